"""NaN, infinities and scores far from zero through every forward kernel, with the keys of a Q block in one
workgroup and dealt out to several. Against plain attention in 64 bits: a row that sees a NaN (or a score of plus
infinity) is NaN, output and row statistics; a score of minus infinity is a key that counts for nothing."""
import math

import pytest

pytestmark = pytest.mark.gpu

# dtype, B, H, Hkv, N, Nk, d, Br, causal
FEW = [("bf16", 1, 4, 2, 3, 4096, 64, 64, True), ("bf16", 2, 2, 2, 5, 3000, 128, 64, True)]
SHARES = [("bf16", 1, 2, 1, 200, 4099, 64, 128, True), ("bf16", 1, 2, 2, 33, 2100, 128, 64, False)]
SHORT = [("bf16", 64, 4, 4, 197, 197, 64, 64, False), ("bf16", 128, 2, 1, 60, 100, 64, 64, True)]
GENERAL = [("bf16", 1, 4, 2, 300, 300, 64, 128, True), ("bf16", 1, 2, 2, 200, 200, 128, 64, False)]
FLOAT = [("f32", 1, 4, 2, 200, 333, 64, 64, True), ("f32", 1, 2, 2, 100, 100, 128, 64, False)]


def _inputs(shape):
    import torch
    dtype, B, H, Hkv, N, Nk, d, Br, causal = shape
    gen = torch.Generator(device="cuda").manual_seed(11)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    return [torch.randn(s, generator=gen, device="cuda").to(t) for s in ((B, H, N, d), (B, Hkv, Nk, d), (B, Hkv, Nk, d))]


def _call(shape, q, k, v, distr=False, undivided=False):
    import torch

    import paper_2507_17245_amd as da
    dtype, B, H, Hkv, N, Nk, d, Br, causal = shape
    print(f"case {shape} distr={distr} undivided={undivided}", flush=True)
    o, lse = torch.zeros_like(q), torch.zeros((B, H, N), device="cuda")
    room = torch.empty(256, dtype=torch.uint8, device="cuda") if undivided else None   # too little for partial sums
    p = da.make_params(q, k, v, Br=Br, n_groups=d // 2 if distr else d, causal=causal, lse_out=lse, workspace=room)
    (da.distr_attn_fwd_ex if distr else da.distr_attn_exact_fwd_ex)(q, k, v, o, p)
    return o, lse


def _visible(shape):
    """[N, Nk] bool on the GPU."""
    import torch
    dtype, B, H, Hkv, N, Nk, d, Br, causal = shape
    i, n = torch.arange(N, device="cuda")[:, None], torch.arange(Nk, device="cuda")[None, :]
    return n <= i + (Nk - N) if causal else torch.ones((N, Nk), dtype=torch.bool, device="cuda")


def _plain(shape, q, k, v):
    """Exact attention and its row statistics in 64 bits."""
    import torch
    dtype, B, H, Hkv, N, Nk, d, Br, causal = shape
    k, v = (x.double().cpu().repeat_interleave(H // Hkv, dim=1) for x in (k, v))
    s = torch.matmul(q.double().cpu(), k.transpose(2, 3).contiguous()) / math.sqrt(d)
    s = s.masked_fill(~_visible(shape).cpu(), -math.inf)
    return torch.matmul(torch.softmax(s, dim=-1), v), torch.logsumexp(s, dim=-1)


@pytest.mark.parametrize("shape", FEW + SHARES + SHORT + GENERAL + FLOAT, ids=str)
@pytest.mark.parametrize("distr,undivided", [(False, False), (False, True), (True, False)])
@pytest.mark.parametrize("at", [0.4, -2])
def test_nan_in_a_key(shape, distr, undivided, at):
    """One NaN in one key (of every head): NaN in every row that sees it, every other row to the bit what it is
    without it."""
    import torch
    q, k, v = _inputs(shape)
    key = int(at * k.shape[2]) if at > 0 else k.shape[2] + at
    clean, clean_lse = _call(shape, q, k, v, distr, undivided)
    k[:, :, key, 7] = math.nan
    o, lse = _call(shape, q, k, v, distr, undivided)
    hit = _visible(shape)[:, key]
    assert hit.any()
    assert torch.isnan(o[:, :, hit]).all() and torch.isnan(lse[:, :, hit]).all()
    assert torch.equal(o[:, :, ~hit], clean[:, :, ~hit]) and torch.equal(lse[:, :, ~hit], clean_lse[:, :, ~hit])


@pytest.mark.parametrize("shape", FEW + SHARES + SHORT + GENERAL + FLOAT, ids=str)
@pytest.mark.parametrize("undivided", [False, True])
@pytest.mark.parametrize("low", [False, True])
def test_infinite_scores(shape, undivided, low):
    """Infinite keys (the first 32 and one more): scores of minus infinity, and of plus infinity for every
    fourth row. `low`: the finite scores lie around -256, where exp(score) is 0 in 32 bits."""
    import torch
    q, k, v = _inputs(shape)
    q[..., 0] = -1.0
    q[:, :, 1::4, 0] = 1.0
    k[:, :, :32, 0] = math.inf
    k[:, :, k.shape[2] // 2, 0] = math.inf
    if low:
        q[..., 1] = 1.0
        k[..., 1] = -256.0 * math.sqrt(shape[6])
    o, lse = _call(shape, q, k, v, undivided=undivided)
    want, want_lse = _plain(shape, q, k, v)
    o, lse = o.double().cpu(), lse.double().cpu()
    assert torch.equal(torch.isnan(o), torch.isnan(want))
    # (a row with a score of plus infinity has no finite statistics); 1e-4 and 2e-2: the parity bars
    rows = ~torch.isnan(want[..., 0])
    assert not torch.isfinite(lse[~rows]).any()
    tol = 1e-4 if shape[0] == "f32" else 2e-2
    assert (o - want)[rows].abs().max() <= tol and (lse - want_lse)[rows].abs().max() <= tol


@pytest.mark.parametrize("shape", FEW + FLOAT, ids=str)
@pytest.mark.parametrize("undivided", [False, True])
@pytest.mark.parametrize("size", [2.0 ** 30, 2.0 ** 101])
@pytest.mark.parametrize("sign", [-1, 1])
def test_scores_far_from_zero(shape, undivided, size, sign):
    """Every score an exact product of one size, the keys 1, 4, 7, .. twice the others: a row's output is the mean
    over the keys with its largest score, however large that is."""
    import torch
    q, k, v = _inputs(shape)
    q.zero_()
    k.zero_()
    q[..., 5] = 1.0
    k[..., 5] = sign * 171 * size          # (not a power of two: its product with the scale is rounded)
    k[:, :, 1::3, 5] *= 2.0
    o, lse = _call(shape, q, k, v, undivided=undivided)
    want, want_lse = _plain(shape, q, k, v)
    assert (o.double().cpu() - want).abs().max() <= (1e-4 if shape[0] == "f32" else 2e-2)
    assert ((lse.double().cpu() - want_lse) / want_lse).abs().max() <= 1e-6


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("d", [64, 128])
def test_float_gradients_at_large_scores(d, G):
    """Scores of up to 150: P = exp(S - lse) of a row with one large score rests on the last bits of both. Relative
    errors (2-norm) against 64 bits; the bounds are twice what sums in short chains, the same in both passes, give.
    Summed over the channels against statistics of sums over groups, dv was at 1.5e-5."""
    import torch

    import paper_2507_17245_amd as da
    B, H, Hkv, N, Nk, Br = 1, 4, 2, 500, 700, 128
    gen = torch.Generator(device="cuda").manual_seed(12)
    q, k, v, dout = (torch.randn(s, generator=gen, device="cuda") for s in ((B, H, N, d), (B, Hkv, Nk, d), (B, Hkv, Nk, d), (B, H, N, d)))
    q *= 30.0
    o, lse = torch.empty_like(q), torch.empty((B, H, N), device="cuda")
    table = torch.empty((B, H, -(-N // Br), d), dtype=torch.uint8, device="cuda")
    print(f"case d {d} G {G}", flush=True)
    da.distr_attn_fwd_ex(q, k, v, o, da.make_params(q, k, v, Br=Br, n_groups=d // G, causal=True, lse_out=lse, perm_out=table))
    dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    da.distr_attn_bwd_ex(q, k, v, o, dout, lse, dq, dk, dv, da.make_params(q, k, v, Br=Br, n_groups=d // G, causal=True, perm_in=table))
    # Q~: every channel replaced by its group's first in the sorted order
    order = table.long().cpu().view(B, H, -1, d // G, G)
    source = torch.empty((B, H, order.shape[2], d), dtype=torch.long)
    source.scatter_(3, order.flatten(3), order[..., :1].expand_as(order).flatten(3))
    source = source.repeat_interleave(Br, dim=2)[:, :, :N]
    qr = torch.gather(q.double().cpu(), 3, source)
    kk, vv = (x.double().cpu().repeat_interleave(H // Hkv, dim=1) for x in (k, v))
    s = torch.matmul(qr, kk.transpose(2, 3).contiguous()) / math.sqrt(d)
    s = s.masked_fill(torch.arange(Nk)[None, :] > torch.arange(N)[:, None] + Nk - N, -math.inf)
    p, g = torch.softmax(s, dim=-1), dout.double().cpu()
    out = torch.matmul(p, vv)
    ds = p * (torch.matmul(g, vv.transpose(2, 3).contiguous()) - (g * out).sum(-1, keepdim=True)) / math.sqrt(d)
    want = {"o": out, "lse": torch.logsumexp(s, dim=-1),
            "dq": torch.zeros_like(qr).scatter_add_(3, source, torch.matmul(ds, kk)),
            "dk": torch.matmul(ds.transpose(2, 3).contiguous(), qr).view(B, Hkv, 2, Nk, d).sum(2),
            "dv": torch.matmul(p.transpose(2, 3).contiguous(), g).view(B, Hkv, 2, Nk, d).sum(2)}
    bound = {"o": 3e-6, "lse": 1.5e-7, "dq": 1e-5, "dk": 1e-5, "dv": 6e-6}
    for name, x in (("o", o), ("lse", lse), ("dq", dq), ("dk", dk), ("dv", dv)):
        err = ((x.double().cpu() - want[name]).norm() / want[name].norm()).item()
        print(f"  {name}: {err:.2e}", flush=True)
        assert err <= bound[name], f"{name}: {err:.3g}"


# Whole tiles of masked keys in front of scores far below zero, in workgroups that walk the keys in one piece: more blocks of 64 rows than
# are taken in two halves, blocks of 128 rows with few tiles, of 256 rows, shares of dealt-out keys that begin with masked tiles,
# K tiles of 32 and 128 rows. q's channels are all alike, so that the grouped form has the exact form's scores.
@pytest.mark.parametrize("B,H,Hkv,N,Nk,d,Br,Bc,causal", [
    (3, 64, 64, 200, 300, 64, 64, 64, True), (3, 32, 16, 200, 300, 128, 64, 64, False), (1, 4, 2, 300, 400, 64, 128, 64, True),
    (1, 2, 2, 200, 700, 128, 128, 64, False), (1, 4, 4, 300, 500, 64, 256, 64, True), (1, 2, 1, 300, 500, 128, 256, 64, False),
    (1, 2, 2, 300, 4096, 64, 256, 64, True), (1, 2, 1, 260, 2100, 128, 128, 64, True), (1, 2, 2, 300, 500, 64, 128, 32, False), (1, 2, 2, 300, 500, 128, 128, 128, True)])
@pytest.mark.parametrize("distr", [False, True])
def test_masked_tiles_before_low_scores(B, H, Hkv, N, Nk, d, Br, Bc, causal, distr):
    import torch

    import paper_2507_17245_amd as da
    gen = torch.Generator(device="cuda").manual_seed(13)
    shape = ("bf16", B, H, Hkv, N, Nk, d, Br, causal)
    q = (torch.randn((B, H, N, 1), generator=gen, device="cuda").abs() + 0.5).expand(B, H, N, d).contiguous().bfloat16()
    k = (-20.0 * torch.randn((B, Hkv, Nk, d), generator=gen, device="cuda").abs() - 1.0).bfloat16()     # scores of -60 .. -600
    v = torch.randn((B, Hkv, Nk, d), generator=gen, device="cuda").bfloat16()
    k[:, 0::2, :200] = -math.inf                          # the first tile of every row, at any tile size
    k[:, 1::2] = torch.where(torch.arange(Nk, device="cuda")[:, None] % 448 < 192, -math.inf, k[:, 1::2])   # and of some shares
    o, lse = torch.full_like(q, math.nan), torch.full((B, H, N), math.nan, device="cuda")
    print(f"case {shape} Bc {Bc} distr={distr}", flush=True)
    p = da.make_params(q, k, v, Br=Br, Bc=Bc, n_groups=d // 2 if distr else d, causal=causal, lse_out=lse)
    (da.distr_attn_fwd_ex if distr else da.distr_attn_exact_fwd_ex)(q, k, v, o, p)
    want, want_lse = _plain(shape, q, k, v)
    o, lse = o.double().cpu(), lse.double().cpu()
    rows = torch.isfinite(want_lse)                       # (a causal row may see masked keys only: NaN in both)
    assert rows.any() and torch.equal(torch.isnan(o[..., 0]), ~rows)
    assert (o - want)[rows].abs().max() <= 2e-2
    assert ((lse - want_lse)[rows].abs() / want_lse[rows].abs().clamp(min=1.0)).max() <= 2e-2


@pytest.mark.parametrize("shape", [("bf16", 1, 4, 2, 300, 300, 64, 128, True), ("bf16", 1, 2, 2, 200, 333, 128, 256, False),
                                   ("bf16", 1, 2, 2, 1100, 1100, 128, 256, False), ("bf16", 1, 2, 1, 200, 4099, 64, 128, True)], ids=str)
@pytest.mark.parametrize("distr", [False, True])
@pytest.mark.parametrize("value", [math.nan, math.inf, 2.0 ** 100])
def test_rows_keep_to_themselves(shape, distr, value):
    """A query row whose scores are NaN, infinite or far above the others', in every 32 rows: sums of rows are
    taken together, and no other row changes by more than the order of its float sums (its P, the same to the bit, is
    summed another way where a row beside it is not finite: 64 additions a tile, 2^-24 each at most, and with them
    outputs move by a bf16 step at most). The tables are given: a block's grouping knows all of its rows."""
    import torch

    import paper_2507_17245_amd as da
    dtype, B, H, Hkv, N, Nk, d, Br, causal = shape
    q, k, v = _inputs(shape)
    table = torch.stack([torch.randperm(d) for _ in range(B * H * -(-N // Br))]).to(torch.uint8).cuda()
    rows = torch.arange(N, device="cuda") % 32 == 5
    outs = []
    for x in (None, value):
        y = q.clone()
        if x is not None:
            y[:, :, rows] = torch.tensor(x, device="cuda").to(y.dtype)
        o, lse = torch.zeros_like(q), torch.zeros((B, H, N), device="cuda")
        p = da.make_params(y, k, v, Br=Br, n_groups=d // 2 if distr else d, causal=causal, lse_out=lse,
                           perm_in=table.view(B, H, -1, d) if distr else None)
        print(f"case {shape} distr={distr} {x}", flush=True)
        (da.distr_attn_fwd_ex if distr else da.distr_attn_exact_fwd_ex)(y, k, v, o, p)
        outs.append((o[:, :, ~rows], lse[:, :, ~rows]))
    assert torch.isfinite(outs[0][0]).all()
    (o, lse), (o1, lse1) = outs
    assert (o1.float() - o.float()).abs().le(2.0 ** -7 * o.float().abs()).all()
    assert (lse1 - lse).abs().max() <= 64 * 2.0 ** -24 + 2.0 ** -20   # (and the rounding of a statistic of up to 16)


@pytest.mark.parametrize("shape", [(4, 300, 300, 64, 128, 64, False), (4, 300, 300, 64, 128, 64, True), (2, 400, 400, 128, 64, 64, True), (16, 1100, 1100, 128, 256, 64, False),
                                   (12, 2200, 2200, 64, 128, 64, True), (2, 200, 6200, 64, 128, 64, False), (4, 300, 300, 64, 128, 128, False),
                                   (4, 300, 300, 128, 64, 32, False)], ids=str)
@pytest.mark.parametrize("distr", [False, True])
def test_reference_moves_for_a_score_far_above(shape, distr):
    """The row sum that moves a row's reference is that of the BC / 2 keys a lane owns: a weight of 2^(1/8) times its limit, BC / 2 times
    2^8, is above it whatever the others are. The reference is then the largest score, whose weight is 1 and half of it 1/2, both exact: what is left is the
    rounding of a statistic of up to 16 in a few operations. Against the old reference both would be rounded to bf16, 2^-8.4 above."""
    import torch

    import paper_2507_17245_amd as da
    H, N, Nk, d, Br, Bc, causal = shape
    far = 7 + math.log2(Bc) + 0.125
    score = torch.full((Nk,), -100.0, dtype=torch.float64)
    score[0], score[Bc + 6], score[Bc + 7] = 0.0, far, far - 1
    q, k = torch.zeros((1, H, N, d), device="cuda"), torch.zeros((1, H, Nk, d), device="cuda")
    q[..., 0], k[..., 0] = 1.0, score.float().cuda()
    q, k = q.bfloat16(), k.bfloat16()
    v, o, lse = torch.randn_like(k), torch.zeros_like(q), torch.zeros((1, H, N), device="cuda")
    table = torch.arange(d, device="cuda").to(torch.uint8).expand(1, H, -(-N // Br), d).contiguous()
    p = da.make_params(q, k, v, Br=Br, Bc=Bc, n_groups=d // 2 if distr else d, causal=causal, lse_out=lse, softmax_scale=math.log(2.0),
                       perm_in=table if distr else None)
    print(f"case {shape} distr={distr}", flush=True)
    (da.distr_attn_fwd_ex if distr else da.distr_attn_exact_fwd_ex)(q, k, v, o, p)
    want = torch.logsumexp(score * math.log(2.0), dim=0).item()
    seen = torch.arange(N) + (Nk - N if causal else Nk) >= Bc + 7
    assert seen.any() and (lse[0, :, seen.cuda()].double() - want).abs().max() <= 2.0 ** -16
