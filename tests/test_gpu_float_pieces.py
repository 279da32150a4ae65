"""Float products taken as bf16 pieces: what pieces do not hold as floats do (infinities, NaN, magnitudes far from one) comes out as
float products give it, row by row, and every other row is what it is without it. Groups of two and four channels and the mirrored
form; sizes around the tiles of 32 rows, and Q blocks that a wave's run of tiles enters and leaves. Products are by pieces from 257 keys on;
with more than 256 row tiles (64 heads of 129 rows) the forward and dQ have four waves per workgroup, with fewer than eight query tiles
per kv head dK/dV has, otherwise eight at d = 64."""
import math

import pytest

pytestmark = pytest.mark.gpu

# H, Hkv, N, Nk, d, G, causal, side
FORWARD = [(2, 1, 33, 65, 64, 2, True, 0), (8, 2, 200, 300, 64, 2, True, 0), (1, 1, 300, 520, 64, 4, True, 0), (3, 3, 1, 31, 64, 4, True, 0),
           (2, 1, 100, 300, 64, 2, True, 1), (2, 2, 97, 129, 128, 4, True, 1), (1, 1, 64, 800, 64, 2, True, 1),
           (64, 64, 129, 300, 64, 2, True, 0), (64, 32, 130, 290, 64, 4, True, 0), (3, 3, 1, 287, 64, 4, True, 0), (2, 1, 33, 257, 64, 2, True, 0),
           (64, 64, 129, 300, 64, 4, True, 1), (64, 64, 129, 300, 64, 2, True, 1), (2, 2, 97, 300, 128, 4, True, 1), (2, 1, 97, 300, 128, 2, True, 1)]
BACKWARD = [(2, 1, 33, 65, 64, 2, True, 0), (8, 2, 300, 300, 64, 2, True, 0), (2, 2, 300, 520, 64, 4, True, 0), (1, 1, 257, 257, 64, 2, True, 0),
            (64, 64, 129, 300, 64, 2, True, 0), (64, 64, 130, 290, 64, 4, True, 0), (2, 1, 33, 300, 64, 2, True, 0), (2, 1, 33, 260, 64, 4, True, 0)]


def _inputs(case):
    import torch
    H, Hkv, N, Nk, d, G, causal, side = case
    gen = torch.Generator(device="cuda").manual_seed(21)
    # channels alike on the sampled side, so that the grouped scores are the exact ones whatever the grouping
    q = torch.randn((1, H, N, 1 if side == 0 else d), generator=gen, device="cuda").abs().expand(1, H, N, d) + 0.5
    k = torch.randn((1, Hkv, Nk, d if side == 0 else 1), generator=gen, device="cuda").expand(1, Hkv, Nk, d)
    v = torch.randn((1, Hkv, Nk, d), generator=gen, device="cuda")
    return q.contiguous(), k.contiguous(), v


def _params(da, case, q, k, v, **more):
    H, Hkv, N, Nk, d, G, causal, side = case
    return da.make_params(q, k, v, Br=64, Bc=32, n_groups=d // G, causal=causal, side=side, softmax_scale=0.02, **more)


def _forward(case, q, k, v):
    import torch

    import paper_2507_17245_amd as da
    print(f"case {case}", flush=True)
    o, lse = torch.zeros_like(q), torch.zeros(q.shape[:3], device="cuda")
    da.distr_attn_fwd_ex(q, k, v, o, _params(da, case, q, k, v, **({} if case[7] else {"lse_out": lse})))
    return o, lse


def _plain(case, q, k, v):
    import torch
    H, Hkv, N, Nk, d, G, causal, side = case
    k, v = (x.double().repeat_interleave(H // Hkv, dim=1) for x in (k, v))
    s = torch.matmul(q.double(), k.transpose(2, 3).contiguous()) * 0.02
    hidden = torch.arange(Nk, device="cuda")[None, :] > torch.arange(N, device="cuda")[:, None] + Nk - N
    s = s.masked_fill(hidden, -math.inf)
    return torch.matmul(torch.softmax(s, dim=-1), v), torch.logsumexp(s, dim=-1), hidden


@pytest.mark.parametrize("case", FORWARD, ids=str)
def test_infinite_keys(case):
    import torch
    q, k, v = _inputs(case)
    Nk, at = k.shape[2], k.shape[2] - 1 - q.shape[2] // 2
    k[:, :, :Nk // 8] = -math.inf
    low, low_lse = _forward(case, q, k, v)
    want, want_lse, hidden = _plain(case, q, k, v)
    assert torch.isfinite(want).all()
    assert (low - want).abs().max() <= 1e-4 and (case[7] or (low_lse - want_lse).abs().max() <= 1e-4)
    k[:, :, at] = math.inf        # a row that sees it is NaN, every other row the same to the bit
    o, lse = _forward(case, q, k, v)
    assert torch.isnan(o[:, :, ~hidden[:, at]]).all()
    assert torch.equal(o[:, :, hidden[:, at]], low[:, :, hidden[:, at]])
    assert case[7] or torch.equal(lse[:, :, hidden[:, at]], low_lse[:, :, hidden[:, at]])


@pytest.mark.parametrize("case", FORWARD, ids=str)
@pytest.mark.parametrize("by", [(1.0, 1.0, 2.0 ** -100), (1.0, 1.0, 2.0 ** 100), (2.0 ** 70, 2.0 ** -70, 1.0), (2.0 ** -110, 2.0 ** 110, 1.0)])
def test_magnitudes(case, by):
    """Bound: four times what the same inputs give at magnitude one (3e-7 at most)."""
    q, k, v = _inputs(case)
    o, lse = _forward(case, q * by[0], k * by[1], v * by[2])
    want = _plain(case, q, k, v)[0] * by[2]
    assert ((o.double() - want) / by[2]).norm() <= 1.2e-6 * (want / by[2]).norm()


def _backward(case, q, k, v, dout):
    import torch

    import paper_2507_17245_amd as da
    o, lse = _forward(case, q, k, v)
    grads = [torch.zeros_like(x) for x in (q, k, v)]
    da.distr_attn_bwd_ex(q, k, v, o, dout, lse, *grads, _params(da, case, q, k, v))
    return grads


@pytest.mark.parametrize("case", BACKWARD, ids=str)
@pytest.mark.parametrize("value", [math.inf, math.nan])
def test_gradients_that_are_not_finite(case, value):
    """One element of dout: its row of dq and the keys that the row sees are not finite; every other row of dq, and the keys of tiles
    that no row of its tile sees, are the same to the bit."""
    import torch
    q, k, v = _inputs(case)
    dout = torch.randn(q.shape, generator=torch.Generator(device="cuda").manual_seed(22), device="cuda")
    clean = _backward(case, q, k, v, dout)
    row = q.shape[2] // 3
    dout[:, :, row, 9] = value
    dq, dk, dv = _backward(case, q, k, v, dout)
    seen = k.shape[2] - q.shape[2] + row + 1
    sampled = clean[0][:, :, row] != 0
    assert not torch.isfinite(dq[:, :, row][sampled]).any()
    dq[:, :, row] = clean[0][:, :, row]
    assert torch.equal(dq, clean[0])
    assert not torch.isfinite(dk[:, :, :seen]).any() and not torch.isfinite(dv[:, :, :seen, 9]).any()
    far = -(-(k.shape[2] - q.shape[2] + (row | 31) + 1) // 32) * 32
    assert torch.equal(dk[:, :, far:], clean[1][:, :, far:]) and torch.equal(dv[:, :, far:], clean[2][:, :, far:])


@pytest.mark.parametrize("case", BACKWARD, ids=str)
@pytest.mark.parametrize("size", [2.0 ** -100, 2.0 ** 60])
def test_gradients_far_from_one(case, size):
    """dout times a power of two: the gradients' distance from 64 bits stays what it is at one (bound: four times that, 1e-6)."""
    import torch
    H, Hkv, N, Nk, d, G, causal, side = case
    q, k, v = _inputs(case)
    dout = torch.randn(q.shape, generator=torch.Generator(device="cuda").manual_seed(23), device="cuda")
    dq, dk, dv = _backward(case, q, k, v, dout * size)
    o, lse, hidden = _plain(case, q, k, v)
    kk, vv = (x.double().repeat_interleave(H // Hkv, dim=1) for x in (k, v))
    p = torch.exp((torch.matmul(q.double(), kk.transpose(2, 3).contiguous()) * 0.02).masked_fill(hidden, -math.inf) - lse[..., None])
    g = dout.double()
    ds = p * (torch.matmul(g, vv.transpose(2, 3).contiguous()) - (g * o).sum(-1, keepdim=True)) * 0.02
    # dq's sampled channels hold the sum over their groups: summed over all channels it is the exact gradient's sum
    for got, want in ((dq.double().sum(-1), torch.matmul(ds, kk).sum(-1)),
                      (dk.double(), torch.matmul(ds.transpose(2, 3).contiguous(), q.double()).view(1, Hkv, -1, Nk, d).sum(2)),
                      (dv.double(), torch.matmul(p.transpose(2, 3).contiguous(), g).view(1, Hkv, -1, Nk, d).sum(2))):
        assert (got / size - want).norm() <= 4e-6 * want.norm()


# the keys of every row apart by more than exp() reaches: P is 1 at the last key with the largest score and 0 elsewhere
ONE_KEY = [(8, 2, 300, 300, 64, 2, True, 0), (1, 1, 290, 320, 64, 4, True, 0), (64, 64, 129, 300, 64, 2, True, 0), (64, 64, 130, 290, 64, 4, True, 0)]


@pytest.mark.parametrize("case", ONE_KEY, ids=str)
@pytest.mark.parametrize("what", ["ordinary", "small q", "small k", "large q", "large k", "infinite k", "no q"])
def test_scores_of_both_passes(case, what):
    """P = exp(S - lse) of the backward is of the very scores that the forward's lse is of, whichever way they are summed: with one key that
    counts it is exactly 1 at scores of 1e4 and more, where the two ways differ by up to 1 %. Bound: the rounding of a float sum of 600."""
    import torch
    H, Hkv, N, Nk, d, G, causal, side = case
    q, k, v = _inputs(case)
    gen = torch.Generator(device="cuda").manual_seed(24)
    k = 100.0 * torch.arange(1, Nk + 1, device="cuda")[None, None, :, None] * (1.0 + 1e-3 * torch.randn(k.shape, generator=gen, device="cuda"))
    if what == "small q":
        q[:, :, 2::7, 5] = 1e-20
    elif what == "small k":
        k[:, :, 3::7, 10] += k[:, :, 3::7, 9]
        k[:, :, 3::7, 9] = 1e-20
    elif what == "large q":
        q[:, :, 1::5] *= 2.0 ** 70
    elif what == "large k":
        k[:, :, 5::50] *= 2.0 ** 70
    elif what == "infinite k":
        k[:, :, 7::40] = -math.inf
    elif what == "no q":
        q[:, :, 2::9] = 0.0
        k[:, :, 20::30] *= 2.0 ** 70
    dout = torch.randn(q.shape, generator=gen, device="cuda")
    o, _ = _forward(case, q, k, v)
    dv = _backward(case, q, k, v, dout)[2]
    kk, vv = (x.double().repeat_interleave(H // Hkv, dim=1) for x in (k, v))
    hidden = torch.arange(Nk, device="cuda")[None, :] > torch.arange(N, device="cuda")[:, None] + Nk - N
    s = torch.matmul(q.double(), kk.transpose(2, 3).contiguous()) * 0.02
    p = torch.softmax(s.masked_fill(hidden, -math.inf), dim=-1)
    want = torch.matmul(p, vv)
    assert (o.double() - want).norm() <= 1e-6 * want.norm()
    want = torch.matmul(p.transpose(2, 3).contiguous(), dout.double()).view(1, Hkv, -1, Nk, d).sum(2)
    assert (dv.double() - want).norm() <= 2e-6 * want.norm()


def _apart(x, channel, by, others):
    """One channel times `by`, the others times `others`."""
    y = x * others
    y[..., channel] = x[..., channel] * by
    return y


@pytest.mark.parametrize("case", [c for c in BACKWARD if c[3] > 256], ids=str)
@pytest.mark.parametrize("what", ["small v", "small v, large dout", "large v, small dout", "a channel of v and dout", "a channel of v and dout, small others",
                                  "small k"])
def test_gradients_of_operands_far_apart(case, what):
    """V and dO, or K, that are far from one in all channels or in one: every product of the backward keeps the bits of its operands. Against
    64 bits, what is of another size by itself; bound as above."""
    import torch
    H, Hkv, N, Nk, d, G, causal, side = case
    q, k, v = _inputs(case)
    dout = torch.randn(q.shape, generator=torch.Generator(device="cuda").manual_seed(25), device="cuda")
    if what == "small v":
        v = v * 2.0 ** -115
    elif what == "small v, large dout":
        v, dout = v * 2.0 ** -118, dout * 2.0 ** 70
    elif what == "large v, small dout":
        v, dout = v * 2.0 ** 110, dout * 2.0 ** -118
    elif what == "a channel of v and dout":
        v, dout = _apart(v, 9, 2.0 ** 120, 1.0), _apart(dout, 9, 2.0 ** -120, 1.0)
    elif what == "a channel of v and dout, small others":
        v, dout = _apart(v, 9, 2.0 ** 90, 2.0 ** -16), _apart(dout, 9, 2.0 ** -122, 2.0 ** -16)
    elif what == "small k":
        k = k * 2.0 ** -105
    dq, dk, dv = _backward(case, q, k, v, dout)
    o, lse, hidden = _plain(case, q, k, v)
    kk, vv = (x.double().repeat_interleave(H // Hkv, dim=1) for x in (k, v))
    p = torch.exp((torch.matmul(q.double(), kk.transpose(2, 3).contiguous()) * 0.02).masked_fill(hidden, -math.inf) - lse[..., None])
    g = dout.double()
    ds = p * (torch.matmul(g, vv.transpose(2, 3).contiguous()) - (g * o).sum(-1, keepdim=True)) * 0.02
    for name, got, want in (("dq", dq.double().sum(-1), torch.matmul(ds, kk).sum(-1)),
                            ("dk", dk.double(), torch.matmul(ds.transpose(2, 3).contiguous(), q.double()).view(1, Hkv, -1, Nk, d).sum(2)),
                            ("dv", dv.double(), torch.matmul(p.transpose(2, 3).contiguous(), g).view(1, Hkv, -1, Nk, d).sum(2))):
        for part in (slice(0, 9), slice(9, 10), slice(10, None)) if name == "dv" else (slice(None),):
            a, b = got[..., part], want[..., part]
            unit = b.abs().max()
            assert unit > 0 and ((a - b) / unit).norm() <= 4e-6 * (b / unit).norm(), (name, part)


PIECES_FORWARD = [(2, 1, 33, 300, 64, 2, True, 0), (64, 64, 129, 300, 64, 2, True, 0), (64, 64, 130, 290, 64, 4, True, 0), (1, 1, 300, 520, 64, 4, True, 0),
                  (2, 1, 100, 300, 64, 2, True, 1), (64, 64, 129, 300, 64, 2, True, 1), (2, 2, 97, 300, 128, 4, True, 1), (2, 1, 97, 300, 128, 2, True, 1)]


@pytest.mark.parametrize("case", PIECES_FORWARD, ids=str)
@pytest.mark.parametrize("by,others", [(2.0 ** -115, 1.0), (2.0 ** 115, 1.0), (2.0 ** 60, 2.0 ** -60), (2.0 ** -60, 2.0 ** 60), (2.0 ** -118, 2.0 ** 70)])
def test_a_channel_of_v_by_itself(case, by, others):
    """Every channel of the output is as near to 64 bits as it is at magnitude one (bound: test_magnitudes), whatever the others are."""
    q, k, v = _inputs(case)
    v = _apart(v, 9, by, others)
    o = _forward(case, q, k, v)[0].double()
    want = _plain(case, q, k, v)[0]
    for part in (slice(0, 9), slice(9, 10), slice(10, None)):
        unit = want[..., part].abs().max()
        assert ((o - want)[..., part] / unit).norm() <= 1.2e-6 * (want[..., part] / unit).norm()


@pytest.mark.parametrize("case", PIECES_FORWARD, ids=str)
@pytest.mark.parametrize("size", [2.0 ** 122, 2.0 ** 86, 2.0 ** 66])
def test_small_weights_of_large_values(case, size):
    """Weights of 2^-122 that alone have values. Bound: P = exp2 of -122, whose argument has the rounding of three products and one difference."""
    import torch
    q, k, v = _inputs(case)
    q.fill_(1.0)
    k.zero_()
    k[:, :, :3] = -66.0 * 64 / case[4]
    v[:, :, 3:] = 0.0
    v[:, :, :3] *= size
    o = _forward(case, q, k, v)[0].double() / size
    want = _plain(case, q, k, v / size)[0]
    assert (o - want).norm() <= 122 * 0.7 * 4 * 2.0 ** -24 * want.norm()


@pytest.mark.parametrize("case", [c for c in PIECES_FORWARD if c[7]], ids=str)
@pytest.mark.parametrize("what", ["ordinary", "infinite k", "nan", "large k", "large q", "a channel of v", "infinite v"])
def test_mirrored_form_of_bf16_tensors(case, what):
    """The same arithmetic as for float tensors of these values, rounded at the end."""
    import torch
    q, k, v = (x.bfloat16() for x in _inputs(case))
    if what == "infinite k":
        k[:, :, 4:40] = -math.inf
    elif what == "nan":
        k[:, :, -3, 7] = math.nan
    elif what == "large k":
        k[:, :, 11::37] *= 2.0 ** 70
    elif what == "large q":
        q[:, :, 1::9] *= 2.0 ** 70
    elif what == "a channel of v":
        v = _apart(v, 9, 2.0 ** -115, 1.0)
    elif what == "infinite v":
        v[:, :, -2, 3] = math.inf
    o = _forward(case, q, k, v)[0]
    want = _forward(case, q.float(), k.float(), v.float())[0].bfloat16()
    assert torch.equal(torch.isnan(o), torch.isnan(want)) and torch.isnan(o).any() == (what in ("nan", "infinite v"))
    assert torch.equal(o.nan_to_num(nan=0.0, posinf=1.0), want.nan_to_num(nan=0.0, posinf=1.0))
