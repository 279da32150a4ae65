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
