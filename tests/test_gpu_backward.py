"""GPU parity of the backward pass (float tensors: float matrix instructions; bf16 tensors: bf16 ones) against the CPU oracle (gradient of the forward with the
grouping held fixed; the paper, Sec. 4.3-4.4, trains through the method without giving one)."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

TOL = 1e-4   # float path, relative to the larger of 1 and the gradient's largest magnitude

CASES = [
    ("one-block", dict(N=50)),
    ("tiny", dict()),
    ("ragged-causal", dict(N=150, causal=True)),
    ("gqa-more-keys-causal", dict(H=4, Hkv=2, N=100, Nk=173, causal=True, Br=128)),
    ("fewer-keys", dict(B=2, N=130, Nk=45)),
    ("d128-groups-of-4", dict(H=2, Hkv=1, N=200, d=128, n_groups=32, Br=128, recipe="rho_pairs")),
    ("blocks-of-256", dict(N=300, Br=256, causal=True, n_groups=16)),
    ("one-channel-per-group", dict(N=90, n_groups=64, causal=True)),
]


def run_backward(cfg, q, k, v, dout, distr, perm_in=None):
    import torch

    import gpu_util as U
    import paper_2507_17245_amd as da
    tq, tk, tv, tdo = (U.to_dev(x, cfg.dtype) for x in (q, k, v, dout))
    o = torch.full_like(tq, float("nan"))
    lse = torch.full((cfg.B, cfg.H, cfg.N), float("nan"), dtype=torch.float32, device="cuda")
    t_perm = None if perm_in is None else torch.from_numpy(np.ascontiguousarray(perm_in)).cuda()
    p = da.make_params(tq, tk, tv, Br=cfg.Br, Bc=cfg.Bc, n_groups=cfg.n_groups, causal=cfg.causal,
                       lsh_seed=cfg.lsh_seed, n_planes=cfg.n_planes, lse_out=lse, perm_in=t_perm)
    fwd, bwd = (da.distr_attn_fwd_ex, da.distr_attn_bwd_ex) if distr else (da.distr_attn_exact_fwd_ex, da.distr_attn_exact_bwd_ex)
    fwd(tq, tk, tv, o, p)
    dq = torch.full_like(tq, float("nan"))
    dk = torch.full_like(tk, float("nan"))
    dv = torch.full_like(tk, float("nan"))
    bwd(tq, tk, tv, o, tdo, lse, dq, dk, dv, p)
    torch.cuda.synchronize()
    return [t.float().cpu().numpy().astype(np.float64) for t in (dq, dk, dv)]


@pytest.mark.parametrize("name,kw", CASES, ids=[c[0] for c in CASES])
def test_backward_matches_oracle(name, kw):
    import gpu_util as U
    cfg = W.CONFIGS["tiny"].scaled(**kw)
    print(f"case {cfg}", flush=True)
    q, k, v = W.make(cfg)
    dout = W.make_grad(cfg)
    p = U.oracle_params(cfg)
    for distr in (True, False):
        got = run_backward(cfg, q, k, v, dout, distr)
        ref = oracle.distr_bwd(q, k, v, dout, p) if distr else oracle.exact_bwd(q, k, v, dout, p)
        for what, g, r in zip(("dq", "dk", "dv"), got, ref):
            assert np.isfinite(g).all(), f"{what}: non-finite"
            err = np.abs(g - r).max()
            print(f"  distr={distr} {what}: max-abs {err:.3g} (largest gradient {np.abs(r).max():.3g})", flush=True)
            assert err <= TOL * max(1.0, np.abs(r).max()), f"{name} distr={distr} {what}: {err:.4g}"
        if distr and cfg.n_groups < cfg.d:
            # the unsampled query columns of every block get exactly zero
            _, perm, _ = oracle.lsh_group(q, p)
            G = cfg.d // cfg.n_groups
            for t in range(cfg.Tq):
                unsampled = np.setdiff1d(np.arange(cfg.d), perm[0, 0, t, ::G])
                assert np.all(got[0][0, 0, t * cfg.Br:(t + 1) * cfg.Br][:, unsampled] == 0.0)


def test_backward_is_deterministic_and_takes_a_caller_table():
    import gpu_util as U
    cfg = W.CONFIGS["tiny"].scaled(H=2, Hkv=1, N=140, causal=True)
    q, k, v = W.make(cfg)
    dout = W.make_grad(cfg)
    a = run_backward(cfg, q, k, v, dout, True)
    b = run_backward(cfg, q, k, v, dout, True)
    assert all(np.array_equal(x, y) for x, y in zip(a, b))
    _, perm, _ = oracle.lsh_group(q, U.oracle_params(cfg))
    c = run_backward(cfg, q, k, v, dout, True, perm_in=perm)
    assert all(np.array_equal(x, y) for x, y in zip(a, c))
    rng = np.random.default_rng(5)
    other = np.stack([rng.permutation(cfg.d) for _ in range(cfg.B * cfg.H * cfg.Tq)]).astype(np.uint8).reshape(cfg.B, cfg.H, cfg.Tq, cfg.d)
    got = run_backward(cfg, q, k, v, dout, True, perm_in=other)
    ref = oracle.distr_bwd(q, k, v, dout, U.oracle_params(cfg), perm=other)
    for g, r in zip(got, ref):
        assert np.abs(g - r).max() <= TOL * max(1.0, np.abs(r).max())


BF16_CASES = [
    ("vit", dict(B=1, H=3, Hkv=3, N=150)),
    ("llama", dict(H=4, Hkv=2, N=300)),
    ("llama", dict(H=4, Hkv=2, N=100, Nk=260)),
    ("mid", dict(B=1, H=2, Hkv=2, N=260, n_groups=32)),
    ("long", dict(H=2, Hkv=1, N=200, Br=64)),
    ("long", dict(H=2, Hkv=1, N=700)),                          # causal, several workgroups per head
    ("llama", dict(H=4, Hkv=2, N=300, Br=256)),
    ("vit", dict(B=2, H=2, Hkv=2, N=130, Nk=45)),               # fewer keys than one tile
    ("mid", dict(B=1, H=2, Hkv=1, N=200, n_groups=16)),         # groups of eight channels
    ("vit", dict(B=1, H=2, Hkv=2, N=129, n_groups=64)),         # one channel per group
    ("vit", dict(B=1, H=2, Hkv=1, N=1, Nk=70)),                 # a single query row
    ("llama", dict(H=4, Hkv=1, N=4096)),                        # the full sequence length of "llama", one kv head
    ("mid", dict(B=1, H=2, Hkv=2, N=2048)),                     # 32 tiles per workgroup at d = 128
    ("long", dict(B=2, H=4, Hkv=2, N=150, Nk=290)),             # batch x grouped heads x more keys, causal
]


@pytest.mark.parametrize("base,kw", BF16_CASES, ids=[f"{b}-{i}" for i, (b, _) in enumerate(BF16_CASES)])
def test_backward_on_bf16_tensors(base, kw):
    """bf16 tensors on the matrix cores, fed the bf16 forward's output and row statistics: within
    the bf16 tolerances relative to the gradient's scale; the unsampled query columns exactly zero."""
    import gpu_util as U
    cfg = W.CONFIGS[base].scaled(**kw)
    print(f"case {cfg}", flush=True)
    q, k, v = W.make(cfg)
    dout = W.make_grad(cfg)
    p = U.oracle_params(cfg)
    for distr in (True, False):
        got = run_backward(cfg, q, k, v, dout, distr)
        ref = oracle.distr_bwd(q, k, v, dout, p) if distr else oracle.exact_bwd(q, k, v, dout, p)
        for what, g, r in zip(("dq", "dk", "dv"), got, ref):
            assert np.isfinite(g).all(), f"{what}: non-finite"
            err = np.abs(g - r)
            unit = max(1.0, np.abs(r).max())
            print(f"  distr={distr} {what}: max-abs {err.max():.3g} mean-abs {err.mean():.3g} (largest gradient {np.abs(r).max():.3g})", flush=True)
            assert err.max() <= 2e-2 * unit and err.mean() <= 2e-3 * unit, f"{base} distr={distr} {what}"
            # regression bound: twice the largest errors these kernels showed on any case when
            # they were tuned (0.65 % / 0.03 % of the gradient's scale)
            assert err.max() <= 1.3e-2 * unit and err.mean() <= 6e-4 * unit, f"{base} distr={distr} {what}: regression"
        if distr and cfg.n_groups < cfg.d:
            _, perm, _ = oracle.lsh_group(q, p)
            G = cfg.d // cfg.n_groups
            for t in range(cfg.Tq):
                unsampled = np.setdiff1d(np.arange(cfg.d), perm[0, 0, t, ::G])
                assert np.all(got[0][0, 0, t * cfg.Br:(t + 1) * cfg.Br][:, unsampled] == 0.0)


def test_bf16_backward_is_deterministic_and_takes_a_workspace():
    import torch

    import gpu_util as U
    import paper_2507_17245_amd as da
    cfg = W.CONFIGS["llama"].scaled(H=4, Hkv=2, N=333)
    q, k, v = W.make(cfg)
    dout = W.make_grad(cfg)
    a = run_backward(cfg, q, k, v, dout, True)
    b = run_backward(cfg, q, k, v, dout, True)
    assert all(np.array_equal(x, y) for x, y in zip(a, b))
    # the same through a caller's workspace of exactly the size the library asks for
    tq, tk, tv, tdo = (U.to_dev(x, cfg.dtype) for x in (q, k, v, dout))
    o = torch.empty_like(tq)
    lse = torch.empty((cfg.B, cfg.H, cfg.N), dtype=torch.float32, device="cuda")
    p = da.make_params(tq, tk, tv, Br=cfg.Br, Bc=cfg.Bc, n_groups=cfg.n_groups, causal=cfg.causal,
                       lsh_seed=cfg.lsh_seed, n_planes=cfg.n_planes, lse_out=lse)
    da.distr_attn_fwd_ex(tq, tk, tv, o, p)
    need = da.distr_attn_bwd_workspace_bytes(p)
    assert need >= cfg.B * cfg.H * cfg.N * (4 + 2 * cfg.d)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    pw = da.make_params(tq, tk, tv, Br=cfg.Br, Bc=cfg.Bc, n_groups=cfg.n_groups, causal=cfg.causal,
                        lsh_seed=cfg.lsh_seed, n_planes=cfg.n_planes, workspace=ws)
    outs = [torch.full_like(t, float("nan")) for t in (tq, tk, tk)]
    da.distr_attn_bwd_ex(tq, tk, tv, o, tdo, lse, *outs, pw)
    torch.cuda.synchronize()
    assert all(np.array_equal(x, t.float().cpu().numpy()) for x, t in zip(a, outs))
    small = torch.empty(need - 256, dtype=torch.uint8, device="cuda")
    ps = da.make_params(tq, tk, tv, Br=cfg.Br, Bc=cfg.Bc, n_groups=cfg.n_groups, causal=cfg.causal,
                        lsh_seed=cfg.lsh_seed, n_planes=cfg.n_planes, workspace=small)
    with pytest.raises(da.DistrAttnError) as e:
        da.distr_attn_bwd_ex(tq, tk, tv, o, tdo, lse, *outs, ps)
    assert e.value.code == da.DA_ERR_WORKSPACE


def test_backward_refuses_the_mirrored_form():
    import torch

    import paper_2507_17245_amd as da
    x = torch.zeros((1, 2, 64, 64), dtype=torch.float32, device="cuda")
    lse = torch.zeros((1, 2, 64), dtype=torch.float32, device="cuda")
    outs = [torch.zeros_like(x) for _ in range(5)]
    p = da.make_params(x, x, x, Br=64, n_groups=32, side=1)
    with pytest.raises(da.DistrAttnError) as e:
        da.distr_attn_bwd_ex(x, x, x, outs[0], outs[1], lse, outs[2], outs[3], outs[4], p)
    assert e.value.code == da.DA_ERR_UNSUPPORTED


def test_forward_and_backward_replay_from_a_hip_graph():
    """With caller-provided workspaces a training step's attention (forward with row statistics,
    then the backward) is launches only, so it can be captured once and replayed: every replay,
    with eager work and synchronisations in between, must equal the eager result on the inputs of
    that moment."""
    import torch

    import gpu_util as U
    import paper_2507_17245_amd as da
    cfg = W.CONFIGS["llama"].scaled(H=4, Hkv=2, N=333)
    q, k, v = W.make(cfg)
    tq, tk, tv, tdo = (U.to_dev(x, "bf16") for x in (q, k, v, W.make_grad(cfg)))
    common = dict(Br=cfg.Br, n_groups=cfg.n_groups, causal=cfg.causal, lsh_seed=cfg.lsh_seed)
    probe = da.make_params(tq, tk, tv, **common)
    bytes_f, bytes_b = da.distr_attn_workspace_bytes(probe), da.distr_attn_bwd_workspace_bytes(probe)

    def buffers():
        return dict(o=torch.empty_like(tq), lse=torch.empty((cfg.B, cfg.H, cfg.N), dtype=torch.float32, device="cuda"),
                    dq=torch.empty_like(tq), dk=torch.empty_like(tk), dv=torch.empty_like(tk),
                    wf=torch.empty(bytes_f, dtype=torch.uint8, device="cuda"),
                    wb=torch.empty(bytes_b, dtype=torch.uint8, device="cuda"))

    def step(x):
        da.distr_attn_fwd_ex(tq, tk, tv, x["o"], da.make_params(tq, tk, tv, workspace=x["wf"], lse_out=x["lse"], **common))
        da.distr_attn_bwd_ex(tq, tk, tv, x["o"], tdo, x["lse"], x["dq"], x["dk"], x["dv"],
                             da.make_params(tq, tk, tv, workspace=x["wb"], **common))

    g, e = buffers(), buffers()
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        step(g)
    torch.cuda.synchronize()
    gen = torch.Generator(device="cuda").manual_seed(7)
    for rep in range(4):
        if rep:   # new inputs in the captured buffers
            for t in (tq, tk, tv, tdo):
                t.copy_(torch.randn(t.shape, device="cuda", generator=gen).to(torch.bfloat16))
        for name in ("dq", "dk", "dv"):
            g[name].fill_(float("nan"))
        step(e)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for name in ("o", "dq", "dk", "dv"):
            assert torch.equal(g[name].view(torch.int16), e[name].view(torch.int16)), (name, rep)
