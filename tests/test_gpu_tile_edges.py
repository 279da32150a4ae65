"""GPU parity at the sizes where a kernel's tiling can go wrong: around the edges of its tiles, with
fewer rows or keys than a tile, with tiles that only some waves get, at every group size it is
built for. Against the CPU oracle, with the parity bar of gpu_util."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


def _forward(cfg, distr=True):
    import gpu_util as U
    print(f"case {cfg} distr={distr}", flush=True)
    q, k, v = W.make(cfg)
    p = U.oracle_params(cfg)
    o, _, _ = U.run_gpu(cfg, q, k, v, distr=distr)
    U.assert_close(o, oracle.distr_fwd(q, k, v, p) if distr else oracle.exact_fwd(q, k, v, p), cfg.dtype)


# Float kernel: 32-row workgroups, 32-key tiles dealt out to 4 waves.
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N,Nk,causal", [(1, 1, False), (31, 33, True), (32, 32, True), (33, 31, False), (65, 129, True), (70, 160, False)])
@pytest.mark.parametrize("side,Bc,G", [(0, 64, 1), (0, 64, 2), (0, 64, 4), (0, 64, 8), (1, 32, 2), (1, 64, 4), (1, 128, 2), (1, 64, 8), (1, 32, 1)])
def test_float_forward(d, N, Nk, causal, side, Bc, G):
    cfg = W.CONFIGS["tiny"].scaled(B=2, H=4, Hkv=2, N=N, Nk=Nk, d=d, causal=causal, side=side, Bc=Bc, n_groups=d // G,
                                   recipe="normal", n_planes=16)
    _forward(cfg)
    if side == 0 and G == 1:
        _forward(cfg, distr=False)


# Float backward: 32-row tiles on both sides, dealt out to 4 waves; groups of 2 and 4 have products
# over the groups, other sizes over the channels. Bound: float rounding, the parity bar of the backward tests.
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N,Nk,causal", [(1, 1, False), (31, 33, True), (33, 31, False), (129, 290, True)])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_float_backward(d, N, Nk, causal, G):
    import gpu_util as U
    from test_gpu_backward import TOL, run_backward
    cfg = W.CONFIGS["tiny"].scaled(B=2, H=4, Hkv=2, N=N, Nk=Nk, d=d, causal=causal, n_groups=d // G, recipe="normal")
    print(f"case {cfg}", flush=True)
    q, k, v = W.make(cfg)
    dout = W.make_grad(cfg)
    got = run_backward(cfg, q, k, v, dout, True)
    for what, g, r in zip(("dq", "dk", "dv"), got, oracle.distr_bwd(q, k, v, dout, U.oracle_params(cfg))):
        err = np.abs(g - r).max()
        assert err <= TOL * max(1.0, np.abs(r).max()), f"{what}: {err:.4g}"
