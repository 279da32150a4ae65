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


# Float backward: 32-row tiles on both sides, dealt out to 4 waves (dK/dV at d = 64 from 8 query tiles on: 8); groups of 2 and 4 have products
# over the groups, other sizes over the channels. Bound: float rounding, the parity bar of the backward tests.
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N,Nk,causal", [(1, 1, False), (31, 33, True), (33, 31, False), (96, 97, False), (97, 33, False), (129, 290, True), (289, 320, True)])
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


# Float dK/dV over the groups: a wave takes a run of the query tiles of all heads of a kv head. Runs of one tile, of none, runs that begin
# inside a Q block, cover several, cross from one head into the next and, under the mask, skip the tiles above a key tile.
@pytest.mark.parametrize("H,Hkv,N,Nk,Br,causal", [(1, 1, 40, 33, 64, False), (2, 1, 97, 40, 64, False), (6, 1, 330, 70, 64, False), (6, 1, 330, 350, 64, True),
                                                  (5, 1, 200, 200, 128, True), (3, 1, 500, 33, 256, False)])
@pytest.mark.parametrize("d,G", [(64, 2), (64, 4), (128, 2), (128, 4)])
def test_float_dkv_runs(H, Hkv, N, Nk, Br, causal, d, G):
    import gpu_util as U
    from test_gpu_backward import TOL, run_backward
    cfg = W.CONFIGS["tiny"].scaled(B=2, H=H, Hkv=Hkv, N=N, Nk=Nk, d=d, Br=Br, causal=causal, n_groups=d // G, recipe="normal", n_planes=16)
    print(f"case {cfg}", flush=True)
    q, k, v = W.make(cfg)
    dout = W.make_grad(cfg)
    for what, g, r in zip(("dq", "dk", "dv"), run_backward(cfg, q, k, v, dout, True), oracle.distr_bwd(q, k, v, dout, U.oracle_params(cfg))):
        err = np.abs(g - r).max()
        assert err <= TOL * max(1.0, np.abs(r).max()), f"{what}: {err:.4g}"


# bf16, few query rows against many keys: rows of all query heads of a kv head packed into tiles of 32,
# key tiles of 64 (d = 64) or 32 (d = 128) dealt out to four waves of each share.
@pytest.mark.parametrize("base,d", [("llama", 64), ("long", 128)])
@pytest.mark.parametrize("B,H,Hkv,N,Nk,causal", [(1, 4, 1, 1, 256, True), (2, 8, 2, 3, 300, True), (1, 4, 4, 32, 1000, True), (1, 2, 1, 64, 513, False),
                                                 (1, 32, 1, 1, 777, True), (1, 12, 2, 17, 4100, True), (3, 2, 2, 5, 16383, False), (300, 1, 1, 2, 320, True),
                                                 # around the lengths from which keys are dealt out, and from which exact calls come here
                                                 (1, 4, 4, 2, 1345, True), (1, 4, 4, 2, 1409, True), (1, 8, 2, 4, 672, False), (1, 8, 2, 4, 705, False),
                                                 (2, 4, 4, 3, 512, True), (2, 4, 4, 3, 513, True), (2, 4, 2, 3, 257, True)])
def test_bf16_few_rows(base, d, B, H, Hkv, N, Nk, causal):
    cfg = W.CONFIGS[base].scaled(B=B, H=H, Hkv=Hkv, N=N, Nk=Nk, Br=64, n_groups=d // 2, causal=causal, recipe="normal")
    assert cfg.d == d
    import gpu_util as U
    print(f"case {cfg}", flush=True)
    q, k, v = W.make(cfg)
    p = U.oracle_params(cfg)
    import torch
    lse = torch.empty((B, H, N), dtype=torch.float32, device="cuda")
    o, perm, _ = U.run_gpu(cfg, q, k, v, want_perm_only=True, lse_out=lse)
    assert np.array_equal(perm, oracle.lsh_group(q, p)[1])
    U.assert_close(o, oracle.distr_fwd(q, k, v, p), "bf16")
    tab, _, _ = U.run_gpu(cfg, q, k, v, want_tables=True)      # the LSH kernel's table: the same output
    assert np.array_equal(tab, o)
    assert np.abs(lse.cpu().numpy() - oracle.lse(q, k, p)).max() <= 2e-2
    o, _, _ = U.run_gpu(cfg, q, k, v, distr=False)
    U.assert_close(o, oracle.exact_fwd(q, k, v, p), "bf16")


# bf16, a Q block's keys dealt out to several workgroups (general kernel and combine kernel): ragged last
# rows and keys, shares that the causal mask leaves empty for some rows, more shares than a block has tiles.
@pytest.mark.parametrize("base", ["llama", "long"])
@pytest.mark.parametrize("H,Hkv,N,Nk,Br,causal", [(2, 1, 200, 4099, 128, True), (1, 1, 33, 2100, 64, False), (4, 2, 130, 2500, 64, True), (2, 2, 2300, 2300, 256, True)])
def test_bf16_key_shares(base, H, Hkv, N, Nk, Br, causal):
    import torch

    import gpu_util as U
    cfg = W.CONFIGS[base].scaled(B=1, H=H, Hkv=Hkv, N=N, Nk=Nk, Br=Br, causal=causal, recipe="normal")
    print(f"case {cfg}", flush=True)
    q, k, v = W.make(cfg)
    p = U.oracle_params(cfg)
    lse = torch.empty((1, H, N), dtype=torch.float32, device="cuda")
    for distr in (True, False):
        o, _, _ = U.run_gpu(cfg, q, k, v, distr=distr, lse_out=lse)
        U.assert_close(o, oracle.distr_fwd(q, k, v, p) if distr else oracle.exact_fwd(q, k, v, p), "bf16")
        assert np.abs(lse.cpu().numpy() - oracle.lse(q, k, p, distr=distr)).max() <= 2e-2


def test_bf16_key_shares_with_little_room():
    """A caller's workspace that only holds what a call must have: the keys stay together, the result
    is the same to rounding. Threads on one stream and on several: each call's own result."""
    import threading

    import torch

    import paper_2507_17245_amd as da
    gen = torch.Generator(device="cuda").manual_seed(3)
    q = torch.randn((1, 4, 100, 64), generator=gen, device="cuda").bfloat16()
    k, v = (torch.randn((1, 4, 4096, 64), generator=gen, device="cuda").bfloat16() for _ in range(2))
    whole = da.make_params(q, k, v, Br=64, causal=True)
    o = da.distr_attn_exact_fwd_ex(q, k, v, torch.empty_like(q), whole).float()
    small = torch.empty(256, dtype=torch.uint8, device="cuda")
    o1 = da.distr_attn_exact_fwd_ex(q, k, v, torch.empty_like(q), da.make_params(q, k, v, Br=64, causal=True, workspace=small)).float()
    assert (o - o1).abs().max() <= 2.0 ** -7 * o.abs().max()
    scale = [1.0, 0.5, 2.0, 4.0]
    vs = [(v * s).contiguous() for s in scale]
    torch.cuda.synchronize()
    for shared in (True, False):
        outs = [[] for _ in scale]
        streams = [torch.cuda.Stream()] * 4 if shared else [torch.cuda.Stream() for _ in scale]

        def work(i):
            with torch.cuda.stream(streams[i]):
                params = da.make_params(q, k, vs[i], Br=64, causal=True)
                for _ in range(8):
                    outs[i].append(da.distr_attn_exact_fwd_ex(q, k, vs[i], torch.empty_like(q), params))
        threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
        [t.start() for t in threads]
        [t.join() for t in threads]
        torch.cuda.synchronize()
        for i, s in enumerate(scale):
            for x in outs[i]:
                assert torch.equal(x.float(), o * s)     # powers of two scale every step exactly


def test_bf16_key_shares_under_capture():
    """A captured call without a workspace uses no library-owned buffer: graphs captured on one stream replay
    on different streams at once, each with its own result, beside eager calls on the capture stream."""
    import torch

    import paper_2507_17245_amd as da
    gen = torch.Generator(device="cuda").manual_seed(4)
    q = torch.randn((1, 4, 100, 64), generator=gen, device="cuda").bfloat16()
    k, v = (torch.randn((1, 4, 4096, 64), generator=gen, device="cuda").bfloat16() for _ in range(2))
    scale = [1.0, 0.5, 2.0]
    vs, outs = [(v * s).contiguous() for s in scale], [torch.empty_like(q) for _ in scale]
    side = torch.cuda.Stream()

    def call(i, o):
        return da.distr_attn_exact_fwd_ex(q, k, vs[i], o, da.make_params(q, k, vs[i], Br=64, causal=True))
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        eager = call(0, torch.empty_like(q))     # the capture stream has a buffer before the captures
    torch.cuda.synchronize()
    graphs = [torch.cuda.CUDAGraph() for _ in scale]
    for i, g in enumerate(graphs):
        with torch.cuda.graph(g, stream=side):
            call(i, outs[i])
    streams = [torch.cuda.Stream() for _ in scale]
    torch.cuda.synchronize()
    for _ in range(4):
        for s, g in zip(streams, graphs):
            with torch.cuda.stream(s):
                g.replay()
        with torch.cuda.stream(side):
            again = call(0, torch.empty_like(q))
        torch.cuda.synchronize()
        assert torch.equal(again, eager)
        for i, s in enumerate(scale):
            assert torch.equal(outs[i].float(), outs[0].float() * s)      # powers of two scale every step exactly
            assert (outs[i].float() - eager.float() * s).abs().max() <= 2.0 ** -7 * s * eager.float().abs().max()


def test_bf16_key_shares_on_many_streams():
    """However many streams a process has used one after the other, a call deals its keys out and gives the same bits;
    and again when a stream is destroyed with its work in flight and another takes its place."""
    import torch

    import paper_2507_17245_amd as da
    gen = torch.Generator(device="cuda").manual_seed(5)
    q = torch.randn((1, 4, 100, 64), generator=gen, device="cuda").bfloat16()
    k, v = (torch.randn((1, 4, 4096, 64), generator=gen, device="cuda").bfloat16() for _ in range(2))

    def call(vx, o, **kw):
        return da.distr_attn_exact_fwd_ex(q, k, vx, o, da.make_params(q, k, vx, Br=64, causal=True, **kw))
    small = torch.empty(256, dtype=torch.uint8, device="cuda")
    undivided = call(v, torch.empty_like(q), workspace=small)
    outs = [torch.empty_like(q) for _ in range(24)]
    torch.cuda.synchronize()
    for stream, o in zip([torch.cuda.Stream() for _ in outs], outs):
        with torch.cuda.stream(stream):
            call(v, o)
        stream.synchronize()
    assert not torch.equal(undivided, outs[0])      # (the two ways differ in rounding: equal bits say which was taken)
    for i, o in enumerate(outs):
        assert torch.equal(o, outs[0]), f"stream {i}"
    # streams of the runtime's own, each destroyed as soon as its call is queued
    import ctypes
    hip = ctypes.CDLL("libamdhip64.so")
    vs = [(v * s).contiguous() for s in (1.0, 0.5, 2.0, 4.0)]
    outs = [torch.empty_like(q) for _ in range(40)]
    torch.cuda.synchronize()
    for i, o in enumerate(outs):
        handle = ctypes.c_void_p()
        assert hip.hipStreamCreate(ctypes.byref(handle)) == 0
        with torch.cuda.stream(torch.cuda.ExternalStream(handle.value)):
            call(vs[i % 4], o)
        assert hip.hipStreamDestroy(handle) == 0
    torch.cuda.synchronize()
    for i, o in enumerate(outs):
        assert torch.equal(o.float(), outs[0].float() * (1.0, 0.5, 2.0, 4.0)[i % 4])   # powers of two scale every step exactly


# LSH kernel: blocks staged 128 rows at a time (float) or whole (bf16, matrix pipe), 16 projections at a time;
# a tensor that is not 16-byte aligned takes a path of its own; a sequence shorter than a block takes the kernel of a
# shorter one. Tables and hashes to the bit.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,Br", [(64, 64), (64, 256), (128, 64), (128, 128), (128, 256)])
@pytest.mark.parametrize("N,n_planes,offset", [(1, 16, 0), (65, 3, 0), (257, 17, 0), (300, 32, 1), (129, 16, 1),
                                                 (32, 17, 0), (33, 32, 1), (64, 16, 0), (128, 17, 0)])
def test_lsh_kernel(dtype, d, Br, N, n_planes, offset):
    import torch

    import gpu_util as U
    import paper_2507_17245_amd as da
    cfg = W.CONFIGS["tiny"].scaled(B=2, H=2, Hkv=1, N=N, d=d, Br=Br, n_groups=d // 2, n_planes=n_planes, recipe="normal")
    q = W.make(cfg)[0]
    if dtype == "bf16":
        q = torch.from_numpy(q).bfloat16().float().numpy()
    print(f"case {cfg} {dtype} offset {offset}", flush=True)
    room = torch.empty(q.size + 8, dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
    tq = room[offset:offset + q.size].view(q.shape)
    tq.copy_(torch.from_numpy(q))
    perm = torch.zeros((2, 2, cfg.Tq, d), dtype=torch.uint8, device="cuda")
    hsh = torch.zeros((2, 2, cfg.Tq, d), dtype=torch.int32, device="cuda")
    da.distr_attn_lsh_group(tq, da.make_params(tq, tq, tq, Br=Br, n_groups=d // 2, lsh_seed=cfg.lsh_seed, n_planes=n_planes,
                                               perm_out=perm, hash_out=hsh))
    want_hash, want_perm, _ = oracle.lsh_group(q, U.oracle_params(cfg))
    assert np.array_equal(perm.cpu().numpy(), want_perm)
    assert np.array_equal(hsh.cpu().numpy().view(np.uint32), want_hash)


# The same with more blocks than compute units, where a bf16 block has 256 threads instead of 512.
@pytest.mark.parametrize("d,Br", [(64, 64), (64, 256), (128, 64), (128, 128), (128, 256)])
@pytest.mark.parametrize("N,n_planes,offset", [(1, 16, 0), (65, 3, 0), (257, 17, 0), (300, 32, 1), (129, 16, 1), (33, 32, 1)])
def test_lsh_kernel_many_blocks(d, Br, N, n_planes, offset):
    import torch

    import gpu_util as U
    import paper_2507_17245_amd as da
    cfg = W.CONFIGS["tiny"].scaled(B=1, H=260, Hkv=260, N=N, d=d, Br=Br, n_groups=d // 2, n_planes=n_planes, recipe="normal")
    q = torch.from_numpy(W.make(cfg)[0]).bfloat16()
    print(f"case {cfg} offset {offset}", flush=True)
    tq = torch.empty(q.numel() + 8, dtype=torch.bfloat16, device="cuda")[offset:offset + q.numel()].view(q.shape)
    tq.copy_(q)
    perm = torch.zeros((1, 260, cfg.Tq, d), dtype=torch.uint8, device="cuda")
    hsh = torch.zeros((1, 260, cfg.Tq, d), dtype=torch.int32, device="cuda")
    da.distr_attn_lsh_group(tq, da.make_params(tq, tq, tq, Br=Br, n_groups=d // 2, lsh_seed=cfg.lsh_seed, n_planes=n_planes,
                                               perm_out=perm, hash_out=hsh))
    want_hash, want_perm, _ = oracle.lsh_group(q.float().numpy(), U.oracle_params(cfg))
    assert np.array_equal(perm.cpu().numpy(), want_perm)
    assert np.array_equal(hsh.cpu().numpy().view(np.uint32), want_hash)


# Projections the matrix pipe leaves in doubt: `n` channels of every 16 sum to almost nothing along one projection (columns
# built as in test_projections_that_nearly_cancel). One at a time is summed by the wave, a few by a lane each, many by
# every lane for its own channels; in the LSH kernel and in the forward kernels' own stages. Tables to the bit.
@pytest.mark.parametrize("base,N,Br", [("vit", 128, 64), ("vit", 250, 128), ("vit", 256, 256), ("llama", 300, 64), ("llama", 384, 128), ("llama", 300, 256), ("mid", 256, 128)])
@pytest.mark.parametrize("n", [1, 2, 5, 12, 13])
def test_doubtful_projections(base, N, Br, n):
    import gpu_util as U
    import paper_2507_17245_amd as da
    cfg = W.CONFIGS[base].scaled(B=1, H=2, Hkv=1, N=N, Br=Br, recipe="normal", data_seed=4000 + n)
    q, k, v = W.make(cfg)
    R = da.distr_attn_hyperplanes(cfg.lsh_seed, cfg.n_planes, cfg.Br).astype(np.float64)
    for t in range(cfg.Tq):
        r0, rows = t * Br, min(Br, N - t * Br)
        for c in [c for c in range(cfg.d) if c % 16 < n]:
            w, col, run = R[c % cfg.n_planes, :rows], np.zeros(rows), 0.0
            for r in range(rows):
                if r >= rows - 3 and abs(w[r]) > 0.1:
                    col[r] = float(W.round_to_bf16(np.array([-run / w[r]], dtype=np.float32))[0])
                else:
                    col[r] = -1.0 if run * w[r] > 0 else 1.0
                run += col[r] * w[r]
            q[:, :, r0:r0 + rows, c] = col
    print(f"case {cfg} n {n}", flush=True)
    want_hash, want_perm, _ = oracle.lsh_group(q, U.oracle_params(cfg))
    o, perm, hsh = U.run_gpu(cfg, q, k, v, want_tables=True)
    assert np.array_equal(hsh, want_hash) and np.array_equal(perm, want_perm)
    own, perm, _ = U.run_gpu(cfg, q, k, v, want_perm_only=True)
    assert np.array_equal(perm, want_perm) and np.array_equal(own, o)


def test_zero_queries_cost_what_others_do():
    """Queries of zeros (padding) leave every projection in doubt; summed one by one they took 33 times as long."""
    import torch

    import paper_2507_17245_amd as da
    gen = torch.Generator(device="cuda").manual_seed(6)
    for B, N, d, Br in ((8, 512, 64, 64), (2, 1024, 64, 256), (16, 197, 64, 64)):
        q, k, v = (torch.randn((B, 12, N, d), generator=gen, device="cuda").bfloat16() for _ in range(3))
        o, zero = torch.empty_like(q), torch.zeros_like(q)
        p = da.make_params(q, k, v, Br=Br, n_groups=d // 2)
        times = []
        for x in (q, zero) * 4:
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(10):
                da.distr_attn_fwd_ex(x, k, v, o, p)
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end))
        print(f"  B{B} N{N} Br{Br}: {min(times[0::2]):.3f} | {min(times[1::2]):.3f} ms", flush=True)
        assert min(times[1::2]) < 4 * min(times[0::2])


# bf16 backward of short sequences in one workgroup per head: 32 keys per wave (4 waves up to 128 keys, 8 up to 256),
# row tiles of 64 in blocks of 32 and 16; one past the range on either side takes the general kernels. Same bar as the
# bf16 backward tests; a call's results do not depend on the run.
@pytest.mark.parametrize("N,Nk,causal", [(1, 1, False), (31, 33, True), (33, 31, False), (64, 128, True), (65, 129, False), (127, 64, False),
                                         (128, 128, True), (196, 225, True), (256, 256, True), (256, 256, False), (257, 256, False), (200, 257, True)])
@pytest.mark.parametrize("Br,G", [(64, 2), (128, 4), (256, 1)])
def test_bf16_backward_short(N, Nk, causal, Br, G):
    import gpu_util as U
    from test_gpu_backward import run_backward
    cfg = W.CONFIGS["vit"].scaled(B=2, H=3, Hkv=3, N=N, Nk=Nk, Br=Br, causal=causal, n_groups=64 // G, recipe="normal")
    print(f"case {cfg}", flush=True)
    q, k, v = W.make(cfg)
    dout = W.make_grad(cfg)
    p = U.oracle_params(cfg)
    for distr in (True, False):
        got = run_backward(cfg, q, k, v, dout, distr)
        ref = oracle.distr_bwd(q, k, v, dout, p) if distr else oracle.exact_bwd(q, k, v, dout, p)
        for what, g, r in zip(("dq", "dk", "dv"), got, ref):
            err, unit = np.abs(g - r), max(1.0, np.abs(r).max())
            assert np.isfinite(g).all(), what
            assert err.max() <= 2e-2 * unit and err.mean() <= 2e-3 * unit, f"distr={distr} {what}: {err.max():.4g}"
        assert all(np.array_equal(x, y) for x, y in zip(got, run_backward(cfg, q, k, v, dout, distr)))


# bf16 forward of short sequences, one workgroup per head: 32 rows per wave, two, four or eight waves by the longer
# side; one past the range takes the general kernel. Tables to the bit, row statistics, the table handed in.
@pytest.mark.parametrize("N,Nk,causal", [(1, 1, False), (31, 33, True), (64, 64, True), (65, 64, False), (33, 129, True), (128, 128, False),
                                         (197, 197, False), (256, 255, False), (256, 256, True), (257, 256, False)])
@pytest.mark.parametrize("B,Br,G", [(2, 64, 2), (2, 128, 4), (80, 256, 8)])
def test_bf16_short(N, Nk, causal, B, Br, G):
    import torch

    import gpu_util as U
    cfg = W.CONFIGS["vit"].scaled(B=B, H=4, Hkv=2, N=N, Nk=Nk, Br=Br, causal=causal, n_groups=64 // G, recipe="normal")
    print(f"case {cfg}", flush=True)
    q, k, v = W.make(cfg)
    p = U.oracle_params(cfg)
    lse = torch.empty((B, 4, N), dtype=torch.float32, device="cuda")
    o, perm, _ = U.run_gpu(cfg, q, k, v, want_perm_only=True, lse_out=lse)
    assert np.array_equal(perm, oracle.lsh_group(q, p)[1])
    U.assert_close(o, oracle.distr_fwd(q, k, v, p), "bf16")
    assert np.abs(lse.cpu().numpy() - oracle.lse(q, k, p)).max() <= 2e-2
    assert np.array_equal(U.run_gpu(cfg, q, k, v, perm_in=perm)[0], o)
    o, _, _ = U.run_gpu(cfg, q, k, v, distr=False, lse_out=lse)
    U.assert_close(o, oracle.exact_fwd(q, k, v, p), "bf16")
    assert np.abs(lse.cpu().numpy() - oracle.lse(q, k, p, distr=False)).max() <= 2e-2


# Causal launches whose second round of workgroups is issued in the opposite order: in the forward a whole second round and one that
# the tiles end inside of, in the backward (tiles of 128 rows) the same at d = 64 and 128; more heads than half the compute units, or than all
# of them, where nothing is reversed (300 rows; 200 take the one-workgroup kernels). Every row of every head, forward and gradients.
@pytest.mark.parametrize("base,B,H,Hkv,N,Br", [("llama", 1, 100, 50, 500, 64), ("llama", 2, 12, 4, 910, 64), ("llama", 2, 70, 70, 600, 128), ("llama", 1, 300, 300, 200, 64), ("llama", 1, 300, 100, 300, 64),
                                               ("llama", 1, 40, 20, 1100, 128), ("llama", 1, 64, 64, 1030, 64), ("long", 1, 40, 40, 1100, 128), ("long", 1, 64, 32, 900, 64)])
def test_causal_order(base, B, H, Hkv, N, Br):
    import gpu_util as U
    from test_gpu_backward import run_backward
    cfg = W.CONFIGS[base].scaled(B=B, H=H, Hkv=Hkv, N=N, Br=Br, recipe="normal")
    _forward(cfg)
    _forward(cfg, distr=False)
    q, k, v = W.make(cfg)
    dout = W.make_grad(cfg)
    for what, g, r in zip(("dq", "dk", "dv"), run_backward(cfg, q, k, v, dout, True), oracle.distr_bwd(q, k, v, dout, U.oracle_params(cfg))):
        err, unit = np.abs(g - r), max(1.0, np.abs(r).max())
        assert err.max() <= U.BF16_MAX_ABS * unit and err.mean() <= U.BF16_MEAN_ABS * unit, f"{what}: {err.max():.4g} {err.mean():.4g}"


# Float kernels at d = 64 with eight waves (more than eight key tiles, at most 256 row tiles): around the number of tiles from which
# they are taken, tiles that only some waves get, K blocks of the mirrored form dealt out to them.
@pytest.mark.parametrize("B,H,Hkv,N,Nk,causal", [(1, 4, 2, 33, 256, False), (1, 4, 2, 33, 257, True), (1, 2, 1, 290, 545, True), (2, 2, 2, 70, 1000, False),
                                                 (1, 64, 32, 128, 300, False), (1, 64, 32, 129, 300, True)])
@pytest.mark.parametrize("side,Bc,G", [(0, 64, 1), (0, 64, 2), (0, 64, 4), (0, 64, 8), (1, 32, 2), (1, 128, 4), (1, 64, 8)])
def test_float_eight_waves(B, H, Hkv, N, Nk, causal, side, Bc, G):
    import gpu_util as U
    from test_gpu_backward import TOL, run_backward
    cfg = W.CONFIGS["tiny"].scaled(B=B, H=H, Hkv=Hkv, N=N, Nk=Nk, causal=causal, side=side, Bc=Bc, n_groups=64 // G, recipe="normal", n_planes=16)
    _forward(cfg)
    if side:
        return
    q, k, v = W.make(cfg)
    dout = W.make_grad(cfg)
    for what, g, r in zip(("dq", "dk", "dv"), run_backward(cfg, q, k, v, dout, True), oracle.distr_bwd(q, k, v, dout, U.oracle_params(cfg))):
        err = np.abs(g - r).max()
        assert err <= TOL * max(1.0, np.abs(r).max()), f"{what}: {err:.4g}"


# Two halves of the keys per workgroup: blocks whose second half has no tile (causal, one tile) or one less than the first, ragged last
# tiles, halves of a share of dealt-out keys (blocks of 64 rows and, with 24 tiles a share, of 128), the edges of the rule. Exact and Q~ K^T; the
# fused product is in test_fused_in_halves.
@pytest.mark.parametrize("base,Br,B,H,Hkv,N,Nk,causal,G", [
    ("llama", 64, 1, 4, 2, 200, 200, True, 2), ("llama", 64, 2, 3, 3, 257, 449, False, 4), ("long", 64, 1, 4, 4, 300, 330, True, 2),
    ("long", 64, 1, 2, 1, 65, 197, False, 8), ("llama", 64, 1, 2, 2, 130, 3000, True, 2), ("long", 64, 1, 3, 3, 100, 2500, True, 4),
    ("llama", 128, 1, 2, 1, 1537, 1537, True, 2), ("long", 128, 1, 2, 2, 1600, 1637, True, 2), ("llama", 128, 1, 1, 1, 140, 4700, True, 2),
    ("long", 128, 1, 2, 1, 130, 6001, False, 4), ("llama", 128, 1, 64, 64, 140, 3900, True, 2), ("long", 128, 1, 64, 32, 140, 3900, True, 4), ("llama", 64, 1, 64, 64, 512, 512, True, 2), ("llama", 64, 1, 65, 65, 512, 512, True, 2)])
def test_halves(base, Br, B, H, Hkv, N, Nk, causal, G):
    import gpu_util as U
    import torch
    d = W.CONFIGS[base].d
    cfg = W.CONFIGS[base].scaled(B=B, H=H, Hkv=Hkv, N=N, Nk=Nk, Br=Br, n_groups=d // G, causal=causal, recipe="normal")
    print(f"case {cfg}", flush=True)
    q, k, v = W.make(cfg)
    p = U.oracle_params(cfg)
    lse = torch.empty((B, H, N), dtype=torch.float32, device="cuda")
    o, perm, _ = U.run_gpu(cfg, q, k, v, want_perm_only=True, lse_out=lse)
    assert np.array_equal(perm, oracle.lsh_group(q, p)[1])
    U.assert_close(o, oracle.distr_fwd(q, k, v, p), "bf16")
    assert np.abs(lse.cpu().numpy() - oracle.lse(q, k, p)).max() <= 2e-2
    _forward(cfg, distr=False)


# A half whose first tiles hold only scores of minus infinity for a row, and finite ones far below zero behind them: the row's
# reference is its first finite score, whichever half that is in.
@pytest.mark.parametrize("d,Br,H,N,Nk", [(64, 64, 2, 70, 640), (128, 64, 2, 70, 640), (64, 128, 66, 130, 1664)])
def test_halves_with_masked_keys(d, Br, H, N, Nk):
    import torch
    import paper_2507_17245_amd as da
    g = torch.Generator().manual_seed(5)
    q = torch.randn(1, H, N, d, generator=g).abs() + 0.5
    k = torch.randn(1, H, Nk, d, generator=g)
    k = -k.abs() * 20.0 - 1.0                       # scores around -10^2 .. -10^3
    half = (Nk // 64 + 1) // 2 * 64
    k[:, 0::2, half:half + 130] = -float("inf")                 # even heads: the second half begins with masked keys
    k[:, 1::2, :Nk - 70] = -float("inf")                        # odd heads: all but the last tiles are masked
    v = torch.randn(1, H, Nk, d, generator=g)
    q, k, v = (x.to(torch.bfloat16).cuda() for x in (q, k, v))
    o = torch.full_like(q, float("nan"))
    print(f"case d{d} Br{Br} N{N} Nk{Nk}", flush=True)
    da.distr_attn_exact_fwd_ex(q, k, v, o, da.make_params(q, k, v, Br=Br, Bc=64, n_groups=d))
    s = q.double().cpu() @ k.double().cpu().transpose(-1, -2) / d ** 0.5
    want = torch.softmax(s, -1) @ v.double().cpu()
    got = o.double().cpu()
    assert torch.isfinite(got).all() and (got - want).abs().max() <= 2e-2


# Grouped heads whose dK/dV workgroups take some of a kv head's query heads: all of them, a half, a third, a quarter, one each beside the
# edge of the rule (7/8 of a full chip) and for a ragged tile of keys.
@pytest.mark.parametrize("base,H,Hkv,N,Nk,causal", [("long", 480, 240, 64, 128, False), ("long", 480, 120, 64, 128, False), ("long", 480, 80, 64, 128, False),
                                                    ("long", 448, 112, 64, 128, False), ("long", 480, 120, 64, 127, False), ("long", 480, 60, 70, 256, True),
                                                    ("llama", 480, 120, 64, 256, False), ("llama", 480, 60, 70, 256, True)])
@pytest.mark.parametrize("distr", [True, False])
def test_head_shares(base, H, Hkv, N, Nk, causal, distr):
    import gpu_util as U
    from test_gpu_backward import run_backward
    cfg = W.CONFIGS[base].scaled(B=1, H=H, Hkv=Hkv, N=N, Nk=Nk, causal=causal, Br=64, n_groups=W.CONFIGS[base].d // 2, recipe="normal")
    print(f"case {cfg}", flush=True)
    q, k, v = W.make(cfg)
    dout = W.make_grad(cfg)
    ref = (oracle.distr_bwd if distr else oracle.exact_bwd)(q, k, v, dout, U.oracle_params(cfg))
    for what, g, r in zip(("dq", "dk", "dv"), run_backward(cfg, q, k, v, dout, distr), ref):
        err, unit = np.abs(g - r), max(1.0, np.abs(r).max())
        assert err.max() <= U.BF16_MAX_ABS * unit and err.mean() <= U.BF16_MEAN_ABS * unit, f"{what}: {err.max():.4g} {err.mean():.4g}"


# Dealt-out keys by the number of workgroups a block takes and whether each walks its keys whole or in halves, on both sides of the rules: shares
# whose blocks find nothing of each other in an L2 (few heads on an XCD), short, middling and long ones.
@pytest.mark.parametrize("base,Br,H,N,Nk", [("llama", 64, 150, 64, 2500), ("llama", 64, 130, 40, 2250), ("long", 128, 100, 33, 3200), ("long", 128, 100, 33, 8400)])
@pytest.mark.parametrize("distr", [True, False])
def test_shares_whole_and_in_halves(base, Br, H, N, Nk, distr):
    _forward(W.CONFIGS[base].scaled(B=1, H=H, Hkv=H, N=N, Nk=Nk, Br=Br, causal=True, recipe="normal"), distr)


# Blocks of 64 rows at d = 128: one workgroup or two for each compute unit, by the tiles of a share and by whether blocks share an L2.
@pytest.mark.parametrize("H,Hkv,N,Nk", [(128, 128, 65, 4096), (128, 16, 65, 4160), (32, 8, 129, 2900), (32, 8, 129, 3900), (8, 8, 64, 2100), (250, 50, 33, 4200)])
@pytest.mark.parametrize("distr", [True, False])
def test_one_workgroup_or_two(H, Hkv, N, Nk, distr):
    _forward(W.CONFIGS["long"].scaled(B=1, H=H, Hkv=Hkv, N=N, Nk=Nk, Br=64, causal=True, recipe="normal"), distr)


@pytest.mark.parametrize("B,H,N,causal", [(1, 1, 1, False), (1, 2, 33, True), (1, 1, 256, False), (2, 3, 300, True), (1, 8, 1000, False), (1, 256, 32, False)])
@pytest.mark.parametrize("Br,G", [(64, 2), (128, 4), (256, 2), (256, 8)])
@pytest.mark.parametrize("n_planes", [1, 4, 5, 16, 17, 32])
def test_float_groups_itself(B, H, N, causal, Br, G, n_planes):
    """Float calls whose workgroups have a compute unit each group their Q blocks themselves: the tables are the LSH
    kernel's (which the oracle pins), and the output is to the bit what that table gives when it is handed in."""
    import torch

    import paper_2507_17245_amd as da
    gen = torch.Generator(device="cuda").manual_seed(N + n_planes)
    q, k, v = (torch.randn((B, H, N, 64), generator=gen, device="cuda") for _ in range(3))
    want, got = (torch.zeros((B, H, -(-N // Br), 64), dtype=torch.uint8, device="cuda") for _ in range(2))
    o, o_given, o_quiet = (torch.zeros_like(q) for _ in range(3))
    options = dict(Br=Br, n_groups=64 // G, causal=causal, lsh_seed=9, n_planes=n_planes)
    print(f"case {(B, H, N, causal, Br, G, n_planes)}", flush=True)
    da.distr_attn_lsh_group(q, da.make_params(q, k, v, perm_out=want, **options))
    da.distr_attn_fwd_ex(q, k, v, o, da.make_params(q, k, v, perm_out=got, **options))
    da.distr_attn_fwd_ex(q, k, v, o_given, da.make_params(q, k, v, perm_in=want, **options))
    da.distr_attn_fwd_ex(q, k, v, o_quiet, da.make_params(q, k, v, **options))
    assert torch.equal(got, want)
    assert torch.equal(o, o_given) and torch.equal(o_quiet, o_given)


@pytest.mark.parametrize("B,H,Hkv,N,Nk,d,causal", [
    (1, 8, 8, 2048, 2048, 64, True), (1, 8, 4, 2049, 2049, 128, False), (1, 6, 6, 8129, 8129, 64, True), (16, 12, 12, 280, 280, 64, False),
    (16, 12, 12, 300, 300, 64, False), (1, 16, 16, 2100, 2500, 128, False), (1, 16, 4, 2100, 2100, 64, False), (1, 4, 4, 65, 6000, 128, True),
    (1, 4, 4, 150, 6000, 128, True), (1, 8, 8, 1000, 1000, 128, True), (1, 4, 4, 2299, 2299, 128, False), (1, 4, 4, 2300, 2300, 128, False), (1, 4, 2, 3001, 3001, 64, False),
    (1, 4, 4, 3001, 3001, 128, True), (16, 12, 3, 400, 400, 64, True), (16, 12, 12, 401, 401, 64, True), (8, 12, 12, 315, 315, 128, False), (2, 32, 8, 607, 607, 64, False),
    (1, 32, 32, 1400, 1400, 64, False), (4, 12, 12, 2264, 2264, 128, False), (8, 8, 8, 2100, 2300, 128, False), (1, 8, 2, 558, 9553, 128, True), (1, 16, 16, 127, 1584, 128, False),
    (3, 16, 16, 5, 700, 64, False), (1, 32, 32, 2500, 2500, 64, True)])
def test_exact_rows_of_a_workgroup(B, H, Hkv, N, Nk, d, causal):
    """Exact calls choose their workgroups' rows by the launch: every Br gives the same rows (up to the order of the sums where
    shares of the keys differ), and they are plain attention's, on either side of each line of the rule."""
    import math

    import torch

    import paper_2507_17245_amd as da
    gen = torch.Generator(device="cuda").manual_seed(N)
    q, k, v = (torch.randn(s, generator=gen, device="cuda").bfloat16() for s in ((B, H, N, d), (B, Hkv, Nk, d), (B, Hkv, Nk, d)))
    rows = torch.cat([torch.arange(0, N, max(1, N // 37)), torch.arange(max(0, N - 40), N)]).unique()
    b, h = B - 1, H - 1
    kd, vd = (x[b, h // (H // Hkv)].double().cpu() for x in (k, v))
    s = torch.matmul(q[b, h].double().cpu()[rows], kd.t().contiguous()) / math.sqrt(d)
    if causal:
        s = s.masked_fill(torch.arange(Nk)[None, :] > rows[:, None] + (Nk - N), -math.inf)
    want, want_lse = torch.matmul(torch.softmax(s, dim=-1), vd), torch.logsumexp(s, dim=-1)
    for Br in (64, 128, 256):
        print(f"case {(B, H, Hkv, N, Nk, d, causal)} Br={Br}", flush=True)
        o, lse = torch.zeros_like(q), torch.zeros((B, H, N), device="cuda")
        da.distr_attn_exact_fwd_ex(q, k, v, o, da.make_params(q, k, v, Br=Br, causal=causal, lse_out=lse))
        err = (o[b, h].double().cpu()[rows] - want).abs()
        assert err.max() <= 2e-2 and err.mean() <= 2e-3
        assert (lse[b, h].double().cpu()[rows] - want_lse).abs().max() <= 2e-3
        assert torch.isfinite(o.float()).all() and (o.float().abs().sum(dim=-1) > 0).all()


# Two Q blocks of 64 rows in a workgroup (d = 128, keys dealt out): a second block without rows, of one row and whole, on either side of the
# rule's lines, the table given or made; and waves without rows, which take no products, whole and in halves.
@pytest.mark.parametrize("H,Hkv,N,Nk,Br", [(2, 2, 65, 5999, 64), (2, 2, 65, 6000, 64), (2, 1, 128, 6001, 64), (1, 1, 129, 6400, 64), (3, 3, 190, 6000, 64), (2, 2, 250, 6000, 64),
                                           (2, 2, 100, 6000, 128), (2, 1, 160, 3000, 128), (2, 2, 290, 2000, 256), (70, 70, 65, 1700, 128)])
@pytest.mark.parametrize("n_groups,given", [(64, False), (32, True)])
def test_blocks_that_share_a_workgroup(H, Hkv, N, Nk, Br, n_groups, given):
    import gpu_util as U
    import torch
    cfg = W.CONFIGS["long"].scaled(B=1, H=H, Hkv=Hkv, N=N, Nk=Nk, Br=Br, causal=True, n_groups=n_groups, recipe="normal")
    print(f"case {cfg}", flush=True)
    q, k, v = W.make(cfg)
    p = U.oracle_params(cfg)
    table = oracle.lsh_group(q, p)[1] if given else None
    lse = torch.empty((1, H, N), dtype=torch.float32, device="cuda")
    o, _, _ = U.run_gpu(cfg, q, k, v, lse_out=lse, perm_in=table)
    U.assert_close(o, oracle.distr_fwd(q, k, v, p), "bf16")
    assert np.abs(lse.cpu().numpy() - oracle.lse(q, k, p, distr=True)).max() <= 2e-2


# Workgroups of a part of a Q block (Q~ K^T, keys together): ragged parts, a last block shorter than a part, one part of two; with a table
# handed in, made by the call, asked for, and with a workspace that has no room for one: the same bits.
@pytest.mark.parametrize("base,H,N,Br,causal", [("llama", 4, 830, 128, True), ("llama", 6, 1030, 256, True), ("llama", 2, 300, 256, False), ("long", 4, 810, 128, True),
                                                ("long", 3, 577, 256, False), ("long", 6, 1300, 256, True)])
def test_parts_of_a_block(base, H, N, Br, causal):
    import gpu_util as U
    import torch

    import paper_2507_17245_amd as da
    cfg = W.CONFIGS[base].scaled(B=1, H=H, Hkv=H, N=N, Br=Br, causal=causal, recipe="normal")
    print(f"case {cfg}", flush=True)
    q, k, v = W.make(cfg)
    want = oracle.distr_fwd(q, k, v, U.oracle_params(cfg))
    tq, tk, tv = (U.to_dev(x, "bf16") for x in (q, k, v))
    options = dict(Br=Br, Bc=cfg.Bc, n_groups=cfg.n_groups, causal=causal, lsh_seed=cfg.lsh_seed, n_planes=cfg.n_planes)
    table = torch.zeros((1, H, cfg.Tq, cfg.d), dtype=torch.uint8, device="cuda")
    room = torch.empty(da.distr_attn_kt_bytes(da.make_params(tq, tk, tv, **options)), dtype=torch.uint8, device="cuda")
    outs = []
    for more in (dict(perm_out=table), dict(), dict(perm_in=table), dict(workspace=room)):
        o = torch.zeros_like(tq)
        da.distr_attn_fwd_ex(tq, tk, tv, o, da.make_params(tq, tk, tv, **options, **more))
        outs.append(o)
    U.assert_close(outs[0].float().cpu().numpy().astype(np.float64), want, "bf16")
    assert torch.equal(table.cpu(), torch.from_numpy(oracle.lsh_group(q, U.oracle_params(cfg))[1]))
    assert all(torch.equal(o, outs[0]) for o in outs[1:])


def test_parts_of_a_block_on_many_streams():
    """Calls in flight on several streams, none of which was given a workspace, keep their tables apart."""
    import torch

    import paper_2507_17245_amd as da
    gen = torch.Generator(device="cuda").manual_seed(3)
    qs = [torch.randn((1, 8, 1000, 64), generator=gen, device="cuda").bfloat16() for _ in range(6)]
    k, v = (torch.randn((1, 8, 1000, 64), generator=gen, device="cuda").bfloat16() for _ in range(2))

    def call(q, o):
        da.distr_attn_fwd_ex(q, k, v, o, da.make_params(q, k, v, Br=256, n_groups=32, causal=True))
    want, got = ([torch.zeros_like(q) for q in qs] for _ in range(2))
    for q, o in zip(qs, want):
        call(q, o)
        torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in qs]
    for _ in range(10):
        for q, o, stream in zip(qs, got, streams):
            with torch.cuda.stream(stream):
                call(q, o)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(want, got))


@pytest.mark.parametrize("base,H,N,Br,causal", [("llama", 8, 1000, 128, True), ("llama", 8, 1000, 256, True), ("llama", 2, 300, 256, False), ("long", 4, 810, 128, True),
                                                ("long", 6, 1301, 256, True)])
def test_parts_of_a_block_wherever_called(base, H, N, Br, causal):
    """Which rows a workgroup takes follows from the arguments alone: the same bits without allocations, with a workspace
    that holds no table and from a graph that is replayed. o comes with the bytes 0xff, which neither
    the tables that lie in it meanwhile nor the results may keep."""
    import torch

    import paper_2507_17245_amd as da
    cfg = W.CONFIGS[base].scaled(B=1, H=H, Hkv=H, N=N, Br=Br, causal=causal)
    gen = torch.Generator(device="cuda").manual_seed(N)
    q, k, v = (torch.randn((1, H, N, cfg.d), generator=gen, device="cuda").bfloat16() for _ in range(3))
    options = dict(Br=Br, Bc=cfg.Bc, n_groups=cfg.n_groups, causal=causal, lsh_seed=5)
    fresh = lambda: torch.full((1, H, N, cfg.d), -1, dtype=torch.int16, device="cuda").view(torch.bfloat16)
    print(f"case {(base, H, N, Br, causal)}", flush=True)
    want, table = fresh(), torch.zeros((1, H, cfg.Tq, cfg.d), dtype=torch.uint8, device="cuda")
    da.distr_attn_fwd_ex(q, k, v, want, da.make_params(q, k, v, perm_out=table, **options))
    assert torch.isfinite(want.float()).all()

    def check(o, how):
        torch.cuda.synchronize()
        assert torch.equal(o.view(torch.int16), want.view(torch.int16)), how
    o = fresh()
    da.distr_attn_fwd_ex(q, k, v, o, da.make_params(q, k, v, **options))
    check(o, "plain")
    o = fresh()
    da.distr_attn_fwd_noalloc(q, k, v, o, da.make_params(q, k, v, **options))
    check(o, "without allocations")
    room = torch.empty(da.distr_attn_kt_bytes(da.make_params(q, k, v, **options)), dtype=torch.uint8, device="cuda")
    o = fresh()
    da.distr_attn_fwd_ex(q, k, v, o, da.make_params(q, k, v, workspace=room, **options))
    check(o, "a workspace for the keys alone")
    side, graph, o = torch.cuda.Stream(), torch.cuda.CUDAGraph(), fresh()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        da.distr_attn_fwd_ex(q, k, v, o, da.make_params(q, k, v, **options))
    for rep in range(3):
        o.view(torch.int16).fill_(-1)
        torch.cuda.synchronize()
        graph.replay()
        check(o, f"replay {rep}")


@pytest.mark.parametrize("H,Hkv,N,Nk,causal", [(2, 2, 130, 1535, False), (2, 2, 130, 1601, False), (16, 16, 1030, 1600, True), (16, 16, 1030, 2100, True), (9, 3, 2000, 2000, False)])
def test_row_sums_either_way(H, Hkv, N, Nk, causal):
    """Grouped blocks of 64 rows at d = 128 take the row sums of P by dot products or on the matrix pipe by the length of the walk and the mask: on
    either side of the rule's lines, whole and in halves, the output is the method's."""
    _forward(W.CONFIGS["long"].scaled(B=1, H=H, Hkv=Hkv, N=N, Nk=Nk, Br=64, causal=causal, recipe="normal"), True)
