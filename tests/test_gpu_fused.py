"""GPU parity of the bf16 product over the groups (Q_r K_f^T, read from the transposed keys) at sizes that the forward
would otherwise take over the channels: with kt_in the transposed keys are at hand and the fused kernel is the faster
one. That it ran is checked by handing in the transposed keys of another K, which has to change the output."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


def _cfg(d, **kw):
    return W.CONFIGS["vit" if d == 64 else "mid"].scaled(**{**dict(B=1, recipe="normal"), **kw})


def _call(cfg, q, k, v, kt, **kw):
    """One forward -> (o, lse) as float64 numpy."""
    import torch

    import paper_2507_17245_amd as da
    o = torch.full_like(q, float("nan"))
    lse = torch.full((cfg.B, cfg.H, cfg.N), float("nan"), device="cuda")
    da.distr_attn_fwd_ex(q, k, v, o, da.make_params(q, k, v, Br=cfg.Br, Bc=cfg.Bc, n_groups=cfg.n_groups, causal=cfg.causal,
                                                   lsh_seed=cfg.lsh_seed, n_planes=cfg.n_planes, lse_out=lse, kt_in=kt, **kw))
    return o.double().cpu().numpy(), lse.double().cpu().numpy()


def _transposed(cfg, q, k):
    import torch

    import paper_2507_17245_amd as da
    p = da.make_params(q, k, k, Br=cfg.Br, Bc=cfg.Bc, n_groups=cfg.n_groups, causal=cfg.causal, lsh_seed=cfg.lsh_seed,
                       n_planes=cfg.n_planes)
    return da.distr_attn_key_prepass(k, torch.zeros(da.distr_attn_kt_bytes(p), dtype=torch.uint8, device="cuda"), p)


def _check(cfg, heads=None, batches=(0,)):
    """Every route to the grouping through the fused kernel, against the oracle (sampled Q blocks if `heads` names some)."""
    import torch

    import gpu_util as U
    print(f"case {cfg}", flush=True)
    host = W.make(cfg)
    q, k, v = (U.to_dev(x, "bf16") for x in host)
    kt = _transposed(cfg, q, k)
    perm = torch.full((cfg.B, cfg.H, cfg.Tq, cfg.d), 255, dtype=torch.uint8, device="cuda")
    o, lse = _call(cfg, q, k, v, kt, perm_out=perm)                       # the kernel's own LSH stage
    p = U.oracle_params(cfg)
    assert np.array_equal(perm.cpu().numpy(), oracle.lsh_group(host[0], p)[1])
    if heads is None:
        U.assert_close(o, oracle.distr_fwd(*host, p), "bf16", "fused")
        assert np.abs(lse - oracle.lse(host[0], host[1], p)).max() <= 2e-2
    else:
        tiles = [t for b in batches for t in W.sample_tiles(cfg, heads=heads, batch=b)]
        ref = oracle.distr_fwd_tiles(*host, p, tiles)
        for i, (b, h, t) in enumerate(tiles):
            rows = min(cfg.Br, cfg.N - t * cfg.Br)
            U.assert_close(o[b, h, t * cfg.Br:t * cfg.Br + rows], ref[i, :rows], "bf16", f"block {b, h, t}")
        assert np.isfinite(o).all() and np.isfinite(lse).all()
    hashes = torch.empty(perm.shape, dtype=torch.int32, device="cuda")
    for kw in (dict(hash_out=hashes), dict(perm_in=perm)):                # the LSH kernel's table, the caller's
        o2, lse2 = _call(cfg, q, k, v, kt, **kw)
        assert np.array_equal(o2, o) and np.array_equal(lse2, lse)
    # the transposed keys do not depend on the grouping's options: those of a call with others serve as well
    with_others = cfg.scaled(lsh_seed=cfg.lsh_seed + 1, n_planes=cfg.n_planes + 3, Br=64 if cfg.Br == 128 else 128)
    o3, _ = _call(cfg, q, k, v, _transposed(with_others, q, k))
    assert np.array_equal(o3, o)
    other, _ = _call(cfg, q, k, v, _transposed(cfg, q, -k))
    assert np.abs(other - o).max() > 0.1, "kt_in was not read"
    return q, k, v, o


SHAPES_64 = [(Br, Bc, G) for Br in (64, 128, 256) for Bc in (32, 64, 128) for G in (2, 4)] + [(Br, 64, 8) for Br in (64, 128, 256)]


@pytest.mark.parametrize("Br,Bc,G", SHAPES_64)
@pytest.mark.parametrize("N,Nk,causal", [(450, 450, False), (300, 651, True), (700, 700, True)])
def test_fused_d64(N, Nk, causal, Br, Bc, G):
    _check(_cfg(64, H=32, Hkv=2, N=N, Nk=Nk, causal=causal, Br=Br, Bc=Bc, n_groups=64 // G))


SHAPES_128 = [(Br, Bc, G) for Br in (64, 128, 256) for Bc in (32, 64, 128) for G in (2, 8)] + [(64, 64, 4), (128, 128, 4), (256, 32, 4)]


@pytest.mark.parametrize("Br,Bc,G", SHAPES_128)
@pytest.mark.parametrize("N,Nk,causal", [(1100, 1900, True), (1391, 1391, False)])
def test_fused_d128(N, Nk, causal, Br, Bc, G):
    _check(_cfg(128, H=32, Hkv=2, N=N, Nk=Nk, causal=causal, Br=Br, Bc=Bc, n_groups=128 // G), heads=(0, 15, 31))


# Few enough workgroups for two halves of the keys in each (up to 256; 512 of 64 rows at d = 64; blocks of 128 rows from 24 tiles on): K_f of
# either half from its own tiles of K^T, zero rows that pad 4 and 8 groups in both. Halves of a tile each, of an odd number, none at all (causal).
@pytest.mark.parametrize("d,Br,G,H,Hkv,N,Nk,causal", [
    (d, Br, G, *shape) for d, Br, shapes in ((64, 64, ((8, 2, 1000, 1000, True), (16, 16, 520, 700, False))),
                                             (64, 128, ((16, 4, 1600, 1600, True), (16, 16, 300, 1563, False))),
                                             (128, 64, ((8, 2, 1391, 1391, True), (16, 16, 300, 1473, False))),
                                             (128, 128, ((16, 4, 1600, 1600, True), (16, 16, 700, 1540, False))))
    for G in (2, 4, 8) for shape in shapes] + [
    (64, 64, 16, 32, 1, 490, 9000, False), (64, 128, 16, 32, 1, 700, 6000, False), (128, 64, 16, 32, 1, 490, 4400, False), (128, 128, 16, 32, 1, 700, 3000, False)])
def test_fused_in_halves(d, Br, G, H, Hkv, N, Nk, causal):
    assert H * -(-N // Br) <= 256 and (Br == 64 or Nk > 23 * 64)
    _check(_cfg(d, H=H, Hkv=Hkv, N=N, Nk=Nk, causal=causal, Br=Br, n_groups=d // G), heads=None if Nk < 1000 else (0, H // 2, H - 1))


# Blocks of 64 x 128 at d = 128 take the fused product as soon as there are more workgroups than compute units, with kt_in
# or without: the same bits.
@pytest.mark.parametrize("G", [4, 8])
@pytest.mark.parametrize("N,Nk,causal", [(513, 700, False), (577, 901, True)])
def test_blocks_of_64_by_128(N, Nk, causal, G):
    cfg = _cfg(128, H=32, Hkv=4, N=N, Nk=Nk, causal=causal, Br=64, Bc=128, n_groups=128 // G)
    q, k, v, o = _check(cfg, heads=(0, 31))
    assert np.array_equal(_call(cfg, q, k, v, None)[0], o)


# groups of 16 (contraction zero-padded to one matrix step): fused from many rows per key on
@pytest.mark.parametrize("d,N,Br", [(64, 2070, 64), (64, 2070, 256), (128, 1590, 64), (128, 1590, 128)])
def test_fused_groups_of_16(d, N, Br):
    _check(_cfg(d, H=32, Hkv=1, N=N, Nk=N, causal=False, Br=Br, n_groups=d // 16), heads=(0, 13, 31))


def test_fused_head_major_causal_order():
    """More than 2048 causal query blocks: head by head."""
    cfg = _cfg(64, B=4, H=16, Hkv=16, N=2100, Nk=2100, causal=True, Br=64, n_groups=32)
    assert cfg.B * cfg.H * cfg.Tq > 2048
    _check(cfg, heads=(0, 7, 15), batches=(0, 3))


def test_fused_without_kt_in():
    """Large enough for the call to transpose the keys itself: into the library's workspace, a caller's, or the fixed array of
    the entry that allocates nothing. The same bits as with kt_in, which the product over the channels does not give."""
    import torch

    import paper_2507_17245_amd as da
    cfg = _cfg(64, H=32, Hkv=1, N=1300, Nk=4500, causal=False, Br=64, n_groups=16)
    q, k, v, o = _check(cfg, heads=(0, 31))
    options = dict(Br=cfg.Br, n_groups=cfg.n_groups, n_planes=cfg.n_planes, lsh_seed=cfg.lsh_seed)
    room = torch.empty(da.distr_attn_workspace_bytes(da.make_params(q, k, v, **options)), dtype=torch.uint8, device="cuda")
    for entry, kw in ((da.distr_attn_fwd_ex, {}), (da.distr_attn_fwd_ex, dict(workspace=room)), (da.distr_attn_fwd_noalloc, {})):
        got = entry(q, k, v, torch.empty_like(q), da.make_params(q, k, v, **options, **kw))
        assert np.array_equal(got.double().cpu().numpy(), o)


def test_no_room_for_the_transposed_keys():
    """Transposed keys that the fixed array does not hold: the entry that allocates nothing takes the product over the channels
    where that is light enough, instead of refusing the call; with room it is fused."""
    import torch

    import gpu_util as U
    import paper_2507_17245_amd as da
    cfg = _cfg(64, B=2, H=16, Hkv=16, N=1000, Nk=8192, causal=False, Br=128, n_groups=32)
    print(f"case {cfg}", flush=True)
    host = W.make(cfg)
    q, k, v = (U.to_dev(x, "bf16") for x in host)
    p = da.make_params(q, k, v, Br=cfg.Br, n_groups=cfg.n_groups, n_planes=cfg.n_planes, lsh_seed=cfg.lsh_seed)
    assert da.distr_attn_kt_bytes(p) > da.distr_attn_noalloc_max_bytes()
    fused = da.distr_attn_fwd_ex(q, k, v, torch.empty_like(q), p).double().cpu().numpy()
    assert np.array_equal(fused, _call(cfg, q, k, v, _transposed(cfg, q, k))[0])
    o = da.distr_attn_fwd_noalloc(q, k, v, torch.empty_like(q), p).double().cpu().numpy()
    tiles = W.sample_tiles(cfg, heads=(0, 15), batch=1)
    ref = oracle.distr_fwd_tiles(*host, U.oracle_params(cfg), tiles)
    for i, (b, h, t) in enumerate(tiles):
        rows = min(cfg.Br, cfg.N - t * cfg.Br)
        for x in (fused, o):
            U.assert_close(x[b, h, t * cfg.Br:t * cfg.Br + rows], ref[i, :rows], "bf16", f"block {b, h, t}")


def test_fused_clamps_to_half_range():
    """|q| * scale * log2 e beyond 65504 and |k| beyond 65504 / G* are clamped (documented limit of the product over the
    groups). One large value in head 0's queries, one in head 1's keys, on a channel that is sampled, against small
    ones: the clamped scores spread by 2 to 3, the others by 8. The oracle on clamped values agrees, on the others not."""
    import gpu_util as U
    for n_groups in (32, 16):
        G = 64 // n_groups
        cfg = _cfg(64, H=32, Hkv=32, N=400, Nk=400, causal=False, Br=64, n_groups=n_groups)
        q, k, v = (x.copy() for x in W.make(cfg))
        q *= np.float32(0.25)
        big, tiny = np.float32(2.0 ** 17), np.float32(2.0 ** -14)
        q[0, 0, 70] = 0.0
        q[0, 0, 70, 0] = big
        k[0, 0, :, :G] *= tiny                 # the group of channel 0
        k[0, 1, 10, 0] = big
        q[0, 1, :, 0] *= np.float32(4.0) * tiny
        perm = np.broadcast_to(np.arange(64, dtype=np.uint8), (1, cfg.H, cfg.Tq, 64)).copy()
        tq, tk, tv = (U.to_dev(x, "bf16") for x in (q, k, v))
        import torch
        print(f"case {cfg} clamp", flush=True)
        import paper_2507_17245_amd as da
        o = torch.empty_like(tq)
        da.distr_attn_fwd_ex(tq, tk, tv, o, da.make_params(tq, tk, tv, Br=64, n_groups=n_groups, softmax_scale=1.0,
                                                           perm_in=torch.from_numpy(perm).cuda(), kt_in=_transposed(cfg, tq, tk)))
        o = o.double().cpu().numpy()
        p = U.oracle_params(cfg, scale=1.0)
        q_lim = 65504.0 / np.log2(np.e)
        qc = np.clip(q, -q_lim, q_lim).astype(np.float32)
        kc = np.clip(k, -65504.0 / G, 65504.0 / G).astype(np.float32)
        U.assert_close(o, oracle.distr_fwd(qc, kc, v, p, perm=perm), "bf16", f"clamped, G*={G}")
        plain = oracle.distr_fwd(q, k, v, p, perm=perm)
        for h, rows in ((0, [70]), (1, slice(None))):
            assert np.abs(o[0, h, rows] - plain[0, h, rows]).max() > 0.1      # five times the bar
