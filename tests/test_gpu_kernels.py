"""Kernel-level parity through the measurement hooks: every tile shape of the bf16 GEMM and
the bf16 attention kernel against the oracle's plain loops, at shapes that leave ragged
tiles in every dimension, and the DiT-XL-shaped pass at its benchmark launch size on
sampled slots."""
import numpy as np
import pytest

from paper_2603_25872_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


@pytest.fixture(scope="module")
def drf():
    from paper_2603_25872_amd import drf as d
    d.lib()
    return d


def bf16_round(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(torch.bfloat16)


def block_routes(drf, M, D, tokens):
    """How the four GEMMs of a bf16 block of M rows are run (see drf.probe_gemm_route)."""
    gemms = dict(qkv=(3 * D, D, 1), proj=(D, D, 2), fc1=(4 * D, D, 3), fc2=(D, 4 * D, 2))
    return {name: drf.probe_gemm_route(M, N, K, kind, tokens) for name, (N, K, kind) in gemms.items()}


@pytest.mark.parametrize("variant", [0, 1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("M,N,K", [(300, 292, 128), (517, 1156, 192), (1024, 576, 64), (33, 8, 64), (260, 148, 384)])
def test_gemm_bf16_every_tile_shape(torch, drf, orc, variant, M, N, K):
    rng = np.random.default_rng(M + N + K)
    A = bf16_round(torch, rng.standard_normal((M, K)))
    W = bf16_round(torch, rng.standard_normal((N, K)) * 0.1)
    b = rng.standard_normal(N).astype(np.float32)
    if variant == 8 and K % 128:                 # 16's tile for whole pairs of k-tiles only
        with pytest.raises(drf.DrfError):
            drf.probe_gemm_bf16(A.cuda(), W.cuda(), torch.from_numpy(b).cuda(), variant=variant)
        return
    out = drf.probe_gemm_bf16(A.cuda(), W.cuda(), torch.from_numpy(b).cuda(), variant=variant).float().cpu().numpy()
    want = orc.linear(A.float().numpy(), W.float().numpy(), b)
    err = np.abs(out - want).max() / np.abs(want).max()
    assert err < 6e-3, err                       # bf16 rounding of the stored result: 2^-8 relative at worst


@pytest.mark.parametrize("M,N,K", [(512, 1152, 4608), (300, 292, 2304), (1024, 576, 2304), (130, 132, 2560)])
def test_gemm_bf16_split_k(torch, drf, orc, M, N, K):
    """Few 128 x 128 tiles and a long K: K is split across workgroups and the partial tiles are added by a second
    launch (5 or 6 splits here); same tolerance as the unsplit tile, whose result it must also track closely."""
    rng = np.random.default_rng(M + N + K)
    A = bf16_round(torch, rng.standard_normal((M, K)))
    W = bf16_round(torch, rng.standard_normal((N, K)) * 0.1)
    b = rng.standard_normal(N).astype(np.float32)
    out = drf.probe_gemm_bf16(A.cuda(), W.cuda(), torch.from_numpy(b).cuda(), variant=10).float().cpu().numpy()
    again = drf.probe_gemm_bf16(A.cuda(), W.cuda(), torch.from_numpy(b).cuda(), variant=10).float().cpu().numpy()
    assert np.array_equal(out, again)            # fixed summation order
    whole = drf.probe_gemm_bf16(A.cuda(), W.cuda(), torch.from_numpy(b).cuda(), variant=5).float().cpu().numpy()
    want = orc.linear(A.float().numpy(), W.float().numpy(), b)
    scale = np.abs(want).max()
    assert np.abs(out - want).max() / scale < 6e-3
    assert np.abs(out - whole).max() / scale < 6e-3   # both are bf16 roundings of nearly the same fp32 sums


@pytest.mark.parametrize("variant", [9, 11, 12, 13, 14, 501, 505, 406, 409, 412])
@pytest.mark.parametrize("M,N,K", [(300, 292, 1152), (33, 8, 1152), (1, 64, 1280), (130, 100, 1408)])
def test_gemm_bf16_small_tiles_and_splits(torch, drf, orc, variant, M, N, K):
    """Tiles of two K groups (9, 11, 12), three-stage tiles (13, 14) and 100 s + tile: K in s parts whose k-steps do not divide evenly (18, 20, 22
    steps in 5 parts; 9, 10, 11 pairs in 4)."""
    rng = np.random.default_rng(M + N + K)
    A = bf16_round(torch, rng.standard_normal((M, K)))
    W = bf16_round(torch, rng.standard_normal((N, K)) * 0.1)
    b = rng.standard_normal(N).astype(np.float32)
    out = drf.probe_gemm_bf16(A.cuda(), W.cuda(), torch.from_numpy(b).cuda(), variant=variant).float().cpu().numpy()
    want = orc.linear(A.float().numpy(), W.float().numpy(), b)
    err = np.abs(out - want).max() / np.abs(want).max()
    assert err < 6e-3, err                       # bf16 rounding of the stored result: 2^-8 relative at worst
    if variant in (9, 11, 12):                   # an odd number of k-tiles has no pairs
        with pytest.raises(drf.DrfError):
            drf.probe_gemm_bf16(A[:, :192].contiguous().cuda(), W[:, :192].contiguous().cuda(), torch.from_numpy(b).cuda(), variant=variant)


@pytest.mark.parametrize("variant", [2, 3, 13, 16, 17, 18, 19, 20])
@pytest.mark.parametrize("M,N,K", [(300, 292, 64), (33, 8, 128), (256, 288, 192), (517, 580, 256), (130, 148, 320), (512, 576, 1088)])
def test_gemm_bf16_four_wave_tiles(torch, drf, orc, variant, M, N, K):
    """With the eight-wave forms of the 256-row ones (18, 19, 20).  1 to 5 and 17 k-tiles: fewer than the stages, as many, one more, odd and even numbers; whole and ragged tiles."""
    rng = np.random.default_rng(M + N + K)
    A = bf16_round(torch, rng.standard_normal((M, K)))
    W = bf16_round(torch, rng.standard_normal((N, K)) * 0.1)
    b = rng.standard_normal(N).astype(np.float32)
    out = drf.probe_gemm_bf16(A.cuda(), W.cuda(), torch.from_numpy(b).cuda(), variant=variant).float().cpu().numpy()
    want = orc.linear(A.float().numpy(), W.float().numpy(), b)
    err = np.abs(out - want).max() / np.abs(want).max()
    assert err < 6e-3, err                       # bf16 rounding of the stored result: 2^-8 relative at worst


@pytest.mark.parametrize("variant,bm,bn", [(21, 256, 192), (22, 192, 288)])
@pytest.mark.parametrize("dm,dn,K", [(0, 0, 64), (1, 4, 128), (-1, -4, 192), (0, 0, 1088), (37, 100, 320), (-150, -180, 256)])
def test_gemm_bf16_tiles_for_part_filled_rounds(torch, drf, orc, variant, bm, bn, K, dm, dn):
    """Two tiles each way, whole, one row and four columns more and less, ragged, and fewer than one wave's rows and columns; 1 to 5 and 17 k-tiles."""
    M, N = 2 * bm + dm, 2 * bn + dn
    rng = np.random.default_rng(M + N + K)
    A = bf16_round(torch, rng.standard_normal((M, K)))
    W = bf16_round(torch, rng.standard_normal((N, K)) * 0.1)
    b = rng.standard_normal(N).astype(np.float32)
    out = drf.probe_gemm_bf16(A.cuda(), W.cuda(), torch.from_numpy(b).cuda(), variant=variant).float().cpu().numpy()
    want = orc.linear(A.float().numpy(), W.float().numpy(), b)
    err = np.abs(out - want).max() / np.abs(want).max()
    assert err < 6e-3, err                       # bf16 rounding of the stored result: 2^-8 relative at worst


@pytest.mark.parametrize("M,N,K", [(20011, 1152, 384), (12803, 1540, 384), (10957, 1540, 384)])
def test_gemm_bf16_rows_in_two_launches(torch, drf, M, N, K):
    """Full rounds of one tile and the remaining rows with another: same sums in the same order as one launch of a
    third tile (neither splits K), so the same bits; ragged last row and column tiles."""
    tile, _, first_tile, first_rows = drf.probe_gemm_route(M, N, K)
    assert 0 < first_rows < M and not {tile, first_tile} & {9, 11, 12, 13, 16, 17}      # (those add two halves of the sums)
    g = torch.Generator(device="cuda").manual_seed(M)
    A = torch.randn((M, K), generator=g, device="cuda").bfloat16()
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.1).bfloat16()
    b = torch.randn((N,), generator=g, device="cuda")
    out = drf.probe_gemm_bf16(A, W, b)
    assert torch.equal(out, drf.probe_gemm_bf16(A, W, b, variant=1))


@pytest.mark.parametrize("variant", [-1, 15, 99, 100])
def test_gemm_bf16_number_that_names_no_tile(torch, drf, variant):
    """Taken by the 128 x 128 tile, as such numbers always were by a general one."""
    g = torch.Generator(device="cuda").manual_seed(5)
    A = torch.randn((130, 192), generator=g, device="cuda").bfloat16()
    W = (torch.randn((100, 192), generator=g, device="cuda") * 0.1).bfloat16()
    b = torch.randn((100,), generator=g, device="cuda")
    assert torch.equal(drf.probe_gemm_bf16(A, W, b, variant=variant), drf.probe_gemm_bf16(A, W, b, variant=5))


def test_gemm_bf16_rejects_bad_k(torch, drf):
    A = torch.zeros((64, 72), dtype=torch.bfloat16, device="cuda")
    W = torch.zeros((64, 72), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(drf.DrfError):
        drf.probe_gemm_bf16(A, W, torch.zeros(64, device="cuda"))


@pytest.mark.parametrize("slots,T,H,d", [(3, 256, 2, 72), (2, 77, 3, 64), (5, 15, 4, 32), (1, 300, 1, 96), (2, 130, 2, 48),
                                          (1, 1, 2, 16), (2, 192, 1, 80), (1, 129, 1, 80), (2, 640, 2, 72), (1, 255, 2, 24),
                                          (40, 200, 8, 72), (65, 136, 4, 40)])     # more work items than CUs
def test_attention_bf16_shapes(torch, drf, orc, slots, T, H, d):
    rng = np.random.default_rng(T + d)
    qkv = bf16_round(torch, rng.standard_normal((slots * T, 3 * H * d)) * 1.5)
    out = drf.probe_attn_bf16(qkv.cuda(), slots, T, H, d).float().cpu().numpy()
    want = orc.attention_packed(qkv.float().numpy(), T, H, d)
    err = np.abs(out - want).max() / np.abs(want).max()
    assert err < 1.5e-2, err


@pytest.mark.parametrize("d", [8, 16, 24, 32, 40, 48, 56, 64, 72, 80, 88, 96])
@pytest.mark.parametrize("T", [257, 320, 545])
def test_attention_bf16_long_sequences(torch, drf, orc, d, T):
    """More than 256 kv rows: every head width, last steps of 1 and 32 rows, a last chunk of one row, and a last query
    block in which three of four waves have no query."""
    slots, H = 2, 3
    rng = np.random.default_rng(1000 * d + T)
    qkv = bf16_round(torch, rng.standard_normal((slots * T, 3 * H * d)) * 1.5)
    out = drf.probe_attn_bf16(qkv.cuda(), slots, T, H, d).float().cpu().numpy()
    want = orc.attention_packed(qkv.float().numpy(), T, H, d)
    err = np.abs(out - want).max() / np.abs(want).max()
    assert err < 1.5e-2, err                     # P and the result rounded to bf16: 2^-8 relative each at worst


@pytest.mark.parametrize("d", [8, 16, 24, 32, 40, 48, 56, 64, 72, 80, 88, 96])
@pytest.mark.parametrize("slots,T,H,scale", [(3, 1, 2, 1.5), (2, 31, 3, 1.5), (2, 64, 1, 1.5), (3, 65, 2, 1.5), (1, 193, 2, 1.5),
                                             (1, 256, 2, 6.0), (300, 40, 8, 1.5)])
def test_attention_bf16_one_wave_per_64_rows(torch, drf, orc, slots, T, H, scale, d):
    """Up to 256 kv rows split over the waves of a workgroup: every head width, one to four waves, last waves of 1 and
    64 rows, partly empty query blocks, large scores (the waves' maxima differ), and enough items for 64-query blocks."""
    rng = np.random.default_rng(1000 * d + T)
    qkv = bf16_round(torch, rng.standard_normal((slots * T, 3 * H * d)) * scale)
    out = drf.probe_attn_bf16(qkv.cuda(), slots, T, H, d).float().cpu().numpy()
    want = orc.attention_packed(qkv.float().numpy(), T, H, d)
    err = np.abs(out - want).max() / np.abs(want).max()
    assert err < 1.5e-2, err                     # P and the result rounded to bf16: 2^-8 relative each at worst


def test_attention_bf16_large_scores_and_lazy_rescale(torch, drf, orc):
    # score ranges far beyond the lazy-rescale headroom, increasing along kv so the reference moves often
    slots, T, H, d = 1, 512, 1, 64
    rng = np.random.default_rng(3)
    q = rng.standard_normal((T, d)) * 4
    k = rng.standard_normal((T, d)) * np.linspace(0.2, 6, T)[:, None]
    v = rng.standard_normal((T, d))
    qkv = bf16_round(torch, np.concatenate([q, k, v], axis=1))
    out = drf.probe_attn_bf16(qkv.cuda(), slots, T, H, d).float().cpu().numpy()
    want = orc.attention_packed(qkv.float().numpy(), T, H, d)
    assert np.isfinite(out).all()
    assert np.abs(out - want).max() / np.abs(want).max() < 2e-2


def test_config3_pass_at_benchmark_size_sampled_slots(torch, drf, orc):
    """The 64-slot draft pass of configuration 3 (8 drafts-by-guidance groups of batch 8, distinct
    timesteps per group) as bench.py launches it; the oracle evaluates two sampled slots."""
    cfg = I.config(3)
    dit = cfg["dit"]
    w = I.weights(dit, 3)
    den = drf.Denoiser(dit, w)
    slots = cfg["n"] * 2 * cfg["batch"]
    rng = np.random.default_rng(33)
    x = rng.standard_normal((slots, 4, 32, 32)).astype(np.float32)
    stride = 1000 // cfg["sched"]["steps"]
    t = np.repeat(np.array([(49 - i) * stride for i in range(4)], np.int32), 16)       # tau of s = 50..47, per group
    cls = I.conditioning(dit, slots, 3)
    cls[1::2] = dit["cond_dim"]                                                         # null class on odd slots
    got = den.eps_batched(torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda(), torch.from_numpy(cls).cuda())
    got = got.cpu().numpy()
    den.close()
    assert np.isfinite(got).all()
    wd = orc.prepare_weights(w)
    for j in (5, 62):
        want = orc.dit_eps(dit, wd, x[j:j + 1], t[j:j + 1], cls[j:j + 1])[0]
        err = np.abs(got[j] - want).max() / np.abs(want).max()
        assert err < 2e-2, (j, err)


@pytest.mark.parametrize("slots,gemms", [(34, {"proj", "fc1", "fc2"}), (23, {"qkv", "fc1"})])
def test_pass_whose_gemms_run_in_two_launches_sampled_slots(torch, drf, orc, slots, gemms):
    """247-token slots, no multiple of any tile: the GEMMs named run as full rounds of one tile and the remaining rows with another,
    whose first row lies inside a slot: gates, head-major planes and GELU across it.  The slots at each seam are compared."""
    dit = dict(I.CONFIGS[3]["dit"], depth=2, lat_h=26, lat_w=38)
    seams = {name: r[3] // 247 for name, r in block_routes(drf, slots * 247, 1152, 247).items() if r[3]}
    assert set(seams) == gemms
    w = I.weights(dit, 3, "loud")
    den = drf.Denoiser(dit, w)
    rng = np.random.default_rng(slots)
    x = rng.standard_normal((slots, 4, 26, 38)).astype(np.float32)
    t = rng.integers(0, 1000, size=slots).astype(np.int32)
    cls = I.conditioning(dit, slots, 3)
    got = den.eps_batched(torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda(), torch.from_numpy(cls).cuda()).cpu().numpy()
    den.close()
    wd = orc.prepare_weights(w)
    for j in sorted({0, slots - 1} | set(seams.values()) | {j - 1 for j in seams.values()}):
        want = orc.dit_eps(dit, wd, x[j:j + 1], t[j:j + 1], cls[j:j + 1])[0]
        err = np.abs(got[j] - want).max() / np.abs(want).max()
        assert err < 2e-2, (j, err)


@pytest.mark.parametrize("lat,slots,tiles", [
    ((36, 28), 5, dict(qkv=16)), ((36, 28), 8, dict(proj=17, fc1=18, fc2=17)), ((36, 28), 10, dict(qkv=18, proj=7, fc1=3, fc2=7)),
    ((36, 28), 15, dict(qkv=3, proj=16, fc1=2, fc2=16)), ((36, 28), 19, dict(qkv=20)), ((36, 28), 31, dict(qkv=19, proj=18, fc1=20, fc2=13)),
    ((36, 28), 24, dict(fc1=19)),
    ((18, 14), 10, dict(qkv=17, fc1=7)), ((18, 14), 15, dict(fc1=16)), ((18, 14), 19, dict(qkv=16)), ((18, 14), 29, dict(proj=17, fc1=18, fc2=17)),
    ((18, 14), 57, dict(qkv=3, proj=16, fc1=2, fc2=16)), ((18, 14), 122, dict(qkv=19, proj=18, fc1=20, fc2=13)),
    ((8, 8), 37, dict(qkv=17)), ((8, 8), 41, dict(qkv=7)), ((8, 8), 73, dict(qkv=16)), ((8, 8), 113, dict(proj=17, fc1=18, fc2=17)),
    ((8, 8), 145, dict(qkv=18, fc1=3)), ((8, 8), 225, dict(proj=16, fc1=2, fc2=16)), ((8, 8), 481, dict(proj=18, fc1=20, fc2=13))])
def test_pass_of_ragged_slots_on_every_middle_tile_sampled_slots(torch, drf, orc, lat, slots, tiles):
    """252, 63 and 16 tokens a slot at row counts that no tile divides: the tiles of two pairs of waves (13, 16, 17), 256-row ones on
    four and eight waves (2, 3, 18, 19, 20) and 128 x 96 with head-major stores whose 32 rows cross slots, gates of two to four
    rows in LDS and of more from memory, GELU, and the last block's gated update of the stream; slots at tile edges are compared."""
    T = lat[0] * lat[1] // 4
    M = slots * T
    routes = block_routes(drf, M, 1152, T)
    assert {name: routes[name][:2] for name in tiles} == {name: (tile, 1) for name, tile in tiles.items()}
    dit = dict(I.CONFIGS[3]["dit"], depth=2, lat_h=lat[0], lat_w=lat[1])
    w = I.weights(dit, 3, "loud")
    den = drf.Denoiser(dit, w)
    rng = np.random.default_rng(slots)
    x = rng.standard_normal((slots, 4, *lat)).astype(np.float32)
    t = rng.integers(0, 1000, size=slots).astype(np.int32)
    cls = I.conditioning(dit, slots, 3)
    got = den.eps_batched(torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda(), torch.from_numpy(cls).cuda()).cpu().numpy()
    den.close()
    wd = orc.prepare_weights(w)
    for j in sorted({r // T for r in (0, 64, 128, 255, 256, M // 256 * 256 - 1, M - 1) if r < M}):
        want = orc.dit_eps(dit, wd, x[j:j + 1], t[j:j + 1], cls[j:j + 1])[0]
        err = np.abs(got[j] - want).max() / np.abs(want).max()
        assert err < 2e-2, (j, err)


@pytest.mark.parametrize("text,lat,slots,tiles", [
    (False, (36, 28), 13, dict(qkv=21)), (False, (32, 32), 13, dict(qkv=21)), (False, (18, 14), 56, dict(qkv=21)),
    (False, (36, 28), 40, dict(proj=21, fc2=21)), (False, (18, 14), 160, dict(proj=21, fc2=21)),
    (False, (36, 28), 45, dict(proj=22, fc2=22)), (False, (18, 14), 180, dict(proj=22, fc2=22)),
    (False, (32, 28), 17, dict(qkv=22)), (False, (8, 16), 120, dict(qkv=22)), (False, (32, 32), 48, dict(qkv=22, proj=22, fc2=22)),
    (True, (32, 32), 34, dict(proj=21, xq=21, xo=21, fc2=21)), (True, (36, 28), 45, dict(proj=22, xq=22, xo=22, fc2=22))])
def test_pass_on_tiles_for_part_filled_rounds_sampled_slots(torch, drf, orc, text, lat, slots, tiles):
    """256 x 192 (21) and 192 x 288 (22) in the launches that take them: head-major planes of slots of whole 32-row passes, whose tiles begin
    inside slots of 224 and cover several of 32, and (21) of others; one gate row, two, and more than LDS holds; the plain store and the update of the
    stream, gated (last block) and not (behind the cross-attention).  The slots at tile edges are compared."""
    T = lat[0] * lat[1] // 4
    M = slots * T
    routes = dict(block_routes(drf, M, 1152, T), xq=drf.probe_gemm_route(M, 1152, 1152, 4, T), xo=drf.probe_gemm_route(M, 1152, 1152, 4, T))
    assert {name: routes[name] for name in tiles} == {name: (tile, 1, 0, 0) for name, tile in tiles.items()}
    dit = dict(I.CONFIGS[4 if text else 3]["dit"], depth=2, lat_h=lat[0], lat_w=lat[1])
    assert dit["hidden"] == 1152
    w = I.weights(dit, 3, "loud")
    den = drf.Denoiser(dit, w)
    rng = np.random.default_rng(slots)
    x = rng.standard_normal((slots, dit["in_ch"], *lat)).astype(np.float32)
    t = rng.integers(0, 1000, size=slots).astype(np.int32)
    cond = I.conditioning(dit, slots, 3)
    got = den.eps_batched(torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda(), torch.from_numpy(cond).cuda()).cpu().numpy()
    den.close()
    assert np.isfinite(got).all()
    wd = orc.prepare_weights(w)
    for j in sorted({r // T for r in (0, 191, 256, M // 192 * 192 - 1, M - 1)}):
        want = orc.dit_eps(dit, wd, x[j:j + 1], t[j:j + 1], cond[j:j + 1])[0]
        err = np.abs(got[j] - want).max() / np.abs(want).max()
        assert err < 2e-2, (j, err)


@pytest.mark.parametrize("g,n_chain,n_draft", [(2, 4, 4), (1, 3, 0), (2, 0, 4), (1, 1, 1)])
def test_fused_update_probe_equals_its_parts(torch, drf, orc, g, n_chain, n_draft):
    """The measurement hook that launches the fused guidance + chain + draft update once, against the same steps
    made of refine_step / skip_transition calls and against the oracle's operator."""
    sd = dict(train_steps=1000, beta_start=1e-4, beta_end=0.02, steps=50, eta=0.0)
    rng = np.random.default_rng(g * 100 + n_chain * 10 + n_draft)
    shape, s_from, w = (3, 4, 8, 8), 20, 4.0
    x = rng.standard_normal(shape).astype(np.float32)
    eps = rng.standard_normal((max(n_chain, 1), g) + shape).astype(np.float32)
    xd, ed = torch.from_numpy(x).cuda(), torch.from_numpy(eps).cuda()
    x_out, drafts = drf.probe_update_fused(sd, s_from, n_chain, n_draft, g, w, xd, ed)
    guided = ed[:, 0] if g == 1 else ed[:, 1] + w * (ed[:, 0] - ed[:, 1])
    y, s = xd, s_from
    want = x.astype(np.float64)
    gn = guided.cpu().numpy().astype(np.float64)
    for i in range(n_chain):
        y = drf.refine_step(sd, y, guided[i].contiguous(), s)
        want = orc.skip(want, gn[i], orc.abar_at(sd, s), orc.abar_at(sd, s - 1))
        s -= 1
    assert np.abs(x_out.cpu().numpy() - y.cpu().numpy()).max() < 1e-5
    assert np.abs(x_out.cpu().numpy() - want).max() / np.abs(want).max() < 1e-5
    if n_draft:
        anchor = guided[n_chain - 1 if n_chain else 0].contiguous()
        parts = drf.skip_transition(sd, y, anchor, s, [s - j - 1 for j in range(n_draft)])
        assert np.abs(drafts.cpu().numpy() - parts.cpu().numpy()).max() < 1e-5


@pytest.mark.parametrize("hidden", [128, 384, 576, 768, 1024, 1152])
@pytest.mark.parametrize("slots,in_ch", [(1, 4), (65, 5), (66, 4)])
def test_final_layer_of_one_and_two_rounds_of_workgroups(torch, drf, orc, hidden, slots, in_ch):
    """A model without blocks, 63 tokens a slot: 63, 4095 and 4158 rows (4, 256 and 260 workgroups of 16 rows), the last of them ragged;
    16 and 20 outputs a token.  fp32 sums of at most 1152 products: 1152 x 2^-24 relative at worst."""
    dit = dict(I.CONFIGS[1]["dit"], depth=0, hidden=hidden, heads=hidden // 64, lat_h=18, lat_w=14, in_ch=in_ch)
    w = I.weights(dit, 5, "loud")
    den = drf.Denoiser(dit, w)
    rng = np.random.default_rng(hidden + slots)
    x = rng.standard_normal((slots, in_ch, 18, 14)).astype(np.float32)
    t = rng.integers(0, 1000, size=slots).astype(np.int32)
    cond = I.conditioning(dit, slots, 5)
    got = den.eps_batched(torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda(), torch.from_numpy(cond).cuda()).cpu().numpy()
    den.close()
    wd = orc.prepare_weights(w)
    for j in {0, slots // 2, slots - 1}:
        want = orc.dit_eps(dit, wd, x[j:j + 1], t[j:j + 1], cond[j:j + 1])[0]
        err = np.abs(got[j] - want).max() / np.abs(want).max()
        assert err < 7e-5, (j, err)
