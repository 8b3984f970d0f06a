"""Parity of the HIP path (through the C ABI) with the CPU oracle on the same seeded
inputs.  Tolerances are the workload's: plan/timestep bookkeeping bit-exact (checked
on the host in test_host_abi.py), fp32 path max-norm relative error <= 1e-4, bf16
path <= 2e-2, where error = max|gpu - oracle| / max|oracle| per sample; the same numbers
also bound every element's error against |oracle| + rms(oracle) (tests/parity.py)."""
import os

import numpy as np
import pytest

from paper_2603_25872_amd import inputs as I
from parity import TOL_BF16, TOL_F32, check, relerr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


@pytest.fixture(scope="module")
def drf():
    from paper_2603_25872_amd import drf as d
    d.lib()
    return d


def dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


SCHED20 = dict(train_steps=1000, beta_start=1e-4, beta_end=0.02, steps=20, eta=0.0)


# ------------------------------------------------------------ update kernels

@pytest.mark.parametrize("shape", [(1, 4, 16, 16), (3, 1021), (2, 4, 32, 32), (5, 3)])
def test_skip_transition_matches_oracle(torch, drf, orc, shape):
    rng = np.random.default_rng(1)
    x = rng.standard_normal(shape).astype(np.float32)
    e = rng.standard_normal(shape).astype(np.float32)
    for s_from, targets in [(20, [19, 18, 17]), (7, [6]), (3, [2, 1, 0]), (5, [9, 5])]:
        got = drf.skip_transition(SCHED20, dev(torch, x), dev(torch, e), s_from, targets).cpu().numpy()
        for j, s_to in enumerate(targets):
            want = orc.skip(x, e, orc.abar_at(SCHED20, s_from), orc.abar_at(SCHED20, s_to))
            assert relerr(got[j], want) < 1e-5, (s_from, s_to)


def test_refine_step_is_the_unit_skip_bit_for_bit(torch, drf, orc):
    rng = np.random.default_rng(2)
    x = rng.standard_normal((2, 4, 16, 16)).astype(np.float32)
    e = rng.standard_normal((2, 4, 16, 16)).astype(np.float32)
    xd, ed = dev(torch, x), dev(torch, e)
    for s in (20, 11, 1):
        a = drf.refine_step(SCHED20, xd, ed, s).cpu().numpy()
        b = drf.skip_transition(SCHED20, xd, ed, s, [s - 1]).cpu().numpy()[0]
        assert np.array_equal(a, b)
        assert relerr(a, orc.skip(x, e, orc.abar_at(SCHED20, s), orc.abar_at(SCHED20, s - 1))) < 1e-5
    # in-place refine
    y = xd.clone()
    drf.refine_step(SCHED20, y, ed, 9, out=y)
    assert np.array_equal(y.cpu().numpy(), drf.refine_step(SCHED20, xd, ed, 9).cpu().numpy())


def test_update_edge_cases(torch, drf):
    empty = torch.empty((0, 16), dtype=torch.float32, device="cuda")
    assert drf.skip_transition(SCHED20, empty, empty, 5, [4]).shape == (1, 0, 16)
    x = torch.ones((1, 8), dtype=torch.float32, device="cuda")
    with pytest.raises(drf.DrfError):
        drf.skip_transition(SCHED20, x, x, 21, [3])
    with pytest.raises(drf.DrfError):
        drf.skip_transition(SCHED20, x, x, 5, [-1])
    with pytest.raises(drf.DrfError):
        drf.refine_step(dict(SCHED20, eta=1.0), x, x, 5)
    # many targets (more than one argument block)
    tg = [i % 21 for i in range(70)]
    out = drf.skip_transition(SCHED20, x, x * 0.5, 10, tg)
    assert out.shape == (70, 1, 8)
    assert torch.equal(out[3], out[3 + 21]) and torch.equal(out[10], x)


# ------------------------------------------------------------------ DiT forward

def small_dit(cond, dtype, **kw):
    base = dict(depth=2, hidden=128, heads=4, mlp_ratio=4, patch=2, in_ch=4, lat_h=10, lat_w=6, dtype=dtype,
                cond=cond, cond_dim={0: 24, 1: 10, 2: 64}[cond], ctx_len=7 if cond == I.COND_TEXT else 0)
    base.update(kw)
    return base


def make_cond(dit, slots, seed):
    rng = np.random.default_rng(seed)
    if dit["cond"] == I.COND_VECTOR:
        return rng.standard_normal((slots, dit["cond_dim"])).astype(np.float32)
    if dit["cond"] == I.COND_CLASS:
        return rng.integers(0, dit["cond_dim"] + 1, size=slots).astype(np.int32)
    return rng.standard_normal((slots, dit["ctx_len"], dit["cond_dim"])).astype(np.float32)


def check_forward(torch, drf, orc, dit, init, slots, tol, seed=0, trace=True):
    w = I.weights(dit, 40 + seed, init)
    rng = np.random.default_rng(50 + seed)
    x = rng.standard_normal((slots, dit["in_ch"], dit["lat_h"], dit["lat_w"])).astype(np.float32)
    t = rng.integers(0, 1000, size=slots).astype(np.int32)
    t[0], t[-1] = 0, 999
    cond = make_cond(dit, slots, 60 + seed)
    den = drf.Denoiser(dit, w)
    xd, td, cd = dev(torch, x), dev(torch, t), dev(torch, cond)
    errs = {}
    if trace:
        for k in range(dit["depth"] + 1):
            got = den.eps_trace(xd, td, cd, k).cpu().numpy()
            errs["resid%d" % k] = check(got, orc.dit_eps(dit, w, x, t, cond, stop_blocks=k), tol, "resid%d" % k)[0]
    got = den.eps_batched(xd, td, cd).cpu().numpy()
    want = orc.dit_eps(dit, w, x, t, cond)
    errs["eps"] = check(got, want, tol, "eps")[0]
    den.close()
    return errs


@pytest.mark.parametrize("cond", [I.COND_VECTOR, I.COND_CLASS, I.COND_TEXT])
@pytest.mark.parametrize("init", ["paper", "loud"])
def test_fp32_forward_matches_oracle(torch, drf, orc, cond, init):
    check_forward(torch, drf, orc, small_dit(cond, I.F32), init, slots=3, tol=TOL_F32, seed=cond)


def test_fp32_forward_odd_shapes(torch, drf, orc):
    # hidden 72 with 3 heads of 24, one token row, patch 1
    dit = small_dit(I.COND_CLASS, I.F32, hidden=72, heads=3, patch=1, lat_h=3, lat_w=5, depth=1, mlp_ratio=2)
    check_forward(torch, drf, orc, dit, "loud", slots=5, tol=TOL_F32, seed=7)


@pytest.mark.parametrize("kw", [dict(cond=I.COND_VECTOR, hidden=20, heads=4, cond_dim=7, lat_h=6, lat_w=6),          # d = 5
                                dict(cond=I.COND_TEXT, hidden=36, heads=2, cond_dim=6, ctx_len=35, lat_h=8, lat_w=8),   # d = 18
                                dict(cond=I.COND_CLASS, hidden=128, heads=1, lat_h=24, lat_w=24, depth=1),              # 144 rows, d = 128
                                dict(cond=I.COND_CLASS, hidden=132, heads=2, lat_h=14, lat_w=4, patch=1, in_ch=5)])     # d = 66, P = 5
def test_fp32_forward_operands_that_no_vector_load_takes(torch, drf, orc, kw):
    """Widths that are not multiples of 4 or 16, K remainders, kv rows beyond one round of the waves."""
    cond = kw.pop("cond")
    check_forward(torch, drf, orc, small_dit(cond, I.F32, **kw), "loud", slots=3, tol=TOL_F32, seed=70 + kw["hidden"])


def test_fp32_attention_scores_of_minus_infinity_in_one_waves_rows(torch, drf, orc):
    """Context rows 32-63, one wave's share, score below the range of fp32: they get no weight."""
    dit = small_dit(I.COND_TEXT, I.F32, depth=1, ctx_len=70)
    w, D = I.weights(dit, 11, "loud"), dit["hidden"]
    p = I.param_views(dit, w)
    p["blk0.xq_w"][:], p["blk0.xq_b"][:] = 0, 1e19
    p["blk0.xkv_w"][:D] *= 1e-19
    p["blk0.xkv_b"][:D] = 0
    p["blk0.xkv_w"][:D, 0] = -1e25
    rng = np.random.default_rng(12)
    ctx = rng.standard_normal((2, 70, dit["cond_dim"])).astype(np.float32)
    ctx[:, :, 0] = 0
    ctx[:, 32:64, 0] = 1
    x = rng.standard_normal((2, dit["in_ch"], dit["lat_h"], dit["lat_w"])).astype(np.float32)
    t = np.array([3, 900], np.int32)
    den = drf.Denoiser(dit, w)
    got = den.eps_trace(dev(torch, x), dev(torch, t), dev(torch, ctx), 1).cpu().numpy()
    den.close()
    check(got, orc.dit_eps(dit, w, x, t, ctx, stop_blocks=1), TOL_F32, "resid1")


def test_fp32_conditioning_from_an_unaligned_buffer(torch, drf, orc):
    dit = small_dit(I.COND_VECTOR, I.F32)
    w, cond = I.weights(dit, 3, "loud"), make_cond(dit, 2, 4)
    rng = np.random.default_rng(5)
    x = rng.standard_normal((2, dit["in_ch"], dit["lat_h"], dit["lat_w"])).astype(np.float32)
    t = np.array([3, 900], np.int32)
    den = drf.Denoiser(dit, w)
    room = torch.zeros(cond.size + 1, device="cuda")
    room[1:] = dev(torch, cond).ravel()
    got = den.eps_batched(dev(torch, x), dev(torch, t), room[1:].view(cond.shape)).cpu().numpy()
    check(got, orc.dit_eps(dit, w, x, t, cond), TOL_F32, "eps")
    den.close()


@pytest.mark.parametrize("cond", [I.COND_VECTOR, I.COND_CLASS, I.COND_TEXT])
@pytest.mark.parametrize("init", ["paper", "loud"])
def test_bf16_forward_matches_oracle(torch, drf, orc, cond, init):
    # 15 tokens per slot: ragged against every tile size; head dim 32
    check_forward(torch, drf, orc, small_dit(cond, I.BF16), init, slots=3, tol=TOL_BF16, seed=10 + cond)


@pytest.mark.parametrize("hidden,heads,lat", [(576, 8, (18, 14)), (384, 6, (32, 32)), (192, 2, (8, 8)), (128, 1, (4, 2))])
def test_bf16_forward_head_dims_and_tiles(torch, drf, orc, hidden, heads, lat):
    # head dims 72, 64, 96, 128->rejected below; 63 / 256 / 16 / 2 tokens per slot
    dit = small_dit(I.COND_CLASS, I.BF16, hidden=hidden, heads=heads, lat_h=lat[0], lat_w=lat[1], depth=2)
    if hidden // heads > 96:
        with pytest.raises(drf.DrfError):
            drf.Denoiser(dit, I.weights(dit, 1))
        return
    check_forward(torch, drf, orc, dit, "loud", slots=5, tol=TOL_BF16, seed=20 + heads)


@pytest.mark.parametrize("cond", [I.COND_CLASS, I.COND_TEXT])
@pytest.mark.parametrize("hidden,heads", [(128, 4), (384, 6), (768, 8), (1024, 16), (1152, 16)])
def test_bf16_thin_pass_branch_outputs_left_as_partial_tiles(torch, drf, orc, hidden, heads, cond):
    # 45 rows: the branch GEMMs split K and the LayerNorm launches add their partial tiles; odd row count
    dit = small_dit(cond, I.BF16, hidden=hidden, heads=heads, depth=2)
    check_forward(torch, drf, orc, dit, "loud", slots=3, tol=TOL_BF16, seed=80 + heads)


@pytest.mark.parametrize("hidden,heads,slots", [(4, 1, 1), (20, 1, 3), (128, 4, 1), (260, 4, 3), (512, 8, 1), (516, 6, 1), (256, 4, 20)])
def test_fp32_forward_rows_normalised_in_the_gemm(torch, drf, orc, hidden, heads, slots):
    """Rows of 4 to 512 (one wave's single step, ragged steps, every wave's full batch) inside the GEMM; 516 and 300 rows of
    256 through a LayerNorm launch; 15 tokens a slot, so row tiles run over slots."""
    check_forward(torch, drf, orc, small_dit(I.COND_CLASS, I.F32, hidden=hidden, heads=heads), "loud", slots=slots, tol=TOL_F32, seed=70 + heads)
    check_forward(torch, drf, orc, small_dit(I.COND_TEXT, I.F32, hidden=hidden, heads=heads, depth=1), "loud", slots=slots, tol=TOL_F32, seed=71)


@pytest.mark.parametrize("hidden,heads,in_ch,patch,lat,slots", [
    (276, 4, 5, 1, (33, 31), 8), (276, 4, 4, 2, (66, 62), 8),       # six column tiles a wave, the last group part-filled, scalar and 16-byte weights
    (276, 4, 5, 1, (33, 31), 7), (132, 2, 5, 1, (33, 31), 17)])     # two: few rows; a group that six would leave mostly empty
def test_patch_embedding_of_ragged_rows_and_columns(torch, drf, orc, hidden, heads, in_ch, patch, lat, slots):
    dit = small_dit(I.COND_CLASS, I.F32, hidden=hidden, heads=heads, in_ch=in_ch, patch=patch, lat_h=lat[0], lat_w=lat[1], depth=1)
    w = I.weights(dit, 48, "loud")
    rng = np.random.default_rng(58)
    x = rng.standard_normal((slots, in_ch, *lat)).astype(np.float32)
    t = rng.integers(0, 1000, size=slots).astype(np.int32)
    c = make_cond(dit, slots, 68)
    den = drf.Denoiser(dit, w)
    got = den.eps_trace(dev(torch, x), dev(torch, t), dev(torch, c), 0).cpu().numpy()
    den.close()
    check(got, orc.dit_eps(dit, w, x, t, c, stop_blocks=0), TOL_F32, "resid0")


@pytest.mark.parametrize("cond,lat,slots", [(I.COND_CLASS, (32, 32), 65), (I.COND_TEXT, (36, 28), 67), (I.COND_CLASS, (18, 14), 261),
                                            (I.COND_CLASS, (8, 8), 1030)])
def test_bf16_whole_and_edge_tiles_of_a_fat_pass(torch, drf, orc, cond, lat, slots):
    """More rows than one round of the largest GEMM tiles: 256 tokens (whole tiles, one gate row each), 252 and 63 (tiles over
    two to six slots, a ragged last row tile), 16 (more slots to a tile than gate rows are kept); slots at both ends, at a
    seam of the first tiles and in the middle against the oracle."""
    dit = small_dit(cond, I.BF16, hidden=1152, heads=16, depth=2, lat_h=lat[0], lat_w=lat[1])
    w = I.weights(dit, 47, "loud")
    rng = np.random.default_rng(57)
    x = rng.standard_normal((slots, dit["in_ch"], dit["lat_h"], dit["lat_w"])).astype(np.float32)
    t = rng.integers(0, 1000, size=slots).astype(np.int32)
    c = make_cond(dit, slots, 67)
    den = drf.Denoiser(dit, w)
    got = den.eps_batched(dev(torch, x), dev(torch, t), dev(torch, c)).cpu().numpy()
    den.close()
    pick = [0, 1, slots // 2, slots - 1]
    check(got[pick], orc.dit_eps(dit, w, x[pick], t[pick], c[pick]), TOL_BF16, "eps")


@pytest.mark.parametrize("hidden,heads,lat,slots,ratio,route", [
    (256, 4, (10, 6), 3, 4, 16),        # 15 tokens: one part-filled row tile a slot; no room for whole key groups in the buffers
    (256, 4, (2, 2), 5, 2, 16),         # one token
    (256, 4, (16, 16), 5, 2, 21016), (256, 4, (8, 16), 4, 3, 21016), (256, 4, (16, 16), 50, 2, 1016),
    (256, 4, (18, 14), 1, 4, 41016), (384, 6, (26, 38), 4, 4, 41016), (512, 8, (26, 38), 3, 4, 41016),
    (384, 6, (26, 38), 5, 4, 21016), (256, 4, (26, 38), 8, 4, 21016), (512, 8, (26, 38), 7, 4, 21016),    # q, k, v in three parts, in two
    (384, 6, (26, 38), 12, 4, 1016),    # 247 tokens: a row tile and a key group of 15 and 23
    (384, 6, (26, 38), 25, 4, 1032), (256, 4, (26, 38), 30, 4, 1032), (512, 8, (26, 38), 25, 4, 1032),
    (512, 8, (26, 38), 16, 4, 1016),
    (384, 12, (26, 38), 10, 4, 16), (384, 12, (26, 38), 25, 4, 32), (384, 4, (26, 38), 50, 4, 64), (256, 8, (26, 38), 60, 4, 64),
    (512, 16, (26, 38), 30, 1, 32),
    (384, 6, (48, 50), 8, 4, 1032),     # 600 tokens
    (384, 6, (8, 8), 5, 4, 0)])
def test_bf16_rows_of_a_block_in_one_launch(torch, drf, orc, hidden, heads, lat, slots, ratio, route):
    """Narrow models: the launch of a block's row-local part at 16, 32 and 64 rows, with and without the self-attention, whole and
    part-filled row tiles and key groups, every MLP ratio, the hidden units in one, two and four parts; slots at both ends and in the middle against the oracle."""
    dit = small_dit(I.COND_CLASS, I.BF16, hidden=hidden, heads=heads, depth=2, mlp_ratio=ratio, lat_h=lat[0], lat_w=lat[1])
    w = I.weights(dit, 49, "loud")
    assert drf.probe_block_route(slots, lat[0] * lat[1] // 4, hidden, heads, ratio) == route
    rng = np.random.default_rng(59)
    x = rng.standard_normal((slots, dit["in_ch"], dit["lat_h"], dit["lat_w"])).astype(np.float32)
    t = rng.integers(0, 1000, size=slots).astype(np.int32)
    c = make_cond(dit, slots, 69)
    den = drf.Denoiser(dit, w)
    args = dev(torch, x), dev(torch, t), dev(torch, c)
    got, resid = den.eps_batched(*args).cpu().numpy(), den.eps_trace(*args, 1).cpu().numpy()
    assert np.array_equal(got, den.eps_batched(*args).cpu().numpy())
    den.close()
    pick = [0, slots // 2, slots - 1]
    check(resid.reshape(slots, -1)[pick], orc.dit_eps(dit, w, x[pick], t[pick], c[pick], stop_blocks=1).reshape(len(pick), -1), TOL_BF16, "resid1")
    check(got[pick], orc.dit_eps(dit, w, x[pick], t[pick], c[pick]), TOL_BF16, "eps")


@pytest.mark.parametrize("hidden,heads,lat,slots,route", [(256, 8, (26, 38), 17, 32), (512, 16, (26, 38), 13, 16)])
def test_bf16_rows_of_a_block_behind_their_own_attention_launch(torch, drf, orc, hidden, heads, lat, slots, route):
    """The forms without the self-attention at 32 rows of hidden 256 and at 16 of hidden 512, a part-filled row tile in every slot."""
    test_bf16_rows_of_a_block_in_one_launch(torch, drf, orc, hidden, heads, lat, slots, 4, route)


@pytest.mark.parametrize("hidden,slots,route", [(256, 12, 1016), (384, 5, 21016), (384, 4, 41016), (384, 25, 1032), (512, 12, 1016), (512, 25, 1032)])
def test_bf16_scores_of_minus_infinity_in_the_block_launch(torch, drf, orc, hidden, slots, route):
    """Tokens are of two kinds, told apart by one large channel each.  Keys of the second kind score below the range of fp32, those of
    the first around 2e37: the second kind gets no weight, also where it fills the first step of 64 keys, the last or several.  Values
    differ by kind, and hardly within one, so it does not matter which of the far-apart scores of the first kind is the largest."""
    dit = small_dit(I.COND_CLASS, I.BF16, hidden=hidden, heads=hidden // 64, lat_h=26, lat_w=38)
    T, D = 247, hidden
    assert drf.probe_block_route(slots, T, D, D // 64, 4) == route
    w = I.weights(dit, 53, "loud")
    v = I.param_views(dit, w)
    c1, c2 = 5, 70
    v["patch_w"][c1, 0] = v["patch_w"][c2, 4] = 1e4             # channel 0's, channel 1's first pixel of a patch
    v["blk0.ada_w"][:] = 0
    v["blk0.ada_b"][:] = np.repeat(np.float32([0, 0, 1, 0, 0, 1]), D)
    qw, qb = v["blk0.qkv_w"], v["blk0.qkv_b"]
    qw[:D] = 0
    qb[:D:64] = 1e19
    qw[D:2 * D:64] = 0
    qw[D:2 * D:64, c2] = -2.2e20                                # LN gives -1 / sqrt(D) there for the first kind, sqrt(D) for the second
    qb[D:2 * D:64] = 0
    qw[2 * D:] *= 3000
    rng = np.random.default_rng(67)
    x = rng.standard_normal((slots, 4, 13, 2, 19, 2)).astype(np.float32)
    second = [range(0, 64), range(T - 40, T), range(64, 128), range(0, 200)]
    for s in range(slots):
        kind = np.isin(np.arange(T), second[s % 4]).astype(np.float32).reshape(13, 19)
        x[s, 0, :, 0, :, 0], x[s, 1, :, 0, :, 0] = 1 - kind, kind
    x = x.reshape(slots, 4, 26, 38)
    t = rng.integers(0, 1000, size=slots).astype(np.int32)
    c = make_cond(dit, slots, 71)
    den = drf.Denoiser(dit, w)
    args = dev(torch, x), dev(torch, t), dev(torch, c)
    got, resid = den.eps_batched(*args).cpu().numpy(), den.eps_trace(*args, 1).cpu().numpy()
    den.close()
    check(resid.reshape(slots, -1)[:4], orc.dit_eps(dit, w, x[:4], t[:4], c[:4], stop_blocks=1).reshape(4, -1), TOL_BF16, "resid1")
    check(got[:4], orc.dit_eps(dit, w, x[:4], t[:4], c[:4]), TOL_BF16, "eps")


@pytest.mark.parametrize("hidden,heads,lat,slots,route", [(256, 4, (18, 14), 1, 41016), (384, 6, (32, 32), 2, 41016), (512, 8, (26, 38), 7, 21016)])
def test_bf16_every_block_of_a_dealt_pass_is_dealt(torch, drf, orc, hidden, heads, lat, slots, route):
    """The hidden units of every block are dealt, the last one's too: an evaluation has one launch a block more than one whose blocks
    are one launch each, at any depth.  A last block in one launch of few row tiles costs shallow models what dealing gains."""
    rng = np.random.default_rng(61)
    for depth in (1, 3):
        dit = small_dit(I.COND_CLASS, I.BF16, hidden=hidden, heads=heads, depth=depth, mlp_ratio=4, lat_h=lat[0], lat_w=lat[1])
        w = I.weights(dit, 51, "loud")
        den = drf.Denoiser(dit, w)
        tokens, launches = lat[0] * lat[1] // 4, {}
        single = next(s for s in range(slots, 400) if drf.probe_block_route(s, tokens, hidden, heads) == 1016)
        assert drf.probe_block_route(slots, tokens, hidden, heads) == route
        for s in (slots, single):
            x = rng.standard_normal((s, dit["in_ch"], dit["lat_h"], dit["lat_w"])).astype(np.float32)
            t = rng.integers(0, 1000, size=s).astype(np.int32)
            c = make_cond(dit, s, 69)
            args = dev(torch, x), dev(torch, t), dev(torch, c)
            den.profile_enable(True)
            got = den.eps_batched(*args).cpu().numpy()
            launches[s] = den.profile_read(drf.PROF_GEMM)["launches"]
            den.profile_enable(False)
            check(got[:1], orc.dit_eps(dit, w, x[:1], t[:1], c[:1]), TOL_BF16, "eps")
        den.close()
        assert launches[slots] - launches[single] == depth


@pytest.mark.parametrize("lat", [(10, 6), (24, 24)])
def test_bf16_text_context_of_300_rows(torch, drf, orc, lat):
    # 15 and 144 queries over 300 kv rows: the chunked kernel's forms with four and with eight waves
    dit = small_dit(I.COND_TEXT, I.BF16, lat_h=lat[0], lat_w=lat[1], ctx_len=300)
    check_forward(torch, drf, orc, dit, "loud", slots=3, tol=TOL_BF16, seed=90 + lat[0])


@pytest.mark.parametrize("hidden,heads,slots", [(64, 8, 2), (192, 8, 2), (320, 8, 2), (384, 8, 1), (448, 8, 1), (576, 8, 2), (640, 8, 1), (1152, 16, 1),
                                                (128, 8, 17), (256, 8, 17)])
def test_bf16_long_self_attention_with_scaled_queries(torch, drf, orc, hidden, heads, slots):
    """272 tokens at head widths 8 to 80: the projection stores q multiplied by log2(e) / sqrt(d), whole and split GEMMs."""
    dit = small_dit(I.COND_CLASS, I.BF16, hidden=hidden, heads=heads, depth=1, lat_h=32, lat_w=34)
    assert drf.probe_attn_route(slots, 272, 272, heads, hidden // heads, 1) == 7
    check_forward(torch, drf, orc, dit, "loud", slots=slots, tol=TOL_BF16, seed=100 + heads, trace=slots < 17)


def test_bf16_text_cross_attention_77(torch, drf, orc):
    dit = small_dit(I.COND_TEXT, I.BF16, hidden=576, heads=8, lat_h=12, lat_w=12, depth=2, cond_dim=128, ctx_len=77)
    check_forward(torch, drf, orc, dit, "loud", slots=2, tol=TOL_BF16, seed=31)


def test_bf16_attention_with_more_work_items_than_cus(torch, drf, orc):
    # launches whose (query block, head, slot) items outnumber the CUs: self-attention over a ragged 200-token sequence on
    # persistent workgroups, and cross-attention of 1024 queries (four query blocks per head) against a 77-row context on
    # workgroups of 64 queries a wave
    assert drf.probe_attn_route(70, 200, 200, 4, 32) == 4 and drf.probe_attn_route(17, 1024, 77, 4, 32) == 7
    dit = small_dit(I.COND_CLASS, I.BF16, depth=1, lat_h=20, lat_w=40)
    check_forward(torch, drf, orc, dit, "loud", slots=70, tol=TOL_BF16, seed=41, trace=False)
    dit = small_dit(I.COND_TEXT, I.BF16, depth=1, lat_h=64, lat_w=64, ctx_len=77)
    check_forward(torch, drf, orc, dit, "loud", slots=17, tol=TOL_BF16, seed=42, trace=False)


def test_eps_batched_edge_cases(torch, drf):
    dit = small_dit(I.COND_CLASS, I.F32, depth=1)
    den = drf.Denoiser(dit, I.weights(dit, 2))
    x = torch.zeros((0, 4, 10, 6), dtype=torch.float32, device="cuda")
    t = torch.zeros((0,), dtype=torch.int32, device="cuda")
    assert den.eps_batched(x, t, t).shape == (0, 4, 10, 6)
    x1 = torch.randn((2, 4, 10, 6), dtype=torch.float32, device="cuda")
    t1 = torch.tensor([5, 5], dtype=torch.int32, device="cuda")
    # out-of-range class ids are clamped to the null class
    a = den.eps_batched(x1, t1, torch.tensor([10, 10], dtype=torch.int32, device="cuda"))
    b = den.eps_batched(x1, t1, torch.tensor([99, -3], dtype=torch.int32, device="cuda"))
    assert torch.equal(a, b)
    # deterministic: same inputs, same bits; slot order does not matter
    c = den.eps_batched(x1.flip(0).contiguous(), t1, torch.tensor([10, 10], dtype=torch.int32, device="cuda"))
    assert torch.equal(a, c.flip(0))
    with pytest.raises(drf.DrfError):
        drf.Denoiser(dit, I.weights(dit, 2)[:-1])
    den.close()


# ------------------------------------------------------------------ whole path

def run_sample(torch, drf, orc, cfg, tol, mode=None, n=None, batch=None, init="paper", seed=0):
    dit, sd = cfg["dit"], cfg["sched"]
    mode = cfg["mode"] if mode is None else mode
    n = cfg["n"] if n is None else n
    batch = cfg["batch"] if batch is None else batch
    w = I.weights(dit, 70 + seed, init)
    xT = I.latent_noise(dit, batch, 70 + seed)
    cond = I.conditioning(dit, batch, 70 + seed)
    null = I.conditioning(dit, batch, 70 + seed, null=True) if cfg["guidance"] else None
    den = drf.Denoiser(dit, w)
    got = den.sample(sd, mode, n, dev(torch, xT), dev(torch, cond), None if null is None else dev(torch, null),
                     cfg["guidance"] or 0.0).cpu().numpy()
    den.close()
    want = orc.sample_dit(dit, w, sd, mode, n, xT, cond, null, cfg["guidance"] or 0.0)
    return check(got, want, tol, "x_0 %s" % cfg["name"])[0]


@pytest.mark.parametrize("mode", [I.CONSERVATIVE, I.AGGRESSIVE])
@pytest.mark.parametrize("n", [1, 2, 3, 20])
def test_sample_config1_fp32(torch, drf, orc, mode, n):
    # configuration 1 as specified (tiny fp32 DiT, 20-step DDIM), all block sizes incl. n > remaining steps
    run_sample(torch, drf, orc, I.config(1), TOL_F32, mode=mode, n=n)


def test_sample_config1_fp32_loud_with_guidance(torch, drf, orc):
    cfg = I.config(1)
    cfg["guidance"] = 3.0
    run_sample(torch, drf, orc, cfg, TOL_F32, batch=2, init="loud", seed=1)


@pytest.mark.parametrize("mode", [I.CONSERVATIVE, I.AGGRESSIVE])
def test_sample_config2_shape_bf16_reduced(torch, drf, orc, mode):
    # DiT-S width and head count on a 16x16 latent, 3 blocks, 10 steps: the oracle finishes in seconds
    cfg = I.config(2, depth=3, lat_h=16, lat_w=16)
    cfg["sched"]["steps"] = 10
    run_sample(torch, drf, orc, cfg, TOL_BF16, mode=mode, n=3, batch=2)


def test_sample_bf16_guidance_head72(torch, drf, orc):
    # DiT-XL head width (72) and guidance, narrow and shallow
    cfg = I.config(3, depth=2, hidden=576, heads=8, lat_h=8, lat_w=8)
    cfg["sched"]["steps"] = 9
    run_sample(torch, drf, orc, cfg, TOL_BF16, n=4, batch=2)
    run_sample(torch, drf, orc, cfg, TOL_BF16, mode=I.AGGRESSIVE, n=4, batch=2, init="loud", seed=3)


def test_sample_config3_full_depth_against_the_stored_oracle_sample(torch, drf):
    """Configuration 3 exactly as benchmarked except for the batch (1 instead of 8: samples are
    independent): 28 blocks, 50-step DDIM, conservative n = 4, guidance 4.  The expected x_0 was written by
    tests/golden/make_cfg3_sample.py, which calls the CPU oracle only (about half an hour on 8 cores, so
    it is stored instead of recomputed)."""
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "cfg3_batch1_x0.txt")
    cfg = I.config(3)
    dit, sd = cfg["dit"], cfg["sched"]
    want = np.loadtxt(path).reshape(1, dit["in_ch"], dit["lat_h"], dit["lat_w"])
    w = I.weights(dit, 3)
    xT, cond, null = I.latent_noise(dit, 1, 3), I.conditioning(dit, 1, 3), I.conditioning(dit, 1, 3, null=True)
    den = drf.Denoiser(dit, w)
    got = den.sample(sd, cfg["mode"], cfg["n"], dev(torch, xT), dev(torch, cond), dev(torch, null), cfg["guidance"]).cpu().numpy()
    den.close()
    check(got, want, TOL_BF16, "cfg3 batch 1 x_0")


def test_sample_bf16_text_guidance(torch, drf, orc):
    cfg = I.config(4, depth=2, hidden=192, heads=3, lat_h=8, lat_w=8, cond_dim=64, ctx_len=9)
    cfg["sched"]["steps"] = 7
    run_sample(torch, drf, orc, cfg, TOL_BF16, batch=2, init="loud", seed=4)


def test_sample_equals_manual_loop_over_the_plan(torch, drf, orc):
    """The fused loop against its parts: replay the oracle's plan table with separate
    eps_batched / skip_transition / refine_step calls.  Holds at any size."""
    cfg = I.config(2, depth=2, lat_h=16, lat_w=16)
    cfg["sched"]["steps"] = 11
    dit, sd = cfg["dit"], cfg["sched"]
    B = 2
    w = I.weights(dit, 5)
    den = drf.Denoiser(dit, w)
    xT = dev(torch, I.latent_noise(dit, B, 5))
    cond = dev(torch, I.conditioning(dit, B, 5))
    for mode in (I.CONSERVATIVE, I.AGGRESSIVE):
        got = den.sample(sd, mode, 3, xT, cond)
        rows = orc.plan(sd, mode, 3)
        X, NA, ND = {sd["steps"]: xT}, {}, {}       # refined states, anchor noises, draft noises

        def eps_at(state, tau):
            return den.eps_batched(state, torch.full((B,), tau, dtype=torch.int32, device="cuda"), cond)

        for _, kind, s_from, s_to, tau in rows.tolist():
            if kind == 0:
                NA[s_from] = eps_at(X[s_from], tau)
            elif kind == 1:
                anchor_noise = NA[s_from] if s_from in NA else ND[s_from]
                d = drf.skip_transition(sd, X[s_from], anchor_noise, s_from, [s_to])[0]
                if tau >= 0:
                    ND[s_to] = eps_at(d, tau)
                if s_from - s_to == 1:
                    X[s_to] = d
            else:
                X[s_to] = drf.refine_step(sd, X[s_from], ND[s_from] if s_from in ND else NA[s_from], s_from)
        x = X[0]
        assert relerr(got.cpu().numpy(), x.cpu().numpy()) < 1e-6, mode
    den.close()


def test_sample_edge_cases(torch, drf):
    dit = small_dit(I.COND_CLASS, I.F32, depth=1)
    den = drf.Denoiser(dit, I.weights(dit, 2))
    x = torch.randn((2, 4, 10, 6), dtype=torch.float32, device="cuda")
    c = torch.tensor([1, 2], dtype=torch.int32, device="cuda")
    sd = dict(SCHED20, steps=4)
    a = den.sample(sd, I.CONSERVATIVE, 100, x, c)            # n beyond S
    b = den.sample(sd, I.CONSERVATIVE, 4, x, c)
    assert torch.equal(a, b)
    one = den.sample(dict(SCHED20, steps=1), I.AGGRESSIVE, 3, x, c)
    assert torch.isfinite(one).all()
    y = x.clone()
    den.sample(sd, I.AGGRESSIVE, 2, y, c, out=y)             # in place
    assert torch.equal(y, den.sample(sd, I.AGGRESSIVE, 2, x, c))
    for bad in (dict(n=0), dict(mode=3)):
        with pytest.raises(drf.DrfError):
            den.sample(sd, bad.get("mode", 0), bad.get("n", 2), x, c)
    empty = torch.empty((0, 4, 10, 6), dtype=torch.float32, device="cuda")
    assert den.sample(sd, 0, 2, empty, c[:0]).shape == (0, 4, 10, 6)
    den.close()


@pytest.mark.parametrize("steps,batch,guidance", [(50, 24, 3.0), (100, 2, None)])
def test_sample_with_more_conditioning_rows_than_one_chunk_or_flush(torch, drf, orc, steps, batch, guidance):
    """The modulation rows of a call are produced per chunk of passes (at most 1024 rows unless one pass has more)
    and per flush of 64 timestep groups: 50 steps x 48 slot rows = 2400 rows make three chunks, and 100 steps at
    batch 2 make one chunk of two flushes.  Tiny fp32 DiT of configuration 1, aggressive n = 3, against the oracle."""
    cfg = I.config(1)
    cfg["sched"]["steps"] = steps
    cfg["guidance"] = guidance
    run_sample(torch, drf, orc, cfg, TOL_F32, mode=I.AGGRESSIVE, n=3, batch=batch, seed=8)
