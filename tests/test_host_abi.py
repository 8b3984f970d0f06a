"""Host-side checks that need no GPU: the library loads, exports every symbol the
header declares, its plan table equals the oracle's bit for bit, and bad arguments
come back as status codes."""
import ctypes as C
import os
import re
import subprocess
import sys

import numpy as np
import pytest

from paper_2603_25872_amd import drf, inputs as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_symbols(name):
    text = open(os.path.join(ROOT, "include", name)).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(drf_[a-z_0-9]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    L = drf.lib()
    assert sorted(os.listdir(os.path.join(ROOT, "include"))) == ["drf.h", "drf_measure.h"]
    assert header_symbols("drf.h") == sorted(drf.SYMBOLS)
    assert header_symbols("drf_measure.h") == sorted(drf.MEASURE_SYMBOLS)
    for n in drf.SYMBOLS + drf.MEASURE_SYMBOLS:
        assert getattr(L, n) is not None
    # the measurement hooks stay out of the method's header
    assert not set(drf.MEASURE_SYMBOLS) & set(header_symbols("drf.h"))


def sched(S):
    return dict(train_steps=1000, beta_start=1e-4, beta_end=0.02, steps=S, eta=0.0)


@pytest.mark.parametrize("mode", [drf.CONSERVATIVE, drf.AGGRESSIVE])
@pytest.mark.parametrize("S", [1, 2, 3, 5, 20, 28, 30, 50, 1000])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 8, 9, 64, 100])
def test_plan_table_bit_exact_with_oracle(orc, mode, S, n):
    got = drf.plan_build(sched(S), mode, n)
    want = orc.plan(sched(S), mode, n)
    assert got.dtype == want.dtype == np.int32
    assert got.shape == want.shape
    assert np.array_equal(got, want)


def test_plan_for_the_five_workloads(orc):
    for idx, c in I.CONFIGS.items():
        assert np.array_equal(drf.plan_build(c["sched"], c["mode"], c["n"]), orc.plan(c["sched"], c["mode"], c["n"]))


def test_plan_capacity_is_respected():
    sc = drf.sched_config(sched(20))
    cnt = C.c_size_t(0)
    rows = np.full((3, 5), -7, np.int32)
    assert drf.lib().drf_plan_build(C.byref(sc), 0, 2, rows.ctypes.data_as(C.c_void_p), 2, C.byref(cnt)) == 0
    assert cnt.value > 3
    assert (rows[2] == -7).all() and (rows[:2] != -7).any()


@pytest.mark.parametrize("bad", [dict(steps=0), dict(steps=1001), dict(eta=1.5), dict(eta=-0.1), dict(beta_start=0.0),
                                 dict(beta_end=1.0), dict(train_steps=1), dict(sampler=3), dict(sampler=-1),
                                 dict(sampler=drf.EULER, shift=0.0)])
def test_bad_schedule_is_a_status_code(bad):
    sc = drf.sched_config(dict(sched(20), **bad))
    cnt = C.c_size_t(0)
    st = drf.lib().drf_plan_build(C.byref(sc), 0, 2, None, 0, C.byref(cnt))
    assert st == -1
    assert len(drf.lib().drf_last_error()) > 0


@pytest.mark.parametrize("mode", [drf.CONSERVATIVE, drf.AGGRESSIVE])
@pytest.mark.parametrize("S", [1, 2, 3, 7, 28, 50])
@pytest.mark.parametrize("n", [1, 2, 4, 9])
@pytest.mark.parametrize("extra", [dict(eta=1.0), dict(sampler=drf.DDPM), dict(sampler=drf.EULER),
                                   dict(sampler=drf.EULER, shift=3.0)])
def test_plan_and_draw_count_of_the_other_samplers(orc, mode, S, n, extra):
    sd = dict(sched(S), **extra)
    got = drf.plan_build(sd, mode, n)
    assert np.array_equal(got, orc.plan(sd, mode, n))
    assert drf.noise_count(sd, mode, n) == orc.noise_count(sd, mode, n) == int((got[:, 1] != 0).sum())


def test_euler_plan_feeds_sigma_scaled_times(orc):
    sd = dict(sched(28), sampler=drf.EULER, shift=3.0)
    rows = drf.plan_build(sd, drf.CONSERVATIVE, 4)
    evald = rows[rows[:, 4] >= 0]
    for r in evald:
        u = r[3] / 28
        assert r[4] == int(np.floor(3 * u / (1 + 2 * u) * 1000 + 0.5))
    assert evald[0, 4] == 1000


def test_stochastic_sampler_without_noise_source_is_rejected_before_any_launch():
    # validation happens on the host: fake (never dereferenced) device addresses are enough
    L = drf.lib()
    fake = C.c_void_p(0x1000)
    to = (C.c_int * 2)(4, 3)
    for extra in (dict(eta=0.5), dict(sampler=drf.DDPM)):
        sc = drf.sched_config(dict(sched(20), **extra))
        assert L.drf_skip_transition_noise(C.byref(sc), fake, fake, 5, to, 2, 1, 16, None, fake, None) == -1
        assert b"noise source" in L.drf_last_error()
        assert L.drf_skip_transition(C.byref(sc), fake, fake, 5, to, 2, 1, 16, fake, None) == -1
        # a transition with variance has to move towards data
        up = (C.c_int * 1)(7)
        nz = drf.Noise(None, 1, 0)
        assert L.drf_skip_transition_noise(C.byref(sc), fake, fake, 5, up, 1, 1, 16, C.byref(nz), fake, None) == -1
        assert b"towards data" in L.drf_last_error()
    cnt = C.c_size_t(0)
    sc = drf.sched_config(sched(20))
    assert L.drf_noise_count(C.byref(sc), 0, 2, None) == -1
    assert L.drf_noise_count(C.byref(sc), 0, 0, C.byref(cnt)) == -1
    assert L.drf_normal_fill(1, 0, 4, 16, None, None) == -1
    assert L.drf_normal_fill(1, 0, 0, 16, None, None) == 0
    assert L.drf_normal_fill(1, 0xffffffff, 2, 16, fake, None) == -1


def test_bad_plan_arguments():
    sc = drf.sched_config(sched(20))
    cnt = C.c_size_t(0)
    L = drf.lib()
    assert L.drf_plan_build(C.byref(sc), 0, 0, None, 0, C.byref(cnt)) == -1
    assert L.drf_plan_build(C.byref(sc), 5, 2, None, 0, C.byref(cnt)) == -1
    assert L.drf_plan_build(None, 0, 2, None, 0, C.byref(cnt)) == -1
    assert L.drf_plan_build(C.byref(sc), 0, 2, None, 0, None) == -1


def test_weight_count_matches_layout_and_oracle(orc):
    for idx, c in I.CONFIGS.items():
        n = drf.denoiser_weight_count(c["dit"])
        assert n == I.param_count(c["dit"]) == orc.weight_count(c["dit"])
    assert drf.denoiser_weight_count(dict(I.CONFIGS[1]["dit"], hidden=130)) == 0       # not divisible by heads
    assert drf.denoiser_weight_count(dict(I.CONFIGS[2]["dit"], hidden=390)) == 0       # bf16 needs % 64


def test_null_handles_are_rejected_without_touching_the_gpu():
    L = drf.lib()
    assert L.drf_eps_batched(None, None, None, None, 1, None, None) == -1
    assert L.drf_sample(None, None, 0, 1, 1, None, None, None, C.c_float(0), None, None) == -1
    assert L.drf_denoiser_reserve(None, 4) == -1
    L.drf_denoiser_destroy(None)
    sc = drf.sched_config(sched(20))
    to = (C.c_int * 1)(3)
    # zero-sized work is a no-op, NULL buffers with real sizes are an error
    assert L.drf_skip_transition(C.byref(sc), None, None, 5, to, 1, 0, 16, None, None) == 0
    assert L.drf_skip_transition(C.byref(sc), None, None, 5, to, 1, 2, 16, None, None) == -1
    assert L.drf_refine_step(C.byref(sc), None, None, 0, 1, 16, None, None) == -1
    # the entry point that allocates nothing, the graph switch and the measurement hooks
    assert L.drf_eps_batched_static(None, None, None, None, 1, None, None) == -1
    assert L.drf_denoiser_use_graphs(None, 1) == -1
    a, b, c = C.c_int(0), C.c_int(0), C.c_longlong(0)
    assert L.drf_graph_stats(None, C.byref(a), C.byref(b), C.byref(c)) == -1
    assert L.drf_profile_enable(None, 1) == -1
    v = C.c_double(0)
    assert L.drf_calibrate_mfma_bf16(1, 0, C.byref(v), None) == -1           # iters < 1
    assert L.drf_calibrate_copy(None, None, 1024, 1, C.byref(v), None) == -1
    # the fused-update probe validates its counts and indices on the host before any launch
    assert L.drf_probe_update_fused(C.byref(sc), 20, 4, 4, 3, C.c_float(1), 16, None, None, None, None, None) == -1   # g not 1 | 2
    assert L.drf_probe_update_fused(C.byref(sc), 5, 4, 4, 2, C.c_float(1), 16, None, None, None, None, None) == -1    # runs past index 0
    assert L.drf_probe_update_fused(C.byref(sc), 20, 4, 4, 2, C.c_float(1), 0, None, None, None, None, None) == 0     # empty field: no-op
    assert L.drf_probe_update_fused(C.byref(sc), 20, 4, 4, 2, C.c_float(1), 16, None, None, None, None, None) == -1   # NULL buffers
    assert len(L.drf_last_error()) > 0


def test_bench_refuses_more_than_one_gpu():
    # the contract: bench.py --gpus N with N > 1 exits with a message that says so (no GPU is touched)
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode != 0
    assert "one GPU" in (r.stderr + r.stdout)


@pytest.mark.parametrize("d", range(8, 97, 8))
@pytest.mark.parametrize("scaled", [0, 1])
def test_long_attention_goes_to_the_kernel_that_measured_faster(d, scaled):
    """More than 256 kv rows.  One workgroup of 256 queries to a CU (here 4 and 256 of them): 64 queries per wave lose at widths
    16, 32 and 64 (0.76-0.95x of the chunked kernel, queries scaled or not) and never beyond 80; many workgroups: they win at every
    width up to 80."""
    few, full, many = (drf.probe_attn_route(s, 1024, 1024, h, d, scaled) for s, h in ((1, 1), (8, 8), (64, 8)))
    assert many == (7 if d <= 80 else 5)
    if d in (16, 32, 64, 88, 96):
        assert (few, full) == (5, 5)
    elif scaled or d in (56, 72):
        assert (few, full) == (7, 7)


@pytest.mark.parametrize("d", range(8, 97, 8))
def test_long_attention_of_a_few_rows_more_than_256(d):
    """Up to 352 rows the chunked kernel fills its third chunk of 128 in part and keeps fewer widths."""
    few, many = drf.probe_attn_route(2, 300, 300, 4, d, 0), drf.probe_attn_route(64, 300, 300, 8, d, 0)
    assert few == (5 if d in (16, 32, 64, 88, 96) else 7) and many == (7 if d <= 88 else 5)


def test_attention_routes_by_rows():
    route = drf.probe_attn_route
    for d in range(8, 97, 8):
        assert route(2, 64, 64, 4, d) == 1 and route(300, 40, 40, 16, d) == 2         # up to 128 queries: 32 at a time, 64 of many
        assert route(2, 256, 256, 4, d) == 1                                            # fits the chip at once
        assert route(32, 256, 256, 8, d) == 3 and route(64, 256, 256, 8, d) == 4
        assert route(2, 128, 257, 4, d) == 6 and route(2, 128, 256, 4, d) == 1
        assert route(3, 129, 257, 4, d) in (5, 7)
    assert route(0, 64, 64, 4, 64) == route(1, 64, 64, 4, 12) == route(1, 64, 64, 4, 104) == 0


@pytest.mark.parametrize("d", range(8, 97, 8))
def test_wide_heads_share_kv_between_two_query_blocks_from_the_second_round_on(d):
    """Up to 256 rows and 97 to 128 queries at widths 88 and 96: with 32 queries per workgroup a launch that does not fit the chip at once is
    slower than with 64 (18.9 against 15.9 us) and than one chunk per head was (17.1 us)."""
    route = drf.probe_attn_route
    assert route(64, 128, 256, 4, d) == route(16, 128, 200, 16, d) == (2 if d > 80 else 1)
    assert route(64, 96, 256, 4, d) == 1 and route(8, 128, 256, 4, d) == 1


@pytest.mark.parametrize("d", [8, 40, 72, 80, 88])
def test_many_queries_over_short_kv_stay_within_a_grid(d):
    """One workgroup of 256 threads to 256 queries of a head, up to 2^32 threads a launch; persistent workgroups beyond."""
    route = drf.probe_attn_route
    assert route(2 ** 18 - 1, 1024, 77, 16, d) == 7 and route(2 ** 18, 1024, 77, 16, d) == route(2 ** 20, 1024, 256, 16, d) == 4


def test_gemm_routes_are_readable():
    """Small problems split K where they may, a part-filled last round goes to a second launch, bad arguments are refused."""
    tile, parts, first_tile, first_rows = drf.probe_gemm_route(512, 1152, 4608, 2)
    assert parts > 1 and (first_tile, first_rows) == (0, 0)
    assert drf.probe_gemm_route(512, 1152, 4608, 0)[1] == 1
    for args in ((0, 64, 64, 0), (64, 64, 72, 0), (64, 64, 64, 5), (64, 64, 64, 1, 0)):
        with pytest.raises(drf.DrfError):
            drf.probe_gemm_route(*args)


@pytest.mark.parametrize("tile,eight,cols", [(2, 20, 288), (3, 19, 256)])
def test_gemm_256_row_tiles_take_the_form_that_measured_faster(tile, eight, cols):
    """One and two rounds of 256 x 288 or 256 x 256 tiles: eight waves where GELU or the head-major store weighs more than the
    loop, four elsewhere (times inside a pass beside the rule)."""
    for rounds in (1, 2):
        def route(K, kind, rows_per_slot=256):
            return drf.probe_gemm_route(16384, 4 * rounds * cols, K, kind, rows_per_slot)[0]
        for K in (384, 512, 768, 1152, 1536, 2048, 4608):
            assert route(K, 3) == (eight if K < (1024 if rounds == 1 else 1536) else tile)
            assert route(K, 1) == (eight if K < 512 else tile)
            assert route(K, 1, 252) == (eight if K < (1024 if rounds == 1 and tile == 3 else 1536) else tile)
            assert route(K, 2) == route(K, 4) == route(K, 0) == tile


@pytest.mark.parametrize("K,tile", [(384, 18), (768, 18), (1152, 18), (2048, 13), (4608, 13)])
def test_gemm_one_round_of_256_x_144_tiles(K, tile):
    """Eight waves for short K, two pairs of waves for long K (times inside a pass beside the tile table)."""
    assert drf.probe_gemm_route(8192, 1152, K, 2) == (tile, 1, 0, 0)


@pytest.mark.parametrize("M,N,K", [(2560, 1152, 4608), (2470, 1152, 1152), (8192, 384, 1536), (7904, 384, 1536)])
def test_gemm_one_round_of_128_x_96_tiles(M, N, K):
    """193 to 256 of them, where 128 x 128 tiles leave CUs idle and smaller ones need a second round."""
    assert drf.probe_gemm_route(M, N, K, 2) == (7, 1, 0, 0)
    assert drf.probe_gemm_route(4096, 1536, 6144, 2)[0] != 7       # two rounds: 84 us, one of 256 x 128 75
    assert drf.probe_gemm_route(8192, 384, 384, 2)[0] != 7         # a short launch: 0.6 us, which the next kernels' code loads cost


@pytest.mark.parametrize("M,N,K,kind,rows_per_slot,tile", [
    (3072, 3456, 1152, 1, 256, 21), (3276, 3456, 1152, 1, 252, 21), (10240, 1152, 4608, 2, 256, 21),
    (24576, 1152, 4608, 2, 4096, 22), (24576, 1152, 1152, 4, 4096, 22), (12288, 3456, 1152, 1, 256, 22)])
def test_gemm_tiles_for_part_filled_rounds(M, N, K, kind, rows_per_slot, tile):
    """One round of 256 x 192, one to three of 192 x 288 where other tiles leave a round part-filled; neither for GELU or as one of two
    launches, the latter not where head-major rows cross slots (times inside a pass beside the tile table)."""
    assert drf.probe_gemm_route(M, N, K, kind, rows_per_slot) == (tile, 1, 0, 0)
    for rows in range(2048, 65536, 512):
        tile, _, first_tile, _ = drf.probe_gemm_route(rows, N, K, kind, rows_per_slot)
        assert first_tile not in (21, 22)
        if tile == 21:
            assert -(-rows // 256) * -(-N // 192) <= 256
        if tile == 22:
            assert -(-rows // 192) * -(-N // 288) <= 768 and not (kind == 1 and rows_per_slot % 32)
        assert not {21, 22} & set(drf.probe_gemm_route(rows, N, K, 3)[::2])


@pytest.mark.parametrize("M,N,K,tile", [(2816, 4608, 1152, 3), (3072, 4608, 1152, 19), (3276, 4608, 1152, 19), (3584, 4608, 1152, 19),
                                        (3328, 4096, 1024, 3), (3584, 4096, 1024, 19), (4096, 4096, 1024, 3)])
def test_gemm_gelu_in_a_round_that_is_nearly_full_takes_eight_waves(M, N, K, tile):
    """216 to 255 tiles of 256 x 256; fewer, and a full round, stay on four (times beside the rule)."""
    assert drf.probe_gemm_route(M, N, K, 3) == (tile, 1, 0, 0)


def test_cross_attention_of_many_queries_takes_the_kernel_for_long_sequences():
    """More than 256 queries over at most 256 rows, from the second workgroup of a CU on (at widths 72 and 80 the first)."""
    for d in range(8, 97, 8):
        for Nk in (77, 128, 256):
            route = [drf.probe_attn_route(slots, Nq, Nk, 16, d) for slots, Nq in ((4, 1024), (8, 1024), (5, 1025), (2, 1024), (32, 256))]
            assert (route[0] == 7) == (d in (72, 80)) and 7 not in route[3:]
            assert [r == 7 for r in route[1:3]] == [d <= 88] * 2


def test_block_routes_stay_inside_their_buffers():
    """Keys and values in whole groups of 32 fit the buffers of q | k | v and of the hidden units, the shares of a dealt block the split
    GEMMs' partial tiles (2^22 floats), the launches of a dealt block the chip; widths, head widths and ratios without the form have none."""
    for D, heads in ((256, 4), (384, 6), (512, 8), (384, 12), (512, 16), (256, 8)):
        for ratio in (1, 2, 3, 4):
            for tokens in (1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 247, 256, 257, 1000, 4096):
                for slots in (1, 2, 3, 5, 8, 16, 17, 64, 300):
                    r = drf.probe_block_route(slots, tokens, D, heads, ratio)
                    parts, attention, rows = max(r // 10000, 1), r // 1000 % 10, r % 1000
                    assert rows in (0, 16, 32, 64) and parts <= ratio and (rows or r == 0) and (rows < 64 or D < 512)
                    if attention:
                        assert D // heads == 64 and rows <= 32 and 2 * ((tokens + 31) // 32 * 32) <= min(ratio, 3) * tokens
                    if parts > 1:
                        assert attention and rows == 16 and slots * ((tokens + 15) // 16) * parts <= 256 and parts * slots * tokens * D <= 1 << 22
    for D, heads, ratio in ((128, 4, 4), (1152, 16, 4), (768, 12, 4), (384, 6, 5), (384, 5, 4)):
        assert drf.probe_block_route(12, 256, D, heads, ratio) == 0


@pytest.mark.parametrize("slots,tokens", [(17, 32), (10, 64), (6, 128), (4, 256)])
def test_block_route_of_three_pieces_of_hidden_units(slots, tokens):
    """Three pieces do not deal evenly over two workgroups: at hidden 512 and few rows the launches one by one are the faster form; two
    and four pieces, longer sequences and hidden 384 keep the dealt one."""
    assert drf.probe_block_route(slots, tokens, 512, 8, 3) == 0
    assert drf.probe_block_route(slots, tokens, 512, 8, 2) == 21016 and drf.probe_block_route(slots, tokens, 512, 8, 4) == 41016
    for slots, tokens, hidden in ((2, 400, 512), (5, 247, 512), (2, 256, 384)):
        assert drf.probe_block_route(slots, tokens, hidden, hidden // 64, 3) == 21016


def test_bf16_gemm_refuses_the_fp32_paths_activation():
    """SiLU is an epilogue of the fp32 GEMM only: the bf16 launch must say so (checked on the host, before anything else is looked
    at) instead of storing without it."""
    launch = drf.lib()._ZN3drf16launch_gemm_bf16EPKDF16bS1_iiiRKNS_8EpilogueEP12ihipStream_tiPfPNS_10PartialSumE
    launch.argtypes = [C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_void_p, C.c_void_p, C.c_int, C.c_void_p, C.c_void_p]
    epilogue = (C.c_int * 128)(5)                # Epilogue starts with its mode: EPI_STORE_SILU
    assert launch(None, None, 64, 64, 64, epilogue, None, 0, None, None) == -2
    assert b"SiLU" in drf.lib().drf_last_error()


class DeviceTensor:
    """What the skip calls ask of a tensor, without a device."""
    is_cuda = True

    def __init__(self, shape, dtype, contiguous=True):
        self.shape, self.dtype, self.contiguous = shape, dtype, contiguous

    def is_contiguous(self):
        return self.contiguous

    def data_ptr(self):
        return 4096


def test_skip_calls_take_and_refuse_what_their_arguments_say():
    """The native marshalling: mappings and sequences of every kind, defaults of absent options, the errors of bad values; nothing is
    launched, as the batch is empty or the indices are refused."""
    torch = pytest.importorskip("torch")
    import collections
    drf.lib()
    sched = dict(train_steps=1000, beta_start=1e-4, beta_end=0.02, steps=50)
    none, one = DeviceTensor((0, 8), torch.float32), DeviceTensor((1, 8), torch.float32)
    skip = lambda sc, x, to, s_from=50, net=one, out=one: drf._skip(sc, x, net, s_from, to, None, out, torch.float32, 0)
    for sc in (sched, dict(sched, eta=0.5, sampler=2, shift=3), dict(sched, eta="0.25"), collections.UserDict(sched)):
        for to in ([1, 2], (3,), range(40), np.arange(3)):
            assert skip(sc, none, to) == 0
    assert skip(dict(sched, steps=0), none, [1]) != 0 and skip(dict(sched, sampler=9), none, [1]) != 0
    assert skip(dict(sched, eta=1.5), none, [1]) != 0
    assert skip(sched, one, [51]) != 0 and skip(sched, one, [1], s_from=51) != 0 and skip(sched, one, [1], net=None) != 0
    for error, call in ((KeyError, lambda: skip(dict(train_steps=1000), none, [1])), (TypeError, lambda: skip(dict(sched, steps=5.0), none, [1])),
                        (TypeError, lambda: skip(sched, none, [1.0])), (TypeError, lambda: skip(sched, none, 3)), (TypeError, lambda: skip(sched, none, [1], s_from=1.5)),
                        (AssertionError, lambda: skip(sched, torch.zeros(1, 8), [1])), (AssertionError, lambda: skip(sched, DeviceTensor((1, 8), torch.float32, False), [1])),
                        (AssertionError, lambda: skip(sched, one, [1], net=DeviceTensor((1, 8), torch.float16))), (ValueError, lambda: skip(dict(sched, eta="x"), none, [1]))):
        with pytest.raises(error):
            call()


def test_skip_calls_keep_target_indices_of_their_own(monkeypatch):
    """An index is whatever has __index__, which may change the caller's list: the call goes on with the list as it was."""
    torch = pytest.importorskip("torch")
    drf.lib()
    sched = dict(train_steps=1000, beta_start=1e-4, beta_end=0.02, steps=50)
    none = DeviceTensor((0, 8), torch.float32)

    class Index:
        def __init__(self, act):
            self.act = act

        def __index__(self):
            self.act()
            return 1

    for act in (list.clear, lambda to: to.extend([2] * 100000), lambda to: to.__setitem__(slice(1, None), ["no index"])):
        to = []
        to += [Index(lambda: act(to)), *(Index(lambda: None) for _ in range(40))]
        assert drf._skip(sched, none, none, 50, to, None, none, torch.float32, 0) == 0
        assert drf._targets(to) == tuple(to)

    class Longer(list):                              # says 1, holds 2: the second would be written past an output for one
        def __len__(self):
            return 1

    with pytest.raises(IndexError):
        drf._targets(Longer([1, 2]))
    with pytest.raises(IndexError):
        drf._skip(sched, none, none, 50, Longer([1, 2]), None, none, torch.float32, 0)
    with pytest.raises(TypeError):
        drf._targets(i for i in (1, 2))
    # what sizes the output is what is launched, whatever becomes of the list
    for call in (drf.skip_transition, drf.skip_transition_noise):
        to, handed = [1, 2], []
        monkeypatch.setattr(drf, "_stream", lambda: to.append(3))
        monkeypatch.setattr(drf, "_skip", lambda *a: a[8]() or handed.append(a[4]) or 0)
        out = call(sched, torch.zeros(1, 8), torch.zeros(1, 8), 50, to)
        assert out.shape == (2, 1, 8) and handed == [(1, 2)]


def test_skip_calls_read_a_schedules_options_as_the_other_calls_do():
    """An option that is there and None is refused, in a dict, a class of it and another mapping; absent ones have their defaults."""
    torch = pytest.importorskip("torch")
    import collections
    drf.lib()
    sched = dict(train_steps=1000, beta_start=1e-4, beta_end=0.02, steps=50)
    none = DeviceTensor((0, 8), torch.float32)
    for kind in (dict, collections.UserDict, collections.OrderedDict, collections.ChainMap):
        assert drf._skip(kind(sched), none, none, 50, [1], None, none, torch.float32, 0) == 0
        for option in ("eta", "sampler", "shift"):
            for read in (drf.sched_config, lambda sc: drf._skip(sc, none, none, 50, [1], None, none, torch.float32, 0)):
                with pytest.raises(TypeError):
                    read(kind(dict(sched, **{option: None})))


def test_skip_calls_refuse_host_tensors_before_they_ask_for_a_stream(monkeypatch):
    torch = pytest.importorskip("torch")
    sched = dict(train_steps=1000, beta_start=1e-4, beta_end=0.02, steps=50)
    asked = []
    monkeypatch.setattr(drf, "_stream", lambda: asked.append(1) or 0)
    host = torch.zeros(1, 8)
    for call in (drf.skip_transition, drf.skip_transition_noise):
        with pytest.raises(AssertionError, match="contiguous device tensor"):
            call(sched, host, host, 50, [1])
        with pytest.raises(KeyError):
            call({}, host, host, 50, [1])
        assert not asked
        none = DeviceTensor((0, 8), torch.float32)
        assert call(sched, none, none, 50, [1], out=none) is none and asked.pop()


def test_library_loads_without_the_binding_module():
    """Another interpreter than the build's has no such module: every call is there all the same, the skip calls through ctypes."""
    code = ("import sys; sys.modules['paper_2603_25872_amd._native'] = None\n"
            "from paper_2603_25872_amd import drf\n"
            "sched = dict(train_steps=1000, beta_start=1e-4, beta_end=0.02, steps=50)\n"
            "assert len(drf.plan_build(sched, drf.CONSERVATIVE, 4)) and drf._skip is drf._skip_ctypes\n")
    subprocess.run([sys.executable, "-c", code], check=True, cwd=ROOT, timeout=120)


def test_both_marshallings_of_the_skip_calls_agree():
    """The same calls through the CPython module and through ctypes: status, message and type of error, over schedules, shapes, indices and
    tensors that are taken and refused (nothing is launched: the batch is empty, or the call is refused)."""
    torch = pytest.importorskip("torch")
    import collections
    drf.lib()
    assert drf._skip is not drf._skip_ctypes         # built beside the library here
    sched = dict(train_steps=1000, beta_start=1e-4, beta_end=0.02, steps=50)
    tensor = lambda *shape, dtype=torch.float32, **kw: DeviceTensor(shape, dtype, **kw)
    none, one = tensor(0, 8), tensor(1, 8)

    def outcome(form, *args):
        try:
            status = form(*args)
            return status, drf.lib().drf_last_error() if status else None
        except Exception as e:
            return TypeError if isinstance(e, C.ArgumentError) else type(e)      # (how ctypes reports one of its arguments)

    def same(sc=sched, x=none, net=one, s_from=50, to=(1, 2), noise=None, out=one, stream=0):
        a, b = (outcome(form, sc, x, net, s_from, to, noise, out, torch.float32, stream) for form in (drf._skip, drf._skip_ctypes))
        assert a == b, (sc, x.shape, to, a, b)
        return a

    values = (0, 1, 3, -1, 50, 51, 2 ** 31, 2 ** 40, -2 ** 70, True, 1.0, "1", "x", None, np.int64(4), np.float64(0.5), torch.tensor(2), float("nan"))
    for v in values:
        for field in ("train_steps", "beta_start", "beta_end", "steps", "eta", "sampler", "shift"):
            for kind in (dict, collections.UserDict):
                same(kind(dict(sched, **{field: v})))
        same(x=one, to=[v], net=None)
        same(x=one, to=[v, v], out=None)
        same(x=one, s_from=v, out=None)
    for field in sched:
        assert same({k: sched[k] for k in sched if k != field}) is KeyError
    for to in ([], (), range(3), {1, 2}, {1: 0}, np.arange(3), torch.arange(3), list(range(40)), 3, None, "12", iter([1])):
        same(to=to)
    for shape in ((), (0,), (3,), (0, 0), (2, 0), (1, 0, 4), (5, 2, 3, 4)):
        same(x=tensor(*shape), net=None)
    for bad in (tensor(1, 8, contiguous=False), tensor(1, 8, dtype=torch.float16), torch.zeros(1, 8), 3, None):
        same(net=bad), same(out=bad)
        if hasattr(bad, "shape"):
            same(x=bad)
    same(stream=lambda: 0)
