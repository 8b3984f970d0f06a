"""Every bf16 attention kernel at sizes that its route takes, against softmax(q k^T) v in float64.  Each case names the kernel
that it is there for and fails if the launch would go to another one."""
import numpy as np
import pytest

from paper_2603_25872_amd import drf as D_

pytestmark = pytest.mark.gpu
WIDTHS = list(range(8, 97, 8))


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


@pytest.fixture(scope="module")
def drf():
    D_.lib()
    return D_


def reference(q, kv, slot, kv_slots, Nq, Nk, H, d, scaled):
    """Rows of one slot in float64; scaled queries make scores exponents of two."""
    qs = q[slot * Nq:(slot + 1) * Nq].astype(np.float64).reshape(Nq, H, d)
    k, v = np.split(kv[(slot % kv_slots) * Nk:(slot % kv_slots + 1) * Nk].astype(np.float64), 2, axis=1)
    out = np.empty((Nq, H, d))
    for h in range(H):
        s = qs[:, h] @ k[:, h * d:(h + 1) * d].T * (np.log(2.0) if scaled else d ** -0.5)
        p = np.exp(s - s.max(axis=1, keepdims=True))
        out[:, h] = p @ v[:, h * d:(h + 1) * d] / p.sum(axis=1, keepdims=True)
    return out.reshape(Nq, H * d)


def run(torch, drf, route, q, kv, slots, kv_slots, Nq, Nk, H, d, scaled, tol, look=None):
    """q [slots*Nq][H*d], kv [kv_slots*Nk][2*H*d] as float arrays; compares the slots in `look` (default: first and last)."""
    assert drf.probe_attn_route(slots, Nq, Nk, H, d, scaled) == route
    if scaled:
        q = q * (np.log2(np.e) / d ** 0.5)
    q, kv = (torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(torch.bfloat16) for a in (q, kv))
    out = drf.probe_cross_attn_bf16(q.cuda(), kv.cuda(), slots, kv_slots, Nq, Nk, H, d, q_scaled=scaled).float().cpu().numpy()
    qn, kvn = q.float().numpy(), kv.float().numpy()
    for s in look or (0, slots - 1):
        want, got = reference(qn, kvn, s, kv_slots, Nq, Nk, H, d, scaled), out[s * Nq:(s + 1) * Nq]
        err = np.abs(got - want).max() / np.abs(want).max()
        assert np.isfinite(got).all() and err < tol, (s, err)


def normal(rng, slots, kv_slots, Nq, Nk, H, d, scale=1.5):
    return tuple(rng.standard_normal(shape, np.float32) * np.float32(scale) for shape in ((slots * Nq, H * d), (kv_slots * Nk, 2 * H * d)))


def growing(rng, slots, kv_slots, Nq, Nk, H, d):
    """Scores of tens of exponents of two that grow along kv: the reference of the online softmax moves again and again."""
    q, kv = normal(rng, slots, kv_slots, Nq, Nk, H, d, 1)
    kv[:, :H * d] *= np.tile(np.linspace(0.2, 6, Nk, dtype=np.float32), kv_slots)[:, None]
    return 4 * q, kv


# tolerances: P and the result rounded to bf16, 2^-8 relative each at worst (about 0.8 % together), as for the other shapes


@pytest.mark.parametrize("scaled", [False, True])
@pytest.mark.parametrize("d,Nq,Nk", [(d, *n) for d in WIDTHS for n in ((257, 257), (320, 320), (545, 545), (129, 300), (300, 1030))
                                     if d <= 80 or d == 88 and n[1] <= 352])
def test_64_queries_per_wave(torch, drf, d, scaled, Nq, Nk):
    """Both forms of the queries at every width: last steps of 1 and 32 rows, last chunks of one and a few rows, query blocks in
    which waves have no query, kv shared between slots."""
    H = 8
    slots = 130 if d in (16, 32) and not scaled else 34
    args = (slots, 17, Nq, Nk, H, d)
    run(torch, drf, 7, *normal(np.random.default_rng(d + Nq + Nk), *args), *args, scaled, 1.5e-2, look=(0, 18, slots - 1))


@pytest.mark.parametrize("scaled", [False, True])
@pytest.mark.parametrize("d", [w for w in WIDTHS if w <= 80])
def test_64_queries_per_wave_moving_reference(torch, drf, d, scaled):
    """Spare score columns (odd d / 8), the 16-row tail (d = 8, 40, 72) and neither of them, under a reference that keeps moving."""
    slots, H = 130 if d in (16, 32) and not scaled else 34, 8
    args = (slots, 5, 300, 512, H, d)
    run(torch, drf, 7, *growing(np.random.default_rng(d), *args), *args, scaled, 2e-2)


@pytest.mark.parametrize("d", WIDTHS)
@pytest.mark.parametrize("Nq,Nk", [(129, 257), (300, 385), (256, 513)])
def test_chunks_of_128_rows(torch, drf, d, Nq, Nk):
    """More than 256 kv rows and few workgroups: the 8-wave chunked kernel at every width that comes to it."""
    args, route = (3, 2, Nq, Nk, 2, d), 7 if d in (56, 72) or Nk <= 352 and d in (8, 24, 40, 48, 80) else 5
    run(torch, drf, route, *normal(np.random.default_rng(d), *args), *args, False, 1.5e-2)
    run(torch, drf, route, *growing(np.random.default_rng(d), *args), *args, False, 2e-2)


@pytest.mark.parametrize("d", WIDTHS)
@pytest.mark.parametrize("Nq,Nk", [(1, 257), (16, 300), (128, 384), (100, 640)])
def test_few_queries_over_long_kv(torch, drf, d, Nq, Nk):
    """Cross-attention of a small latent with a long context: 128 queries per workgroup, kv shared between slots."""
    args = (5, 2, Nq, Nk, 3, d)
    run(torch, drf, 6, *normal(np.random.default_rng(d + Nq), *args), *args, False, 1.5e-2, look=(0, 3, 4))
    run(torch, drf, 6, *growing(np.random.default_rng(d + Nq), *args), *args, False, 2e-2)


@pytest.mark.parametrize("d", WIDTHS)
@pytest.mark.parametrize("slots,T,route", [(33, 200, 3), (17, 256, 3), (34, 193, 4), (70, 130, 4)])
def test_chunks_of_64_rows(torch, drf, d, slots, T, route):
    """130 to 256 rows, more than the one-wave-per-64-rows kernel holds at once: plain and persistent workgroups."""
    args = (slots, 9, T, T, 12 if route == 4 else 7, d)
    run(torch, drf, route, *normal(np.random.default_rng(d + T), *args), *args, False, 1.5e-2)
    run(torch, drf, route, *growing(np.random.default_rng(d + T), *args), *args, False, 2e-2)


@pytest.mark.parametrize("d,slots,Nq,Nk,H,route", [(96, 17, 1024, 77, 4, 4), (96, 33, 300, 200, 8, 4), (96, 32, 513, 256, 3, 4)] +
                         [(d, 15, 513, 256, 5, 3) for d in WIDTHS] + [(d, 8, 1000, 200, 7, 3) for d in (32, 64, 72, 88, 96)])
def test_chunks_of_64_rows_with_several_query_blocks_a_head(torch, drf, d, slots, Nq, Nk, H, route):
    """Cross-attention of more than 256 queries over at most 256 rows: persistent workgroups (width 96 only) and plain ones, two to four query
    blocks to a head, the last of them of 1 to 256 queries, kv shared between slots."""
    args = (slots, 5, Nq, Nk, H, d)
    run(torch, drf, route, *normal(np.random.default_rng(d + Nk), *args), *args, False, 1.5e-2, look=(0, 7, slots - 1))
    run(torch, drf, route, *growing(np.random.default_rng(d + Nk), *args), *args, False, 2e-2)


@pytest.mark.parametrize("d", WIDTHS)
@pytest.mark.parametrize("Nq,Nk", [(97, 97), (128, 128), (33, 192), (128, 193), (65, 256)])
def test_64_queries_per_workgroup_of_several_waves(torch, drf, d, Nq, Nk):
    """Two to four waves of 64 kv rows: the second query block's maxima and partial sums, ragged blocks and last waves."""
    H = 8
    slots = 4096 // (H * -(-Nq // 32)) + 3
    args = (slots, 7, Nq, Nk, H, d)
    run(torch, drf, 2, *normal(np.random.default_rng(d + Nk), *args), *args, False, 1.5e-2, look=(0, 1, slots - 1))
    run(torch, drf, 2, *growing(np.random.default_rng(d + Nk), *args), *args, False, 2e-2)


@pytest.mark.parametrize("d", WIDTHS)
@pytest.mark.parametrize("Nq,Nk", [(5, 70), (32, 129), (100, 256), (200, 193)])
def test_one_wave_per_64_rows_over_shared_kv(torch, drf, d, Nq, Nk):
    args = (5, 2, Nq, Nk, 3, d)
    run(torch, drf, 1, *normal(np.random.default_rng(d + Nq), *args), *args, False, 1.5e-2, look=(0, 3, 4))
    run(torch, drf, 1, *growing(np.random.default_rng(d + Nq), *args), *args, False, 2e-2)


def overflowing(rng, slots, kv_slots, Nq, Nk, H, d, rows):
    """Finite queries and keys whose products with the keys of `rows` are below the range of fp32 (scores of -inf); the other
    scores are of order one."""
    q, kv = normal(rng, slots, kv_slots, Nq, Nk, H, d, 1)
    q = np.abs(q) * 1e19 + 1e19
    kv[:, :H * d] *= 1e-19
    for s in range(kv_slots):
        kv[s * Nk + rows.start:s * Nk + rows.stop, :H * d] = -1e25
    return q, kv


@pytest.mark.parametrize("d", [16, 64, 72, 96])
@pytest.mark.parametrize("slots,Nq,Nk,rows,route", [(3, 40, 128, range(64, 128), 1), (3, 40, 200, range(0, 64), 1), (131, 256, 70, range(64, 70), 4),
                                                    (180, 96, 256, range(64, 192), 2)])
def test_scores_of_minus_infinity_in_a_whole_wave(torch, drf, d, slots, Nq, Nk, rows, route):
    """The rows of one wave have no finite score: they get no weight, and the rest of the row is what it is without them."""
    args = (slots, 2, Nq, Nk, 8, d)
    run(torch, drf, route, *overflowing(np.random.default_rng(d), *args, rows), *args, False, 1.5e-2)


@pytest.mark.parametrize("scaled", [False, True])
@pytest.mark.parametrize("d", [w for w in WIDTHS if w <= 80])
@pytest.mark.parametrize("rows", [range(0, 32), range(32, 96), range(256, 300)])
@pytest.mark.parametrize("every", [1, 2])
def test_scores_of_minus_infinity_in_a_step_of_64_queries(torch, drf, d, scaled, rows, every):
    """The same for steps of the kernel for long sequences, the first of which sets the reference: for every query, and for
    every second one while the others' scores stay finite; the scores of all other rows are far below zero."""
    args = (130 if d in (16, 32) and not scaled else 34, 2, 300, 300, 8, d)
    q, kv = overflowing(np.random.default_rng(d), *args, rows)
    for r in set(range(300)) - set(rows):
        kv[[r, 300 + r], :8 * d] -= 1.5e-17 * d ** -0.5
    if every == 2:
        q[::2] *= 1e-9
    run(torch, drf, 7, q, kv, *args, scaled, 1.5e-2)


@pytest.mark.parametrize("d", [w for w in WIDTHS if w <= 88])
@pytest.mark.parametrize("Nq,Nk", [(257, 1), (300, 31), (257, 33), (513, 77), (257, 128), (600, 129), (257, 256)])
def test_64_queries_per_wave_over_short_kv(torch, drf, d, Nq, Nk):
    """Cross-attention of many queries over at most 256 rows: one step or less, last steps of 1 and 13 rows, one and two chunks, kv shared
    between slots, the references of growing scores."""
    args = (100, 5, Nq, Nk, 8, d)
    run(torch, drf, 7, *normal(np.random.default_rng(d + Nk), *args), *args, False, 1.5e-2, look=(0, 7, 33))
    run(torch, drf, 7, *growing(np.random.default_rng(d + Nk), *args), *args, False, 2e-2)


@pytest.mark.parametrize("d", [w for w in WIDTHS if w <= 88])
@pytest.mark.parametrize("rows", [range(0, 32), range(0, 96), range(32, 120)])
def test_scores_of_minus_infinity_over_short_kv(torch, drf, d, rows):
    """One to three steps without a finite score, the first ones or the last; the other scores are far below zero, so that the reference
    has to come from the first step that has some."""
    args = (34, 2, 257, 120, 8, d)
    q, kv = overflowing(np.random.default_rng(d), *args, rows)
    for r in set(range(120)) - set(rows):
        kv[[r, 120 + r], :8 * d] -= 1.5e-17 * d ** -0.5
    run(torch, drf, 7, q, kv, *args, False, 1.5e-2)


@pytest.mark.parametrize("scaled", [False, True])
@pytest.mark.parametrize("d", [w for w in WIDTHS if w <= 80])
@pytest.mark.parametrize("far", [1e3, 1e5, 1e8, 1e20])
def test_scores_far_above_the_reference_so_far(torch, drf, d, scaled, far):
    """The first rows, as many as a step or a little more, score far below the rest, whose differences decide the result: they
    must not be rounded to the distance."""
    args = (130 if d in (16, 32) and not scaled else 34, 2, 300, 300, 8, d)
    q, kv = normal(np.random.default_rng(d), *args, 1)
    q = np.abs(q) + 1
    for s in range(2):
        kv[s * 300:s * 300 + 32, :8 * d] = -far
        kv[s * 300 + 32:s * 300 + 40, :8 * d] = -far / 2
    run(torch, drf, 7, q, kv, *args, scaled, 1.5e-2)
