// Multi-head attention softmax(q k^T / sqrt(d)) v for sequences of more than 256 kv rows, and of many queries over fewer (bf16, no mask).
#include <type_traits>

#include "common.h"

namespace drf {

namespace {

typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
#define DRF_LDS_PTR __attribute__((address_space(3)))

constexpr int kWaves = 4, kQpw = 64, kQpg = kWaves * kQpw;     // waves, queries per wave and per workgroup
constexpr int kStep = 32;                                       // kv rows per softmax step
constexpr float kTau = 8.f;                                     // lazy-rescale headroom of the online softmax, in log2 units
constexpr float kFar = 1024.f;                                  // see settle: scores closer than this to the reference keep 2^-13

__device__ inline float max3(float a, float b, float c) { return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c); }

// Shapes that follow from the head width d = 8 P8.
template <int P8> struct LongCfg {
    static constexpr int d = P8 * 8, KS = (P8 + 1) / 2;
    static constexpr bool TAIL = d % 32 == 8;                   // the last 8 rows of O^T and the denominator: one 16-row tile
    static constexpr int DT = TAIL ? d / 32 : (d + 31) / 32;    // 32-row tiles of O^T
    static constexpr bool ONES = d % 32 != 0;                   // O^T has a padding row: it accumulates the denominator
    static constexpr int KP = P8 | 1;                           // 16-byte pieces per K row in LDS
    static constexpr int VP0 = ONES ? P8 + 1 : P8, VP = VP0 == 8 ? 9 : VP0;   // and per V row
    static constexpr int PAD = 64;                              // zero bytes behind each V buffer
    static constexpr int KC = 2 * 128 * (KP + VP) * 16 + 3 * PAD <= 80 * 1024 ? 128 : 64;   // kv rows per chunk
    static constexpr int KBYTES = KC * KP * 16, VBYTES = KC * VP * 16 + PAD, BUF = KBYTES + VBYTES;
    static constexpr int LDO = DT * 32 + (TAIL ? 16 : 0) + 8;                     // row stride of a wave's output tile
    static constexpr int OUT = kWaves * 32 * LDO * 2;
    static constexpr bool PADM = P8 % 2 == 1;                   // the last k-step of the score MFMA has 8 spare columns
    static constexpr int CONST = 2 * BUF;                       // one 16-byte piece (1, 1, 1, 0, ...): K in those columns
    static constexpr int SMEM = CONST + 16 > OUT ? CONST + 16 : OUT;
    static_assert(SMEM <= 80 * 1024 && SMEM % 16 == 0, "two workgroups per CU");
    static_assert((DT * 4 + (TAIL ? 2 : 0) - VP) * 16 <= PAD, "reads past the last V row end in the pad");
};

// What bounds it: the matrix and the vector units about equally (per 32 x 64 scores of a wave 640 MFMA cycles at d = 72,
// 440 cycles of exponentials, conversions and maxima), then the power both draw together; memory is idle (a workgroup
// reads 36 KB per chunk).  Hence:
//  - A wave owns 64 queries (two blocks of 32) and uses every K and V^T fragment twice: with 32 queries per wave, as for
//    short sequences, the fragment reads alone fill the LDS port (22 KB per wave and 64 kv rows at 128 bytes per clock
//    take as long as the MFMAs).
//  - The two blocks take turns, so that independent work is always at hand: while one block's scores become P (vector
//    unit) the next scores of the other block are computed (matrix unit).  A step has no branch but the lazy rescale, so
//    the compiler interleaves the two streams instruction by instruction, and fragments are re-read right after their last
//    use, half a step before they are needed.
//  - Four waves per workgroup and two workgroups per CU (80 KB of LDS each): the barrier that hands over a chunk of 128
//    kv rows stops half of a CU's waves, and one workgroup's prologue and epilogue run beside the other's steps.
//  - K and V go to LDS as stored, by direct copies.  Rows are an odd number of 16-byte pieces (K) or a number that keeps
//    four rows of the transpose read on different banks (V).
//  - The reference score is subtracted by the score MFMA (spare columns of the head width, see settle) and the softmax
//    scale is in the queries, so an exponential has nothing before it but the MFMA; the denominator is a row of O^T.
//  - Head widths of 8 more than a multiple of 32 (72: DiT-XL) put the last 8 rows of O^T and the denominator into one
//    16-row tile (16 x 16 x 32 MFMAs) instead of a 32-row one.
// Measured inside a predictor pass, before (32 queries per wave, 8 waves, register-staged K and V) and after: 6 slots x 4096
// tokens x 16 heads of 72: 576 -> 410 us (805 -> 1133 TFLOP/s); 64 slots x 1024 tokens: 496 -> 314 us (623 -> 985 TFLOP/s).
// PRE: the queries come multiplied by log2(e) / sqrt(d), so that scores are exponents of two; otherwise by nothing and
// scores are scaled by scale_log2 here.
template <int P8, bool PRE>
__global__ void __launch_bounds__(kWaves * 64, 2) attn_long_kernel(const AttnArgs a, float scale_log2, int nqb, int n_items)
{
    using C = LongCfg<P8>;
    constexpr int d = C::d, KS = C::KS, DT = C::DT, KP = C::KP, VP = C::VP, KC = C::KC, LDO = C::LDO, NT = kWaves * 64;
    extern __shared__ __attribute__((aligned(16))) unsigned char attn_smem[];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // work item: query block fastest; consecutive items on one XCD (ids are dealt round-robin over the 8 XCDs)
    int item = blockIdx.x;
    if (nqb > 1) {
        const int q8 = n_items >> 3, rem = n_items & 7, xcd = item & 7;
        item = xcd * q8 + (xcd < rem ? xcd : rem) + (item >> 3);
    }
    const int qb = item % nqb, hs = item / nqb, h = hs % a.heads, slot = hs / a.heads;
    const int kvb = a.kv_mod ? slot % a.kv_mod : slot;
    const bf16_t* Q = (const bf16_t*)a.q + slot * a.q_slot_stride + h * a.q_head_stride;
    const bf16_t* Kp = (const bf16_t*)a.k + kvb * a.kv_batch_stride + h * a.kv_head_stride;
    const bf16_t* Vp = (const bf16_t*)a.v + kvb * a.kv_batch_stride + h * a.kv_head_stride;
    const int q0 = qb * kQpg + wave * kQpw;
    const int Nk = a.Nk, ldk = a.ldk;

    // constant parts of the LDS image: pads, and the pieces of a V row behind its d columns (1, 0, 0, ...); zeros for rows past the end of
    // a first chunk that is not full, as other threads write there too (issue)
    const bf16x8 zero8 = { 0, 0, 0, 0, 0, 0, 0, 0 };
    if (tid < 2 * (C::PAD / 16)) {
        const int buf = tid / (C::PAD / 16), p = tid % (C::PAD / 16);
        *reinterpret_cast<bf16x8*>(attn_smem + (buf + 1) * C::BUF - C::PAD + p * 16) = zero8;
    }
    if (tid == 64) {
        const bf16_t one = (bf16_t)1.f;
        const bf16x8 ones3 = { one, one, one, 0, 0, 0, 0, 0 };
        *reinterpret_cast<bf16x8*>(attn_smem + C::CONST) = ones3;
    }
    if constexpr (VP > P8) {
        for (int i = tid; i < 2 * KC * (VP - P8); i += NT) {
            const int buf = i / (KC * (VP - P8)), r = i % (KC * (VP - P8)), row = r / (VP - P8), p = r % (VP - P8);
            bf16x8 v = zero8;
            if (C::ONES && p == 0 && row < Nk) v[0] = (bf16_t)1.f;
            *reinterpret_cast<bf16x8*>(attn_smem + buf * C::BUF + C::KBYTES + (row * VP + P8 + p) * 16) = v;
        }
    }

    bf16x8 qf[2][KS];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        int q = q0 + b * 32 + l32;
        q = q < a.Nq ? q : a.Nq - 1;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int dd = ks * 16 + half * 8;
            qf[b][ks] = dd < d ? *reinterpret_cast<const bf16x8*>(Q + (size_t)q * a.ldq + dd) : zero8;
        }
    }

    // chunk copies global -> LDS, 64 pieces of 16 bytes per wave-wide instruction (lane i's piece lands at byte 16 i
    // behind the wave-uniform destination; lanes whose piece is row padding are masked off and leave it as it is)
    const uint32_t lds_base = (uint32_t)(uintptr_t)(DRF_LDS_PTR unsigned char*)attn_smem;
    auto copy_rows = [&](auto pieces_c, const bf16_t* src, int rows_left, bool clamp, uint32_t dst) {
        constexpr int PP = decltype(pieces_c)::value, NI = KC * PP / 64;
#pragma unroll
        for (int j = 0; j < (NI + kWaves - 1) / kWaves; ++j) {
            const int i = wave + j * kWaves;
            if (i < NI) {
                const int id = i * 64 + lane, row = id / PP, c = id % PP;
                const int rowc = row < rows_left ? row : rows_left - 1;
                const uint32_t vo = (uint32_t)(rowc * ldk + c * 8) * 2u;
                if ((PP == P8 || c < P8) && (clamp || row < rows_left))
                    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                                 :: "s"(dst + (uint32_t)i * 1024u), "v"(vo), "s"(src) : "memory");
            }
        }
    };
    // Rows past the end of the last chunk: K repeats the last row (a score that is there already, so the running
    // maximum is right), V and its ones are zero, so those rows add nothing to O or to the denominator.  (Without an
    // ones column the denominator is summed from the scores, and these are masked instead.)
    auto issue = [&](int c0, int buf) {
        const uint32_t b = lds_base + (uint32_t)buf * C::BUF;
        const int left = Nk - c0;
        copy_rows(std::integral_constant<int, KP>{}, Kp + (size_t)c0 * ldk, left, true, b);
        copy_rows(std::integral_constant<int, VP>{}, Vp + (size_t)c0 * ldk, left, false, b + C::KBYTES);
        if (left < KC)
            for (int i = left * VP + tid; i < KC * VP; i += NT)
                *reinterpret_cast<bf16x8*>(attn_smem + buf * C::BUF + C::KBYTES + i * 16) = zero8;
    };
    // every copy of this wave has landed and its LDS reads are done, for every wave behind the barrier
    auto sync_all = [&]() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // chunk c is ready and chunk c - 1's buffer is free: refill it
    auto next_chunk = [&](int c) {
        sync_all();
        if ((c + 1) * KC < Nk) issue((c + 1) * KC, (c + 1) & 1);
    };

    issue(0, 0);
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[b][ks]));
    sync_all();
    if (KC < Nk) issue(KC, 1);

    const int nsteps = (Nk + kStep - 1) / kStep;
    constexpr int DT1 = DT > 0 ? DT : 1;
    f32x16 o[2][DT1];
    f32x4 ot[2][2];                                 // TAIL: rows 32 DT .. 32 DT + 15, queries 0-15 and 16-31 of block b
    // Lazy rescaling: exponents are taken against a reference score m_run that only moves when some query of the wave would
    // otherwise exceed 2^kTau.
    const float tau = PRE ? kTau : kTau / scale_log2;
    float m_run[2] = { 0.f, 0.f }, l_run[2] = { 0.f, 0.f };
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[b][t][r] = 0.f;
#pragma unroll
    for (int b = 0; b < 2; ++b) ot[b][0] = ot[b][1] = (f32x4){ 0.f, 0.f, 0.f, 0.f };

    if (q0 < a.Nq) {
        bf16x8 kf[KS], vf[2][DT1], vt;
        f32x16 s[2];
        const f32x16 zero16 = { 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f };
        const int koff = l32 * KP * 8 + half * 8;
        const int voff = C::KBYTES / 2 + (4 * half + ((lane & 15) >> 2)) * VP * 8 + (l32 & 16) + 4 * (lane & 3);
        // tail tile: k-slices of the 16 x 16 x 32 MFMA are (chunk 0, half 0), (1, 0), (0, 1), (1, 1), see soft_pv
        const int voff_t = C::KBYTES / 2 + (16 * ((lane >> 4) & 1) + 4 * half + ((lane & 15) >> 2)) * VP * 8 + DT * 32 + 4 * (lane & 3);
        const bf16_t* base = reinterpret_cast<const bf16_t*>(attn_smem);
        auto load_k = [&](const bf16_t* p) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bf16_t* pk = p + ks * 16;
                if (C::PADM && ks == KS - 1) pk = half ? reinterpret_cast<const bf16_t*>(attn_smem + C::CONST) : pk;
                kf[ks] = *reinterpret_cast<const bf16x8*>(pk);
            }
        };
        auto load_v = [&](const bf16_t* rows) {
            const bf16_t* p = rows + voff;
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int t = 0; t < DT; ++t) {
                    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((DRF_LDS_PTR s16x4*)(p + 16 * c * VP * 8 + t * 32));
                    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((DRF_LDS_PTR s16x4*)(p + (16 * c + 8) * VP * 8 + t * 32));
                    vf[c][t] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                }
            if constexpr (C::TAIL) {
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((DRF_LDS_PTR s16x4*)(rows + voff_t));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((DRF_LDS_PTR s16x4*)(rows + voff_t + 8 * VP * 8));
                vt = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        };
        auto qk = [&](int b) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) s[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[b][ks], ks == 0 ? zero16 : s[b], 0, 0, 0);
        };
        auto largest = [&](const f32x16& v) {
            float mx = max3(v[0], v[1], v[2]);
#pragma unroll
            for (int r = 3; r < 15; r += 2) mx = max3(mx, v[r], v[r + 1]);
            return __builtin_elementwise_maximum(mx, v[15]);
        };
        // Largest score of this lane's kv rows.  Register r of s[b] holds kv row 8 (r / 4) + 4 half + r % 4 of the step.
        auto top = [&](int b, int kv0) {
            if constexpr (!C::ONES) {
                if (kv0 + kStep > Nk) {
                    const int left = Nk - kv0 - 4 * half;
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (8 * (r >> 2) + (r & 3) >= left) s[b][r] = -INFINITY;
                }
            }
            return largest(s[b]);
        };
        // Scores of block b and a step without any reference, with K straight from memory (its LDS rows may be gone): for the
        // rare cases of settle.  The spare columns meet zeros.
        auto raw = [&](int b, int step, f32x16& v) {
            const int row = step * kStep + l32;
            const bf16_t* kr = Kp + (size_t)(row < Nk ? row : Nk - 1) * ldk;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int dd = ks * 16 + half * 8;
                const bf16x8 kk = dd < d ? *reinterpret_cast<const bf16x8*>(kr + dd) : zero8;
                v = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk, qf[b][ks], ks == 0 ? zero16 : v, 0, 0, 0);
            }
        };
        // PADM: the reference is subtracted by the score MFMA itself, as three bf16 parts in Q's spare columns (24 bits: all
        // of m_run) against ones in K's, so scores arrive relative to it and need no arithmetic before the exponential.
        auto settle = [&](int b, float mx, int step, bool first) {
            const float rel = C::PADM ? mx : mx - m_run[b];
            if (__any(rel >= (first ? -INFINITY : tau))) {
                // the largest of both halves' rows; m_new: never below the reference so far
                auto both = [&](float v, float least) {
                    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
                    return max3(__uint_as_float(sw[0]), __uint_as_float(sw[1]), least);
                };
                float m_new = C::PADM ? m_run[b] + both(rel, first ? -INFINITY : 0.f) : both(mx, first ? -INFINITY : m_run[b]);
                if (first && __any(m_new == -INFINITY)) {
                    // a query that scores -infinity against all of the first 32 rows takes its reference from the next 32 that have
                    // a finite score, in the registers of the other block's scores, which hold nothing yet; failing that, 0
                    for (int st = 1; st < nsteps && __any(m_new == -INFINITY); ++st) {
                        raw(b, st, s[1 - b]);
                        const float m2 = both(largest(s[1 - b]), -INFINITY);
                        if (m_new == -INFINITY) m_new = m2;
                    }
                    if (m_new == -INFINITY) m_new = 0.f;
                }
                float delta = m_new - m_run[b], shift = delta;
                // scores far above the reference have lost their low bits to it (2^-24 of the distance): formed anew
                if (C::PADM && !first && __any(delta > kFar)) {
                    raw(b, step, s[b]);
                    shift = m_new = both(largest(s[b]), m_run[b]);
                    delta = m_new - m_run[b];
                }
                const float alpha = first ? 1.f : __builtin_amdgcn_exp2f(PRE ? -delta : -delta * scale_log2);
                m_run[b] = m_new;
                l_run[b] *= alpha;
                if constexpr (C::PADM) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) s[b][r] -= shift;
                    const bf16_t hi = (bf16_t)-m_new, mid = (bf16_t)(-m_new - (float)hi), lo = (bf16_t)((-m_new - (float)hi) - (float)mid);
                    const bf16x8 parts = { hi, mid, lo, 0, 0, 0, 0, 0 };
                    qf[b][KS - 1] = half ? parts : qf[b][KS - 1];
                }
#pragma unroll
                for (int t = 0; t < DT; ++t)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o[b][t][r] *= alpha;
                if constexpr (C::TAIL) {            // here a lane's query is lane % 16 (+ 16)
                    const auto al = __builtin_amdgcn_permlane16_swap(__float_as_uint(alpha), __float_as_uint(alpha), false, false);
#pragma unroll
                    for (int r = 0; r < 4; ++r) { ot[b][0][r] *= __uint_as_float(al[0]); ot[b][1][r] *= __uint_as_float(al[1]); }
                }
            }
        };
        auto prob = [&](int b, float v) {
            if constexpr (C::PADM) return __builtin_amdgcn_exp2f(PRE ? v : v * scale_log2);
            else return __builtin_amdgcn_exp2f(PRE ? v - m_run[b] : (v - m_run[b]) * scale_log2);
        };
        // P of block b and O^T[d][q] += sum_kv V^T[d][kv] P^T[kv][q], 16 kv rows (8 of a lane's scores) at a time
        auto soft_pv = [&](int b) {
            bf16x8 pf[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
#pragma unroll
                for (int e = 0; e < 8; ++e) s[b][8 * c + e] = prob(b, s[b][8 * c + e]);
                if constexpr (!C::ONES) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) l_run[b] += s[b][8 * c + e];
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) pf[c][e] = (bf16_t)s[b][8 * c + e];
#pragma unroll
                for (int t = 0; t < DT; ++t) o[b][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[c][t], pf[c], o[b][t], 0, 0, 0);
            }
            if constexpr (C::TAIL) {
                // 16 x 16 x 32 operands of queries 0-15 and 16-31: rows of 16 lanes 1, 3 of chunk 0 against 0, 2 of chunk 1
                u32x4 p0 = __builtin_bit_cast(u32x4, pf[0]), p1 = __builtin_bit_cast(u32x4, pf[1]);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const auto sw = __builtin_amdgcn_permlane16_swap(p0[i], p1[i], false, false);
                    p0[i] = sw[0]; p1[i] = sw[1];
                }
                ot[b][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt, __builtin_bit_cast(bf16x8, p0), ot[b][0], 0, 0, 0);
                ot[b][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt, __builtin_bit_cast(bf16x8, p1), ot[b][1], 0, 0, 0);
            }
        };
        auto pin = []() { __builtin_amdgcn_sched_barrier(0x40f); };      // LDS accesses stay on their side, the rest may cross
        constexpr int SPC = KC / kStep;             // steps per chunk
        load_k(base + koff);
        load_v(base);
        qk(0);
        settle(0, top(0, 0), 0, true);
        static_assert(SPC > 1, "the pipeline runs one step ahead");
        for (int kv = 0; kv < nsteps; ++kv) {
            // position n's fragments are read as soon as the last MFMA that needs this one's is issued (past the end: the
            // same fragments again, their scores are not used)
            const int n = kv + 1 < nsteps ? kv + 1 : kv;
            const bf16_t* nb = base + ((n / SPC) & 1) * (C::BUF / 2);
            qk(1);
            load_k(nb + (n % SPC) * (kStep * KP * 8) + koff);
            pin();
            soft_pv(0);
            settle(1, top(1, kv * kStep), kv, kv == 0);
            qk(0);
            soft_pv(1);
            load_v(nb + (n % SPC) * (kStep * VP * 8));
            pin();
            settle(0, top(0, n * kStep), n, false);
            // every fragment of this chunk has been read when step kv + 2 opens the next one
            if ((kv + 2) % SPC == 0 && kv + 2 < nsteps) next_chunk((kv + 2) / SPC);
        }
    } else {
        // no query of this wave exists: it only takes part in the copies and barriers
        for (int c = 1; c * KC < Nk; ++c) next_chunk(c);
    }
    __syncthreads();                                // the chunk buffers are free
    bf16_t* sOut = reinterpret_cast<bf16_t*>(attn_smem) + wave * (32 * LDO);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        if (q0 + b * 32 >= a.Nq) break;
        float l_tot;
        if constexpr (C::TAIL) {
            // row d of O^T is row 8 of the tail tile: register 0 of lanes 32-47, query lane % 16 (+ 16)
            const float l0 = __shfl(ot[b][0][0], 32 + (lane & 15), 64), l1 = __shfl(ot[b][1][0], 32 + (lane & 15), 64);
            l_tot = l32 < 16 ? l0 : l1;
        } else if constexpr (C::ONES) {
            constexpr int lr = d & 31, r = 4 * (lr >> 3) + (lr & 3), owner = (lr >> 2) & 1;
            const float mine = o[b][DT1 - 1][r], other = __shfl_xor(mine, 32, 64);
            l_tot = half == owner ? mine : other;
        } else {
            l_tot = l_run[b] + __shfl_xor(l_run[b], 32, 64);
        }
        // the block's 32 x d tile is transposed through the wave's LDS slice, so that rows leave in 16-byte pieces
        // (a wave's LDS operations complete in order: no barrier)
        const float inv = 1.f / l_tot;
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const bf16x4 w = { (bf16_t)(o[b][t][4 * g4] * inv), (bf16_t)(o[b][t][4 * g4 + 1] * inv),
                                   (bf16_t)(o[b][t][4 * g4 + 2] * inv), (bf16_t)(o[b][t][4 * g4 + 3] * inv) };
                *reinterpret_cast<bf16x4*>(sOut + l32 * LDO + t * 32 + 8 * g4 + 4 * half) = w;
            }
        if constexpr (C::TAIL) {
            if (lane < 32) {                        // rows 0-7 of the tail tile: four rows of query lane % 16 (+ 16) per lane
#pragma unroll
                for (int qh = 0; qh < 2; ++qh) {
                    const float iv = __shfl(inv, (lane & 15) + 16 * qh, 64);
                    const bf16x4 w = { (bf16_t)(ot[b][qh][0] * iv), (bf16_t)(ot[b][qh][1] * iv),
                                       (bf16_t)(ot[b][qh][2] * iv), (bf16_t)(ot[b][qh][3] * iv) };
                    *reinterpret_cast<bf16x4*>(sOut + ((lane & 15) + 16 * qh) * LDO + DT * 32 + 4 * (lane >> 4)) = w;
                }
            }
        }
        bf16_t* op = (bf16_t*)a.out + ((size_t)slot * a.Nq + q0 + b * 32) * a.ldo + h * d;
        for (int id = lane; id < 32 * P8; id += 64) {
            const int r = id / P8, c = id % P8;
            if (q0 + b * 32 + r < a.Nq)
                *reinterpret_cast<bf16x8*>(op + (size_t)r * a.ldo + c * 8) = *reinterpret_cast<const bf16x8*>(sOut + r * LDO + c * 8);
        }
    }
}

template <int P8, bool PRE> drf_status launch_inst(const AttnArgs& a, hipStream_t st)
{
    auto kern = attn_long_kernel<P8, PRE>;
    static bool attr_set = false;
    if (!attr_set) {
        DRF_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LongCfg<P8>::SMEM));
        attr_set = true;
    }
    const int nqb = (a.Nq + kQpg - 1) / kQpg;
    const long long n_items = (long long)nqb * a.heads * a.slots;
    if (n_items > 0x7fffffffLL) DRF_FAIL(DRF_ESHAPE, "attention: too many (query block, head, slot) items");
    hipLaunchKernelGGL(kern, dim3((unsigned)n_items), dim3(kWaves * 64), LongCfg<P8>::SMEM, st, a, attn_scale_log2(a), nqb, (int)n_items);
    DRF_HIP(hipGetLastError());
    return DRF_OK;
}

template <bool PRE> drf_status launch_width(const AttnArgs& a, hipStream_t st)
{
    switch (a.d / 8) {
    case 1: return launch_inst<1, PRE>(a, st);
    case 2: return launch_inst<2, PRE>(a, st);
    case 3: return launch_inst<3, PRE>(a, st);
    case 4: return launch_inst<4, PRE>(a, st);
    case 5: return launch_inst<5, PRE>(a, st);
    case 6: return launch_inst<6, PRE>(a, st);
    case 7: return launch_inst<7, PRE>(a, st);
    case 8: return launch_inst<8, PRE>(a, st);
    case 9: return launch_inst<9, PRE>(a, st);
    case 10: return launch_inst<10, PRE>(a, st);
    case 11: return launch_inst<11, PRE>(a, st);
    default: DRF_FAIL(DRF_ESHAPE, "attention with 64 queries per wave: head dim <= 88 (got %d)", a.d);
    }
}

}  // namespace

drf_status launch_attn_long_bf16(const AttnArgs& a, hipStream_t st)
{
    return a.q_scaled ? launch_width<true>(a, st) : launch_width<false>(a, st);
}

}  // namespace drf
