// Attention over up to 256 kv rows, bf16: softmax(q k^T / sqrt(d)) v in one step.
//
// A workgroup takes 32 QB queries of one (slot, head); its wave w owns kv rows 64 w .. 64 w + 63 and no loop over kv
// is left: every load of the workgroup is issued at once, each wave forms its scores, its own softmax numerators and
// its partial O, and the partial results (numerators relative to the wave's own maximum) are combined through LDS.
// K and V are private to their wave, so the only block barriers are those of the combination.
// Such a launch is bound by latency and by the rate at which a CU takes loads, not by arithmetic: the kernel that walks
// the kv rows in chunks spends 12-15 us on anything up to 256 work items, in four chains of load, barrier, step.
#include "common.h"

namespace drf {

namespace {

typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
#define DRF_LDS_PTR __attribute__((address_space(3)))

constexpr int kRows = 64;           // kv rows per wave
constexpr int kMaxWaves = 4;

__host__ __device__ constexpr int short_ldk(int KS) { return KS * 16 + 8; }
__host__ __device__ constexpr int short_ldv(int DT) { return DT * 32 + 16; }    // 4 rows x 32 bytes tile the 32 banks
__host__ __device__ constexpr int short_ldo(int DT) { return DT * 32 + 4; }     // floats; column DT * 32 holds the sum when no padding column does
__host__ __device__ constexpr int short_region(int KS, int DT)                  // bytes of a wave's LDS
{
    const int k = kRows * short_ldk(KS) * 2, v = kRows * short_ldv(DT) * 2, o = 32 * short_ldo(DT) * 4;
    return (k > v ? (k > o ? k : o) : (v > o ? v : o));
}

// KS = ceil(d / 16) k-steps of the score MFMA; DT = ceil(d / 32) row tiles of O^T; QB blocks of 32 queries.
// Scores are computed transposed (S^T = K Q^T): a lane owns one query column, register r of tile t holds kv row
// t * 32 + 8 * (r / 4) + 4 * half + r % 4, and P^T feeds the second MFMA from registers.  V is staged as stored and its
// transposed operand comes from the LDS transpose read, whose groups of four kv rows are those of a lane's P values.
template <int KS, int DT, int QB>
__global__ void __launch_bounds__(kMaxWaves * 64, 2)
attn_short_kernel(const AttnArgs a, float scale_log2, int nqb, int n_items, uint32_t dch_magic)
{
    constexpr int LDK = short_ldk(KS), LDV = short_ldv(DT), LDO = short_ldo(DT), REGION = short_region(KS, DT);
    extern __shared__ __attribute__((aligned(16))) unsigned char short_smem[];
    __shared__ float s_max[kMaxWaves][QB][32];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
    const int d = a.d, dch = d >> 3;
    const bf16x8 zero8 = { 0, 0, 0, 0, 0, 0, 0, 0 };

    // ids are dealt round-robin over the 8 XCDs: consecutive items, the query blocks of one head, go to one XCD's L2
    const int q8 = n_items >> 3, rem = n_items & 7, xcd = blockIdx.x & 7;
    const int item = xcd * q8 + (xcd < rem ? xcd : rem) + ((int)blockIdx.x >> 3);
    const int qb = item % nqb, hs = item / nqb, h = hs % a.heads, slot = hs / a.heads;
    const int kvb = a.kv_mod ? slot % a.kv_mod : slot;
    const bf16_t* Q = (const bf16_t*)a.q + slot * a.q_slot_stride + h * a.q_head_stride;
    const bf16_t* Kp = (const bf16_t*)a.k + kvb * a.kv_batch_stride + h * a.kv_head_stride;
    const bf16_t* Vp = (const bf16_t*)a.v + kvb * a.kv_batch_stride + h * a.kv_head_stride;
    const int q0 = qb * (32 * QB), kv0 = wave * kRows;

    // all loads: K and V as the wave's 64 rows in 16-byte pieces (consecutive lanes on consecutive pieces), Q fragments
    bf16x8 rk[2 * KS], rv[2 * KS], qf[QB][KS];
    int at[2 * KS];                                 // row * 16 + piece of this lane's c-th piece
#pragma unroll
    for (int c = 0; c < 2 * KS; ++c) {
        const int id = lane + c * 64, r = (int)(((uint32_t)id * dch_magic) >> 16), cc = id - r * dch;
        at[c] = r * 16 + cc;
        rk[c] = zero8;
        if (c < dch && kv0 + r < a.Nk) rk[c] = *reinterpret_cast<const bf16x8*>(Kp + (size_t)(kv0 + r) * a.ldk + cc * 8);
    }
#pragma unroll
    for (int b = 0; b < QB; ++b) {
        const int q = q0 + b * 32 + l32, qc = q < a.Nq ? q : a.Nq - 1;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int dd = ks * 16 + half * 8;
            qf[b][ks] = dd < d ? *reinterpret_cast<const bf16x8*>(Q + (size_t)qc * a.ldq + dd) : zero8;
        }
    }
#pragma unroll
    for (int c = 0; c < 2 * KS; ++c) {
        const int r = at[c] >> 4, cc = at[c] & 15;
        rv[c] = zero8;
        if (c < dch && kv0 + r < a.Nk) rv[c] = *reinterpret_cast<const bf16x8*>(Vp + (size_t)(kv0 + r) * a.ldk + cc * 8);
    }

    // K through the wave's LDS into fragments, then the scores
    bf16_t* buf = reinterpret_cast<bf16_t*>(short_smem + wave * REGION);
    if (d < KS * 16) *reinterpret_cast<bf16x8*>(buf + lane * LDK + d) = zero8;
#pragma unroll
    for (int c = 0; c < 2 * KS; ++c)
        if (c < dch) *reinterpret_cast<bf16x8*>(buf + (at[c] >> 4) * LDK + (at[c] & 15) * 8) = rk[c];
    bf16x8 kf[2][KS];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            kf[t][ks] = *reinterpret_cast<const bf16x8*>(buf + (t * 32 + l32) * LDK + ks * 16 + half * 8);
    f32x16 s[QB][2];
#pragma unroll
    for (int b = 0; b < QB; ++b)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const f32x16 zero16 = { 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f };
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                s[b][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t][ks], qf[b][ks], ks == 0 ? zero16 : s[b][t], 0, 0, 0);
        }
    // V takes the place of K.  When the head width leaves a padding column, its last one is set to ones: row
    // DT * 32 - 1 of O^T is then the softmax denominator.
    const bool ones_row = d < DT * 32;
#pragma unroll
    for (int c = 0; c < 2 * KS; ++c)
        if (c < dch) *reinterpret_cast<bf16x8*>(buf + (at[c] >> 4) * LDV + (at[c] & 15) * 8) = rv[c];
    if (ones_row) buf[lane * LDV + DT * 32 - 1] = (bf16_t)1.f;

    if (kv0 + kRows > a.Nk) {                       // ragged last wave: rows past the end do not take part
#pragma unroll
        for (int b = 0; b < QB; ++b)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (kv0 + t * 32 + 8 * (r >> 2) + 4 * half + (r & 3) >= a.Nk) s[b][t][r] = -INFINITY;
    }
    float m_own[QB], l_own[QB];
    bf16x8 pf[QB][2][2];
#pragma unroll
    for (int b = 0; b < QB; ++b) {
        float mx = fmaxf(s[b][0][0], s[b][1][0]);
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, fmaxf(s[b][0][r], s[b][1][r]));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        m_own[b] = mx * scale_log2;
        if (half == 0) s_max[wave][b][l32] = m_own[b];
        // (a wave whose 64 rows all score -infinity has no reference: its numerators are zero against any)
        const float ref = m_own[b] == -INFINITY ? 0.f : m_own[b];
        float sum = 0.f;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float p = __builtin_amdgcn_exp2f(fmaf(s[b][t][r], scale_log2, -ref));
                sum += p;
                pf[b][t][r >> 3][r & 7] = (bf16_t)p;
            }
        l_own[b] = sum;                             // this half's share (used when there is no ones row)
    }
    // O^T[d][q] = sum_kv V^T[d][kv] P^T[kv][q]
    f32x16 o[QB][DT];
#pragma unroll
    for (int b = 0; b < QB; ++b)
#pragma unroll
        for (int tt = 0; tt < DT; ++tt)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[b][tt][r] = 0.f;
    const bf16_t* vl = buf + (4 * half + ((lane & 15) >> 2)) * LDV + (l32 & 16) + 4 * (lane & 3);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int tt = 0; tt < DT; ++tt) {
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((DRF_LDS_PTR s16x4*)(vl + (t * 32 + 16 * c) * LDV + tt * 32));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((DRF_LDS_PTR s16x4*)(vl + (t * 32 + 16 * c + 8) * LDV + tt * 32));
                const bf16x8 vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
                for (int b = 0; b < QB; ++b) o[b][tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[b][t][c], o[b][tt], 0, 0, 0);
            }
    __syncthreads();                                // every wave's maxima are visible

    // Combination, one block of 32 queries at a time: every wave leaves its partial O, scaled to the common maximum, in
    // its own region ([query][d], the denominator in column `lcol`), then the workgroup adds them and stores whole rows.
    float* po = reinterpret_cast<float*>(short_smem);
    const int lcol = ones_row ? DT * 32 - 1 : DT * 32;
#pragma unroll
    for (int b = 0; b < QB; ++b) {
        float m = m_own[b];
        for (int w = 0; w < nw; ++w) m = fmaxf(m, s_max[w][b][l32]);
        const float f = __builtin_amdgcn_exp2f(m_own[b] - m);
        float* mine = po + wave * (REGION / 4) + l32 * LDO;
#pragma unroll
        for (int tt = 0; tt < DT; ++tt)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
                *reinterpret_cast<float4*>(mine + tt * 32 + 8 * g4 + 4 * half) =
                    make_float4(o[b][tt][4 * g4] * f, o[b][tt][4 * g4 + 1] * f, o[b][tt][4 * g4 + 2] * f, o[b][tt][4 * g4 + 3] * f);
        if (!ones_row) {
            const float l = l_own[b] + __shfl_xor(l_own[b], 32, 64);
            if (half == 0) mine[DT * 32] = l * f;
        }
        __syncthreads();
        const int qn = a.Nq - (q0 + b * 32);        // rows of this block that exist (may be <= 0)
        bf16_t* op = (bf16_t*)a.out + ((size_t)slot * a.Nq + q0 + b * 32) * a.ldo + h * d;
        for (int id = tid; id < 32 * dch; id += blockDim.x) {
            const int r = (int)(((uint32_t)id * dch_magic) >> 16), cc = id - r * dch;
            const float* src = po + r * LDO;
            float l = src[lcol];
            float4 x = *reinterpret_cast<const float4*>(src + cc * 8), y = *reinterpret_cast<const float4*>(src + cc * 8 + 4);
            for (int w = 1; w < nw; ++w) {
                const float* sw = src + w * (REGION / 4);
                l += sw[lcol];
                const float4 x2 = *reinterpret_cast<const float4*>(sw + cc * 8), y2 = *reinterpret_cast<const float4*>(sw + cc * 8 + 4);
                x.x += x2.x; x.y += x2.y; x.z += x2.z; x.w += x2.w;
                y.x += y2.x; y.y += y2.y; y.z += y2.z; y.w += y2.w;
            }
            const float inv = 1.f / l;
            const bf16x8 w8 = { (bf16_t)(x.x * inv), (bf16_t)(x.y * inv), (bf16_t)(x.z * inv), (bf16_t)(x.w * inv),
                                (bf16_t)(y.x * inv), (bf16_t)(y.y * inv), (bf16_t)(y.z * inv), (bf16_t)(y.w * inv) };
            if (r < qn) *reinterpret_cast<bf16x8*>(op + (size_t)r * a.ldo + cc * 8) = w8;
        }
        if (b + 1 < QB) __syncthreads();
    }
}

template <int KS, int DT, int QB>
drf_status launch_short(const AttnArgs& a, float scale_log2, hipStream_t st)
{
    const int nw = (a.Nk + kRows - 1) / kRows, nqb = (a.Nq + 32 * QB - 1) / (32 * QB), dch = a.d / 8;
    const size_t smem = (size_t)nw * short_region(KS, DT);
    static_assert(2 * (kMaxWaves * short_region(KS, DT) + kMaxWaves * QB * 128) <= 160 * 1024, "two workgroups per CU");
    const long long n_items = (long long)nqb * a.heads * a.slots;
    if (n_items > 0x7fffffffLL) DRF_FAIL(DRF_ESHAPE, "attention: too many (query block, head, slot) items");
    // floor(id / dch) == id * magic >> 16 for id < 64 * 12: the error term id * (magic - 65536 / dch) stays below 65536 / dch
    const uint32_t magic = 65536u / (uint32_t)dch + 1u;
    hipLaunchKernelGGL((attn_short_kernel<KS, DT, QB>), dim3((unsigned)n_items), dim3(nw * 64), smem, st, a, scale_log2, nqb, (int)n_items, magic);
    DRF_HIP(hipGetLastError());
    return DRF_OK;
}

// Work items of 32 queries that run at once: workgroups per CU by LDS and by the three waves a SIMD's registers hold.
template <int KS, int DT> int short_round(int nw)
{
    const int by_lds = 160 * 1024 / (nw * short_region(KS, DT) + kMaxWaves * 128), by_regs = 12 / nw;
    return 256 * (by_lds < by_regs ? by_lds : by_regs);
}

}  // namespace

int attn_short_items_at_once(int Nk, int d)
{
    const int nw = (Nk + kRows - 1) / kRows;
    switch ((d + 15) / 16) {
    case 1: return short_round<1, 1>(nw);
    case 2: return short_round<2, 1>(nw);
    case 3: return short_round<3, 2>(nw);
    case 4: return short_round<4, 2>(nw);
    case 5: return short_round<5, 3>(nw);
    default: return short_round<6, 3>(nw);
    }
}

drf_status launch_attn_short_bf16(const AttnArgs& a, int queries, hipStream_t st)
{
    if (a.Nk > kRows * kMaxWaves) DRF_FAIL(DRF_ESHAPE, "one wave per 64 rows: at most %d kv rows", kRows * kMaxWaves);
    const float sl2 = attn_scale_log2(a);
#define DRF_SHORT(KS, DT) (queries == 32 ? launch_short<KS, DT, 1>(a, sl2, st) : launch_short<KS, DT, 2>(a, sl2, st))
    switch ((a.d + 15) / 16) {
    case 1: return DRF_SHORT(1, 1);
    case 2: return DRF_SHORT(2, 1);
    case 3: return DRF_SHORT(3, 2);
    case 4: return DRF_SHORT(4, 2);
    case 5: return DRF_SHORT(5, 3);
    default: return DRF_SHORT(6, 3);
    }
#undef DRF_SHORT
}

}  // namespace drf
