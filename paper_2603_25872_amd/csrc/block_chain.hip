// The part of a transformer block that works on rows alone, as one launch for narrow models: attention projection, gated residual, LayerNorm,
// fc1, GELU, fc2, gated residual, the next block's LayerNorm and its q | k | v projection; with heads of 64, the self-attention before it too.
#include <type_traits>

#include "common.h"

namespace drf {

namespace {

typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
#define DRF_LDS_PTR __attribute__((address_space(3)))

constexpr int kChainWaves = 8, kChainRatio = 4;     // waves of a workgroup; largest MLP ratio
constexpr int kChainHead = 64;                      // head width of the self-attention form

template <int NI, int MI> struct ChainCfg {
    static constexpr int D = 128 * NI, KS = D / 32, ROWS = 16 * MI;
    static constexpr int PITCH = D * 2 + 16;                    // bytes per row in LDS: 16 rows of 16-byte reads on distinct banks
    static constexpr int TILE = ROWS * PITCH;
    static constexpr int MODS = 6 * D * 4;                      // six modulation rows
    static constexpr int BIAS = (5 + kChainRatio) * D * 4;      // proj | fc1 | fc2 | q k v
    static constexpr int RED = kChainWaves * ROWS * 8;          // a wave's mean and squares of every row
    static constexpr int HB = 3 * TILE + MODS + BIAS + RED <= 160 * 1024 ? 2 : 1;       // tiles of hidden units
    static constexpr int SMEM = (1 + HB) * TILE + MODS + BIAS + RED;
    static constexpr int PD = 4;                                // k-steps of weights in flight
    static constexpr int FD = MI == 1 ? 4 : 2;                  // k-steps of activation fragments: those read ahead and the one in use
    static_assert(KS % PD == 0 && SMEM <= 160 * 1024, "shape");
};

__device__ inline float chain_gelu(float x)         // as gelu_tanh in gemm_device.h
{
    const float t = x * x;
    const float m2u_log2e = x * fmaf(t, -0.1029432f, -2.3022082f);
    return x * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(m2u_log2e));
}

// LDS accesses of every wave of the workgroup are done; loads to registers stay in flight.
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The larger of a value of this lane and those of the three lanes with the same l16.
__device__ inline float quarters_max(float v)
{
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

__device__ inline float quarters_sum(float v)
{
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Self-attention of one head (width 64) for 16 MI queries of a slot over its T keys; queries are scaled to exponents of two.  q: this lane's
// first query piece, rows of ldq; k, v: the head's keys and values in fragments of 32 keys (see ChainArgs).  The scores are computed
// transposed, a lane holding keys 8 quarter .. + 7 of every 32 for query l16, which is the operand layout of P in O^T += V^T P^T; the
// denominator is the product of P, as rounded, with ones.  Results as bf16 into `out`.
template <int MI>
__device__ __forceinline__ void head_attention(const bf16_t* const (&q)[MI], const bf16_t* k, const bf16_t* v, int T, unsigned char* out, int pitch)
{
    constexpr int U = 2, CK = U * 32;               // keys per softmax step (four groups of 32 spill)
    constexpr int STEP = 32 * kChainHead * 2;       // bytes of 32 keys
    const int lane = threadIdx.x & 63, l16 = lane & 15, quarter = lane >> 4, lane16 = lane * 16, groups = (T + 31) / 32;
    const bf16_t one = (bf16_t)1.f;
    const bf16x8 ones = { one, one, one, one, one, one, one, one };
    const auto krsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(k), 0, groups * STEP, 0x00020000);
    const auto vrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(v), 0, groups * STEP, 0x00020000);
    bf16x8 qf[MI][2], kf[U][4], vf[U][4];           // k: [32 keys][16 of them, half of the head], v: [32 keys][16 columns]
    auto load = [&](bf16x8 (&f)[U][4], decltype(krsrc) rsrc, int g0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                f[u][i] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane16 + i * 1024, (g0 + u < groups ? g0 + u : groups - 1) * STEP, 0));
    };
#pragma unroll
    for (int j = 0; j < MI; ++j)
#pragma unroll
        for (int s = 0; s < 2; ++s) qf[j][s] = *reinterpret_cast<const bf16x8*>(q[j] + s * 32);
    load(kf, krsrc, 0);
    f32x4 o[4][MI], den[MI];
    float m_run[MI];
#pragma unroll
    for (int j = 0; j < MI; ++j) {
        m_run[j] = -INFINITY;
        den[j] = (f32x4){ 0.f, 0.f, 0.f, 0.f };
#pragma unroll
        for (int d = 0; d < 4; ++d) o[d][j] = (f32x4){ 0.f, 0.f, 0.f, 0.f };
    }
    for (int k0 = 0; k0 < T; k0 += CK) {
        load(vf, vrsrc, k0 / 32);
        f32x4 s[U][2][MI];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int j = 0; j < MI; ++j) {
                    s[u][b][j] = (f32x4){ 0.f, 0.f, 0.f, 0.f };
#pragma unroll
                    for (int h = 0; h < 2; ++h) s[u][b][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[u][2 * b + h], qf[j][h], s[u][b][j], 0, 0, 0);
                }
        __builtin_amdgcn_sched_barrier(0);
        if (k0 + CK < T) load(kf, krsrc, k0 / 32 + U);
        else if (k0 + CK > T) {
            // keys past the end score -infinity, and whatever their values' places hold is not met by their zero weights
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (k0 + u * 32 + 8 * quarter + e >= T) {
#pragma unroll
                        for (int j = 0; j < MI; ++j) s[u][e >> 2][j][e & 3] = -INFINITY;
#pragma unroll
                        for (int d = 0; d < 4; ++d) vf[u][d][e] = (bf16_t)0.f;
                    }
        }
        bf16x8 pf[U][MI];
#pragma unroll
        for (int j = 0; j < MI; ++j) {
            f32x4 m4 = s[0][0][j];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r) m4[r] = fmaxf(m4[r], s[u][b][j][r]);
            const float m_new = fmaxf(m_run[j], quarters_max(fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3])))), ref = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = __builtin_amdgcn_exp2f(m_run[j] - ref);
            m_run[j] = m_new;
            den[j] *= alpha;
#pragma unroll
            for (int d = 0; d < 4; ++d) o[d][j] *= alpha;
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r) pf[u][j][4 * b + r] = (bf16_t)__builtin_amdgcn_exp2f(s[u][b][j][r] - ref);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < MI; ++j) {
#pragma unroll
                for (int d = 0; d < 4; ++d) o[d][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[u][d], pf[u][j], o[d][j], 0, 0, 0);
                den[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[u][j], den[j], 0, 0, 0);
            }
    }
#pragma unroll
    for (int j = 0; j < MI; ++j) {
        const float inv = 1.f / den[j][0];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const bf16x4 w = { (bf16_t)(o[d][j][0] * inv), (bf16_t)(o[d][j][1] * inv), (bf16_t)(o[d][j][2] * inv), (bf16_t)(o[d][j][3] * inv) };
            *reinterpret_cast<bf16x4*>(out + (j * 16 + l16) * pitch + d * 32 + quarter * 8) = w;
        }
    }
}

// A workgroup takes 16 MI rows of one slot through the whole chain.  The rows stay on the chip: activations as bf16 tiles in LDS, the stream in
// registers in the accumulators' layout; a wave owns 16 NI columns of every D x D unit of weights.
// What bounds it: the weights, which every workgroup reads in full (3.5 MB a block at hidden 384, ratio 4) through its CU's 64 bytes a
// clock: 23 us of the 41 that a launch of 16 rows takes (with or without the attention, 192 and 224 workgroups), however many there are
// up to 256; the attention, barriers, LayerNorms and GELU take the rest.  Against that stand seven launches of 5 to 13 us with their
// results through memory.  Hence:
//  - weights go from memory to registers in a layout of their own (1 KB of consecutive bytes per 16 x 32 fragment; 16 rows of 64
//    bytes an instruction take the vector-memory path two to three times as long), each fragment read by one wave once, four k-steps
//    ahead of their use and across the barriers (six steps ahead: no gain; each XCD's workgroups touching all lines first: no gain);
//  - 16 rows while all workgroups run at once, since the stream costs the same for 32 (47 us without the attention, 52 with it and
//    200 workgroups, 56 with 256) and 64 (65 with 200, 72 with 256: matrix unit, and at hidden 384 all 256 registers and 9 more in
//    scratch, 40 bytes a lane; 64 x 256 rows are still faster so than at 32 rows a workgroup, 1129 against 1229 us an evaluation);
//  - biases, modulation rows and the attention output are asked for together ahead of everything (asked for where they were used,
//    they cost 64 rows 10 us);
//  - ATT: the self-attention of these rows' queries, a head a wave, from keys and values that the launch before left as operand fragments:
//    5 us at 256 keys by its clocks, 3 of them more than the form that reads an attention output takes, where a launch of its own
//    takes 10; from head-major planes, transposing values through LDS in every workgroup, it took 7.5 us;
//  - few rows leave CUs idle, each of the others streaming all weights: the hidden units are then dealt over two or four workgroups a row
//    tile (projection and 2 ratio / parts units each: 19 us at 4 x 256 rows in four parts, 23 at 5 x 247 in two), and a second launch adds
//    their shares of the stream and deals q, k and v over two or three (9 to 12 us; 5 us to add up behind the last block, and for
//    the first q, k and v).  5 slots of 247 rows 525 us an evaluation of 12 blocks in one launch each, 422 so, one by one 510.
// A call of 16 passes of 3072 rows and two of 1024 (hidden 384, 12 blocks) 11.78 -> 8.84 ms; passes of 6175 rows 998 -> 618 us, of 16384 1756 -> 1129.
template <int NI, int MI, bool ATT>
__global__ void __launch_bounds__(kChainWaves * 64)
block_chain_kernel(const ChainArgs a, int tiles)
{
    using C = ChainCfg<NI, MI>;
    constexpr int D = C::D, KS = C::KS, ROWS = C::ROWS, PITCH = C::PITCH, PD = C::PD, FD = C::FD, HB = C::HB, NT = kChainWaves * 64;
    constexpr int UNIT = D * D * 2;                 // bytes of a D x D weight unit
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char* const ybuf = smem;
    unsigned char* const hbuf = smem + C::TILE;
    float* const mods = reinterpret_cast<float*>(smem + (1 + HB) * C::TILE);
    float* const biases = mods + C::MODS / 4;
    float2* const red = reinterpret_cast<float2*>(biases + C::BIAS / 4);

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, quarter = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // a workgroup's rows belong to one slot; the tiles of a slot run on one XCD (ids are dealt round-robin over the 8 of them)
    const int nb = gridDim.x, xcd = blockIdx.x & 7, per = nb >> 3, rem = nb & 7;
    const int idx = xcd * per + (xcd < rem ? xcd : rem) + (blockIdx.x >> 3);
    const int part = a.parts > 1 ? idx % a.parts : 0, tile = a.parts > 1 ? idx / a.parts : idx;
    const int slot = tile / tiles, t0 = (tile - slot * tiles) * ROWS, T = a.tokens, row0 = slot * T + t0;
    const int left = T - t0;                        // rows of the tile that exist
    const size_t part_len = (size_t)a.slots * T * D;
    if constexpr (!ATT && MI == 1) {
        if (!a.attn && !a.qkv && !a.kv_out) {       // behind the last block only the shares are added up, in their order
            for (int id = tid; id < ROWS * D / 4; id += NT) {
                const size_t at = (size_t)row0 * D + id * 4;
                if (id / (D / 4) >= left) break;
                f32x4 v = *reinterpret_cast<const f32x4*>(a.part_in + at);
                for (int s = 1; s < a.n_in; ++s) v += *reinterpret_cast<const f32x4*>(a.part_in + s * part_len + at);
                *reinterpret_cast<f32x4*>(a.resid + at) = v;
            }
            return;
        }
    }
    const int col = wave * (16 * NI) + 4 * quarter;             // this lane's columns of a unit: col + 16 i .. + 3
    const bool has_mlp = ATT || a.attn, has_qkv = a.qkv || a.kv_out;
    // this workgroup's pieces of D hidden units, and of q, k, v
    const int c0 = part * a.mlp_ratio / a.parts, c1 = (part + 1) * a.mlp_ratio / a.parts, p0 = has_mlp ? 0 : part * 3 / a.parts, p1 = has_mlp ? 3 : (part + 1) * 3 / a.parts;

    // behind the attention, every operand is asked for before the first is used, in the order of their use
    constexpr int PIECES = ROWS * D / 8, PU = (PIECES + NT - 1) / NT;             // 16-byte pieces of a bf16 row tile
    constexpr int D4 = D / 4, MU = (6 * D4 + NT - 1) / NT, BU = ((5 + kChainRatio) * D4 + NT - 1) / NT;
    bf16x8 rows_in[ATT ? 1 : PU];
    f32x4 mod_in[MU], bias_in[BU];
    const int n_bias = (a.mlp_ratio + 5) * D4, fc2_at = (a.mlp_ratio + 1) * D4;
    if (!ATT && a.attn) {
#pragma unroll
        for (int u = 0; u < PU; ++u) {
            const int id = tid + u * NT, r = id / (D / 8), c = id % (D / 8);
            if (PIECES % NT == 0 || id < PIECES) rows_in[u] = *reinterpret_cast<const bf16x8*>(a.attn + (size_t)(row0 + (r < left ? r : left - 1)) * D + c * 8);
        }
    }
    bf16x8 ring[PD][NI];
    const auto wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.weights), 0, ((has_mlp ? 1 + 2 * a.mlp_ratio : 0) + (has_qkv ? 3 : 0)) * UNIT, 0x00020000);
    const int lane16 = lane * 16;
    auto load_step = [&](bf16x8 (&dst)[NI], int p) {
#pragma unroll
        for (int i = 0; i < NI; ++i) dst[i] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, lane16 + i * 1024, p, 0));
    };
    int wp = wave * (KS * NI * 1024) + p0 * UNIT;
    float* xp[MI];
    f32x4 x[NI][MI];
#pragma unroll
    for (int j = 0; j < MI; ++j) {
        const int r = j * 16 + l16;
        xp[j] = a.resid + (size_t)(row0 + (r < left ? r : left - 1)) * D + col;
    }
    if constexpr (ATT) {
        const size_t head = (size_t)((T + 31) / 32 * 32) * kChainHead;          // elements of a head's keys
        for (int h = wave; h < a.heads; h += kChainWaves) {
            const bf16_t *q[MI], *k = a.kv_in + (slot * a.heads + h) * head;
#pragma unroll
            for (int j = 0; j < MI; ++j) {
                const int r = j * 16 + l16;
                q[j] = a.q + (size_t)(row0 + (r < left ? r : left - 1)) * D + h * kChainHead + quarter * 8;
            }
            head_attention<MI>(q, k, k + a.slots * a.heads * head, T, ybuf + h * kChainHead * 2, PITCH);
        }
    }
#pragma unroll
    for (int u = 0; u < MU; ++u) {
        const int id = tid + u * NT;
        if (id < 6 * D4 && (has_mlp || id >= 4 * D4)) mod_in[u] = *reinterpret_cast<const f32x4*>(a.mod + (ptrdiff_t)slot * a.mod_ld + id * 4);
    }
#pragma unroll
    for (int u = 0; u < BU; ++u) {
        const int id = tid + u * NT;
        const float* src = id < D4 ? a.b_proj + id * 4 : id < fc2_at ? a.b_fc1 + (id - D4) * 4 : id < fc2_at + D4 ? a.b_fc2 + (id - fc2_at) * 4 : a.b_qkv + (id - fc2_at - D4) * 4;
        if (id < n_bias && (id < fc2_at + D4 ? has_mlp : has_qkv)) bias_in[u] = *reinterpret_cast<const f32x4*>(src);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < PD; ++s) load_step(ring[s], wp + s * NI * 1024);
    __builtin_amdgcn_sched_barrier(0);
    // (not where the stream is the sum of shares: another workgroup of the row tile stores it in this launch)
    if (ATT || MI > 1 || !a.part_in)
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < MI; ++j) x[i][j] = *reinterpret_cast<const f32x4*>(xp[j] + i * 16);
    __builtin_amdgcn_sched_barrier(0);
    if (!ATT && a.attn) {
#pragma unroll
        for (int u = 0; u < PU; ++u) {
            const int id = tid + u * NT, r = id / (D / 8), c = id % (D / 8);
            if (PIECES % NT == 0 || id < PIECES) *reinterpret_cast<bf16x8*>(ybuf + r * PITCH + c * 16) = rows_in[u];
        }
    }
#pragma unroll
    for (int u = 0; u < MU; ++u)
        if (tid + u * NT < 6 * D4) reinterpret_cast<f32x4*>(mods)[tid + u * NT] = mod_in[u];
#pragma unroll
    for (int u = 0; u < BU; ++u)
        if (tid + u * NT < n_bias) reinterpret_cast<f32x4*>(biases)[tid + u * NT] = bias_in[u];

    // acc[i][j] += this wave's 16 NI columns of a weight unit times the rows in `tile`; the ring then holds the first steps of `next`
    const int a_ofs = l16 * PITCH + quarter * 16;
    auto unit = [&](f32x4 (&acc)[NI][MI], const unsigned char* tile, int cur, int next) {
        bf16x8 fa[FD][MI];
        auto read = [&](int ks) {
#pragma unroll
            for (int j = 0; j < MI; ++j) fa[ks % FD][j] = *reinterpret_cast<const bf16x8*>(tile + a_ofs + j * 16 * PITCH + ks * 64);
        };
#pragma unroll
        for (int ks = 0; ks < FD - 1; ++ks) read(ks);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks + FD - 1 < KS) read(ks + FD - 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < MI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ring[ks % PD][i], fa[ks % FD][j], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            load_step(ring[ks % PD], ks + PD < KS ? cur + (ks + PD) * NI * 1024 : next + (ks + PD - KS) * NI * 1024);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto zero = [&](f32x4 (&acc)[NI][MI]) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < MI; ++j) acc[i][j] = (f32x4){ 0.f, 0.f, 0.f, 0.f };
    };
    auto mod_at = [&](int which, int i) -> f32x4 { return *reinterpret_cast<const f32x4*>(mods + which * D + col + i * 16); };
    auto bias_at = [&](int row, int i) -> f32x4 { return *reinterpret_cast<const f32x4*>(biases + row * D + col + i * 16); };
    // x += gate * (acc + bias)
    auto add_branch = [&](const f32x4 (&acc)[NI][MI], int bias, int gate) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const f32x4 g = mod_at(gate, i), b = bias_at(bias, i);
#pragma unroll
            for (int j = 0; j < MI; ++j) {
                const f32x4 v = acc[i][j] + b;
#pragma unroll
                for (int r = 0; r < 4; ++r) x[i][j][r] = fmaf(g[r], v[r], x[i][j][r]);
            }
        }
    };
    // ybuf = LN(x) * (1 + scale) + shift.  A wave's mean and squares about it are combined with those of the others, so one exchange will do.
    auto norm = [&](int shift, int scale) {
        constexpr float per_wave = 16.f * NI;
#pragma unroll
        for (int j = 0; j < MI; ++j) {
            float s = 0.f, q = 0.f;
#pragma unroll
            for (int i = 0; i < NI; ++i) s += (x[i][j][0] + x[i][j][1]) + (x[i][j][2] + x[i][j][3]);
            s = quarters_sum(s);
            const float mean = s * (1.f / per_wave);
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) { const float c = x[i][j][r] - mean; q = fmaf(c, c, q); }
            q = quarters_sum(q);
            if (quarter == 0) red[wave * ROWS + j * 16 + l16] = make_float2(mean, q);
        }
        lds_barrier();
        float mean[MI], rstd[MI];
#pragma unroll
        for (int j = 0; j < MI; ++j) {
            float2 p[kChainWaves];
            float q = 0.f;
            mean[j] = 0.f;
#pragma unroll
            for (int w = 0; w < kChainWaves; ++w) { p[w] = red[w * ROWS + j * 16 + l16]; mean[j] += p[w].x; q += p[w].y; }
            mean[j] *= 1.f / kChainWaves;
#pragma unroll
            for (int w = 0; w < kChainWaves; ++w) { const float c = p[w].x - mean[j]; q = fmaf(per_wave * c, c, q); }
            rstd[j] = rsqrtf(q * (1.f / (float)D) + 1e-6f);
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const f32x4 sc = mod_at(scale, i), sh = mod_at(shift, i);
#pragma unroll
            for (int j = 0; j < MI; ++j) {
                bf16x4 o;
#pragma unroll
                for (int r = 0; r < 4; ++r) o[r] = (bf16_t)fmaf((x[i][j][r] - mean[j]) * rstd[j], 1.f + sc[r], sh[r]);
                *reinterpret_cast<bf16x4*>(ybuf + (j * 16 + l16) * PITCH + (col + i * 16) * 2) = o;
            }
        }
        lds_barrier();
    };
    // the ring's last loads, which nothing uses, are not left to a wave's end
    auto drain = []() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };

    if (has_mlp) {
        f32x4 acc[NI][MI], sum[NI][MI];
        zero(sum);
        lds_barrier();
        unit(sum, ybuf, wp, wp + (1 + 2 * c0) * UNIT);
        wp += (1 + 2 * c0) * UNIT;
        add_branch(sum, 0, 0);
        norm(1, 2);
        zero(sum);
        for (int c = c0; c < c1; ++c) {
            unsigned char* const h = hbuf + (HB == 2 && (c & 1) ? C::TILE : 0);
            zero(acc);
            unit(acc, ybuf, wp, wp + UNIT);
            wp += UNIT;
            if (HB == 1) lds_barrier();             // every wave has read the previous tile
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const f32x4 b = bias_at(1 + c, i);
#pragma unroll
                for (int j = 0; j < MI; ++j) {
                    const f32x4 v = acc[i][j] + b;
                    const bf16x4 o = { (bf16_t)chain_gelu(v[0]), (bf16_t)chain_gelu(v[1]), (bf16_t)chain_gelu(v[2]), (bf16_t)chain_gelu(v[3]) };
                    *reinterpret_cast<bf16x4*>(h + (j * 16 + l16) * PITCH + (col + i * 16) * 2) = o;
                }
            }
            lds_barrier();
            const bool more = has_qkv || c + 1 < c1;
            unit(sum, h, wp, more ? wp + UNIT : wp);
            wp += UNIT;
        }
        if (part == 0) add_branch(sum, 1 + a.mlp_ratio, 3);
        else {
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const f32x4 g = mod_at(3, i);
#pragma unroll
                for (int j = 0; j < MI; ++j) x[i][j] = g * sum[i][j];
            }
        }
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < MI; ++j)
                if (j * 16 + l16 < left) {
                    float* to = a.part_out ? a.part_out + part * part_len + (xp[j] - a.resid) : xp[j];
                    *reinterpret_cast<f32x4*>(to + i * 16) = x[i][j];
                }
    } else {
        if constexpr (MI == 1) {
            if (a.part_in) {                        // the stream is the sum of the parts' shares, added in their order
                f32x4 more[kChainRatio][NI];
#pragma unroll
                for (int s = 0; s < kChainRatio; ++s)
#pragma unroll
                    for (int i = 0; i < NI; ++i)
                        if (s < a.n_in) more[s][i] = *reinterpret_cast<const f32x4*>(a.part_in + s * part_len + (xp[0] - a.resid) + i * 16);
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    x[i][0] = more[0][i];
#pragma unroll
                    for (int s = 1; s < kChainRatio; ++s)
                        if (s < a.n_in) x[i][0] += more[s][i];
                    if (part == 0 && l16 < left) *reinterpret_cast<f32x4*>(xp[0] + i * 16) = x[i][0];
                }
            }
        }
        lds_barrier();
    }
    if (!has_qkv) { drain(); return; }
    norm(4, 5);
    for (int p = p0; p < p1; ++p) {
        f32x4 acc[NI][MI];
        unsigned char* const h = hbuf + (HB == 2 && (p & 1) ? C::TILE : 0);
        zero(acc);
        unit(acc, ybuf, wp, p + 1 < p1 ? wp + UNIT : wp);
        wp += UNIT;
        const float scale = p == 0 ? a.q_scale : 1.f;
        if (HB == 1) lds_barrier();
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const f32x4 b = bias_at(2 + a.mlp_ratio + p, i);
#pragma unroll
            for (int j = 0; j < MI; ++j) {
                const f32x4 v = (acc[i][j] + b) * scale;
                const bf16x4 o = { (bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3] };
                *reinterpret_cast<bf16x4*>(h + (j * 16 + l16) * PITCH + (col + i * 16) * 2) = o;
            }
        }
        lds_barrier();
        if (a.kv_out && p == 2) {
            // value fragments: columns of 8 rows, transposed on the way out of LDS
            const size_t head_len = (size_t)((T + 31) / 32 * 32) * kChainHead;
#pragma unroll
            for (int u = 0; u < PU; ++u) {
                const int id = tid + u * NT, g = (id >> 4) % (ROWS / 8), ct = (id >> 4) / (ROWS / 8), key = t0 + g * 8;
                if (PIECES % NT == 0 || id < PIECES) {
                    const unsigned char* src = h + (g * 8 + (l16 >> 2)) * PITCH + ct * 32 + (lane & 3) * 8;
                    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((DRF_LDS_PTR s16x4*)src);
                    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((DRF_LDS_PTR s16x4*)(src + 4 * PITCH));
                    bf16_t* out = a.kv_out + (a.slots * a.heads + slot * a.heads + (ct >> 2)) * head_len + (key >> 5) * (32 * kChainHead);
                    *reinterpret_cast<bf16x8*>(out + ((ct & 3) * 64 + ((key >> 3) & 3) * 16 + l16) * 8) = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                }
            }
            continue;
        }
        if (a.kv_out && p == 1) {
            const size_t head_len = (size_t)((T + 31) / 32 * 32) * kChainHead;
#pragma unroll
            for (int u = 0; u < PU; ++u) {
                const int id = tid + u * NT, r = id % ROWS, c = id / ROWS, key = t0 + r, half = (c >> 2) & 1;
                if ((PIECES % NT == 0 || id < PIECES) && r < left) {
                    bf16_t* out = a.kv_out + (slot * a.heads + (c >> 3)) * head_len + (key >> 5) * (32 * kChainHead);
                    *reinterpret_cast<bf16x8*>(out + (((key >> 2) & 1) * 128 + half * 64 + (c & 3) * 16 + ((key >> 3) & 3) * 4 + (key & 3)) * 8) =
                        *reinterpret_cast<const bf16x8*>(h + r * PITCH + c * 16);
                }
            }
            continue;
        }
#pragma unroll
        for (int u = 0; u < PU; ++u) {
            const int id = tid + u * NT, r = id / (D / 8), c = id % (D / 8);
            if ((PIECES % NT == 0 || id < PIECES) && r < left) {
                const bf16x8 v = *reinterpret_cast<const bf16x8*>(h + r * PITCH + c * 16);
                if (a.kv_out) *reinterpret_cast<bf16x8*>(a.q + (size_t)(row0 + r) * D + c * 8) = v;
                else {
                    const int head = a.hd_magic ? (int)(__umulhi((uint32_t)(c * 8), a.hd_magic) >> a.hd_shift) : (c * 8) >> a.hd_shift;
                    *reinterpret_cast<bf16x8*>(a.qkv + (size_t)p * a.plane + ((size_t)(slot * a.heads + head) * T + t0 + r) * a.hd + (c * 8 - head * a.hd)) = v;
                }
            }
        }
    }
    drain();
}

// Weight units in the order and layout that the kernel streams: unit, wave, k-step, 16-column piece, lane.
__global__ void __launch_bounds__(256) chain_pack_kernel(const bf16_t* __restrict__ w, int ld, int NI, int KS, bf16_t* __restrict__ out)
{
    const int id = blockIdx.x * 256 + threadIdx.x, lane = id & 63;      // one 16-byte piece
    int f = id >> 6;
    const int i = f % NI; f /= NI;
    const int ks = f % KS, wave = f / KS;
    if (wave >= kChainWaves) return;
    const int n = (wave * NI + i) * 16 + (lane & 15), k = ks * 32 + (lane >> 4) * 8;
    *reinterpret_cast<bf16x8*>(out + (size_t)id * 8) = *reinterpret_cast<const bf16x8*>(w + (size_t)n * ld + k);
}

template <int NI, int MI, bool ATT> drf_status launch_inst(const ChainArgs& a, hipStream_t st)
{
    using C = ChainCfg<NI, MI>;
    auto kern = block_chain_kernel<NI, MI, ATT>;
    static bool attr_set = false;
    if (!attr_set) {
        DRF_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, C::SMEM));
        attr_set = true;
    }
    const int tiles = (a.tokens + C::ROWS - 1) / C::ROWS;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.slots * tiles * a.parts)), dim3(kChainWaves * 64), C::SMEM, st, a, tiles);
    DRF_HIP(hipGetLastError());
    return DRF_OK;
}

template <int NI, bool ATT> drf_status launch_rows(const ChainArgs& a, int rows, hipStream_t st)
{
    switch (rows) {
    case 16: return launch_inst<NI, 1, ATT>(a, st);
    case 32: return launch_inst<NI, 2, ATT>(a, st);
    case 64: if constexpr (!ATT && NI <= 3) return launch_inst<NI, 4, false>(a, st); [[fallthrough]];
    default: DRF_FAIL(DRF_ESHAPE, "block chain of %d rows a workgroup", rows);
    }
}

}  // namespace

bool chain_width(int D, int mlp_ratio) { return (D == 256 || D == 384 || D == 512) && mlp_ratio <= kChainRatio; }

// Modelled times in us: a round of the chip (256 workgroups) of each form, per launch and, with the attention, per 1000 keys; the block's
// launches one by one without the attention's, at 0 rows and per 1000 rows.  Fitted to whole evaluations of 1 to 64 slots of 16 to 1024
// tokens, e.g. in us per evaluation of 12 blocks one by one | 16 rows with attention | 32 | the best plain form:
//   hidden 256: 256 rows 422 | 323 | 378 | 357, 4096 565 | 342 | 375 | 394, 8192 792 | 583 | 403 | 510, 16384 1114 | 1060 | 739 | 678 (64 rows)
//   hidden 384: 256 rows 408 | 535 | 622 | 560, 1024 488 | 512 | 600 | 539, 2048 591 | 514 | 597 | 554, 6175 (247 tokens a slot) 998 | 1016 | 618 | 683,
//               16384 1756 | 2000 | 1229 | 1129 (64 rows), 64 x 1024 6453 | 10570 | 6773 | 5066 (64 rows)
//   hidden 512: 2048 rows 701 | 829 | 912 | 861, 4096 998 | 875 | 925 | 949, 8192 1367 | 1655 | 1012 | 1063, 64 x 1024 9731 | 16532 | 10265 | 9405 (32 rows)
// With few rows most CUs would idle while each workgroup streams all weights; the hidden units in two or four parts cost a second launch and
// a repeated attention and projection: hidden 384, one launch | two parts | four: 1 x 256 rows 535 | 426 | 382 (one by one 410), 4 x 256 518 |
// 421 | 390 (487), 5 x 247 525 | 431 | 563 (510), 1 x 1024 627 | 528 | 502; hidden 256, 4 x 256 322 | 300 | 288; hidden 512 825 | 625 | 567 (609).
// Fitted while the last block and the first q, k and v were not dealt; now 1 x 256 371, 4 x 256 380, 5 x 247 422, 1 x 1024 493, hidden 256 283,
// hidden 512 550.  At hidden 512 the launches one by one are modelled too long from 2048 rows on (8 x 256 767 us against 707), and two
// parts too short (8 x 256 600 against 689): the choice there is between near equals.
// The models are of ratio 4.  At ratios 1 to 3 both sides shrink: the one-launch forms by 5.0 us a unit of ratio (hidden 384), two parts by
// 0.6 us from 4 to 3 and 5 from 3 to 2, the launches one by one by 0.4 us and 0.65 per 1000 rows.  Over 20 sizes of 1 to 64 slots of 64 to
// 2304 tokens with heads of 32, 64 and 96 no choice at these ratios is slower than one by one beyond the spread of 1 to 2 %.
struct ChainModel { int D; double att16, att16_key, att32, att32_key, plain16, plain32, plain64, two, two_key, four, four_key, apart, apart_row; };
const ChainModel kChainModels[] = {
    { 256, 23.0,  9.5, 27.5, 13.5, 23.0, 29.0, 40.0, 20.3,  9.8, 18.6, 10.8, 27.0, 3.0 },
    { 384, 38.5, 12.0, 44.0, 20.0, 38.5, 45.0, 70.0, 30.6, 11.5, 26.6, 12.9, 25.5, 6.3 },
    { 512, 66.5, 16.0, 78.0, 27.0, 67.0, 77.0, 0.00, 46.0, 15.6, 40.0, 17.0, 36.0, 10.0 },
};

ChainRoute chain_route(int slots, int D, int mlp_ratio, int tokens, int hd)
{
    ChainRoute best{ 0, false, 1, 1 };
    for (const ChainModel& m : kChainModels) {
        if (m.D != D) continue;
        const double rows = (double)slots * tokens, keys = 1e-3 * tokens;
        // the attention's own launch: a base, and its operations or, with few heads, the steps over the keys one after the other
        const double attn = 5.0 + fmax(4.0 * rows * tokens * D / (tokens > 256 ? 0.9e9 : 0.45e9), 0.0235 * (tokens - 256));
        double us = m.apart + m.apart_row * 1e-3 * rows + attn;
        auto consider = [&](int r, bool att, double round) {
            const double tiles = (double)slots * ((tokens + r - 1) / r), t = ceil(tiles / 256.0) * round + (att ? 0.0 : attn);
            if (round > 0.0 && t < us) { us = t; best = ChainRoute{ r, att, 1, 1 }; }
        };
        consider(16, false, m.plain16);
        consider(32, false, m.plain32);
        consider(64, false, m.plain64);
        // (keys and values of a slot are kept in whole groups of 32, in the buffers of q | k | v and of the hidden units)
        if (hd == kChainHead && 2 * ((tokens + 31) / 32 * 32) <= (mlp_ratio < 3 ? mlp_ratio : 3) * tokens) {
            consider(16, true, m.att16 + m.att16_key * keys);
            consider(32, true, m.att32 + m.att32_key * keys);
            // two launches a block, each of all its workgroups at once
            const double tiles = (double)slots * ((tokens + 15) / 16);
            for (int p = 2; p <= 4; p += 2) {
                // Three pieces in two parts take what four take, the launches one by one less: at hidden 512 they are ahead up to 256 keys
                // (us a block, one by one | two parts: 4 x 200 rows 47.9 | 51.2, 4 x 256 48.2 | 50.9, 17 x 32 46.3 | 47.8, 12 x 64 48.2 | 47.4),
                // not beyond, where their attention is another kernel (2 x 400 56.9 | 54.5), nor at hidden 384 (2 x 256 35.4 | 34.2).
                const double uneven = mlp_ratio % p && D == 512 && tokens <= 256 ? 1.05 : 1.0;
                const double t = (p == 2 ? m.two + m.two_key * keys : m.four + m.four_key * keys) * uneven;
                if (p <= mlp_ratio && tiles * p <= 256.0 && t < us) { us = t; best = ChainRoute{ 16, true, p, tiles * 3 <= 256.0 ? 3 : 2 }; }
            }
        }
    }
    return best;
}

float chain_q_scale() { return 1.4426950408889634f / sqrtf((float)kChainHead); }

drf_status launch_chain_pack(const bf16_t* w, int ld, int D, bf16_t* out, hipStream_t st)
{
    hipLaunchKernelGGL(chain_pack_kernel, dim3((unsigned)(D * D / 8 / 256)), dim3(256), 0, st, w, ld, D / 128, D / 32, out);
    DRF_HIP(hipGetLastError());
    return DRF_OK;
}

drf_status launch_block_chain(const ChainArgs& a, int D, int rows, hipStream_t st)
{
    if (a.slots == 0) return DRF_OK;
    if (a.mod_ld % 4 != 0 || !chain_width(D, a.mlp_ratio) || (a.attn && a.kv_in) || (a.qkv && a.kv_out) || ((a.kv_in || a.kv_out) && (a.hd != kChainHead || !a.q || rows > 32)))
        DRF_FAIL(DRF_ESHAPE, "block chain: hidden %d, MLP ratio %d, head width %d", D, a.mlp_ratio, a.hd);
    // parts: of the hidden units, each leaving its share of the stream, or of q, k, v
    if (!a.attn && !a.kv_in && !a.qkv && !a.kv_out && !a.part_in) DRF_FAIL(DRF_EINVAL, "block chain with nothing to do");
    if (a.parts < 1 || (a.parts > 1 && (rows != 16 || (a.kv_in || a.attn ? a.parts > a.mlp_ratio || !a.part_out || a.qkv || a.kv_out : a.parts > 3))) ||
        (a.part_in && (rows != 16 || a.kv_in || a.attn || a.n_in < 1 || a.n_in > kChainRatio)))
        DRF_FAIL(DRF_ESHAPE, "block chain in %d parts", a.parts);
    switch (D) {
    case 256: return a.kv_in ? launch_rows<2, true>(a, rows, st) : launch_rows<2, false>(a, rows, st);
    case 384: return a.kv_in ? launch_rows<3, true>(a, rows, st) : launch_rows<3, false>(a, rows, st);
    default: return a.kv_in ? launch_rows<4, true>(a, rows, st) : launch_rows<4, false>(a, rows, st);
    }
}

}  // namespace drf
