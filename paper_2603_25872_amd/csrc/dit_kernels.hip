// Bandwidth-bound pieces of the DiT forward: conditioning front-end, patch embedding,
// LayerNorm + adaLN modulation, final projection + unpatchify.
#include <type_traits>

#include "common.h"

namespace drf {

namespace {

constexpr int kWave = 64;
constexpr int kTFreq = 256;
typedef float f32x4m __attribute__((ext_vector_type(4)));

// Sum over the 64 lanes with DPP adds (no LDS traffic): inclusive scan inside each row of 16
// lanes (row_shr 1, 2, 4, 8 with zero fill), then the row totals are passed on with
// row_bcast:15 (into rows 1 and 3) and row_bcast:31 (into rows 2 and 3); lane 63 ends with
// the wave total, which readlane hands to every lane.
template <int CTRL, int ROW_MASK>
__device__ inline float dpp_add(float v)
{
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xf, true));
}
__device__ inline float wave_sum(float v)
{
    v = dpp_add<0x111, 0xf>(v);
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);
    v = dpp_add<0x143, 0xc>(v);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

__device__ inline int slot_tau(const SlotMap& m, int slot) { return m.t_dev ? m.t_dev[slot] : m.taus[slot / m.group]; }
__device__ inline int slot_xrow(const SlotMap& m, int slot) { return (slot / m.x_group) * m.x_batch + slot % m.x_batch; }
__device__ inline int slot_crow(const SlotMap& m, int slot) { return m.cond_mod ? slot % m.cond_mod : slot; }

// Conditioning front-end, four small launches:
//   femb(tau) per slot -> Linear + SiLU -> Linear -> add cond embedding, SiLU  (fp32 GEMMs).

// femb[slot][256] = [cos(tau f_i) | sin(tau f_i)], f_i = 10000^(-i/128).  Double precision:
// tau * f reaches ~1e3 rad, beyond what fp32 range reduction keeps to 1e-7.
__global__ void __launch_bounds__(kTFreq / 2) time_features_kernel(const SlotMap map, int slots, float* __restrict__ femb)
{
    const int slot = blockIdx.x, i = threadIdx.x;
    if (slot >= slots) return;
    const double f = exp(-9.210340371976184 * (double)i / (double)(kTFreq / 2));
    const double ang = (double)slot_tau(map, slot) * f;
    femb[(size_t)slot * kTFreq + i] = (float)cos(ang);
    femb[(size_t)slot * kTFreq + kTFreq / 2 + i] = (float)sin(ang);
}

// c = t_emb + cond embedding; writes SiLU(c) as float and, if asked, bf16.
__global__ void __launch_bounds__(256) cond_finish_kernel(const float* __restrict__ temb, const float* __restrict__ vemb,
                                                          const float* __restrict__ table, const int32_t* __restrict__ cls,
                                                          const SlotMap map, int n_classes, int slots, int D,
                                                          float* __restrict__ act_f32, bf16_t* __restrict__ act_bf16)
{
    const int slot = blockIdx.y, j = blockIdx.x * blockDim.x + threadIdx.x;
    if (slot >= slots || j >= D) return;
    float c = temb[(size_t)slot * D + j];
    if (vemb) c += vemb[(size_t)slot * D + j];
    if (table) {
        int k = cls[slot_crow(map, slot)];
        if (k < 0 || k > n_classes) k = n_classes;
        c += table[(size_t)k * D + j];
    }
    const float s = silu(c);
    act_f32[(size_t)slot * D + j] = s;
    if (act_bf16) act_bf16[(size_t)slot * D + j] = (bf16_t)s;
}

// resid[m][j] = sum_k token[m][k] w[j][k] + b[j] + pos[token][j], on the fp32 matrix instruction.  A workgroup takes 16
// tokens and (blockIdx.y) 4 * kPatchTiles tiles of 16 columns, dealt over its four waves; a wave gathers its tokens'
// patches once, in the operand layout (lane: token lane % 16, k = 4 * (lane / 16) + (0..3) of every 16).  Bound by the
// store of the stream: the row-per-thread form, whose weight reads touched 64 lines per instruction, took 25 us for 512
// rows and 44 us for 16384 (hidden 1152), this one 7.6 and 33.5 us.
// VEC: P % 4 == 0 (16-byte loads of the weight rows).
template <bool VEC, int kPatchTiles>
__global__ void __launch_bounds__(256) patch_embed_kernel(const float* __restrict__ x, const SlotMap map,
                                                          const float* __restrict__ w, const float* __restrict__ b,
                                                          const float* __restrict__ pos, const DitDims dm, int M,
                                                          float* __restrict__ resid)
{
    const int lane = threadIdx.x & 63, l16 = lane & 15, quarter = lane >> 4, wave = threadIdx.x >> 6;
    const size_t E = (size_t)dm.C * dm.H * dm.W;
    const int row = blockIdx.x * 16 + l16, m = row < M ? row : M - 1;
    const int slot = m / dm.T, t = m - slot * dm.T, py = t / dm.gw, px = t - py * dm.gw;
    const float* xp = x + (size_t)slot_xrow(map, slot) * E + (size_t)py * dm.patch * dm.W + px * dm.patch;
    const int pp = dm.patch * dm.patch, first = (blockIdx.y * 4 + wave) * kPatchTiles * 16;
    f32x4m acc[kPatchTiles];
#pragma unroll
    for (int i = 0; i < kPatchTiles; ++i) acc[i] = (f32x4m){ 0.f, 0.f, 0.f, 0.f };
    f32x4m code[kPatchTiles];                       // position code, asked for with the operands and not after them
#pragma unroll
    for (int i = 0; i < kPatchTiles; ++i) {
        const int j = first + i * 16 + 4 * quarter, jc = j < dm.D ? j : 0;      // hidden is a multiple of 4
        code[i] = *reinterpret_cast<const f32x4m*>(pos + (size_t)t * dm.D + jc);
    }
    for (int k0 = 0; k0 < dm.P; k0 += 16) {
        f32x4m tok = { 0.f, 0.f, 0.f, 0.f }, wf[kPatchTiles];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = k0 + 4 * quarter + j, ch = k / pp, dy = (k - ch * pp) / dm.patch, dx = k - ch * pp - dy * dm.patch;
            if (k < dm.P) tok[j] = xp[((size_t)ch * dm.H + dy) * dm.W + dx];
        }
#pragma unroll
        for (int i = 0; i < kPatchTiles; ++i) {
            const int j = first + i * 16 + l16, k = k0 + 4 * quarter;
            const float* wr = w + (size_t)(j < dm.D ? j : dm.D - 1) * dm.P;
            wf[i] = (f32x4m){ 0.f, 0.f, 0.f, 0.f };
            if constexpr (VEC) {
                if (k < dm.P) wf[i] = *reinterpret_cast<const f32x4m*>(wr + k);
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (k + u < dm.P) wf[i][u] = wr[k + u];
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int i = 0; i < kPatchTiles; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[i][u], tok[u], acc[i], 0, 0, 0);
    }
    if (row >= M) return;
#pragma unroll
    for (int i = 0; i < kPatchTiles; ++i) {         // acc[i][r]: column first + 16 i + 4 quarter + r of row l16
        const int j = first + i * 16 + 4 * quarter;
        if (j < dm.D) {
            const f32x4m bj = *reinterpret_cast<const f32x4m*>(b + j);
            *reinterpret_cast<f32x4m*>(resid + (size_t)m * dm.D + j) = acc[i] + bj + code[i];
        }
    }
}

// One wave per row; the row stays in registers between the statistics and the output.
// Lanes hold pairs of adjacent columns (8-byte loads, 4- or 8-byte stores); PER pairs per lane.
template <typename OutT> struct Pair;
template <> struct Pair<float> { typedef float2 type; };
template <> struct Pair<bf16_t> { typedef bf16_t type __attribute__((ext_vector_type(2))); };

template <int PER, typename OutT>
__global__ void __launch_bounds__(256) ln_modulate_kernel(float* __restrict__ resid, const bf16_t* __restrict__ add,
                                                          const bf16_t* __restrict__ add2, int write_back,
                                                          const float* __restrict__ shift,
                                                          const float* __restrict__ scale, int mod_ld, int rows_per_slot,
                                                          int M, int D, OutT* __restrict__ out)
{
    typedef typename Pair<OutT>::type out2;
    typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
    const int lane = threadIdx.x & 63, row = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (row >= M) return;
    const int D2 = D >> 1;
    float2* xr = reinterpret_cast<float2*>(resid + (size_t)row * D);
    float2 v[PER];
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int j = i * kWave + lane;
        v[i] = j < D2 ? xr[j] : make_float2(0.f, 0.f);
        if (add && j < D2) {                   // pending branch outputs: x = resid + add (+ add2), stored if asked
            const bf16x2 a2 = reinterpret_cast<const bf16x2*>(add + (size_t)row * D)[j];
            v[i].x += (float)a2.x; v[i].y += (float)a2.y;
            if (add2) {
                const bf16x2 b2 = reinterpret_cast<const bf16x2*>(add2 + (size_t)row * D)[j];
                v[i].x += (float)b2.x; v[i].y += (float)b2.y;
            }
            if (write_back) xr[j] = v[i];
        }
        sum += v[i].x + v[i].y;
    }
    const float mean = wave_sum(sum) / (float)D;
    float sq = 0.f;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int j = i * kWave + lane;
        const float dx = j < D2 ? v[i].x - mean : 0.f, dy = j < D2 ? v[i].y - mean : 0.f;
        sq = fmaf(dx, dx, fmaf(dy, dy, sq));
    }
    const float rstd = rsqrtf(wave_sum(sq) / (float)D + 1e-6f);
    const size_t mrow = (size_t)(row / rows_per_slot) * mod_ld;
    const float2* sh = shift ? reinterpret_cast<const float2*>(shift + mrow) : nullptr;
    const float2* sc = shift ? reinterpret_cast<const float2*>(scale + mrow) : nullptr;
    out2* orow = reinterpret_cast<out2*>(out + (size_t)row * D);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int j = i * kWave + lane;
        if (j < D2) {
            float y0 = (v[i].x - mean) * rstd, y1 = (v[i].y - mean) * rstd;
            if (sh) {
                const float2 s2 = sc[j], h2 = sh[j];
                y0 = fmaf(y0, 1.f + s2.x, h2.x);
                y1 = fmaf(y1, 1.f + s2.y, h2.y);
            }
            out2 o;
            o.x = (OutT)y0; o.y = (OutT)y1;
            orow[j] = o;
        }
    }
}

// Same operation for hidden sizes that are multiples of 128: half a wave per row, 16-byte loads
// of the residual row (PER4 float4 per lane) and 8-byte (bf16) or 16-byte (fp32) stores.
__device__ inline float half_wave_sum(float v)
{
#pragma unroll
    for (int o = 16; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
template <int PER4, typename OutT, int ADD, bool WB>
__global__ void __launch_bounds__(256) ln_modulate4_kernel(float* __restrict__ resid, const bf16_t* __restrict__ add,
                                                           const bf16_t* __restrict__ add2,
                                                           const float* __restrict__ shift,
                                                           const float* __restrict__ scale, int mod_ld, int rows_per_slot,
                                                           int M, OutT* __restrict__ out)
{
    constexpr int D = PER4 * 128;
    typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));
    typedef float f32x4n __attribute__((ext_vector_type(4)));
    const int l32 = threadIdx.x & 31, row = blockIdx.x * (blockDim.x >> 5) + (threadIdx.x >> 5);
    if (row >= M) return;                       // M is even here or the spare half wave idles: no block barrier below
    float4* xr = reinterpret_cast<float4*>(resid + (size_t)row * D);
    float4 v[PER4];
    bf16x4 a4[ADD >= 1 ? PER4 : 1], b4[ADD >= 2 ? PER4 : 1];
#pragma unroll
    for (int i = 0; i < PER4; ++i) {
        // The residual stream and the pending branch outputs are streaming data here: each is next needed a
        // few hundred microseconds and several hundred megabytes of other traffic later, so they are read and
        // written with the non-temporal hint and leave the caches to the activations that the next kernel
        // consumes (the GEMMs of a call run 2 % faster for it, this launch 5 % slower).
        { const f32x4n t4 = __builtin_nontemporal_load(reinterpret_cast<const f32x4n*>(xr) + i * 32 + l32); v[i] = make_float4(t4[0], t4[1], t4[2], t4[3]); }
        if constexpr (ADD >= 1) a4[i] = __builtin_nontemporal_load(&reinterpret_cast<const bf16x4*>(add + (size_t)row * D)[i * 32 + l32]);
        if constexpr (ADD >= 2) b4[i] = __builtin_nontemporal_load(&reinterpret_cast<const bf16x4*>(add2 + (size_t)row * D)[i * 32 + l32]);
    }
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < PER4; ++i) {
        if constexpr (ADD >= 1) {               // pending branch outputs: x = resid + add (+ add2), stored if WB
            v[i].x += (float)a4[i][0]; v[i].y += (float)a4[i][1]; v[i].z += (float)a4[i][2]; v[i].w += (float)a4[i][3];
            if constexpr (ADD >= 2) {
                v[i].x += (float)b4[i][0]; v[i].y += (float)b4[i][1]; v[i].z += (float)b4[i][2]; v[i].w += (float)b4[i][3];
            }
        }
        sum += (v[i].x + v[i].y) + (v[i].z + v[i].w);
    }
    // Every load of the kernel is issued before its first store: loads and stores share one in-order counter, so a
    // load behind a store is only seen once the memory system has taken the store.  The modulation rows are asked
    // for here, all at once, and arrive during the two reductions; the stream's write-back waits until the end.
    // (132-170 registers, two or three waves per SIMD: capping the kernel at 168 or 128 registers for more waves
    // was measured 2 % and 50 % slower for these launches.)
    float4 s4[PER4], h4[PER4];
    if (shift) {
        const size_t mrow = (size_t)(row / rows_per_slot) * mod_ld;
        const float4* sh = reinterpret_cast<const float4*>(shift + mrow);
        const float4* sc = reinterpret_cast<const float4*>(scale + mrow);
#pragma unroll
        for (int i = 0; i < PER4; ++i) { s4[i] = sc[i * 32 + l32]; h4[i] = sh[i * 32 + l32]; }
    } else {
#pragma unroll
        for (int i = 0; i < PER4; ++i) { s4[i] = make_float4(0.f, 0.f, 0.f, 0.f); h4[i] = s4[i]; }
    }
    const float mean = half_wave_sum(sum) * (1.f / (float)D);
    float sq = 0.f;
#pragma unroll
    for (int i = 0; i < PER4; ++i) {
        const float dx = v[i].x - mean, dy = v[i].y - mean, dz = v[i].z - mean, dw = v[i].w - mean;
        sq = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, fmaf(dw, dw, sq))));
    }
    const float rstd = rsqrtf(half_wave_sum(sq) * (1.f / (float)D) + 1e-6f);
#pragma unroll
    for (int i = 0; i < PER4; ++i) {
        const int j = i * 32 + l32;
        float y0 = (v[i].x - mean) * rstd, y1 = (v[i].y - mean) * rstd, y2 = (v[i].z - mean) * rstd, y3 = (v[i].w - mean) * rstd;
        if (shift) {                            // (without modulation y * 1 + 0 would be the same value; kept exact in form)
            y0 = fmaf(y0, 1.f + s4[i].x, h4[i].x); y1 = fmaf(y1, 1.f + s4[i].y, h4[i].y);
            y2 = fmaf(y2, 1.f + s4[i].z, h4[i].z); y3 = fmaf(y3, 1.f + s4[i].w, h4[i].w);
        }
        if constexpr (sizeof(OutT) == 4) {
            reinterpret_cast<float4*>(out + (size_t)row * D)[j] = make_float4(y0, y1, y2, y3);
        } else {
            const bf16x4 o = { (bf16_t)y0, (bf16_t)y1, (bf16_t)y2, (bf16_t)y3 };
            reinterpret_cast<bf16x4*>(out + (size_t)row * D)[j] = o;
        }
        if constexpr (ADD >= 1 && WB) { const f32x4n t4 = { v[i].x, v[i].y, v[i].z, v[i].w }; __builtin_nontemporal_store(t4, reinterpret_cast<f32x4n*>(xr) + i * 32 + l32); }
    }
}

// ln_modulate4_kernel with the output of a split GEMM as the branch to add: the partial tiles are summed here in a fixed
// order instead of by a reduction launch between the GEMM and this one (thin passes: 4.5 us of a 75 us block at 512
// rows), and the branch output takes the rounding that a stored one takes, so that launch by launch a sample's result does not
// depend on the size of the pass it was part of beyond the order of those sums (narrow models round elsewhere in passes that
// block_chain.hip takes: there the branch outputs stay fp32).  Always stores the stream, since the partials do not outlive the
// next split launch.  A workgroup of one wave per row: these launches have few rows (us a launch at two rows a workgroup | one: hidden
// 1152, 250 rows 5.0 | 4.2, 500 5.3 | 4.9, 1000 7.2 | 6.75; 384, 250 3.95 | 3.3, 1000 5.2 | 4.65; four rows: whole evaluations of 256 rows 1604 us against 1583 at two).
template <int D, bool ADD>
__global__ void __launch_bounds__(64) ln_partial_kernel(float* __restrict__ resid, const bf16_t* __restrict__ add, const PartialBranch br,
                                                         const float* __restrict__ shift, const float* __restrict__ scale, int mod_ld,
                                                         int rows_per_slot, bf16_t* __restrict__ out)
{
    constexpr int D4 = D / 4, PER = (D4 + 63) / 64;                  // float4 pieces of a row, pieces per lane
    typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x, row = blockIdx.x;
    f32x4m* xr = reinterpret_cast<f32x4m*>(resid + (size_t)row * D);
    const size_t mrow = (size_t)(row / rows_per_slot) * mod_ld;
    // (a lane without a last piece repeats the row's last one, counts nothing for it and stores nothing)
    auto at = [&](int i) { const int j = i * 64 + lane; return j < D4 ? j : D4 - 1; };
    auto mine = [&](int i) { return i * 64 + lane < D4; };
    f32x4m v[PER], p[PER], g[PER], b[PER];
    bf16x4 a4[ADD ? PER : 1];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        v[i] = xr[at(i)];
        if constexpr (ADD) a4[i] = reinterpret_cast<const bf16x4*>(add + (size_t)row * D)[at(i)];
        p[i] = reinterpret_cast<const f32x4m*>(br.sum.part + (size_t)row * br.sum.ldp)[at(i)];
        g[i] = reinterpret_cast<const f32x4m*>(br.gate + mrow)[at(i)];
        b[i] = reinterpret_cast<const f32x4m*>(br.bias)[at(i)];
    }
    // every partial tile's row is asked for before the first is added: added one by one they were five round trips
    f32x4m more[kMaxSplits - 1][PER];
#pragma unroll
    for (int s = 1; s < kMaxSplits; ++s)
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            more[s - 1][i] = (f32x4m){ 0.f, 0.f, 0.f, 0.f };
            if (s < br.sum.splits) more[s - 1][i] = reinterpret_cast<const f32x4m*>(br.sum.part + s * br.sum.stride + (size_t)row * br.sum.ldp)[at(i)];
        }
    f32x4m s4[PER], h4[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        s4[i] = h4[i] = (f32x4m){ 0.f, 0.f, 0.f, 0.f };
        if (shift) {
            s4[i] = reinterpret_cast<const f32x4m*>(scale + mrow)[at(i)];
            h4[i] = reinterpret_cast<const f32x4m*>(shift + mrow)[at(i)];
        }
    }
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
#pragma unroll
        for (int s = 1; s < kMaxSplits; ++s) p[i] += more[s - 1][i];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (ADD) v[i][j] += (float)a4[i][j];
            v[i][j] += (float)(bf16_t)(g[i][j] * (p[i][j] + b[i][j]));      // rounded as a stored branch output is
        }
        if (mine(i)) sum += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
    }
    const float mean = wave_sum(sum) * (1.f / (float)D);
    float sq = 0.f;
#pragma unroll
    for (int i = 0; i < PER; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) { const float c = mine(i) ? v[i][j] - mean : 0.f; sq = fmaf(c, c, sq); }
    const float rstd = rsqrtf(wave_sum(sq) * (1.f / (float)D) + 1e-6f);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        bf16x4 o;
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = (bf16_t)fmaf((v[i][j] - mean) * rstd, 1.f + s4[i][j], h4[i][j]);
        if (mine(i)) {
            reinterpret_cast<bf16x4*>(out + (size_t)row * D)[at(i)] = o;
            xr[at(i)] = v[i];
        }
    }
}

// Final layer: LN + modulate, Linear(D -> P), scatter to [C][H][W].  A block of 4 waves takes
// kFinalRowsPerBlock token rows; wave w keeps the weights of outputs w, w+4, w+8, w+12 (of each
// group of 16) in registers and sweeps the rows, so nothing but the residual rows is re-read.
constexpr int kFinalRowsPerBlock = 16;
template <int PER>
__global__ void __launch_bounds__(256) final_kernel(const float* __restrict__ resid, const float* __restrict__ shift,
                                                    const float* __restrict__ scale, int mod_ld,
                                                    const float* __restrict__ w, const float* __restrict__ b,
                                                    const DitDims dm, int M, float* __restrict__ eps_out)
{
    const int D = dm.D, P = dm.P;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t E = (size_t)dm.C * dm.H * dm.W;
    const int pp = dm.patch * dm.patch;
    const int row0 = blockIdx.x * kFinalRowsPerBlock, row_end = min(M, row0 + kFinalRowsPerBlock);
    for (int kbase = 0; kbase < P; kbase += 16) {
        float wr[4][PER], bias[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = kbase + wave + 4 * q;
            bias[q] = k < P ? b[k] : 0.f;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int j = i * kWave + lane;
                wr[q][i] = (k < P && j < D) ? w[(size_t)k * D + j] : 0.f;
            }
        }
        for (int row = row0; row < row_end; ++row) {
            const float* xr = resid + (size_t)row * D;
            float v[PER];
            float sum = 0.f;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int j = i * kWave + lane;
                v[i] = j < D ? xr[j] : 0.f;
                sum += v[i];
            }
            const float mean = wave_sum(sum) / (float)D;
            float sq = 0.f;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int j = i * kWave + lane;
                const float dlt = j < D ? v[i] - mean : 0.f;
                sq = fmaf(dlt, dlt, sq);
            }
            const float rstd = rsqrtf(wave_sum(sq) / (float)D + 1e-6f);
            const int slot = row / dm.T, t = row % dm.T, py = t / dm.gw, px = t % dm.gw;
            const size_t mrow = (size_t)slot * mod_ld;
            float acc[4] = { 0.f, 0.f, 0.f, 0.f };
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int j = i * kWave + lane;
                const float y = j < D ? fmaf((v[i] - mean) * rstd, 1.f + scale[mrow + j], shift[mrow + j]) : 0.f;
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[q] = fmaf(y, wr[q][i], acc[q]);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float tot = wave_sum(acc[q]);
                const int k = kbase + wave + 4 * q;
                if (lane == 0 && k < P) {
                    const int ch = k / pp, dy = (k % pp) / dm.patch, dx = k % dm.patch;
                    eps_out[(size_t)slot * E + ((size_t)ch * dm.H + py * dm.patch + dy) * dm.W + px * dm.patch + dx] = tot + bias[q];
                }
            }
        }
    }
}

// Final layer for hidden sizes that are multiples of 64, on the fp32 matrix instruction: a workgroup takes 16 rows, its
// NW waves a share of the columns each (NS steps of 16), a row piece in the operand layout staying in registers
// through the statistics (two exchanges through LDS), the modulation and the product with 16 output weights at a time;
// the waves' partial products are added through LDS.  One chain of loads and no weights staged: with the weights in LDS
// and a row per half wave a launch took 23 us for 512 rows and 42 us for 16384 (hidden 1152, P = 16), four waves 15 and 27 us.
// EARLY: a single round of workgroups is bound by latency, so modulation and the first 16 outputs' weights are asked for together
// with the rows, ahead of the statistics, by eight waves, which have the registers for it (hidden 1152, 512 to 4096 rows:
// 14.5-15.5 -> 8.9-9.5 us; 384, 3072 rows 5.5 -> 4.9; 128, 64 rows 3.2 -> 2.9).  Such a workgroup fills a CU: over several rounds it loses (16384 rows 33.7 us, four waves 27.4).
template <int NS, int NW, bool EARLY>
__global__ void __launch_bounds__(NW * 64) final_mfma_kernel(const float* __restrict__ resid, const float* __restrict__ shift,
                                                             const float* __restrict__ scale, int mod_ld,
                                                             const float* __restrict__ w, const float* __restrict__ b,
                                                             const DitDims dm, int M, float* __restrict__ eps_out)
{
    constexpr int D = NS * NW * 16;
    __shared__ float s_sum[NW][16], s_sq[NW][16];
    __shared__ f32x4m part[NW][64];
    const int lane = threadIdx.x & 63, l16 = lane & 15, quarter = lane >> 4, wave = threadIdx.x >> 6;
    const int m0 = blockIdx.x * 16, row = m0 + l16, m = row < M ? row : M - 1;
    const size_t col0 = (size_t)wave * (NS * 16) + 4 * quarter;
    f32x4m v[NS], w4[NS], s4[NS], h4[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) v[i] = *reinterpret_cast<const f32x4m*>(resid + (size_t)m * D + col0 + i * 16);
    auto load_w = [&](int kbase) {
        const float* wr = w + (size_t)(kbase + l16 < dm.P ? kbase + l16 : dm.P - 1) * D + col0;
#pragma unroll
        for (int i = 0; i < NS; ++i) w4[i] = *reinterpret_cast<const f32x4m*>(wr + i * 16);
    };
    auto load_mod = [&]() {
        const size_t mod = (size_t)(m / dm.T) * mod_ld + col0;
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            s4[i] = *reinterpret_cast<const f32x4m*>(scale + mod + i * 16);
            h4[i] = *reinterpret_cast<const f32x4m*>(shift + mod + i * 16);
        }
    };
    if constexpr (EARLY) {
        load_mod();
        load_w(0);
        __builtin_amdgcn_sched_barrier(0);          // (the loads would otherwise move behind the exchanges)
    }
    // sums of a row over its four lanes, then over the waves
    auto total = [&](float t, float (&over)[NW][16]) {
        t += __shfl_xor(t, 16, 64);
        t += __shfl_xor(t, 32, 64);
        if (quarter == 0) over[wave][l16] = t;
        __syncthreads();
        t = 0.f;
#pragma unroll
        for (int k = 0; k < NW; ++k) t += over[k][l16];
        return t * (1.f / (float)D);
    };
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < NS; ++i) sum += (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]);
    const float mean = total(sum, s_sum);
    float sq = 0.f;
#pragma unroll
    for (int i = 0; i < NS; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) { v[i][j] -= mean; sq = fmaf(v[i][j], v[i][j], sq); }
    const float rstd = rsqrtf(total(sq, s_sq) + 1e-6f);
    if constexpr (!EARLY) load_mod();
#pragma unroll
    for (int i = 0; i < NS; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) v[i][j] = fmaf(v[i][j] * rstd, 1.f + s4[i][j], h4[i][j]);
    const size_t E = (size_t)dm.C * dm.H * dm.W;
    const int pp = dm.patch * dm.patch;
    const int orow = m0 + (threadIdx.x & 15), oslot = orow / dm.T, t = orow - oslot * dm.T, py = t / dm.gw, px = t - py * dm.gw;
    for (int kbase = 0; kbase < dm.P; kbase += 16) {
        if (!EARLY || kbase) load_w(kbase);
        f32x4m acc[2] = { { 0.f, 0.f, 0.f, 0.f }, { 0.f, 0.f, 0.f, 0.f } };
#pragma unroll
        for (int i = 0; i < NS; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[j & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(w4[i][j], v[i][j], acc[j & 1], 0, 0, 0);
        part[wave][lane] = acc[0] + acc[1];         // element r: output kbase + 4 quarter + r of row l16
        __syncthreads();
        const int kk = threadIdx.x >> 4, k = kbase + kk, src = (kk >> 2) * 16 + (threadIdx.x & 15);
        if (kk < 16 && k < dm.P && orow < M) {
            float tot = 0.f;
#pragma unroll
            for (int q = 0; q < NW; ++q) tot += part[q][src][kk & 3];
            const int ch = k / pp, dy = (k % pp) / dm.patch, dx = k % dm.patch;
            eps_out[(size_t)oslot * E + ((size_t)ch * dm.H + py * dm.patch + dy) * dm.W + px * dm.patch + dx] = tot + b[k];
        }
        __syncthreads();
    }
}

__global__ void f32_to_bf16_kernel(const float* __restrict__ in, bf16_t* __restrict__ out, size_t n)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) out[i] = (bf16_t)in[i];
}

}  // namespace

drf_status launch_cond_embed(const CondArgs& a, hipStream_t st)
{
    if (a.slots == 0) return DRF_OK;
    const int D = a.D, S = a.slots;
    // scratch rows: femb [S][256] | h1 [S][D] | temb [S][D] | vemb [S][D]
    float* femb = a.scratch;
    float* h1 = femb + (size_t)S * kTFreq;
    float* temb = h1 + (size_t)S * D;
    float* vemb = temb + (size_t)S * D;
    hipLaunchKernelGGL(time_features_kernel, dim3(S), dim3(kTFreq / 2), 0, st, a.map, S, femb);
    auto linear = [&](const float* x, int K, const float* w, const float* b, float* y, bool act, int row_mod) -> drf_status {
        Epilogue e{};
        e.mode = act ? EPI_STORE_SILU : EPI_STORE; e.out = y; e.ldo = D; e.out_f32 = 1; e.bias = b;
        return launch_gemm_f32(x, w, S, D, K, e, st, row_mod);
    };
    drf_status rc;
    if ((rc = linear(femb, kTFreq, a.t_w1, a.t_b1, h1, true, 0)) != DRF_OK) return rc;
    if ((rc = linear(h1, D, a.t_w2, a.t_b2, temb, false, 0)) != DRF_OK) return rc;
    const bool vec = a.cond_kind == DRF_COND_VECTOR;
    if (vec && (rc = linear((const float*)a.cond, a.cond_dim, a.c_w, a.c_b, vemb, false, a.map.cond_mod)) != DRF_OK) return rc;
    const bool cls = a.cond_kind == DRF_COND_CLASS;
    hipLaunchKernelGGL(cond_finish_kernel, dim3((D + 255) / 256, S), dim3(256), 0, st, temb, vec ? vemb : nullptr,
                       cls ? a.table : nullptr, cls ? (const int32_t*)a.cond : nullptr, a.map, a.cond_dim, S, D,
                       a.act_f32, a.act_bf16);
    DRF_HIP(hipGetLastError());
    return DRF_OK;
}

drf_status launch_patch_embed(const float* x, const SlotMap& map, const float* w, const float* b, const float* pos,
                              const DitDims& dm, int slots, float* resid, hipStream_t st)
{
    const int M = slots * dm.T;
    if (M == 0) return DRF_OK;
    auto go = [&](auto tiles_c) {
        constexpr int TILES = decltype(tiles_c)::value, per = 4 * TILES * 16;
        const dim3 grid((M + 15) / 16, (dm.D + per - 1) / per);
        if (dm.P % 4 == 0 && (reinterpret_cast<uintptr_t>(w) & 15u) == 0)
            hipLaunchKernelGGL((patch_embed_kernel<true, TILES>), grid, dim3(256), 0, st, x, map, w, b, pos, dm, M, resid);
        else
            hipLaunchKernelGGL((patch_embed_kernel<false, TILES>), grid, dim3(256), 0, st, x, map, w, b, pos, dm, M, resid);
    };
    // Two column tiles a wave or six.  Six gather the patches once for 24 tiles, two put more workgroups on the chip and waste less of a
    // last group: where a third of the six-tile groups' columns are padding, two are the faster form at every size (us, two against
    // six: hidden 128 4.5 : 5.6 at 4096 rows, 14.9 : 19.1 at 24576; 256 14.8 : 16.8 at 16384; 512 9.1 : 9.3 and 25.8 : 28.0), otherwise up
    // to about 2.2 million elements of the stream (384: 9.0 : 9.6 at 5120 rows, 10.3 : 10.1 at 6144, 12.6 : 11.5 at 8192; 640: 8.9 : 9.4 at 3072,
    // 10.5 : 10.0 at 4096; 768: 7.7 : 8.3 at 2048, 9.6 : 9.4 at 3072, 14.4 : 13.4 at 8192; 1152: 6.3 : 6.9 at 1024, 8.1 : 8.2 at 2048,
    // 10.8 : 10.6 at 3328, 12.0 : 11.1 at 4096, 36.9 : 34.4 at 16384; 1536: 6.0 : 6.6 at 1024, 9.1 : 8.2 at 2048).
    const int tiles = (dm.D + 15) / 16, padded = (tiles + 23) / 24 * 24;
    if (3 * tiles <= 2 * padded || (long long)M * dm.D < 2200000) go(std::integral_constant<int, 2>{});
    else go(std::integral_constant<int, 6>{});
    DRF_HIP(hipGetLastError());
    return DRF_OK;
}

template <int PER>
static void launch_ln_inst(float* resid, const bf16_t* add, const bf16_t* add2, int write_back, const float* shift, const float* scale,
                           int mod_ld, int rows_per_slot, int M, int D, void* out, int out_f32, hipStream_t st)
{
    const dim3 grid((M + 3) / 4), block(256);
    if (out_f32)
        hipLaunchKernelGGL((ln_modulate_kernel<PER, float>), grid, block, 0, st, resid, add, add2, write_back, shift, scale, mod_ld,
                           rows_per_slot, M, D, (float*)out);
    else
        hipLaunchKernelGGL((ln_modulate_kernel<PER, bf16_t>), grid, block, 0, st, resid, add, add2, write_back, shift, scale, mod_ld,
                           rows_per_slot, M, D, (bf16_t*)out);
}

template <int PER4>
void launch_ln4_inst(float* resid, const bf16_t* add, const bf16_t* add2, int write_back, const float* shift, const float* scale,
                     int mod_ld, int rows_per_slot, int M, void* out, int out_f32, hipStream_t st)
{
    // Rows a workgroup: eight, four up to 5120 rows and two up to 1024, so that few rows still reach all CUs and leave no round in part.
    // Times of a launch, us, eight | that many, one pending branch, then two: hidden 1152, 500 rows 4.9 | 4.4; 1000 5.3 | 4.85; 2250 9.5 |
    // 8.8, 10.2 | 9.05; 3000 9.85 | 9.25, 11.2 | 10.0; 4000 10.6 | 10.4, 12.9 | 13.0; 6000 at four rows 12.15 | 12.4, 18.4 | 18.75.  768: 3000 8.05 |
    // 7.55, 8.0 | 7.2; 4000 8.65 | 8.55, 9.3 | 9.6; 6000 even.  384: 2250 4.5 | 4.3, 4.7 | 4.65; 4000 4.95 | 4.95, 5.2 | 5.5; 6000 6.5 | 6.65, 7.2 |
    // 7.6.  128: within 0.1 at all of these.  Whole evaluations of six blocks at eight | four rows: 4608 rows of 384, 768, 1024, 1152
    // 453 | 451, 757 | 751, 1207 | 1199, 1392 | 1386; 5120 489 | 485, 775 | 771, 1250 | 1241, 1423 | 1420; 5632 513 | 514, 957 | 957, 1320 | 1320,
    // 1522 | 1525; 6144 521 | 521, 1023 | 1025, 1391 | 1395, 1571 | 1575.
    const int rows = M <= 1024 ? 2 : M <= 5120 ? 4 : 8;
    const dim3 grid((M + rows - 1) / rows), block(rows * 32);
#define DRF_LN4(OUT, ADD, WB) \
    hipLaunchKernelGGL((ln_modulate4_kernel<PER4, OUT, ADD, WB>), grid, block, 0, st, resid, add, add2, shift, scale, mod_ld, \
                       rows_per_slot, M, (OUT*)out)
    if (out_f32) DRF_LN4(float, 0, false);
    else if (!add) DRF_LN4(bf16_t, 0, false);
    else if (!add2 && write_back) DRF_LN4(bf16_t, 1, true);
    else if (!add2) DRF_LN4(bf16_t, 1, false);
    else if (write_back) DRF_LN4(bf16_t, 2, true);
    else DRF_LN4(bf16_t, 2, false);
#undef DRF_LN4
}

drf_status launch_ln_modulate(float* resid, const bf16_t* add, const bf16_t* add2, bool write_back, const float* shift,
                              const float* scale, int mod_ld, int rows_per_slot, int M, int D, void* out, int out_f32,
                              hipStream_t st)
{
    if (M == 0) return DRF_OK;
    if (add && out_f32) DRF_FAIL(DRF_ESHAPE, "the pending-branch add is a bf16-path feature");
    if (add2 && !add) DRF_FAIL(DRF_EINVAL, "a second pending branch output needs a first one");
    if (D > 2048 || D % 2 != 0 || mod_ld % 2 != 0) DRF_FAIL(DRF_ESHAPE, "LayerNorm kernel needs even hidden <= 2048 (got %d)", D);
    const int wb = write_back ? 1 : 0;
    const bool al16 = mod_ld % 4 == 0 && ((reinterpret_cast<uintptr_t>(resid) | reinterpret_cast<uintptr_t>(out) |
                                           reinterpret_cast<uintptr_t>(shift) | reinterpret_cast<uintptr_t>(scale) |
                                           reinterpret_cast<uintptr_t>(add) | reinterpret_cast<uintptr_t>(add2)) & 15u) == 0;
    if (al16 && (D == 1152 || D == 384 || D == 768 || D == 1024 || D == 128)) {
        switch (D / 128) {
        case 1: launch_ln4_inst<1>(resid, add, add2, wb, shift, scale, mod_ld, rows_per_slot, M, out, out_f32, st); break;
        case 3: launch_ln4_inst<3>(resid, add, add2, wb, shift, scale, mod_ld, rows_per_slot, M, out, out_f32, st); break;
        case 6: launch_ln4_inst<6>(resid, add, add2, wb, shift, scale, mod_ld, rows_per_slot, M, out, out_f32, st); break;
        case 8: launch_ln4_inst<8>(resid, add, add2, wb, shift, scale, mod_ld, rows_per_slot, M, out, out_f32, st); break;
        default: launch_ln4_inst<9>(resid, add, add2, wb, shift, scale, mod_ld, rows_per_slot, M, out, out_f32, st); break;
        }
        DRF_HIP(hipGetLastError());
        return DRF_OK;
    }
    const int per = (D / 2 + kWave - 1) / kWave;      // column pairs per lane
    if (per <= 1) launch_ln_inst<1>(resid, add, add2, wb, shift, scale, mod_ld, rows_per_slot, M, D, out, out_f32, st);
    else if (per <= 3) launch_ln_inst<3>(resid, add, add2, wb, shift, scale, mod_ld, rows_per_slot, M, D, out, out_f32, st);
    else if (per <= 5) launch_ln_inst<5>(resid, add, add2, wb, shift, scale, mod_ld, rows_per_slot, M, D, out, out_f32, st);
    else if (per <= 9) launch_ln_inst<9>(resid, add, add2, wb, shift, scale, mod_ld, rows_per_slot, M, D, out, out_f32, st);
    else launch_ln_inst<16>(resid, add, add2, wb, shift, scale, mod_ld, rows_per_slot, M, D, out, out_f32, st);
    DRF_HIP(hipGetLastError());
    return DRF_OK;
}

bool ln_partial_width(int D) { return D == 128 || D == 384 || D == 768 || D == 1024 || D == 1152; }

drf_status launch_ln_modulate_partial(float* resid, const bf16_t* add, const PartialBranch& br, const float* shift, const float* scale,
                                      int mod_ld, int rows_per_slot, int M, int D, bf16_t* out, hipStream_t st)
{
    if (M == 0) return DRF_OK;
    if (!ln_partial_width(D) || mod_ld % 4 != 0 || br.sum.ldp % 4 != 0 || br.sum.splits < 1 || br.sum.splits > kMaxSplits) DRF_FAIL(DRF_ESHAPE, "LayerNorm of partial tiles: hidden %d", D);
    const dim3 grid(M), block(64);
    auto go = [&](auto with, auto without) -> drf_status {
        if (add) hipLaunchKernelGGL(with, grid, block, 0, st, resid, add, br, shift, scale, mod_ld, rows_per_slot, out);
        else hipLaunchKernelGGL(without, grid, block, 0, st, resid, add, br, shift, scale, mod_ld, rows_per_slot, out);
        DRF_HIP(hipGetLastError());
        return DRF_OK;
    };
    switch (D) {
    case 128: return go(ln_partial_kernel<128, true>, ln_partial_kernel<128, false>);
    case 384: return go(ln_partial_kernel<384, true>, ln_partial_kernel<384, false>);
    case 768: return go(ln_partial_kernel<768, true>, ln_partial_kernel<768, false>);
    case 1024: return go(ln_partial_kernel<1024, true>, ln_partial_kernel<1024, false>);
    default: return go(ln_partial_kernel<1152, true>, ln_partial_kernel<1152, false>);
    }
}

drf_status launch_final(const float* resid, const float* shift, const float* scale, int mod_ld, const float* w,
                        const float* b, const DitDims& dm, int slots, float* eps_out, hipStream_t st)
{
    const int M = slots * dm.T;
    if (M == 0) return DRF_OK;
    if (dm.D > 2048) DRF_FAIL(DRF_ESHAPE, "final layer needs hidden <= 2048");
    const bool al16 = mod_ld % 4 == 0 && ((reinterpret_cast<uintptr_t>(resid) | reinterpret_cast<uintptr_t>(shift) |
                                           reinterpret_cast<uintptr_t>(scale) | reinterpret_cast<uintptr_t>(w)) & 15u) == 0;
    if (al16) {
        auto go = [&](auto ns_c) -> drf_status {    // ns: column steps of a wave, of four
            constexpr int NS = decltype(ns_c)::value;
            const dim3 groups((M + 15) / 16);
            if constexpr (NS % 2 == 0) {
                if (groups.x <= 256) {
                    hipLaunchKernelGGL((final_mfma_kernel<NS / 2, 8, true>), groups, dim3(512), 0, st, resid, shift, scale, mod_ld, w, b, dm, M, eps_out);
                    DRF_HIP(hipGetLastError());
                    return DRF_OK;
                }
            }
            hipLaunchKernelGGL((final_mfma_kernel<NS, 4, false>), groups, dim3(256), 0, st, resid, shift, scale, mod_ld, w, b, dm, M, eps_out);
            DRF_HIP(hipGetLastError());
            return DRF_OK;
        };
        switch (dm.D) {
        case 128: return go(std::integral_constant<int, 2>{});
        case 384: return go(std::integral_constant<int, 6>{});
        case 576: return go(std::integral_constant<int, 9>{});
        case 768: return go(std::integral_constant<int, 12>{});
        case 1024: return go(std::integral_constant<int, 16>{});
        case 1152: return go(std::integral_constant<int, 18>{});
        default: break;
        }
    }
    const dim3 grid((M + kFinalRowsPerBlock - 1) / kFinalRowsPerBlock), block(256);
    const int per = (dm.D + kWave - 1) / kWave;
    if (per <= 6) hipLaunchKernelGGL(final_kernel<6>, grid, block, 0, st, resid, shift, scale, mod_ld, w, b, dm, M, eps_out);
    else if (per <= 18) hipLaunchKernelGGL(final_kernel<18>, grid, block, 0, st, resid, shift, scale, mod_ld, w, b, dm, M, eps_out);
    else hipLaunchKernelGGL(final_kernel<32>, grid, block, 0, st, resid, shift, scale, mod_ld, w, b, dm, M, eps_out);
    DRF_HIP(hipGetLastError());
    return DRF_OK;
}

drf_status launch_f32_to_bf16(const float* in, bf16_t* out, size_t n, hipStream_t st)
{
    if (n == 0) return DRF_OK;
    size_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(f32_to_bf16_kernel, dim3((unsigned)blocks), dim3(256), 0, st, in, out, n);
    DRF_HIP(hipGetLastError());
    return DRF_OK;
}

}  // namespace drf
