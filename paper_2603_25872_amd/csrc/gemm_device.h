// Device code shared by the GEMM kernels: epilogue arithmetic, hand-written LDS reads and waits, the store of a wave's tile.
#pragma once
#include <type_traits>

#include "common.h"

namespace drf {

namespace {

typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));

// GELU (tanh form): 0.5 x (1 + tanh(u)) = x * sigmoid(2u), u = sqrt(2/pi) (x + 0.044715 x^3).
// One exp2 and one reciprocal (both hardware transcendental ops, ~1 ulp).
__device__ inline float gelu_tanh(float x)
{
    const float t = x * x;
    const float m2u_log2e = x * fmaf(t, -0.1029432f, -2.3022082f);   // -2 u log2(e)
    return x * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(m2u_log2e));
}

// floor(n / d) for 0 <= n < 2^31 with a host-made magic number (d >= 1).
__device__ inline int fast_div(int n, uint32_t magic, int shift)
{
    return magic ? (int)(__umulhi((uint32_t)n, magic) >> shift) : (n >> shift);
}

// Element offset of (row m, column n) in the head-major q | k | v planes (n is a multiple of 4 or 8
// and the head width a multiple of 8, so a vector never straddles a head).
__device__ inline size_t heads_offset(const Epilogue& e, int m, int n)
{
    const int which = fast_div(n, e.hid_magic, e.hid_shift), c = n - which * e.hid;
    const int head = fast_div(c, e.hd_magic, e.hd_shift), dd = c - head * e.hd;
    const int slot = fast_div(m, e.rps_magic, e.rps_shift), t = m - slot * e.rows_per_slot;
    return (size_t)which * e.plane + ((size_t)(slot * e.heads + head) * e.rows_per_slot + t) * e.hd + dd;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
#define DRF_GLOBAL_AS __attribute__((address_space(1)))
#define DRF_LDS_AS __attribute__((address_space(3)))
template <int N> __device__ inline void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
template <int N> __device__ inline void wait_lgkmcnt() { asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory"); }
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// 16 bytes per lane from LDS byte address addr + OFF, asynchronously: dst is valid only after an
// s_waitcnt lgkmcnt that covers it.
template <int OFF> __device__ inline void lds_read16(u32x4& dst, uint32_t addr)
{
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF));
}
// Waits until at most N LDS reads are outstanding.  The fragments that the following MFMAs consume
// pass through the statement as in/out operands, so no use of them can be scheduled above the wait.
template <int N> __device__ inline void wait_frag(u32x4& w) { asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(w) : "n"(N)); }
// Keeps a fragment's registers its own up to this point.
__device__ inline void hold_frag(u32x4& w) { asm volatile("" : "+v"(w)); }
template <int N, int MI> __device__ inline void wait_frags(u32x4& w, u32x4 (&a)[MI])
{
    static_assert(MI == 2 || MI == 4, "activation fragments per k-step");
    if constexpr (MI == 2) asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(w), "+v"(a[0]), "+v"(a[1]) : "n"(N));
    else asm volatile("s_waitcnt lgkmcnt(%5)" : "+v"(w), "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]) : "n"(N));
}
// c += w . a on the matrix unit, the accumulator's register file named: where it is left to the compiler, it has moved whole
// sets of accumulators between the two files in every k-tile (128 x 96 tile: 47.8 instead of 37.4 us).  The compiler knows nothing
// of the instruction's latency: before the first one, a hold_acc() of every accumulator and settle_mfma() (their zeros are
// written); after the last one, settle_mfma() and a hold_acc() of each (their results are read).
template <bool AGPR> __device__ __forceinline__ void mfma(f32x4& c, const u32x4& w, const u32x4& a)
{
    if constexpr (AGPR) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(w), "v"(a));
    else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(w), "v"(a));
}
template <bool AGPR> __device__ __forceinline__ void hold_acc(f32x4& c)
{
    if constexpr (AGPR) asm volatile("" : "+a"(c));
    else asm volatile("" : "+v"(c));
}

__device__ inline void settle_mfma() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }

template <int I, int N, typename F> __device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// Rows of epilogue operands that a workgroup keeps in LDS behind its stages: the bias of its columns, then the gate rows
// of the slots that its rows belong to (up to kGateRows; beyond, gates are read from global memory).  They are copied
// between the first stage and the second, so the wait for the first covers them and the epilogue meets no memory round trip.
constexpr int kGateRows = 4;
__host__ __device__ constexpr int epi_row_bytes(int BN) { return (BN + 63) / 64 * 256; }
__host__ __device__ constexpr int epi_lds_bytes(int BN) { return (1 + kGateRows) * epi_row_bytes(BN); }

struct GateRows { int slot0, rows; };               // first slot of the workgroup's rows; rows in LDS (0: none)
template <int BM> __device__ inline GateRows gate_rows(const Epilogue& e, int m0, int M)
{
    if (!e.gate) return { 0, 0 };
    const int last = m0 + BM < M ? m0 + BM - 1 : M - 1;
    const int s0 = fast_div(m0, e.rps_magic, e.rps_shift), s1 = fast_div(last, e.rps_magic, e.rps_shift);
    return { s0, s1 - s0 < kGateRows ? s1 - s0 + 1 : 0 };
}
// Copies those rows (4 bytes per lane: no alignment beyond a float's is asked of bias and gate).
template <int BN> __device__ inline void stage_epilogue_rows(const Epilogue& e, const GateRows& gr, uint32_t lds, int wave, int n_waves, int n0, int N)
{
    constexpr int PIECES = (BN + 63) / 64;
    const int lane = threadIdx.x & 63;
    for (int r = wave; r < 1 + gr.rows; r += n_waves) {
        const float* src = r == 0 ? e.bias : e.gate + (size_t)(gr.slot0 + r - 1) * e.gate_ld;
#pragma unroll
        for (int c = 0; c < PIECES; ++c) {
            int n = n0 + c * 64 + lane;
            n = n < N ? n : N - 1;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                         :: "s"(lds + (uint32_t)(r * epi_row_bytes(BN) + c * 256)), "v"((uint32_t)n * 4u), "s"(src) : "memory");
        }
    }
}

// Cache warm-up for a later launch (see Epilogue::warm): the lines are dealt over the workgroups of the last round, one word
// per line and lane, into 256 bytes of LDS that nobody reads (a register destination would be waited for: with it the
// prologue took the time of its stages and of these lines from HBM).  Whoever calls it waits for vmcnt 0 once before
// its workgroup ends: nothing may land in LDS after that.
__device__ inline void warm_caches(const Epilogue& e, uint32_t lds, int nb, int b, int wave, int n_waves)
{
    if (!e.warm_lines) return;
    const uint32_t first = nb > 256 ? (uint32_t)nb - 256u : 0u, cnt = (uint32_t)nb - first;
    const uint32_t per = (e.warm_lines + cnt - 1u) / cnt;
    if ((uint32_t)b < first) return;
    for (uint32_t t = (uint32_t)wave * 64u; t < per; t += (uint32_t)n_waves * 64u) {
        uint32_t line = ((uint32_t)b - first) * per + t + (threadIdx.x & 63u);
        line = line < e.warm_lines ? line : e.warm_lines - 1u;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" :: "s"(lds), "v"(line * 128u), "s"(e.warm) : "memory");
    }
}

// Epilogue of a wave's tile of TM x TN from its accumulators, acc[i][j][r] being (m = j*16 + l16, n = i*16 + 4*quarter + r).
// bf16: a lane's four columns of two neighbouring pieces are exchanged between the quarters of the wave (two lane swaps),
// after which every lane holds 16 bytes of one row and a store covers 64 bytes of each of 16 rows.  Launches of one short
// round gain 0.2-0.5 us on the way through LDS (512 x 1152 x 1152: 6.9 -> 6.5 us, 1024 x 384 x 384: 4.2 -> 3.9); where the chip
// is full, store_rows is the better one.
// EDGES_ONLY: every piece is checked against M and N, also where the whole tile is inside (less code).
// erows: this wave's columns of the workgroup's bias row in LDS, the gate rows behind it, `rstride` bytes apart.
template <int TM, int TN, int MODE, bool F32, bool EDGES_ONLY = false>
__device__ __forceinline__ void store_tile_as(const f32x4 (&acc)[TN / 16][TM / 16], const Epilogue& e, int mw, int nw, int M, int N,
                                              const unsigned char* erows, int rstride, const GateRows& gr, int lane)
{
    constexpr int MI = TM / 16, NI = TN / 16;
    static_assert(MI % 2 == 0, "pieces are paired");
    const int l16 = lane & 15, quarter = lane >> 4, odd = quarter & 1;
    const bool inside = mw + TM <= M && nw + TN <= N;
    const float* gate_lds = reinterpret_cast<const float*>(erows + rstride);
    // GATE: 0 none | 1 one row in LDS | 2 several rows in LDS | 3 global memory
    auto run = [&](auto gate_c, auto inside_c) {
        constexpr int GATE = decltype(gate_c)::value;
        constexpr bool IN = decltype(inside_c)::value;
        int gofs[MI];                               // gate row of this lane's row j: floats from gate_lds / from e.gate's slot row
#pragma unroll
        for (int j = 0; j < MI; ++j) {
            int m = mw + j * 16 + l16;
            m = IN || m < M ? m : M - 1;
            if constexpr (GATE == 2) gofs[j] = (fast_div(m, e.rps_magic, e.rps_shift) - gr.slot0) * (rstride / 4);
            else if constexpr (GATE == 3) gofs[j] = fast_div(m, e.rps_magic, e.rps_shift);
            else gofs[j] = 0;
        }
        auto gate_at = [&](int i, int j) -> f32x4 {
            const int c = i * 16 + 4 * quarter;
            if constexpr (GATE == 3) return *reinterpret_cast<const f32x4*>(e.gate + (size_t)gofs[j] * e.gate_ld + (IN || nw + c < N ? nw + c : 0));
            else return *reinterpret_cast<const f32x4*>(gate_lds + gofs[j] + c);
        };
        auto bias_at = [&](int i) -> f32x4 { return *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(erows) + i * 16 + 4 * quarter); };
        // the epilogue's arithmetic on piece (i, j); b: bias, g: the gate where it is the same for all rows
        auto value = [&](int i, int j, const f32x4& b, const f32x4& g) -> f32x4 {
            f32x4 v = acc[i][j] + b;
            if constexpr (MODE == EPI_STORE_GELU) { v[0] = gelu_tanh(v[0]); v[1] = gelu_tanh(v[1]); v[2] = gelu_tanh(v[2]); v[3] = gelu_tanh(v[3]); }
            if constexpr (MODE == EPI_STORE_HEADS) v *= nw + i * 16 < e.hid ? e.q_scale : 1.f;     // hid is a multiple of 16
            if constexpr (MODE == EPI_STORE_GATED) {
                if constexpr (GATE == 1) v *= g; else v *= gate_at(i, j);
            }
            return v;
        };
        if constexpr (F32) {
            float* op = (float*)e.out + (size_t)(mw + l16) * e.ldo + nw + 4 * quarter;
            auto ok = [&](int i, int j) { return IN || (mw + j * 16 + l16 < M && nw + i * 16 + 4 * quarter < N); };
            f32x4 x[2][MODE == EPI_RESID ? MI : 1];
            auto fetch_x = [&](int i) {
                if constexpr (MODE == EPI_RESID) {
#pragma unroll
                    for (int j = 0; j < MI; ++j)
                        if (ok(i, j)) x[i & 1][j] = *reinterpret_cast<const f32x4*>(op + (size_t)j * 16 * e.ldo + i * 16);
                }
            };
            fetch_x(0);
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                if (i + 1 < NI) fetch_x(i + 1);     // asked for ahead of this piece's stores
                __builtin_amdgcn_sched_barrier(0);
                const f32x4 b = bias_at(i);
                f32x4 g = { 1.f, 1.f, 1.f, 1.f };
                if constexpr (GATE == 1) g = gate_at(i, 0);
#pragma unroll
                for (int j = 0; j < MI; ++j) {
                    f32x4 v = value(i, j, b, g);
                    if constexpr (MODE == EPI_RESID) {
                        if constexpr (GATE >= 2) g = gate_at(i, j);
                        if (ok(i, j)) {
                            f32x4 y = x[i & 1][j];
                            y[0] = fmaf(g[0], v[0], y[0]); y[1] = fmaf(g[1], v[1], y[1]); y[2] = fmaf(g[2], v[2], y[2]); y[3] = fmaf(g[3], v[3], y[3]);
                            v = y;
                        }
                    }
                    if (ok(i, j)) *reinterpret_cast<f32x4*>(op + (size_t)j * 16 * e.ldo + i * 16) = v;
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        } else {
            // element offset of a row, and of a column relative to its row
            size_t rofs[MI];
#pragma unroll
            for (int j = 0; j < MI; ++j) {
                const int m = mw + j * 16 + l16;
                if constexpr (MODE == EPI_STORE_HEADS) {
                    const int slot = fast_div(m, e.rps_magic, e.rps_shift);
                    rofs[j] = ((size_t)slot * e.heads * e.rows_per_slot + (m - slot * e.rows_per_slot)) * e.hd;
                } else rofs[j] = (size_t)m * e.ldo;
            }
            auto cofs = [&](int n) -> size_t {
                if constexpr (MODE == EPI_STORE_HEADS) {
                    const int which = fast_div(n, e.hid_magic, e.hid_shift), c = n - which * e.hid, head = fast_div(c, e.hd_magic, e.hd_shift);
                    return (size_t)which * e.plane + (size_t)head * e.rows_per_slot * e.hd + (c - head * e.hd);
                } else return (size_t)n;
            };
            auto packed = [&](const f32x4& v, uint32_t (&p)[2]) {
                const bf16x4 o = { (bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3] };
                const uint2 u = __builtin_bit_cast(uint2, o);
                p[0] = u.x; p[1] = u.y;
            };
            // after the swap: even quarters hold the first piece's columns 0..7 (quarter 0) and 8..15 (2), odd ones the second's
            auto swap_store = [&](uint32_t (&d)[2], uint32_t (&s)[2], size_t ofs, bool row_ok, int n) {
                const auto r0 = __builtin_amdgcn_permlane16_swap(d[0], s[0], false, false);
                const auto r1 = __builtin_amdgcn_permlane16_swap(d[1], s[1], false, false);
                const u32x4 v = { r0[0], r1[0], r0[1], r1[1] };
                bf16_t* p = (bf16_t*)e.out + ofs;
                if (IN || (row_ok && n + 8 <= N)) *reinterpret_cast<u32x4*>(p) = v;
                else if (row_ok && n < N) *reinterpret_cast<uint2*>(p) = make_uint2(v[0], v[1]);       // N is a multiple of 4: half a chunk
            };
#pragma unroll
            for (int i = 0; i + 1 < NI; i += 2) {
                const f32x4 b0 = bias_at(i), b1 = bias_at(i + 1);
                f32x4 g0 = b0, g1 = b1;
                if constexpr (GATE == 1) { g0 = gate_at(i, 0); g1 = gate_at(i + 1, 0); }
                const int n = nw + (i + odd) * 16 + (quarter >> 1) * 8;
                const size_t co = cofs(n);
#pragma unroll
                for (int j = 0; j < MI; ++j) {
                    uint32_t d[2], s[2];
                    packed(value(i, j, b0, g0), d);
                    packed(value(i + 1, j, b1, g1), s);
                    swap_store(d, s, rofs[j] + co, mw + j * 16 + l16 < M, n);
                    __builtin_amdgcn_sched_barrier(0);      // (pieces computed far ahead of their stores would spill)
                }
            }
            if constexpr (NI % 2 == 1) {            // the last piece pairs with itself 16 rows further down
                constexpr int i = NI - 1;
                const f32x4 b = bias_at(i);
                f32x4 g = b;
                if constexpr (GATE == 1) g = gate_at(i, 0);
                const int n = nw + i * 16 + (quarter >> 1) * 8;
                const size_t co = cofs(n);
#pragma unroll
                for (int j = 0; j < MI; j += 2) {
                    uint32_t d[2], s[2];
                    packed(value(i, j, b, g), d);
                    packed(value(i, j + 1, b, g), s);
                    swap_store(d, s, (odd ? rofs[j + 1] : rofs[j]) + co, mw + (j + odd) * 16 + l16 < M, n);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    };
    auto pick = [&](auto gate_c) {
        if constexpr (!EDGES_ONLY) {
            if (inside) { run(gate_c, std::true_type{}); return; }
        }
        run(gate_c, std::false_type{});
    };
    if (MODE == EPI_STORE_GATED || (MODE == EPI_RESID && e.gate)) {
        if (gr.rows == 1) pick(std::integral_constant<int, 1>{});
        else if (gr.rows > 1) pick(std::integral_constant<int, 2>{});
        else pick(std::integral_constant<int, 3>{});
    } else pick(std::integral_constant<int, 0>{});
}

// The same for a whole tile with bf16 results, in whole rows: transposed through LDS of the wave's own (wbuf,
// rows_tile_bytes), 32 rows at a time, a store instruction covering 1 KB of consecutive 16-byte pieces of the rows.  For
// launches that fill the chip, where the lane-swapped stores of 64-byte pieces cost the memory system 2-3 us a round more
// (128 x 144 per wave, 256 CUs: 6.2-7.0 us against 4.0; with an address computed per store 5.9): bias and gate stay in
// registers, and the offsets of a pass of 32 rows are those of every pass.  GATE: 0 none | 1 one gate row in LDS.
// HEADS: the rows of a pass belong to one slot, and offsets stay below 2^32 bytes.
__host__ __device__ constexpr int rows_pitch(int TN) { return TN * 2 + 16; }     // 16 rows of 8-byte writes on distinct banks
__host__ __device__ constexpr int rows_tile_bytes(int TM, int TN) { return TM * rows_pitch(TN); }
template <int TM, int TN, int MODE, int GATE>
__device__ __forceinline__ void store_rows(const f32x4 (&acc)[TN / 16][TM / 16], const Epilogue& e, int mw, int nw, unsigned char* wbuf,
                                           const unsigned char* erows, int rstride)
{
    constexpr int NI = TN / 16, PITCH = rows_pitch(TN), CH = TN / 8, U = 32 * CH / 64;
    static_assert(TM % 32 == 0 && 32 * CH % 64 == 0, "passes of 32 rows");
    const int lane = threadIdx.x & 63, l16 = lane & 15, quarter = lane >> 4;
    f32x4 bias[NI], gate[GATE ? NI : 1];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        bias[i] = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(erows) + i * 16 + 4 * quarter);
        if constexpr (GATE) gate[i] = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(erows + rstride) + i * 16 + 4 * quarter);
    }
    uint32_t lo[U], go[U];                          // this lane's pieces of a pass: bytes in LDS, bytes from the pass's first row
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int id = lane + u * 64, r = id / CH, c = id - r * CH, n = nw + c * 8;
        lo[u] = (uint32_t)(r * PITCH + c * 16);
        if constexpr (MODE == EPI_STORE_HEADS) {
            const int which = fast_div(n, e.hid_magic, e.hid_shift), cc = n - which * e.hid, head = fast_div(cc, e.hd_magic, e.hd_shift);
            go[u] = (uint32_t)(which * e.plane + (size_t)(head * e.rows_per_slot + r) * e.hd + (cc - head * e.hd)) * 2u;
        } else go[u] = (uint32_t)(r * e.ldo + n) * 2u;
    }
    unsigned char* wrow = wbuf + l16 * PITCH + quarter * 8;
    auto write = [&](int p) {
#pragma unroll
        for (int j = 2 * p; j < 2 * p + 2; ++j)
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                if (i % 3 == 0) __builtin_amdgcn_sched_barrier(0);      // (pieces computed far ahead of their stores would spill)
                f32x4 v = acc[i][j] + bias[i];
                if constexpr (MODE == EPI_STORE_GELU) { v[0] = gelu_tanh(v[0]); v[1] = gelu_tanh(v[1]); v[2] = gelu_tanh(v[2]); v[3] = gelu_tanh(v[3]); }
                if constexpr (MODE == EPI_STORE_HEADS) v *= nw + i * 16 < e.hid ? e.q_scale : 1.f;     // hid is a multiple of 16
                if constexpr (MODE == EPI_STORE_GATED) v *= gate[i];
                const bf16x4 o = { (bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3] };
                *reinterpret_cast<bf16x4*>(wrow + j * 16 * PITCH + i * 32) = o;
            }
    };
    write(0);
#pragma unroll
    for (int p = 0; p < TM / 32; ++p) {
        if (p + 1 < TM / 32) write(p + 1);          // the next pass's arithmetic covers this one's way through LDS
        __builtin_amdgcn_sched_barrier(0);
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const u32x4*>(wbuf + p * 32 * PITCH + lo[u]);
        const int m = __builtin_amdgcn_readfirstlane(mw + p * 32);
        char* out;
        if constexpr (MODE == EPI_STORE_HEADS) {
            const int slot = fast_div(m, e.rps_magic, e.rps_shift);
            out = (char*)e.out + ((size_t)slot * e.heads * e.rows_per_slot + (m - slot * e.rows_per_slot)) * e.hd * 2;
        } else out = (char*)e.out + (size_t)m * e.ldo * 2;
#pragma unroll
        for (int u = 0; u < U; ++u) *reinterpret_cast<u32x4*>(out + go[u]) = v[u];
    }
}

// The epilogue's mode found at run time.
template <int TM, int TN, bool EDGES_ONLY = false>
__device__ __forceinline__ void store_tile(const f32x4 (&acc)[TN / 16][TM / 16], const Epilogue& e, int mw, int nw, int M, int N,
                                           const unsigned char* erows, int rstride, const GateRows& gr)
{
    const int lane = threadIdx.x & 63;
    if (e.mode == EPI_RESID) store_tile_as<TM, TN, EPI_RESID, true, EDGES_ONLY>(acc, e, mw, nw, M, N, erows, rstride, gr, lane);
    else if (e.out_f32) {
        if (e.mode == EPI_STORE_GELU) store_tile_as<TM, TN, EPI_STORE_GELU, true, EDGES_ONLY>(acc, e, mw, nw, M, N, erows, rstride, gr, lane);
        else store_tile_as<TM, TN, EPI_STORE, true, EDGES_ONLY>(acc, e, mw, nw, M, N, erows, rstride, gr, lane);
    } else if (e.mode == EPI_STORE_GELU) store_tile_as<TM, TN, EPI_STORE_GELU, false, EDGES_ONLY>(acc, e, mw, nw, M, N, erows, rstride, gr, lane);
    else if (e.mode == EPI_STORE_HEADS) store_tile_as<TM, TN, EPI_STORE_HEADS, false, EDGES_ONLY>(acc, e, mw, nw, M, N, erows, rstride, gr, lane);
    else if (e.mode == EPI_STORE_GATED) store_tile_as<TM, TN, EPI_STORE_GATED, false, EDGES_ONLY>(acc, e, mw, nw, M, N, erows, rstride, gr, lane);
    else store_tile_as<TM, TN, EPI_STORE, false, EDGES_ONLY>(acc, e, mw, nw, M, N, erows, rstride, gr, lane);
}

// Whether the workgroup's tile (rows m0 .., columns n0 ..) may go through store_rows.
template <int BM, int BN>
__device__ inline bool may_store_rows(const Epilogue& e, int m0, int n0, int M, int N, const GateRows& gr)
{
    if (m0 + BM > M || n0 + BN > N || e.out_f32 || e.mode == EPI_RESID) return false;
    if (e.mode == EPI_STORE_GATED) return gr.rows == 1;
    if (e.mode == EPI_STORE_HEADS) return e.rows_per_slot % 32 == 0 && e.plane <= ((size_t)1 << 29);
    return true;
}

}  // namespace

}  // namespace drf
