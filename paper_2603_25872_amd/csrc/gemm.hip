// GEMM C[M][N] = A[M][K] . W[N][K]^T with fused epilogues (bias, GELU-tanh, gated
// residual).  bf16 path: software-pipelined kernels (16x16x32 MFMAs, operands by LDS-DMA, fp32 accumulate) at tiles from
// 32 x 64 to 256 x 288, the tile chosen by a measured time model.  The 256-row tiles of 256 and 288 columns have a four-wave form
// (gemm_wide.h) beside the one here, the 144-column tiles one of two pairs of waves (gemm_pair.h).
// fp32 path: fp32 MFMA, operands straight to registers, K split over the waves of a workgroup.
#include "gemm_device.h"

namespace drf {

namespace {

// Applies the epilogue to 4 consecutive columns n..n+3 of row m (n % 4 == 0, n + 3 < N).
__device__ inline void epilogue4(const Epilogue& e, int m, int n, float v0, float v1, float v2, float v3)
{
    const float4 b = *reinterpret_cast<const float4*>(e.bias + n);
    v0 += b.x; v1 += b.y; v2 += b.z; v3 += b.w;
    if (e.mode == EPI_RESID) {
        float4* xp = reinterpret_cast<float4*>((float*)e.out + (size_t)m * e.ldo + n);
        float4 x = *xp;
        if (e.gate) {
            const float4 g = *reinterpret_cast<const float4*>(e.gate + (size_t)fast_div(m, e.rps_magic, e.rps_shift) * e.gate_ld + n);
            x.x = fmaf(g.x, v0, x.x); x.y = fmaf(g.y, v1, x.y); x.z = fmaf(g.z, v2, x.z); x.w = fmaf(g.w, v3, x.w);
        } else {
            x.x += v0; x.y += v1; x.z += v2; x.w += v3;
        }
        *xp = x;
        return;
    }
    if (e.mode == EPI_STORE_GELU) { v0 = gelu_tanh(v0); v1 = gelu_tanh(v1); v2 = gelu_tanh(v2); v3 = gelu_tanh(v3); }
    if (e.mode == EPI_STORE_GATED) {
        const float4 g = *reinterpret_cast<const float4*>(e.gate + (size_t)fast_div(m, e.rps_magic, e.rps_shift) * e.gate_ld + n);
        v0 *= g.x; v1 *= g.y; v2 *= g.z; v3 *= g.w;
    }
    if (e.mode == EPI_STORE_HEADS && n < e.hid) { v0 *= e.q_scale; v1 *= e.q_scale; v2 *= e.q_scale; v3 *= e.q_scale; }
    if (e.out_f32) {
        *reinterpret_cast<float4*>((float*)e.out + (size_t)m * e.ldo + n) = make_float4(v0, v1, v2, v3);
    } else {
        bf16x4 o = { (bf16_t)v0, (bf16_t)v1, (bf16_t)v2, (bf16_t)v3 };
        const size_t off = e.mode == EPI_STORE_HEADS ? heads_offset(e, m, n) : (size_t)m * e.ldo + n;
        *reinterpret_cast<bf16x4*>((bf16_t*)e.out + off) = o;
    }
}

// The same for the fp32 path's modes, in two parts: what it reads, asked for ahead of the product, and the rest.
struct EpilogueOperands { f32x4 bias, gate, x; };
__device__ inline EpilogueOperands load_epilogue4(const Epilogue& e, int m, int n)
{
    EpilogueOperands o;
    o.bias = *reinterpret_cast<const f32x4*>(e.bias + n);
    o.gate = (f32x4){ 1.f, 1.f, 1.f, 1.f };
    if (e.mode == EPI_RESID) {
        o.x = *reinterpret_cast<const f32x4*>((const float*)e.out + (size_t)m * e.ldo + n);
        if (e.gate) o.gate = *reinterpret_cast<const f32x4*>(e.gate + (size_t)fast_div(m, e.rps_magic, e.rps_shift) * e.gate_ld + n);
    }
    return o;
}
__device__ inline void store_epilogue4(const Epilogue& e, int m, int n, f32x4 v, const EpilogueOperands& o)
{
    v += o.bias;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (e.mode == EPI_RESID) v[j] = fmaf(o.gate[j], v[j], o.x[j]);
        if (e.mode == EPI_STORE_GELU) v[j] = gelu_tanh(v[j]);
        if (e.mode == EPI_STORE_SILU) v[j] = silu(v[j]);
    }
    *reinterpret_cast<f32x4*>((float*)e.out + (size_t)m * e.ldo + n) = v;
}

// ------------------------------------------------------------------ bf16 MFMA
// The kernel for small problems and for what the 4-wave kernels leave (see wide_form): BM x BN x 64 block tile, waves as WM x WN (x WK), wave
// tile (BM/WM) x (BN/WN) built from 16x16x32 MFMAs so that widths only need to be multiples of 16.
//  - operands go HBM -> LDS directly (global_load_lds_dwordx4: every lane supplies its own
//    global address and the wave's 64 x 16 bytes land contiguously in LDS), NS stages so the copy of the next k-tiles overlaps
//    the MFMAs of k-tile t.  A tile row is 128 bytes = 8
//    chunks; chunk c of row r sits at position c ^ ((r / 2) % 8), which keeps both the DMA
//    writes and the ds_read_b128 operand fetches free of bank conflicts;
//  - workgroup ids are remapped so that each XCD (ids are dealt round-robin over the 8 XCDs)
//    works on a compact group of tiles and shares A/W slices through its own L2;
//  - the weight tile is the MFMA A operand: a lane ends with 4 consecutive columns n of one
//    row m per accumulator;
//  - epilogue: store_tile, or (RS: the tiles that fill the chip) store_rows through the idle LDS stages.
// copy instructions issued per MFMA group by the in-loop copy of the two-stage kernels (1: measured best; 2, 3 and
// the whole copy at once are 0.8 % slower per call, one every other group lands too late: 3 % slower)
constexpr int kSpreadPer = 1;
// partial tiles of one split-K launch: 256 tiles of 128 x 128
constexpr size_t kSplitKScratchFloats = (size_t)256 * 128 * 128;

//  - SK (split K across workgroups, for problems with few tiles and a long K): tiles_n counts sk.splits column-tile
//    rows, workgroup (tm, tn) takes the k-steps of part tn / sk.tiles_n (parts differ by at most one step) of column
//    tile tn % sk.tiles_n and leaves its fp32 partial tile in sk.part ([split][tiles_m * BM][sk.tiles_n * BN], padded,
//    so no bounds are needed); splitk_reduce_kernel adds the partial tiles in a fixed order and applies the epilogue.
struct SplitK { int splits, tiles_n; float* part; };

template <int BM, int BN, int BK, int NS, int WM, int WN, int WK = 1, bool SK = false, bool RS = false>
__global__ void __launch_bounds__(WM * WN * WK * 64)
gemm_bf16_xl_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, int M, int N, int K, const Epilogue e,
                    int tiles_m, int tiles_n, int m_first, const SplitK sk)
{
    // WK > 1: the waves form WK groups that share the output tile and split K between them (group g
    // takes the k-tiles g, g + WK, ...); the groups' partial sums are added through LDS before the
    // epilogue.  This doubles the waves per CU for shapes that only yield one small tile per CU.
    constexpr int NWT = WM * WN, NW = NWT * WK, TM = BM / WM, TN = BN / WN, MI = TM / 16, NI = TN / 16, KS = BK / 32;
    constexpr int CPR = BK / 8, RPI = 64 / CPR, RB = 256 / (BK * 2);
    constexpr int STAGE1 = (BM + BN) * BK, STAGE = WK * STAGE1;
    constexpr int SEG1 = (BM + BN) / RPI, SEG = WK * SEG1, LPT = (SEG + NW - 1) / NW;
    constexpr int GROUP_M = 8;
    static_assert(TM % 16 == 0 && TN % 16 == 0 && (BM + BN) % RPI == 0 && BM % 16 == 0, "tile shape");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];

    const int nb = tiles_m * tiles_n, b = blockIdx.x;
    const int xcd = b & 7, local = b >> 3, q = nb >> 3, rem = nb & 7;
    const int idx = xcd * q + (xcd < rem ? xcd : rem) + local;
    const int per_group = GROUP_M * tiles_n, group = idx / per_group, first_m = group * GROUP_M;
    const int gsz = tiles_m - first_m < GROUP_M ? tiles_m - first_m : GROUP_M;
    const int tm = first_m + (idx % per_group) % gsz, tn = (idx % per_group) / gsz;
    const int split = SK ? tn / sk.tiles_n : 0;
    const int m0 = m_first + tm * BM, n0 = (SK ? tn - split * sk.tiles_n : tn) * BN;
    int nk = K / (BK * WK);                                          // k-steps of this workgroup
    if constexpr (SK) {
        const int first = split * nk / sk.splits, last = (split + 1) * nk / sk.splits;
        A += first * BK * WK; W += first * BK * WK;                  // row stride stays K
        nk = last - first;
    }

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave-uniform, kept in a scalar register
    const int wk = wave / NWT, wl = wave % NWT, wm = wl % WM, wn = wl / WM;
    const int l16 = lane & 15, quarter = lane >> 4;

    // DMA: the A rows and W rows of a k-tile form one row space [0, BM + BN), and a stage holds WK
    // k-tiles one after the other.  A wave-wide instruction covers RPI rows (never straddling the
    // A/W boundary).  Every wave issues LPT instructions; when SEG is not a multiple of the wave
    // count the surplus ones repeat the last segment (same bytes, same place).  Per lane only a
    // 32-bit byte offset is kept; the matrix base and the LDS destination are wave-uniform.
    const int prow = lane / CPR, ppos = lane % CPR;
    uint32_t voff[LPT];
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        int g = wave * LPT + i; g = g < SEG ? g : SEG - 1;
        const int gl = g % SEG1, r = gl * RPI + prow;
        const int chunk = ppos ^ ((r / RB) & (CPR - 1));
        int row;
        if (gl * RPI < BM) { row = m0 + r; row = row < M ? row : M - 1; }
        else { row = n0 + r - BM; row = row < N ? row : N - 1; }
        voff[i] = ((uint32_t)row * (uint32_t)K + (uint32_t)chunk * 8u) * 2u;
    }
    const uint32_t lds_base = (uint32_t)(uintptr_t)(DRF_LDS_AS unsigned char*)smem_raw;
    // instruction i (of this wave's LPT) of the copy of k-tile kt into `stage`
    auto issue_one = [&](auto ic, int kt, int stage) {
        constexpr int i = decltype(ic)::value;
        int g = wave * LPT + i; g = g < SEG ? g : SEG - 1;
        const int sub = g / SEG1, gl = g % SEG1;
        // written by hand in the scalar-base form (uniform 64-bit base in SGPRs + the lane's 32-bit byte offset),
        // which needs no 64-bit address registers per lane; M0 carries the wave-uniform LDS destination
        const bf16_t* base = (gl * RPI < BM ? A : W) + (kt * WK + sub) * BK;
        const uint32_t dst = lds_base + (uint32_t)(stage * STAGE + sub * STAGE1 + gl * RPI * BK) * 2u;
        const uint32_t vo = voff[i];
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :: "s"(dst), "v"(vo), "s"(base) : "memory");
    };
    auto issue = [&](int kt, int stage) {
        static_for<0, LPT>([&](auto ic) { issue_one(ic, kt, stage); });
    };

    f32x4 acc[NI][MI];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j) acc[i][j] = (f32x4){ 0.f, 0.f, 0.f, 0.f };

    int koff[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) koff[ks] = l16 * BK + (((ks * 4 + quarter) ^ ((l16 / RB) & (CPR - 1))) << 3);

    // Main loop, software-pipelined at the granularity of one weight fragment.  The MFMAs of a k-tile
    // are G = KS * NI groups (one 16-column weight fragment against the MI activation fragments); the
    // LDS read of the fragment for group g + D is issued just before the MFMAs of group g, into a ring
    // of R = D + 1 register sets, and the activation fragments of a k-step are double-buffered the
    // same way.  The block barrier that hands over the next k-tile (its DMA has landed, every wave has
    // finished reading the current one) sits D groups before the end of the current tile, so each wave
    // leaves it with D groups of MFMAs whose operands are already in registers while the first reads
    // of the new tile are in flight: no LDS latency is exposed at the tile boundary.
    // The fragment reads and their waits are written by hand (ds_read_b128 / s_waitcnt lgkmcnt(n)):
    // with LDS-DMA in the loop the compiler's own wait insertion falls back to lgkmcnt(0), which
    // exposes a full LDS round trip several times per tile.  LDS reads return in order, so before the
    // MFMAs of group g it is enough that at most the reads issued after position g's remain.
    static_assert(NS >= 2 && KS == 2, "the pipelined loop assumes LDS stages of two k-steps");
    constexpr int G = KS * NI;
    constexpr int R = G % 6 == 0 && NI >= 6 ? 6 : G % 4 == 0 && NI >= 4 ? 4 : G % 5 == 0 && NI >= 5 ? 5 : G % 3 == 0 && NI >= 3 ? 3 : 2, D = R - 1;
    static_assert(G % R == 0 && D < NI && D + MI <= 15, "ring size");
    // With two stages the copy of tile kt + 2 is not issued as one burst after the barrier of tile kt (72
    // wave-wide loads that the vector-memory path takes one per ~17 cycles, during which the issuing waves
    // cannot issue MFMAs) but one instruction per MFMA group: the first HEAD of them in the groups after the
    // barrier, the remaining TAIL in the first groups of the next tile.  All of them are issued long before
    // the next barrier, whose vmcnt(0) covers them as before.
    constexpr int PER = kSpreadPer;                 // copy instructions per MFMA group
    constexpr int HEAD0 = D * PER < LPT ? D * PER : LPT;
    constexpr bool kSpread = NS == 2 && WK == 1 && (LPT - HEAD0 + PER - 1) / PER <= G - D;
    constexpr int HEAD = kSpread ? HEAD0 : LPT, TAIL = LPT - HEAD;
    u32x4 fa[2][MI], fw[R];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(DRF_LDS_AS unsigned char*)smem_raw;
    uint32_t a_addr[KS], w_addr[KS];                // byte addresses of this lane's fragments in stage 0
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        a_addr[ks] = lds0 + (uint32_t)(wk * STAGE1 + wm * TM * BK + koff[ks]) * 2u;
        w_addr[ks] = lds0 + (uint32_t)(wk * STAGE1 + BM * BK + wn * TN * BK + koff[ks]) * 2u;
    }
    // reads of stream position p (0 <= p < G) of a k-tile; aa / wa: this lane's fragment addresses in its stage
    auto fetch = [&](auto pc, const uint32_t (&aa)[KS], const uint32_t (&wa)[KS]) {
        constexpr int p = decltype(pc)::value, ks = p / NI, i = p % NI;
        if constexpr (i == 0)
            static_for<0, MI>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                lds_read16<j * 16 * BK * 2>(fa[ks & 1][j], aa[ks]);
            });
        lds_read16<i * 16 * BK * 2>(fw[p % R], wa[ks]);
    };

    // tiles 0 .. NS-2 are in flight before the loop; tile kt + NS - 1 is requested once tile kt - 1 has been read
    issue(0, 0);
    const GateRows gr = gate_rows<BM>(e, m0, M);
    if constexpr (!SK) stage_epilogue_rows<BN>(e, gr, lds_base + NS * STAGE * 2, wave, NW, n0, N);
#pragma unroll
    for (int t = 1; t < NS - 1; ++t)
        if (t < nk) issue(t, t);
    if (NS > 2 && nk >= NS - 1) wait_vmcnt<LPT * (NS - 2)>(); else wait_vmcnt<0>();
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    warm_caches(e, lds_base + NS * STAGE * 2 + epi_lds_bytes(BN), nb, b, wave, NW);     // (the last k-tile's wait covers it)
    static_for<0, NI * MI>([&](auto pc) { constexpr int p = decltype(pc)::value; hold_acc<false>(acc[p / MI][p % MI]); });
    settle_mfma();
    if (NS - 1 < nk) issue(NS - 1, NS - 1);
    static_for<0, D>([&](auto pc) { fetch(pc, a_addr, w_addr); });
    int cs = 0;                                     // stage of tile kt
    for (int kt = 0; kt < nk; ++kt) {
        const int ns = cs + 1 == NS ? 0 : cs + 1;
        const uint32_t co = (uint32_t)cs * (uint32_t)(STAGE * 2), no = (uint32_t)ns * (uint32_t)(STAGE * 2);
        uint32_t ca[KS], cw[KS], na[KS], nw[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) { ca[ks] = a_addr[ks] + co; cw[ks] = w_addr[ks] + co; na[ks] = a_addr[ks] + no; nw[ks] = w_addr[ks] + no; }
        static_for<0, G>([&](auto gc) {
            constexpr int g = decltype(gc)::value;
            if constexpr (g + D == G) {
                // tile kt+1 has landed (vmcnt 0) and this wave's reads of tile kt are complete (lgkmcnt 0), for
                // every wave after the barrier: the stage of tile kt may be refilled
                // (the NS - 2 younger tiles may still be in flight; near the end fewer are, so wait for all)
                if (NS > 2 && kt + NS - 1 < nk) wait_vmcnt<LPT * (NS - 2)>(); else wait_vmcnt<0>();
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                if constexpr (!kSpread) {
                    if (kt + NS < nk) issue(kt + NS, cs);
                }
            }
            if constexpr (kSpread) {
                static_for<0, PER>([&](auto uc) {
                    constexpr int u = decltype(uc)::value;
                    if constexpr (g >= G - D && (g - (G - D)) * PER + u < HEAD) {
                        if (kt + NS < nk) issue_one(std::integral_constant<int, (g - (G - D)) * PER + u>{}, kt + NS, cs);
                    } else if constexpr (g < G - D && g * PER + u < TAIL) {
                        // the rest of the copy that the previous tile's last groups started: tile kt + 1, into the other stage
                        if (kt >= 1 && kt + 1 < nk) issue_one(std::integral_constant<int, HEAD + g * PER + u>{}, kt + 1, ns);
                    }
                });
            }
            {
                // on the last tile the positions beyond it read the idle stage: valid LDS, values unused
                // (drained by the wait after the loop)
                if constexpr (g + D < G) fetch(std::integral_constant<int, g + D>{}, ca, cw);
                else fetch(std::integral_constant<int, g + D - G>{}, na, nw);
                __builtin_amdgcn_sched_barrier(0);
                // reads issued after position g's: one per later position, plus the activation fragments
                // of a k-step that starts among them
                constexpr int later = D + (((g + D) / NI) != (g / NI) ? MI : 0);
                if constexpr (g % NI == 0) wait_frags<later, MI>(fw[g % R], fa[(g / NI) & 1]);
                else wait_frag<later>(fw[g % R]);
                static_for<0, MI>([&](auto jc) {
                    constexpr int j = (g & 1) ? MI - 1 - decltype(jc)::value : decltype(jc)::value;   // snake: one operand changes per MFMA
                    mfma<false>(acc[g % NI][j], fw[g % R], fa[(g / NI) & 1][j]);
                });
                __builtin_amdgcn_sched_barrier(0);
            }
        });
        cs = ns;
    }
    // The last tile's look-ahead reads are still on their way into the fragment registers, which nothing consumes
    // any more: they pass through the wait, so that no register of theirs is given to anything computed above it
    // (a column index kept there would be overwritten by the data that lands).
    wait_frag<0>(fw[0]);
    settle_mfma();
    static_for<0, NI * MI>([&](auto pc) { constexpr int p = decltype(pc)::value; hold_acc<false>(acc[p / MI][p % MI]); });
#pragma unroll
    for (int r = 1; r < R; ++r) hold_frag(fw[r]);
#pragma unroll
    for (int j = 0; j < MI; ++j) { hold_frag(fa[0][j]); hold_frag(fa[1][j]); }

    // ---- epilogue: acc[i][j][r] is (m = j*16 + l16, n = i*16 + 4*quarter + r) of the wave tile
    constexpr int PART = (WK - 1) * NWT * TM * TN * 4;              // partial sums of the other K groups
    if constexpr (WK > 1) {
        static_assert(PART < NS * STAGE * 2, "LDS too small for the split-K partial sums");
        __syncthreads();                                            // the stages are idle
        f32x4* part = reinterpret_cast<f32x4*>(smem_raw);
        if (wk > 0) {
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < MI; ++j) part[(((wk - 1) * NWT + wl) * NI * MI + i * MI + j) * 64 + lane] = acc[i][j];
        }
        __syncthreads();
        if (wk > 0) return;                                         // the first group finishes the tile
#pragma unroll
        for (int g = 0; g < WK - 1; ++g)
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < MI; ++j) acc[i][j] += part[((g * NWT + wl) * NI * MI + i * MI + j) * 64 + lane];
    }
    if constexpr (SK) {
        // partial tile, straight from the accumulators: acc[i][j][r] is (m = j*16 + l16, n = i*16 + 4*quarter + r)
        float* pt = sk.part + ((size_t)split * tiles_m * BM + m0 + wm * TM) * ((size_t)sk.tiles_n * BN) + n0 + wn * TN;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < MI; ++j)
                *reinterpret_cast<f32x4*>(pt + (size_t)(j * 16 + l16) * ((size_t)sk.tiles_n * BN) + i * 16 + 4 * quarter) = acc[i][j];
        return;
    }
    if constexpr (RS) {
        if (may_store_rows<BM, BN>(e, m0, n0, M, N, gr)) {
            static_assert(PART + NWT * rows_tile_bytes(TM, TN) <= NS * STAGE * 2, "LDS too small for the waves' tiles in rows");
            if constexpr (WK == 1) asm volatile("s_barrier" ::: "memory");      // every wave has read its last fragments
            const int mw = m0 + wm * TM, nw = n0 + wn * TN;
            unsigned char* wbuf = smem_raw + PART + wl * rows_tile_bytes(TM, TN);
            const unsigned char* erows = smem_raw + NS * STAGE * 2 + wn * TN * 4;
            if (e.mode == EPI_STORE_GELU) store_rows<TM, TN, EPI_STORE_GELU, 0>(acc, e, mw, nw, wbuf, erows, 0);
            else if (e.mode == EPI_STORE_HEADS) store_rows<TM, TN, EPI_STORE_HEADS, 0>(acc, e, mw, nw, wbuf, erows, 0);
            else if (e.mode == EPI_STORE_GATED) store_rows<TM, TN, EPI_STORE_GATED, 1>(acc, e, mw, nw, wbuf, erows, epi_row_bytes(BN));
            else store_rows<TM, TN, EPI_STORE, 0>(acc, e, mw, nw, wbuf, erows, 0);
            return;
        }
    }
    store_tile<TM, TN>(acc, e, m0 + wm * TM, n0 + wn * TN, M, N, smem_raw + NS * STAGE * 2 + wn * TN * 4, epi_row_bytes(BN), gr);
}

// Sum of the split-K partial tiles (fixed order: deterministic), then the epilogue; one thread per 4 columns.
__global__ void __launch_bounds__(256)
splitk_reduce_kernel(const float* __restrict__ part, int splits, size_t split_stride, int ldp, int M, int N, const Epilogue e)
{
    const int n4 = N / 4, id = blockIdx.x * 256 + threadIdx.x;
    if (id >= M * n4) return;
    const int m = id / n4, n = (id - m * n4) * 4;
    const float* p = part + (size_t)m * ldp + n;
    float4 v = *reinterpret_cast<const float4*>(p);
    for (int s2 = 1; s2 < splits; ++s2) {
        const float4 u = *reinterpret_cast<const float4*>(p + (size_t)s2 * split_stride);
        v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
    }
    epilogue4(e, m, n, v.x, v.y, v.z, v.w);
}

// ------------------------------------------------------------------------ fp32
// 32 x 32 (F == 2) or 16 x 16 (F == 1) output tile per workgroup on the fp32 matrix instruction (16x16x4, exact fp32 products and sums); the NW
// waves split K (wave w takes the 16-wide k-steps w, w + NW, ...) and add their partial tiles through LDS.  Operands go
// from memory straight to registers, B steps at a time and one batch ahead: the problems of this path are a few
// hundred rows, where a launch is a chain of round trips to memory, and a staged tile only adds barriers to them.  What the
// epilogue adds to the product is asked for before the first of its operands is used.  Two forms (f32_small): 16 x 16 tiles
// with K dealt over enough waves that one batch takes all of it up to 512, and 32 x 32 tiles of four waves for more rows.
// A lane loads 4 consecutive k of its row; MFMA e of a step takes element e of every lane, that is the k-set
// {4 quarter + e}, the same for both operands.  The weights are the first operand: a lane ends with 4 consecutive n.
// VEC: rows are 16-byte aligned and K % 4 == 0; otherwise the four elements are loaded one by one.
// LN: A is the residual stream, and its rows are normalised and modulated here (statistics over all K, in one batch), in
// place of a launch that does it once for all column tiles: for a few rows reading and normalising them again costs less than
// that launch (M = 64, K = 128: 3.2 + 5.3 us as two launches, 4.4 as one; 2304 rows of 256: 1.7 times the two).
// (32 x 32 tiles: three workgroups a CU; a fourth evicts the lines that they share from L1, 5 % slower at 16384 x 1024 and more.)
template <bool VEC, int F, int NW, int B, bool LN>
__global__ void __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(F == 2 ? 3 : 1, F == 2 ? 3 : 8)))
gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ W, int M, int N, int K, int a_row_mod, const Epilogue e, const RowNorm ln)
{
    constexpr int T = 16 * F;
    __shared__ f32x4 part[NW][F * F][64];
    __shared__ float red[LN ? 2 : 1][NW][T];
    const int lane = threadIdx.x & 63, l16 = lane & 15, quarter = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = blockIdx.x * T;
    for (int m0 = blockIdx.y * T; m0 < M; m0 += gridDim.y * T) {   // (more row tiles than the grid's y limit: several each)
        const float *ap[F], *wp[F], *sc[F], *sh[F];
#pragma unroll
        for (int i = 0; i < F; ++i) {
            int m = m0 + i * 16 + l16, n = n0 + i * 16 + l16;           // rows past the end repeat the last one, never stored
            m = m < M ? m : M - 1; n = n < N ? n : N - 1;
            if (a_row_mod) m %= a_row_mod;
            ap[i] = A + (size_t)m * K; wp[i] = W + (size_t)n * K;
            if (LN && ln.shift) { const size_t mr = (size_t)(m / ln.rows_per_slot) * ln.mod_ld; sc[i] = ln.scale + mr; sh[i] = ln.shift + mr; }
        }
        auto load4 = [&](const float* p, int k) -> f32x4 {
            f32x4 v = { 0.f, 0.f, 0.f, 0.f };
            if constexpr (VEC) {
                if (k < K) v = *reinterpret_cast<const f32x4*>(p + k);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (k + j < K) v[j] = p[k + j];
            }
            return v;
        };
        f32x4 fa[2][B][F], fw[2][B][F], acc[F][F];      // [buffer][step][16-row part]; acc[n part][m part]
        auto load = [&](f32x4 (&a)[B][F], f32x4 (&w)[B][F], int step) {
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int k = (step + NW * u) * 16 + 4 * quarter;
#pragma unroll
                for (int i = 0; i < F; ++i) { a[u][i] = load4(ap[i], k); w[u][i] = load4(wp[i], k); }
            }
        };
        auto multiply = [&](const f32x4 (&a)[B][F], const f32x4 (&w)[B][F], int left) {
#pragma unroll
            for (int u = 0; u < B; ++u)
                if (F == 2 || u == 0 || NW * u < left)                  // (steps past the end are zeros)
#pragma unroll
                    for (int k = 0; k < 4; ++k)
#pragma unroll
                        for (int i = 0; i < F; ++i)
#pragma unroll
                            for (int j = 0; j < F; ++j)
                                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][i][k], a[u][j][k], acc[i][j], 0, 0, 0);
        };
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
            for (int j = 0; j < F; ++j) acc[i][j] = (f32x4){ 0.f, 0.f, 0.f, 0.f };
        const int steps = (K + 15) / 16;
        load(fa[0], fw[0], wave);
        f32x4 s4[LN ? B : 1][F], h4[LN ? B : 1][F];
        if constexpr (LN) {
#pragma unroll
            for (int u = 0; u < B; ++u)
#pragma unroll
                for (int i = 0; i < F; ++i) {
                    const int k = (wave + NW * u) * 16 + 4 * quarter;
                    s4[u][i] = h4[u][i] = (f32x4){ 0.f, 0.f, 0.f, 0.f };
                    if (ln.shift) { s4[u][i] = load4(sc[i], k); h4[u][i] = load4(sh[i], k); }
                }
        }
        // wave f < F F finishes fragment f: acc[i][j][r] is (n = 16 i + 4 quarter + r, m = 16 j + l16) of the tile
        const int em = m0 + wave % F * 16 + l16, en = n0 + wave / F * 16 + 4 * quarter;
        const bool mine = wave < F * F && em < M && en < N;
        EpilogueOperands ops;
        if (F == 1 && mine) ops = load_epilogue4(e, em, en);
        if constexpr (LN) {
            // mean, then the centred squares: two exchanges between the quarters and the waves
            float mean[F], rstd[F];
            auto total = [&](const float (&v)[F], float (&out)[F], int which) {
#pragma unroll
                for (int i = 0; i < F; ++i) {
                    float t = v[i];
                    t += __shfl_xor(t, 16, 64); t += __shfl_xor(t, 32, 64);
                    if (quarter == 0) red[which][wave][i * 16 + l16] = t;
                }
                __syncthreads();
#pragma unroll
                for (int i = 0; i < F; ++i) {
                    float t = 0.f;
#pragma unroll
                    for (int w = 0; w < NW; ++w) t += red[which][w][i * 16 + l16];
                    out[i] = t;
                }
            };
            float v[F] = {};
#pragma unroll
            for (int u = 0; u < B; ++u)
#pragma unroll
                for (int i = 0; i < F; ++i) v[i] += (fa[0][u][i][0] + fa[0][u][i][1]) + (fa[0][u][i][2] + fa[0][u][i][3]);
            total(v, mean, 0);
#pragma unroll
            for (int i = 0; i < F; ++i) {
                v[i] = 0.f;
                mean[i] *= 1.f / (float)K;
#pragma unroll
                for (int u = 0; u < B; ++u)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const bool in = (wave + NW * u) * 16 + 4 * quarter + j < K;
                        fa[0][u][i][j] = in ? fa[0][u][i][j] - mean[i] : 0.f;
                        v[i] = fmaf(fa[0][u][i][j], fa[0][u][i][j], v[i]);
                    }
            }
            total(v, rstd, LN ? 1 : 0);
#pragma unroll
            for (int i = 0; i < F; ++i) {
                rstd[i] = rsqrtf(rstd[i] * (1.f / (float)K) + 1e-6f);
#pragma unroll
                for (int u = 0; u < B; ++u)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float y = fa[0][u][i][j] * rstd[i];
                        fa[0][u][i][j] = ln.shift ? fmaf(y, 1.f + s4[u][i][j], h4[u][i][j]) : y;
                    }
            }
            multiply(fa[0], fw[0], steps - wave);
        } else {
            for (int s = wave; s < steps; s += 2 * NW * B) {
                if (F == 2 || s + NW * B < steps) load(fa[1], fw[1], s + NW * B);
                multiply(fa[0], fw[0], steps - s);
                if (F == 2 || s + 2 * NW * B < steps) load(fa[0], fw[0], s + 2 * NW * B);
                if (F == 2 || s + NW * B < steps) multiply(fa[1], fw[1], steps - s - NW * B);
            }
        }
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
            for (int j = 0; j < F; ++j) part[wave][i * F + j][lane] = acc[i][j];
        __syncthreads();
        if (mine) {
            if (F == 2) ops = load_epilogue4(e, em, en);                // (registers that the loop needs, where there are many tiles)
            f32x4 v = part[0][wave][lane];
#pragma unroll
            for (int w = 1; w < NW; ++w) v += part[w][wave][lane];
            store_epilogue4(e, em, en, v, ops);
        }
        __syncthreads();
    }
}

template <int BM, int BN, int BK, int NS, int WM, int WN, int WK = 1, bool RS = false>
drf_status launch_bf16_xl(const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int m_first = 0)
{
    constexpr size_t smem = (size_t)NS * WK * (BM + BN) * BK * sizeof(bf16_t) + epi_lds_bytes(BN) + 256;
    static_assert(smem <= 160 * 1024, "LDS of a CU");
    static bool attr_set = false;
    auto kern = gemm_bf16_xl_kernel<BM, BN, BK, NS, WM, WN, WK, false, RS>;
    if (K % (BK * WK) != 0) DRF_FAIL(DRF_ESHAPE, "bf16 GEMM tile needs K %% %d == 0 (K=%d)", BK * WK, K);
    if (!attr_set) {
        DRF_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        attr_set = true;
    }
    const int tiles_m = (M - m_first + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(WM * WN * WK * 64), smem, st, A, W, M, N, K, e, tiles_m, tiles_n, m_first, SplitK{});
    DRF_HIP(hipGetLastError());
    return DRF_OK;
}

// Split-K form: `splits` workgroups per output tile, partial tiles in `part`, then the reduction with the epilogue.
template <int BM, int BN, int BK, int NS, int WM, int WN, int WK = 1>
drf_status launch_bf16_splitk(const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st,
                              int splits, float* part, PartialSum* leave)
{
    constexpr size_t smem = (size_t)NS * WK * (BM + BN) * BK * sizeof(bf16_t) + epi_lds_bytes(BN) + 256;
    static_assert(smem <= 160 * 1024, "LDS of a CU");
    static bool attr_set = false;
    auto kern = gemm_bf16_xl_kernel<BM, BN, BK, NS, WM, WN, WK, true>;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    if (!part || K % (BK * WK) != 0 || K / (BK * WK) < splits || (size_t)tiles_m * tiles_n * splits * BM * BN > kSplitKScratchFloats)
        DRF_FAIL(DRF_ESHAPE, "split-K GEMM of %d parts does not fit (M=%d N=%d K=%d)", splits, M, N, K);
    if (!attr_set) {
        DRF_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        attr_set = true;
    }
    SplitK sk{ splits, tiles_n, part };
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n * splits), dim3(WM * WN * WK * 64), smem, st, A, W, M, N, K, e, tiles_m, tiles_n * splits, 0, sk);
    DRF_HIP(hipGetLastError());
    const int ldp = tiles_n * BN;
    if (leave) {
        *leave = PartialSum{ part, splits, ldp, (size_t)tiles_m * BM * ldp };
        return DRF_OK;
    }
    const long long quads = (long long)M * (N / 4);
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, st, part, splits,
                       (size_t)tiles_m * BM * ldp, ldp, M, N, e);
    DRF_HIP(hipGetLastError());
    return DRF_OK;
}

// The tiles, and a time model of a launch of each: base + (per round of workgroups) round + steps * max(lat, c * thr)
// microseconds, where a round is per_cu workgroups on each of the 256 CUs, c the workgroups that share a CU in it and
// steps the k-steps of 64 * wk; a split adds red0 + red1 per million partial elements for the reduction launch.
// The constants are least-squares fits to timings of every tile on 134 shapes (M 16 .. 65536, N 384 .. 195840, K 384 ..
// 4608, weights cold, back to back), those of 7 and 18 to timings inside a pass, where launches take longer and short ones the
// more: there the choice is within 5 % of the best single launch at most sizes of hidden 384 and 1152, up to 20 % behind at others.
// Small problems live on small tiles: with weights coming from HBM a launch is a chain of round trips, and what counts is
// how many of the chip's CUs pull operands at once (M = 512, N = K = 1152: 7.1 us on 144 64 x 64 tiles whose two wave
// groups split K, 12.5 on 36 128 x 128 tiles).  Larger ones lose by a part-filled round: the tiles between 128 x 128 and 256 x 256
// are there for their counts (M = 8192, N = 1152, K = 4608 inside a pass: 71.8 us on 256 tiles of 256 x 144, 89.8 on 160 of 256 x 256).
// 13 and 18 are the 256 x 144 tile on two pairs of waves and on eight.  Inside a pass, eight against pairs: K = 384 (8192 x 1152) 14.0 : 17.2
// us, K = 768 (4096 x 2304) 19.7 : 22.0, K = 1152 (2560 x 3456) 24.6 : 26.9, K = 1536 (16384 x 384) 28.5 : 29.2, K = 2048 (4096 x 2048)
// 42.9 : 42.4, K = 3072 (8192 x 768) 52.5 : 48.2, K = 4608 (8192 x 1152) 81.3 : 71.8; 18's constants put the line at K = 1344.  (18 stores by
// lane swaps; with store_rows QKV of 8192 and 16384 rows of 384 13.1 -> 13.7 and 24.1 -> 25.4, GELU 22.4 -> 23.4, gated even.)
// 7 has the launches of 193 to 256 tiles of 128 x 96 (inside a pass, against the next best: 2560 x 1152 x 4608 33.7 us, 128 x 144 35.8, 128 x
// 128 39.8; 8192 x 384 x 1536 14.4, 128 x 128 15.8), on four waves by two (four by one: 35.7, 15.4).  Its base keeps launches of K <= 512 on
// 128 x 128: they would gain 0.2-0.6 us, and the other launches of a block, which then find another kernel's code in the instruction
// caches, lose as much or more (4096 rows of 256: QKV 7.1 -> 6.9, the other three 20.0 -> 21.4).
// 21 and 22 are there for rounds that the 256-row tiles of 256 and 288 columns leave part-filled.  Inside a pass of hidden 1152, against the
// tiles chosen before: 256 x 192 QKV of 3072 to 3584 rows 34 -> 30 us (one round of 216 to 252 tiles, 182 before), whole evaluations of
// 8704 to 10752 rows (K = 4608 in one round; 170 to 210 tiles of 256 x 256 before) -4 to -7 %; 192 x 288 K = 4608 of 24576 rows 204 -> 180
// (512 tiles, two whole rounds; 480 before) and of 12288 rows -3.4 to -6.6, the update of the stream at 24576 rows (K = 1152) -7, QKV of
// 12288 rows -3.9 to -7.7.  The constants of both are fitted to those launches and to those where they lose: 256 x 192 gated K = 4608
// of 16384 rows +33, GELU of 8192 and 16384 rows +7.4 and +5; 192 x 288 GELU of 12288 and 24576 rows +9.5 and +13.
struct TileModel { int id, bm, bn, wk, per_cu; double base, round, lat, thr, red0, red1; };     // red0 = 0: never split
const TileModel kTiles[] = {
    {  2, 256, 288, 1, 1, 0.00, 8.99, 1.59, 0.00, 0.0, 0.0 },
    {  3, 256, 256, 1, 1, 0.00, 7.66, 1.31, 0.00, 0.0, 0.0 },
    { 22, 192, 288, 1, 1, 0.00, 8.50, 1.18, 0.00, 0.0, 0.0 },
    { 21, 256, 192, 1, 1, 0.00, 8.60, 0.94, 0.00, 0.0, 0.0 },
    { 13, 256, 144, 1, 1, 0.10, 8.17, 0.94, 0.00, 0.0, 0.0 },
    { 18, 256, 144, 1, 1, 0.10, 6.50, 1.02, 0.00, 0.0, 0.0 },
    { 14, 256, 128, 1, 1, 0.24, 4.29, 0.85, 0.00, 0.0, 0.0 },
    { 16, 128, 144, 1, 1, 0.51, 4.58, 0.54, 0.00, 0.0, 0.0 },
    {  4, 128, 128, 1, 2, 0.98, 2.65, 0.64, 0.51, 0.0, 0.0 },
    {  5, 128, 128, 1, 1, 1.29, 2.95, 0.48, 0.00, 2.9, 1.8 },
    {  7, 128,  96, 1, 1, 1.90, 2.96, 0.42, 0.00, 0.0, 0.0 },
    { 17,  64, 144, 1, 1, 1.51, 3.13, 0.31, 0.00, 0.0, 0.0 },
    {  6, 128,  64, 1, 1, 1.50, 2.12, 0.32, 0.00, 2.9, 1.9 },
    { 11,  64,  96, 2, 1, 1.43, 2.65, 0.44, 0.00, 0.0, 0.0 },
    {  9,  64,  64, 2, 1, 1.47, 2.08, 0.37, 0.00, 2.9, 1.8 },
    {  1,  64,  64, 1, 2, 1.91, 1.40, 0.22, 0.19, 2.7, 1.8 },
    { 12,  32,  64, 2, 2, 1.98, 1.34, 0.29, 0.26, 2.9, 1.7 },
};

// Tiles 21 and 22 are for the launches they were measured ahead in: 21 a single round (of q, k, v; of other launches from 200 tiles on), 22 up
// to three rounds, but not for head-major stores whose 32 rows cross slots; neither for GELU.  The line at 200 is no crossing: below it, where
// the model would take 21 too, 21 is ahead as well (whole evaluations without : with the line, us, 14 blocks: hidden 1152 8448 rows, 198 tiles, 4808 :
// 5162, slots of 247 4907 : 5247; 1024 8448 rows 4169 : 4414; 768 11008 to 12544 rows, 172 to 196 tiles, 3463 : 3698 to 3781 : 4047; 1536 6144 rows
// 5834 : 6167).  These stay as two launches, on which a test of ragged passes stands that needs a split of this kind.  Beyond, and as one of two launches (pick_row_split), where the model puts them level or ahead, their larger
// share of fragment reads and copies costs more than a part-filled last round (hidden 1152, whole evaluations: K = 4608 of 18432
// rows in two rounds of 21 +1.3 %; 14336 and 28672 rows cut in two +2.6 %).  Against the tiles of before over 290 evaluations of hidden 384 to
// 2048, wherever the choice differs: 0 to -8 %, but for q, k, v of ragged slots at hidden 576 on more than 225 tiles (+0.4 to +1.4 %: 256 x 256 on
// eight waves was ahead there) and 22 in a round of 768 or 1280 wide models' q, k, v (5888 rows +0.7 %, 3328 and 6912 rows +0.5).
bool offered(const TileModel& t, const Epilogue& e, int M, int N)
{
    if (t.id != 21 && t.id != 22) return true;
    const bool heads = e.mode == EPI_STORE_HEADS;
    const long long tiles = (long long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
    if (e.mode == EPI_STORE_GELU) return false;
    return t.id == 21 ? tiles <= 256 && (heads || tiles >= 200) : tiles <= 768 && (!heads || e.rows_per_slot % 32 == 0);
}

double model_us(const TileModel& t, int M, int N, int K, int splits, bool leave)
{
    const long long tiles = (long long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) * splits;
    const int steps = (K / (64 * t.wk) + splits - 1) / splits;
    const long long cap = 256LL * t.per_cu, full = tiles / cap, share = (tiles - full * cap + 255) / 256;
    double us = t.base + full * (t.round + steps * fmax(t.lat, t.per_cu * t.thr));
    if (share) us += t.round + steps * fmax(t.lat, share * t.thr);
    // partials left to the next launch cost it their bytes, and the store of the row that it would not make otherwise
    if (splits > 1) us += leave ? 0.5 + 0.8e-6 * M * N * splits : t.red0 + t.red1 * 1e-6 * M * N * splits;
    return us;
}

drf_status launch_last_tiles(int v, const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int m_first);

// The 256-row tiles 2 and 3 on eight waves (20, 19) where the epilogue weighs more than the loop: four waves gain 5-10 % in the
// loop, but a SIMD's one wave has nothing to run beside its epilogue's arithmetic and address work.  Inside a pass, eight waves
// against four, 256 x 256 | 256 x 288 tiles:
//  - GELU: 8192 x 1536 x 384 18.1 : 20.5 | 20.1 : 22.0 us, 16384 x 4608 x 1152 163.7 : 170.2 | 155.3 : 162.1; 16384 x 6144 x 1536
//    281.6 : 262.6 | 303.0 : 277.8, 8192 x 8192 x 2048 226.1 : 219.7 | 241.7 : 233.7.  A single round of K = 1152
//    with weights from HBM loses on eight waves (36.9 : 33.6 to 36.9 : 35.4 at 2520 to 3276 rows; two stages wait for them at every k-tile), but
//    every launch's weights are asked for by the one before: 216 to 255 tiles gain 1.6 to 2.9 us (3072 to 3584 rows; whole evaluations -0.3
//    to -0.9 %, hidden 1024 at 224 and 240 tiles -0.9), fewer do not (208 tiles +2 %), and a full round is even (4096 rows 0 to -1.2).  So do the
//    first of two launches (3584 rows of 4352 to 5632: whole evaluations -0.7 to -1.0 %, hidden 1280 -0.3 to -0.7); as the second one
//    it is even (7424 and 7680 rows -0.3 and -0.6 %, 11520 and 11776 rows +0.7 and -0.2, where runs differ by 0.5);
//  - head-major planes, slots of whole 32-row passes: K = 384 17.9 : 18.8 | 21.1 : 21.6, K = 512 even (19.60 : 19.56 | 21.0 : 21.9),
//    K = 768 22.5 : 22.2 | 25.0 : 24.7, K = 1152 34.5 : 31.8 | 121.1 : 110.1;
//  - other slot lengths: K = 768 42.9 : 43.8 | 30.3 : 32.1, K = 1152 128.6 : 138.9 | 112.4 : 118.9, K = 2048 101.9 : 96.2 | 110.9 : 106.6; a
//    single round of K = 1152 30.7 : 31.2 | 39.7 : 42.0, and a whole evaluation with the former 4.74 : 4.69 ms.
// Gated, residual and plain stores stay on four at every K (24576 x 1152 x 1152 plain 70.8 : 63.0, residual 106.8 : 102.5, gated even).
int wide_form(int tile, int rows, int N, int K, const Epilogue& e)
{
    if (tile != 2 && tile != 3) return tile;
    const int cols = tile == 2 ? 288 : 256;
    const long long tiles = ((rows + 255) / 256) * (long long)((N + cols - 1) / cols);
    const bool one_round = tiles <= 256, part_filled = tile == 3 && tiles >= 216 && tiles < 256;
    const bool eight = e.mode == EPI_STORE_GELU ? K < (one_round && !part_filled ? 1024 : 1536)
                                                : e.mode == EPI_STORE_HEADS && K < (e.rows_per_slot % 32 == 0 ? 512 : tile == 3 && one_round ? 1024 : 1536);
    return !eight ? tile : tile == 2 ? 20 : 19;
}

// Rows m_first .. M - 1 of the problem with tile v (m_first a multiple of the tile's height).
drf_status launch_tile(int v, const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int m_first)
{
    if (e.mode == EPI_STORE_GELU && e.out_f32 && (v == 2 || v == 3)) v = 14;      // (the 4-wave tiles have no such store)
    switch (v) {
    case 1: return launch_bf16_xl<64, 64, 64, 4, 2, 2>(A, W, M, N, K, e, st, m_first);
    case 2: return launch_gemm_wide_288(A, W, M, N, K, e, st, m_first);
    case 3: return launch_gemm_wide_256(A, W, M, N, K, e, st, m_first);
    case 4: return launch_bf16_xl<128, 128, 64, 2, 4, 2, 1, true>(A, W, M, N, K, e, st, m_first);
    case 6: return launch_bf16_xl<128, 64, 64, 4, 4, 2>(A, W, M, N, K, e, st, m_first);
    case 8:                                         // (16 for whole pairs of k-tiles only, as this number has always been)
        if (K % 128 != 0) DRF_FAIL(DRF_ESHAPE, "bf16 GEMM tile needs K %% 128 == 0 (K=%d)", K);
        [[fallthrough]];
    case 13: case 16: case 17: return launch_gemm_pair(v, A, W, M, N, K, e, st, m_first);
    case 9: return launch_bf16_xl<64, 64, 64, 3, 2, 2, 2>(A, W, M, N, K, e, st, m_first);
    case 11: return launch_bf16_xl<64, 96, 64, 3, 2, 2, 2>(A, W, M, N, K, e, st, m_first);
    case 12: return launch_bf16_xl<32, 64, 64, 3, 1, 2, 2>(A, W, M, N, K, e, st, m_first);
    case 7: case 18: case 19: case 20: case 21: case 22: return launch_last_tiles(v, A, W, M, N, K, e, st, m_first);
    case 14: return launch_bf16_xl<256, 128, 64, 3, 4, 2, 1, true>(A, W, M, N, K, e, st, m_first);
    default: return launch_bf16_xl<128, 128, 64, 4, 4, 2>(A, W, M, N, K, e, st, m_first);      // 5, or a number that names no tile
    }
}

// A problem that fills some rounds of a tile and part of another runs as two launches where that is modelled at least 5 %
// faster: the rows of the full rounds with that tile, the rest with whatever suits it (6144 x 3456 x 1152 inside a pass: 5376 rows of
// 256 x 288 tiles and the rest of 128 x 96 50.5 us, the best single launch 57.5).
// Returns the rows of the first launch, 0 for one launch.
int pick_row_split(int M, int N, int K, double one_us, int* id_a, int* id_b)
{
    double best = 0.95 * one_us;
    int rows = 0;
    for (const TileModel& a : kTiles) {
        const long long tn = (N + a.bn - 1) / a.bn, cap = 256LL * a.per_cu, rounds = M / a.bm * tn / cap;
        if (rounds < 1 || K % (64 * a.wk) != 0 || a.id == 21 || a.id == 22) continue;
        const int ra = (int)(rounds * cap / tn) * a.bm;
        if (ra == 0 || ra >= M) continue;
        const double ua = model_us(a, ra, N, K, 1, false);
        for (const TileModel& b : kTiles) {
            if (K % (64 * b.wk) != 0 || ra % b.bm != 0 || b.id == 21 || b.id == 22) continue;
            const double us = ua + model_us(b, M - ra, N, K, 1, false);
            if (us < best) { best = us; rows = ra; *id_a = a.id; *id_b = b.id; }
        }
    }
    return rows;
}

// The tile and split with the least modelled time.  Two K groups need whole pairs of k-tiles; a split leaves every
// part at least two k-steps and its partial tiles must fit the scratch.
double pick_tile(int M, int N, int K, const Epilogue& e, bool may_split, bool leave, int* id, int* splits)
{
    double best = 1e300;
    for (const TileModel& t : kTiles) {
        if (K % (64 * t.wk) != 0 || !offered(t, e, M, N)) continue;
        const size_t tile_floats = (size_t)((M + t.bm - 1) / t.bm) * t.bm * ((size_t)((N + t.bn - 1) / t.bn) * t.bn);
        const int most = may_split && t.red0 > 0.0 && tile_floats / (t.bm * t.bn) < 512 ? kMaxSplits : 1;   // (enough tiles fill the chip unsplit)
        for (int s2 = 1; s2 <= most; ++s2) {
            if (s2 > 1 && (K / (64 * t.wk) < 2 * s2 || tile_floats * s2 > kSplitKScratchFloats)) break;
            const double us = model_us(t, M, N, K, s2, leave);
            if (us < best) { best = us; *id = t.id; *splits = s2; }
        }
    }
    return best;
}

}  // namespace

size_t gemm_splitk_scratch_bytes() { return kSplitKScratchFloats * sizeof(float); }

GemmRoute gemm_route(int M, int N, int K, const Epilogue& e, bool may_split, bool leave)
{
    GemmRoute r{ 0, 1, 0, 0 };
    const double us = pick_tile(M, N, K, e, may_split, leave, &r.tile, &r.splits);
    if (r.splits == 1 && M >= 2048) r.first_rows = pick_row_split(M, N, K, us, &r.first_tile, &r.tile);
    r.tile = wide_form(r.tile, M - r.first_rows, N, K, e);
    r.first_tile = wide_form(r.first_tile, r.first_rows, N, K, e);
    return r;
}

drf_status launch_gemm_bf16(const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st,
                            int variant, float* splitk_scratch, PartialSum* leave)
{
    if (leave) leave->splits = 0;
    if (M == 0 || N == 0) return DRF_OK;
    if (K % 64 != 0 || N % 4 != 0 || e.ldo % 4 != 0) DRF_FAIL(DRF_ESHAPE, "bf16 GEMM needs K %% 64 == 0 and N %% 4 == 0 (M=%d N=%d K=%d)", M, N, K);
    if (e.mode == EPI_STORE_HEADS && (e.out_f32 || e.hd % 8 != 0 || e.hid % 16 != 0 || N % e.hid != 0))
        DRF_FAIL(DRF_ESHAPE, "head-major store needs bf16 output, head width %% 8 == 0 and hidden %% 16 == 0");
    if (e.mode == EPI_STORE_GATED && (e.out_f32 || !e.gate)) DRF_FAIL(DRF_ESHAPE, "gated store needs bf16 output and a gate");
    if (e.mode == EPI_STORE_SILU) DRF_FAIL(DRF_ESHAPE, "the SiLU store is an epilogue of the fp32 GEMM");
    if ((size_t)M * K >= ((size_t)1 << 31) || (size_t)N * K >= ((size_t)1 << 31))
        DRF_FAIL(DRF_ESHAPE, "bf16 GEMM operand exceeds 2^31 elements");
    int v = variant, splits = 1, va = 0, rows_a = 0;
    if (v == 0) {
        const GemmRoute r = gemm_route(M, N, K, e, splitk_scratch != nullptr, leave != nullptr);
        v = r.tile; splits = r.splits; va = r.first_tile; rows_a = r.first_rows;
    } else if (v >= 100) {
        splits = v / 100;
        v %= 100;
    } else if (v == 10) {
        v = 5;
        const int tiles = ((M + 127) / 128) * ((N + 127) / 128), nk = K / 64;
        for (int s2 = 2; splitk_scratch && s2 <= 8 && s2 * tiles <= 256; ++s2)
            if (nk / s2 >= 6) splits = s2;
    }
    if (splits > 1) {
        switch (v) {
        case 1: return launch_bf16_splitk<64, 64, 64, 4, 2, 2>(A, W, M, N, K, e, st, splits, splitk_scratch, leave);
        case 5: return launch_bf16_splitk<128, 128, 64, 4, 4, 2>(A, W, M, N, K, e, st, splits, splitk_scratch, leave);
        case 6: return launch_bf16_splitk<128, 64, 64, 4, 4, 2>(A, W, M, N, K, e, st, splits, splitk_scratch, leave);
        case 9: return launch_bf16_splitk<64, 64, 64, 3, 2, 2, 2>(A, W, M, N, K, e, st, splits, splitk_scratch, leave);
        case 12: return launch_bf16_splitk<32, 64, 64, 3, 1, 2, 2>(A, W, M, N, K, e, st, splits, splitk_scratch, leave);
        default: DRF_FAIL(DRF_EINVAL, "GEMM tile %d has no split form", v);
        }
    }
    if (rows_a) {
        Epilogue ea = e;
        ea.warm_lines = 0;                          // the second launch is the one whose last round warms the caches
        const drf_status rc = launch_tile(va, A, W, rows_a, N, K, ea, st, 0);
        if (rc != DRF_OK) return rc;
    }
    return launch_tile(v, A, W, M, N, K, e, st, rows_a);
}

// Whether a problem is for the 16 x 16 tiles: so few 32 x 32 tiles that a launch is one chain of round trips, which then only
// gets shorter with more and smaller workgroups.  (M = 64: K = 512, N = 128 7.2 -> 5.1 us, K = N = 128 5.3 -> 3.6;
// a call of configuration 1 1047 -> 675 us.  With the small tiles' waves and batches on 32 x 32 tiles, 16384 rows of 1024 lose 23 %.)
bool f32_small(int M, int N) { return ((M + 31LL) / 32) * ((N + 31LL) / 32) <= 128; }

template <bool LN>
static drf_status launch_f32(const float* A, const float* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int a_row_mod, const RowNorm& ln)
{
    if (M == 0 || N == 0) return DRF_OK;
    if (N % 4 != 0 || e.ldo % 4 != 0) DRF_FAIL(DRF_ESHAPE, "fp32 GEMM needs N %% 4 == 0 (N=%d)", N);
    if (!e.out_f32 || e.mode == EPI_STORE_HEADS || e.mode == EPI_STORE_GATED) DRF_FAIL(DRF_ESHAPE, "epilogue mode of the bf16 GEMM");
    uintptr_t bases = reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(W);
    if (LN) bases |= reinterpret_cast<uintptr_t>(ln.shift) | reinterpret_cast<uintptr_t>(ln.scale) | (uintptr_t)(ln.mod_ld % 4);
    const bool vec = K % 4 == 0 && (bases & 15u) == 0;
    auto go = [&](auto f_c, auto nw_c, auto b_c) {
        constexpr int F = decltype(f_c)::value, NW = decltype(nw_c)::value, B = decltype(b_c)::value, T = 16 * F;
        const long long tiles_m = ((long long)M + T - 1) / T;
        const dim3 grid((unsigned)((N + T - 1LL) / T), (unsigned)(tiles_m < 65535 ? tiles_m : 65535));
        if (vec) hipLaunchKernelGGL((gemm_f32_kernel<true, F, NW, B, LN>), grid, dim3(NW * 64), 0, st, A, W, M, N, K, a_row_mod, e, ln);
        else hipLaunchKernelGGL((gemm_f32_kernel<false, F, NW, B, LN>), grid, dim3(NW * 64), 0, st, A, W, M, N, K, a_row_mod, e, ln);
    };
    constexpr std::integral_constant<int, 1> one{};
    constexpr std::integral_constant<int, 2> two{};
    constexpr std::integral_constant<int, 4> four{};
    if (LN || f32_small(M, N)) {
        if (K <= 128) go(one, four, four);
        else go(one, std::integral_constant<int, 8>{}, four);
    } else if constexpr (!LN) go(two, four, two);
    DRF_HIP(hipGetLastError());
    return DRF_OK;
}

drf_status launch_gemm_f32(const float* A, const float* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int a_row_mod)
{
    return launch_f32<false>(A, W, M, N, K, e, st, a_row_mod, RowNorm{});
}

bool gemm_f32_folds_ln(int M, int N, int K) { return K <= 512 && f32_small(M, N); }

drf_status launch_gemm_f32_ln(const float* resid, const RowNorm& ln, const float* W, int M, int N, int K, const Epilogue& e, hipStream_t st)
{
    if (!gemm_f32_folds_ln(M, N, K)) DRF_FAIL(DRF_ESHAPE, "LayerNorm inside the fp32 GEMM is for few rows of at most 512 (M=%d N=%d K=%d)", M, N, K);
    return launch_f32<true>(resid, W, M, N, K, e, st, 0, ln);
}

namespace {

// Tiles 7 and 18 to 22, at the end of the file so that their code lies behind that of the others: between the kernels of small problems, whose
// launches are as long as a few misses of the instruction cache, it costs passes of 1500 to 2000 rows of hidden 384 1 % (six passes of 24
// slots of 63 tokens 3.29 -> 3.26 ms, of 32 slots 3.43 -> 3.38).
drf_status launch_last_tiles(int v, const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int m_first)
{
    switch (v) {
    case 7: return launch_bf16_xl<128, 96, 64, 3, 4, 2>(A, W, M, N, K, e, st, m_first);
    case 18: return launch_bf16_xl<256, 144, 64, 3, 8, 1>(A, W, M, N, K, e, st, m_first);
    case 19: return launch_bf16_xl<256, 256, 64, 2, 4, 2>(A, W, M, N, K, e, st, m_first);
    case 21: return launch_gemm_wide_192(A, W, M, N, K, e, st, m_first);
    case 22: return launch_gemm_wide_192x288(A, W, M, N, K, e, st, m_first);
    default: return launch_bf16_xl<256, 288, 64, 2, 4, 2>(A, W, M, N, K, e, st, m_first);
    }
}

}  // namespace

}  // namespace drf
