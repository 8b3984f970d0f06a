// bf16 GEMM at middle tiles: four waves, one per SIMD, in two pairs; a pair takes every k-tile's first k-step of 32, the other
// pair the second, a wave half of the tile's rows and all of its columns.
//
// What bounds these tiles is the LDS: fragment reads and copies share it (128 x 144: a k-tile takes 0.31 us without the copies,
// 0.37 without the reads, 0.60 with both; the MFMAs 0.26).  Halving K between the pairs makes the waves' tiles as large as
// the accumulators allow, 64 x 144 of a 128 x 144 tile, where four row blocks that share K by k-tiles read 90 KB a k-tile; now
// 53.  Fragments are double-buffered a k-tile ahead, so a stage is free as soon as its k-tile begins and one block
// barrier a k-tile does for both hand-overs.  Back to back with warm weights, 8-wave forms before: 8192 x 1152 x 4608 77.9 -> 66.0 us
// (256 x 144), 4096 x 1152 x 4608 44.3 -> 38.7 (128 x 144), 2048 x 1152 x 4608 33.7 (128 x 96) -> 26.0 (64 x 144).
// Inside a pass of 4096 rows: 128 x 144 at K = 4608 48.7 -> 43.1, at K = 1152 19.1 -> 17.5.  Below K = 1400 the exchange of the
// partial sums and the one wave's epilogue cost the 256 x 144 tile more than the loop gains, and it runs on eight waves (tile 18
// in gemm.hip).
// Four more waves that only copy gained nothing (38.7 -> 42.8, 66.0 -> 64.0), copies by way of registers lost 20-40 %.
#pragma once
#include "gemm_device.h"

namespace drf {

namespace {

__host__ __device__ constexpr int pair_lds_rows_at(int BM, int BN, int NS) { return NS * (BM + BN) * 128; }

template <int BM, int BN, int NS>
__global__ void __launch_bounds__(256, 1)
gemm_bf16_pair_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, int M, int N, int K, const Epilogue e,
                      int tiles_m, int tiles_n, int m_first)
{
    constexpr int TM = BM / 2, TN = BN, MI = TM / 16, NI = TN / 16, S = MI * NI, RD = MI + NI;
    constexpr int STAGE = (BM + BN) * 128, SEG = (BM + BN) / 8, NL = (SEG + 3) / 4;          // bytes of a stage; copies per wave
    constexpr int ROWS = pair_lds_rows_at(BM, BN, NS), DUMMY = ROWS + epi_lds_bytes(BN);
    constexpr int GROUP_M = 8, AGPR = S < 60 ? S : 60;
    static_assert(BM % 32 == 0 && BN % 16 == 0 && (BM + BN) % 8 == 0, "tile shape");
    extern __shared__ __attribute__((aligned(128))) unsigned char smem_raw[];

    const int nb = tiles_m * tiles_n, b = blockIdx.x;
    const int xcd = b & 7, local = b >> 3, q = nb >> 3, rem = nb & 7;
    const int idx = xcd * q + (xcd < rem ? xcd : rem) + local;
    const int per_group = GROUP_M * tiles_n, group = idx / per_group, first_m = group * GROUP_M;
    const int gsz = tiles_m - first_m < GROUP_M ? tiles_m - first_m : GROUP_M;
    const int tm = first_m + (idx % per_group) % gsz, tn = (idx % per_group) / gsz;
    const int m0 = m_first + tm * BM, n0 = tn * BN, nk = K / 64;

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, quarter = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave & 1, wk = wave >> 1;

    // Copies: a wave-wide instruction moves 8 rows of 128 bytes of the stage's row space (BM activation rows, BN weight rows);
    // wave w takes NL in a row, the surplus ones of the last wave repeat the last segment
    uint32_t voff[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        int g = wave * NL + i; g = g < SEG ? g : SEG - 1;
        const int r = g * 8 + (lane >> 3), chunk = (lane & 7) ^ ((r >> 1) & 7);
        int row = g * 8 < BM ? m0 + r : n0 + r - BM;
        const int last = (g * 8 < BM ? M : N) - 1;
        row = row < last ? row : last;
        voff[i] = ((uint32_t)row * (uint32_t)K + (uint32_t)chunk * 8u) * 2u;
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(DRF_LDS_AS unsigned char*)smem_raw;
    auto copy_one = [&](auto ic, int kt, uint32_t so) {
        constexpr int i = decltype(ic)::value;
        int g = wave * NL + i; g = g < SEG ? g : SEG - 1;
        const bf16_t* base = (g * 8 < BM ? A : W) + kt * 64;
        const uint32_t dst = lds0 + so + (uint32_t)g * 1024u, vo = voff[i];
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(dst), "v"(vo), "s"(base) : "memory");
    };

    f32x4 acc[NI][MI];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j) acc[i][j] = (f32x4){ 0.f, 0.f, 0.f, 0.f };
    u32x4 fa[2][MI], fw[2][NI];
    const int pos = ((wk * 4 + quarter) ^ ((l16 >> 1) & 7)) * 16;
    const uint32_t a0 = lds0 + (uint32_t)(wm * TM + l16) * 128u + pos, w0 = lds0 + (uint32_t)(BM + l16) * 128u + pos;
    // r-th fragment read of a k-tile: the first weight fragment, the activation fragments, the other weight fragments
    auto read_one = [&](auto rc, auto sc, uint32_t so) {
        constexpr int r = decltype(rc)::value, s = decltype(sc)::value;
        if constexpr (r == 0) lds_read16<0>(fw[s][0], w0 + so);
        else if constexpr (r <= MI) lds_read16<(r - 1) * 2048>(fa[s][r - 1], a0 + so);
        else lds_read16<(r - MI) * 2048>(fw[s][r - MI], w0 + so);
    };
    auto hold_set = [&](auto sc) {
        constexpr int s = decltype(sc)::value;
        static_for<0, MI>([&](auto jc) { hold_frag(fa[s][decltype(jc)::value]); });
        static_for<0, NI>([&](auto ic) { hold_frag(fw[s][decltype(ic)::value]); });
    };

    static_for<0, NL>([&](auto ic) { copy_one(ic, 0, 0u); });
    const GateRows gr = gate_rows<BM>(e, m0, M);
    stage_epilogue_rows<BN>(e, gr, lds0 + ROWS, wave, 4, n0, N);
#pragma unroll
    for (int t = 1; t < NS; ++t)
        if (t < nk) static_for<0, NL>([&](auto ic) { copy_one(ic, t, (uint32_t)(t * STAGE)); });
    if (nk >= NS) wait_vmcnt<NL * (NS - 1)>(); else wait_vmcnt<0>();
    asm volatile("s_barrier" ::: "memory");
    warm_caches(e, lds0 + DUMMY, nb, b, wave, 4);
    if (nk == 1) wait_vmcnt<0>();                   // (otherwise the last k-tile's wait covers it)
    static_for<0, S>([&](auto pc) { constexpr int p = decltype(pc)::value; hold_acc<(p < AGPR)>(acc[p / MI][p % MI]); });
    settle_mfma();

    // One k-tile: its fragments are in set P, so its stage is free once every wave is here; the next k-tile's are read
    // into the other set, and the copy of k-tile kt + NS refills the stage.  YOUNGER: k-tiles whose copies were requested
    // after the next one's (-1: there is no next one).
    constexpr int RSTEP = (S - 8) / RD < 1 ? 1 : (S - 8) / RD, LSTEP = (S - 1) / NL < 1 ? 1 : (S - 1) / NL;
    static_assert(RSTEP * RD <= S && 1 + LSTEP * (NL - 1) < S, "schedule");
    int cs = 0;                                     // stage of k-tile kt
    auto tile = [&](auto set_c, auto load_c, auto younger_c, int kt) {
        constexpr int P = decltype(set_c)::value, YOUNGER = decltype(younger_c)::value;
        constexpr bool LOAD = decltype(load_c)::value, NEXT = YOUNGER >= 0;
        const int ns = cs + 1 == NS ? 0 : cs + 1;
        const uint32_t so = (uint32_t)cs * STAGE, no = (uint32_t)ns * STAGE;
        if constexpr (NEXT) { wait_vmcnt<YOUNGER * NL>(); asm volatile("s_barrier" ::: "memory"); }
        static_for<0, S>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            if constexpr (NEXT && m % RSTEP == 0 && m / RSTEP < RD) read_one(std::integral_constant<int, m / RSTEP>{}, std::integral_constant<int, 1 - P>{}, no);
            if constexpr (LOAD && m >= 1 && (m - 1) % LSTEP == 0 && (m - 1) / LSTEP < NL)
                copy_one(std::integral_constant<int, (m - 1) / LSTEP>{}, kt + NS, so);
            constexpr int i = m / MI, j = i & 1 ? MI - 1 - m % MI : m % MI;      // snake: one operand changes per MFMA
            mfma<(i * MI + j < AGPR)>(acc[i][j], fw[P][i], fa[P][j]);
        });
        if constexpr (NEXT) { wait_lgkmcnt<0>(); hold_set(std::integral_constant<int, 1 - P>{}); }
        cs = ns;
    };
    // k-tile kt takes set (nk - 1 - kt) & 1, so that the last ones' sets are known
    auto first_reads = [&](auto sc) {
        static_for<0, RD>([&](auto rc) { read_one(rc, sc, 0); });
        wait_lgkmcnt<0>();
        hold_set(sc);
    };
    constexpr std::integral_constant<int, 0> C0{};
    constexpr std::integral_constant<int, 1> C1{};
    if ((nk - 1) & 1) first_reads(C1); else first_reads(C0);
    constexpr std::integral_constant<int, (NS - 1) & 1> PA{};       // set of a k-tile NS (+ 2, 4, ..) before the end
    constexpr std::integral_constant<int, NS & 1> PB{};
    constexpr std::integral_constant<int, NS - 2> YA{};
    int kt = 0;
    if (nk > NS && ((nk - NS) & 1)) { tile(PB, std::true_type{}, YA, 0); kt = 1; }
    for (; kt + NS < nk; kt += 2) {
        tile(PA, std::true_type{}, YA, kt);
        tile(PB, std::true_type{}, YA, kt + 1);
    }
    static_for<0, NS>([&](auto tc) {
        constexpr int left = NS - 1 - decltype(tc)::value;          // k-tiles after this one
        if (nk > left) tile(std::integral_constant<int, left & 1>{}, std::false_type{}, std::integral_constant<int, left - 1>{}, nk - 1 - left);
    });
    settle_mfma();
    static_for<0, S>([&](auto pc) { constexpr int p = decltype(pc)::value; hold_acc<(p < AGPR)>(acc[p / MI][p % MI]); });

    // The pairs' partial sums meet in LDS: with an even number of 32-row blocks each pair finishes half of the rows, otherwise
    // the first pair all of them.
    constexpr bool HALVES = MI % 4 == 0;
    constexpr int MF = HALVES ? MI / 2 : MI, PART = 4 * NI * MF * 1024;
    static_assert(PART / (HALVES ? 1 : 2) <= NS * STAGE, "LDS too small for the partial sums");
    asm volatile("s_barrier" ::: "memory");         // every wave has read its last fragments
    f32x4* part = reinterpret_cast<f32x4*>(smem_raw);
    f32x4 fin[NI][MF];
    if constexpr (HALVES) {
        auto give = [&](auto jc) {                  // pieces of the other pair's half
            constexpr int j0 = decltype(jc)::value;
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < MF; ++j) part[(wave * NI * MF + i * MF + j) * 64 + lane] = acc[i][j0 + j];
        };
        if (wk == 0) give(std::integral_constant<int, MF>{}); else give(C0);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        auto take = [&](auto jc) {
            constexpr int j0 = decltype(jc)::value;
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < MF; ++j) fin[i][j] = acc[i][j0 + j] + part[((wave ^ 2) * NI * MF + i * MF + j) * 64 + lane];
        };
        if (wk == 0) take(C0); else take(std::integral_constant<int, MF>{});
    } else {
        if (wk == 1) {
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < MI; ++j) part[(wm * NI * MI + i * MI + j) * 64 + lane] = acc[i][j];
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (wk == 1) return;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < MI; ++j) fin[i][j] = acc[i][j] + part[(wm * NI * MI + i * MI + j) * 64 + lane];
    }
    const int mw = m0 + wm * TM + (HALVES ? wk * (TM / 2) : 0);
    const unsigned char* erows = smem_raw + ROWS;
    if (may_store_rows<BM, BN>(e, m0, n0, M, N, gr)) {
        // (a wave's rows in LDS take the place of partial sums: all are read)
        if constexpr (HALVES) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        constexpr int FIN = MF * 16;
        unsigned char* wbuf = HALVES ? smem_raw + wave * rows_tile_bytes(FIN, TN) : smem_raw + PART / 2 + wm * rows_tile_bytes(FIN, TN);
        static_assert(HALVES ? 4 * rows_tile_bytes(FIN, TN) <= NS * STAGE : PART / 2 + 2 * rows_tile_bytes(FIN, TN) <= NS * STAGE, "LDS");
        if (e.mode == EPI_STORE_GELU) store_rows<FIN, TN, EPI_STORE_GELU, 0>(fin, e, mw, n0, wbuf, erows, 0);
        else if (e.mode == EPI_STORE_HEADS) store_rows<FIN, TN, EPI_STORE_HEADS, 0>(fin, e, mw, n0, wbuf, erows, 0);
        else if (e.mode == EPI_STORE_GATED) store_rows<FIN, TN, EPI_STORE_GATED, 1>(fin, e, mw, n0, wbuf, erows, epi_row_bytes(BN));
        else store_rows<FIN, TN, EPI_STORE, 0>(fin, e, mw, n0, wbuf, erows, 0);
        return;
    }
    store_tile<MF * 16, TN, true>(fin, e, mw, n0, M, N, erows, epi_row_bytes(BN), gr);
}

template <int BM, int BN, int NS>
drf_status launch_pair(const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int m_first)
{
    constexpr size_t smem = pair_lds_rows_at(BM, BN, NS) + epi_lds_bytes(BN) + 256;
    static_assert(smem <= 160 * 1024, "LDS of a CU");
    static bool attr_set = false;
    auto kern = gemm_bf16_pair_kernel<BM, BN, NS>;
    if (!attr_set) {
        DRF_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        attr_set = true;
    }
    const int tiles_m = (M - m_first + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(256), smem, st, A, W, M, N, K, e, tiles_m, tiles_n, m_first);
    DRF_HIP(hipGetLastError());
    return DRF_OK;
}

}  // namespace

}  // namespace drf
