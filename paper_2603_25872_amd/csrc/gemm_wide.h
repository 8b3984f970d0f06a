// bf16 GEMM at tiles of 256 or 192 rows for problems that fill the chip with them: four waves, one per SIMD, each with a
// quarter of the tile (128 x 144, 128 x 128, 128 x 96 or 96 x 144) and a SIMD's whole register file.
//
// Against the 8-wave form of the same tile (64 x 144 per wave) the fragment reads of a k-tile fall from 213 to 139 KB, which
// with the 70 KB that the copies write was 96 % of what the LDS port moves in the k-tile's MFMA time and is now 70 %.  What is
// left of a long loop is held by power (8192 x 8192 x 8192, 256 columns: 1310 -> 1520 TFLOP/s with random operands, 1420 -> 1850 with
// zeros).  Inside a pass of 16384 rows (hidden 1152): gated K = 4608 135.1 -> 122.4 us and K = 1152 43.2 -> 39.8, QKV 120.6 -> 114.1;
// the GELU launch did not gain (166.3 and 166.7, 639 -> 562 back to back at 65536 rows): a quarter of a K = 1152 round lies outside the
// loop, where one wave per SIMD has nothing beside it, and such launches run on eight waves (wide_form in gemm.hip).
//  - one wave per SIMD hides nothing behind another wave, so the loop is a fixed sequence: both k-steps' fragments are
//    double-buffered in registers, every MFMA slot has at most one LDS read or one copy beside it, and nothing but the two
//    block barriers of a k-tile waits.  Accumulators are named by inline assembly (AGPRs as far as they go): left to the
//    compiler, 256 of them are copied about;
//  - copies go out one per 7 MFMAs over the whole k-tile: the vector-memory path takes one per ~17 cycles and CU, and a
//    wave that meets it busy issues no MFMA meanwhile (one per 2: 10 % slower, all at once: 14 %);
//  - two barriers: a stage is free once every wave has read its second k-step (slot REL), the next one is needed only from
//    slot LAND of the second k-step on; with one barrier for both, the copies have 40 % less time to land (6-9 % slower);
//  - epilogue: see store_rows; bias and gate rows wait in LDS.
#pragma once
#include "gemm_device.h"

namespace drf {

namespace {

// Accumulator pieces kept in AGPRs (of at most 72; 256 registers there, the rest with the fragments in VGPRs).
constexpr int kAgprPieces = 60;
__host__ __device__ constexpr int wide_rows_at(int BM, int BN)
{
    const int stages = 2 * (BM + BN) * 128, tiles = 4 * rows_tile_bytes(BM / 2, BN / 2);
    return stages > tiles ? stages : tiles;
}

template <int BM, int BN, int MODE, bool F32>
__global__ void __launch_bounds__(256, 1)
gemm_bf16_wide_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, int M, int N, int K, const Epilogue e,
                      int tiles_m, int tiles_n, int m_first)
{
    constexpr int TM = BM / 2, TN = BN / 2, MI = TM / 16, NI = TN / 16, S = MI * NI, RD = MI + NI;
    constexpr int STAGE = (BM + BN) * 128, NLA = BM / 32, NLW = BN / 32, NL = NLA + NLW;     // bytes of a stage; copies per wave
    constexpr int GROUP_M = 8;
    // LDS: two stages, later the waves' tiles in rows | epilogue rows | 256 bytes nobody reads
    constexpr int ROWS = wide_rows_at(BM, BN), DUMMY = ROWS + epi_lds_bytes(BN);
    static_assert(BM % 32 == 0 && BN % 32 == 0, "tile shape");
    extern __shared__ __attribute__((aligned(128))) unsigned char smem_raw[];

    const int nb = tiles_m * tiles_n, b = blockIdx.x;
    const int xcd = b & 7, local = b >> 3, q = nb >> 3, rem = nb & 7;
    const int idx = xcd * q + (xcd < rem ? xcd : rem) + local;
    const int per_group = GROUP_M * tiles_n, group = idx / per_group, first_m = group * GROUP_M;
    const int gsz = tiles_m - first_m < GROUP_M ? tiles_m - first_m : GROUP_M;
    const int tm = first_m + (idx % per_group) % gsz, tn = (idx % per_group) / gsz;
    const int m0 = m_first + tm * BM, n0 = tn * BN, nk = K / 64;

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, quarter = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave & 1, wn = wave >> 1;

    // Copies: a wave-wide instruction moves 8 rows of 128 bytes; wave w takes the activation rows [w BM/4, ..) and the
    // weight rows [w BN/4, ..) of a k-tile.
    uint32_t voff[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int r = (i < NLA ? wave * (BM / 4) + i * 8 : wave * (BN / 4) + (i - NLA) * 8) + (lane >> 3);
        const int chunk = (lane & 7) ^ ((r >> 1) & 7);
        int row = i < NLA ? m0 + r : n0 + r;
        const int last = (i < NLA ? M : N) - 1;
        row = row < last ? row : last;
        voff[i] = ((uint32_t)row * (uint32_t)K + (uint32_t)chunk * 8u) * 2u;
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(DRF_LDS_AS unsigned char*)smem_raw;
    const uint32_t dst_a = lds0 + (uint32_t)wave * (BM / 4) * 128u, dst_w = lds0 + (uint32_t)(BM + wave * (BN / 4)) * 128u;
    auto copy_one = [&](auto ic, int kt, uint32_t so) {
        constexpr int i = decltype(ic)::value;
        const bf16_t* base = (i < NLA ? A : W) + kt * 64;
        const uint32_t dst = (i < NLA ? dst_a : dst_w) + so;
        constexpr int step = (i < NLA ? i : i - NLA) * 1024;
        const uint32_t vo = voff[i];
        asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"
                     :: "s"(dst), "n"(step), "v"(vo), "s"(base) : "memory", "scc");
    };

    f32x4 acc[NI][MI];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j) acc[i][j] = (f32x4){ 0.f, 0.f, 0.f, 0.f };

    u32x4 fa[2][MI], fw[2][NI];
    const int pos0 = (quarter ^ ((l16 >> 1) & 7)) * 16, pos1 = ((4 + quarter) ^ ((l16 >> 1) & 7)) * 16;
    const uint32_t a_row = lds0 + (uint32_t)(wm * TM + l16) * 128u, w_row = lds0 + (uint32_t)(BM + wn * TN + l16) * 128u;
    const uint32_t a0 = a_row + pos0, a1 = a_row + pos1, w0 = w_row + pos0, w1 = w_row + pos1;
    // r-th fragment read of a k-step: the first weight fragment, the activation fragments, the other weight fragments
    auto read_one = [&](auto rc, auto sc, uint32_t aa, uint32_t wa) {
        constexpr int r = decltype(rc)::value, s = decltype(sc)::value;
        if constexpr (r == 0) lds_read16<0>(fw[s][0], wa);
        else if constexpr (r <= MI) lds_read16<(r - 1) * 2048>(fa[s][r - 1], aa);
        else lds_read16<(r - MI) * 2048>(fw[s][r - MI], wa);
    };
    auto hold_set = [&](auto sc) {
        constexpr int s = decltype(sc)::value;
        static_for<0, MI>([&](auto jc) { hold_frag(fa[s][decltype(jc)::value]); });
        static_for<0, NI>([&](auto ic) { hold_frag(fw[s][decltype(ic)::value]); });
    };
    // schedule of a k-tile (see tile below): reads every RSTEP slots; REL, LAND: slots of the two barriers; copies from LFIRST on, one every LSTEP
    // slots, the FIRST_TILE first of them in the tile whose stage they refill, the others in the next tile
    constexpr int RSTEP = 2, REL = RSTEP * RD + 2, LAND = S + 24 < 2 * S - RSTEP * RD ? S + 24 : 2 * S - RSTEP * RD, LFIRST = REL + 1, LSTEP = 7;
    constexpr int FIRST_TILE = (2 * S - LFIRST + LSTEP - 1) / LSTEP < NL ? (2 * S - LFIRST + LSTEP - 1) / LSTEP : NL;
    static_assert(REL < S && LAND + RSTEP * RD <= 2 * S && LFIRST + (NL - 1) * LSTEP - 2 * S < REL, "schedule");
    auto copies_before = [](int slot) constexpr { return (slot - LFIRST + LSTEP - 1) / LSTEP < NL ? (slot - LFIRST + LSTEP - 1) / LSTEP : NL; };
    auto copy_at = [](int m) constexpr {            // the copy issued at slot m of a tile, -1: none
        for (int c = 0; c < NL; ++c)
            if ((LFIRST + c * LSTEP) % (2 * S) == m) return c;
        return -1;
    };
    constexpr auto C0 = std::integral_constant<int, 0>{};
    constexpr auto C1 = std::integral_constant<int, 1>{};

    static_for<0, NL>([&](auto ic) { copy_one(ic, 0, 0); });
    const GateRows gr = gate_rows<BM>(e, m0, M);
    stage_epilogue_rows<BN>(e, gr, lds0 + ROWS, wave, 4, n0, N);
    if (nk > 1) {
        static_for<0, FIRST_TILE>([&](auto ic) { copy_one(ic, 1, STAGE); });
        wait_vmcnt<FIRST_TILE>();
    } else wait_vmcnt<0>();
    asm volatile("s_barrier" ::: "memory");
    warm_caches(e, lds0 + DUMMY, nb, b, wave, 4);
    if (nk == 1) wait_vmcnt<0>();                   // (otherwise the last k-tile's wait covers it)
    static_for<0, RD>([&](auto rc) { read_one(rc, C0, a0, w0); });
    static_for<0, S>([&](auto pc) { constexpr int p = decltype(pc)::value; hold_acc<(p < kAgprPieces)>(acc[p / MI][p % MI]); });
    settle_mfma();
    wait_lgkmcnt<0>();
    hold_set(C0);

    // One k-tile: MFMA slots 0 .. S-1 on the first k-step's fragments, S .. 2S-1 on the second's.
    auto tile = [&](auto load_c, auto next_c, int kt, uint32_t so, uint32_t no) {
        constexpr bool LOAD = decltype(load_c)::value, NEXT = decltype(next_c)::value;
        const uint32_t ca1 = a1 + so, cw1 = w1 + so, na0 = a0 + no, nw0 = w0 + no;
        static_for<0, 2 * S>([&](auto mc) {
            constexpr int m = decltype(mc)::value, s = m / S, p = m % S;
            if constexpr (m == REL) {
                wait_lgkmcnt<0>();
                hold_set(C1);
                if constexpr (NEXT) asm volatile("s_barrier" ::: "memory");
            }
            if constexpr (m == LAND && NEXT) { wait_vmcnt<LOAD ? copies_before(LAND) : 0>(); asm volatile("s_barrier" ::: "memory"); }
            if constexpr (m < RSTEP * RD && m % RSTEP == 0) read_one(std::integral_constant<int, m / RSTEP>{}, C1, ca1, cw1);
            if constexpr (NEXT && m >= LAND && m < LAND + RSTEP * RD && (m - LAND) % RSTEP == 0) read_one(std::integral_constant<int, (m - LAND) / RSTEP>{}, C0, na0, nw0);
            if constexpr (copy_at(m) >= 0) {
                if constexpr (copy_at(m) < FIRST_TILE) { if constexpr (LOAD) copy_one(std::integral_constant<int, copy_at(m)>{}, kt + 2, so); }
                else if constexpr (NEXT) copy_one(std::integral_constant<int, copy_at(m)>{}, kt + 1, no);
            }
            constexpr int i = p / MI, j = i & 1 ? MI - 1 - p % MI : p % MI;      // snake: one operand changes per MFMA
            mfma<(i * MI + j < kAgprPieces)>(acc[i][j], fw[s][i], fa[s][j]);
        });
        if constexpr (NEXT) { wait_lgkmcnt<0>(); hold_set(C0); }
    };
    uint32_t so = 0;
    int kt = 0;
    for (; kt + 2 < nk; ++kt) {
        tile(std::true_type{}, std::true_type{}, kt, so, (uint32_t)STAGE - so);
        so = (uint32_t)STAGE - so;
    }
    if (kt + 1 < nk) {
        tile(std::false_type{}, std::true_type{}, kt, so, (uint32_t)STAGE - so);
        so = (uint32_t)STAGE - so;
    }
    tile(std::false_type{}, std::false_type{}, kt, so, (uint32_t)STAGE - so);
    // (the last MFMAs' results are read by ordinary instructions from here on)
    settle_mfma();
    static_for<0, S>([&](auto pc) { constexpr int p = decltype(pc)::value; hold_acc<(p < kAgprPieces)>(acc[p / MI][p % MI]); });

    const int mw = m0 + wm * TM, nw = n0 + wn * TN;
    const unsigned char* erows = smem_raw + ROWS + wn * TN * 4;
    if constexpr (F32) store_tile_as<TM, TN, MODE, true>(acc, e, mw, nw, M, N, erows, epi_row_bytes(BN), gr, lane);
    else if (may_store_rows<BM, BN>(e, m0, n0, M, N, gr)) {
        asm volatile("s_barrier" ::: "memory");     // every wave has read its last fragments
        store_rows<TM, TN, MODE, MODE == EPI_STORE_GATED>(acc, e, mw, nw, smem_raw + wave * rows_tile_bytes(TM, TN), erows, epi_row_bytes(BN));
    } else store_tile_as<TM, TN, MODE, false, true>(acc, e, mw, nw, M, N, erows, epi_row_bytes(BN), gr, lane);
}

template <int BM, int BN, int MODE, bool F32>
drf_status launch_wide(const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int m_first)
{
    constexpr size_t smem = wide_rows_at(BM, BN) + epi_lds_bytes(BN) + 256;
    static_assert(smem <= 160 * 1024, "LDS of a CU");
    static bool attr_set = false;
    auto kern = gemm_bf16_wide_kernel<BM, BN, MODE, F32>;
    if (!attr_set) {
        DRF_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        attr_set = true;
    }
    const int tiles_m = (M - m_first + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(256), smem, st, A, W, M, N, K, e, tiles_m, tiles_n, m_first);
    DRF_HIP(hipGetLastError());
    return DRF_OK;
}

// GELU: whether the shape has instances of that store.
template <int BM, int BN, bool GELU = true>
drf_status launch_wide_mode(const bf16_t* A, const bf16_t* W, int M, int N, int K, const Epilogue& e, hipStream_t st, int m_first)
{
    if (!GELU && e.mode == EPI_STORE_GELU) DRF_FAIL(DRF_EINVAL, "no GELU on tiles of %d x %d", BM, BN);
    if (e.mode == EPI_RESID) return launch_wide<BM, BN, EPI_RESID, true>(A, W, M, N, K, e, st, m_first);
    if (e.out_f32) return launch_wide<BM, BN, EPI_STORE, true>(A, W, M, N, K, e, st, m_first);
    if constexpr (GELU) {
        if (e.mode == EPI_STORE_GELU) return launch_wide<BM, BN, EPI_STORE_GELU, false>(A, W, M, N, K, e, st, m_first);
    }
    if (e.mode == EPI_STORE_HEADS) return launch_wide<BM, BN, EPI_STORE_HEADS, false>(A, W, M, N, K, e, st, m_first);
    if (e.mode == EPI_STORE_GATED) return launch_wide<BM, BN, EPI_STORE_GATED, false>(A, W, M, N, K, e, st, m_first);
    return launch_wide<BM, BN, EPI_STORE, false>(A, W, M, N, K, e, st, m_first);
}

}  // namespace

}  // namespace drf
