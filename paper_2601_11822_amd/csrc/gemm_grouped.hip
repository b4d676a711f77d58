// The experts' products: the grouped form of the large-tile GEMM, whose tiles each belong to one expert.
#include <algorithm>

#include "gemm_tiles.h"

// Grouped GEMM: rows laid out expert by expert, every unit of the work list (moe_plan_kernel) a tile of 128 to 256
// rows, in steps of 32, of one expert by 256 columns.  The arithmetic of an output element does not depend on the tile that holds it.
// Blocks of 32 rows that are padding are not fetched (64 rows of 8 experts in tiles of 128 rows: gate/up 337 -> 333 us).  What they are multiplied
// with is whatever their stage holds, and the sums are stored with the others, to rows that nobody reads.
// An expert's rows are cut into units of one height (two from four units on), so that the units that share its weights run
// through K at one pace and fetch them together.  A 256-row tile beside a shorter one that runs ahead of it had every weight leave the L2 in
// between (8 experts of 275 rows of the 8B widths, 256 + 128 rows each against 192 + 192: gate/up 801 -> 649 us, down 395 -> 324 us).
template <int EPI, bool NT>
__global__ __launch_bounds__(256) void gemm_grouped_kernel(GemmArgs a, int n_tiles, int cus) {
    extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
    const int nu = __builtin_amdgcn_readfirstlane(a.units[0]) & 0xffff;
    if (nu <= 0) return;
    const bool narrow = grouped_narrow(EPI == EPI_STORE, nu, n_tiles, cus);
    if (narrow) n_tiles = (a.N + 127) / 128;
    const GroupTile t = grouped_tile(blockIdx.x & 7, blockIdx.x >> 3, nu, n_tiles);
    if (t.u < 0) return;
    const int code = __builtin_amdgcn_readfirstlane(a.units[2 + t.u]);
    const int row0 = (code >> 13) * 32, height = (code >> 5) & 15, blocks = (code >> 9) & 15;
    GemmArgs g = a;
    g.Wp += (size_t)(code & 31) * a.expert_stride;
    if (EPI == EPI_SWIGLU) g.Wp2 += (size_t)(code & 31) * a.expert_stride;
    auto tile = [&](auto bm, auto bn, auto ns) {
        gemm_direct_tile<decltype(bm)::value, decltype(bn)::value, EPI, decltype(ns)::value, false, false, NT>(g, row0, t.nb, smem, 0, 0, nullptr, 0, nullptr, blocks);
    };
#define RS_T(bm, bn, ns) tile(std::integral_constant<int, bm>{}, std::integral_constant<int, bn>{}, std::integral_constant<int, ns>{})
    if constexpr (EPI == EPI_STORE) {
        if (narrow) {
            if (height == 8) RS_T(256, 128, 5);
            else if (height == 7) RS_T(224, 128, 5);
            else if (height == 6) RS_T(192, 128, 6);
            else if (height == 5) RS_T(160, 128, 7);
            else RS_T(128, 128, 8);
            return;
        }
    }
    if (height == 8) RS_T(256, 256, RS_NS_FULL);
    else if (height == 7) RS_T(224, 256, 4);
    else if (height == 6) RS_T(192, 256, 4);
    else if (height == 5) RS_T(160, 256, 4);
    else RS_T(128, 256, 5);
#undef RS_T
}

// The same with tiles of up to 320 rows, by eight waves (grouped_cut says when): an XCD's tall units (more than 256 rows) first, then the others, so that
// those that share weights still run side by side and the last tiles to start are the short ones (1300 rows of 8 experts, half of them cut in two: 1153 -> 1100 us);
// a last round of few tiles is cut into halves of 128 columns (grouped_piece: 1100 rows 926 -> 894 us).
template <int EPI, bool NT>
__global__ __launch_bounds__(512) void gemm_grouped_tall_kernel(GemmArgs a, int cus) {
    extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
    const int nus = __builtin_amdgcn_readfirstlane(a.units[0]), nu = nus & 0xffff, nu_tall = nus >> 16;
    if (nu <= 0) return;
    const GroupTallTile t = grouped_tall_tile(blockIdx.x & 7, blockIdx.x >> 3, nu_tall, nu, a.N, EPI == EPI_STORE, cus);
    if (t.u < 0) return;
    const int code = __builtin_amdgcn_readfirstlane(a.units[2 + t.u]);
    const int row0 = (code >> 13) * 32, height = (code >> 5) & 15, blocks = (code >> 9) & 15;
    GemmArgs g = a;
    g.Wp += (size_t)(code & 31) * a.expert_stride;
    if (EPI == EPI_SWIGLU) g.Wp2 += (size_t)(code & 31) * a.expert_stride;
    auto tile = [&](auto xf, auto wgm, auto ns) {
        gemm_tall_tile<decltype(xf)::value, decltype(wgm)::value, EPI, decltype(ns)::value, NT>(g, row0, t.nb, smem, blocks, row0 + 32 * height);
    };
#define RS_T(xf, wgm, ns) tile(std::integral_constant<int, xf>{}, std::integral_constant<int, wgm>{}, std::integral_constant<int, ns>{})
    if (t.half) {
        if (height > 8) RS_T(5, 4, 5);
        else if (height > 6) RS_T(4, 4, 6);
        else if (height > 4) RS_T(3, 4, 8);
        else RS_T(2, 4, 8);
        return;
    }
    if (height == 10) RS_T(10, 2, 4);
    else if (height == 9) RS_T(9, 2, 4);
    else if (height == 8) RS_T(8, 2, 5);
    else if (height == 7) RS_T(7, 2, 5);
    else if (height == 6) RS_T(6, 2, 5);
    else if (height == 5) RS_T(5, 2, 6);
    else RS_T(4, 2, 6);
#undef RS_T
}

template <int EPI, bool NT>
static void launch_grouped_nt(hipStream_t st, const GemmArgs &a) {
    const int n_tiles = (EPI == EPI_SWIGLU) ? (a.N + 127) / 128 : (a.N + 255) / 256;
    const int cus = a.cus > 0 ? a.cus : 256, units = a.M >> 7;   // as many as there can be
    if (a.tall) {
        hipLaunchKernelGGL((gemm_grouped_tall_kernel<EPI, NT>), dim3(grouped_tall_grid(units, n_tiles, cus)), dim3(512), RS_TALL_LDS, st, a, cus);
    } else {   // of narrow tiles no more than CUs
        const int grid = (std::max(units * n_tiles, EPI == EPI_STORE ? cus : 0) + 7) / 8 * 8;
        hipLaunchKernelGGL((gemm_grouped_kernel<EPI, NT>), dim3(grid), dim3(256), RS_NS_FULL * 32768, st, a, n_tiles, cus);
    }
}
template <int EPI>
static void launch_grouped_epi(hipStream_t st, const GemmArgs &a) {
    a.stream_weights ? launch_grouped_nt<EPI, true>(st, a) : launch_grouped_nt<EPI, false>(st, a);
}

bool launch_gemm_grouped(hipStream_t st, const GemmArgs &a) {
    if (!(a.K % 32 == 0 && a.K >= 32 && a.Wp && a.N >= 1024 && a.M % 128 == 0 && a.units)) return false;
    if (a.epi == EPI_SWIGLU) launch_grouped_epi<EPI_SWIGLU>(st, a);
    else if (a.epi == EPI_STORE) launch_grouped_epi<EPI_STORE>(st, a);
    else return false;
    return true;
}

void grouped_kernels_init() {
    auto set = [](const void *f, int lds) { (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds); };
    set((const void *)gemm_grouped_tall_kernel<EPI_STORE, true>, RS_TALL_LDS);
    set((const void *)gemm_grouped_tall_kernel<EPI_SWIGLU, true>, RS_TALL_LDS);
    set((const void *)gemm_grouped_tall_kernel<EPI_STORE, false>, RS_TALL_LDS);
    set((const void *)gemm_grouped_tall_kernel<EPI_SWIGLU, false>, RS_TALL_LDS);
    set((const void *)gemm_grouped_kernel<EPI_STORE, true>, RS_NS_FULL * 32768);
    set((const void *)gemm_grouped_kernel<EPI_SWIGLU, true>, RS_NS_FULL * 32768);
    set((const void *)gemm_grouped_kernel<EPI_STORE, false>, RS_NS_FULL * 32768);
    set((const void *)gemm_grouped_kernel<EPI_SWIGLU, false>, RS_NS_FULL * 32768);
}
