// bf16 GEMMs out = epi(A[M,K] * W[N,K]^T) on the gfx950 matrix cores (fp32 accumulation).
//
// A lane's 8-element MFMA fragment is 8 consecutive k of one row: one 16-byte chunk, and the unit
// of the fragment-packed operand layout (packed_offset) that the activations are always stored in.
// The weight tile is the MFMA "row" operand and the activation tile the "column" operand:
// a lane then owns 4 consecutive output columns of one output row, which makes the epilogues
// (residual add, SwiGLU, bf16 pack) per-lane code; the direct kernel's row-major outputs pass through LDS on their way (store_rows).
#include <algorithm>

#include "gemm_tiles.h"

// ---------------------------------------------------------------------------------------------
// Tiled kernel: BM x BN output tile per 256-thread workgroup (2x2 waves), BK = 64, operands
// (fragment-packed A, row-major W) staged global -> registers -> LDS (16-byte chunks, chunk index XOR (row>>1)&7 against bank
// conflicts on the 64-bank LDS), next tile's global loads in flight during the MFMAs.  Every tail (M, N, K) is
// handled by predicated zero-filled loads and predicated stores.
//
// SwiGLU: the B tile interleaves 32 gate rows with the 32 matching up rows, so gate and up of
// one output element sit in the same lane and register index of neighbouring accumulators.
// ---------------------------------------------------------------------------------------------
template <int BM, int BN, int EPI>
__global__ __launch_bounds__(256) void gemm_tiled_kernel(GemmArgs a) {
    constexpr int BK = 64;
    constexpr int WM = BM / 2, WN = BN / 2;
    constexpr int TM = WM / 32, TN = WN / 32;
    constexpr int CA = BM / 32, CB = BN / 32;  // 16-byte chunks per thread per tile
    __shared__ __attribute__((aligned(16))) bf16_t As[BM * BK];
    __shared__ __attribute__((aligned(16))) bf16_t Bs[BN * BK];

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wm = wave >> 1, wn = wave & 1;
    const int c32 = lane & 31, h = lane >> 5;
    const int M = a.M, N = a.N, K = a.K;
    const int bm = blockIdx.y * BM;
    const int nb = blockIdx.x;

    // global row pointers of this thread's chunks
    const bf16_t *pa[CA];
    const bf16_t *pb[CB];
    const int cc = tid & 7;  // chunk column (same for all of a thread's chunks)
    const int Mt = packed_mt(M);
#pragma unroll
    for (int j = 0; j < CA; ++j) {
        const int r = (tid >> 3) + 32 * j;
        const int m = bm + r;
        pa[j] = (m < M) ? a.A + packed_offset(m, cc * 8, Mt) : nullptr;   // chunk (m, k0 + 8cc) for k0 = 0
    }
    const size_t a_kmul = (size_t)Mt * 32;   // a step of 64 in k is 4 k blocks of Mt KB
#pragma unroll
    for (int j = 0; j < CB; ++j) {
        const int r = (tid >> 3) + 32 * j;  // row of the B tile
        if (EPI == EPI_SWIGLU) {
            const int t = r >> 5;
            const int f = nb * (BN / 2) + (t >> 1) * 32 + (r & 31);
            pb[j] = (f < N) ? ((t & 1) ? a.W2 : a.W) + (size_t)f * K + cc * 8 : nullptr;
        } else {
            const int n = nb * BN + r;
            pb[j] = (n < N) ? a.W + (size_t)n * K + cc * 8 : nullptr;
        }
    }

    f32x16 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    bf16x8 ra[CA], rb[CB];
    auto gload = [&](int k0) {
        const bool kin = k0 + cc * 8 < K;
#pragma unroll
        for (int j = 0; j < CA; ++j) ra[j] = (kin && pa[j]) ? ld_bf16x8(pa[j] + k0 * a_kmul) : zero_bf16x8();
#pragma unroll
        for (int j = 0; j < CB; ++j) rb[j] = (kin && pb[j]) ? ld_bf16x8(pb[j] + k0) : zero_bf16x8();
    };
    gload(0);
    for (int k0 = 0; k0 < K; k0 += BK) {
#pragma unroll
        for (int j = 0; j < CA; ++j) {
            const int r = (tid >> 3) + 32 * j;
            *(bf16x8 *)&As[r * BK + ((cc ^ ((r >> 1) & 7)) << 3)] = ra[j];
        }
#pragma unroll
        for (int j = 0; j < CB; ++j) {
            const int r = (tid >> 3) + 32 * j;
            *(bf16x8 *)&Bs[r * BK + ((cc ^ ((r >> 1) & 7)) << 3)] = rb[j];
        }
        __syncthreads();
        if (k0 + BK < K) gload(k0 + BK);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            bf16x8 wf[TN], xf[TM];
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                const int r = wn * WN + 32 * tn + c32;
                wf[tn] = *(const bf16x8 *)&Bs[r * BK + (((2 * s + h) ^ ((r >> 1) & 7)) << 3)];
            }
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                const int r = wm * WM + 32 * tm + c32;
                xf[tm] = *(const bf16x8 *)&As[r * BK + (((2 * s + h) ^ ((r >> 1) & 7)) << 3)];
            }
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) acc[tn][tm] = mfma32(wf[tn], xf[tm], acc[tn][tm]);
        }
        __syncthreads();
    }

    // epilogue: lane owns row m, columns n0 + 8j + 4h + (0..3)
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        const int m = bm + wm * WM + 32 * tm + c32;
        if (m >= M) continue;
        if (EPI == EPI_SWIGLU) {
#pragma unroll
            for (int p = 0; p < TN / 2; ++p)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int f = nb * (BN / 2) + (wn * (TN / 2) + p) * 32 + 8 * j + 4 * h;
                    if (f >= N) continue;
                    bf16x4 v;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        v[i] = (bf16_t)(silu_f(acc[2 * p][tm][4 * j + i]) * acc[2 * p + 1][tm][4 * j + i]);
                    store_out4<EPI>(a, m, f, v);
                }
        } else {
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int n = nb * BN + wn * WN + 32 * tn + 8 * j + 4 * h;
                    if (n >= N) continue;
                    bf16x4 v;
                    if (EPI == EPI_RESIDUAL) {
                        const bf16x4 r = *(const bf16x4 *)(a.resid + (size_t)m * N + n);
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = (bf16_t)(acc[tn][tm][4 * j + i] + (float)r[i]);
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = (bf16_t)acc[tn][tm][4 * j + i];
                    }
                    store_out4<EPI>(a, m, n, v);
                }
        }
    }
}

// The flat workgroup id is remapped so that the workgroups resident on one XCD (ids congruent
// mod 8) own a contiguous run of tiles in that order, served by that XCD's L2.
template <int BM, int BN, int EPI, int NS, bool NT>
__global__ __launch_bounds__(256) void gemm_direct_kernel(GemmArgs a, int m_tiles, int n_tiles) {
    extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
    const int total = m_tiles * n_tiles;
    const int per_xcd = (total + 7) >> 3;
    const int t = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (t >= total) return;
    int r, c;
    tile_rc(t, m_tiles, n_tiles, r, c);
    gemm_direct_tile<BM, BN, EPI, NS, false, false, NT>(a, r * BM, c, smem);
}

// Tiles of 128 x 256 with the residual, or stored as they are: the loads by four more waves (FED).  These products are long rounds of a CU's loads (2048x4096x14336: 192 us,
// its loads alone 160, its products 131), and a wave that multiplies no longer stands at a load that the full queue does not take.  Layers of the 8B widths on 256 CUs: 1536 rows
// 628 -> 612 us, 2048 748 -> 733; of the 70B widths 768 1154 -> 1124.  Not the short ones, whose first bytes come later so: gate/up and K slices of 160 rows +4 % of the layer, of 512 +1.5.
#define RS_FED_LDS 147456   // 6 x 24 KB
template <int EPI, bool NT>
__global__ __launch_bounds__(512) void gemm_fed_kernel(GemmArgs a, int m_tiles, int n_tiles) {
    extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
    const int total = m_tiles * n_tiles;
    const int per_xcd = (total + 7) >> 3;
    const int t = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (t >= total) return;
    int r, c;
    tile_rc(t, m_tiles, n_tiles, r, c);
    gemm_direct_tile<128, 256, EPI, 6, false, false, NT, true>(a, r * 128, c, smem);
}

// The same with tiles of eight waves.
template <int XF, int EPI, int NS, bool NT>
__global__ __launch_bounds__(512) void gemm_tall_kernel(GemmArgs a, int m_tiles, int n_tiles) {
    extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
    const int total = m_tiles * n_tiles;
    const int per_xcd = (total + 7) >> 3;
    const int t = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (t >= total) return;
    int r, c;
    tile_rc(t, m_tiles, n_tiles, r, c);
    gemm_tall_tile<XF, 2, EPI, NS, NT>(a, r * 32 * XF, c, smem, XF, a.M);
}

// Whole rounds of large tiles, then a last half round: when the tiles do not divide by the number of compute units, the first
// n_full workgroups (a multiple of the unit count) take whole tiles and the remaining tiles are cut in two, one workgroup each,
// which are dispatched last: 256x256 into two of 128x256, 192x256 (TALL false) into two of 192x128.
// The arithmetic of an output element does not depend on the tile
// that holds it, so the schedule may follow the size of the partition.
template <int EPI, bool TALL, bool NT>
__global__ __launch_bounds__(256) void gemm_direct_mixed_kernel(GemmArgs a, int m_tiles, int n_full, int n_half) {
    extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
    constexpr int BM = TALL ? 256 : 192;
    const int id = blockIdx.x;
    const int n_tiles = (n_full + (n_half >> 1)) / m_tiles;   // column tiles
    int r, c;
    if (id < n_full) {
        const int t = (id & 7) * (n_full >> 3) + (id >> 3);          // n_full is a multiple of 8
        tile_rc(t, m_tiles, n_tiles, r, c);
        gemm_direct_tile<BM, 256, EPI, RS_NS_FULL, false, false, NT>(a, r * BM, c, smem);
    } else {
        const int j = id - n_full;
        const int u = (j & 7) * ((n_half + 7) >> 3) + (j >> 3);
        if (u >= n_half) return;
        const int t = n_full + (u >> 1);
        tile_rc(t, m_tiles, n_tiles, r, c);
        if (TALL) {
            const int bm = r * 256 + (u & 1) * 128;
            if (bm < a.M) gemm_direct_tile<128, 256, EPI, 5, false, false, NT>(a, bm, c, smem);
        } else {
            const int nb = 2 * c + (u & 1);
            if (nb * (EPI == EPI_SWIGLU ? 64 : 128) < a.N) gemm_direct_tile<192, 128, EPI, 5, false, false, NT>(a, r * 192, nb, smem);
        }
    }
}

// Few output tiles and a long K (the projections at a few hundred rows): the K range is cut into S slices, one workgroup per
// (tile, slice), and an epilogue kernel adds the slices in order.  Workgroups that run on one XCD own a contiguous run of tiles of
// one slice in tile_rc's order, as in gemm_direct_kernel: dealt out in turn every XCD fetched every slab (576x6144x4096 in two
// slices: 318 MB past the L2s for operands of 55, 49 -> 40 us).
template <int BM, int NS>
__global__ __launch_bounds__(256) void gemm_direct_splitk_kernel(GemmArgs a, int m_tiles, int n_tiles, int S, int nk_per, float *part) {
    extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
    const int tiles = m_tiles * n_tiles, total = tiles * S, per_xcd = (total + 7) >> 3;
    const int id = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (id >= total) return;
    const int z = id / tiles, t = id % tiles;
    const int kt0 = z * nk_per;
    int r, c;
    tile_rc(t, m_tiles, n_tiles, r, c);
    gemm_direct_tile<BM, 256, EPI_STORE, NS, true>(a, r * BM, c, smem, kt0, min(nk_per, a.K / 32 - kt0), part, z);
}

template <int XF, int NS>
__global__ __launch_bounds__(512) void gemm_tall_splitk_kernel(GemmArgs a, int m_tiles, int n_tiles, int S, int nk_per, float *part) {
    extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
    const int tiles = m_tiles * n_tiles, total = tiles * S, per_xcd = (total + 7) >> 3;
    const int id = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (id >= total) return;
    const int z = id / tiles, t = id % tiles, kt0 = z * nk_per;
    int r, c;
    tile_rc(t, m_tiles, n_tiles, r, c);
    gemm_tall_tile<XF, 2, EPI_STORE, NS, true, true>(a, r * 32 * XF, c, smem, XF, a.M, kt0, min(nk_per, a.K / 32 - kt0), part + (size_t)z * a.M * a.N);
}

// ---------------------------------------------------------------------------------------------
// The schedule of a large-tile product: tile shape and K slices by what they are expected to cost.
// A round of w workgroups of one tile shape takes 4.8 + nk * (a + b * w / 256) us for nk K tiles: 4.8 are the first loads and the
// tile's stores, b is what the units cost one another (fabric, power).  Fitted to 1215 timings of cold weights on 64, 96, 128,
// 192 and 256 CUs (150 to 2048 rows; K 4096, 8192, 14336; N 4096 to 28672 pairs; the shapes of 128, 192 and 256 rows, 1 to 6 slices): 6 % rms.
// 160 and 224 rows, whose waves stand side by side and read more LDS per product, follow from 1176 products of one layer of the 8B and 70B
// widths (150 to 4000 rows, 64 to 256 CUs, each with every form): with b = 0.10 and 0.17 the choice was 0.2 % slower than the fastest form
// on average, 10 % at most.  With constants found on 256 CUs (0.415 + 0.055 and 0.495 + 0.12) it was 1.4 % and 21 %, nearly all on half of
// the chip and less; layers at those and these: 8B 1150 rows on 128 CUs 773 -> 750 us, 576 rows 483 -> 466, 800 rows on 96 CUs 762 -> 715,
// 70B 1153 rows on 128 CUs 2723 -> 2555, 620 rows on 96 1869 -> 1785.
// 288 and 320 rows (eight waves) stand where layers with them and without them crossed: 8B widths on 256 CUs, without / with: 576 rows 293 / 273 us, 640 318 / 300,
// 1152 487 / 471, 1280 521 / 505 (their gate/up; forced at 512 rows 250 / 250, at 700 353 / 380, at 1400 602 / 639, at 2048 742 / 816); on 128 CUs 288 rows 293 / 232, 576 458 / 369,
// 1088 716 / 641, 1400 827 / 781 (slices too); 70B widths on 256 CUs 288 rows 540 / 490.  What they save is what a CU loads: 34 KB a K tile for 288 x 256 where two of 160 x 256 take 52.
// Their b is 0.005 dearer than those timings gave: among forms that cost the same to 1 %, the larger tile is the faster one in passes back to
// back, where power sets the clock (gate/up of 224 rows or of 256 with a last round of halves: 70B 5482 rows 7887 and 7783 us a layer,
// 8B 7050 rows 2898 and 2876, 6460 rows on 192 CUs 3072 and 3032).
// A slice adds its partial sums, written and read back, 0.3 us, and once 2 us for the epilogue kernel.
// (All of these are timings of the loop with 32x32x16 products; the present one takes 0.89 to 0.95 of the times of long products, so a slice's
// cost, which stands beside them in microseconds, counts for that much less than it should.  With the present loop every form and every count of
// slices was forced in turn, those of eight waves and the fed one among them, 12 row counts of the 8B widths from 200 to 8000 on 256 and 128 CUs, five on 192 and seven
// passes of the 70B widths (profiles/large_tile_forms_forced.md): the forms are within 1 % of the fastest layer; the slices, which may not follow the CUs, within 1 %
// on the whole chip, 2 % on 192 CUs and 4 % on half of it.  With every tile of 288 and 320 rows of whole products left out, 1400 to 12000 rows take 0.99 to 1.14 times as long;
// 70B widths, 7000 rows on 192 CUs 0.98.)
// Against the rule before it (128-row tiles for slices, their count a power of two up to half the chip; no 192-row tiles), product and
// epilogue, on 256 CUs: 576x4096x14336 94 -> 74 us, 1152x4096x14336 172 -> 127, 576x8192x28672 330 -> 252, gate/up 576x14336x4096
// 157 -> 133, 384x14336x4096 107 -> 75, 192x28672x8192 231 -> 175; over the products timed 4 % on 256 CUs and 10 % on 128.
// ---------------------------------------------------------------------------------------------
static double direct_round_us(DirectForm f, int nk, long w) {
    constexpr double A[] = {0.30, 0.365, 0.38, 0.44, 0.44, 0.36, 0.225, 0, 0, 0.50, 0.56}, B[] = {0.10, 0.105, 0.145, 0.175, 0.25, 0.165, 0.09, 0, 0, 0.28, 0.31};
    return 4.8 + nk * (A[f] + B[f] * (double)w / 256.0);
}
static long direct_tiles(DirectForm f, int M, int nv) {
    constexpr int BM[] = {128, 160, 192, 224, 256, 256, 192, 0, 0, 288, 320}, BN[] = {256, 256, 256, 256, 256, 192, 128, 0, 0, 256, 256};
    return (long)((M + BM[f] - 1) / BM[f]) * ((nv + BN[f] - 1) / BN[f]);
}
static double direct_rounds_us(DirectForm f, int nk, long wgs, int cus) {
    return (double)(wgs / cus) * direct_round_us(f, nk, cus) + (wgs % cus ? direct_round_us(f, nk, wgs % cus) : 0.0);
}
// Whole rounds of `full` tiles and one round of `half` ones: cost, or a huge one where there is no such schedule.
static double direct_mixed_us(DirectForm full, DirectForm half, int nk, long tiles, int cus, int &n_full) {
    n_full = (int)(tiles / cus) * cus;
    const long rest = tiles - n_full;
    if (!n_full || n_full % 8 || !rest || 2 * rest > cus) return 1e30;
    return (double)(n_full / cus) * direct_round_us(full, nk, cus) + direct_round_us(half, nk, 2 * rest);
}

// The fastest form for S slices (1: the finished product) on `cus` compute units, and its cost.  all: with the heights of an odd
// number of row blocks and those of eight waves.
static double direct_best_form(int M, int N, int K, int epi, int S, int cus, DirectForm &form, bool all = true) {
    const int nv = epi == EPI_SWIGLU ? (N + 127) / 128 * 256 : N, nk = (K / 32 + S - 1) / S;
    double best = 1e30;
    auto consider = [&](DirectForm f, double us) { if (us < best) { best = us; form = f; } };
    for (DirectForm f : {FORM_320x256, FORM_288x256, FORM_256x256, FORM_224x256, FORM_192x256, FORM_160x256, FORM_128x256})
        if (all || (f != FORM_160x256 && f != FORM_224x256 && f != FORM_288x256 && f != FORM_320x256)) consider(f, direct_rounds_us(f, nk, S * direct_tiles(f, M, nv), cus));
    if (S > 1) return best;
    int n_full;
    if (epi == EPI_SWIGLU) {
        consider(FORM_192x128, direct_rounds_us(FORM_192x128, nk, direct_tiles(FORM_192x128, M, nv), cus));
        consider(FORM_MIXED_192, direct_mixed_us(FORM_192x256, FORM_192x128, nk, direct_tiles(FORM_192x256, M, nv), cus, n_full));
    } else {
        consider(FORM_256x192, direct_rounds_us(FORM_256x192, nk, direct_tiles(FORM_256x192, M, nv), cus));
    }
    consider(FORM_MIXED_256, direct_mixed_us(FORM_256x256, FORM_128x256, nk, direct_tiles(FORM_256x256, M, nv), cus, n_full));
    return best;
}

DirectForm direct_form(int M, int N, int K, int epi, int S, int cus) {
    DirectForm f;
    direct_best_form(M, N, K, epi, S, cus, f);
    return f;
}

// K slices: from (M, N, K) alone, so that results do not depend on the CU share; the whole chip's time counts four times what half
// of it takes.  At least 16 K tiles a slice, one round of workgroups, and no more partial sums than RS_DIRECT_PARTIAL_ELEMS.
// (With the whole chip alone 576 to 1150 rows lost up to 15 % of a product on 128 CUs.  What is left: two slices of 1150x4096x14336 gain 33 us
// of the layer on 256 CUs and cost 18 on 128.)  Heights of an odd number of row blocks take no part in the choice: counted in, they
// raised the slices of 680 to 770 rows of a 4096-wide down projection from two to three, 2 % of the layer on 256 CUs for 8 % on 128.
int direct_splits(int M, int N, int K) {
    DirectForm f;
    auto us = [&](int epi, int S) { return direct_best_form(M, N, K, epi, S, 256, f, false) + 0.25 * direct_best_form(M, N, K, epi, S, 128, f, false); };
    int S = 1;
    double best = us(EPI_RESIDUAL, 1);
    const int nk = K / 32;
    for (int s = 2; s <= 8 && nk / s >= 16 && (size_t)s * M * N <= RS_DIRECT_PARTIAL_ELEMS; ++s) {
        if ((nk + s - 1) / s * (s - 1) >= nk || s * direct_tiles(FORM_256x256, M, N) > 256) continue;   // no empty slice, no second round
        const double t = us(EPI_STORE, s) + 1.25 * (1.2e-6 * s * M * N + 2.0 + 0.3 * s);
        if (t < best) { best = t; S = s; }
    }
    return S;
}

// Slices for a pass of at most 64 rows (launch_gemm_skinny): doubled while the chip has a unit for every 256-column tile, at least 16
// K tiles each.  Not the rows: a row's sums are in the same order whatever else is in its batch, and the costs above are fitted
// from 150 rows on (by them 6144x6144 took 8 slices up to 55 rows and 5 from 56).
static int skinny_direct_splits(int N, int K) {
    int S = 1;
    while ((N + 255) / 256 * S * 2 <= 256 && S < 8 && K / 32 / (S * 2) >= 16) S *= 2;
    return S;
}

template <int EPI>
__global__ __launch_bounds__(256) void skinny_epilogue_kernel(GemmArgs a, const float *__restrict__ part, int S, int Nv);

template <int BM, int NS>
static void launch_direct_splitk_tiles(hipStream_t st, const GemmArgs &a, int S) {
    const int m_tiles = (a.M + BM - 1) / BM, n_tiles = (a.N + 255) / 256, nk_per = (a.K / 32 + S - 1) / S;
    const dim3 grid((m_tiles * n_tiles * S + 7) / 8 * 8);
    if constexpr (BM > 256) hipLaunchKernelGGL((gemm_tall_splitk_kernel<BM / 32, NS>), grid, dim3(512), NS * (BM + 256) * 64, st, a, m_tiles, n_tiles, S, nk_per, a.partials);
    else hipLaunchKernelGGL((gemm_direct_splitk_kernel<BM, NS>), grid, dim3(256), NS * (BM + 256) * 64, st, a, m_tiles, n_tiles, S, nk_per, a.partials);
}
static void launch_direct_splitk_main(hipStream_t st, const GemmArgs &a, int S) {
    const DirectForm f = direct_form(a.M, a.N, a.K, EPI_STORE, S, a.cus > 0 ? a.cus : 256);
    if (f == FORM_256x256) launch_direct_splitk_tiles<256, RS_NS_FULL>(st, a, S);
    else if (f == FORM_320x256) launch_direct_splitk_tiles<320, 4>(st, a, S);
    else if (f == FORM_288x256) launch_direct_splitk_tiles<288, 4>(st, a, S);
    else if (f == FORM_224x256) launch_direct_splitk_tiles<224, 4>(st, a, S);
    else if (f == FORM_192x256) launch_direct_splitk_tiles<192, 4>(st, a, S);
    else if (f == FORM_160x256) launch_direct_splitk_tiles<160, 4>(st, a, S);
    else launch_direct_splitk_tiles<128, 5>(st, a, S);
}

static void launch_direct_splitk(hipStream_t st, const GemmArgs &a, int S) {
    launch_direct_splitk_main(st, a, S);
    const int eblocks = (a.M * (a.N / 4) + 255) / 256;
    if (a.epi == EPI_RESIDUAL)
        hipLaunchKernelGGL(skinny_epilogue_kernel<EPI_RESIDUAL>, dim3(eblocks), dim3(256), 0, st, a, a.partials, S, a.N);
    else
        hipLaunchKernelGGL(skinny_epilogue_kernel<EPI_STORE>, dim3(eblocks), dim3(256), 0, st, a, a.partials, S, a.N);
}

static int direct_sliced(const GemmArgs &a) {   // K slices of launch_gemm_tiled's sliced path, or 0 where it is not taken
    if (!(a.K % 32 == 0 && a.K >= 32 && a.Wp && a.M > 64 && a.N >= 1024 && a.epi != EPI_SWIGLU && a.partials && a.N % 4 == 0)) return 0;
    const int S = direct_splits(a.M, a.N, a.K);
    return S > 1 && (size_t)S * a.M * a.N <= a.partial_cap ? S : 0;
}

int launch_gemm_tiled_partials(hipStream_t st, const GemmArgs &a) {
    const int S = direct_sliced(a);
    if (S) launch_direct_splitk_main(st, a, S);
    return S;
}

// LM head of more than 64 rows: whole K per tile, all row tiles of a column tile next to each other on one XCD.
template <int BM, int NS>
__global__ __launch_bounds__(256) void gemm_head_kernel(GemmArgs a, HeadOut o, int m_tiles, int n_tiles) {
    extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
    const int total = m_tiles * n_tiles, per_xcd = (total + 7) >> 3;
    const int t = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (t >= total) return;
    gemm_direct_tile<BM, 256, EPI_STORE, NS, false, true>(a, (t % m_tiles) * BM, t / m_tiles, smem, 0, 0, nullptr, 0, &o);
}

// Whether a whole product's weights are a stream (non-temporal).  tile_rc runs up to four row tiles of a column side by side: with no more than those nobody
// reads the weights again.  Layers of the 8B widths on 256 CUs, not streamed / streamed: 160 rows 165.9 / 162.5 us, 512 249.6 / 247.4, 768 369.6 / 360.8,
// 1024 429 / 418; of the 70B widths 160 rows 376 / 360; streamed throughout 1300 rows of the 8B widths 579 / 602, 4000 of the 70B widths 5140 / 5269.
// Not three row tiles on 32 or 64 CUs: an XCD runs four or eight tiles at a time there, so that one column in three has its last tile in the next round, which
// reads the weights again.  70B widths, 660 to 768 rows: on 64 CUs 2727 - 2869 / 2853 - 2967 us, on 32 4994 - 5320 / 5215 - 5534; 8B widths on 32 1521 - 1573 /
// 1554 - 1605, on 64 level.  On 128 CUs, one column in five: 8B widths 0.7 to 1.4 % for streams, 70B widths 1.4 % against to 0.4 % for; 96 and 192 split none.
// Weights few enough to stay in the memory-side cache from pass to pass lose by it: four layers of d 1024, f 3584 at 512 rows 85.4 / 87.5 us; twenty of them level.
bool direct_streams(int m_tiles, int cus) { return m_tiles <= 4 && (m_tiles != 3 || cus > 64); }

template <int EPI, bool TALL>
static void launch_direct_mixed(hipStream_t st, const GemmArgs &a, int cus) {
    constexpr int BM = TALL ? 256 : 192;
    const int m_tiles = (a.M + BM - 1) / BM, n_tiles = EPI == EPI_SWIGLU ? (a.N + 127) / 128 : (a.N + 255) / 256;
    const int n_full = m_tiles * n_tiles / cus * cus, n_half = 2 * (m_tiles * n_tiles - n_full);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(n_full + (n_half + 7) / 8 * 8), dim3(256), RS_NS_FULL * (BM + 256) * 64, st, a, m_tiles, n_full, n_half);
    };
    direct_streams(m_tiles, cus) ? go(gemm_direct_mixed_kernel<EPI, TALL, true>) : go(gemm_direct_mixed_kernel<EPI, TALL, false>);
}

template <int BM, int BN, int EPI, int NS>
static void launch_direct_epi(hipStream_t st, const GemmArgs &a) {
    const int m_tiles = (a.M + BM - 1) / BM;
    const int n_tiles = (EPI == EPI_SWIGLU) ? (a.N + BN / 2 - 1) / (BN / 2) : (a.N + BN - 1) / BN;
    const int total = m_tiles * n_tiles;
    const int grid = ((total + 7) / 8) * 8;
    constexpr int lds = NS * (BM + BN) * 32 * 2;
    constexpr bool fed = BM == 128 && BN == 256 && EPI != EPI_SWIGLU;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(BM > 256 || fed ? 512 : 256), fed ? RS_FED_LDS : lds, st, a, m_tiles, n_tiles);
    };
    const bool nt = direct_streams(m_tiles, a.cus > 0 ? a.cus : 256);
    if constexpr (fed) nt ? go(gemm_fed_kernel<EPI, true>) : go(gemm_fed_kernel<EPI, false>);
    else if constexpr (BM > 256) nt ? go(gemm_tall_kernel<BM / 32, EPI, NS, true>) : go(gemm_tall_kernel<BM / 32, EPI, NS, false>);
    else nt ? go(gemm_direct_kernel<BM, BN, EPI, NS, true>) : go(gemm_direct_kernel<BM, BN, EPI, NS, false>);
}

template <int BM, int BN, int NS>
static void launch_direct(hipStream_t st, const GemmArgs &a) {
    switch (a.epi) {
        case EPI_STORE: launch_direct_epi<BM, BN, EPI_STORE, NS>(st, a); break;
        case EPI_RESIDUAL: launch_direct_epi<BM, BN, EPI_RESIDUAL, NS>(st, a); break;
        default: launch_direct_epi<BM, BN, EPI_SWIGLU, NS>(st, a); break;
    }
}

template <int BM, int BN>
static void launch_tiled(hipStream_t st, const GemmArgs &a) {
    const int n_virtual = (a.epi == EPI_SWIGLU) ? 2 * a.N : a.N;
    // SwiGLU tiles hold BN/2 output columns, padded per 32-column group
    dim3 grid(a.epi == EPI_SWIGLU ? (a.N + BN / 2 - 1) / (BN / 2) : (n_virtual + BN - 1) / BN,
              (a.M + BM - 1) / BM);
    switch (a.epi) {
        case EPI_STORE:
            hipLaunchKernelGGL((gemm_tiled_kernel<BM, BN, EPI_STORE>), grid, dim3(256), 0, st, a);
            break;
        case EPI_RESIDUAL:
            hipLaunchKernelGGL((gemm_tiled_kernel<BM, BN, EPI_RESIDUAL>), grid, dim3(256), 0, st, a);
            break;
        default:
            hipLaunchKernelGGL((gemm_tiled_kernel<BM, BN, EPI_SWIGLU>), grid, dim3(256), 0, st, a);
            break;
    }
}

bool launch_gemm_tiled(hipStream_t st, const GemmArgs &a) {
    if (a.M <= 0 || a.N <= 0) return true;
    const bool aligned = (a.K % 32 == 0) && a.K >= 32;
    if (aligned && a.Wp && a.M > 64 && a.N >= 1024) {
        if (const int S = direct_sliced(a)) {
            launch_direct_splitk(st, a, S);
            return true;
        }
        const int cus = a.cus > 0 ? a.cus : 256;
        switch (direct_form(a.M, a.N, a.K, a.epi, 1, cus)) {
            case FORM_256x256: launch_direct<256, 256, RS_NS_FULL>(st, a); break;   // RS_NS_FULL x 32 KB of LDS
            case FORM_320x256: launch_direct<320, 256, 4>(st, a); break;            // 4 x 36 KB
            case FORM_288x256: launch_direct<288, 256, 4>(st, a); break;            // 4 x 34 KB
            case FORM_224x256: launch_direct<224, 256, 4>(st, a); break;            // 4 x 30 KB
            case FORM_192x256: launch_direct<192, 256, 4>(st, a); break;            // 4 x 28 KB
            case FORM_160x256: launch_direct<160, 256, 4>(st, a); break;            // 4 x 26 KB
            case FORM_128x256: launch_direct<128, 256, 5>(st, a); break;            // 5 x 24 KB, fed 6
            case FORM_256x192:                                                         // 4 x 28 KB
                if (a.epi == EPI_STORE) launch_direct_epi<256, 192, EPI_STORE, 4>(st, a);
                else launch_direct_epi<256, 192, EPI_RESIDUAL, 4>(st, a);
                break;
            case FORM_192x128: launch_direct_epi<192, 128, EPI_SWIGLU, 5>(st, a); break;   // 5 x 20 KB
            case FORM_MIXED_192: launch_direct_mixed<EPI_SWIGLU, false>(st, a, cus); break;
            default:
                if (a.epi == EPI_STORE) launch_direct_mixed<EPI_STORE, true>(st, a, cus);
                else if (a.epi == EPI_RESIDUAL) launch_direct_mixed<EPI_RESIDUAL, true>(st, a, cus);
                else launch_direct_mixed<EPI_SWIGLU, true>(st, a, cus);
        }
    } else {
        // the generic kernel reads the caller's row-major matrices: refuse when they have been released
        if (!a.W || (a.epi == EPI_SWIGLU && !a.W2)) return false;
        if (a.M >= 1024 && a.N >= 1024) launch_tiled<256, 256>(st, a);
        else launch_tiled<128, 128>(st, a);
    }
    return true;
}

// ---------------------------------------------------------------------------------------------
// Skinny kernel (M <= 64): bandwidth bound, so built for bytes in flight.  Both operands arrive in
// MFMA fragment order -- the activations fragment-packed by their producer, the weights repacked
// once when they are set -- so every load is one contiguous 1 KB per wave straight into the
// registers that feed the matrix core: no LDS staging, and since only register loads are
// outstanding they complete in order and the compiler's own wait counts are exact.
//
// Packed weights: [ceil(K/16) k blocks][ceil(N/64)*2 row tiles of 32][64 lanes][8], zero padded;
// lane h*32 + r of block (kb, t) holds W[32t + r][16kb + 8h .. +8).  k-block major: the waves of
// all workgroups advance through K together, so at any moment the chip reads a few contiguous
// regions that spread evenly over the memory channels (row-tile-major streams would all sit at
// the same offset within their 2^n-spaced rows and crowd the same channels).
//
// Workgroup = 64 (virtual) weight rows x one K slice; its 4 waves split the slice.  Each wave keeps
// PD k-blocks (4 KB each: two weight and two activation fragments) in flight in a register ring;
// two workgroups fit a CU, i.e. 8 waves x 32 KB in flight per CU.  Loads past the wave's range
// re-fetch the last block (cache hits, never used), which keeps the ring's wait counts static.
// The 4 waves are summed in wave order through LDS; the S slices of K are summed in slice order
// by the epilogue kernel.  S depends on (N, K) only, so results never depend on the CU share.
// ---------------------------------------------------------------------------------------------
// RT = 32-row weight tiles per workgroup (and per wave: the 4 waves split K, not rows)
#define RS_SKINNY_RT 2
static inline int skinny_virtual_n(int N, int epi) {
    constexpr int VT = 32 * RS_SKINNY_RT;   // virtual rows per workgroup; SwiGLU: half gate, half up
    return epi == EPI_SWIGLU ? ((N + VT / 2 - 1) / (VT / 2)) * VT : ((N + VT - 1) / VT) * VT;
}
static inline int skinny_kblocks(int K) { return (K + 15) / 16; }
static inline int skinny_splits(int N, int K, int epi) {
    const int tiles = skinny_virtual_n(N, epi) / (32 * RS_SKINNY_RT);
    const int Kb = skinny_kblocks(K);
    int S = 1;
    // enough workgroups for one per CU and more, but at least 8 k-blocks per wave
    while (tiles * S < RS_SKINNY_TARGET_WGS && S < 16 && Kb / (2 * S) >= 32) S *= 2;
    return S;
}
static inline int skinny_kb_per_wg(int K, int S) {
    const int per = (skinny_kblocks(K) + S - 1) / S;
    return ((per + 3) / 4) * 4;  // 4 waves
}
static inline int shared_virtual_n(int N, int epi);
static inline int shared_splits(int N, int K, int epi);
size_t skinny_partial_elems(int M, int N, int K, int epi) {
    const size_t plain = (size_t)skinny_splits(N, K, epi) * (size_t)M * (size_t)skinny_virtual_n(N, epi);
    const size_t shared = (size_t)shared_splits(N, K, epi) * (size_t)M * (size_t)shared_virtual_n(N, epi);
    return std::max(plain, shared);
}
size_t packed_weight_elems(int N, int K) {
    return (size_t)((N + 63) / 64) * 2 * (size_t)skinny_kblocks(K) * 512;
}

// One thread per 16-byte chunk of the packed matrix.
__global__ __launch_bounds__(256) void pack_weights_kernel(const bf16_t *__restrict__ W, bf16_t *__restrict__ Wp,
                                                           int N, int K, int Kb, long n_chunks) {
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n_chunks) return;
    const int lane = (int)(idx & 63);
    const long blk = idx >> 6;
    const int Nt = ((N + 63) / 64) * 2;
    const int t = (int)(blk % Nt), kb = (int)(blk / Nt);
    const int row = 32 * t + (lane & 31), k0 = 16 * kb + 8 * (lane >> 5);
    bf16x8 v = zero_bf16x8();
    if (row < N) {
        if (k0 + 8 <= K) {
            v = ld_bf16x8(W + (size_t)row * K + k0);
        } else {
            for (int i = 0; i < 8; ++i)
                if (k0 + i < K) v[i] = W[(size_t)row * K + k0 + i];
        }
    }
    st_bf16x8(Wp + idx * 8, v);
}

void launch_pack_weights(hipStream_t st, const bf16_t *W, bf16_t *Wp, int N, int K) {
    const long n_chunks = (long)(packed_weight_elems(N, K) / 8);
    hipLaunchKernelGGL(pack_weights_kernel, dim3((unsigned)((n_chunks + 255) / 256)), dim3(256), 0, st, W, Wp, N, K,
                       skinny_kblocks(K), n_chunks);
}

template <int EPI, int RT, int PD>
__global__ __launch_bounds__(256, RT <= 2 ? 2 : 1) void gemm_skinny_kernel(GemmArgs a, float *__restrict__ part,
                                                          int kb_per_wg, int Kb, int Nv) {
    // RT * 32 KB: the waves' accumulators for the in-order reduction, [wave][tile][lane][16]
    extern __shared__ __attribute__((aligned(1024))) float red[];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int c32 = lane & 31, h = lane >> 5;
    const int M = a.M;
    const int kbw = kb_per_wg >> 2;
    const int kb0 = __builtin_amdgcn_readfirstlane(blockIdx.y * kb_per_wg + wave * kbw);
    const int nsteps = max(min(kb0 + kbw, Kb) - kb0, 0);
    const int kb_last = Kb - 1;

    // the workgroup's RT row tiles in the packed matrices.  SwiGLU: virtual tile t is gate (t even) or
    // up (t odd) tile RT/2 * blockIdx.x + t/2, so gate and up of a feature sit 32 virtual columns apart
    const int Nt = ((a.N + 63) / 64) * 2;
    const size_t wstride = (size_t)Nt * 512, tstride = 512;   // elements per k block / per row tile
    const bf16_t *w[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        if (EPI == EPI_SWIGLU)
            w[t] = ((t & 1) ? a.Wp2 : a.Wp) + (size_t)min((RT / 2) * (int)blockIdx.x + (t >> 1), Nt - 1) * tstride + lane * 8;
        else
            w[t] = a.Wp + (size_t)min(RT * (int)blockIdx.x + t, Nt - 1) * tstride + lane * 8;
    }
    const bf16_t *x = a.A + lane * 8;

    f32x16 acc[RT][2];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    bf16x8 rw[PD][RT], rx[PD][2];
    auto load = [&](int p, int step) {
        const size_t kb = (size_t)min(kb0 + step, kb_last);
#pragma unroll
        for (int t = 0; t < RT; ++t) rw[p][t] = ld_bf16x8_stream(w[t] + kb * wstride);
        rx[p][0] = ld_bf16x8(x + kb * 1024);
        rx[p][1] = ld_bf16x8(x + kb * 1024 + 512);
    };
#pragma unroll
    for (int p = 0; p < PD; ++p) load(p, p);
    auto step = [&](int p) {
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            acc[t][0] = mfma32(rw[p][t], rx[p][0], acc[t][0]);
            acc[t][1] = mfma32(rw[p][t], rx[p][1], acc[t][1]);
        }
    };
    // whole rings: branch free, so the wait in front of each step is "all but the PD-1 younger steps"
    int i = 0;
    for (; i + PD <= nsteps; i += PD) {
#pragma unroll
        for (int p = 0; p < PD; ++p) {
            step(p);
            load(p, i + p + PD);
            __builtin_amdgcn_sched_barrier(0);   // refill the ring slot at once: keeps the bytes in flight level
        }
    }
    // the last, partial ring is already in flight
    const int rem = nsteps - i;
#pragma unroll
    for (int p = 0; p < PD; ++p)
        if (p < rem) step(p);
    // in-order reduction of the 4 waves
#pragma unroll
    for (int tn = 0; tn < RT; ++tn)
#pragma unroll
        for (int tm = 0; tm < 2; ++tm)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f32x4 v = {acc[tn][tm][4 * j], acc[tn][tm][4 * j + 1], acc[tn][tm][4 * j + 2], acc[tn][tm][4 * j + 3]};
                *(f32x4 *)&red[(((wave * (2 * RT) + tn * 2 + tm) * 4 + j) * 64 + lane) * 4] = v;   // lanes 16 bytes apart: no bank conflicts
            }
    __syncthreads();
    // wave w finishes tiles w, w + 4, ...: sum of the 4 waves in wave order
#pragma unroll
    for (int q = 0; q < (2 * RT) / 4; ++q) {
        const int tile = wave + 4 * q, tn = tile >> 1, tm = tile & 1;
        const int m = 32 * tm + c32;
        if (m < M) {
            float *dst = part + ((size_t)blockIdx.y * M + m) * Nv + blockIdx.x * (32 * RT) + 32 * tn;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f32x4 v = *(const f32x4 *)&red[(((0 * (2 * RT) + tile) * 4 + j) * 64 + lane) * 4];
#pragma unroll
                for (int ww = 1; ww < 4; ++ww) v += *(const f32x4 *)&red[(((ww * (2 * RT) + tile) * 4 + j) * 64 + lane) * 4];
                *(f32x4 *)(dst + 8 * j + 4 * h) = v;
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Skinny kernel, shared activations (used for the wide gate/up matrix).  A CU moves about 55 GB/s
// through its vector memory path whether the bytes come from HBM or from L2 (measured: the plain
// weight stream of gemm_skinny_kernel reaches 50 GB/s per CU, and 30 once every wave also fetches
// its own activation fragments, which are as many bytes as the weights).  Here the 4 waves of a
// workgroup take different rows over the SAME K slice, so the slice's activation k-blocks are
// fetched once per workgroup into LDS (a quarter of the bytes) and read from there:
//   * K is cut into chunks of CH k-blocks; the chunk's activations (CH x 2 KB) sit in one of two
//     LDS slabs; while chunk c is computed each wave fetches its 8 pieces of chunk c+1's slab, one
//     per step, through the same register ring as its weights (so all loads stay register loads,
//     in order, exact wait counts) and stores them to the other slab when their ring slot comes
//     up; one barrier per chunk (s_barrier after lgkmcnt(0): the weight ring is NOT drained);
//   * no K split inside the workgroup, hence no LDS reduction: each wave writes its own 64 x 64
//     partial tile; K is split S ways across workgroups, summed in slice order by the epilogue
//     kernel as before (S depends on the shape only).
// ---------------------------------------------------------------------------------------------
#define RS_SHARED_CH 16
static inline bool skinny_shared_applies(const GemmArgs &a) {
    if (skinny_kblocks(a.K) % (4 * RS_SHARED_CH) != 0 || a.N < 4096) return false;
    return a.epi == EPI_SWIGLU || (a.epi == EPI_RESIDUAL && a.K >= 8192);   // wide, or long enough in K to split 8 ways
}
static inline int shared_virtual_n(int N, int epi) {
    return epi == EPI_SWIGLU ? ((N + 127) / 128) * 256 : ((N + 255) / 256) * 256;
}
static inline int shared_splits(int N, int K, int epi) {
    const int tiles = shared_virtual_n(N, epi) / 256;
    const int Kb = skinny_kblocks(K);
    int S = 1;
    while (tiles * S < 224 && S < 16 && Kb % (2 * S * RS_SHARED_CH) == 0 && Kb / (2 * S) >= 4 * RS_SHARED_CH) S *= 2;
    return S;
}

template <int EPI, int CH, bool HEAD = false>
__global__ __launch_bounds__(256, 2) void gemm_skinny_shared_kernel(GemmArgs a, float *__restrict__ part, int kb_per_wg,
                                                                     int Kb, int Nv, HeadOut ho) {
    constexpr int PD = 8;                      // ring depth; divides CH, so ring slots are static in the unrolled chunk
    static_assert(CH % PD == 0 && CH * 2 == 32, "4 waves x 8 pieces fill one slab");
    extern __shared__ __attribute__((aligned(1024))) bf16_t slab[];   // [2][CH][2 token tiles][64 lanes][8]
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int c32 = lane & 31, h = lane >> 5;
    const int M = a.M;
    const int kb_begin = blockIdx.y * kb_per_wg;
    const int nchunks = kb_per_wg / CH;
    const int kb_last = Kb - 1;
    const int Nt = ((a.N + 63) / 64) * 2;
    const size_t wstride = (size_t)Nt * 512;
    const bf16_t *w0, *w1;
    if (EPI == EPI_SWIGLU) {   // wave w: gate tile and up tile of feature tile 4 * blockIdx.x + w
        const int f = min(4 * (int)blockIdx.x + wave, Nt - 1);
        w0 = a.Wp + (size_t)f * 512 + lane * 8;
        w1 = a.Wp2 + (size_t)f * 512 + lane * 8;
    } else {
        w0 = a.Wp + (size_t)min(8 * (int)blockIdx.x + 2 * wave, Nt - 1) * 512 + lane * 8;
        w1 = a.Wp + (size_t)min(8 * (int)blockIdx.x + 2 * wave + 1, Nt - 1) * 512 + lane * 8;
    }
    const bf16_t *x = a.A + lane * 8;

    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // piece q (0..31) of a chunk's slab = 1 KB = (k-block q/2, token tile q%2); wave w fetches pieces 8w .. 8w+7
    auto x_piece = [&](int chunk, int j) {
        const int q = 8 * wave + j;
        const size_t kb = (size_t)min(kb_begin + chunk * CH + (q >> 1), kb_last);
        return ld_bf16x8(x + kb * 1024 + (q & 1) * 512);
    };
    // chunk 0's slab, up front
    {
        bf16x8 t[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = x_piece(0, j);
#pragma unroll
        for (int j = 0; j < 8; ++j) *(bf16x8 *)&slab[(8 * wave + j) * 512 + lane * 8] = t[j];
    }
    bf16x8 rw0[PD], rw1[PD], rxs[PD];
    auto load_w = [&](int p, int step) {   // step counts k-blocks from kb_begin
        const size_t kb = (size_t)min(kb_begin + step, kb_last);
        rw0[p] = ld_bf16x8_stream(w0 + kb * wstride);
        rw1[p] = ld_bf16x8_stream(w1 + kb * wstride);
    };
#pragma unroll
    for (int p = 0; p < PD; ++p) load_w(p, p);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");

    for (int c = 0; c < nchunks; ++c) {
        const bf16_t *cur = slab + (c & 1) * (CH * 1024) + lane * 8;
        bf16_t *nxt = slab + ((c + 1) & 1) * (CH * 1024);
#pragma unroll
        for (int s = 0; s < CH; ++s) {
            const int p = s % PD;
            const bf16x8 x0 = *(const bf16x8 *)&cur[(2 * s) * 512], x1 = *(const bf16x8 *)&cur[(2 * s + 1) * 512];
            acc[0][0] = mfma32(rw0[p], x0, acc[0][0]);
            acc[0][1] = mfma32(rw0[p], x1, acc[0][1]);
            acc[1][0] = mfma32(rw1[p], x0, acc[1][0]);
            acc[1][1] = mfma32(rw1[p], x1, acc[1][1]);
            // the piece of the next slab that was fetched into this slot PD steps ago
            if (s >= PD && s - PD < 8) *(bf16x8 *)&nxt[(8 * wave + (s - PD)) * 512 + lane * 8] = rxs[p];
            load_w(p, c * CH + s + PD);
            if (s < 8) rxs[p] = x_piece(c + 1, s);
            __builtin_amdgcn_sched_barrier(0);
        }
        // every wave has read slab c and written its pieces of slab c+1; the weight loads stay in flight
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
    if (HEAD) {
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            f32x4 row[8];
#pragma unroll
            for (int v = 0; v < 8; ++v)
#pragma unroll
                for (int i = 0; i < 4; ++i) row[v][i] = acc[v >> 2][tm][4 * (v & 3) + i];
            const int m = 32 * tm + c32, n0 = blockIdx.x * 256 + wave * 64 + 4 * h;
            head_row<2>(ho, row, [&](int v) { return n0 + 8 * v; }, m, m < M, a.N, h == 0, blockIdx.x * 4 + wave);
        }
        return;
    }
    // each wave owns its rows: partial tile straight from the accumulators
#pragma unroll
    for (int tn = 0; tn < 2; ++tn)
#pragma unroll
        for (int tm = 0; tm < 2; ++tm) {
            const int m = 32 * tm + c32;
            if (m >= M) continue;
            float *dst = part + ((size_t)blockIdx.y * M + m) * Nv + blockIdx.x * 256 + wave * 64 + 32 * tn;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f32x4 v = {acc[tn][tm][4 * j], acc[tn][tm][4 * j + 1], acc[tn][tm][4 * j + 2], acc[tn][tm][4 * j + 3]};
                *(f32x4 *)(dst + 8 * j + 4 * h) = v;
            }
        }
}

// Sums the K slices in order and applies the epilogue; one thread per 4 output columns.
template <int EPI>
__global__ __launch_bounds__(256) void skinny_epilogue_kernel(GemmArgs a, const float *__restrict__ part,
                                                              int S, int Nv) {
    const int M = a.M, N = a.N;
    const int groups = N >> 2;
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= M * groups) return;
    const int m = idx / groups, n = (idx % groups) * 4;
    bf16x4 v;
    if (EPI == EPI_SWIGLU) {
        const int col = (n >> 5) * 64 + (n & 31);
        f32x4 g = {0.f, 0.f, 0.f, 0.f}, u = {0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < S; ++s) {
            const float *p = part + ((size_t)s * M + m) * Nv + col;
            g += *(const f32x4 *)p;
            u += *(const f32x4 *)(p + 32);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = (bf16_t)(silu_f(g[i]) * u[i]);
    } else {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < S; ++s) acc += *(const f32x4 *)(part + ((size_t)s * M + m) * Nv + n);
        if (EPI == EPI_RESIDUAL) {
            const bf16x4 r = *(const bf16x4 *)(a.resid + (size_t)m * N + n);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = (bf16_t)(acc[i] + (float)r[i]);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = (bf16_t)acc[i];
        }
    }
    store_out4<EPI>(a, m, n, v);
}

template <int EPI>
static void launch_skinny_epi(hipStream_t st, const GemmArgs &a, float *partials) {
    if (EPI != EPI_STORE && skinny_shared_applies(a)) {
        constexpr int CH = RS_SHARED_CH, lds = 2 * CH * 2048;
        const int Nv = shared_virtual_n(a.N, a.epi), S = shared_splits(a.N, a.K, a.epi);
        const int kbpw = skinny_kblocks(a.K) / S;
        hipLaunchKernelGGL((gemm_skinny_shared_kernel<EPI, CH>), dim3(Nv / 256, S), dim3(256), lds, st, a, partials, kbpw,
                           skinny_kblocks(a.K), Nv, HeadOut{});
        hipLaunchKernelGGL(skinny_epilogue_kernel<EPI>, dim3((a.M * (a.N / 4) + 255) / 256), dim3(256), 0, st, a, partials, S, Nv);
        return;
    }
    constexpr int RT = RS_SKINNY_RT, PD = 10;   // (RT + 2) * PD loads per wave in flight; at most 63 can be outstanding (gemm_kernels_init uses the same pair)
    constexpr int lds = RT * 32768;
    const int Nv = skinny_virtual_n(a.N, a.epi);
    const int S = skinny_splits(a.N, a.K, a.epi);
    const int kbpw = skinny_kb_per_wg(a.K, S);
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void *)gemm_skinny_kernel<EPI, RT, PD>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        attr_set = true;
    }
    const int eblocks = (a.M * (a.N / 4) + 255) / 256;
    hipLaunchKernelGGL((gemm_skinny_kernel<EPI, RT, PD>), dim3(Nv / (32 * RT), S), dim3(256), lds, st, a, partials, kbpw,
                       skinny_kblocks(a.K), Nv);
    hipLaunchKernelGGL(skinny_epilogue_kernel<EPI>, dim3(eblocks), dim3(256), 0, st, a, partials, S, Nv);
}

static inline bool head_streams(int N, int K) { return K % 16 == 0 && skinny_kblocks(K) % (4 * RS_SHARED_CH) == 0 && N >= 4096; }

void launch_gemm_skinny_partials(hipStream_t st, const GemmArgs &a, float *partials, int *S_out, int *Nv_out) {
    if (head_streams(a.N, a.K)) {
        constexpr int CH = RS_SHARED_CH;
        const int Nv = shared_virtual_n(a.N, EPI_STORE), S = shared_splits(a.N, a.K, EPI_STORE);
        *S_out = S;
        *Nv_out = Nv;
        if (a.M <= 0 || a.N <= 0) return;
        hipLaunchKernelGGL((gemm_skinny_shared_kernel<EPI_STORE, CH>), dim3(Nv / 256, S), dim3(256), 2 * CH * 2048, st, a, partials,
                           skinny_kblocks(a.K) / S, skinny_kblocks(a.K), Nv, HeadOut{});
        return;
    }
    constexpr int RT = RS_SKINNY_RT, PD = 10;
    const int Nv = skinny_virtual_n(a.N, EPI_STORE), S = skinny_splits(a.N, a.K, EPI_STORE);
    *S_out = S;
    *Nv_out = Nv;
    if (a.M <= 0 || a.N <= 0) return;
    hipLaunchKernelGGL((gemm_skinny_kernel<EPI_STORE, RT, PD>), dim3(Nv / (32 * RT), S), dim3(256), RT * 32768, st, a, partials,
                       skinny_kb_per_wg(a.K, S), skinny_kblocks(a.K), Nv);
}

// LM head with the greedy choice begun in the epilogue.  Up to 64 rows the weight-streaming kernel, one workgroup per 256
// columns over the whole K (a vocabulary too narrow to fill the chip that way takes K slices and launch_head_argmax);
// above that the large-tile kernel, tiles of 128, 192 or 256 rows (a decode step of one layer and the head, without and with
// 192: 130 rows 429 -> 400 us, 150 rows 464 -> 408, 192 rows 484 -> 451).
// The product used to leave its float32 sums in a scratch matrix that one workgroup per row read back, chose from and
// copied to the caller's logits: at 256 rows of a 128256-wide head 106 us of argmax behind 323 us of product (131 MB
// written, read and written again, and 1002 tiles of 128x256 where 501 of 256x256 are two rounds); now 251 + 4 us.
int head_candidates(int M, int N, int K) {
    if (M < 1 || N % 4) return 0;
    if (M <= 64 && head_streams(N, K)) return shared_splits(N, K, EPI_STORE) == 1 ? shared_virtual_n(N, EPI_STORE) / 64 : 0;
    return K % 32 == 0 && K >= 32 && N >= 1024 ? (N + 255) / 256 * 2 : 0;
}
void launch_gemm_head(hipStream_t st, const GemmArgs &a, const HeadOut &o) {
    if (a.M <= 64 && head_streams(a.N, a.K)) {
        hipLaunchKernelGGL((gemm_skinny_shared_kernel<EPI_STORE, RS_SHARED_CH, true>), dim3(shared_virtual_n(a.N, EPI_STORE) / 256), dim3(256),
                           2 * RS_SHARED_CH * 2048, st, a, (float *)nullptr, skinny_kblocks(a.K), skinny_kblocks(a.K), 0, o);
        return;
    }
    // as few row tiles of at most 256 rows as hold the batch, each no higher than needed (of heights whose waves stand two by
    // two: head_candidates counts on two column halves)
    const int n_tiles = (a.N + 255) / 256, m_tiles = (a.M + 255) / 256, height = (a.M + 32 * m_tiles - 1) / (32 * m_tiles);
    const dim3 grid((m_tiles * n_tiles + 7) / 8 * 8);
    auto go = [&](auto kernel, int bm, int ns) { hipLaunchKernelGGL(kernel, grid, dim3(256), ns * (bm + 256) * 64, st, a, o, m_tiles, n_tiles); };
    if (height <= 4) go(gemm_head_kernel<128, 5>, 128, 5);
    else if (height <= 6) go(gemm_head_kernel<192, 4>, 192, 4);
    else go(gemm_head_kernel<256, RS_NS_FULL>, 256, RS_NS_FULL);
}

void launch_gemm_skinny(hipStream_t st, const GemmArgs &a, float *partials) {
    if (a.M <= 0 || a.N <= 0) return;
    // A residual projection too short in K for the shared-activation kernel (the attention output projection)
    // has few, short K ranges per wave in the streaming kernel; the K-sliced large-tile kernel serves it better
    // on a partition (8B layer, 64 rows: 27 -> 21 us on 128 CUs, equal on 256).  A function of the shape alone.
    if (a.epi == EPI_RESIDUAL && !skinny_shared_applies(a) && a.K % 32 == 0 && a.K >= 512 && a.Wp && a.N >= 1024 && a.N % 4 == 0 &&
        a.partials == partials && a.partial_cap > 0) {
        int S = skinny_direct_splits(a.N, a.K);
        while (S > 1 && (size_t)S * a.M * a.N > a.partial_cap) S /= 2;
        if (S > 1) {
            launch_direct_splitk(st, a, S);
            return;
        }
    }
    switch (a.epi) {
        case EPI_STORE: launch_skinny_epi<EPI_STORE>(st, a, partials); break;
        case EPI_RESIDUAL: launch_skinny_epi<EPI_RESIDUAL>(st, a, partials); break;
        default: launch_skinny_epi<EPI_SWIGLU>(st, a, partials); break;
    }
}

// Raises the dynamic-LDS limit of every kernel that needs more than the default, once, at context
// creation: nothing but launches is then left for a call that may run under stream capture.
void gemm_kernels_init() {
    auto set = [](const void *f, int lds) { (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds); };
    auto set_nt = [&](const void *f, const void *nt, int lds) { set(f, lds), set(nt, lds); };
    grouped_kernels_init();
    constexpr int RT = RS_SKINNY_RT, PD = 10;
    set((const void *)gemm_skinny_kernel<EPI_STORE, RT, PD>, RT * 32768);
    set((const void *)gemm_skinny_kernel<EPI_RESIDUAL, RT, PD>, RT * 32768);
    set((const void *)gemm_skinny_kernel<EPI_SWIGLU, RT, PD>, RT * 32768);
    set((const void *)gemm_skinny_shared_kernel<EPI_SWIGLU, RS_SHARED_CH>, 2 * RS_SHARED_CH * 2048);
    set((const void *)gemm_skinny_shared_kernel<EPI_STORE, RS_SHARED_CH>, 2 * RS_SHARED_CH * 2048);
    set((const void *)gemm_skinny_shared_kernel<EPI_STORE, RS_SHARED_CH, true>, 2 * RS_SHARED_CH * 2048);
    set((const void *)gemm_head_kernel<128, 5>, 122880);
    set((const void *)gemm_head_kernel<192, 4>, 114688);
    set((const void *)gemm_head_kernel<256, RS_NS_FULL>, RS_NS_FULL * 32768);
    set((const void *)gemm_skinny_shared_kernel<EPI_RESIDUAL, RS_SHARED_CH>, 2 * RS_SHARED_CH * 2048);
    set((const void *)gemm_direct_splitk_kernel<128, 5>, 122880);
    set((const void *)gemm_direct_splitk_kernel<160, 4>, 106496);
    set((const void *)gemm_tall_splitk_kernel<9, 4>, 139264);
    set((const void *)gemm_tall_splitk_kernel<10, 4>, 147456);
    set_nt((const void *)gemm_tall_kernel<9, EPI_STORE, 4, false>, (const void *)gemm_tall_kernel<9, EPI_STORE, 4, true>, 139264);
    set_nt((const void *)gemm_tall_kernel<9, EPI_RESIDUAL, 4, false>, (const void *)gemm_tall_kernel<9, EPI_RESIDUAL, 4, true>, 139264);
    set_nt((const void *)gemm_tall_kernel<9, EPI_SWIGLU, 4, false>, (const void *)gemm_tall_kernel<9, EPI_SWIGLU, 4, true>, 139264);
    set_nt((const void *)gemm_tall_kernel<10, EPI_STORE, 4, false>, (const void *)gemm_tall_kernel<10, EPI_STORE, 4, true>, 147456);
    set_nt((const void *)gemm_tall_kernel<10, EPI_RESIDUAL, 4, false>, (const void *)gemm_tall_kernel<10, EPI_RESIDUAL, 4, true>, 147456);
    set_nt((const void *)gemm_tall_kernel<10, EPI_SWIGLU, 4, false>, (const void *)gemm_tall_kernel<10, EPI_SWIGLU, 4, true>, 147456);
    set((const void *)gemm_direct_splitk_kernel<192, 4>, 114688);
    set((const void *)gemm_direct_splitk_kernel<224, 4>, 122880);
    set((const void *)gemm_direct_splitk_kernel<256, RS_NS_FULL>, RS_NS_FULL * 32768);
    set_nt((const void *)gemm_direct_mixed_kernel<EPI_STORE, true, false>, (const void *)gemm_direct_mixed_kernel<EPI_STORE, true, true>, RS_NS_FULL * 32768);
    set_nt((const void *)gemm_direct_mixed_kernel<EPI_RESIDUAL, true, false>, (const void *)gemm_direct_mixed_kernel<EPI_RESIDUAL, true, true>, RS_NS_FULL * 32768);
    set_nt((const void *)gemm_direct_mixed_kernel<EPI_SWIGLU, true, false>, (const void *)gemm_direct_mixed_kernel<EPI_SWIGLU, true, true>, RS_NS_FULL * 32768);
    set_nt((const void *)gemm_direct_kernel<256, 256, EPI_STORE, RS_NS_FULL, false>, (const void *)gemm_direct_kernel<256, 256, EPI_STORE, RS_NS_FULL, true>, RS_NS_FULL * 32768);
    set_nt((const void *)gemm_direct_kernel<256, 256, EPI_RESIDUAL, RS_NS_FULL, false>, (const void *)gemm_direct_kernel<256, 256, EPI_RESIDUAL, RS_NS_FULL, true>, RS_NS_FULL * 32768);
    set_nt((const void *)gemm_direct_kernel<256, 256, EPI_SWIGLU, RS_NS_FULL, false>, (const void *)gemm_direct_kernel<256, 256, EPI_SWIGLU, RS_NS_FULL, true>, RS_NS_FULL * 32768);
    set_nt((const void *)gemm_fed_kernel<EPI_STORE, false>, (const void *)gemm_fed_kernel<EPI_STORE, true>, RS_FED_LDS);
    set_nt((const void *)gemm_direct_kernel<160, 256, EPI_STORE, 4, false>, (const void *)gemm_direct_kernel<160, 256, EPI_STORE, 4, true>, 106496);
    set_nt((const void *)gemm_direct_kernel<192, 256, EPI_STORE, 4, false>, (const void *)gemm_direct_kernel<192, 256, EPI_STORE, 4, true>, 114688);
    set_nt((const void *)gemm_direct_kernel<224, 256, EPI_STORE, 4, false>, (const void *)gemm_direct_kernel<224, 256, EPI_STORE, 4, true>, 122880);
    set_nt((const void *)gemm_fed_kernel<EPI_RESIDUAL, false>, (const void *)gemm_fed_kernel<EPI_RESIDUAL, true>, RS_FED_LDS);
    set_nt((const void *)gemm_direct_kernel<160, 256, EPI_RESIDUAL, 4, false>, (const void *)gemm_direct_kernel<160, 256, EPI_RESIDUAL, 4, true>, 106496);
    set_nt((const void *)gemm_direct_kernel<192, 256, EPI_RESIDUAL, 4, false>, (const void *)gemm_direct_kernel<192, 256, EPI_RESIDUAL, 4, true>, 114688);
    set_nt((const void *)gemm_direct_kernel<224, 256, EPI_RESIDUAL, 4, false>, (const void *)gemm_direct_kernel<224, 256, EPI_RESIDUAL, 4, true>, 122880);
    set_nt((const void *)gemm_direct_kernel<128, 256, EPI_SWIGLU, 5, false>, (const void *)gemm_direct_kernel<128, 256, EPI_SWIGLU, 5, true>, 122880);
    set_nt((const void *)gemm_direct_kernel<160, 256, EPI_SWIGLU, 4, false>, (const void *)gemm_direct_kernel<160, 256, EPI_SWIGLU, 4, true>, 106496);
    set_nt((const void *)gemm_direct_kernel<192, 256, EPI_SWIGLU, 4, false>, (const void *)gemm_direct_kernel<192, 256, EPI_SWIGLU, 4, true>, 114688);
    set_nt((const void *)gemm_direct_kernel<224, 256, EPI_SWIGLU, 4, false>, (const void *)gemm_direct_kernel<224, 256, EPI_SWIGLU, 4, true>, 122880);
    set_nt((const void *)gemm_direct_mixed_kernel<EPI_SWIGLU, false, false>, (const void *)gemm_direct_mixed_kernel<EPI_SWIGLU, false, true>, RS_NS_FULL * 28672);
    set_nt((const void *)gemm_direct_kernel<192, 128, EPI_SWIGLU, 5, false>, (const void *)gemm_direct_kernel<192, 128, EPI_SWIGLU, 5, true>, 102400);
    set_nt((const void *)gemm_direct_kernel<256, 192, EPI_STORE, 4, false>, (const void *)gemm_direct_kernel<256, 192, EPI_STORE, 4, true>, 114688);
    set_nt((const void *)gemm_direct_kernel<256, 192, EPI_RESIDUAL, 4, false>, (const void *)gemm_direct_kernel<256, 192, EPI_RESIDUAL, 4, true>, 114688);
}

