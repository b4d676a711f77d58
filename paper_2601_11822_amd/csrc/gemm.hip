// bf16 GEMMs out = epi(A[M,K] * W[N,K]^T) on the gfx950 matrix cores (fp32 accumulation).
//
// A lane's 8-element MFMA fragment is 8 consecutive k of one row: one 16-byte chunk, and the unit
// of the fragment-packed operand layout (packed_offset) that the activations are always stored in.
// The weight tile is the MFMA "row" operand and the activation tile the "column" operand:
// a lane then owns 4 consecutive output columns of one output row, which makes the epilogues
// (residual add, SwiGLU, bf16 pack) per-lane code; the direct kernel's row-major outputs pass through LDS on their way (store_rows).
#include <algorithm>
#include <type_traits>
#include <utility>

#include "kernels.h"

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// z * sigmoid(z); the reciprocal is the hardware's one-instruction approximation (1 ulp): an IEEE division costs
// ten more vector instructions per element of a 256x256 epilogue, for digits far below the bf16 the result is rounded to
__device__ __forceinline__ float silu_f(float z) { return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
// f(integral_constant 0) .. f(integral_constant N - 1): straight-line code whose indices are constants before the optimizer runs
template <class F, int... I>
__device__ __forceinline__ void static_for_each(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_each(f, std::make_integer_sequence<int, N>{});
}
#define RS_INLINE __attribute__((always_inline))
// 4 consecutive output columns (n % 4 == 0) of row m
template <int EPI>
__device__ __forceinline__ void store_out4(const GemmArgs &a, int m, int n, bf16x4 v) {
    bf16_t *dst = EPI == EPI_SWIGLU ? a.out + packed_offset(m, n, packed_mt(a.M)) + (n & 7) : a.out + (size_t)m * a.N + n;
    *(bf16x4 *)dst = v;
}

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

// ---------------------------------------------------------------------------------------------
// Direct kernel (K % 32 == 0): the tiled kernel's product with larger tiles of more shapes; both operands
// are read in the fragment-packed layout (activations as their producers wrote them, weights from
// the library's packed copies) and go global -> LDS with the 16-byte LDS-DMA load (no register
// staging) through a ring of NS LDS stages of BK = 32, so that a K tile is requested NS-1 tiles
// (several microseconds of MFMA work) before it is consumed: HBM latency is covered although only
// one wave runs per SIMD.
//
// A wave-wide load moves one 1 KB fragment block (32 rows x 16 k), lane l fetching and storing
// chunk l: the slab of a K tile is BM/32 + BN/32 contiguous kilobytes per k block, which spreads
// over the memory channels (a row-major operand would give one 64-byte piece per 2K-byte-strided
// row, crowding a few channels: the DMA fill rate of this tile walk measured 13 TB/s row-major
// and 22 TB/s packed).  In LDS a block keeps the lane order, so a fragment read is four runs of 16
// consecutive 16-byte chunks: conflict free without a swizzle.  Row tiles past M or N are not fetched
// (their results are never stored); K tiles past the end re-fetch the last tile into a stage
// nobody reads, which keeps the loop body branch free.
//
// Per K tile (one MFMA step of K = 32, one barrier): the loads of tile kt+NS-1 and the reads of tile kt+1's
// fragments, into the register set that tile kt does not use, trickle out between the MFMAs.  The barrier stands in the
// middle (vmcnt counts the younger loads that may still fly): tile kt+1 has landed, and every wave has read tile kt.
// Earlier slots for it cost 0.2 to 0.5 % of a layer, other slots for the reads and loads nothing, a fifth stage nothing.
//
// 16x16x32 products, not 32x32x16: a product of some rounds of tiles on the whole chip runs at the power limit, and the smaller
// accumulator tile moves half as many accumulator bits per multiplication.  Four waves a CU on random operands, registers
// alone, hold 1.77 PFLOP/s with 32x32x16 and 2.05 with 16x16x32; with the fragment reads of this tile 1.68 and 1.92.
// The sums are the same bits.
//
// One wave runs per SIMD, so every instruction issued between two MFMAs that takes longer than the
// MFMA itself (16 cycles) leaves the matrix core idle.  The loop therefore issues one fragment read or one load between
// two MFMAs, and a load is one instruction: a buffer load whose constant offset counts in memory and in LDS alike, so
// that the loads of a wave, consecutive kilobytes of one k block, share their lane offset and LDS address; the slab bases
// advance by scalar adds once per K tile.  Layers of the 8B widths with 32x32x16 / 16x16x32 and vector addresses /
// this: 2048 rows 818 / 784 / 750 us, 16384 rows 7870 / 7600 / 7370, 5444 rows of the 70B widths 7690 / 7400 / 7000; gate/up of the
// latter 3908 -> 3472 us, 1.31 -> 1.47 PFLOP/s (matrix cores 80 % busy in both, at 1.61 and 1.82 GHz).
// (One copy of the loop serves all four waves; a copy each, so that a wave could place its loads a quarter-spacing after its
// neighbour's, costs the registers their allocation: the copies' 256 accumulators meet behind the loop, through scratch memory.)
// ---------------------------------------------------------------------------------------------
// LM head: the float32 logits (if wanted) and the best (value, column) of row m, taken straight from the accumulators: a lane has
// the columns col(v) .. col(v) + 3 in vector v, ascending, the GROUPS lanes of equal lane % (64 / GROUPS) have the whole row between
// them.  NaN never wins; the lowest column wins among equals.
template <int GROUPS, int NV, class Col>
__device__ __forceinline__ void head_row(const HeadOut &o, const f32x4 (&acc)[NV], Col col, int m, bool m_ok, int N, bool first, int cand) {
    float best = -__builtin_huge_valf();
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int n = col(v);
        if (n >= N) continue;
        if (o.logits && m_ok) *(f32x4 *)(o.logits + (size_t)m * N + n) = acc[v];
#pragma unroll
        for (int i = 0; i < 4; ++i) best = fmaxf(best, acc[v][i]);
    }
    int arg = 0x7fffffff;
#pragma unroll
    for (int v = NV - 1; v >= 0; --v)
#pragma unroll
        for (int i = 3; i >= 0; --i) {
            const int n = col(v) + i;
            if (n < N && acc[v][i] == best) arg = n;
        }
#pragma unroll
    for (int x = 64 / GROUPS; x < 64; x *= 2) {
        const float vo = __shfl_xor(best, x, 64);
        const int ao = __shfl_xor(arg, x, 64);
        if (vo > best || (vo == best && ao < arg)) { best = vo; arg = ao; }
    }
    if (first && m_ok) {
        o.cand_val[(size_t)m * o.n_cand + cand] = best;
        o.cand_idx[(size_t)m * o.n_cand + cand] = arg;
    }
}

// A wave's accumulators leave as whole rows.  In a register a lane holds 4 consecutive columns of one row, so a store from there
// touches 32 rows, 16 (bf16) or 32 bytes (float32) of a line each; through LDS, 32 rows at a time, it writes runs as long as the wave's
// columns (128 of them 256 or 512 bytes; 64, in tiles of 160 and 224 rows, half that; 96 of 256x192 192 bytes, not all on a line's
// start), and the residual is read the same way.  The wave's strip (32 rows of 4 more floats than it has columns, so that the 16-byte
// writes of 8 neighbouring rows fall on different banks) is its own: no barrier after the first, which frees the ring.
// Bound by the write of the tile, once every compute unit stores at the same time.  2048x4096x4096 with residual 72 -> 62 us,
// 2048x8192x512 30 -> 23 us; K slices of 128x256 sums 37.8 -> 34.8 us (576x6144x4096 in two).
// F32: raw sums to dst[m][n] (row stride N, a multiple of 4), else bf16 to a.out (a multiple of 8), with the residual if RES.
template <int TM, int TN, bool F32, bool RES>
__device__ __forceinline__ void store_rows(const GemmArgs &a, const f32x4 (&acc)[2 * TN][2 * TM], float *dst, int m_base, int n0, bf16_t *smem, int wave, int lane) {
    constexpr int WN = 32 * TN, LD = WN + 4, EPC = F32 ? 4 : 8, CPR = WN / EPC, IT = 32 * CPR / 64;   // 16-byte chunks: per row, per lane
    const int c16 = lane & 15, g = lane >> 4, M = a.M, N = a.N;
    float *buf = (float *)smem + wave * (32 * LD);
    __syncthreads();
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
        const int m0 = m_base + 32 * tm;
        if (m0 >= M) break;
        bf16x8 r[IT];
        if (RES) {
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int q = it * 64 + lane;
                r[it] = ld_bf16x8(a.resid + (size_t)min(m0 + q / CPR, M - 1) * N + min(n0 + (q % CPR) * EPC, N - 8));
            }
        }
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
            for (int tn = 0; tn < 2 * TN; ++tn) *(f32x4 *)&buf[(16 * half + c16) * LD + 16 * tn + 4 * g] = acc[tn][2 * tm + half];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the strip is read by other lanes than wrote it
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int q = it * 64 + lane, row = q / CPR, col = (q % CPR) * EPC;
            const int m = m0 + row, n = n0 + col;
            const f32x4 lo = *(const f32x4 *)&buf[row * LD + col];
            if (F32) {
                if (m < M && n < N) *(f32x4 *)(dst + (size_t)m * N + n) = lo;
            } else {
                const f32x4 hi = *(const f32x4 *)&buf[row * LD + col + 4];
                bf16x8 v;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float x = i < 4 ? lo[i & 3] : hi[i & 3];
                    v[i] = (bf16_t)(RES ? x + (float)r[it][i] : x);
                }
                if (m < M && n < N) st_bf16x8(a.out + (size_t)m * N + n, v);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read before the next rows overwrite it
    }
}

// One output tile: rows [bm, bm + BM), column tile nb (of width BN; BN/2 output columns for SwiGLU).
// HEAD: the epilogue is head_row above.  PARTIAL: the tile covers K tiles [kt0, kt0 + nk_part) only and stores its raw float32 sums to
// part[z][m][n] (row stride N), for an epilogue pass that adds the slices in order.
// NT: the weights are fetched as a stream (non-temporal: first out of the L2).  Right where few row tiles share a slab and all of
// them run at once: K slices, the head, expert tiles (grouped_streams_weights), whole products of few row tiles (direct_streams).
// LDS stages of the 256x256 tile's ring (32 KB each): a K tile is requested three tiles ahead.  A fifth stage (the
// whole 160 KB of a compute unit) measured the same, alone and beside a bandwidth-bound kernel on the other
// partition: what that neighbour costs is not memory latency the ring could cover.
#define RS_NS_FULL 4
template <int BM, int BN, int EPI, int NS, bool PARTIAL = false, bool HEAD = false, bool NT = PARTIAL || HEAD>
__device__ __forceinline__ void gemm_direct_tile(const GemmArgs &a, const int bm, const int nb, bf16_t *smem,
                                                 const int kt0 = 0, const int nk_part = 0, float *part = nullptr, const int z = 0,
                                                 const HeadOut *ho = nullptr, const int blocks = BM / 32) {
    constexpr int BK = 32;
    constexpr int WGM = BM % 64 ? 1 : 2;             // four waves: 2 along M x 2 along N, or all along N (a height of an odd number of row blocks)
    constexpr int WGN = 4 / WGM;
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int TM = WM / 32, TN = WN / 32;
    constexpr int TA = BM / 32, TB = BN / 32;        // 32-row blocks per k block of the tile
    constexpr int LB = TB / 2;                       // wave-wide loads of weights per wave per stage
    constexpr int STAGE = (BM + BN) * BK;            // elements per stage: [2][TA] A blocks, then [2][TB] B blocks
    constexpr int D = NS - 1;                        // prefetch distance in K tiles
    // the slots of a K tile that the barrier is in front of (the fragment reads follow it), and that its first load is behind
    constexpr int BAR = 2 * TN * TM < 4 * TN * TM - 1 - 2 * (TN + TM) ? 2 * TN * TM : 4 * TN * TM - 1 - 2 * (TN + TM), LSLOT = 2;
    static_assert(!HEAD || WGN == 2, "two candidates per row and column tile");
    static_assert(BAR > 0, "a K tile must have a slot per fragment read");

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wm = wave / WGN, wn = wave % WGN;
    const int c16 = lane & 15, g16 = lane >> 4;
    const int M = a.M, N = a.N, K = a.K;
    const int Mt = packed_mt(M), Nt = ((N + 63) / 64) * 2;   // row tiles per k block of A and of the weights

    const size_t ksa = (size_t)Mt * 1024, ksb = (size_t)Nt * 1024;   // elements per K tile (2 k blocks)
    const int nk = PARTIAL ? nk_part : K / BK;

    f32x4 acc[2 * TN][2 * TM];
#pragma unroll
    for (int i = 0; i < 2 * TN; ++i)
#pragma unroll
        for (int j = 0; j < 2 * TM; ++j) {
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            asm volatile("" : "+a"(acc[i][j]));
        }

    {
        // A wave brings half of one k block of either operand: consecutive kilobytes in memory and in LDS, so that its loads share a
        // lane offset and an LDS address and differ in the instruction's constant.  (An odd number of blocks: the first half is larger.)
        constexpr int LA = (TA + 1) / 2, LEAST = TA / 2 + LB;   // loads of a K tile of the waves that have fewer
        constexpr int SL = 4 * TN * TM, LT = LA + LB, SP = SL / LT, NF = 2 * (TN + TM);
        // loads of the current K tile already issued when the barrier of slot BAR is reached, by the waves that skip load LA - 1 too
        constexpr int PLACED = BAR > LSLOT ? (BAR - 1 - LSLOT) / SP + 1 : 0, EARLY = PLACED - (TA % 2 && PLACED >= LA ? 1 : 0);
        const int W = __builtin_amdgcn_readfirstlane(wave), kb = W >> 1, second = W & 1;
        const bool more = !second || TA % 2 == 0;
        constexpr int TBH = TB / 2;   // SwiGLU: a k block's first half is gate rows, its second half the matching up rows
        // Its part of K tile 0: from there to the last block that there is (of a tile past the edge, or of an expert's last unit) is the
        // buffer of its loads; what lies behind is not fetched, and the results it gives are of no row that anybody reads.
        const int t0a = (bm >> 5) + second * LA, t0b = EPI == EPI_SWIGLU ? nb * TBH : nb * TB + second * TBH;
        const int bytes_a = max(min(Mt - t0a, blocks - second * LA), 0) * 1024, bytes_b = max(Nt - t0b, 0) * 1024;
        const char *ga = (const char *)(a.A + (size_t)kt0 * ksa + (size_t)(kb * Mt + t0a) * 512);
        const char *gb = (const char *)((EPI == EPI_SWIGLU && second ? a.Wp2 : a.Wp) + (size_t)kt0 * ksb + (size_t)(kb * Nt + t0b) * 512);
        int fetch_kt = 0;   // the K tile they point at
        auto advance = [&]() RS_INLINE {   // to the next K tile, staying on the last one (its re-fetches land in a stage nobody reads)
            const size_t in = fetch_kt + 1 < nk ? 1 : 0;
            ga += in * ksa * 2;
            gb += in * ksb * 2;
            ++fetch_kt;
        };
        // the j-th of this wave's LA + LB loads that bring the K tile at ga, gb into the stage at element offset so
        auto issue = [&](int so, auto jtag) RS_INLINE {
            constexpr int j = decltype(jtag)::value;
            if constexpr (j < LA) {
                if (j >= TA / 2 && !more) return;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void *)ga, 0, bytes_a, 0x00020000),
                                                         (__attribute__((address_space(3))) void *)(smem + so + (kb * TA + second * LA) * 512), 16, lane * 16, 0, j * 1024, 0);
            } else {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void *)gb, 0, bytes_b, 0x00020000),
                                                         (__attribute__((address_space(3))) void *)(smem + so + BM * BK + (kb * TB + second * TBH) * 512), 16, lane * 16, 0,
                                                         (j - LA) * 1024, NT ? 2 : 0);
            }
        };
        bf16x8 wf[2][2 * TN], xf[2][2 * TM];
        // A fragment of 16 rows x 32 k: lane (row c16, 8-wide k group g16) finds its 16 bytes in k block g16 >> 1
        const int la = ((g16 >> 1) * TA + wm * TM) * 512 + ((g16 & 1) * 32 + c16) * 8;
        const int lb = BM * BK + ((g16 >> 1) * TB + wn * (EPI == EPI_SWIGLU ? TN / 2 : TN)) * 512 + ((g16 & 1) * 32 + c16) * 8;
        // the f-th fragment to be used of the K tile in the stage at element offset so: weights 0, all activations, the other weights
        auto read_frag = [&](auto stag, int so, auto ftag) RS_INLINE {
            constexpr int set = decltype(stag)::value, f = decltype(ftag)::value;
            if constexpr (f >= 1 && f <= 2 * TM) {
                constexpr int t = f - 1;
                xf[set][t] = *(const bf16x8 *)&smem[so + la + (t >> 1) * 512 + (t & 1) * 128];
            } else {
                constexpr int t = f == 0 ? 0 : f - 2 * TM;
                constexpr int blk = EPI == EPI_SWIGLU ? (t >> 2) + ((t >> 1) & 1) * TBH : t >> 1;   // gate and up blocks in turn
                wf[set][t] = *(const bf16x8 *)&smem[so + lb + blk * 512 + (t & 1) * 128];
            }
        };
        // prologue: K tiles 0 .. D-1 into stages 0 .. D-1
        static_for<D>([&](auto i) RS_INLINE {
            static_for<LT>([&](auto j) RS_INLINE { issue(decltype(i)::value * STAGE, j); });
            advance();
        });
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((D - 1) * LEAST) : "memory");
        static_for<NF>([&](auto f) RS_INLINE { read_frag(std::integral_constant<int, 0>{}, 0, f); });

        // One K tile = SL MFMA slots; its loads fill the stage before its own (tile kt + D), and it reads the fragments of the
        // next tile into the other register set, both between the MFMAs.
        int so_cur = 0;   // element offset of the stage that holds K tile kt (uniform)
        auto k_tile = [&](auto stag) RS_INLINE {
            constexpr int SET = decltype(stag)::value;
            const int so_ld = so_cur == 0 ? (NS - 1) * STAGE : so_cur - STAGE;
            const int so_nxt = so_cur == (NS - 1) * STAGE ? 0 : so_cur + STAGE;
            static_for<SL>([&](auto sltag) RS_INLINE {
                constexpr int sl = decltype(sltag)::value, tn = sl / (2 * TM), tm = sl % (2 * TM);
                if constexpr (sl == BAR)
                    // tile kt+1 has landed once only the younger loads are outstanding; this wave's
                    // LDS reads are complete before it tells the others so at the barrier
                    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((D - 2) * LEAST + EARLY) : "memory");
                acc[tn][tm] = mfma16(wf[SET][tn], xf[SET][tm], acc[tn][tm]);
                __builtin_amdgcn_sched_barrier(0);
                // read f goes behind slot BAR + f * (SL - BAR - 1) / NF
                constexpr int f = ((sl - BAR) * NF + SL - BAR - 2) / (SL - BAR - 1);
                if constexpr (sl >= BAR && f < NF && BAR + f * (SL - BAR - 1) / NF == sl)
                    read_frag(std::integral_constant<int, 1 - SET>{}, so_nxt, std::integral_constant<int, f>{});
                if constexpr (sl >= LSLOT && (sl - LSLOT) % SP == 0 && (sl - LSLOT) / SP < LT) issue(so_ld, std::integral_constant<int, (sl - LSLOT) / SP>{});
                __builtin_amdgcn_sched_barrier(0);
            });
            advance();
            so_cur = so_nxt;
        };
#pragma clang loop unroll(disable)
        for (int kt = 0; kt < nk >> 1; ++kt) {
            k_tile(std::integral_constant<int, 0>{});
            k_tile(std::integral_constant<int, 1>{});
        }
        if (nk & 1) k_tile(std::integral_constant<int, 0>{});
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");

    if (HEAD) {
#pragma unroll
        for (int tm = 0; tm < 2 * TM; ++tm) {
            const int m = bm + wm * WM + 16 * tm + c16;
            f32x4 row[2 * TN];
#pragma unroll
            for (int tn = 0; tn < 2 * TN; ++tn) row[tn] = acc[tn][tm];
            const int n0 = nb * BN + wn * WN + 4 * g16;
            head_row<4>(*ho, row, [&](int v) { return n0 + 16 * v; }, m, m < M, N, g16 == 0, nb * WGN + wn);
        }
        return;
    }
    if (PARTIAL) {
        store_rows<TM, TN, true, false>(a, acc, part + (size_t)z * M * N, bm + wm * WM, nb * BN + wn * WN, smem, wave, lane);
        return;
    }
    if (EPI != EPI_SWIGLU) {
        store_rows<TM, TN, false, EPI == EPI_RESIDUAL>(a, acc, nullptr, bm + wm * WM, nb * BN + wn * WN, smem, wave, lane);
        return;
    }
    // SwiGLU, fragment-packed, without a branch per store: the 4 columns c0 + 16q + 4g (c0 a multiple of 32) of row m sit at
    // row_term(m) + col_term(c0, g) + q * S16, where a step of 16 columns is S16 = Mt*512 elements.
    // 16 rows of a store are two 256-byte runs.
    const size_t S16 = (size_t)Mt * 512;
    const int c0 = nb * (BN / 2) + wn * (TN / 2) * 32;
    constexpr int NQ = TN / 2;
    const size_t col_term = (size_t)(c0 >> 4) * S16 + (g16 >> 1) * 256 + (g16 & 1) * 4;
    const bool whole = c0 + 32 * NQ <= N;     // wave-uniform: no column of this wave's tile is past the edge
    auto rows = [&](auto checked) {
#pragma unroll
        for (int tm = 0; tm < 2 * TM; ++tm) {
            const int m = bm + wm * WM + 16 * tm + c16;
            if (m >= M) continue;
            bf16_t *dst = a.out + (size_t)(m >> 5) * 512 + (size_t)(m & 31) * 8 + col_term;
#pragma unroll
            for (int q = 0; q < 2 * NQ; ++q) {
                if (decltype(checked)::value && c0 + 16 * q + 4 * g16 >= N) continue;
                const f32x4 &gate = acc[4 * (q >> 1) + (q & 1)][tm], &up = acc[4 * (q >> 1) + 2 + (q & 1)][tm];
                bf16x4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = (bf16_t)(silu_f(gate[i]) * up[i]);
                *(bf16x4 *)(dst + (size_t)q * S16) = v;
            }
        }
    };
    if (whole) rows(std::false_type{});
    else rows(std::true_type{});
}

// One output tile by eight waves, two per SIMD, each with XF x 4 accumulators of 16 x 16 (WGM waves along the rows, the others along the
// columns): tiles of up to 320 x 256 or 640 x 128, where four waves end at 256 x 256.  Every element's sum is in gemm_direct_tile's order.
// What it is for: a CU has some 32 KB of loads in flight however many it has asked for (57 to 61 GB/s from HBM, 131 from L2), and a product of
// a few rounds of tiles is bound by that, not by its matrix instructions; a taller tile asks for its weights once where two lower ones ask for them twice.
// The registers: 160 accumulators, the activations' fragments (40) once and the weights' (32) twice: a wave's products go through the activation
// fragments one after the other, and the one that is done with is read again for the next K tile.  No more than 256 in all, all of them vector
// registers (a function that uses accumulation registers gets half of each, which spills).
// What bounds it: the LDS.  A K tile of 320 x 256 is 112 KB of fragment reads and 36 KB of DMA writes beside 1280 cycles of products, 1156 at 128 bytes
// a cycle; the place of the barrier, the reads and the loads among the products changes nothing.
// rows_end: rows from here on are not stored; blocks: 32-row blocks from here on are not fetched.
#define RS_TALL_LDS 163840   // all of a compute unit's: at most NS stages of BM + BN rows of 64 bytes
template <int XF, int WGM, int EPI, int NS, bool NT, bool PARTIAL = false>
__device__ __forceinline__ void gemm_tall_tile(const GemmArgs &a, const int bm, const int nb, bf16_t *smem, const int blocks, const int rows_end,
                                               const int kt0 = 0, const int nk_part = 0, float *part = nullptr) {
    constexpr int BK = 32, WGN = 8 / WGM, BM = 16 * XF * WGM, BN = 64 * WGN;
    static_assert(WGM == 2 || WGM == 4, "the wave's 16-row units lie WGM apart, which puts them at one LDS stride");
    static_assert(NS * (BM + BN) * 64 <= RS_TALL_LDS, "the ring");
    constexpr int TA = BM / 32, TB = BN / 32, LA = (TA + 3) / 4, LB = TB / 4, LT = LA + LB, LEAST = TA / 4 + LB;
    constexpr int STAGE = (BM + BN) * BK, SL = 4 * XF, NF = 4 + XF;
    constexpr int BAR = SL / 4 < 4 ? 4 : SL / 4;                          // the slot that the barrier is in front of
    constexpr int RSTEP = (SL - 1 - BAR) / (NF - 1) < 1 ? 1 : (SL - 1 - BAR) / (NF - 1), LSTEP = (SL - 2 - BAR) / LT < 1 ? 1 : (SL - 2 - BAR) / LT;

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wm = wave / WGN, wn = wave % WGN;
    const int c16 = lane & 15, g16 = lane >> 4;
    const int M = a.M, N = a.N, K = a.K;
    const int Mt = packed_mt(M), Nt = ((N + 63) / 64) * 2;
    const size_t ksa = (size_t)Mt * 1024, ksb = (size_t)Nt * 1024;
    const int nk = PARTIAL ? nk_part : K / BK;

    f32x4 acc[4][XF];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < XF; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    {
        constexpr int TBH = TB / 2;
        const int W = __builtin_amdgcn_readfirstlane(wave), kb = W >> 2, q = W & 3;
        const int na = TA / 4 + (q < TA % 4 ? 1 : 0), sa = q * (TA / 4) + min(q, TA % 4);
        const int t0a = (bm >> 5) + sa, t0b = EPI == EPI_SWIGLU ? nb * TBH + (q & 1) * LB : nb * TB + q * LB;
        const int bytes_a = __builtin_amdgcn_readfirstlane(max(min(min(Mt - t0a, blocks - sa), na), 0) * 1024), bytes_b = __builtin_amdgcn_readfirstlane(max(min(Nt - t0b, LB), 0) * 1024);
        const char *ga = (const char *)(a.A + (size_t)kt0 * ksa + (size_t)(kb * Mt + t0a) * 512);
        const char *gb = (const char *)((EPI == EPI_SWIGLU && q >= 2 ? a.Wp2 : a.Wp) + (size_t)kt0 * ksb + (size_t)(kb * Nt + t0b) * 512);
        int fetch_kt = 0;
        auto advance = [&]() RS_INLINE {
            const size_t in = fetch_kt + 1 < nk ? 1 : 0;
            ga += in * ksa * 2;
            gb += in * ksb * 2;
            ++fetch_kt;
        };
        auto issue = [&](int so, auto jtag) RS_INLINE {
            constexpr int j = decltype(jtag)::value;
            if constexpr (j < LA) {
                if (j >= TA / 4 && j >= na) return;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void *)ga, 0, bytes_a, 0x00020000),
                                                         (__attribute__((address_space(3))) void *)(smem + so + (kb * TA + sa) * 512), 16, lane * 16, 0, j * 1024, 0);
            } else {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void *)gb, 0, bytes_b, 0x00020000),
                                                         (__attribute__((address_space(3))) void *)(smem + so + BM * BK + (kb * TB + q * LB) * 512), 16, lane * 16, 0,
                                                         (j - LA) * 1024, NT ? 2 : 0);
            }
        };
        bf16x8 wf[2][4], xf[XF];
        const int la = (g16 >> 1) * TA * 512 + ((g16 & 1) * 32 + c16) * 8 + (WGM == 2 ? wm * 128 : (wm >> 1) * 512 + (wm & 1) * 128);
        const int lb = BM * BK + ((g16 >> 1) * TB + (EPI == EPI_SWIGLU ? wn : 2 * wn)) * 512 + ((g16 & 1) * 32 + c16) * 8;
        auto read_frag = [&](auto stag, int so, auto ftag) RS_INLINE {
            constexpr int set = decltype(stag)::value, f = decltype(ftag)::value;
            if constexpr (f >= 4) xf[f - 4] = *(const bf16x8 *)&smem[so + la + (f - 4) * (WGM == 2 ? 512 : 1024)];
            else wf[set][f] = *(const bf16x8 *)&smem[so + lb + (f >> 1) * (EPI == EPI_SWIGLU ? TBH : 1) * 512 + (f & 1) * 128];
        };
        static_for<NS>([&](auto i) RS_INLINE {
            static_for<LT>([&](auto j) RS_INLINE { issue(decltype(i)::value * STAGE, j); });
            advance();
        });
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 1) * LEAST) : "memory");
        static_for<NF>([&](auto f) RS_INLINE { read_frag(std::integral_constant<int, 0>{}, 0, f); });

        int so_cur = 0;
        auto k_tile = [&](auto stag) RS_INLINE {
            constexpr int SET = decltype(stag)::value;
            const int so_nxt = so_cur == (NS - 1) * STAGE ? 0 : so_cur + STAGE;
            static_for<SL>([&](auto sltag) RS_INLINE {
                constexpr int sl = decltype(sltag)::value, t = sl >> 2, c = sl & 3;
                if constexpr (sl == BAR) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 2) * LEAST) : "memory");
                acc[c][t] = mfma16(wf[SET][c], xf[t], acc[c][t]);
                __builtin_amdgcn_sched_barrier(0);
                static_for<NF>([&](auto ftag) RS_INLINE {
                    constexpr int f = decltype(ftag)::value, due = BAR + f * RSTEP > SL - 1 ? SL - 1 : BAR + f * RSTEP, last = 4 * (f - 4) + 3;
                    if constexpr ((f >= 4 && last > due ? last : due) == sl) read_frag(std::integral_constant<int, 1 - SET>{}, so_nxt, ftag);
                });
                static_for<LT>([&](auto jtag) RS_INLINE {
                    constexpr int j = decltype(jtag)::value, due = BAR + 1 + j * LSTEP > SL - 1 ? SL - 1 : BAR + 1 + j * LSTEP;
                    if constexpr (due == sl) issue(so_cur, jtag);
                });
                __builtin_amdgcn_sched_barrier(0);
            });
            advance();
            so_cur = so_nxt;
        };
#pragma clang loop unroll(disable)
        for (int kt = 0; kt < nk >> 1; ++kt) {
            k_tile(std::integral_constant<int, 0>{});
            k_tile(std::integral_constant<int, 1>{});
        }
        if (nk & 1) k_tile(std::integral_constant<int, 0>{});
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    const int m_end = min(M, rows_end);
    if constexpr (EPI == EPI_SWIGLU) {
        const size_t S16 = (size_t)Mt * 512;
        const int c0 = nb * (BN / 2) + wn * 32;
        const size_t col_term = (size_t)(c0 >> 4) * S16 + (g16 >> 1) * 256 + (g16 & 1) * 4;
#pragma unroll
        for (int t = 0; t < XF; ++t) {
            const int m = bm + (t * WGM + wm) * 16 + c16;
            if (m >= m_end) continue;
            bf16_t *dst = a.out + (size_t)(m >> 5) * 512 + (size_t)(m & 31) * 8 + col_term;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (c0 + 16 * q + 4 * g16 >= N) continue;
                const f32x4 &gate = acc[q][t], &up = acc[2 + q][t];
                bf16x4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = (bf16_t)(silu_f(gate[i]) * up[i]);
                *(bf16x4 *)(dst + (size_t)q * S16) = v;
            }
        }
    } else {
        // rows of the wave's 64 columns, 16 at a time through LDS (store_rows)
        constexpr int LD = 68, EPC = PARTIAL ? 4 : 8, CPR = 64 / EPC, IT = 16 * CPR / 64;
        float *buf = (float *)smem + wave * (16 * LD);
        const int n0 = nb * BN + wn * 64;
        __syncthreads();
#pragma unroll
        for (int t = 0; t < XF; ++t) {
            const int m0 = bm + (t * WGM + wm) * 16;
            if (m0 >= m_end) break;
            bf16x8 r[IT];
            if (EPI == EPI_RESIDUAL && !PARTIAL) {
#pragma unroll
                for (int it = 0; it < IT; ++it) {
                    const int q = it * 64 + lane;
                    r[it] = ld_bf16x8(a.resid + (size_t)min(m0 + q / CPR, m_end - 1) * N + min(n0 + (q % CPR) * EPC, N - 8));
                }
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) *(f32x4 *)&buf[c16 * LD + 16 * c + 4 * g16] = acc[c][t];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the strip is read by other lanes than wrote it
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int q = it * 64 + lane, row = q / CPR, col = (q % CPR) * EPC, m = m0 + row, n = n0 + col;
                const f32x4 lo = *(const f32x4 *)&buf[row * LD + col];
                if constexpr (PARTIAL) {
                    if (m < m_end && n < N) *(f32x4 *)(part + (size_t)m * N + n) = lo;
                } else {
                    const f32x4 hi = *(const f32x4 *)&buf[row * LD + col + 4];
                    bf16x8 v;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const float x = i < 4 ? lo[i & 3] : hi[i & 3];
                        v[i] = (bf16_t)(EPI == EPI_RESIDUAL ? x + (float)r[it][i] : x);
                    }
                    if (m < m_end && n < N) st_bf16x8(a.out + (size_t)m * N + n, v);
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read before the next rows overwrite it
        }
    }
}

// Order of the output tiles: super columns of four column tiles, inside one the row tiles four at a time, a
// 4 x 4 block column by column.  Tiles that run at the same time on an XCD (16 on half the chip, 32 on the whole
// chip) then share four weight slabs and four or eight activation slabs, whatever the number of row tiles: with
// plain column-major order an XCD's set was all rows of one or two columns, and each round re-read the whole
// activation matrix.
__device__ __forceinline__ void tile_rc(int t, int m_tiles, int n_tiles, int &r, int &c) {
    constexpr int CW = 4, RH = 4;
    const int per_sc = CW * m_tiles;
    const int sc = t / per_sc, c0 = sc * CW;
    const int w = min(CW, n_tiles - c0);      // the last super column may be narrower
    const int u = t - sc * per_sc;
    const int rb = u / (RH * w), r0 = rb * RH;
    const int hgt = min(RH, m_tiles - r0);    // the last row block may be lower
    const int v = u - rb * (RH * w);
    r = r0 + v % hgt;
    c = c0 + v / hgt;
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
// slices was forced in turn, 12 row counts of the 8B widths from 200 to 8000 on 256 and 128 CUs and four of the 70B widths
// (profiles/large_tile_forms_forced.md): the forms are within 1 % of the fastest layer; the slices, which may not follow the CUs, within 2 %
// on the whole chip and 6 % on half of it.)
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
static bool direct_streams(int m_tiles) { return m_tiles <= 4; }

template <int EPI, bool TALL>
static void launch_direct_mixed(hipStream_t st, const GemmArgs &a, int cus) {
    constexpr int BM = TALL ? 256 : 192;
    const int m_tiles = (a.M + BM - 1) / BM, n_tiles = EPI == EPI_SWIGLU ? (a.N + 127) / 128 : (a.N + 255) / 256;
    const int n_full = m_tiles * n_tiles / cus * cus, n_half = 2 * (m_tiles * n_tiles - n_full);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(n_full + (n_half + 7) / 8 * 8), dim3(256), RS_NS_FULL * (BM + 256) * 64, st, a, m_tiles, n_full, n_half);
    };
    direct_streams(m_tiles) ? go(gemm_direct_mixed_kernel<EPI, TALL, true>) : go(gemm_direct_mixed_kernel<EPI, TALL, false>);
}

template <int BM, int BN, int EPI, int NS>
static void launch_direct_epi(hipStream_t st, const GemmArgs &a) {
    const int m_tiles = (a.M + BM - 1) / BM;
    const int n_tiles = (EPI == EPI_SWIGLU) ? (a.N + BN / 2 - 1) / (BN / 2) : (a.N + BN - 1) / BN;
    const int total = m_tiles * n_tiles;
    const int grid = ((total + 7) / 8) * 8;
    constexpr int lds = NS * (BM + BN) * 32 * 2;
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(grid), dim3(BM > 256 ? 512 : 256), lds, st, a, m_tiles, n_tiles); };
    if constexpr (BM > 256) direct_streams(m_tiles) ? go(gemm_tall_kernel<BM / 32, EPI, NS, true>) : go(gemm_tall_kernel<BM / 32, EPI, NS, false>);
    else direct_streams(m_tiles) ? go(gemm_direct_kernel<BM, BN, EPI, NS, true>) : go(gemm_direct_kernel<BM, BN, EPI, NS, false>);
}

template <int BM, int BN, int NS>
static void launch_direct(hipStream_t st, const GemmArgs &a) {
    switch (a.epi) {
        case EPI_STORE: launch_direct_epi<BM, BN, EPI_STORE, NS>(st, a); break;
        case EPI_RESIDUAL: launch_direct_epi<BM, BN, EPI_RESIDUAL, NS>(st, a); break;
        default: launch_direct_epi<BM, BN, EPI_SWIGLU, NS>(st, a); break;
    }
}

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
__global__ __launch_bounds__(512) void gemm_grouped_tall_kernel(GemmArgs a, int n_tiles, int cus) {
    extern __shared__ __attribute__((aligned(1024))) bf16_t smem[];
    const int nus = __builtin_amdgcn_readfirstlane(a.units[0]), nu = nus & 0xffff, nu_tall = nus >> 16;
    if (nu <= 0) return;
    const bool narrow = grouped_narrow(EPI == EPI_STORE, nu, n_tiles, cus);
    if (narrow) n_tiles = (a.N + 127) / 128;
    const int x = blockIdx.x & 7;
    const GroupPiece p = grouped_piece(x, blockIdx.x >> 3, nu_tall, nu - nu_tall, n_tiles, cus);
    GroupTile t = grouped_tile(x, p.i, p.tall ? nu_tall : nu - nu_tall, n_tiles);
    if (t.u < 0) return;
    if (!p.tall) t.u += nu_tall;
    const int code = __builtin_amdgcn_readfirstlane(a.units[2 + t.u]);
    const int row0 = (code >> 13) * 32, height = (code >> 5) & 15, blocks = (code >> 9) & 15;
    GemmArgs g = a;
    g.Wp += (size_t)(code & 31) * a.expert_stride;
    if (EPI == EPI_SWIGLU) g.Wp2 += (size_t)(code & 31) * a.expert_stride;
    const bool half = p.half >= 0 || narrow;
    const int nb = p.half >= 0 ? 2 * t.nb + p.half : t.nb;
    auto tile = [&](auto xf, auto wgm, auto ns) {
        gemm_tall_tile<decltype(xf)::value, decltype(wgm)::value, EPI, decltype(ns)::value, NT>(g, row0, nb, smem, blocks, row0 + 32 * height);
    };
#define RS_T(xf, wgm, ns) tile(std::integral_constant<int, xf>{}, std::integral_constant<int, wgm>{}, std::integral_constant<int, ns>{})
    if (half) {
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
    const int cus = a.cus > 0 ? a.cus : 256, most = (a.M >> 7) * n_tiles;   // of as many units as there can be
    if (a.tall) {   // and the second halves
        const int grid = (std::max(most + cus / 2, cus) + 7) / 8 * 8 + 8;
        hipLaunchKernelGGL((gemm_grouped_tall_kernel<EPI, NT>), dim3(grid), dim3(512), RS_TALL_LDS, st, a, n_tiles, cus);
    } else {        // of narrow tiles no more than CUs
        const int grid = (std::max(most, EPI == EPI_STORE ? cus : 0) + 7) / 8 * 8;
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
            case FORM_128x256: launch_direct<128, 256, 5>(st, a); break;            // 5 x 24 KB
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
    set((const void *)gemm_grouped_tall_kernel<EPI_STORE, true>, RS_TALL_LDS);
    set((const void *)gemm_grouped_tall_kernel<EPI_SWIGLU, true>, RS_TALL_LDS);
    set((const void *)gemm_grouped_tall_kernel<EPI_STORE, false>, RS_TALL_LDS);
    set((const void *)gemm_grouped_tall_kernel<EPI_SWIGLU, false>, RS_TALL_LDS);
    set((const void *)gemm_grouped_kernel<EPI_STORE, true>, RS_NS_FULL * 32768);
    set((const void *)gemm_grouped_kernel<EPI_SWIGLU, true>, RS_NS_FULL * 32768);
    set((const void *)gemm_grouped_kernel<EPI_STORE, false>, RS_NS_FULL * 32768);
    set((const void *)gemm_grouped_kernel<EPI_SWIGLU, false>, RS_NS_FULL * 32768);
    set_nt((const void *)gemm_direct_mixed_kernel<EPI_STORE, true, false>, (const void *)gemm_direct_mixed_kernel<EPI_STORE, true, true>, RS_NS_FULL * 32768);
    set_nt((const void *)gemm_direct_mixed_kernel<EPI_RESIDUAL, true, false>, (const void *)gemm_direct_mixed_kernel<EPI_RESIDUAL, true, true>, RS_NS_FULL * 32768);
    set_nt((const void *)gemm_direct_mixed_kernel<EPI_SWIGLU, true, false>, (const void *)gemm_direct_mixed_kernel<EPI_SWIGLU, true, true>, RS_NS_FULL * 32768);
    set_nt((const void *)gemm_direct_kernel<256, 256, EPI_STORE, RS_NS_FULL, false>, (const void *)gemm_direct_kernel<256, 256, EPI_STORE, RS_NS_FULL, true>, RS_NS_FULL * 32768);
    set_nt((const void *)gemm_direct_kernel<256, 256, EPI_RESIDUAL, RS_NS_FULL, false>, (const void *)gemm_direct_kernel<256, 256, EPI_RESIDUAL, RS_NS_FULL, true>, RS_NS_FULL * 32768);
    set_nt((const void *)gemm_direct_kernel<256, 256, EPI_SWIGLU, RS_NS_FULL, false>, (const void *)gemm_direct_kernel<256, 256, EPI_SWIGLU, RS_NS_FULL, true>, RS_NS_FULL * 32768);
    set_nt((const void *)gemm_direct_kernel<128, 256, EPI_STORE, 5, false>, (const void *)gemm_direct_kernel<128, 256, EPI_STORE, 5, true>, 122880);
    set_nt((const void *)gemm_direct_kernel<160, 256, EPI_STORE, 4, false>, (const void *)gemm_direct_kernel<160, 256, EPI_STORE, 4, true>, 106496);
    set_nt((const void *)gemm_direct_kernel<192, 256, EPI_STORE, 4, false>, (const void *)gemm_direct_kernel<192, 256, EPI_STORE, 4, true>, 114688);
    set_nt((const void *)gemm_direct_kernel<224, 256, EPI_STORE, 4, false>, (const void *)gemm_direct_kernel<224, 256, EPI_STORE, 4, true>, 122880);
    set_nt((const void *)gemm_direct_kernel<128, 256, EPI_RESIDUAL, 5, false>, (const void *)gemm_direct_kernel<128, 256, EPI_RESIDUAL, 5, true>, 122880);
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

