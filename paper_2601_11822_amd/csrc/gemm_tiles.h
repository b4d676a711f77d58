// Output tiles of the large-tile products on the gfx950 matrix cores: the device code that whole products, K slices, the head (gemm.hip) and
// the experts' products (gemm_grouped.hip) share.
#pragma once
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
// FED: eight waves, of which the last four only load.
#define RS_NS_FULL 4
template <int BM, int BN, int EPI, int NS, bool PARTIAL = false, bool HEAD = false, bool NT = PARTIAL || HEAD, bool FED = false>
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
    static_assert(!FED || (EPI != EPI_SWIGLU && !HEAD), "the barrier of store_rows");
    static_assert(BAR > 0, "a K tile must have a slot per fragment read");

    // The mask is the fed form's alone: in the others the compiler then forms the lanes' addresses in another way, and the experts' gate/up
    // tiles spill a register (300 rows through 16 experts of the 8B widths on 160 CUs: gate/up 831 us with it, 822 without).
    const int tid = threadIdx.x, wave = FED ? (tid >> 6) & 3 : tid >> 6, lane = tid & 63;
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
        if constexpr (FED) {
            // four more waves bring the operands, a whole ring ahead: the ones that multiply never wait to issue a load
            if (__builtin_amdgcn_readfirstlane(tid >> 8)) {
                static_for<NS>([&](auto i) RS_INLINE {
                    static_for<LT>([&](auto j) RS_INLINE { issue(decltype(i)::value * STAGE, j); });
                    advance();
                });
                asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 1) * LEAST) : "memory");
                int so = 0;
#pragma clang loop unroll(disable)
                for (int kt = 0; kt < nk; ++kt) {   // a barrier a K tile: the next one has landed, and this one's stage is free
                    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NS - 2) * LEAST) : "memory");
                    static_for<LT>([&](auto j) RS_INLINE { issue(so, j); });
                    advance();
                    so = so == (NS - 1) * STAGE ? 0 : so + STAGE;
                }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();   // store_rows' own
                return;
            }
        }
        // prologue: K tiles 0 .. D-1 into stages 0 .. D-1
        if constexpr (FED) {
            asm volatile("s_barrier" ::: "memory");
        } else {
            static_for<D>([&](auto i) RS_INLINE {
                static_for<LT>([&](auto j) RS_INLINE { issue(decltype(i)::value * STAGE, j); });
                advance();
            });
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((D - 1) * LEAST) : "memory");
        }
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
                if constexpr (FED && sl == BAR) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                if constexpr (!FED && sl == BAR)
                    // tile kt+1 has landed once only the younger loads are outstanding; this wave's
                    // LDS reads are complete before it tells the others so at the barrier
                    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((D - 2) * LEAST + EARLY) : "memory");
                acc[tn][tm] = mfma16(wf[SET][tn], xf[SET][tm], acc[tn][tm]);
                __builtin_amdgcn_sched_barrier(0);
                // read f goes behind slot BAR + f * (SL - BAR - 1) / NF
                constexpr int f = ((sl - BAR) * NF + SL - BAR - 2) / (SL - BAR - 1);
                if constexpr (sl >= BAR && f < NF && BAR + f * (SL - BAR - 1) / NF == sl)
                    read_frag(std::integral_constant<int, 1 - SET>{}, so_nxt, std::integral_constant<int, f>{});
                if constexpr (!FED && sl >= LSLOT && (sl - LSLOT) % SP == 0 && (sl - LSLOT) / SP < LT) issue(so_ld, std::integral_constant<int, (sl - LSLOT) / SP>{});
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (!FED) advance();
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
// columns): tiles of up to 320 x 256, and of 320 x 128, where four waves end at 256 x 256.  Every element's sum is in gemm_direct_tile's order.
// What it is for: a CU has some 32 KB of loads in flight however many it has asked for (57 to 61 GB/s from HBM, 131 from L2), and a product of
// a few rounds of tiles is bound by that, not by its matrix instructions; a taller tile asks for its weights once where two lower ones ask for them twice.
// The registers: 160 accumulators, the activations' fragments (40) once and the weights' (32) twice: a wave's products go through the activation
// fragments one after the other, and the one that is done with is read again for the next K tile.  No more than 256 in all, all of them vector
// registers (a function that uses accumulation registers gets half of each, which spills).
// What bounds it: the LDS.  A K tile of 320 x 256 is 112 KB of fragment reads and 36 KB of DMA writes beside 1280 cycles of products, 1184 at 128 bytes
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
