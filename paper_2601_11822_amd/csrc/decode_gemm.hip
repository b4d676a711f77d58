// Projections of a pass of at most RS_STREAM_ROWS rows: weight-streaming GEMMs with the RMSNorm folded in.
//
// Such a pass multiplies a few rows by every weight of the layer once (paper section 2.1: decode is
// bound by reading weights and cache, not by arithmetic; so is a prompt this short), so each of the four projections
// is a stream of its matrix through the matrix cores at the rate the partition's memory path allows, and everything
// around that stream is overhead to be removed:
//
//   * RMSNorm needs a whole row before it can scale an element, which would cost a kernel of its own in
//     front of the QKV and the gate/up projection.  But the row's scale is one scalar: with
//     s = 1/sqrt(mean(x^2) + eps),  RMSNorm(x; g) W^T = s * ((x . g) W^T).  The streaming kernel therefore
//     (QKV) reads the hidden state x row-major as it is, multiplies by the gain while it stages the rows in
//     LDS, and adds up the squares of the part of each row it sees; the per-slice sums of squares go out
//     beside the partial products, and their consumer (the rotary/KV epilogue) forms s and applies it.  The
//     gate/up projection's input has a producer, the output projection's epilogue: that writes x1 . g2 and the
//     sums of squares itself, so the widest stream of the layer copies its activations and converts nothing.
//   * The 4 waves of a workgroup take different weight rows over the SAME K slice, so the slice's
//     activation rows are fetched once per workgroup into LDS (double buffered, 16 k-blocks at a time)
//     and every wave's vector memory path carries weights only: each wave keeps PD one-kilobyte weight
//     fragments in flight in a register ring that is refilled right after the MFMAs that free a slot.
//   * K is cut into S slices so that every compute unit of a partition holds several workgroups; S and
//     the tile counts follow from (N, K) alone, and the slices are added in slice order by the epilogue,
//     so results do not depend on the CU share.  Loads past a slice's end re-read its last k-block
//     (cache hits), so the ring's wait counts stay static without fetching a byte of another slice.
#include <algorithm>

#include "kernels.h"

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// z * sigmoid(z); the reciprocal is the hardware's one-instruction approximation (1 ulp): an IEEE division costs
// ten more vector instructions per element of a 256x256 epilogue, for digits far below the bf16 the result is rounded to
__device__ __forceinline__ float silu_f(float z) { return z * __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

// The RMSNorm scale of row m from the sums of squares of its parts, added in order.  The first SSQ_BATCH parts (all of them
// up to a width of 8192) are requested together, wherever the caller has something to do meanwhile, and added later.
#define SSQ_BATCH 8
struct RowSsq {
    float v[SSQ_BATCH];
    __device__ __forceinline__ void request(const float *ssq_part, int S_ssq, int m) {
#pragma unroll
        for (int s = 0; s < SSQ_BATCH; ++s) v[s] = ssq_part[min(s, S_ssq - 1) * RS_SSQ_ROWS + m];
    }
    __device__ __forceinline__ float scale(const float *ssq_part, int S_ssq, int m, int d, float eps) const {
        float t = 0.f;
#pragma unroll
        for (int s = 0; s < SSQ_BATCH; ++s)
            if (s < S_ssq) t += v[s];
        for (int s = SSQ_BATCH; s < S_ssq; ++s) t += ssq_part[s * RS_SSQ_ROWS + m];
        return 1.0f / sqrtf(t / (float)d + eps);
    }
};

// Sum over the K slices, in slice order, of NV 4-float columns at p[0], p[off], ...; slices are requested SB at a time (one
// after the other they are a chain of memory round trips, which is all that bounds the small kernels here: a layer of one
// decode row 103.5 -> 97 us with this, RowSsq and decode_combine_kernel's batches).
template <int SB, int NV>
__device__ __forceinline__ void sum_slices(const float *p, int off, size_t stride, int S, f32x4 (&acc)[NV]) {
#pragma unroll
    for (int i = 0; i < NV; ++i) acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < S; s0 += SB) {
        f32x4 v[SB][NV];
#pragma unroll
        for (int s = 0; s < SB; ++s)
#pragma unroll
            for (int i = 0; i < NV; ++i) v[s][i] = *(const f32x4 *)(p + (size_t)min(s0 + s, S - 1) * stride + i * off);
#pragma unroll
        for (int s = 0; s < SB; ++s)
#pragma unroll
            for (int i = 0; i < NV; ++i)
                if (s0 + s < S) acc[i] += v[s][i];
    }
}

#define DS_INLINE_PIECES 12
#define FEW_PARTS (RS_FEW_COLS / 1024)   // parts of a row's sum of squares, where a pass of few rows forms it
#define DS_CH 16   // k-blocks per activation chunk: two slabs of MT x 16 KB in LDS

// ACT 0: activations fragment-packed (packed_mt(M) row tiles per k-block), as their producers write them.
// ACT 1: activations row-major [M][K]; multiplied by gain[K] while staged; sums of squares written out.
// RT   : 32-row weight tiles per wave.  MT: 32-row activation tiles, ceil(M / 32): rows past M are neither fetched
//        (their lanes repeat row M - 1) nor multiplied beyond the last tile that holds a row.
// PAIR : RT == 2 and the wave's two tiles are row tile f of Wp (gate) and of Wp2 (up); else RT tiles of Wp.
// PSPLIT: RT == 1 and the pair is spread over waves: waves 0-1 take gate tiles 2x, 2x+1 of Wp, waves 2-3 the matching
//         up tiles of Wp2 (half as many features per workgroup as PAIR, the same sums and the same output columns).
// A pair covers the whole K (one slice): its accumulators are the finished sums, so the row scale, SwiGLU and the packed
// output are the epilogue of this kernel and no partial products are written.
// Llama-3-8B gate/up on 256 CUs: at 64 rows 51.6 + 5.7 us with the gain and the squares formed in this stream (about 50
// vector instructions per staged kilobyte, more cycles than its matrix instructions) and SwiGLU in a kernel of its own,
// 47 us now; at one row 37.4 + 4.8 -> 36.8 us (6.4 TB/s).  A second row tile that holds no row is not staged or
// multiplied (QKV at one row 13.0 -> 10.9 us).
template <int ACT, int RT, bool PAIR, bool PSPLIT, int MT, bool SELF = false>
__global__ __launch_bounds__(256, MT > 2 ? 1 : 2) void dstream_kernel(DGemmArgs a, int kb_per_wg, int Nv, DFuseArgs fz) {
    constexpr int CH = DS_CH, PD = 8;
    // An activation piece is stored 8 steps after its load was issued, right behind a weight fragment that is
    // consumed PD steps after ITS issue: with PD == 8 the two are due together and the in-order wait counts cost
    // nothing; a deeper ring would make every piece wait for weights that are not needed yet (measured: 2x slower).
    // Taking the pieces out of these waves altogether -- one or two extra waves per workgroup that only stage the
    // next slab, the four streaming waves with a ring of 16 (128 KB of weights in flight per workgroup) -- gave the
    // same results and was slower on all 256 CUs (QKV 20.2 -> 23.9 us, gate/up 42.6 -> 50.4, output/down 21.3 -> 22.3)
    // and no faster beside a prefill pass on 128: depth in flight is not what bounds this stream.
    static_assert(CH % PD == 0, "ring slots are static inside an unrolled chunk");
    static_assert(!PAIR || RT == 2, "a pair is a gate tile and an up tile");
    static_assert(!PSPLIT || (RT == 1 && !PAIR), "a split pair is one tile per wave");
    constexpr bool FUSED = PAIR || PSPLIT;
    static_assert(!FUSED || ACT == 0, "a pair reads what the output projection's epilogue wrote");
    constexpr int NPC = 4 * MT;   // activation pieces (1 KB) a wave brings per chunk
    extern __shared__ __attribute__((aligned(1024))) bf16_t slab[];   // [2][CH][MT row tiles][64 lanes][8]
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int c32 = lane & 31, h = lane >> 5;
    const int M = a.M, K = a.K;
    const int kb_begin = blockIdx.y * kb_per_wg;
    const int kb_end = kb_begin + kb_per_wg - 1;     // loads past the slice re-read its last k-block
    const int nchunks = kb_per_wg / CH;
    const int Nt = ((a.N + 63) / 64) * 2;
    const size_t wstride = (size_t)Nt * 512, xstride = (size_t)packed_mt(M) * 512;
    const bf16_t *w[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        if (PAIR)
            w[t] = (t ? a.Wp2 : a.Wp) + (size_t)min(4 * (int)blockIdx.x + wave, Nt - 1) * 512 + lane * 8;
        else if (PSPLIT)
            w[t] = (wave >= 2 ? a.Wp2 : a.Wp) + (size_t)min(2 * (int)blockIdx.x + (wave & 1), Nt - 1) * 512 + lane * 8;
        else
            w[t] = a.Wp + (size_t)min((4 * (int)blockIdx.x + wave) * RT + t, Nt - 1) * 512 + lane * 8;
    }

    f32x16 acc[RT][MT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // ---- activation pieces: a chunk's slab is 16 MT pieces of 1 KB; wave w brings 4 MT of them per chunk
    // ACT 0: piece q = 4 MT w + j is (k-block q/MT, row tile q%MT) of the packed matrix.
    // ACT 1: piece j of wave w is rows 8j..8j+7 x the chunk's 16-byte columns 8w..8w+7 (lane l: row 8j + l%8,
    //        column 8w + l/8): eight 128-byte runs of eight rows, stored to the fragment order
    //        ((k-block*MT + row tile)*64 + half*32 + row%32).
    float ssq[NPC];
#pragma unroll
    for (int j = 0; j < NPC; ++j) ssq[j] = 0.f;
    const int k8 = 8 * wave + (lane >> 3);            // ACT 1: this lane's 16-byte column inside a chunk
    int xoff[MT];                                     // ACT 0: this lane's chunk of row tile t within a k-block
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const int r = min(32 * t + c32, M - 1);
        xoff[t] = (r >> 5) * 512 + (h * 32 + (r & 31)) * 8;
    }
    auto x_addr = [&](int chunk, int j) -> const bf16_t * {
        if (ACT == 0) {
            const size_t kb = (size_t)min(kb_begin + chunk * CH + 4 * wave + j / MT, kb_end);
            return a.A_packed + kb * xstride + xoff[j % MT];
        } else {
            const int m = min(8 * j + (lane & 7), M - 1);
            const int ch = min(chunk, nchunks - 1);
            return a.X_rows + (size_t)m * K + (size_t)(kb_begin + ch * CH) * 16 + k8 * 8;
        }
    };
    auto g_addr = [&](int chunk) -> const bf16_t * {
        const int ch = min(chunk, nchunks - 1);
        return a.gain + (size_t)(kb_begin + ch * CH) * 16 + k8 * 8;
    };
    const bool counts = ACT == 1 && blockIdx.x == 0;
    auto x_store = [&](bf16_t *dst_slab, int j, bf16x8 xv, const float (&gf)[8], bool count) {
        if (ACT == 0) {
            *(bf16x8 *)&dst_slab[(NPC * wave + j) * 512 + lane * 8] = xv;
        } else {
            const int m = 8 * j + (lane & 7);
            bf16x8 hv;
#pragma unroll
            for (int e = 0; e < 8; ++e) hv[e] = (bf16_t)((float)xv[e] * gf[e]);
            if (counts && count) {
                float s = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) s += (float)xv[e] * (float)xv[e];
                ssq[j] += s;
            }
            *(bf16x8 *)&dst_slab[(((k8 >> 1) * MT + (m >> 5)) * 64 + (k8 & 1) * 32 + (m & 31)) * 8] = hv;
        }
    };
    RowSsq rs[MT];   // FUSED: what this lane's rows' RMSNorm scales are made of
    __shared__ f32x4 self_ssq[SELF ? RS_FEW_ROWS : 1][FEW_PARTS];   // SELF: by row, part of 1024 and wave
    if (FUSED && !SELF) {
#pragma unroll
        for (int tm = 0; tm < MT; ++tm) rs[tm].request(fz.ssq_part, fz.S_ssq, 32 * tm + c32);
    }
    bf16x4 self[SELF ? RS_FEW_ROWS : 1][FEW_PARTS];   // requested in front of the weights, whose ring must not be waited for
    if (SELF)
#pragma unroll
        for (int r = 0; r < RS_FEW_ROWS; ++r) {
            if (r >= M) break;
#pragma unroll
            for (int i = 0; i < FEW_PARTS; ++i) self[r][i] = *(const bf16x4 *)(fz.rows + (size_t)r * K + min(1024 * i + 4 * tid, K - 4));
        }
    float gf[8];
    auto gains = [&](bf16x8 g) {
#pragma unroll
        for (int e = 0; e < 8; ++e) gf[e] = (float)g[e];
    };
    {   // chunk 0's slab, up front
        bf16x8 t[NPC];
        if (ACT == 1) gains(ld_bf16x8(g_addr(0)));
#pragma unroll
        for (int j = 0; j < NPC; ++j) t[j] = ld_bf16x8(x_addr(0, j));
#pragma unroll
        for (int j = 0; j < NPC; ++j) x_store(slab, j, t[j], gf, true);
    }
    bf16x8 rw[PD][RT], rxs[NPC], rg = zero_bf16x8();
    auto load_w = [&](int p, int step) {
        const size_t kb = (size_t)min(kb_begin + step, kb_end);
#pragma unroll
        for (int t = 0; t < RT; ++t) rw[p][t] = ld_bf16x8_stream(w[t] + kb * wstride);
    };
    // (SELF: in this order, which the loop's wait counts go by; left to the scheduler, gate/up of one row on 128 CUs takes 49.7 us
    // instead of 47.3)
    if (SELF) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < PD; ++p) {
        load_w(p, p);
        if (SELF) __builtin_amdgcn_sched_barrier(0);
    }
    if (SELF) {   // a few rows: the sums of squares are formed here, from the rows themselves, as dgemm_epilogue_kernel forms them
#pragma unroll
        for (int r = 0; r < RS_FEW_ROWS; ++r) {
            if (r >= M) break;
            float s[FEW_PARTS] = {};
#pragma unroll
            for (int i = 0; i < FEW_PARTS; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float f = 1024 * i + 4 * tid < K ? (float)self[r][i][e] : 0.f;
                    s[i] += f * f;
                }
            // wave_sum of all four, each with the other half's or quarter's: lanes 16 i .. 16 i + 15 end with part i
            const bool up = lane & 32, odd = lane & 16;
            const float s0 = (up ? s[2] : s[0]) + __shfl_xor(up ? s[0] : s[2], 32, 64), s1 = (up ? s[3] : s[1]) + __shfl_xor(up ? s[1] : s[3], 32, 64);
            float t = (odd ? s1 : s0) + __shfl_xor(odd ? s0 : s1, 16, 64);
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
            if ((lane & 15) == 0) self_ssq[r][lane >> 4][wave] = t;
        }
    }
    float sc[MT];
    if (FUSED && !SELF) {
#pragma unroll
        for (int tm = 0; tm < MT; ++tm) sc[tm] = rs[tm].scale(fz.ssq_part, fz.S_ssq, 32 * tm + c32, K, fz.eps);
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (SELF) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < FEW_PARTS; ++i) {
            const f32x4 s = self_ssq[min(c32, M - 1)][i];
            if (1024 * i < K) t += (s[0] + s[1]) + (s[2] + s[3]);
        }
        sc[0] = 1.0f / sqrtf(t / (float)K + fz.eps);
    }

    for (int c = 0; c < nchunks; ++c) {
        const bf16_t *cur = slab + (c & 1) * (CH * MT * 512) + lane * 8;
        bf16_t *nxt = slab + ((c + 1) & 1) * (CH * MT * 512);
        const bool more = c + 1 < nchunks;
        bf16x8 xf[2][MT];   // activation fragments, read one step ahead of their MFMAs
#pragma unroll
        for (int tm = 0; tm < MT; ++tm) xf[0][tm] = *(const bf16x8 *)&cur[tm * 512];
#pragma unroll
        for (int s = 0; s < CH; ++s) {
            const int p = s % PD;
            if (s + 1 < CH)
#pragma unroll
                for (int tm = 0; tm < MT; ++tm) xf[(s + 1) & 1][tm] = *(const bf16x8 *)&cur[((s + 1) * MT + tm) * 512];
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int tm = 0; tm < MT; ++tm) acc[t][tm] = mfma32(rw[p][t], xf[s & 1][tm], acc[t][tm]);
            // the pieces of the next slab that were fetched eight steps ago
            if (ACT == 1 && s == 8) gains(rg);
#pragma unroll
            for (int j = 0; j < NPC; ++j)
                if (j * 8 / NPC == s - 8) x_store(nxt, j, rxs[j], gf, more);
            load_w(p, c * CH + s + PD);
            if (ACT == 1 && s == 0) rg = ld_bf16x8(g_addr(c + 1));
#pragma unroll
            for (int j = 0; j < NPC; ++j)
                if (j * 8 / NPC == s) rxs[j] = ld_bf16x8(x_addr(c + 1, j));
            __builtin_amdgcn_sched_barrier(0);
        }
        // every wave has read slab c and written its pieces of slab c+1; the weight loads stay in flight
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
    if (FUSED) {
        const int Mt_out = packed_mt(M);
        auto emit = [&](const f32x16 &g, const f32x16 &u, int tm, int ftile) {
            const int m = 32 * tm + c32;
            if (m >= M) return;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int n = 32 * ftile + 8 * j + 4 * h;
                if (n >= a.N) continue;
                bf16x4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = (bf16_t)(silu_f(g[4 * j + i] * sc[tm]) * (u[4 * j + i] * sc[tm]));
                *(bf16x4 *)(fz.out + packed_offset(m, n, Mt_out) + (n & 7)) = v;
            }
        };
        if (PAIR) {
#pragma unroll
            for (int tm = 0; tm < MT; ++tm) emit(acc[0][tm], acc[RT - 1][tm], tm, 4 * (int)blockIdx.x + wave);
        } else {
            // gate and up of a feature tile sit in waves w and w + 2, which trade halves through LDS: w finishes the
            // first H row tiles, w + 2 the rest
            constexpr int H = (MT + 1) / 2;
            f32x4 *xch = (f32x4 *)slab;   // free since the last barrier: [wave][H][4][64 lanes]
            const bool up = wave >= 2;
#pragma unroll
            for (int q = 0; q < H; ++q)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    f32x4 v;
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = up ? acc[0][q][4 * j + i] : acc[0][min(H + q, MT - 1)][4 * j + i];
                    xch[((wave * H + q) * 4 + j) * 64 + lane] = v;
                }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < H; ++q) {
                f32x16 other;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const f32x4 v = xch[(((wave ^ 2) * H + q) * 4 + j) * 64 + lane];
#pragma unroll
                    for (int i = 0; i < 4; ++i) other[4 * j + i] = v[i];
                }
                const int ftile = 2 * (int)blockIdx.x + (wave & 1);
                if (!up) emit(acc[0][q], other, q, ftile);
                else if (H + q < MT) emit(other, acc[0][min(H + q, MT - 1)], min(H + q, MT - 1), ftile);
            }
        }
        return;
    }
    // each wave owns its rows: partial tile straight from the accumulators
#pragma unroll
    for (int tn = 0; tn < RT; ++tn)
#pragma unroll
        for (int tm = 0; tm < MT; ++tm) {
            const int m = 32 * tm + c32;
            if (m >= M) continue;
            float *dst = a.part + ((size_t)blockIdx.y * M + m) * Nv + (int)blockIdx.x * (128 * RT) + wave * (32 * RT) + 32 * tn;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f32x4 v = {acc[tn][tm][4 * j], acc[tn][tm][4 * j + 1], acc[tn][tm][4 * j + 2], acc[tn][tm][4 * j + 3]};
                *(f32x4 *)(dst + 8 * j + 4 * h) = v;
            }
        }
    if (ACT == 1 && blockIdx.x == 0) {
        // sums of squares of the slice: lanes with the same l%8 hold the same row, then the 4 waves in wave order
        float *red = (float *)slab;   // free since the last barrier
#pragma unroll
        for (int j = 0; j < NPC; ++j) {
            float v = ssq[j];
            v += __shfl_xor(v, 8, 64);
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            if (lane < 8) red[wave * (32 * MT) + 8 * j + lane] = v;
        }
        __syncthreads();
        if (tid < 32 * MT)
            a.ssq_part[blockIdx.y * RS_SSQ_ROWS + tid] = ((red[tid] + red[32 * MT + tid]) + red[64 * MT + tid]) + red[96 * MT + tid];
    }
}

// ---------------------------------------------------------------------------------------------
// The schedule of a projection: a function of (N, K, pair) alone.
// ---------------------------------------------------------------------------------------------
bool dgemm_applies(int N, int K) { return K >= 256 && K % 256 == 0 && N >= 128 && N % 4 == 0; }

DGemmPlan dgemm_plan(int N, int K, bool pair) {
    DGemmPlan p{};
    p.pair = pair;
    // a workgroup's 4 waves take two 32-row weight tiles each: 256 rows, or 128 gate rows and their up rows
    p.cols = pair ? (N + 127) / 128 : (N + 255) / 256;
    p.Nv = p.cols * 256;
    const int Kb = K / 16;
    // K slices: as many as keep the launch within about one workgroup per compute unit of a half-chip partition
    // (128) with at least 32 k-blocks (two chunks) per slice, in whole chunks.  Measured on the Llama-3-8B shapes: on
    // a partition the stream is bound by what one compute unit can pull, so one large workgroup per unit beats two
    // half-sized ones (the activation rows are staged once instead of twice); on the whole chip more, smaller
    // workgroups win a little -- this is the better compromise.
    // A gate/up pair is never cut: a slice of it would have to leave partial sums for a kernel of its own to finish,
    // and the pair is wide enough to fill the chip (two slices: 2 % slower on 128 CUs even before its epilogue moved
    // into the stream).
    const int cap = 128;
    int S = 1;
    for (int s = 2; s <= 64 && !pair; ++s)
        if (Kb % (s * DS_CH) == 0 && Kb / s >= 2 * DS_CH && p.cols * s <= cap) S = s;
    p.S = S;
    p.kb_per_wg = Kb / S;
    return p;
}

size_t dgemm_partial_elems(int M, int N, int K) {
    const DGemmPlan p = dgemm_plan(N, K, false);
    return (size_t)p.S * (size_t)M * (size_t)p.Nv;
}

// `narrow`: workgroups of 128 weight rows (one tile per wave) instead of 256, twice as many of them; for a gate/up
// pair, 64 features per workgroup (two gate tiles and their two up tiles, one per wave) instead of 128.
// The K slices and the order of every sum are those of the plan, so the
// results are the same bits; only the number of compute units that have a workgroup changes.  The caller picks the
// form per projection with dgemm_prefers_half_height: on the whole chip the plan's 96-128 workgroups leave too many
// units idle (Llama-3-8B decode step alone on 256 CUs 0.243 -> 0.2325 ms with half-height workgroups), on a 128-CU
// partition one large workgroup per unit is the faster shape (0.2914 against 0.2992 ms), and where the full-height
// count fills the units badly (128 workgroups on 96 units: two rounds, the second a third full) the half-height
// form's three shorter rounds win (decode step on 96 CUs 0.402 -> 0.393 ms, on 192 CUs 0.265 -> 0.261 ms).
//
// The rule: rounds of workgroups (one per unit) times what a workgroup moves.  A full-height workgroup streams its weights plus a
// quarter as many activation bytes (64 rows against 256), a half-height one half the weights and the same activations: 0.6
// of the bytes.  (0.56 at 32 rows and 0.67 at 128; with 0.6 throughout the rule agreed with the faster of the two within 3 %
// for the four projections of the 8B and 70B shapes at 1 to 128 rows on 64 to 256 CUs, but for QKV of the 8B shape at 65 to
// 96 rows on 64 CUs, 55 us where full height takes 49, and gate/up of the 70B shape at up to 16 rows on 96, 250 where half height
// takes 235.)
bool dgemm_prefers_half_height(const DGemmPlan &p, int cus) {
    if (cus <= 0) return false;
    const int wgs = p.cols * p.S;
    const double full = (double)((wgs + cus - 1) / cus), half = 0.6 * (double)((2 * wgs + cus - 1) / cus);
    return half < full;
}

constexpr int ds_lds(int mt) { return 2 * DS_CH * mt * 1024; }

template <int MT>
static void launch_dstream(hipStream_t st, const DGemmArgs &a, const DGemmPlan &p, const DFuseArgs &f, bool narrow) {
    const dim3 grid(narrow ? 2 * p.cols : p.cols, p.S), block(256);
    const bool rows = a.X_rows != nullptr;
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, ds_lds(MT), st, a, p.kb_per_wg, p.Nv, f); };
    if constexpr (MT == 1) {
        if (f.rows) {
            narrow ? go(dstream_kernel<0, 1, false, true, 1, true>) : go(dstream_kernel<0, 2, true, false, 1, true>);
            return;
        }
    }
    if (p.pair) narrow ? go(dstream_kernel<0, 1, false, true, MT>) : go(dstream_kernel<0, 2, true, false, MT>);
    else if (rows) narrow ? go(dstream_kernel<1, 1, false, false, MT>) : go(dstream_kernel<1, 2, false, false, MT>);
    else narrow ? go(dstream_kernel<0, 1, false, false, MT>) : go(dstream_kernel<0, 2, false, false, MT>);
}

void launch_dgemm_stream(hipStream_t st, const DGemmArgs &a, const DGemmPlan &p, const DFuseArgs &f, bool narrow) {
    switch ((a.M + 31) / 32) {
        case 1: launch_dstream<1>(st, a, p, f, narrow); break;
        case 2: launch_dstream<2>(st, a, p, f, narrow); break;
        case 3: launch_dstream<3>(st, a, p, f, narrow); break;
        default: launch_dstream<4>(st, a, p, f, narrow); break;
    }
}

// ---------------------------------------------------------------------------------------------
// Epilogues: the K slices are added in slice order; where the projection's input was an RMSNorm, the
// row's scale is formed here from the slices' sums of squares (in slice order) and applied first.
// ---------------------------------------------------------------------------------------------
// out = resid + sum, row-major; one thread per 4 columns, one workgroup per 1024 columns of a row.  With a gain (the
// next RMSNorm's) also out . gain, fragment-packed, and the sum of squares of the workgroup's part of the row.
template <int SB>
__global__ __launch_bounds__(256) void dgemm_epilogue_kernel(DEpiArgs a) {
    const int M = a.M, N = a.N;
    const int m = blockIdx.y, n = (blockIdx.x * 256 + threadIdx.x) * 4;
    float ss = 0.f;
    if (n < N) {
        const bf16x4 r = *(const bf16x4 *)(a.resid + (size_t)m * N + n);
        const bf16x4 g = *(const bf16x4 *)((a.gain ? a.gain : a.resid) + n);
        f32x4 acc[1];
        sum_slices<SB, 1>(a.part + (size_t)m * a.Nv + n, 0, (size_t)M * a.Nv, a.S, acc);
        bf16x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = (bf16_t)(acc[0][i] + (float)r[i]);
        *(bf16x4 *)(a.out + (size_t)m * N + n) = v;
        if (a.gain) {
            bf16x4 w;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float f = (float)v[i];
                ss += f * f;
                w[i] = (bf16_t)(f * (float)g[i]);
            }
            *(bf16x4 *)(a.out_gain + packed_offset(m, n, packed_mt(M)) + (n & 7)) = w;
        }
    }
    if (!a.gain) return;
    __shared__ float red[4];
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    if (threadIdx.x == 0) a.ssq_out[blockIdx.x * RS_SSQ_ROWS + m] = (red[0] + red[1]) + (red[2] + red[3]);
}

// The operand of a projection behind an RMSNorm, made in front of its stream: x . gain fragment-packed and the sums of
// squares of each row's parts (as dgemm_epilogue_kernel leaves them).
__global__ __launch_bounds__(256) void gain_pack_kernel(const bf16_t *__restrict__ x, const bf16_t *__restrict__ gain, bf16_t *__restrict__ out,
                                                        float *__restrict__ ssq_out, int M, int N) {
    const int m = blockIdx.y, n = (blockIdx.x * 256 + threadIdx.x) * 4;
    float ss = 0.f;
    if (n < N) {
        const bf16x4 v = *(const bf16x4 *)(x + (size_t)m * N + n), g = *(const bf16x4 *)(gain + n);
        bf16x4 w;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float f = (float)v[i];
            ss += f * f;
            w[i] = (bf16_t)(f * (float)g[i]);
        }
        *(bf16x4 *)(out + packed_offset(m, n, packed_mt(M)) + (n & 7)) = w;
    }
    __shared__ float red[4];
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    if (threadIdx.x == 0) ssq_out[blockIdx.x * RS_SSQ_ROWS + m] = (red[0] + red[1]) + (red[2] + red[3]);
}

void launch_gain_pack(hipStream_t st, const bf16_t *x, const bf16_t *gain, bf16_t *out, float *ssq_out, int M, int N) {
    hipLaunchKernelGGL(gain_pack_kernel, dim3((N + 1023) / 1024, M), dim3(256), 0, st, x, gain, out, ssq_out, M, N);
}

// Whether the stream forms x . gain itself.  That costs a workgroup 0.3 to 0.5 us per staged chunk and row tile (vector
// instructions in front of its matrix instructions); launch_gain_pack is a launch of 5 us.  QKV on 256 CUs, inline /
// packed first: 8B shape (4 chunks) at 64 rows 16.8 / 14.4 + 4.8 us, at 77 rows 20.1 / 15.6 + 5.0 (equal in the layer's
// time); 70B shape (16 chunks) at 101 rows 76 / 45 + 5 us.
bool dgemm_gains_inline(int M, const DGemmPlan &p) { return (p.kb_per_wg / DS_CH) * ((M + 31) / 32) <= DS_INLINE_PIECES; }

void launch_dgemm_epilogue(hipStream_t st, const DEpiArgs &a) {
    const dim3 grid((a.N + 1023) / 1024, a.M);
    if (a.S <= 4) hipLaunchKernelGGL(dgemm_epilogue_kernel<4>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(dgemm_epilogue_kernel<8>, grid, dim3(256), 0, st, a);
}

// QKV epilogue: sums the K slices, applies the first RMSNorm's row scale, rotates q and k at the row's position
// (rotate-half pairs (i, i + hd/2), angles from the host-built table), stores q | k | v as bf16 rows for the
// attention kernels, and writes k and v to the paged cache through the block table (rows [0, T) are prompt rows,
// the rest decode rows):
// K in the pool's fragment order (kpool_chunk_offset), V token-minor.  One thread owns 4 dims of a pair's
// lower half and the matching 4 of the upper half.  A position outside the rotary table or a block id
// outside the pool is never used as an index: the row's cache write is skipped (without a position q and k stay as they are) and
// the error word raised.
struct QkvPlace {   // of row m: what depends on its position alone, requested before the sums are waited for
    int pos, blk;
    bool pos_ok;
    f32x4 cs01, cs23;   // cos and sin of the angles of dims i0 .. i0 + 3
};
template <int HD>
__device__ __forceinline__ QkvPlace qkv_place(const QkvEpiArgs &a, int m, int head, int i0) {
    QkvPlace p;
    int max_blk;
    const int32_t *tab_row;
    if (m < a.T) {
        int req = 0;
        while (req + 1 < a.seq.n_req && m >= a.seq.cu[req + 1]) ++req;
        p.pos = a.seq.start[req] + m - a.seq.cu[req];
        max_blk = a.max_blk_p;
        tab_row = a.ptables + (size_t)req * max_blk;
    } else {
        p.pos = a.ctx_lens[m - a.T];
        max_blk = a.max_blk;
        tab_row = a.tables + (size_t)(m - a.T) * max_blk;
    }
    p.pos_ok = p.pos >= 0 && p.pos < a.max_pos;
    const int bi = p.pos_ok ? p.pos / RS_BLOCK_TOKENS : 0;
    p.blk = -1;
    if (head >= a.Hq && bi < max_blk) p.blk = tab_row[bi];
    const f32x4 *tab = (const f32x4 *)(a.table + (size_t)(p.pos_ok ? p.pos : 0) * (HD / 2) + i0);
    p.cs01 = tab[0];
    p.cs23 = tab[1];
    return p;
}
// lo, hi: dims i0 .. i0 + 3 of the head's halves.  first: one thread of the row's; of_head: one thread of the head's.
template <int HD>
__device__ __forceinline__ void qkv_finish(const QkvEpiArgs &a, const QkvPlace &p, int m, int head, int i0, const f32x4 &lo, const f32x4 &hi, bool first,
                                           bool of_head) {
    constexpr int half = HD / 2;
    const int n_heads = a.Hq + 2 * a.Hkv;
    if (!p.pos_ok && first) atomicOr(a.err_flag, 1);
    bf16x4 olo, ohi;
    if (head < a.Hq + a.Hkv && p.pos_ok) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f32x4 &t = i < 2 ? p.cs01 : p.cs23;
            const float cc = t[2 * (i & 1)], ss = t[2 * (i & 1) + 1];
            olo[i] = (bf16_t)(lo[i] * cc - hi[i] * ss);
            ohi[i] = (bf16_t)(hi[i] * cc + lo[i] * ss);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            olo[i] = (bf16_t)lo[i];
            ohi[i] = (bf16_t)hi[i];
        }
    }
    bf16_t *row = a.qkv + (size_t)m * (n_heads * HD) + head * HD;
    *(bf16x4 *)(row + i0) = olo;
    *(bf16x4 *)(row + half + i0) = ohi;
    if (head < a.Hq || !p.pos_ok) return;
    if ((unsigned)p.blk >= (unsigned)a.n_blocks) {
        if (of_head && head == a.Hq) atomicOr(a.err_flag, 2);
        return;
    }
    const int slot = p.pos % RS_BLOCK_TOKENS;
    if (head < a.Hq + a.Hkv) {
        bf16_t *dst = a.k_pool + ((size_t)p.blk * a.Hkv + (head - a.Hq)) * RS_BLOCK_TOKENS * HD;
        *(bf16x4 *)(dst + kpool_chunk_offset(slot, i0 & ~7) + (i0 & 7)) = olo;
        *(bf16x4 *)(dst + kpool_chunk_offset(slot, (half + i0) & ~7) + (i0 & 7)) = ohi;
    } else {
        bf16_t *dst = a.v_pool + ((size_t)p.blk * a.Hkv + (head - a.Hq - a.Hkv)) * HD * RS_BLOCK_TOKENS + slot;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            dst[(i0 + i) * RS_BLOCK_TOKENS] = olo[i];
            dst[(half + i0 + i) * RS_BLOCK_TOKENS] = ohi[i];
        }
    }
}

template <int HD>
__global__ __launch_bounds__(256) void qkv_rope_epilogue_kernel(QkvEpiArgs a) {
    constexpr int TPH = HD / 8;           // threads per head
    constexpr int HPW = 256 / TPH;        // heads per workgroup
    const int m = row_of(blockIdx.x, gridDim.x), tid = threadIdx.x;
    const int head = blockIdx.y * HPW + tid / TPH;
    if (m >= a.M || head >= a.Hq + 2 * a.Hkv) return;
    const int i0 = (tid % TPH) * 4;
    const QkvPlace place = qkv_place<HD>(a, m, head, i0);
    RowSsq rs;
    if (a.S_ssq) rs.request(a.ssq_part, a.S_ssq, m);
    f32x4 sum[2];
    sum_slices<4, 2>(a.part + (size_t)m * a.Nv + head * HD + i0, HD / 2, (size_t)a.M * a.Nv, a.S, sum);
    const float sc = a.S_ssq ? rs.scale(a.ssq_part, a.S_ssq, m, a.d, a.eps) : 1.0f;
    qkv_finish<HD>(a, place, m, head, i0, sum[0] * sc, sum[1] * sc, tid == 0 && blockIdx.y == 0, tid % TPH == 0);
}

// ---------------------------------------------------------------------------------------------
// A pass of at most RS_FEW_ROWS rows: the projections that a stream cuts in K for enough workgroups, whole.  A workgroup's two to seven waves
// take the plan's K slices between them, of the same R x 16 weight rows (QKV: R x 16 dims and those that they are rotated with), the slices' sums
// are added in their order through LDS, and the workgroup finishes its columns: no partial sums in memory and no epilogue kernel that reads
// them, and the bits are the stream's.  What bounds a layer of one row, beside its weights, is some 4 us of every kernel in it (launch, first
// bytes, last ones), and so it is six of them instead of nine.  The activation fragments come with the weights from memory (the L2); of QKV
// every wave forms x . gain of its slices' columns in LDS, and their sums of squares.  Four layers of the 8B widths on 256 CUs behind 900
// cached tokens, streams / this: 1 row 389 / 355 us, 4 rows 395 / 365.  More rows are slower on partitions (8 rows on 128 CUs, a layer
// 114.5 / 116.6): the lines that the rows' fragments touch grow with the rows.  More bytes in flight are slower (eight waves of eight
// steps each 1.066 of the streams' rate where four of four have 1.084).
// ---------------------------------------------------------------------------------------------
#define FEW_PD 4   // 16x32 weight fragments in flight per wave and tile
#define FEW_LEAST 2     // fewest and
#define FEW_SLICES 16   // most slices that a workgroup's waves share
#define FEW_WAVES 7     // most waves
#define FEW_PAIRS 2     // QKV: most pairs of activation chunks of a wave, of rows of RS_FEW_COLS columns
// Slices of a wave: the fewest waves, from four on, among those that leave the last one the least idle.
static int few_slices_of_wave(int S) {
    int best = std::min(S, 4);
    for (int w = best; w <= FEW_WAVES; ++w)
        if ((S + w - 1) / w * w < (S + best - 1) / best * best) best = w;
    return (S + best - 1) / best;
}
static_assert(DS_CH % (2 * FEW_PD) == 0, "a slice is whole rounds of the ring");

// HD: head_dim of the QKV projection, 0: a residual projection.  R: 16-row tiles of a workgroup (QKV: of either half of a head).
template <int HD, int R>
__global__ __launch_bounds__(64 * FEW_WAVES) void few_kernel(FewArgs a, QkvEpiArgs q) {
    constexpr bool QKV = HD > 0;
    constexpr int NT = QKV ? 2 * R : R, PD = FEW_PD;
    extern __shared__ __attribute__((aligned(16))) f32x4 few_lds[];
    __shared__ float ssq[RS_FEW_ROWS][FEW_SLICES];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, c16 = lane & 15, g = lane >> 4;
    const int M = a.M, N = a.N, K = a.K, S = a.S, m = min(c16, M - 1);
    f32x4 *red = few_lds;                                   // [S][NT][4 column groups][RS_FEW_ROWS]
    bf16_t *xs = (bf16_t *)(red + S * NT * 4 * RS_FEW_ROWS);   // QKV: [M][K + 8], every wave the columns of its slices
    const int sl0 = wave * a.wave_slices, sl1 = min(sl0 + a.wave_slices, S);   // this wave's slices
    const int ns = K / (32 * S), n = (sl1 - sl0) * ns, k0 = sl0 * ns;          // steps of 32 of one and of all, and the first
    const int Nt = ((N + 63) / 64) * 2;
    const size_t wstride = (size_t)Nt * 512, xstride = (size_t)packed_mt(M) * 512;   // per k block
    // columns n0 (and n0 + HD / 2) .. + 16 R - 1; wave j finishes the j-th 16 of them
    constexpr int GPH = QKV ? HD / (32 * R) : 1;   // workgroups per head
    const int head = blockIdx.x / GPH, i0 = 16 * (R * (blockIdx.x % GPH) + wave) + 4 * g;
    const int n0 = QKV ? head * HD + 16 * R * (blockIdx.x % GPH) : 16 * R * (int)blockIdx.x;
    const bf16_t *w[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int r = n0 + 16 * (t % R) + (t / R) * (HD / 2);
        w[t] = a.Wp + (size_t)(2 * k0 + (g >> 1)) * wstride + (size_t)(r >> 5) * 512 + ((g & 1) * 32 + (r & 16) + c16) * 8;
    }
    const bf16_t *x = QKV ? nullptr : a.A + (size_t)(2 * k0 + (g >> 1)) * xstride + ((g & 1) * 32 + m) * 8;
    bf16x8 rw[PD][NT], rx[PD];
    auto load = [&](int p, int step) {
        const size_t s = (size_t)min(step, n - 1);   // (past the end: the last one again)
#pragma unroll
        for (int t = 0; t < NT; ++t) rw[p][t] = ld_bf16x8_stream(w[t] + s * 2 * wstride);
        if (!QKV) rx[p] = ld_bf16x8(x + s * 2 * xstride);
    };
    // QKV: a wave brings the columns of its own slices, two chunks of 16 k-blocks at a time (a half-wave each), requested in front of the
    // weights and waited for alone
    const int nch = K / (16 * DS_CH * S), pairs = (nch + 1) >> 1, k8 = lane & 31, half = lane >> 5;   // chunks of a slice, and pairs of them
    bf16x8 xv[FEW_PAIRS][RS_FEW_ROWS], gv[FEW_PAIRS];
    auto column = [&](int i) { return ((sl0 + i / pairs) * nch + min(2 * (i % pairs) + half, nch - 1)) * 32 + k8; };   // of 8 elements
    const int items = (sl1 - sl0) * pairs;
    // a residual projection: what the finished columns are added to and multiplied by
    const int col = min(n0 + 16 * wave, N - 16) + 4 * g;
    bf16x4 resid{}, gain{};
    if (!QKV) {
        resid = *(const bf16x4 *)(a.resid + (size_t)m * N + col);
        gain = *(const bf16x4 *)((a.gain ? a.gain : a.resid) + col);
    }
    if (QKV)
#pragma unroll
        for (int i = 0; i < FEW_PAIRS; ++i) {
            const int c = column(min(i, items - 1));
            gv[i] = ld_bf16x8(a.gain + c * 8);
#pragma unroll
            for (int r = 0; r < RS_FEW_ROWS; ++r) xv[i][r] = ld_bf16x8(a.X_rows + (size_t)min(r, M - 1) * K + c * 8);
        }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < PD; ++p) load(p, p);
    __builtin_amdgcn_sched_barrier(0);
    QkvPlace place{};
    const int ld = K + 8;
    if (QKV) {
        // x . gain to LDS, and a slice's sums of squares in the stream's order: over the chunks for each 16-byte column of a chunk, then
        // eight columns as a tree, then the four eights one after the other
        float t[RS_FEW_ROWS];
#pragma unroll
        for (int i = 0; i < FEW_PAIRS; ++i) {
            if (i >= items) break;
            const int j = i % pairs, c = column(i);
            const bool two = 2 * j + 1 < nch;   // else the upper half-wave has the lower one's chunk
#pragma unroll
            for (int r = 0; r < RS_FEW_ROWS; ++r) {
                if (r >= M) break;
                bf16x8 h;
                float s = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    s += (float)xv[i][r][e] * (float)xv[i][r][e];
                    h[e] = (bf16_t)((float)xv[i][r][e] * (float)gv[i][e]);
                }
                *(bf16x8 *)&xs[r * ld + c * 8] = h;
                const float other = __shfl_xor(s, 32, 64);
                t[r] = (j ? t[r] : 0.f) + (half ? other : s);
                if (two) t[r] += half ? s : other;
            }
            if (j + 1 < pairs) continue;
#pragma unroll
            for (int r = 0; r < RS_FEW_ROWS; ++r) {
                if (r >= M) break;
#pragma unroll
                for (int o = 1; o < 8; o *= 2) t[r] += __shfl_xor(t[r], o, 64);
                const float q = ((__shfl(t[r], 0, 64) + __shfl(t[r], 8, 64)) + __shfl(t[r], 16, 64)) + __shfl(t[r], 24, 64);
                if (lane == 0) ssq[r][sl0 + i / pairs] = q;
            }
        }
        if (wave < R) place = qkv_place<QKV ? HD : 64>(q, m, head, i0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the rows are read by other lanes of the wave; the weight loads stay in flight
    }
    const bf16_t *xr = xs + m * ld + k0 * 32 + 8 * g;
    for (int sl = sl0; sl < sl1; ++sl) {
        f32x4 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int s0 = (sl - sl0) * ns; s0 < (sl - sl0 + 1) * ns; s0 += PD) {
#pragma unroll
            for (int p = 0; p < PD; ++p) {
                const bf16x8 xf = QKV ? *(const bf16x8 *)&xr[(s0 + p) * 32] : rx[p];
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(rw[p][t], xf, acc[t], 0, 0, 0);
                load(p, s0 + p + PD);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // lane: columns n0 + 4g .. + 3 of row c16
        if (c16 < RS_FEW_ROWS)
#pragma unroll
            for (int t = 0; t < NT; ++t) red[((sl * NT + t) * 4 + g) * RS_FEW_ROWS + c16] = acc[t];
    }
    __syncthreads();
    if (wave >= R || c16 >= M) return;
    f32x4 sum[NT / R];
#pragma unroll
    for (int t = 0; t < NT / R; ++t) sum[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma clang loop unroll(disable)
    for (int s0 = 0; s0 < S; s0 += 8) {
        f32x4 v[8][NT / R];
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int t = 0; t < NT / R; ++t) v[s][t] = red[((min(s0 + s, S - 1) * NT + t * R + wave) * 4 + g) * RS_FEW_ROWS + c16];
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int t = 0; t < NT / R; ++t)
                if (s0 + s < S) sum[t] += v[s][t];
    }
    if constexpr (QKV) {
        float t = 0.f;
        for (int s = 0; s < S; ++s) t += ssq[m][s];
        const float sc = 1.0f / sqrtf(t / (float)K + a.eps);
        qkv_finish<HD>(q, place, m, head, i0, sum[0] * sc, sum[1] * sc, blockIdx.x == 0 && wave == 0 && g == 0, i0 == 0);
    } else {
        bf16x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = (bf16_t)(sum[0][i] + (float)resid[i]);
        *(bf16x4 *)(a.out + (size_t)m * N + col) = v;
        if (a.gain) {
            bf16x4 h;
#pragma unroll
            for (int i = 0; i < 4; ++i) h[i] = (bf16_t)((float)v[i] * (float)gain[i]);
            *(bf16x4 *)(a.out_gain + packed_offset(m, col, packed_mt(M)) + (col & 7)) = h;
        }
    }
}

// Tiles of a workgroup: rounds of workgroups (one per CU) times what a workgroup moves, its tiles of weights and `act` of one for the rows.
// The same sums whatever the number.  One row of the 8B widths, streams / one tile throughout / this in all three projections, four layers: on 128 CUs 446 / 469 / 438 us,
// on 64 698 / 767 / 680 (four rows), on 192 437 / 459 / 428.
static int few_rounds(int tiles, int R, int cus) { return (tiles / R + cus - 1) / cus; }
static int few_tiles(int tiles, int cus, double act, int most) {
    int best = 1;
    double least = 1e30;
    for (int R = 1; R <= most; R *= 2) {
        const double cost = few_rounds(tiles, R, cus) * (R + act);
        if (cost < least) { least = cost; best = R; }
    }
    return best;
}
// (A tile is finished by a wave of its own.)
static int few_residual_tiles(int N, int S, int cus) { return few_tiles(N / 16, cus, 0.6, S < 4 ? 1 : N % 64 ? 2 : 4); }
static int few_qkv_tiles(int N, int S, int hd, int cus) { return few_tiles(N / 32, cus, 0.1, S < 4 ? 1 : hd == 64 ? 2 : 4); }

// Whether a projection of a few rows is finished in one kernel or streamed, with the same bits.  It saves the partial sums and a kernel of some
// 4 us; what can cost more is a CU's load, in 16-row tiles of K: the most of them that any CU has, here and in the stream's chosen form.
// Measured for each projection by itself, one row, four layers, against the streams on 256 / 224 / 192 / 160 / 128 / 96 / 64 / 32 CUs:
//   8B widths, QKV -12 -11 -11 -10 -11 -11 0 -7 us, output -13 -4 -1 -2 -3 0 -8 -13, down (K = 14336) -10 +3 +4 +5 +5 +27 -3 -4
//   3072 columns, QKV -10 -14 -15 -15 -3 -14 +2 -1, output -6 -5 -6 +4 -6 -5 -2 -10, down (K = 8192) -1 -1 -2 +1 0 +1 +16 +13
//   2560 columns, QKV -8 -8 -8 -8 -16 -6 -17 -18, output -8 -8 -8 -8 +1 -10 +6 -1, down (K = 10240) +4 +4 -8 -8 +19 -3 +36 +15
// (and five other widths, four rows).  So a residual projection where a CU's load does not grow; QKV, whose rows cost a workgroup less than
// the stream's, where it grows by no more than what a CU moves in 2 us (57 KB each).  Long K with several tiles a workgroup loses even at
// equal loads: the rows' fragments come with every step.  Two or three slices are two or three waves, too few to load a CU at its rate:
// where a workgroup a tile is one round (down projection of 3584 columns, K = 18944: -35 us on 256 CUs; on 96, three rounds, +12).
static double stream_load(const DGemmPlan &p, int cus) {
    const int wgs = p.cols * p.S;
    return dgemm_prefers_half_height(p, cus) ? (2 * wgs + cus - 1) / cus * (8.0 / p.S) : (wgs + cus - 1) / cus * (16.0 / p.S);
}
static bool few_applies(int M, int N, const DGemmPlan &p) { return M <= RS_FEW_ROWS && N % 32 == 0 && p.S >= FEW_LEAST && p.S <= FEW_SLICES; }
bool few_takes_residual(int M, int N, int K, int cus) {
    const DGemmPlan p = dgemm_plan(N, K, false);
    if (N > RS_FEW_COLS || !dgemm_applies(N, K) || !few_applies(M, N, p)) return false;
    const int R = few_residual_tiles(N, p.S, cus);
    return few_rounds(N / 16, R, cus) * R <= stream_load(p, cus) && (R == 1 || K <= 8192) && (p.S >= 4 || N / 16 <= cus);
}
bool few_takes_qkv(int M, int N, int K, int hd, int cus) {
    const DGemmPlan p = dgemm_plan(N, K, false);
    if (K > RS_FEW_COLS || !dgemm_gains_inline(M, p) || !few_applies(M, N, p)) return false;
    if (few_slices_of_wave(p.S) * ((p.kb_per_wg / DS_CH + 1) / 2) > FEW_PAIRS) return false;
    const int R = few_qkv_tiles(N, p.S, hd, cus);
    return (p.S >= 4 || N / 32 <= cus) && (few_rounds(N / 32, R, cus) * 2 * R - stream_load(p, cus)) * (32.0 * K) <= 2 * 57e3;
}
// (At most 50 KB, which needs no leave: rows of RS_FEW_COLS columns, 32 KB, have up to eight slices, 16 KB of sums.)
static size_t few_lds_bytes(int S, int tiles) { return (size_t)S * tiles * 4 * RS_FEW_ROWS * sizeof(f32x4); }
static int few_threads(FewArgs &a) {
    a.wave_slices = few_slices_of_wave(a.S);
    return 64 * ((a.S + a.wave_slices - 1) / a.wave_slices);
}
void launch_few_residual(hipStream_t st, FewArgs a, int cus) {
    const int R = few_residual_tiles(a.N, a.S, cus), threads = few_threads(a);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(a.N / (16 * R)), dim3(threads), few_lds_bytes(a.S, R), st, a, QkvEpiArgs{}); };
    R == 4 ? go(few_kernel<0, 4>) : R == 2 ? go(few_kernel<0, 2>) : go(few_kernel<0, 1>);
}
void launch_few_qkv(hipStream_t st, FewArgs a, const QkvEpiArgs &q, int cus) {
    const int R = few_qkv_tiles(a.N, a.S, q.hd, cus);
    const dim3 grid(a.N / (32 * R)), block(few_threads(a));
    const size_t lds = few_lds_bytes(a.S, 2 * R) + (size_t)a.M * (a.K + 8) * sizeof(bf16_t);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, lds, st, a, q); };
    if (q.hd == 128) R == 4 ? go(few_kernel<128, 4>) : R == 2 ? go(few_kernel<128, 2>) : go(few_kernel<128, 1>);
    else R == 2 ? go(few_kernel<64, 2>) : go(few_kernel<64, 1>);
}

void launch_qkv_rope_epilogue(hipStream_t st, const QkvEpiArgs &a) {
    const int n_heads = a.Hq + 2 * a.Hkv;
    if (a.hd == 128) {
        hipLaunchKernelGGL(qkv_rope_epilogue_kernel<128>, dim3(row_grid(a.M), (n_heads + 15) / 16), dim3(256), 0, st, a);
    } else {
        hipLaunchKernelGGL(qkv_rope_epilogue_kernel<64>, dim3(row_grid(a.M), (n_heads + 31) / 32), dim3(256), 0, st, a);
    }
}

// The output projection of a pass that multiplies in K slices, finished: residual, and the RMSNorm in front of the
// feed-forward block.  A thread owns 8 columns of every 2048; NG = ceil(N / 2048).
// In place of an epilogue and a norm kernel (576 rows of 4096, 2 slices: 7.0 + 7.6 us, 9.3 now).
template <int NG>
__global__ __launch_bounds__(256) void residual_norm_kernel(ResidualNormArgs a) {
    const int m = row_of(blockIdx.x, gridDim.x), tid = threadIdx.x;
    if (m >= a.M) return;
    bf16x8 r[NG], g[NG], v[NG];
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        const int n = min((q * 256 + tid) * 8, a.N - 8);
        r[q] = ld_bf16x8(a.resid + (size_t)m * a.N + n);
        g[q] = ld_bf16x8(a.gain + n);
    }
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        const int n = (q * 256 + tid) * 8;
        if (n >= a.N) continue;
        f32x4 sum[2];
        sum_slices<4, 2>(a.part + (size_t)m * a.N + n, 4, (size_t)a.M * a.N, a.S, sum);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            v[q][i] = (bf16_t)(sum[i >> 2][i & 3] + (float)r[q][i]);
            const float f = (float)v[q][i];
            ss += f * f;
        }
        st_bf16x8(a.x1 + (size_t)m * a.N + n, v[q]);
    }
    __shared__ float red[4];
    ss = wave_sum(ss);
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    const float inv = 1.0f / sqrtf(((red[0] + red[1]) + (red[2] + red[3])) / (float)a.N + a.eps);
    const int Mt = packed_mt(a.M);
#pragma unroll
    for (int q = 0; q < NG; ++q) {
        const int n = (q * 256 + tid) * 8;
        if (n >= a.N) continue;
        bf16x8 o;
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = (bf16_t)((float)v[q][i] * inv * (float)g[q][i]);
        st_bf16x8(a.h + packed_offset(m, n, Mt), o);
    }
}

bool residual_norm_applies(int N) { return N % 8 == 0 && N >= 8 && N <= 8192; }
void launch_residual_norm(hipStream_t st, const ResidualNormArgs &a) {
    const dim3 grid(row_grid(a.M));
    if (a.N <= 2048) hipLaunchKernelGGL(residual_norm_kernel<1>, grid, dim3(256), 0, st, a);
    else if (a.N <= 4096) hipLaunchKernelGGL(residual_norm_kernel<2>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(residual_norm_kernel<4>, grid, dim3(256), 0, st, a);
}

template <int MT>
static void dstream_init() {
    auto set = [](const void *f) { (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, ds_lds(MT)); };
    set((const void *)dstream_kernel<0, 1, false, true, MT>);
    set((const void *)dstream_kernel<0, 2, true, false, MT>);
    set((const void *)dstream_kernel<1, 1, false, false, MT>);
    set((const void *)dstream_kernel<1, 2, false, false, MT>);
    set((const void *)dstream_kernel<0, 1, false, false, MT>);
    set((const void *)dstream_kernel<0, 2, false, false, MT>);
}
void decode_gemm_kernels_init() {
    auto set = [](const void *f, int lds) { (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds); };
    set((const void *)dstream_kernel<0, 1, false, true, 1, true>, ds_lds(1));
    set((const void *)dstream_kernel<0, 2, true, false, 1, true>, ds_lds(1));
    dstream_init<1>();
    dstream_init<2>();
    dstream_init<3>();
    dstream_init<4>();
}
