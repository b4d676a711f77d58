// Attention kernels over the paged KV cache (gfx950, bf16 MFMA, fp32 softmax).
//
// Pool layouts (one layer):  K [n_blocks][Hkv][hd/32][4][16][8] (see kpool_chunk_offset)
// V [n_blocks][Hkv][hd][16], so one (block, kv head) is a contiguous 16*hd*2-byte run in each
// pool, a K fragment of the MFMA "row x k" operand is one contiguous 1 KB, and V, being token-
// minor, feeds the operand whose contraction index is the token without any transpose.
//
// Both kernels evaluate S^T = K Q^T and O^T = V^T P^T, so that a lane owns one query column:
// the running maximum and sum of the online softmax are per-lane scalars.
#include <algorithm>
#include <type_traits>

#include "kernels.h"

#define NEG_INF (-__builtin_huge_valf())
#define PREFILL_TAB_LDS 2048   // block ids of a prompt kept in LDS by the prefill kernel (32K tokens)

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// =============================================================================================
// Decode: one query token per request, keys gathered through the block table.
// Workgroup = (512-token chunk, kv head, request); its 4 waves take 128 tokens (8 blocks) each,
// two blocks per iteration.  The G = Hq/Hkv query heads that share the kv head are the (zero
// padded) 16 columns of the MFMA tiles, so every K/V byte is fetched once per kv head, straight
// from the pools into MFMA fragments with 16-byte loads (no LDS staging).
// The chunking depends on the context length only, never on the launch's CU share.
//
// Measured alternatives that were no better (Llama-3-8B shape, batch 64, contexts U[512,4096]; whole chip /
// 128-CU partition / partition beside a prefill pass; this kernel: 110 / 144 / 172 us):
//   * a persistent launch whose waves are independent workers on 128-token items, the next item's block ids
//     and first K/V loads in flight while an item is computed, items dealt round-robin: 126 / 156 / 171 us
//     (no round trip is exposed any more, yet nothing is gained: the kernel is not bound by the start-up of
//     its workgroups); the same with a device-side item counter: 200 us on any partition (12 500
//     single-address atomics serialise at about 16 ns each);
//   * the kv heads of one (request, chunk) on ONE XCD instead of eight: 7-10 % slower everywhere.
// What the measurements fit: a compute unit sustains a bounded number of outstanding lines, so its rate is
// that bound over the memory latency of the access pattern -- 47 GB/s for a linear stream, 34 GB/s for
// these 4 KB pieces of shuffled 32 KB blocks (38 GB/s with consecutive block ids), on a 128-CU partition.
//
// Row permutation: the two 16x16 score tiles of an iteration do not hold "block 0" and "block 1"
// but, with h = lane>>4, tile A row 4h+i <- token 8(h&1)+i of block h>>1 and tile B row 4h+i <-
// token 8(h&1)+4+i of block h>>1.  A lane's 4+4 score registers are then 8 consecutive tokens of
// one block, exactly the contraction slice k' = 8h..8h+7 that lane supplies to the 16x16x32 P V
// product, and the matching V fragment V[block h>>1][d][8(h&1)..+8] is one 16-byte load.
// =============================================================================================
static __host__ __device__ inline int decode_attn_lds_floats(int hd, int G) { return 4 * hd * G + 8 * G; }   // <= 33 KB at G = 16

// Column col of row b of the output, the output projection's operand
__device__ __forceinline__ bf16_t *decode_out(const DecodeAttnArgs &a, int b, int col) {
    return a.out + packed_offset(a.out_row0 + b, col, a.out_Mt ? a.out_Mt : packed_mt(a.B)) + (col & 7);
}

// One (kv head, request, chunk), by 256 threads; smem_dec: [4][HD][G] partial outputs, then [4][G] max, [4][G] sum
template <int HD>
__device__ __forceinline__ void decode_attn_chunk(const DecodeAttnArgs &a, const int hk, const int b, const int chunk, const int tid, float *smem_dec) {
    constexpr int KS = HD / 32;  // 16x16x32 steps over head_dim for S^T
    constexpr int DT = HD / 16;  // 16-row tiles of O^T
    const int wave = tid >> 6, lane = tid & 63;
    const int c16 = lane & 15, h = lane >> 4;
    const int G = a.Hq / a.Hkv;
    float *s_o = smem_dec;
    float *s_m = smem_dec + 4 * HD * G;
    float *s_l = s_m + 4 * G;

    int n_keys = a.ctx_lens[b] + 1;
    if (n_keys < 1 || n_keys > a.max_ctx) {
        if (tid == 0 && chunk == 0 && hk == 0) atomicOr(a.err_flag, 8);
        if (n_keys < 1) {
            if (a.n_chunks == 1)
                for (int col = hk * G * HD + tid; col < (hk + 1) * G * HD; col += 256) *decode_out(a, b, col) = (bf16_t)0.f;
            return;
        }
        n_keys = a.max_ctx;
    }
    if (chunk * RS_DECODE_CHUNK >= n_keys) return;

    constexpr int WT = RS_DECODE_CHUNK / 4;   // tokens per wave
    const int t0 = chunk * RS_DECODE_CHUNK + wave * WT;
    const int t1 = min(t0 + WT, n_keys);
    // the wave's (up to) WT/16 block ids, fetched once: lane i holds the id of block i of the range
    int my_blk = -1;
    {
        const int nb = t1 > t0 ? (t1 - t0 + 15) >> 4 : 0;
        if (lane < nb) {
            my_blk = a.tables[(size_t)b * a.max_blk + (t0 >> 4) + lane];
            if ((unsigned)my_blk >= (unsigned)a.n_blocks) {
                atomicOr(a.err_flag, 2);
                my_blk = -1;
            }
        }
    }

    bf16x8 qf[KS];
    {
        const bf16_t *qp = a.q + (size_t)b * a.q_stride + (size_t)(hk * G + c16) * HD;
#pragma unroll
        for (int s = 0; s < KS; ++s) qf[s] = (c16 < G) ? ld_bf16x8(qp + 32 * s + 8 * h) : zero_bf16x8();
    }

    float m_run = NEG_INF, l_run = 0.f;
    f32x4 o[DT];
#pragma unroll
    for (int i = 0; i < DT; ++i) o[i] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // K operand: MFMA row c16 = 4 hr + ir comes from block (hr>>1), token 8(hr&1)+ir (+4 for tile
    // B): in the pool's permuted row order these are rows c16&7 (tile A) and 8 + (c16&7) (tile B)
    const bool k_second = (c16 >> 3) != 0;   // this lane's K rows come from the iteration's second block
    const bool v_second = (h >> 1) != 0;     // this lane's V slice comes from the second block
    const size_t k_lane = (size_t)(h * 16 + (c16 & 7)) * 8;
    const size_t v_lane = (size_t)c16 * 16 + 8 * (h & 1);
    const size_t blk_stride = (size_t)a.Hkv * 16 * HD;
    const bf16_t *k_head = a.k_pool + (size_t)hk * 16 * HD;
    const bf16_t *v_head = a.v_pool + (size_t)hk * 16 * HD;
    const float sc = a.scale_log2;

    // Two register buffers of one iteration's K and V fragments (32 tokens, 16 KB per wave): the loads
    // of iteration it+1 are issued before iteration it is computed, so the wave always has bytes in
    // flight.  The number of iterations is wave-uniform; each count gets its own straight-line copy
    // of the schedule, which keeps the compiler's wait counts exact (a load issued under a branch
    // would force a wait for everything at the join).
    bf16x8 kA[2][KS], kB[2][KS], vf[2][DT];
    auto issue = [&](int it, int buf) {
        // the iteration's two block ids as wave-uniform scalars; blocks that are missing (past the
        // context, or rejected) read block 0: valid memory whose contents are masked out in compute()
        const int b0 = __builtin_amdgcn_readlane(my_blk, 2 * it);
        const int b1 = __builtin_amdgcn_readlane(my_blk, 2 * it + 1);
        const size_t o0 = (size_t)max(b0, 0) * blk_stride, o1 = (size_t)max(b1, 0) * blk_stride;
        const bf16_t *kp = k_head + (k_second ? o1 : o0) + k_lane;
        const bf16_t *vp = v_head + (v_second ? o1 : o0) + v_lane;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            kA[buf][s] = ld_bf16x8_stream(kp + 512 * s);
            kB[buf][s] = ld_bf16x8_stream(kp + 512 * s + 64);
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) vf[buf][dt] = ld_bf16x8_stream(vp + dt * 256);
    };
    auto compute = [&](int it, int buf) {
        const int base = t0 + 32 * it;
        const int b0 = __builtin_amdgcn_readlane(my_blk, 2 * it);
        const int b1 = __builtin_amdgcn_readlane(my_blk, 2 * it + 1);
        const bool full = base + 32 <= n_keys && b0 >= 0 && b1 >= 0;   // uniform: every token valid
        f32x4 sA = {0.f, 0.f, 0.f, 0.f}, sB = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            sA = mfma16(kA[buf][s], qf[s], sA);
            sB = mfma16(kB[buf][s], qf[s], sB);
        }
        // this lane's 8 scores are tokens tok0 .. tok0+7 (A: +0..3, B: +4..7) of its V block
        if (!full) {
            const int tok0 = base + 16 * (h >> 1) + 8 * (h & 1);
            const int nv = ((v_second ? b1 : b0) >= 0) ? min(max(n_keys - tok0, 0), 8) : 0;   // valid tokens
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (i >= nv) sA[i] = NEG_INF;
                if (4 + i >= nv) sB[i] = NEG_INF;
            }
            // zero V of invalid tokens so that 0 * garbage cannot produce NaN: dword j holds tokens 2j, 2j+1
            uint32_t msk[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) msk[j] = nv >= 2 * j + 2 ? 0xffffffffu : (nv == 2 * j + 1 ? 0x0000ffffu : 0u);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
                u32x4v raw = __builtin_bit_cast(u32x4v, vf[buf][dt]);
#pragma unroll
                for (int j = 0; j < 4; ++j) raw[j] &= msk[j];
                vf[buf][dt] = __builtin_bit_cast(bf16x8, raw);
            }
        }
        float m_tile = fmaxf(fmaxf(fmaxf(sA[0], sA[1]), fmaxf(sA[2], sA[3])), fmaxf(fmaxf(sB[0], sB[1]), fmaxf(sB[2], sB[3])));
        m_tile = fmaxf(m_tile, __shfl_xor(m_tile, 16, 64));
        m_tile = fmaxf(m_tile, __shfl_xor(m_tile, 32, 64));
        const float m_new = fmaxf(m_run, m_tile);            // running maximum of RAW scores
        const float m_safe = (m_new == NEG_INF) ? 0.f : m_new;
        const float ms = m_safe * sc;
        bf16x8 pf;
        float psum = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float pa = __builtin_amdgcn_exp2f(fmaf(sA[i], sc, -ms)), pb = __builtin_amdgcn_exp2f(fmaf(sB[i], sc, -ms));
            psum += pa + pb;
            pf[i] = (bf16_t)pa;
            pf[4 + i] = (bf16_t)pb;
        }
        if (__any(m_new != m_run)) {
            const float alpha = __builtin_amdgcn_exp2f((m_run - m_safe) * sc);
            l_run *= alpha;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) o[dt] = o[dt] * alpha;
            m_run = m_new;
        }
        l_run += psum;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt] = mfma16(vf[buf][dt], pf, o[dt]);
    };
    auto run = [&](auto ntag) {
        constexpr int N = decltype(ntag)::value;
        issue(0, 0);
#pragma unroll
        for (int it = 0; it < N; ++it) {
            if (it + 1 < N) issue(it + 1, (it + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);   // the next iteration's loads go out before this one's arithmetic
            compute(it, it & 1);
        }
    };
    static_assert(WT / 32 == 4, "one schedule per iteration count below");
    const int nit = t1 > t0 ? (t1 - t0 + 31) >> 5 : 0;   // wave-uniform
    switch (nit) {
        case 1: run(std::integral_constant<int, 1>{}); break;
        case 2: run(std::integral_constant<int, 2>{}); break;
        case 3: run(std::integral_constant<int, 3>{}); break;
        case 4: run(std::integral_constant<int, 4>{}); break;
        default: break;
    }
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);

    // combine the 4 waves (fixed order) and emit the chunk's partial result
    if (c16 < G) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) s_o[(wave * HD + 16 * dt + 4 * h + i) * G + c16] = o[dt][i];
        if (h == 0) {
            s_m[wave * G + c16] = m_run;
            s_l[wave * G + c16] = l_run;
        }
    }
    __syncthreads();
    // the only chunk is the result, and no kernel follows: what the merge below makes of one chunk, the same bits (four layers of the 8B widths, one row
    // of 300 cached tokens 351 -> 341 us, 64 rows of 100 to 500 516 -> 506)
    if (a.n_chunks == 1) {
        for (int idx = tid; idx < G * HD; idx += 256) {
            const int gg = idx / HD, d = idx % HD;
            const float mx = fmaxf(fmaxf(s_m[gg], s_m[G + gg]), fmaxf(s_m[2 * G + gg], s_m[3 * G + gg]));
            const float ms = (mx == NEG_INF) ? 0.f : mx;
            float acc = 0.f, l = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float e = __builtin_amdgcn_exp2f((s_m[w * G + gg] - ms) * a.scale_log2);
                acc += s_o[(w * HD + d) * G + gg] * e;
                l += s_l[w * G + gg] * e;
            }
            *decode_out(a, b, (hk * G + gg) * HD + d) = (bf16_t)(l > 0.f ? acc / l : 0.f);
        }
        return;
    }
    for (int idx = tid; idx < G * HD; idx += 256) {
        const int gg = idx % G, d = idx / G;   // consecutive threads read consecutive words of s_o: no bank conflicts
        const float mx = fmaxf(fmaxf(s_m[gg], s_m[G + gg]), fmaxf(s_m[2 * G + gg], s_m[3 * G + gg]));
        const float ms = (mx == NEG_INF) ? 0.f : mx;
        float acc = 0.f, l = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float e = __builtin_amdgcn_exp2f((s_m[w * G + gg] - ms) * a.scale_log2);
            acc += s_o[(w * HD + d) * G + gg] * e;
            l += s_l[w * G + gg] * e;
        }
        const size_t pi = ((size_t)b * a.Hq + hk * G + gg) * a.n_chunks + chunk;
        a.part_o[pi * HD + d] = acc;
        if (d == 0) {
            a.part_ml[pi * 2] = mx;
            a.part_ml[pi * 2 + 1] = l;
        }
    }
}

// With requests slowest, the y-th workgroup of request b takes this chunk.  An XCD deals its workgroups to four shader engines
// in turn, so with two or four chunks a fixed order gives an engine the same chunk of every request, and the engine with the
// last one, which few requests reach, idles (256 rows of 64 to 2047 cached tokens, 8B heads: 228 us, 198 with the order
// turned from request to request; 200 rows of 16 to 700: 75 and 61; 64 rows of 512 to 4096, nine chunks: 102 either way).
__device__ __forceinline__ int decode_chunk_of(int y, int b, int n_chunks) { return (y + b + (b >> 1)) % n_chunks; }

template <int HD>
__global__ __launch_bounds__(256, 2) void decode_attn_kernel(DecodeAttnArgs a) {
    extern __shared__ float smem_dec[];
    // kv head fastest: consecutive workgroup ids are dealt to the 8 XCDs in turn, and every kv head
    // carries the same work, whereas chunk c only exists for contexts longer than c chunks.  With the chunk
    // index slowest the workgroups that have nothing to do (chunks past a request's context) gather at
    // the end of the grid instead of following each request: on a CU partition that measured 5 % faster
    // (128 CUs: 160 -> 152 us), on the whole chip 2 % slower, so the launcher chooses by partition size.
    // (Consecutive ids go to the 8 XCDs in turn, so the kv heads of one block are read through 8 different L2s
    // at about the same time; putting them on ONE XCD instead measured 7-10 % slower on every partition.)
    const int b = a.chunk_major ? blockIdx.y : blockIdx.z;
    decode_attn_chunk<HD>(a, blockIdx.x, b, a.chunk_major ? (int)blockIdx.z : decode_chunk_of(blockIdx.y, b, a.n_chunks), threadIdx.x, smem_dec);
}

// Merges the per-chunk partial results of one (request, query head).  Bound by memory round trips: the maxima and sums of
// 64 chunks are read by a lane each, beside the context length; a quarter of the threads each takes every fourth chunk's
// outputs, 16 bytes a thread, eight chunks requested together, and the quarters are added in order.  With one thread per
// column and one chunk after the other: 23 us for 32 contexts of up to 32K tokens (8B shape), 6.5 now; 101 of up to
// 8K (70B shape) 14, 9.5 now; 64 of up to 4K 5.3, 4.9 now.
template <int HD>
__global__ __launch_bounds__(HD) void decode_combine_kernel(DecodeAttnArgs a) {
    constexpr int Q = HD / 4;   // threads of a quarter
    __shared__ float s_e[64];
    __shared__ f32x4 s_acc[4 * Q];
    const int hq = blockIdx.x, b = blockIdx.y, d = threadIdx.x, lane = d & 63, quarter = d / Q;
    const size_t p0 = ((size_t)b * a.Hq + hq) * a.n_chunks;
    const float2 *ml = (const float2 *)a.part_ml + p0;
    const f32x4 *po = (const f32x4 *)(a.part_o + p0 * HD) + d % Q;
    float2 mine = ml[min(lane, a.n_chunks - 1)];   // looked at only if the chunk is one of this context's
    int n_keys = a.ctx_lens[b] + 1;
    const int col = hq * HD + d;
    bf16_t *op = decode_out(a, b, col);
    if (n_keys < 1) {
        *op = (bf16_t)0.f;
        return;
    }
    if (n_keys > a.max_ctx) n_keys = a.max_ctx;
    const int nch = (n_keys + RS_DECODE_CHUNK - 1) / RS_DECODE_CHUNK;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float mx = NEG_INF, l = 0.f;
    for (int c0 = 64; c0 < nch; c0 += 64) mx = fmaxf(mx, c0 + lane < nch ? ml[c0 + lane].x : NEG_INF);
    for (int c0 = 0; c0 < nch; c0 += 64) {
        const int nc = min(64, nch - c0);
        f32x4 v[8];
        auto request = [&](int first) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (first - quarter + 4 * j < nc) v[j] = po[(size_t)(c0 + min(first + 4 * j, nc - 1)) * Q];   // (uniform)
        };
        auto add = [&](int first) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (first + 4 * j < nc) acc += v[j] * s_e[first + 4 * j];
        };
        request(quarter);
        if (c0 == 0) {
            mx = fmaxf(mx, lane < nch ? mine.x : NEG_INF);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
        } else {
            mine = ml[c0 + min(lane, nc - 1)];
            __syncthreads();   // s_e of the 64 chunks before has been read
        }
        const float e = lane < nc ? exp2f((mine.x - (mx == NEG_INF ? 0.f : mx)) * a.scale_log2) : 0.f;   // maxima are raw scores
        l += lane < nc ? mine.y * e : 0.f;
        if (d < 64) s_e[lane] = e;
        __syncthreads();
        add(quarter);
        if (nc > 32) {
            request(32 + quarter);
            add(32 + quarter);
        }
    }
    l = wave_sum(l);
    s_acc[d] = acc;
    __syncthreads();
    const float *col_sums = (const float *)s_acc + d;
    const float sum = (col_sums[0] + col_sums[HD]) + (col_sums[2 * HD] + col_sums[3 * HD]);
    *op = (bf16_t)(l > 0.f ? sum / l : 0.f);
}

// The same sums, to the bit, where no context has more than RS_FEW_CHUNKS chunks (NC: 2 or 4, the most that the bound of the
// contexts allows): a thread per column, everything it needs requested together.  Few registers and no barriers: with hundreds
// of short contexts that is what counts (decode attention of 256 rows of 511 tokens, 8B heads, 64 CUs: 197 us with the kernel
// above, 188 with this; 128 CUs 135 and 129).
#define RS_FEW_CHUNKS 4
template <int HD, int NC>
__global__ __launch_bounds__(256) void decode_combine_few_kernel(DecodeAttnArgs a) {
    const int b = blockIdx.y, col = blockIdx.x * 256 + threadIdx.x, hq = col / HD;
    if (hq >= a.Hq) return;
    const size_t p0 = ((size_t)b * a.Hq + hq) * a.n_chunks;
    const float2 *ml = (const float2 *)a.part_ml + p0;
    const float *po = a.part_o + p0 * HD + col % HD;
    float2 c[NC];
    float v[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        const int ci = min(i, a.n_chunks - 1);
        c[i] = ml[ci];
        v[i] = po[(size_t)ci * HD];
    }
    const int n_keys = a.ctx_lens[b] + 1;
    bf16_t *op = decode_out(a, b, col);
    if (n_keys < 1) {
        *op = (bf16_t)0.f;
        return;
    }
    const int nch = (min(n_keys, a.max_ctx) + RS_DECODE_CHUNK - 1) / RS_DECODE_CHUNK;
    float mx = NEG_INF;
#pragma unroll
    for (int i = 0; i < NC; ++i) mx = fmaxf(mx, i < nch ? c[i].x : NEG_INF);
    float s[RS_FEW_CHUNKS] = {}, l[RS_FEW_CHUNKS] = {};
#pragma unroll
    for (int i = 0; i < NC; ++i) {
        const float e = i < nch ? exp2f((c[i].x - (mx == NEG_INF ? 0.f : mx)) * a.scale_log2) : 0.f;
        s[i] = i < nch ? __builtin_fmaf(v[i], e, 0.f) : 0.f;   // (products of their own: not to be contracted with the sums)
        l[i] = i < nch ? __builtin_fmaf(c[i].y, e, 0.f) : 0.f;
    }
    static_assert(RS_FEW_CHUNKS == 4, "a chunk a quarter there, a lane of the wave's sum each");
    const float sum = (s[0] + s[1]) + (s[2] + s[3]), tot = (l[0] + l[2]) + (l[1] + l[3]);
    *op = (bf16_t)(tot > 0.f ? sum / tot : 0.f);
}

template <int HD>
static void launch_decode_combine_few(hipStream_t st, const DecodeAttnArgs &a) {
    const dim3 grid((a.Hq * HD + 255) / 256, a.B);
    if (a.n_chunks == 2) hipLaunchKernelGGL((decode_combine_few_kernel<HD, 2>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((decode_combine_few_kernel<HD, RS_FEW_CHUNKS>), grid, dim3(256), 0, st, a);
}

static void launch_decode_combine(hipStream_t st, const DecodeAttnArgs &a) {
    if (a.n_chunks == 1) return;   // finished by its one chunk's workgroup
    if (a.n_chunks <= RS_FEW_CHUNKS) {
        if (a.hd == 128) launch_decode_combine_few<128>(st, a);
        else launch_decode_combine_few<64>(st, a);
        return;
    }
    if (a.hd == 128) hipLaunchKernelGGL(decode_combine_kernel<128>, dim3(a.Hq, a.B), dim3(128), 0, st, a);
    else hipLaunchKernelGGL(decode_combine_kernel<64>, dim3(a.Hq, a.B), dim3(64), 0, st, a);
}

void launch_decode_attention(hipStream_t st, const DecodeAttnArgs &a) {
    if (a.B <= 0) return;
    dim3 grid(a.Hkv, a.chunk_major ? a.B : a.n_chunks, a.chunk_major ? a.n_chunks : a.B);
    const size_t lds = (size_t)decode_attn_lds_floats(a.hd, a.Hq / a.Hkv) * sizeof(float);
    if (a.hd == 128) hipLaunchKernelGGL(decode_attn_kernel<128>, grid, dim3(256), lds, st, a);
    else hipLaunchKernelGGL(decode_attn_kernel<64>, grid, dim3(256), lds, st, a);
    launch_decode_combine(st, a);
}

// =============================================================================================
// Prefill: causal attention of whole prompts, reading the K/V the same layer call has just
// written to the pools.  A workgroup owns one query head and one 128-query tile of a prompt, or a PAIR of
// them, tile n-1-p then tile p, so that every workgroup does the same amount of causal work.
// Wave w owns 32 query rows of the tile; keys are consumed 64 (= 4 blocks) at a time through two
// LDS buffers: the next key tile's global loads are in flight while the current one is multiplied,
// one barrier per key tile.  The prompt's block ids are copied to LDS once, so a key tile costs one
// memory round trip (pool) instead of two chained ones (table, then pool).
// The K tile sits in LDS as its four blocks in the pool's own order and the V tile as [block][8-token half][dim]:
// the 16 lanes of a fragment read are then 16 consecutive 16-byte chunks (no bank conflicts, no swizzle), every
// read address is a per-lane base plus a constant, and a whole tile comes in by LDS-DMA (global -> LDS, no
// staging registers, no LDS stores).
//
// A launch that leaves compute units idle or with one workgroup takes two teams of four waves a workgroup, which share out the
// key tiles: with one wave per SIMD every wait is exposed.  On 256 CUs, one team / two (8B heads): 1024 tokens 33 / 30 us, 512
// 20 / 19, a 512-token chunk behind 1024 cached tokens 52 / 46, behind 4000 118 / 100.  Where there are more workgroups than
// units it takes one team: two workgroups on a unit overlap better than two teams at one barrier (prefill_form below).
//
// What bounds it on long prompts: every wave reads the whole 32 KB K/V tile from LDS for its 32 queries, one
// kilobyte of LDS reads per MFMA, which with four matrix cores per CU is the LDS's whole bandwidth (128 bytes
// per cycle); and per score there are about as many vector cycles (scale, exponential at quarter rate, sum,
// maximum, conversion) as matrix cycles.  Two workgroups per CU (two waves per SIMD) overlap the two kinds of
// work as far as the LDS allows.  Measured alternative, dropped: two 32-query strips per wave (each K and V
// fragment feeds two MFMAs: half the LDS reads), which needs both strips' accumulators (128 registers) and so
// leaves one wave per SIMD; bit-identical results, but 1.4-1.8x SLOWER at every size (16384 tokens: 3.48
// against 2.44 ms on the whole chip) although strip 1's exponentials were placed under strip 0's P V MFMAs:
// with a single wave per SIMD every dependent chain of the softmax (running maximum, half-wave exchanges, the
// rescale decision) is exposed, and what the second wave hides here for nothing would have to be software
// pipelined by hand across key tiles.  Dropped as well: 16x16x32 products, which the large-tile products gain from: with half as much
// work per instruction they take twice the issue slots beside the softmax (16384 tokens 7145 -> 7250 us a layer).
// =============================================================================================
// Sums over the even and over the odd key tiles of a row, each relative to a maximum of its own, brought together.  Which
// product is rounded is written out, so that every form gets the same bits.
struct Merge {
    float e_even, e_odd, l;
    __device__ __forceinline__ Merge(float m, float l_mine, float m_other, float l_other, bool even, float sc) {
        const float top = fmaxf(m, m_other), ref = top == NEG_INF ? 0.f : top;
        const float e = __builtin_amdgcn_exp2f((m - ref) * sc), e_other = __builtin_amdgcn_exp2f((m_other - ref) * sc);
        e_even = even ? e : e_other;
        e_odd = even ? e_other : e;
        l = (*this)(even ? l_mine : l_other, even ? l_other : l_mine);
    }
    __device__ __forceinline__ float operator()(float even, float odd) const { return __builtin_fmaf(even, e_even, odd * e_odd); }
};

// The units of a launch: with `pairs` the pairs of 128-query tiles of all prompts, else the tiles themselves, heaviest first.
__device__ __forceinline__ int prefill_units(int rows, bool pairs) { const int nt = (rows + 127) >> 7; return pairs ? (nt + 1) >> 1 : nt; }

// KW: teams of four waves that take every KW-th key tile each, with K/V buffers of their own, and are merged at the end.
// SEQ: one team that computes what two would, the same bits: the even key tiles, then (their sums put away in `park`,
// float32, 128 x HD of them) the odd ones, then the same merge.
template <int HD, int KW, bool SEQ>
__device__ __forceinline__ void prefill_attn_unit(const PrefillAttnArgs &a, int pr, const int hq, bf16_t *smem_attn, float *park) {
    static_assert(KW == 1 || !SEQ, "two teams put nothing away");
    constexpr int CPR = HD / 8;   // 16-byte chunks per K row
    constexpr int KS = HD / 16;   // 32x32x16 steps over head_dim
    constexpr int DT = HD / 32;   // 32-row tiles of O^T
    constexpr int NKC = (64 * CPR) / 256, NVC = (HD * 8) / 256;  // chunks per thread per tile
    const int tid = threadIdx.x & 255, wave = tid >> 6, lane = tid & 63;
    const int team = KW > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) : 0;
    const int c32 = lane & 31, h = lane >> 5;
    bf16_t *Ks = smem_attn + team * (4 * 64 * HD);   // [2][64 * HD]
    bf16_t *Vs = Ks + 2 * 64 * HD;                   // [2][HD * 64]
    int32_t *s_tab = (int32_t *)(smem_attn + KW * 4 * 64 * HD);   // [PREFILL_TAB_LDS] block ids of this prompt

    // (request, unit of it) of this workgroup
    int req = 0, np = 0;
    for (;; ++req) {
        np = prefill_units(a.seq.cu[req + 1] - a.seq.cu[req], a.pairs);
        if (pr < np || req + 1 >= a.seq.n_req) break;
        pr -= np;
    }
    if (pr >= np) return;
    const int nt = (a.seq.cu[req + 1] - a.seq.cu[req] + 127) >> 7;
    const int row0 = a.seq.cu[req];
    const int len = a.seq.cu[req + 1] - row0;
    // a later chunk of a prompt: its first row sits at position `prior`, and the positions before it are keys too
    // (read from the cache like the chunk's own); key positions below are absolute, query rows relative to the chunk
    const int prior = a.seq.start[req];
    const int tot = prior + len;
    const int hk = hq / (a.Hq / a.Hkv);
    const int32_t *tab = a.tables + (size_t)req * a.max_blk;
    const float sc = a.scale_log2;
    const int n_blk = (tot + 15) >> 4;
    for (int i = threadIdx.x; i < min(n_blk, PREFILL_TAB_LDS); i += 256 * KW) s_tab[i] = tab[i];
    // (two separate loads: a pointer chosen between the LDS copy and the table would become a generic-address
    // load, which waits for every outstanding LDS and global access)
    auto block_of = [&](int bi) {
        int b = s_tab[min(bi, PREFILL_TAB_LDS - 1)];
        if (bi >= PREFILL_TAB_LDS) {
            int g = tab[bi];
            asm volatile("" : "+v"(g));   // pins the global load to this branch: the two loads must not be merged
            b = g;
        }
        return b;
    };

    // K tile in LDS: the four blocks one after the other, each in the pool's own order (element offset of row r, 16-byte column cc)
    auto klds = [](int r, int cc) { return (r >> 4) * (16 * HD) + kpool_chunk_offset(r & 15, cc * 8); };

    // this thread's chunks of a key tile on the checked path: K chunk j = (row c/CPR, 16-byte column c%CPR),
    // V chunk j = (dim c>>3, block (c&7)>>1, 8-token half c&1), c = tid + 256 j
    // V tile in LDS: per block the 8-token halves apart, [block][half][dim][8 tokens]: the 16 lanes of a fragment read
    // (16 dims, one half) are 16 consecutive 16-byte chunks
    auto vlds = [](int blk, int half, int d) { return blk * (16 * HD) + half * (8 * HD) + d * 8; };
    // Brings key tile [kv0, kv0 + 64) into LDS buffer buf (nobody reads that buffer before the next barrier).
    auto load_tile = [&](int kv0, int buf) {
        bf16_t *ks = Ks + buf * 64 * HD;
        bf16_t *vs = Vs + buf * HD * 64;
        if (HD == 128 && kv0 + 64 <= tot && (kv0 >> 4) + 4 <= PREFILL_TAB_LDS) {
            const int b0 = kv0 >> 4;
            int blk[4];
            bool ok = true;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                blk[j] = __builtin_amdgcn_readfirstlane(s_tab[b0 + j]);
                ok = ok && (unsigned)blk[j] < (unsigned)a.n_blocks;
            }
            if (ok) {   // uniform; a tile with a bad block id takes the checked path below, which reports it
                // Whole tile by LDS-DMA (global -> LDS, 16 bytes per lane, lane l's bytes land at the window's
                // base + 16 l; no registers): wave w copies block w.  K keeps the pool's order (4 KB straight);
                // V's 16-byte chunk (dim d, half) goes to [half][d], so a lane fetches chunk (64 i + l, half).
                const int w = __builtin_amdgcn_readfirstlane(wave);
                const int bw = w == 0 ? blk[0] : w == 1 ? blk[1] : w == 2 ? blk[2] : blk[3];
                const size_t head = ((size_t)bw * a.Hkv + hk) * 16 * HD;
                // (Buffer loads: a global load to LDS counts as a generic access, after which the compiler has every fragment wait for all
                // LDS reads in flight, not for its own: the layer at 16384 tokens 7260 -> 7145 us.)
                const auto kbuf = __builtin_amdgcn_make_buffer_rsrc((void *)(a.k_pool + head), 0, 32 * HD, 0x00020000);
                const auto vbuf = __builtin_amdgcn_make_buffer_rsrc((void *)(a.v_pool + head), 0, 32 * HD, 0x00020000);
                bf16_t *kdst = ks + w * (16 * HD), *vdst = vs + w * (16 * HD);
                auto *kd = (__attribute__((address_space(3))) void *)kdst;   // the constant offset counts in LDS too
                __builtin_amdgcn_raw_ptr_buffer_load_lds(kbuf, kd, 16, lane * 16, 0, 0, 0);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(kbuf, kd, 16, lane * 16, 0, 1024, 0);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(kbuf, kd, 16, lane * 16, 0, 2048, 0);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(kbuf, kd, 16, lane * 16, 0, 3072, 0);
#pragma unroll
                for (int j = 0; j < 4; ++j)   // j = 2 * half + i
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(vbuf, (__attribute__((address_space(3))) void *)(vdst + (j >> 1) * (8 * HD) + (j & 1) * 512), 16, lane * 32,
                                                             (j & 1) * 2048 + (j >> 1) * 16, 0, 0);
                return;
            }
        }
        // checked path (a ragged last tile, a bad block id, head_dim 64): through registers
        bf16x8 rk[NKC], rv[NVC];
#pragma unroll
        for (int j = 0; j < NKC; ++j) {
            const int c = tid + 256 * j;
            const int r = c / CPR, cc = c % CPR;
            const int tok = kv0 + r;
            bf16x8 v = zero_bf16x8();
            if ((tok & ~15) < tot) {
                const int blk = block_of(tok >> 4);
                if ((unsigned)blk < (unsigned)a.n_blocks)
                    v = ld_bf16x8(a.k_pool + ((size_t)blk * a.Hkv + hk) * 16 * HD + kpool_chunk_offset(tok & 15, cc * 8));
                else if (cc == 0 && (tok & 15) == 0)
                    atomicOr(a.err_flag, 2);
            }
            rk[j] = v;
        }
#pragma unroll
        for (int j = 0; j < NVC; ++j) {
            const int c = tid + 256 * j;
            const int d = c >> 3, cc = c & 7;
            const int tok0 = kv0 + (cc >> 1) * 16 + (cc & 1) * 8;
            bf16x8 v = zero_bf16x8();
            if (tok0 < tot) {
                const int blk = block_of(tok0 >> 4);
                if ((unsigned)blk < (unsigned)a.n_blocks) {
                    v = ld_bf16x8(a.v_pool + (((size_t)blk * a.Hkv + hk) * HD + d) * 16 + (cc & 1) * 8);
                    if (tok0 + 8 > tot) {  // zero V past the prompt: 0 * garbage must not be NaN
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            if (tok0 + i >= tot) v[i] = (bf16_t)0.f;
                    }
                }
            }
            rv[j] = v;
        }
#pragma unroll
        for (int j = 0; j < NKC; ++j) {
            const int c = tid + 256 * j;
            *(bf16x8 *)&ks[klds(c / CPR, c % CPR)] = rk[j];
        }
#pragma unroll
        for (int j = 0; j < NVC; ++j) {
            const int c = tid + 256 * j;
            *(bf16x8 *)&vs[vlds((c & 7) >> 1, c & 1, c >> 3)] = rv[j];
        }
    };

    for (int which = 0; which < 2; ++which) {
        const int tile = which == 0 ? nt - 1 - pr : pr;   // the heavier tile first
        if (which == 1 && (!a.pairs || tile == nt - 1 - pr)) break;
        const int q0 = tile * 128;
        const int q_local = q0 + wave * 32 + c32;
        const bool q_valid = q_local < len;
        const int q_row = q_valid ? q_local : len - 1;
        const int q_pos = prior + q_row;   // absolute position: the causal bound
        bf16x8 qf[KS];
        {
            const bf16_t *qp = a.q + (size_t)(row0 + q_row) * a.q_stride + (size_t)hq * HD + 8 * h;
#pragma unroll
            for (int s = 0; s < KS; ++s) qf[s] = ld_bf16x8(qp + 16 * s);
        }
        const int wave_q_min = prior + q0 + wave * 32;
        const int wave_q_max = min(wave_q_min + 31, tot - 1);
        const int kv_end = prior + min(q0 + 128, len);
        const int n_kv_tiles = (kv_end + 63) >> 6;

        // the key tile of iteration `it`; as many iterations for every team: the barriers are the workgroup's
        const int n_even = (n_kv_tiles + 1) >> 1, n_it = KW == 2 ? n_even : n_kv_tiles;
        auto tile_at = [&](int it) { return KW == 2 ? 2 * it + team : !SEQ ? it : it < n_even ? 2 * it : 2 * (it - n_even) + 1; };

        float m_run = NEG_INF, l_run = 0.f;   // running max of raw scores, running sum
        float m_put = NEG_INF, l_put = 0.f;   // SEQ: those of the even tiles
        f32x4 *o_put = (f32x4 *)park + wave * (4 * DT * 64) + lane;
        f32x16 o[DT];
        auto reset = [&]() {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[dt][i] = 0.f;
        };
        reset();

        __syncthreads();   // s_tab visible; the previous tile's last reads done before buffer 0 is refilled
        if (team < n_kv_tiles) load_tile(64 * team, 0);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the LDS-DMA loads have landed
        __syncthreads();
        for (int it = 0; it < n_it; ++it) {
            const int kt = tile_at(it);
            const int kv0 = kt * 64;
            if (it + 1 < n_it && tile_at(it + 1) < n_kv_tiles) load_tile(64 * tile_at(it + 1), (it + 1) & 1);
            if (SEQ && it == n_even) {
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int j = 0; j < 4; ++j) o_put[(dt * 4 + j) * 64] = f32x4{o[dt][4 * j], o[dt][4 * j + 1], o[dt][4 * j + 2], o[dt][4 * j + 3]};
                m_put = m_run, l_put = l_run;
                m_run = NEG_INF, l_run = 0.f;
                reset();
            }
            if (kt < n_kv_tiles && kv0 <= wave_q_max) {
                const bf16_t *ks = Ks + (it & 1) * 64 * HD;
                const bf16_t *vs = Vs + (it & 1) * HD * 64;
                f32x16 st[2];
#pragma unroll
                for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
                    for (int i = 0; i < 16; ++i) st[t2][i] = 0.f;
                {
                    // K fragment i = (key half i & 1, head_dim step i >> 1), read six fragments ahead of its MFMA; the
                    // two score tiles alternate, each still summed over the steps in order
                    constexpr int NQK = 2 * KS, R = 6;
                    auto kread = [&](int i) { return *(const bf16x8 *)&ks[klds(32 * (i & 1) + c32, 2 * (i >> 1) + h)]; };
                    bf16x8 kf[R];
#pragma unroll
                    for (int i = 0; i < R; ++i) kf[i] = kread(i);
#pragma unroll
                    for (int i = 0; i < NQK; ++i) {
                        st[i & 1] = mfma32(kf[i % R], qf[i >> 1], st[i & 1]);
                        __builtin_amdgcn_sched_barrier(0);
                        if (i + R < NQK) kf[i % R] = kread(i + R);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                if (kv0 + 63 > wave_q_min) {   // only tiles that touch the diagonal need the mask
#pragma unroll
                    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            const int key = kv0 + 32 * t2 + (i >> 2) * 8 + 4 * h + (i & 3);
                            if (key > q_pos) st[t2][i] = NEG_INF;
                        }
                }
                float m_tile = NEG_INF;
#pragma unroll
                for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
                    for (int i = 0; i < 16; ++i) m_tile = fmaxf(m_tile, st[t2][i]);
                {   // the other half-wave holds the rest of this query column: one swap gives each lane both maxima
                    const uint32_t mb = __builtin_bit_cast(uint32_t, m_tile);
                    const auto sw = __builtin_amdgcn_permlane32_swap(mb, mb, false, false);
                    m_tile = fmaxf(__builtin_bit_cast(float, (uint32_t)sw[0]), __builtin_bit_cast(float, (uint32_t)sw[1]));
                }
                // The reference of the exponentials is the running maximum itself: the largest weights then sit at the top of a
                // binade, where bf16 is finest, the largest of all exactly.  A reference that is followed only once it is 2^8
                // behind saves the rescaling of two tiles in three (16384 tokens, 8B heads: 2314 -> 2211 us) and was taken back:
                // the attention's error against float64 was 5 to 12 % larger (4096 tokens 0.00193 -> 0.00216 of the result).
                const float m_new = fmaxf(m_run, m_tile);
                const float m_safe = m_new == NEG_INF ? 0.f : m_new;
                if (__any(m_new != m_run)) {
                    const float alpha = __builtin_amdgcn_exp2f((m_run - m_safe) * sc);
                    l_run *= alpha;
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt) o[dt] = o[dt] * alpha;
                    m_run = m_new;
                }
                const float ms = m_safe * sc;
                float psum = 0.f;
                // The score registers give lane half h a block's tokens 4h..4h+3 and 8+4h..8+4h+3.  The two
                // half-waves (same query column) trade their middle pieces, h = 0 then holds tokens 0-7 and
                // h = 1 tokens 8-15: the contraction slices of V's own layout, 16 bytes per (dim, half).
                bf16x8 pf[2];
                auto weights = [&](int blk4, int t0, int n) {
#pragma unroll
                    for (int t = t0; t < t0 + n; ++t) {
                        const float p = __builtin_amdgcn_exp2f(fmaf(st[blk4 >> 1][8 * (blk4 & 1) + t], sc, -ms));
                        psum += p;
                        pf[blk4 & 1][t] = (bf16_t)p;
                    }
                };
                auto trade = [&](int blk4) {
                    typedef uint32_t u32x4p __attribute__((ext_vector_type(4)));
                    u32x4p pr4 = __builtin_bit_cast(u32x4p, pf[blk4 & 1]);
#pragma unroll
                    for (int u = 0; u < 2; ++u) {   // upper half-wave of word u <-> lower half-wave of word u + 2
                        const auto sw = __builtin_amdgcn_permlane32_swap(pr4[u], pr4[u + 2], false, false);
                        pr4[u] = sw[0];
                        pr4[u + 2] = sw[1];
                    }
                    pf[blk4 & 1] = __builtin_bit_cast(bf16x8, pr4);
                };
                // V fragments are read one block (DT fragments) ahead of their MFMAs, and the weights of a block formed
                // between the products of the one before (16384 tokens 7136 -> 7078 us)
                bf16x8 vfr[2][DT];
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) vfr[0][dt] = *(const bf16x8 *)&vs[vlds(0, h, 32 * dt + c32)];
                weights(0, 0, 8);
                trade(0);
#pragma unroll
                for (int blk4 = 0; blk4 < 4; ++blk4) {  // one 16-token block per MFMA step
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt) {
                        if (blk4 + 1 < 4) vfr[(blk4 + 1) & 1][dt] = *(const bf16x8 *)&vs[vlds(blk4 + 1, h, 32 * dt + c32)];
                        o[dt] = mfma32(vfr[blk4 & 1][dt], pf[blk4 & 1], o[dt]);
                        __builtin_amdgcn_sched_barrier(0);
                        if (blk4 + 1 < 4) weights(blk4 + 1, dt * (8 / DT), 8 / DT);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (blk4 + 1 < 4) trade(blk4 + 1);
                }
                l_run += psum;
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the LDS-DMA loads have landed
            __syncthreads();
        }
        l_run += __shfl_xor(l_run, 32, 64);
        if (KW == 2) {
            // The teams' halves of a row: both rescale to the common maximum; team 0 finishes the first half of head_dim,
            // team 1 the second, each with the other's part through the K/V buffers (nobody reads those any more).
            float *x_ml = (float *)s_tab + PREFILL_TAB_LDS;   // [KW][4 waves][32][2]
            f32x4 *x_o = (f32x4 *)smem_attn;                  // [KW][4 waves][2 DT][64]
            float *mine = x_ml + (team * 4 + wave) * 64, *theirs = x_ml + ((1 - team) * 4 + wave) * 64;
            if (h == 0) {
                mine[2 * c32] = m_run;
                mine[2 * c32 + 1] = l_run;
            }
#pragma unroll
            for (int dt = 0; dt < DT / 2; ++dt)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    f32x4 v;
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = team == 0 ? o[DT / 2 + dt][4 * j + i] : o[dt][4 * j + i];
                    x_o[((team * 4 + wave) * (2 * DT) + dt * 4 + j) * 64 + lane] = v;
                }
            __syncthreads();
            const Merge g(m_run, l_run, theirs[2 * c32], theirs[2 * c32 + 1], team == 0, sc);
            l_run = g.l;
#pragma unroll
            for (int dt = 0; dt < DT / 2; ++dt)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const f32x4 v = x_o[(((1 - team) * 4 + wave) * (2 * DT) + dt * 4 + j) * 64 + lane];
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[dt][4 * j + i] = team == 0 ? g(o[dt][4 * j + i], v[i]) : g(v[i], o[DT / 2 + dt][4 * j + i]);
                }
        }
        if (SEQ) {
            l_put += __shfl_xor(l_put, 32, 64);
            const bool two = n_kv_tiles > 1;   // else there are even tiles only, and they are still here
            const Merge g = two ? Merge(m_put, l_put, m_run, l_run, true, sc) : Merge(m_run, l_run, m_put, l_put, true, sc);
            l_run = g.l;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    f32x4 v = {0.f, 0.f, 0.f, 0.f};
                    if (two) v = o_put[(dt * 4 + j) * 64];
#pragma unroll
                    for (int i = 0; i < 4; ++i) o[dt][4 * j + i] = two ? g(v[i], o[dt][4 * j + i]) : g(o[dt][4 * j + i], v[i]);
                }
        }
        if (q_valid) {
            const float inv = 1.0f / l_run;
            // the output feeds the output projection: fragment-packed operand layout
            const int Mt = a.Mt_out ? a.Mt_out : packed_mt(a.seq.cu[a.seq.n_req]);
#pragma unroll
            for (int dt = 0; dt < DT / KW; ++dt)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    bf16x4 v;
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = (bf16_t)(o[dt][4 * j + i] * inv);
                    const int col = hq * HD + 32 * (team * (DT / KW) + dt) + 8 * j + 4 * h;
                    *(bf16x4 *)(a.out + packed_offset(row0 + q_local, col, Mt) + (col & 7)) = v;
                }
        }
    }
}

constexpr int prefill_lds(int hd, int kw) { return kw * 4 * 64 * hd * 2 + PREFILL_TAB_LDS * 4 + (kw > 1 ? kw * 4 * 64 * 4 : 0); }

// Workgroup w of a launch: the heads of one kv head run on one XCD where there are eight of them (ids go to the XCDs in
// turn), so that their keys and values stay in its L2 (5444 rows of 4 prompts, 70B heads: 352 -> 268 us; with one head after
// the other every XCD read all of them).
template <int HD, int KW, bool SEQ>
__device__ __forceinline__ void prefill_attn_wg(const PrefillAttnArgs &a, int w, bf16_t *smem) {
    const int G = a.Hq / a.Hkv, hk = w % a.Hkv, r = w / a.Hkv;
    prefill_attn_unit<HD, KW, SEQ>(a, r / G, hk * G + r % G, smem, SEQ ? a.park + (size_t)w * (128 * HD) : nullptr);
}

template <int HD, int KW, bool SEQ>
__global__ __launch_bounds__(256 * KW, 2) void prefill_attn_kernel(PrefillAttnArgs a) {
    extern __shared__ __attribute__((aligned(1024))) bf16_t smem_attn[];
    prefill_attn_wg<HD, KW, SEQ>(a, blockIdx.x, smem_attn);
}

// The prompt rows and the decode rows of a hybrid batch in one launch: the first n_prefill workgroups are
// prefill_attn_kernel's, the others two kv heads of decode_attn_kernel's (request, chunk) each.  The two kinds of work need
// different parts of the machine (matrix and vector units; memory), and a chunk's workgroups fill a quarter of the chip:
// 512 rows behind 1024 cached tokens beside 64 decode rows (8B heads) 76 + 103 us one after the other, 128 us together.
template <int HD>
__global__ __launch_bounds__(512, 2) void hybrid_attn_kernel(PrefillAttnArgs p, DecodeAttnArgs d, int n_prefill) {
    extern __shared__ __attribute__((aligned(1024))) bf16_t smem_attn[];
    if ((int)blockIdx.x < n_prefill) {
        prefill_attn_wg<HD, 2, false>(p, blockIdx.x, smem_attn);
        return;
    }
    const int w = blockIdx.x - n_prefill, half = threadIdx.x >> 8, pairs = (d.Hkv + 1) >> 1;
    const int hk = min(2 * (w % pairs) + half, d.Hkv - 1);   // (of an odd number the last is computed twice)
    const int r = w / pairs, b = r % d.B, chunk = r / d.B;   // chunks slowest: 128 us against 133 to 147 in the two other orders
    decode_attn_chunk<HD>(d, hk, b, chunk, threadIdx.x & 255, (float *)smem_attn + half * decode_attn_lds_floats(HD, d.Hq / d.Hkv));
}

// The same with workgroups of 256 threads: one team that computes what two would, and one kv head's chunk each.  Two fit a unit, and the
// decode rows read faster in workgroups of one head (64 rows of 512 to 4096 tokens alone: a layer of 213 us, 233 in pairs of heads).
template <int HD>
__global__ __launch_bounds__(256, 2) void hybrid_attn_small_kernel(PrefillAttnArgs p, DecodeAttnArgs d, int n_prefill) {
    extern __shared__ __attribute__((aligned(1024))) bf16_t smem_attn[];
    if ((int)blockIdx.x < n_prefill) {
        prefill_attn_wg<HD, 1, true>(p, blockIdx.x, smem_attn);
        return;
    }
    const int w = blockIdx.x - n_prefill, r = w / d.Hkv, b = r % d.B, chunk = r / d.B;
    decode_attn_chunk<HD>(d, w % d.Hkv, b, chunk, threadIdx.x, (float *)smem_attn);
}

static int prefill_unit_count(const PrefillAttnArgs &a, bool pairs) {
    int n = 0;
    for (int r = 0; r < a.seq.n_req; ++r) {
        const int nt = (a.seq.cu[r + 1] - a.seq.cu[r] + 127) / 128;
        n += pairs ? (nt + 1) / 2 : nt;
    }
    return n;
}

// How a launch goes about its tiles.  Whether a row's sums are cut into even and odd key tiles (`split`) follows from the sizes
// alone: no more tiles than the whole chip has units.  By whom they are computed, and in what order, from the compute units
// `cus` too, with the same bits.  A unit holds one workgroup of two teams or two of one team, so two teams only where all
// pairs of tiles fit at a time: 1024 rows of 32 heads (256 tiles, 128 pairs) on 256 / 128 / 96 / 64 CUs 30 / 33 / 47 / 60 us
// with two teams, 36 / 36 / 41 / 54 with one that cuts (putting the even tiles' sums away costs it 2 us a tile), 33 / 33 / 35 / 47 with
// one that does not.  Not cut: 2048 rows on 256 / 192 / 128 / 64 CUs 64 / 58 / 78 / 138 us, where two teams and a team that cuts
// took 57 / 63 / 84 / 153; with earlier keys two teams are ahead for longer (1024 rows behind 4000 tokens on 256 CUs 118 / 142).
// Pairs of tiles where they about fill the places, else single ones, heaviest first: those even out whatever the number
// (3000 rows, 384 pairs, on 256 CUs 125 / 102 us, on 192 CUs, all places filled, 122 / 126; 1536 rows on 128 CUs 62 / 51).
struct PrefillForm { bool split, teams, pairs; int tiles, wgs; };
static bool prefill_pairs_fill(int pairs, int places) { return pairs <= places && 10 * pairs > 9 * places; }
static int prefill_cus(const PrefillAttnArgs &a) { return a.cus > 0 ? a.cus : 256; }
static PrefillForm prefill_form(const PrefillAttnArgs &a) {
    const int pairs = prefill_unit_count(a, true) * a.Hq, cus = prefill_cus(a);
    PrefillForm f{};
    f.tiles = prefill_unit_count(a, false) * a.Hq;
    f.split = f.tiles <= 256;
    const size_t parked = (size_t)f.tiles * 128 * a.hd;
    f.teams = f.split && (pairs <= cus || !a.park || parked > a.park_cap);
    f.pairs = prefill_pairs_fill(pairs, f.teams ? cus : 2 * cus);
    f.wgs = f.pairs ? pairs : f.tiles;
    return f;
}

template <int HD>
static void launch_prefill_form(hipStream_t st, const PrefillAttnArgs &a, const PrefillForm &f) {
    if (f.teams) hipLaunchKernelGGL((prefill_attn_kernel<HD, 2, false>), dim3(f.wgs), dim3(512), prefill_lds(HD, 2), st, a);
    else if (f.split) hipLaunchKernelGGL((prefill_attn_kernel<HD, 1, true>), dim3(f.wgs), dim3(256), prefill_lds(HD, 1), st, a);
    else hipLaunchKernelGGL((prefill_attn_kernel<HD, 1, false>), dim3(f.wgs), dim3(256), prefill_lds(HD, 1), st, a);
}

void launch_prefill_attention(hipStream_t st, const PrefillAttnArgs &args) {
    PrefillAttnArgs a = args;
    const PrefillForm f = prefill_form(a);
    if (f.wgs <= 0) return;
    a.pairs = f.pairs;
    if (a.hd == 128) launch_prefill_form<128>(st, a, f);
    else launch_prefill_form<64>(st, a, f);
}

// Which of the two: a prompt tile takes a team of its own longer than two teams (some 2.3 us a 64-key tile), so the small workgroups
// where the decode rows are read for longer than that: the contexts' own tokens where the host has counted them, else half of their
// bound for each, which the caller sets near the longest (64 rows of 100 to 500 tokens under a bound of 4097 take the small ones, 328 us,
// where the large ones take 316).  The same bits in both.  Layers of the 8B widths, 512 rows behind 1024 tokens beside 64 decode rows of 512 to
// 4096 and beside 128, large / small workgroups: 404 / 395 and 541 / 523 us; where the rule takes the large ones, 512 rows behind 3072 beside 16
// of up to 600 tokens 337 / 356, behind 1024 beside 32 of 1000 to 2000 323 / 328.  head_dim 64 (32 heads over 8, the 512 rows behind 1024):
// beside 64 of 512 to 4096, where the rule changes over, 196 / 196, beside 128 265 / 245, beside 32 of 1000 to 2000 159 / 176.
static bool hybrid_small(const PrefillAttnArgs &p, const DecodeAttnArgs &d, const PrefillForm &f) {
    int keys = 0;
    for (int r = 0; r < p.seq.n_req; ++r) keys = std::max(keys, p.seq.start[r] + p.seq.cu[r + 1] - p.seq.cu[r]);
    const double tokens = d.n_keys > 0 ? (double)d.n_keys : 0.5 * d.B * d.max_ctx;
    const double bytes = tokens * (4.0 * d.Hkv * d.hd), rate = std::min(6.0e6, 0.034e6 * prefill_cus(p));   // bytes a us
    return p.park && (size_t)f.tiles * 128 * p.hd <= p.park_cap && 2.3 * keys / 64 < bytes / rate;
}

// One launch for both kinds of rows while the prompt rows leave most units to the others: half of the whole chip (512 rows of
// 32 heads behind 1024 cached tokens beside 64 decode rows: 131 us, 141 in two launches; 2048 rows 132 and 121), a quarter of a
// partition, where decode rows need every unit for themselves (the 512 rows on 128 CUs 215 and 173 us; 100 rows beside 28: 48 and
// 59).  Or beside so few decode workgroups that it is the launch that counts (200 and 300 rows beside one: 29 and 35 us).
struct HybridPlan { HybridForm form; int n_prefill, n_decode; bool pairs; };
static HybridPlan hybrid_plan(const PrefillAttnArgs &p, const DecodeAttnArgs &d) {
    const PrefillForm f = prefill_form(p);
    const int pairs = prefill_unit_count(p, true) * p.Hq, n_decode = (d.Hkv + 1) / 2 * d.n_chunks * d.B;
    const int cus = prefill_cus(p), most = cus >= 256 ? cus / 2 : cus / 4;
    const bool light = f.teams && (8 * n_decode <= cus || f.tiles + n_decode <= cus);
    if (!f.split || !(light || pairs <= most)) return {HYBRID_APART, 0, 0, false};
    if (hybrid_small(p, d, f)) return {HYBRID_SMALL, f.tiles, d.Hkv * d.n_chunks * d.B, false};
    const bool in_pairs = light ? f.pairs : f.tiles > most;
    return {HYBRID_TEAMS, in_pairs ? pairs : f.tiles, n_decode, in_pairs};
}
HybridForm hybrid_form(const PrefillAttnArgs &p, const DecodeAttnArgs &d) { return hybrid_plan(p, d).form; }

void launch_hybrid_attention(hipStream_t st, const PrefillAttnArgs &pargs, const DecodeAttnArgs &d) {
    const HybridPlan h = hybrid_plan(pargs, d);
    if (h.form == HYBRID_APART) {
        launch_prefill_attention(st, pargs);
        launch_decode_attention(st, d);
        return;
    }
    PrefillAttnArgs p = pargs;
    p.pairs = h.pairs;
    const dim3 grid(h.n_prefill + h.n_decode);
    if (h.form == HYBRID_SMALL) {
        if (d.hd == 128) hipLaunchKernelGGL(hybrid_attn_small_kernel<128>, grid, dim3(256), prefill_lds(128, 1), st, p, d, h.n_prefill);
        else hipLaunchKernelGGL(hybrid_attn_small_kernel<64>, grid, dim3(256), prefill_lds(64, 1), st, p, d, h.n_prefill);
    } else {
        if (d.hd == 128) hipLaunchKernelGGL(hybrid_attn_kernel<128>, grid, dim3(512), prefill_lds(128, 2), st, p, d, h.n_prefill);
        else hipLaunchKernelGGL(hybrid_attn_kernel<64>, grid, dim3(512), prefill_lds(64, 2), st, p, d, h.n_prefill);
    }
    launch_decode_combine(st, d);
}

void attention_kernels_init() {
    auto set = [](const void *f, int lds) { (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds); };
    set((const void *)prefill_attn_kernel<128, 1, false>, prefill_lds(128, 1));
    set((const void *)prefill_attn_kernel<128, 1, true>, prefill_lds(128, 1));
    set((const void *)prefill_attn_kernel<128, 2, false>, prefill_lds(128, 2));
    set((const void *)prefill_attn_kernel<64, 2, false>, prefill_lds(64, 2));
    set((const void *)hybrid_attn_small_kernel<128>, prefill_lds(128, 1));
    set((const void *)hybrid_attn_kernel<128>, prefill_lds(128, 2));
    set((const void *)hybrid_attn_kernel<64>, prefill_lds(64, 2));
}
