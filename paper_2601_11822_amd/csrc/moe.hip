// Sparse (mixture-of-experts) feed-forward block around the grouped form of the large-tile GEMM:
// route each row to its two experts, lay the (row, expert) assignments out expert by expert in
// whole tiles, gather the normalised rows into that order, run gate/up and down once over
// all tiles (each tile reads its own expert's weights), and add the two weighted results back.
#include "kernels.h"

// ---------------------------------------------------------------------------------------------
// Router: logits of row m = h[m] . Wr[e] for the E experts (h fragment-packed, Wr row-major), then
// the two largest (lower index first on ties) and the softmax over those two.  One workgroup per 32
// rows, on the matrix cores: the experts are the 32x32x16 product's rows (those past E repeat the last
// one and are not looked at), 16 waves take a sixteenth of K each and are summed in wave order (1100 rows of 4096, 8
// experts: 73 us with vector arithmetic, 32 threads a row and one weight row at a time, 13 us now).  What
// bounds it is one round trip to memory, so a wave requests RS_ROUTER_KB k-blocks at a time.
// ---------------------------------------------------------------------------------------------
#define RS_ROUTER_KB 8
__global__ __launch_bounds__(1024) void moe_router_kernel(MoeArgs a) {
    __shared__ float red[16][RS_MOE_MAX_EXPERTS][32];
    __shared__ float logit[RS_MOE_MAX_EXPERTS][33];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, c32 = lane & 31, h = lane >> 5;
    const int Mt = packed_mt(a.M), Kb = a.d >> 4, per = (Kb + 15) >> 4;
    const int kb0 = wave * per, kb1 = min(kb0 + per, Kb);
    const bf16_t *hp = a.h + (size_t)blockIdx.x * 512 + lane * 8;
    const bf16_t *wp = a.router + (size_t)min(c32, a.E - 1) * a.d + 8 * h;
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    int kb = kb0;
    for (; kb + RS_ROUTER_KB <= kb1; kb += RS_ROUTER_KB) {
        bf16x8 hv[RS_ROUTER_KB], wv[RS_ROUTER_KB];
#pragma unroll
        for (int j = 0; j < RS_ROUTER_KB; ++j) {
            hv[j] = ld_bf16x8(hp + (size_t)(kb + j) * Mt * 512);
            wv[j] = ld_bf16x8(wp + (kb + j) * 16);
        }
#pragma unroll
        for (int j = 0; j < RS_ROUTER_KB; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv[j], hv[j], acc, 0, 0, 0);
    }
    for (; kb < kb1; ++kb) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ld_bf16x8(wp + kb * 16), ld_bf16x8(hp + (size_t)kb * Mt * 512), acc, 0, 0, 0);
    // registers 0..7 hold experts 4h..4h+3 and 8+4h..8+4h+3 of row c32
#pragma unroll
    for (int e = 0; e < 8; ++e) red[wave][8 * (e >> 2) + 4 * h + (e & 3)][c32] = acc[e];
    __syncthreads();
    if (tid < 32 * RS_MOE_MAX_EXPERTS) {
        const int e = tid >> 5;
        float v = red[0][e][c32];
#pragma unroll
        for (int w = 1; w < 16; ++w) v += red[w][e][c32];
        logit[e][c32] = v;
    }
    __syncthreads();
    const int m = blockIdx.x * 32 + tid;
    if (tid < 32 && m < a.M) {
        int e0 = 0;
        for (int e = 1; e < a.E; ++e)
            if (logit[e][tid] > logit[e0][tid]) e0 = e;
        int e1 = -1;
        for (int e = 0; e < a.E; ++e)
            if (e != e0 && (e1 < 0 || logit[e][tid] > logit[e1][tid])) e1 = e;
        const float eb = expf(logit[e1][tid] - logit[e0][tid]);
        a.sel[2 * m] = e0;
        a.sel[2 * m + 1] = e1;
        a.wt[2 * m] = 1.0f / (1.0f + eb);
        a.wt[2 * m + 1] = eb / (1.0f + eb);
    }
}

// ---------------------------------------------------------------------------------------------
// Plan (one workgroup): per-expert counts, each expert's segment in whole tiles (of one height per expert: as few tiles of
// at most a.limit rows as hold it, each no higher than needed, in steps of 32 rows and at least 128; of four or more the last ones
// a step lower where that still holds it: four tiles hide that one of them runs ahead, which two do not; 4000 rows through 8 experts
// of the 8B widths 3247 -> 3130 us, on 64 CUs 8057 -> 7888, in steps of 64; steps of 32 against 64, the whole layer: 600 rows 764 -> 758 us,
// 1100 1160 -> 1130, 1500 1273 -> 1226, 2500 2086 -> 1957, 4000 2959 -> 2922), the grouped GEMM's work
// list (units, rows in use, then per unit its first row / 32, blocks with rows, height / 32 and expert), the source row of every grouped row
// (-1 for padding) and the grouped position of every assignment.  The order of rows inside a
// segment is arbitrary (an atomic cursor): a row's result does not depend on where it sits.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void moe_plan_kernel(MoeArgs a) {
    __shared__ int cnt[RS_MOE_MAX_EXPERTS], off[RS_MOE_MAX_EXPERTS], cur[RS_MOE_MAX_EXPERTS];
    const int tid = threadIdx.x;
    if (tid < RS_MOE_MAX_EXPERTS) cnt[tid] = cur[tid] = 0;
    __syncthreads();
    for (int i = tid; i < 2 * a.M; i += 1024) atomicAdd(&cnt[a.sel[i]], 1);
    for (int i = tid; i < a.Mg_cap; i += 1024) a.src[i] = -1;
    __syncthreads();
    __shared__ int units[RS_MOE_MAX_EXPERTS], h32[RS_MOE_MAX_EXPERTS], lower[RS_MOE_MAX_EXPERTS], first[RS_MOE_MAX_EXPERTS];
    if (tid < a.E) {
        const int c = cnt[tid], k = (c + a.limit - 1) / a.limit, h = k ? max(4, (c + 32 * k - 1) / (32 * k)) : 0;
        units[tid] = k;
        h32[tid] = h;
        lower[tid] = k >= 4 ? k * h - ((c + 31) >> 5) : 0;   // this many of the last ones
    }
    __syncthreads();
    if (tid == 0) {
        int row = 0, nu = 0, nu_tall = 0;
        for (int tall = 1; tall >= 0; --tall) {   // experts whose units are of more than 256 rows first
            for (int e = 0; e < a.E; ++e) {
                if ((h32[e] > 8) != tall) continue;
                off[e] = row;
                first[e] = nu;
                nu += units[e];
                row += 32 * (units[e] * h32[e] - lower[e]);
            }
            if (tall) nu_tall = nu;
        }
        a.units[0] = nu_tall << 16 | nu;
        a.units[1] = row;
    }
    __syncthreads();
    if (tid < a.E)
        for (int j = 0, left = cnt[tid], row = off[tid]; j < units[tid]; ++j) {
            const int h = j < units[tid] - lower[tid] ? h32[tid] : h32[tid] - 1;
            a.units[2 + first[tid] + j] = (row >> 5) << 13 | min((left + 31) >> 5, h) << 9 | h << 5 | tid;
            row += 32 * h;
            left -= 32 * h;
        }
    __syncthreads();
    for (int i = tid; i < 2 * a.M; i += 1024) {
        const int e = a.sel[i];
        const int p = off[e] + atomicAdd(&cur[e], 1);
        a.pos[i] = p;
        a.src[p] = i >> 1;
    }
}

// Gathered, fragment-packed GEMM input: grouped row g takes the chunks of its source row (zeros for padding).
// A workgroup has 256 rows of one 16-byte column; all workgroups of a column run on one XCD, since the lines that they read, eight rows' chunks each, are the same ones
// in another order (dealt out in turn every XCD fetched all of the rows: 1100 rows of 4096 and 8 experts 12.3 -> 9.0 us, 4000 24.6 -> 20.6; 64 to 450 rows 5.4 to 5.6 either way).
__global__ __launch_bounds__(256) void moe_gather_kernel(MoeArgs a, int row_groups) {
    const int i = blockIdx.x >> 3, c = (i / row_groups) * 8 + (blockIdx.x & 7), g = (i % row_groups) * 256 + threadIdx.x;
    // consecutive threads take consecutive rows of one k chunk: whole 128-byte lines on the writing side
    if (c >= a.d >> 3 || g >= a.units[1]) return;   // past the last tile in use
    const int s = a.src[g];
    const bf16x8 v = s >= 0 ? ld_bf16x8(a.h + packed_offset(s, c * 8, packed_mt(a.M))) : zero_bf16x8();
    st_bf16x8(a.a_g + packed_offset(g, c * 8, a.Mg_cap >> 5), v);
}

// y[m] = x1[m] + w0 * out[pos0] + w1 * out[pos1], float32 arithmetic.  One workgroup per row.
__global__ __launch_bounds__(256) void moe_combine_kernel(MoeArgs a) {
    const int m = blockIdx.x;
    const float w0 = a.wt[2 * m], w1 = a.wt[2 * m + 1];
    const bf16_t *o0 = a.out_g + (size_t)a.pos[2 * m] * a.d, *o1 = a.out_g + (size_t)a.pos[2 * m + 1] * a.d;
    const bf16_t *xr = a.x1 + (size_t)m * a.d;
    bf16_t *yr = a.y + (size_t)m * a.d;
    for (int c = threadIdx.x; c < (a.d >> 3); c += 256) {
        const bf16x8 x = ld_bf16x8(xr + c * 8), p = ld_bf16x8(o0 + c * 8), q = ld_bf16x8(o1 + c * 8);
        bf16x8 r;
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] = (bf16_t)((float)x[i] + (w0 * (float)p[i] + w1 * (float)q[i]));
        st_bf16x8(yr + c * 8, r);
    }
}

void launch_moe_route_and_gather(hipStream_t st, const MoeArgs &a) {
    if (a.M <= 0) return;
    hipLaunchKernelGGL(moe_router_kernel, dim3((a.M + 31) / 32), dim3(1024), 0, st, a);
    hipLaunchKernelGGL(moe_plan_kernel, dim3(1), dim3(1024), 0, st, a);
    const int row_groups = (a.Mg_cap + 255) / 256, columns = (a.d / 8 + 7) / 8 * 8;
    hipLaunchKernelGGL(moe_gather_kernel, dim3(row_groups * columns), dim3(256), 0, st, a, row_groups);
}

void launch_moe_combine(hipStream_t st, const MoeArgs &a) {
    if (a.M <= 0) return;
    hipLaunchKernelGGL(moe_combine_kernel, dim3(a.M), dim3(256), 0, st, a);
}
