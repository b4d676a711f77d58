// Host-callable launchers of the gfx950 kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

// out[m,:] = x[m,:] * rsqrt(mean(x[m,:]^2) + eps) * g      (bf16 in, fp32 math, bf16 out)
// x is row-major [M][d]; `out` is written fragment-packed (packed_offset with packed_mt(M) row tiles).
void launch_rmsnorm(hipStream_t st, const bf16_t *x, const bf16_t *g, bf16_t *out, int M, int d, float eps);

// A launch of 128 rows or more (row_grid rounds it up to whole groups of 128) gives an XCD 16 consecutive rows of each group:
// the pieces of a line that belong to neighbouring rows (a K or V block's tokens, a fragment-packed operand's rows) meet in one L2.
__device__ __forceinline__ int row_of(int x, int grid) { return grid < 128 ? x : (x & ~127) + (x & 7) * 16 + ((x >> 3) & 15); }
static int row_grid(int M) { return M < 128 ? M : (M + 127) / 128 * 128; }

struct RopeKvArgs {
    bf16_t *qkv;            // [M][nqkv]; q part rotated in place
    const CosSin *table;    // [max_pos][hd/2]
    bf16_t *k_pool;         // this layer: [n_blocks][Hkv][16][hd]
    bf16_t *v_pool;         // this layer: [n_blocks][Hkv][hd][16]
    const int32_t *tables;  // [n_req][max_blk]
    const int32_t *ctx_lens;  // decode: position of row m (and request = m); prefill: nullptr
    int32_t *err_flag;
    int M, Hq, Hkv, hd, max_blk, n_blocks, max_pos;
    SeqInfo seq;  // prefill only
};
void launch_rope_kvwrite(hipStream_t st, const RopeKvArgs &a);

struct PrefillAttnArgs {
    const bf16_t *q;  // [T][q_stride] (rotated)
    int q_stride;
    bf16_t *out;  // [T][Hq*hd], fragment-packed (packed_mt(T) row tiles)
    const bf16_t *k_pool, *v_pool;
    const int32_t *tables;
    int32_t *err_flag;
    int Hq, Hkv, hd, max_blk, n_blocks;
    float scale_log2;  // log2(e)/sqrt(hd)
    SeqInfo seq;       // seq.start[r] > 0: the rows are a later chunk of prompt r and also attend to its cached positions before them
    int Mt_out = 0;    // row tiles of the packed output matrix when it holds more rows than this call's (0: packed_mt of this call's rows)
    int cus = 0;       // compute units of the launching stream's partition (0: the whole chip); scheduling only
    float *park = nullptr;   // float32 scratch, free until the launch is done: without it two teams of waves where one would be faster
    size_t park_cap = 0;     // elements
    bool pairs = true; // set by the launchers
};
void launch_prefill_attention(hipStream_t st, const PrefillAttnArgs &a);

struct DecodeAttnArgs {
    const bf16_t *q;  // [B][q_stride]
    int q_stride;
    bf16_t *out;  // [B][Hq*hd], fragment-packed (packed_mt(B) row tiles)
    const bf16_t *k_pool, *v_pool;
    const int32_t *tables;
    const int32_t *ctx_lens;
    int32_t *err_flag;
    float *part_o;   // [B][Hq][n_chunks][hd]
    float *part_ml;  // [B][Hq][n_chunks][2]
    int B, Hq, Hkv, hd, max_blk, n_blocks, max_ctx, n_chunks;
    float scale_log2;
    int chunk_major;   // order of the workgroups only (results do not depend on it): chunks slowest, else requests slowest
    int out_row0 = 0, out_Mt = 0;   // the packed output matrix holds other rows first / more row tiles (0: packed_mt(B))
    int64_t n_keys = 0;             // tokens of all contexts, where the host knows them (0: it knows max_ctx alone); scheduling only
};
#define RS_SKINNY_TARGET_WGS 384  // the skinny GEMM splits K until it has about this many workgroups
#define RS_DECODE_CHUNK 512  // tokens per workgroup of the decode attention
void launch_decode_attention(hipStream_t st, const DecodeAttnArgs &a);
// Both.  HYBRID_APART: a launch each; else one launch, in workgroups of 512 threads (HYBRID_TEAMS) or of 256 (HYBRID_SMALL).
enum HybridForm { HYBRID_APART, HYBRID_TEAMS, HYBRID_SMALL };
HybridForm hybrid_form(const PrefillAttnArgs &p, const DecodeAttnArgs &d);
void launch_hybrid_attention(hipStream_t st, const PrefillAttnArgs &p, const DecodeAttnArgs &d);

enum GemmEpilogue { EPI_STORE = 0, EPI_RESIDUAL = 1, EPI_SWIGLU = 2 };

// out[M,N] = epi(A[M,K] * W[N,K]^T).  EPI_RESIDUAL adds resid[M,N].  EPI_SWIGLU:
// out[M,N] = silu(A*W^T) * (A*W2^T) with W, W2 both [N,K].
// A is always fragment-packed (packed_offset, packed_mt(M) row tiles).  W / W2 are the caller's
// row-major matrices (read by the tail-safe tiled kernel), Wp / Wp2 the library's fragment-packed
// copies of the same matrices (launch_pack_weights; read by the direct and the skinny kernels).
struct GemmArgs {
    const bf16_t *A;
    const bf16_t *W, *W2;
    const bf16_t *Wp, *Wp2;
    const bf16_t *resid;  // row-major [M][N]
    bf16_t *out;          // row-major [M][N]; EPI_SWIGLU: fragment-packed (it feeds another GEMM)
    int M, N, K;
    int epi;
    int cus = 0;  // compute units of the launching stream's partition (0: the whole chip); scheduling only
    // float32 scratch for launch_gemm_tiled's K-sliced path (few tiles, long K); without it that path is not taken
    float *partials = nullptr;
    size_t partial_cap = 0;   // elements
    // grouped form (launch_gemm_grouped): the work list, and the distance in elements between consecutive experts'
    // packed matrices (Wp and Wp2 alike)
    const int32_t *units = nullptr;
    size_t expert_stride = 0;
    bool stream_weights = false;   // grouped_streams_weights
    bool tall = false;             // grouped_cut
};
// Upper bound of what the K-sliced path of launch_gemm_tiled needs, for any M: S * M * N <= this.
#define RS_DIRECT_PARTIAL_ELEMS ((size_t)10 << 20)
// false (nothing launched): the shape needs the generic kernel, which reads a.W / a.W2, and they are null
bool launch_gemm_tiled(hipStream_t st, const GemmArgs &a);
// The main pass alone where launch_gemm_tiled would cut K into slices: leaves part[s][M][N] in a.partials and returns the
// number of slices; otherwise launches nothing and returns 0.
int launch_gemm_tiled_partials(hipStream_t st, const GemmArgs &a);

// How launch_gemm_tiled cuts a large-tile product: K slices (1: none) and, for S of them, tile rows x columns (MIXED: whole rounds of the
// tile of these rows, then a round of half tiles).
enum DirectForm { FORM_128x256, FORM_160x256, FORM_192x256, FORM_224x256, FORM_256x256, FORM_256x192, FORM_192x128, FORM_MIXED_256, FORM_MIXED_192, FORM_288x256, FORM_320x256 };
int direct_splits(int M, int N, int K);
DirectForm direct_form(int M, int N, int K, int epi, int S, int cus);
bool direct_streams(int m_tiles, int cus);   // whether a whole product of so many row tiles reads its weights as a stream

// Skinny variant for M <= 64 (decode): weight-streaming, deterministic split-K through
// `partials` (fp32, at least skinny_partial_elems(...) elements).  Reads A, Wp and Wp2.
// a.partial_cap (elements, in proportion to M) limits the slices of a residual projection that takes the large tiles.
size_t skinny_partial_elems(int M, int N, int K, int epi);
void launch_gemm_skinny(hipStream_t st, const GemmArgs &a, float *partials);
// Main pass only (a.epi must be EPI_STORE): leaves part[s][m][n], s < *S_out K-slices, row stride
// *Nv_out floats; the product's element (m, n) is the sum of its slices in slice order.
void launch_gemm_skinny_partials(hipStream_t st, const GemmArgs &a, float *partials, int *S_out, int *Nv_out);
// LM head (a.epi EPI_STORE) with the greedy choice begun in the epilogue: every wave writes the float32 logits of its
// tile, if wanted, and the best (value, column) of each row among its columns to cand_val / cand_idx [M][n_cand].
struct HeadOut {
    float *logits;       // [M][N] or nullptr
    float *cand_val;     // [M][n_cand]
    int32_t *cand_idx;
    int n_cand;
};
// Candidates per row of the pass for M rows, or 0 where the shape is not one the pass takes.
int head_candidates(int M, int N, int K);
void launch_gemm_head(hipStream_t st, const GemmArgs &a, const HeadOut &o);
size_t packed_weight_elems(int N, int K);
void launch_pack_weights(hipStream_t st, const bf16_t *W, bf16_t *Wp, int N, int K);

// ---- projections of a pass of few rows (decode_gemm.hip): weights streamed once, RMSNorm folded in ----
#define RS_STREAM_ROWS 128   // most rows of such a pass
#define RS_SSQ_ROWS RS_STREAM_ROWS   // row stride of the sums of squares below
struct DGemmArgs {
    const bf16_t *A_packed;   // activations fragment-packed (packed_mt(M) row tiles), or
    const bf16_t *X_rows;     // row-major [M][K] hidden state: multiplied by gain[K] on the way in, and
    const bf16_t *gain;       //   the sums of squares of each row over each K slice go to
    float *ssq_part;          //   ssq_part[slice][RS_SSQ_ROWS]  (the epilogue turns them into the RMSNorm scale)
    const bf16_t *Wp, *Wp2;   // fragment-packed weights [N][K]; Wp2: the up matrix of a gate/up pair
    float *part;              // out: float32 partial products [S][M][Nv]  (not for a pair)
    int M, N, K;
};
struct DFuseArgs {            // a gate/up pair: out = silu(s g) * (s u) with the row's RMSNorm scale s
    const float *ssq_part = nullptr;    // [S_ssq][RS_SSQ_ROWS] sums of squares of the parts of each row of K elements
    int S_ssq = 0;
    float eps = 0.f;
    bf16_t *out = nullptr;              // fragment-packed [M][N]
    const bf16_t *rows = nullptr;       // instead of ssq_part, up to RS_FEW_ROWS rows of RS_FEW_COLS: the rows [M][K] themselves
};
struct DGemmPlan {
    bool pair;
    int cols, S, kb_per_wg, Nv;   // workgroups along N, K slices, k-blocks per slice, row stride of the partial products
};
// True if the streaming kernel takes this projection (K a multiple of 256, N a multiple of 4 and at least 128).
bool dgemm_applies(int N, int K);
DGemmPlan dgemm_plan(int N, int K, bool pair);
size_t dgemm_partial_elems(int M, int N, int K);
// The stream: partial products of a plain projection, or a pair's finished output (f).
// narrow: half-height workgroups, twice as many (same sums, same bits); dgemm_prefers_half_height says when, from the
// number of compute units the side owns
void launch_dgemm_stream(hipStream_t st, const DGemmArgs &a, const DGemmPlan &p, const DFuseArgs &f, bool narrow);
bool dgemm_gains_inline(int M, const DGemmPlan &p);
void launch_gain_pack(hipStream_t st, const bf16_t *x, const bf16_t *gain, bf16_t *out, float *ssq_out, int M, int N);
bool dgemm_prefers_half_height(const DGemmPlan &p, int cus);
struct DEpiArgs {
    const float *part;        // [S][M][Nv]
    int S, Nv;
    const bf16_t *resid;      // row-major [M][N]
    bf16_t *out;              // row-major [M][N]
    int M, N;
    // or nullptr: the next RMSNorm's gain [N]; out . gain goes fragment-packed to out_gain and the sums of squares of
    // out's rows to ssq_out [ceil(N / 1024)][RS_SSQ_ROWS]
    const bf16_t *gain = nullptr;
    bf16_t *out_gain = nullptr;
    float *ssq_out = nullptr;
};
void launch_dgemm_epilogue(hipStream_t st, const DEpiArgs &a);
struct QkvEpiArgs {
    const float *part;        // [S][M][Nv] partial q | k | v
    const float *ssq_part;    // [S_ssq][RS_SSQ_ROWS]; S_ssq 0: the product's input was normalised already
    int S, S_ssq, Nv, d;
    float eps;
    bf16_t *qkv;              // out: [M][(Hq+2Hkv)*hd] with q and k rotated
    const CosSin *table;
    bf16_t *k_pool, *v_pool;  // this layer
    const int32_t *tables, *ctx_lens;   // of the decode rows [T, M)
    int32_t *err_flag;
    int M, Hq, Hkv, hd, max_blk, n_blocks, max_pos;
    // rows [0, T): prompts, delimited and placed by seq
    int T = 0;
    const int32_t *ptables = nullptr;
    int max_blk_p = 0;
    SeqInfo seq{};
};
void launch_qkv_rope_epilogue(hipStream_t st, const QkvEpiArgs &a);
// The projections of at most RS_FEW_ROWS rows, finished in one kernel: the bits of the stream and its epilogue.
#define RS_FEW_ROWS 4
#define RS_FEW_COLS 4096   // most columns of such rows
struct FewArgs {
    const bf16_t *A;          // fragment-packed activations, or (QKV)
    const bf16_t *X_rows;     // the rows [M][K], normalised with
    const bf16_t *gain;       //   this gain [K]; of a residual projection: the next RMSNorm's gain [N] or nullptr
    const bf16_t *Wp;
    int M, N, K, S;           // S: the plan's K slices
    float eps;
    const bf16_t *resid;      // row-major [M][N]
    bf16_t *out, *out_gain;   // resid + product, row-major; times the gain, fragment-packed
    int wave_slices = 0;      // of each wave; set by the launch
};
// Whether they are the faster (and take the projection: 2 to 16 K slices, N a multiple of 32, rows of at most RS_FEW_COLS columns).
bool few_takes_residual(int M, int N, int K, int cus);
bool few_takes_qkv(int M, int N, int K, int hd, int cus);
void launch_few_residual(hipStream_t st, FewArgs a, int cus);
void launch_few_qkv(hipStream_t st, FewArgs a, const QkvEpiArgs &q, int cus);   // rotated q | k | v and the cache write, as launch_qkv_rope_epilogue
// x1 = resid + the slices' sum (row-major) and h = RMSNorm(x1; gain) (fragment-packed), a row a workgroup.  Needs
// residual_norm_applies: rows of at most 8192, a multiple of 8.
struct ResidualNormArgs {
    const float *part;        // [S][M][N]
    int S;
    const bf16_t *resid, *gain;
    bf16_t *x1, *h;
    int M, N;
    float eps;
};
bool residual_norm_applies(int N);
void launch_residual_norm(hipStream_t st, const ResidualNormArgs &a);
void decode_gemm_kernels_init();

// Grouped GEMM over tiles that each belong to one expert: STORE or SWIGLU epilogue, a.M = the padded row capacity (a
// multiple of 128), a.expert_stride set and a.units the work list that moe_plan_kernel writes.  Needs K % 32 == 0 and
// N >= 1024.
bool launch_gemm_grouped(hipStream_t st, const GemmArgs &a);

// The grouped GEMM's order of tiles.  An XCD takes an eighth of them, counted column by column, so that every one has the same
// number of them and its share of every expert.  (Dealt in jobs of 4 units by 8 columns some XCDs had four jobs and others
// three, or three and two; 8 experts of the 8B widths, jobs / this: gate/up of 16 rows on 64 CUs 923 / 820 us and on 128 532 /
// 492, down of 4000 rows on 64 CUs 2872 / 2194, gate/up of 300 rows of which most share an expert on 256 CUs 483 / 395.)
// An XCD's whole columns go in blocks of 8, four units (neighbours in the list, mostly of one expert) at a time: 32 tiles in
// flight then read 4 activation slabs and, with two units an expert, 16 weight slabs, where all units of one column
// after another read 16 and 32 for as many tiles.
#define RS_GROUP_UNITS 4
#define RS_GROUP_COLS 8
struct GroupTile { int u, nb; };   // unit, column tile
// The i-th tile (0 <= i) of XCD x, or u = -1 past its share.
__host__ __device__ inline GroupTile grouped_tile(int x, int i, int nu, int n_tiles) {
    const int total = nu * n_tiles, per = (total + 7) >> 3;
    const int first = x * per, end = first + per < total ? first + per : total;
    if (i >= end - first) return {-1, 0};
    const int col0 = (first + nu - 1) / nu, col1 = end / nu;   // its whole columns [col0, col1)
    const int t = first + i, j = t - col0 * nu;
    if (j < 0 || t >= col1 * nu) return {t % nu, t / nu};      // of a column shared with a neighbour
    const int block = j / (RS_GROUP_COLS * nu), c0 = col0 + block * RS_GROUP_COLS, cols = col1 - c0 < RS_GROUP_COLS ? col1 - c0 : RS_GROUP_COLS;
    const int r = j - block * (RS_GROUP_COLS * nu), g = r / (RS_GROUP_UNITS * cols);
    const int units = nu - g * RS_GROUP_UNITS < RS_GROUP_UNITS ? nu - g * RS_GROUP_UNITS : RS_GROUP_UNITS, v = r - g * (RS_GROUP_UNITS * cols);
    return {g * RS_GROUP_UNITS + v % units, c0 + v / units};
}

// Whether the down projection's tiles are 128 columns wide instead of 256: where all of them then run at once, on twice as many CUs.
// What bounds them is what a CU loads, 57 GB/s however deep the ring (from HBM and L2 alike: the times of the two add up); 8
// experts of one unit each leave half of 256 CUs idle with 256 columns.  Down of the 8B widths through 8 experts on 256 CUs,
// 256 / 128 columns: 64 rows 223 / 154 us, 256 rows 222 / 171, 600 rows 252 / 201, 900 rows 343 / 237.
static __host__ __device__ inline bool grouped_narrow(bool store, int nu, int n_tiles, int cus) { return store && 2 * nu * n_tiles <= cus; }

// The i-th workgroup of XCD x: first the XCD's tiles of the tall units, then those of the others; where its last round is of tiles for no more than
// half of its compute units, those are cut in two (half 0, 1; -1: a whole tile).
struct GroupPiece { int i, half; bool tall; };
__host__ __device__ inline int grouped_share(int x, int total) {
    const int per = (total + 7) >> 3, first = x * per;
    return first >= total ? 0 : (first + per < total ? per : total - first);
}
__host__ __device__ inline GroupPiece grouped_piece(int x, int i, int nu_tall, int nu_low, int n_tiles, int cus) {
    const int n0 = grouped_share(x, nu_tall * n_tiles), n = n0 + grouped_share(x, nu_low * n_tiles);
    const int units = cus >> 3, rest = n % units, whole = 2 * rest <= units && n > rest ? n - rest : n;
    int half = -1;
    if (i >= whole) {
        if (whole == n) return {n, -1, false};
        half = (i - whole) & 1;
        i = whole + ((i - whole) >> 1);
    }
    return i < n0 ? GroupPiece{i, half, true} : GroupPiece{i - n0, half, false};
}
// What the i-th workgroup of XCD x computes in the eight-wave kernel: column tile nb of unit u (-1: nothing), nb counted in whole tiles (256
// columns of the down projection, 128 of gate and up) or, if half, in tiles of half as many.
struct GroupTallTile { int u, nb; bool half; };
__host__ __device__ inline GroupTallTile grouped_tall_tile(int x, int i, int nu_tall, int nu, int N, bool store, int cus) {
    const int n_tiles = store ? (N + 255) / 256 : (N + 127) / 128;
    if (grouped_narrow(store, nu, n_tiles, cus)) {
        // all run at once, so the tall units need not come first, and there is no last round to cut: dealt apart, their share of an
        // XCD and the others', each rounded up, can be one tile more than it has compute units
        const GroupTile t = grouped_tile(x, i, nu, (N + 127) / 128);
        return {t.u, t.nb, true};
    }
    const GroupPiece p = grouped_piece(x, i, nu_tall, nu - nu_tall, n_tiles, cus);
    const GroupTile t = grouped_tile(x, p.i, p.tall ? nu_tall : nu - nu_tall, n_tiles);
    if (t.u < 0) return {-1, 0, false};
    return {p.tall ? t.u : t.u + nu_tall, p.half >= 0 ? 2 * t.nb + p.half : t.nb, p.half >= 0};
}
// Its workgroups, where there can be `units` units: their tiles and the second halves of a last round; narrow tiles are no more than CUs.
static inline int grouped_tall_grid(int units, int n_tiles, int cus) {
    const int most = units * n_tiles + cus / 2;
    return ((most > cus ? most : cus) + 7) / 8 * 8 + 8;
}

#define RS_MOE_MAX_EXPERTS 16
// Whether the grouped GEMM fetches the weights as a stream (non-temporal): `rows` rows go to two of E experts each, and where an expert
// has one tile or two on average (at most 512 rows) they run at once and nobody reads its weights again.  The layer of the 8B widths,
// not streamed / streamed: decode of 64 rows through 2, 4, 16 experts 369 / 355, 472 / 451, 1154 / 1096 us; prefill through 2 experts
// of 300, 500, 900, 1500 rows 456 / 443, 582 / 574, 823 / 825, 1134 / 1155; through 4 of 600, 1000, 1500 rows 659 / 639, 893 / 889,
// 1178 / 1180; through 8 of 900, 1100, 1500, 2048 rows 971 / 952, 1018 / 1011, 1224 / 1212, 1707 / 1710, of 3000 2322 / 2359; through 16
// of 600, 1500, 2500, 3000 rows 1191 / 1121, 1461 / 1424, 2124 / 2104, 2474 / 2457.
static inline bool grouped_streams_weights(int rows, int E) { return rows <= 256 * E; }
// How the experts' rows are cut into units: `limit` rows at most, and whether by the kernel of eight waves, which alone takes more than 256.
// An expert has `rows` rows in E to two of them; its share and a deviation above it is what the fullest are taken to have.  On more than 128 CUs
// taller tiles are worth it where fewer of them hold that, but three of 288 are 1 % slower than four of 224 rows; where their number stays the
// same the four-wave tiles are 2 % faster on 256 CUs (LDS traffic).  On 128 and fewer, where the loads of a CU count for more, eight waves are the
// faster from 256 rows on.  Prefill through 8 experts of the 8B widths, us, units of 256 rows by four waves / of 320 by eight ("-": not taken; on 128 CUs
// those go by eight waves in units of 256):
//            950 rows      1000        1100       1250         1500         2048         2400         3300         4000
//   256 CUs  827 / 818 -   890 / 843   1022 / 906 1012 / 1030 - 1142 / 1147 - 1590 / 1437 1850 / 1644 2291 / 2330 - 2837 / 2702
//   192 CUs  925 / 927 -   995 / 951   1247 / 1017 1247 / 1103 - 1381 / 1322 - 1778 / 1662 1985 / 1914 2670 / 2579 - 3156 / 3124
//   128 CUs  1058 / 1052 - 1324 / 1079 1507 / 1134 1494 / 1328 - 1643 / 1621 - 2322 / 1960 2586 / 2235 3369 / 3168   4074 / 3793
// (So the line of 256 CUs is not that of 160 to 224, nor is a deviation above the share always the fullest.  Half of the rows on one of the experts,
// which no rule on the host sees: 2400 rows on 192 CUs 1840 / 1894, 1000 to 4000 rows otherwise 0.91 to 1.01.)
// Not where the lower tiles of the down projection, 128 columns wide, leave CUs idle as it is: fewer and taller ones leave half of what works.
// With all but an eighth of the CUs at work they do that for what a taller tile saves only if the projection is long (f) and nearly every expert
// fills its lower tiles.  The same pair, of E experts of `mean` rows:
//   256 CUs: E 8, 290 rows, d 1024, f 14336 367 / 428;  E 4, 290, d 2816, f 4096 196 / 231;  E 4, 290, d 2048, f 8192 237 / 271
//            E 4, d 4096, f 14336: 266 rows 568 / 542 (taken), 275 539 / 558, 300 553 / 582;  E 16, 290, d 1024, f 3584 277 / 256 (taken)
//   128 CUs: E 4, 290 rows, d 2048, f 8192 293 / 306;  E 4, 290, d 1024, f 3584 147 / 158
struct GroupCut { int limit; bool tall; };
static inline GroupCut grouped_cut(int rows, int E, int d, int f, int cus) {
    if (cus <= 0) cus = 256;
    const double mean = 2.0 * rows / E, dev = __builtin_sqrt(mean);
    const int of320 = (int)__builtin_ceil((mean + dev) / 320), of256 = (int)__builtin_ceil((mean + dev) / 256), low = E * of256 * ((d + 127) / 128);
    const bool idle = 8 * low <= 7 * cus || (low <= cus && f >= 8192 && mean - dev > 256 * (of256 - 1));
    const bool fewer = of320 < of256 && !idle;
    if (cus <= 128) return {fewer ? 320 : 256, of256 > 1};
    return fewer && of320 != 3 ? GroupCut{320, true} : GroupCut{256, false};
}
// Rows of the grouped (expert-major) layout that M rows with two experts each can need: an expert's segment is less than
// 256 rows longer than its rows.
static inline int moe_row_cap(int M, int E) { return ((2 * M + 255 * E + 127) / 128) * 128; }
struct MoeArgs {
    const bf16_t *h;        // normalised rows, fragment-packed with packed_mt(M) row tiles
    const bf16_t *router;   // [E][d] row-major
    int32_t *sel;           // [M][2] experts of each row
    float *wt;              // [M][2] their weights
    int32_t *pos;           // [M][2] grouped row of each assignment
    int32_t *src;           // [Mg_cap] source row of each grouped row, -1 for padding
    int32_t *units;         // [2 + Mg_cap / 128]: units of more than 256 rows << 16 | units, rows in use, first row / 32 << 13 | 32-row blocks with rows << 9 | height / 32 << 5 | expert of each
    bf16_t *a_g;            // gathered rows, fragment-packed with Mg_cap / 32 row tiles
    const bf16_t *out_g;    // [Mg_cap][d] expert outputs, row-major
    const bf16_t *x1;       // [M][d]
    bf16_t *y;              // [M][d]
    int M, d, E, Mg_cap;
    int limit;              // rows of a unit at most: 256 or 320 (grouped_cut)
};
void launch_moe_route_and_gather(hipStream_t st, const MoeArgs &a);
void launch_moe_combine(hipStream_t st, const MoeArgs &a);

struct EmbedArgs {
    const int32_t *tokens;     // [n], or per-slot tokens when row_slot is given, or slot regions when slots is given
    const int32_t *row_slot;   // [n] or nullptr
    const bf16_t *table;       // [vocab][d]
    bf16_t *x;                 // [n][d] row-major
    int32_t *err_flag;
    int n, d, vocab;
    // several prompts (or a chunk of each, from position seq.start[q]) in one call: row r of prompt q (seq.cu
    // delimits them) is token tokens[slots[q] * slot_stride + seq.start[q] + (r - seq.cu[q])]
    const int32_t *slots = nullptr;
    int slot_stride = 0;
    SeqInfo seq{};
};
void launch_embed(hipStream_t st, const EmbedArgs &a);
// out[q][:] = x[seq.cu[q+1] - 1][:]: the last row of each prompt, for the LM head.
void launch_gather_last_rows(hipStream_t st, const bf16_t *x, bf16_t *out, int d, const SeqInfo &seq);

struct HeadArgmaxArgs {
    const float *part;         // [S][M][Nv] partial logits
    float *logits;             // [M][N] or nullptr
    int32_t *tokens;           // [M] or nullptr
    const int32_t *row_slot;   // [M] or nullptr
    int32_t *tok_by_slot;      // scattered copy of the tokens, or nullptr
    int S, M, N, Nv;
};
void launch_head_argmax(hipStream_t st, const HeadArgmaxArgs &a);
// The same choice over the candidates that launch_gemm_head left.
struct HeadPickArgs {
    const float *cand_val;
    const int32_t *cand_idx;
    int32_t *tokens;
    const int32_t *row_slot;
    int32_t *tok_by_slot;
    int M, n_cand;
};
void launch_head_pick(hipStream_t st, const HeadPickArgs &a);

// Counts workgroups per physical CU: hist[(xcc << 8) | (se << 5) | (sh << 4) | cu] += 1.
void launch_cu_probe(hipStream_t st, int32_t *hist, int n_workgroups);

// Reads `bytes` (multiple of 16) once with coalesced 16-byte loads.
void launch_stream_read(hipStream_t st, const void *src, size_t bytes, int n_workgroups);

// Back-to-back register-only 32x32x16 bf16 MFMAs; returns the flops the launch performs.
double launch_mfma_probe(hipStream_t st, float *sink, int n_workgroups, int iters);

void launch_noop(hipStream_t st);

// Zeroes `bytes` (a multiple of 16) of device memory with a kernel (usable under stream capture).
void launch_fill_zero(hipStream_t st, void *dst, size_t bytes);

// Called once per context creation (see gemm.hip).
void gemm_kernels_init();
void grouped_kernels_init();
void attention_kernels_init();

