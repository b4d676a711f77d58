// Host-side check of the rules by which passes take their kernels (no GPU call), at sizes where both sides were measured
// and at those where tests compare the two.  Built against the library and run by tests/test_host_abi.py.
#include <algorithm>
#include <cstdio>
#include <utility>
#include <vector>

#include "../paper_2601_11822_amd/csrc/kernels.h"

static int fails = 0;
#define CHECK(c, ...) do { if (!(c)) { if (fails++ < 10) { std::printf("FAIL %s:%d: ", __FILE__, __LINE__); std::printf(__VA_ARGS__); std::printf("\n"); } } } while (0)

static void few_rows() {
    // one to four rows of the 8B widths: on the whole chip all three projections in one kernel each; on 96 compute units, which no
    // number of tiles a workgroup fills, the residual ones streamed; the long down projection streamed on every partition
    struct { int cus; bool q, o, d; } of8b[] = {{256, true, true, true}, {224, true, true, false}, {192, true, true, false}, {160, true, true, false},
                                                {128, true, true, false}, {96, true, false, false}, {64, true, true, false}, {32, true, true, false}};
    for (auto &w : of8b)
        for (int M = 1; M <= 5; ++M) {
            CHECK(few_takes_qkv(M, 6144, 4096, 128, w.cus) == (w.q && M <= 4), "QKV of %d rows on %d", M, w.cus);
            CHECK(few_takes_residual(M, 4096, 4096, w.cus) == (w.o && M <= 4), "output of %d rows on %d", M, w.cus);
            CHECK(few_takes_residual(M, 4096, 14336, w.cus) == (w.d && M <= 4), "down of %d rows on %d", M, w.cus);
        }
    // narrower: streamed where a compute unit would have more to load
    CHECK(!few_takes_residual(1, 3072, 8192, 64) && few_takes_residual(1, 3072, 8192, 128), "down of 3072 columns");
    CHECK(!few_takes_residual(1, 3072, 3072, 160) && few_takes_residual(1, 3072, 3072, 192), "output of 3072 columns");
    CHECK(!few_takes_residual(1, 2560, 10240, 64) && few_takes_residual(1, 2560, 10240, 192), "down of 2560 columns");
    CHECK(!few_takes_qkv(1, 4608, 3584, 128, 64) && few_takes_qkv(1, 4608, 3584, 128, 192), "QKV of 3584 columns");
    // two or three slices: where a workgroup a tile is one round
    CHECK(few_takes_residual(1, 3584, 18944, 256) && !few_takes_residual(1, 3584, 18944, 192), "down of 3584 columns");
    CHECK(few_takes_residual(1, 1024, 1024, 64) && !few_takes_residual(1, 1024, 1024, 32) && few_takes_qkv(1, 1536, 1024, 64, 48) && !few_takes_qkv(1, 1536, 1024, 64, 32), "1024 columns");
    // what the kernels cannot take: one slice, wider rows, columns off the grid
    CHECK(!few_takes_residual(1, 1024, 2816, 256), "down of 1024 columns");
    CHECK(!few_takes_residual(1, 8192, 8192, 256) && !few_takes_qkv(1, 10240, 8192, 128, 256), "8192 columns");
    CHECK(!few_takes_residual(1, 2064, 4096, 256), "2064 columns");
    // the sizes at which the GPU tests compare both
    CHECK(few_takes_qkv(1, 3072, 2048, 64, 256) && few_takes_residual(1, 2048, 2048, 256) && few_takes_residual(1, 2048, 4608, 64), "2048 columns");
}

// The form of hybrid attention: prompts of `lens` rows behind `starts` tokens, B decode rows of at most max_ctx tokens (all of them n_keys)
struct Heads { int Hq, Hkv, hd; };
static HybridForm form_of(Heads h, std::vector<int> lens, std::vector<int> starts, int B, int max_ctx, int64_t n_keys, int cus) {
    static float park;
    PrefillAttnArgs p{};
    p.Hq = h.Hq, p.Hkv = h.Hkv, p.hd = h.hd, p.cus = cus, p.park = &park, p.park_cap = (size_t)1 << 40;
    p.seq.n_req = (int)lens.size();
    for (size_t r = 0; r < lens.size(); ++r) p.seq.cu[r + 1] = p.seq.cu[r] + lens[r], p.seq.start[r] = starts[r];
    DecodeAttnArgs d{};
    d.B = B, d.Hq = h.Hq, d.Hkv = h.Hkv, d.hd = h.hd, d.max_ctx = max_ctx, d.n_chunks = (max_ctx + RS_DECODE_CHUNK - 1) / RS_DECODE_CHUNK, d.n_keys = n_keys;
    return hybrid_form(p, d);
}

static void hybrid_forms() {
    const Heads of8b{32, 8, 128}, mid{8, 2, 128}, odd{9, 3, 128}, tiny{4, 4, 64};
    // 512 rows of the 8B heads: small workgroups where the decode rows are read for longer than the longest prompt tile takes
    CHECK(form_of(of8b, {512}, {1024}, 64, 4097, 0, 256) == HYBRID_SMALL, "64 rows of up to 4096");
    CHECK(form_of(of8b, {512}, {3072}, 16, 601, 0, 256) == HYBRID_TEAMS, "16 rows of up to 600");
    CHECK(form_of(of8b, {512}, {1024}, 32, 2001, 0, 256) == HYBRID_TEAMS, "32 rows of up to 2000");
    CHECK(form_of(of8b, {512}, {1024}, 64, 4097, 0, 128) == HYBRID_APART, "a partition");
    // by the tokens themselves where they are known: one long context among short ones is not 64 long ones, and many long ones are more than half
    CHECK(form_of(of8b, {512}, {1024}, 64, 4097, 4097 + 63 * 300, 256) == HYBRID_TEAMS, "63 rows of 300 beside one of 4096");
    CHECK(form_of(of8b, {512}, {1024}, 64, 3001, 64 * 3001, 256) == HYBRID_SMALL, "64 rows of 3000");
    CHECK(form_of(of8b, {512}, {1536}, 64, 4097, 0, 256) == HYBRID_SMALL && form_of(of8b, {512}, {1536}, 64, 4097, 64 * 1000, 256) == HYBRID_TEAMS, "bound and tokens");
    // the sizes at which a GPU test compares the forms
    struct { Heads h; std::vector<int> lens, starts; int B; } tests[] = {{mid, {90}, {16}, 40}, {odd, {200, 31}, {0, 48}, 50}, {tiny, {140, 1}, {32, 0}, 50}};
    for (auto &t : tests) {
        CHECK(form_of(t.h, t.lens, t.starts, t.B, 301, 0, 256) == HYBRID_TEAMS, "%d rows of up to 300", t.B);
        CHECK(form_of(t.h, t.lens, t.starts, t.B, 2600, 0, 256) == HYBRID_SMALL, "%d rows of up to 2600", t.B);
    }
    for (int cus : {256, 128, 64}) CHECK(form_of(mid, {16}, {0}, 60, 301, 0, cus) == HYBRID_SMALL, "one chunk on %d", cus);
    CHECK(form_of(mid, {16}, {0}, 2, 301, 0, 256) == HYBRID_TEAMS, "2 rows of one chunk");
}

// Large tiles of an odd number of 32-row blocks: each of the passes that a GPU test repeats for their sake has a product in them
static void odd_heights() {
    const struct { int M, cus; } passes[] = {{576, 256}, {300, 256}, {1120, 128}, {650, 96}};
    const int N[] = {6144, 4096, 4096}, K[] = {4096, 4096, 14336};   // QKV, output, down of the 8B widths; gate/up below
    auto odd = [](DirectForm f) { return f == FORM_160x256 || f == FORM_224x256; };
    for (auto &p : passes) {
        bool any = odd(direct_form(p.M, 14336, 4096, EPI_SWIGLU, 1, p.cus));
        for (int j = 0; j < 3; ++j) {
            const int S = direct_splits(p.M, N[j], K[j]);
            any = any || odd(direct_form(p.M, N[j], K[j], S > 1 || j == 0 ? EPI_STORE : EPI_RESIDUAL, S, p.cus));
        }
        CHECK(any, "%d rows on %d compute units have no tile of 160 or 224 rows", p.M, p.cus);
    }
}

// Every kind of product in tiles of 288 and 320 rows and, of 128, in the fed form, that GPU tests are about: on one of the partitions that they run, is it chosen?
struct Widths { int d, qkv, q, f; };
enum Kind { GATE_UP, STORED, RESIDUAL, SLICED };
struct Wanted { Kind kind; DirectForm form; int rows_over; bool streamed; int nk; };   // rows_over: in the last tile (0: full); streamed: of whole products; nk: K tiles (0: any)
static void forms_of(const char *what, std::vector<std::pair<Widths, std::vector<int>>> passes, std::vector<Wanted> wanted) {
    for (auto &w : wanted) {
        const int bm = w.form == FORM_320x256 ? 320 : w.form == FORM_288x256 ? 288 : 128;
        bool any = false;
        for (auto &p : passes)
            for (int M : p.second)
                for (int cus : {256, 128, 64, 96}) {
                    const Widths &s = p.first;
                    const struct { Kind kind; int N, K; } products[] = {{GATE_UP, s.f, s.d}, {STORED, s.qkv, s.d}, {RESIDUAL, s.d, s.q}, {RESIDUAL, s.d, s.f}};
                    for (auto &q : products) {
                        if (q.N < 1024) continue;
                        const int S = q.kind == GATE_UP ? 1 : direct_splits(M, q.N, q.K), tiles = (M + bm - 1) / bm;
                        const DirectForm f = direct_form(M, q.N, q.K, S > 1 || q.kind == STORED ? EPI_STORE : q.kind == GATE_UP ? EPI_SWIGLU : EPI_RESIDUAL, S, cus);
                        any = any || (f == w.form && (S > 1 ? SLICED : q.kind) == w.kind && M % bm == w.rows_over && (!w.nk || q.K / 32 == w.nk) &&
                                      (S > 1 || direct_streams(tiles, cus) == w.streamed));
                    }
                }
        CHECK(any, "%s: kind %d, form %d, %d rows over, streamed %d, %d K tiles", what, w.kind, w.form, w.rows_over, w.streamed, w.nk);
    }
}
static void tall_and_fed_forms() {
    const Widths of8b{4096, 6144, 4096, 14336}, of70b{8192, 10240, 8192, 28672}, odd{1152, 1920, 1152, 3104};
    forms_of("tall", {{of8b, {288, 320, 640, 832, 1280, 1600, 1800}}, {of70b, {290, 1100}}, {odd, {310, 640, 2593, 2881, 3169, 3521}}},
             {{GATE_UP, FORM_288x256, 0, true, 0}, {GATE_UP, FORM_320x256, 0, true, 0}, {GATE_UP, FORM_288x256, 1, false, 0}, {GATE_UP, FORM_320x256, 1, false, 0},
              {SLICED, FORM_288x256, 0, true, 0}, {SLICED, FORM_320x256, 0, true, 0}, {SLICED, FORM_320x256, 290, true, 0}, {SLICED, FORM_288x256, 256, true, 0},
              {STORED, FORM_320x256, 0, true, 0}, {STORED, FORM_320x256, 0, false, 0}, {STORED, FORM_288x256, 1, false, 36}, {STORED, FORM_320x256, 1, false, 36},
              {RESIDUAL, FORM_288x256, 236, true, 0}, {RESIDUAL, FORM_320x256, 0, true, 0}, {RESIDUAL, FORM_288x256, 1, false, 97}, {RESIDUAL, FORM_320x256, 1, false, 97}});
    // fed: fewer K tiles than the ring has stages, an odd number of them, one row tile and many
    const Widths one_head{1024, 384, 128, 1056}, odd_k{1056, 1280, 1024, 1120}, narrow{160, 1280, 1024, 1024};
    forms_of("fed", {{one_head, {128, 129, 500, 641, 897}}, {odd_k, {897, 1300, 1500}}, {narrow, {128, 129, 400, 641}}, {of8b, {1537}}},
             {{RESIDUAL, FORM_128x256, 0, true, 4}, {RESIDUAL, FORM_128x256, 1, true, 4}, {RESIDUAL, FORM_128x256, 1, false, 4}, {RESIDUAL, FORM_128x256, 1, false, 33},
              {RESIDUAL, FORM_128x256, 20, false, 35}, {STORED, FORM_128x256, 1, false, 33}, {STORED, FORM_128x256, 0, true, 5}, {STORED, FORM_128x256, 1, true, 5},
              {STORED, FORM_128x256, 1, false, 5}, {RESIDUAL, FORM_128x256, 1, false, 448}});
    // the passes that are repeated: fed on the whole chip
    for (int K : {4096, 14336}) CHECK(direct_splits(1536, 4096, K) == 1 && direct_form(1536, 4096, K, EPI_RESIDUAL, 1, 256) == FORM_128x256, "1536 rows, K %d", K);
}

// Weights as a stream: only where a column's row tiles run side by side (three of them do not on 32 or 64 units, where an XCD runs four or eight tiles at a time)
static void streamed_weights() {
    for (int cus = 32; cus <= 256; cus += 32)
        for (int m_tiles = 1; m_tiles <= 8; ++m_tiles)
            CHECK(direct_streams(m_tiles, cus) == (m_tiles <= 4 && !(m_tiles == 3 && cus <= 64)), "%d row tiles on %d", m_tiles, cus);
}

// The experts' down projection: of up to 8 units 4 (1024 columns) tiles each, narrow on the whole chip, not on 32 units
static void expert_tiles() {
    for (int nu = 1; nu <= 64; ++nu)
        for (int cus : {32, 64, 128, 256}) {
            CHECK(grouped_narrow(true, nu, 4, cus) == (8 * nu <= cus), "%d units on %d", nu, cus);
            CHECK(!grouped_narrow(false, nu, 4, cus), "gate/up");
        }
}

// Eight-wave expert tiles: the launched workgroups have each column of each unit once, whatever the units, the width and the partition.
// `cells` are as many columns as half a tile has.
static void expert_pieces() {
    std::vector<unsigned char> seen;
    for (bool store : {true, false})
        for (int N = 1024; N <= 8192; N += store ? 128 : 640)
            for (int cus = 32; cus <= 256; cus += 32)
                for (int nu = 1; nu <= 24; ++nu)
                    for (int tall = 0; tall <= nu; ++tall) {
                        const int n_tiles = store ? (N + 255) / 256 : (N + 127) / 128, cells = store ? (N + 127) / 128 : (N + 63) / 64;
                        const int grid = grouped_tall_grid(nu, n_tiles, cus);   // no unit is lower than 128 rows
                        seen.assign((size_t)nu * cells, 0);
                        bool inside = true;
                        for (int id = 0; id < grid; ++id) {
                            const GroupTallTile t = grouped_tall_tile(id & 7, id >> 3, tall, nu, N, store, cus);
                            if (t.u < 0) continue;
                            inside = inside && t.u < nu && t.nb >= 0 && t.nb < (t.half ? 2 : 1) * n_tiles;
                            for (int c = t.half ? t.nb : 2 * t.nb; inside && c < (t.half ? t.nb + 1 : 2 * t.nb + 2); ++c)
                                if (c < cells) ++seen[(size_t)t.u * cells + c];
                        }
                        const bool once = std::all_of(seen.begin(), seen.end(), [](unsigned char v) { return v == 1; });
                        CHECK(inside && once, "%s: %d tall of %d units, %d columns on %d", store ? "down" : "gate/up", tall, nu, N, cus);
                    }
    // the kernel and the limit, where both were measured: 8 experts
    struct { int rows, cus, limit; bool tall; } of8[] = {{64, 256, 256, false}, {950, 256, 256, false}, {1000, 256, 320, true}, {1100, 256, 320, true}, {1250, 256, 256, false},
                                                         {1900, 256, 256, false}, {2048, 256, 320, true}, {3300, 256, 256, false}, {4000, 256, 320, true},
                                                         {900, 128, 256, false}, {1000, 128, 320, true}, {1300, 128, 256, true}, {3300, 128, 320, true}};
    for (auto &w : of8) {
        const GroupCut c = grouped_cut(w.rows, 8, 4096, 14336, w.cus);
        CHECK(c.limit == w.limit && c.tall == w.tall, "%d rows on %d: %d %d", w.rows, w.cus, c.limit, c.tall);
    }
    // where a lower down projection leaves compute units idle, and where it nearly does: experts of `mean` rows, of other widths
    struct { int mean, E, d, f, cus, limit; bool tall; } others[] = {
        {290, 8, 1024, 14336, 256, 256, false}, {270, 8, 1024, 14336, 224, 256, false}, {290, 4, 1024, 3584, 160, 256, false}, {600, 4, 2048, 8192, 256, 256, false}, {290, 4, 2816, 4096, 256, 256, false},
        {290, 4, 2048, 8192, 192, 256, false}, {290, 2, 4096, 14336, 192, 256, false}, {250, 4, 4096, 14336, 256, 320, true}, {266, 4, 4096, 14336, 256, 320, true}, {276, 4, 4096, 14336, 256, 256, false}, {300, 4, 4096, 14336, 256, 256, false},
        {300, 4, 4096, 14336, 224, 320, true}, {600, 4, 4096, 14336, 256, 320, true}, {290, 16, 1024, 3584, 256, 320, true}, {270, 8, 2048, 8192, 256, 320, true}, {290, 8, 2048, 8192, 256, 256, false}, {290, 8, 2048, 8192, 192, 320, true},
        {290, 8, 2816, 4096, 256, 320, true}, {290, 4, 2048, 8192, 128, 256, true}, {290, 4, 1024, 3584, 128, 256, true}, {290, 4, 2048, 8192, 96, 320, true}, {290, 4, 1024, 3584, 64, 320, true}, {600, 4, 2048, 8192, 128, 320, true}};
    for (auto &w : others) {
        const GroupCut c = grouped_cut(w.mean * w.E / 2, w.E, w.d, w.f, w.cus);
        CHECK(c.limit == w.limit && c.tall == w.tall, "%d experts of %d rows, %d x %d, on %d: %d %d", w.E, w.mean, w.d, w.f, w.cus, c.limit, c.tall);
    }
    // the GPU tests of units of up to 320 rows, down projection 128 columns wide or 256
    for (int E : {3, 7}) CHECK(grouped_cut(E == 3 ? 450 : 1000, E, 1024, 2816, 32).limit == 320 && !grouped_narrow(true, E, 4, 32) == (E == 7), "%d experts on 32", E);
    CHECK(grouped_cut(1000, 7, 1024, 2816, 64).limit == 320 && grouped_narrow(true, 7, 4, 64), "7 experts on 64");
    struct { int d, T, E, cus; } of128[] = {{1280, 380, 3, 32}, {1280, 400, 3, 32}, {1536, 1000, 8, 96}, {1536, 1060, 8, 96}, {3584, 1040, 8, 224}};
    for (auto &w : of128) CHECK(grouped_cut(w.T, w.E, w.d, 1024, w.cus).limit == 320, "%d rows, width %d on %d", w.T, w.d, w.cus);
}

int main() {
    expert_pieces();
    few_rows();
    hybrid_forms();
    odd_heights();
    tall_and_fed_forms();
    streamed_weights();
    expert_tiles();
    if (fails) { std::printf("%d checks failed\n", fails); return 1; }
    std::printf("dispatch ok\n");
    return 0;
}
