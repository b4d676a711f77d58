// Host-side check of the rules by which passes take their kernels (no GPU call), at sizes where both sides were measured
// and at those where tests compare the two.  Built against the library and run by tests/test_host_abi.py.
#include <cstdio>

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

int main() {
    few_rows();
    if (fails) { std::printf("%d checks failed\n", fails); return 1; }
    std::printf("dispatch ok\n");
    return 0;
}
