// The rules that choose a launch's form (ddp_plan.h), on both sides of their lines, for 256 compute units.
#include <cstdio>
#include <cstdlib>

#include "ddp_plan.h"

#define CHECK(cond)                                                                       \
    do {                                                                                  \
        if (!(cond)) {                                                                    \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
            std::exit(1);                                                                 \
        }                                                                                 \
    } while (0)

using namespace ddp;

int main() {
    // two vectors per thread in flight: bf16 peers, a kernel laid out for 16 or 32 replicas, two vectors for each of 256 threads,
    // three scheduled chunks per CU in a call on 4.5
    for (int N = 1; N <= DDP_MAX_REPLICAS; ++N) {
        const int64_t many = 1 << 30;
        CHECK(takes_pairs(256, 2048, 1152, 768, N, true) == (N >= 9 && N <= 32) && takes_pairs(256, 1 << 20, many, many, N, true) == (N >= 9 && N <= 32));
        CHECK(!takes_pairs(256, 2048, 1151, 768, N, true) && !takes_pairs(256, 2048, many, 767, N, true));
        CHECK(!takes_pairs(256, 1024, many, many, N, true) && !takes_pairs(256, 2048, many, many, N, false));
    }
    // every average that is cut finds two pairs a chunk in its context's scratch; slots that are never cut have one
    for (int64_t n : {1, 100, 319, 320, 321, 384, 385, 2048, 100000, 520000, 524288, 600000})
        for (int64_t layers : {1, 32, 100})
            for (int N = 1; N <= DDP_MAX_REPLICAS; ++N)
                for (bool wire16 : {false, true}) CHECK(!mean_cut(256, 2048, n, layers, N, wire16) || mean_pairs(256, 2048, n, layers) == 2);
    CHECK(mean_pairs(256, 2048, 524288 - 32, 1) == 2 && mean_pairs(256, 2048, 524288 - 31, 1) == 1);
    // statistics folded into the launch: 5/4 workgroups per CU with a pair, as many pairs in a layer as it has counters for
    CHECK(folds(256, 1, 1) && folds(256, 320, 1) && folds(256, 320, 320) && !folds(256, 321, 1) && folds(304, 380, 320) && !folds(304, 321, 321));
    // chunks of the average cut in two: 12 to 16 fp32 replicas over small slots; 17 to 31 over small and large ones, with a bf16 wire
    // and from 32 replicas over all; none above 32
    for (int N = 1; N <= DDP_MAX_REPLICAS; ++N) {
        const bool few = N >= 12 && N <= 16, many = N >= 17 && N <= 32;
        for (int64_t n : {1, 320, 321, 384, 385, 2047, 2048}) {
            CHECK(mean_cut(256, 2048, n, 4, N, true) == (many ? 1024 : 0));
            const bool line = few ? n <= 320 : many && (N == 32 || n <= 384 || n >= 2048);
            CHECK(mean_cut(256, 2048, n, 4, N, false) == (line ? 1024 : 0));
        }
    }
    CHECK(mean_cut(256, 4096, 1, 4, 16, false) == 2048);
    // small models: 4.5 chunks of 2048 per CU, without a second moment more than 5/4; short AdamW updates: 7/4
    const int64_t lo = 320 * 2048, hi = 1152 * 2048, sh = 448 * 2048;
    CHECK(small_model(256, 1, true) && small_model(256, hi, true) && !small_model(256, hi + 1, true));
    CHECK(!small_model(256, 1, false) && !small_model(256, lo, false) && small_model(256, lo + 1, false) && small_model(256, hi, false) && !small_model(256, hi + 1, false));
    CHECK(short_update(256, 1, true) && short_update(256, sh, true) && !short_update(256, sh + 1, true) && !short_update(256, 1, false));
    std::printf("rules ok\n");
    return 0;
}
