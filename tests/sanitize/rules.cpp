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
    std::printf("rules ok\n");
    return 0;
}
