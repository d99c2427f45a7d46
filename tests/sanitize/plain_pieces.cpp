// The plan of the fused step over dense arenas where a workgroup of an unscheduled piece takes several chunks: random models, whole
// and clipped to ranges of layers; every element belongs to one piece and every launch is wide enough for what the kernel makes of
// its pieces.  And the rules of the fused step's shape on both sides of their lines, for 256 compute units.
#include <cstdio>
#include <cstdlib>
#include <random>

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
    std::mt19937_64 rng(5);
    auto pick = [&](int64_t lo, int64_t hi) { return lo + (int64_t)(rng() % (uint64_t)(hi - lo + 1)); };
    long calls = 0;
    for (int r = 0; r < 500; ++r) {
        const int64_t chunk = 1024, plain = pick(1, 3);
        const int L = (int)pick(1, 30), keep = (int)pick(0, 4);
        SlotTables st;
        std::vector<int64_t> e(1, 0), wg(1, 0);
        for (int l = 0; l < L; ++l) {
            e.push_back(e.back() + std::max<int64_t>(1, chunk * pick(0, 5) + pick(-70, 70) + (pick(0, 9) ? 0 : (int64_t)1 << pick(10, 33))));
            wg.push_back(wg.back() + dense_workgroups(e[(size_t)l], e[(size_t)l + 1], chunk, kLine));
        }
        st.layer_pos.assign((size_t)L, -1);
        int64_t off = 0;
        for (int l = L - 1; l >= 0; --l)
            if (pick(1, 4) <= keep) {
                st.layer_pos[(size_t)l] = (int32_t)st.layers.size();
                st.layers.push_back(l);
                st.layer_begin.push_back(off);
                st.update_ranges.push_back((int32_t)wg[(size_t)l]);
                st.update_ranges.push_back((int32_t)wg[(size_t)l + 1]);
                off += e[(size_t)l + 1] - e[(size_t)l];
            }
        plan_dense(st, L, [&](int l) { return e[(size_t)l]; }, chunk, kLine, plain);
        for (int k = 0; k < 20; ++k, ++calls) {
            const int first = k ? (int)pick(0, L - 1) : 0, last = k ? (int)pick(first + 1, L) : L;
            int64_t at = e[(size_t)first];
            const int64_t e1 = e[(size_t)last];
            for (auto pass = first_pass(st, at); pass != st.dense_passes.end() && pass->begin < e1; ++pass) {
                static DensePass part;
                clip_pass(*pass, e[(size_t)first], e1, chunk, part, kLine, plain);
                CHECK(part.begin == at);
                if (part.width == 0) at = part.end;
                int64_t widest = 0;
                for (int i = 0; i < part.n_pieces; ++i) {
                    const Piece &q = part.pieces[i];
                    CHECK(q.begin == at && q.count > 0);
                    at += q.count;
                    // as the kernel counts: the last workgroup with elements
                    const int64_t step = q.flat0 < 0 ? plain * chunk : chunk, past = q.begin & (kLine - 1);
                    const int64_t x = (q.count + past - 1) / step;
                    CHECK(x < part.width && (part.width + 1) * step <= INT32_MAX);
                    widest = std::max(widest, x + 1);
                    if (q.flat0 < 0) continue;
                    CHECK(q.first == st.update_ranges[2 * (size_t)q.pos] && q.first + q.n == st.update_ranges[2 * (size_t)q.pos + 1]);
                    CHECK(q.pbase >= q.first && q.pbase + x < q.first + q.n);
                }
                CHECK(at == part.end && widest == part.width);
            }
            if (!st.dense_passes.empty()) CHECK(at == e1);
        }
    }
    // workgroups per CU: with SGD four below 96 bytes per thread, with AdamW for three bf16 replicas, in calls of up to 24 chunks per CU with less than 96 bytes,
    // over dense arenas from 6 to 16 chunks per CU in slots of 3/2, and where that makes the call one round of them; else three; two over dense arenas for
    // 16 to 32 fp32 replicas from 64 M elements on
    const int64_t some = 1, large = (int64_t)1 << 26, cu = 256 * 2048;
    auto sgd = [&](int N, bool wire16, bool grad16 = false) { return fused_wg_per_cu(256, true, N, wire16, false, grad16, 1 << 24, some, 1 << 24); };
    CHECK(sgd(2, false) == 4 && sgd(3, false) == 4 && sgd(4, false) == 3 && sgd(5, false) == 3 && sgd(8, false) == 3);  // 64, 80, 96, 112, 160 bytes
    CHECK(sgd(6, true) == 4 && sgd(7, true) == 3 && sgd(7, true, true) == 4 && sgd(8, true, true) == 3 && sgd(64, true) == 3);  // 88, 96, 88, 96
    for (bool dense : {true, false}) {
        auto adamw = [&](int N, bool wire16, int64_t e, int64_t slot = 3 * 128 * 2048) { return fused_wg_per_cu(256, dense, N, wire16, true, true, e, some, slot); };
        CHECK(adamw(2, true, large) == 3 && adamw(3, true, large) == 4 && adamw(3, false, large) == 3 && adamw(4, true, large) == 3);
        CHECK(adamw(3, false, 1) == 4 && adamw(4, false, 1) == 3 && adamw(6, true, 1) == 3 && adamw(5, true, 1) == 4 && adamw(2, true, 24 * cu) == 3);  // 88, 104, 96
        const int four = dense ? 4 : 3;
        CHECK(adamw(8, false, 6 * cu - 2048) == 3 && adamw(8, false, 6 * cu) == four && adamw(32, true, 16 * cu - 2048) == four && adamw(32, true, 16 * cu) == 3);
        CHECK(adamw(8, false, 6 * cu, 3 * cu / 2 - 2048) == 3 && adamw(3, false, 24 * cu - 2048, 0) == 4 && adamw(3, false, 24 * cu, 0) == 3);
        CHECK(adamw(16, false, large) == (dense ? 2 : 3) && adamw(16, false, large - 1) == 3 && adamw(15, false, large) == 3 && adamw(16, true, large) == 3);
        CHECK(adamw(32, false, large) == (dense ? 2 : 3) && adamw(33, false, large) == 3 && adamw(64, false, large) == 3);
        for (int N : {8, 40}) {
            auto round = [&](int cus, int64_t halves) { return fused_wg_per_cu(cus, dense, N, false, N == 8, true, 1, halves, 1); };
            CHECK(round(256, 768) == 3 && round(256, 769) == 4 && round(256, 1024) == 4 && round(256, 1025) == 3 && round(304, 1216) == 4);
        }
    }
    // small models, table-driven, SGD with fp32 gradients: three for 16 fp32 replicas from 45/8 workgroups per CU on, four for 32 bf16 ones from 7 on
    CHECK(small_wg_per_cu(256, 16, false, false, false, 1439) == 0 && small_wg_per_cu(256, 16, false, false, false, 1440) == 3);
    CHECK(small_wg_per_cu(256, 32, true, false, false, 1791) == 0 && small_wg_per_cu(256, 32, true, false, false, 1792) == 4);
    for (int N : {2, 8, 15, 16, 17, 31, 32, 33})
        for (int k = 0; k < 8; ++k) {
            const bool w = k & 1, adamw = k & 2, g = k & 4, has = !adamw && !g && N == (w ? 32 : 16);
            CHECK((small_wg_per_cu(256, N, w, adamw, g, 1 << 20) != 0) == has);
        }
    // halves of chunks: no layer of 128 M elements, over separate tensors with one moment fewer than 16 M elements
    const int64_t layer = (int64_t)1 << 27, model = (int64_t)1 << 24;
    CHECK(takes_halves(1, 1, true, false) && takes_halves(100 * layer, layer - 1, true, false) && !takes_halves(layer, layer, true, true));
    CHECK(takes_halves(model - 1, 1, false, false) && !takes_halves(model, 1, false, false) && takes_halves(model, 1, false, true));
    // ... in calls as measured: whole chunks from 6 to 10 chunks of 2048 per CU for vectors of less than 200 bytes, with SGD below 6 too for less than
    // 120, in slots of some size; over separate tensors whatever the slot, with SGD from 5/4 on, but for vectors of 300 bytes and more
    const int64_t per = 256 * 2048;
    for (bool dense : {true, false}) {
        auto halves = [&](int64_t numel, int N, bool wire16, bool adamw, int64_t slot = 2 * 256 * 2048, int64_t layer = 128) {
            return call_takes_halves(256, numel, slot, layer, dense, N, wire16, adamw, adamw);
        };
        CHECK(halves(6 * per - 2048, 4, false, true) && !halves(6 * per, 4, false, true) && !halves(10 * per - 2048, 4, false, true) && halves(10 * per, 4, false, true));
        CHECK(!halves(8 * per, 9, false, true) && halves(8 * per, 10, false, true) && !halves(8 * per, 18, true, true) && halves(8 * per, 19, true, true));  // 184, 200, 192, 200
        CHECK(halves(8 * per, 4, false, true, 2 * per, 127));                                                                     // layers of less than half a chunk per CU
        CHECK(halves(8 * per, 4, false, true, 3 * per / 4 - 2048) == dense && !halves(8 * per, 4, false, true, 3 * per / 4));
        CHECK(halves(8 * per, 8, false, true, 3 * per / 2 - 2048) == dense && !halves(8 * per, 8, false, true, 3 * per / 2));     // 168 bytes
        CHECK(!halves(8 * per, 4, false, true, 5 * per / 2 - 2048) && halves(8 * per, 4, false, true, 5 * per / 2) == dense);
        CHECK(halves(8 * per, 5, true, true, 5 * per / 2) == dense && !halves(8 * per, 6, true, true, 5 * per / 2));              // 88, 96
        CHECK(halves(per * 5 / 4, 4, false, false, per, 127) && !halves(per * 5 / 4, 4, false, false, per, 128) && halves(per * 5 / 4, 6, false, false, per, 128) &&
              halves(per * 5 / 4, 8, true, false, per, 128) && halves(per * 5 / 4, 7, true, false, per, 128) && !halves(per * 5 / 4, 6, true, false, per, 128));
        CHECK(!halves(per * 5, 4, false, false) && halves(5 * per, 32, false, false) && halves(9 * per, 18, false, false));
        CHECK(halves(8 * per, 4, false, false, 5 * per / 4 - 2048) == dense && !halves(8 * per, 4, false, false, 5 * per / 4) && !halves(8 * per, 4, false, false, 6 * per));
        CHECK(halves(8 * per, 8, false, false, 7 * per / 4 - 2048) == dense && !halves(8 * per, 8, false, false, 7 * per / 4));   // 160
        CHECK(!halves(5 * per, 4, false, false, 5 * per / 2 - 2048) && halves(5 * per, 4, false, false, 5 * per / 2) == dense);
        CHECK(!halves(5 * per, 5, false, false) && halves(5 * per, 6, false, false) == dense && halves(6 * per, 11, false, false) == dense);  // 112, 128, 208
        CHECK(!halves(10 * per - 2048, 4, false, false) && halves(10 * per, 4, false, false) == dense && halves(10 * per, 2, true, false) == dense);
    }
    // ... and a grid of less than 2^32 threads
    CHECK(halves_fit(1) && halves_fit(((int64_t)1 << 23) - 1) && !halves_fit((int64_t)1 << 23) && !halves_fit(INT32_MAX));
    // statistics put together in the launch: 5/2 pairs per CU, 5/4 a layer where less than half the call's chunks have none and the call is one of 24 MB
    const int64_t beside = 1 << 20, mb = 1000000;
    CHECK(folds_fused(256, 640, 640, beside, 0) && !folds_fused(256, 641, 1, beside, 0) && !folds_fused(304, 641, 641, beside, 0));
    CHECK(folds_fused(304, 760, 640, beside, 99 * mb) && folds_fused(256, 640, 640, 640, 24 * mb - 1) && !folds_fused(256, 641, 641, 641, 1));
    auto of_24 = [&](int cus, int64_t partials, int64_t chunks) { return folds_fused(cus, partials, partials, chunks, 24 * mb); };
    CHECK(of_24(256, 640, 1280) && !of_24(256, 640, 1279) && of_24(256, 320, 320) && !of_24(256, 321, 321));
    CHECK(folds_fused(256, 640, 320, 640, 99 * mb) && !folds_fused(256, 640, 321, 640, 99 * mb));
    CHECK(of_24(256, 321, 642) && !of_24(256, 321, 641) && of_24(304, 380, 380) && !of_24(304, 381, 381));
    std::printf("plain pieces ok: %ld calls\n", calls);
    return 0;
}
