// The plan of the fused step over dense arenas with chunks that end on cache lines (kLine): random models, whole and clipped to
// ranges of layers.  Every element belongs to one piece, pieces are cut on lines, every scheduled workgroup has a partial of its
// own layer's, and the launch is wide enough for what the kernel makes of a piece.
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
    std::mt19937_64 rng(11);
    auto pick = [&](int64_t lo, int64_t hi) { return lo + (int64_t)(rng() % (uint64_t)(hi - lo + 1)); };
    long calls = 0;
    for (int r = 0; r < 500; ++r) {
        const int64_t chunk = 1024 * pick(1, 3);
        const int L = (int)pick(1, 30), keep = (int)pick(0, 4);
        SlotTables st;
        std::vector<int64_t> e(1, 0), wg(1, 0);
        for (int l = 0; l < L; ++l) {
            e.push_back(e.back() + std::max<int64_t>(1, chunk * pick(0, 3) + pick(-70, 70) + (pick(0, 9) ? 0 : (int64_t)1 << pick(10, 33))));
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
        plan_dense(st, L, [&](int l) { return e[(size_t)l]; }, chunk, kLine);
        for (int k = 0; k < 20; ++k, ++calls) {
            const int first = k ? (int)pick(0, L - 1) : 0, last = k ? (int)pick(first + 1, L) : L;
            const int64_t e0 = e[(size_t)first], e1 = e[(size_t)last];
            int64_t at = e0;
            for (auto pass = first_pass(st, e0); pass != st.dense_passes.end() && pass->begin < e1; ++pass) {
                static DensePass part;
                clip_pass(*pass, e0, e1, chunk, part, kLine);
                CHECK(part.begin == at);
                if (part.width == 0) {  // a plain update: unscheduled layers alone, wherever they start
                    for (int l = first; l < last; ++l) CHECK(st.layer_pos[(size_t)l] < 0 || e[(size_t)l + 1] <= part.begin || e[(size_t)l] >= part.end);
                    at = part.end;
                    continue;
                }
                for (int i = 0; i < part.n_pieces; ++i) {
                    const Piece &q = part.pieces[i];
                    CHECK(q.begin == at && q.count > 0);
                    at += q.count;
                    const int past = (int)q.begin & (kLine - 1);  // as the kernel counts
                    int64_t chunks = 0;
                    while ((chunks + 1) * chunk - past < q.count) ++chunks;
                    ++chunks;
                    CHECK(chunks <= part.width && (part.width + 1) * chunk <= INT32_MAX);
                    if (q.flat0 < 0) continue;
                    const int64_t l0 = e[(size_t)q.layer], l1 = e[(size_t)q.layer + 1];
                    CHECK(q.begin >= l0 && at <= l1 && (q.begin == l0 || q.begin % kLine == 0) && (at == l1 || at % kLine == 0));
                    CHECK(q.flat0 == st.layer_begin[(size_t)q.pos] + q.begin - l0);
                    const int64_t before = q.begin == l0 ? 0 : (q.begin - l0 / kLine * kLine) / chunk;
                    CHECK(q.pbase == st.update_ranges[2 * (size_t)q.pos] + before);
                    CHECK(at == l1 ? q.pbase + chunks == st.update_ranges[2 * (size_t)q.pos + 1] : (at - l0 / kLine * kLine) == (before + chunks) * chunk);
                }
                CHECK(at == part.end);
            }
            if (!st.dense_passes.empty()) CHECK(at == e1);
        }
    }
    std::printf("plan lines ok: %ld calls\n", calls);
    return 0;
}
