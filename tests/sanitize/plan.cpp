// The launches of the fused step over dense arenas (ddp_plan.h), built for the host with sanitizers: random models and
// schedules, whole-model calls and ranges of layers, against the rules that the kernel relies on.  Every element of the range
// belongs to exactly one piece, with its own flat index; every scheduled workgroup writes the partial of its own place; the
// 32-bit indexes hold; a range call allocates nothing.  Sizes up to 2^36 elements: the arithmetic needs no memory.
#include <cstdio>
#include <cstdlib>
#include <new>
#include <random>

#include "ddp_plan.h"

static long g_allocations = 0;
void *operator new(std::size_t n) {
    ++g_allocations;
    if (void *p = std::malloc(n ? n : 1)) return p;
    std::abort();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

#define CHECK(cond)                                                                          \
    do {                                                                                     \
        if (!(cond)) {                                                                       \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond);    \
            std::exit(1);                                                                    \
        }                                                                                    \
    } while (0)

using namespace ddp;

struct Model {
    std::vector<int64_t> e;  // first element of every layer, and the end
    SlotTables st;
    int64_t chunk;
    int L() const { return (int)e.size() - 1; }
};

static Model make(const std::vector<int64_t> &sizes, const std::vector<int> &order, int64_t chunk) {
    Model m;
    m.chunk = chunk;
    m.e.push_back(0);
    for (int64_t n : sizes) m.e.push_back(m.e.back() + n);
    std::vector<int64_t> wg(1, 0);
    for (size_t l = 0; l < sizes.size(); ++l) wg.push_back(wg.back() + dense_workgroups(m.e[l], m.e[l + 1], chunk, kLine));
    m.st.layer_pos.assign(sizes.size(), -1);
    int64_t off = 0;
    for (int l : order) {
        m.st.layer_pos[(size_t)l] = (int32_t)m.st.layers.size();
        m.st.layers.push_back(l);
        m.st.layer_begin.push_back(off);
        m.st.update_ranges.push_back((int32_t)wg[(size_t)l]);
        m.st.update_ranges.push_back((int32_t)wg[(size_t)l + 1]);
        off += sizes[(size_t)l];
    }
    m.st.layer_begin.push_back(off);
    plan_dense(m.st, m.L(), [&](int l) { return m.e[(size_t)l]; }, chunk, kLine);
    return m;
}

// The launches of a call on layers [first, first + count); their number is returned.
static int check_call(const Model &m, int first, int count) {
    const int64_t e0 = m.e[(size_t)first], e1 = m.e[(size_t)(first + count)];
    int64_t at = e0;
    int launches = 0;
    for (auto pass = first_pass(m.st, e0); pass != m.st.dense_passes.end() && pass->begin < e1; ++pass) {
        const DensePass &whole = *pass;
        static DensePass part;
        const long before = g_allocations;
        clip_pass(whole, e0, e1, m.chunk, part, kLine);
        CHECK(g_allocations == before);
        if (whole.begin >= e0 && whole.end <= e1) {  // inside: the clipped form is the launch itself
            CHECK(part.width == whole.width && part.n_pieces == whole.n_pieces && part.begin == whole.begin && part.end == whole.end);
        }
        ++launches;
        CHECK(part.begin == at && part.begin < part.end);
        if (part.width == 0) {
            CHECK(part.n_pieces == 0);
            for (int l = 0; l < m.L(); ++l)
                if (m.e[(size_t)l] < part.end && m.e[(size_t)l + 1] > part.begin) CHECK(m.st.layer_pos[(size_t)l] < 0);
            at = part.end;
            continue;
        }
        CHECK(part.n_pieces >= 1 && part.n_pieces <= kMaxPieces);
        CHECK(((int64_t)part.width + 1) * m.chunk <= INT32_MAX);
        int64_t widest = 0;
        bool scheduled = false;
        for (int i = 0; i < part.n_pieces; ++i) {
            const Piece &q = part.pieces[i];
            scheduled = scheduled || q.flat0 >= 0;
            CHECK(q.begin == at && q.count > 0);
            at += q.count;
            const int64_t wg = dense_workgroups(q.begin, at, m.chunk, kLine);
            CHECK(wg <= part.width);
            widest = std::max(widest, wg);
            if (q.flat0 < 0) {
                for (int l = first; l < first + count; ++l)
                    if (m.e[(size_t)l] < at && m.e[(size_t)l + 1] > q.begin) CHECK(m.st.layer_pos[(size_t)l] < 0);
                continue;
            }
            CHECK(q.pos >= 0 && q.pos < (int)m.st.layers.size() && m.st.layers[(size_t)q.pos] == q.layer);
            const int64_t l0 = m.e[(size_t)q.layer], l1 = m.e[(size_t)q.layer + 1];
            CHECK(q.begin >= l0 && at <= l1 && q.flat0 == m.st.layer_begin[(size_t)q.pos] + (q.begin - l0));
            // its workgroups follow each other in the layer's partials: the first one's place, and the last one's
            CHECK(q.begin == l0 || q.begin % kLine == 0);
            CHECK(q.pbase == m.st.update_ranges[2 * (size_t)q.pos] + (q.begin / kLine * kLine - l0 / kLine * kLine) / m.chunk);
            CHECK((q.begin / kLine * kLine - l0 / kLine * kLine) % m.chunk == 0);
            CHECK(at == l1 ? q.pbase + wg == m.st.update_ranges[2 * (size_t)q.pos + 1] : at % kLine == 0 && wg == (at - q.begin / kLine * kLine) / m.chunk);
        }
        CHECK(at == part.end && widest == part.width && scheduled);  // unscheduled layers alone are a plain update
    }
    CHECK(at == e1);
    CHECK(takes_pieces(m.st, first_pass(m.st, e0), e1) == (!m.st.table_first || launches == 1));
    return launches;
}

int main(int argc, char **argv) {
    const int rounds = argc > 1 ? std::atoi(argv[1]) : 300;
    std::mt19937_64 rng(7);
    auto pick = [&](int64_t lo, int64_t hi) { return lo + (int64_t)(rng() % (uint64_t)(hi - lo + 1)); };
    long planned = 0, ranges = 0;
    for (int r = 0; r < rounds; ++r) {
        const int64_t chunk = 1024 * (r % 3 == 0 ? 1 : r % 3 == 1 ? 2 : pick(1, 1024));
        const int L = (int)pick(1, r % 5 == 0 ? 1000 : 40);
        std::vector<int64_t> sizes;
        const int spread = (int)pick(1, 30);
        for (int l = 0; l < L; ++l) sizes.push_back(pick(1, ((int64_t)1 << pick(0, spread))));
        if (r % 7 == 0) sizes[(size_t)pick(0, L - 1)] = pick((int64_t)1 << 31, (int64_t)1 << 36);
        std::vector<int> order;
        const int keep = (int)pick(0, 4);  // of four layers: none to all scheduled
        for (int l = L - 1; l >= 0; --l)
            if (pick(1, 4) <= keep) order.push_back(l);
        if (r % 2) std::shuffle(order.begin(), order.end(), rng);
        int64_t total = 0;
        for (int64_t n : sizes) total += (n + chunk - 1) / chunk + 1;
        if (total > INT32_MAX) continue;  // registration refuses it
        const Model m = make(sizes, order, chunk);
        if (m.st.dense_passes.empty()) continue;
        ++planned;
        check_call(m, 0, L);
        for (int k = 0; k < 40; ++k, ++ranges) {
            const int first = (int)pick(0, L - 1);
            check_call(m, first, (int)pick(1, L - first));
        }
    }
    CHECK(planned > rounds / 2);
    {  // small layers beside one that has a launch of its own, and a run of unscheduled layers cut at odd elements
        std::vector<int64_t> sizes(21, 1001);
        sizes[0] = (int64_t)1 << 30;
        const Model m = make(sizes, {20, 19, 18, 17, 16, 15, 14, 13, 12, 11, 10, 9, 8, 7, 6, 5, 4, 3, 2, 1, 0}, 2048);
        CHECK(check_call(m, 0, 21) == 2 && check_call(m, 1, 20) == 1 && check_call(m, 5, 7) == 1);
        const Model u = make(std::vector<int64_t>(9, ((int64_t)1 << 25) + 1), {8}, 2048);
        CHECK(u.st.dense_passes.size() == 2 && u.st.dense_passes[0].width == 0);
        for (int first = 0; first < 9; ++first)
            for (int count = 1; first + count <= 9; ++count) check_call(u, first, count);
        const Model v = make({8, 1000, 1001, 4000, 6, 12}, {2, 4}, 2048);  // one launch; unscheduled ranges are plain updates
        CHECK(v.st.dense_passes.size() == 1);
        static DensePass part;
        auto range = [&](int first, int last) { clip_pass(v.st.dense_passes[0], v.e[(size_t)first], v.e[(size_t)last], 2048, part, kLine); };
        range(0, 2);
        CHECK(part.width == 0);
        range(1, 2);
        CHECK(part.width == 0);
        range(3, 4);  // begins at element 2009
        CHECK(part.width == 0 && part.n_pieces == 0 && part.begin == 2009 && part.end == 6009);
        range(0, 3);
        CHECK(part.width == 1 && part.n_pieces == 2 && part.pieces[1].flat0 == 0);
    }
    // the number of launches, on both sides of each line; 0: the table's single one
    auto launches = [&](std::vector<int64_t> sizes) {
        std::vector<int> order;
        for (int l = (int)sizes.size() - 1; l >= 0; --l) order.push_back(l);
        const Model m = make(sizes, order, 2048);
        return m.st.table_first ? 0 : (int)m.st.dense_passes.size();
    };
    auto layers = [](size_t n, int64_t size) { return std::vector<int64_t>(n, size); };
    const int64_t large = (int64_t)3 << 23;
    CHECK(launches(layers(20, 1)) == 1 && launches(layers(21, 1)) == 0 && launches(layers(400, 1000)) == 0);
    CHECK(launches(layers(32, 1 << 19)) == 2 && launches(layers(32, (1 << 19) - 1)) == 0);
    CHECK(launches(layers(20, large - 1)) == 1 && launches(layers(20, large)) == 20);
    CHECK(launches({large, 5, 7, large, 9}) == 4 && launches({5, large, 7}) == 3 && launches({5, large - 1, 7, large - 1, 9}) == 1);
    // more pieces of 2^31 elements than a launch takes: no plan (the slot takes the table), and nothing written out of range
    CHECK(make({(int64_t)1 << 37, 5}, {1, 0}, 2048 * 64).st.dense_passes.empty());
    CHECK(make({5, (int64_t)1 << 37}, {0}, 2048 * 64).st.dense_passes.empty());
    std::printf("plan sweep ok: %ld slots, %ld ranges\n", planned, ranges);
    return 0;
}
