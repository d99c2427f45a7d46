// The launches of the fused step over dense arenas: how the model is cut into pieces, once per slot, and what of them a call
// on a range of layers runs.  Arithmetic on the host only.
#ifndef DDP_PLAN_H
#define DDP_PLAN_H

#include <algorithm>

#include "ddp_internal.h"

namespace ddp {

// Workgroups of the table-free fused kernel over elements [e0, e1) of the arenas: chunks counted from the multiple of four at
// or below e0, where every stream is vector-aligned.
inline int64_t dense_workgroups(int64_t e0, int64_t e1, int64_t chunk) { return (e1 - e0 / 4 * 4 + chunk - 1) / chunk; }

// Chunks of the widest piece that the kernel's 32-bit indexes allow.
inline int64_t widest_piece(int64_t chunk) { return INT32_MAX / chunk - 1; }

// Elements [begin, end), all of one scheduled layer (flat0 >= 0) or all unscheduled, as pieces of at most `width` chunks behind
// those that p has.
inline void add_pieces(DensePass &p, int64_t begin, int64_t end, int64_t flat0, int64_t pbase, int32_t pos, int32_t layer, int64_t width,
                       int64_t chunk) {
    const int64_t base = begin / 4 * 4, wg = dense_workgroups(begin, end, chunk);
    for (int64_t b = 0; b < wg; b += width) {
        const int64_t at = b == 0 ? begin : base + b * chunk, to = std::min(end, base + (b + width) * chunk);
        p.pieces[p.n_pieces++] = {at, flat0 < 0 ? -1 : flat0 + (at - begin), (int32_t)(to - at), (int32_t)(pbase + b), pos, layer};
    }
}

// The launches over the whole model of L layers, layer l being elements [elem0(l), elem0(l + 1)) of the arenas.  A segment is a
// scheduled layer or a run of unscheduled ones.  Where segments average fewer than 2^25 elements all of them share one launch
// (one per kMaxSegments), cut into pieces of about the same width: a launch of its own costs a segment some 3 us of ramp (GPT-2
// small, AdamW, N = 8, 20 M per segment: 701 us in one launch, 726 in six; 12 layers of 512^2: 25 against 47).  Larger ones get
// a launch each, the unscheduled ones that of the plain update, whose workgroups start sooner (Llama-2-7B blocks, 380 M per
// segment: 11.8 ms in one launch, 11.5 in five; about equal at 40 M), and small ones between them share.  Empty where a launch would need more than kMaxPieces
// pieces (segments of tens of 2^31 elements): such a slot takes the table.
template <class Elem0>
std::vector<DensePass> plan_dense(const SlotTables &st, int L, Elem0 &&elem0, int64_t chunk) {
    constexpr int kMaxSegments = 20;
    struct Segment {
        int64_t begin, end, flat0, pbase, wg;
        int32_t pos, layer;
    };
    std::vector<Segment> all;
    for (int l = 0; l < L;) {
        const int i = st.layer_pos[(size_t)l];
        int m = l + 1;
        while (i < 0 && m < L && st.layer_pos[(size_t)m] < 0) ++m;
        all.push_back({elem0(l), elem0(m), i < 0 ? -1 : st.layer_begin[(size_t)i], i < 0 ? 0 : st.dense_ranges[2 * (size_t)i],
                       dense_workgroups(elem0(l), elem0(m), chunk), i, l});
        l = m;
    }
    std::vector<DensePass> passes;
    if (all.empty()) return passes;
    constexpr int64_t kApart = (int64_t)1 << 25;
    const bool apart = (all.back().end - all[0].begin) / (int64_t)all.size() >= kApart;
    auto alone = [&](size_t k) { return apart && all[k].end - all[k].begin >= kApart; };
    const int64_t widest = widest_piece(chunk);
    for (size_t i = 0; i < all.size();) {
        const Segment *seg = &all[i];
        int n = 1;
        while (!alone(i) && n < kMaxSegments && i + (size_t)n < all.size() && !alone(i + (size_t)n)) ++n;
        i += (size_t)n;
        int64_t least = 0;
        for (int k = 0; k < n; ++k) least += (seg[k].wg + widest - 1) / widest;
        if (least > kMaxPieces) return {};
        passes.emplace_back();
        DensePass &p = passes.back();
        p.width = p.n_pieces = 0;
        p.begin = seg[0].begin;
        p.end = seg[n - 1].end;
        if (n == 1 && seg[0].flat0 < 0 && seg[0].begin % 4 == 0) continue;
        // the width that leaves the fewest workgroups without work among those that cut some segment evenly
        int64_t width = widest, best = INT64_MAX;
        for (int k = 0; k < n; ++k)
            for (int64_t parts : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24}) {
                const int64_t w = (seg[k].wg + parts - 1) / parts;
                if (w > widest) continue;
                int64_t rows = 0;
                for (int j = 0; j < n; ++j) rows += (seg[j].wg + w - 1) / w;
                if (rows <= kMaxPieces && (rows * w < best || (rows * w == best && w > width))) {
                    best = rows * w;
                    width = w;
                }
            }
        p.width = (int)width;
        for (int k = 0; k < n; ++k)
            add_pieces(p, seg[k].begin, seg[k].end, seg[k].flat0, seg[k].pbase, seg[k].pos, seg[k].layer, width, chunk);
    }
    return passes;
}

// What a call on elements [e0, e1), whole layers, runs of launch p: the pieces inside, runs of unscheduled layers cut at the
// range's ends.  No search and nothing allocated; part is written only as far as its pieces go.
inline void clip_pass(const DensePass &p, int64_t e0, int64_t e1, int64_t chunk, DensePass &part) {
    part.begin = std::max(p.begin, e0);
    part.end = std::min(p.end, e1);
    part.width = part.n_pieces = 0;
    if (part.begin >= part.end) return;
    if (p.width == 0) {
        if (part.begin % 4 == 0) return;  // a plain update as well
        // (no more pieces than the whole run would have, which plan_dense has counted)
        const int64_t wg = dense_workgroups(part.begin, part.end, chunk);
        part.width = (int)std::min(wg, widest_piece(chunk));
        add_pieces(part, part.begin, part.end, -1, 0, -1, -1, part.width, chunk);
        return;
    }
    for (int i = 0; i < p.n_pieces; ++i) {
        const Piece &whole = p.pieces[i];
        const int64_t b = std::max(whole.begin, e0), e = std::min(whole.begin + whole.count, e1);
        if (b >= e) continue;
        Piece &q = part.pieces[part.n_pieces++];
        q = whole;
        q.begin = b;  // (moves in unscheduled pieces only: a scheduled one is part of one layer)
        q.count = (int32_t)(e - b);
        part.width = std::max(part.width, (int)dense_workgroups(b, e, chunk));
    }
}

}  // namespace ddp

#endif
