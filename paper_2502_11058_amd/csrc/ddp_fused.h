// The averaging + update of one run of elements, shared by the table-driven and the table-free fused kernels.
#ifndef DDP_FUSED_H
#define DDP_FUSED_H

#include <type_traits>

#include "ddp_device.h"

#pragma clang fp contract(off)

namespace ddp {
namespace {

struct Peers {
    const void *x[DDP_MAX_REPLICAS - 1];  // the N-1 peers' flat buffers (fp32 or bf16) in rank order
    float inv_n;
    int n;
    int local_rank;
    int stage_threads;  // run-time replica count with statistics: threads that take part in the vector loop
};

// The peers' pointers as they lie in the launch's arguments, whose first bytes they are in every fused kernel, as an address that the compiler takes for
// a new one: what it has in registers from an earlier read is not kept for this one.
typedef const void *const __attribute__((address_space(4))) *PeerPointers;
__device__ __forceinline__ PeerPointers peers_again() {
    auto p = (PeerPointers)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// (entries from N-1 on are never used)
inline void fill_peers(Peers &p, const FusedLaunch &f) {
    for (int k = 0; k + 1 < f.n_replicas; ++k) p.x[k] = f.x[k];
    p.inv_n = f.inv_n;
    p.n = f.n_replicas;
    p.local_rank = f.local_rank;
    p.stage_threads = stage_threads(f.n_replicas - kRegReps);  // only the terms beyond the registers are staged
}

// Both cases of Eq. (5) in one pass over the run c, whose peers' values start at flat index fo: the average over the N
// replicas is formed from the local tensor and the peers' flat buffers (same rank-ordered fp32 sum and 1/N multiply as
// mean_kernel) and the optimizer step is applied.
//   UTS = false: average, then update the average (the bits of pack -> partial average -> unpack -> local update);
//   UTS = true:  update the local value, then average it with the peers (Eq. (5) and Algorithm 1 as printed: the
//                replicas that are averaged have taken this iteration's step; the bits of local update -> pack ->
//                partial average -> unpack).
// W16: peers are bf16 and the local replica contributes its bf16 rounding.  NREP > 0: the replica count (EXACT), or the
// largest one that the registers are laid out for; 0: run-time loop, for more than kFixedReps.  gsum, msum: this thread's statistics (STATS).
template <bool ADAM, bool GBF16, bool MODEL, int NREP, bool EXACT, bool STATS, bool W16, bool UTS, bool PAIRS, bool BUF>
__device__ __forceinline__ void fused_body(const Streams<GBF16> c, int64_t fo, const Peers &a, const UpdateScalars &s, double &gsum, double &msum) {
    typedef GradVec<GBF16> G;
    typedef typename G::vec gvec;
    constexpr bool NT = true;
    const int tid = threadIdx.x;
    const int nrep = EXACT ? NREP : a.n;
    const int lr = a.local_rank;
    const float inv_n = a.inv_n;
    auto step1 = [&](float gi, float &x, float &av, float &bv) {
        if constexpr (ADAM)
            adamw_one(gi, x, av, bv, s);
        else
            sgdm_one(gi, x, av, s);
    };

    // The parameters' accesses are aligned; the peers' flat offset, and any stream that lies differently against its own
    // vectors, take unaligned ones.  Bound by HBM either way: a slot whose flat offsets are odd runs at the rate of an aligned
    // one (28 M parameters, N = 24, fp32 peers: 583 us with a scalar loop over such chunks, 259 us so, 259 us aligned).
    const int h = head_to_16B(c.p, c.n);
    const int nv = (c.n - h) >> 2;
    const Vectors<GBF16, BUF> b(c, h, nv);
    const int64_t bfo = fo + h;
    typedef typename WireVec<W16>::elem xelem;
    // A buffer's base must be dword-aligned, which a bf16 peer's need not be; and the kernels for 17 to 31 replicas, whose conditions take
    // scalar registers too, have none to spare for four per peer (10 layers of 3000^2, N = 24, SGD 738 us with buffers, 724 without, AdamW 868 /
    // 853; N = 32, all unconditional, 906 / 923 and 1052 / 1064).
    constexpr bool kPeerBuffers = BUF && !W16 && (EXACT || NREP <= 16);

    auto stats4 = [&](f32x4 m, f32x4 x) {
        const f32x4 d = m - x;
        add_square(gsum, d.x);
        add_square(gsum, d.y);
        add_square(gsum, d.z);
        add_square(gsum, d.w);
    };
    auto msq4 = [&](f32x4 m) {
        add_square(msum, m.x);
        add_square(msum, m.y);
        add_square(msum, m.z);
        add_square(msum, m.w);
    };
    auto step4 = [&](gvec gv, f32x4 &x, f32x4 &av, f32x4 &bv) {
        const f32x4 gw = G::widen(gv);
        float G4[4] = {gw.x, gw.y, gw.z, gw.w};
        float P4[4] = {x.x, x.y, x.z, x.w};
        float A4[4] = {av.x, av.y, av.z, av.w};
        float B4[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) step1(G4[j], P4[j], A4[j], B4[j]);
        x = f32x4{P4[0], P4[1], P4[2], P4[3]};
        av = f32x4{A4[0], A4[1], A4[2], A4[3]};
        bv = f32x4{B4[0], B4[1], B4[2], B4[3]};
    };
    auto store4 = [&](unsigned i, f32x4 res, f32x4 av, f32x4 bv) {
        b.p.template st<NT>(i, res);
        b.s0.template st<NT>(i, av);
        if constexpr (ADAM) b.s1.template st<NT>(i, bv);
        if constexpr (MODEL) b.mdl.template st<NT>(i, bf16_rne4(res));
    };
    if constexpr (NREP > 1) {
        // The local contribution may be computed (updated and / or rounded) and a branch on it per replica would serialise
        // the loads: the N-1 peers are loaded by their position among the peers, all in flight before the first use.
        // One vector of all streams in flight per thread, or two (PAIRS, a kernel of its own: takes_pairs): with many bf16 peers, half
        // the bytes a peer, nothing else would be asked for while one vector's long sum is formed.
        typedef typename WireVec<W16>::type raw4;
        auto groups = [&](int v, auto count) {
            constexpr int K = decltype(count)::value;
            raw4 pv[K][NREP - 1];
            f32x4 pl[K], av[K], bv[K];
            gvec gv[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const unsigned i = 4u * (v + k * kThreads);
#pragma unroll
                for (int j = 0; j < NREP - 1; ++j) {
                    pv[k][j] = raw4{};
                    if (j < kPeersAlways<NREP, EXACT> || j < nrep - 1) {
                        const Stream<kPeerBuffers, xelem> x(reinterpret_cast<const xelem *>(a.x[j]) + bfo, nv);
                        pv[k][j] = __builtin_bit_cast(raw4, x.template ld<NT>(i));
                    }
                }
                pl[k] = b.p.template ld<NT>(i);
                gv[k] = b.g.template ld<NT>(i);
                av[k] = b.s0.template ld<NT>(i);
                bv[k] = f32x4{};
                if constexpr (ADAM) bv[k] = b.s1.template ld<NT>(i);
            }
            if constexpr (K > 1) __builtin_amdgcn_sched_barrier(0);  // all requested before the first vector's arithmetic
#pragma unroll
            for (int k = 0; k < K; ++k) {
                fused_math4<ADAM, GBF16, NREP, EXACT, STATS, W16, UTS>(pv[k], gv[k], pl[k], av[k], bv[k], nrep, lr, inv_n, s, gsum, msum);
                store4(4u * (v + k * kThreads), pl[k], av[k], bv[k]);
            }
        };
        int v = tid;
        if constexpr (PAIRS)
            for (; v + kThreads < nv; v += 2 * kThreads) groups(v, std::integral_constant<int, 2>());
        for (; v < nv; v += kThreads) groups(v, std::integral_constant<int, 1>());
    } else {
        // run-time replica count, above kFixedReps; with statistics the terms beyond the first kRegReps are parked in LDS (see
        // stage_threads) so that the peers are fetched once; only the first `vt` threads take part (192 at N = 33, 64 at 64)
        extern __shared__ __align__(16) unsigned char dyn_lds[];
        f32x4 *stage = reinterpret_cast<f32x4 *>(dyn_lds);
        const int vt = STATS ? a.stage_threads : kThreads;
        for (int v = tid; v < nv && tid < vt; v += vt) {
            const unsigned i = 4u * v;
            f32x4 pl = b.p.template ld<NT>(i);
            const gvec gv = b.g.template ld<NT>(i);
            f32x4 av = b.s0.template ld<NT>(i);
            f32x4 bv{};
            if constexpr (ADAM) bv = b.s1.template ld<NT>(i);
            if constexpr (UTS) step4(gv, pl, av, bv);
            f32x4 loc = pl;
            if constexpr (W16) loc = bf16_widen4(bf16_rne4(pl));
            auto term = [&](int k) -> f32x4 { return k == lr ? loc : WireVec<W16>::widen(wire_raw4<W16, NT>(a.x[k - (k > lr ? 1 : 0)], bfo, i)); };
            // the first kRegReps terms of the rank-order sum stay in registers, the rest are parked in LDS
            f32x4 r[kRegReps];
#pragma unroll
            for (int k = 0; k < kRegReps; ++k) r[k] = term(k);
            f32x4 acc = r[0];
#pragma unroll
            for (int k = 1; k < kRegReps; ++k) acc = acc + r[k];
            for (int k0 = kRegReps; k0 < nrep; k0 += 8) {  // eight more peers in flight, then park and add them in rank order
                f32x4 x[8];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (k0 + j < nrep) x[j] = term(k0 + j);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (k0 + j < nrep) {
                        if constexpr (STATS) stage[(k0 + j - kRegReps) * vt + tid] = x[j];
                        acc = acc + x[j];
                    }
            }
            f32x4 m = acc * inv_n;
            if constexpr (STATS) {
#pragma unroll
                for (int k = 0; k < kRegReps; ++k) stats4(m, r[k]);
                for (int k = kRegReps; k < nrep; ++k) stats4(m, stage[(k - kRegReps) * vt + tid]);
                msq4(m);
            }
            if constexpr (!UTS) step4(gv, m, av, bv);
            store4(i, m, av, bv);
        }
    }
    // head and tail together, element by element, behind the vectors: only a tensor's first and last chunk have any
    if (tid < c.n - 4 * nv) {
        const unsigned i = tid < h ? tid : 4 * nv + tid;
        // Replicas that the registers are laid out for are asked for together, as the vectors are, others eight at a time: one after the other
        // they are a chain of 2 N trips to memory, which a short launch waits for.  Fused step, us, one after the other / so: 14 layers of
        // 226^2, N = 32 bf16 16.3 / 9.7, 5 of 282^2, AdamW, N = 6 7.2 / 6.3, 15 of 166^2, AdamW, N = 24 13.7 / 11.2 (all at once 9.8, but the scalar
        // registers that the kernels for 17 to 31 spill then cost 10 layers of 3000^2 845 / 850), N = 40 27.6 / 23.1.
        constexpr bool kTogether = NREP > 1 && (EXACT || NREP <= 16);
        // The table-driven kernels of 9 and more replicas read the peers' pointers again: kept over the vector loop, for a handful of elements, they
        // made up to 94 scalar registers spill (12 layers of 2304^2, separate tensors, bf16 peers, us kept / read again: SGD, N = 12 269.1 / 262.0,
        // N = 32 387.0 / 373.2, layer by layer 441.0 / 418.5).  The table-free ones keep them without, and read again a short call is slower (15 layers
        // of 166^2, AdamW, N = 32 bf16 9.2 / 9.9).  Eight pointers are read at a time: one by one each element waits for its pointer (13 layers of 142^2,
        // separate tensors, one by one / eight, AdamW, N = 12 bf16 7.7 / 7.4, N = 32 bf16 9.3 / 8.5, SGD 8.6 / 8.1; large calls alike).
        // With two vectors in flight, which only long calls have, one by one: eight would make up to 86 more spill.
        constexpr bool kAgain = !BUF && NREP >= 16, kEight = kAgain && !PAIRS;
        xelem peer[kTogether ? NREP - 1 : 1];
        if constexpr (kTogether) {
            PeerPointers again = nullptr;
#pragma unroll
            for (int j = 0; j < NREP - 1; ++j) {
                if constexpr (kEight)
                    if (j % 8 == 0) again = peers_again();
                peer[j] = xelem{};
                if (j < kPeersAlways<NREP, EXACT> || j < nrep - 1)
                    peer[j] = ld1(reinterpret_cast<const xelem *>(kEight ? again[j] : a.x[kAgain ? fresh(j) : j]) + fo, i);
            }
        }
        float pl = ld1(c.p, i), av = ld1(c.s0, i), bv = ADAM ? ld1(c.s1, i) : 0.0f;
        const float gi = G::widen1(ld1(c.g, i));
        if constexpr (UTS) step1(gi, pl, av, bv);
        // what this worker contributes: its value, rounded to bf16 first if that is what its peers received
        const float loc = W16 ? bf16_widen(bf16_rne(pl)) : pl;
        float m;
        if constexpr (kTogether) {
            constexpr int ALWAYS = kPeersAlways<NREP, EXACT>;
            const int n = fresh(nrep), at = fresh(lr);
            float acc = -0.0f;
#pragma unroll
            for (int j = 0; j < NREP - 1; ++j) {
                if (j == at) acc = acc + loc;
                if (j < ALWAYS || j < n - 1) acc = acc + WireVec<W16>::widen1(peer[j]);
            }
            if constexpr (EXACT)
                if (at == NREP - 1) acc = acc + loc;
            m = acc * inv_n;
            if constexpr (STATS) {
#pragma unroll
                for (int j = 0; j < NREP - 1; ++j) {
                    if (j == at) add_square(gsum, m - loc);
                    if (j < ALWAYS || j < n - 1) add_square(gsum, m - WireVec<W16>::widen1(peer[j]));
                }
                if constexpr (EXACT)
                    if (at == NREP - 1) add_square(gsum, m - loc);
                add_square(msum, m);
            }
        } else {
            auto each = [&](auto &&f) {  // f(value) of every replica, in rank order
                for (int k0 = 0; k0 < nrep; k0 += 8) {
                    float x[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) {  // (the last peer again where the local replica or none is meant)
                        const int q = k0 + k - (k0 + k > lr ? 1 : 0);
                        x[k] = wire1<W16>(a.x[q < nrep - 1 ? q : nrep - 2], fo + i);
                    }
#pragma unroll
                    for (int k = 0; k < 8; ++k)
                        if (k0 + k < nrep) f(k0 + k == lr ? loc : x[k]);
                }
            };
            float acc = -0.0f;
            each([&](float x) { acc = acc + x; });
            m = acc * inv_n;
            if constexpr (STATS) {
                each([&](float x) { add_square(gsum, m - x); });
                add_square(msum, m);
            }
        }
        float res = m;
        if constexpr (!UTS) step1(gi, res, av, bv);
        st1(c.p, i, res);
        st1(c.s0, i, av);
        if constexpr (ADAM) st1(c.s1, i, bv);
        if constexpr (MODEL) st1(c.mdl, i, bf16_rne(res));
    }
}

// The instantiation for a launch: K::go<ADAM, GBF16, MODEL, NREP, EXACT, STATS, W16, UTS, PAIRS>(lds), lds = the dynamic LDS it needs
// (the residency pad, or the staging area of the run-time replica count if that is larger).
template <bool A, bool G, bool M, int NR, bool EXACT, bool W, bool PAIRS, class K>
int dispatch_fused_w(const FusedLaunch &f, const K &k, int lds) {
    if (f.update_first) return f.st.partials ? k.template go<A, G, M, NR, EXACT, true, W, true, PAIRS>(lds) : k.template go<A, G, M, NR, EXACT, false, W, true, PAIRS>(lds);
    return f.st.partials ? k.template go<A, G, M, NR, EXACT, true, W, false, PAIRS>(lds) : k.template go<A, G, M, NR, EXACT, false, W, false, PAIRS>(lds);
}

template <bool A, bool G, bool M, int NR, bool EXACT, class K>
int dispatch_fused_n(const FusedLaunch &f, const K &k) {
    const int need = NR == 0 && f.st.partials ? stage_bytes(f.n_replicas - kRegReps) : 0;
    const int lds = f.lds_pad > need ? f.lds_pad : need;
    if (!f.wire16) return dispatch_fused_w<A, G, M, NR, EXACT, false, false>(f, k, lds);
    if constexpr (NR >= 16)
        if (f.pairs) return dispatch_fused_w<A, G, M, NR, EXACT, true, true>(f, k, lds);
    return dispatch_fused_w<A, G, M, NR, EXACT, true, false>(f, k, lds);
}

template <bool A, bool G, bool M, class K>
int dispatch_fused_t(const FusedLaunch &f, const K &k) {
    const int n = f.n_replicas;
    switch (n) {
        case 2: return dispatch_fused_n<A, G, M, 2, true>(f, k);
        case 4: return dispatch_fused_n<A, G, M, 4, true>(f, k);
        case 8: return dispatch_fused_n<A, G, M, 8, true>(f, k);
        case 16: return dispatch_fused_n<A, G, M, 16, true>(f, k);
        case kFixedReps: return dispatch_fused_n<A, G, M, kFixedReps, true>(f, k);
    }
    // Other counts up to 31 take the kernel laid out for the next power of two, whose upper loads are conditional: within 3 %
    // of the rate of the exact kernels beside them (28 M parameters, SGD-m, bf16 peers, N = 12: 130 us; 192 us with the
    // run-time loop, which stays for what does not fit the registers).
    if (n < 4) return dispatch_fused_n<A, G, M, 4, false>(f, k);
    if (n < 8) return dispatch_fused_n<A, G, M, 8, false>(f, k);
    if (n < 16) return dispatch_fused_n<A, G, M, 16, false>(f, k);
    if (n < kFixedReps) return dispatch_fused_n<A, G, M, kFixedReps, false>(f, k);
    return dispatch_fused_n<A, G, M, 0, false>(f, k);
}

template <bool A, class K>
int dispatch_fused(const FusedLaunch &f, const K &k) {
    const bool gb = f.grad_dtype == DDP_BF16;
    if (!gb && !f.with_model) return dispatch_fused_t<A, false, false>(f, k);
    if (!gb) return dispatch_fused_t<A, false, true>(f, k);
    if (!f.with_model) return dispatch_fused_t<A, true, false>(f, k);
    return dispatch_fused_t<A, true, true>(f, k);
}

}  // namespace
}  // namespace ddp

#endif
