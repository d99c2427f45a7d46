// partial average (Eq. (5), second case) and the per-layer statistics (Sec. 3.4).
#include <type_traits>

#include "ddp_device.h"

namespace ddp {
namespace {

template <int R>
struct MeanArgs {
    const void *x[R];  // fp32 or bf16 flat buffers, rank order; first, so that they lie where wide scalar loads take them
    float *out;
    const MeanChunk *chunks;
    StatsLaunch st;
    float inv_n;
    int n;
    int cut;            // MeanLaunch
    int stage_threads;  // run-time replica count with statistics: threads that take part in the vector loop
};
// Replica pointers among the arguments of a kernel: as many as it can use, since every launch writes and reads all of them.
template <int NREP>
constexpr int kArgReps = NREP > 0 ? NREP : DDP_MAX_REPLICAS;

// Eq. (5), second case.  NREP > 0: the replica count (EXACT), or the largest count that the kernel's registers are laid out
// for, serving the counts above half of it (loads and sum fully unrolled, wave-uniform conditions on the upper half);
// NREP == 0: run-time count.  The sum runs left to right over replicas in rank order, in fp32, then one multiply by 1/N.
// STATS adds, per chunk, sum_k sum_i (out_i - x_k,i)^2 and sum_i out_i^2 in fp64.
// Bound by HBM; with bf16 replicas also by how many wavefronts the registers let in, so a group is kept as it was loaded and
// widened at each use (N = 32: 241 -> 82 VGPRs).
template <int NREP, bool EXACT, bool STATS, bool NT, bool W16, bool CUT>
__global__ __launch_bounds__(kThreads) void mean_kernel(const MeanArgs<kArgReps<NREP>> a) {
    __shared__ double lds[2][kThreads / kWave];
    // CUT: two workgroups a chunk (mean_cut).  A kernel of its own: what the others spent on it before their first load was 0.3 %.
    MeanChunk ch = a.chunks[CUT ? blockIdx.x >> 1 : blockIdx.x];
    if constexpr (CUT) {
        const int half = (int)blockIdx.x & 1, first = a.cut - ((int)ch.begin & (kLine - 1)), at = first < ch.count ? first : ch.count;
        ch.begin += half ? at : 0;
        ch.count = half ? ch.count - at : at;
        ch.partial = 2 * ch.partial + half;
    }
    // (in a vector register until the end: the kernels with conditions have no scalar one to spare)
    if constexpr (STATS && !EXACT && NREP > 0) asm("" : "+v"(ch.of.n));
    const int n = ch.count;
    const int tid = threadIdx.x;
    const int nrep = EXACT ? NREP : a.n;
    const float inv_n = a.inv_n;
    const int64_t base = ch.begin;
    double gsum = 0.0, msum = 0.0;

    // A single element.  Where the replica count is not compiled in, eight replicas are asked for together: one after the other they are
    // a chain of 2 N trips to memory, which a short launch waits for (11 layers of 201^2, N = 20, 10.2 / 8.6 us).
    auto one = [&](int64_t i) {
        auto each = [&](auto &&f) {  // f(value) of every replica, in rank order
            constexpr int U = EXACT ? 1 : 8;
            for (int k0 = 0; k0 < nrep; k0 += U) {
                float x[U];
#pragma unroll
                for (int j = 0; j < U; ++j) x[j] = wire1<W16>(a.x[EXACT || k0 + j < nrep ? k0 + j : 0], i);
#pragma unroll
                for (int j = 0; j < U; ++j)
                    if (EXACT || k0 + j < nrep) f(x[j]);
            }
        };
        float acc = -0.0f;  // (leaves the first term as it is, whatever it is)
        each([&](float x) { acc = acc + x; });
        const float m = acc * inv_n;
        if constexpr (STATS) {
            each([&](float x) { add_square(gsum, m - x); });
            add_square(msum, m);
        }
        a.out[i] = m;
    };

    // all buffers are 16-byte aligned at element 0, so the flat index decides the alignment
    int h = (int)((4 - (base & 3)) & 3);
    if (h > n) h = n;
    const int nv = (n - h) >> 2;
    // Head and tail, which only a layer's first and last chunk have, come before the vectors: behind them all replica pointers stay
    // live across the loop, and the kernel for 32 replicas spilled 54 scalar registers into 36 bytes of scratch per lane (none so).
    // No time either way, alternating builds: TinyLlama-1.1B, us, first / behind, N = 5 1066 / 1059, N = 6 1193 / 1203, N = 8
    // 1536 / 1533, N = 24 4344 / 4397, N = 32 5812 / 5791 (runs of one build differ by 2 %).
    if (tid < n - 4 * nv) one(base + (tid < h ? tid : 4 * nv + tid));

    const int64_t vbase = (base + h) >> 2;  // index in 16-byte units
    f32x4 *o4 = reinterpret_cast<f32x4 *>(a.out) + vbase;

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

    if constexpr (NREP > 0) {
        // vectors per thread in flight: 2 * NREP loads (a 2048-element chunk is 2 vectors per thread); beyond 16 replicas one
        // vector, so that the loads still fit the register file
        constexpr int B = NREP > 16 ? 1 : 2;
        // a replica's vector as it sits in memory: kept in that form (bf16: half the registers) until it is used
        typedef WireVec<W16> V;
        typedef typename V::type raw4;
        auto groups = [&](int v, auto count) {
            constexpr int C = decltype(count)::value;
            raw4 x[C][NREP];
#pragma unroll
            for (int b = 0; b < C; ++b)
#pragma unroll
                for (int k = 0; k < NREP; ++k) {
                    x[b][k] = raw4{};
                    if (EXACT || k <= NREP / 2 || k < nrep) x[b][k] = ld<NT>(reinterpret_cast<const raw4 *>(a.x[k]) + vbase + v + b * kThreads);
                }
            const int n = fresh(nrep);
#pragma unroll
            for (int b = 0; b < C; ++b) {
                f32x4 acc = V::widen(x[b][0]);
#pragma unroll
                for (int k = 1; k < NREP; ++k)
                    if (EXACT || k <= NREP / 2 || k < n) acc = acc + V::widen(x[b][k]);
                const f32x4 m = acc * inv_n;
                if constexpr (STATS) {
#pragma unroll
                    for (int k = 0; k < NREP; ++k)
                        if (EXACT || k <= NREP / 2 || k < n) stats4(m, widen_again<W16>(x[b][k]));
                    msq4(m);
                }
                st<NT>(o4 + v + b * kThreads, m);
            }
        };
        int v = tid;
        for (; v + (B - 1) * kThreads < nv; v += B * kThreads) groups(v, std::integral_constant<int, B>());
        if constexpr (B > 1)
            for (; v < nv; v += kThreads) groups(v, std::integral_constant<int, 1>());
    } else if constexpr (STATS) {
        // Run-time replica count (above kFixedReps) with statistics: the first kRegReps replicas of a vector stay in registers,
        // the rest are parked in LDS (one column per thread), so every replica is fetched from memory once; 192 threads take
        // part at N = 33, 64 at N = 64.
        extern __shared__ __align__(16) unsigned char dyn_lds[];
        f32x4 *stage = reinterpret_cast<f32x4 *>(dyn_lds);
        const int vt = a.stage_threads;
        if (tid < vt) {
            for (int v = tid; v < nv; v += vt) {
                f32x4 r[kRegReps];
#pragma unroll
                for (int k = 0; k < kRegReps; ++k) r[k] = wire4<W16, NT>(a.x[k], vbase + v);
                f32x4 acc = r[0];
#pragma unroll
                for (int k = 1; k < kRegReps; ++k) acc = acc + r[k];
                for (int k0 = kRegReps; k0 < nrep; k0 += 4) {  // four more loads in flight, then park and add them in rank order
                    f32x4 x[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (k0 + j < nrep) x[j] = wire4<W16, NT>(a.x[k0 + j], vbase + v);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (k0 + j < nrep) {
                            stage[(k0 + j - kRegReps) * vt + tid] = x[j];
                            acc = acc + x[j];
                        }
                }
                const f32x4 m = acc * inv_n;
#pragma unroll
                for (int k = 0; k < kRegReps; ++k) stats4(m, r[k]);
                for (int k = kRegReps; k < nrep; ++k) stats4(m, stage[(k - kRegReps) * vt + tid]);
                msq4(m);
                st<NT>(o4 + v, m);
            }
        }
    } else {
        for (int v = tid; v < nv; v += kThreads) {
            f32x4 acc = wire4<W16, NT>(a.x[0], vbase + v);
            for (int k = 1; k < nrep; ++k) acc = acc + wire4<W16, NT>(a.x[k], vbase + v);
            st<NT>(o4 + v, acc * inv_n);
        }
    }

    if constexpr (STATS) {
        // Up to four replicas, with three and four workgroups per CU, the two sums of a long launch come one after the other
        // (TinyLlama-1.1B, us, side by side / so: N = 4 860 / 831, N = 2 508 / 501, N = 3 661 / 653);
        // with 9 to 16 fp32 replicas from 8192 workgroups on (N = 16, 218 M 2469 / 2454, 67 M 774 / 771, N = 14, 37 M 362 / 361, N = 12, 27 M
        // 222.0 / 221.4; N = 12, 2.4 M 17.4 / 17.9).  Five to eight (N = 6, 159.3 / 160.0) and bf16 replicas gain nothing.
        constexpr bool kApart = NREP > 0 && NREP <= 4, kLongApart = NREP > 8 && NREP <= 16 && !W16;
        if ((kApart && !a.st.counters) || (kLongApart && gridDim.x >= 8192)) {
            gsum = block_sum(gsum, lds[0]);
            msum = block_sum(msum, lds[1]);
        } else {
            block_sum2(gsum, msum, lds);
        }
        if constexpr (!EXACT && NREP > 0) ch.of.n = __builtin_amdgcn_readfirstlane(ch.of.n);
        put_partial<CUT ? 2 : 1>(a.st, ch.partial, ch.of, ch.of.pos, nrep, gsum, msum);
    }
}

// Per-layer statistics from the per-chunk partials, in two fixed-order stages so that a layer with 10^5 chunks does
// not hang on one workgroup: stage 1 cuts layer l's partials [ranges[2l], ranges[2l+1]) into kStatSlices contiguous
// slices, one workgroup each (thread-strided sums, then the workgroup tree); stage 2 adds the slice sums of a layer
// in slice order and scales the divergence by 1/N (Sec. 3.4: Gamma = 1/K sum_k ||wbar - w^k||^2, per layer).
__global__ __launch_bounds__(kThreads) void stats_slices_kernel(const double *__restrict__ partials,
                                                                const int32_t *__restrict__ ranges, int pairs, double *__restrict__ slice_sums) {
    __shared__ double lds[2][kThreads / kWave];
    const int l = blockIdx.y, j = blockIdx.x;
    const int64_t c0 = (int64_t)pairs * ranges[2 * l], c1 = (int64_t)pairs * ranges[2 * l + 1];
    const int64_t lo = c0 + (c1 - c0) * j / kStatSlices, hi = c0 + (c1 - c0) * (j + 1) / kStatSlices;
    double g = 0.0, m = 0.0;
    for (int64_t c = lo + (int64_t)threadIdx.x; c < hi; c += kThreads) {
        g += partials[2 * c];
        m += partials[2 * c + 1];
    }
    block_sum2(g, m, lds);
    if (threadIdx.x == 0) {
        slice_sums[2 * ((int64_t)l * kStatSlices + j)] = g;
        slice_sums[2 * ((int64_t)l * kStatSlices + j) + 1] = m;
    }
}

__global__ __launch_bounds__(kWave) void stats_finalize_kernel(const double *__restrict__ slice_sums, int n_replicas,
                                                               double *__restrict__ stats) {
    const int l = blockIdx.x;
    if (threadIdx.x == 0) {
        double g = 0.0, m = 0.0;
        for (int j = 0; j < kStatSlices; ++j) {
            g += slice_sums[2 * ((int64_t)l * kStatSlices + j)];
            m += slice_sums[2 * ((int64_t)l * kStatSlices + j) + 1];
        }
        stats[2 * l] = g / (double)n_replicas;
        stats[2 * l + 1] = m;
    }
}

// The same reduction in one launch, for layers with few partials (launch-bound slots): one workgroup per layer adds the
// layer's partials thread-strided, then the workgroup tree.  Fixed order as well.  Bound by the start of the workgroups where layers are many: those of
// up to kThreads partials each take workgroups of that size (average, N = 4, 1024 threads / 256, us: 1000 layers of 700 elements 9.0 / 7.3, 500 of 2000
// 7.7 / 7.1, 200 of 5000 6.8 / 6.6, 100 of 40000 16.0 / 15.8).
template <int THREADS>
__global__ __launch_bounds__(THREADS) void stats_single_kernel(const double *__restrict__ partials, const int32_t *__restrict__ ranges,
                                                               int pairs, int n_replicas, double *__restrict__ stats) {
    __shared__ double lds[2][THREADS / kWave];
    const int l = blockIdx.x;
    sum_partials<THREADS>(partials, (int64_t)pairs * ranges[2 * l], (int64_t)pairs * ranges[2 * l + 1], n_replicas, stats + 2 * l, lds);
}

// Dynamic LDS of a launch: the residency pad, or the staging area of the run-time replica count if that is larger.
template <int NREP>
int mean_lds(const MeanLaunch &a) {
    const int need = NREP == 0 && a.st.partials ? stage_bytes(a.n_replicas - kRegReps) : 0;
    return a.lds_pad > need ? a.lds_pad : need;
}

template <int NREP, bool EXACT, bool CUT>
int launch_mean_c(const MeanLaunch &a, void *stream) {
    MeanArgs<kArgReps<NREP>> ma;
    for (int k = 0; k < kArgReps<NREP>; ++k) ma.x[k] = k < a.n_replicas ? a.x[k] : nullptr;
    ma.out = a.out;
    ma.chunks = a.chunks;
    ma.st = a.st;
    ma.inv_n = a.inv_n;
    ma.n = a.n_replicas;
    ma.cut = a.cut;
    ma.stage_threads = stage_threads(a.n_replicas - kRegReps);  // the replicas beyond the registers are staged
    const int64_t grid = CUT ? 2 * a.n_chunks : a.n_chunks;
    if constexpr (!CUT || NREP >= kCutReps16) {
        if (a.wire16) {
            if (a.st.partials) return launch(mean_kernel<NREP, EXACT, true, true, true, CUT>, grid, stream, mean_lds<NREP>(a), ma);
            return launch(mean_kernel<NREP, EXACT, false, true, true, CUT>, grid, stream, a.lds_pad, ma);
        }
    }
    if (a.st.partials) return a.nontemporal ? launch(mean_kernel<NREP, EXACT, true, true, false, CUT>, grid, stream, mean_lds<NREP>(a), ma)
                                         : launch(mean_kernel<NREP, EXACT, true, false, false, CUT>, grid, stream, mean_lds<NREP>(a), ma);
    return a.nontemporal ? launch(mean_kernel<NREP, EXACT, false, true, false, CUT>, grid, stream, a.lds_pad, ma)
                         : launch(mean_kernel<NREP, EXACT, false, false, false, CUT>, grid, stream, a.lds_pad, ma);
}

template <int NREP, bool EXACT>
int launch_mean_n(const MeanLaunch &a, void *stream) {
    if constexpr (NREP >= kCutReps)
        if (a.cut) return launch_mean_c<NREP, EXACT, true>(a, stream);
    return launch_mean_c<NREP, EXACT, false>(a, stream);
}

}  // namespace

int launch_stats(const double *partials, double *slice_sums, const int32_t *ranges, int pairs, int n_layers, int n_replicas, double *stats,
                 int64_t max_partials_per_layer, void *stream) {
    if (n_layers <= 0) return 0;
    if (max_partials_per_layer <= kStatSingleMax) {
        const int threads = max_partials_per_layer <= kThreads ? kThreads : kSumThreads;
        hipLaunchKernelGGL(threads == kThreads ? stats_single_kernel<kThreads> : stats_single_kernel<kSumThreads>, dim3((unsigned)n_layers),
                           dim3((unsigned)threads), 0, (hipStream_t)stream, partials, ranges, pairs, n_replicas, stats);
        return (int)hipGetLastError();
    }
    hipLaunchKernelGGL(stats_slices_kernel, dim3(kStatSlices, (unsigned)n_layers), dim3(kThreads), 0, (hipStream_t)stream, partials,
                       ranges, pairs, slice_sums);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
    hipLaunchKernelGGL(stats_finalize_kernel, dim3((unsigned)n_layers), dim3(kWave), 0, (hipStream_t)stream,
                       (const double *)slice_sums, n_replicas, stats);
    return (int)hipGetLastError();
}

int launch_mean(const MeanLaunch &a, void *stream) {
    int rc;
    switch (a.n_replicas) {
        case 1: rc = launch_mean_n<1, true>(a, stream); break;
        case 2: rc = launch_mean_n<2, true>(a, stream); break;
        case 3: rc = launch_mean_n<3, true>(a, stream); break;
        case 4: rc = launch_mean_n<4, true>(a, stream); break;
        case 5: rc = launch_mean_n<5, true>(a, stream); break;
        case 6: rc = launch_mean_n<6, true>(a, stream); break;
        case 7: rc = launch_mean_n<7, true>(a, stream); break;
        case 8: rc = launch_mean_n<8, true>(a, stream); break;
        case 9: rc = launch_mean_n<9, true>(a, stream); break;
        case 10: rc = launch_mean_n<10, true>(a, stream); break;
        case 11: rc = launch_mean_n<11, true>(a, stream); break;
        case 12: rc = launch_mean_n<12, true>(a, stream); break;
        case 13: rc = launch_mean_n<13, true>(a, stream); break;
        case 14: rc = launch_mean_n<14, true>(a, stream); break;
        case 15: rc = launch_mean_n<15, true>(a, stream); break;
        case 16: rc = launch_mean_n<16, true>(a, stream); break;
        case kFixedReps: rc = launch_mean_n<kFixedReps, true>(a, stream); break;
        default: rc = a.n_replicas < kFixedReps ? launch_mean_n<kFixedReps, false>(a, stream) : launch_mean_n<0, false>(a, stream); break;
    }
    return rc;
}

}  // namespace ddp
