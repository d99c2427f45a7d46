// fused synchronisation + update over dense arenas (table-free).
//
// Compiled twice, once per optimizer, like the table-driven kernel.
#include "ddp_fused.h"

#ifndef DDP_FUSED_ADAM
#error "compile with -DDDP_FUSED_ADAM=0 or -DDDP_FUSED_ADAM=1"
#endif

namespace ddp {
namespace {

struct FusedDenseArgs {
    Peers peers;
    DenseLaunch d;
    StatsLaunch st;
    UpdateScalars s;
    int plain;  // elements per workgroup of an unscheduled piece (d.chunk: of a scheduled one)
    Piece pieces[kMaxPieces];
};

// fused_kernel for a model registered as dense arenas: a workgroup's addresses follow from its indexes and its piece, which is
// part of the launch's arguments.  Bound by HBM with two workgroups per CU, so what a workgroup spends before its first load
// counts: with the pieces searched by workgroup index instead of indexed (about 0.2 us) TinyLlama-1.1B at N = 2 took 5450 us,
// so 5220.
template <bool ADAM, bool GBF16, bool MODEL, int NREP, bool EXACT, bool STATS, bool W16, bool UTS, bool PAIRS>
__global__ __launch_bounds__(kThreads, 2) void fused_dense_kernel(const FusedDenseArgs a) {
    __shared__ double lds[2][kThreads / kWave];
    const Piece t = a.pieces[blockIdx.y];
    // Two workgroups per CU do not hide what one spends before its first load: the arguments are requested together, not
    // where each is first used behind a branch.
    asm volatile("" ::"s"(a.d.g), "s"(a.d.p), "s"(a.d.s0), "s"(a.d.s1), "s"(a.d.mdl));
#pragma unroll
    for (int j = 0; j < (NREP < 16 ? NREP : 16) - 1; ++j) asm volatile("" ::"s"(a.peers.x[j]));
    const int past = (int)t.begin & (kLine - 1);             // chunks end at multiples of kLine
    const int chunk = t.flat0 < 0 ? a.plain : a.d.chunk;
    const int hi = ((int)blockIdx.x + 1) * chunk - past;
    int at = hi - chunk;
    at = at > 0 ? at : 0;
    const int n = (hi < t.count ? hi : t.count) - at;
    if (n <= 0) return;  // a piece narrower than the widest
    const int64_t begin = t.begin + at;
    const Streams<GBF16> c{reinterpret_cast<const typename GradVec<GBF16>::elem *>(a.d.g) + begin, a.d.p + begin, a.d.s0 + begin, a.d.s1 + begin,
                           a.d.mdl + begin, n};
    if (t.flat0 < 0) {
        update_body<ADAM, GBF16, MODEL, true, true>(c, a.s);
        return;
    }
    double gsum = 0.0, msum = 0.0;
    fused_body<ADAM, GBF16, MODEL, NREP, EXACT, STATS, W16, UTS, PAIRS, true>(c, t.flat0 + at, a.peers, a.s, gsum, msum);
    if constexpr (STATS) {
        block_sum2(gsum, msum, lds);
        put_partial<1>(a.st, (int64_t)t.pbase + blockIdx.x, LayerSums{t.pos, t.first, t.n}, t.layer, a.peers.n, gsum, msum);
    }
}

struct LaunchDense {
    const FusedDense &f;
    const FusedDenseArgs &a;
    void *stream;
    template <bool A, bool G, bool M, int NR, bool EXACT, bool STATS, bool W, bool U, bool PAIRS>
    int go(int lds) const {
        return launch2(fused_dense_kernel<A, G, M, NR, EXACT, STATS, W, U, PAIRS>, f.pass->width, f.pass->n_pieces, stream, lds, a);
    }
};

}  // namespace

#if DDP_FUSED_ADAM
#define DDP_FUSED_HALF launch_fused_dense_adamw
#else
#define DDP_FUSED_HALF launch_fused_dense_sgdm
#endif

int DDP_FUSED_HALF(const FusedDense &f, void *stream) {
    FusedDenseArgs a;
    fill_peers(a.peers, f);
    a.d = f.d;
    a.plain = f.plain;
    a.st = f.st;
    a.s = f.s;
    for (int i = 0; i < f.pass->n_pieces; ++i) a.pieces[i] = f.pass->pieces[i];
    return dispatch_fused<DDP_FUSED_ADAM != 0>(f, LaunchDense{f, a, stream});
}

#if !DDP_FUSED_ADAM
int launch_fused_dense_adamw(const FusedDense &f, void *stream);

int launch_fused_dense(const FusedDense &f, void *stream) {
    return f.kind == DDP_OPT_ADAMW ? launch_fused_dense_adamw(f, stream) : launch_fused_dense_sgdm(f, stream);
}
#endif

}  // namespace ddp
