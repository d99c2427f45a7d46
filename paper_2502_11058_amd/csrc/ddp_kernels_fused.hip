// fused synchronisation + update, table-driven (both cases of Eq. (5) in one pass).
//
// Compiled twice, once per optimizer (-DDDP_FUSED_ADAM=0: SGD with momentum, =1: AdamW), so that the two halves of the
// kernel's instantiations build in parallel; the first half also holds the dispatcher.
#include "ddp_fused.h"

#ifndef DDP_FUSED_ADAM
#error "compile with -DDDP_FUSED_ADAM=0 or -DDDP_FUSED_ADAM=1"
#endif

namespace ddp {
namespace {

struct FusedArgs {
    Peers peers;
    const TensorDesc *runs;
    const UpdateChunk *chunks;
    const RunSlot *run_slot;
    const int32_t *run_chunk_base;      // per run: index of its first chunk in registration order
    StatsLaunch st;                     // partials: a pair per scheduled chunk, or per half of one
    UpdateScalars s;
    int chunk_elems;
    int halved;  // 1: two workgroups a chunk
};
static_assert(offsetof(FusedArgs, peers) == 0 && offsetof(Peers, x) == 0, "peers_again reads them at the start of the arguments");

// At least two wavefronts per SIMD (the launch bounds), the residency that the launch asks for.  SGD on 16 fp32 replicas with fp32 gradients: four,
// which its 128 to 130 registers otherwise have or miss with any change (small_wg_per_cu, where both are measured).
template <bool ADAM, bool GBF16, int NREP, bool EXACT, bool W16>
constexpr int kWavesPerSimd = !ADAM && !GBF16 && NREP == 16 && EXACT && !W16 ? 4 : 2;

// A chunk of a scheduled run takes fused_body, every other chunk the optimizer step only.
template <bool ADAM, bool GBF16, bool MODEL, int NREP, bool EXACT, bool STATS, bool W16, bool UTS, bool PAIRS>
__global__ __launch_bounds__(kThreads, (kWavesPerSimd<ADAM, GBF16, NREP, EXACT, W16>)) void fused_kernel(const FusedArgs a) {
    __shared__ double lds[2][kThreads / kWave];
    const bool paced = ADAM && long_launch();  // (of use to whole chunks: half a chunk is one vector a thread)
    UpdateChunk ch = a.chunks[blockIdx.x >> a.halved];
    const TensorDesc td = a.runs[ch.run];
    const RunSlot ts = a.run_slot[ch.run];
    // Where this chunk's partial pair goes: chunks end on cache lines, chunk c of a run begins less than kLine elements before
    // c * chunk_elems.  (A division: behind the loads.)
    const int64_t chunk_begin = ch.begin;
    auto partial = [&] {
        const int64_t p = (int64_t)a.run_chunk_base[ch.run] + (chunk_begin + kLine - 1) / a.chunk_elems;
        return a.halved ? 2 * p + (blockIdx.x & 1) : p;
    };
    if (a.halved) {
        const int half = (int)blockIdx.x & 1, first = a.chunk_elems / 2 - ((int)(ch.begin + td.past) & (kLine - 1)), at = first < ch.count ? first : ch.count;
        ch.begin += half ? at : 0;
        ch.count = half ? ch.count - at : at;
        // an empty half has its place among the partials only where another run of the layer lies behind it
        if (ch.count == 0 && (ts.flat0 < 0 || partial() >= ts.of.first + ts.of.n)) return;
    }
    const Streams<GBF16> c = chunk_streams<GBF16>(td, ch);
    if (ts.flat0 < 0) {  // uniform for the workgroup
        update_body<ADAM, GBF16, MODEL, true, false>(c, a.s, paced);
        return;
    }
    double gsum = 0.0, msum = 0.0;
    fused_body<ADAM, GBF16, MODEL, NREP, EXACT, STATS, W16, UTS, PAIRS, false>(c, ts.flat0 + ch.begin, a.peers, a.s, gsum, msum);
    if constexpr (STATS) {
        block_sum2(gsum, msum, lds);
        put_partial<1>(a.st, partial(), ts.of, ts.layer, a.peers.n, gsum, msum);
    }
}

}  // namespace

namespace {

struct LaunchTable {
    const FusedTable &f;
    const FusedArgs &a;
    void *stream;
    template <bool A, bool G, bool M, int NR, bool EXACT, bool STATS, bool W, bool U, bool PAIRS>
    int go(int lds) const {
        return launch(fused_kernel<A, G, M, NR, EXACT, STATS, W, U, PAIRS>, f.halved ? 2 * f.n_chunks : f.n_chunks, stream, lds, a);
    }
};

}  // namespace

#if DDP_FUSED_ADAM
#define DDP_FUSED_HALF launch_fused_adamw
#else
#define DDP_FUSED_HALF launch_fused_sgdm
#endif

// The kernel launch of this file's optimizer.
int DDP_FUSED_HALF(const FusedTable &f, void *stream) {
    FusedArgs a;
    fill_peers(a.peers, f);
    a.runs = f.runs;
    a.chunks = f.chunks;
    a.run_slot = f.run_slot;
    a.run_chunk_base = f.run_chunk_base;
    a.st = f.st;
    a.s = f.s;
    a.chunk_elems = f.chunk_elems;
    a.halved = f.halved;
    return dispatch_fused<DDP_FUSED_ADAM != 0>(f, LaunchTable{f, a, stream});
}

#if !DDP_FUSED_ADAM
int launch_fused_adamw(const FusedTable &f, void *stream);

int launch_fused(const FusedTable &f, void *stream) {
    return f.kind == DDP_OPT_ADAMW ? launch_fused_adamw(f, stream) : launch_fused_sgdm(f, stream);
}
#endif

}  // namespace ddp
