// local update (Eq. (5), first case): table-driven and table-free kernels.
#include "ddp_device.h"

namespace ddp {
namespace {

template <bool ADAM, bool GBF16, bool MODEL, bool NT>
__global__ __launch_bounds__(kThreads) void update_kernel(const TensorDesc *__restrict__ runs, const UpdateChunk *__restrict__ chunks,
                                                          const UpdateScalars s) {
    const bool paced = ADAM && long_launch();
    const UpdateChunk ch = chunks[blockIdx.x];
    const TensorDesc td = runs[ch.run];
    update_body<ADAM, GBF16, MODEL, NT, false>(chunk_streams<GBF16>(td, ch), s, paced);
}

// The update when the registered tensors lie back to back in every stream (one arena per stream): workgroup b takes
// elements [b * chunk, (b + 1) * chunk) of the arenas, counted from the cache line (kLine) that the range starts in, addresses
// follow from the block index alone (no table), and chunks end on lines: only the first workgroup of a range that starts inside a
// vector has a head, of up to three elements, and only the last a tail.
// Same operations per element as update_kernel, hence the same bits.
// PAST: the range starts inside a line.  (A kernel of its own: the 15 ns that the first chunk's correction costs each workgroup
// before its first load are 0.3 % of TinyLlama-1.1B's update.)
template <bool ADAM, bool GBF16, bool MODEL, int AUX, bool PAST>
__global__ __launch_bounds__(kThreads) void update_dense_kernel(const DenseArgs a) {
    int64_t b = (int64_t)blockIdx.x * a.chunk - (PAST ? a.past : 0);
    const int64_t left = a.n - b;
    int count = left < (int64_t)a.chunk ? (int)left : a.chunk;
    if (PAST && b < 0) {
        count -= a.past;
        b = 0;
    }
    const Streams<GBF16> c{reinterpret_cast<const typename GradVec<GBF16>::elem *>(a.g) + b, a.p + b, a.s0 + b, a.s1 + b, a.mdl + b, count};
    update_body<ADAM, GBF16, MODEL, AUX != 0, true>(c, a.s);
}

}  // namespace

int launch_update(int kind, int grad_dtype, bool with_model, const TensorDesc *runs, const UpdateChunk *chunks, int64_t n_chunks,
                  const UpdateScalars &s, bool nontemporal, int lds_pad, void *stream) {
    const bool adam = kind == DDP_OPT_ADAMW, gb = grad_dtype == DDP_BF16;
#define DDP_UPD(A, G, M)                                                                               \
    if (adam == A && gb == G && with_model == M)                                                       \
        return nontemporal ? launch(update_kernel<A, G, M, true>, n_chunks, stream, lds_pad, runs, chunks, s) \
                           : launch(update_kernel<A, G, M, false>, n_chunks, stream, lds_pad, runs, chunks, s);
    DDP_UPD(false, false, false)
    DDP_UPD(false, false, true)
    DDP_UPD(false, true, false)
    DDP_UPD(false, true, true)
    DDP_UPD(true, false, false)
    DDP_UPD(true, false, true)
    DDP_UPD(true, true, false)
    DDP_UPD(true, true, true)
#undef DDP_UPD
    return (int)hipErrorInvalidValue;
}

int launch_update_dense(int kind, int grad_dtype, bool with_model, const DenseLaunch &d, const UpdateScalars &s, bool nontemporal,
                        int lds_pad, void *stream) {
    if (d.n <= 0) return 0;
    DenseArgs a{};
    a.g = d.g;
    a.p = d.p;
    a.s0 = d.s0;
    a.s1 = d.s1;
    a.mdl = d.mdl;
    a.n = d.n;
    a.chunk = d.chunk;
    a.past = d.past;
    a.s = s;
    const int64_t grid = (d.n + d.past + d.chunk - 1) / d.chunk;
    const bool adam = kind == DDP_OPT_ADAMW, gb = grad_dtype == DDP_BF16;
#define DDP_UPD(A, G, M)                                                                                \
    if (adam == A && gb == G && with_model == M)                                                        \
        return !nontemporal ? launch(update_dense_kernel<A, G, M, 0, true>, grid, stream, lds_pad, a)   \
               : a.past     ? launch(update_dense_kernel<A, G, M, 2, true>, grid, stream, lds_pad, a)   \
                            : launch(update_dense_kernel<A, G, M, 2, false>, grid, stream, lds_pad, a);
    DDP_UPD(false, false, false)
    DDP_UPD(false, false, true)
    DDP_UPD(false, true, false)
    DDP_UPD(false, true, true)
    DDP_UPD(true, false, false)
    DDP_UPD(true, false, true)
    DDP_UPD(true, true, false)
    DDP_UPD(true, true, true)
#undef DDP_UPD
    return (int)hipErrorInvalidValue;
}

}  // namespace ddp
