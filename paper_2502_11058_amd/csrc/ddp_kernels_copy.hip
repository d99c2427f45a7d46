// pack / unpack kernels (Algorithm 1: the operand of the average, and writing the average back).
#include "ddp_device.h"

namespace ddp {
namespace {

// UNPACK = false: flat[flat_begin + i] = sync[t_begin + i]           (Algorithm 1: operand of the average)
// UNPACK = true : sync[t_begin + i] = flat[flat_begin + i], and the bf16 model copy = RNE of the same value.
// The fp32 stores are always 16-byte aligned; loads, and the bf16 stores, start wherever the other side lies.
template <bool UNPACK, bool MODEL, bool NT>
__global__ __launch_bounds__(kThreads) void copy_kernel(const TensorDesc *__restrict__ runs, const CopyChunk *__restrict__ chunks,
                                                        float *__restrict__ flat) {
    const CopyChunk ch = chunks[blockIdx.x];
    float *tptr = ch.sync;
    float *fptr = flat + ch.flat_begin;
    const float *src = UNPACK ? fptr : tptr;
    float *dst = UNPACK ? tptr : fptr;
    // (the copy's address is needed after the first loads only; unused without MODEL)
    unsigned short *mdl = MODEL ? runs[ch.run].model + (tptr - runs[ch.run].sync) : reinterpret_cast<unsigned short *>(dst);
    const int n = ch.count;
    const int tid = threadIdx.x;

    const int h = head_to_16B(dst, n);
    const int nv = (n - h) >> 2;
    const float *bsrc = src + h;
    float *bdst = dst + h;
    unsigned short *bmdl = mdl + h;

    auto put = [&](unsigned i, f32x4 val) {
        st4<NT>(bdst, i, val);
        if constexpr (MODEL) st4<NT>(bmdl, i, bf16_rne4(val));
    };
    int v = tid;
    // a chunk of 2048 elements is two vectors per thread: both in flight (12 layers of 512^2, the four calls on
    // a bf16 wire: 30.6 -> 29.4 us; within the noise from GPT-2 small on)
    for (; v + kThreads < nv; v += 2 * kThreads) {
        const unsigned i = 4u * v, j = i + 4u * kThreads;
        const f32x4 a0 = ld4<NT>(bsrc, i), a1 = ld4<NT>(bsrc, j);
        put(i, a0);
        put(j, a1);
    }
    for (; v < nv; v += kThreads) put(4u * v, ld4<NT>(bsrc, 4u * v));
    if (tid < n - 4 * nv) {  // head and tail
        const unsigned i = tid < h ? tid : 4 * nv + tid;
        const float x = ld1(src, i);
        st1(dst, i, x);
        if constexpr (MODEL) st1(mdl, i, bf16_rne(x));
    }
}

// Pack for a bf16 wire: flat16[flat_begin + i] = bf16_rne(sync[t_begin + i]).  Stores are 8-byte aligned groups of
// four; the loads start wherever the tensor lies.
template <bool NT>
__global__ __launch_bounds__(kThreads) void pack16_kernel(const CopyChunk *__restrict__ chunks, unsigned short *__restrict__ flat16) {
    const CopyChunk ch = chunks[blockIdx.x];
    const float *src = ch.sync;
    unsigned short *dst = flat16 + ch.flat_begin;
    const int n = ch.count;
    const int tid = threadIdx.x;
    int h = (int)((4 - (ch.flat_begin & 3)) & 3);  // the flat buffer is 16-byte aligned at element 0
    if (h > n) h = n;
    const int nv = (n - h) >> 2;
    const float *bsrc = src + h;
    unsigned short *bdst = dst + h;
    int v = tid;
    for (; v + kThreads < nv; v += 2 * kThreads) {
        const unsigned i = 4u * v, j = i + 4u * kThreads;
        const f32x4 a0 = ld4<NT>(bsrc, i), a1 = ld4<NT>(bsrc, j);
        st4<NT>(bdst, i, bf16_rne4(a0));
        st4<NT>(bdst, j, bf16_rne4(a1));
    }
    for (; v < nv; v += kThreads) st4<NT>(bdst, 4u * v, bf16_rne4(ld4<NT>(bsrc, 4u * v)));
    if (tid < n - 4 * nv) {  // head and tail
        const unsigned i = tid < h ? tid : 4 * nv + tid;
        st1(dst, i, bf16_rne(ld1(src, i)));
    }
}

}  // namespace

int launch_copy(bool unpack, const TensorDesc *runs, const CopyChunk *chunks, int64_t n_chunks, float *flat, bool with_model,
                bool nontemporal, int lds_pad, void *stream) {
    if (!unpack) return nontemporal ? launch(copy_kernel<false, false, true>, n_chunks, stream, lds_pad, runs, chunks, flat)
                                    : launch(copy_kernel<false, false, false>, n_chunks, stream, lds_pad, runs, chunks, flat);
    if (with_model) return nontemporal ? launch(copy_kernel<true, true, true>, n_chunks, stream, lds_pad, runs, chunks, flat)
                                       : launch(copy_kernel<true, true, false>, n_chunks, stream, lds_pad, runs, chunks, flat);
    return nontemporal ? launch(copy_kernel<true, false, true>, n_chunks, stream, lds_pad, runs, chunks, flat)
                       : launch(copy_kernel<true, false, false>, n_chunks, stream, lds_pad, runs, chunks, flat);
}

int launch_pack16(const CopyChunk *chunks, int64_t n_chunks, uint16_t *flat16, bool nontemporal, int lds_pad, void *stream) {
    return nontemporal ? launch(pack16_kernel<true>, n_chunks, stream, lds_pad, chunks, flat16)
                       : launch(pack16_kernel<false>, n_chunks, stream, lds_pad, chunks, flat16);
}

}  // namespace ddp
