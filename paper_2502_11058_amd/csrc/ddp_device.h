// Device-side helpers shared by the kernel files of the library (gfx950).
//
//
// All kernels are HBM streaming kernels (well under 1 flop per byte): no MFMA, no data reuse.  The design
// rules are the same everywhere:
//   - one workgroup (256 threads = 4 wavefronts of 64) per table entry ("chunk"), a run of elements inside one
//     tensor or one layer, so the ragged boundaries of tensors and layers are handled by the table, not by
//     per-element searches; where the registered tensors form dense arenas the update and the fused step need no
//     table at all (the *_dense_kernel variants: addresses from the block index, buffer accesses);
//   - inside a chunk: a scalar head of < 4 elements up to the next 16-byte boundary of the destination, a body
//     of 128-bit accesses (lane i of a wavefront touches bytes [16i, 16i+16) of a 1 KiB line, fully coalesced),
//     and a scalar tail of < 4 elements;
//   - several independent 128-bit loads are issued before the first use, to keep enough bytes in flight per CU;
//   - streaming (nontemporal) cache hints, since nothing is read twice;
//   - floating-point contraction is off: every product and sum below is its own IEEE fp32 operation, and
//     division and square root are the correctly rounded ones, so results do not depend on instruction selection.
#ifndef DDP_DEVICE_H
#define DDP_DEVICE_H

#include <hip/hip_runtime.h>

#include <cstdint>

#include "ddp_internal.h"

#pragma clang fp contract(off)

namespace ddp {
namespace {

constexpr int kThreads = 256;
constexpr int kWave = 64;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <bool NT, class T>
__device__ __forceinline__ T ld(const T *p) {
    if constexpr (NT)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}

template <bool NT, class T>
__device__ __forceinline__ void st(T *p, T v) {
    if constexpr (NT)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

// Groups of four elements at any element: gfx950 takes 128- and 64-bit global accesses at any address, so a stream whose
// start is not a multiple of its vector needs no scalar loop.  A wavefront's 1 KiB then touches one cache line more than an
// aligned one, mostly out of the cache: a fused step with odd offsets reads 1.017 times and writes 1.000 times its algorithmic
// bytes.  base is wave-uniform and i, an element index, an unsigned 32-bit one: the access takes its base from scalar registers
// and one offset register serves all streams of a type.  The address space is stated because a pointer that a kernel reads
// from a table is a generic one, whose accesses (flat) also wait for and occupy the LDS counter.
#define DDP_GLOBAL __attribute__((address_space(1)))
typedef f32x4 f32x4_any __attribute__((aligned(4)));
typedef u16x4 u16x4_any __attribute__((aligned(2)));

template <class T>
struct AnyVec;  // element type -> its group of four with the alignment of one element
template <>
struct AnyVec<float> {
    typedef f32x4 vec;
    static __device__ __forceinline__ const DDP_GLOBAL f32x4_any *at(const float *p, unsigned i) {
        return (const DDP_GLOBAL f32x4_any *)((const DDP_GLOBAL char *)p + 4u * i);
    }
};
template <>
struct AnyVec<unsigned short> {
    typedef u16x4 vec;
    static __device__ __forceinline__ const DDP_GLOBAL u16x4_any *at(const unsigned short *p, unsigned i) {
        return (const DDP_GLOBAL u16x4_any *)((const DDP_GLOBAL char *)p + 2u * i);
    }
};

template <bool NT, class T>
__device__ __forceinline__ typename AnyVec<T>::vec ld4(const T *base, unsigned i) {
    if constexpr (NT) return __builtin_nontemporal_load(AnyVec<T>::at(base, i));
    return *AnyVec<T>::at(base, i);
}
__device__ __forceinline__ float ld1(const float *base, unsigned i) { return *(const DDP_GLOBAL float *)((const DDP_GLOBAL char *)base + 4u * i); }
__device__ __forceinline__ unsigned short ld1(const unsigned short *base, unsigned i) {
    return *(const DDP_GLOBAL unsigned short *)((const DDP_GLOBAL char *)base + 2u * i);
}
template <bool NT>
__device__ __forceinline__ void st4(float *base, unsigned i, f32x4 v) {
    DDP_GLOBAL f32x4_any *q = (DDP_GLOBAL f32x4_any *)((DDP_GLOBAL char *)base + 4u * i);
    if constexpr (NT)
        __builtin_nontemporal_store(v, q);
    else
        *q = v;
}
template <bool NT>
__device__ __forceinline__ void st4(unsigned short *base, unsigned i, u16x4 v) {
    DDP_GLOBAL u16x4_any *q = (DDP_GLOBAL u16x4_any *)((DDP_GLOBAL char *)base + 2u * i);
    if constexpr (NT)
        __builtin_nontemporal_store(v, q);
    else
        *q = v;
}
__device__ __forceinline__ void st1(float *base, unsigned i, float v) { *(DDP_GLOBAL float *)((DDP_GLOBAL char *)base + 4u * i) = v; }
__device__ __forceinline__ void st1(unsigned short *base, unsigned i, unsigned short v) {
    *(DDP_GLOBAL unsigned short *)((DDP_GLOBAL char *)base + 2u * i) = v;
}

// fp32 -> bf16, round to nearest, ties to even (add 0x7fff plus the lowest kept bit, then truncate); NaN -> quiet NaN.
__device__ __forceinline__ unsigned short bf16_rne(float f) {
    unsigned int u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x0040u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

__device__ __forceinline__ float bf16_widen(unsigned short h) { return __uint_as_float(((unsigned int)h) << 16); }

__device__ __forceinline__ u16x4 bf16_rne4(f32x4 v) {
    u16x4 r;
    r.x = bf16_rne(v.x);
    r.y = bf16_rne(v.y);
    r.z = bf16_rne(v.z);
    r.w = bf16_rne(v.w);
    return r;
}

__device__ __forceinline__ f32x4 bf16_widen4(u16x4 h) {
    return f32x4{bf16_widen(h.x), bf16_widen(h.y), bf16_widen(h.z), bf16_widen(h.w)};
}

// One replica's flat buffer as it arrives: fp32 (W16 = false) or bf16 bit patterns (W16 = true, widened exactly).
// Element index i, or index v of a group of 4 elements (16 bytes of fp32, 8 bytes of bf16).
template <bool W16>
__device__ __forceinline__ float wire1(const void *base, int64_t i) {
    if constexpr (W16)
        return bf16_widen(reinterpret_cast<const unsigned short *>(base)[i]);
    else
        return reinterpret_cast<const float *>(base)[i];
}
template <bool W16, bool NT>
__device__ __forceinline__ f32x4 wire4(const void *base, int64_t v) {
    if constexpr (W16)
        return bf16_widen4(ld<NT>(reinterpret_cast<const u16x4 *>(base) + v));
    else
        return ld<NT>(reinterpret_cast<const f32x4 *>(base) + v);
}

// A group of four elements of a replica as it sits in memory, and its exact widening to fp32.
template <bool W16>
struct WireVec;
template <>
struct WireVec<false> {
    typedef float elem;
    typedef f32x4 type;
    static __device__ __forceinline__ f32x4 widen(f32x4 v) { return v; }
    static __device__ __forceinline__ float widen1(float v) { return v; }
};
template <>
struct WireVec<true> {
    typedef unsigned short elem;
    typedef u32x2 type;  // whole registers: 16-bit lanes kept over the loads of a group make the compiler copy them about
    static __device__ __forceinline__ f32x4 widen(u32x2 v) {
        return f32x4{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u)};
    }
    static __device__ __forceinline__ float widen1(unsigned short v) { return bf16_widen(v); }
};
// The group for its second use: bf16 is widened anew, or the compiler keeps the widened form, twice the registers, from the
// first use on.
template <bool W16>
__device__ __forceinline__ f32x4 widen_again(typename WireVec<W16>::type v) {
    if constexpr (W16) asm("" : "+v"(v));
    return WireVec<W16>::widen(v);
}
// ... loaded from element first + i of the replica (first wave-uniform).
template <bool W16, bool NT>
__device__ __forceinline__ typename WireVec<W16>::type wire_raw4(const void *base, int64_t first, unsigned i) {
    return __builtin_bit_cast(typename WireVec<W16>::type, ld4<NT>(reinterpret_cast<const typename WireVec<W16>::elem *>(base) + first, i));
}

// Buffer (MUBUF) accesses: a per-workgroup descriptor (base in SGPRs, extent = the workgroup's part of the stream)
// plus a 32-bit byte offset per lane.  Accesses past the extent read zero / are dropped by the hardware.
// AUX: cache policy bits of the instruction (2 = nt, the streaming hint; 0 = default).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00020000);  // raw dword format
}

template <int AUX, class T>
__device__ __forceinline__ T bld(__amdgpu_buffer_rsrc_t r, int byte_off) {
    static_assert(sizeof(T) == 16 || sizeof(T) == 8, "128- or 64-bit access");
    if constexpr (sizeof(T) == 16)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(r, byte_off, 0, AUX));
    else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, byte_off, 0, AUX));
}

template <int AUX, class T>
__device__ __forceinline__ void bst(__amdgpu_buffer_rsrc_t r, int byte_off, T v) {
    static_assert(sizeof(T) == 16 || sizeof(T) == 8, "128- or 64-bit access");
    if constexpr (sizeof(T) == 16)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, byte_off, 0, AUX);
    else
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, byte_off, 0, AUX);
}

// One stream of a run of whole vectors, nv groups of four from a wave-uniform base on: through a buffer descriptor (BUF; the
// base must be dword-aligned) or as global accesses.
template <bool BUF, class T>
struct Stream;
template <class T>
struct Stream<true, T> {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ Stream(const T *base, int nv) : r(make_rsrc(base, nv * 4 * (int)sizeof(T))) {}
    template <bool NT>
    __device__ __forceinline__ typename AnyVec<T>::vec ld(unsigned i) const {
        return bld<NT ? 2 : 0, typename AnyVec<T>::vec>(r, (int)(i * (unsigned)sizeof(T)));
    }
    template <bool NT>
    __device__ __forceinline__ void st(unsigned i, typename AnyVec<T>::vec v) const {
        bst<NT ? 2 : 0>(r, (int)(i * (unsigned)sizeof(T)), v);
    }
};
template <class T>
struct Stream<false, T> {
    T *p;
    __device__ __forceinline__ Stream(const T *base, int) : p(const_cast<T *>(base)) {}
    template <bool NT>
    __device__ __forceinline__ typename AnyVec<T>::vec ld(unsigned i) const {
        return ld4<NT>(p, i);
    }
    template <bool NT>
    __device__ __forceinline__ void st(unsigned i, typename AnyVec<T>::vec v) const {
        st4<NT>(p, i, v);
    }
};

__device__ __forceinline__ int head_to_16B(const void *p, int n) {  // fp32 elements until p is 16-byte aligned
    int h = (int)((4u - (unsigned)((reinterpret_cast<uintptr_t>(p) >> 2) & 3u)) & 3u);
    return h < n ? h : n;
}

// sum + d * d in fp64.  The product of two widened fp32 values is exact, so one fused operation gives the bits of the two
// (average, us: 10 layers of 1536^2, N = 24 124.0 -> 121.7, N = 32 157.3 -> 155.7; 9 of 900^2, N = 12 19.1 -> 18.7, N = 16 23.8 -> 23.3).
__device__ __forceinline__ void add_square(double &sum, float d) { sum = __builtin_fma((double)d, (double)d, sum); }

// Sum of a double over the wavefront, valid in lane 0: lane i and lane i + 32, then 16, 8, 4, 2, 1, the order of a shuffle-down tree.
// The halves come by lane swaps and row shifts of the vector unit; through the LDS crossbar (ds_bpermute, __shfl_down) each of the
// six steps waits some 100 cycles, and a short kernel waits for the whole chain, twice where its workgroups put the layers'
// sums together.  With that, the layer's range in the chunk's record and one wavefront behind the counters, us a call: fused step, 8
// layers of 256^2, N = 4 6.44 -> 5.95, 13 of 172^2, AdamW 6.97 -> 6.44; average, 9 layers of 145^2, N = 32 8.29 -> 7.62.
template <int CTRL>
__device__ __forceinline__ double row_shifted(double v) {
    const u32x2 w = __builtin_bit_cast(u32x2, v);
    return __builtin_bit_cast(double, u32x2{(unsigned)__builtin_amdgcn_update_dpp(0, (int)w.x, CTRL, 0xf, 0xf, true),
                                            (unsigned)__builtin_amdgcn_update_dpp(0, (int)w.y, CTRL, 0xf, 0xf, true)});
}
__device__ __forceinline__ double wave_sum(double v) {
    u32x2 w = __builtin_bit_cast(u32x2, v);
    auto lo = __builtin_amdgcn_permlane32_swap(w.x, w.x, false, false), hi = __builtin_amdgcn_permlane32_swap(w.y, w.y, false, false);
    v = __builtin_bit_cast(double, u32x2{lo[0], hi[0]}) + __builtin_bit_cast(double, u32x2{lo[1], hi[1]});
    w = __builtin_bit_cast(u32x2, v);
    lo = __builtin_amdgcn_permlane16_swap(w.x, w.x, false, false);
    hi = __builtin_amdgcn_permlane16_swap(w.y, w.y, false, false);
    v = __builtin_bit_cast(double, u32x2{lo[0], hi[0]}) + __builtin_bit_cast(double, u32x2{lo[1], hi[1]});
    constexpr int kRowShl = 0x100;  // lane i takes lane i + n of its row of 16
    v += row_shifted<kRowShl + 8>(v);
    v += row_shifted<kRowShl + 4>(v);
    v += row_shifted<kRowShl + 2>(v);
    v += row_shifted<kRowShl + 1>(v);
    return v;
}

// Sum of a double over the workgroup, in the order of block_sum2.  Result valid in thread 0.
__device__ __forceinline__ double block_sum(double v, double *lds) {
    v = wave_sum(v);
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    if (lane == 0) lds[wave] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 0; w < kThreads / kWave; ++w) r += lds[w];
    }
    __syncthreads();
    return r;
}

// Sums of two doubles over the workgroup in a fixed order: a tree inside each wavefront (wave_sum), then the wavefronts' sums
// added in wavefront order by thread 0.  Results valid in thread 0.  Both trees side by side, one barrier.
template <int WAVES = kThreads / kWave>
__device__ __forceinline__ void block_sum2(double &g, double &m, double (*lds)[WAVES]) {
    g = wave_sum(g);
    m = wave_sum(m);
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    if (lane == 0) {
        lds[0][wave] = g;
        lds[1][wave] = m;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        g = m = 0.0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            g += lds[0][w];
            m += lds[1][w];
        }
    }
}

// The sums of a layer from its partials by a workgroup of kSumThreads, in a fixed order: thread-strided, then the workgroup tree.
// Eight pairs in flight per thread, all that a layer summed in one launch has: the loop is bound by latency.  Up to kThreads partials are
// added to the same bits by THREADS = kThreads: a thread has one of them, and what the other wavefronts would have added are zeros.
constexpr int kSumThreads = 1024;
template <int THREADS>
__device__ __forceinline__ void sum_partials(const double *partials, int64_t c0, int64_t c1, int n_replicas, double *stats, double (*lds)[THREADS / kWave]) {
    static_assert(THREADS == kSumThreads || THREADS == kThreads, "of two widths");
    double g = 0.0, m = 0.0;
    typedef double f64x2 __attribute__((ext_vector_type(2)));
    constexpr int U = THREADS == kSumThreads ? (int)(kStatSingleMax / kSumThreads) : 1;  // pairs in flight per thread
    for (int64_t c = c0 + (int64_t)threadIdx.x; c < c1; c += U * THREADS) {
        f64x2 x[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            x[j] = f64x2{};
            if (c + j * THREADS < c1) x[j] = reinterpret_cast<const f64x2 *>(partials)[c + j * THREADS];
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {  // (both sums are of squares: adding zero changes nothing)
            g += x[j].x;
            m += x[j].y;
        }
    }
    block_sum2<THREADS / kWave>(g, m, lds);
    if (threadIdx.x == 0) {
        stats[0] = g / (double)n_replicas;
        stats[1] = m;
    }
}

// The same sums, of up to kFoldGroup * kFoldGroups partials and in the same order, by one wavefront: its lane stands for the
// threads lane, lane + 64, .. of sum_partials, whose trees have no barrier between them here.
__device__ __forceinline__ void sum_partials_wave(const double *partials, int n, int n_replicas, double *stats) {
    constexpr int kParts = kFoldGroup * kFoldGroups / kWave;
    static_assert(kParts * kWave == kFoldGroup * kFoldGroups && kParts * kWave <= kSumThreads, "a thread of sum_partials has one of these partials");
    const int lane = (int)threadIdx.x;
    double x[kParts], y[kParts];
#pragma unroll
    for (int w = 0; w < kParts; ++w) {
        const int c = w * kWave + lane;
        x[w] = y[w] = 0.0;
        if (c < n) {
            x[w] = __hip_atomic_load(partials + 2 * c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            y[w] = __hip_atomic_load(partials + 2 * c + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    double g = 0.0, m = 0.0;
#pragma unroll
    for (int w = 0; w < kParts; ++w)
        if (w * kWave < n) {
            g += wave_sum(x[w]);
            m += wave_sum(y[w]);
        }
    if (lane == 0) {
        stats[0] = g / (double)n_replicas;
        stats[1] = m;
    }
}

// A workgroup's partial pair of the statistics (valid in thread 0) and, with counters, the layer's sums: the last workgroup of a
// layer to arrive adds the partials up, in the order of sum_partials whichever it is.  Partials and counter are accessed at
// agent scope: the workgroups of a layer run on several XCDs, each with an L2 of its own.  The pair is exchanged, not stored: the
// old values come back from where all XCDs see the new ones, so once they have arrived the counter may be raised without the
// release that would write the XCD's whole L2 back, and the last workgroup reads the pairs past its own L2 without an acquire
// that would empty it (8 layers of 256^2, N = 4, us a call: fused step 6.9 -> 6.3, average 6.1 -> 5.3).  The language orders none of
// this, every access is relaxed; gfx950 does: an agent-scope atomic that has returned was performed where the agent-scope accesses
// of all XCDs meet, the wave waits for the returned values (s_waitcnt, which the empty asm that uses them forces) before it issues
// the counter's atomic, each further atomic depends on the value of the one before, and the loads, of agent scope too, are issued
// behind the branch on the last one's value.  Any other target needs release and acquire at the counters.
// All of it is the first wavefront's, which has the pair: no barrier behind the counters, and the others are done.  PAIRS: partial
// pairs per chunk.
template <int PAIRS>
__device__ __forceinline__ void put_partial(const StatsLaunch &st, int64_t partial, const LayerSums &of, int layer, int n_replicas, double g, double m) {
    if (threadIdx.x >= kWave) return;
    if (st.counters == nullptr) {
        if (threadIdx.x == 0) {
            st.partials[2 * partial] = g;
            st.partials[2 * partial + 1] = m;
        }
        return;
    }
    const int n = PAIRS * of.n;
    const int64_t c0 = (int64_t)PAIRS * of.first;
    int is_last = 0;
    if (threadIdx.x == 0) {
        const double was_g = __hip_atomic_exchange(st.partials + 2 * partial, g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const double was_m = __hip_atomic_exchange(st.partials + 2 * partial + 1, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("" ::"v"(was_g), "v"(was_m) : "memory");  // (waits for them)
        int32_t *const of_layer = st.counters + (int64_t)layer * kFoldStride;
        auto last = [](int32_t *counter, int n) {
            const bool yes = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == n;
            if (yes) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // for the next launch
            return yes;
        };
        const int group = (int)(partial - c0) / kFoldGroup, groups = (n + kFoldGroup - 1) / kFoldGroup;
        const int left = n - group * kFoldGroup, members = left < kFoldGroup ? left : kFoldGroup;
        is_last = last(of_layer + (1 + group) * kFoldLine, members) && (groups == 1 || last(of_layer, groups));
    }
    is_last = __builtin_amdgcn_readfirstlane(is_last);
    asm volatile("" ::: "memory");  // (the loads stay behind the branch)
    if (!is_last) return;
    sum_partials_wave(st.partials + 2 * c0, n, n_replicas, st.stats + 2 * of.pos);
}

// ---------------------------------------------------------------------------------------------------------------
// local update
// ---------------------------------------------------------------------------------------------------------------

// buf = mu*buf + g;  p = p - lr*buf
__device__ __forceinline__ void sgdm_one(float g, float &p, float &buf, const UpdateScalars &s) {
    float b = s.mu * buf;
    b = b + g;
    buf = b;
    const float u = s.lr * b;
    p = p - u;
}

// m = beta1*m + (1-beta1)*g;  v = beta2*v + ((1-beta2)*g)*g;  p = p*decay;  p = p - step_size*(m / (sqrt(v)*rsqrt_bc2 + eps))
__device__ __forceinline__ void adamw_one(float g, float &p, float &m, float &v, const UpdateScalars &s) {
    const float a = s.beta1 * m;
    const float b = s.omb1 * g;
    const float mi = a + b;
    const float c = s.beta2 * v;
    const float d = s.omb2 * g;
    const float e = d * g;
    const float vi = c + e;
    float pi = p * s.decay;
    const float r = __builtin_sqrtf(vi);  // correctly rounded (hipcc default -fhip-fp32-correctly-rounded-divide-sqrt)
    float den = r * s.rsqrt_bc2;
    den = den + s.eps;
    const float q = mi / den;  // IEEE division, correctly rounded
    const float u = s.step_size * q;
    pi = pi - u;
    m = mi;
    v = vi;
    p = pi;
}

template <bool BF16>
struct GradVec;
template <>
struct GradVec<false> {
    typedef float elem;
    typedef f32x4 vec;
    static __device__ __forceinline__ f32x4 widen(f32x4 g) { return g; }
    static __device__ __forceinline__ float widen1(float g) { return g; }
};
template <>
struct GradVec<true> {
    typedef unsigned short elem;
    typedef u16x4 vec;
    static __device__ __forceinline__ f32x4 widen(u16x4 g) {
        return f32x4{bf16_widen(g.x), bf16_widen(g.y), bf16_widen(g.z), bf16_widen(g.w)};
    }
    static __device__ __forceinline__ float widen1(unsigned short g) { return bf16_widen(g); }
};

// The local streams of one run of n elements (wave-uniform pointers to its first element; s1 and mdl unused without AdamW /
// a model copy).
template <bool GBF16>
struct Streams {
    typedef typename GradVec<GBF16>::elem gelem;
    const gelem *g;
    float *p, *s0, *s1;
    unsigned short *mdl;
    int n;
};
// ... and their whole vectors, nv groups of four from element h on.
template <bool GBF16, bool BUF>
struct Vectors {
    Stream<BUF, typename GradVec<GBF16>::elem> g;
    Stream<BUF, float> p, s0, s1;
    Stream<BUF, unsigned short> mdl;
    __device__ __forceinline__ Vectors(const Streams<GBF16> &c, int h, int nv)
        : g(c.g + h, nv), p(c.p + h, nv), s0(c.s0 + h, nv), s1(c.s1 + h, nv), mdl(c.mdl + h, nv) {}
};

template <bool GBF16>
__device__ __forceinline__ Streams<GBF16> chunk_streams(const TensorDesc &td, const UpdateChunk &ch) {
    return {reinterpret_cast<const typename GradVec<GBF16>::elem *>(td.grad) + ch.begin, td.sync + ch.begin, td.state0 + ch.begin,
            td.state1 + ch.begin, td.model + ch.begin, ch.count};
}

// Table-driven AdamW updates from 34 M elements on (in workgroups of the default size) ask for less at a time, so that the memory
// serves fewer rows at once.  Update over separate tensors, us, all in flight / paced: TinyLlama-1.1B 5305 / 5065, Llama blocks
// of 340 M 1254 / 1214, 200 M 977 / 909, GPT-2 small 563 / 553, 28 M 127 / 127, 3 M 16.6 / 17.5.
__device__ __forceinline__ bool long_launch() { return gridDim.x >= 16384; }

// Eq. (5), first case, fused: one pass reads gradient, parameter and optimizer state and writes parameter,
// state and (if present) the bf16 model copy.  ADAM selects AdamW, else SGD with momentum.
template <bool ADAM, bool GBF16, bool MODEL, bool NT, bool BUF>
__device__ __forceinline__ void update_body(const Streams<GBF16> c, const UpdateScalars &s, bool paced = false) {
    typedef GradVec<GBF16> G;
    typedef typename G::vec gvec;
    // the parameters' accesses are aligned; a stream that lies differently against its own vectors takes unaligned ones
    const int h = head_to_16B(c.p, c.n);
    const int nv = (c.n - h) >> 2;
    const Vectors<GBF16, BUF> b(c, h, nv);

    auto compute_store = [&](unsigned i, gvec gv, f32x4 pv, f32x4 av, f32x4 bv) {
        const f32x4 gw = G::widen(gv);
        float G4[4] = {gw.x, gw.y, gw.z, gw.w};
        float P4[4] = {pv.x, pv.y, pv.z, pv.w};
        float A4[4] = {av.x, av.y, av.z, av.w};
        float B4[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (ADAM)
                adamw_one(G4[j], P4[j], A4[j], B4[j], s);
            else
                sgdm_one(G4[j], P4[j], A4[j], s);
        }
        const f32x4 pn{P4[0], P4[1], P4[2], P4[3]};
        b.p.template st<NT>(i, pn);
        b.s0.template st<NT>(i, f32x4{A4[0], A4[1], A4[2], A4[3]});
        if constexpr (ADAM) b.s1.template st<NT>(i, f32x4{B4[0], B4[1], B4[2], B4[3]});
        if constexpr (MODEL) b.mdl.template st<NT>(i, bf16_rne4(pn));
    };

    // Two vectors of every stream in flight; paced (long_launch): the second one's fp32 streams are requested when the first
    // vector has arrived.
    int v = threadIdx.x;
    for (; v + kThreads < nv; v += 2 * kThreads) {
        const unsigned i = 4u * v, j = i + 4u * kThreads;
        const gvec g0 = b.g.template ld<NT>(i);
        const f32x4 p0 = b.p.template ld<NT>(i), a0 = b.s0.template ld<NT>(i);
        f32x4 b0{}, b1{};
        if constexpr (ADAM) b0 = b.s1.template ld<NT>(i);
        const gvec g1 = b.g.template ld<NT>(j);
        if constexpr (ADAM && !BUF) {
            if (paced) asm volatile("" ::"v"(g0), "v"(p0), "v"(a0), "v"(b0), "v"(g1));  // (waits for them)
        }
        const f32x4 p1 = b.p.template ld<NT>(j), a1 = b.s0.template ld<NT>(j);
        if constexpr (ADAM) b1 = b.s1.template ld<NT>(j);
        if constexpr (ADAM && !BUF) __builtin_amdgcn_sched_barrier(0);  // requested before the first vector's arithmetic
        compute_store(i, g0, p0, a0, b0);
        compute_store(j, g1, p1, a1, b1);
    }
    for (; v < nv; v += kThreads) {
        const unsigned i = 4u * v;
        const gvec g0 = b.g.template ld<NT>(i);
        const f32x4 p0 = b.p.template ld<NT>(i);
        const f32x4 a0 = b.s0.template ld<NT>(i);
        f32x4 b0{};
        if constexpr (ADAM) b0 = b.s1.template ld<NT>(i);
        compute_store(i, g0, p0, a0, b0);
    }
    // head and tail together, behind the vectors: only a tensor's first and last chunk have any
    if ((int)threadIdx.x < c.n - 4 * nv) {
        const unsigned i = (int)threadIdx.x < h ? threadIdx.x : 4 * nv + threadIdx.x;
        float pi = ld1(c.p, i), av = ld1(c.s0, i);
        const float gi = G::widen1(ld1(c.g, i));
        if constexpr (ADAM) {
            float bv = ld1(c.s1, i);
            adamw_one(gi, pi, av, bv, s);
            st1(c.s1, i, bv);
        } else {
            sgdm_one(gi, pi, av, s);
        }
        st1(c.p, i, pi);
        st1(c.s0, i, av);
        if constexpr (MODEL) st1(c.mdl, i, bf16_rne(pi));
    }
}

// ---------------------------------------------------------------------------------------------------------------
// local update over dense arenas
// ---------------------------------------------------------------------------------------------------------------

struct DenseArgs {
    const void *g;  // the five streams at the first element of the range, any of arenas that are aligned for 128-bit (bf16: 64-bit) access
    float *p;
    float *s0;
    float *s1;
    unsigned short *mdl;
    int64_t n;  // elements in the range
    int chunk;  // elements per workgroup, a multiple of 1024
    int past;   // elements of the first workgroup's chunk that lie before the range (kLine)
    UpdateScalars s;
};

// ---------------------------------------------------------------------------------------------------------------
// fused synchronisation + update
// ---------------------------------------------------------------------------------------------------------------

// Peers that every replica count served by a fused kernel has: all of them when the kernel is compiled for one count
// (EXACT), half the registers' worth when it serves the counts above NREP / 2 (and none for the smallest such kernel).
template <int NREP, bool EXACT>
constexpr int kPeersAlways = EXACT ? NREP - 1 : (NREP > 4 ? NREP / 2 : 0);

// A wave-uniform value that the compiler takes for a new one: conditions on it are formed where they are used, instead of
// being kept for a whole loop in more scalar registers than there are.
__device__ __forceinline__ int fresh(int v) {
    asm volatile("" : "+s"(v));
    return v;
}

// One group of four elements of a scheduled tensor: raw = the peers' values as they sit in memory (rank order, local rank
// left out), x = the local parameter on entry and the value to store on return, av / bv = optimizer state (updated in
// place).  NREP is the replica count (EXACT) or the largest count that the kernel's registers are laid out for, n the count
// itself.  Rank-order fp32 sum with the local contribution (x, stepped first if UTS, rounded to bf16 if W16) before the peer
// at position lr; the sum starts from -0, which leaves the first term as it is, whatever it is.  One multiply by 1/N;
// statistics in fp64.
template <bool ADAM, bool GBF16, int NREP, bool EXACT, bool STATS, bool W16, bool UTS>
__device__ __forceinline__ void fused_math4(const typename WireVec<W16>::type (&raw)[NREP - 1], typename GradVec<GBF16>::vec gv, f32x4 &x,
                                            f32x4 &av, f32x4 &bv, int n_, int lr_, float inv_n, const UpdateScalars &s, double &gsum,
                                            double &msum) {
    constexpr int ALWAYS = kPeersAlways<NREP, EXACT>;
    const int n = fresh(n_), lr = fresh(lr_);
    auto step4 = [&](f32x4 &q) {
        const f32x4 gw = GradVec<GBF16>::widen(gv);
        float G4[4] = {gw.x, gw.y, gw.z, gw.w};
        float P4[4] = {q.x, q.y, q.z, q.w};
        float A4[4] = {av.x, av.y, av.z, av.w};
        float B4[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (ADAM)
                adamw_one(G4[j], P4[j], A4[j], B4[j], s);
            else
                sgdm_one(G4[j], P4[j], A4[j], s);
        }
        q = f32x4{P4[0], P4[1], P4[2], P4[3]};
        av = f32x4{A4[0], A4[1], A4[2], A4[3]};
        bv = f32x4{B4[0], B4[1], B4[2], B4[3]};
    };
    if constexpr (UTS) step4(x);
    f32x4 loc = x;
    if constexpr (W16) loc = bf16_widen4(bf16_rne4(x));
    typedef WireVec<W16> V;
    f32x4 acc{-0.0f, -0.0f, -0.0f, -0.0f};
#pragma unroll
    for (int j = 0; j < NREP - 1; ++j) {
        if (j == lr) acc = acc + loc;
        if (j < ALWAYS || j < n - 1) acc = acc + V::widen(raw[j]);
    }
    if constexpr (EXACT)  // otherwise n < NREP and the loop has come past the last position
        if (lr == NREP - 1) acc = acc + loc;
    f32x4 m = acc * inv_n;
    if constexpr (STATS) {
        auto add_sq = [](double &sum, f32x4 d) {
            add_square(sum, d.x);
            add_square(sum, d.y);
            add_square(sum, d.z);
            add_square(sum, d.w);
        };
#pragma unroll
        for (int j = 0; j < NREP - 1; ++j) {
            if (j < ALWAYS || j < n - 1) add_sq(gsum, m - widen_again<W16>(raw[j]));
            if (NREP > 16 && j % 8 == 7) __builtin_amdgcn_sched_barrier(0);  // few differences in flight: the peers fill the registers
        }
        add_sq(gsum, m - loc);
        add_sq(msum, m);
    }
    if constexpr (!UTS) step4(m);
    x = m;
}

// Run-time replica counts, those above kFixedReps (the kernels up to there keep all replicas in registers): the first kRegReps
// replicas of a vector stay in registers; a thread parks the rest in LDS while it forms the rank-order sum and reads them back
// for the statistics, so every replica is fetched from memory once.  The staging area is dynamic LDS laid out
// [replica][thread] (each thread only ever touches its own column: no barrier needed, no bank conflicts); with kStageBytes of
// it, stage_threads(staged replicas) threads of the workgroup (whole wavefronts) take part in the vector loop.
constexpr int kStageBytes = 65536;
constexpr int kFixedReps = 32;
constexpr int kRegReps = 16;
inline int stage_threads(int staged) {
    const int t = kStageBytes / 16 / (staged > 0 ? staged : 1) / kWave * kWave;
    return t > kThreads ? kThreads : t;  // at least one wavefront up to DDP_MAX_REPLICAS
}
inline int stage_bytes(int staged) { return staged * stage_threads(staged) * 16; }
static_assert(kStageBytes / 16 / (DDP_MAX_REPLICAS - kRegReps) >= kWave, "the staging area must hold one wavefront at the largest replica count");
static_assert(kRegReps <= kFixedReps, "the run-time loop takes its register replicas without a condition");

// lds_pad: bytes of dynamic LDS requested per workgroup although no kernel uses them.  A CU has 160 KiB, so the pad
// caps how many workgroups are resident per CU, i.e. how wide the window of addresses in flight is.
template <class K, class... Args>
int launch2(K kernel, int64_t grid, int rows, void *stream, int lds_pad, const Args &...args) {
    if (grid <= 0 || rows <= 0) return 0;
    if (grid > 0x7fffffff || rows > 65535) return (int)hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid, (unsigned)rows), dim3(kThreads), (size_t)lds_pad, (hipStream_t)stream, args...);
    return (int)hipGetLastError();
}
template <class K, class... Args>
int launch(K kernel, int64_t grid, void *stream, int lds_pad, const Args &...args) {
    return launch2(kernel, grid, 1, stream, lds_pad, args...);
}

}  // namespace
}  // namespace ddp

#endif
