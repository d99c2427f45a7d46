// Internal declarations shared by the host side of the library (context, tables) and its kernels.
#ifndef DDP_INTERNAL_H
#define DDP_INTERNAL_H

#include <cstdint>
#include <string>
#include <vector>

#include "dreamddp.h"

namespace ddp {

// Record a failure message (on the context, or thread-local when ctx is NULL) and return the code.
int fail(const ddp_ctx *ctx, int code, const std::string &msg);

// The same from a catch block: if recording the message throws as well, the code alone is returned.
inline int fail_nothrow(const ddp_ctx *ctx, int code, const char *msg) noexcept {
    try {
        return fail(ctx, code, msg);
    } catch (...) {
        return code;
    }
}

// No C++ exception crosses the C boundary: the entry points build messages and small host vectors, so a failed host
// allocation (or anything else thrown) is turned into DDP_ENOMEM here.
template <class F>
int guarded(const ddp_ctx *ctx, F &&body) noexcept {
    try {
        return body();
    } catch (...) {
        return fail_nothrow(ctx, DDP_ENOMEM, "host allocation failed");
    }
}

// ---- device tables -------------------------------------------------------------------------------------------
// Everything a kernel needs to find its work is in small read-only tables in HBM, built once when the model
// is registered or the schedule installed.  One workgroup handles one "chunk": a run of elements that lies
// inside one tensor (copy, update) or one layer (mean), so ragged tensor and layer boundaries never fall
// inside a workgroup's vector loop, and per-layer reductions never mix layers.

struct TensorDesc {   // one registered tensor
    float *sync;      // fp32 params or master weights
    uint16_t *model;  // bf16 model copy or nullptr
    void *grad;       // fp32 or bf16
    float *state0;    // momentum / first moment
    float *state1;    // second moment or nullptr
    int64_t numel;
    int32_t past;     // elements of its first cache line (kLine) before it
};

// Inside a run, chunks end at multiples of kLine elements, counted where the run's fp32 streams have a 256-byte boundary (over
// dense arenas from the arenas' first element): a cache line of any stream, 128 bytes of 16-bit elements too, then belongs to one
// chunk.  Lines that two workgroups shared were read twice and written in parts, by two XCDs' L2s: 16 layers of 1533^2, AdamW
// with bf16 gradients and copy, N = 8, fused: 226 us with chunks that end at multiples of four elements, 218 so; average of N = 16 over layers of 3001^2: 207 and 200.
// Where flat element 0 meets a layer that starts inside a line, the peers' lines are shared instead, most of the bytes from about 24
// replicas on: 4 layers of 1448^2, layer by layer, fp32, N = 4 69.3 and 65.3, N = 32 84.0 and 86.3.
constexpr int kLine = 64;

struct UpdateChunk {  // local_update: elements [begin, begin+count) of run `run` (a tensor; over dense arenas a whole layer)
    int64_t begin;
    int32_t run;
    int32_t count;
};

// pack / unpack: `count` elements at `sync`, in run `run` of the update table, <-> flat elements [flat_begin, +count).  The address is
// in the record: a workgroup's first load waits for one table, not for a chunk and then a tensor.
struct CopyChunk {
    float *sync;
    int64_t flat_begin;
    int32_t run;
    int32_t count;
};

// A layer of the slot as its statistics are put together: `n` chunks from `first` on, each with its partial sums.  Every chunk's
// record has it, so that a workgroup has it at hand with its first load and not, behind its last store, from a table of its own.
struct LayerSums {
    int32_t pos;  // position of the layer in the slot
    int32_t first, n;
};

struct alignas(32) MeanChunk {  // partial_average: flat elements [begin, +count), all inside one layer of the slot
    int64_t begin;
    int32_t count;
    int32_t partial;  // where this chunk's partial sums go: its index in flat order, whatever the dispatch order
    LayerSums of;
};

struct alignas(32) RunSlot {  // a run of the update table in one slot
    int64_t flat0;            // first flat index, -1 if it is not scheduled
    int32_t layer;
    LayerSums of;  // chunks of the fused step
};

// One launch of the fused step over dense arenas: consecutive pieces of the model, each part of a scheduled layer or of a run
// of unscheduled ones.  Workgroup (x, y) takes chunk x of piece y, counted from the multiple of kLine at or below the piece's
// first element; it writes its partial pair at partials[2 * (pbase + x)].
constexpr int kMaxPieces = 32;  // the pieces travel with the launch's arguments
struct Piece {
    int64_t begin;  // first element of the arenas
    int64_t flat0;  // its flat index, -1 if the piece is not scheduled
    int32_t count;  // elements
    int32_t pbase;
    int32_t pos, layer;  // position of the layer in the slot, and the layer
    int32_t first, n;    // LayerSums
};
struct DensePass {
    int width;          // chunks of the widest piece; 0: a plain update of elements [begin, end)
    int n_pieces;
    int64_t begin, end;
    Piece pieces[kMaxPieces];
};

// A slot as the fused step cuts it, in one of its two sizes of chunk.
struct FusedPlan {
    RunSlot *d_run_slot = nullptr;         // per run of the update table
    std::vector<int32_t> update_ranges;    // per layer of the slot: [first, last) chunk of the fused step (registration order), whose
    int32_t *d_update_ranges = nullptr;    // places its partials have, table-driven or table-free
    int64_t max_update_partials = 0;       // largest count of a layer
    std::vector<DensePass> dense_passes;   // dense arenas: the launches of the fused step over the whole model
    bool table_first = false;              // ... for which the table's single launch is the better one
};

struct SlotTables : FusedPlan {  // (the plan in the update table's own chunks)
    // host copies (introspection, validation)
    std::vector<int32_t> layers;       // layer ids in flat order
    std::vector<int64_t> layer_begin;  // n_layers + 1 flat offsets
    std::vector<int32_t> tensors;      // tensor ids in flat order
    std::vector<int64_t> tensor_off;
    int64_t numel = 0;
    // device tables
    // each covers the slot in chunks that end on the lines (kLine) of what is written; one table where those are the same, else
    // one allocation, d_pack's
    CopyChunk *d_pack = nullptr, *d_unpack = nullptr;
    int64_t n_pack = 0, n_unpack = 0;
    MeanChunk *d_mean = nullptr;
    int64_t n_mean = 0;
    int32_t *d_layer_ranges = nullptr;     // per layer of the slot: [first, last) mean chunk
    int64_t max_mean_partials = 0;         // largest count of a layer
    std::vector<int32_t> layer_pos;        // [L] layer -> position in this slot, -1 if not scheduled
    FusedPlan halves;                      // ... and in halves of those chunks (ddp_ctx::halves); its device tables lie behind the others
};

// Counters of a layer whose workgroups add the statistics up themselves, in 32-bit words: one per group of kFoldGroup partials
// and one over the groups, each in a cache line of its own.  Arrivals at one counter are served
// one after the other, 20-25 ns each: 128 of them on one 6.3 us, in groups 5.7 (average, N = 4).
constexpr int kFoldGroup = 32, kFoldGroups = 20, kFoldLine = 32, kFoldStride = (1 + kFoldGroups) * kFoldLine;

// How the per-layer statistics of a launch are put together from its workgroups' partial pairs.
struct StatsLaunch {
    double *partials;   // nullptr: no statistics
    double *stats;      // [positions][2]
    int32_t *counters;  // kFoldStride per layer, zero between launches: the layer's last workgroup adds the partials up
                        // in the kernel itself; nullptr: a launch of its own follows (launch_stats)
};

// ---- launchers (ddp_kernels_*.hip) -------------------------------------------------------------------------------
constexpr int kCutReps = 12, kCutReps16 = 17;  // fewest replicas, fp32 and bf16, whose average may cut chunks (mean_cut)
struct MeanLaunch {
    const void *x[DDP_MAX_REPLICAS];  // replicas in rank order (fp32, or bf16 when wire16)
    bool wire16;
    int n_replicas;
    float inv_n;
    float *out;
    const MeanChunk *chunks;
    int64_t n_chunks;
    int cut;                   // elements after which a chunk is cut in two, a workgroup each; 0: not cut
    StatsLaunch st;            // two partial pairs per chunk where chunks are cut
    bool nontemporal;
    int lds_pad;
};

struct UpdateScalars {
    float lr, mu;                                                // SGD-m
    float beta1, beta2, omb1, omb2, decay, step_size, rsqrt_bc2, eps;  // AdamW
};

int launch_copy(bool unpack, const TensorDesc *runs, const CopyChunk *chunks, int64_t n_chunks, float *flat, bool with_model,
                bool nontemporal, int lds_pad, void *stream);
int launch_mean(const MeanLaunch &a, void *stream);
// Per-layer statistics from per-chunk partials: layer l of n_layers adds the `pairs` partials of each of the chunks
// [ranges[2l], ranges[2l+1]) in a fixed order through kStatSlices slice sums (slice_sums: [n_layers][kStatSlices][2]) into
// stats[2l], stats[2l+1].
// With at most kStatSingleMax partials in any of the layers (max_partials_per_layer, an upper bound is enough) one launch
// does it all; beyond that the two stages.
constexpr int kStatSlices = 64;
constexpr int64_t kStatSingleMax = 8192;
int launch_stats(const double *partials, double *slice_sums, const int32_t *ranges, int pairs, int n_layers, int n_replicas, double *stats,
                 int64_t max_partials_per_layer, void *stream);
int launch_pack16(const CopyChunk *chunks, int64_t n_chunks, uint16_t *flat16, bool nontemporal, int lds_pad, void *stream);
// The fused step: what both forms of the kernel take ...
struct FusedLaunch {
    const void *x[DDP_MAX_REPLICAS - 1];  // the N-1 peers in rank order; fp32, or bf16 when wire16
    bool wire16;
    bool update_first;  // Eq. (5) as printed: the local value takes the optimizer step before it is averaged
    int n_replicas, local_rank;
    float inv_n;
    int kind, grad_dtype;
    bool with_model;
    UpdateScalars s;
    StatsLaunch st;
    int lds_pad;
    bool pairs;  // two vectors of all streams in flight per thread (takes_pairs)
};
// ... the table-driven one, over chunks of the update table ...
struct FusedTable : FusedLaunch {
    const TensorDesc *runs;
    const UpdateChunk *chunks;
    int64_t n_chunks;
    const RunSlot *run_slot;
    const int32_t *run_chunk_base;
    int chunk_elems;
    bool halved;  // two workgroups a chunk
};
int launch_fused(const FusedTable &f, void *stream);
// The update over tensors that lie back to back in every stream: the range's first element in each stream (any element of arenas
// that are aligned for 128-bit access, bf16 ones for 64-bit), its length, the elements per workgroup and where in a line (kLine) it starts.
struct DenseLaunch {
    const void *g;
    float *p, *s0, *s1;
    uint16_t *mdl;
    int64_t n;
    int chunk, past;
};
int launch_update_dense(int kind, int grad_dtype, bool with_model, const DenseLaunch &d, const UpdateScalars &s, bool nontemporal,
                        int lds_pad, void *stream);
// ... and the one over dense arenas (d: the arenas' first elements; d.n is not used).
struct FusedDense : FusedLaunch {
    DenseLaunch d;
    int plain;  // elements per workgroup of an unscheduled piece
    const DensePass *pass;
};
int launch_fused_dense(const FusedDense &f, void *stream);
int launch_update(int kind, int grad_dtype, bool with_model, const TensorDesc *runs, const UpdateChunk *chunks,
                  int64_t n_chunks, const UpdateScalars &s, bool nontemporal, int lds_pad, void *stream);

// Shared body of the averaging entry points (ddp_context.hip).  scratch == nullptr: the context's reduction scratch.
int partial_average_impl(ddp_ctx *ctx, const char *who, bool wire16, int slot, const void *flat_local, const void *const *peers, int N,
                         int local_rank, float *flat_out, double *layer_stats, void *stream, double *scratch, int64_t scratch_bytes);

// The fixed reduction scratch of ddp_partial_average_static on the current device (ddp_noalloc.hip): resolves the
// device address of the library's static array once per device.  Call with `device` current.
int static_scratch_for(const ddp_ctx *ctx, int device, double **ptr);

}  // namespace ddp

struct ddp_ctx {
    int device = 0;
    mutable std::string err;
    // options
    int64_t update_chunk = 2048, mean_chunk = 2048, copy_chunk = 2048;
    bool nontemporal = true;
    int dispatch_ways = 1;
    int lds_per_cu = 163840, lds_per_wg_max = 65536;  // what the device reports (ddp_create); gfx950 values until then
    int update_lds = 64512, mean_lds = 64512, copy_lds = 26112;  // dynamic-LDS pad per workgroup: caps residency per CU (2 / 2 / 6)
    bool update_chunk_set = false, update_lds_set = false;  // ... given by the caller, whatever the model's size (small_model)
    bool mean_lds_set = false;  // the average's residency was given by the caller, whatever the replica count
    // model
    bool registered = false;
    int64_t run_chunk = 2048;  // elements per chunk of the update table and the table-free kernels: update_chunk, or small_model's
    bool halves = false;       // the fused step may have a workgroup for each half of such a chunk (takes_halves, call_takes_halves)
    bool small = false;
    int L = 0, T = 0;
    int param_dtype = DDP_F32, grad_dtype = DDP_F32;
    bool has_state1 = false;
    std::vector<int32_t> layer_of;
    std::vector<int64_t> numel;
    std::vector<ddp::TensorDesc> tensors;
    std::vector<int32_t> layer_first_tensor;  // L + 1
    std::vector<int64_t> tensor_elem_off;     // T + 1: elements before each tensor, registration order
    bool dense = false;      // tensors lie back to back in every stream and the streams' starts are vector-aligned
    bool dense_path = true;  // option: use the table-free kernels where `dense` allows it
    std::vector<int32_t> layer_first_run;  // L + 1: runs of the update table
    std::vector<ddp::TensorDesc> runs;
    ddp::TensorDesc *d_runs = nullptr;
    ddp::UpdateChunk *d_update = nullptr;
    int64_t n_update = 0;
    std::vector<int32_t> run_chunk_base;  // first update chunk of each run, registration order, and their number
    int32_t *d_run_chunk_base = nullptr;
    // schedule
    int H = 0;
    std::vector<ddp::SlotTables> slots;
    double *d_partials = nullptr;  // reduction scratch for per-layer statistics: one partial pair per chunk ...
    double *d_slice_sums = nullptr;  // ... followed by 64 slice sums per layer (same allocation)
    int32_t *d_counters = nullptr;   // ... and the layers' counters, zero between launches (StatsLaunch)
    int cus = 256;                   // compute units of the device (ddp_create)
    int64_t partials_cap = 0;
    double *static_scratch = nullptr;  // this device's copy of the library's fixed scratch array (ddp_partial_average_static)
    std::string static_scratch_err;    // why it could not be resolved, if it could not
};

#endif
