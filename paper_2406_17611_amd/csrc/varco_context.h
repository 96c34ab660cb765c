// The context behind the C ABI and the host-side helpers its translation units share (varco_api.hip: one partition's
// calls; varco_network.hip: the calls that serve all partitions of a device at once).
#pragma once

#include <initializer_list>
#include <string>
#include <vector>

#include "varco_internal.h"

namespace varco {

struct LayerState {
    uint32_t num = 1, den = 1;
    int32_t k = 0;
    int32_t n_units = 0;
    std::vector<uint16_t> h_units, h_units_inv;   // host copies; uploaded on first device use
    uint16_t* units = nullptr;       // device
    uint16_t* units_inv = nullptr;   // device
    bool ran_forward = false;        // in the current step
    int32_t order = VARCO_ORDER_AGGREGATE_FIRST;
};

struct PartState {
    bool registered = false;
    varco_partition_desc d{};
    SpmmPlan fwd, t_local, t_halo;
    VarcoEdge* edges = nullptr;      // device [nnz]: per-entry {source row, node id}
    int32_t* prow = nullptr;         // device [nnz]: per-entry row of the halo-gradient product buffer
    int32_t* boundary_gid = nullptr; // device [n_boundary]
    int64_t nnz_t_local = 0;         // transposed entries whose row is a local node
    int64_t z_rows = 0;              // 1 + the largest row of the compressed buffer a halo entry refers to
    std::vector<int32_t> t_local_ptr;   // host copy of the transpose's row pointer over the local rows
    int64_t n_returned = 0;          // rows of the registered owner-side map (d.ret_ptr / d.ret_src), 0 without one
};

// All registered partitions as one block of rows in arena order (partition 0's local rows, then partition 1's, ...), for
// the calls that serve them with one launch per kernel. Built by varco_link_partitions; owned by the library.
struct NetState {
    bool linked = false;
    int64_t rows = 0, nnz = 0, nnz_local = 0, nnz_cross = 0, halo_rows = 0, boundary = 0;
    int64_t largest = 0;              // rows of the largest partition
    std::vector<int64_t> row_off, halo_off;   // first arena row / halo row of every partition, and the total
    SpmmPlan fwd;                     // the partitions' forward work lists, one after the other
    VarcoEdge* edges = nullptr;       // [nnz] {arena row, -1} or {compressed-buffer row, node id}
    int32_t* arow = nullptr;          // [nnz] arena row of every entry's column (the owner's row for a halo column)
    float* vals = nullptr;            // [nnz]
    int32_t* prow = nullptr;          // [nnz] row of the product buffer of a halo entry (node order, see NodeItem), else -1
    uint2* t_local = nullptr;         // [nnz_local] transposed local entries {arena row of dM, value bits}, node order
    uint2* t_cross = nullptr;         // [nnz_cross] transposed halo entries, node order, consumers ascending
    NodePlan nodes;
    int32_t* brow = nullptr;          // [boundary] arena rows of the boundary nodes, in compressed-buffer order
    int32_t* bgid = nullptr;          // [boundary] their node ids
    int32_t* zrow_of = nullptr;       // [rows] compressed-buffer row of an arena row, -1 for a row that is no boundary node
};

// Device scratch of the layer calls. Calls issued on different streams may run concurrently, so every
// stream that calls into a context gets a set of its own (up to kMaxStreams), sized from what the
// registered partitions need.
struct Workspace {
    hipStream_t stream = nullptr;
    bool used = false;
    bool captured = false;              // a call on it was recorded into a graph, which goes on using its buffers: they are
    std::vector<float*> kept;           // kept here, not freed, when larger ones take their place
    float* dm = nullptr;        size_t dm_elems = 0;        // dM: n_local x width (elements of the storage type)
    float* spmm = nullptr;      size_t spmm_elems = 0;      // partial rows of split CSR rows
    float* gemm = nullptr;      size_t gemm_elems = 0;      // split-K partial products
    float* prod = nullptr;      size_t prod_elems = 0;      // halo-gradient products: (halo entries) x k elements
    size_t prod_refused = SIZE_MAX;     // floats of rows of whole 64-byte pieces that the device had no room for
    float* w = nullptr;         size_t w_elems = 0;         // converted copies of the weights, one slot per (layer, weight, orientation)
    float* tf = nullptr;        size_t tf_elems = 0;        // transform-first layers: [Y_loc ; Y_halo], (n_local + n_halo) x width[l+1]
    float* hrows = nullptr;     size_t hrows_elems = 0;     // and one record (two words) per halo row
    float* loss = nullptr;      size_t loss_elems = 0;      // the loss's sums per workgroup
    struct WeightTag {          // what a slot holds: made from `h` during step epoch `epoch` in the form `terms`
        const void* h = nullptr;
        uint64_t epoch = 0;
        int32_t terms = -1;
    };
    std::vector<WeightTag> w_tags;
};
constexpr int kMaxStreams = 8;

}  // namespace varco

struct varco_ctx {
    int32_t n_layers = 0, n_parts = 0, conv = 0, dtype = 0;
    int32_t f32_terms = 3;           // fp32 storage: bf16 terms per operand on the matrix cores (0: fp32 instructions)
    uint64_t weight_epoch = 1;       // converted weight copies are reused within an epoch (= a step)
    std::vector<size_t> w_slot;      // offset (bf16 elements) of every slot in a workspace's weight buffer, and the total
    uint64_t key = 0, step = 0;
    std::vector<int32_t> widths, act;
    std::vector<varco::LayerState> layers;
    std::vector<varco::PartState> parts;
    uint64_t* d_step = nullptr;      // device-resident step state (varco_step_table_enable), or null
    uint32_t* d_table = nullptr;     // its key words: 2 per tap address
    varco::Workspace ws[varco::kMaxStreams];
    varco::NetState net;             // all partitions as one block (varco_link_partitions), or empty
    size_t need_dm = 0, need_spmm = 0, need_gemm = 0, need_w = 0;   // what the registered partitions ask for
    int32_t* d_flags = nullptr;      // device word the index checks of a registration report into
    varco_stats stats{};
    VarcoProfiler prof;
    double prof_ms[VARCO_K_COUNT] = {}, prof_bytes[VARCO_K_COUNT] = {}, prof_flops[VARCO_K_COUNT] = {};
    double prof_stream_bytes[VARCO_K_COUNT] = {};
    int64_t prof_launches[VARCO_K_COUNT] = {};
    mutable std::string error;
    mutable hipError_t last_hip = hipSuccess;      // of the last failed runtime call
    double elem_bytes() const { return dtype == VARCO_BF16 ? 2.0 : 4.0; }
    LaunchTag tag(int cls, double bytes, double flops, double stream_bytes = -1.0) {
        LaunchTag t;
        t.prof = prof.on ? &prof : nullptr;
        t.cls = cls, t.bytes = bytes, t.flops = flops, t.stream_bytes = stream_bytes;
        return t;
    }
};

namespace varco {

int32_t hip_fail(const varco_ctx* ctx, hipError_t e, const char* what);

#define VARCO_HIP(ctx, call)                                          \
    do {                                                              \
        hipError_t e_ = (call);                                       \
        if (e_ != hipSuccess) return varco::hip_fail(ctx, e_, #call); \
    } while (0)

// The rule of the kept positions of `layer` (hop > 0: of that hop's exchange inside a K-tap layer) at the context's step.
MaskRule make_rule(const varco_ctx* ctx, int32_t layer, int32_t hop = 0);
// A rule that keeps every element of `width`-wide rows (used for purely dense aggregations).
MaskRule full_rule(int32_t width);
void free_plan(SpmmPlan& p);
void free_network(NetState& net);
// Floats of a workspace's product buffer that the calls on all partitions ask for at the current ratios, and at most at any.
size_t network_prod_need(const varco_ctx* ctx, bool whole, size_t* most);
// Whether the input gradient of layer l can be formed from errors summed at the width of its outputs, and the workspace's
// floats for the rows of a class layer over all partitions: [Y ; Y_z], or dZ, G_loc and G_z (two_terms: each sum as two bf16 numbers).
bool narrow_sums_possible(const varco_ctx* ctx, int32_t l);
size_t class_block_floats(const varco_ctx* ctx, bool two_terms);
enum GemmKind { kGemmF32 = 0, kGemmBf16 = 1, kGemmExpanded = 2 };     // kGemmBf16: as weight gradients
int32_t gemm_split_for(int32_t m, int32_t n, int64_t k, int kind);
int32_t plain_bf16_split(int32_t m, int32_t n, int64_t k);      // the same for bf16 in tiles of 256 x 128, two workgroups per compute unit
int gemm_kind(const GemmArgs& g);
int64_t wgrad_slots(int32_t m, int32_t n, int kind, int products);     // slabs that fill the device once
constexpr int kWeightSlots = 4;       // converted copies held per layer and orientation: of the two taps of a layer, or of the first taps of a K-tap layer
bool prep_slot(varco_ctx* ctx, Workspace& ws, int32_t layer, const void* h, int32_t fi, int32_t fo, bool transpose, int which, bool as_b2,
               GemmArgs& g, PrepJob* job);
hipError_t prep_weight(varco_ctx* ctx, Workspace& ws, int32_t layer, const void* h, int32_t fi, int32_t fo, bool transpose,
                       int which, bool as_b2, hipStream_t st, GemmArgs& g);
int32_t size_all_workspaces(varco_ctx* ctx);
int32_t workspace_for(varco_ctx* ctx, hipStream_t st, Workspace** out, const char* fn);
int32_t check_tables(const varco_ctx* ctx, const char* fn);
int32_t check_layer(const varco_ctx* ctx, int32_t layer, const char* fn);
int32_t split_tap(const varco_ctx* ctx, int32_t* layer, int32_t* hop, const char* fn);
int32_t check_wide_rows(const varco_ctx* ctx, int32_t width, std::initializer_list<const void*> ptrs, const char* fn);

}  // namespace varco
