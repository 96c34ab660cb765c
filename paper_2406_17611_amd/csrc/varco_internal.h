// Internal declarations shared by the translation units of libvarco (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "varco.h"

// Brackets kernel launches with HIP events on the launch stream (see varco_profile_enable). When a launch
// follows the previous bracketed launch on the same stream, the previous stop event doubles as its start
// event: an event record is a marker in the queue that keeps the next kernel from starting early, so half as
// many markers disturb the run half as much.
struct VarcoProfiler {
    struct Rec {
        int cls;
        int start, stop;     // indices into `events`
        double bytes, flops;
        double stream_bytes;   // bytes when no cache serves a re-read (one source row per entry); = bytes for streaming kernels
    };
    bool on = false;
    std::vector<Rec> recs;
    std::vector<hipEvent_t> events;   // recorded since the last read
    std::vector<hipEvent_t> pool;     // free
    hipStream_t last_stream = nullptr;
    int last_stop = -1;               // event index of the last stop record, still the tail of last_stream's queue
    int record(hipStream_t st) {
        hipEvent_t e = nullptr;
        if (!pool.empty()) {
            e = pool.back();
            pool.pop_back();
        } else {
            (void)hipEventCreate(&e);
        }
        (void)hipEventRecord(e, st);
        events.push_back(e);
        return int(events.size()) - 1;
    }
    void begin(int cls, hipStream_t st, double bytes, double flops, double stream_bytes = -1.0) {
        if (!on) return;
        const int start = (last_stop >= 0 && last_stream == st) ? last_stop : record(st);
        recs.push_back(Rec{cls, start, -1, bytes, flops, stream_bytes < 0 ? bytes : stream_bytes});
        last_stop = -1;
    }
    void end(hipStream_t st) {
        if (!on) return;
        recs.back().stop = record(st);
        last_stream = st;
        last_stop = recs.back().stop;
    }
    // An untimed launch went to `st`: the next bracket on it needs a start event of its own.
    void interrupt() { last_stop = -1; }
};
// Work attributed to one launch, handed from the API layer to the launchers.
struct LaunchTag {
    VarcoProfiler* prof = nullptr;
    int cls = 0;
    double bytes = 0, flops = 0;
    double stream_bytes = -1;   // < 0: same as bytes
    void begin(hipStream_t st) const { if (prof) prof->begin(cls, st, bytes, flops, stream_bytes); }
    void begin_as(int other, hipStream_t st, double other_bytes) const { if (prof) prof->begin(other, st, other_bytes, 0); }
    void end(hipStream_t st) const { if (prof) prof->end(st); }
};

// Records `msg` as the last error of ctx (or of the process when ctx is null) and returns `code`.
int32_t varco_fail(const varco_ctx* ctx, int32_t code, const char* msg);

// The kept positions of a node vector (Definition 1 / Appendix A of the paper, with this library's keyed
// rule): pi_v(j) = (a_v * j + b_v) mod width, j < k, where b_v = floor(h1 * width / 2^32), a_v =
// units[floor(h2 * n_units / 2^32)], h1 = mix(v ^ s0), h2 = mix(h1 ^ s1), and (s0, s1) are derived on the
// host from (key, step, layer). k == width means the identity. Passed by value to kernels.
struct MaskRule {
    uint32_t s0, s1;
    uint32_t width, k;
    uint32_t n_units;
    uint32_t width_magic;       // floor(2^32 / width), 0xFFFFFFFF for width 1
    const uint16_t* units;      // device: ascending multipliers coprime with width
    const uint16_t* units_inv;  // device: their inverses modulo width
    const uint32_t* words;      // device, or null: when set, (s0, s1) are read from here instead (step table)
};

// One unit of SpMM work: entries [e0, e1) of CSR row `row`; dst < 0 writes the output row directly, else
// the partial sum goes to slot dst of the partial buffer (rows longer than the chunk length are split).
struct SpmmItem {
    int32_t row, e0, e1, dst;
};
// A split row and the contiguous range of partial slots that add up to it.
struct SpmmSplit {
    int32_t row, first, count, pad;
};
struct SpmmPlan {
    int32_t n_items = 0, n_splits = 0, n_partials = 0;
    // dense-only blocks with very short rows: rows short_r0 .. short_r0 + short_rows - 1 with at most short_max_len
    // entries are not on `items` but taken four to a wavefront, straight from the row pointer (device, borrowed)
    int32_t short_r0 = 0, short_rows = 0, short_max_len = 0;
    const int32_t* short_rowptr = nullptr;
    SpmmItem* items = nullptr;    // device
    SpmmSplit* splits = nullptr;  // device
};

// Per-entry record of a partition's row block, derived by the library at registration: a local column
// becomes {local row, -1}; a halo column becomes {row of that node in the concatenated compressed buffer,
// node id} (the id keys the node's kept positions).
struct VarcoEdge {
    int32_t src, gid;
};

// Backward aggregation seen from the nodes of all partitions at once: node row `row` of the arena receives
//   sum of its local entries [l0, l1) (dense rows of dM) + its kept positions of the sum of its cross entries [c0, c1),
// both ranges in node order. When a range is longer than a wavefront should take, it is cut into pieces whose partial
// sums lie in slots [l0, l1) / [c0, c1) of the partial buffer instead (flags).
struct NodeItem {
    int32_t row;
    uint32_t gid;
    int32_t l0, l1, c0, c1;
    int32_t flags, pad;
};
enum { VARCO_NODE_LOCAL_SPLIT = 1, VARCO_NODE_CROSS_SPLIT = 2 };
struct NodePlan {
    int32_t n_nodes = 0, n_pieces = 0;     // pieces: row = 0 for a local range, 1 for a cross range; dst = its slot
    int32_t n_whole = 0;                   // the nodes without pieces come first
    NodeItem* nodes = nullptr;             // device
    SpmmItem* pieces = nullptr;            // device
};

// `dtype` (VARCO_F32 / VARCO_BF16) is the storage type of every activation, message and gradient buffer
// passed as void*; sums are formed in fp32 and rounded to nearest even on store.
hipError_t varco_launch_compress(int dtype, const MaskRule& rule, const int32_t* gids, const int32_t* rows, int64_t n_rows,
                                 const void* x, int64_t ldx, void* z, hipStream_t stream, const LaunchTag& tag);
hipError_t varco_launch_decompress(int dtype, const MaskRule& rule, const int32_t* gids, const int32_t* rows,
                                   int64_t n_rows, const void* z, void* x, int64_t ldx, int accumulate,
                                   hipStream_t stream, const LaunchTag& tag);

// x[rows[b], pi_v(j)] += sum_{e in [ptr[b], ptr[b+1])} returned[src[e] * k + j], v = gids[b].
hipError_t varco_launch_accumulate_returned(int dtype, const MaskRule& rule, const int32_t* gids, const int32_t* rows,
                                            int64_t n_rows, const int32_t* ptr, const int32_t* src, const void* returned,
                                            void* x, int64_t ldx, hipStream_t stream, const LaunchTag& tag);

hipError_t varco_launch_calibration_copy(void* dst, const void* src, int64_t bytes, hipStream_t stream);
hipError_t varco_launch_sum_gradients(float* dst, const float* src, int64_t n, hipStream_t stream);

// out[s] = {(a << 16) | b of node gids[s] under `rule` (1 << 16, the identity, when every element is kept), zrow[s]}:
// element j of halo row s sits at position (a j + b) mod width; the per-row records of HaloTransform. zrow null: row s.
hipError_t varco_launch_halo_rows(const MaskRule& rule, const int32_t* gids, const int32_t* zrow, int32_t n, uint2* out,
                                  hipStream_t stream);

// Device-resident step state: *d_step = the step (set to `value` when set != 0, else incremented), and
// table[2 t], table[2 t + 1] = the two key words of tap address t (0 .. 255) for that step and `key`.
hipError_t varco_launch_step_table(uint64_t* d_step, uint32_t* table, uint64_t key, int set, uint64_t value,
                                   hipStream_t stream);

// Index checks at registration: bits set in *flags (device int32, zeroed by the caller) by the first failed check
// of each kind.
enum {
    VARCO_BAD_COLUMN_RANGE = 1, VARCO_BAD_COLUMN_ORDER = 2, VARCO_BAD_TROW_RANGE = 4, VARCO_BAD_TROW_ORDER = 8,
    VARCO_BAD_TRANSPOSE = 16, VARCO_BAD_ID = 32, VARCO_BAD_BOUNDARY = 64, VARCO_BAD_RETURN_MAP = 128,
    VARCO_BAD_LINK = 256
};
hipError_t varco_launch_validate_partition(const varco_partition_desc& d, int32_t* flags, hipStream_t stream);

hipError_t varco_launch_build_edges(const int32_t* colidx, int64_t nnz, int32_t n_local, const int32_t* halo_zrow,
                                    const int32_t* halo_gid, VarcoEdge* edge, hipStream_t stream);

// Where a launch finds the owners' rows: the row of `dense` of every entry's column, and row and node of every row of z.
// jobs: weight copies to be made by the launch as well (at most kFewPrepJobs).
struct PrepJob;
struct SpmmOwners {
    const int32_t *arow, *brow, *bgid;
    PrepJob* jobs;
    int n_jobs;
};

// out[row - row_base, :] = sum_e vals[e] * source_row(e) for the rows of `plan`, width = rule.width.
//   edge != null (forward): entry e reads dense + edge[e].src * width when edge[e].gid < 0, else the k kept
//       elements z[edge[e].src * k + j], which land at pi_gid(j) (a full row of z when k == width);
//   edge == null (transposed, all dense): entry e reads dense + colidx[e] * width.
// partial: workspace of plan.n_partials * width floats (fp32 for either storage type). z_rows: rows of z (0 when
// unknown); a compressed buffer below 4 GiB is addressed with 32-bit offsets.
hipError_t varco_launch_spmm(int dtype, const SpmmPlan& plan, const VarcoEdge* edge, const int32_t* colidx,
                             const float* vals, const void* dense, const void* z, int64_t z_rows, const MaskRule& rule,
                             void* out, int32_t row_base, float* partial, hipStream_t stream, const LaunchTag& tag,
                             const SpmmOwners* owners = nullptr);
// Whether one launch may aggregate and write the messages (`owners`: z is written, not read) instead of varco_launch_compress before it.
bool varco_spmm_owners_pay(int dtype, const SpmmPlan& plan, const MaskRule& rule, int64_t rows, int64_t cross, int64_t boundary, const void* dense,
                           const void* out, const void* partial);

// prow[e] = position of forward entry e among the halo entries of the transposed order (-1 for local entries).
hipError_t varco_launch_build_prow(const int32_t* rowptr, const int32_t* colidx, int32_t n_local,
                                   const int32_t* t_rowptr, const int32_t* t_colidx, int32_t* prow, hipStream_t stream);

// out[s, j] = sum over local rows i of S[i, halo s] * dm[i, pi_v(j)], j < k (the halo rows of the transposed
// aggregation, produced directly in compressed form) in two streaming passes through the product buffer
// `prod` ((halo entries) x k elements of the storage type). prod_base = transposed position of the first halo entry.
hipError_t varco_launch_halo_grad(int dtype, const SpmmPlan& fwd_plan, const SpmmPlan& t_halo_plan, const VarcoEdge* edge,
                                  const float* vals, const int32_t* prow, int32_t prod_base, const void* dm,
                                  const MaskRule& rule, void* prod, void* out, int32_t row_base, float* partial,
                                  hipStream_t stream, const LaunchTag& tag, const LaunchTag& sum_tag);

// Elements between the rows of a product buffer of the library's own: k rounded up to whole 16-byte stores, and above 32 bytes to 64 bytes, so
// that no row shares a 64-byte piece of memory with another: rows are written in row order and lie in node order, and a shared piece is written
// twice, in parts. (An odd k, as compression schedules give, otherwise means element stores: 31 of 256 fp32 values per message, 1.75 million
// messages, 272 us against 108. Whole steps with rows rounded to 16 bytes / to 64, us, 200,003 nodes, two hidden layers of 256 fp32: rows of 36 bytes
// 1,798 / 1,719, 68 1,854 / 1,757, 132 2,032 / 1,919, 180 1,917 / 1,928, 260 2,274 / 2,157; of 512 bf16: 36 2,057 / 1,982, 68 2,104 / 2,000, 132
// 2,285 / 2,163, 228 2,386 / 2,227. To 32 bytes: as 16 where that leaves half a piece. To 128 above 128: 1 % slower.) The buffer grows by up to 1.8 times
// (a third beyond the next 16 bytes); `whole` false, to 16 bytes, where that leaves no room for it. The sums are the same either way.
inline int32_t varco_product_pitch(const MaskRule& rule, int elem_bytes, bool whole) {
    const uint32_t unit = (whole && rule.k * uint32_t(elem_bytes) > 32 ? 64u : 16u) / uint32_t(elem_bytes), up = (rule.k + unit - 1) / unit * unit;
    return int32_t(up <= rule.width ? up : rule.k);
}
// First pass of the product form: prod[prow[e] * pitch + j] = vals[e] * dm[row of e, pi_v(j)], j < k, for the halo entries of
// `fwd_plan` (and up to the pitch, which is at most the width).
hipError_t varco_launch_halo_products(int dtype, const SpmmPlan& fwd_plan, const VarcoEdge* edge, const float* vals, const int32_t* prow,
                                      const void* dm, const MaskRule& rule, void* prod, int32_t pitch, hipStream_t stream, const LaunchTag& tag);

// Bytes of a row above which products may be formed (products_pay draws the lines, from here on); there are no kernels for the products of shorter ones.
constexpr int kProductRowBytes = 320;

// How the cross entries of varco_launch_node_sum are taken: not at all (k = 0); summed from the product buffer (rows of
// `pitch` elements, whole 16-byte pieces, already weighted; for rows of more than kProductRowBytes); gathered as whole rows of dm and kept only at the node's positions; gathered as whole rows (k = width).
enum VarcoCross { kCrossNone = 0, kCrossProducts = 1, kCrossMasked = 2, kCrossFull = 3 };
// out[row, :] (+)= sum of local entries + cross entries for every node of the plan (see NodeItem). partial: one
// width-float row per piece.
hipError_t varco_launch_node_sum(int dtype, const NodePlan& plan, const uint2* t_local, const uint2* t_cross, const void* dm,
                                 const void* prod, int32_t pitch, const MaskRule& rule, VarcoCross cross, void* out, bool add_old, float* partial,
                                 hipStream_t stream, const LaunchTag& tag);

// Set-up kernels of the network block (kernels_network.hip); *flags collects VARCO_BAD_* bits.
struct LinkPartition {           // one partition inside the block
    varco_partition_desc d;
    int64_t row_off, ent_off, local_off;
};
hipError_t varco_launch_link_edges(const LinkPartition& p, const int32_t* prow_part, const int32_t* owner_row, const int32_t* prod_start,
                                   VarcoEdge* edges, int32_t* arow, float* vals, int32_t* prow, hipStream_t stream);
hipError_t varco_launch_link_halo(const LinkPartition& p, int32_t* halo_len, int32_t* halo_gid, int32_t* halo_zrow, hipStream_t stream);
hipError_t varco_launch_link_owner(const LinkPartition& p, int64_t halo_total, const int32_t* halo_len, const int32_t* halo_gid,
                                   const int32_t* halo_zrow, int32_t* owner_row, int32_t* cross_len, int32_t* brow, int32_t* bgid,
                                   int32_t* zrow_of, int32_t* flags, hipStream_t stream);
hipError_t varco_launch_link_starts(const LinkPartition& p, const int32_t* halo_len, const int32_t* cross_ptr, int32_t* prod_start,
                                    hipStream_t stream);
hipError_t varco_launch_link_transposed(const LinkPartition& p, const int32_t* prod_start, uint2* t_local, uint2* t_cross, hipStream_t stream);
hipError_t varco_launch_link_items(const SpmmPlan& part, int32_t row_off, int32_t ent_off, int32_t slot_off, int32_t item_off,
                                   int32_t split_off, const SpmmPlan& out, hipStream_t stream);

// Forms of weight copies beside a number of bf16 terms (varco_launch_prep_weights).
constexpr int kHalfTerms = 4, kExactTerms = 5;

// C (+)= op(A) op(B) in fp32 on the matrix cores, row-major everywhere.
struct GemmOperand {
    const void* ptr = nullptr;    // matrix as stored
    const void* gate = nullptr;   // optional, same shape and type: elements are used only where gate > 0 (ReLU mask)
    int dtype = VARCO_F32;        // storage type of ptr and gate
    int64_t ld = 0;
    bool transposed = false;      // false: stored [rows=M or K][cols=K or N]; true: stored the other way round
};
struct GemmArgs {
    int32_t m = 0, n = 0, k = 0;
    GemmOperand a, b;             // first product
    GemmOperand a2, b2;           // optional second product summed into the same C (k2 reduction length)
    int32_t k2 = 0;
    // optional bf16 copies of B / B2 laid out [n][pitch] (reduction index contiguous, zero-padded to the pitch),
    // made by varco_launch_prep_weights: with them, bf16 activations go through the bf16 matrix-core kernel
    const void* b_prep = nullptr;
    const void* b2_prep = nullptr;
    int64_t b_prep_ld = 0, b2_prep_ld = 0;
    // fp32 operands on the 16-bit matrix cores: 0 = no (fp32 matrix instructions); 2 or 3 = in the transform each operand is
    // expanded into that many bf16 terms, in the gradients into two scaled fp16 terms, and b_prep / b2_prep are expanded copies made
    // by varco_launch_prep_weights (by tile and stage, `plane` elements per term in all)
    int32_t f32_terms = 0;
    int64_t b_prep_plane = 0, b2_prep_plane = 0;
    int32_t bf16_terms = 1;       // bf16 operands: form of b_prep and b2_prep, one rounded copy (1) or kExactTerms
    bool b_halves = false;        // b_prep (and b_dual_prep) hold two scaled fp16 terms instead (kHalfTerms)
    void* c = nullptr;
    int c_dtype = VARCO_F32;
    int64_t ldc = 0;
    bool accumulate = false;      // C += instead of C =
    bool relu = false;            // C = max(., 0)
    int32_t split_k = 1;          // > 1: partial products into `partial` then reduced in a second kernel
    float* partial = nullptr;     // split_k * m * n floats
    // A second product of the same shape that shares an operand, formed by the same launch (varco_gemm_dual_usable): with A
    // transposed another A against the same B (the two taps' weight gradients), else another B against the same A (the two
    // taps' input gradients); its result goes to c_dual, its partial products behind the first product's.
    const void* a_dual = nullptr;
    const void* b_dual = nullptr;         // the weights as given, and their copy (same layout as b_prep)
    const void* b_dual_prep = nullptr;
    void* c_dual = nullptr;
    int32_t* deferred = nullptr;  // when set: the number of partial products written to `partial` (1: C holds the result); the
                                  // caller sums them (varco_launch_gemm_reduce_jobs)
};
hipError_t varco_launch_gemm(const GemmArgs& g, hipStream_t stream, const LaunchTag& tag);
// c (+)= sum over s < slabs of partial[s][m x n], in a fixed order (the second pass of every split reduction).
hipError_t varco_launch_gemm_reduce(const float* partial, int32_t slabs, int32_t m, int32_t n, float* c, int64_t ldc,
                                    bool accumulate, hipStream_t stream, const LaunchTag& tag);

// The same for several products in one launch; splits <= 1 are skipped. At most kMaxReduceJobs jobs.
struct ReduceJob {
    const float* partial;
    float* c;
    int64_t ldc;
    int32_t splits, m, n, first_block;
};
constexpr int kMaxReduceJobs = 2 * VARCO_MAX_LAYERS;
hipError_t varco_launch_gemm_reduce_jobs(ReduceJob* jobs, int n, bool accumulate, hipStream_t stream, const LaunchTag& tag);

// The halo rows of a partition as an exchange delivered them (kernels_halo_transform.hip; bf16 storage): row s holds
// the k elements z[rec[s].y * k + j] at positions (a j + b) mod width, (a << 16) | b = rec[s].x, of a width-wide row
// that is zero elsewhere. width: a multiple of 16, at most 512; fo <= 64 columns on the other side of the weights.
struct HaloTransform {
    const void* z = nullptr;
    const uint2* rec = nullptr;
    int32_t n = 0;
    uint32_t width = 0, k = 0, width_magic = 0;
    int32_t fo = 0;
    int32_t ldy = 0;              // elements between rows of y / dy (0: fo)
};

constexpr int kHaloTransformGroups = 512;      // workgroups that are resident at a time: two per compute unit
// Most shares of a weight gradient over n rows: whole rounds of workgroups, none summing more than 1,024 rows (the error of an
// fp32 sum grows with the square root of its length).
inline int64_t varco_halo_transform_shares(int64_t n) {
    constexpr int64_t round = int64_t(kHaloTransformGroups) * 1024;
    return kHaloTransformGroups * (n > round ? (n + round - 1) / round : 1);
}

// The same layer for all partitions at once (kernels_class_first.hip): rows of Y, G and dZ take kClassPitch elements.
constexpr int kClassPitch = 64;
// fp32 rows of at most 32 outputs take 32 elements, one line, in the sums of the backward pass.
inline int32_t varco_class_pitch(int dtype, int32_t fo) { return dtype == VARCO_F32 && fo <= 32 ? 32 : kClassPitch; }
hipError_t varco_launch_narrow_forward(const SpmmPlan& plan, const VarcoEdge* edge, const float* vals, const void* y, int32_t rows, void* out,
                                       int32_t fo, float* partial, hipStream_t stream, const LaunchTag& tag);
// g_z may be null (nothing exchanged). dz: rows x fo; dz_padded: the same with rows of varco_class_pitch, made here, or dz itself where
// its rows are whole aligned 16-byte pieces; g_loc, g_z: rows of varco_class_pitch, or (bf16) of twice that with every sum in two terms;
// partial: kClassPitch floats per piece.
hipError_t varco_launch_narrow_backward(int dtype, const NodePlan& plan, const uint2* t_local, const uint2* t_cross, const void* dz, int64_t rows,
                                        const int32_t* zrow_of, void* dz_padded, void* g_loc, void* g_z, bool two_terms, int32_t fo, float* partial,
                                        hipStream_t stream, const LaunchTag& tag);
hipError_t varco_launch_class_dgrad(const void* g_loc, const void* g_z, bool two_terms, const int32_t* zrow_of, const int32_t* bgid, int64_t rows,
                                    const MaskRule& rule, int32_t fo, const void* wr, int32_t cpitch, void* dx, hipStream_t stream,
                                    const LaunchTag& tag);
// The same for fp32 storage from the weights as they are; with h0 and dz (rows dz_ld apart, whole 16-byte pieces) dX takes the self tap dZ H0^T as well.
hipError_t varco_launch_class_dgrad_f32(const void* g_loc, const void* g_z, const void* dz, int32_t dz_ld, const int32_t* zrow_of, const int32_t* bgid, int64_t rows,
                                        const MaskRule& rule, int32_t fo, const void* h1, const void* h0, void* dx, hipStream_t stream,
                                        const LaunchTag& tag);
// y[s, :] = X~[s, :] H (n x fo, bf16), H as its bf16 copy wt[column][position] (pitch wpitch).
hipError_t varco_launch_halo_transform_fwd(const HaloTransform& h, const void* wt, int32_t wpitch, void* y, hipStream_t stream);
// dz[s, j] = (dy[s, :] H^T)[position of j] (n x k, bf16), H as its bf16 copy wr[position][column] (pitch cpitch).
hipError_t varco_launch_halo_transform_bwd(const HaloTransform& h, const void* dy, const void* wr, int32_t cpitch, void* dz,
                                           hipStream_t stream);
// partial[g][width x fo] = workgroup g's share of X~^T dy; *slabs = number of shares written (sum them with
// varco_launch_gemm_reduce). partial_elems: floats the buffer holds.
hipError_t varco_launch_halo_transform_wgrad(const HaloTransform& h, const void* dy, float* partial, int64_t partial_elems,
                                             int32_t* slabs, hipStream_t stream);

// bf16 matrix-core path (bf16 operands, fp32 accumulation). `usable` says whether the shapes, types and
// alignments of `g` fit it; the launcher runs the product kernel only and reports the number of reduction
// slabs it wrote to g.partial (1: the result is already in C).
bool varco_gemm_bf16_usable(const GemmArgs& g);
hipError_t varco_launch_gemm_bf16(const GemmArgs& g, hipStream_t stream, const LaunchTag& tag, int32_t* split_used);
// Its weight gradients (A transposed; kernels_gemm_tn_bf16.hip), and their tile and resident workgroups per compute unit.
bool varco_gemm_tn_bf16_usable(const GemmArgs& g);
void varco_gemm_tn_bf16_tile(int32_t m, int32_t n, int32_t* bm, int32_t* bn, int32_t* per_cu);
hipError_t varco_launch_gemm_tn_bf16(const GemmArgs& g, hipStream_t stream, const LaunchTag& tag, int32_t* split_used);
// fp32 operands as sums of bf16 terms on the bf16 matrix cores (kernels_gemm_split.hip, kernels_gemm_split_rows.hip): the transform.
bool varco_gemm_split_usable(const GemmArgs& g);
hipError_t varco_launch_gemm_split(const GemmArgs& g, hipStream_t stream, const LaunchTag& tag);
// Products that each add to what the one before them wrote, by one launch (the taps of a K-tap layer): the same bits.
bool varco_gemm_split_taps_usable(const GemmArgs* g, int n);
hipError_t varco_launch_gemm_split_taps(const GemmArgs* g, int n, hipStream_t stream, const LaunchTag& tag);
bool varco_gemm_split_rows_usable(const GemmArgs& g);   // of 65 to 256 reduction steps, where weights in registers are faster
hipError_t varco_launch_gemm_split_rows(const GemmArgs& g, hipStream_t stream, const LaunchTag& tag);
// The transform in fp32 instructions, up to 256 steps a tap, where the forms above do not take it (kernels_gemm_rows.hip): the sums of the general tiles.
bool varco_gemm_rows_usable(const GemmArgs& g);
hipError_t varco_launch_gemm_rows(const GemmArgs& g, hipStream_t stream, const LaunchTag& tag);
// fp32 operands as two scaled fp16 terms on the fp16 matrix cores: input gradients (kernels_gemm_half.hip, kernels_gemm_half_nt.hip) and weight
// gradients (A transposed, kernels_gemm_half_tn.hip); same contract as the bf16 path above.
bool varco_gemm_half_usable(const GemmArgs& g);
hipError_t varco_launch_gemm_half(const GemmArgs& g, hipStream_t stream, const LaunchTag& tag);
bool varco_gemm_half_nt_usable(const GemmArgs& g);      // input gradients with 65 to 512 reduction steps (kernels_gemm_half_nt.hip)
hipError_t varco_launch_gemm_half_nt(const GemmArgs& g, hipStream_t stream, const LaunchTag& tag);
hipError_t varco_launch_gemm_half_tn(const GemmArgs& g, hipStream_t stream, const LaunchTag& tag, int32_t* split_used);
// Several of them by one launch, of 128 x 128 tiles (128 x 64 where none has more than 64 columns) and g[i].split_k slabs; their tiles.
constexpr int kMaxWeightJobs = 8;
hipError_t varco_launch_gemm_half_tn_jobs(const GemmArgs* g, int32_t n, hipStream_t stream, const LaunchTag& tag, int32_t* split_used);
int64_t varco_gemm_half_tn_tiles(const GemmArgs& g);
// Copies of weight matrices in the form the bf16 matrix-core kernels take, several per launch: (transpose ? h[c][r] : h[r][c])
// for r < rows, c < cols, zero beyond.
//   terms = 1: one rounded bf16 copy [row][pitch], rows_padded = rows;
//   terms = 2, 3: the terms of the exact expansion, rows padded to rows_padded (a multiple of 128) and columns to pitch (a
//   multiple of 32), stored by row tile and stage of 32 columns as the product kernel fetches it (kernels_gemm_split.hip);
//   kHalfTerms: two scaled fp16 terms in the same order, then the rows' scale exponents (kernels_gemm_half.hip).
//   kExactTerms: three bf16 terms of the value's sign that add up to it (below 2^-109: to 2^-131), none of them zero, stored as terms = 3.
struct PrepJob {
    const float* h;
    void* out;
    int32_t ld, rows, cols, rows_padded, pitch, transpose, terms, first_block;
};
constexpr int kMaxPrepJobs = 4 * VARCO_MAX_LAYERS;
constexpr int kFewPrepJobs = 8;         // copies that a launch which does something else as well may carry
hipError_t varco_launch_prep_weights(PrepJob* jobs, int n, hipStream_t stream);
int64_t varco_prep_blocks(PrepJob* jobs, int n);       // sets their first_block; workgroups of all copies, -1: a job that is none

// Whether varco_launch_gemm forms g and its dual product in one launch.
bool varco_gemm_dual_usable(const GemmArgs& g);
// Whether varco_launch_gemm takes the short-reduction kernels, which read the weights as they are.
bool varco_gemm_short_usable(const GemmArgs& g);

// C (+)= A B^T with at most 64 reduction steps on the bf16 matrix units (terms: 1 for bf16 storage, 2 or 3 bf16 terms
// per fp32 operand); same operand contract as the fp32-instruction kernel of kernels_gemm.hip that it replaces.
hipError_t varco_launch_gemm_short_k(const GemmArgs& g, int terms, hipStream_t stream);

// Loss and update of a training iteration (kernels_train.hip). row_loss / row_correct: n_rows each; totals
// (2 floats) may be null. block_sums: 2 * kLossBlocks floats of scratch of the stream, or null (then the rows are summed by
// one workgroup from row_loss / row_correct).
constexpr int kLossBlocks = 2048;
hipError_t varco_launch_softmax_xent(int dtype, const void* logits, int64_t ld, const int32_t* labels, int64_t n_rows,
                                     int32_t n_classes, float scale, void* dlogits, int64_t ldd, float* row_loss,
                                     int32_t* row_correct, float* totals, float* block_sums, hipStream_t stream);
hipError_t varco_launch_sgd(float* w, const float* dw, int64_t n, float lr, hipStream_t stream);
