// The calls that serve all partitions of one device at once: the layers of Algorithm 1 with every kernel launched once
// for all partitions instead of once per partition. The arithmetic is that of varco_layer_fwd / varco_layer_bwd /
// varco_accumulate_returned; the partitions' rows lie one after the other in one arena (partition 0 first), the dense
// products run over the arena, and the exchange goes through the same compressed buffer.
#include <algorithm>
#include <cstring>
#include <string>
#include <vector>

#include "varco_context.h"

using namespace varco;

namespace {

// Longest range of local / cross entries that one wavefront of the node sums takes; longer ones (hub nodes) are cut.
constexpr int32_t kNodeLocal = 64, kNodeCross = 128;
// Largest product buffer (bytes); beyond it the masked form is used, which needs none.
constexpr double kProdBytes = 48.0 * (1ull << 30);
constexpr int64_t kFewStages = 128;
// Most floats of partial products that one launch writes out for the sake of shorter sums (4 GiB).
constexpr int64_t kPartialElems = int64_t(1) << 30;

// Products of k values per cross entry are written and read back (2 k elements at about 4.8 TB/s), or whole rows are
// gathered (width elements at about 7 TB/s).
// (Rows of whole 64-byte pieces, `whole`, only where the buffer then stays within its limit.)
int32_t product_pitch(const varco_ctx* ctx, int32_t layer, int64_t k, bool whole) {
    MaskRule r{};
    r.k = uint32_t(k), r.width = uint32_t(ctx->widths[layer]);
    const int32_t pitch = varco_product_pitch(r, ctx->elem_bytes(), whole);
    return whole && double(ctx->net.nnz_cross) * pitch * ctx->elem_bytes() > kProdBytes ? varco_product_pitch(r, ctx->elem_bytes(), false) : pitch;
}
// A message's products go to a place of their own, at least 35 to 48 ps each however few they are, and are read back: rows below some length are gathered whole.
// Steps with products / with gathered rows in the hidden layer of widths 32-w-72-8, us, 8 partitions, ratios 4, 8, 16 and 32:
// few entries to a row (at most 16):
//   800,011 nodes of 12            f32 128 3,943/3,760 3,895/3,783 3,953/3,693 3,935/3,677, 160 4,579/4,342 4,298/4,286 4,137/4,189 4,274/4,163
//                                 bf16 320 4,813/4,502 4,398/4,314 4,258/4,246 4,332/4,166, 384 4,991/4,796 4,571/4,597 4,435/4,527 4,538/4,459, 448
//                                 5,319/5,203 4,809/5,001 4,673/4,925 4,771/4,861
//   60,011 nodes of 12 neighbours  f32 128 412/370 398/372 374/365 370/362    bf16 384 544/485 494/462 476/448 456/452
// more:
//   60,011 nodes of 60             f32 96 659/567 583/541 594/509 571/501, 160 859/747 699/714 616/686 650/674    bf16 256 721/672 644/642 656/624
//                                 631/602, 288 967/842 784/766 698/729 710/704, 384 1,003/917 801/841 728/807 741/801
//   200,003 nodes of 24            bf16 256 1,318/1,261 1,228/1,224 1,250/1,192 1,204/1,169, 320 1,689/1,518 1,436/1,423 1,361/1,395 1,368/1,358
//   83,480 nodes of 41             f32 96 719/658 645/627 655/603 628/602, 128 736/736 666/706 671/679 650/674    bf16 256 777/751 708/732 724/705
//                                 688/698, 288 1,016/920 835/852 763/819 767/798
// and rows that the last cache does not hold, as far as others are in use:
//   400,003 nodes of 50            f32 96 3,435/3,321 3,027/3,110 3,211/2,946 3,100/2,890, 128 3,448/3,715 3,111/3,573 3,337/3,440 3,222/3,351
//                                 bf16 192 3,597/3,434 3,240/3,279 3,446/3,148 3,344/3,058, 256 3,624/3,874 3,317/3,772 3,568/3,655 3,458/3,571, 288
//                                 4,934/4,677 3,906/4,323 3,569/4,180 3,798/4,050, 320 4,949/4,748 3,943/4,376 3,596/4,252 3,840/4,136
// (bf16: products of more than 128 bytes, ratio 4 from 288 columns on here, pay from a longer row on.)
// Rows whose length is no multiple of 4 are gathered one element to a lane (node_sum_kernel), a product's row is read by wide loads whatever the width:
//   60,011 nodes of 12 neighbours  f32 127 442/420 421/414 404/405 398/405    bf16 127 398/394 386/385 378/383 377/370, 191 462/457 429/445 415/438
//                                 407/435
//   83,480 nodes of 41             f32 79 737/694 670/664 679/640 654/631, 127 781/814 709/789 717/763 687/749    bf16 127 720/679 697/641 670/626
//                                 652/617, 191 881/884 789/847 787/819 758/818
//   400,003 nodes of 50            f32 79 3,496/3,462 3,106/3,266 3,249/3,085 3,155/3,001, 95 3,571/3,686 3,181/3,482 3,339/3,309 3,207/3,202    bf16
//                                 127 3,331/3,334 3,515/3,204 3,381/3,101 3,313/3,041, 191 4,045/4,284 3,689/4,102 3,828/3,950 3,716/3,872
bool products_pay(const varco_ctx* ctx, int32_t layer, int64_t k) {
    const int32_t width = ctx->widths[layer], row = width * int32_t(ctx->elem_bytes());
    const bool bf16 = ctx->dtype == VARCO_BF16, few = ctx->net.nnz_cross <= 16 * ctx->net.rows;
    int32_t gathered = few ? 512 : 384;                      // bytes of a row up to which it is gathered
    if (width % 4 != 0)
        gathered = !bf16 && few ? 512 : kProductRowBytes;
    else if (bf16)
        gathered = few ? 768 : product_pitch(ctx, layer, k, true) > 64 ? 640 : ctx->net.rows * row > (int64_t(128) << 20) ? 448 : 512;
    return k > 0 && 3 * k < width && row > gathered && double(ctx->net.nnz_cross) * product_pitch(ctx, layer, k, false) * ctx->elem_bytes() <= kProdBytes;
}
size_t prod_floats(const varco_ctx* ctx, int32_t layer, int64_t k, bool whole) {
    return (size_t(ctx->net.nnz_cross) * size_t(product_pitch(ctx, layer, k, whole)) * size_t(ctx->elem_bytes()) + 3) / 4;
}

// Split of a weight gradient's reduction over the arena's rows: whole rounds of resident workgroups, at least two
// stages of 32 rows each (one, where there are few). (The per-partition calls stop at eight stages: with few rows - 2,000 rows and a
// 32 x 8 weight matrix - a handful of workgroups then walks a chain of round trips while the device idles, 16 us against 6.)
// The fp32 sum of a slab loses accuracy with the square root of its length, so that there is a longest slab. With fp32 instructions it is
// that of the partitions' gradients formed one after the other (`alone` rows); with bf16 4 rows per slab and 16 per partition more, which is
// what adding a partition's gradient to the last one's cost (these sums are exact now): no less accurate than those. With two
// fp16 terms (kernels_gemm_half.hip) it is longer by a factor that grows with the rows, and the result up to 4 times as far from exact as the
// partitions' own: slabs as short as theirs took 7 (2,449,029 rows) to 32 % longer. What the factor keeps is an error below that of three
// bf16 terms in their slabs: 0.45 to 0.85 of it at 13 shapes of 2,000 to 2,449,029 rows. Relative error against fp64 of independent products,
// partition after partition / slabs as short as theirs / now, and the time of the last two:
//   fp32  256 x 256   2,449,029 rows, 8 parts   3.3e-7 / 3.1e-7 / 8.8e-7  (1,993, 1,864 us; three bf16 terms 2.0e-6)
//            two taps in a launch               3.3e-7 / 3.1e-7 / 1.2e-6  (3,748, 3,500 us; 2.7e-6)
//                     600,000 rows, 8 parts     1.9e-7 / 1.7e-7 / 4.5e-7  (582, 471 us; 7.1e-7)
//                     169,343 rows, 4 parts     1.5e-7 / 1.4e-7 / 2.5e-7  (198, 150 us; 3.9e-7)
//         200 x 136   50,021 rows, 5 parts      1.5e-7 / 1.3e-7 / 1.6e-7  (61, 50 us; 3.0e-7)
// and partition after partition / one round / now:
//   bf16  512 x 512   2,449,029 rows, 32 parts  2.1e-7 / 1.2e-6 / 2.0e-7  (1.81, 2.26 ms)
//                     169,343 rows, 4 parts     1.5e-7 / 2.6e-7 / 1.3e-7  (158, 210 us: writing and reading the partial products)
int32_t wgrad_splits(const varco_ctx* ctx, int32_t m, int32_t n, int64_t rows, int kind, int products) {
    const int64_t step = kind == kGemmF32 ? 16 : 32;
    const int64_t slots = wgrad_slots(m, n, kind, products), most = ctx->net.largest;
    const int64_t split = kind == kGemmBf16 ? plain_bf16_split(m, n, most) : gemm_split_for(m, n, most, kind), alone = most / split;
    const int64_t longest = kind == kGemmExpanded ? alone * (137'500 + rows) / 73'300 : kind == kGemmBf16 ? alone + 4 * split + 16 * ctx->n_parts : alone;
    const int64_t round = slots * std::max<int64_t>(1, longest);
    const int64_t rounds = std::max<int64_t>(1, std::min((rows + round - 1) / round, kPartialElems / (slots * products * m * n)));
    // (The stages of a slab follow one another, 1.4 us each: few rows take slabs of a single one. Beyond, and with large weights, adding the
    // partial products costs more; their sums are the more accurate all the same. Slabs of two stages / of one, one tap with its sums, us:
    //   fp32 16 x 32     2,000 rows 11.5 / 9.4    4,000 11.4 / 9.7    6,000 11.0 / 10.6   16,000 12.5 / 15.6
    //        64 x 128               16.1 / 13.2         16.0 / 14.4         15.4 / 16.0          19.1 / 24.2
    //        128 x 256              15.2 / 14.9         16.8 / 18.3         17.1 / 20.7
    //   bf16 64 x 128                9.9 / 9.8          10.4 / 11.2         11.0 / 12.3          14.0 / 19.2)
    const int64_t stages = (rows + step - 1) / step;
    return int32_t(std::min<int64_t>(rounds * slots, stages <= kFewStages ? stages : stages / 2));
}

// Whether the input gradient of a class layer that aggregated first is formed from errors summed at the width of the outputs
// (class_sums, class_input). Bytes per entry: a row of varco_class_pitch elements, against a whole row of dM for a local entry and,
// for a cross one, a row of products written and read back (which costs no less than 128 bytes do, however short) or a whole row
// of dM; dM itself is then neither written nor read. A whole step, widths at the layer's inputs and products, us:
//   bf16, 2,449,029 nodes, 97 % of 126,167,309 entries cross, 512 inputs: ratio 4 54,160 -> 44,070, 32 38,620 -> 33,160,
//     64 38,000 -> 32,540
//   bf16, 169,343 nodes, 75 % of 2,501,829 entries cross: 512 inputs, ratio 1 2,577 -> 2,343, 4 2,190 -> 1,931, 64 1,871 -> 1,737;
//     64 inputs, ratio 32 1,029 -> 939; 128 inputs, ratio 8, SAGE 1,314 -> 1,255, ratio 16, GCN 1,098 -> 1,039
//   fp32, 2,449,029 nodes, 88 % of 123,718,280 entries cross, 256 inputs, SAGE: ratio 8 47,900 -> 44,200
//   fp32, 169,343 nodes, as above: 256 inputs, ratio 8 1,763 -> 1,650, 1 2,587 -> 2,335; 32 inputs, 24 outputs 1,274 -> 1,197; 64 inputs
//     and 40 outputs, where the rule says no, 1,329 and 1,326 with all other steps
bool narrow_sums_pay(const varco_ctx* ctx, int32_t l) {
    if (!narrow_sums_possible(ctx, l)) return false;
    const NetState& net = ctx->net;
    const double row = ctx->widths[l] * ctx->elem_bytes(), k = ctx->layers[l].k, cross = k > 0 ? double(net.nnz_cross) : 0.0;
    const double wide = double(net.nnz_local) * row + cross * std::min(std::max(2.0 * k * ctx->elem_bytes(), 128.0), row) + 2.0 * double(net.rows) * row;
    return (double(net.nnz_local) + cross) * varco_class_pitch(ctx->dtype, ctx->widths[l + 1]) * ctx->elem_bytes() <= wide;
}

template <typename P>
hipError_t alloc(P*& p, size_t n) {
    return n ? hipMalloc(reinterpret_cast<void**>(&p), n * sizeof(P)) : hipSuccess;
}

// An allocation of varco_link_partitions.
#define VARCO_ROOM(ctx, call)                                                            \
    do {                                                                                 \
        const hipError_t e_ = (call);                                                    \
        if (e_ == hipErrorOutOfMemory) return no_room(ctx);                              \
        if (e_ != hipSuccess) return varco::hip_fail(ctx, e_, #call);                    \
    } while (0)
int32_t no_room(const varco_ctx* ctx) {
    (void)hipGetLastError();
    return varco_fail(ctx, VARCO_ERR_UNSUPPORTED, "varco_link_partitions: the device has no room for the joined partitions (the per-partition calls need none)");
}

struct Temp {                     // device memory of the set-up, given back on every path
    void* p = nullptr;
    ~Temp() {
        if (p) (void)hipFree(p);
    }
    hipError_t make(size_t bytes) { return bytes ? hipMalloc(&p, bytes) : hipSuccess; }
    int32_t* i32() const { return static_cast<int32_t*>(p); }
};

int32_t link_impl(varco_ctx* ctx) {
    NetState& net = ctx->net;
    const int32_t P = ctx->n_parts;
    std::vector<LinkPartition> lp(P);
    net.row_off.assign(P + 1, 0), net.halo_off.assign(P + 1, 0);
    int64_t ent = 0, local = 0, items = 0, splits = 0, slots = 0, returned = 0;
    for (int32_t q = 0; q < P; ++q) {
        const PartState& ps = ctx->parts[q];
        if (!ps.registered) return varco_fail(ctx, VARCO_ERR_STATE, "varco_link_partitions: every partition must be registered first");
        lp[q].d = ps.d;
        lp[q].row_off = net.row_off[q], lp[q].ent_off = ent, lp[q].local_off = local;
        if (ps.d.z_row_offset != net.boundary || ps.d.halo_row_offset != net.halo_off[q])
            return varco_fail(ctx, VARCO_ERR_SHAPE, "varco_link_partitions: the partitions' boundary or halo rows do not follow one another");
        if (ps.d.n_boundary > 0 && !ps.d.ret_ptr)
            return varco_fail(ctx, VARCO_ERR_UNSUPPORTED, "varco_link_partitions: a partition has no map of returned rows");
        net.row_off[q + 1] = net.row_off[q] + ps.d.n_local;
        net.largest = std::max<int64_t>(net.largest, ps.d.n_local);
        net.halo_off[q + 1] = net.halo_off[q] + ps.d.n_halo;
        net.boundary += ps.d.n_boundary;
        ent += ps.d.nnz, local += ps.nnz_t_local;
        items += ps.fwd.n_items, splits += ps.fwd.n_splits, slots += ps.fwd.n_partials;
        returned += ps.n_returned;
    }
    net.rows = net.row_off[P], net.halo_rows = net.halo_off[P];
    net.nnz = ent, net.nnz_local = local, net.nnz_cross = ent - local;
    const int64_t lim = (int64_t(1) << 31) - 1;
    if (ent > lim || net.rows > lim || net.halo_rows > lim || items > lim || slots > lim)
        return varco_fail(ctx, VARCO_ERR_UNSUPPORTED, "varco_link_partitions: 2^31 or more entries over all partitions");
    if (returned != net.halo_rows)
        return varco_fail(ctx, VARCO_ERR_SHAPE, "varco_link_partitions: the maps of returned rows do not cover the halo rows");

    // everything whose size is known, before the first kernel: a device without room for it is left as it was
    VARCO_ROOM(ctx, alloc(net.edges, size_t(net.nnz)));
    VARCO_ROOM(ctx, alloc(net.arow, size_t(net.nnz)));
    VARCO_ROOM(ctx, alloc(net.vals, size_t(net.nnz)));
    VARCO_ROOM(ctx, alloc(net.prow, size_t(net.nnz)));
    VARCO_ROOM(ctx, alloc(net.t_local, size_t(net.nnz_local)));
    VARCO_ROOM(ctx, alloc(net.t_cross, size_t(net.nnz_cross)));
    net.fwd.n_items = int32_t(items), net.fwd.n_splits = int32_t(splits), net.fwd.n_partials = int32_t(slots);
    VARCO_ROOM(ctx, alloc(net.fwd.items, size_t(items)));
    VARCO_ROOM(ctx, alloc(net.fwd.splits, size_t(splits)));
    VARCO_ROOM(ctx, alloc(net.nodes.nodes, size_t(net.rows)));
    Temp halo_len, halo_gid, halo_zrow, owner_row, cross_len, cross_ptr_d, prod_start;
    for (Temp* t : {&halo_len, &halo_gid, &halo_zrow, &owner_row, &prod_start}) VARCO_ROOM(ctx, t->make(size_t(net.halo_rows) * 4));
    VARCO_ROOM(ctx, cross_len.make(size_t(net.rows) * 4));
    VARCO_ROOM(ctx, cross_ptr_d.make(size_t(net.rows + 1) * 4));
    VARCO_ROOM(ctx, alloc(net.brow, size_t(net.boundary)));
    VARCO_ROOM(ctx, alloc(net.bgid, size_t(net.boundary)));
    VARCO_ROOM(ctx, alloc(net.zrow_of, size_t(net.rows)));

    // halo rows, their owners, and the number of cross entries of every arena row
    if (net.rows) VARCO_HIP(ctx, hipMemset(net.zrow_of, 0xFF, size_t(net.rows) * 4));
    if (net.halo_rows) VARCO_HIP(ctx, hipMemset(owner_row.p, 0xFF, size_t(net.halo_rows) * 4));
    if (net.rows) VARCO_HIP(ctx, hipMemset(cross_len.p, 0, size_t(net.rows) * 4));
    if (!ctx->d_flags) VARCO_HIP(ctx, hipMalloc(reinterpret_cast<void**>(&ctx->d_flags), sizeof(int32_t)));
    int32_t flags = 0;
    VARCO_HIP(ctx, hipMemcpy(ctx->d_flags, &flags, sizeof(flags), hipMemcpyHostToDevice));
    for (int32_t q = 0; q < P; ++q) VARCO_HIP(ctx, varco_launch_link_halo(lp[q], halo_len.i32(), halo_gid.i32(), halo_zrow.i32(), nullptr));
    for (int32_t q = 0; q < P; ++q)
        VARCO_HIP(ctx, varco_launch_link_owner(lp[q], net.halo_rows, halo_len.i32(), halo_gid.i32(), halo_zrow.i32(), owner_row.i32(),
                                               cross_len.i32(), net.brow, net.bgid, net.zrow_of, ctx->d_flags, nullptr));
    VARCO_HIP(ctx, hipMemcpy(&flags, ctx->d_flags, sizeof(flags), hipMemcpyDeviceToHost));
    if (flags) return varco_fail(ctx, VARCO_ERR_SHAPE, "varco_link_partitions: a map of returned rows does not fit the consumers' halo rows");
    std::vector<int32_t> len(size_t(net.rows)), cross_ptr(size_t(net.rows) + 1, 0);
    if (net.rows) VARCO_HIP(ctx, hipMemcpy(len.data(), cross_len.p, len.size() * 4, hipMemcpyDeviceToHost));
    for (int64_t r = 0; r < net.rows; ++r) cross_ptr[r + 1] = cross_ptr[r] + len[r];
    if (cross_ptr[net.rows] != net.nnz_cross)
        return varco_fail(ctx, VARCO_ERR_SHAPE, "varco_link_partitions: the returned rows do not hold every entry of the halo columns");
    VARCO_HIP(ctx, hipMemcpy(cross_ptr_d.p, cross_ptr.data(), cross_ptr.size() * 4, hipMemcpyHostToDevice));

    // entry arrays of both directions
    for (int32_t q = 0; q < P; ++q)
        VARCO_HIP(ctx, varco_launch_link_starts(lp[q], halo_len.i32(), cross_ptr_d.i32(), prod_start.i32(), nullptr));
    items = splits = slots = 0;
    for (int32_t q = 0; q < P; ++q) {
        const PartState& ps = ctx->parts[q];
        VARCO_HIP(ctx, varco_launch_link_edges(lp[q], ps.prow, owner_row.i32(), prod_start.i32(), net.edges, net.arow, net.vals, net.prow, nullptr));
        VARCO_HIP(ctx, varco_launch_link_transposed(lp[q], prod_start.i32(), net.t_local, net.t_cross, nullptr));
        VARCO_HIP(ctx, varco_launch_link_items(ps.fwd, int32_t(lp[q].row_off), int32_t(lp[q].ent_off), int32_t(slots), int32_t(items),
                                               int32_t(splits), net.fwd, nullptr));
        items += ps.fwd.n_items, splits += ps.fwd.n_splits, slots += ps.fwd.n_partials;
    }

    // work list of the node sums
    std::vector<NodeItem> nodes(static_cast<size_t>(net.rows));
    std::vector<SpmmItem> pieces;
    int32_t n_slots = 0;
    auto cut = [&](int32_t kind, int32_t& e0, int32_t& e1, int32_t longest, int32_t flag, int32_t& f) {
        if (e1 - e0 <= longest) return;
        const int32_t first = n_slots;
        for (int32_t e = e0; e < e1; e += longest) pieces.push_back({kind, e, std::min(e + longest, e1), n_slots++});
        e0 = first, e1 = n_slots, f |= flag;
    };
    for (int32_t q = 0; q < P; ++q) {
        const PartState& ps = ctx->parts[q];
        std::vector<int32_t> gid(size_t(ps.d.n_local));
        if (!gid.empty()) VARCO_HIP(ctx, hipMemcpy(gid.data(), ps.d.local_gid, gid.size() * 4, hipMemcpyDeviceToHost));
        for (int32_t i = 0; i < ps.d.n_local; ++i) {
            const int64_t r = lp[q].row_off + i;
            NodeItem& it = nodes[size_t(r)];
            it.row = int32_t(r), it.gid = uint32_t(gid[size_t(i)]);
            it.l0 = int32_t(lp[q].local_off) + ps.t_local_ptr[size_t(i)], it.l1 = int32_t(lp[q].local_off) + ps.t_local_ptr[size_t(i) + 1];
            it.c0 = cross_ptr[size_t(r)], it.c1 = cross_ptr[size_t(r) + 1];
            it.flags = it.pad = 0;
            cut(0, it.l0, it.l1, kNodeLocal, VARCO_NODE_LOCAL_SPLIT, it.flags);
            cut(1, it.c0, it.c1, kNodeCross, VARCO_NODE_CROSS_SPLIT, it.flags);
        }
    }
    net.nodes.n_whole = int32_t(std::stable_partition(nodes.begin(), nodes.end(), [](const NodeItem& it) { return it.flags == 0; }) - nodes.begin());
    net.nodes.n_nodes = int32_t(nodes.size()), net.nodes.n_pieces = int32_t(pieces.size());
    VARCO_ROOM(ctx, alloc(net.nodes.pieces, pieces.size()));
    if (!nodes.empty()) VARCO_HIP(ctx, hipMemcpy(net.nodes.nodes, nodes.data(), nodes.size() * sizeof(NodeItem), hipMemcpyHostToDevice));
    if (!pieces.empty()) VARCO_HIP(ctx, hipMemcpy(net.nodes.pieces, pieces.data(), pieces.size() * sizeof(SpmmItem), hipMemcpyHostToDevice));
    VARCO_HIP(ctx, hipDeviceSynchronize());

    // workspace: dM over the arena, partial rows, partial products of the weight gradients
    const int32_t wmax = *std::max_element(ctx->widths.begin(), ctx->widths.end());
    int64_t gemm_elems = 0;
    for (int32_t l = 0; l < ctx->n_layers; ++l) {     // the partial products of all layers wait for one sum
        const int32_t fi = ctx->widths[l], fo = ctx->widths[l + 1];
        const int usual = ctx->dtype == VARCO_BF16 ? kGemmBf16 : kGemmExpanded;
        const bool other = ctx->dtype == VARCO_F32 || fi < 8 || fo < 8;        // fp32 instructions, on request or for narrow bf16 weights
        const int taps = ctx->conv == VARCO_CONV_SAGE ? 2 : 1;
        int64_t splits = 0;
        for (int products = 1; products <= taps; ++products)                   // taps one by one, or sharing a launch
            for (int kind : {usual, other ? int(kGemmF32) : usual})
                splits = std::max(splits, int64_t(taps) * wgrad_splits(ctx, fi, fo, net.rows, kind, products));
        gemm_elems += splits * fi * fo;
    }
    ctx->need_dm = std::max(ctx->need_dm, (size_t(net.rows) * size_t(wmax) * size_t(ctx->elem_bytes()) + 3) / 4);
    ctx->need_spmm = std::max(ctx->need_spmm, size_t(std::max<int64_t>(net.fwd.n_partials, n_slots)) * size_t(std::max(wmax, kClassPitch)));
    ctx->need_gemm = std::max(ctx->need_gemm, size_t(gemm_elems));
    net.linked = true;
    const int32_t rc = size_all_workspaces(ctx);
    return rc != VARCO_OK && ctx->last_hip == hipErrorOutOfMemory ? no_room(ctx) : rc;
}

int32_t check_linked(const varco_ctx* ctx, const char* fn) {
    if (!ctx) return varco_fail(nullptr, VARCO_ERR_INVALID_ARG, "null context");
    if (ctx->net.linked) return VARCO_OK;
    std::string m = std::string(fn) + ": call varco_link_partitions first";
    return varco_fail(ctx, VARCO_ERR_STATE, m.c_str());
}

int32_t null_pointer(const varco_ctx* ctx, const char* fn) {
    std::string m = std::string(fn) + ": null pointer";
    return varco_fail(ctx, VARCO_ERR_INVALID_ARG, m.c_str());
}

// M = S [local rows of x; compressed rows of z] for all partitions.
// with_z: z is written by the same launch and not read (varco_spmm_owners_pay), and the given weight copies are made by it.
struct PrepList {
    PrepJob job[kMaxPrepJobs];
    int n = 0;
};
int32_t aggregate_fwd(varco_ctx* ctx, Workspace& ws, int32_t layer, const MaskRule& rule, const void* x, const void* z, void* m, hipStream_t st,
                      PrepList* with_z = nullptr) {
    const NetState& net = ctx->net;
    const double es = ctx->elem_bytes();
    const int32_t fi = ctx->widths[layer];
    // one launch: kept elements come from the owners' rows, the messages and the copies are written (and the copies' weights read)
    double extra = 0;
    if (with_z) {
        extra = double(net.boundary) * rule.k * es;
        for (int i = 0; i < with_z->n; ++i) {
            const PrepJob& j = with_z->job[i];
            extra += 4.0 * j.rows * j.cols + double(j.rows_padded) * (2.0 * j.pitch * (j.terms == kHalfTerms ? 2 : j.terms == kExactTerms ? 3 : j.terms) + (j.terms == kHalfTerms ? 4.0 : 0.0));
        }
    }
    const double entries = double(net.nnz) * 8.0 + (double(net.rows) + 1.0) * 4.0;
    const double bytes = entries + (2.0 * double(net.rows) * fi + (with_z ? 0.0 : double(net.halo_rows) * rule.k)) * es + extra;
    const double stream = entries + (double(net.rows) * fi + double(net.nnz_local) * fi + (double(net.nnz_cross) + (with_z ? double(net.boundary) : 0.0)) * rule.k) * es + extra;
    const LaunchTag tag = ctx->tag(VARCO_K_AGG_FWD, bytes, 0, stream);
    if (rule.k == rule.width)   // lossless: a message equals the owner's row, which is nearer (the same rows serve the local entries)
        VARCO_HIP(ctx, varco_launch_spmm(ctx->dtype, net.fwd, nullptr, net.arow, net.vals, x, nullptr, 0, full_rule(fi), m, 0, ws.spmm, st, tag));
    else {
        SpmmOwners owners{net.arow, net.brow, net.bgid, nullptr, 0};
        if (with_z) owners.jobs = with_z->job, owners.n_jobs = with_z->n;
        VARCO_HIP(ctx, varco_launch_spmm(ctx->dtype, net.fwd, net.edges, nullptr, net.vals, x, z, net.boundary, rule, m, 0, ws.spmm, st, tag,
                                         with_z ? &owners : nullptr));
    }
    ctx->stats.fwd_elems[layer] += net.halo_rows * rule.k;
    ctx->stats.full_fwd_elems[layer] += net.halo_rows * fi;
    return VARCO_OK;
}

// dX (+)= S^T dM, cross entries at the kept positions of their node.
int32_t aggregate_bwd(varco_ctx* ctx, Workspace& ws, int32_t layer, const MaskRule& rule, const void* dm, void* dx, bool add_old, hipStream_t st) {
    const NetState& net = ctx->net;
    const double es = ctx->elem_bytes();
    const int32_t fi = ctx->widths[layer];
    VarcoCross cross = net.nnz_cross == 0 || rule.k == 0 ? kCrossNone : rule.k == rule.width ? kCrossFull : kCrossMasked;
    const bool whole = prod_floats(ctx, layer, rule.k, true) <= ws.prod_elems;
    const int32_t pitch = product_pitch(ctx, layer, rule.k, whole);
    if (cross == kCrossMasked && products_pay(ctx, layer, rule.k) && (whole || prod_floats(ctx, layer, rule.k, false) <= ws.prod_elems)) {
        cross = kCrossProducts;
        const double bytes = double(net.nnz_cross) * 8.0 + double(net.rows) * fi * es;
        VARCO_HIP(ctx, varco_launch_halo_products(ctx->dtype, net.fwd, net.edges, net.vals, net.prow, dm, rule, ws.prod, pitch, st,
                                                  ctx->tag(VARCO_K_AGG_BWD_HALO, bytes, 0)));
    }
    const double bytes = double(net.nnz_local) * 8.0 + (double(net.rows) + 1.0) * 4.0 + 2.0 * double(net.rows) * fi * es;
    const double stream = double(net.nnz_local) * (8.0 + fi * es) + (double(net.rows) + 1.0) * 4.0 + double(net.rows) * fi * es;
    VARCO_HIP(ctx, varco_launch_node_sum(ctx->dtype, net.nodes, net.t_local, net.t_cross, dm, ws.prod, pitch, rule, cross, dx, add_old, ws.spmm, st,
                                         ctx->tag(VARCO_K_AGG_BWD_LOCAL, bytes, 0, stream)));
    if (rule.k > 0) {
        ctx->stats.bwd_elems[layer] += net.halo_rows * rule.k;
        ctx->stats.full_bwd_elems[layer] += net.halo_rows * fi;
    }
    return VARCO_OK;
}

int32_t compress_all(varco_ctx* ctx, int32_t layer, const MaskRule& rule, const void* x, void* z, hipStream_t st) {
    const NetState& net = ctx->net;
    if (net.boundary == 0 || rule.k == 0) return VARCO_OK;
    ctx->layers[layer].ran_forward = true;
    VARCO_HIP(ctx, varco_launch_compress(ctx->dtype, rule, net.bgid, net.brow, net.boundary, x, ctx->widths[layer], z, st,
                                         ctx->tag(VARCO_K_COMPRESS, double(net.boundary) * (rule.width + rule.k) * ctx->elem_bytes(), 0)));
    return VARCO_OK;
}

// Partial products of the weight gradients of a backward pass, summed by one launch at its end.
struct WeightSums {
    ReduceJob job[kMaxReduceJobs];
    int n = 0;
    size_t used = 0;              // floats of the workspace's partial buffer
    GemmArgs waiting[kMaxWeightJobs];      // small products, for one launch at the end
    int n_waiting = 0;
};

// A layer that transforms before it aggregates (kernels_class_first.hip).
int32_t class_fits(varco_ctx* ctx, const Workspace& ws, const char* fn) {
    const NetState& net = ctx->net;
    if (class_block_floats(ctx, false) <= ws.tf_elems && size_t(net.boundary) * 2 <= ws.hrows_elems) return VARCO_OK;
    std::string m = std::string(fn) + ": the stream's workspace is too small; call varco_prepare";
    return varco_fail(ctx, VARCO_ERR_STATE, m.c_str());
}

HaloTransform boundary_transform(const varco_ctx* ctx, const Workspace& ws, const MaskRule& rule, const void* z, int32_t fo) {
    HaloTransform h;
    h.z = z;
    h.rec = reinterpret_cast<const uint2*>(ws.hrows);
    h.n = int32_t(ctx->net.boundary);
    h.width = rule.width, h.k = rule.k, h.width_magic = rule.width_magic;
    h.fo = fo, h.ldy = kClassPitch;
    return h;
}

int32_t class_fwd(varco_ctx* ctx, Workspace& ws, const varco_network_buffers& b, int32_t l, hipStream_t st) {
    const NetState& net = ctx->net;
    const int32_t fi = ctx->widths[l], fo = ctx->widths[l + 1];
    const int dt = ctx->dtype;
    const double es = ctx->elem_bytes();
    const MaskRule rule = make_rule(ctx, l);
    ctx->layers[l].ran_forward = true;
    ctx->stats.fwd_elems[l] += net.halo_rows * rule.k;
    ctx->stats.full_fwd_elems[l] += net.halo_rows * fi;
    if (net.rows == 0) return VARCO_OK;
    if (int32_t rc = class_fits(ctx, ws, "varco_network_forward")) return rc;
    uint16_t* const y = reinterpret_cast<uint16_t*>(ws.tf);
    uint16_t* const yz = y + net.rows * kClassPitch;
    GemmArgs g;
    g.m = int32_t(net.rows), g.n = fo, g.k = fi;
    g.a.ptr = b.x[l], g.a.ld = fi, g.a.dtype = dt;
    g.b.ptr = b.h1[l], g.b.ld = fo;
    g.c = y, g.ldc = kClassPitch, g.c_dtype = dt;
    VARCO_HIP(ctx, prep_weight(ctx, ws, l, b.h1[l], fi, fo, true, 0, false, st, g));
    VARCO_HIP(ctx, varco_launch_gemm(g, st, ctx->tag(VARCO_K_GEMM_FWD, 0, 2.0 * double(net.rows) * fo * fi)));
    if (net.boundary > 0) {          // k = 0: rows of zeros
        ctx->prof.interrupt();
        VARCO_HIP(ctx, varco_launch_halo_rows(rule, net.bgid, nullptr, int32_t(net.boundary), reinterpret_cast<uint2*>(ws.hrows), st));
        const LaunchTag tag = ctx->tag(VARCO_K_GEMM_FWD, double(net.boundary) * (rule.k + fo) * es, 2.0 * double(net.boundary) * fo * rule.k);
        tag.begin(st);
        const hipError_t e = varco_launch_halo_transform_fwd(boundary_transform(ctx, ws, rule, b.z[l], fo), g.b_prep, int32_t(g.b_prep_ld), yz, st);
        tag.end(st);
        VARCO_HIP(ctx, e);
    }
    const double entries = double(net.nnz) * 8.0 + (double(net.rows) + 1.0) * 4.0;
    VARCO_HIP(ctx, varco_launch_narrow_forward(net.fwd, net.edges, net.vals, y, int32_t(net.rows), b.x[l + 1], fo, ws.spmm, st,
                                               ctx->tag(VARCO_K_AGG_FWD, entries + (2.0 * double(net.rows) + double(net.boundary)) * fo * es, 0,
                                                        entries + (double(net.rows) + double(net.nnz)) * fo * es)));
    if (ctx->conv == VARCO_CONV_SAGE) {   // self tap
        GemmArgs g0;
        g0.m = int32_t(net.rows), g0.n = fo, g0.k = fi;
        g0.a = g.a;
        g0.b.ptr = b.h0[l], g0.b.ld = fo;
        g0.c = b.x[l + 1], g0.ldc = fo, g0.c_dtype = dt;
        g0.accumulate = true;
        VARCO_HIP(ctx, prep_weight(ctx, ws, l, b.h0[l], fi, fo, true, 1, false, st, g0));
        VARCO_HIP(ctx, varco_launch_gemm(g0, st, ctx->tag(VARCO_K_GEMM_FWD, 0, 2.0 * double(net.rows) * fo * fi)));
    }
    return VARCO_OK;
}

int32_t sum_later(varco_ctx* ctx, const GemmArgs& g, int32_t split, WeightSums& sums) {
    const int products = g.c_dual ? 2 : 1;
    if (sums.n + products > kMaxReduceJobs) return varco_fail(ctx, VARCO_ERR_STATE, "varco_network_backward: workspace too small");
    for (int i = 0; split > 1 && i < products; ++i)
        sums.job[sums.n++] = ReduceJob{g.partial + size_t(i) * split * g.m * g.n, static_cast<float*>(i ? g.c_dual : g.c), g.ldc, split, g.m, g.n, 0};
    return VARCO_OK;
}

// One split product into the weight sums; `g` with everything but the split set.
int32_t add_weight_product(varco_ctx* ctx, Workspace& ws, GemmArgs& g, WeightSums& sums, hipStream_t st) {
    const int products = g.c_dual ? 2 : 1;
    const size_t one = size_t(g.m) * g.n;
    int32_t split = 1;
    g.deferred = &split;
    g.split_k = wgrad_splits(ctx, g.m, g.n, g.k, gemm_kind(g), products);
    if (sums.used + size_t(g.split_k) * one * products > ws.gemm_elems || sums.n + products > kMaxReduceJobs)
        return varco_fail(ctx, VARCO_ERR_STATE, "varco_network_backward: workspace too small");
    g.partial = ws.gemm + sums.used;
    VARCO_HIP(ctx, varco_launch_gemm(g, st, ctx->tag(VARCO_K_GEMM_WGRAD, 0, 2.0 * products * double(one) * double(g.k))));
    if (split > 1) sums.used += size_t(split) * one * products;
    return sum_later(ctx, g, split, sums);
}

// Whether a layer's weight products may wait for the end of the pass, where one launch takes them all: stages of 32 rows times 128 x 128 tiles
// are few, and nothing that the layers below write lies in what they read. A launch of few stages is a chain of round trips on a device that the
// next one could use. Backward passes layer by layer / together, us: 2,000 nodes 16-32-8 21.9 / 17.8, 16,000 nodes 32-64-8 33.9 / 30.1, 5,000 nodes
// 200-64-64-64-10, two taps 87.0 / 64.6, 3,997 nodes 93-208-120-14, two taps 79.7 / 80.4; 53 networks of 2,000 to 300,000 nodes take 0.73 to 1.009, 0.933 in the
// mean. Limits of 256 and 2,048: 0.944; of 4,096 and 16,384 0.933, but up to 1.024 (300,000 nodes 32-32-32-8: 460 / 472, 457 with these).
constexpr int64_t kFewTiles = 1024, kFewNarrowTiles = 4096;
bool may_wait(const varco_ctx* ctx, const varco_network_buffers& b, int32_t l, const GemmArgs& g, const WeightSums& sums) {
    if (sums.n_waiting == kMaxWeightJobs || gemm_kind(g) != kGemmExpanded || int64_t((g.k + 31) / 32) * varco_gemm_half_tn_tiles(g) > (g.n <= 64 ? kFewNarrowTiles : kFewTiles)) return false;
    const size_t rows = size_t(g.k) * sizeof(float);
    auto apart = [](const void* p, size_t np, const void* q, size_t nq) {
        const uintptr_t a = reinterpret_cast<uintptr_t>(p), c = reinterpret_cast<uintptr_t>(q);
        return a + np <= c || c + nq <= a;
    };
    for (int32_t j = 1; j <= l; ++j) {
        const size_t written = rows * size_t(ctx->widths[j]);
        for (const void* p : {g.a.ptr, g.a_dual})
            if (p && !apart(p, rows * size_t(g.m), b.dx[j], written)) return false;
        for (const void* p : {g.b.ptr, g.b.gate})
            if (p && !apart(p, rows * size_t(g.n), b.dx[j], written)) return false;
    }
    return true;
}

// The products that waited, one launch for those of up to 64 columns and one for the others. Every product keeps the slabs it has in a launch of
// its own, hence its bits and its accuracy. (The device divided among them means longer slabs, whose sums are further from exact:
// 100,000 nodes 64-64-64-40, two partitions, 1.30e-7 -> 1.81e-7, and a backward pass of 203 us where it takes 218 with these slabs and 224 layer by layer.)
int32_t launch_together(varco_ctx* ctx, Workspace& ws, GemmArgs* g, int n, WeightSums& sums, hipStream_t st) {
    if (n == 0) return VARCO_OK;
    if (n == 1) return add_weight_product(ctx, ws, *g, sums, st);
    double flops = 0;
    int32_t split[kMaxWeightJobs] = {};
    for (int i = 0; i < n; ++i) {
        const int products = g[i].c_dual ? 2 : 1;
        g[i].split_k = wgrad_splits(ctx, g[i].m, g[i].n, g[i].k, kGemmExpanded, products);
        g[i].partial = ws.gemm + sums.used;
        sums.used += size_t(g[i].split_k) * size_t(g[i].m) * size_t(g[i].n) * size_t(products);
        flops += 2.0 * products * double(g[i].m) * double(g[i].n) * double(g[i].k);
    }
    if (sums.used > ws.gemm_elems) return varco_fail(ctx, VARCO_ERR_STATE, "varco_network_backward: workspace too small");
    VARCO_HIP(ctx, varco_launch_gemm_half_tn_jobs(g, n, st, ctx->tag(VARCO_K_GEMM_WGRAD, 0, flops), split));
    for (int i = 0; i < n; ++i)
        if (int32_t rc = sum_later(ctx, g[i], split[i], sums)) return rc;
    return VARCO_OK;
}
int32_t launch_waiting(varco_ctx* ctx, Workspace& ws, WeightSums& sums, hipStream_t st) {
    GemmArgs* const end = sums.waiting + sums.n_waiting;
    GemmArgs* const wide = std::stable_partition(sums.waiting, end, [](const GemmArgs& g) { return g.n <= 64; });
    sums.n_waiting = 0;
    if (int32_t rc = launch_together(ctx, ws, sums.waiting, int(wide - sums.waiting), sums, st)) return rc;
    return launch_together(ctx, ws, wide, int(end - wide), sums, st);
}

// Backward pass of a narrowing class layer in two steps that do not depend on the order of its forward pass: the errors of all
// its consumers are summed at the width of the outputs, G = S^T dZ, and then taken back through the weights,
//   dX[v] = G_loc[v] H1^T + kept positions of (G_z[v] H1^T) (+ dZ[v] H0^T),
// instead of through the weights first and summed at the width of the inputs (dM = dZ H1^T; dX = S^T dM).
// With bf16 storage a sum that stands in for rows of dM is kept as two bf16 numbers. Rounded to one, errors of one sign (neighbours of
// one class) cost dX accuracy that dM, rounded for each consumer, had kept; with two, dX has its own rounding and no other. Relative error
// of dX, through dM / one / two, 3 outputs, errors of one sign 1.76e-3 / 1.91e-3 / 1.66e-3, 47 outputs of any sign 2.56e-3 / 2.35e-3 / 1.66e-3; a
// whole step of 2,449,029 nodes and 512 inputs 43.3 ms with one, 43.7 with two. A layer that transforms first rounds its sums to bf16 as it
// always did: its weight gradients read them as such.
struct ClassRows {
    void *dz, *g_loc, *g_z;          // rows of varco_class_pitch elements, twice as many with two_terms, of dz dz_ld; g_z null: no errors come back
    int32_t dz_ld;
    bool two_terms;
};
// What such a pass is given: dZ, the weights of the aggregated tap and of the one that is not (or null), and where dX goes.
struct ClassCall {
    void* dz;
    const void *h1, *h0;
    void* dx;
};
ClassCall class_call(const varco_ctx* ctx, const varco_network_buffers& b, int32_t l) {
    return {b.dx[l + 1], b.h1[l], ctx->conv == VARCO_CONV_SAGE ? b.h0[l] : nullptr, b.dx[l]};
}
ClassRows class_rows(const varco_ctx* ctx, const Workspace& ws, const ClassCall& c, int32_t l, const MaskRule& rule) {
    const NetState& net = ctx->net;
    const int32_t pitch = varco_class_pitch(ctx->dtype, ctx->widths[l + 1]);
    const size_t bytes = size_t(net.rows) * size_t(pitch) * size_t(ctx->elem_bytes());
    char* const at = reinterpret_cast<char*>(ws.tf);
    ClassRows r;
    // dZ as it is where its rows are whole aligned 16-byte pieces, else a padded copy
    const bool whole = ctx->widths[l + 1] * int(ctx->elem_bytes()) % 16 == 0 && (reinterpret_cast<uintptr_t>(c.dz) & 15u) == 0;
    r.dz = whole ? c.dz : at, r.dz_ld = whole ? ctx->widths[l + 1] : pitch;
    r.two_terms = ctx->dtype == VARCO_BF16 && ctx->layers[l].order == VARCO_ORDER_AGGREGATE_FIRST;
    r.g_loc = at + bytes;
    r.g_z = net.nnz_cross > 0 && rule.k > 0 ? at + (r.two_terms ? 3 : 2) * bytes : nullptr;
    return r;
}
int32_t class_sums(varco_ctx* ctx, Workspace& ws, const ClassCall& c, int32_t l, const ClassRows& r, hipStream_t st) {
    const NetState& net = ctx->net;
    const int32_t fo = ctx->widths[l + 1];
    const double es = ctx->elem_bytes();
    const double entries = double(net.nnz) * 8.0 + (double(net.rows) + 1.0) * 4.0;
    VARCO_HIP(ctx, varco_launch_narrow_backward(ctx->dtype, net.nodes, net.t_local, net.t_cross, c.dz, net.rows, net.zrow_of, r.dz, r.g_loc, r.g_z,
                                                r.two_terms, fo, ws.spmm, st,
                                                ctx->tag(VARCO_K_AGG_BWD_LOCAL, entries + (2.0 * double(net.rows) + double(net.boundary)) * fo * es, 0,
                                                         entries + (double(net.rows) + double(net.nnz)) * fo * es)));
    return VARCO_OK;
}
int32_t class_input(varco_ctx* ctx, Workspace& ws, const ClassCall& c, int32_t l, const MaskRule& rule, const ClassRows& r, hipStream_t st) {
    const NetState& net = ctx->net;
    const int32_t fi = ctx->widths[l], fo = ctx->widths[l + 1];
    const int dt = ctx->dtype;
    if (rule.k > 0) {
        ctx->stats.bwd_elems[l] += net.halo_rows * rule.k;
        ctx->stats.full_bwd_elems[l] += net.halo_rows * fi;
    }
    if (dt == VARCO_F32) {
        VARCO_HIP(ctx, varco_launch_class_dgrad_f32(r.g_loc, r.g_z, r.dz, r.dz_ld, net.zrow_of, net.bgid, net.rows, rule, fo, c.h1, c.h0,
                                                    c.dx, st, ctx->tag(VARCO_K_GEMM_DGRAD, 0, (c.h0 ? 4.0 : 2.0) * fi * fo * double(net.rows))));
        return VARCO_OK;
    }
    GemmArgs gw;                       // carries the slot of the weights' bf16 copy [position][column]
    VARCO_HIP(ctx, prep_weight(ctx, ws, l, c.h1, fi, fo, false, 0, false, st, gw));
    VARCO_HIP(ctx, varco_launch_class_dgrad(r.g_loc, r.g_z, r.two_terms, net.zrow_of, net.bgid, net.rows, rule, fo, gw.b_prep, int32_t(gw.b_prep_ld),
                                            c.dx, st, ctx->tag(VARCO_K_GEMM_DGRAD, 0, 2.0 * fi * fo * double(net.rows))));
    if (c.h0) {                        // + dZ H0^T
        GemmArgs g0;
        g0.m = int32_t(net.rows), g0.n = fi, g0.k = fo;
        g0.a.ptr = c.dz, g0.a.ld = fo, g0.a.dtype = dt;
        g0.b.ptr = c.h0, g0.b.ld = fo, g0.b.transposed = true;
        g0.c = c.dx, g0.ldc = fi, g0.c_dtype = dt;
        g0.accumulate = true;
        VARCO_HIP(ctx, varco_launch_gemm(g0, st, ctx->tag(VARCO_K_GEMM_DGRAD, 0, 2.0 * fi * fo * double(net.rows))));
    }
    return VARCO_OK;
}

bool narrow_sums_taken(const varco_ctx* ctx, const Workspace& ws, int32_t l, const ClassCall& c) {
    const bool bf16 = ctx->dtype == VARCO_BF16;
    return narrow_sums_pay(ctx, l) && class_block_floats(ctx, bf16) <= ws.tf_elems && (!bf16 || (reinterpret_cast<uintptr_t>(c.dx) & 15u) == 0);
}
int32_t narrow_bwd(varco_ctx* ctx, Workspace& ws, const ClassCall& c, int32_t l, const MaskRule& rule, hipStream_t st) {
    const ClassRows r = class_rows(ctx, ws, c, l, rule);
    if (int32_t rc = class_sums(ctx, ws, c, l, r, st)) return rc;
    return class_input(ctx, ws, c, l, rule, r, st);
}

int32_t class_bwd(varco_ctx* ctx, Workspace& ws, const varco_network_buffers& b, int32_t l, WeightSums& sums, hipStream_t st) {
    const NetState& net = ctx->net;
    const int32_t fi = ctx->widths[l], fo = ctx->widths[l + 1];
    const int dt = ctx->dtype;
    const double es = ctx->elem_bytes();
    const MaskRule rule = make_rule(ctx, l);
    if (int32_t rc = class_fits(ctx, ws, "varco_network_backward")) return rc;
    const ClassCall c = class_call(ctx, b, l);
    const ClassRows r = class_rows(ctx, ws, c, l, rule);
    if (int32_t rc = class_sums(ctx, ws, c, l, r, st)) return rc;
    GemmArgs g;
    g.m = fi, g.n = fo, g.k = int32_t(net.rows);
    g.a.ptr = b.x[l], g.a.ld = fi, g.a.transposed = true, g.a.dtype = dt;
    g.b.ptr = r.g_loc, g.b.ld = kClassPitch, g.b.dtype = dt;
    g.c = b.dh1[l], g.ldc = fo;
    g.accumulate = true;
    if (int32_t rc = add_weight_product(ctx, ws, g, sums, st)) return rc;
    if (ctx->conv == VARCO_CONV_SAGE) {
        g.b.ptr = r.dz, g.b.ld = r.dz_ld, g.c = b.dh0[l];
        if (int32_t rc = add_weight_product(ctx, ws, g, sums, st)) return rc;
    }
    if (r.g_z) {   // + X~_z^T G_z: per-workgroup shares
        VARCO_HIP(ctx, varco_launch_halo_rows(rule, net.bgid, nullptr, int32_t(net.boundary), reinterpret_cast<uint2*>(ws.hrows), st));
        const LaunchTag tag = ctx->tag(VARCO_K_GEMM_WGRAD, double(net.boundary) * (rule.k + fo) * es, 2.0 * double(rule.k) * fo * double(net.boundary));
        int32_t slabs = 0;
        float* const partial = ws.gemm + sums.used;
        tag.begin(st);
        const hipError_t e = varco_launch_halo_transform_wgrad(boundary_transform(ctx, ws, rule, b.z[l], fo), r.g_z, partial,
                                                               int64_t(ws.gemm_elems - sums.used), &slabs, st);
        tag.end(st);
        VARCO_HIP(ctx, e);
        // (added by a launch of its own: the sums of a pass go to distinct results)
        VARCO_HIP(ctx, varco_launch_gemm_reduce(partial, slabs, fi, fo, static_cast<float*>(b.dh1[l]), fo, true, st, tag));
    }
    return l > 0 ? class_input(ctx, ws, c, l, rule, r, st) : VARCO_OK;
}

// copies: weight copies that have not been made yet (the pass's first layer); made here.
int32_t layer_fwd(varco_ctx* ctx, Workspace& ws, const varco_network_buffers& b, int32_t l, PrepList& copies, hipStream_t st) {
    const NetState& net = ctx->net;
    const int32_t fi = ctx->widths[l], fo = ctx->widths[l + 1];
    const bool sage = ctx->conv == VARCO_CONV_SAGE;
    const int dt = ctx->dtype;
    const double es = ctx->elem_bytes();
    const bool first = ctx->layers[l].order == VARCO_ORDER_TRANSFORM_FIRST;
    const MaskRule rule = make_rule(ctx, l);
    const bool together = !first && varco_spmm_owners_pay(dt, net.fwd, rule, net.rows, net.nnz_cross, net.boundary, b.x[l], b.m[l], ws.spmm);
    if (copies.n > 0 && !(together && copies.n <= kFewPrepJobs)) {
        ctx->prof.interrupt();
        VARCO_HIP(ctx, varco_launch_prep_weights(copies.job, copies.n, st));
        copies.n = 0;
    }
    if (!together)
        if (int32_t rc = compress_all(ctx, l, rule, b.x[l], b.z[l], st)) return rc;
    if (first) return class_fwd(ctx, ws, b, l, st);
    ctx->layers[l].ran_forward = true;
    if (int32_t rc = aggregate_fwd(ctx, ws, l, rule, b.x[l], b.z[l], b.m[l], st, together ? &copies : nullptr)) return rc;
    copies.n = 0;
    if (net.rows > 0) {
        GemmArgs g;
        g.m = int32_t(net.rows), g.n = fo, g.k = fi;
        g.a.ptr = b.m[l], g.a.ld = fi, g.a.dtype = dt;
        g.b.ptr = b.h1[l], g.b.ld = fo;
        if (sage) {
            g.k2 = fi;
            g.a2.ptr = b.x[l], g.a2.ld = fi, g.a2.dtype = dt;
            g.b2.ptr = b.h0[l], g.b2.ld = fo;
        }
        g.c = b.x[l + 1], g.ldc = fo, g.c_dtype = dt;
        g.relu = ctx->act[l] == VARCO_ACT_RELU;
        VARCO_HIP(ctx, prep_weight(ctx, ws, l, b.h1[l], fi, fo, true, 0, false, st, g));
        if (sage) VARCO_HIP(ctx, prep_weight(ctx, ws, l, b.h0[l], fi, fo, true, 1, true, st, g));
        VARCO_HIP(ctx, varco_launch_gemm(g, st, ctx->tag(VARCO_K_GEMM_FWD, 0, 2.0 * g.m * double(g.n) * (double(g.k) + g.k2))));
    }
    return VARCO_OK;
}

int32_t layer_bwd(varco_ctx* ctx, Workspace& ws, const varco_network_buffers& b, int32_t l, WeightSums& sums, hipStream_t st) {
    const NetState& net = ctx->net;
    const int32_t fi = ctx->widths[l], fo = ctx->widths[l + 1];
    const bool sage = ctx->conv == VARCO_CONV_SAGE, need = l > 0;
    const int dt = ctx->dtype;
    const double es = ctx->elem_bytes();
    if (net.rows == 0) return VARCO_OK;
    const int32_t nl = int32_t(net.rows);
    if (ctx->layers[l].order == VARCO_ORDER_TRANSFORM_FIRST) return class_bwd(ctx, ws, b, l, sums, st);
    const void* gate = ctx->act[l] == VARCO_ACT_RELU ? b.x[l + 1] : nullptr;
    {   // weight gradients: one reduction over the rows of all partitions (their sum is what Algorithm 1 asks for)
        GemmArgs g;
        g.m = fi, g.n = fo, g.k = nl;
        g.a.ptr = b.m[l], g.a.ld = fi, g.a.transposed = true, g.a.dtype = dt;
        g.b.ptr = b.dx[l + 1], g.b.gate = gate, g.b.ld = fo, g.b.dtype = dt;
        g.c = b.dh1[l], g.ldc = fo;
        g.accumulate = true;
        g.f32_terms = dt == VARCO_F32 ? ctx->f32_terms : 0;
        // both taps' gradients by one launch where the kernels can: they share dZ (and its mask)
        if (sage) {
            int32_t unused = 0;
            g.deferred = &unused;
            g.a_dual = b.x[l], g.c_dual = b.dh0[l];
            if (!varco_gemm_dual_usable(g)) g.a_dual = nullptr, g.c_dual = nullptr;
        }
        const int products = g.c_dual ? 2 : 1;
        for (int tap = 0; tap < (sage ? 2 : 1); tap += products) {
            if (tap == 1) g.a.ptr = b.x[l], g.c = b.dh0[l];
            if (may_wait(ctx, b, l, g, sums))
                g.deferred = nullptr, sums.waiting[sums.n_waiting++] = g;
            else if (int32_t rc = add_weight_product(ctx, ws, g, sums, st))
                return rc;
        }
    }
    if (!need) return VARCO_OK;
    if (const ClassCall c = class_call(ctx, b, l); narrow_sums_taken(ctx, ws, l, c)) return narrow_bwd(ctx, ws, c, l, make_rule(ctx, l), st);
    GemmArgs g;                    // dM = dZ H1^T
    g.m = nl, g.n = fi, g.k = fo;
    g.a.ptr = b.dx[l + 1], g.a.gate = gate, g.a.ld = fo, g.a.dtype = dt;
    g.b.ptr = b.h1[l], g.b.ld = fo, g.b.transposed = true;
    g.c = ws.dm, g.ldc = fi, g.c_dtype = dt;
    g.f32_terms = dt == VARCO_F32 ? ctx->f32_terms : 0;
    const bool short_k = varco_gemm_short_usable(g);      // reads the weights as they are
    const double flops = 2.0 * fi * fo * double(nl);
    if (!short_k) VARCO_HIP(ctx, prep_weight(ctx, ws, l, b.h1[l], fi, fo, false, 0, false, st, g));
    GemmArgs g0 = g;               // self tap: dZ H0^T
    if (sage) {
        g0.b.ptr = b.h0[l], g0.c = b.dx[l];
        if (!short_k) VARCO_HIP(ctx, prep_weight(ctx, ws, l, b.h0[l], fi, fo, false, 1, false, st, g0));
    }
    // fp32 storage: the aggregated part is added to the self tap, whose product can share a launch with dM. With bf16 storage the
    // self tap, the larger part, would be rounded once more that way (relative error of dX at ratio 4: 2.86e-3 against 2.55e-3
    // with the product added to the aggregated part).
    const bool self_first = sage && dt == VARCO_F32;
    if (self_first) {
        g.b_dual = b.h0[l], g.b_dual_prep = g0.b_prep, g.c_dual = b.dx[l];
        if (!varco_gemm_dual_usable(g)) {
            g.b_dual = g.b_dual_prep = nullptr, g.c_dual = nullptr;
            VARCO_HIP(ctx, varco_launch_gemm(g0, st, ctx->tag(VARCO_K_GEMM_DGRAD, 0, flops)));
        }
    }
    VARCO_HIP(ctx, varco_launch_gemm(g, st, ctx->tag(VARCO_K_GEMM_DGRAD, 0, g.c_dual ? 2.0 * flops : flops)));
    if (int32_t rc = aggregate_bwd(ctx, ws, l, make_rule(ctx, l), ws.dm, b.dx[l], self_first, st)) return rc;
    if (sage && !self_first) {
        g0.accumulate = true;
        VARCO_HIP(ctx, varco_launch_gemm(g0, st, ctx->tag(VARCO_K_GEMM_DGRAD, 0, flops)));
    }
    return VARCO_OK;
}

int32_t finish_sums(varco_ctx* ctx, WeightSums& sums, hipStream_t st) {
    VARCO_HIP(ctx, varco_launch_gemm_reduce_jobs(sums.job, sums.n, true, st, ctx->tag(VARCO_K_REDUCE, 0, 0)));
    sums.n = 0, sums.used = 0;
    return VARCO_OK;
}

// All weight copies a pass needs, for one launch: those of the forward products, and when the buffers hold weight gradients
// (a backward pass follows) those of the input gradients as well.
void prep_all(varco_ctx* ctx, Workspace& ws, const varco_network_buffers& b, PrepList& list) {
    PrepJob* const jobs = list.job;
    int& n = list.n;
    GemmArgs unused;
    for (int32_t l = 0; l < ctx->n_layers; ++l) {
        const int32_t fi = ctx->widths[l], fo = ctx->widths[l + 1];
        const bool first = ctx->layers[l].order == VARCO_ORDER_TRANSFORM_FIRST;
        for (int which = 0; which < (ctx->conv == VARCO_CONV_SAGE ? 2 : 1); ++which) {
            const void* h = which ? b.h0[l] : b.h1[l];
            n += prep_slot(ctx, ws, l, h, fi, fo, true, which, false, unused, jobs + n) ? 1 : 0;
            // (fp32 layers of at most 64 outputs take their weights as they are, or, from 17 outputs on where no narrow sums are formed, have them
            // copied by layer_bwd)
            if (b.dh1[l] && l > 0 && (fo > 64 || (which == 0 && ctx->dtype == VARCO_BF16 && (first || narrow_sums_pay(ctx, l)))))
                n += prep_slot(ctx, ws, l, h, fi, fo, false, which, false, unused, jobs + n) ? 1 : 0;
        }
    }
}

int32_t check_buffers(const varco_ctx* ctx, const varco_network_buffers* b, bool backward, const char* fn) {
    if (!b) return null_pointer(ctx, fn);
    const NetState& net = ctx->net;
    const int32_t L = ctx->n_layers;
    const bool sage = ctx->conv == VARCO_CONV_SAGE;
    for (int32_t l = 0; l < L; ++l) {
        const bool first = ctx->layers[l].order == VARCO_ORDER_TRANSFORM_FIRST, sent = net.halo_rows > 0 && ctx->layers[l].k > 0;
        if (!b->h1[l] || (sage && !b->h0[l]) || (net.rows > 0 && (!b->x[l] || (!first && !b->m[l]))) || (sent && !b->z[l])) return null_pointer(ctx, fn);
        if (backward && (!b->dh1[l] || (sage && !b->dh0[l]) || (net.rows > 0 && !b->dx[l + 1]) ))
            return null_pointer(ctx, fn);
        if (int32_t rc = check_wide_rows(ctx, ctx->widths[l], {b->x[l], b->z[l], b->m[l], backward ? b->dx[l + 1] : nullptr}, fn)) return rc;
    }
    return net.rows > 0 && !b->x[L] ? null_pointer(ctx, fn) : VARCO_OK;
}

// Shared prologue of the calls on one buffer pair (a tap of a K-tap layer).
int32_t tap_prologue(varco_ctx* ctx, int32_t tap, varco_stream stream, const char* fn, int32_t* layer, int32_t* hop, Workspace** ws) {
    if (int32_t rc = check_linked(ctx, fn)) return rc;
    ctx->prof.interrupt();
    *layer = tap;
    if (int32_t rc = split_tap(ctx, layer, hop, fn)) return rc;
    return workspace_for(ctx, static_cast<hipStream_t>(stream), ws, fn);
}

}  // namespace

size_t varco::network_prod_need(const varco_ctx* ctx, bool whole, size_t* most) {
    size_t need = 0;
    *most = 0;
    for (int32_t l = 1; l < ctx->n_layers; ++l) {     // the first layer's input needs no gradient
        if (products_pay(ctx, l, ctx->layers[l].k)) need = std::max(need, prod_floats(ctx, l, ctx->layers[l].k, whole));
        int64_t k = (ctx->widths[l] - 1) / 3;
        while (k > 0 && !products_pay(ctx, l, k)) --k;
        if (k > 0) *most = std::max(*most, prod_floats(ctx, l, k, whole));
    }
    return need;
}

extern "C" int32_t varco_link_partitions(varco_ctx* ctx) {
    if (!ctx) return varco_fail(nullptr, VARCO_ERR_INVALID_ARG, "varco_link_partitions: null context");
    VARCO_HIP(ctx, hipDeviceSynchronize());
    free_network(ctx->net);
    const size_t need_dm = ctx->need_dm, need_spmm = ctx->need_spmm, need_gemm = ctx->need_gemm;
    ctx->last_hip = hipSuccess;
    const int32_t rc = link_impl(ctx);
    if (rc == VARCO_OK) return VARCO_OK;
    // as before the call: workspaces of the per-partition calls, which go on
    free_network(ctx->net);
    ctx->need_dm = need_dm, ctx->need_spmm = need_spmm, ctx->need_gemm = need_gemm;
    const std::string why = ctx->error;
    if (int32_t lost = size_all_workspaces(ctx)) return lost;
    return varco_fail(ctx, rc, why.c_str());
}

extern "C" int32_t varco_network_forward(varco_ctx* ctx, const varco_network_buffers* b, varco_stream stream) {
    const char* fn = "varco_network_forward";
    if (int32_t rc = check_linked(ctx, fn)) return rc;
    ctx->prof.interrupt();
    if (int32_t rc = check_buffers(ctx, b, false, fn)) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    Workspace* ws = nullptr;
    if (int32_t rc = workspace_for(ctx, st, &ws, fn)) return rc;
    PrepList copies;
    prep_all(ctx, *ws, *b, copies);
    for (int32_t l = 0; l < ctx->n_layers; ++l)
        if (int32_t rc = layer_fwd(ctx, *ws, *b, l, copies, st)) return rc;
    return VARCO_OK;
}

extern "C" int32_t varco_network_backward(varco_ctx* ctx, const varco_network_buffers* b, varco_stream stream) {
    const char* fn = "varco_network_backward";
    if (int32_t rc = check_linked(ctx, fn)) return rc;
    ctx->prof.interrupt();
    if (int32_t rc = check_buffers(ctx, b, true, fn)) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    Workspace* ws = nullptr;
    if (int32_t rc = workspace_for(ctx, st, &ws, fn)) return rc;
    WeightSums sums;
    for (int32_t l = ctx->n_layers - 1; l >= 0; --l)
        if (int32_t rc = layer_bwd(ctx, *ws, *b, l, sums, st)) return rc;
    if (int32_t rc = launch_waiting(ctx, *ws, sums, st)) return rc;
    return finish_sums(ctx, sums, st);
}

extern "C" int32_t varco_network_compress(varco_ctx* ctx, int32_t tap, const void* x, void* z, varco_stream stream) {
    const char* fn = "varco_network_compress";
    int32_t layer = 0, hop = 0;
    Workspace* ws = nullptr;
    if (int32_t rc = tap_prologue(ctx, tap, stream, fn, &layer, &hop, &ws)) return rc;
    if (ctx->net.boundary > 0 && ctx->layers[layer].k > 0 && (!x || !z)) return null_pointer(ctx, fn);
    return compress_all(ctx, layer, make_rule(ctx, layer, hop), x, z, static_cast<hipStream_t>(stream));
}

extern "C" int32_t varco_network_aggregate_fwd(varco_ctx* ctx, int32_t tap, const void* y, const void* z_in, void* y_out, varco_stream stream) {
    const char* fn = "varco_network_aggregate_fwd";
    int32_t layer = 0, hop = 0;
    Workspace* ws = nullptr;
    if (int32_t rc = tap_prologue(ctx, tap, stream, fn, &layer, &hop, &ws)) return rc;
    if ((ctx->net.rows > 0 && (!y || !y_out)) || (ctx->net.halo_rows > 0 && ctx->layers[layer].k > 0 && !z_in)) return null_pointer(ctx, fn);
    if (int32_t rc = check_wide_rows(ctx, ctx->widths[layer], {y, z_in, y_out}, fn)) return rc;
    ctx->layers[layer].ran_forward = true;
    return aggregate_fwd(ctx, *ws, layer, make_rule(ctx, layer, hop), y, z_in, y_out, static_cast<hipStream_t>(stream));
}

extern "C" int32_t varco_network_aggregate_bwd(varco_ctx* ctx, int32_t tap, const void* g_out, void* g_in, int32_t accumulate, varco_stream stream) {
    const char* fn = "varco_network_aggregate_bwd";
    int32_t layer = 0, hop = 0;
    Workspace* ws = nullptr;
    if (int32_t rc = tap_prologue(ctx, tap, stream, fn, &layer, &hop, &ws)) return rc;
    if (ctx->net.rows > 0 && (!g_out || !g_in)) return null_pointer(ctx, fn);
    if (int32_t rc = check_wide_rows(ctx, ctx->widths[layer], {g_out, g_in}, fn)) return rc;
    return aggregate_bwd(ctx, *ws, layer, make_rule(ctx, layer, hop), g_out, g_in, accumulate != 0, static_cast<hipStream_t>(stream));
}

// The dense products of all taps of a layer over the arena. The copies of all weights are made by one launch (as many as there
// are slots); forward, fp32 storage, so are their products, in the order of varco_transform_fwd; backward, the products of two taps, which
// share dZ, are formed by one launch where the kernels can. (Chained products of bf16 storage would be rounded once less.)
namespace {
int32_t taps_prologue(varco_ctx* ctx, int32_t layer, int32_t n_taps, varco_stream stream, const char* fn, Workspace** ws) {
    if (int32_t rc = check_linked(ctx, fn)) return rc;
    ctx->prof.interrupt();
    if (layer < 0 || layer >= ctx->n_layers || n_taps < 1) {
        std::string m = std::string(fn) + ": no such layer, or no tap";
        return varco_fail(ctx, VARCO_ERR_INVALID_ARG, m.c_str());
    }
    return workspace_for(ctx, static_cast<hipStream_t>(stream), ws, fn);
}
bool any_null(int32_t n, const void* const* p) {
    if (!p) return true;
    for (int32_t i = 0; i < n; ++i)
        if (!p[i]) return true;
    return false;
}
}  // namespace

extern "C" int32_t varco_network_taps_fwd(varco_ctx* ctx, int32_t layer, int32_t n_taps, const void* const* y, const void* const* h, void* c,
                                          varco_stream stream) {
    const char* fn = "varco_network_taps_fwd";
    hipStream_t st = static_cast<hipStream_t>(stream);
    Workspace* ws = nullptr;
    if (int32_t rc = taps_prologue(ctx, layer, n_taps, stream, fn, &ws)) return rc;
    if (ctx->net.rows == 0) return VARCO_OK;
    if (any_null(n_taps, y) || any_null(n_taps, h) || !c) return null_pointer(ctx, fn);
    const int32_t fi = ctx->widths[layer], fo = ctx->widths[layer + 1], rows = int32_t(ctx->net.rows);
    const int dt = ctx->dtype;
    for (int32_t t0 = 0; t0 < n_taps; t0 += kWeightSlots) {
        const int32_t n = std::min(kWeightSlots, n_taps - t0);
        GemmArgs g[kWeightSlots];
        PrepJob jobs[kWeightSlots];
        int n_jobs = 0;
        for (int32_t i = 0; i < n; ++i) {
            GemmArgs& p = g[i];
            p.m = rows, p.n = fo, p.k = fi;
            p.a.ptr = y[t0 + i], p.a.ld = fi, p.a.dtype = dt;
            p.b.ptr = h[t0 + i], p.b.ld = fo;
            n_jobs += prep_slot(ctx, *ws, layer, h[t0 + i], fi, fo, true, i, false, p, jobs + n_jobs) ? 1 : 0;
            p.c = c, p.ldc = fo, p.c_dtype = dt;
            p.accumulate = t0 + i > 0;
            p.relu = t0 + i + 1 == n_taps && ctx->act[layer] == VARCO_ACT_RELU;
        }
        ctx->prof.interrupt();
        VARCO_HIP(ctx, varco_launch_prep_weights(jobs, n_jobs, st));
        const double flops = 2.0 * double(rows) * fo * fi;
        if (varco_gemm_split_taps_usable(g, n)) {
            VARCO_HIP(ctx, varco_launch_gemm_split_taps(g, n, st, ctx->tag(VARCO_K_GEMM_FWD, 0, n * flops)));
            continue;
        }
        for (int32_t i = 0; i < n; ++i) VARCO_HIP(ctx, varco_launch_gemm(g[i], st, ctx->tag(VARCO_K_GEMM_FWD, 0, flops)));
    }
    return VARCO_OK;
}

extern "C" int32_t varco_network_taps_bwd_weight(varco_ctx* ctx, int32_t layer, int32_t n_taps, const void* const* y, const void* dx_out,
                                                 const void* x_out, void* const* dh, varco_stream stream) {
    const char* fn = "varco_network_taps_bwd_weight";
    hipStream_t st = static_cast<hipStream_t>(stream);
    Workspace* ws = nullptr;
    if (int32_t rc = taps_prologue(ctx, layer, n_taps, stream, fn, &ws)) return rc;
    if (ctx->net.rows == 0) return VARCO_OK;
    const bool relu = ctx->act[layer] == VARCO_ACT_RELU;
    if (any_null(n_taps, y) || any_null(n_taps, dh) || !dx_out || (relu && !x_out)) return null_pointer(ctx, fn);
    const int32_t fi = ctx->widths[layer], fo = ctx->widths[layer + 1];
    const int dt = ctx->dtype;
    WeightSums sums;
    for (int32_t i = 0; i < n_taps;) {
        GemmArgs g;
        g.m = fi, g.n = fo, g.k = int32_t(ctx->net.rows);
        g.a.ptr = y[i], g.a.ld = fi, g.a.transposed = true, g.a.dtype = dt;
        g.b.ptr = dx_out, g.b.gate = relu ? x_out : nullptr, g.b.ld = fo, g.b.dtype = dt;
        g.c = dh[i], g.ldc = fo;
        g.accumulate = true;
        g.f32_terms = dt == VARCO_F32 ? ctx->f32_terms : 0;
        if (i + 1 < n_taps) {
            int32_t unused = 0;
            g.deferred = &unused;
            g.a_dual = y[i + 1], g.c_dual = dh[i + 1];
            // (a context of one tap per layer has room for one tap's partial products, which two taps may exceed)
            if (!varco_gemm_dual_usable(g) || size_t(wgrad_splits(ctx, fi, fo, g.k, gemm_kind(g), 2)) * 2 * fi * fo > ws->gemm_elems)
                g.a_dual = nullptr, g.c_dual = nullptr;
        }
        const int32_t products = g.c_dual ? 2 : 1;
        const size_t want = size_t(wgrad_splits(ctx, fi, fo, g.k, gemm_kind(g), products)) * products * fi * fo;
        if (sums.n > 0 && (sums.used + want > ws->gemm_elems || sums.n + products > kMaxReduceJobs))
            if (int32_t rc = finish_sums(ctx, sums, st)) return rc;
        if (int32_t rc = add_weight_product(ctx, *ws, g, sums, st)) return rc;
        i += products;
    }
    return finish_sums(ctx, sums, st);
}

extern "C" int32_t varco_network_taps_bwd_input(varco_ctx* ctx, int32_t layer, int32_t n_taps, const void* dx_out, const void* x_out,
                                                const void* const* h, void* const* g_out, varco_stream stream) {
    const char* fn = "varco_network_taps_bwd_input";
    hipStream_t st = static_cast<hipStream_t>(stream);
    Workspace* ws = nullptr;
    if (int32_t rc = taps_prologue(ctx, layer, n_taps, stream, fn, &ws)) return rc;
    if (ctx->net.rows == 0) return VARCO_OK;
    const bool relu = ctx->act[layer] == VARCO_ACT_RELU;
    if (n_taps > 2) return varco_fail(ctx, VARCO_ERR_INVALID_ARG, "varco_network_taps_bwd_input: one or two taps");
    if (any_null(n_taps, h) || any_null(n_taps, g_out) || !dx_out || (relu && !x_out)) return null_pointer(ctx, fn);
    const int32_t fi = ctx->widths[layer], fo = ctx->widths[layer + 1];
    const int dt = ctx->dtype;
    GemmArgs g[2];
    PrepJob jobs[2];
    int n_jobs = 0;
    for (int32_t i = 0; i < n_taps; ++i) {
        g[i].m = int32_t(ctx->net.rows), g[i].n = fi, g[i].k = fo;
        g[i].a.ptr = dx_out, g[i].a.gate = relu ? x_out : nullptr, g[i].a.ld = fo, g[i].a.dtype = dt;
        g[i].b.ptr = h[i], g[i].b.ld = fo, g[i].b.transposed = true;
        g[i].c = g_out[i], g[i].ldc = fi, g[i].c_dtype = dt;
        g[i].f32_terms = dt == VARCO_F32 ? ctx->f32_terms : 0;
        if (!varco_gemm_short_usable(g[i]))      // (short reductions take the weights as they are)
            n_jobs += prep_slot(ctx, *ws, layer, h[i], fi, fo, false, i, false, g[i], jobs + n_jobs) ? 1 : 0;
    }
    ctx->prof.interrupt();
    VARCO_HIP(ctx, varco_launch_prep_weights(jobs, n_jobs, st));
    int32_t launches = n_taps;
    if (n_taps == 2) {
        g[0].b_dual = g[1].b.ptr, g[0].b_dual_prep = g[1].b_prep, g[0].c_dual = g[1].c;
        if (varco_gemm_dual_usable(g[0]))
            launches = 1;
        else
            g[0].c_dual = nullptr;
    }
    for (int32_t i = 0; i < launches; ++i)
        VARCO_HIP(ctx, varco_launch_gemm(g[i], st, ctx->tag(VARCO_K_GEMM_DGRAD, 0, (g[i].c_dual ? 4.0 : 2.0) * fi * fo * double(g[i].m))));
    return VARCO_OK;
}

// The hop of the last tap is the same product either way round: S^T (dZ H^T), or (S^T dZ) H^T as a class layer forms it (class_sums, class_input),
// with the next tap's dZ H'^T in the same launch. A step of 60,013 nodes 64-128-24, three taps, ratio 4: 633 -> 576 us.
extern "C" int32_t varco_network_taps_bwd_last_hop(varco_ctx* ctx, int32_t tap, const void* dx_out, const void* h_last, const void* h_next, void* g_in,
                                                   int32_t* formed, varco_stream stream) {
    const char* fn = "varco_network_taps_bwd_last_hop";
    int32_t layer = 0, hop = 0;
    Workspace* ws = nullptr;
    if (int32_t rc = tap_prologue(ctx, tap, stream, fn, &layer, &hop, &ws)) return rc;
    if (!formed || !h_last || !h_next || (ctx->net.rows > 0 && (!dx_out || !g_in))) return null_pointer(ctx, fn);
    if (int32_t rc = check_wide_rows(ctx, ctx->widths[layer], {g_in}, fn)) return rc;
    const ClassCall c{const_cast<void*>(dx_out), h_last, h_next, g_in};
    *formed = ctx->net.rows > 0 && narrow_sums_taken(ctx, *ws, layer, c) ? 1 : 0;
    return *formed ? narrow_bwd(ctx, *ws, c, layer, make_rule(ctx, layer, hop), static_cast<hipStream_t>(stream)) : VARCO_OK;
}
