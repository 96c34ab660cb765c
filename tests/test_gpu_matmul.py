"""GPU accuracy of the dense products of eq. (2) in their three forms for fp32 storage (fp32 matrix
instructions; fp32 operands expanded into three or two bf16 terms on the bf16 matrix units), through the
building-block calls of the C ABI, against fp64 products of the same inputs (numpy matmul on the CPU).

terms = 3 must be as accurate as fp32 arithmetic itself, not merely inside the 1e-4 parity bound: the
bound asserted is the one derived for an fp32 product-sum of this length."""
import numpy as np
import pytest
import torch

from gpu_common import KEY, assert_close, dev
from paper_2406_17611_amd import binding as vb
from paper_2406_17611_amd import synth
from paper_2406_17611_amd.runner import PartitionedNetwork

pytestmark = pytest.mark.gpu

# rows: several 128-row tiles and a ragged tail; widths: multiples of 8, of 4 only, and one that forces the
# fallback (47: rows not 16-byte aligned)
SHAPES = [(1000, 256, 256), (777, 100, 256), (1301, 256, 47), (515, 136, 72), (64, 32, 512), (130, 47, 64),
          # one row; exactly one tile; one row past a tile; the narrowest widths; a wide reduction with few rows
          (1, 256, 256), (128, 128, 128), (129, 8, 8), (255, 1, 3), (300, 4, 1), (9, 2048, 40), (2100, 24, 2048),
          # more steps than wavefronts keep in registers, more than 64 columns
          (515, 512, 130), (300, 260, 72)]


def _ctx(fi, fo, act, terms):
    ctx = vb.Context([fi, fo], [act], vb.CONV_GCN, 1, KEY)
    ctx.set_matmul_terms(terms)
    ctx.prepare()
    return ctx


def _bound(terms, length):
    # fp32 accumulation over `length` products: error grows like sqrt(length) * 2^-24 norm-wise; the
    # two-term form adds its 2^-16 per-product truncation
    u = 2.0 ** -24 * max(4.0, np.sqrt(length))
    return 8 * u if terms in (0, 3) else 2.0 ** -14


@pytest.mark.parametrize("terms", [3, 0, 2])
@pytest.mark.parametrize("n,fi,fo", SHAPES)
def test_transform_products(n, fi, fo, terms):
    rng = np.random.default_rng(1000 * fi + fo + n)
    # values over many binades, both signs, some exact zeros: every term of the expansion is exercised
    y = (rng.standard_normal((n, fi)) * np.exp2(rng.integers(-6, 7, size=(n, fi)))).astype(np.float32)
    y[rng.random((n, fi)) < 0.05] = 0.0
    h = synth.glorot(fi, fo, 7, fi + fo).astype(np.float32)
    c0 = rng.standard_normal((n, fo)).astype(np.float32)
    dxo = (rng.standard_normal((n, fo)) / n).astype(np.float32)
    ctx = _ctx(fi, fo, vb.ACT_RELU, terms)
    tol = _bound(terms, max(fi, fo))

    # forward: C = relu(C0 + Y H)
    c = dev(c0)
    ctx.transform_fwd(0, dev(y), dev(h), c, True, True)
    torch.cuda.synchronize()
    ref_c = np.maximum(c0.astype(np.float64) + y.astype(np.float64) @ h.astype(np.float64), 0.0)
    assert_close(c.cpu().numpy(), ref_c, "relu(C0 + Y H)", tol)

    # gradients, with the ReLU mask taken on a stored activation that both sides share
    xo = np.maximum(rng.standard_normal((n, fo)), 0.0).astype(np.float32)
    dz = dxo.astype(np.float64) * (xo > 0)
    dh = torch.zeros(fi, fo, device="cuda")
    ctx2 = _ctx(fi, fo, vb.ACT_RELU, terms)
    # the split of the node dimension needs a partial buffer: sized by a registered partition
    g = synth.small_random_graph(max(n, 8), 3.0, "gcn", seed=5)
    host = vb.partition_build(g.n, g.rowptr, g.colidx, g.vals, np.zeros(g.n, dtype=np.int32), 1)
    ctx2.register_partition(0, host[0])       # (the prepared workspace set follows the registration)
    ctx2.transform_bwd_weight(0, dev(y), dev(dxo), dev(xo), dh)
    torch.cuda.synchronize()
    assert_close(dh.cpu().numpy(), y.astype(np.float64).T @ dz, "Y^T dZ", _bound(terms, n))

    gin0 = rng.standard_normal((n, fi)).astype(np.float32)
    gin = dev(gin0)
    ctx.transform_bwd_input(0, dev(dxo), dev(xo), dev(h), gin, True)
    torch.cuda.synchronize()
    assert_close(gin.cpu().numpy(), gin0.astype(np.float64) + dz @ h.astype(np.float64).T, "G0 + dZ H^T",
                 max(tol, 2.0 ** -22))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("first_row", [0, 1, 3])
def test_input_gradient_short_reduction(first_row, dtype):
    """dZ H^T with 47 reduction steps (the class logits' gradient) on row ranges that start at any row of a
    larger tensor, so that the rows are neither 16-byte aligned nor is the range's start; masked and not. (fp32 storage:
    products from two fp16 terms; bf16 storage: the kernel for short reductions.)"""
    from oracle.rounding import round_bf16
    n, fi, fo = 700, 256, 47
    rng = np.random.default_rng(40 + first_row)
    bf16 = dtype == "bf16"
    tdt = torch.bfloat16 if bf16 else torch.float32
    rnd = (lambda a: round_bf16(a).astype(np.float32)) if bf16 else (lambda a: a.astype(np.float32))
    h = synth.glorot(fi, fo, 9, 1).astype(np.float32)
    dxo_all = rnd(rng.standard_normal((n + first_row, fo)))
    xo_all = rnd(np.maximum(rng.standard_normal((n + first_row, fo)), 0.0))
    dxo_d, xo_d = dev(dxo_all, tdt), dev(xo_all, tdt)
    tol = 2.0 ** -7 if bf16 else 8 * 2.0 ** -24 * np.sqrt(fo)
    for act in (vb.ACT_IDENTITY, vb.ACT_RELU):
        ctx = vb.Context([fi, fo], [act], vb.CONV_GCN, 1, KEY, vb.BF16 if bf16 else vb.F32)
        ctx.prepare()
        g0 = rnd(rng.standard_normal((n, fi)))
        gout = dev(g0, tdt)
        ctx.transform_bwd_input(0, dxo_d[first_row:], xo_d[first_row:], dev(h), gout, True)
        torch.cuda.synchronize()
        dz = dxo_all[first_row:].astype(np.float64)
        if act == vb.ACT_RELU:
            dz = dz * (xo_all[first_row:] > 0)
        ref = g0.astype(np.float64) + dz @ h.astype(np.float64).T
        assert_close(gout.float().cpu().numpy(), ref, f"G0 + dZ H^T from row {first_row}", tol)


@pytest.mark.parametrize("terms", [3, 2])
@pytest.mark.parametrize("fo", [33, 47, 48])
def test_input_gradient_short_reduction_over_many_rows(fo, terms):
    """fp32 input gradients of 33 to 48 steps, more than 128 columns and 300,000 rows: the kernel for short reductions, from any row,
    masked, alone (adding to the result) and for two taps in one launch."""
    from test_gpu_weight_gradients import _linked_context
    n, fi = 300_013, 132
    gen = torch.Generator(device="cuda")
    gen.manual_seed(fo)
    randn = lambda *s: torch.randn(*s, generator=gen, device="cuda")     # noqa: E731
    h = [randn(fi, fo) for _ in range(2)]
    d, x = randn(n + 1, fo), randn(n + 1, fo)
    dz = torch.where(x > 0, d, torch.zeros_like(d)).double()
    # a product-sum in fp32 (terms 3), 2^-16 per product and operand (terms 2); adding to g0 rounds once more
    tol = 8 * 2.0 ** -24 * np.sqrt(fo) if terms == 3 else 2.0 ** -14

    def check(got, ref):
        assert float((got.double() - ref).norm()) <= tol * float(ref.norm())
        assert float((got.double() - ref).abs().max()) <= tol * float(ref.abs().max())

    ctx = _ctx(fi, fo, vb.ACT_RELU, terms)
    g0 = randn(n, fi)
    out = g0.clone()
    ctx.transform_bwd_input(0, d[1:], x[1:], h[0], out, True)
    torch.cuda.synchronize()
    check(out, g0.double() + dz[1:] @ h[0].double().t())
    ctx, held = _linked_context(n, 2, fi, fo, vb.F32, terms)
    pair = [torch.empty(n, fi, device="cuda") for _ in range(2)]
    ctx.network_taps_bwd_input(0, d[:n], x[:n], h, pair)
    torch.cuda.synchronize()
    for got, ht in zip(pair, h):
        check(got, dz[:n] @ ht.double().t())
    ctx.close()
    del held


@pytest.mark.parametrize("n,wide,short", [(8100, 2040, 48), (8065, 2048, 70), (16350, 1012, 200)])
def test_bf16_products_of_whole_device_tiles(n, wide, short):
    """bf16 products wide and tall enough for 128 x 256 tiles (512 of them or more): ragged last tiles in both directions,
    reductions shorter than a stage of 64 steps, past one and over several, rows of any alignment; plain and masked."""
    from oracle.rounding import round_bf16
    rng = np.random.default_rng(n + wide + short)
    rnd = lambda a: round_bf16(a).astype(np.float32)
    bf = torch.bfloat16
    y = rnd(rng.standard_normal((n, short)))
    h = synth.glorot(short, wide, 5, 2).astype(np.float32)
    c = torch.empty(n, wide, dtype=bf, device="cuda")
    ctx = vb.Context([short, wide], [vb.ACT_IDENTITY], vb.CONV_GCN, 1, KEY, vb.BF16)
    ctx.prepare()
    ctx.transform_fwd(0, dev(y, bf), dev(h), c, False, False)
    torch.cuda.synchronize()
    # weights and results are rounded to bf16 (2^-9 relative each)
    assert_close(c.float().cpu().numpy(), y.astype(np.float64) @ h.astype(np.float64), "Y H", 2.0 ** -7)

    ctx = vb.Context([wide, short], [vb.ACT_RELU], vb.CONV_GCN, 1, KEY, vb.BF16)
    ctx.prepare()
    xo = rnd(np.maximum(rng.standard_normal((n, short)), 0.0))
    gin = torch.empty(n, wide, dtype=bf, device="cuda")
    ctx.transform_bwd_input(0, dev(y, bf), dev(xo, bf), dev(np.ascontiguousarray(h.T)), gin, False)
    torch.cuda.synchronize()
    ref = (y.astype(np.float64) * (xo > 0)) @ h.astype(np.float64)
    assert_close(gin.float().cpu().numpy(), ref, "masked dZ H^T", 2.0 ** -7)


@pytest.mark.parametrize("mode", ["f32x3", "f32x2", "bf16"])
@pytest.mark.parametrize("fo", [47, 3, 1, 62])
@pytest.mark.parametrize("first_row", [0, 1])
def test_weight_gradient_of_unaligned_columns(first_row, fo, mode):
    """Y^T dZ where dZ has a width that is no multiple of 4 and no activation mask (the class logits of the last
    layer): its rows are not aligned, and the range may start at any row of a larger tensor. The reduction over
    the rows spans several tiles, a ragged last tile and several workgroups."""
    from oracle.rounding import round_bf16
    n, fi = 2333, 256
    rng = np.random.default_rng(300 + fo + first_row)
    bf16 = mode == "bf16"
    tdt = torch.bfloat16 if bf16 else torch.float32
    rnd = (lambda a: round_bf16(a).astype(np.float32)) if bf16 else (lambda a: a.astype(np.float32))
    y = rnd(rng.standard_normal((n, fi)) * np.exp2(rng.integers(-4, 5, size=(n, fi))))
    dz_all = rnd(rng.standard_normal((n + first_row, fo)) / n)
    ctx = vb.Context([fi, fo], [vb.ACT_IDENTITY], vb.CONV_GCN, 1, KEY, vb.BF16 if bf16 else vb.F32)
    if not bf16:
        ctx.set_matmul_terms(3 if mode == "f32x3" else 2)
    g = synth.small_random_graph(n, 3.0, "gcn", seed=5)
    host = vb.partition_build(g.n, g.rowptr, g.colidx, g.vals, np.zeros(g.n, dtype=np.int32), 1)
    ctx.register_partition(0, host[0])
    ctx.prepare()
    dh0 = rng.standard_normal((fi, fo)).astype(np.float32)
    dh = dev(dh0)
    ctx.transform_bwd_weight(0, dev(y, tdt), dev(dz_all, tdt)[first_row:], None, dh)      # adds to dh
    torch.cuda.synchronize()
    ref = dh0.astype(np.float64) + y.astype(np.float64).T @ dz_all[first_row:].astype(np.float64)
    tol = 2.0 ** -14 if mode == "f32x2" else 8 * 2.0 ** -24 * np.sqrt(n)
    assert_close(dh.cpu().numpy(), ref, f"dH0 + Y^T dZ, {fo} columns from row {first_row}", tol)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_weights_changed_between_steps_are_seen(dtype):
    """The library may keep converted copies of the weights during a step; after an in-place update and the
    next step call the new values must be used (both orientations: transform and input gradient)."""
    n, fi, fo = 300, 64, 96
    rng = np.random.default_rng(77)
    bf16 = dtype == "bf16"
    tdt = torch.bfloat16 if bf16 else torch.float32
    tol = 2.0 ** -7 if bf16 else 1e-5
    ctx = vb.Context([fi, fo], [vb.ACT_IDENTITY], vb.CONV_GCN, 1, KEY, vb.BF16 if bf16 else vb.F32)
    ctx.prepare()
    y = torch.from_numpy(rng.standard_normal((n, fi)).astype(np.float32)).to(tdt).cuda()
    d = torch.from_numpy(rng.standard_normal((n, fo)).astype(np.float32)).to(tdt).cuda()
    h = dev(synth.glorot(fi, fo, 3, 0))
    c = torch.empty(n, fo, dtype=tdt, device="cuda")
    gin = torch.empty(n, fi, dtype=tdt, device="cuda")
    for step in range(3):
        ctx.set_step(step)
        for _ in range(2):          # the second call of a step may reuse the first one's copies
            ctx.transform_fwd(0, y, h, c, False, False)
            ctx.transform_bwd_input(0, d, None, h, gin, False)
        torch.cuda.synchronize()
        hh = h.cpu().numpy().astype(np.float64)
        assert_close(c.float().cpu().numpy(), y.float().cpu().numpy().astype(np.float64) @ hh, f"Y H at step {step}", tol)
        assert_close(gin.float().cpu().numpy(), d.float().cpu().numpy().astype(np.float64) @ hh.T, f"dZ H^T at step {step}", tol)
        h.mul_(-1.5).add_(0.01)     # in-place update, same address
    torch.cuda.synchronize()


@pytest.mark.parametrize("terms", [3, 0])
def test_non_finite_operand_stays_in_its_row(terms):
    """An infinite activation makes its own output row non-finite (NaN with the bf16-term products, infinite or
    NaN with fp32 instructions) and leaves every other row as it was."""
    n, fi, fo = 300, 128, 128
    rng = np.random.default_rng(5)
    y = rng.standard_normal((n, fi)).astype(np.float32)
    h = (synth.glorot(fi, fo, 2, 0) + 0.01).astype(np.float32)
    ref = y.astype(np.float64) @ h.astype(np.float64)
    y[137, 5] = np.inf
    ctx = _ctx(fi, fo, vb.ACT_IDENTITY, terms)
    c = torch.empty(n, fo, device="cuda")
    ctx.transform_fwd(0, dev(y), dev(h), c, False, False)
    torch.cuda.synchronize()
    got = c.cpu().numpy()
    assert not np.isfinite(got[137]).any()
    if terms == 3:
        assert np.isnan(got[137]).all()
    keep = np.arange(n) != 137
    assert_close(got[keep], ref[keep], "rows without the infinite element", _bound(terms, fi))


@pytest.mark.parametrize("fi,fo", [(65, 8), (75, 200), (96, 72), (100, 256), (127, 130), (131, 40), (160, 129), (192, 136), (200, 257), (224, 65), (255, 512), (256, 256)])
@pytest.mark.parametrize("taps", [1, 2])
@pytest.mark.parametrize("n", [2, 31, 33, 3001, 32801])
def test_transform_at_the_edges_of_blocks(n, taps, fi, fo):
    """One tap: rows in blocks of 32 of workgroups that walk over them, columns in units of 32 of wavefronts, every number of stages, added to
    what is there. Two: the chained tiles of a K-tap layer. Rows that start at any word of a larger tensor."""
    from test_gpu_weight_gradients import _linked_context
    rng = np.random.default_rng(n + fi + fo)
    y = [rng.standard_normal((n, fi)).astype(np.float32) for _ in range(taps)]
    h = [synth.glorot(fi, fo, 3, 1 + t).astype(np.float32) for t in range(taps)]
    old = rng.standard_normal((n + 1, fo)).astype(np.float32)
    out = dev(old)
    held = [torch.zeros(n * fi + 1, device="cuda") for _ in y]
    for t, one in zip(held, y):
        t[1:] = dev(one).flatten()
    rows = [t[1:].view(n, fi) for t in held]
    if taps == 1:
        ctx, parts = _ctx(fi, fo, vb.ACT_RELU, 3), None
        ctx.transform_fwd(0, rows[0], dev(h[0]), out[:n], True, True)
    else:
        ctx, parts = _linked_context(n, 2, fi, fo, vb.F32, 3)
        ctx.network_taps_fwd(0, rows, [dev(w) for w in h], out[:n])
    torch.cuda.synchronize()
    want = sum(a.astype(np.float64) @ b.astype(np.float64) for a, b in zip(y, h)) + (old[:n] if taps == 1 else 0.0)
    size = sum(np.abs(a) @ np.abs(b) for a, b in zip(y, h))
    # terms left out are below 2^-24 of a product; one rounding of 2^-24 per instruction (six per 16 steps) on a partial sum that is at most `size`:
    # sqrt of their number for independent ones, four times that for the tail; the addition rounds once more
    bound = (2.0 ** -24 + 4 * 2.0 ** -24 * np.sqrt(6 * taps * np.ceil(fi / 16))) * size + (2.0 ** -24 * np.abs(want) if taps == 1 else 0.0)
    got = out.cpu().numpy()
    assert (np.abs(got[:n] - np.maximum(want, 0.0)) <= bound).all()
    assert np.array_equal(got[n], old[n])                             # the row behind the last one
    ctx.close()
    del parts


@pytest.mark.parametrize("fi,fo", [(68, 65), (80, 132), (96, 72), (100, 256), (104, 257), (124, 136), (128, 130)])
@pytest.mark.parametrize("n", [2, 33, 3001, 32801])
def test_layer_of_two_taps_at_the_edges_of_blocks(n, fi, fo):
    """A SAGE layer's transform, both taps' weights in the wavefronts: blocks of 32 rows, a tap at a time, units of 32 columns, three and four
    stages to a tap, the rows of either tap from any word of a larger tensor on."""
    graph = synth.small_random_graph(n, 2.0, "sage", seed=n)
    host = vb.partition_build(graph.n, graph.rowptr, graph.colidx, graph.vals, synth.random_partition(graph.n, 2, seed=5), 2)
    rng = np.random.default_rng(n + fi + fo)
    net = PartitionedNetwork(host, (fi, fo, 4), "sage", 17, need_backward=False)
    moved = [torch.zeros(n * fi + 1, device="cuda") for _ in range(2)]
    net.x[0], net.m[0] = (t[1:].view(n, fi) for t in moved)
    whole = torch.full((n + 1, fo), 7.0, device="cuda")
    net.x[1] = whole[:n]
    h = [[synth.glorot(a, b, 3, 1 + t).astype(np.float32) for a, b in ((fi, fo), (fo, 4))] for t in range(2)]
    net.set_weights(*h)
    net.set_inputs(rng.standard_normal((n, fi)).astype(np.float32))
    net.forward(1, (4, 1))
    torch.cuda.synchronize()
    taps = [(net.m[0].cpu().numpy().astype(np.float64), h[0][0]), (net.x[0].cpu().numpy().astype(np.float64), h[1][0])]
    want = sum(a @ b.astype(np.float64) for a, b in taps)
    size = sum(np.abs(a) @ np.abs(b) for a, b in taps)
    bound = (2.0 ** -24 + 4 * 2.0 ** -24 * np.sqrt(6 * 2 * np.ceil(fi / 16))) * size       # as above
    got = whole.cpu().numpy()
    assert (np.abs(got[:n] - np.maximum(want, 0.0)) <= bound).all()
    assert (got[n] == 7.0).all()                                      # the row behind the last one
    net.ctx.close()


@pytest.mark.parametrize("fi,fo", [(68, 72), (80, 132), (96, 130), (100, 256), (128, 136), (144, 96), (180, 257), (224, 65), (256, 512)])
@pytest.mark.parametrize("conv", ["gcn", "sage"])
@pytest.mark.parametrize("n", [2, 33, 3001, 32801])
def test_transform_sums_do_not_depend_on_the_kernel(n, conv, fi, fo):
    """Outputs of up to 64 columns are formed by tiles, wider ones mostly by wavefronts that keep the weights: the same bits, since a ReLU whose
    argument is within rounding of zero must not open by the width of its layer or the number of rows."""
    graph = synth.small_random_graph(n, 2.0, conv, seed=n)
    host = vb.partition_build(graph.n, graph.rowptr, graph.colidx, graph.vals, synth.random_partition(graph.n, 2, seed=5), 2)
    h1, h0 = (synth.glorot(fi, fo, 7, 1 + t).astype(np.float32) for t in range(2))
    x0 = np.random.default_rng(n + fi).standard_normal((n, fi)).astype(np.float32)

    def outputs(c0, c1):
        net = PartitionedNetwork(host, (fi, c1 - c0), conv, 17, need_backward=False)
        net.set_inputs(x0)
        net.set_weights([np.ascontiguousarray(h1[:, c0:c1])], [np.ascontiguousarray(h0[:, c0:c1])])
        net.forward(1, (4, 1))
        torch.cuda.synchronize()
        return net.x[1].clone()

    whole = outputs(0, fo)
    for c0 in range(0, fo, 64):
        assert torch.equal(whole[:, c0:c0 + 64].view(torch.int32), outputs(c0, min(c0 + 64, fo)).view(torch.int32)), c0


@pytest.mark.parametrize("fi,fo", [(8, 8), (64, 128), (64, 24), (100, 130), (256, 256), (76, 64), (75, 40)])
@pytest.mark.parametrize("n,taps", [(1, 2), (127, 3), (129, 4), (3001, 3), (3001, 5)])
def test_taps_together_are_the_taps_in_turn(n, taps, fi, fo):
    """The products of all taps of a layer in one launch: the bits of one launch after the other, each adding to the one before."""
    from test_gpu_weight_gradients import _linked_context
    rng = np.random.default_rng(n + fi + fo)
    y = [dev(rng.standard_normal((n, fi)).astype(np.float32)) for _ in range(taps)]
    h = [dev(synth.glorot(fi, fo, 3, 1 + t).astype(np.float32)) for t in range(taps)]
    ctx, parts = _linked_context(n, min(n, 2), fi, fo, vb.F32, 3)
    together, in_turn = (torch.full((n + 1, fo), 7.0, device="cuda") for _ in range(2))
    ctx.network_taps_fwd(0, y, h, together[:n])
    for t in range(taps):
        ctx.transform_fwd(0, y[t], h[t], in_turn[:n], t > 0, t == taps - 1)
    torch.cuda.synchronize()
    assert torch.equal(together.view(torch.int32), in_turn.view(torch.int32))
    ctx.close()
    del parts
