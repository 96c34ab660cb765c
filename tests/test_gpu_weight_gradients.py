"""Accuracy of weight gradients formed over all partitions at once: sums over many rows are cut so that no fp32 accumulator
takes longer chains than the rule for its kind of product allows, and partial sums are added in fp64."""
import numpy as np
import pytest
import torch

from gpu_common import KEY
from paper_2406_17611_amd import binding as vb
from paper_2406_17611_amd import synth
from paper_2406_17611_amd.runner import PartitionedNetwork

pytestmark = pytest.mark.gpu


def _linked_context(n, n_parts, fi, fo, dtype, terms):
    """Partitions without edges: the dense products over the arena are all that is used."""
    none = np.zeros(0, dtype=np.int64)
    g = synth.gcn_operator(n, none, none)
    part = np.sort(np.arange(n) % n_parts).astype(np.int32)
    host = vb.partition_build(g.n, g.rowptr, g.colidx, g.vals, part, n_parts)
    ctx = vb.Context([fi, fo], [vb.ACT_RELU], vb.CONV_SAGE, n_parts, KEY, dtype)
    if dtype == vb.F32:
        ctx.set_matmul_terms(terms)
    held = [ctx.register_partition(q, hp) for q, hp in enumerate(host)]
    assert ctx.link_partitions()
    ctx.prepare()
    return ctx, held


# rows a slab may hold for these sizes, and roundings per row. With two fp16 terms the large sum takes one per 16 rows; operands are
# within 2^-23, 7.5e-8 in the root mean square of a product; and the matrix unit cuts instead of rounding, an error of one sign
# that slabs of alternating sign do not cancel altogether: a quarter. fp32 instructions round once per 2 rows, bf16 once per 8.
@pytest.mark.parametrize("dtype,terms,fi,fo,slab_rows,roundings,operands,margin",
                         [(vb.F32, 3, 256, 256, 330 * (137_500 + 169_343) / 73_300, 1 / 16, 7.5e-8, 1.25), (vb.F32, 0, 256, 256, 220, 1 / 2, 0.0, 1.0),
                          (vb.BF16, 1, 512, 512, 661 + 4 * 64 + 16 * 4, 1 / 8, 0.0, 1.0)])
def test_long_reductions_keep_the_accuracy_of_short_ones(dtype, terms, fi, fo, slab_rows, roundings, operands, margin):
    n, n_parts = 169_343, 4
    ctx, held = _linked_context(n, n_parts, fi, fo, dtype, terms)
    tdt = torch.bfloat16 if dtype == vb.BF16 else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    randn = lambda *s: torch.randn(*s, generator=gen, device="cuda")     # noqa: E731
    y = [randn(n, fi).to(tdt) for _ in range(2)]
    d = (randn(n, fo) / n).to(tdt)
    x = randn(n, fo).clamp_min(0).to(tdt)
    dh = [torch.zeros(fi, fo, device="cuda") for _ in range(2)]
    ctx.network_taps_bwd_weight(0, y, d, x, dh)
    dz = torch.where(x > 0, d, torch.zeros_like(d)).double()
    # a rounding of a sum s is within 2^-24 |s|, 2^-24 / sqrt(3) of it in the root mean square; independent products make s^2 grow
    # linearly along a chain, so that its mean is half of the end's
    bound = margin * np.hypot(2.0 ** -24 / np.sqrt(3) * np.sqrt(slab_rows * roundings / 2), operands)
    for yt, got in zip(y, dh):
        ref = yt.double().t() @ dz
        err = float((got.double() - ref).norm() / ref.norm())
        assert err <= bound, (err, bound)
    ctx.close()
    del held


def test_received_rows_of_many_shares():
    """More boundary rows than one round of workgroups may sum (512 shares of 1,024 rows), a remainder included, against the
    other order of the layer's products."""
    n = 2 * 512 * 1024 + 77                            # every node of a ring dealt to two partitions is a boundary node
    u = np.arange(n - 1, dtype=np.int64)
    g = synth.gcn_operator(n, u, u + 1)
    host = vb.partition_build(g.n, g.rowptr, g.colidx, g.vals, (np.arange(n) % 2).astype(np.int32), 2)
    widths = (16, 32, 5)
    h1 = [synth.glorot(widths[l], widths[l + 1], 11, l) for l in range(2)]
    got = []
    for first in ((1,), ()):
        net = PartitionedNetwork(host, widths, "gcn", KEY, dtype="bf16", transform_first=first)
        net.set_weights(h1)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(3)
        net.x[0].copy_(torch.randn(n, 16, generator=gen, device="cuda"))
        net.dx[2].copy_((torch.randn(n, 5, generator=gen, device="cuda") + 0.5) / n)
        net.step(3, (2, 1))
        torch.cuda.synchronize()
        got.append(net.dh1[1].double().cpu().numpy())
        net.ctx.close()
    # three bf16 roundings of 2^-9 at most lie between the stored activations and a gradient in either order
    assert np.abs(got[0] - got[1]).max() <= 6 * 2.0 ** -9 * np.abs(got[1]).max()


@pytest.mark.parametrize("conv,widths", [("sage", (33, 64, 65, 40, 7)), ("gcn", (130, 128, 200, 64, 3)), ("sage", (16, 32, 8)), ("gcn", (7, 129, 130, 131))])
@pytest.mark.parametrize("n", [31, 700])
@pytest.mark.parametrize("shared", [False, True])
def test_products_of_all_layers_in_one_launch(n, conv, widths, shared):
    """Products of layers of few rows wait for the end of the pass: narrow and wide outputs, masked and not, one tap and two, one layer of a kind.
    shared: the rows that a product reads are where a lower layer's gradient goes."""
    g = synth.small_random_graph(n, 5.0, conv, seed=7)
    host = vb.partition_build(g.n, g.rowptr, g.colidx, g.vals, synth.random_partition(g.n, 3, seed=8), 3)
    net = PartitionedNetwork(host, widths, conv, KEY)
    layers = range(len(widths) - 1)
    rng = np.random.default_rng(n)
    net.set_inputs(rng.standard_normal((n, widths[0])).astype(np.float32))
    weights = [[rng.standard_normal((widths[l], widths[l + 1])).astype(np.float32) for l in layers] for _ in range(2)]
    net.set_weights(weights[0], weights[1] if conv == "sage" else None)
    net.set_upstream(rng.standard_normal((n, widths[-1])).astype(np.float32))
    net.zero_grads()
    net.forward(0, (2, 1))
    m = [net.m[l].double() for l in layers]
    if shared:
        for l in layers[1:]:
            net.dx[l] = net.m[l]
    net.backward()
    torch.cuda.synchronize()
    for l in layers:
        dz = net.dx[l + 1].double()
        if l < layers[-1]:
            dz = torch.where(net.x[l + 1] > 0, dz, torch.zeros_like(dz))
        for got, a in [(net.dh1[l], m[l])] + ([(net.dh0[l], net.x[l].double())] if conv == "sage" else []):
            # two scaled terms within 2^-23 of either operand, a rounding of 2^-24 per 16 rows of a slab and per slab, and four times their root for the tail
            bound = (2.0 ** -21 + 4 * 2.0 ** -23 * (n / 16 + 1) ** 0.5) * (a.abs().t() @ dz.abs())
            # values far below the largest of their column keep 2^-42 of that one
            floor = 2.0 ** -42 * (a.abs().max() * dz.abs().sum(0)[None, :] + a.abs().sum(0)[:, None] * dz.abs().max())
            assert ((got.double() - a.t() @ dz).abs() <= bound + floor).all(), l


@pytest.mark.parametrize("n,parts,conv,widths", [(100_000, 2, "gcn", (64, 64, 64, 40)), (6_000, 3, "gcn", (128, 256, 256, 40)), (3_997, 4, "sage", (93, 208, 120, 14)),
                                                 (2_000, 2, "gcn", (16, 32, 8))])
def test_products_that_share_a_launch_keep_their_slabs(n, parts, conv, widths):
    """The same bits as in launches of their own: as accurate as those, whatever else a network's layers have the device do."""
    g = synth.small_random_graph(n, 4.0, conv, seed=5)
    host = vb.partition_build(g.n, g.rowptr, g.colidx, g.vals, synth.random_partition(g.n, parts, seed=6), parts)
    net = PartitionedNetwork(host, widths, conv, KEY)
    layers = range(len(widths) - 1)
    rng = np.random.default_rng(n)
    net.set_inputs(rng.standard_normal((n, widths[0])).astype(np.float32))
    weights = [[rng.standard_normal((widths[l], widths[l + 1])).astype(np.float32) for l in layers] for _ in range(2)]
    net.set_weights(weights[0], weights[1] if conv == "sage" else None)
    net.set_upstream(rng.standard_normal((n, widths[-1])).astype(np.float32))
    net.zero_grads()
    net.forward(0, (4, 1))
    net.backward()
    for l in layers:
        rows, got = ([net.m[l], net.x[l]], [net.dh1[l], net.dh0[l]]) if conv == "sage" else ([net.m[l]], [net.dh1[l]])
        want = [torch.zeros_like(t) for t in got]
        net.ctx.network_taps_bwd_weight(l, rows, net.dx[l + 1], net.x[l + 1], want)
        for a, b in zip(got, want):
            assert torch.equal(a, b), (l, float((a - b).abs().max()))
    net.ctx.close()


@pytest.mark.parametrize("fi,fo", [(16, 200), (100, 130), (129, 65), (200, 136), (300, 60), (257, 257)])
@pytest.mark.parametrize("n", [31, 1_999, 5_003, 20_011])
def test_tiles_of_any_size(n, fi, fo):
    """Few slabs, which take small tiles, to many: one tap and two, masked, columns and rows that no tile divides."""
    ctx, held = _linked_context(n, 3, fi, fo, vb.F32, 3)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + fi)
    randn = lambda *s: torch.randn(*s, generator=gen, device="cuda")     # noqa: E731
    y, d, x = [randn(n, fi) for _ in range(2)], randn(n, fo), randn(n, fo)
    dz = torch.where(x > 0, d, torch.zeros_like(d)).double()
    for taps in (1, 2):
        dh = [torch.full((fi, fo), 3.0, device="cuda") for _ in range(taps)]
        ctx.network_taps_bwd_weight(0, y[:taps], d, x, dh)
        for yt, got in zip(y, dh):
            # two scaled terms within 2^-23 of either operand, a rounding of 2^-24 per 16 rows of a slab and per slab, four times their root for the tail
            bound = (2.0 ** -21 + 4 * 2.0 ** -23 * (n / 16 + 1) ** 0.5) * (yt.double().abs().t() @ dz.abs()) + 2.0 ** -23 * 3.0
            assert ((got.double() - 3.0 - yt.double().t() @ dz).abs() <= bound + 2.0 ** -42 * n * float(yt.abs().max() * d.abs().max())).all()
    ctx.close()
    del held
