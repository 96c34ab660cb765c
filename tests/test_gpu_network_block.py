"""The calls that serve all partitions at once (varco_link_partitions, varco_network_*) at the sizes where their node
sums change form: hub nodes whose local and cross entries are cut into pieces, widths that need one to several loads per
lane or element loads, messages summed from the product buffer, taken from whole rows, complete or absent."""
import numpy as np
import pytest
import torch

from gpu_common import KEY, both_partitions, hub_graph
from paper_2406_17611_amd import binding as vb
from paper_2406_17611_amd import synth
from paper_2406_17611_amd.runner import PartitionedNetwork
from test_gpu_network import BF16_TOL, _compare_network

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("conv,widths,dtype", [("gcn", (20, 64, 9), "f32"), ("sage", (33, 30, 7), "f32"), ("gcn", (16, 256, 12), "f32"),
                                               ("sage", (24, 516, 5), "f32"), ("gcn", (20, 96, 9), "bf16"), ("sage", (17, 512, 6), "bf16")])
def test_node_sums_with_hubs(conv, widths, dtype):
    g = hub_graph(1500, 3, 1100, 6.0, conv, seed=81)
    part = synth.random_partition(g.n, 3, seed=82)
    # 1/8 and 1/5 (ragged k) of a row: products, where a row is long enough (256 and 516 fp32 columns), or masked; 2/3: whole rows masked; all; nothing
    ratios = [(8, 1), (5, 1), (3, 2), (1, 1), (1, 0)]
    _compare_network(g, part, 3, conv, widths, ratios, steps=list(range(5)), tol=BF16_TOL if dtype == "bf16" else 1e-4, dtype=dtype)


@pytest.mark.parametrize("conv,widths", [("gcn", (16, 48, 5)), ("sage", (24, 512, 64)), ("gcn", (40, 208, 47)), ("sage", (32, 7))])
def test_class_layer_transforms_first_with_hubs(conv, widths):
    # rows of 1 to 64 outputs; k ragged, complete and 0; tiles of 32 and 64 rows with a remainder
    g = hub_graph(1500, 3, 1100, 6.0, conv, seed=86)
    part = synth.random_partition(g.n, 3, seed=87)
    ratios = [(8, 1), (5, 1), (3, 2), (1, 1), (1, 0)]
    _compare_network(g, part, 3, conv, widths, ratios, steps=list(range(5)), tol=BF16_TOL, dtype="bf16", transform_first=(len(widths) - 2,))


@pytest.mark.parametrize("conv,widths,dtype", [("gcn", (20, 112, 1), "bf16"), ("sage", (16, 64, 33), "bf16"), ("sage", (24, 512, 64), "bf16"),
                                               ("gcn", (40, 208, 47), "bf16"), ("gcn", (20, 24, 96, 80), "bf16"), ("sage", (17, 512, 72), "bf16"),
                                               ("gcn", (20, 112, 1), "f32"), ("sage", (16, 65, 33), "f32"), ("sage", (24, 512, 64), "f32"),
                                               ("gcn", (40, 208, 47), "f32"), ("sage", (17, 72, 16), "f32"), ("sage", (16, 61, 32), "f32"),
                                               ("gcn", (24, 516, 48), "f32"), ("gcn", (20, 64, 80), "f32"), ("sage", (33, 30, 70), "f32"),
                                               ("gcn", (16, 256, 72), "f32"), ("sage", (24, 516, 70), "f32")])
def test_class_layer_errors_with_hubs(conv, widths, dtype):
    # an aggregated-first class layer sums its errors at the width of its outputs (1 to 64 of them), wider outputs at the width of
    # the inputs; k short, ragged, complete and 0
    g = hub_graph(1500, 3, 1100, 6.0, conv, seed=91)
    part = synth.random_partition(g.n, 3, seed=92)
    ratios = [(16, 1), (5, 1), (3, 2), (1, 1), (1, 0)]
    _compare_network(g, part, 3, conv, widths, ratios, steps=list(range(5)), tol=BF16_TOL if dtype == "bf16" else 1e-4, dtype=dtype)


@pytest.mark.parametrize("conv,widths,dtype", [("gcn", (16, 48, 3), "bf16"), ("sage", (16, 144, 33), "bf16"), ("sage", (16, 144, 33), "f32"),
                                               ("gcn", (16, 40, 47), "f32"), ("sage", (16, 65, 50), "f32")])
def test_class_layer_errors_over_many_tiles(conv, widths, dtype):
    # more tiles of rows than workgroups, several times over: both LDS buffers are written again, the last tile has a remainder; rows
    # of dZ of any length padded (shorter than 16 bytes, and longer)
    g = hub_graph(131_100, 3, 900, 2.0, conv, seed=93)
    part = synth.random_partition(g.n, 3, seed=94)
    _compare_network(g, part, 3, conv, widths, [(5, 1), (1, 1)], steps=[0, 1], tol=BF16_TOL if dtype == "bf16" else 1e-4, dtype=dtype)


def test_uneven_and_empty_partitions():
    g = synth.small_random_graph(300, 5.0, "gcn", seed=83)
    part = np.zeros(g.n, dtype=np.int32)
    part[20:] = 2                                        # partition 1 owns nothing
    _compare_network(g, part, 3, "gcn", (12, 40, 5), [(4, 1), (1, 1)], steps=[0, 1])


def test_linked_calls_need_a_link_and_a_changed_partition_drops_it():
    g = synth.small_random_graph(200, 5.0, "gcn", seed=84)
    host, _ = both_partitions(g, synth.random_partition(g.n, 2, seed=85), 2)
    net = PartitionedNetwork(host, (8, 16, 4), "gcn", KEY)
    assert net.linked
    net.set_weights([synth.glorot(8, 16, 1), synth.glorot(16, 4, 2)])
    net.set_inputs(synth.features(g.n, 8, 3))
    net.forward(0, (2, 1))
    torch.cuda.synchronize()
    want = net.x[2].clone()
    net.ctx.register_partition(1, host[1])
    with pytest.raises(vb.VarcoError) as e:
        net.forward(0, (2, 1))
    assert e.value.code == vb.ERR_STATE
    assert net.ctx.link_partitions()
    net.forward(0, (2, 1))
    torch.cuda.synchronize()
    assert torch.equal(net.x[2], want)
    # a map of returned rows that names another node's rows is refused
    bad = host[0]
    bad.ret_src = bad.ret_src[::-1].copy()
    net.ctx.register_partition(0, bad)
    with pytest.raises(vb.VarcoError) as e:
        net.ctx.link_partitions()
    assert e.value.code == vb.ERR_SHAPE


@pytest.mark.parametrize("widths,ratio,dtype,n", [((4, 8, 4), (2, 1), "f32", 900), ((20, 36, 7), (3, 1), "f32", 900), ((128, 256, 5), (8, 1), "bf16", 900),
                                                  ((252, 60, 9), (4, 1), "f32", 700), ((256, 128, 9), (4, 1), "f32", 1), ((64, 256, 9), (2, 1), "bf16", 700),
                                                  ((100, 256, 9), (4, 1), "f32", 600), ((75, 130, 9), (3, 1), "f32", 500)])
def test_messages_written_with_the_sums(widths, ratio, dtype, n):
    """A forward pass of few entries writes the messages and sums their kept elements from the owners' rows in one launch: the same bits
    as messages first and their sums after, for every lane layout, rows long enough to be split, and widths that keep to two launches."""
    if n == 1:
        g = synth.small_random_graph(6, 2.0, "gcn", seed=90)
    else:
        g = synth.gcn_operator(n, *synth.chung_lu_edges(n, 12 * n, 2.1, 91))
    host, _ = both_partitions(g, synth.random_partition(g.n, 3, seed=92), 3)
    net = PartitionedNetwork(host, widths, "gcn", KEY, dtype=dtype)
    net.set_inputs(synth.features(g.n, widths[0], synth.SEED_FEAT))
    net.set_weights([synth.glorot(widths[l], widths[l + 1], synth.SEED_WEIGHT, 2 * l) for l in range(2)])
    for step in (3, 4):
        net.forward(step, ratio)
        for l in range(2):
            z, m = torch.full_like(net.z[l], 7.0), torch.full_like(net.m[l], 7.0)
            net.ctx.network_compress(l, net.x[l], z)
            net.ctx.network_aggregate_fwd(l, net.x[l], z, m)
            torch.cuda.synchronize()
            sent = net.b_total * net.ctx.keep(l)
            assert torch.equal(net.z[l][:sent], z[:sent]) and torch.equal(net.m[l], m), (l, step)


@pytest.mark.parametrize("conv,widths", [("gcn", (20, 96, 130, 72, 9)), ("sage", (24, 96, 8)), ("sage", (20, 96, 130, 72, 9)), ("gcn", (21, 256, 66, 5))])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_weight_copies_made_with_the_first_sums(conv, widths, dtype):
    """At most eight copies, for products and input gradients, made by the first aggregation's launch; more than eight, an input width that
    is no multiple of 4 and a lossless first layer, where they have a launch of their own."""
    g = synth.small_random_graph(700, 7.0, conv, seed=95)
    _compare_network(g, synth.random_partition(g.n, 3, seed=96), 3, conv, widths, [(4, 1), (3, 1), (1, 1)], steps=[0, 1, 2],
                     tol=BF16_TOL if dtype == "bf16" else 1e-4, dtype=dtype)


@pytest.mark.parametrize("widths,together", [((16, 32, 8), True), ((75, 130, 9), False)])
def test_bytes_of_a_launch_that_writes_the_messages_too(widths, together):
    """What the per-kernel profile counts: one launch per layer with the bytes of the sums and of the messages, or two launches."""
    g = synth.small_random_graph(700, 7.0, "gcn", seed=97)
    host, _ = both_partitions(g, synth.random_partition(g.n, 3, seed=98), 3)
    net = PartitionedNetwork(host, widths, "gcn", KEY)
    net.set_inputs(synth.features(g.n, widths[0], synth.SEED_FEAT))
    net.set_weights([synth.glorot(widths[l], widths[l + 1], synth.SEED_WEIGHT, 2 * l) for l in range(2)])
    net.forward(0, (4, 1))
    net.ctx.profile_enable(True)
    net.ctx.profile_read()
    net.ctx.network_forward(net._network_buffers())            # in the same step: the copies of the weights are there
    p = net.ctx.profile_read()
    net.forward(1)                                             # the first layer's launch makes them
    first = net.ctx.profile_read()
    nnz, n_halo = sum(h.nnz for h in host), sum(h.n_halo for h in host)
    moved = sum(8 * nnz + 4 * (g.n + 1) + 4 * (2 * g.n * widths[l] + (net.b_total if together else n_halo) * net.ctx.keep(l)) for l in range(2))
    assert p["agg_fwd"]["launches"] == 2 and p["compress"]["launches"] == (0 if together else 2)
    assert abs(p["agg_fwd"]["bytes"] - moved) <= 1e-9 * moved
    weights = 4 * sum(widths[l] * widths[l + 1] for l in range(2))
    assert first["agg_fwd"]["bytes"] >= moved + weights if together else first["agg_fwd"]["bytes"] == p["agg_fwd"]["bytes"]
