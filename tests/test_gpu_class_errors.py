"""Input gradient of a class layer that aggregated first, formed from errors summed at the width of the outputs: element by element
against fp64 of the same inputs, with data on which rounding shows (errors of one sign, sources and weights of very different size)."""
import numpy as np
import pytest
import torch

from dense_reference import dense_operator, split_operator
from gpu_common import KEY, hub_graph
from oracle import mask as omask
from oracle.rounding import round_bf16
from paper_2406_17611_amd import binding as vb
from paper_2406_17611_amd import synth
from paper_2406_17611_amd.runner import PartitionedNetwork

pytestmark = pytest.mark.gpu


def _class_layer(conv, fi, fo, ratio, dtype, dz, h1, h0, seed=7, n=500):
    """dX of the class layer on the device, the same in fp64, and what bounds its error: sums of |S| |dZ| |H| (all that reaches an
    element, and its aggregated part), 0 where nothing does. dz(part, rng) and the weights are made by the caller."""
    g = hub_graph(n, 2, 300, 5.0, conv, seed=seed)
    part = synth.random_partition(g.n, 3, seed=seed + 1)
    host = vb.partition_build(g.n, g.rowptr, g.colidx, g.vals, part, 3)
    net = PartitionedNetwork(host, (8, fi, fo), conv, KEY, dtype=dtype)
    net.set_inputs(synth.features(g.n, 8, 3))
    first = synth.glorot(8, fi, 3, 0)
    net.set_weights([first, h1], [first, h0] if conv == "sage" else None)
    net.set_upstream(dz)
    net.zero_grads()
    net.forward(2, ratio)
    net.ctx.profile_enable(True)
    net.ctx.profile_read()
    net.backward()
    torch.cuda.synchronize()
    launches = {name: p["launches"] for name, p in net.ctx.profile_read().items()}
    # sums at the width of the outputs: no products handed back, one product for dX (bf16 storage adds the self tap by another)
    assert launches["agg_bwd_halo"] == 0 and launches["gemm_dgrad"] == (2 if conv == "sage" and dtype == "bf16" else 1), launches
    got = net.to_global(net.dx[1]).astype(np.float64)
    net.ctx.close()

    s_intra, s_cross = split_operator(dense_operator(g), part)
    keep = omask.keep_count(fi, *ratio)
    mask = omask.keep_mask(np.arange(g.n), fi, keep, KEY, 2, 1)
    def dx(absolute):
        a = np.abs if absolute else (lambda x: x)
        dm = a(dz.astype(np.float64)) @ a(h1.astype(np.float64)).T
        aggregated = a(s_intra).T @ dm + mask * (a(s_cross).T @ dm)
        return aggregated, aggregated + (a(dz.astype(np.float64)) @ a(h0.astype(np.float64)).T if conv == "sage" else 0.0)
    return got, dx(False), dx(True)


@pytest.mark.parametrize("conv,fi,fo,ratio", [("gcn", 64, 1, (8, 1)), ("gcn", 256, 3, (8, 1)), ("sage", 128, 16, (8, 1)), ("gcn", 512, 47, (5, 1)),
                                              ("sage", 272, 33, (1, 1)), ("gcn", 208, 64, (8, 1))])
def test_bf16_errors_of_one_sign(conv, fi, fo, ratio):
    """Errors that agree in sign from node to node: what rounds the sums of errors does not average out."""
    rng = np.random.default_rng(fi + fo)
    bf = lambda a: round_bf16(a).astype(np.float32)
    dz = bf(np.abs(rng.standard_normal((500, fo))) * np.where(rng.random(fo) < 0.5, -1.0, 1.0))
    h1, h0 = bf(rng.standard_normal((fi, fo))), bf(rng.standard_normal((fi, fo)))
    got, (agg, ref), (_, absolute) = _class_layer(conv, fi, fo, ratio, "bf16", dz, h1, h0)
    # every store of dX rounds to 8 bits, to within 2^-8 (SAGE stores the aggregated part first); sums of errors keep 16 bits
    # (2^-16) and are added in fp32: up to 300 entries a sum over 64 lanes, at most 64 products
    bound = 2.0 ** -8 * (np.abs(ref) + (np.abs(agg) if conv == "sage" else 0.0)) * (1 + 2.0 ** -7) + (2.0 ** -16 + 80 * 2.0 ** -24) * absolute
    assert (np.abs(got - ref) <= bound).all(), float((np.abs(got - ref) / bound.clip(1e-300)).max())
