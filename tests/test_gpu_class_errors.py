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
    """dX of the class layer on the device; the same in fp64, aggregated part and whole; what bounds its error, sums of |S| |dZ| |H|
    alike (0 where nothing reaches an element). dz: the errors, or what makes them from the nodes' partitions; nodes whose errors are
    not finite count as zeros in the fp64 values, and the elements they reach are returned as well. Last: the nodes' entries."""
    g = hub_graph(n, 2, 300, 5.0, conv, seed=seed)
    part = synth.random_partition(g.n, 3, seed=seed + 1)
    dz = dz(part) if callable(dz) else dz
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
    finite = np.isfinite(dz).all(1)
    dz = np.where(finite[:, None], dz, 0.0)

    def dx(kind, absolute=False):
        a = lambda x: (np.abs(x) if absolute else x).astype(kind)
        dm = a(dz) @ a(h1).T
        aggregated = a(s_intra).T @ dm + mask.astype(kind) * (a(s_cross).T @ dm)
        return aggregated, aggregated + (a(dz) @ a(h0).T if conv == "sage" else kind(0))
    lost = (~finite).astype(np.float64)[:, None]
    reached = (np.abs(s_intra).T @ lost) + mask * (np.abs(s_cross).T @ lost) + (lost if conv == "sage" else 0.0) > 0
    return got, dx(np.float64), dx(np.float64, True), reached, ((s_intra + s_cross) != 0).sum(0)[:, None], dx(np.float32)[1]


def _bf16_bound(conv, agg, ref, absolute):
    """Every store of dX rounds to 8 bits, to within 2^-8 (SAGE stores the aggregated part first); sums of errors keep 16 bits (2^-16) and
    are added in fp32: up to 300 entries a sum over 64 lanes, at most 64 products."""
    return 2.0 ** -8 * (np.abs(ref) + (np.abs(agg) if conv == "sage" else 0.0)) * (1 + 2.0 ** -7) + (2.0 ** -16 + 80 * 2.0 ** -24) * absolute


@pytest.mark.parametrize("conv,fi,fo,ratio", [("gcn", 64, 1, (8, 1)), ("gcn", 256, 3, (8, 1)), ("sage", 128, 16, (8, 1)), ("gcn", 512, 47, (5, 1)),
                                              ("sage", 272, 33, (1, 1)), ("gcn", 208, 64, (8, 1))])
def test_bf16_errors_of_one_sign(conv, fi, fo, ratio):
    """Errors that agree in sign from node to node: what rounds the sums of errors does not average out."""
    rng = np.random.default_rng(fi + fo)
    bf = lambda a: round_bf16(a).astype(np.float32)
    dz = bf(np.abs(rng.standard_normal((500, fo))) * np.where(rng.random(fo) < 0.5, -1.0, 1.0))
    h1, h0 = bf(rng.standard_normal((fi, fo))), bf(rng.standard_normal((fi, fo)))
    got, (agg, ref), (_, absolute), *_ = _class_layer(conv, fi, fo, ratio, "bf16", dz, h1, h0)
    bound = _bf16_bound(conv, agg, ref, absolute)
    assert (np.abs(got - ref) <= bound).all(), float((np.abs(got - ref) / bound.clip(1e-300)).max())


def _fp32_bound(fo, entries, absolute):
    """Both terms of either operand within 2^-23 of the value; three products of ceil(fo / 16) steps that each round the sum so far
    (the matrix unit cuts: 2^-23), the two sums of terms and the result; the fp32 sums of errors, four entries at a time and 16 lanes."""
    return (2.0 ** -22 + (3 * -(-fo // 16) + 2) * 2.0 ** -23 + (entries / 4 + 8) * 2.0 ** -24) * absolute


_SHAPES = [("gcn", 64, 1, (8, 1)), ("sage", 128, 3, (8, 1)), ("gcn", 96, 16, (8, 1)), ("sage", 256, 17, (8, 1)), ("sage", 132, 47, (8, 1)),
           ("gcn", 256, 47, (8, 1)), ("gcn", 300, 64, (8, 1)), ("sage", 516, 64, (3, 1))]


@pytest.mark.parametrize("conv,fi,fo,ratio", _SHAPES)
@pytest.mark.parametrize("spread", ["none", "rows", "sources", "taps", "positions", "all"])
def test_fp32_sources_and_weights_of_any_magnitude(conv, fi, fo, ratio, spread):
    """rows: errors of every node at a size of its own, some zero. sources: those of one partition far larger than the others', which
    leaves rows whose received errors exceed their own 2^35 times (all: 2^75) at the positions they do not reach. taps: self weights far smaller or
    larger than the others. positions: weights of every input feature at a size of its own."""
    rng = np.random.default_rng(fi + fo)

    def errors(part):
        dz = rng.standard_normal((500, fo))
        if spread in ("rows", "all"):
            dz *= np.exp2(rng.integers(-30, 10, size=(500, 1)))
            dz[::9] = 0.0
        if spread in ("sources", "all"):
            dz *= np.exp2(np.where(part == 1, 35.0, 0.0))[:, None]
        return dz.astype(np.float32)

    h1, h0 = rng.standard_normal((fi, fo)), rng.standard_normal((fi, fo))
    if spread in ("taps", "all"):
        h0 *= np.exp2(np.where(np.arange(fi) % 3 == 0, 30.0, np.where(np.arange(fi) % 3 == 1, -30.0, -4.0)))[:, None]
    if spread in ("positions", "all"):
        sizes = np.exp2(rng.integers(-20, 20, size=(fi, 1)))
        h1, h0 = h1 * sizes, h0 * sizes
    h1, h0 = h1.astype(np.float32), h0.astype(np.float32)
    got, (_, ref), (_, absolute), _, entries, plain = _class_layer(conv, fi, fo, ratio, "f32", errors, h1, h0)
    bound = _fp32_bound(fo, entries, absolute)
    assert (np.abs(got - ref) <= bound).all(), float((np.abs(got - ref) / bound.clip(1e-300)).max())
    if spread == "none":                                  # as a whole as accurate as products and sums in fp32
        assert np.linalg.norm(got - ref) <= 1.25 * np.linalg.norm(plain - ref)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("conv,fi,fo,ratio", _SHAPES)
def test_infinite_errors_stay_where_they_are_received(conv, fi, fo, ratio, dtype):
    """An infinite error of one node: its consumers' elements are lost, all others keep their accuracy, the positions of the same row that
    a message did not carry among them."""
    rng = np.random.default_rng(fi + fo)
    fi = min(fi // 16 * 16, 512) if dtype == "bf16" else fi      # (what bf16 storage sums at the width of the outputs)
    stored = (lambda a: round_bf16(a).astype(np.float32)) if dtype == "bf16" else (lambda a: a.astype(np.float32))
    dz, h1, h0 = [stored(rng.standard_normal(shape)) for shape in ((500, fo), (fi, fo), (fi, fo))]
    dz[123, fo // 2] = np.inf
    got, (agg, ref), (_, absolute), reached, entries, _ = _class_layer(conv, fi, fo, ratio, dtype, dz, h1, h0)
    assert reached.any() and not reached.all() and not np.isfinite(got[reached]).any()
    bound = _fp32_bound(fo, entries, absolute) if dtype == "f32" else _bf16_bound(conv, agg, ref, absolute)
    assert (np.abs(got - ref) <= bound)[~reached].all()
