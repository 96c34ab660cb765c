"""The transform in fp32 matrix instructions with the weights in registers (rows whose length is no multiple of 4): blocks of 32 rows, units of 32 columns
on two or four wavefronts, pieces of 64 steps, tiles of 16, halves of a tile."""
import numpy as np
import pytest
import torch

from gpu_common import KEY, dev
from paper_2406_17611_amd import binding as vb
from paper_2406_17611_amd import synth
from paper_2406_17611_amd.runner import PartitionedNetwork

pytestmark = pytest.mark.gpu


def _bound(taps, fi, size):
    # every step of a tap is multiplied and added with a rounding of 2^-24 on a partial sum that is at most `size`: sqrt of their number for
    # independent ones, four times that for the tail; an addition to what was there rounds once more
    return 4 * 2.0 ** -24 * np.sqrt(taps * fi + 1) * size


@pytest.mark.parametrize("fi,fo", [(5, 1), (17, 33), (31, 64), (63, 65), (65, 96), (71, 160), (81, 129), (127, 256), (129, 288), (150, 32), (191, 40), (193, 200), (250, 130), (255, 512), (257, 70)])
@pytest.mark.parametrize("n", [1, 31, 33, 3001, 32801])
def test_one_tap(n, fi, fo):
    """Added to what is there, from any word of a larger tensor on; nothing behind the last row is read into it or written."""
    rng = np.random.default_rng(n + fi + fo)
    y = rng.standard_normal((n, fi)).astype(np.float32)
    h = synth.glorot(fi, fo, 3, 1).astype(np.float32)
    old = rng.standard_normal((n + 1, fo)).astype(np.float32)
    held = torch.full((n * fi + 2,), float("nan"), device="cuda")
    held[1:-1] = dev(y).flatten()
    out = dev(old)
    ctx = vb.Context([fi, fo], [vb.ACT_RELU], vb.CONV_GCN, 1, KEY)
    ctx.prepare()
    ctx.transform_fwd(0, held[1:-1].view(n, fi), dev(h), out[:n], True, True)
    torch.cuda.synchronize()
    want = y.astype(np.float64) @ h.astype(np.float64) + old[:n]
    size = np.abs(y) @ np.abs(h) + np.abs(old[:n])
    got = out.cpu().numpy()
    assert (np.abs(got[:n] - np.maximum(want, 0.0)) <= _bound(1, fi, size)).all()
    assert np.array_equal(got[n], old[n])
    ctx.close()


@pytest.mark.parametrize("fi,fo", [(6, 40), (33, 96), (63, 70), (65, 256), (127, 160), (130, 48), (159, 130), (193, 288), (255, 257)])
@pytest.mark.parametrize("n", [2, 33, 3001, 32801])
def test_two_taps(n, fi, fo):
    """A layer's two products in one chain. A row that is not finite leaves the others as they are."""
    graph = synth.small_random_graph(n, 2.0, "sage", seed=n)
    host = vb.partition_build(graph.n, graph.rowptr, graph.colidx, graph.vals, synth.random_partition(graph.n, 2, seed=5), 2)
    rng = np.random.default_rng(n + fi + fo)
    net = PartitionedNetwork(host, (fi, fo, 4), "sage", 17, need_backward=False)
    whole = torch.full((n + 1, fo), 7.0, device="cuda")
    net.x[1] = whole[:n]
    h = [[synth.glorot(a, b, 3, 1 + t).astype(np.float32) for a, b in ((fi, fo), (fo, 4))] for t in range(2)]
    net.set_weights(*h)
    x0 = rng.standard_normal((n, fi)).astype(np.float32)
    for bad in (False, True):
        if bad:
            x0[n // 2, 0] = np.inf
        net.set_inputs(x0)
        net.forward(1, (1, 0))                      # (no exchange, and half of the neighbours elsewhere)
        torch.cuda.synchronize()
        taps = [(net.m[0].cpu().numpy().astype(np.float64), h[0][0]), (net.x[0].cpu().numpy().astype(np.float64), h[1][0])]
        finite = np.isfinite(taps[0][0]).all(1) & np.isfinite(taps[1][0]).all(1)
        assert not bad or finite.sum() < n
        taps = [(a[finite], b) for a, b in taps]
        want = sum(a @ b.astype(np.float64) for a, b in taps)
        size = sum(np.abs(a) @ np.abs(b) for a, b in taps)
        got = whole.cpu().numpy()
        assert (np.abs(got[:n][finite] - np.maximum(want, 0.0)) <= _bound(2, fi, size)).all()
        assert (got[n] == 7.0).all()
    net.ctx.close()


def _bits(t):
    return t.view(torch.int32)


@pytest.mark.parametrize("fi,fo,n", [(17, 64, 991_003), (45, 47, 1_450_007), (16, 64, 991_003), (20, 30, 1_450_007)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_bits_do_not_depend_on_the_number_of_rows(fi, fo, n, accumulate):
    """So many rows that tiles of 256 x 64 take them (results or operands beyond the last cache), and ranges of them that wavefronts with the weights in
    registers take, which start at any row: the same bits, added to what is there and through the ReLU as well."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(fi)
    y, h = (torch.randn(*shape, generator=gen, device="cuda") for shape in ((n, fi), (fi, fo)))
    old = torch.randn(n, fo, generator=gen, device="cuda")
    ctx = vb.Context([fi, fo], [vb.ACT_RELU], vb.CONV_GCN, 1, KEY)
    ctx.set_matmul_terms(3 if fi % 4 else 0)
    ctx.prepare()
    whole = old.clone()
    ctx.transform_fwd(0, y, h, whole, accumulate, True)
    for first, rows in ((0, 3001), (1, 33), (n - 40_007, 40_007)):
        part = old[first:first + rows].clone()
        ctx.transform_fwd(0, y[first:first + rows], h, part, accumulate, True)
        assert torch.equal(_bits(part), _bits(whole[first:first + rows])), first
    ctx.close()


@pytest.mark.parametrize("fi,fo,terms", [(150, 384, 3), (161, 500, 3), (200, 384, 0)])
def test_bits_of_two_taps_do_not_depend_on_the_columns(fi, fo, terms):
    """A layer's two products of more than 256 columns and 100,000 rows, which tiles of 128 x 128 take, and the same columns by the wavefronts that keep
    the weights, in units with and without a remainder."""
    n = 100_013
    graph = synth.small_random_graph(n, 2.0, "sage", seed=n)
    host = vb.partition_build(graph.n, graph.rowptr, graph.colidx, graph.vals, synth.random_partition(graph.n, 2, seed=5), 2)
    h1, h0 = (synth.glorot(fi, fo, 7, 1 + t).astype(np.float32) for t in range(2))
    x0 = np.random.default_rng(fi).standard_normal((n, fi)).astype(np.float32)

    def outputs(c0, c1):
        net = PartitionedNetwork(host, (fi, c1 - c0, 4), "sage", 17, need_backward=False)      # (two layers: the first has a ReLU)
        net.ctx.set_matmul_terms(terms)
        net.set_inputs(x0)
        narrow = np.zeros((c1 - c0, 4), dtype=np.float32)
        net.set_weights([np.ascontiguousarray(h1[:, c0:c1]), narrow], [np.ascontiguousarray(h0[:, c0:c1]), narrow])
        net.forward(1, (1, 0))
        torch.cuda.synchronize()
        out = net.x[1].clone()
        net.ctx.close()
        return out

    whole = outputs(0, fo)
    for c0, c1 in ((0, 256), (200, 247), (256, fo)):
        assert torch.equal(_bits(whole[:, c0:c1]), _bits(outputs(c0, c1))), c0
