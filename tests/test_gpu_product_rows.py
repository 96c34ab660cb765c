"""Rows of the product buffer on both sides of the sizes that they are rounded up to (16 bytes, 32, 64 and more), and rows on both sides of the length below
which they are gathered whole instead, with few neighbours and with many."""
import pytest
import torch

from gpu_common import hub_graph, products_taken
from paper_2406_17611_amd import binding as vb
from paper_2406_17611_amd import synth
from test_gpu_graph import _network, _snapshot
from test_gpu_network import BF16_TOL, _compare_network

pytestmark = pytest.mark.gpu


def _check(dtype, width, kept, degree, products=None):
    g = hub_graph(500, 2, 200, degree, "gcn", seed=width + kept)
    part = synth.random_partition(g.n, 4, seed=92)
    net = _compare_network(g, part, 4, "gcn", (12, width, 72, 6), [(width, kept)] * 2, steps=[0, 1], tol=BF16_TOL if dtype == "bf16" else 1e-4, dtype=dtype)
    taken = products_taken(net.ctx, lambda: net.step(2, (width, kept)))
    assert taken is products or products is None


@pytest.mark.parametrize("dtype,width,kept", [("f32", 132, 4), ("f32", 136, 5), ("f32", 148, 8), ("f32", 150, 9), ("f32", 160, 16), ("f32", 200, 17), ("f32", 256, 33),
                                              ("f32", 299, 20), ("f32", 300, 67), ("f32", 516, 21), ("f32", 1028, 33), ("bf16", 392, 8), ("bf16", 392, 9), ("bf16", 400, 16), ("bf16", 404, 17), ("bf16", 512, 32), ("bf16", 512, 33), ("bf16", 516, 20), ("bf16", 520, 20),
                                              ("bf16", 1028, 40), ("bf16", 1032, 40), ("bf16", 163, 9), ("bf16", 251, 20)])
def test_products_of_any_length(dtype, width, kept):
    _check(dtype, width, kept, 6.0, True)


@pytest.mark.parametrize("dtype,width", [("f32", 40), ("f32", 96), ("f32", 100), ("f32", 128), ("bf16", 56), ("bf16", 320), ("bf16", 328), ("bf16", 384)])
@pytest.mark.parametrize("degree", [6.0, 30.0])
def test_rows_gathered_or_not(dtype, width, degree):
    for kept in (1, 9):
        _check(dtype, width, kept, degree)


@pytest.mark.parametrize("dtype,width,kept,degree,products",
                         [("f32", 127, 7, 6.0, False), ("f32", 128, 7, 6.0, False), ("f32", 129, 7, 6.0, True), ("f32", 132, 7, 6.0, True), ("f32", 79, 7, 30.0, False),
                          ("f32", 80, 7, 30.0, False), ("f32", 81, 7, 30.0, True), ("f32", 96, 7, 30.0, False), ("f32", 100, 7, 30.0, True), ("bf16", 159, 7, 6.0, False),
                          ("bf16", 161, 7, 6.0, True), ("bf16", 384, 7, 6.0, False), ("bf16", 388, 7, 6.0, True), ("bf16", 159, 7, 30.0, False), ("bf16", 161, 7, 30.0, True),
                          ("bf16", 256, 7, 30.0, False), ("bf16", 260, 7, 30.0, True), ("bf16", 264, 64, 30.0, True), ("bf16", 264, 65, 30.0, False),
                          ("bf16", 320, 65, 30.0, False), ("bf16", 324, 65, 30.0, True)])
def test_lines_of_the_form(dtype, width, kept, degree, products):
    """Rows of odd lengths are gathered an element to a lane, so products are formed from shorter ones on; long products pay from longer rows on."""
    _check(dtype, width, kept, degree, products)


@pytest.mark.parametrize("width,products", [(224, False), (228, True), (232, True)])
def test_line_of_many_rows(monkeypatch, width, products):
    """bf16 rows that take more than 128 MiB together, at most 512 bytes each: products from 448 bytes on, the errors of which are those that partition after partition
    gives."""
    n, ratio = 310_007, (width, 7)
    g = synth.gcn_operator(n, *synth.chung_lu_edges(n, 4_000_000, 2.5, 5))
    part = synth.random_partition(n, 4, seed=6)
    nets = []
    for linked in (True, False):
        with monkeypatch.context() as m:
            if not linked:
                m.setattr(vb.Context, "link_partitions", lambda ctx: False)
            nets.append(_network(g, part, 4, (8, width, 72, 4), "gcn", 1, dtype="bf16"))
    for net in nets:
        net.forward(5, ratio)
    torch.cuda.synchronize()
    for l in range(1, 4):
        nets[1].x[l].copy_(nets[0].x[l])
    assert products_taken(nets[0].ctx, nets[0].backward) is products
    nets[1].backward()
    torch.cuda.synchronize()
    a, b = (net.dx[1].double() for net in nets)
    assert float((a - b).norm()) <= 2.0 ** -5 * float(a.norm())         # (as test_linked_and_partition_after_partition_agree)
    for net in nets:
        net.ctx.close()


def test_rows_of_less_than_64_bytes_where_the_device_is_full():
    """Rows of 36 bytes take 64 bytes each, 4 million of them 244 MiB; on a device that has no room for that, 48 bytes and 183 MiB. The sums are the same."""
    n, ratio = 60_000, (256, 9)
    g = synth.gcn_operator(n, *synth.chung_lu_edges(n, 3_000_000, 2.5, 5))
    part = synth.random_partition(n, 3, seed=6)
    got = []
    for room in (None, 212 << 20):
        net = _network(g, part, 3, (8, 256, 72, 4), "gcn", 1)
        entries = net.nnz_total - sum(int(hp.t_rowptr[hp.n_local]) for hp in net.host_parts)
        assert 64 * entries > 240 << 20 and 48 * entries < 184 << 20
        net.step(4, (1, 1))
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        filler = []
        try:
            while room and (left := torch.cuda.mem_get_info()[0] - room) >= 8 << 20:
                while left >= 8 << 20:                       # what cannot be had in one piece is taken in smaller ones
                    try:
                        filler.append(torch.empty(left, dtype=torch.uint8, device="cuda"))
                        break
                    except torch.OutOfMemoryError:
                        left //= 2
                else:
                    break
            assert products_taken(net.ctx, lambda: (net.zero_grads(), net.step(5, ratio)))
            got.append(_snapshot(net))
        finally:
            filler.clear()
            torch.cuda.empty_cache()
        net.ctx.close()
        del net
    for a, b in zip(*got):
        assert (a == b).all()
