"""A schedule that raises k step by step: how often the library's product buffer is allocated anew, and steps captured at
earlier ratios, whose buffers must outlive that."""
import numpy as np
import pytest
import torch

from gpu_common import hub_graph, products_taken
from paper_2406_17611_amd import synth
from test_gpu_graph import _network, _snapshot

pytestmark = pytest.mark.gpu


def test_product_buffer_grows_in_few_steps():
    n = 40_000
    g = synth.gcn_operator(n, *synth.chung_lu_edges(n, 600_000, 2.5, 7))
    net = _network(g, synth.random_partition(n, 4, seed=8), 4, (16, 256, 8), "gcn", 1)
    ctx, steps, sizes = net.ctx, 120, []
    for step in range(steps):
        ctx.set_step(step)
        ctx.set_ratio(-1, 16 * steps - 15 * step, steps)           # 16 -> 1, as an exact rational
        sizes.append(torch.cuda.mem_get_info()[0])
    # k from 16 to 85 takes the product form, in rows of 16, 32, ... 96 values; beyond, the calls per partition ask for (halo entries of the largest
    # partition, fewer than half of all) x k, up to 255. Growing by a quarter, that is 1 + log(128 / 16) / log(1.25) = 10 allocations at most
    changes = sum(a != b for a, b in zip(sizes, sizes[1:]))
    assert 1 <= changes <= 1 + int(np.log(128 / 16) / np.log(1.25)), changes


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_graphs_of_a_rising_schedule_keep_replaying(dtype):
    g = hub_graph(5000, 3, 1200, 7.0, "gcn", seed=35)
    part = synth.random_partition(g.n, 4, seed=36)
    widths, first = (64, 400 if dtype == "bf16" else 160, 128, 16), 70           # rows long enough for products
    ratios = [(32, 1), (16, 1), (12, 1), (8, 1), (6, 1), (5, 1), (4, 1), (7, 2), (2, 1), (1, 1)]     # more than a context has streams
    kw = dict(dtype=dtype)
    eager = _network(g, part, 4, widths, "gcn", 1, **kw)
    want = []
    for ratio in ratios:
        eager.zero_grads()
        assert products_taken(eager.ctx, lambda: eager.step(first + 1, ratio)) is (ratio[0] > 3 * ratio[1])
        want.append(_snapshot(eager))
    eager.ctx.close()
    net = _network(g, part, 4, widths, "gcn", 1, **kw)
    graphs = [net.capture_step(ratio) for ratio in ratios]
    filler = [torch.full((1 << 18,), float("nan"), device="cuda") for _ in range(64)]    # takes whatever memory was given back
    for repeat in range(2):
        for i in (list(range(len(ratios))) if repeat == 0 else reversed(range(len(ratios)))):
            net.zero_grads()
            net.ctx.set_step(first)
            torch.cuda.synchronize()
            graphs[i].replay()
            for a, b in zip(_snapshot(net), want[i]):
                assert np.array_equal(a, b), (repeat, ratios[i])
    assert all(bool(torch.isnan(f).all()) for f in filler)
