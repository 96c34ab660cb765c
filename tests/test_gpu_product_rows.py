"""Rows of the product buffer on both sides of the sizes that they are rounded up to: 16 bytes, 32, 64 and more."""
import pytest

from gpu_common import hub_graph
from paper_2406_17611_amd import synth
from test_gpu_network import BF16_TOL, _compare_network

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,width,kept", [("f32", 60, 4), ("f32", 60, 5), ("f32", 60, 8), ("f32", 60, 9), ("f32", 60, 16), ("f32", 60, 17), ("f32", 100, 33),
                                              ("bf16", 104, 8), ("bf16", 104, 9), ("bf16", 104, 16), ("bf16", 104, 17), ("bf16", 104, 32), ("bf16", 104, 33)])
def test_products_of_any_length(dtype, width, kept):
    g = hub_graph(500, 2, 200, 6.0, "gcn", seed=width + kept)
    part = synth.random_partition(g.n, 4, seed=92)
    _compare_network(g, part, 4, "gcn", (12, width, 72, 6), [(width, kept)] * 2, steps=[0, 1], tol=BF16_TOL if dtype == "bf16" else 1e-4, dtype=dtype)
