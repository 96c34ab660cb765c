"""Rows of the product buffer on both sides of the sizes that they are rounded up to (16 bytes, 32, 64 and more), and rows on both sides of the length below
which they are gathered whole instead, with few neighbours and with many."""
import pytest

from gpu_common import hub_graph
from paper_2406_17611_amd import synth
from test_gpu_network import BF16_TOL, _compare_network

pytestmark = pytest.mark.gpu


def _check(dtype, width, kept, degree):
    g = hub_graph(500, 2, 200, degree, "gcn", seed=width + kept)
    part = synth.random_partition(g.n, 4, seed=92)
    _compare_network(g, part, 4, "gcn", (12, width, 72, 6), [(width, kept)] * 2, steps=[0, 1], tol=BF16_TOL if dtype == "bf16" else 1e-4, dtype=dtype)


@pytest.mark.parametrize("dtype,width,kept", [("f32", 132, 4), ("f32", 136, 5), ("f32", 148, 8), ("f32", 150, 9), ("f32", 160, 16), ("f32", 200, 17), ("f32", 256, 33),
                                              ("f32", 300, 67), ("bf16", 392, 8), ("bf16", 392, 9), ("bf16", 400, 16), ("bf16", 404, 17), ("bf16", 512, 32), ("bf16", 512, 33)])
def test_products_of_any_length(dtype, width, kept):
    _check(dtype, width, kept, 6.0)


@pytest.mark.parametrize("dtype,width", [("f32", 40), ("f32", 96), ("f32", 100), ("f32", 128), ("bf16", 56), ("bf16", 320), ("bf16", 328), ("bf16", 384)])
@pytest.mark.parametrize("degree", [6.0, 30.0])
def test_rows_gathered_or_not(dtype, width, degree):
    for kept in (1, 9):
        _check(dtype, width, kept, degree)
