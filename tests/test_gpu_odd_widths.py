"""Dense products whose rows have any length and alignment: groups of four or eight that cross the end of a row, with 1 to 3
(1 to 7) elements of it inside, alone in the last stage or tile, masked and not, for both taps at once."""
import pytest

from paper_2406_17611_amd import synth
from test_gpu_matmul import test_transform_products as check_products
from test_gpu_network import BF16_TOL, _compare_network

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,fi,fo", [(1000, 75, 200), (129, 131, 129), (517, 201, 77), (33, 33, 67), (40, 5, 6), (300, 98, 130), (4, 4, 257), (131, 3, 2), (70, 2, 131)])
def test_products_of_odd_widths(n, fi, fo):
    check_products(n, fi, fo, 3)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("conv,widths", [("gcn", (75, 130, 66, 5)), ("sage", (97, 129, 47)), ("sage", (22, 67, 258, 9)), ("gcn", (39, 70, 64))])
def test_layers_of_odd_widths(conv, widths, dtype):
    g = synth.small_random_graph(700, 7.0, conv, seed=91)
    part = synth.random_partition(g.n, 3, seed=92)
    _compare_network(g, part, 3, conv, widths, [(4, 1), (2, 1)], steps=[0, 1], tol=BF16_TOL if dtype == "bf16" else 1e-4, dtype=dtype)
