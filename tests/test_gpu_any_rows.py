"""Forward aggregation of rows whose length is no multiple of 4: two or four elements to a load from any address of an element, the end of a row by loads
that overlap the ones before. Hubs (rows in several runs, partial sums of odd length), compressed, whole and no messages."""
import pytest

from gpu_common import hub_graph
from paper_2406_17611_amd import synth
from test_gpu_network import BF16_TOL, _compare_network

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("width", [63, 65, 66, 67, 127, 129, 131, 254, 255, 257, 330, 511])
def test_rows_of_any_length(width, dtype):
    g = hub_graph(420, 3, 300, 5.0, "sage" if width % 2 else "gcn", seed=width)
    part = synth.random_partition(g.n, 3, seed=92)
    conv = "sage" if width % 2 else "gcn"
    _compare_network(g, part, 3, conv, (width, 6), [(3, 1), (1, 1), (1, 0)], steps=[0, 1, 2], tol=BF16_TOL if dtype == "bf16" else 1e-4, dtype=dtype)
