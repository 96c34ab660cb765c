"""Forward aggregation of rows whose length is no multiple of 4: two or four elements to a load from any address of an element, the end of a row by loads
that overlap the ones before. Hubs (rows in several runs, partial sums of odd length), compressed, whole and no messages."""
import pytest
import torch

from gpu_common import KEY, hub_graph
from paper_2406_17611_amd import binding as vb
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


def _aggregate(host, y, kept, dtype, shift_rows=0, shift_messages=0):
    """Sums of all partitions' rows y (whole ones, some elements or none of the others' rows), from buffers that start `shift` elements behind an address of
    16 bytes."""
    n, width = y.shape
    ctx = vb.Context([width, 4], [vb.ACT_IDENTITY], vb.CONV_GCN, len(host), KEY, vb.BF16 if dtype == "bf16" else vb.F32)
    held = [ctx.register_partition(q, hp) for q, hp in enumerate(host)]
    assert ctx.link_partitions()
    ctx.set_ratio(-1, *((width, kept) if kept else (1, 0)))
    ctx.prepare()
    assert ctx.keep(0) == kept

    def buffer(elements, shift):
        return torch.zeros(elements + shift, dtype=y.dtype, device="cuda")[shift:]

    rows, out = buffer(n * width, shift_rows), buffer(n * width, shift_rows)
    z = buffer(sum(hp.n_boundary for hp in host) * kept, shift_messages)
    rows.copy_(y.flatten())
    ctx.begin_step(3)
    ctx.network_compress(0, rows, z)
    ctx.network_aggregate_fwd(0, rows, z, out)
    torch.cuda.synchronize()
    got = out.view(n, width).clone()
    ctx.close()
    del held
    return got


def _same_bits(a, b):
    kind = torch.int16 if a.dtype == torch.bfloat16 else torch.int32
    return torch.equal(a.contiguous().view(kind), b.contiguous().view(kind))


def _rows(width, dtype, seed):
    g = hub_graph(420, 3, 300, 5.0, "gcn", seed=seed)
    host = vb.partition_build(g.n, g.rowptr, g.colidx, g.vals, synth.random_partition(g.n, 3, seed=92), 3)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return host, torch.randn(g.n, width, generator=gen, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)


@pytest.mark.parametrize("width", [1, 2, 3, 5, 7, 9, 13, 17, 25, 33, 47, 63, 126, 127, 129])
def test_narrow_bf16_rows_of_any_length(width):
    """One element to a load beside compressed messages, up to 64 private rows; four beside whole ones."""
    g = hub_graph(420, 3, 300, 5.0, "gcn", seed=width)
    part = synth.random_partition(g.n, 3, seed=92)
    _compare_network(g, part, 3, "gcn", (width, 6), [(3, 1), (8, 1), (1, 0), (1, 1)], steps=[0, 1, 2, 3], tol=BF16_TOL, dtype="bf16")


@pytest.mark.parametrize("width,shift", [(65, 0), (66, 0), (75, 0), (100, 1), (127, 0), (128, 3), (130, 0), (147, 0), (209, 0), (255, 0), (256, 1), (257, 0), (330, 0), (511, 0)])
@pytest.mark.parametrize("whole", [True, False])
def test_bits_do_not_depend_on_the_width(width, shift, whole):
    """fp32 rows by two or four elements to a load: every column has the bits that it has among at most 63, which take one element to a load."""
    host, y = _rows(width, "f32", width)
    got = _aggregate(host, y, width if whole else 0, "f32", shift)
    for c0 in range(0, width, 50):
        c1 = min(c0 + 63, width)
        c0 += (c1 - c0) % 4 == 0              # (rows of aligned length, and of at most 32 elements, are summed in groups of lanes)
        if c1 - c0 > 32:
            assert _same_bits(got[:, c0:c1], _aggregate(host, y[:, c0:c1].contiguous(), c1 - c0 if whole else 0, "f32")), c0


@pytest.mark.parametrize("width,dtype,whole", [(132, "f32", True), (132, "f32", False), (256, "f32", True), (260, "f32", False), (512, "f32", True), (512, "f32", False),
                                               (20, "bf16", True), (100, "bf16", True), (132, "bf16", True), (132, "bf16", False), (260, "bf16", False)])
def test_bits_do_not_depend_on_the_address(width, dtype, whole):
    """(bf16 rows of at most 128 elements beside compressed messages take one element to a load there, in another order.)"""
    host, y = _rows(width, dtype, width)
    aligned, shifted = (_aggregate(host, y, width if whole else 0, dtype, shift, shift) for shift in (0, 1))
    assert _same_bits(aligned, shifted)


@pytest.mark.parametrize("width,kept", [(256, 66), (256, 126), (256, 132), (300, 70), (300, 172), (512, 200), (512, 332)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_bits_do_not_depend_on_the_address_of_messages(width, kept, dtype):
    """Messages of 65 elements and more: two or four to a lane from any address, the end of one by a load that overlaps the one before."""
    host, y = _rows(width, dtype, width + kept)
    aligned, shifted = (_aggregate(host, y, kept, dtype, 0, shift) for shift in (0, 1))
    assert _same_bits(aligned, shifted)
