"""Accuracy of weight gradients formed over all partitions at once: sums over many rows are cut so that no fp32 accumulator
takes longer chains than the rule for its kind of product allows, and partial sums are added in fp64."""
import numpy as np
import pytest
import torch

from gpu_common import KEY
from paper_2406_17611_amd import binding as vb
from paper_2406_17611_amd import synth
from paper_2406_17611_amd.runner import PartitionedNetwork

pytestmark = pytest.mark.gpu


def _linked_context(n, n_parts, fi, fo, dtype, terms):
    """Partitions without edges: the dense products over the arena are all that is used."""
    none = np.zeros(0, dtype=np.int64)
    g = synth.gcn_operator(n, none, none)
    part = np.sort(np.arange(n) % n_parts).astype(np.int32)
    host = vb.partition_build(g.n, g.rowptr, g.colidx, g.vals, part, n_parts)
    ctx = vb.Context([fi, fo], [vb.ACT_RELU], vb.CONV_SAGE, n_parts, KEY, dtype)
    if dtype == vb.F32:
        ctx.set_matmul_terms(terms)
    held = [ctx.register_partition(q, hp) for q, hp in enumerate(host)]
    assert ctx.link_partitions()
    ctx.prepare()
    return ctx, held


# rows a slab may hold for these sizes, and roundings per row. With two fp16 terms the large sum takes one per 16 rows; operands are
# within 2^-23, 7.5e-8 in the root mean square of a product; and the matrix unit cuts instead of rounding, an error of one sign
# that slabs of alternating sign do not cancel altogether: a quarter. fp32 instructions round once per 2 rows, bf16 once per 8.
@pytest.mark.parametrize("dtype,terms,fi,fo,slab_rows,roundings,operands,margin",
                         [(vb.F32, 3, 256, 256, 330 * (137_500 + 169_343) / 73_300, 1 / 16, 7.5e-8, 1.25), (vb.F32, 0, 256, 256, 220, 1 / 2, 0.0, 1.0),
                          (vb.BF16, 1, 512, 512, 661 + 4 * 64 + 16 * 4, 1 / 8, 0.0, 1.0)])
def test_long_reductions_keep_the_accuracy_of_short_ones(dtype, terms, fi, fo, slab_rows, roundings, operands, margin):
    n, n_parts = 169_343, 4
    ctx, held = _linked_context(n, n_parts, fi, fo, dtype, terms)
    tdt = torch.bfloat16 if dtype == vb.BF16 else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    randn = lambda *s: torch.randn(*s, generator=gen, device="cuda")     # noqa: E731
    y = [randn(n, fi).to(tdt) for _ in range(2)]
    d = (randn(n, fo) / n).to(tdt)
    x = randn(n, fo).clamp_min(0).to(tdt)
    dh = [torch.zeros(fi, fo, device="cuda") for _ in range(2)]
    ctx.network_taps_bwd_weight(0, y, d, x, dh)
    dz = torch.where(x > 0, d, torch.zeros_like(d)).double()
    # a rounding of a sum s is within 2^-24 |s|, 2^-24 / sqrt(3) of it in the root mean square; independent products make s^2 grow
    # linearly along a chain, so that its mean is half of the end's
    bound = margin * np.hypot(2.0 ** -24 / np.sqrt(3) * np.sqrt(slab_rows * roundings / 2), operands)
    for yt, got in zip(y, dh):
        ref = yt.double().t() @ dz
        err = float((got.double() - ref).norm() / ref.norm())
        assert err <= bound, (err, bound)
    ctx.close()
    del held


def test_received_rows_of_many_shares():
    """More boundary rows than one round of workgroups may sum (512 shares of 1,024 rows), a remainder included, against the
    other order of the layer's products."""
    n = 2 * 512 * 1024 + 77                            # every node of a ring dealt to two partitions is a boundary node
    u = np.arange(n - 1, dtype=np.int64)
    g = synth.gcn_operator(n, u, u + 1)
    host = vb.partition_build(g.n, g.rowptr, g.colidx, g.vals, (np.arange(n) % 2).astype(np.int32), 2)
    widths = (16, 32, 5)
    h1 = [synth.glorot(widths[l], widths[l + 1], 11, l) for l in range(2)]
    got = []
    for first in ((1,), ()):
        net = PartitionedNetwork(host, widths, "gcn", KEY, dtype="bf16", transform_first=first)
        net.set_weights(h1)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(3)
        net.x[0].copy_(torch.randn(n, 16, generator=gen, device="cuda"))
        net.dx[2].copy_((torch.randn(n, 5, generator=gen, device="cuda") + 0.5) / n)
        net.step(3, (2, 1))
        torch.cuda.synchronize()
        got.append(net.dh1[1].double().cpu().numpy())
        net.ctx.close()
    # three bf16 roundings of 2^-9 at most lie between the stored activations and a gradient in either order
    assert np.abs(got[0] - got[1]).max() <= 6 * 2.0 ** -9 * np.abs(got[1]).max()
