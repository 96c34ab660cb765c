"""The entry point that allocates nothing, varco_transform_bwd_weight_static, against the entry point it is a
variant of (varco_transform_bwd_weight), through the C ABI: same kernels and the same split of the reduction, the
partial products in the library's static device array instead of a prepared workspace. Two calls in a row, the
second with a smaller input (the array keeps the first call's contents), must both give the existing entry point's
bits; a shape whose partial products exceed the array is refused with the sizes in the error text."""
import numpy as np
import pytest
import torch

from gpu_common import KEY, assert_close, dev
from paper_2406_17611_amd import binding as vb
from paper_2406_17611_amd import synth

pytestmark = pytest.mark.gpu


def _prepared_reference_context(fi, fo, act, dtype, n_rows):
    """A context whose prepared workspace holds the full split for n_rows (sized by a registered partition)."""
    ctx = vb.Context([fi, fo], [act], vb.CONV_GCN, 1, KEY, dtype)
    g = synth.small_random_graph(n_rows, 3.0, "gcn", seed=5)
    host = vb.partition_build(g.n, g.rowptr, g.colidx, g.vals, np.zeros(g.n, dtype=np.int32), 1)
    ctx.register_partition(0, host[0])
    ctx.prepare()
    return ctx


@pytest.mark.parametrize("dtype,fi,fo,sizes", [("f32", 256, 256, (40000, 3001)), ("f32", 100, 47, (20000, 777)),
                                               ("bf16", 512, 512, (8192, 1000)), ("bf16", 100, 512, (30000, 129))])
def test_static_scratch_variant_gives_the_existing_entry_points_bits(dtype, fi, fo, sizes):
    bf16 = dtype == "bf16"
    tdt = torch.bfloat16 if bf16 else torch.float32
    rng = np.random.default_rng(fi + fo)
    ref_ctx = _prepared_reference_context(fi, fo, vb.ACT_RELU, vb.BF16 if bf16 else vb.F32, max(sizes))
    ctx = vb.Context([fi, fo], [vb.ACT_RELU], vb.CONV_GCN, 1, KEY, vb.BF16 if bf16 else vb.F32)   # never prepared
    for n in sizes:                                   # the second call is smaller and sees the first one's leftovers
        y = dev(rng.standard_normal((n, fi)).astype(np.float32), tdt)
        dxo = dev((rng.standard_normal((n, fo)) / n).astype(np.float32), tdt)
        xo = dev(np.maximum(rng.standard_normal((n, fo)), 0.0).astype(np.float32), tdt)
        start = rng.standard_normal((fi, fo)).astype(np.float32)
        want, got = dev(start), dev(start)
        ref_ctx.transform_bwd_weight(0, y, dxo, xo, want)
        ctx.transform_bwd_weight_static(0, y, dxo, xo, got)
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), want.cpu().numpy()), f"{n} rows"
        # and both are the weight gradient: dH += Y^T (dX * [X > 0]) in fp64 on the stored values
        dz = dxo.float().cpu().numpy().astype(np.float64) * (xo.float().cpu().numpy() > 0)
        assert_close(got.cpu().numpy(), start + y.float().cpu().numpy().astype(np.float64).T @ dz, f"dH, {n} rows", 1e-4)
    ctx.close()
    ref_ctx.close()


def test_static_scratch_variant_refuses_what_does_not_fit():
    fi = fo = 512
    ctx = vb.Context([fi, fo], [vb.ACT_IDENTITY], vb.CONV_GCN, 1, KEY, vb.BF16)
    n = 16384                                          # full split of the bf16 kernel: 64 slabs of 1 MiB
    y = torch.zeros((n, fi), dtype=torch.bfloat16, device="cuda")
    d = torch.zeros((n, fo), dtype=torch.bfloat16, device="cuda")
    dh = torch.zeros((fi, fo), device="cuda")
    with pytest.raises(vb.VarcoError) as e:
        ctx.transform_bwd_weight_static(0, y, d, None, dh)
    assert e.value.code == vb.ERR_SHAPE and "67108864 bytes of scratch" in str(e.value) and "33554432" in str(e.value)
    ctx.transform_bwd_weight_static(0, y[:8192], d[:8192], None, dh)      # exactly the array's size: accepted
    torch.cuda.synchronize()
    assert float(dh.abs().max()) == 0.0
    ctx.close()


@pytest.mark.parametrize("fi,fo,n", [(100, 512, 65536), (128, 512, 33024), (100, 256, 83968), (128, 256, 65792), (100, 512, 41983)])
def test_static_scratch_variant_takes_flat_bf16_weights_of_any_row_count(fi, fo, n):
    """Weights of at most 128 rows: the split that fills the device would exceed the array, the one that fits it is taken, by
    both entry points."""
    ref_ctx = _prepared_reference_context(fi, fo, vb.ACT_IDENTITY, vb.BF16, n)
    ctx = vb.Context([fi, fo], [vb.ACT_IDENTITY], vb.CONV_GCN, 1, KEY, vb.BF16)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    y = torch.randn(n, fi, generator=gen, device="cuda").to(torch.bfloat16)
    d = (torch.randn(n, fo, generator=gen, device="cuda") / n).to(torch.bfloat16)
    want, got = torch.zeros(fi, fo, device="cuda"), torch.zeros(fi, fo, device="cuda")
    ref_ctx.transform_bwd_weight(0, y, d, None, want)
    ctx.transform_bwd_weight_static(0, y, d, None, got)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    assert_close(got.cpu().numpy(), (y.double().t() @ d.double()).cpu().numpy(), f"dH, {n} rows", 1e-5)
    ctx.close()
    ref_ctx.close()
