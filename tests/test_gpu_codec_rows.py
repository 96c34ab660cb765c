"""Encoder and decoders on aligned rows (16-byte accesses, rows through LDS) at the edges of their groups of rows and of the
rules that choose between the forms; compared bit for bit with the oracle."""
import numpy as np
import pytest
import torch

from gpu_common import KEY, dev
from oracle import layer as olayer
from oracle import mask as omask
from oracle.rounding import round_bf16
from paper_2406_17611_amd import binding as vb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rows", [1, 3, 4, 1025])
@pytest.mark.parametrize("dtype,width,ratio", [("f32", 256, (8, 1)), ("f32", 256, (32, 1)), ("f32", 260, (2, 1)), ("f32", 12, (4, 1)),
                                               ("f32", 2048, (4, 1)), ("f32", 256, (1, 1)), ("bf16", 512, (4, 1)), ("bf16", 512, (7, 1)),
                                               ("bf16", 520, (64, 1)), ("bf16", 8, (2, 1)), ("bf16", 2048, (3, 1)), ("bf16", 256, (1, 1))])
def test_aligned_rows(dtype, width, ratio, n_rows):
    bf16 = dtype == "bf16"
    rng = np.random.default_rng(width + n_rows)
    stored = (lambda a: round_bf16(a).astype(np.float32)) if bf16 else (lambda a: np.asarray(a, dtype=np.float32))
    tdt = torch.bfloat16 if bf16 else torch.float32
    n_src = n_rows + 7
    x = stored(rng.standard_normal((n_src, width)))
    rows = np.sort(rng.permutation(n_src)[:n_rows]).astype(np.int32)
    gids = rng.integers(0, 2_449_029, size=n_rows).astype(np.int32)
    ctx = vb.Context([8, width, 8], [1, 0], vb.CONV_GCN, 1, KEY, vb.BF16 if bf16 else vb.F32)
    ctx.prepare()
    ctx.begin_step(6)
    ctx.set_ratio(1, *ratio)
    k = ctx.keep(1)
    cols = omask.kept_columns(gids, width, k, KEY, 6, 1)
    xd, rd, gd = dev(x, tdt), dev(rows), dev(gids)
    z = torch.zeros((n_rows + 1, k), dtype=tdt, device="cuda")          # one row of slack: must stay untouched
    ctx.compress(1, gd, rd, n_rows, xd, width, z)
    want_z = olayer.compress(x, rows, cols).astype(np.float32)
    assert np.array_equal(z[:n_rows].float().cpu().numpy(), want_z) and not z[n_rows].any()
    out = torch.full((n_src, width), 7.0, dtype=tdt, device="cuda")
    ctx.decompress(1, gd, rd, n_rows, z, out, width, 0)
    want = np.full((n_src, width), 7.0, dtype=np.float32)
    want[rows] = olayer.decompress(want_z.astype(np.float64), cols, width).astype(np.float32)
    assert np.array_equal(out.float().cpu().numpy(), want)
    acc = dev(x, tdt)
    ctx.decompress(1, gd, rd, n_rows, z, acc, width, 1)
    want_acc = x.copy()
    for i in range(n_rows):
        want_acc[rows[i], cols[i]] = stored(want_acc[rows[i], cols[i]] + want_z[i])
    assert np.array_equal(acc.float().cpu().numpy(), want_acc)
    ctx.close()


@pytest.mark.parametrize("dtype,width,ratio,n_rows", [("f32", 256, (7, 1), 1025), ("f32", 255, (2, 1), 1025), ("f32", 380, (2, 1), 3), ("f32", 384, (2, 1), 1025),
                                                      ("f32", 385, (2, 1), 5), ("bf16", 511, (2, 1), 1025), ("bf16", 516, (2, 1), 3),
                                                      ("f32", 12, (3, 1), 131_107), ("bf16", 16, (2, 1), 262_147)])
def test_both_sides_of_the_line_by_row_length(dtype, width, ratio, n_rows):
    test_aligned_rows(dtype, width, ratio, n_rows)      # the last two: wavefronts that walk take more than one group


@pytest.mark.parametrize("dtype,width,ratio,n_rows", [("f32", 256, (8, 1), 33_001), ("f32", 384, (4, 1), 22_003), ("f32", 385, (2, 1), 22_001), ("f32", 505, (2, 1), 3),
                                                      ("bf16", 512, (4, 1), 33_001), ("bf16", 772, (2, 1), 22_003), ("bf16", 768, (8, 1), 1025)])
@pytest.mark.parametrize("listed", [True, False])
def test_adding_decoder_of_many_rows(dtype, width, ratio, n_rows, listed):
    """Groups of two rows, an odd number of them, on either side of what the caches hold; rows of a list or in order."""
    bf16 = dtype == "bf16"
    rng = np.random.default_rng(width)
    stored = (lambda a: round_bf16(a).astype(np.float32)) if bf16 else (lambda a: np.asarray(a, dtype=np.float32))
    tdt = torch.bfloat16 if bf16 else torch.float32
    n_src = n_rows + 9
    x = stored(rng.standard_normal((n_src, width), dtype=np.float32))
    rows = np.sort(rng.permutation(n_src)[:n_rows]).astype(np.int32) if listed else np.arange(n_rows, dtype=np.int32)
    gids = rng.integers(0, 2_449_029, size=n_rows).astype(np.int32)
    ctx = vb.Context([8, width, 8], [1, 0], vb.CONV_GCN, 1, KEY, vb.BF16 if bf16 else vb.F32)
    ctx.prepare()
    ctx.begin_step(6)
    ctx.set_ratio(1, *ratio)
    k = ctx.keep(1)
    z = stored(rng.standard_normal((n_rows, k), dtype=np.float32))
    cols = np.asarray(omask.kept_columns(gids, width, k, KEY, 6, 1), dtype=np.int64).reshape(n_rows, k)
    acc = dev(x, tdt)
    ctx.decompress(1, dev(gids), dev(rows) if listed else None, n_rows, dev(z, tdt), acc, width, 1)
    at = rows.astype(np.int64)[:, None]
    x[at, cols] = stored(x[at, cols] + z)
    assert np.array_equal(acc.float().cpu().numpy(), x)
    ctx.close()


@pytest.mark.parametrize("dtype,width,ratio,n_rows", [("f32", 256, (8, 1), 327_679), ("f32", 256, (8, 1), 327_683), ("f32", 320, (2, 1), 262_145), ("f32", 512, (16, 1), 163_841),
                                                      ("f32", 896, (32, 1), 93_623), ("bf16", 512, (4, 1), 163_839), ("bf16", 512, (4, 1), 163_843), ("bf16", 516, (2, 1), 325_145)])
def test_on_both_sides_of_the_line_by_all_rows(dtype, width, ratio, n_rows):
    """Rows that the last-level cache holds, or half of it, and more: all three calls, against index operations on the same device."""
    bf16 = dtype == "bf16"
    tdt, idt = (torch.bfloat16, torch.int16) if bf16 else (torch.float32, torch.int32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(width)
    n_src = n_rows + 5
    x = torch.randn(n_src, width, generator=gen, device="cuda").to(tdt)
    rows = torch.randperm(n_src, generator=gen, device="cuda")[:n_rows].sort().values
    gids = (rows * 3 + 1).to(torch.int32)
    ctx = vb.Context([8, width, 8], [1, 0], vb.CONV_GCN, 1, KEY, vb.BF16 if bf16 else vb.F32)
    ctx.prepare()
    ctx.begin_step(6)
    ctx.set_ratio(1, *ratio)
    k = ctx.keep(1)
    cols = dev(np.asarray(omask.kept_columns(gids.cpu().numpy(), width, k, KEY, 6, 1), dtype=np.int64).reshape(n_rows, k))
    z = torch.zeros((n_rows + 1, k), dtype=tdt, device="cuda")
    ctx.compress(1, gids, rows.to(torch.int32), n_rows, x, width, z)
    want = x[rows].gather(1, cols)
    assert torch.equal(z[:n_rows].view(idt), want.view(idt)) and not z[n_rows].any()
    out = torch.full((n_src, width), 7.0, dtype=tdt, device="cuda")
    ctx.decompress(1, gids, None, n_rows, z, out, width, 0)
    assert torch.equal(out[:n_rows].view(idt), torch.zeros_like(out[:n_rows]).scatter_(1, cols, want).view(idt)) and bool((out[n_rows:] == 7.0).all())
    add = torch.randn(n_rows, k, generator=gen, device="cuda").to(tdt)
    old = x.clone()
    ctx.decompress(1, gids, rows.to(torch.int32), n_rows, add, x, width, 1)
    old[rows] = old[rows].scatter(1, cols, (want.float() + add.float()).to(tdt))
    assert torch.equal(x.view(idt), old.view(idt))
    ctx.close()


@pytest.mark.parametrize("dtype,width,ratio", [("f32", 256, (8, 1)), ("f32", 2048, (4, 1)), ("f32", 75, (2, 1)), ("bf16", 512, (4, 1)),
                                               ("bf16", 2048, (3, 1)), ("bf16", 256, (1, 1))])
def test_adding_decoder_leaves_other_elements_alone(dtype, width, ratio):
    bf16 = dtype == "bf16"
    tdt, idt = (torch.bfloat16, torch.int16) if bf16 else (torch.float32, torch.int32)
    n = 37
    # negative zeros, both infinities and NaNs with a payload, quiet and signalling
    odd = np.array([0x8000, 0x7F80, 0xFF80, 0x7FC1, 0xFF81], dtype=np.uint16) if bf16 else \
        np.array([0x80000000, 0x7F800000, 0xFF800000, 0x7FC00123, 0xFF800321], dtype=np.uint32)
    bits = odd[np.random.default_rng(width).integers(0, len(odd), size=(n, width))]
    signed = bits.view(np.int16 if bf16 else np.int32)
    gids = (np.arange(n) * 3 + 1).astype(np.int32)
    ctx = vb.Context([8, width, 8], [1, 0], vb.CONV_GCN, 1, KEY, vb.BF16 if bf16 else vb.F32)
    ctx.prepare()
    ctx.begin_step(6)
    ctx.set_ratio(1, *ratio)
    k = ctx.keep(1)
    cols = omask.kept_columns(gids, width, k, KEY, 6, 1)
    kept = np.zeros((n, width), dtype=bool)
    np.put_along_axis(kept, np.asarray(cols, dtype=np.int64).reshape(n, k), True, axis=1)
    x = dev(signed)
    z = torch.full((n, k), -0.0, dtype=tdt, device="cuda")
    ctx.decompress(1, dev(gids), None, n, z, x.view(tdt), width, 1)
    got = x.view(idt).cpu().numpy()
    assert np.array_equal(got[~kept], signed[~kept])
    zero = kept & (bits == odd[0])
    assert zero.any() and np.array_equal(got[zero], signed[zero])          # -0 + -0
    ctx.close()


def test_more_rows_than_32_bits_count():
    n = (1 << 31) + 5                                     # without a row list, rows are numbered by the kernels themselves
    ctx = vb.Context([8, 2, 8], [1, 0], vb.CONV_GCN, 1, KEY, vb.BF16)
    ctx.prepare()
    ctx.begin_step(2)
    ctx.set_ratio(1, 2, 1)
    gids = torch.zeros(n, dtype=torch.int32, device="cuda")
    col = int(np.asarray(omask.kept_columns(np.zeros(1, dtype=np.int32), 2, 1, KEY, 2, 1)).ravel()[0])
    x = torch.zeros(n, 2, dtype=torch.bfloat16, device="cuda")
    some = torch.tensor([0, 1, 7, (1 << 31) - 1, 1 << 31, n - 1], device="cuda")
    val = torch.arange(1, 7, device="cuda").to(torch.bfloat16)
    x[some, col] = val
    z = torch.full((n,), 9.0, dtype=torch.bfloat16, device="cuda")
    ctx.compress(1, gids, None, n, x, 2, z)
    assert torch.equal(z[some], val) and int((z != 0).sum()) == 6
    ctx.decompress(1, gids, None, n, z, x, 2, 1)
    assert torch.equal(x[some, col], 2 * val) and int((x != 0).sum()) == 6
    x.fill_(5.0)
    ctx.decompress(1, gids, None, n, z, x, 2, 0)
    assert torch.equal(x[some, col], val) and int((x != 0).sum()) == 6
    ctx.close()
