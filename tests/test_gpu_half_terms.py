"""Gradients of the dense transform as products of two scaled fp16 terms (fp32 storage), where their scales have work to do: rows and
columns of very different magnitude, values that grow along the reduction, leading zeros, reductions of any length, values that are
not finite. Against fp64 products of the same inputs."""
import numpy as np
import pytest
import torch

from gpu_common import KEY, dev
from paper_2406_17611_amd import binding as vb
from paper_2406_17611_amd import synth

pytestmark = pytest.mark.gpu


def _context(fi, fo, rows=0, conv=vb.CONV_GCN):
    ctx = vb.Context([fi, fo], [vb.ACT_RELU], conv, 1, KEY)
    if rows:                    # the partial products of a weight gradient are sized by a registered partition
        g = synth.small_random_graph(max(rows, 8), 3.0, "gcn", seed=5)
        host = vb.partition_build(g.n, g.rowptr, g.colidx, g.vals, np.zeros(g.n, dtype=np.int32), 1)
        ctx.register_partition(0, host[0])
    ctx.prepare()
    return ctx


def _bound(length, a, b):
    """Per element: both terms of either operand within 2^-23 of the value, one rounding of 2^-24 per 16 products on a partial sum,
    which is at most sum |a||b|: sqrt of their number for the error of independent roundings, four times that for the tail."""
    return (2.0 ** -21 + 4 * 2.0 ** -23 * np.sqrt(np.ceil(length / 16) + 1)) * (np.abs(a) @ np.abs(b))


@pytest.mark.parametrize("fo", [65, 66, 75, 96, 97, 128, 200, 260, 321, 352, 384, 385, 417, 448, 449, 512])
@pytest.mark.parametrize("growth", [0, 5, 7, 12])
def test_input_gradient_rows_of_any_magnitude(fo, growth):
    n, fi = 300, 136
    rng = np.random.default_rng(fo + growth)
    d = rng.standard_normal((n, fo)) * np.exp2(rng.integers(-90, 20, size=(n, 1)))
    d *= np.exp2(growth * (np.arange(fo) // 32))[None, :] if growth * (fo // 32) < 60 else np.exp2(growth * (np.arange(fo) >= 64))[None, :]
    d[::7, :32] = 0.0                                     # nothing in the first stage
    d[5] = 0.0
    d = d.astype(np.float32)
    xo = rng.standard_normal((n, fo)).astype(np.float32)
    h = (synth.glorot(fi, fo, 3, 1) * np.exp2(rng.integers(-30, 30, size=(fi, 1)))).astype(np.float32)
    taps = [h, h[::-1].copy()]
    out = [torch.empty(n, fi, device="cuda") for _ in range(3)]
    ctx = _context(fi, fo, n, vb.CONV_SAGE)
    ctx.transform_bwd_input(0, dev(d), dev(xo), dev(h), out[0], False)
    assert ctx.link_partitions()
    ctx.prepare()
    ctx.set_step(1)
    ctx.network_taps_bwd_input(0, dev(d), dev(xo), [dev(a) for a in taps], out[1:])      # two taps share the rows of dZ and their scales
    torch.cuda.synchronize()
    dz = d.astype(np.float64) * (xo > 0)
    for a, got in zip((h, *taps), out):
        err = np.abs(got.cpu().numpy() - dz @ a.astype(np.float64).T)
        assert (err <= _bound(fo, dz, a.astype(np.float64).T)).all()


@pytest.mark.parametrize("fo", [17, 24, 32, 33, 47, 48, 49, 64])
@pytest.mark.parametrize("growth", [0, 7, 12])
def test_short_input_gradient_rows_of_any_magnitude(fo, growth):
    test_input_gradient_rows_of_any_magnitude(fo, growth)      # one stage or two, with a remainder or none


@pytest.mark.parametrize("fi,fo", [(1, 65), (31, 127), (33, 128), (64, 129), (129, 159), (255, 192), (257, 225), (300, 256), (15, 257), (65, 289), (128, 320), (250, 511), (48, 512), (40, 516),
                                   (100, 193), (130, 200), (70, 321), (96, 352), (65, 353), (129, 384), (77, 385), (128, 416), (100, 417), (250, 448), (66, 449)])
@pytest.mark.parametrize("n,accumulate", [(1, False), (33, True), (63, False), (64, True), (8225, False)])
def test_input_gradient_at_the_edges_of_blocks(n, accumulate, fi, fo):
    """Rows in blocks of 32 or 64 of workgroups that walk over them, columns in units of 16 or 32 of wavefronts, every number of stages from three to
    sixteen (those that an odd number leaves empty among them), and what is left to the tiles."""
    rng = np.random.default_rng(n + fi + fo)
    d, xo = (rng.standard_normal((n, fo)).astype(np.float32) for _ in range(2))
    h = synth.glorot(fi, fo, 3, 1).astype(np.float32)
    old = rng.standard_normal((n + 1, fi)).astype(np.float32)
    out = dev(old)
    _context(fi, fo).transform_bwd_input(0, dev(d), dev(xo), dev(h), out[:n], accumulate)
    torch.cuda.synchronize()
    dz, got = d.astype(np.float64) * (xo > 0), out.cpu().numpy()
    want = dz @ h.astype(np.float64).T + (old[:n] if accumulate else 0.0)
    slack = 2.0 ** -24 * np.abs(want) if accumulate else 0.0          # the addition's own rounding
    assert (np.abs(got[:n] - want) <= _bound(fo, dz, h.astype(np.float64).T) + slack).all()
    assert np.array_equal(got[n], old[n])                             # the row behind the last one


@pytest.mark.parametrize("n,fi,fo", [(65_537, 16, 120), (65_500, 16, 120), (262_145, 33, 96), (261_990, 33, 80), (2_001, 32, 102), (24_001, 32, 102), (24_575, 48, 225),
                                     (32_767, 48, 225), (32_769, 64, 225), (8_192, 384, 96), (8_193, 384, 96), (21_889, 384, 66), (21_762, 384, 128)])
def test_input_gradient_on_both_sides_of_the_lines(n, fi, fo):
    test_input_gradient_at_the_edges_of_blocks(n, False, fi, fo)      # few outputs, and a last group with idle wavefronts: tiles or blocks of rows


@pytest.mark.parametrize("n,fi,fo", [(32_768, 16, 96), (32_769, 16, 96), (16_129, 33, 100), (33_025, 33, 100)])
def test_two_input_gradients_on_both_sides_of_the_line(n, fi, fo):
    rng = np.random.default_rng(n + fi + fo)
    d, xo = (rng.standard_normal((n, fo)).astype(np.float32) for _ in range(2))
    h = [synth.glorot(fi, fo, 3, t).astype(np.float32) for t in range(2)]
    out = [torch.full((n + 1, fi), 7.0, device="cuda") for _ in range(2)]
    ctx = _context(fi, fo, n, vb.CONV_SAGE)
    assert ctx.link_partitions()
    ctx.prepare()
    ctx.network_taps_bwd_input(0, dev(d), dev(xo), [dev(a) for a in h], out)
    torch.cuda.synchronize()
    dz = d.astype(np.float64) * (xo > 0)
    for a, got in zip(h, out):
        got = got.cpu().numpy()
        assert (np.abs(got[:n] - dz @ a.astype(np.float64).T) <= _bound(fo, dz, a.astype(np.float64).T)).all()
        assert (got[n] == 7.0).all()


@pytest.mark.parametrize("fi,fo", [(4, 4), (75, 47), (64, 65), (130, 136)])
@pytest.mark.parametrize("growth", [0, 7])
@pytest.mark.parametrize("n", [1, 31, 33, 2333])
def test_weight_gradient_of_growing_values(n, growth, fi, fo):
    rng = np.random.default_rng(n + fi + growth)
    steps = np.exp2(growth * np.minimum(np.arange(n) // 32 % 8, 6))[:, None]      # up to 2^42 larger than the first stage, and back
    y = (rng.standard_normal((n, fi)) * steps * 2.0 ** -40).astype(np.float32)
    y[: min(n - 1, 40)] = 0.0
    d = (rng.standard_normal((n, fo)) * 2.0 ** 30 / steps[::-1]).astype(np.float32)
    xo = rng.standard_normal((n, fo)).astype(np.float32)
    dh = torch.zeros(fi, fo, device="cuda")
    _context(fi, fo, n).transform_bwd_weight(0, dev(y), dev(d), dev(xo), dh)
    torch.cuda.synchronize()
    dz = d.astype(np.float64) * (xo > 0)
    err = np.abs(dh.cpu().numpy() - y.astype(np.float64).T @ dz)
    # a value far below the largest of its 64 columns and slab is within 2^-42 of that one
    floor = 2.0 ** -42 * (np.abs(y).max() * np.abs(dz).sum(0)[None, :] + np.abs(y).sum(0)[:, None] * np.abs(dz).max())
    assert (err <= _bound(n, y.astype(np.float64).T, dz) + floor).all()


@pytest.mark.parametrize("fi,fo", [(4, 4), (75, 47), (64, 65), (130, 136)])
@pytest.mark.parametrize("growth", [0, 7])
@pytest.mark.parametrize("n", [1, 33, 2333])
def test_weight_gradient_of_columns_of_any_magnitude(n, growth, fi, fo):
    """Features of different units, outputs of different weight: every column keeps its own bits, alone and where two taps share
    the errors."""
    rng = np.random.default_rng(n + fi + growth)
    steps = np.exp2(growth * np.minimum(np.arange(n) // 32 % 8, 6))[:, None]
    y = [(rng.standard_normal((n, fi)) * np.exp2(rng.integers(-60, 30, size=(1, fi))) * steps).astype(np.float32) for _ in range(2)]
    d = (rng.standard_normal((n, fo)) * np.exp2(rng.integers(-50, 30, size=(1, fo))) / steps[::-1]).astype(np.float32)
    xo = rng.standard_normal((n, fo)).astype(np.float32)
    xo[0] = 1.0                                           # (no column without a value)
    ctx = _context(fi, fo, n, vb.CONV_SAGE)
    single, pair = torch.zeros(fi, fo, device="cuda"), [torch.zeros(fi, fo, device="cuda") for _ in range(2)]
    ctx.transform_bwd_weight(0, dev(y[0]), dev(d), dev(xo), single)
    rows = max(n, 8)                                      # (the partition's: zeros follow)
    padded = lambda a: dev(np.concatenate([a, np.zeros((rows - n, a.shape[1]), dtype=np.float32)]))
    assert ctx.link_partitions()
    ctx.prepare()
    ctx.network_taps_bwd_weight(0, [padded(a) for a in y], padded(d), padded(xo), pair)
    torch.cuda.synchronize()
    dz = d.astype(np.float64) * (xo > 0)
    for a, got in zip((y[0], *y), (single, *pair)):
        a = a.astype(np.float64)
        err = np.abs(got.cpu().numpy() - a.T @ dz)
        # a value far below the largest of its own column is within 2^-42 of that one
        floor = 2.0 ** -42 * (np.abs(a).max(0)[:, None] * np.abs(dz).sum(0)[None, :] + np.abs(a).sum(0)[:, None] * np.abs(dz).max(0)[None, :])
        assert (err <= _bound(n, a.T, dz) + floor).all()


@pytest.mark.parametrize("fi,fo", [(5, 63), (63, 129), (65, 64), (127, 4), (128, 128), (129, 66), (192, 127), (193, 5), (256, 130), (257, 64), (321, 47)])
@pytest.mark.parametrize("n", [31, 97])
def test_weight_gradient_at_the_edges_of_tiles(n, fi, fo):
    test_weight_gradient_of_columns_of_any_magnitude(n, 7, fi, fo)      # 64 columns a unit, 128 or 256 a tile, one tap and two


def test_infinite_values_stay_in_their_rows_and_columns():
    n, fi, fo = 700, 128, 96
    rng = np.random.default_rng(9)
    y, d = rng.standard_normal((n, fi)).astype(np.float32), rng.standard_normal((n, fo)).astype(np.float32)
    h = synth.glorot(fi, fo, 3, 1).astype(np.float32)
    ones = torch.ones(n, fo, device="cuda")
    y[321, 17], d[650, 40] = np.inf, -np.inf
    ctx = _context(fi, fo, n)
    dh, dx = torch.zeros(fi, fo, device="cuda"), torch.empty(n, fi, device="cuda")
    ctx.transform_bwd_weight(0, dev(y), dev(d), ones, dh)
    ctx.transform_bwd_input(0, dev(d), ones, dev(h), dx, False)
    torch.cuda.synchronize()
    got_h, got_x = dh.cpu().numpy(), dx.cpu().numpy()
    assert not np.isfinite(got_h[17]).any() and not np.isfinite(got_h[:, 40]).any() and not np.isfinite(got_x[650]).any()
    rows, cols, nodes = np.arange(fi) != 17, np.arange(fo) != 40, np.arange(n) != 650
    ref_h = y[:, rows].astype(np.float64).T @ d[:, cols].astype(np.float64)
    assert (np.abs(got_h[rows][:, cols] - ref_h) <= _bound(n, y[:, rows].astype(np.float64).T, d[:, cols].astype(np.float64))).all()
    ref_x = d[nodes].astype(np.float64) @ h.astype(np.float64).T
    assert (np.abs(got_x[nodes] - ref_x) <= _bound(fo, d[nodes].astype(np.float64), h.astype(np.float64).T)).all()
