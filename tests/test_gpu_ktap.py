"""GPU parity of general K-tap layers (one compressed exchange per hop) built from the library's
building-block calls, against the K-tap oracle."""
import numpy as np
import pytest
import torch

from gpu_common import KEY, TOL, assert_close, both_partitions, products_taken
from oracle import ktap as oktap
from oracle import layer as olayer
from oracle import mask as omask
from oracle.rounding import round_bf16
from paper_2406_17611_amd import binding as vb
from paper_2406_17611_amd import synth
from paper_2406_17611_amd.runner import KTapNetwork

pytestmark = pytest.mark.gpu


def _gather(parts, per_part, n):
    out = np.empty((n, per_part[0].shape[1]))
    for p in parts:
        out[p.local_gid] = per_part[p.q]
    return out


@pytest.mark.parametrize("n_taps,ratio,dtype", [(3, (4, 1), "f32"), (4, (2, 1), "f32"), (3, (1, 1), "f32"), (2, (8, 1), "f32"),
                                                (1, (4, 1), "f32"), (3, (1, 0), "f32"), (3, (4, 1), "bf16")])
def test_ktap_network(n_taps, ratio, dtype):
    g = synth.small_random_graph(2500, 9.0, "sage", seed=70 + n_taps)
    part = synth.random_partition(g.n, 3, seed=71)
    host, orc = both_partitions(g, part, 3)
    bf16 = dtype == "bf16"
    widths = (64, 400 if bf16 else 160, 24)           # rows long enough for products
    L = 2
    # bf16: the sum of K products is rounded after every product, each hop's aggregate once more
    tol = 2.0 ** -6 if bf16 else TOL
    x0 = synth.features(g.n, widths[0], synth.SEED_FEAT)
    dxl = synth.upstream_grad(g.n, widths[-1], synth.SEED_GRAD)
    if bf16:
        x0, dxl = round_bf16(x0).astype(np.float32), round_bf16(dxl).astype(np.float32)
    weights = [[synth.glorot(widths[l], widths[l + 1], synth.SEED_WEIGHT, 8 * l + hop) for hop in range(n_taps)]
               for l in range(L)]
    net = KTapNetwork(host, widths, n_taps, KEY, dtype=dtype)
    net.set_inputs(x0)
    net.set_tap_weights(weights)
    net.set_upstream(dxl)
    acts = [olayer.RELU, olayer.IDENTITY]
    keep = [omask.keep_count(w, *ratio) for w in widths[:-1]]
    step = 5
    ref = oktap.network_step(orc, [x0[p.local_gid] for p in orc], weights, acts, keep, KEY, step,
                             [dxl[p.local_gid] for p in orc])
    net.zero_grads()
    net.ctx.reset_stats()
    net.forward(step, ratio)
    torch.cuda.synchronize()
    for l in range(L):
        for hop in range(1, n_taps):
            assert_close(net.to_global(net.y[l][hop]), _gather(orc, ref["y"][l][hop], g.n), f"Y_{l},{hop}", tol)
        assert_close(net.to_global(net.x[l + 1]), _gather(orc, ref["x"][l + 1], g.n), f"X_{l + 1}", tol)
    # the ReLU gates of the backward pass are taken on the oracle's stored activations (as in the network tests)
    stored = (lambda a: round_bf16(a).astype(np.float32)) if bf16 else (lambda a: np.asarray(a, dtype=np.float32))
    for l in range(L):
        net.x[l + 1].copy_(torch.from_numpy(stored(np.vstack(ref["x"][l + 1]))))
        for hop in range(1, n_taps):
            net.y[l][hop].copy_(torch.from_numpy(stored(np.vstack(ref["y"][l][hop]))))
    # (the hop of the last tap may sum the errors of the narrow outputs instead, the others don't)
    assert products_taken(net.ctx, net.backward) or not net.linked or n_taps < 3 or not ratio[0] > 3 * ratio[1] > 0
    for l in range(L):
        for hop in range(n_taps):
            assert_close(net.dh[l][hop].cpu().numpy(), ref["dh"][l][hop], f"dH_{l},{hop}", tol)
    assert_close(net.to_global(net.dx[1]), _gather(orc, ref["dx"][1], g.n), "dX_1", tol)
    st = net.ctx.stats()
    assert st["fwd_elems"] == ref["fwd_elems"] and st["bwd_elems"] == ref["bwd_elems"]


def test_zero_grads_clears_a_replaced_gradient():
    g = synth.small_random_graph(200, 5.0, "sage", seed=75)
    host, _ = both_partitions(g, synth.random_partition(g.n, 2, seed=76), 2)
    net = KTapNetwork(host, (8, 16, 4), 3, KEY)
    net.dh[1][2] = torch.ones(16, 4, device="cuda")
    net.dh[0][0].fill_(1.0)
    net.zero_grads()
    assert not any(bool(m.any()) for taps in net.dh for m in taps)


@pytest.mark.parametrize("widths,n_taps,ratio,dtype", [((8, 75, 47), 2, (3, 1), "f32"), ((8, 130, 5), 4, (8, 1), "f32"), ((8, 516, 64), 3, (1, 1), "f32"),
                                                       ((8, 40, 33), 3, (1, 0), "f32"), ((16, 144, 17), 3, (7, 2), "bf16"), ((16, 512, 64), 2, (16, 1), "bf16")])
def test_hop_of_the_last_tap_in_one_call(widths, n_taps, ratio, dtype):
    """The errors of a narrow layer summed before they pass the weights: the same dX as through the separate calls (either form is
    within the tolerance of the exact one), from whichever hop, and left alone where the library says that it does not form it."""
    g = synth.small_random_graph(1500, 11.0, "sage", seed=80)
    host, _ = both_partitions(g, synth.random_partition(g.n, 3, seed=81), 3)
    net = KTapNetwork(host, widths, n_taps, KEY, dtype=dtype)
    net.set_tap_weights([[synth.glorot(widths[l], widths[l + 1], synth.SEED_WEIGHT, 8 * l + hop) for hop in range(n_taps)] for l in range(2)])
    net.set_inputs(synth.features(g.n, widths[0], synth.SEED_FEAT))
    net.set_upstream(synth.upstream_grad(g.n, widths[-1], synth.SEED_GRAD))
    net.forward(3, ratio)
    tap, far, near = vb.tap(1, n_taps - 1), net.h[1][n_taps - 1], net.h[1][n_taps - 2]
    got, through, want = (torch.full_like(net.x[1], 7.0) for _ in range(3))
    net.ctx.reset_stats()
    formed = net.ctx.network_taps_bwd_last_hop(tap, net.dx[2], far, near, got)
    handed = net.ctx.stats()["bwd_elems"]
    net.ctx.reset_stats()
    net.ctx.network_taps_bwd_input(1, net.dx[2], net.x[2], [far], [through])
    net.ctx.network_aggregate_bwd(tap, through, want, False)
    assert not formed or handed == net.ctx.stats()["bwd_elems"]
    net.ctx.transform_bwd_input(1, net.dx[2], net.x[2], near, want, True)
    torch.cuda.synchronize()
    if not formed:                   # few errors are sent: the sums at the width of the inputs move less
        assert bool((got == 7.0).all()) and ratio == (1, 0)
    else:
        assert_close(net.to_global(got), net.to_global(want), "dX", 2.0 ** -6 if dtype == "bf16" else 2 * TOL)
    assert not net.ctx.network_taps_bwd_last_hop(vb.tap(0, 1), net.dx[1], net.h[0][1], net.h[0][0], net.x[0].clone())      # a layer with an activation
