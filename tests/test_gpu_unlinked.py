"""The form of the runner that serves partition after partition, which it takes when the partitions cannot be linked (2^31
entries, no room on the device): the same tests as for the linked form, on one and several streams, and both against each other."""
import pytest
import torch

import test_gpu_graph
import test_gpu_ktap
import test_gpu_network
import test_gpu_train
from gpu_common import assert_close, hub_graph, products_taken
from paper_2406_17611_amd import binding as vb
from paper_2406_17611_amd import synth
from test_gpu_graph import _network

pytestmark = pytest.mark.gpu


def test_link_without_room_falls_back(monkeypatch):
    """The device is filled for the time of the link call, whose first allocations then fail; nothing was launched, and the
    partitions are served one after the other with the results of the linked form."""
    n = 60_000
    g = synth.gcn_operator(n, *synth.chung_lu_edges(n, 3_000_000, 2.5, 5))
    part = synth.random_partition(n, 3, seed=6)
    widths, ratio = (8, 16, 4), (4, 1)
    link = vb.Context.link_partitions

    def link_on_a_full_device(ctx):
        torch.cuda.empty_cache()
        filler, left = [], torch.cuda.mem_get_info()[0] - (32 << 20)
        while left >= 32 << 20:                          # what cannot be had in one piece is taken in smaller ones
            try:
                filler.append(torch.empty(left, dtype=torch.uint8, device="cuda"))
                left = torch.cuda.mem_get_info()[0] - (32 << 20)
            except torch.OutOfMemoryError:
                left //= 2
        try:
            return link(ctx)
        finally:
            filler.clear()
            torch.cuda.empty_cache()

    nets = []
    for patched in (False, True):
        monkeypatch.setattr(vb.Context, "link_partitions", link_on_a_full_device if patched else link)
        net = _network(g, part, 3, widths, "gcn", 1)     # 6 million entries: 168 MB of joined arrays, 64 MB at most are free
        assert net.linked is not patched
        net.zero_grads()
        net.step(4, ratio)
        torch.cuda.synchronize()
        nets.append(net)
    _compare(nets[0], nets[1], 1e-5)
    assert nets[0].ctx.stats() == nets[1].ctx.stats()
    # with room again the same context links
    monkeypatch.setattr(vb.Context, "link_partitions", link)
    assert nets[1].ctx.link_partitions()


def _compare(a, b, tol):
    for l in range(1, a.L + 1):
        assert_close(b.x[l].float().cpu().numpy(), a.x[l].float().cpu().numpy(), f"X_{l}", tol)
    for l in range(a.L):
        assert_close(b.dh1[l].cpu().numpy(), a.dh1[l].cpu().numpy(), f"dH1_{l}", tol)
        if a.dh0[l] is not None:
            assert_close(b.dh0[l].cpu().numpy(), a.dh0[l].cpu().numpy(), f"dH0_{l}", tol)
    for l in range(1, a.L):
        assert_close(b.dx[l].float().cpu().numpy(), a.dx[l].float().cpu().numpy(), f"dX_{l}", tol)


@pytest.fixture
def unlinked(monkeypatch):
    monkeypatch.setattr(vb.Context, "link_partitions", lambda ctx: False)


@pytest.mark.parametrize("conv,dtype,n_streams,first", [("sage", "f32", 1, ()), ("gcn", "f32", 2, ()), ("sage", "f32", 3, ()),
                                                        ("sage", "bf16", 2, ()), ("gcn", "bf16", 2, (2,))])
def test_linked_and_partition_after_partition_agree(monkeypatch, conv, dtype, n_streams, first):
    g = hub_graph(3000, 3, 1100, 6.0, conv, seed=91)
    part = synth.random_partition(g.n, 4, seed=92)
    widths = (33, 400 if dtype == "bf16" else 136, 80, 9)           # rows long enough for products
    nets = []
    for linked in (True, False):
        with monkeypatch.context() as m:
            if not linked:
                m.setattr(vb.Context, "link_partitions", lambda ctx: False)
            nets.append(_network(g, part, 4, widths, conv, n_streams, dtype=dtype, transform_first=first))
        assert nets[-1].linked is linked
    # bf16: at most six roundings of 2^-9 lie between the inputs and a gradient, in different places in the two forms; a ReLU
    # gate within rounding of zero may open on one side only, so both sides take the gates (and saved rows) of the linked form
    tol = 2.0 ** -5 if dtype == "bf16" else 2e-5
    for step, ratio in enumerate([(4, 1), (5, 1), (3, 2), (1, 1), (1, 0)]):
        for net in nets:
            net.zero_grads()
            net.ctx.reset_stats()
            net.forward(step, ratio)
        torch.cuda.synchronize()
        for l in range(1, nets[0].L + 1):
            assert_close(nets[1].x[l].float().cpu().numpy(), nets[0].x[l].float().cpu().numpy(), f"X_{l}", tol)
            nets[1].x[l].copy_(nets[0].x[l])
        for l in range(nets[0].L):
            if l not in first:
                nets[1].m[l].copy_(nets[0].m[l])
        assert products_taken(nets[0].ctx, nets[0].backward) is (ratio[0] > 3 * ratio[1] > 0)
        nets[1].backward()
        torch.cuda.synchronize()
        _compare(nets[0], nets[1], tol)
        assert nets[0].ctx.stats() == nets[1].ctx.stats()


@pytest.mark.parametrize("n_streams", [2, 3])
def test_partitions_dealt_to_several_streams(unlinked, n_streams):
    test_gpu_network.test_partitions_dealt_to_several_streams(n_streams)


@pytest.mark.parametrize("n_streams", [1, 2])
def test_graph_replays_equal_eager_steps(unlinked, n_streams):
    test_gpu_graph.test_graph_replays_equal_eager_steps(n_streams)


def test_graph_replays_with_the_class_layer_transforming_first(unlinked):
    test_gpu_graph.test_graph_replays_with_the_class_layer_transforming_first()


@pytest.mark.parametrize("n_taps,ratio,dtype", [(3, (4, 1), "f32"), (4, (2, 1), "f32"), (3, (1, 1), "f32"), (1, (4, 1), "f32"),
                                                (3, (1, 0), "f32"), (3, (4, 1), "bf16")])
def test_ktap_network(unlinked, n_taps, ratio, dtype):
    test_gpu_ktap.test_ktap_network(n_taps, ratio, dtype)


@pytest.mark.parametrize("conv,dtype", [("sage", "f32"), ("sage", "bf16")])
def test_training_iterations_match_the_oracle(unlinked, conv, dtype):
    test_gpu_train.test_training_iterations_match_the_oracle(conv, dtype)


@pytest.mark.parametrize("n_streams", [1, 2])
def test_free_running_training(unlinked, n_streams):
    test_gpu_train.test_free_running_training_learns_and_tracks_the_oracle(n_streams)
