"""The form of the runner that serves partition after partition, which it takes when the partitions cannot be linked (2^31
entries, no room on the device)."""
import pytest
import torch

from gpu_common import assert_close
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
