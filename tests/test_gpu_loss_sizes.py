"""The cross-entropy kernel at the class counts where its lane groups change, with and without a prepared stream (which
decides how the rows' losses are summed) and with the gradient written over the logits."""
import numpy as np
import pytest
import torch

from gpu_common import KEY, assert_close, dev
from oracle import train as otrain
from paper_2406_17611_amd import binding as vb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 33, 40000])
@pytest.mark.parametrize("n_classes", [1, 8, 9, 16, 17, 64, 65, 512, 516])
def test_class_counts(n_classes, n):
    rng = np.random.default_rng(n_classes + n)
    z = (rng.standard_normal((n, n_classes)) * 3).astype(np.float32)
    y = rng.integers(-1, n_classes, size=n).astype(np.int32)
    scale = 1.0 / max(1, int((y >= 0).sum()))
    loss_ref, d_ref, correct_ref = otrain.softmax_xent(z, y, scale)
    ctx = vb.Context([8, n_classes], [0], vb.CONV_GCN, 1, KEY)
    row_loss = torch.empty(n, dtype=torch.float32, device="cuda")
    row_correct = torch.empty(n, dtype=torch.int32, device="cuda")
    for prepared in (False, True):
        if prepared:
            ctx.prepare()
        zd = dev(z)
        totals = torch.zeros(2, dtype=torch.float32, device="cuda")
        ctx.softmax_xent(zd, dev(y), n_classes, scale, zd, row_loss, row_correct, totals)
        got = totals.cpu().numpy()
        assert abs(got[0] - loss_ref) <= 1e-5 * abs(loss_ref) + 1e-6
        assert int(round(got[1])) == correct_ref == int(row_correct.sum().item())
        assert_close(zd.cpu().numpy(), d_ref, "dlogits", 1e-5)
    ctx.close()
