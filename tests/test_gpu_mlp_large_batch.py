"""The surrogate's forward pass beyond the largest training batch (8192 rows),
where a work-group takes 64 rows: predictions and every saved activation are
those of the same rows in training-sized batches, byte for byte; the backward
pass refuses such batches; a workspace for many rows serves fewer.
"""
import numpy as np
import pytest
import torch

from paper_2407_02363_amd import edt, inputs, mlp
from paper_2407_02363_amd.surrogate import Surrogate
from tests.gpu_util import dev, say
from tests.test_gpu_mlp import ws_views

pytestmark = pytest.mark.gpu


def test_workspace_never_shrinks():
    sizes = [mlp.sdf_mlp_workspace_bytes(b) for b in (1, 64, 65, 4096, 8191, 8192, 8193, 10000, 33000, 65536, 262144)]
    assert sizes == sorted(sizes)


@pytest.mark.parametrize("batch", [8193, 8255, 8256, 12301, 20000])
def test_forward_of_many_rows(batch):
    say("[mlp] forward of", batch)
    d = dev()
    s = Surrogate(d, seed=3, batch=batch)
    q = torch.from_numpy(inputs.random_joint_states(batch + 9, 5).astype(np.float32)).to(d)
    idx = torch.from_numpy(inputs.rng(7).permutation(batch + 9)[:batch].astype(np.int32)).to(d)
    idx[5], idx[batch - 1] = -1, batch + 9      # rows of NaN
    s.ws.fill_(0xFF)
    y = torch.empty((batch, mlp.N_OUT), dtype=torch.float32, device=d)
    mlp.sdf_mlp_forward(s.w16, s.master, q, y, s.ws, idx=idx)
    big = {k: v.copy() for k, v in ws_views(s.ws, batch).items()}
    t = torch.zeros((batch, mlp.N_OUT), dtype=torch.float32, device=d)
    with pytest.raises(edt.EdtError) as e:
        mlp.sdf_mlp_backward(s.w16, t, s.grad, s.loss, s.ws)
    assert e.value.status == -5
    for r0 in range(0, batch, 8192):
        n = min(8192, batch - r0)
        part = torch.empty((n, mlp.N_OUT), dtype=torch.float32, device=d)
        mlp.sdf_mlp_forward(s.w16, s.master, q, part, s.ws, idx=idx[r0:r0 + n])
        assert torch.equal(part.view(torch.int32), y[r0:r0 + n].view(torch.int32))
        small = ws_views(s.ws, n)
        for k in ("x", "h1", "h2", "h3"):
            assert np.array_equal(small[k][:n], big[k][r0:r0 + n], equal_nan=True), (k, r0)
    # a training step on the same workspace
    s.train_step(q, torch.zeros((batch + 9, mlp.N_OUT), device=d), idx=idx[6:4000].contiguous())
    assert torch.isfinite(s.loss).all() and torch.isfinite(s.grad).all()
