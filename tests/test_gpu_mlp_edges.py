"""The surrogate's kernels at the batch sizes where their tiles end: 16-row
tiles, 64-row padding, gradient chunks of unequal length, the largest batch;
inference tiles of 16 and 64 rows and several tiles per work-group.  Weight
gradients against the oracle within 2e-3 of their largest entry (one-ulp
bfloat16 flips of masked upstream gradients), inference bit for bit against
the forward pass.
"""
import numpy as np
import pytest
import torch

from oracle import mlp_ref as M
from paper_2407_02363_amd import inputs, mlp
from paper_2407_02363_amd.surrogate import Surrogate
from tests.gpu_util import dev, say
from tests.test_gpu_mlp import device_params, ws_views

pytestmark = pytest.mark.gpu


def surrogate(batch, seed):
    s = Surrogate(dev(), seed=seed, batch=batch)
    g = inputs.rng(seed + 100)
    p = s.master.cpu().numpy()
    for (_, bo, _, _), (ro, _) in zip(mlp.LAYOUT, mlp.REAL):
        p[bo:bo + ro] = g.normal(0, 0.1, ro)
    s.master.copy_(torch.from_numpy(p))
    mlp.sdf_mlp_pack(s.master, s.w16)
    return s


@pytest.mark.parametrize("batch", [1, 16, 17, 64, 65, 1000, 3578, 6942, 8192])
def test_backward_at_tile_ends(batch):
    rows = batch + 37
    s = surrogate(batch, 4)
    q = torch.from_numpy(inputs.random_joint_states(rows, 5).astype(np.float32)).to(dev())
    t_np = inputs.rng(6).uniform(0, 40, (rows, 12)).astype(np.float32)
    idx = torch.from_numpy(inputs.rng(7).permutation(rows)[:batch].astype(np.int32)).to(dev())
    s.ws.fill_(0xFF)   # nothing may depend on what the workspace held
    y = torch.empty((batch, 12), dtype=torch.float32, device=dev())
    mlp.sdf_mlp_forward(s.w16, s.master, q, y, s.ws, idx=idx)
    mlp.sdf_mlp_backward(s.w16, torch.from_numpy(t_np).to(dev()), s.grad, s.loss, s.ws, idx=idx, clip_vox=24.0)
    say("[mlp] backward", batch)
    acts = ws_views(s.ws, batch)
    a = [acts["x"][:batch, :14], acts["h1"][:batch], acts["h2"][:batch], acts["h3"][:batch]]
    loss, dy = M.loss_and_dy(y.cpu().numpy().astype(np.float64), t_np[idx.cpu().numpy()].astype(np.float64), clip=24.0)
    assert abs(float(s.loss.item()) - loss) <= 1e-5 * loss
    g = s.grad.cpu().numpy()
    for (wo, bo, nr, nc), (ro, ci), (rdW, rdb) in zip(mlp.LAYOUT, mlp.REAL, M.backward(device_params(s), a, dy)):
        dW, db = g[wo:wo + nr * nc].reshape(nr, nc), g[bo:bo + nr]
        assert (dW[ro:] == 0).all() and (dW[:, ci:] == 0).all() and (db[ro:] == 0).all()
        assert np.abs(dW[:ro, :ci] - rdW).max() <= 2e-3 * np.abs(rdW).max() + 1e-7
        assert np.abs(db[:ro] - rdb).max() <= 2e-3 * np.abs(rdb).max() + 1e-7


@pytest.mark.parametrize("batch", [1, 15, 16, 17, 4097, 8192, 8193, 16384 + 5, 40001])
def test_infer_tiles(batch):
    """Bit for bit the forward pass (in batches the workspace holds), NaN rows
    and the fallback flags among them."""
    s = surrogate(4096, 8)
    q = torch.from_numpy(inputs.random_joint_states(batch, 9).astype(np.float32)).to(dev())
    q[batch // 2, 3] = float("nan")
    y = torch.full((batch, 12), 7.0, dtype=torch.float32, device=dev())
    need = torch.full((batch,), -1, dtype=torch.int32, device=dev())
    radii = torch.full((12,), 0.03, dtype=torch.float32, device=dev())
    eps = torch.linspace(0.0, 2.0, 12, dtype=torch.float32, device=dev())
    say("[mlp] infer", batch)
    mlp.sdf_mlp_infer(s.w16, s.master, q, y, radii, eps, 0.01, 0.05, need)
    ref = torch.empty_like(y)
    for b0 in range(0, batch, 4096):
        mlp.sdf_mlp_forward(s.w16, s.master, q[b0:b0 + 4096], ref[b0:b0 + 4096], s.ws)
    assert torch.isnan(ref[batch // 2]).all()
    ok = torch.arange(batch, device=dev()) != batch // 2
    assert torch.equal(y[ok], ref[ok]) and torch.isnan(y[batch // 2]).all()
    want, count = torch.empty_like(need), torch.empty(1, dtype=torch.int32, device=dev())
    mlp.sdf_mlp_fallback(ref, radii, eps, 0.01, 0.05, want, count)
    assert torch.equal(need, want)
