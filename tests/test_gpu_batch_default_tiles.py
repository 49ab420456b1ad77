"""The tiles a persistent batch takes by itself: the kernel that runs, by its
name, and its results against the oracle, on either side of every line of the
rule (192 and 320 slices, 320 rows) and for a batch the lean tiles take.
"""
import numpy as np
import pytest
import torch

from paper_2407_02363_amd import edt, inputs
from tests.gpu_util import dev, grid_of, say

pytestmark = pytest.mark.gpu


def batch(shapes, seed):
    occs = [inputs.random_grid(s, 0.01, seed + i) for i, s in enumerate(shapes)]
    o = [torch.from_numpy(np.ascontiguousarray(x).ravel()).to(dev()) for x in occs]
    d2 = [torch.full((x.size,), -7, dtype=torch.int32, device=dev()) for x in occs]
    st = [torch.full((x.size,), -7, dtype=torch.int32, device=dev()) for x in occs]
    return occs, edt.batch_maps([grid_of(s) for s in shapes], o, d2, st), (o, d2, st)


def launched(fn):
    """Names of the library's persistent kernels that fn launches."""
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as p:
        fn()
        torch.cuda.synchronize()
    return [e.name for e in p.events() if "k_edt_batched" in e.name]


@pytest.mark.parametrize("shapes,kernel", [
    ([(192, 20, 40), (5, 30, 33)], "k_edt_batched<32, 64>"),
    ([(193, 20, 40), (5, 30, 33)], "k_edt_batched<32, 32>"),
    ([(320, 20, 40)], "k_edt_batched<32, 32>"),
    ([(321, 20, 40), (2, 320, 9)], "k_edt_batched<32, 16>"),
    ([(321, 20, 40), (2, 321, 9)], "k_edt_batched<32, 32>"),
    ([(512, 16, 20)], "k_edt_batched<32, 16>"),
    ([(4, 512, 64), (128, 9, 64)], "k_edt_batched<32, 64>"),
    ([(128, 30, 64), (9, 256, 70)], "k_edt_batched_lean"),
])
def test_default_tiles(oracle_lib, shapes, kernel):
    say("default batch tiles", shapes)
    occs, maps, (o, d2, st) = batch(shapes, 40)
    ws = edt.new_batch_workspace(len(shapes), dev())
    edt.edt_tuning_cache_clear()
    names = launched(lambda: edt.edt_compute_batched(maps, ws))
    assert len(names) == 1 and kernel in names[0], names
    assert not edt.edt_batch_status(ws)
    for x, a, b in zip(occs, d2, st):
        rd2, rsite = oracle_lib.edt(x)
        assert np.array_equal(a.cpu().numpy().reshape(x.shape), rd2)
        assert np.array_equal(b.cpu().numpy().reshape(x.shape), rsite)


@pytest.mark.parametrize("shape", [(20, 257, 64), (30, 30, 63), (129, 20, 64), (257, 300, 9), (2, 2, 2), (64, 64, 64)])
def test_the_default_tuning_of_a_map_serves_a_batch(oracle_lib, shape):
    """What edt_default_tuning answers for a map is accepted for a batch of
    such maps, with and without a workspace; 64 / 64 without the groups stays
    the lean tiles, refused past their limits."""
    say("batch with the map's tuning", shape)
    nz, ny, nx = shape
    tiles = edt.edt_default_tuning(grid_of(shape))
    occs, maps, (o, d2, st) = batch([shape] * 3, 60)
    ws = edt.new_batch_workspace(3, dev())
    refs = [oracle_lib.edt(x) for x in occs]
    for call in (lambda: edt.edt_compute_batched(maps, ws, tiles), lambda: edt.edt_compute_batched_noalloc(maps, tiles)):
        for a in d2 + st:
            a.fill_(-7)
        call()
        torch.cuda.synchronize()
        for x, a, b, (rd2, rsite) in zip(occs, d2, st, refs):
            assert np.array_equal(a.cpu().numpy().reshape(x.shape), rd2)
            assert np.array_equal(b.cpu().numpy().reshape(x.shape), rsite)
    if nx >= 64 and ny <= 256 and nz <= 128:
        edt.edt_compute_batched(maps, ws, (64, 64))
    else:
        for refused in ((64, 64), (64, 64, 256, 256)):
            with pytest.raises(edt.EdtError) as e:
                edt.edt_compute_batched(maps, ws, refused)
            assert e.value.status == -5
