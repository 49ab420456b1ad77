"""Maps whose rows are of one tile (up to 64 columns), which the xy search reads
from the occupancy bytes: row lengths and counts around the ends of words, bands
and work-groups, maps of a few voxels, occupancy at every offset from 16 bytes
with occupied bytes right before and after it, sets with idle bands and gated
maps, and a set that holds one wider row (read from bits).  Integers throughout:
nothing may differ from the oracle.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2407_02363_amd import edt, inputs
from tests.gpu_util import dev, gpu_edt, grid_of, say

pytestmark = pytest.mark.gpu

# (nz, ny, nx)
SHAPES = [(1, 1, 1), (2, 2, 2), (1, 1, 15), (1, 1, 16), (1, 1, 64), (3, 7, 1), (5, 8, 31), (4, 9, 32), (6, 16, 33),
          (70, 31, 63), (3, 33, 64), (2, 65, 5), (9, 129, 48), (2, 257, 64), (3, 512, 17), (300, 4, 40)]


def scene(shape, density, seed):
    occ = (inputs.rng(seed).random(shape) < density).astype(np.uint8) * 255
    if density > 0:
        occ[tuple(int(v) for v in inputs.rng(seed + 1).integers(0, shape))] = 1
    return occ


@pytest.mark.parametrize("density", [0.0, 1e-9, 0.02, 0.5, 1.0])
@pytest.mark.parametrize("shape", SHAPES)
def test_narrow_maps(shape, density):
    occ = scene(shape, density, 17 + SHAPES.index(shape))
    rd2, rsite = oracle.edt(occ)
    for off in (0, 1, 7, 15):
        d2, site = gpu_edt(occ, occ_offset=off)
        assert np.array_equal(d2, rd2) and np.array_equal(site, rsite), off


@pytest.mark.parametrize("off", range(16))
def test_every_offset(off):
    """The last voxels of an allocation too: the buffer ends with the map."""
    for shape in [(3, 37, 61), (1, 3, 5)]:
        occ = scene(shape, 0.03, off)
        buf = torch.full((off + occ.size,), 0xFF, dtype=torch.uint8, device=dev())
        buf[off:] = torch.from_numpy(occ.ravel()).to(dev())
        d2, site = (torch.full((occ.size,), -7, dtype=torch.int32, device=dev()) for _ in range(2))
        edt.edt_compute(grid_of(shape), buf[off:], d2, site)
        rd2, rsite = oracle.edt(occ)
        assert np.array_equal(d2.cpu().numpy().reshape(shape), rd2)
        assert np.array_equal(site.cpu().numpy().reshape(shape), rsite)


@pytest.mark.parametrize("wider", [0, 1, 3])
@pytest.mark.parametrize("gated", [False, True])
def test_sets(gated, wider):
    shapes = [(9, 200, 60), (130, 4, 9), (64, 64, 64), (1, 1, 8), (40, 100, 33)]
    if wider == 1:      # one map read from bits, behind and before others
        shapes = [(1, 1, 1), (20, 30, 65)] + shapes
    elif wider == 3:
        shapes = [(4, 9, 300), (3, 3, 3), (64, 64, 65)] + shapes + [(128, 20, 129)]
    gates = [(i + i // 3) % 2 for i in range(len(shapes))]
    say("narrow set", shapes, gated)
    occs = [scene(s, 0.01, 5 + i) for i, s in enumerate(shapes)]
    o = [torch.from_numpy(x.ravel()).to(dev()) for x in occs]
    d2 = [torch.full((x.size,), -7, dtype=torch.int32, device=dev()) for x in occs]
    site = [torch.full((x.size,), -7, dtype=torch.int32, device=dev()) for x in occs]
    maps = edt.batch_maps([grid_of(s) for s in shapes], o, d2, site)
    if gated:
        edt.edt_compute_many_gated(maps, torch.tensor(gates, dtype=torch.int32, device=dev()))
    else:
        edt.edt_compute_many(maps)
    for i, x in enumerate(occs):
        a, b = d2[i].cpu().numpy().reshape(x.shape), site[i].cpu().numpy().reshape(x.shape)
        if gated and not gates[i]:
            assert (a == -7).all() and (b == -7).all()
        else:
            ref = oracle.edt(x)
            assert np.array_equal(a, ref[0]) and np.array_equal(b, ref[1])


@pytest.mark.parametrize("shape", [(1, 1, 3), (7, 40, 64), (7, 40, 65), (5, 30, 200)])
def test_xy_stage_without_d2(shape):
    """The xy stage takes a NULL d2: the packed 2D sites are those it gives with
    one, and finish to the transform."""
    import ctypes
    g = edt.make_grid(grid_of(shape))
    occ = scene(shape, 0.02, 3)
    n = occ.size
    o = torch.from_numpy(occ.ravel()).to(dev())
    a, b, d2 = (torch.full((n,), -7, dtype=torch.int32, device=dev()) for _ in range(3))
    rc = edt.lib().edt_compute_stage(ctypes.byref(g), ctypes.c_void_p(o.data_ptr()), None,
                                     ctypes.c_void_p(a.data_ptr()), edt.STAGE_XY, None, edt._stream(None))
    assert rc == 0
    edt.edt_compute_stage(g, o, d2, b, edt.STAGE_XY)
    assert torch.equal(a, b)
    edt.edt_compute_stage(g, o, d2, a, edt.STAGE_Z)
    rd2, rsite = oracle.edt(occ)
    assert np.array_equal(d2.cpu().numpy().reshape(shape), rd2) and np.array_equal(a.cpu().numpy().reshape(shape), rsite)
