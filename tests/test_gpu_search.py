"""The search tiles (every axis up to 512) at the sizes where they can go
wrong, bit for bit against the oracle: the ends of blocks (8 positions),
bands (8, 16, 32), groups and work-group sizes (64, 128, 256, 512 positions),
tiles of 64 columns, maps too small for the bits; maps with one site, sites far
apart (the bounds by groups), dense maps (the bounds by neighbours), no site.
Integers throughout: nothing may differ.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2407_02363_amd import edt, inputs
from tests.gpu_util import dev, gpu_edt, grid_of, say

pytestmark = pytest.mark.gpu

# (nz, ny, nx)
SHAPES = [(1, 1, 8), (8, 8, 7), (9, 7, 9), (64, 64, 64), (65, 63, 65), (3, 128, 63), (128, 3, 130), (129, 17, 20),
          (5, 129, 40), (256, 5, 66), (7, 256, 70), (257, 9, 33), (4, 257, 72), (512, 6, 30), (3, 512, 68),
          (2, 5, 512), (31, 33, 257)]


def scene(kind, shape, seed):
    g = inputs.rng(seed)
    occ = np.zeros(shape, np.uint8)
    if kind == "one":
        occ[tuple(int(g.integers(0, n)) for n in shape)] = 1
    elif kind == "far":          # a few sites: distances across the map
        for _ in range(5):
            occ[tuple(int(g.integers(0, n)) for n in shape)] = 255
    elif kind == "corners":      # the largest distances, many ties
        occ[np.ix_(*[[0, n - 1] for n in shape])] = 1
    elif kind == "half":         # sites in one half of every axis only
        occ[tuple(slice(0, (n + 1) // 2) for n in shape)] = (
            g.random(tuple((n + 1) // 2 for n in shape)) < 0.03).astype(np.uint8)
    elif kind == "dense":
        occ = (g.random(shape) < 0.2).astype(np.uint8)
    return occ


@pytest.mark.parametrize("kind", ["one", "far", "corners", "half", "dense", "empty"])
@pytest.mark.parametrize("shape", SHAPES)
def test_search_tiles(shape, kind):
    occ = scene(kind, shape, 11 + SHAPES.index(shape))
    d2, site = gpu_edt(occ)
    rd2, rsite = oracle.edt(occ)
    assert np.array_equal(d2, rd2) and np.array_equal(site, rsite)


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_outputs_off_16_bytes(shift):
    """The occupancy bits stay inside d2, wherever it starts, also for the
    smallest maps that hold them."""
    for shape in [(3, 5, 8), (20, 33, 70)]:
        occ = scene("half", shape, 3)
        n = occ.size
        buf = torch.full((2, n + 8), -7, dtype=torch.int32, device=dev())
        d2, site = buf[0, shift:shift + n], buf[1, shift:shift + n]
        edt.edt_compute(grid_of(shape), torch.from_numpy(occ.ravel()).to(dev()), d2, site)
        got = buf.cpu().numpy()
        rd2, rsite = oracle.edt(occ)
        assert np.array_equal(got[0, shift:shift + n].reshape(shape), rd2)
        assert np.array_equal(got[1, shift:shift + n].reshape(shape), rsite)
        assert (got[:, :shift] == -7).all() and (got[:, shift + n:] == -7).all()


def test_many_maps_of_mixed_lengths():
    """One launch whose longest lines exceed most maps' (idle bands), some
    maps gated off."""
    shapes = [(9, 200, 70), (130, 4, 9), (64, 64, 64), (1, 1, 8), (40, 100, 200)]
    say("many", shapes)
    for gates in (None, [1, 0, 1, 1, 0]):
        occs = [scene("half", s, 5 + i) for i, s in enumerate(shapes)]
        o = [torch.from_numpy(x.ravel()).to(dev()) for x in occs]
        d2 = [torch.full((x.size,), -7, dtype=torch.int32, device=dev()) for x in occs]
        site = [torch.full((x.size,), -7, dtype=torch.int32, device=dev()) for x in occs]
        maps = edt.batch_maps([grid_of(s) for s in shapes], o, d2, site)
        if gates is None:
            edt.edt_compute_many(maps)
        else:
            edt.edt_compute_many_gated(maps, torch.tensor(gates, dtype=torch.int32, device=dev()))
        for i, x in enumerate(occs):
            got = d2[i].cpu().numpy().reshape(x.shape), site[i].cpu().numpy().reshape(x.shape)
            if gates is not None and not gates[i]:
                assert (got[0] == -7).all() and (got[1] == -7).all()
                continue
            ref = oracle.edt(x)
            assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])


def test_same_as_the_general_tiles():
    """The general tiles (any explicit tuning) give the same bits."""
    g = inputs.rng(17)
    for _ in range(12):
        shape = tuple(int(g.integers(lo, hi)) for lo, hi in ((1, 140), (1, 140), (8, 200)))
        kind = ["one", "far", "corners", "half", "dense"][int(g.integers(0, 5))]
        occ = torch.from_numpy(scene(kind, shape, int(g.integers(0, 1 << 20))).ravel()).to(dev())
        out = [torch.empty(occ.numel(), dtype=torch.int32, device=dev()) for _ in range(4)]
        edt.edt_compute(grid_of(shape), occ, out[0], out[1])
        edt.edt_compute_tuned(grid_of(shape), occ, out[2], out[3], (16, 16, 64, 64))
        assert torch.equal(out[0], out[2]) and torch.equal(out[1], out[3]), (shape, kind)
