"""The z pass of lines longer than 256, where a work-group walks over several
tiles: more tiles than CUs, the last tile short, maps of a set gated off
anywhere in a work-group's walk.  Bit for bit against the oracle.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2407_02363_amd import edt, inputs
from tests.gpu_util import dev, grid_of, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes,gates", [
    ([(257, 130, 133)], None),                                             # 271 tiles
    ([(300, 150, 260)], None),                                             # 610
    ([(260, 120, 130), (40, 33, 70), (512, 60, 70)], None),                # a set, 349
    ([(260, 120, 130), (40, 33, 70), (512, 60, 70)], [0, 1, 1]),
    ([(260, 120, 130), (40, 33, 70), (290, 60, 140)], [1, 0, 0]),
])
def test_walk(shapes, gates):
    say("walk", shapes, gates)
    g = inputs.rng(23)
    occs = [(g.random(s) < 0.002).astype(np.uint8) for s in shapes]
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
