"""The FP32 120 x 20 step of up to 768 tiles and of more: two forms of one
kernel, the same bits as any other tile shape."""
from __future__ import annotations

import pytest
import torch

from paper_1102_1343_amd import fire as F

from test_gpu_small import _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(1440, 1280), (1440, 1281), (961, 780)])
def test_few_tiles_and_more_equal_another_shape(nx, ny):
    """768 tiles, 780, and a ragged mesh of 351."""
    prob = _problem(nx, ny, 10, 10)
    u, v = (torch.from_numpy(a).to("cuda", torch.float32) for a in prob.wind[0])
    res = []
    for tile in (None, (60, 10)):
        f = F.Fire.from_problem(prob, dtype=torch.float32)
        if tile:
            f.set_tile(*tile)
        for _ in range(6):
            out = f.step(u, v, prob.dt)
        res.append([f.psi.clone(), f.tign.clone(), f.frac.clone(), *out])
        st = f.status()
    for name, a, b in zip(("psi", "tign", "frac", "sens", "lat"), *res):
        assert torch.equal(a, b), name
    assert bool((res[0][2] < 1).any()) and st & F.STATUS_BOUNDARY
