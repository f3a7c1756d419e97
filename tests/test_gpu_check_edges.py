"""lb_check's reduction at the edges of its grid (a workgroup of 256 sites, 2048
workgroups) and its test for bad sites in every position of the state: sums
against numpy, one planted infinity, NaN or negative density at a time."""
import numpy as np
import pytest
import torch

import paper_0707_1581_amd as lbf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(1, 1, 1), (5, 3, 17), (16, 16, 1), (257, 1, 1), (64, 64, 128), (524289, 1, 1)])
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
def test_sums(dims, storage):
    lat = lbf.Lattice(*dims, storage=storage, kT=1e-3, gamma_shear=0.5, seed=3, init="thermal")
    for n in (0, 1):
        lat.step(n)
        bad, sums = lat.check()
        m = lat.moments().double().cpu().numpy().reshape(4, -1)
        assert bad == 0
        # every site's rho and j are rounded once more in fp32 by the gather
        tol = 2.0 ** -24 * np.abs(m).sum(axis=1) + 1e-12
        assert np.all(np.abs(np.asarray(sums) - m.sum(axis=1)) <= tol), (sums, m.sum(axis=1))
    lat.close()


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
def test_one_bad_population(value, storage):
    dims = (33, 17, 5)
    lat = lbf.Lattice(*dims, storage=storage, kT=1e-4, gamma_shear=0.5, seed=3, init="thermal")
    for i, z, y, x in [(0, 0, 0, 0), (7, 2, 9, 11), (18, 4, 16, 32), (5, 4, 0, 31)]:
        keep = lat.state[i, z, y, x].clone()
        lat.state[i, z, y, x] = value
        assert lat.check()[0] == 1, (i, z, y, x)
        lat.state[i, z, y, x] = keep
    assert lat.check()[0] == 0
    lat.state[:, 1, 2, 3] = -1.5  # finite, rho < 0
    assert lat.check()[0] == 1
    big = torch.finfo(lat.state.dtype).max
    lat.state[:, 1, 2, 3] = 0
    lat.state[0, 1, 2, 3] = big if storage == "f16" else 1e30  # finite and large, rho > 0
    assert lat.check()[0] == 0
    lat.close()
