"""The collision leaves the kinetic modes' forward transform out when both
kinetic rates are zero: every combination of zero and non-zero kinetic rates,
with and without noise and on both lattices, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
import paper_0707_1581_amd as lbf
from tests.gpu_util import gpu_pops

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lattice,dims", [("d3q19", (7, 6, 5)), ("d2q9", (13, 11, 1))])
@pytest.mark.parametrize("rates", [(0.0, 0.0), (0.3, 0.0), (0.0, -0.2), (-1.0, 1.0)])
@pytest.mark.parametrize("kT", [0.0, 1e-3])
def test_kinetic_rates_match_oracle(lattice, dims, rates, kT):
    cfg = dict(nx=dims[0], ny=dims[1], nz=dims[2], rho0=1.0, kT=kT, gamma_bulk=0.5, gamma_shear=0.8,
               gamma_odd=rates[0], gamma_even=rates[1], seed=77)
    # a start whose kinetic modes are away from zero: the thermal state at kT = 1e-3
    a = oracle.D2Q9 if lattice == "d2q9" else oracle.D3Q19
    start = lbf.Lattice(**dict(cfg, kT=1e-3), storage="f32", init="thermal", lattice=lattice)
    lat = lbf.Lattice(**cfg, storage="f32", init="keep", lattice=lattice, state=start.state.clone())
    n = oracle.init(oracle.params(**dict(cfg, kT=1e-3), lattice=a), oracle.INIT_THERMAL)
    lat.step(5)
    want = oracle.run(oracle.params(**cfg, lattice=a), n, 0, 5)
    weights = oracle.tables(a)[1]
    err = float((np.abs(gpu_pops(lat) - want).max(axis=(1, 2, 3)) / (weights * cfg["rho0"])).max())
    assert err < 1e-5, err  # the parity bar of the fp32 state
    start.close()
    lat.close()
