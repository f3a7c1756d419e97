"""The branches of the collision, the step counter and the graph chunks inside
the passes of larger lattices: k_pass3d (D3Q19 above 16384 sites) and k_strip2d
(D2Q9 above 64 MB), which hold the collision's coefficients in registers of
their own and count the steps of a pass themselves.  Bit for bit against AA
steps, and k_pass3d on a box of medium size against the FP64 oracle; and the
16-bit cases of the random sweep against AA steps, whatever the default
schedule of their small boxes is."""
import numpy as np
import pytest
import torch

import oracle
import paper_0707_1581_amd as lbf
from tests import test_gpu_random_sweep as sweep
from tests.gpu_util import gpu_pops, oracle_params, say, scaled_err

pytestmark = pytest.mark.gpu

BOXES = [("d3q19", (65, 14, 19)), ("d2q9", (59, 61007, 1))]


def _cfg(lattice, dims, **variant):
    cfg = dict(nx=dims[0], ny=dims[1], nz=dims[2], rho0=1.0, kT=1e-4, gamma_bulk=0.5, gamma_shear=0.8, gamma_odd=-0.3,
               gamma_even=0.2, seed=99, lattice=lattice)
    cfg.update(variant)
    return cfg


def _pair(cfg, storage, t0=0, chunk=16):
    start = lbf.Lattice(**dict(cfg, kT=1e-4), storage=storage, init="thermal")
    lats = [lbf.Lattice(**cfg, storage=storage, init="keep", state=start.state.clone(), t0=t0) for _ in range(2)]
    for lat, fused in zip(lats, (0, 1)):
        lat.set_schedule(block=128, graph_chunk=chunk, fused=fused)
    start.close()
    return lats


def _same(lats, counts):
    for n in counts:
        for lat in lats:
            lat.step(n)
        assert torch.equal(lats[0].state, lats[1].state), (n, lats[0].t)
    for lat in lats:
        lat.close()


@pytest.mark.parametrize("lattice,dims", BOXES)
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("variant", [dict(kT=0.0, gamma_bulk=-0.4, gamma_shear=0.9, gamma_odd=0.0, gamma_even=0.0),
                                     dict(thermal_modes="stress_only", gamma_odd=0.0, gamma_even=0.0),
                                     dict(thermal_modes="stress_only"),
                                     dict(gamma_odd=0.0, gamma_even=0.0),
                                     dict(gamma_bulk=1.0, gamma_shear=-1.0, gamma_odd=1.0, gamma_even=-1.0),
                                     dict(seed=2 ** 40 + 3, rho0=1.7)])
def test_branches_in_the_passes(lattice, dims, storage, variant):
    """From a count that crosses 2^32 inside a pass: the count's high word
    changes between the steps of one launch."""
    if storage == "bf16" and variant.get("kT") == 0.0:
        pytest.skip("bf16 storage is for fluctuating runs")
    _same(_pair(_cfg(lattice, dims, **variant), storage, t0=2 ** 32 - 5), (5, 9, 16))


@pytest.mark.parametrize("start", range(1, 9))
@pytest.mark.parametrize("lattice,dims", BOXES)
def test_counts_cross_2_32_at_every_step_of_a_pass(lattice, dims, start):
    _same(_pair(_cfg(lattice, dims), "f32", t0=2 ** 32 - start), (8,))


@pytest.mark.parametrize("chunk", [2, 4, 6, 8, 30])
@pytest.mark.parametrize("dims", [(65, 14, 19), (129, 27, 10)])
def test_graph_chunks_of_the_tiles(chunk, dims):
    _same(_pair(_cfg("d3q19", dims), "f32", chunk=chunk), (2 * chunk + 1, chunk, 3))


@pytest.mark.parametrize("dims", [(65, 14, 19), (33, 27, 20)])
@pytest.mark.parametrize("kT", [0.0, 1e-4])
def test_tiles_match_oracle(dims, kT):
    cfg = _cfg("d3q19", dims, kT=kT)
    p = oracle_params(cfg)
    init, kind = ("thermal", oracle.INIT_THERMAL) if kT > 0 else ("fields", oracle.INIT_FIELDS)
    f = None
    if kT == 0.0:
        rng = np.random.default_rng(4)
        f = (0.01 * rng.standard_normal((4, *dims[::-1]))).astype(np.float32)
        f[0] += 1.0
    lat = lbf.Lattice(**cfg, storage="f32", init=init, **({} if f is None else {"fields": torch.from_numpy(f)}))
    lat.set_schedule(fused=1)
    n = oracle.init(p, kind, None if f is None else f.astype(np.float64))
    for t, target in ((0, 8), (8, 17)):
        lat.step(target - t)
        n = oracle.run(p, n, t, target - t)
        err = scaled_err(gpu_pops(lat), n, cfg["rho0"])
        say(f"{dims} kT={kT} t={target}: max scaled err {err:.2e}")
        assert err < 1e-5, (target, err)  # the parity bar of the fp32 state
    lat.close()


@pytest.mark.parametrize("k", [k for k in range(sweep.CASES) if sweep._case(k)[1] != "f32"])
@pytest.mark.parametrize("default", [False, True])
def test_random_16_bit_cases_equal_single_steps(k, default):
    cfg, storage, t0, steps, sched, fields = sweep._case(k)
    init = "thermal" if cfg["kT"] > 0 else "fields"
    fkw = {} if fields is None else {"fields": torch.from_numpy(fields)}
    lats = [lbf.Lattice(**cfg, storage=storage, init=init, t0=t0, **fkw) for _ in range(2)]
    if not default:
        lats[0].set_schedule(**sched)
    lats[1].set_schedule(fused=0)
    for lat in lats:
        lat.step(steps)
        lat.step(16)
    assert torch.equal(lats[0].state, lats[1].state)
    for lat in lats:
        lat.close()
