"""The D2Q9 passes of two, three and four steps at the sizes where they can go
wrong: strips whose width is one site off a multiple of the interior (58, 60
and 62 sites), a box narrower than the halo, the last strip and the last chunk
ragged, step counts that take every combination of passes, an odd start.  Bit
for bit against AA steps (which are pinned to the oracle), and propagation
only as an exact shift.  Long narrow boxes: passes of three and four steps are
taken where a strip walks eight rows or more."""
import numpy as np
import pytest
import torch

import oracle
import paper_0707_1581_amd as lbf

pytestmark = pytest.mark.gpu

# above the 64 MB of state up to which passes take blocks instead, in every storage form
BOXES = [(1, 3600007), (2, 1800011), (58, 62003), (59, 61007), (61, 59009), (117, 31013), (3600011, 1)]


def _cfg(dims, kT=1e-4):
    return dict(nx=dims[0], ny=dims[1], nz=1, rho0=1.0, kT=kT, gamma_bulk=0.5, gamma_shear=0.8, gamma_odd=-0.3,
                gamma_even=0.2, seed=4321, lattice="d2q9")


@pytest.mark.parametrize("dims", BOXES)
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
def test_strips_equal_single_steps(dims, storage):
    a = lbf.Lattice(**_cfg(dims), storage=storage, init="thermal")
    b = lbf.Lattice(**_cfg(dims), storage=storage, init="thermal")
    a.set_schedule(fused=0)
    b.set_schedule(fused=1)
    for n in (4, 6, 8, 1, 13, 20, 34):
        a.step(n)
        b.step(n)
        assert torch.equal(a.state, b.state), (dims, storage, n, a.t)
    a.close()
    b.close()


@pytest.mark.parametrize("dims", [(59, 61007)])
def test_strips_propagate_exactly(dims):
    lat = lbf.Lattice(**_cfg(dims), storage="bf16", init="thermal")
    lat.set_schedule(fused=1)
    c = oracle.tables(oracle.D2Q9)[0]
    before = lat.populations().clone()
    for n in (4, 6, 8, 14):
        lat.propagate(n)
        after = lat.populations()
        for i in range(9):
            want = torch.roll(before[i], shifts=(lat.t * int(c[i, 1]), lat.t * int(c[i, 0])), dims=(1, 2))
            assert torch.equal(after[i], want), (n, i)
    lat.close()


@pytest.mark.parametrize("dims", [(58, 41001)])
@pytest.mark.parametrize("steps", [4, 8])
def test_strips_match_oracle(dims, steps):
    """Noiseless and noisy passes against the oracle at the first and last
    columns and rows (a band of the box evolved alone: its inner rows depend
    on nothing outside it for `steps` steps)."""
    for kT in (0.0, 1e-3):
        cfg = _cfg(dims, kT)
        start = lbf.Lattice(**_cfg(dims, 1e-3), storage="f32", init="thermal")
        lat = lbf.Lattice(**cfg, storage="f32", init="keep", state=start.state.clone())
        lat.set_schedule(fused=1)
        n0 = lat.populations().double().cpu().numpy()
        lat.step(steps)
        got = lat.populations().double().cpu().numpy()
        keys = ("nx", "ny", "nz", "rho0", "kT", "gamma_bulk", "gamma_shear", "gamma_odd", "gamma_even", "seed")
        p = {k: cfg[k] for k in keys}
        if dims[1] > 64:  # the first rows: row 0 is site 0 of the box and of the band alike
            rows = 40
            p["ny"] = rows
            n0, got = n0[:, :, :rows], got[:, :, :rows]
        want = oracle.run(oracle.params(**p, lattice=oracle.D2Q9), np.ascontiguousarray(n0), 0, steps)
        inner = slice(steps, p["ny"] - steps) if dims[1] > 64 else slice(None)
        a = oracle.tables(oracle.D2Q9)[1]
        err = float((np.abs(got - want)[:, :, inner].max(axis=(1, 2, 3)) / a).max())
        assert err < 1e-5, (dims, kT, err)  # the parity bar of the fp32 state
        start.close()
        lat.close()


@pytest.mark.parametrize("storage,dims", [("f16", (4096, 3700)), ("bf16", (3900, 4001)), ("f32", (857, 911)),
                                          ("f32", (1023, 901))])
def test_passes_before_a_schedule_is_set(storage, dims):
    """Lattices that report fused = 0 but take several steps per launch until
    a schedule is set: the bits of single steps, also after a propagation and
    once a schedule has been set."""
    lats = [lbf.Lattice(dims[0], dims[1], 1, lattice="d2q9", storage=storage, kT=1e-4, gamma_bulk=0.5,
                        gamma_shear=0.8, seed=11, init="thermal", t0=3) for _ in range(2)]
    assert lats[0].schedule()["fused"] == 0
    lats[1].set_schedule(fused=0)
    for n in (4, 1, 19, 32, 7):
        for lat in lats:
            lat.step(n)
        assert torch.equal(lats[0].state, lats[1].state), n
    for lat in lats:
        lat.propagate(3)
        lat.step(6)
    assert torch.equal(lats[0].state, lats[1].state)
    lats[0].set_schedule(fused=0)
    for lat in lats:
        lat.step(17)
    assert torch.equal(lats[0].state, lats[1].state)
    for lat in lats:
        lat.close()


@pytest.mark.parametrize("storage,dims", [("f32", (3001, 3011)), ("f32", (59, 153001)), ("f32", (200003, 47)),
                                          ("f32", (61, 70001)), ("f32", (2111, 1999)),
                                          ("f16", (4801, 3903)), ("bf16", (117, 160001))])
def test_strips_in_step(storage, dims):
    """State whose strips walk in step (beyond the Infinity Cache, and passes of
    two fp32 steps from 140 MB on): ragged last strips, chunks and workgroups,
    workgroups over several chunks, passes of two, three and four steps."""
    lats = [lbf.Lattice(**_cfg(dims), storage=storage, init="thermal") for _ in range(2)]
    lats[0].set_schedule(fused=1)
    lats[1].set_schedule(fused=0)
    for n in (4, 6, 8, 21):
        for lat in lats:
            lat.step(n)
        assert torch.equal(lats[0].state, lats[1].state), n
    for lat in lats:
        lat.close()
