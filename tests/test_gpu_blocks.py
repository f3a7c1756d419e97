"""Small lattices take several steps per launch in blocks with a halo
(k_block), by default and under the fused schedule: bit for bit against AA
steps, which are pinned to the oracle, at the edges of the blocks (4^3; 8 x 8,
16 x 16 and 58 x 10), at both ends of the range of sizes, on boxes narrower than
the halo, for step counts that take passes of every length."""
import pytest
import torch

import oracle
import paper_0707_1581_amd as lbf

pytestmark = pytest.mark.gpu

BOXES = {"d3q19": [(1, 1, 1), (2, 1, 3), (4, 4, 4), (5, 4, 3), (8, 9, 7), (16, 16, 16), (25, 25, 26)],
         "d2q9": [(1, 1), (3, 2), (8, 8), (9, 7), (64, 48), (65, 49), (130, 131), (257, 300), (580, 101), (666, 665)]}
CASES = [(lat, d) for lat in BOXES for d in BOXES[lat]]


def _cfg(lattice, dims, kT):
    return dict(nx=dims[0], ny=dims[1], nz=dims[2] if lattice == "d3q19" else 1, rho0=1.0, kT=kT, gamma_bulk=0.5,
                gamma_shear=0.8, gamma_odd=-0.3, gamma_even=0.2, seed=2 ** 33 + 5, lattice=lattice)


@pytest.mark.parametrize("lattice,dims", CASES)
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
def test_blocks_equal_single_steps(lattice, dims, storage):
    t0 = 2 ** 32 - 20
    lats = [lbf.Lattice(**_cfg(lattice, dims, 1e-4), storage=storage, init="thermal", t0=t0) for _ in range(3)]
    assert lats[0].schedule()["fused"] == 0
    lats[1].set_schedule(fused=0)
    lats[2].set_schedule(fused=1)
    for n in (4, 6, 8, 10, 1, 2, 3, 16, 35, 100):
        for lat in lats:
            lat.step(n)
        assert torch.equal(lats[0].state, lats[1].state), ("default", n)
        assert torch.equal(lats[2].state, lats[1].state), ("fused", n)
    for lat in lats:
        lat.close()


@pytest.mark.parametrize("lattice,dims", [("d3q19", (8, 9, 7)), ("d2q9", (65, 49))])
def test_blocks_noiseless(lattice, dims):
    start = lbf.Lattice(**_cfg(lattice, dims, 1e-3), storage="f32", init="thermal")
    lats = [lbf.Lattice(**_cfg(lattice, dims, 0.0), storage="f32", init="keep", state=start.state.clone())
            for _ in range(2)]
    lats[1].set_schedule(fused=0)
    for lat in lats:
        lat.step(23)
    assert torch.equal(lats[0].state, lats[1].state)
    for lat in lats + [start]:
        lat.close()


@pytest.mark.parametrize("lattice,dims", [("d3q19", (9, 5, 6)), ("d2q9", (65, 49))])
def test_blocks_propagate_exactly(lattice, dims):
    lat = lbf.Lattice(**_cfg(lattice, dims, 1e-4), storage="f16", init="thermal")
    lat.set_schedule(fused=1)
    c = oracle.tables(oracle.D2Q9 if lattice == "d2q9" else oracle.D3Q19)[0]
    before = lat.populations().clone()
    for n in (4, 6, 8, 16):
        lat.propagate(n)
        after = lat.populations()
        for i in range(len(c)):
            v = [int(a) for a in c[i]] + [0] * (3 - len(c[i]))
            want = torch.roll(before[i], shifts=tuple(lat.t * v[a] for a in (2, 1, 0)), dims=(0, 1, 2))
            assert torch.equal(after[i], want), (n, i)
    lat.close()
