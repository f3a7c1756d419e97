"""Propagation takes the launches of the steps it is the movement floor of, also
on lattices that take several steps per launch before a schedule is set: the
same exact shift, in less time than the steps."""
import pytest
import torch

import oracle
import paper_0707_1581_amd as lbf
from tests.gpu_util import LATTICES, say

pytestmark = pytest.mark.gpu


def _lat(lattice, dims, storage):
    return lbf.Lattice(*dims, kT=1e-4, gamma_shear=0.5, seed=5, init="thermal", lattice=lattice, storage=storage)


@pytest.mark.parametrize("lattice,dims,storage", [("d3q19", (16, 15, 17), "f32"), ("d2q9", (64, 48, 1), "f16"),
                                                  ("d2q9", (701, 699, 1), "f32"), ("d2q9", (3900, 4001, 1), "bf16")])
def test_default_passes_propagate_exactly(lattice, dims, storage):
    lat = _lat(lattice, dims, storage)
    assert lat.schedule()["fused"] == 0
    c = oracle.tables(LATTICES[lattice])[0]
    before = lat.populations().clone()
    for n in (4, 1, 16, 7):
        lat.propagate(n)
        after = lat.populations()
        for i in range(len(c)):
            v = [int(a) for a in c[i]] + [0] * (3 - len(c[i]))
            want = torch.roll(before[i], shifts=tuple(lat.t * v[a] for a in (2, 1, 0)), dims=(0, 1, 2))
            assert torch.equal(after[i], want), (n, i)
    lat.close()


def test_propagation_is_the_floor_of_the_step():
    """701 x 699 fp32 (17.6 MB): 16 steps take 70 to 100 us in blocks, AA
    propagation 120 or more; the launches of the blocks without their
    collisions cannot take longer than the blocks."""
    lat = _lat("d2q9", (701, 699, 1), "f32")
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    best = {}
    for name, call in (("step", lat.step), ("propagate", lat.propagate)):
        for _ in range(9):
            ev[0].record()
            for _ in range(4):
                call(16)
            ev[1].record()
            torch.cuda.synchronize()
            best[name] = min(best.get(name, 1e9), ev[0].elapsed_time(ev[1]))
    say(f"64 steps {1e3 * best['step']:.0f} us, propagation {1e3 * best['propagate']:.0f} us")
    assert best["propagate"] <= 1.05 * best["step"]
    lat.close()
