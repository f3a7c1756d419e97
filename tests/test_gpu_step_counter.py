"""The device's step counter over every kind of run: runs of one launch and of
many, odd and even, from odd and even counts beyond 2^32, and runs that a
caller captures into a graph of its own and replays between eager steps (each
replay goes on from where the counter is).  The populations depend on the
count through the noise, so they are compared, bit for bit, with one call."""
import pytest
import torch

import paper_0707_1581_amd as lbf

pytestmark = pytest.mark.gpu


def _lat(lattice, dims, t0, fused=None, stream=None):
    lat = lbf.Lattice(*dims, storage="f32", kT=1e-4, gamma_shear=0.8, seed=5, init="thermal", t0=t0, lattice=lattice,
                      stream=stream)
    if fused is not None:
        lat.set_schedule(fused=fused, block=64)
    return lat


@pytest.mark.parametrize("lattice,dims", [("d3q19", (9, 8, 7)), ("d2q9", (40, 33, 1))])
@pytest.mark.parametrize("t0", [0, 2 ** 32 - 7])
@pytest.mark.parametrize("fused", [None, 0, 1])
def test_runs_add_up(lattice, dims, t0, fused):
    a, b = (_lat(lattice, dims, t0, fused) for _ in range(2))
    for n in (1, 1, 2, 3, 1, 5, 16, 1, 33, 4, 7):
        a.step(n)
    b.step(a.t - t0)
    assert a.t == b.t and torch.equal(a.state, b.state)
    a.propagate(3)
    a.step(2)
    b.propagate(1)
    b.propagate(2)
    b.step(1)
    b.step(1)
    assert torch.equal(a.state, b.state)
    a.close()
    b.close()


@pytest.mark.parametrize("steps", [(2,), (4,), (1, 1), (3, 5)])
def test_captured_runs_go_on(steps):
    dims = (9, 8, 7)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        lat = _lat("d3q19", dims, 0, 0, side)
        lat.step(2)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        for n in steps:
            lat.step(n)
    ref = _lat("d3q19", dims, 0, 0)
    done = 2
    with torch.cuda.stream(side):
        for k in range(4):
            graph.replay()
            done += sum(steps)
            torch.cuda.synchronize()
            for n in (1, 3, 2, 16)[:k]:
                lat.step(n)
                done += n
            if k % 2:  # back to the parity that the graph was captured at
                lat.step(1)
                done += 1
            torch.cuda.synchronize()
            if done % 2:
                lat.step(1)
                done += 1
                torch.cuda.synchronize()
            ref.step(done - ref.t)
            torch.cuda.synchronize()
            assert torch.equal(lat.state, ref.state), k
    lat.close()
    ref.close()
