"""Host-side replay of the passes of several steps: the D3Q19 tiles that walk z
(k_pass3d), the D2Q9 strips that walk y (k_strip2d) and the blocks of small
lattices (k_block).

Lane by lane and phase by phase, with the kernels' own index arithmetic, tile
sizes and delays: what each lane loads, the site and step it collides for, the
neighbour it takes a population from (LDS planes in the kernel's layout, lane
shifts), the phases a population waits, and what each lane stores.  The
collision is a stand-in that mixes every population of a site with the site,
the step and the population's number, in wrapping integers: the result equals
so many steps of collide and stream only if every value came from the right
site at the right step and every collision was given its own.  Places that
nothing has written hold a poison.  Every value of the destination must be
written, once.  The compiled kernels are compared with single steps and the
oracle in the GPU tests."""
import os
import re

import numpy as np
import pytest

import oracle
from paper_0707_1581_amd import build

C3 = np.asarray(oracle.tables(oracle.D3Q19)[0], dtype=int)
C2 = np.asarray(oracle.tables(oracle.D2Q9)[0], dtype=int)
C2 = np.hstack([C2, np.zeros((9, 1), dtype=int)]) if C2.shape[1] == 2 else C2
POISON = np.uint64(0xDEADBEEFDEADBEEF)


def _constants(header):
    text = open(os.path.join(build.HERE, "csrc", header)).read()
    return {m.group(1): int(m.group(2)) for m in re.finditer(r"\b(P3_T[XY]) = (\d+)", text)}


P3 = _constants("lbf_pass3d.h")
TX, TY = P3["P3_TX"], P3["P3_TY"]
ROW, PLANE, PAD = TX + 2, (TX + 2) * (TY + 2), TX + 3


def collide(d, site, t):
    """(q, n) populations of the n sites at step t."""
    i = np.arange(d.shape[0], dtype=np.uint64)[:, None]
    with np.errstate(over="ignore"):
        key = np.asarray(site).astype(np.uint64) * np.uint64(0x9E3779B97F4A7C15) + np.uint64(t) * np.uint64(0xBF58476D1CE4E5B9)
        return (d * np.uint64(0x94D049BB133111EB) + d.sum(0, dtype=np.uint64) * np.uint64(0xD6E8FEB86659FD93)
                + key * (np.uint64(2) * i + np.uint64(1)))


def steps(state, c, t, k):
    """k steps of collide and push on (q, nz, ny, nx)."""
    q, nz, ny, nx = state.shape
    for s in range(k):
        post = collide(state.reshape(q, -1), np.arange(nx * ny * nz), t + s).reshape(state.shape)
        state = np.stack([np.roll(post[i], (c[i, 2], c[i, 1], c[i, 0]), (0, 1, 2)) for i in range(q)])
    return state


def start(c, dims, seed=3):
    nx, ny, nz = dims
    return np.random.default_rng(seed).integers(0, 2 ** 63, size=(len(c), nz, ny, nx), dtype=np.uint64)


class Out:
    def __init__(self, like):
        self.data = np.full_like(like, POISON)
        self.count = np.zeros(like.shape, dtype=int)

    def put(self, i, z, y, x, v):
        np.add.at(self.count[i], (z, y, x), 1)
        self.data[i, z, y, x] = v

    def done(self):
        assert (self.count == 1).all()
        return self.data


# ---------------------------------------------------------------- k_pass3d
MOVES = [int(bool(c[0] or c[1])) for c in C3]
SLOT = np.concatenate([[0], np.cumsum(MOVES)[:-1]])
ZIDX = [sum(1 for j in range(i) if C3[j, 2] == C3[i, 2]) for i in range(19)]


def pass3d(src, t, ty, zlen, pull, own):
    q, nz, ny, nx = src.shape
    out = Out(src)
    w, lane = (a.ravel() for a in np.meshgrid(np.arange(ty + 3), np.arange(64), indexing="ij"))
    inner = w < ty
    for z0 in range(0, nz, zlen):
        for y0 in range(0, ny, ty):
            for x0 in range(0, nx, TX):
                tw, th, zc_n = min(TX, nx - x0), min(ty, ny - y0), min(zlen, nz - z0)
                cols = w == ty + 2
                assert th + 2 <= 32 and tw <= 64  # the column wave's lanes cover both halo columns
                lx = np.where(cols, np.where(lane < 32, 0, tw + 1), lane + 1)
                ly = np.where(cols, lane & 31, np.where(w == ty, 0, np.where(w == ty + 1, th + 1, w + 1)))
                mine = (w < th) & (lane < tw)
                lx, ly = np.minimum(lx, tw + 1), np.minimum(ly, th + 1)
                pos = ly * ROW + lx
                gx, gy = x0 + lx, y0 + ly
                x = np.where(gx == 0, nx - 1, np.where(gx > nx, gx - nx - 1, gx - 1))
                y = np.where(gy == 0, ny - 1, np.where(gy > ny, gy - ny - 1, gy - 1))
                lds = np.full(2 * PAD + 2 * 16 * PLANE, POISON, dtype=np.uint64)
                flat = np.full((9, len(w)), POISON)
                ua, ub = np.full((5, len(w)), POISON), np.full((5, len(w)), POISON)
                zc = zprev = (z0 - 1) % nz
                for it in range(zc_n + 2):
                    v = np.stack([src[i, (zc - pull * C3[i, 2]) % nz, (y - pull * C3[i, 1]) % ny,
                                      (x - pull * C3[i, 0]) % nx] for i in range(q)])
                    post = collide(v, x + nx * (y + ny * zc), t)
                    base, following = (PAD + (p & 1) * 16 * PLANE + pos for p in (it, it + 1))
                    for i in range(q):
                        if MOVES[i]:
                            lds[base + SLOT[i] * PLANE] = post[i]
                    for i in range(q):  # past the one barrier, a faster wave may write the next phase's already
                        if MOVES[i]:
                            lds[following + SLOT[i] * PLANE] = POISON
                    h, now = np.empty_like(post), np.empty_like(post)
                    for i in range(q):
                        now[i] = lds[base + SLOT[i] * PLANE - C3[i, 1] * ROW - C3[i, 0]] if MOVES[i] else post[i]
                        k = ZIDX[i]
                        h[i] = now[i] if C3[i, 2] < 0 else (flat[k] if C3[i, 2] == 0 else ua[k])
                    if it >= 2:
                        h = collide(h, x + nx * (y + ny * zprev), t + 1)
                        on = mine & inner
                        for i in range(q):
                            m = 0 if own else 1
                            out.put(i, (zprev + m * C3[i, 2]) % nz, (y[on] + m * C3[i, 1]) % ny,
                                    (x[on] + m * C3[i, 0]) % nx, h[i][on])
                    for i in range(q):
                        if C3[i, 2] == 0:
                            flat[ZIDX[i]] = now[i]
                        elif C3[i, 2] > 0:
                            ua[ZIDX[i]], ub[ZIDX[i]] = ub[ZIDX[i]], now[i]
                    zprev, zc = zc, (zc + 1) % nz
    return out.done()


@pytest.mark.parametrize("dims,ty,zlen", [((64, 13, 5), 13, 5), ((65, 14, 7), 7, 3), ((3, 27, 4), 9, 8), ((1, 1, 1), 1, 8),
                                          ((130, 5, 3), 5, 2), ((2, 2, 9), 2, 4), ((70, 40, 2), 10, 16)])
def test_tiles_take_two_steps(dims, ty, zlen):
    """Chains of two and of four passes: the first reads streamed populations
    and stores them at their own sites, those between pull and store there, the
    last pulls and pushes."""
    a = start(C3, dims)
    for chain in (2, 4):
        s = a
        for n in range(chain):
            s = pass3d(s, 10 + 2 * n, ty, zlen, int(n > 0), n + 1 < chain)
        assert np.array_equal(s, steps(a, C3, 10, 2 * chain)), chain


# ---------------------------------------------------------------- k_strip2d
YIDX = [sum(1 for j in range(i) if C2[j, 1] == C2[i, 1]) for i in range(9)]


def strip2d(src, t, K, rows):
    q, _, ny, nx = src.shape
    out = Out(src)
    halo = K - 1
    ntx = -(-nx // (64 - 2 * halo))
    tx = -(-nx // ntx)
    lane = np.arange(64)
    for y0 in range(0, ny, rows):
        for x0 in range(0, nx, tx):
            tw, yc = min(tx, nx - x0), min(rows, ny - y0)
            col = np.minimum(lane, tw + 2 * halo - 1)
            mine = (lane >= halo) & (lane < halo + tw)
            hx, hy = halo % nx, halo % ny
            x = (x0 + col - hx if x0 >= hx else np.where(x0 + col >= hx, x0 + col - hx, x0 + col + nx - hx)) % nx
            flat, ua, ub = (np.full((halo, 3, 64), POISON) for _ in range(3))
            yr = [y0 - hy if y0 >= hy else y0 + ny - hy] * K
            for it in range(rows + 2 * halo):  # past yc + 2 halo: the loop of a longer strip, without effect
                h = src[:, 0, yr[0], x]
                for k in range(K):
                    if k > 0 and it < 2 * k:
                        break
                    h = collide(h, x + nx * yr[k], t + k)
                    if k + 1 < K:
                        nxt = np.empty_like(h)
                        for i in range(q):
                            now = h[i].copy()
                            if C2[i, 0] > 0:
                                now = np.concatenate([[np.uint64(0)], now[:-1]])
                            elif C2[i, 0] < 0:
                                now = np.concatenate([now[1:], [np.uint64(0)]])
                            j = YIDX[i]
                            if C2[i, 1] == 0:
                                nxt[i], flat[k, j] = flat[k, j], now
                            elif C2[i, 1] > 0:
                                nxt[i], ua[k, j], ub[k, j] = ua[k, j].copy(), ub[k, j], now
                            else:
                                nxt[i] = now
                        h = nxt
                if 2 * halo <= it < yc + 2 * halo:
                    for i in range(q):
                        out.put(i, 0, (yr[K - 1] + C2[i, 1]) % ny, (x[mine] + C2[i, 0]) % nx, h[i][mine])
                yr = [(yr[0] + 1) % ny] + yr[:-1]
    return out.done()


@pytest.mark.parametrize("dims,rows", [((58, 9), 9), ((61, 7), 4), ((125, 5), 3), ((1, 6), 6), ((2, 3), 2), ((200, 1), 1),
                                       ((59, 20), 7)])
@pytest.mark.parametrize("K", [2, 3, 4])
def test_strips_take_their_steps(dims, rows, K):
    a = start(C2, (*dims, 1))
    assert np.array_equal(strip2d(a, 20, K, rows), steps(a, C2, 20, K))


# ---------------------------------------------------------------- k_block
def block(src, c, t, K, size):
    q, nz, ny, nx = src.shape
    out = Out(src)
    h, d3 = K - 1, len(c) == 19
    bx, by, bz = size
    n = (nx, ny, nz)
    r = (bx + 2 * h, by + 2 * h, bz + 2 * h if d3 else 1)
    lanes = -(-(r[0] * r[1] * r[2]) // 64) * 64
    assert lanes <= (512 if d3 else 1024)
    nl = 256 if lanes <= 256 else 512 if lanes <= 512 else 1024  # the LDS plane of the kernel's form
    tid = np.arange(lanes)
    rxy = r[0] * r[1]
    mx, mxy = -(-(1 << 20) // r[0]), -(-(1 << 20) // rxy)
    lz = (tid * mxy) >> 20 if d3 else 0 * tid
    rem = tid - lz * rxy
    ly = (rem * mx) >> 20
    lx = rem - ly * r[0]
    assert np.array_equal(lz, tid // rxy if d3 else 0 * tid) and np.array_equal(ly, rem // r[0])
    for z0 in range(0, nz, bz):
        for y0 in range(0, ny, by):
            for x0 in range(0, nx, bx):
                first, halo = (x0, y0, z0), (h, h, h if d3 else 0)
                ln = [min(b, m - f) for b, m, f in zip(size, n, first)]
                loc = (lx, ly, lz)
                pos = [(f + np.minimum(l, k + 2 * a - 1) - a) % m for f, l, k, a, m in zip(first, loc, ln, halo, n)]
                edge = [np.where(l < k + 2 * a, np.minimum(l, k + 2 * a - 1 - l), 0) for l, k, a in zip(loc, ln, halo)]
                depth = np.minimum.reduce(edge[:3 if d3 else 2])
                there = np.logical_and.reduce([l < k + 2 * a for l, k, a in zip(loc, ln, halo)][:3 if d3 else 2])
                site = pos[0] + nx * (pos[1] + ny * pos[2])
                own = src[:, pos[2], pos[1], pos[0]]
                for k in range(K):
                    wave = (there & (depth >= k)).reshape(-1, 64).any(1).repeat(64)
                    own = np.where(wave, collide(own, site, t + k), own)
                    if k == h:
                        break
                    lds = np.full((q, nl), POISON)
                    lds[:, :lanes] = own
                    for i in range(1, q):
                        f = tid - c[i, 0] - c[i, 1] * r[0] - (c[i, 2] * rxy if d3 else 0)
                        own[i] = lds[i, np.where(f < 0, nl - 1, np.minimum(f, nl - 1))]
                on = there & (depth >= h)
                for i in range(q):
                    out.put(i, (pos[2][on] + c[i, 2]) % nz, (pos[1][on] + c[i, 1]) % ny, (pos[0][on] + c[i, 0]) % nx,
                            own[i][on])
    return out.done()


@pytest.mark.parametrize("K", [2, 3])
@pytest.mark.parametrize("dims,size", [((4, 4, 4), (4, 4, 4)), ((9, 5, 6), (3, 3, 3)), ((1, 1, 1), (1, 1, 1)),
                                       ((2, 7, 3), (2, 4, 3)), ((13, 1, 4), (4, 1, 4))])
def test_blocks_3d_take_their_steps(dims, size, K):
    a = start(C3, dims)
    assert np.array_equal(block(a, C3, 30, K, size), steps(a, C3, 30, K))


@pytest.mark.parametrize("K", range(2, 9))
@pytest.mark.parametrize("dims,size", [((16, 9), (8, 8)), ((3, 2), (3, 2)), ((17, 25), (6, 7))])
def test_small_blocks_2d_take_their_steps(dims, size, K):
    a = start(C2, (*dims, 1))
    assert np.array_equal(block(a, C2, 40, K, (*size, 1)), steps(a, C2, 40, K))


@pytest.mark.parametrize("K", [2, 3, 4])
@pytest.mark.parametrize("dims,size", [((116, 20), (58, 10)), ((59, 11), (30, 6)), ((32, 17), (16, 9))])
def test_blocks_2d_take_their_steps(dims, size, K):
    a = start(C2, (*dims, 1))
    assert np.array_equal(block(a, C2, 50, K, (*size, 1)), steps(a, C2, 50, K))
