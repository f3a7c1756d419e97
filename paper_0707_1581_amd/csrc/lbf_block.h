// Fused steps of a small lattice: K per launch, one site per lane.
//
// What bounds the steps of a small lattice is latency: an AA launch of 16^3
// sites takes 3.9 us, about 2 of them the launch, the descriptor and the state
// on their way and the stores draining.  k_block advances the lattice by K
// steps per launch instead.  A workgroup owns a block of sites and holds it
// with a halo of K - 1 sites, one site per lane (at most NL); each step is
// collided on every lane, and between two steps the populations go through LDS
// to their neighbours.  Of the halo one layer per step loses its neighbours
// and is no longer right; after the last step the block itself is pushed to
// the destination.  Neighbouring workgroups repeat each other's halo: the
// blocks are small where the lattice leaves compute units idle, and large
// where it does not (see plan_blocks in lbf.hip, with the figures).
//
// The steps compute exactly what AA launches compute (same collision code, same
// noise keys, 16-bit values rounded between the steps as they would be stored),
// so the result is bit-identical.  PROP: the identity collision.
#pragma once

#include "lbf_kernels.h"

namespace lbf {

struct BlockGeom {
  uint64_t from, to;        // the state read and the one written, same layout
  uint32_t nx, ny, nz;
  uint32_t bx, by, bz;      // sites of a block
  uint32_t rx, rxy;         // row and plane of a block with its halo
  uint32_t mx, mxy;         // ceil(2^20 / rx), ceil(2^20 / rxy): exact for lanes below 1024
  uint32_t steps;           // K
};

template <class M> struct BlockSlot {
  static constexpr int of(int i) { return i - 1; }  // LDS plane of population i > 0; the rest one stays
};

template <class M, int S, bool PROP, int NL>
__global__ void __launch_bounds__(NL)
k_block(const LatDesc* __restrict__ src, Clock ck, BlockGeom g) {
  using C = Codec<S>;
  using T = typename C::T;
  constexpr int Q = M::Q;
  constexpr uint32_t ES = sizeof(T);
  constexpr uint32_t NOWHERE = 0u - ES;
  __shared__ T lds[(Q - 1) * NL];
  const LatDesc& L = *src;
  const uint32_t tid = threadIdx.x;
  const uint32_t h = g.steps - 1u, hz = M::D == 3 ? h : 0u;

  // this lane's place in the block with its halo; lanes past it repeat its
  // last plane, row or site
  uint32_t lz = 0, r = tid;
  if constexpr (M::D == 3) {
    lz = (tid * g.mxy) >> 20;
    r = tid - lz * g.rxy;
  }
  const uint32_t ly = (r * g.mx) >> 20, lx = r - ly * g.rx;
  auto place = [](uint32_t b, uint32_t l, uint32_t size, uint32_t n, uint32_t halo, uint32_t& len) {
    const uint32_t first = b * size;
    len = min(size, n - first);
    int v = (int)(first + min(l, len + 2u * halo - 1u)) - (int)halo;
    while (v < 0) v += (int)n;          // a box narrower than the halo wraps more than once
    while (v >= (int)n) v -= (int)n;
    return (uint32_t)v;
  };
  uint32_t TX, TY, TZ;
  const uint32_t x = place(blockIdx.x, lx, g.bx, g.nx, h, TX);
  const uint32_t y = place(blockIdx.y, ly, g.by, g.ny, h, TY);
  const uint32_t z = M::D == 3 ? place(blockIdx.z, lz, g.bz, g.nz, hz, TZ) : 0u;
  if constexpr (M::D == 2) TZ = 1u;
  const uint32_t site = x + g.nx * (y + g.ny * z);
  const uint32_t pbytes = g.nx * g.ny * g.nz * ES;

  const __amdgpu_buffer_rsrc_t in = __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)g.from, 0, (int)(Q * pbytes),
                                                                      RAW_BUFFER_WORD3);
  T own[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) own[i] = Raw<T>::template ld<0>(in, site * ES, (uint32_t)i * pbytes);
  const uint64_t t = ck.read();

  // distance of this lane from the edge of the block with its halo: its site
  // is right up to the step of that number
  auto edge = [](uint32_t l, uint32_t len, uint32_t halo) {
    const uint32_t n = len + 2u * halo;
    return l < n ? min(l, n - 1u - l) : 0u;
  };
  uint32_t depth = min(edge(lx, TX, h), edge(ly, TY, h));
  bool there = lx < TX + 2u * h && ly < TY + 2u * h;
  if constexpr (M::D == 3) {
    depth = min(depth, edge(lz, TZ, hz));
    there = there && lz < TZ + 2u * hz;
  }

  for (uint32_t k = 0;; ++k) {
    if constexpr (!PROP) {
      if (__builtin_amdgcn_ballot_w64(there && depth >= k) != 0) {  // a wave past its last right site is done
        float d[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) d[i] = C::dec(own[i]);
        const uint64_t tk = t + k;
        collide<M, S>(L, d, site, (uint32_t)tk, (uint32_t)(tk >> 32));
#pragma unroll
        for (int i = 0; i < Q; ++i) own[i] = C::enc(d[i]);
      }
    }
    if (k == h) break;
    if (k > 0) __syncthreads();  // every lane has pulled the step before
#pragma unroll
    for (int i = 1; i < Q; ++i) lds[BlockSlot<M>::of(i) * NL + tid] = own[i];
    __syncthreads();
    const uint32_t most = (uint32_t)NL - 1u;
#pragma unroll
    for (int i = 1; i < Q; ++i) {
      uint32_t from = tid - (uint32_t)M::CX[i] - (uint32_t)M::CY[i] * g.rx;
      if constexpr (M::D == 3) from -= (uint32_t)M::CZ[i] * g.rxy;
      own[i] = lds[BlockSlot<M>::of(i) * NL + min(from, most)];  // edge lanes have no neighbour: any value
    }
  }

  const bool mine = there && depth >= h;
  const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)g.to, 0, (int)(Q * pbytes),
                                                                       RAW_BUFFER_WORD3);
  const uint32_t xm = x == 0u ? g.nx - 1u : x - 1u, xp = x + 1u >= g.nx ? 0u : x + 1u;
  const uint32_t ym = (y == 0u ? g.ny - 1u : y - 1u) * g.nx, y0 = y * g.nx, yp = (y + 1u >= g.ny ? 0u : y + 1u) * g.nx;
  const uint32_t nxy = g.nx * g.ny;
  const uint32_t zm = (z == 0u ? g.nz - 1u : z - 1u) * nxy, z0 = z * nxy, zp = (z + 1u >= g.nz ? 0u : z + 1u) * nxy;
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const uint32_t s = (M::CX[i] > 0 ? xp : (M::CX[i] < 0 ? xm : x)) + (M::CY[i] > 0 ? yp : (M::CY[i] < 0 ? ym : y0)) +
                       (M::CZ[i] > 0 ? zp : (M::CZ[i] < 0 ? zm : z0));
    Raw<T>::template st<0>(out, mine ? s * ES : NOWHERE, own[i], (uint32_t)i * pbytes);
  }
  ck.tick(t, ck.ticks());
}

}  // namespace lbf
