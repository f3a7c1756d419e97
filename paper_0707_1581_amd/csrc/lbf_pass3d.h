// Two fused steps of a D3Q19 lattice per launch.
//
// k_pass3d advances a D3Q19 lattice from even t by two steps in one pass over
// memory, from one buffer to another.
//
// Work split.  A workgroup of up to 16 waves owns a column of 64 x-y sites by up
// to 13 rows and walks a chunk of planes along z.  One wave holds each x-row, two
// the halo rows and one the halo columns (periodic; ragged tiles leave lanes
// idle).  Tiles split the rows of the box evenly and the workgroup has as many
// waves as its tile needs: a wave without a row of its own would load and collide
// all the same (512 x 7 x 1200 fp32, 16 steps, 1744 to 1309 us; 512 x 14 x 600
// 1907 to 1341; 512 x 40 x 300 2120 to 1795).  In each phase every wave collides the first step of its sites of the
// next plane u and writes the populations that move in x or y to LDS; after
// one barrier the row waves pull what arrives at their sites and collide the
// second step of plane u - 1: its down-going populations have just come from u,
// the flat ones waited one phase in registers, the up-going ones two.  The
// LDS holds two planes in turn, so the one barrier a phase suffices.
//
// The memory operations stand outside every branch (lanes and phases with
// nothing to move use an offset beyond the descriptor, which the range check
// drops, and the waves without a second step have a loop of their own), so the
// compiler waits for exactly the loads of one plane ahead and never for a
// store.
//
// Layouts.  Between the passes of one call the state need not be streamed: all
// but the last pass store the second step's populations at their own site
// (whole aligned rows, past the caches), and all but the first pull them from
// r - c_i.  The first pass reads and the last writes the even AA layout.  NT:
// the destination's rows are whole 128-byte lines; where they are not, a tile's
// row ends inside lines, and streaming the parts costs more than caching them
// (with the pitch of the second buffer, 441 x 318 x 225 fp32 takes 651 us per
// step instead of 784).  The second buffer holds the 19 populations of an x-row
// side by side: with planes on both sides a workgroup would have 38 pages or
// more in use at a time, more than the CU's address translation cache holds
// (22e6 misses a pass at 512^3, now 66e3; that alone took a pass from 6.59 to
// 5.53 ms).
//
// What bounds it: the movement (4.1 ms of the pass with the identity
// collision, 22.8 GB past the L2) and, nearly level with it, the collisions
// (3.6 ms without stores).  512^3 fp32, a pass: 4.55 ms first, 4.77 between,
// 5.21 last, against 5.27 for the former pass (64 x 10 tiles, planes in both
// buffers, pushes, waits for every store) and 7.05 for two AA steps.  Other
// tiles: 64 x 12 4% slower (more halo rows), rows of 66 or 62 lanes across
// waves 10% (every load crosses rows).
//
// The two steps compute exactly what two AA launches compute (same collision
// code, same noise keys, 16-bit values rounded between the steps as they would
// be stored), so the result is bit-identical.  PROP: the identity collision.
#pragma once

#include "lbf_kernels.h"

namespace lbf {

constexpr int P3_TX = 64, P3_TY = 13;                // most interior sites of a tile
constexpr int P3_THREADS = (P3_TY + 3) * 64;         // its row, halo-row and halo-column waves
constexpr int P3_ROW = P3_TX + 2;                    // LDS row: the tile's with its halo
constexpr int P3_PLANE = P3_ROW * (P3_TY + 2);       // LDS values of one population
constexpr int P3_XCH = 16;                           // populations that move in x or y
constexpr int P3_PAD = P3_ROW + 1;                   // what the edge lanes' pulls may pass the planes by

struct P3Slot {
  static constexpr bool moves(int i) { return D3Q19::CX[i] != 0 || D3Q19::CY[i] != 0; }
  // LDS plane of population i
  static constexpr int of(int i) {
    int n = 0;
    for (int j = 0; j < i; ++j) n += moves(j) ? 1 : 0;
    return n;
  }
  // index of population i among those with its c_z
  static constexpr int zidx(int i) {
    int n = 0;
    for (int j = 0; j < i; ++j) n += D3Q19::CZ[j] == D3Q19::CZ[i] ? 1 : 0;
    return n;
  }
};

// Tiles along x and y, the sites of a tile (a workgroup has ty + 3 waves), and
// the planes of a chunk.
struct PassGeom {
  uint32_t ntx, nty, tx, ty, len;
};

template <int S, bool PROP, bool PULL, bool OWN, bool NT>
__global__ void __launch_bounds__(P3_THREADS)
k_pass3d(const LatDesc* __restrict__ src, PassSide from, PassSide to, Clock ck, PassGeom g) {
  using M = D3Q19;
  using C = Codec<S>;
  using T = typename C::T;
  using U = typename Carry<T>::U;  // register form of the prefetched values
  constexpr int Q = M::Q;
  constexpr uint32_t ES = sizeof(T);
  constexpr uint32_t NOWHERE = 0u - ES;  // beyond every span: the range check drops the access
  __shared__ T lds[P3_PAD + 2 * P3_XCH * P3_PLANE + P3_PAD];
  const LatDesc& L = *src;
  Coef<M> cf(L);

  // tile: each XCD takes one contiguous eighth of the tiles (x fastest, then
  // y, then z chunk), so the tiles sharing halo lines run on one L2
  const uint32_t b = xcd_remap(blockIdx.x, gridDim.x, 1);
  const uint32_t txi = b % g.ntx, rest = b / g.ntx;
  const uint32_t tyi = rest % g.nty, tzi = rest / g.nty;
  const uint32_t nx = L.nx, ny = L.ny, nz = L.nz, nxy = L.nxy;
  const uint32_t x0 = txi * g.tx, y0 = tyi * g.ty, z0 = tzi * g.len;
  const uint32_t TW = min(g.tx, nx - x0), TH = min(g.ty, ny - y0), ZC = min(g.len, nz - z0);
  const uint32_t NIT = ZC + 2u;  // phase it: first step of plane z0 + it - 1, second of the one before
  const uint64_t t = ck.read();
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;

  // this lane's site in tile coordinates plus one, 0..TW + 1 and 0..TH + 1;
  // idle lanes repeat one at the far edge
  uint32_t lx = lane + 1u, ly = w + 1u;
  if (w == g.ty) ly = 0u;
  else if (w == g.ty + 1u) ly = TH + 1u;
  else if (w > g.ty + 1u) {
    lx = lane < 32u ? 0u : TW + 1u;
    ly = lane & 31u;
  }
  const bool mine = w < TH && lane < TW;
  lx = min(lx, TW + 1u);
  ly = min(ly, TH + 1u);
  const uint32_t pos = ly * (uint32_t)P3_ROW + lx;
  const uint32_t gx = x0 + lx, gy = y0 + ly;  // lattice coordinates plus one
  const uint32_t x = gx == 0u ? nx - 1u : (gx > nx ? gx - nx - 1u : gx - 1u);
  const uint32_t y = gy == 0u ? ny - 1u : (gy > ny ? gy - ny - 1u : gy - 1u);
  const uint32_t sxy = x + nx * y;
  // the x and y neighbours, periodic
  const uint32_t xm = x == 0u ? nx - 1u : x - 1u, xp = x + 1u >= nx ? 0u : x + 1u;
  const uint32_t ym = y == 0u ? ny - 1u : y - 1u, yp = y + 1u >= ny ? 0u : y + 1u;
  auto zm = [&](uint32_t z) { return z == 0u ? nz - 1u : z - 1u; };
  auto zp = [&](uint32_t z) { return z + 1u >= nz ? 0u : z + 1u; };

  // A running address, opaque to the optimiser, which would otherwise keep all
  // 38 plane addresses in scalar registers across the loop and spill.
  auto start = [](uint64_t a) {
    asm volatile("" : "+s"(a));
    return a;
  };
  auto load_plane = [&](uint32_t z, bool on, U (&v)[Q]) {
    uint64_t a = start(from.base);
    const uint64_t o0 = (uint64_t)z * from.slice;
    const uint64_t om = PULL ? (uint64_t)zm(z) * from.slice : 0u, op = PULL ? (uint64_t)zp(z) * from.slice : 0u;
    static_for<0, Q>([&](auto I) {
      constexpr int i = decltype(I)::value;
      constexpr int cx = PULL ? M::CX[i] : 0, cy = PULL ? M::CY[i] : 0, cz = PULL ? M::CZ[i] : 0;
      const uint32_t xs = cx > 0 ? xm : (cx < 0 ? xp : x), ys = cy > 0 ? ym : (cy < 0 ? yp : y);
      const uint64_t zo = cz > 0 ? om : (cz < 0 ? op : o0);
      v[i] = Carry<T>::wrap(Raw<T>::template ld<0>(span_rsrc(a + zo, from.span), on ? xs * ES + ys * from.row : NOWHERE));
      a += from.plane;
    });
  };
  using H = typename std::conditional<PROP, T, float>::type;
  auto store_plane = [&](uint32_t z, bool on, const H (&h)[Q]) {
    uint64_t a = start(to.base);
    const uint64_t o0 = (uint64_t)z * to.slice;
    const uint64_t om = OWN ? 0u : (uint64_t)zm(z) * to.slice, op = OWN ? 0u : (uint64_t)zp(z) * to.slice;
    static_for<0, Q>([&](auto J) {
      constexpr int j = decltype(J)::value;
      constexpr int cx = OWN ? 0 : M::CX[j], cy = OWN ? 0 : M::CY[j], cz = OWN ? 0 : M::CZ[j];
      const uint32_t xd = cx > 0 ? xp : (cx < 0 ? xm : x), yd = cy > 0 ? yp : (cy < 0 ? ym : y);
      const uint64_t zo = cz > 0 ? op : (cz < 0 ? om : o0);
      T o;
      if constexpr (PROP) o = h[j]; else o = C::enc(h[j]);
      // rows that share lines with the neighbouring tiles are cached, whole lines stream
      Raw<T>::template st<pol(NT && cx == 0)>(span_rsrc(a + zo, to.span), on ? xd * ES + yd * to.row : NOWHERE, o);
      a += to.plane;
    });
  };

  // populations that wait in registers for the second step: flat ones of the
  // last plane, up-going ones of the last two
  H hf[9], ua[5], ub[5];
#pragma unroll
  for (int k = 0; k < 9; ++k) hf[k] = (H)0;
#pragma unroll
  for (int k = 0; k < 5; ++k) ua[k] = ub[k] = (H)0;

  auto walk = [&](auto inner) {
    constexpr bool INNER = decltype(inner)::value;  // a wave of interior rows
    U v[Q];
    uint32_t zc = zm(z0), zprev = zc;
    load_plane(zc, true, v);
    if constexpr (INNER) {  // as many (dropped) stores behind the loads as in every later phase
      H h[Q];
#pragma unroll
      for (int i = 0; i < Q; ++i) h[i] = (H)0;
      store_plane(zc, false, h);
    }
    for (uint32_t it = 0; it < NIT; ++it) {
      T own[Q];
      float d[Q];
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        own[i] = Carry<T>::unwrap(v[i]);
        d[i] = C::dec(own[i]);
      }
      const uint32_t zn = zp(zc);
      load_plane(zn, it + 1u < NIT, v);
      if constexpr (!PROP) {
        cf.fresh_keys();
        collide<M, S>(cf, d, sxy + zc * nxy, (uint32_t)t, (uint32_t)(t >> 32));
#pragma unroll
        for (int i = 0; i < Q; ++i) own[i] = C::enc(d[i]);
      }
      T* const buf = lds + P3_PAD + (it & 1u) * (P3_XCH * P3_PLANE) + pos;
      static_for<0, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if constexpr (P3Slot::moves(i)) buf[P3Slot::of(i) * P3_PLANE] = own[i];
      });
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
      if constexpr (INNER) {
        H now[Q], h[Q];
        static_for<0, Q>([&](auto I) {
          constexpr int i = decltype(I)::value;
          T s = own[i];
          if constexpr (P3Slot::moves(i)) s = buf[P3Slot::of(i) * P3_PLANE - M::CY[i] * P3_ROW - M::CX[i]];
          if constexpr (PROP) now[i] = s; else now[i] = C::dec(s);
          constexpr int k = P3Slot::zidx(i);
          if constexpr (M::CZ[i] == 0) h[i] = hf[k];
          else if constexpr (M::CZ[i] > 0) h[i] = ua[k];
          else h[i] = now[i];
        });
        if constexpr (!PROP) {
          if (it >= 2u) {
            const uint64_t t1 = t + 1u;
            cf.fresh_keys();
            collide<M, S>(cf, h, sxy + zprev * nxy, (uint32_t)t1, (uint32_t)(t1 >> 32));
          }
        }
        store_plane(zprev, mine && it >= 2u, h);
        static_for<0, Q>([&](auto I) {
          constexpr int i = decltype(I)::value;
          constexpr int k = P3Slot::zidx(i);
          if constexpr (M::CZ[i] == 0) hf[k] = now[i];
          if constexpr (M::CZ[i] > 0) {
            ua[k] = ub[k];
            ub[k] = now[i];
          }
        });
      }
      zprev = zc;
      zc = zn;
    }
  };
  if (w < g.ty) walk(std::true_type{});
  else walk(std::false_type{});
  ck.tick(t, ck.ticks());
}

}  // namespace lbf
