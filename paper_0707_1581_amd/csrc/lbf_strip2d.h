// Fused steps of a D2Q9 lattice: K per launch (2 to 4).
//
// k_strip2d advances a D2Q9 lattice from even t by K steps in one pass over
// memory: it reads the state in the even AA layout (plane i at site r holds
// n_i(r)) from one buffer and writes the state at t + K, in the same layout,
// to another, so each population is read and written once per K steps.
//
// Work split.  A wave owns a strip of x-columns, one lane each, and walks a
// chunk of rows along y with everything in registers; waves share no data, so
// there is no LDS and, but for passes in step (below), no barrier, and the waves
// of a SIMD cover each other's loads.  The strip carries a halo of K - 1 columns on either side and the
// chunk one of K - 1 rows: step k is collided on K - k of them, which the
// neighbouring waves collide too (58 of 64 lanes are interior at K = 4).  In
// each phase the wave collides step 1 of the next row, step 2 of the row
// before it, and so on; between two steps the x-shifts are lane shifts (DPP)
// and the y-shifts are the phases the values wait in registers: nine of them
// per pair of steps, the flat populations of one row and the up-going ones of
// two.  The loads of the next row are in flight while a row is collided.
// The loop has no memory operation under a branch: rows and lanes with nothing
// to move use an offset beyond the descriptor, which the range check drops, so
// the compiler can wait for exactly the loads it needs.
//
// The strips of a workgroup share lines at their edges, but no data.  With
// sync they walk in step all the same, one barrier a phase, so that such a line
// is read once and leaves the L2 whole: state that streams through HBM gains
// (16384^2 fp32, 2.87 to 2.39 ms per step with K = 2 and 2.02 with 16 strips
// side by side, 2.00 to 1.62 with K = 3, 1.61 as before with K = 4, which its
// collisions hold in step; the second buffer's writes in partial lines were
// 12% at K = 2), state the Infinity Cache holds loses 1-2%.  All waves run the
// same phases, those past the last strip or row without effect.
//
// What bounds it: the issue of vector instructions for K = 3 and 4 (bf16 takes
// as long as the collisions alone).  16384^2, 20 steps, per step: fp32 1.62 ms
// (1.49 of 8 TB/s in algorithmic bytes) against 2.17 for the former two-step
// pass (256-site segments with an LDS ring) and 3.36 for AA steps; bf16 1.55
// against 1.86 and 1.76.
//
// Addressing.  One descriptor per row of one population, so a plane may exceed
// 4 GiB.  The second buffer holds the nine populations of a row side by side:
// a wave that reads nine planes and writes nine more would have 18 pages or
// more in use at a time, and the CU's address translation cache thrashes.
//
// The K steps compute exactly what K AA launches compute (same collision code,
// same noise keys, 16-bit values rounded between the steps as they would be
// stored), so the result is bit-identical.  PROP: the identity collision.
#pragma once

#include "lbf_kernels.h"

namespace lbf {

struct StripGeom {
  uint32_t ntx;  // strips along x
  uint32_t tx;   // interior sites of a strip, at most 64 - 2 (K - 1)
  uint32_t nty;  // chunks of rows
  uint32_t len;  // rows of a chunk
  uint32_t sync;  // the strips of a workgroup walk in step
};

// Strips of a workgroup, side by side: four, or 16 or eight where the movement
// bounds the pass (two fp32 steps, in step with each other).
constexpr int S2_WAVES = 4, S2_WIDE_WAVES = 16;

template <class M> struct YIndex {
  static constexpr int idx(int i) {
    int n = 0;
    for (int j = 0; j < i; ++j) n += (M::CY[j] == M::CY[i]) ? 1 : 0;
    return n;
  }
};

// The value of the lane to the left (D = 1) or right (D = -1).
template <int D, class T>
__device__ __forceinline__ T lane_from(T v) {
  uint32_t u;
  if constexpr (sizeof(T) == 4) u = __builtin_bit_cast(uint32_t, v);
  else u = (uint32_t)__builtin_bit_cast(uint16_t, v);
  u = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u, D > 0 ? 0x138 : 0x130, 0xF, 0xF, true);
  if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, u);
  else return __builtin_bit_cast(T, (uint16_t)u);
}

template <int S, bool PROP, int K, int W = S2_WAVES>
__global__ void __launch_bounds__(64 * W)
k_strip2d(const LatDesc* __restrict__ src, PassSide from, PassSide to, Clock ck, StripGeom g) {
  using M = D2Q9;
  using C = Codec<S>;
  using T = typename C::T;
  using U = typename Carry<T>::U;
  constexpr int Q = M::Q;
  constexpr uint32_t ES = sizeof(T);
  constexpr uint32_t NOWHERE = 0u - ES;  // beyond every span: the range check drops the access
  constexpr int HALO = K - 1;
  const LatDesc& L = *src;
  Coef<M> cf(L);
  const uint32_t nx = L.nx, ny = L.ny;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = xcd_remap(blockIdx.x, gridDim.x, 1) * W + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t wid = min(wave, g.ntx * g.nty - 1u);  // waves past the last strip walk it too and store nothing
  const uint64_t t = ck.read();
  const bool ticks = ck.ticks();
  const uint32_t txi = wid % g.ntx, tyi = wid / g.ntx;
  const uint32_t x0 = txi * g.tx, y0 = tyi * g.len;
  const uint32_t TW = min(g.tx, nx - x0), YC = min(g.len, ny - y0);
  const uint32_t NIT = wave == wid ? YC + 2u * HALO : 0u;

  // this lane's column: lanes past the strip and its halo repeat the last one
  const uint32_t col = min(lane, TW + 2u * HALO - 1u);
  const bool mine = lane >= (uint32_t)HALO && lane < (uint32_t)HALO + TW;
  const uint32_t hx = (uint32_t)HALO % nx, hy = (uint32_t)HALO % ny;  // the halo of a box narrower than it wraps
  const uint32_t xs = x0 + col, x = (xs >= hx ? xs - hx : xs + (nx - hx)) % nx;
  const uint32_t xm = x == 0u ? nx - 1u : x - 1u, xp = x + 1u >= nx ? 0u : x + 1u;
  const uint32_t vo = x * ES;
  const uint32_t so = mine ? vo : NOWHERE, som = mine ? xm * ES : NOWHERE, sop = mine ? xp * ES : NOWHERE;

  auto next = [&](uint32_t y) { return y + 1u >= ny ? 0u : y + 1u; };
  auto load_row = [&](uint32_t y, uint32_t v_off, U (&v)[Q]) {
    uint64_t a = from.base + (uint64_t)y * from.slice;
    asm volatile("" : "+s"(a));
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      v[i] = Carry<T>::wrap(Raw<T>::template ld<0>(span_rsrc(a, from.span), v_off));
      a += from.plane;
    }
  };
  using H = typename std::conditional<PROP, T, float>::type;
  auto store_row = [&](uint32_t y, bool on, const H (&h)[Q]) {
    const uint32_t ym = y == 0u ? ny - 1u : y - 1u, yp = next(y);
    uint64_t a = to.base;
    asm volatile("" : "+s"(a));
    const uint64_t o0 = (uint64_t)y * to.slice, om = (uint64_t)ym * to.slice, op = (uint64_t)yp * to.slice;
    const uint32_t v0 = on ? so : NOWHERE, vm = on ? som : NOWHERE, vp = on ? sop : NOWHERE;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      T o;
      if constexpr (PROP) o = h[j]; else o = C::enc(h[j]);
      Raw<T>::template st<0>(span_rsrc(a + (M::CY[j] > 0 ? op : (M::CY[j] < 0 ? om : o0)), to.span),
                             M::CX[j] > 0 ? vp : (M::CX[j] < 0 ? vm : v0), o);
      a += to.plane;
    }
  };

  // populations in flight between step k and step k + 1: flat ones of the
  // last row, up-going ones of the last two
  H hf[HALO][3], ua[HALO][3], ub[HALO][3];
#pragma unroll
  for (int k = 0; k < HALO; ++k)
#pragma unroll
    for (int j = 0; j < 3; ++j) hf[k][j] = ua[k][j] = ub[k][j] = (H)0;

  U v[Q];
  uint32_t yr[K];  // row of step k + 1 in this phase
  yr[0] = y0 >= hy ? y0 - hy : y0 + (ny - hy);
#pragma unroll
  for (int k = 1; k < K; ++k) yr[k] = yr[0];
  load_row(yr[0], vo, v);
  {  // as many (dropped) stores behind the loads as in every later phase
    H h[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) h[i] = (H)0;
    store_row(yr[0], false, h);
  }
  for (uint32_t it = 0; it < g.len + 2u * HALO; ++it) {
    if (g.sync) __builtin_amdgcn_s_barrier();
    H h[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      if constexpr (PROP) h[i] = Carry<T>::unwrap(v[i]);
      else h[i] = C::dec(Carry<T>::unwrap(v[i]));
    }
    const uint32_t yn = next(yr[0]);
    load_row(yn, it + 1u < NIT ? vo : NOWHERE, v);
    static_for<0, K>([&](auto KK) {
      constexpr int k = decltype(KK)::value;
      if (k > 0 && it < 2u * k) return;  // its rows start 2 k phases later
      if constexpr (!PROP) {
        const uint64_t tk = t + (uint64_t)k;
        cf.fresh_keys();
        collide<M, S>(cf, h, x + yr[k] * nx, (uint32_t)tk, (uint32_t)(tk >> 32));
      }
      if constexpr (k + 1 < K) {
        H now[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) {
          H o;
          if constexpr (PROP) o = h[i]; else o = C::dec(C::enc(h[i]));
          now[i] = M::CX[i] > 0 ? lane_from<1>(o) : (M::CX[i] < 0 ? lane_from<-1>(o) : o);
        }
#pragma unroll
        for (int i = 0; i < Q; ++i) {
          constexpr auto I = [](int j) { return YIndex<M>::idx(j); };
          if (M::CY[i] == 0) { h[i] = hf[k][I(i)]; hf[k][I(i)] = now[i]; }
          else if (M::CY[i] > 0) { h[i] = ua[k][I(i)]; ua[k][I(i)] = ub[k][I(i)]; ub[k][I(i)] = now[i]; }
          else h[i] = now[i];
        }
      }
    });
    store_row(yr[K - 1], it >= 2u * HALO && it < NIT, h);
#pragma unroll
    for (int k = K - 1; k > 0; --k) yr[k] = yr[k - 1];
    yr[0] = yn;
  }
  ck.tick(t, ticks);
}

}  // namespace lbf
