// Several time steps per launch on two-dimensional lattices (k_tile).
//
// A single-step pass moves 2 q b bytes per node and step and costs a launch
// of ~4 us however small the grid.  Here a workgroup takes a tile of nodes
// and a ring around it through `steps` steps with the populations in LDS:
// step s covers the tile and the steps - 1 - s nodes around it, so the ring
// is computed by several workgroups and nothing is exchanged between them.
// HBM sees each population once per launch.  In LDS the populations stream in
// place (even steps store each one in its opposite slot at the node, odd
// steps gather from the opposite slots upstream and scatter downstream), so
// each slot is read and written by one thread per step and one barrier per
// step is enough.  Values are rounded to the storage type at every step and
// the collision is collide_node, so the result has the bits of single steps.
#pragma once

#include "kernels.hpp"

namespace lbmrv {

constexpr int kTileMaxSteps = 8;
// The LDS region (tile and ring) is kTileP x kTileP nodes.  A fixed pitch
// makes every LDS offset of the unrolled population loops an immediate: with
// run-time pitches the kernel spilled scalar registers and took 11.5 instead
// of 9.7 us for eight steps of D2Q9 64^2 FP32.  40 x 40 FP32 nodes are 57.6 KB,
// two workgroups per CU; a 48 x 48 region (one per CU) ran 20 % slower at
// 1024^2, and FP64's 28 x 28 (two per CU) 5 % slower than its 40 x 40 (one).
constexpr int kTileP = 40;

struct TileArgs {
  uint32_t steps;    // 1 .. kTileMaxSteps
  uint32_t t[2];     // tile extents, t[a] + 2 (steps - 1) <= kTileP
  uint32_t gather;   // 1: fin holds post-collision values, the first step gathers from x - c_j
  uint32_t scatter;  // 1: the last step stores at x + c_j (pre-collision result), 0: at the node
  uint32_t m[kTileMaxSteps];  // step s: 2^18 / (t[0] + 2 (steps - 1 - s)), rounded up
};

// Tile and step count for an nx x ny grid; steps < 2: single steps are the
// better choice.  The tile plus its ring must fit in one period of the grid
// (t + steps - 1 <= extent), so that a coordinate wraps at most once.
struct TilePlan {
  uint32_t t[2];
  uint32_t steps;    // most steps per launch
  uint32_t threads;
};

inline TilePlan plan_tile(uint32_t nx, uint32_t ny) {
  // Large tiles waste less on the ring (32 x 32, 5 steps: 27 % more node
  // steps; 16 x 16: 57 %), small ones keep the 256 CUs busy on small grids.
  // Measured, us per step, D2Q9 FP32 (one step per launch | 8 | 16 | 32):
  //   64^2    3.6 | 1.2 |  -  |  -      256^2   4.0 |  2  | 1.6 |  -
  //   512^2   4.8 |  -  | 3.6 | 2.8     2048^2 54.5 | 136 |  50 | 29.0
  const uint64_t n = (uint64_t)nx * ny;
  const uint32_t side = n >= 3u << 16 ? 32u : n >= 1u << 15 ? 16u : 8u;
  const uint32_t most = side == 32u ? 5u : 8u;
  const uint32_t lo = nx < ny ? nx : ny;
  TilePlan p{};
  if (lo <= side) return p;  // thinner than a tile: single steps
  // equal tiles: no nearly empty last column or row
  const uint32_t cx = (nx + side - 1) / side, cy = (ny + side - 1) / side;
  p.t[0] = (nx + cx - 1) / cx;
  p.t[1] = (ny + cy - 1) / cy;
  const uint32_t t = p.t[0] > p.t[1] ? p.t[0] : p.t[1];
  p.steps = lo - t + 1 < most ? lo - t + 1 : most;
  // one workgroup per CU wants a thread per region node, two share the CU
  p.threads = side == 32u ? ((uint64_t)cx * cy <= 256u ? 1024u : 768u) : side == 16u ? 768u : 512u;
  return p;
}

template <class B, int ST, int MODE>
constexpr size_t tile_lds_bytes() {
  constexpr size_t R = kTileP * kTileP;
  constexpr size_t f = (B::Q * R * sizeof(typename Store<ST>::S) + 15) / 16 * 16;
  return f + (MODE == UT_FIELD ? B::Lat::D * R * sizeof(float) : 0);
}

template <class B, int ST, int MODE, int RLX>
__global__ __launch_bounds__(1024) void k_tile(StepArgs<typename Store<ST>::T> a, TileArgs g) {
  using L = typename B::Lat;
  using S = typename Store<ST>::S;
  using T = typename Store<ST>::T;
  constexpr int Q = B::Q;
  constexpr int D = L::D;
  constexpr int P = kTileP, R = P * P;
  static_assert(D == 2, "two-dimensional lattices");
  extern __shared__ __align__(16) unsigned char lds_raw[];
  S* lf = reinterpret_cast<S*>(lds_raw);
  float* lu = reinterpret_cast<float*>(lds_raw + tile_lds_bytes<B, ST, UT_ZERO>());

  const int nx = (int)a.nx, ny = (int)a.ny;
  const uint64_t N = a.N;
  const S* fin = static_cast<const S*>(a.fin);
  S* fout = static_cast<S*>(a.fout);
  const uint3 tile = block_tile(a.xcd_remap);
  const int steps = (int)g.steps;
  const int x0 = (int)(tile.x * g.t[0]), y0 = (int)(tile.y * g.t[1]);

  for (int s = 0; s < steps; ++s) {
    const int ring = steps - 1 - s;
    const uint32_t ex = g.t[0] + 2 * ring, ey = g.t[1] + 2 * ring;
    const uint32_t count = ex * ey;
    const uint32_t m = g.m[s];
    for (uint32_t i = threadIdx.x; i < count; i += blockDim.x) {
      const uint32_t iy = __umul24(i, m) >> 18, ix = i - __umul24(iy, ex);
      const int l = (int)__umul24(iy + s, P) + (int)ix + s;
      T h[Q];
      T utf[3] = {T(0), T(0), T(0)};
      int x = 0, y = 0;
      bool inside = false;
      if (s == 0 || ring == 0) {
        x = x0 - ring + (int)ix;
        y = y0 - ring + (int)iy;
        inside = x < nx && y < ny;
        x += x < 0 ? nx : 0;
        x -= x >= nx ? nx : 0;
        y += y < 0 ? ny : 0;
        y -= y >= ny ? ny : 0;
      }
      if (s == 0) {
        const int gs = g.gather ? 1 : 0;
        const int xm = gs ? (x == 0 ? nx - 1 : x - 1) : x, xp = gs ? (x == nx - 1 ? 0 : x + 1) : x;
        const uint32_t r0 = (uint32_t)y * nx, rm = gs ? (uint32_t)(y == 0 ? ny - 1 : y - 1) * nx : r0,
                       rp = gs ? (uint32_t)(y == ny - 1 ? 0 : y + 1) * nx : r0;
        sfor<Q>([&](auto jj) {
          constexpr int cx = L::c[jj].x, cy = L::c[jj].y;
          const uint32_t n = (cy > 0 ? rm : cy < 0 ? rp : r0) + (uint32_t)(cx > 0 ? xm : cx < 0 ? xp : x);
          h[jj] = T(fin[(uint64_t)jj * N + n]);
        });
        if constexpr (MODE == UT_FIELD) {
          sfor<D>([&](auto al) {
            const float v = a.ut[(uint64_t)al * N + r0 + x];
            lu[al * R + l] = v;
            utf[al] = T(v) * a.inv_lambda;
          });
        }
      } else {
        if (s & 1) {
          sfor<Q>([&](auto jj) { h[jj] = T(lf[l + (opposite<L>(jj) * R - L::c[jj].y * P - L::c[jj].x)]); });
        } else {
          sfor<Q>([&](auto jj) { h[jj] = T(lf[l + jj * R]); });
        }
        if constexpr (MODE == UT_FIELD) {
          sfor<D>([&](auto al) { utf[al] = T(lu[al * R + l]) * a.inv_lambda; });
        }
      }
      collide_node<B, T, MODE, RLX>(h, a, utf);
      // rounded to the storage type once, right behind the collision: with FP16
      // storage the compiler merges the last fma of a population and this
      // conversion into one instruction with one rounding, as in k_step; one
      // conversion per branch below kept two roundings
      S o[Q];
      sfor<Q>([&](auto jj) { o[jj] = S(h[jj]); });
      if (ring == 0) {
        if (inside) {
          const int gs = g.scatter ? 1 : 0;
          const int xm = gs ? (x == 0 ? nx - 1 : x - 1) : x, xp = gs ? (x == nx - 1 ? 0 : x + 1) : x;
          const uint32_t r0 = (uint32_t)y * nx, rm = gs ? (uint32_t)(y == 0 ? ny - 1 : y - 1) * nx : r0,
                         rp = gs ? (uint32_t)(y == ny - 1 ? 0 : y + 1) * nx : r0;
          sfor<Q>([&](auto jj) {
            constexpr int cx = L::c[jj].x, cy = L::c[jj].y;
            const uint32_t n = (cy < 0 ? rm : cy > 0 ? rp : r0) + (uint32_t)(cx < 0 ? xm : cx > 0 ? xp : x);
            fout[(uint64_t)jj * N + n] = o[jj];
          });
        }
      } else if (s & 1) {
        sfor<Q>([&](auto jj) { lf[l + (jj * R + L::c[jj].y * P + L::c[jj].x)] = o[jj]; });
      } else {
        sfor<Q>([&](auto jj) { lf[l + opposite<L>(jj) * R] = o[jj]; });
      }
    }
    if (ring) __syncthreads();
  }
}

}  // namespace lbmrv
