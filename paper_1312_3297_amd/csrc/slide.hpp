// Two time steps per launch on three-dimensional lattices (k_slide).
//
// A workgroup owns a tile of columns (x, y) and marches through a chunk of
// planes.  Per plane p it takes the tile and a ring of one node through step
// one, leaves the populations that change column in LDS, and then takes plane
// p - 1 of the tile through step two, so the state crosses HBM once for two
// steps.  One thread per column: the populations that move along z only stay
// in its registers.  A plane's populations with c_z < 0 are read in the same
// iteration (one LDS copy), those with c_z = 0 in the next one (two copies),
// those with c_z > 0 in the one after (three): 32 slots per column for D3Q19,
// 48 for D3Q27, instead of three whole planes.
//
// FP32 is bound by HBM and L2, not by the arithmetic: without its collisions
// the kernel is no faster, and of the fetched bytes a third are ring nodes that
// fell out of L2 before the neighbouring tile took them (D3Q19 256^3: 1.73 GB
// read for 1.28 GB, 592 us for two steps against 2 x 429).  Loading the next
// plane after the first collision instead of before it keeps fewer lines in
// flight and measured 592 against 665 us; 66 x 15 and 34 x 30 columns (1024
// threads) 660, a third LDS copy that saves one of the two barriers 593,
// non-temporal stores 601 us.
#pragma once

#include "kernels.hpp"

namespace lbmrv {

struct SlideArgs {
  uint32_t t[2];     // tile extents in x and y
  uint32_t chunk;    // planes per workgroup
  uint32_t gather;   // 1: fin holds post-collision values, step one gathers from x - c_j
  uint32_t scatter;  // 1: step two stores at x + c_j (pre-collision result), 0: at the node
  void* keep;        // KEEP: where the state between the two steps goes
};

// Most columns of a workgroup, ring included.  34 wide: whole 128-byte lines of
// an FP32 row.  22 rows are 96 KB of LDS for D3Q19 FP32 and 144 KB for D3Q27
// FP32; D3Q19 FP64 has room for 18 (157 KB), D3Q27 FP64 for 26 x 16 (160 KB).
// plan_slide picks the rows.
template <class B, int ST>
struct SlideShape {
  static constexpr bool small = B::Q == 27 && ST == 0;
  static constexpr int PX = small ? 26 : 34, PY = small ? 16 : ST == 0 ? 18 : 22;
  static constexpr int threads = (PX * PY + 63) / 64 * 64;
};

// LDS copies of direction j (see above) and its first slot
template <class B>
struct SlideSlots {
  using L = typename B::Lat;
  static constexpr bool axis(int j) { return L::c[j].x == 0 && L::c[j].y == 0; }
  static constexpr int copies(int j) { return axis(j) ? 0 : L::c[j].z < 0 ? 1 : L::c[j].z == 0 ? 2 : 3; }
  static constexpr int base(int j) {
    int b = 0;
    for (int i = 0; i < j; ++i) b += copies(i);
    return b;
  }
  static constexpr int count = base(B::Q);
};

struct SlidePlan {
  uint32_t t[2];
  uint32_t chunk;  // 0: single steps are the better choice
  uint32_t threads;
};

// FP16 storage keeps single steps: half the bytes leave it bound by the vector
// ALU, and the ring adds to that (D3Q19 256^3: 286 against 250 us per step).
template <class B, int ST>
SlidePlan plan_slide(uint32_t nx, uint32_t ny, uint32_t nz) {
  using Sh = SlideShape<B, ST>;
  SlidePlan p{};
  const uint64_t n = (uint64_t)nx * ny * nz;
  // Small grids have too few columns: each workgroup gets two or three planes
  // and computes four or five.  Measured, us per step, single | two per launch:
  // D3Q19 FP32 117 x 100 x 19 8.3 | 9.4, 64^3 9.0 | 7.9 (k_tile: 7.0), 96^3 28.1 |
  // 16.4; FP64 64^3 17.8 | 12.9, 96^3 53.8 | 29.9; D3Q27 FP32 64^3 10.7 | 11.6,
  // 96^3 41.2 | 26.8; FP64 57 x 207 x 61 64 | 75, 63 x 221 x 96 159 | 124.
  if (ST == 2 || n < (B::Q == 27 ? (ST == 0 ? 1u << 20 : 500000u) : ST == 0 ? 1u << 17 : 1u << 18) || nz < 4) return p;
  if ((uint64_t)nx * ny * sizeof(typename Store<ST>::S) >= 1ull << 32) return p;  // 32-bit byte offsets in a plane
  constexpr uint32_t sx = Sh::PX - 2;
  const uint32_t cx = (nx + sx - 1) / sx, tx = (nx + cx - 1) / cx;
  if (tx + 1 > nx || nx * 4 < cx * sx * 3) return p;  // a coordinate wraps at most once; too many idle columns
  // Rows and chunks: 256 workgroups run at a time, one of c planes takes c + 2
  // iterations and about one to start, and an iteration takes a time in
  // proportion to the wavefronts of the workgroup; in FP64 ten of them, three on
  // two of the SIMDs, take a little more.  (D3Q27 FP32 192^3: 20 rows 467, 16
  // rows 493, 13 rows 517 us for two steps; 201 x 117 x 83: 158, 177, 154; D3Q19
  // FP64 256^3: - , 1154, 1221; 201 x 117 x 83: - , 177, 145.)
  constexpr uint32_t rows[4] = {Sh::PY - 2, 16, 13, 0};
  uint64_t best = ~0ull;
  for (uint32_t sy : rows) {
    if (sy == 0 || sy > (uint32_t)Sh::PY - 2) continue;
    const uint32_t cy = (ny + sy - 1) / sy, ty = (ny + cy - 1) / cy;
    if (ty + 1 > ny || ty * 4 < sy * 3) continue;
    const uint32_t waves = (Sh::PX * (ty + 2) + 63) / 64;
    const uint32_t weight = 2 * waves + (ST == 0 && waves % 4 == 2);
    for (uint32_t c = 1; c <= nz; ++c) {
      const uint32_t chunk = (nz + c - 1) / c;
      const uint64_t groups = (uint64_t)cx * cy * ((nz + chunk - 1) / chunk);
      const uint64_t cost = (groups + 255) / 256 * (chunk + 3) * weight;
      if (cost < best) {
        best = cost;
        p = {{tx, ty}, chunk, waves * 64};
      }
      if (groups > 4096) break;
    }
  }
  return p;
}

// Whether the walled instances exist: the others have no registers left for the
// values more (D3Q19 FP64 spills 88 of them, D3Q27 FP32 18).
constexpr bool slide_walls(int q, int eb) { return q == 19 && eb == 4; }

// KEEP: the state between the two steps is stored too (g.keep); an instance of
// its own, as testing for it took ten registers (D3Q27 FP32 192^3: 480 -> 533 us).
// WALLS: half-way bounce-back on both faces of the x or y axis (not z).  A value
// whose source lies beyond a wall is the node's own opposite one of the same
// plane: step one reads it instead of the shifted value, step two finds it in
// the LDS copy of plane p - 1 or, for c_z > 0 (its opposite has one copy only,
// by now plane p's), in registers kept from the previous iteration.  D3Q19 256^3
// FP32, walls on the y faces: 703 us for two steps, 2 x 434 by single ones (592
// without walls: the tiles along a wall are the slowest of the one round).  Wall
// terms formed on the host and read from the arguments cost 7 % (scalar loads and
// spills in the wall wavefronts), a scatter of its own for the others 1 %.
template <class B, int ST, int MODE, bool KEEP, bool WALLS>
__global__ __launch_bounds__((SlideShape<B, ST>::threads)) void k_slide(StepArgs<typename Store<ST>::T> a, SlideArgs g) {
  using L = typename B::Lat;
  using S = typename Store<ST>::S;
  using T = typename Store<ST>::T;
  using SL = SlideSlots<B>;
  constexpr int Q = B::Q;
  constexpr int D = L::D;
  constexpr int PX = SlideShape<B, ST>::PX, PY = SlideShape<B, ST>::PY, R = PX * PY;
  constexpr uint32_t E = sizeof(S);
  __shared__ S lf[SL::count * R];

  const int nx = (int)a.nx, ny = (int)a.ny, nz = (int)a.nz;
  const uint64_t N = a.N, plane = (uint64_t)nx * ny;
  const uint3 tile = block_tile(a.xcd_remap);
  const int tid = (int)threadIdx.x;
  const int iy = tid / PX, ix = tid - iy * PX;
  const int tx = (int)g.t[0], ty = (int)g.t[1];
  // this thread's column, wrapped once; threads beyond the region take column 0
  // and keep nothing
  int x = (int)tile.x * tx + ix - 1, y = (int)tile.y * ty + iy - 1;
  const bool column = ix < tx + 2 && iy < ty + 2;
  const bool owned = ix >= 1 && ix <= tx && iy >= 1 && iy <= ty && x < nx && y < ny;
  x += x < 0 ? nx : 0;
  x -= x >= nx ? nx : 0;
  y += y < 0 ? ny : 0;
  y -= y >= ny ? ny : 0;
  x = column ? x : 0;
  y = column ? y : 0;
  const int z0 = (int)tile.z * (int)g.chunk;
  const int z1 = z0 + (int)g.chunk < nz ? z0 + (int)g.chunk : nz;  // planes z0 .. z1 - 1 are stored
  auto wrapz = [&](int z) { return z < 0 ? z + nz : (z >= nz ? z - nz : z); };
  // Addresses: a uniform base per population and plane plus a 32-bit byte
  // offset in the plane.  The empty asm statements keep the compiler from
  // hoisting Q 64-bit addresses per thread out of the plane loop (168 VGPRs and
  // spills without them, 95 with) and 2 Q bases into scalar registers.
  const uint32_t at = E * ((uint32_t)y * nx + (uint32_t)x);
  const bool x_lo = x == 0, x_hi = x == nx - 1, y_lo = y == 0, y_hi = y == ny - 1;
  struct Steps {
    uint32_t xm, xp, ym, yp;  // byte offsets to the neighbours along one axis
  };
  auto steps_of = [&]() -> Steps {
    uint32_t wx = E * (uint32_t)(nx - 1), wy = E * (uint32_t)nx * (uint32_t)(ny - 1), sy = E * (uint32_t)nx;
    asm volatile("" : "+s"(wx), "+s"(wy), "+s"(sy));
    return Steps{x_lo ? wx : 0u - E, x_hi ? 0u - wx : E, y_lo ? wy : 0u - sy, y_hi ? 0u - wy : sy};
  };

  // Walls: whether the link from x - c_j to this column's nodes passes one on
  // the x axis, or else on the y axis, and the bounced value (as bounce() of
  // kernels.hpp).  Both faces' terms are formed from uniform values and one is
  // picked per lane: a load of the lane's own face would have to wait for the
  // prefetched plane behind it (D3Q19 256^3 channel: 963 us for two steps).
  // The mask is opaque, so that nothing formed from it stays in the registers
  // of the plane loop.
  auto walls_now = [&]() -> uint32_t {
    uint32_t mask = a.wall_mask;
    if constexpr (WALLS) asm volatile("" : "+v"(mask));
    return mask;
  };
  auto wall_on = [&](auto jj, auto axis, uint32_t mask) -> bool {
    constexpr int c = decltype(axis)::value == 0 ? L::c[jj].x : L::c[jj].y;
    if constexpr (!WALLS || c == 0) return false;
    else if constexpr (decltype(axis)::value == 0) return c > 0 ? x_lo && (mask & 1u) : x_hi && (mask & 2u);
    else return c > 0 ? y_lo && (mask & 4u) : y_hi && (mask & 8u);
  };
  constexpr std::integral_constant<int, 0> x_axis{};
  constexpr std::integral_constant<int, 1> y_axis{};
  auto walled = [&](auto jj, uint32_t mask) -> bool { return wall_on(jj, x_axis, mask) || wall_on(jj, y_axis, mask); };
  auto bounced = [&](auto jj, uint32_t mask, T reflected) -> T {
    constexpr int J = jj;
    constexpr int fx = L::c[J].x > 0 ? 0 : 1, fy = L::c[J].y > 0 ? 2 : 3;
    const T via_x = bounce<B, T, J>(a.wall_coef, fx, reflected), via_y = bounce<B, T, J>(a.wall_coef, fy, reflected);
    return wall_on(jj, x_axis, mask) ? via_x : via_y;
  };
  // whether any column of this wavefront lies at a wall: the others take the
  // plain code
  const bool at_wall = WALLS && __any((x_lo && (a.wall_mask & 1u)) || (x_hi && (a.wall_mask & 2u)) ||
                                      (y_lo && (a.wall_mask & 4u)) || (y_hi && (a.wall_mask & 8u)));

  auto load = [&](int p, T (&h)[Q], T (&u)[3]) {
    const int z = wrapz(p), zm = wrapz(z - 1), zp = wrapz(z + 1);
    const uint64_t bz = (uint64_t)z * plane, bm = (uint64_t)zm * plane, bp = (uint64_t)zp * plane;
    uint64_t stride = N * E;
    asm volatile("" : "+s"(stride));
    const char* pop = static_cast<const char*>(a.fin);
    if (g.gather) {
      const Steps d = steps_of();
      auto gather = [&](auto near) {
        const uint32_t mask = walls_now();
        sfor<Q>([&](auto jj) {
          constexpr int cx = L::c[jj].x, cy = L::c[jj].y, cz = L::c[jj].z;
          uint32_t n = at + (cy > 0 ? d.ym : cy < 0 ? d.yp : 0u) + (cx > 0 ? d.xm : cx < 0 ? d.xp : 0u);
          asm volatile("" : "+v"(n));
          const char* from = pop + E * (cz > 0 ? bm : cz < 0 ? bp : bz) + n;
          if constexpr (decltype(near)::value) {
            if (walled(jj, mask))  // the moving wall's term is added where the value is used
              from = static_cast<const char*>(a.fin) + (uint64_t)opposite<L>(jj) * stride + E * bz + at;
          }
          h[jj] = T(*reinterpret_cast<const S*>(from));
          pop += stride;
        });
      };
      if (at_wall) gather(std::true_type{});
      else gather(std::false_type{});
    } else {
      uint32_t n = at;
      asm volatile("" : "+v"(n));
      pop += E * bz;
      sfor<Q>([&](auto jj) {
        h[jj] = T(*reinterpret_cast<const S*>(pop + n));
        pop += stride;
      });
    }
    if constexpr (MODE == UT_FIELD) {
      sfor<D>([&](auto al) { u[al] = T(a.ut[(uint64_t)al * N + bz + at / E]) * a.inv_lambda; });
    }
  };

  T hn[Q], un[3] = {T(0), T(0), T(0)}, up[3] = {T(0), T(0), T(0)};  // next plane; u~ of the previous one
  S c0 = S(0), cu1 = S(0), cu2 = S(0), cd = S(0);  // own column: rest, +z of the last two planes, -z
  S own_dn[Q];  // WALLS: this column's values with c_z < 0 of the previous plane
  load(z0 - 1, hn, un);
  int k = 0, k3 = 0;  // planes so far, and modulo 3
  for (int p = z0 - 1; p <= z1; ++p) {
    // LDS copies written (planes p) and read (planes p - 1 and p - 2)
    const int w0 = (k & 1) * R, r0 = ((k & 1) ^ 1) * R, wu = k3 * R, ru = (k3 == 2 ? 0 : k3 + 1) * R;
    T h[Q], uc[3] = {T(0), T(0), T(0)};
    sfor<Q>([&](auto jj) { h[jj] = hn[jj]; });
    sfor<3>([&](auto al) { uc[al] = un[al]; });
    if constexpr (WALLS) {
      if (at_wall && g.gather) {
        const uint32_t mask = walls_now();
        sfor<Q>([&](auto jj) {
          h[jj] = walled(jj, mask) ? bounced(jj, mask, h[jj]) : h[jj];
        });
      }
    }
    collide_node<B, T, MODE, 0>(h, a, uc);
    S o[Q];
    sfor<Q>([&](auto jj) { o[jj] = S(h[jj]); });
    if (column) {
      sfor<Q>([&](auto jj) {
        constexpr int J = jj;
        if constexpr (!SL::axis(J)) lf[SL::base(J) * R + (L::c[J].z < 0 ? 0 : L::c[J].z == 0 ? w0 : wu) + tid] = o[J];
      });
    }
    const S rest = c0, up2 = cu2;
    sfor<Q>([&](auto jj) {
      constexpr int J = jj;
      if constexpr (SL::axis(J) && L::c[J].z == 0) c0 = o[J];
      if constexpr (SL::axis(J) && L::c[J].z > 0) {
        cu2 = cu1;
        cu1 = o[J];
      }
      if constexpr (SL::axis(J) && L::c[J].z < 0) cd = o[J];
    });
    if (p < z1) load(p + 1, hn, un);
    __syncthreads();
    const int z = p - 1;
    if (p > z0 && owned) {
      sfor<Q>([&](auto jj) {
        constexpr int J = jj;
        if constexpr (SL::axis(J)) {
          h[J] = T(L::c[J].z == 0 ? rest : L::c[J].z > 0 ? up2 : cd);
        } else {
          h[J] = T(lf[SL::base(J) * R - L::c[J].y * PX - L::c[J].x + (L::c[J].z < 0 ? 0 : L::c[J].z == 0 ? r0 : ru) + tid]);
        }
      });
      if constexpr (WALLS) {
        if (at_wall) {
          const uint32_t mask = walls_now();
          sfor<Q>([&](auto jj) {
            constexpr int J = jj, O = opposite<L>(J);
            if constexpr (!SL::axis(J)) {
              const S back = L::c[J].z > 0
                                 ? own_dn[O]
                                 : lf[SL::base(O) * R + (L::c[J].z == 0 ? r0 : (k3 == 0 ? 2 : k3 - 1) * R) + tid];
              h[J] = walled(jj, mask) ? bounced(jj, mask, T(back)) : h[J];
            }
          });
        }
      }
    }
    if constexpr (WALLS) {
      sfor<Q>([&](auto jj) {
        if constexpr (L::c[jj].z < 0 && !SL::axis(jj)) own_dn[jj] = o[jj];
      });
    }
    __syncthreads();
    if (p > z0 && owned) {
      if constexpr (KEEP) {
        uint64_t stride = N * E;
        asm volatile("" : "+s"(stride));
        char* pop = static_cast<char*>(g.keep) + E * ((uint64_t)z * plane);
        uint32_t n = at;
        asm volatile("" : "+v"(n));
        sfor<Q>([&](auto jj) {
          __builtin_nontemporal_store(S(h[jj]), reinterpret_cast<S*>(pop + n));
          pop += stride;
        });
      }
      collide_node<B, T, MODE, 0>(h, a, up);
      sfor<Q>([&](auto jj) { o[jj] = S(h[jj]); });
      const int zm = wrapz(z - 1), zp = wrapz(z + 1);
      const uint64_t bz = (uint64_t)z * plane, bm = (uint64_t)zm * plane, bp = (uint64_t)zp * plane;
      uint64_t stride = N * E;
      asm volatile("" : "+s"(stride));
      char* pop = static_cast<char*>(a.fout);
      if (g.scatter) {
        const Steps d = steps_of();
        const uint32_t mask = walls_now();
        sfor<Q>([&](auto jj) {
          constexpr int cx = L::c[jj].x, cy = L::c[jj].y, cz = L::c[jj].z;
          uint32_t n = at + (cy < 0 ? d.ym : cy > 0 ? d.yp : 0u) + (cx < 0 ? d.xm : cx > 0 ? d.xp : 0u);
          asm volatile("" : "+v"(n));
          constexpr int O = opposite<L>(jj);
          constexpr std::integral_constant<int, O> oo{};
          if (walled(oo, mask))  // the destination lies beyond a wall: back to this node
            *reinterpret_cast<S*>(static_cast<char*>(a.fout) + (uint64_t)O * stride + E * bz + at) =
                S(bounced(oo, mask, T(o[jj])));
          else *reinterpret_cast<S*>(pop + E * (cz < 0 ? bm : cz > 0 ? bp : bz) + n) = o[jj];
          pop += stride;
        });
      } else {
        uint32_t n = at;
        asm volatile("" : "+v"(n));
        pop += E * bz;
        sfor<Q>([&](auto jj) {
          *reinterpret_cast<S*>(pop + n) = o[jj];
          pop += stride;
        });
      }
    }
    sfor<3>([&](auto al) { up[al] = uc[al]; });
    ++k;
    k3 = k3 == 2 ? 0 : k3 + 1;
  }
}

}  // namespace lbmrv
