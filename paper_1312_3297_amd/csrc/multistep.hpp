// Several time steps per launch, a tile at a time in LDS (k_tile).
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

// The region of k_tile (tile and ring), PX x PY x PZ nodes, and the most
// threads of a workgroup (FP64 D3Q19 and D3Q27 need more than the 128 registers
// that 1024 threads leave).  Fixed extents make every LDS offset of the unrolled
// population loops an immediate: with run-time pitches the kernel spilled scalar
// registers and took 11.5 instead of 9.7 us for eight steps of D2Q9 64^2 FP32.
// 2-D: 40 x 40 FP32 nodes are 57.6 KB, two workgroups per CU; 48 x 48 (one per
// CU) ran 20 % slower at 1024^2, and FP64's 28 x 28 (two per CU) 5 % slower than
// its 40 x 40 (one).  3-D: with u~ a field 158 KB for D3Q19 FP32, 147 KB for
// FP64, 146 KB for D3Q27 FP64, of the CU's 160.
template <class B, int ST>
struct TileShape {
  static constexpr bool plane = B::Lat::D == 2, q27 = B::Q == 27;
  static constexpr int PX = plane ? 40 : q27 ? 10 : ST == 0 ? 14 : 18;
  static constexpr int PY = plane ? 40 : q27 || ST == 0 ? 8 : 10;
  static constexpr int PZ = plane ? 1 : q27 || ST == 0 ? 8 : 10;
  static constexpr int threads = !plane && (q27 || ST == 0) ? 512 : 1024;
  static constexpr int nodes = PX * PY * PZ;
};

struct TileArgs {
  uint32_t steps;    // 1 .. kTileMaxSteps
  uint32_t t[3];     // tile extents, t[a] + 2 (steps - 1) <= region extent
  uint32_t gather;   // 1: fin holds post-collision values, the first step gathers from x - c_j
  uint32_t scatter;  // 1: the last step stores at x + c_j (pre-collision result), 0: at the node
  // step s covers e = t + 2 (steps - 1 - s) nodes along each axis: reciprocals
  // of e[0] (2^18 / e, rounded up) and of e[0] e[1] (2^22 / e, rounded up), exact
  // for the node numbers of a region (below 2^18 / e[0] and 2^22 / (e[0] e[1]))
  uint32_t mx[kTileMaxSteps];
  uint32_t mxy[kTileMaxSteps];
  void* keep;            // KEEP: where the states between the steps go, the state
  uint64_t keep_stride;  // before step s (s >= 1) at keep + (s - 1) keep_stride, in elements
};

// Tile and step count for a grid; steps < 2: single steps (or k_slide) are the
// better choice.  The tile plus its ring must fit in one period of the grid
// (t + steps - 1 <= extent), so that a coordinate wraps at most once.
struct TilePlan {
  uint32_t t[3];
  uint32_t steps;    // most steps per launch
  uint32_t threads;
};

// Equal tiles of at most side[a] nodes (no nearly empty last row) and as many
// steps, up to p.steps, as the ring leaves room for; false if fewer than two.
inline bool fit_tile(TilePlan& p, int d, const uint32_t (&n)[3], const uint32_t (&side)[3]) {
  for (int a = 0; a < d; ++a) {
    const uint32_t c = (n[a] + side[a] - 1) / side[a];
    p.t[a] = (n[a] + c - 1) / c;
    if (p.t[a] + p.steps - 1 > n[a]) p.steps = n[a] - p.t[a] + 1;
  }
  if (p.steps < 2) p.steps = 0;
  return p.steps != 0;
}

template <class B, int ST>
TilePlan plan_tile(uint32_t nx, uint32_t ny, uint32_t nz) {
  using Sh = TileShape<B, ST>;
  const uint32_t n[3] = {nx, ny, nz};
  TilePlan p{{1, 1, 1}, 0, 0};
  if constexpr (B::Lat::D == 2) {
    // Large tiles waste less on the ring (32 x 32, 5 steps: 27 % more node
    // steps; 16 x 16: 57 %), small ones keep the 256 CUs busy on small grids, more
    // steps take fewer launches.  The plan is the one of least cost per step, in
    // units of a wavefront's pass over one region node per lane (62 ns FP32, 80 ns
    // FP64): 64 for a launch that fills at most one workgroup per CU, or 72 per
    // round for its loads and stores, 5 per step, and the wavefronts of all steps;
    // two workgroups that share a CU hide a quarter of each other's time.  Within
    // 8 % of what these measured, us per step, FP32 (tile, steps): 256^2 (16 x 16,
    // 7) 1.37, 384^2 (24 x 24, 7) 1.79 and (16 x 16, 7) 2.6, 512^2 (32 x 32, 5)
    // 2.38, 640^2 (30 x 30, 6) 3.3 and (32 x 32, 5) 3.6, 724^2 (28 x 28, 7) 4.3 and
    // (32 x 32, 5) 5.1, 1024^2 (32 x 32, 5) 6.6 and (30 x 30, 6) 7.1.  The search
    // takes some 10 us: once per context.
    // A wide grid of few rows leaves room for low tiles only (t + steps - 1 <= ny),
    // a launch of which moves little and mostly waits; there a single step, 3.5 us
    // and its bytes at 5.8 TB/s (64 lanes to a row of fewer nodes), may be less.
    // The unit above is 72 ns FP64, 59 FP32 and 31 FP16 over such grids (FP16
    // regions share a CU by more than two).  us per step, single | tiles: FP64
    // 77792 x 5 12.0 | 21.9, 286424 x 8 (a field) 59.6 | 99, 30656 x 13 12.8 | 11.2,
    // FP32 353696 x 7 32 | 51, 58642 x 15 14.3 | 15.1, 29764 x 10 6.3 | 6.0, FP16
    // 320184 x 5 14.9 | 23.0, 35600 x 13 6.1 | 5.3, 31016 x 30 9.0 | 6.4.
    constexpr bool shared = ST != 0;  // two workgroups fit in a CU's LDS
    constexpr uint32_t sides[] = {32, 30, 28, 24, 20, 16, 12, 8, 4};  // of equal plans the widest in x
    double best = 1e300;
    for (uint32_t sx : sides)
      for (uint32_t sy : sides) {
        const uint32_t cx = (nx + sx - 1) / sx, cy = (ny + sy - 1) / sy;
        const uint32_t tx = (nx + cx - 1) / cx, ty = (ny + cy - 1) / cy;  // no nearly empty last row
        if (cx >= 1u << 22) continue;  // a launch holds fewer than 2^32 work-items along x
        const uint64_t rounds = ((uint64_t)cx * cy + 255) / 256;
        double waves = 0;
        for (uint32_t k = 1; k <= kTileMaxSteps; ++k) {
          const uint32_t r = 2 * (k - 1), region = (tx + r) * (ty + r);
          if (tx + r > (uint32_t)Sh::PX || ty + r > (uint32_t)Sh::PY || tx + k - 1 > nx || ty + k - 1 > ny) break;
          waves += (region + 63) / 64;
          if (k < 2) continue;
          const double work = rounds == 1 ? 64 + waves : (72 + waves) * (double)rounds * (shared ? 0.75 : 1.0);
          const double cost = (work + 5.0 * k) / k;
          if (cost < best) {
            best = cost;
            p = {{tx, ty, 1}, k, region < 1024 ? (region + 63) / 64 * 64 : 1024u};
          }
        }
      }
    constexpr double unit = ST == 0 ? 0.072 : ST == 1 ? 0.059 : 0.031;  // us
    const double bytes = 2.0 * B::Q * sizeof(typename Store<ST>::S) * ny * (nx < 64 ? 64 : nx);
    if (unit * best >= 3.5 + bytes / 5.8e6) p.steps = 0;
    return p;
  } else {
    // In space the ring is dear (16 x 8 x 8, two steps: 38 % more node steps;
    // 4 x 4 x 4, three: 4.2 times as many), which only pays while a pass is bound
    // by its launch and latency: the smallest tile that at most 256 workgroups,
    // one per CU, cover the grid with, and no such tile beyond that.  Measured, us
    // per step, single | fused:
    //   D3Q19 FP32  16^3 5.1 | 2.6  32^3 5.2 | 3.2  48^3 5.9 | 5.0  64^3 9.0 | 7.0
    //   D3Q19 FP64  16^3 6.5 | 3.0  32^3 6.0 | 4.4  48^3 10.4 | 7.3
    //   D3Q27 FP32  16^3 6.0 | 4.2  32^3 5.5 | 4.8  48^3 7.2 | 7.4
    // and of FP16 and D3Q27 FP64, us per step of single scatter passes, the fastest of
    // the single steps | by launches of the most steps, u~ = u:
    //   D3Q19 FP16  9 x 8 x 8 3.9 | 2.5  16^3 3.9 | 2.5  32^3 3.8 | 3.3  48^3 5.1 | 4.3
    //   D3Q27 FP16  9 x 8 x 8 4.3 | 3.5  16^3 4.3 | 3.5  27 x 25 x 20 4.2 | 3.7
    //   D3Q27 FP64  9 x 8 x 8 5.1 | 4.3  16^3 5.3 | 4.5  27 x 25 x 20 5.2 | 5.3
    // A fused pass takes its time however many of the 256 CUs it fills, a single
    // one less on a smaller grid, hence the least nodes of the larger tiles: D3Q19
    // FP32 101 x 49 x 15 (12 x 6 x 6) 4.9 | 5.9, 64 x 20 x 73 (16 x 8 x 8) 4.8 |
    // 6.4, FP64 45 x 22 x 49 (12 x 6 x 6) 5.4 | 6.4, D3Q27 FP64 32 x 29 x 17 (8 x
    // 4 x 4) 5.5 | 6.3, FP16 with a field 32 x 10 x 53 4.0 | 4.6.
    struct Side {
      uint32_t s[3];
      uint32_t steps;
      uint64_t least;
    };
    constexpr bool f64 = ST == 0, q27 = B::Q == 27;
    const Side sides[4] = {{{4, 4, 4}, q27 ? 2u : 3u, 0},
                           {{8, 4, 4}, q27 || f64 ? 2u : 4u, q27 && ST != 1 ? ~0ull : 0},
                           {{12, 6, 6}, 2u, f64 ? 1u << 16 : 5u << 14},
                           {{16, 8, 8}, 2u, 9u << 14}};
    for (const Side& c : sides) {
      const uint32_t r = 2 * (c.steps - 1);
      if (c.s[0] + r > (uint32_t)Sh::PX || c.s[1] + r > (uint32_t)Sh::PY || c.s[2] + r > (uint32_t)Sh::PZ) break;
      // FP16 gains nothing beyond 12 x 6 x 6 (64^3: 7.0 against 7.5 us per step)
      if (ST == 2 && c.s[0] > 12u) break;
      uint64_t groups = 1;
      for (int a = 0; a < 3; ++a) groups *= (n[a] + c.s[a] - 1) / c.s[a];
      if (groups > 256) continue;
      if ((uint64_t)nx * ny * nz < c.least) return p;
      p.steps = c.steps;
      if (!fit_tile(p, 3, n, c.s)) return p;
      const uint32_t q = 2 * (p.steps - 1), region = (p.t[0] + q) * (p.t[1] + q) * (p.t[2] + q);
      const uint32_t most = Sh::threads;
      p.threads = region > 1024u ? 768u : (region + 63) / 64 * 64;
      if (p.threads > most) p.threads = most;
      return p;
    }
    return p;
  }
}

// Threads per workgroup where the grid has more than 256 tiles, at most the
// plan's.  One workgroup per CU wants a thread per region node, and so do two
// whose waves all fit; with u~ a field (FP32) two of 768 do better, and FP16,
// whose regions leave room for three or four workgroups, takes 512.  2-D, us per
// launch with 1024 | 768 | 512 threads: FP32 u~ = u 1024^2 29.9 | 31.0 | -, a
// field 40.1 | 32.4 | 34.7; FP16 u~ = 0 2048^2 99 | 103 | 90, a field 151 | 118 |
// 108; FP64 a field 61.4 | 62.3 | 66.9.
template <int D, int ST, int MODE>
constexpr uint32_t tile_threads_shared() {
  return D != 2 || ST == 0 ? 1024u : ST == 2 ? 512u : MODE == UT_FIELD ? 768u : 1024u;
}

template <class B, int ST, int MODE>
constexpr size_t tile_lds_bytes() {
  constexpr size_t R = TileShape<B, ST>::nodes;
  constexpr size_t f = (B::Q * R * sizeof(typename Store<ST>::S) + 15) / 16 * 16;
  return f + (MODE == UT_FIELD ? B::Lat::D * R * sizeof(float) : 0);
}

// KEEP: the states between the steps are stored too (g.keep); an instance of
// its own, as testing for it at every node cost the plain one 9 %.
template <class B, int ST, int MODE, int RLX, bool KEEP>
__global__ __launch_bounds__((TileShape<B, ST>::threads)) void k_tile(StepArgs<typename Store<ST>::T> a, TileArgs g) {
  using L = typename B::Lat;
  using S = typename Store<ST>::S;
  using T = typename Store<ST>::T;
  using Sh = TileShape<B, ST>;
  constexpr int Q = B::Q;
  constexpr int D = L::D;
  constexpr int P = Sh::PX, P2 = Sh::PX * Sh::PY, R = Sh::nodes;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  S* lf = reinterpret_cast<S*>(lds_raw);
  float* lu = reinterpret_cast<float*>(lds_raw + tile_lds_bytes<B, ST, UT_ZERO>());

  const int nx = (int)a.nx, ny = (int)a.ny, nz = (int)a.nz;
  const uint64_t N = a.N;
  const S* fin = static_cast<const S*>(a.fin);
  S* fout = static_cast<S*>(a.fout);
  const uint3 tile = block_tile(a.xcd_remap);
  const int steps = (int)g.steps;
  const int x0 = (int)(tile.x * g.t[0]), y0 = (int)(tile.y * g.t[1]), z0 = (int)(tile.z * g.t[2]);

  for (int s = 0; s < steps; ++s) {
    const int ring = steps - 1 - s;
    const uint32_t ex = g.t[0] + 2 * ring, exy = ex * (g.t[1] + 2 * ring);
    const uint32_t count = D == 3 ? exy * (g.t[2] + 2 * ring) : exy;
    const uint32_t mx = g.mx[s], mxy = g.mxy[s];
    for (uint32_t i = threadIdx.x; i < count; i += blockDim.x) {
      uint32_t iz = 0, r = i;
      if constexpr (D == 3) {
        iz = __umul24(i, mxy) >> 22;
        r = i - __umul24(iz, exy);
      }
      const uint32_t iy = __umul24(r, mx) >> 18, ix = r - __umul24(iy, ex);
      int l = (int)__umul24(iy + s, P) + (int)ix + s;
      if constexpr (D == 3) l += (int)__umul24(iz + s, P2);
      T h[Q];
      T utf[3] = {T(0), T(0), T(0)};
      int x = 0, y = 0, z = 0;
      bool inside = false;
      if (KEEP || s == 0 || ring == 0) {
        x = x0 - ring + (int)ix;
        y = y0 - ring + (int)iy;
        inside = x < nx && y < ny;
        // before the last step: nodes of the tile itself, not of its ring
        if constexpr (KEEP) inside = inside && ix - ring < g.t[0] && iy - ring < g.t[1] && (D == 2 || iz - ring < g.t[2]);
        x += x < 0 ? nx : 0;
        x -= x >= nx ? nx : 0;
        y += y < 0 ? ny : 0;
        y -= y >= ny ? ny : 0;
        if constexpr (D == 3) {
          z = z0 - ring + (int)iz;
          inside = inside && z < nz;
          z += z < 0 ? nz : 0;
          z -= z >= nz ? nz : 0;
        }
      }
      // node offset of x + dir c_j, or the node itself where the launch does not shift
      auto node = [&](auto jj, auto dirc, int shifted) -> uint32_t {
        constexpr int cx = decltype(dirc)::value * L::c[jj].x, cy = decltype(dirc)::value * L::c[jj].y,
                      cz = decltype(dirc)::value * L::c[jj].z;
        int xx = x, yy = y, zz = z;
        if (shifted) {
          if constexpr (cx > 0) xx = x == nx - 1 ? 0 : x + 1;
          if constexpr (cx < 0) xx = x == 0 ? nx - 1 : x - 1;
          if constexpr (cy > 0) yy = y == ny - 1 ? 0 : y + 1;
          if constexpr (cy < 0) yy = y == 0 ? ny - 1 : y - 1;
          if constexpr (cz > 0) zz = z == nz - 1 ? 0 : z + 1;
          if constexpr (cz < 0) zz = z == 0 ? nz - 1 : z - 1;
        }
        return D == 3 ? ((uint32_t)zz * ny + (uint32_t)yy) * nx + (uint32_t)xx : (uint32_t)yy * nx + (uint32_t)xx;
      };
      if (s == 0) {
        const int shifted = g.gather ? 1 : 0;
        // the population's base moves on by an opaque stride: as loop invariants
        // the 2 Q bases of fin and fout overflow the scalar registers
        uint64_t stride = N;
        asm volatile("" : "+s"(stride));
        const S* pop = fin;
        sfor<Q>([&](auto jj) {
          h[jj] = T(pop[node(jj, std::integral_constant<int, -1>{}, shifted)]);
          pop += stride;
        });
        if constexpr (MODE == UT_FIELD) {
          const uint32_t own = node(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{}, 0);
          sfor<D>([&](auto al) {
            const float v = a.ut[(uint64_t)al * N + own];
            lu[al * R + l] = v;
            utf[al] = T(v) * a.inv_lambda;
          });
        }
      } else {
        if (s & 1) {
          sfor<Q>([&](auto jj) {
            h[jj] = T(lf[l + (opposite<L>(jj) * R - L::c[jj].z * P2 - L::c[jj].y * P - L::c[jj].x)]);
          });
        } else {
          sfor<Q>([&](auto jj) { h[jj] = T(lf[l + jj * R]); });
        }
        if constexpr (MODE == UT_FIELD) {
          sfor<D>([&](auto al) { utf[al] = T(lu[al * R + l]) * a.inv_lambda; });
        }
        if (KEEP && inside) {
          const uint32_t own = node(std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{}, 0);
          uint64_t stride = N;
          asm volatile("" : "+s"(stride));
          S* pop = static_cast<S*>(g.keep) + (uint64_t)(s - 1) * g.keep_stride;
          sfor<Q>([&](auto jj) {
            __builtin_nontemporal_store(S(h[jj]), &pop[own]);
            pop += stride;
          });
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
          const int shifted = g.scatter ? 1 : 0;
          uint64_t stride = N;
          asm volatile("" : "+s"(stride));
          S* pop = fout;
          sfor<Q>([&](auto jj) {
            pop[node(jj, std::integral_constant<int, 1>{}, shifted)] = o[jj];
            pop += stride;
          });
        }
      } else if (s & 1) {
        sfor<Q>([&](auto jj) { lf[l + (jj * R + L::c[jj].z * P2 + L::c[jj].y * P + L::c[jj].x)] = o[jj]; });
      } else {
        sfor<Q>([&](auto jj) { lf[l + opposite<L>(jj) * R] = o[jj]; });
      }
    }
    if (ring) __syncthreads();
  }
}

// The whole grid in one workgroup, one thread per node, any number of steps in
// one launch: for grids of at most kClosedNodes nodes, where k_tile would spend
// most of its work on rings and still pay a launch every few steps.  The
// populations stay in LDS in the in-place form of k_tile, wrapped; the last
// step scatters to the natural layout.  Every load from fin comes before the
// first store to fout, so the two may be the same array.  A step costs the
// latency of one collision and one LDS exchange, which a second wavefront per
// SIMD hides half of; D2Q9 16^2 FP64, 50 steps: 32 us, and 82 by k_tile (7
// launches).  At 512 nodes, us for 20 steps, single steps | one launch: D2Q9 16 x 32
// FP64 78 | 21, D3Q19 8^3 FP32 82 | 29, FP16 86 | 30, D3Q27 8^3 FP32 91 | 44, FP16 104 |
// 45, FP64 (110 KB of LDS) 107 | 71; two steps of the last 14.9 | 10.3.
constexpr uint32_t kClosedNodes = 512;

template <class B, int ST, int MODE>
constexpr size_t closed_lds_bytes(size_t nodes) {
  return (B::Q * nodes * sizeof(typename Store<ST>::S) + 15) / 16 * 16;
}

template <class B, int ST, int MODE, int RLX>
__global__ __launch_bounds__(kClosedNodes) void k_closed(StepArgs<typename Store<ST>::T> a, uint64_t steps) {
  using L = typename B::Lat;
  using S = typename Store<ST>::S;
  using T = typename Store<ST>::T;
  constexpr int Q = B::Q;
  constexpr int D = L::D;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  S* lf = reinterpret_cast<S*>(lds_raw);

  const uint32_t nx = a.nx, ny = a.ny, nz = a.nz, n = (uint32_t)a.N;
  const bool active = threadIdx.x < n;
  const uint32_t own = active ? threadIdx.x : n - 1;  // idle threads start from the last node and write nothing
  const uint32_t x = own % nx, row = own / nx, y = D == 3 ? row % ny : row, z = D == 3 ? row / ny : 0;
  const uint32_t xm = x == 0 ? nx - 1 : x - 1, xp = x == nx - 1 ? 0 : x + 1;
  const uint32_t ym = y == 0 ? ny - 1 : y - 1, yp = y == ny - 1 ? 0 : y + 1;
  const uint32_t zm = z == 0 ? nz - 1 : z - 1, zp = z == nz - 1 ? 0 : z + 1;
  uint32_t at[Q];  // slot j of node x + c_j
  sfor<Q>([&](auto jj) {
    constexpr int cx = L::c[jj].x, cy = L::c[jj].y, cz = L::c[jj].z;
    const uint32_t xx = cx > 0 ? xp : cx < 0 ? xm : x, yy = cy > 0 ? yp : cy < 0 ? ym : y, zz = cz > 0 ? zp : cz < 0 ? zm : z;
    at[jj] = jj * n + (zz * ny + yy) * nx + xx;
  });

  const S* fin = static_cast<const S*>(a.fin);
  S* fout = static_cast<S*>(a.fout);
  T h[Q], utf[3] = {T(0), T(0), T(0)};
  sfor<Q>([&](auto jj) { h[jj] = T(fin[jj * n + own]); });
  if constexpr (MODE == UT_FIELD) {
    sfor<D>([&](auto al) { utf[al] = T(a.ut[al * n + own]) * a.inv_lambda; });
  }
  S o[Q];
  for (uint64_t s = 0;; ++s) {
    collide_node<B, T, MODE, RLX>(h, a, utf);
    sfor<Q>([&](auto jj) { o[jj] = S(h[jj]); });
    if (s + 1 == steps) break;
    const bool odd = (s & 1) != 0;
    if (active) {
      if (odd) sfor<Q>([&](auto jj) { lf[at[jj]] = o[jj]; });
      else sfor<Q>([&](auto jj) { lf[opposite<L>(jj) * n + own] = o[jj]; });
    }
    __syncthreads();
    if (active) {
      if (odd) sfor<Q>([&](auto jj) { h[jj] = T(lf[jj * n + own]); });
      else sfor<Q>([&](auto jj) { h[jj] = T(lf[at[opposite<L>(jj)]]); });
    }
  }
  __syncthreads();  // one step: every load before the first store
  if (active) sfor<Q>([&](auto jj) { fout[at[jj]] = o[jj]; });
}

}  // namespace lbmrv
