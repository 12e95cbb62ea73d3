// Several steps of a D2Q9 grid in one pass over memory.
//
// A workgroup takes a tile of OX x OY cells: it pulls and collides the tile
// and a halo of T - 1 cells from the state at t, keeps the result in LDS, and
// repeats from there on a region one cell smaller on every side until the
// tile itself holds the state at t + T, which it stores.  Every cell's step
// is the one-step sweep's own (walls, open faces, layers, inlet cells), so
// the values are bitwise those of T single steps.  Four steps ask for
// (1 + 6/64)(1 + 6/8) = 1.91 times q values per cell, which L2 serves but for the
// first, and write q: 18.2 B per update reach HBM (4000 x 3001 periodic FP32, 18 B
// without a halo), a quarter of a one-step sweep's.  Then the vector
// instructions bound it: at four cycles each and 2.4 GHz they fill 76 % of a
// pass's 283 us, with HBM at 3.1 TB/s (170k MLUPS; one-step sweep 81k at 5.8 TB/s).  Two
// steps on the general path (cylinder channel 2048 x 1024 FP32): 58 % of 36.5 us, 4.2 TB/s.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "kernels.hpp"
#include "launch.hpp"
#include "sweep.hpp"

namespace hrlbm {

template <int T_, int OX_, int OY_>
struct Tile2 {
  static constexpr int T = T_, OX = OX_, OY = OY_, H = T - 1;
  static constexpr int RX = OX + 2 * H, RY = OY + 2 * H, SLOTS = RX * RY;
  // with more than two steps, two LDS states alternate
  static constexpr int NB = T > 2 ? 2 : 1;
};

// Face rules and bounce-back of a cell whose neighbours are in LDS: `cell` is
// its slot of population 0, `mask` its slot of the mask, rows RX apart and
// populations SLOTS apart (see pull_fixup).
template <class L, class S, int RX, int SLOTS>
__device__ __forceinline__ void lds_fixup(const SweepArgs<S>& a, uint32_t x, uint32_t y,
                                          const typename S::T* cell, const uint8_t* mask,
                                          bool near_solid, typename S::T raw[L::Q]) {
  const bool on[2][2] = {{a.face[0] != kPeriodic && any_lane(x == 0),
                          a.face[1] != kPeriodic && any_lane(x + 1 == a.nx)},
                         {a.face[2] != kPeriodic && any_lane(y == 0),
                          a.face[3] != kPeriodic && any_lane(y + 1 == a.ny)}};
  const bool any_solid = any_lane(near_solid);
  static_for<1, L::Q>([&](auto I) {
    constexpr int i = decltype(I)::value;
    constexpr Dir v = L::dir(i);
    bool reach = any_solid;
    if constexpr (v.x != 0) reach = reach || on[0][v.x < 0];
    if constexpr (v.y != 0) reach = reach || on[1][v.y < 0];
    if (!reach) return;
    int dx = -v.x, dy = -v.y;
    bool fx = false, fy = false, cross = false;
    if constexpr (v.x != 0) {
      const int f = v.x > 0 ? 0 : 1;
      if ((v.x > 0 ? x == 0 : x + 1 == a.nx) && a.face[f] != kPeriodic) {
        dx = 0;
        fx = a.face[f] == kFreeSlip;
        cross = true;
      }
    }
    if constexpr (v.y != 0) {
      const int f = v.y > 0 ? 2 : 3;
      if ((v.y > 0 ? y == 0 : y + 1 == a.ny) && a.face[f] != kPeriodic) {
        dy = 0;
        fy = a.face[f] == kFreeSlip;
        cross = true;
      }
    }
    const int off = dx + dy * RX;
    if (near_solid && (mask[off] & kKindBits) == kSolid) {
      raw[i] = cell[opposite<L>(i) * SLOTS];
    } else if (cross) {
      raw[i] = cell[flipped<L, i>(fx, fy, false) * SLOTS + off];
    }
  });
}

// The steps of one tile.  kInside: the tile is whole and every cell its steps
// read lies in the grid, so that nothing wraps and no lane is idle at an edge
// (the arithmetic bounds these kernels: 4000 x 3001 FP32 75 us a step with the
// wrap and edge tests in every tile, 69 without; FP16S 50 / 49; a serving quantum of 12
// jobs 7.02 / 6.84 ms).
template <class L, class S, bool kGeneral, bool kInside, class G>
__device__ __forceinline__ void multi2d_tile(const SweepArgs<S>& a, uint32_t bx, uint32_t by,
                                             typename S::T* lds, uint8_t* lmask, uint32_t tid,
                                             uint32_t nthreads) {
  using T = typename S::T;
  using R = typename S::R;
  constexpr int Q = L::Q;
  const int32_t nx = (int32_t)a.nx, ny = (int32_t)a.ny;
  const int32_t x0 = (int32_t)bx * G::OX, y0 = (int32_t)by * G::OY;
  const int32_t wx = min(G::OX, nx - x0), wy = min(G::OY, ny - y0);
  const bool px = !kGeneral || a.face[0] == kPeriodic, py = !kGeneral || a.face[2] == kPeriodic;
  static_for<1, G::T + 1>([&](auto K) {
    constexpr int k = decltype(K)::value;
    constexpr int h = G::T - k;  // halo of this step's region
    constexpr int W = G::OX + 2 * h, N = W * (G::OY + 2 * h);
    T* const out = lds + (G::NB == 2 && k % 2 == 0 ? Q * G::SLOTS : 0);
    const T* const in = lds + (G::NB == 2 && k % 2 == 1 ? Q * G::SLOTS : 0);
    for (int32_t n = (int32_t)tid; n < N; n += (int32_t)nthreads) {
      const int32_t ly = n / W, lx = n - ly * W;
      int32_t gx = x0 - h + lx, gy = y0 - h + ly;
      if constexpr (!kInside) {
        if (lx >= wx + 2 * h || ly >= wy + 2 * h) continue;
        // periodic axes wrap (a grid is at least T cells wide); beyond the
        // other faces there are no cells
        if (px) {
          gx += gx < 0 ? nx : (gx >= nx ? -nx : 0);
        } else if (gx < 0 || gx >= nx) {
          continue;
        }
        if (py) {
          gy += gy < 0 ? ny : (gy >= ny ? -ny : 0);
        } else if (gy < 0 || gy >= ny) {
          continue;
        }
      }
      const uint32_t x = (uint32_t)gx, y = (uint32_t)gy, c = y * a.nx + x;
      const int32_t slot = (ly + (G::H - h)) * G::RX + lx + (G::H - h);
      T raw[Q];
      R post[Q], rho;
      uint8_t m = kFluid;
      if constexpr (k == 1) {
        if constexpr (kGeneral) m = a.mask ? a.mask[c] : kFluid;
        if constexpr (kInside)
          static_for<0, Q>([&](auto I) {
            constexpr int i = decltype(I)::value;
            raw[i] = load_pop(a.src + (uint64_t)i * a.pstride,
                              (uint32_t)((int32_t)c - L::dir(i).x - L::dir(i).y * nx));
          });
        else
          pull_periodic<L, S, false>(a, c, x, y, 0u, raw);
        if constexpr (kGeneral && G::T > 1) lmask[slot] = m;
      } else {
        if constexpr (kGeneral) m = lmask[slot];
        static_for<0, Q>([&](auto I) {
          constexpr int i = decltype(I)::value;
          raw[i] = in[i * G::SLOTS + slot - L::dir(i).x - L::dir(i).y * G::RX];
        });
      }
      auto fixup = [&](T* r) {
        if (m & (kNearFace | kNearSolid)) {
          if constexpr (k == 1)
            pull_fixup<L, S>(a, x, y, 0u, c, (m & kNearSolid) != 0, r);
          else
            lds_fixup<L, S, G::RX, G::SLOTS>(a, x, y, in + slot, lmask + slot,
                                             (m & kNearSolid) != 0, r);
        }
      };
      if (!collide_cell<L, S, kGeneral>(a, c, x, y, 0u, m, a.t_new + (uint64_t)(k - 1), raw, post,
                                        rho, fixup))
        continue;
      // stability watchdog: a rare, benign racy store of 1
      if (!(rho > (R)0) || !(rho < (R)1e30)) a.status[0] = 1;
      static_for<0, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if constexpr (k == G::T)
          store_at<false>(a.dst + (uint64_t)i * a.pstride, (uint32_t)(a.pstride * sizeof(T)),
                      c * (uint32_t)sizeof(T), 0u, narrow<T>(post[i]));
        else
          out[i * G::SLOTS + slot] = narrow<T>(post[i]);
      });
    }
    if constexpr (k < G::T) __syncthreads();
  });
}

// Whether a tile is whole and the cells its steps read lie in the grid.
template <class S, class G>
__device__ __forceinline__ bool inside(const SweepArgs<S>& a, uint32_t bx, uint32_t by) {
  const uint32_t x0 = bx * G::OX, y0 = by * G::OY;
  return x0 >= (uint32_t)G::T && y0 >= (uint32_t)G::T && x0 + G::OX + G::T <= a.nx &&
         y0 + G::OY + G::T <= a.ny;
}

// Whether every cell of an inside tile's first region is plain fluid outside
// the layers (wave-uniform): its steps are then the periodic path's.  Reads
// the 64-cell summaries the region's rows touch, one per lane.
template <class L, class S, class G>
__device__ __forceinline__ bool plain_region(const SweepArgs<S>& a, uint32_t bx, uint32_t by) {
  const int32_t nx = (int32_t)a.nx, ny = (int32_t)a.ny;
  const int32_t xl = (int32_t)bx * G::OX - G::H, yl = (int32_t)by * G::OY - G::H;
  const int32_t xh = xl + G::RX - 1, yh = yl + G::RY - 1;
  if (!a.tiles) return false;
  if (a.chi_max != (typename S::R)0) {
    if (a.sponge[4] > 0 || a.sponge[5] > 0) return false;
    if (xl < a.sponge[0] || xh >= nx - a.sponge[1] || yl < a.sponge[2] || yh >= ny - a.sponge[3])
      return false;
  }
  constexpr uint32_t kPer = (G::RX + 63) / 64 + 1;  // summaries a row segment touches
  bool plain = true;
  for (uint32_t n = threadIdx.x % 64u; n < kPer * G::RY; n += 64u) {
    const int32_t y = yl + (int32_t)(n / kPer);
    if (y > yh) continue;
    const uint32_t first = (uint32_t)(y * nx + xl) >> 6, last = (uint32_t)(y * nx + xh) >> 6;
    const uint32_t t = first + n % kPer;
    if (t <= last) plain = plain && a.tiles[t];
  }
  return __all(plain);
}

// Tile and threads of a workgroup for T steps: the LDS of the intermediate
// states limits the rows.  Grids of few tiles are cut finer (see small_tiles).
template <int T, bool kSmall>
struct Shape2 {
  using G = Tile2<T, kSmall ? 32 : 64, kSmall ? 4 : 8>;
  static constexpr int NT = kSmall ? 384 : (T == 4 ? 512 : 256);
};
// Wavefronts per SIMD: what the LDS of a CU admits.
template <class S, int T>
struct Waves2 {
  static constexpr int value =
      sizeof(typename S::T) == 8 ? 2 : sizeof(typename S::T) == 4 ? (T == 4 ? 4 : 5) : 6;
};

template <class L, class S, bool kGeneral, class G>
__device__ __forceinline__ void multi2d_any(const SweepArgs<S>& a, uint32_t bx, uint32_t by,
                                            typename S::T* lds, uint8_t* lmask,
                                            uint32_t nthreads) {
  if (inside<S, G>(a, bx, by) && (!kGeneral || plain_region<L, S, G>(a, bx, by)))
    multi2d_tile<L, S, false, true, G>(a, bx, by, lds, lmask, threadIdx.x, nthreads);
  else
    multi2d_tile<L, S, kGeneral, false, G>(a, bx, by, lds, lmask, threadIdx.x, nthreads);
}

template <class L, class S, bool kGeneral, int T, bool kSmall>
__global__ void __launch_bounds__((Shape2<T, kSmall>::NT))
    __attribute__((amdgpu_waves_per_eu(Waves2<S, T>::value)))
    k_multi2d(const SweepArgs<S> a, uint32_t tiles_x, uint32_t ntile) {
  using G = typename Shape2<T, kSmall>::G;
  __shared__ typename S::T lds[G::NB * L::Q * G::SLOTS];
  __shared__ uint8_t lmask[kGeneral ? G::SLOTS : 1];
  // each XCD takes a contiguous range of tiles
  const uint32_t k = blockIdx.x % 8u, per = ntile / 8u, rem = ntile % 8u;
  const uint32_t b = k * per + min(k, rem) + blockIdx.x / 8u;
  multi2d_any<L, S, kGeneral, G>(a, b % tiles_x, b / tiles_x, lds, lmask, Shape2<T, kSmall>::NT);
}

// ------------------------------------------------------------------------
// The same tiles over the (job, tile) list of a batch (serving): a fixed grid
// of workgroups walks the list; launch s advances every job that has at least
// (s + 1) T steps by T.  Tiles go to the XCDs in runs of kRun consecutive
// ones, so that neighbours meet in one L2 and every XCD gets a share of every
// job.
// ------------------------------------------------------------------------
template <class L, class S, bool kGeneral, int T>
__global__ void __launch_bounds__((Shape2<T, false>::NT))
    __attribute__((amdgpu_waves_per_eu(Waves2<S, T>::value)))
    k_batch2d(const BatchJob* __restrict__ jobs, const BatchHeader* __restrict__ hdr,
              int32_t s_off) {
  using G = typename Shape2<T, false>::G;
  constexpr uint32_t kRun = 32;
  __shared__ typename S::T lds[G::NB * L::Q * G::SLOTS];
  __shared__ uint8_t lmask[kGeneral ? G::SLOTS : 1];
  const int32_t s = hdr->step + s_off;
  const uint32_t njobs = hdr->njobs, total = hdr->total_ftiles;
  const uint32_t xcd = blockIdx.x % 8u, per = (gridDim.x + 7u - xcd) / 8u;
  uint32_t lo = 0;  // job of the previous tile: this workgroup's tiles increase
  for (uint32_t j = blockIdx.x / 8u;; j += per) {
    const uint32_t first = (j / kRun * 8u + xcd) * kRun, tile = first + j % kRun;
    if (first >= total) break;
    if (tile >= total) continue;
    if (lo + 1 < njobs && jobs[lo + 1].ftile_begin <= tile) {
      uint32_t hi = njobs;
      ++lo;
      while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (jobs[mid].ftile_begin <= tile) lo = mid; else hi = mid;
      }
    }
    const BatchJob& J = jobs[lo];
    if ((int64_t)s >= J.flips0) continue;
    SweepArgs<S> a = to_args_dev<S>(J.h);
    const int p = (J.cur0 + s) & 1;
    a.src = (const typename S::T*)J.buf[p];
    a.dst = (typename S::T*)J.buf[p ^ 1];
    a.t_new = J.t0 + (uint64_t)s * T + 1ull;
    const uint32_t n = tile - J.ftile_begin, tx = (J.h.nx + G::OX - 1) / G::OX;
    multi2d_any<L, S, kGeneral, G>(a, n % tx, n / tx, lds, lmask, Shape2<T, false>::NT);
    __syncthreads();  // LDS is rewritten by the next tile
  }
}

// Estimated times in microseconds: of a launch whatever it covers, and of its
// tiles (a step: cells) at full load.  A tile costs the same however few
// cells it holds, so a narrow grid pays for lanes that idle, and on the
// general path a tile at an edge of the grid costs up to twice one inside
// it.  Fitted to 64 steps on single grids of 3000 to 12 million cells, 4 to 260
// cells wide, 4 to 40 high or of any side ratio from 0.35 to 3, and on batches of
// 1 to 12 grids of 9000 to 5 million cells together, to 4-20 % (r.m.s.).
struct Fit2d {
  double launch;
  double inside, edge;  // per 1000 tiles (a step: per 1000 cells, per 1000 ends of rows)
};
// periodic and general path; storages of 8, 4 and 2 bytes
constexpr Fit2d kStepFit[2][3] = {{{2.9, 0.0263, 0.0}, {2.8, 0.0127, 0.0}, {2.8, 0.0066, 0.0}},
                                  {{4.3, 0.0256, 0.003}, {4.5, 0.0125, 0.049}, {5.2, 0.0080, 0.177}}};
constexpr Fit2d kBatchStepFit[2][3] = {
    {{3.3, 0.0273, 0.0}, {3.3, 0.0134, 0.0}, {3.5, 0.0070, 0.0}},
    {{5.4, 0.0282, 0.0}, {5.8, 0.0139, 0.099}, {5.8, 0.0105, 0.134}}};
// a batch's pass (two steps on the general path of the 8- and 4-byte storages,
// else four)
constexpr Fit2d kBatchPassFit[2][3] = {{{8.9, 27.0, 23.4}, {7.9, 12.1, 11.8}, {7.5, 9.9, 10.0}},
                                       {{14.2, 17.1, 20.3}, {13.4, 10.0, 12.4}, {19.1, 20.5, 28.6}}};
// a single grid's: two steps, four in the large tiles, four in the small ones
constexpr Fit2d kPassFit[2][3][3] = {
    {{{5.2, 13.2, 9.1}, {6.7, 25.1, 23.1}, {4.4, 11.2, 11.2}},
     {{4.7, 6.6, 4.4}, {5.9, 10.7, 9.9}, {4.6, 3.1, 3.1}},
     {{4.9, 3.5, 3.1}, {6.2, 6.7, 7.0}, {4.5, 2.7, 3.0}}},
    {{{13.2, 14.5, 18.6}, {18.8, 34.8, 61.0}, {9.9, 14.6, 26.9}},
     {{12.9, 7.2, 10.1}, {18.0, 15.6, 30.5}, {9.7, 5.7, 11.6}},
     {{14.0, 5.3, 10.0}, {19.2, 11.9, 24.2}, {10.0, 5.3, 11.8}}}};
static int fit_row(int storage) { return storage == 0 ? 0 : storage == 3 ? 2 : 1; }

Time2d step2d_time(int storage, bool general, bool batch, uint32_t nx, uint32_t ny) {
  const Fit2d& f = (batch ? kBatchStepFit : kStepFit)[general][fit_row(storage)];
  const double cells = (double)nx * ny, ends = 2.0 * std::min((double)ny, cells / 64.0);
  return Time2d{f.launch, 1e-3 * (f.inside * cells + f.edge * ends)};
}

// Tiles of a row (or column) of n cells that are whole and have T cells beside
// them (see inside()).
static double inside_tiles(uint32_t n, uint32_t tile, uint32_t T) {
  const uint32_t first = (T + tile - 1) / tile;
  return n < first * tile + tile + T ? 0.0 : (double)((n - tile - T) / tile - first + 1);
}

// Of a pass of `steps` in tiles of ox x oy cells.
static Time2d tiles_time(const Fit2d& f, uint32_t nx, uint32_t ny, uint32_t steps, uint32_t ox,
                         uint32_t oy) {
  const double all = std::ceil((double)nx / ox) * std::ceil((double)ny / oy);
  const double in = inside_tiles(nx, ox, steps) * inside_tiles(ny, oy, steps);
  return Time2d{f.launch, 1e-3 * (f.inside * in + f.edge * (all - in))};
}

Time2d batch2d_time(int storage, bool general, uint32_t nx, uint32_t ny) {
  return tiles_time(kBatchPassFit[general][fit_row(storage)], nx, ny,
                    (uint32_t)batch2d_steps(storage, general), 64, 8);
}

static Time2d pass2d_time(int storage, bool general, uint32_t nx, uint32_t ny, int steps,
                          bool small) {
  const Fit2d& f = kPassFit[general][fit_row(storage)][steps == 2 ? 0 : small ? 2 : 1];
  return tiles_time(f, nx, ny, (uint32_t)steps, small ? 32 : 64, small ? 4 : 8);
}

// Whether a grid is stepped in the small tiles: where the large ones leave
// CUs idle, more and smaller workgroups step fewer cells one after another;
// past that their wider share of halo costs more.  On the general path a
// workgroup takes several times as long, so a few large ones per CU are
// still too uneven; FP64 pays the halo twice.  us per step, large / small:
// periodic 128 x 128 FP64 1.98 / 1.34, FP32 1.56 / 1.15; 256 x 256 FP64 2.13 / 2.13,
// FP32 1.64 / 1.36; 512 x 512 FP32 2.33 / 2.68; channel 300 x 200 FP32 5.7 / 3.5,
// FP64 6.3 / 5.1; 500 x 400 FP32 6.8 / 5.3, FP64 8.4 / 9.5; 900 x 800 FP32 11.2 / 11.4.
static bool small_tiles(int storage, bool general, uint32_t nx, uint32_t ny, uint32_t cus) {
  const uint32_t tiles = multi2d_tiles(nx, ny);
  const uint32_t limit = general ? 4 * cus : cus;
  return tiles < (storage == 0 ? (general ? limit / 4 : limit / 2) : limit);
}

// Whether a pass is taken in place of single steps: where it is expected to
// take under this share of their time, which balances the fit's errors (of 366
// grids measured 13 have a pass that is slower, by up to 13 %, and 33 miss one
// that is faster).  us per step, one at a time / in the pass a rule without the times
// took: periodic 8 x 112500 FP32 14.8 / 33.4, 8 x 3750 FP64 3.1 / 3.6; channel
// 32 x 28125 FP32 18.2 / 36.1, 96 x 41666 FP64 107 / 118, 130 x 30769 FP16S 51 / 73,
// 700 x 500 FP64 13.9 / 9.2.  What is left over by passes of four is two steps at a
// time only where that is clearly faster.
constexpr double kPays = 0.89, kTwoPays = 0.85;
static bool pays(const Time2d& pass, const Time2d& step, int steps, double share) {
  return pass.launch + pass.cells < share * steps * (step.launch + step.cells);
}

// Steps per pass of a single grid: four, but two on the general path of the
// 4- and 8-byte storages, whose larger halo costs more there than the second
// pass it saves, once the tiles fill the device; one where that does not pay.
// us per step, one at a time / two / four: periodic 4000 x 3001 FP32 147 / 90 / 69,
// FP16S 79 / 58 / 49, 128 x 128 FP64 3.2 / 2.8 / 1.3; cylinder channel
// 2048 x 1024 FP32 32 / 18 / 21, FP16S 26 / 20 / 19, FP64 60 / 38 / 44; 1000 x 700 FP32
// 14.4 / 13.9 / 11.9.
int multi2d_steps(int storage, bool general, uint32_t nx, uint32_t ny, uint32_t cus) {
  if (nx < 4 || ny < 4) return 1;  // the halo wraps once
  const int steps = !general || storage == 3 || (uint64_t)nx * ny < (1u << 20) ? 4 : 2;
  const bool small = steps == 4 && small_tiles(storage, general, nx, ny, cus);
  return pays(pass2d_time(storage, general, nx, ny, steps, small),
              step2d_time(storage, general, false, nx, ny), steps, kPays)
             ? steps
             : 1;
}

// Whether two steps left over by passes of four are taken in one.
bool multi2d_two(int storage, bool general, uint32_t nx, uint32_t ny) {
  return nx >= 4 && ny >= 4 &&
         pays(pass2d_time(storage, general, nx, ny, 2, false),
              step2d_time(storage, general, false, nx, ny), 2, kTwoPays);
}

// Steps per pass of a batch: as of a single grid whose tiles fill the device.
int batch2d_steps(int storage, bool general) { return !general || storage == 3 ? 4 : 2; }

uint32_t multi2d_tiles(uint32_t nx, uint32_t ny) { return (nx + 63) / 64 * ((ny + 7) / 8); }

template <class L, class S, bool kGeneral, int T, bool kSmall>
static hipError_t multi2d_one(const Multi2d& m) {
  using Z = Shape2<T, kSmall>;
  const uint32_t tx = (m.h->nx + Z::G::OX - 1) / Z::G::OX;
  const uint32_t n = tx * ((m.h->ny + Z::G::OY - 1) / Z::G::OY);
  hipLaunchKernelGGL((k_multi2d<L, S, kGeneral, T, kSmall>), dim3(n), dim3(Z::NT), 0, m.st,
                     to_args_dev<S>(*m.h), tx, n);
  return hipGetLastError();
}

template <class L, class S, bool kGeneral, int T>
static hipError_t multi2d_g(const Multi2d& m) {
  const dim3 block(Shape2<T, false>::NT);
  if (m.query)
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(m.query, k_batch2d<L, S, kGeneral, T>,
                                                        Shape2<T, false>::NT, 0);
  if (m.jobs) {
    hipLaunchKernelGGL((k_batch2d<L, S, kGeneral, T>), dim3(m.grid), block, 0, m.st, m.jobs,
                       m.hdr, m.s_off);
    return hipGetLastError();
  }
  if constexpr (T == 4)
    if (small_tiles(m.storage, m.general, m.h->nx, m.h->ny, (uint32_t)m.cus))
      return multi2d_one<L, S, kGeneral, T, true>(m);
  return multi2d_one<L, S, kGeneral, T, false>(m);
}

template <class L, class S>
static hipError_t multi2d_t(const Multi2d& m) {
  if (m.general)
    return m.steps == 4 ? multi2d_g<L, S, true, 4>(m) : multi2d_g<L, S, true, 2>(m);
  return m.steps == 4 ? multi2d_g<L, S, false, 4>(m) : multi2d_g<L, S, false, 2>(m);
}

template <class L>
static hipError_t multi2d_l(const Multi2d& m) {
  switch (m.storage) {
    case 0: return multi2d_t<L, StoreF64>(m);
    case 1: return multi2d_t<L, StoreF32>(m);
    case 2: return multi2d_t<L, StoreF32S>(m);
    case 3: return multi2d_t<L, StoreF16S>(m);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_multi2d(const Multi2d& m) {
  if (m.steps != 2 && m.steps != 4) return hipErrorInvalidValue;
  switch (m.lattice) {
    case 9: return multi2d_l<Lattice<9>>(m);
    case kFullOrderCode + 9: return multi2d_l<Lattice<9, true>>(m);
  }
  return hipErrorInvalidValue;
}

}  // namespace hrlbm
