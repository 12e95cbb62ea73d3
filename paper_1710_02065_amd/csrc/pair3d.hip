// Two steps of a periodic 3D population grid in one pass over HBM.
//
// The one-step sweep reads and writes every population once per step and is
// bound by that traffic.  Here a workgroup marches through its chunk of
// planes with a tile of TX x TY cells and, per plane, (1) pulls and collides
// the tile plus a one-cell halo from the state at t (every slot the values
// the one-step sweep would store), puts what streams into the output plane
// into LDS, and (2) pulls every interior cell's populations from there,
// collides again and stores the state at t + 2.  The state at t + 1 never
// reaches HBM: two steps write q values per cell and read q, where single steps
// take 2 q + 2 q.  A halo cell's first step is computed by the neighbouring tile
// too: a workgroup asks for (1 + 2/TX)(1 + 2/TY) = 1.29 times its tile's cells, and
// the L2 of the XCD that walks its neighbours serves most of the rest (256^3 D3Q19
// FP32: 1.056 reads of the state reach HBM, 78.1 B per update).
//
// Measured on 256^3, one step / two at a time, us per step: D3Q19 FP32 445 /
// 254 (66k MLUPS), FP16S 219 / 173, FP64 915 / 512; D3Q27 FP32 646 / 366, FP16S
// 317 / 254, FP64 1309 / 779; every order FP32 638 / 392, FP16S 317 / 305, FP64
// 1321 / 1102.  D3Q19 FP32 is bound by HBM latency: 5.15 TB/s, with two
// workgroups per CU and two barriers a plane; its vector instructions, at four
// cycles each and 2.4 GHz, fill 43 % of the time.  FP16S moves 3.8 TB/s and is
// bound by those more than by HBM: 4280 of them per plane of a tile, 68 %.
// Tried on the way: populations waiting for their plane in registers instead
// of LDS (103 vector registers, one workgroup less per CU), 4, 6, 7 and 12
// rows per tile (266, 338, 311, 287 us at their best chunk length against
// 258 for 8, D3Q19 FP32), raw buffer loads with scalar offsets instead of
// global ones (278 against 254).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "kernels.hpp"
#include "launch.hpp"

namespace hrlbm {

// Workgroup tile: TY wavefronts of interior cells (one lane per cell, TX =
// 64) and three halo wavefronts (the two halo rows, then both halo columns
// with their corners).
template <class L, class S>
struct PairTile {
  using T = typename S::T;
  static constexpr int TX = 64;
  static constexpr int TY = 8;
  static constexpr int HX = TX + 2;
  static constexpr int HY = TY + 2;
  static constexpr int SLOTS = HX * HY;
  static constexpr int NT = (TY + 3) * 64;
  static_assert(2 * HY <= 64, "one wavefront holds both halo columns");
  // planes of the populations with xi_z = +1 / 0 kept in LDS
  static constexpr int kUpRing = sizeof(T) == 8 ? 1 : 2;
  static constexpr int kMidRing = sizeof(T) == 8 ? 1 : 2;
  // the pulls of the next plane are issued before this plane's second step
  static constexpr bool kAhead = sizeof(T) == 4 || (sizeof(T) == 8 && L::Q == 19);
  // waves per SIMD asked of the compiler
  static constexpr int kWaves = sizeof(T) == 8 ? 3 : (sizeof(T) == 4 && L::Q == 27 ? 3 : 6);
  static constexpr int ring(int dz) { return dz > 0 ? kUpRing : (dz == 0 ? kMidRing : 1); }
  // populations with an in-plane velocity go through LDS
  static constexpr bool staged(int i) { return L::dir(i).x != 0 || L::dir(i).y != 0; }
  // first LDS row of population i; row0(Q): the number of rows
  static constexpr int row0(int i) {
    int r = 0;
    for (int j = 0; j < i; ++j)
      if (staged(j)) r += ring(L::dir(j).z);
    return r;
  }
};

template <class S>
struct PairArgs {
  using T = typename S::T;
  using R = typename S::R;
  const T* src;
  T* dst;
  int* status;
  uint32_t nx, ny, nz;
  uint32_t tiles_x, tiles_y, zc, nblocks;
  uint64_t pstride;
  R omega1, rho0;
};

// What a thread computes: kInner its own output cell, every population;
// kRowLo / kRowHi a halo-row cell below / above the tile, whose populations
// with xi_y = +1 / -1 the interior pulls; kCols a halo-column cell (those
// with xi_x != 0).
enum PairRole { kInner = 0, kRowLo = 1, kRowHi = 2, kCols = 3 };

template <class L, int ROLE>
constexpr bool pair_needs(int i) {
  return ROLE == kRowLo   ? L::dir(i).y == 1
         : ROLE == kRowHi ? L::dir(i).y == -1
         : ROLE == kCols  ? L::dir(i).x != 0
                          : true;
}
// The next population array's base.  The sum is opaque to the compiler, which
// would otherwise keep every population's base in scalar registers across the
// loop and spill them to lanes of vector registers.
template <class T>
__device__ __forceinline__ T* next_array(T* p, uint32_t bytes) {
  p = reinterpret_cast<T*>(reinterpret_cast<uintptr_t>(p) + bytes);
  asm volatile("" : "+s"(p));
  return p;
}

// One collision of pulled values: post-collision values as stored, and rho.
template <class L, class S>
__device__ __forceinline__ typename S::R pair_collide(const typename S::T raw[L::Q],
                                                      typename S::R omega1, typename S::R rho0,
                                                      typename S::T out[L::Q]) {
  using R = typename S::R;
  using T = typename S::T;
  R drho, j[3], P[6], post[L::Q];
  const R zero3[3] = {(R)0, (R)0, (R)0};
  stored_moments<L, S>(raw, rho0, drho, j, P);
  const R rho = collide_moments<L, R, false, !S::kShifted>(
      drho, j, P, omega1, rho0, (R)0, rho0, zero3, S::kShifted ? (R)0 : rho0, post);
#pragma unroll
  for (int i = 0; i < L::Q; ++i) out[i] = narrow<T>(post[i]);
  return rho;
}

// One thread's march through output planes z0 ... z1 - 1.  x, y: the cell
// of the first step, slds its LDS slot; an interior thread's second step is of
// the same cell.  A lane without a cell (own false) takes that of another
// lane of its role: it writes the same values to the same slot, and its
// stores are dropped.  Iteration `it` computes the first step of plane
// z0 + it + 1 and the second of plane z0 + it, which pulls the populations with
// xi_z = -1, 0, +1 from planes it + 1, it and it - 1; two warm-up iterations
// fill what is carried.  Populations wait for their plane in LDS where it
// has room (kUpRing, kMidRing planes), else in registers, and are written
// to LDS as early as the previous iteration's reads allow, so that few
// registers are live through the collisions.  Every thread of a workgroup
// meets the same barriers.
template <class L, class S, int ROLE, bool kNt>
__device__ __forceinline__ void pair_march(const PairArgs<S>& a, typename S::T* lds, uint32_t x,
                                           uint32_t y, uint32_t slds, bool own, uint32_t z0,
                                           uint32_t z1) {
  using G = PairTile<L, S>;
  using T = typename S::T;
  using R = typename S::R;
  constexpr int Q = L::Q;
  const uint64_t P = a.pstride;
  const uint32_t plane = a.nx * a.ny;
  // byte offsets of the nine pull sources in a plane: the row is one for the
  // whole wavefront except in the halo columns, and then a scalar offset
  constexpr uint32_t kB = (uint32_t)sizeof(T);
  constexpr bool kRowLane = ROLE == kCols;
  const uint32_t bytes = (uint32_t)(P * kB);  // below 2^32 (checked on the host)
  uint32_t xb[3] = {(x == 0 ? a.nx - 1 : x - 1) * kB, x * kB,
                    (x + 1 == a.nx ? 0u : x + 1) * kB};
  const uint32_t yu = kRowLane ? y : (uint32_t)__builtin_amdgcn_readfirstlane(y);
  const uint32_t yb[3] = {(yu == 0 ? a.ny - 1 : yu - 1) * a.nx * kB, yu * a.nx * kB,
                          (yu + 1 == a.ny ? 0u : yu + 1) * a.nx * kB};
  auto wrap = [&](uint32_t z, int d) -> uint32_t { return (z + a.nz + (uint32_t)d) % a.nz; };
  // LDS row of population i streaming out of plane it + ring index
  auto row = [&](auto I, int plane_it) -> T* {
    constexpr int i = decltype(I)::value;
    constexpr int n = G::ring(L::dir(i).z);
    T* b = lds + G::row0(i) * G::SLOTS;
    return n == 2 ? b + (plane_it & 1) * G::SLOTS : b;
  };

  // carried: up1 / up2 the populations with xi_z = +1 of planes it / it + 1
  // (after the first step), mid those with xi_z = 0 of plane it + 1
  T up0[Q] = {}, up1[Q] = {}, up2[Q] = {}, mid[Q] = {}, mid0[Q] = {};
  T raw[Q];
  auto load_plane = [&](int it_p) {
    const uint32_t zp = wrap(z0, it_p);
    const uint32_t zb[3] = {(zp == 0 ? a.nz - 1 : zp - 1) * plane * kB, zp * plane * kB,
                            (zp + 1 == a.nz ? 0u : zp + 1) * plane * kB};
    static_for<0, Q>([&](auto I) {
      constexpr int i = decltype(I)::value;
      constexpr Dir d = L::dir(i);
      const char* b = reinterpret_cast<const char*>(a.src + (uint64_t)i * P) + zb[1 - d.z];
      if constexpr (kRowLane)
        b += xb[1 - d.x] + yb[1 - d.y];
      else
        b = b + yb[1 - d.y] + xb[1 - d.x];
      raw[i] = *reinterpret_cast<const T*>(b);
    });
  };
  // State at t + 2 of the output cell of plane offset cb; a lane without one
  // is given an offset past the array, where the store is dropped (no lane
  // mask around the second step: D3Q27 FP64 at 256^3 877 us a step with it,
  // 768 without).
  auto store_plane = [&](uint32_t off, uint32_t cb, const T v[Q]) {
    // kNt: rows of whole 64-cell tiles are stored past the caches; of
    // others, the line a row segment ends in is completed by the next
    // tile or row and should meet it in L2 (250 x 131 x 97 FP32: 78 us a
    // step with the hint, 72 without; 256^3: 255 with, 267 without)
    T* p = a.dst;
    static_for<0, Q>([&](auto I) {
      store_at<kNt>(p, bytes, off, cb, v[decltype(I)::value]);
      p = next_array(p, bytes);
    });
  };
  bool bad = false;  // a density that is not positive and finite was seen
  if constexpr (G::kAhead) load_plane(-1);
  auto iterate = [&](int it, auto out) {
    // (opaque to the compiler, which would otherwise hoist the 64-bit vector
    // sums of these offsets with every population's base out of the loop:
    // 103 vector registers instead of 54)
    asm volatile("" : "+v"(xb[0]), "+v"(xb[1]), "+v"(xb[2]));
    // the carried populations the previous iteration's reads kept out of LDS
    static_for<0, Q>([&](auto I) {
      constexpr int i = decltype(I)::value;
      if constexpr (pair_needs<L, ROLE>(i)) {
        if constexpr (L::dir(i).z > 0) {
          if constexpr (G::staged(i)) {
            row(I, G::kUpRing == 2 ? it : it - 1)[slds] = G::kUpRing == 2 ? up2[i] : up1[i];
          } else {
            up0[i] = up1[i];
          }
          up1[i] = up2[i];
        } else if constexpr (L::dir(i).z == 0) {
          if constexpr (!G::staged(i))
            mid0[i] = mid[i];
          else if constexpr (G::kMidRing == 1)
            row(I, it)[slds] = mid[i];
        }
      }
    });
    T down[Q];
    {
      T post[Q];
      if constexpr (!G::kAhead) load_plane(it + 1);
      const R rho = pair_collide<L, S>(raw, a.omega1, a.rho0, post);
      if (ROLE == kInner) bad = bad || !(rho > (R)0) || !(rho < (R)1e30);
      static_for<0, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if constexpr (pair_needs<L, ROLE>(i)) {
          if constexpr (L::dir(i).z > 0) {
            up2[i] = post[i];
          } else if constexpr (L::dir(i).z == 0) {
            if constexpr (G::staged(i) && G::kMidRing == 2) {
              row(I, it + 1)[slds] = post[i];
            } else {
              mid[i] = post[i];
            }
          } else {
            if constexpr (G::staged(i)) {
              row(I, it + 1)[slds] = post[i];
            } else {
              down[i] = post[i];
            }
          }
        }
      });
    }
    if constexpr (G::kAhead) load_plane(it + 2);
    __syncthreads();
    if constexpr (ROLE == kInner) {
      if (out) {
        T raw2[Q], post[Q];
        static_for<0, Q>([&](auto I) {
          constexpr int i = decltype(I)::value;
          constexpr Dir d = L::dir(i);
          if constexpr (G::staged(i))
            raw2[i] = row(I, it - d.z)[(int)slds - d.x - d.y * G::HX];
          else
            raw2[i] = d.z > 0 ? up0[i] : (d.z == 0 ? mid0[i] : down[i]);
        });
        const R rho = pair_collide<L, S>(raw2, a.omega1, a.rho0, post);
        bad = bad || !(rho > (R)0) || !(rho < (R)1e30);
        store_plane(own ? xb[1] : bytes, (z0 + (uint32_t)it) * plane * kB + yb[1], post);
      }
    }
    __syncthreads();
  };
  // The two warm-up iterations, which store nothing, in a loop of their own:
  // without the branch around the second step its LDS reads and the next
  // plane's loads mix freely (256^3, us per step, branch / two loops: D3Q27
  // FP32 374 / 365, FP16S 277 / 254; 64^3 D3Q19 FP32 6.7 / 6.3).  FP64 keeps
  // the branch: at its 168 registers two loops spill (D3Q27 768 / 798).
  if constexpr (sizeof(T) == 8) {
#pragma clang loop unroll(disable)
    for (int it = -2; it < (int)(z1 - z0); ++it) iterate(it, it >= 0);
  } else {
#pragma clang loop unroll(disable)
    for (int it = -2; it < 0; ++it) iterate(it, std::false_type{});
#pragma clang loop unroll(disable)
    for (int it = 0; it < (int)(z1 - z0); ++it) iterate(it, std::true_type{});
  }
  // stability watchdog: a rare, benign racy store of 1
  if (ROLE == kInner && bad) a.status[0] = 1;
}

template <class L, class S, bool kNt>
__global__ void __launch_bounds__((PairTile<L, S>::NT))
    __attribute__((amdgpu_waves_per_eu(PairTile<L, S>::kWaves))) k_pair3d(const PairArgs<S> a) {
  using G = PairTile<L, S>;
  __shared__ typename S::T lds[G::row0(L::Q) * G::SLOTS];

  // each XCD walks a contiguous range of tiles, so that neighbouring tiles
  // share their halo lines in one L2
  const uint32_t k = blockIdx.x % 8u, per = a.nblocks / 8u, rem = a.nblocks % 8u;
  const uint32_t b = k * per + min(k, rem) + blockIdx.x / 8u;
  const uint32_t bx = b % a.tiles_x;
  const uint32_t r = b / a.tiles_x;
  const uint32_t by = r % a.tiles_y;
  const uint32_t ch = r / a.tiles_y;
  const uint32_t x0 = bx * G::TX, y0 = by * G::TY;
  const uint32_t wx = min((uint32_t)G::TX, a.nx - x0);
  const uint32_t wy = min((uint32_t)G::TY, a.ny - y0);
  const uint32_t z0 = ch * a.zc, z1 = min(a.nz, z0 + a.zc);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64u);
  const uint32_t lane = threadIdx.x % 64u;
  if (wave < (uint32_t)G::TY) {
    const uint32_t ox = min(lane, wx - 1), oy = min(wave, wy - 1);
    pair_march<L, S, kInner, kNt>(a, lds, x0 + ox, y0 + oy, (oy + 1) * G::HX + ox + 1,
                             lane < wx && wave < wy, z0, z1);
  } else if (wave < (uint32_t)G::TY + 2) {
    const uint32_t sx = min(lane, wx - 1);
    if (wave == (uint32_t)G::TY)
      pair_march<L, S, kRowLo, kNt>(a, lds, x0 + sx, y0 == 0 ? a.ny - 1 : y0 - 1, sx + 1, lane < wx,
                               z0, z1);
    else
      pair_march<L, S, kRowHi, kNt>(a, lds, x0 + sx, y0 + wy == a.ny ? 0u : y0 + wy,
                               (wy + 1) * G::HX + sx + 1, lane < wx, z0, z1);
  } else {
    // halo columns x0 - 1 (lanes 0 ... hy - 1) and x0 + wx (the next hy
    // lanes), corners included; the clamp of the idle lanes follows the
    // select
    const uint32_t hy = wy + 2;
    const bool left = lane < hy;
    const uint32_t sy = min(left ? lane : lane - hy, hy - 1);
    const uint32_t sx = left ? 0u : wx + 1;
    const uint32_t gx = left ? (x0 == 0 ? a.nx - 1 : x0 - 1) : (x0 + wx == a.nx ? 0u : x0 + wx);
    const uint32_t gy = (y0 + sy + a.ny - 1) % a.ny;
    pair_march<L, S, kCols, kNt>(a, lds, gx, gy, sy * G::HX + sx, lane < 2 * hy, z0, z1);
  }
}

template <class L, class S>
static hipError_t pair3d_t(const SweepHost& h, uint32_t zc, hipStream_t st) {
  using G = PairTile<L, S>;
  using T = typename S::T;
  using R = typename S::R;
  PairArgs<S> a{};
  a.src = (const T*)h.src;
  a.dst = (T*)h.dst;
  a.status = h.status;
  a.nx = h.nx;
  a.ny = h.ny;
  a.nz = h.nz;
  a.tiles_x = (h.nx + G::TX - 1) / G::TX;
  a.tiles_y = (h.ny + G::TY - 1) / G::TY;
  a.zc = zc;
  a.nblocks = a.tiles_x * a.tiles_y * ((h.nz + zc - 1) / zc);
  a.pstride = h.pstride;
  a.omega1 = (R)(1.0 - 1.0 / h.tau);
  a.rho0 = (R)h.rho0;
  if (h.nx % G::TX == 0)
    hipLaunchKernelGGL((k_pair3d<L, S, true>), dim3(a.nblocks), dim3(G::NT), 0, st, a);
  else
    hipLaunchKernelGGL((k_pair3d<L, S, false>), dim3(a.nblocks), dim3(G::NT), 0, st, a);
  return hipGetLastError();
}

template <class L>
static hipError_t pair3d_l(int storage, const SweepHost& h, uint32_t zc, hipStream_t st) {
  switch (storage) {
    case 0: return pair3d_t<L, StoreF64>(h, zc, st);
    case 1: return pair3d_t<L, StoreF32>(h, zc, st);
    case 2: return pair3d_t<L, StoreF32S>(h, zc, st);
    case 3: return pair3d_t<L, StoreF16S>(h, zc, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_pair3d(int lattice, int storage, const SweepHost& h, uint32_t zc,
                         hipStream_t st) {
  switch (lattice) {
    case 19: return pair3d_l<Lattice<19>>(storage, h, zc, st);
    case 27: return pair3d_l<Lattice<27>>(storage, h, zc, st);
    case kFullOrderCode + 27: return pair3d_l<Lattice<27, true>>(storage, h, zc, st);
  }
  return hipErrorInvalidValue;
}

// Time of one iteration (a plane of a tile) on a CU in microseconds, at
// full load: measured on 256^3 to 64^3 grids, odd sizes among them.  FP32
// and FP64 keep one workgroup's loads a plane ahead, so a CU's workgroups
// take their times one after another; the 2-byte storage needs two
// workgroups per CU to hide its loads and is timed per pair.
static double iteration_us(int q, int storage) {
  const bool q27 = q == 27;
  return storage == 0 ? (q27 ? 12.0 : 7.2) : storage == 3 ? (q27 ? 8.4 : 5.3) : (q27 ? 5.4 : 3.9);
}

// Planes per workgroup of two steps in one pass, 0 where two one-step sweeps
// are faster.  A chunk of zc planes takes zc + 2 iterations, and a CU with
// n workgroups n times as long, so the chunk count minimises
// ceil(workgroups / slots) (zc + 2).  The pass is taken when that many
// iterations cost less than two sweeps at their 5.5 TB/s and 1.7 us a launch
// (4.2 us at least).  Both sides measured, us per step, one-step / pass:
// D3Q19 FP32 256^3 445 / 254, 250 x 131 x 97 87 / 70, 200 x 150 x 130 105 / 101,
// 64^3 8.6 / 6.2, 128 x 64 x 24 6 / 7, 12 x 200 x 64 8 / 14 (lanes of narrow rows
// idle); FP16S 256^3 219 / 173, 250 x 131 x 97 46 / 31, 200 x 150 x 130 55 / 67
// (a quarter of the lanes idle, and the 2-byte pass is bound by its
// arithmetic); D3Q27 FP32 256^3 646 / 366; FP64 256^3 D3Q19 915 / 512.
// The search takes the rounds r in which a CU works off its workgroups, and the
// most chunks that fit them; r rounds take at least 2 r iterations more than
// the cells alone, which ends it after few (10^6 planes of 4 x 4 cells: two).
uint32_t pair3d_planes(int q, int storage, uint32_t nx, uint32_t ny, uint32_t nz, uint32_t cus) {
  if (cus == 0) return 0;
  const uint64_t slots = storage == 3 ? 2ull * cus : cus;
  const uint64_t ntile = (uint64_t)((nx + 63) / 64) * ((ny + 7) / 8);
  uint32_t best = nz;
  uint64_t iterations = ~0ull, chunks = 0;
  for (uint64_t r = (ntile + slots - 1) / slots;
       chunks < nz && (iterations == ~0ull || ntile * nz + 2 * r * slots < iterations * slots); ++r) {
    chunks = std::min<uint64_t>(nz, r * slots / ntile);
    const uint64_t zc = (nz + chunks - 1) / chunks;
    const uint64_t n = r * (zc + 2);
    if (n < iterations) {
      iterations = n;
      best = (uint32_t)zc;
    }
  }
  const double bytes = 2.0 * q * (storage == 0 ? 8 : storage == 3 ? 2 : 4) * nx * ny * nz;
  const double sweep = std::max(4.2, 1.7 + bytes / 5.5e6);
  return 2.0 + (double)iterations * iteration_us(q, storage) < 2.0 * sweep ? best : 0;
}

}  // namespace hrlbm
