// Device code of one cell's step shared by the sweeps: the pull under the face
// rules, refinement records and RING nodes, and the collision of every cell
// kind.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "kernels.hpp"
#include "launch.hpp"

namespace hrlbm {

// Direction i with the components along the flipped axes reversed, selected
// from constants (a table indexed at run time would be a memory access in
// the middle of the pull).
template <class L, int I>
__device__ __forceinline__ int flipped(bool fx, bool fy, bool fz) {
  constexpr Dir v = L::dir(I);
  constexpr int px = find_dir<L>(-v.x, v.y, v.z), py = find_dir<L>(v.x, -v.y, v.z),
                pz = find_dir<L>(v.x, v.y, -v.z), pxy = find_dir<L>(-v.x, -v.y, v.z),
                pxz = find_dir<L>(-v.x, v.y, -v.z), pyz = find_dir<L>(v.x, -v.y, -v.z),
                pxyz = opposite<L>(I);
  const int nz = fx ? (fy ? pxy : px) : (fy ? py : I);
  if constexpr (L::D == 2 || v.z == 0) return nz;
  const int wz = fx ? (fy ? pxyz : pxz) : (fy ? pyz : pz);
  return fz ? wz : nz;
}

// ------------------------------------------------------------------------
// Pull under the face rules and the mask (left side of eq. optimizedLB read
// backwards): the source of population i is x - xi_i, mapped axis by axis
// (periodic wrap, free-slip reflection with the population mirrored,
// zero-gradient clamp, or the neighbour subdomain's values through a halo
// face); a link whose source is SOLID is bounced back halfway from this
// cell.  Applied as corrections to the periodic pull already in raw[]: only
// the directions whose source crosses a non-periodic face, or (for cells
// flagged kNearSolid) is SOLID, are loaded again.
//
// A wavefront holding such a cell waits for its reloads, which sets the time
// of a step on small grids: the mask bytes of the sources are read together
// (nine at a time) and the reloads are issued without waiting for each other
// (one mask byte and one reload after the other were up to two memory
// latencies per direction: D2Q9 300 x 200 channel 6.5 us a step, now 5.5).
// kAtOnce = false reads them one by one, for D3Q27 in a batch, whose sweep has no
// registers left for them (FP32 spilled 2.7 KB a lane; its solo sweep, 200 x 150 x 130
// with a cylinder: FP32 185 us a step one by one, 173 together, FP16S 169 / 152).
// Directions that cross no face any lane of the wavefront lies on are passed
// over by a scalar branch: in an open box most wavefronts hold an end of a row
// and would spend more on the 26 directions than on the collision.
// ------------------------------------------------------------------------
template <class L, class S, bool kAtOnce = true>
__device__ __forceinline__ void pull_fixup(const SweepArgs<S>& a, uint32_t x, uint32_t y,
                                           uint32_t z, uint32_t c, bool near_solid,
                                           typename S::T raw[L::Q]) {
  const uint64_t P = a.pstride;
  const uint32_t dims[3] = {a.nx, a.ny, a.nz};
  const uint32_t pos[3] = {x, y, z};
  // source coordinate along one axis: wrapped, or the face row (crossed, with
  // the population reflected on a free-slip face)
  auto along = [&](int ax, int v, bool& crossed, bool& flip) -> uint32_t {
    if (v == 0) return pos[ax];
    const bool hi = v < 0;
    if (hi ? pos[ax] + 1 < dims[ax] : pos[ax] > 0) return hi ? pos[ax] + 1 : pos[ax] - 1;
    const int32_t bc = a.face[2 * ax + (hi ? 1 : 0)];
    if (bc == kPeriodic) return hi ? 0u : dims[ax] - 1;
    crossed = true;
    flip = bc == kFreeSlip;
    return pos[ax];
  };
  // faces (not periodic) that some lane lies on
  bool on[3][2];
#pragma unroll
  for (int ax = 0; ax < L::D; ++ax) {
    on[ax][0] = a.face[2 * ax] != kPeriodic && any_lane(pos[ax] == 0);
    on[ax][1] = a.face[2 * ax + 1] != kPeriodic && any_lane(pos[ax] + 1 == dims[ax]);
  }
  const bool any_solid = any_lane(near_solid);
  uint32_t solid = 0;  // bit i: the source of population i is SOLID
  if (kAtOnce && near_solid) {
    constexpr int kBatch = 9;
    static_for<0, (L::Q + kBatch - 2) / kBatch>([&](auto B) {
      constexpr int i0 = 1 + decltype(B)::value * kBatch;
      constexpr int i1 = i0 + kBatch < L::Q ? i0 + kBatch : L::Q;
      uint8_t m[kBatch];
      static_for<i0, i1>([&](auto I) {
        constexpr Dir v = L::dir(decltype(I)::value);
        bool cr, fl;
        const uint32_t sx = along(0, v.x, cr, fl), sy = along(1, v.y, cr, fl),
                       sz = along(2, v.z, cr, fl);
        m[decltype(I)::value - i0] = a.mask[(sz * a.ny + sy) * a.nx + sx];
      });
      static_for<i0, i1>([&](auto I) {
        constexpr int i = decltype(I)::value;
        solid |= (m[i - i0] & kKindBits) == kSolid ? 1u << i : 0u;
      });
    });
  }
  static_for<1, L::Q>([&](auto I) {
    constexpr int i = decltype(I)::value;
    constexpr Dir v = L::dir(i);
    bool reach = any_solid;
    if constexpr (v.x != 0) reach = reach || on[0][v.x < 0];
    if constexpr (v.y != 0) reach = reach || on[1][v.y < 0];
    if constexpr (v.z != 0) reach = reach || on[2][v.z < 0];
    if (!reach) return;
    bool cross = false, fx = false, fy = false, fz = false;
    const uint32_t sx = along(0, v.x, cross, fx), sy = along(1, v.y, cross, fy),
                   sz = along(2, v.z, cross, fz);
    // halo side crossed (only the last axis has halo faces)
    constexpr int vl = last_component<L>(v);
    constexpr int la = L::D - 1, hi = vl < 0 ? 1 : 0;
    const bool halo = vl != 0 && (hi ? pos[la] + 1 >= dims[la] : pos[la] == 0) &&
                      a.face[2 * la + hi] == kHalo;
    const uint32_t src = (sz * a.ny + sy) * a.nx + sx;
    bool wall;
    if constexpr (kAtOnce)
      wall = (solid >> i & 1u) && !halo;
    else
      wall = near_solid && !halo && (a.mask[src] & kKindBits) == kSolid;
    if (wall) {
      // halfway bounce-back: the population that left this cell towards
      // the wall comes back reversed (same weight, so the same shift)
      raw[i] = load_pop(a.src + (uint64_t)opposite<L>(i) * P, c);
    } else if (cross) {
      if (halo) {
        // the source lies in the neighbour's face plane (mapped on the
        // other axes as above); a free-slip flip acts on the other axes
        // only, so the row is one of four known at compile time
        constexpr int r00 = halo_rank<L>(i);
        constexpr int r10 = halo_rank<L>(find_dir<L>(-v.x, v.y, v.z));
        constexpr int r01 = halo_rank<L>(find_dir<L>(v.x, -v.y, v.z));
        constexpr int r11 = halo_rank<L>(find_dir<L>(-v.x, -v.y, v.z));
        const int r = fx ? (fy ? r11 : r10) : (fy ? r01 : r00);
        const uint32_t pc = L::D == 3 ? sy * a.nx + sx : sx;
        const typename S::T* rb = hi ? a.hrecv[1] : a.hrecv[0];
        raw[i] = load_pop(rb + (uint64_t)r * a.hplane, pc);
      } else {
        int pop = i;
        if (fx || fy || fz) pop = flipped<L, i>(fx, fy, fz);
        raw[i] = load_pop(a.src + (uint64_t)pop * P, src);
      }
    }
  });
}

// Halo faces on the periodic path (every other face periodic, no mask): a
// face-plane cell replaces the populations the periodic pull wrapped across
// a halo face by the neighbour's values, from the receive buffer at the
// source wrapped on the other axes.
template <class L, class S>
__device__ __forceinline__ void halo_pull_periodic(const SweepArgs<S>& a, uint32_t x,
                                                   uint32_t y, uint32_t z,
                                                   typename S::T raw[L::Q]) {
  const uint32_t zl = L::D == 3 ? z : y, nl = L::D == 3 ? a.nz : a.ny;
  const bool lo = zl == 0 && a.hrecv[0], hi = zl + 1 == nl && a.hrecv[1];
  if (!lo && !hi) return;
  static_for<1, L::Q>([&](auto I) {
    constexpr int i = decltype(I)::value;
    constexpr Dir v = L::dir(i);
    constexpr int vl = last_component<L>(v);
    if constexpr (vl != 0) {
      if ((vl > 0 && lo) || (vl < 0 && hi)) {
        int32_t sx = (int32_t)x - v.x;
        if (sx < 0) sx += (int32_t)a.nx;
        if (sx >= (int32_t)a.nx) sx -= (int32_t)a.nx;
        uint32_t pc = (uint32_t)sx;
        if constexpr (L::D == 3) {
          int32_t sy = (int32_t)y - v.y;
          if (sy < 0) sy += (int32_t)a.ny;
          if (sy >= (int32_t)a.ny) sy -= (int32_t)a.ny;
          pc += (uint32_t)sy * a.nx;
        }
        const typename S::T* rb = vl > 0 ? a.hrecv[0] : a.hrecv[1];
        raw[i] = load_pop(rb + (uint64_t)halo_rank<L>(i) * a.hplane, pc);
      }
    }
  });
}

// Pack of a face-plane cell's post-collision populations that leave
// through a halo face into that face's send buffer.
template <class L, class S>
__device__ __forceinline__ void halo_pack(const SweepArgs<S>& a, uint32_t c, uint32_t zl,
                                          uint32_t nl, const typename S::R post[L::Q]) {
  using T = typename S::T;
  const uint32_t pc = c - zl * a.hplane;
  const bool lo = zl == 0 && a.hsend[0], hi = zl + 1 == nl && a.hsend[1];
  static_for<1, L::Q>([&](auto I) {
    constexpr int i = decltype(I)::value;
    constexpr int vl = last_component<L>(L::dir(i));
    constexpr int r = halo_rank<L>(i);
    if constexpr (vl < 0) {
      if (lo) a.hsend[0][(uint64_t)r * a.hplane + pc] = narrow<T>(post[i]);
    } else if constexpr (vl > 0) {
      if (hi) a.hsend[1][(uint64_t)r * a.hplane + pc] = narrow<T>(post[i]);
    }
  });
}

// Pull of all populations of a cell whose neighbours need no face rule or
// bounce-back: offsets to the x-1 / x+1 (etc.) neighbours, with wrap-around
// on periodic axes.  kNt: rows are whole 64-cell tiles (nx a multiple of
// 64), so each wavefront's cells are one aligned row segment, and the
// populations with no x velocity are loaded with the non-temporal hint.
template <class L, class S, bool kNt>
__device__ __forceinline__ void pull_periodic(const SweepArgs<S>& a, uint32_t c, uint32_t x,
                                              uint32_t y, uint32_t z,
                                              typename S::T raw[L::Q]) {
  const uint64_t P = a.pstride;
  const int32_t nx = (int32_t)a.nx, nxy = (int32_t)(a.nx * a.ny);
  const int32_t ox_m = x == 0 ? nx - 1 : -1;
  const int32_t ox_p = x == a.nx - 1 ? -(nx - 1) : 1;
  const int32_t oy_m = y == 0 ? (int32_t)(a.ny - 1) * nx : -nx;
  const int32_t oy_p = y == a.ny - 1 ? -(int32_t)(a.ny - 1) * nx : nx;
  int32_t oz_m = 0, oz_p = 0;
  if constexpr (L::D == 3) {
    oz_m = z == 0 ? (int32_t)(a.nz - 1) * nxy : -nxy;
    oz_p = z == a.nz - 1 ? -(int32_t)(a.nz - 1) * nxy : nxy;
  }
  static_for<0, L::Q>([&](auto I) {
    constexpr int i = decltype(I)::value;
    constexpr Dir v = L::dir(i);
    int32_t off = 0;
    if constexpr (v.x > 0) off += ox_m;
    if constexpr (v.x < 0) off += ox_p;
    if constexpr (v.y > 0) off += oy_m;
    if constexpr (v.y < 0) off += oy_p;
    if constexpr (v.z > 0) off += oz_m;
    if constexpr (v.z < 0) off += oz_p;
    // With aligned rows, a population with no x velocity comes from a row
    // segment aligned with this wavefront's cells, whose lines no other
    // wavefront reads; the non-temporal hint keeps those lines from
    // displacing the ones at the segment ends of the other populations,
    // which the neighbouring wavefront reads too (1 % faster on D3Q19 FP32
    // 256^3, 6 % on D2Q9 2048 x 1024; with the hint on every population,
    // no faster; on unaligned rows, where wavefronts share those lines
    // too, 3 % slower).  A template choice, not a branch: the compiler
    // merges identical loads on the two sides of a branch and drops the
    // hint.
    if constexpr (kNt && v.x == 0)
      raw[i] = load_pop_nt(a.src + (uint64_t)i * P, (uint32_t)((int32_t)c + off));
    else
      raw[i] = load_pop(a.src + (uint64_t)i * P, (uint32_t)((int32_t)c + off));
  });
}

// Refinement records of one cell's pre-collision moments: on the parent
// side the nodes on the child box's boundary planes, on the child side the
// band its parent's IMPORT nodes filter.
template <class L, class S>
__device__ __forceinline__ void record_moments(const SweepArgs<S>& a,
                                               const CellMoments<typename S::R>& mo,
                                               uint32_t x, uint32_t y, uint32_t z, uint32_t c) {
  const int64_t r =
      a.rec ? record_index<L::D>(a.rec_off, a.rec_dim, a.box_lo, a.box_hi, x, y, z) : -1;
  if (r >= 0) {
    // ten contiguous values per node (read together by the RING fill)
    typename S::R* rr = a.rec + (uint64_t)r * 10;
    rr[0] = mo.drho;
#pragma unroll
    for (int k = 0; k < 3; ++k) rr[1 + k] = mo.u[k];
#pragma unroll
    for (int k = 0; k < 6; ++k) rr[4 + k] = mo.a2[k];
  }
  if (a.recf && in_import_band<L::D>(x, y, z, a.nx, a.ny, a.nz)) {
    // ten contiguous values per node: the IMPORT filter reads a node's
    // stress components together
    typename S::R* rc = a.recf + (uint64_t)c * 10;
    rc[0] = mo.drho;
#pragma unroll
    for (int k = 0; k < 3; ++k) rc[1 + k] = mo.u[k];
#pragma unroll
    for (int k = 0; k < 6; ++k) rc[4 + k] = mo.a2[k];
  }
}

// Interpolation points and weights of a child node coordinate k along one
// axis (the child box starts at parent coordinate lo): a coincident node
// copies its parent node; a midpoint takes the local cubic (-1, 9, 9, -1)/16.
// Point i is first + i (an array of points, indexed at run time, costs the sweep
// registers: D3Q19 refined jet 384 x 256 x 256 FP32 1624 us a coarse step with one, 1604).
struct AxisPoints {
  int32_t first;
  int n;
};
__device__ __forceinline__ AxisPoints axis_points(int32_t lo, uint32_t k) {
  const int32_t j = lo + (int32_t)(k >> 1);
  return (k & 1u) == 0 ? AxisPoints{j, 1} : AxisPoints{j - 1, 4};
}
__device__ __forceinline__ float axis_weight(const AxisPoints& p, int i) {
  return p.n == 1 ? 1.0f : (i == 0 || i == 3 ? -1.0f / 16.0f : 9.0f / 16.0f);
}

// RING node state (eq. couplingFC): interpolated rho~, u~, Pi~_neq (cubic
// in space, linear in time: wa Ma + wb Mb of the parent's two recorded
// time levels), Pi_neq rescaled by alpha_cf = tau_f / (2 tau_c), then
// f = f^{eqH}(rho~, u~) + (1 - 1/tau_f) f^{neqH}(alpha_cf Pi~_neq, u~),
// encoded for storage.  k: the node's coordinates on the child level.
template <class L, class S>
__device__ __forceinline__ void ring_node(const typename S::R* Ma, const typename S::R* Mb,
                                          typename S::R wa, typename S::R wb,
                                          typename S::R alpha, typename S::R omega1,
                                          typename S::R rho0, const int32_t lo[3],
                                          const int32_t rec_off[3], const uint32_t rec_dim[3],
                                          const uint32_t k[3], typename S::T vals[L::Q]) {
  using R = typename S::R;
  const AxisPoints p0 = axis_points(lo[0], k[0]), p1 = axis_points(lo[1], k[1]);
  const AxisPoints p2 = L::D == 3 ? axis_points(lo[2], k[2]) : AxisPoints{rec_off[2], 1};
  R m[10];
  for (int q = 0; q < 10; ++q) m[q] = (R)0;
  // (unrolled, the points' loads would take registers from every cell's sweep:
  // D2Q9 FP64 122 instead of 73)
#pragma unroll 1
  for (int i2 = 0; i2 < p2.n; ++i2)
#pragma unroll 1
    for (int i1 = 0; i1 < p1.n; ++i1)
#pragma unroll 1
      for (int i0 = 0; i0 < p0.n; ++i0) {
        const uint64_t r = ((uint64_t)(p2.first + i2 - rec_off[2]) * rec_dim[1] +
                            (uint64_t)(p1.first + i1 - rec_off[1])) * rec_dim[0] +
                           (uint64_t)(p0.first + i0 - rec_off[0]);
        const R w = (R)axis_weight(p0, i0) * (R)axis_weight(p1, i1) * (R)axis_weight(p2, i2);
        for (int q = 0; q < 10; ++q) {
          const uint64_t o = r * 10 + (uint64_t)q;
          m[q] += w * (wa * Ma[o] + wb * Mb[o]);
        }
      }
  R u[3] = {m[1], m[2], L::D == 3 ? m[3] : (R)0};
  R a2[6];
  for (int q = 0; q < 6; ++q) a2[q] = alpha * m[4 + q];
  if (L::D == 2) a2[2] = a2[4] = a2[5] = (R)0;
  R out[L::Q];
  rebuild_state<L, R>(m[0], rho0, u, a2, omega1, out);
#pragma unroll
  for (int i = 0; i < L::Q; ++i) vals[i] = encode<S>(out[i], (R)L::w(i) * rho0);
}

// Collision of one cell from its pulled values: post-collision values in the
// storage domain (not yet rounded) and the density the watchdog looks at;
// false for a cell that is not updated.  m: the cell's mask byte (kFluid on
// the periodic path), t_new: time index of the state being produced,
// fixup(raw): the face rules and bounce-back of a FLUID cell's pull.
template <class L, class S, bool kGeneral, class F>
__device__ __forceinline__ bool collide_cell(const SweepArgs<S>& a, uint32_t c, uint32_t x,
                                             uint32_t y, uint32_t z, uint8_t m, uint64_t t_new,
                                             typename S::T raw[L::Q],
                                             typename S::R post[L::Q], typename S::R& rho,
                                             F&& fixup) {
  using R = typename S::R;
  // the rebuilt values are produced directly in the storage domain
  const R base = S::kShifted ? (R)0 : a.rho0;
  R drho, j[3], Pm[6];
  if constexpr (!kGeneral) {
    stored_moments<L, S>(raw, a.rho0, drho, j, Pm);
    if constexpr (L::kColl == kCollBGK)
      rho = collide_bgk<L, S>(raw, drho, j, a.omega1, a.rho0, (R)0, a.rho_ref, a.uref, post);
    else if constexpr (L::kColl == kCollMRT)
      rho = collide_mrt<L, S>(raw, drho, j, a.omega1, a.rho0, post);
    else
      rho = collide_moments<L, R, false, !S::kShifted>(drho, j, Pm, a.omega1, a.rho0, (R)0, a.rho_ref,
                                         a.uref, base, post);
  } else {
    const uint8_t kind = m & kKindBits;
    if (kind == kSolid || kind >= kCovered) return false;
    // one rebuild for every kind of cell keeps the kernel's code compact
    // (the comparators collide without it)
    Coeffs<L, R> cf;
    bool rebuild = true;
    if (kind == kInlet) {
      // f^{eqH}(rho0, U u_dir (1 + noise r)), r from SplitMix64
      R u[3];
      const uint64_t bidx =
          ((t_new * (uint64_t)a.lstride + (uint64_t)a.level) * (uint64_t)a.ncell + c) * 3ull;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        // (without noise the generator is not run)
        const R r = a.noise != (R)0 ? (R)splitmix_pm1(a.seed, bidx + (uint64_t)k) : (R)0;
        u[k] = a.uin[k] * ((R)1 + a.noise * r);
      }
      if (L::D == 2) u[2] = (R)0;
      const R zero6[6] = {(R)0, (R)0, (R)0, (R)0, (R)0, (R)0};
      state_coeffs<L, R>((R)0, a.rho0, u, zero6, (R)0, cf);
      rho = a.rho0;
    } else {
      fixup(raw);
      stored_moments<L, S>(raw, a.rho0, drho, j, Pm);
      R chi = (R)0, rref = a.rho_ref, uref[3] = {a.uref[0], a.uref[1], a.uref[2]};
      if (m & kFieldSponge) {
        chi = a.sp[c];
        rref = a.sp[a.ncell + c];
#pragma unroll
        for (int k = 0; k < 3; ++k) uref[k] = a.sp[(uint64_t)(2 + k) * a.ncell + c];
      } else if (a.chi_max != (R)0) {
        chi = sponge_chi<R>(a.sponge, a.chi_max, x, y, z, a.nx, a.ny, a.nz);
      }
      if constexpr (L::kColl == kCollBGK) {
        rho = collide_bgk<L, S>(raw, drho, j, a.omega1, a.rho0, chi, rref, uref, post);
        rebuild = false;
      } else if constexpr (L::kColl == kCollMRT) {
        rho = collide_mrt<L, S>(raw, drho, j, a.omega1, a.rho0, post);
        rebuild = false;
      } else {
        // (the moments are always returned in registers; a conditional
        // pointer here would push them to scratch memory)
        CellMoments<R> mo;
        rho = collide_coeffs<L, R, true>(drho, j, Pm, a.omega1, a.rho0, chi, rref, uref, cf,
                                         &mo);
        if (a.rec || a.recf) record_moments<L, S>(a, mo, x, y, z, c);
      }
    }
    if (rebuild) rebuild_from<L, R, !S::kShifted>(cf, base, post);
  }
  return true;
}

// sweep arguments of one storage format from the format-neutral host block
template <class S>
__host__ __device__ inline SweepArgs<S> to_args_dev(const SweepHost& h) {
  using T = typename S::T;
  using R = typename S::R;
  SweepArgs<S> a;
  a.src = (const T*)h.src;
  a.dst = (T*)h.dst;
  a.mask = h.mask;
  a.tiles = h.tiles;
  a.status = h.status;
  a.nx = h.nx;
  a.ny = h.ny;
  a.nz = h.nz;
  a.ncell = h.nx * h.ny * h.nz;
  a.pstride = h.pstride;
#if !defined(__HIP_DEVICE_COMPILE__)
  a.div_nx = make_fastdiv(h.nx);
  a.div_ny = make_fastdiv(h.ny);
#endif
  a.omega1 = (R)(1.0 - 1.0 / h.tau);
  a.rho0 = (R)h.rho0;
  a.chi_max = (R)h.chi_max;
  a.rho_ref = (R)h.rho_ref;
  for (int k = 0; k < 3; ++k) {
    a.uref[k] = (R)h.uref[k];
    a.uin[k] = (R)h.uin[k];
  }
  a.noise = (R)h.noise;
  for (int f = 0; f < 6; ++f) {
    a.face[f] = h.face[f];
    a.sponge[f] = h.sponge[f];
  }
  a.seed = h.seed;
  a.t_new = h.t_new;
  a.level = h.level;
  a.lstride = h.lstride;
  a.ntiles = 0;
  a.xcd_group = 1;
  a.rec = (R*)h.rec;
  a.recf = (R*)h.recf;
  a.sp = (const R*)h.sp;
  for (int k = 0; k < 3; ++k) {
    a.rec_off[k] = h.rec_off[k];
    a.rec_dim[k] = h.rec_dim[k];
    a.box_lo[k] = h.box_lo[k];
    a.box_hi[k] = h.box_hi[k];
  }
  a.rec_n = h.rec_n;
  a.ring_Ma = (const R*)h.ring_Ma;
  a.ring_Mb = (const R*)h.ring_Mb;
  a.ring_wa = (R)h.ring_wa;
  a.ring_wb = (R)h.ring_wb;
  a.ring_alpha = (R)h.ring_alpha;
  for (int k = 0; k < 3; ++k) {
    a.ring_lo[k] = h.ring_lo[k];
    a.ring_off[k] = h.ring_off[k];
    a.ring_dim[k] = h.ring_dim[k];
  }
  for (int k = 0; k < 2; ++k) {
    a.hrecv[k] = (const T*)h.hrecv[k];
    a.hsend[k] = (T*)h.hsend[k];
  }
  a.hplane = h.hplane;
  return a;
}

}  // namespace hrlbm
