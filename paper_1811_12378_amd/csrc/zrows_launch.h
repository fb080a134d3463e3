// Kernels and launches of zrows.h for one precision (included by zrows_f32.hip and
// zrows_f64.hip, which compile in parallel).
#pragma once

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "zrows.h"

namespace hfci {
namespace zrows {

// Rows per lane and the largest block, by precision, factors and extra stream (f or y1): the
// most rows whose planes of state stay in registers without spills, at three waves per SIMD
// (168 registers, blocks of up to 12 waves), or two where three would leave a lane one row.
// SM: few rows per lane, for launches that cannot fill the chip: a plane then costs the
// barrier and the LDS exchange more than the arithmetic.
template <typename T, int NF, bool EXTRA, bool SM>
struct Cfg {
  static constexpr bool kF32 = sizeof(T) == 4;
  static constexpr int R = SM     ? (kF32 ? 2 : 1)
                           : kF32 ? (NF == 2 ? 4 : NF == 3 ? (EXTRA ? 3 : 4) : (EXTRA ? 2 : 3))
                                  : (NF == 2 ? (EXTRA ? 2 : 3) : (EXTRA ? 3 : 2));
  static constexpr int WPE = SM ? (NF == 4 ? 3 : 4) : (!kF32 && NF == 3 && EXTRA) ? 2 : 3;  // waves per SIMD
  static constexpr int WMAX = 4 * WPE;
};

template <typename T, int KIND, int NF, bool SM>
struct KindCfg : Cfg<T, NF, (KIND & (kFacResid | kFacAdd)) != 0, SM> {};

template <typename T, int KIND, int NF, bool SM>
__global__ __launch_bounds__((64 * KindCfg<T, KIND, NF, SM>::WMAX))
    __attribute__((amdgpu_waves_per_eu((KindCfg<T, KIND, NF, SM>::WPE)))) void zrows_kernel(
        GridDesc g, RowsShape q, int sgrp, FactorArgs<typename V2<T>::t> a, const T* __restrict__ K) {
  extern __shared__ __align__(16) char lds[];
  // block order: see pair_block in stencil.hip
  const int per_sys = q.per_sys, xcd_slab = q.xcd_slab;
  int li, b;
  if (xcd_slab > 0 && sgrp > 1) {
    const int xcd = blockIdx.x % 8, k = blockIdx.x / 8;
    const int gsz = sgrp * xcd_slab;
    const int s0 = (k / gsz) * sgrp, r = k % gsz;
    const int gs = min(sgrp, a.count - s0);
    li = s0 + r % gs;
    b = xcd * xcd_slab + r / gs;
  } else {
    li = blockIdx.x / per_sys;
    b = blockIdx.x % per_sys;
    if (xcd_slab > 0) b = (b % 8) * xcd_slab + b / 8;
  }
  const int s = __builtin_amdgcn_readfirstlane(a.list[li]);
  if (s < 0) return;  // a stopped system past the end of the active list (uniform)
  rows_tile<T, KIND, NF, KindCfg<T, KIND, NF, SM>::R>(g, q, s, b, a, K, lds);
}

// The longest z-chunk whose planes (with the halo) 32-bit offsets reach
template <typename T>
int chunk_limit(const GridDesc& g) {
  const double planes = 2147483647.0 / ((double)g.nx * g.ny * 2 * sizeof(T));
  return (int)std::min(planes, 1e6) - 10;
}

// tiles of `len` points covering n, and the distance between them
template <int NF>
int tiles(int n, int len, int& step) {
  step = 0;
  if (n <= len) return 1;
  const int k = 1 + (n - len + len - 2 * NF - 1) / (len - 2 * NF);
  step = (n - len + k - 2) / (k - 1);
  return k;
}

// The largest number of blocks per system a geometry may have: enough to fill the chip eight
// times over with one system, or what the longest chunks and largest blocks give
template <typename T, int NF, bool EXTRA>
int rows_cap(const GridDesc& g) {
  using C = Cfg<T, NF, EXTRA, false>;
  const KernelTune& t = sizeof(T) == 4 ? g.tune32 : g.tune64;
  const int cz = std::min(t.cz > 0 ? t.cz : 126, chunk_limit<T>(g));
  int step;
  return std::max(2048, tiles<NF>(g.nx, 64, step) * tiles<NF>(g.ny, C::WMAX * C::R, step) * ((g.nz + cz - 1) / cz));
}

// the geometry with blocks of w waves and z-chunks of cz planes; false where it cannot be used
template <typename T, int NF, bool EXTRA, bool SM>
bool shape_of(const GridDesc& g, int w, int cz, RowsShape& s) {
  using C = Cfg<T, NF, EXTRA, SM>;
  const int rb = w * C::R;
  if ((g.ny > rb && rb <= 2 * NF) || lds_bytes(NF, w, 2 * sizeof(T)) > 160 * 1024) return false;
  s.w = w;
  s.small = SM ? 1 : 0;
  s.gx = tiles<NF>(g.nx, 64, s.sx);
  if (s.sx > 0) s.sx = std::min((s.sx + 7) / 8 * 8, 64 - 2 * NF);  // rows start on 64-byte lines where they can
  s.gy = tiles<NF>(g.ny, rb, s.sy);
  s.czlen = std::min(std::min(cz, g.nz), chunk_limit<T>(g));
  s.nzc = (g.nz + s.czlen - 1) / s.czlen;
  s.per_sys = s.gx * s.gy * s.nzc;
  s.xcd_slab = (s.per_sys % 8 == 0 && s.per_sys >= 64) ? s.per_sys / 8 : 0;
  s.inv_sh2 = 1.0 / g.s_h2;
  s.damp_sh2 = g.damp_scale / g.s_h2;
  return true;
}

// Blocks of w waves on a CU at once, by registers (C::WMAX waves) and LDS (complex128 with three
// factors: 30 KB for 2 waves, 55 KB for 4)
template <typename T, int NF, class C>
int blocks_per_cu(int w) {
  return std::max(1, std::min(C::WMAX / w, (int)(160 * 1024 / lds_bytes(NF, w, 2 * sizeof(T)))));
}

// Planes a block steps through for a chunk, and CU cycles (2.4 GHz) of one of them for a block of
// w waves with `conc` blocks on its CU at once; a block costs kBlockCycles beside.
template <int NF>
int block_iters(int czlen) { return (czlen + 2 * (NF - 1) + 3) / 4 * 4; }
template <typename T, int NF, bool EXTRA, bool RESID, bool SM>
double iter_cycles(int w, double conc) {
  const double v = Cfg<T, NF, EXTRA, SM>::R * (NF * (sizeof(T) == 4 ? 83.0 : 137.0) + (RESID ? 72.0 : 0.0));
  return std::max(std::ceil(w * conc / 4) * v * 1.19, 820.0 + v * 1.02);
}
constexpr double kBlockCycles = 6100.0;

// Bytes of HBM of a launch over `count` systems of `pts` points each, and bytes requested of the
// L2s by blocks of w waves that load `planes` planes in all, for `pts` points in all
template <typename T, bool EXTRA, bool RESID>
double hbm_bytes(double pts, double count) {
  const double e = 2 * sizeof(T);
  return pts * count * (2.5 * e + (RESID ? e / std::max(count, 1.0) : EXTRA ? e : 0.0));
}
template <typename T, int NF, bool EXTRA, bool SM>
double l2_bytes(int w, double planes, double pts) {
  const double e = 2 * sizeof(T);
  return planes * 64 * w * Cfg<T, NF, EXTRA, SM>::R * 1.5 * e + pts * (EXTRA ? 2.0 : 1.0) * e;
}

// memory time (cycles) overlaps with all but a quarter of the shorter of the two
inline double launch_cycles(double comp, double hbm, double l2) {
  const double mem = 2400.0 * std::max(hbm / 5.16e6, l2 / 9.34e6);
  return std::max(comp, mem) + 0.25 * std::min(comp, mem);
}

template <typename T, int NF, bool EXTRA, bool RESID, bool SM>
void shape_try(const GridDesc& g, int count, RowsShape& best, double& best_t, RowsShape& any) {
  using C = Cfg<T, NF, EXTRA, SM>;
  const KernelTune& t = sizeof(T) == 4 ? g.tune32 : g.tune64;
  const int climit = chunk_limit<T>(g), cap = rows_cap<T, NF, EXTRA>(g);
  for (int w = C::WMAX; w >= 2; --w) {
    if (w > 2 && (w - 1) * C::R >= g.ny) continue;  // a smaller block covers every row
    const int bpc = blocks_per_cu<T, NF, C>(w);
    for (const int m : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32}) {
      const int cz = t.cz > 0 ? t.cz : 4 * m - 2 * (NF - 1) % 4;
      RowsShape s;
      if (!shape_of<T, NF, EXTRA, SM>(g, w, cz, s)) break;
      const double blocks = (double)s.per_sys * count;
      const double conc = std::max(1.0, std::min((double)bpc, std::ceil(blocks / 256.0)));
      const double full = std::floor(blocks / (256.0 * conc)), rest = blocks - full * 256.0 * conc;
      auto block = [&](double n) {
        return block_iters<NF>(s.czlen) * iter_cycles<T, NF, EXTRA, RESID, SM>(w, n) + kBlockCycles;
      };
      const double comp = full * block(conc) + (rest > 0 ? block(std::ceil(rest / 256.0)) : 0.0);
      const double pts = (double)g.nx * g.ny * g.nz;
      const double tm = launch_cycles(comp, hbm_bytes<T, EXTRA, RESID>(pts, count),
                                      l2_bytes<T, NF, EXTRA, SM>(w, blocks * (s.czlen + 2 * NF), pts * count));
      if (s.per_sys <= cap && tm < best_t) {
        best_t = tm;
        best = s;
      }
      if (any.w == 0 || s.per_sys < any.per_sys) any = s;
      if (t.cz > 0 || cz >= g.nz || cz >= climit) break;
    }
  }
}

// Geometry of a pass over `count` systems.  Candidates: blocks of 2 .. WMAX waves and z-chunks
// of 2 .. 128 planes (those for which a chunk's iterations fill whole trips of four), or the
// launch shape's chunk.  A block's planes cost its vector instructions or, with few waves on
// a CU, the latency of a barrier and the LDS exchange; short chunks repeat 2 (NF - 1) planes,
// small blocks 2 NF rows; long chunks and large blocks leave CUs idle where systems are few.
// The constants are fitted to 6300 measured launches (32^3 to 256^3, 1 to 24 systems, both
// precisions, every kind): the geometry chosen costs 4 % more than the best measured one on
// average (33 % at worst), where one fixed geometry per grid costs 30 % and more at either end.
template <typename T, int NF, bool EXTRA, bool RESID>
RowsShape shape_for(const GridDesc& g, int count) {
  RowsShape best{}, any{};
  double best_t = 1e300;
  shape_try<T, NF, EXTRA, RESID, false>(g, count, best, best_t, any);
  shape_try<T, NF, EXTRA, RESID, true>(g, count, best, best_t, any);
  return best.w == 0 ? any : best;
}

template <typename T, int KIND, int NF>
void run(hipStream_t st, const GridDesc& g, const void* kappa, const FactorArgs<typename V2<T>::t>& a,
         const RowsShape& s) {
  const int sg = sizeof(T) == 4 ? g.tune32.sg : g.tune64.sg;
  const dim3 grid((unsigned)s.per_sys * (unsigned)a.count), block(64 * s.w);
  const size_t lds = lds_bytes(NF, s.w, 2 * sizeof(T));
  if (s.small)
    hipLaunchKernelGGL((zrows_kernel<T, KIND, NF, true>), grid, block, lds, st, g, s, sg, a, (const T*)kappa);
  else
    hipLaunchKernelGGL((zrows_kernel<T, KIND, NF, false>), grid, block, lds, st, g, s, sg, a, (const T*)kappa);
}

template <typename T, int NF>
bool run_kind(hipStream_t st, const GridDesc& g, const void* kappa, const FactorArgs<typename V2<T>::t>& a, int kind,
              const RowsShape& s) {
  switch (kind) {
    case 0: run<T, 0, NF>(st, g, kappa, a, s); return true;
    case kFacResid: run<T, kFacResid, NF>(st, g, kappa, a, s); return true;
    case kFacAdd: run<T, kFacAdd, NF>(st, g, kappa, a, s); return true;
    case kFacDual: run<T, kFacDual, NF>(st, g, kappa, a, s); return true;
    case kFacInF: run<T, kFacInF, NF>(st, g, kappa, a, s); return true;
    case kFacInF | kFacDual: run<T, kFacInF | kFacDual, NF>(st, g, kappa, a, s); return true;
    default: return false;
  }
}

}  // namespace zrows

template <typename T2>
bool Launch<T2>::factor_rows(hipStream_t st, const GridDesc& g, const void* kappa, const FactorArgs<T2>& a, int kind,
                             int nf, const RowsShape& sh) {
  using T = typename zrows::Elem<T2>::t;
  if (a.count <= 0) return true;
  if (nf == 2) return zrows::run_kind<T, 2>(st, g, kappa, a, kind, sh);
  if (nf == 3) return zrows::run_kind<T, 3>(st, g, kappa, a, kind, sh);
  if constexpr (sizeof(T2) == 8)
    if (nf == 4) return zrows::run_kind<T, 4>(st, g, kappa, a, kind, sh);
  return false;
}

template <typename T2>
RowsShape Launch<T2>::rows_shape(const GridDesc& g, int nf, int kind, int count) {
  using T = typename zrows::Elem<T2>::t;
  auto of = [&](auto nfc) {
    constexpr int NF = decltype(nfc)::value;
    return (kind & kFacResid) ? zrows::shape_for<T, NF, true, true>(g, count)
           : (kind & kFacAdd) ? zrows::shape_for<T, NF, true, false>(g, count)
                              : zrows::shape_for<T, NF, false, false>(g, count);
  };
  if (nf == 2) return of(std::integral_constant<int, 2>{});
  if (nf == 3) return of(std::integral_constant<int, 3>{});
  if constexpr (sizeof(T2) == 8)
    if (nf == 4) return of(std::integral_constant<int, 4>{});
  return RowsShape{};
}

template <typename T2>
bool Launch<T2>::rows_fits(const GridDesc& g) {
  return zrows::chunk_limit<typename zrows::Elem<T2>::t>(g) >= 4;
}

template <typename T2>
bool Launch<T2>::rows_run(const GridDesc& g) {
  const KernelTune& t = sizeof(T2) == 8 ? g.tune32 : g.tune64;
  // kerns 2 and 3 are the complex64 kernels that stream into LDS; where the grid does not
  // suit them (an odd nx, vectors of 2 GiB or more) their shapes run these passes too
  return t.fuse != 0 && (t.kern <= 1 || !streams_fit(g)) && rows_fits(g);
}

}  // namespace hfci
