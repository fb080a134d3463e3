// Multi-factor passes in registers (zrows.h) over the systems of many operators (included by
// zrows_multi_f32.hip and zrows_multi_f64.hip).
#pragma once

#include "zrows_launch.h"

namespace hfci {
namespace zrows {

// A block finds its system in the work table (binary search over the first-block column), reads
// the system's vectors, its operator's grid and this pass's geometry for it, and runs that tile.
template <typename T, int KIND, int NF, bool SM>
__global__ __launch_bounds__((64 * KindCfg<T, KIND, NF, SM>::WMAX))
    __attribute__((amdgpu_waves_per_eu((KindCfg<T, KIND, NF, SM>::WPE)))) void zrows_multi_kernel(
        const MultiInst* __restrict__ inst, const RowsShape* __restrict__ shapes,
        const MultiSys<typename V2<T>::t>* __restrict__ sys, const int2* __restrict__ seg, int nseg, int rin, int rout,
        int rout2, int k, int cstride) {
  using T2 = typename V2<T>::t;
  extern __shared__ __align__(16) char lds[];
  const int blk = blockIdx.x;
  int lo = 0, hi = nseg - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (seg[mid].x <= blk) lo = mid;
    else hi = mid - 1;
  }
  const int2 row = seg[lo];
  const int G = __builtin_amdgcn_readfirstlane(row.y);
  if (G < 0) return;  // past the live rows of a table rebuilt since the launch was sized
  int b = __builtin_amdgcn_readfirstlane(blk - row.x);
  // fields are read through the pointer: a dynamic index into a copied descriptor
  // (vec[role]) would put the copy in scratch memory
  const MultiSys<T2>* __restrict__ sd = sys + G;
  const int in = sd->inst;
  const RowsShape q = shapes[in];
  if (q.xcd_slab > 0) b = (b % 8) * q.xcd_slab + b / 8;
  FactorArgs<T2> a{};
  a.win = sd->vec[rin];
  a.f = sd->vec[kRoleF];
  a.y1 = sd->vec[kRoleY1];
  a.wout = sd->vec[rout];
  a.wout2 = rout2 >= 0 ? sd->vec[rout2] : nullptr;
  a.coef = sd->coef;
  a.poles = sd->pole;
  a.partial = sd->partial;
  a.count = 1;
  a.nrhs = 1;
  a.cstride = cstride;
  a.k = k;
  rows_tile<T, KIND, NF, KindCfg<T, KIND, NF, SM>::R>(inst[in].g, q, 0, b, a, (const T*)inst[in].kappa, lds);
}

// Block size and per-instance geometry of a pass over `systems[i]` systems of each instance:
// every block size, with z-chunks of one length for all, by the cost model of shape_for with
// the blocks of all instances in one pool (whole rounds of the chip, and half of the longest
// block for the ragged end).
template <typename T, int NF, bool EXTRA, bool RESID, bool SM>
void class_try(const std::vector<GridDesc>& g, const std::vector<double>& systems, RowsClass& best, double& best_t,
               std::vector<RowsShape>& shapes) {
  using C = Cfg<T, NF, EXTRA, SM>;
  std::vector<RowsShape> s(g.size());
  for (int w = C::WMAX; w >= 2; --w) {
    const int bpc = std::max(1, C::WMAX / w);
    for (const int iters : {8, 12, 16, 24, 32, 48, 64, 96, 128}) {
      const int cz = iters - 2 * (NF - 1);
      double blocks = 0.0, hbm = 0.0, l2 = 0.0;
      bool ok = true;
      for (size_t i = 0; i < g.size() && ok; ++i) {
        ok = shape_of<T, NF, EXTRA, SM>(g[i], w, cz, s[i]) && s[i].per_sys <= rows_cap<T, NF, EXTRA>(g[i]);
        double h, l;
        launch_bytes<T, NF, EXTRA, RESID, SM>(g[i], s[i], systems[i], h, l);
        blocks += systems[i] * s[i].per_sys;
        hbm += h;
        l2 += l;
      }
      if (!ok) continue;
      const double conc = std::max(1.0, std::min((double)bpc, std::ceil(blocks / 256.0)));
      double sum = 0.0, longest = 0.0;
      for (size_t i = 0; i < g.size(); ++i) {
        const double t = block_cycles<T, NF, EXTRA, RESID, SM>(w, s[i].czlen, conc);
        sum += t * systems[i] * s[i].per_sys;
        longest = std::max(longest, t);
      }
      const double comp = std::max(longest, sum / (256.0 * conc) + 0.5 * longest);
      const double tm = launch_cycles(comp, hbm, l2);
      if (tm < best_t) {
        best_t = tm;
        best.w = w;
        best.small = SM ? 1 : 0;
        shapes = s;
      }
    }
  }
}

template <typename T, int NF>
void class_for(const std::vector<GridDesc>& g, const std::vector<double>& systems, int kind, RowsClass& c,
               std::vector<RowsShape>& shapes) {
  double t = 1e300;
  if (kind & kFacResid) {
    class_try<T, NF, true, true, false>(g, systems, c, t, shapes);
    class_try<T, NF, true, true, true>(g, systems, c, t, shapes);
  } else if (kind & kFacAdd) {
    class_try<T, NF, true, false, false>(g, systems, c, t, shapes);
    class_try<T, NF, true, false, true>(g, systems, c, t, shapes);
  } else {
    class_try<T, NF, false, false, false>(g, systems, c, t, shapes);
    class_try<T, NF, false, false, true>(g, systems, c, t, shapes);
  }
}

template <typename T, int KIND, int NF>
void run_multi(hipStream_t st, const RowsClass& c, const MultiInst* inst, const RowsShape* shapes,
               const MultiSys<typename V2<T>::t>* sys, const int2* seg, int nseg, int nblocks, int rin, int rout,
               int rout2, int k, int cstride) {
  const dim3 grid((unsigned)nblocks), block(64 * c.w);
  const size_t lds = lds_bytes(NF, c.w, 2 * sizeof(T));
  if (c.small)
    hipLaunchKernelGGL((zrows_multi_kernel<T, KIND, NF, true>), grid, block, lds, st, inst, shapes, sys, seg, nseg, rin,
                       rout, rout2, k, cstride);
  else
    hipLaunchKernelGGL((zrows_multi_kernel<T, KIND, NF, false>), grid, block, lds, st, inst, shapes, sys, seg, nseg,
                       rin, rout, rout2, k, cstride);
}

template <typename T, int NF, class... A>
bool run_multi_kind(int kind, A... a) {
  switch (kind) {
    case 0: run_multi<T, 0, NF>(a...); return true;
    case kFacResid: run_multi<T, kFacResid, NF>(a...); return true;
    case kFacAdd: run_multi<T, kFacAdd, NF>(a...); return true;
    case kFacDual: run_multi<T, kFacDual, NF>(a...); return true;
    case kFacInF: run_multi<T, kFacInF, NF>(a...); return true;
    case kFacInF | kFacDual: run_multi<T, kFacInF | kFacDual, NF>(a...); return true;
    default: return false;
  }
}

}  // namespace zrows

template <typename T2>
bool MultiLaunch<T2>::factor_rows(hipStream_t st, const RowsClass& c, const MultiInst* inst, const RowsShape* shapes,
                                  const MultiSys<T2>* sys, const int2* seg, int nseg, int nblocks, int kind, int rin,
                                  int rout, int rout2, int k, int cstride) {
  using T = typename zrows::Elem<T2>::t;
  if (nseg <= 0 || nblocks <= 0) return true;
  if (c.width == 2)
    return zrows::run_multi_kind<T, 2>(kind, st, c, inst, shapes, sys, seg, nseg, nblocks, rin, rout, rout2, k, cstride);
  if (c.width == 3)
    return zrows::run_multi_kind<T, 3>(kind, st, c, inst, shapes, sys, seg, nseg, nblocks, rin, rout, rout2, k, cstride);
  if constexpr (sizeof(T2) == 8)
    if (c.width == 4)
      return zrows::run_multi_kind<T, 4>(kind, st, c, inst, shapes, sys, seg, nseg, nblocks, rin, rout, rout2, k,
                                         cstride);
  return false;
}

template <typename T2>
RowsClass MultiLaunch<T2>::rows_class(const std::vector<GridDesc>& g, const std::vector<double>& systems, int width,
                                      int kind, std::vector<RowsShape>& shapes) {
  using T = typename zrows::Elem<T2>::t;
  RowsClass c;
  c.width = width;
  c.kind = kind & (kFacResid | kFacAdd);
  if (width == 2) zrows::class_for<T, 2>(g, systems, kind, c, shapes);
  if (width == 3) zrows::class_for<T, 3>(g, systems, kind, c, shapes);
  if constexpr (sizeof(T2) == 8)
    if (width == 4) zrows::class_for<T, 4>(g, systems, kind, c, shapes);
  return c;
}

}  // namespace hfci
