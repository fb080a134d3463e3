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

// Block size and chunk length of a pass over parts[p] systems[i] systems of each instance, for
// every p at once: every block size, with z-chunks of one length for all, by the cost model of
// shape_for with the blocks of all instances in one pool (whole rounds of the chip, and half of
// the longest block for the ragged end).  What a candidate costs is linear in the systems up to
// the rounds, so an instance is visited once per candidate whatever the parts, with a few
// additions each: the search runs on the host while the GPU waits (512 instances, three kinds of
// pass, four parts: 1.1 ms; rebuilding every geometry for every part took 20 ms).
struct ClassBest {
  double tm = 1e300;
  int w = 0, small = 0, cz = 0;
};
template <typename T, int NF, bool EXTRA, bool RESID, bool SM>
void class_try(const std::vector<GridDesc>& g, const std::vector<double>& systems, const std::vector<double>& parts,
               std::vector<ClassBest>& best) {
  using C = Cfg<T, NF, EXTRA, SM>;
  const size_t n = g.size();
  constexpr int kIters[] = {8, 12, 16, 24, 32, 48, 64, 96, 128}, kN = 9;
  std::vector<int> gx(n), gy(n), cap(n), nzc(n * kN), len(n * kN);
  std::vector<double> hbm(parts.size(), 0.0);
  double pts = 0.0;
  int step;
  for (size_t i = 0; i < n; ++i) {
    gx[i] = tiles<NF>(g[i].nx, 64, step);
    const int limit = std::min(g[i].nz, chunk_limit<T>(g[i]));
    for (int m = 0; m < kN; ++m) {
      len[m * n + i] = std::min(kIters[m] - 2 * (NF - 1), limit);
      nzc[m * n + i] = (g[i].nz + len[m * n + i] - 1) / len[m * n + i];
    }
    // enough blocks to fill the chip eight times over with one system, or what the longest
    // chunks and largest blocks give
    cap[i] = std::max(2048, gx[i] * tiles<NF>(g[i].ny, C::WMAX * C::R, step) * nzc[(kN - 1) * n + i]);
    const double p = (double)g[i].nx * g[i].ny * g[i].nz;
    pts += p * systems[i];
    for (size_t k = 0; k < parts.size(); ++k) hbm[k] += hbm_bytes<T, EXTRA, RESID>(p, systems[i] * parts[k]);
  }
  for (int w = C::WMAX; w >= 2; --w) {
    const int rb = w * C::R, bpc = blocks_per_cu<T, NF, C>(w);
    if (lds_bytes(NF, w, 2 * sizeof(T)) > 160 * 1024) continue;
    bool ok = true;
    for (size_t i = 0; i < n; ++i) {
      ok = ok && (g[i].ny <= rb || rb > 2 * NF);
      gy[i] = ok ? tiles<NF>(g[i].ny, rb, step) : 0;
    }
    if (!ok) continue;
    for (int m = 0; m < kN; ++m) {
      // per unit of parts: blocks, planes they load, planes they step through; the longest block
      double blocks = 0.0, planes = 0.0, iters = 0.0;
      int most = 0, over = 0;
      for (size_t i = 0; i < n; ++i) {
        const int per = gx[i] * gy[i] * nzc[m * n + i], l = len[m * n + i], it = block_iters<NF>(l);
        const double v = systems[i] * per;
        over |= per > cap[i];
        blocks += v;
        planes += v * (l + 2 * NF);
        iters += v * it;
        most = std::max(most, it);
      }
      if (over) continue;
      for (size_t k = 0; k < parts.size(); ++k) {
        const double conc = std::max(1.0, std::min((double)bpc, std::ceil(blocks * parts[k] / 256.0)));
        const double c = iter_cycles<T, NF, EXTRA, RESID, SM>(w, conc), longest = most * c + kBlockCycles;
        const double sum = parts[k] * (iters * c + blocks * kBlockCycles);
        const double comp = std::max(longest, sum / (256.0 * conc) + 0.5 * longest);
        const double tm = launch_cycles(comp, hbm[k], l2_bytes<T, NF, EXTRA, SM>(w, parts[k] * planes, parts[k] * pts));
        if (tm < best[k].tm) best[k] = ClassBest{tm, w, SM ? 1 : 0, kIters[m] - 2 * (NF - 1)};
      }
    }
  }
}

template <typename T, int NF, bool EXTRA, bool RESID>
bool class_of(const std::vector<GridDesc>& g, const std::vector<double>& systems, const std::vector<double>& parts,
              RowsClass* c, std::vector<RowsShape>* shapes) {
  std::vector<ClassBest> best(parts.size());
  class_try<T, NF, EXTRA, RESID, false>(g, systems, parts, best);
  class_try<T, NF, EXTRA, RESID, true>(g, systems, parts, best);
  for (size_t k = 0; k < parts.size(); ++k) {
    const ClassBest& b = best[k];
    if (b.w == 0) return false;
    c[k].w = b.w;
    c[k].small = b.small;
    shapes[k].resize(g.size());
    for (size_t i = 0; i < g.size(); ++i)
      if (b.small) shape_of<T, NF, EXTRA, true>(g[i], b.w, b.cz, shapes[k][i]);
      else shape_of<T, NF, EXTRA, false>(g[i], b.w, b.cz, shapes[k][i]);
  }
  return true;
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
bool MultiLaunch<T2>::rows_class(const std::vector<GridDesc>& g, const std::vector<double>& systems,
                                 const std::vector<double>& parts, RowsClass* c, std::vector<RowsShape>* shapes) {
  using T = typename zrows::Elem<T2>::t;
  auto of = [&](auto nfc) {
    constexpr int NF = decltype(nfc)::value;
    return (c[0].kind & kFacResid) ? zrows::class_of<T, NF, true, true>(g, systems, parts, c, shapes)
           : (c[0].kind & kFacAdd) ? zrows::class_of<T, NF, true, false>(g, systems, parts, c, shapes)
                                   : zrows::class_of<T, NF, false, false>(g, systems, parts, c, shapes);
  };
  if (c[0].width == 2) return of(std::integral_constant<int, 2>{});
  if (c[0].width == 3) return of(std::integral_constant<int, 3>{});
  if constexpr (sizeof(T2) == 8)
    if (c[0].width == 4) return of(std::integral_constant<int, 4>{});
  return false;
}

}  // namespace hfci
