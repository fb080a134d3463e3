// Several consecutive factors of the product-form fixed-point step in one pass over HBM
// (temporal blocking), planes held in registers: the launches of the shapes with fuse 1 and
// kern 0 or 1 (a new operator's among them) and, where the grid does not suit kerns 2 and 3, of theirs.
//
//   t_1 = a_1 (A - z0) w + b_1 w,  t_f = a_f (A - z0) t_{f-1} + b_f t_{f-1},  out = t_NF [+ y1]
//
// with NF = 2, 3 or 4 factors, complex64 or complex128.
//
// What bounds it: a pass moves 16 (8 + 8) bytes per point and system in complex64 whatever the
// number of factors, so at large grids the pass count of a step is what costs time, and at
// small ones the launches are.  The tile-in-LDS kernels (two factors, or three for the middle
// ones) are limited in depth by LDS, by one ring of planes per extra stream, and issue four LDS
// reads per point and factor.  Here a lane owns one column x and R consecutive rows y, a wave
// 64 columns, a block W waves stacked in y:
//   * the z-neighbours are earlier and later planes of the same registers;
//   * the y-neighbours are other registers of the same lane, except at a wave's first and last
//     row, which go through LDS (two rows written and two read per wave, plane and factor);
//   * the x-neighbours are the adjacent lanes' registers (DPP wave shifts, part of the add).
// Per plane k: level 1 (the first factor) at plane k, level 2 at k - 1, ... level NF at
// k - NF + 1, with one barrier: every edge row read after it was written before it, into the
// other of two LDS buffers.  Memory streams (input two planes ahead of its use as centre,
// kappa, and f or y1 one plane ahead) go straight to registers, so an extra stream costs
// registers only, and every kind of launch runs at every NF.
//
// Tiles are 64 x RB points (RB = W R) at every level; a level's outermost points on a side are
// wrong where the tile ends inside the grid (its neighbours there are not known), so outputs
// keep NF points away from such sides and neighbouring tiles overlap by 2 NF.  Where the tile
// ends at the grid's edge the missing neighbours are the Dirichlet zeros: nothing is lost
// there, and tiles are placed so that the last one ends at the edge too.
//
// Arithmetic: a (A - z0) x + b x = a sh2 (m x - nb), nb the sum of the six neighbours and
// m = 6 - z0 / sh2 + b / (a sh2) - kappa / sh2 - i D / sh2; the scalars a sh2 of a pass are
// multiplied together, corrected for the rounding of the constants (complete_coefficients), and
// applied once to its output.  17 vector instructions per point and
// factor in complex64 (10 adds for nb, 3 for m, 4 multiply-adds), 4 more per point and pass.
#pragma once

#include "kernels.h"

namespace hfci {
namespace zrows {

template <typename T> struct V2;
template <> struct V2<float> { using t = float2; };
template <> struct V2<double> { using t = double2; };
template <typename T2> struct Elem;
template <> struct Elem<float2> { using t = float; };
template <> struct Elem<double2> { using t = double; };

using BufRsrc = __amdgpu_buffer_rsrc_t;
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t kOOB = 0x80000000u;  // an offset past every buffer here: loads give zero, stores are dropped

__device__ __forceinline__ BufRsrc rsrc(const void* p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ void load(float& v, const BufRsrc& r, uint32_t vo, uint32_t so) {
  v = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0));
}
__device__ __forceinline__ void load(double& v, const BufRsrc& r, uint32_t vo, uint32_t so) {
  const u32x2 u = __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0);
  v = __hiloint2double((int)u.y, (int)u.x);
}
__device__ __forceinline__ void load(float2& v, const BufRsrc& r, uint32_t vo, uint32_t so) {
  const u32x2 u = __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0);
  v = float2{__uint_as_float(u.x), __uint_as_float(u.y)};
}
__device__ __forceinline__ void load(double2& v, const BufRsrc& r, uint32_t vo, uint32_t so) {
  const u32x4 u = __builtin_amdgcn_raw_buffer_load_b128(r, vo, so, 0);
  v = double2{__hiloint2double((int)u.y, (int)u.x), __hiloint2double((int)u.w, (int)u.z)};
}
__device__ __forceinline__ void store(const BufRsrc& r, uint32_t vo, uint32_t so, const float2& x) {
  const u32x2 v = {__float_as_uint(x.x), __float_as_uint(x.y)};
  __builtin_amdgcn_raw_buffer_store_b64(v, r, vo, so, 0);
}
// The 16-byte store takes its whole offset from the lane's register: with a scalar offset the
// compiler lets the next instruction overwrite the data registers (it inserts the wait state
// that stores of more than 8 bytes need for the form without one only), and then, rarely, four
// lanes' values of a store were those of the next row.
__device__ __forceinline__ void store(const BufRsrc& r, uint32_t vo, uint32_t so, const double2& x) {
  const unsigned long long a = (unsigned long long)__double_as_longlong(x.x);
  const unsigned long long b = (unsigned long long)__double_as_longlong(x.y);
  const u32x4 v = {(unsigned)a, (unsigned)(a >> 32), (unsigned)b, (unsigned)(b >> 32)};
  __builtin_amdgcn_raw_buffer_store_b128(v, r, vo + so, 0, 0);
}

// the value of lane l - 1 (zero in lane 0), of lane l + 1 (zero in lane 63)
constexpr int kWaveShr1 = 0x138, kWaveShl1 = 0x130;
template <int CTRL>
__device__ __forceinline__ int shift32(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ float shift(float v) {
  return __int_as_float(shift32<CTRL>(__float_as_int(v)));
}
template <int CTRL>
__device__ __forceinline__ double shift(double v) {
  return __hiloint2double(shift32<CTRL>(__double2hiint(v)), shift32<CTRL>(__double2loint(v)));
}

__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

__device__ __forceinline__ int layer_depth(int i, int n, int L) { return max(0, L - min(i, n - 1 - i)); }

template <typename T>
__device__ __forceinline__ T uniform(T v);
template <>
__device__ __forceinline__ float uniform<float>(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
template <>
__device__ __forceinline__ double uniform<double>(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                          __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

// Bytes of LDS of a block: per buffer and level the first and last row of each wave, and a row
// of zeros that stands in for the rows beyond the block
constexpr size_t lds_bytes(int nf, int w, size_t elem) { return (size_t)2 * nf * (2 * w + 1) * 64 * elem; }

// The work of one block: tile b of system s.
template <typename T, int KIND, int NF, int R>
__device__ __forceinline__ void rows_tile(const GridDesc& g, const RowsShape& q, int s, int b,
                                          const FactorArgs<typename V2<T>::t>& a, const T* __restrict__ K, char* lds) {
  using T2 = typename V2<T>::t;
  constexpr bool RESID = (KIND & kFacResid) != 0, ADD = (KIND & kFacAdd) != 0, DUAL = (KIND & kFacDual) != 0,
                 INF = (KIND & kFacInF) != 0;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int W = blockDim.x >> 6, RB = W * R;
  const int bx = b % q.gx, by = (b / q.gx) % q.gy, zc = b / (q.gx * q.gy);
  const int xs = min(bx * q.sx, max(g.nx - 64, 0)), ys = min(by * q.sy, max(g.ny - RB, 0));
  const int ox0 = bx == 0 ? 0 : bx * q.sx + NF, ox1 = bx == q.gx - 1 ? g.nx : (bx + 1) * q.sx + NF;
  const int oy0 = by == 0 ? 0 : by * q.sy + NF, oy1 = by == q.gy - 1 ? g.ny : (by + 1) * q.sy + NF;
  const int zb = zc * q.czlen, ze = min(g.nz, zb + q.czlen);
  const size_t n = (size_t)g.nx * g.ny * g.nz, plane = (size_t)g.nx * g.ny;
  const int gsys = a.sys0 + s, pole = gsys / a.nrhs, rhs = gsys % a.nrhs;

  // constants of the pass, in FP64 (uniform)
  T cr[NF], ci[NF];
  const PoleDev pd = a.poles[pole];
  const FactorCoef* __restrict__ cf = a.coef + pole * a.cstride + a.k;
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    cr[f] = uniform<T>((T)cf[f].c_re);
    ci[f] = uniform<T>((T)cf[f].c_im);
  }
  const double alr = sizeof(T) == 4 ? cf[0].al32_re : cf[0].al64_re;
  const double ali = sizeof(T) == 4 ? cf[0].al32_im : cf[0].al64_im;
  const T al_r = uniform<T>((T)alr), al_i = uniform<T>((T)ali);
  // what the last pass of a step in complex64 adds for the rounding of its scalar
  const T lo_r = uniform<T>((T)(alr - (double)al_r)), lo_i = uniform<T>((T)(ali - (double)al_i));
  const T kinv = (T)-q.inv_sh2, dsc = (T)q.damp_sh2;
  // the residual's diagonal 6 - z0 / sh2, and what the first factor adds to it
  const double zcr = __builtin_fma(-pd.z0_re, q.inv_sh2, 6.0), zci = -pd.z0_im * q.inv_sh2;
  const T zr = uniform<T>((T)zcr), zi = uniform<T>((T)zci);
  const T br = uniform<T>((T)(cf[0].c_re - zcr)), bi = uniform<T>((T)(cf[0].c_im - zci));

  // buffers from the chunk's first plane on: offsets stay small whatever the grid
  const int kb = max(zb - NF, 0), kend = min(ze + NF, g.nz);
  const size_t base = plane * (size_t)kb, span = plane * (size_t)(kend - kb);
  const T2* X = INF ? a.f + (size_t)rhs * n : a.win + (size_t)s * n;
  const BufRsrc rX = rsrc(X + base, span * sizeof(T2));
  const BufRsrc rK = rsrc(K + base, span * sizeof(T));
  const BufRsrc rE = rsrc((RESID ? a.f + (size_t)rhs * n : ADD ? a.y1 + (size_t)s * n : X) + base, span * sizeof(T2));
  const BufRsrc rO = rsrc(a.wout + (size_t)s * n + base, span * sizeof(T2));
  const BufRsrc rO2 = rsrc((DUAL ? a.wout2 : a.wout) + (size_t)s * n + base, span * sizeof(T2));
  const uint32_t pb = (uint32_t)(plane * sizeof(T2)), pbk = (uint32_t)(plane * sizeof(T));
  auto zoff = [&](int k) { return __builtin_amdgcn_readfirstlane((uint32_t)(min(max(k, kb), kend - 1) - kb)); };

  const int x = xs + lane;
  // a lane's offset in its row, the rows' offsets in the plane (uniform)
  const uint32_t vx = (uint32_t)(x * sizeof(T2)), vk = (uint32_t)(x * sizeof(T));
  const uint32_t rb = (uint32_t)(g.nx * sizeof(T2)), rbk = (uint32_t)(g.nx * sizeof(T));
  const uint32_t row0 = (uint32_t)(ys + wave * R);
  bool in[R], core[R];
  T dxy[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int y = ys + wave * R + r;
    in[r] = x < g.nx && y < g.ny;
    core[r] = in[r] && x >= ox0 && x < ox1 && y >= oy0 && y < oy1;
    const int d = max(layer_depth(x, g.nx, g.damp_cells), layer_depth(y, g.ny, g.damp_cells));
    dxy[r] = in[r] ? (T)(d * d) * dsc : (T)0;
  }
  const bool ragged = g.nx < 64 || g.ny < RB;  // uniform: some lanes or rows lie outside the grid

  // LDS rows: buffer p, level f, row 2 w (first) and 2 w + 1 (last) of wave w, row 2 W zeros
  T2* const eb = reinterpret_cast<T2*>(lds);
  const int lrow = (2 * W + 1) * 64;
  const int eu = (wave > 0 ? 2 * wave - 1 : 2 * W) * 64 + lane, ed = (wave < W - 1 ? 2 * wave + 2 : 2 * W) * 64 + lane;
  const int ew = 2 * wave * 64 + lane;
  auto edge = [&](int p, int f) { return eb + (p * NF + f) * lrow; };
  if (wave == 0)
#pragma unroll
    for (int i = 0; i < 2 * NF; ++i) eb[i * lrow + 2 * W * 64 + lane] = T2{(T)0, (T)0};

  auto load_x = [&](T2 (&v)[R], int k) {
    const uint32_t so = pb * zoff(k) + rb * row0;
    const bool ok = k >= 0 && k < g.nz && k <= ze + NF - 1;
#pragma unroll
    for (int r = 0; r < R; ++r) load(v[r], rX, (ok && in[r]) ? vx : kOOB, so + r * rb);
  };
  auto load_k = [&](T (&v)[R], int k) {
    const uint32_t so = pbk * zoff(k) + rbk * row0;
#pragma unroll
    for (int r = 0; r < R; ++r) load(v[r], rK, in[r] ? vk : kOOB, so + r * rbk);
  };
  auto load_e = [&](T2 (&v)[R], int k) {
    const uint32_t so = pb * zoff(k) + rb * row0;
    const bool ok = k >= zb && k < ze;
#pragma unroll
    for (int r = 0; r < R; ++r) load(v[r], rE, (ok && core[r]) ? vx : kOOB, so + r * rb);
  };

  // level f + 1 at plane p: out = m cen - nb, zero outside the grid, m from the diagonal
  // (dr, di).  The plane above (the level below's newest) enters last: everything else is
  // ready before the barrier's other levels, so a plane's chain through the levels is one
  // instruction each.
  auto level = [&](T dr, T di, int p, const T2* E, const T2 (&cen)[R], const T2 (&zm)[R], const T2 (&zp)[R],
                   const T (&kap)[R], T2 (&out)[R]) {
    const int dz = layer_depth(p, g.nz, g.damp_cells);
    const T dpz = (T)(dz * dz) * dsc;
    const T2 eup = E[eu], edn = E[ed];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const T2 up = r > 0 ? cen[r > 0 ? r - 1 : 0] : eup, dn = r < R - 1 ? cen[r < R - 1 ? r + 1 : 0] : edn;
      T2 nb = zm[r];
      nb.x += shift<kWaveShr1>(cen[r].x);
      nb.y += shift<kWaveShr1>(cen[r].y);
      nb.x += shift<kWaveShl1>(cen[r].x);
      nb.y += shift<kWaveShl1>(cen[r].y);
      nb.x += up.x + dn.x;
      nb.y += up.y + dn.y;
      const T mr = fma_(kap[r], kinv, dr), mi = di - max(dxy[r], dpz);
      out[r].x = fma_(mr, cen[r].x, fma_(-mi, cen[r].y, -nb.x)) - zp[r].x;
      out[r].y = fma_(mr, cen[r].y, fma_(mi, cen[r].x, -nb.y)) - zp[r].y;
    }
  };
  // the Dirichlet zeros of a level's values outside the grid
  auto ghosts = [&](int p, T2 (&v)[R]) {
    const bool pin = p >= 0 && p < g.nz;
    if (ragged || !pin) {  // uniform
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (!(pin && in[r])) v[r] = T2{(T)0, (T)0};
    }
  };

  double acc = 0.0;
  if (zb < ze) {
    // registers: input planes k - 1, k, k + 1 (and k + 2 in flight); per level its planes
    // p - 1, p; kappa of planes k + 1 (in flight), k, ..., k - NF + 1
    T2 x0[R], x1[R], xn[R], xf[R], ex[R], exf[R];
    T2 tm[NF][R], tc[NF][R];
    T kq[NF][R], kf[R];
    const int k0 = zb - (NF - 1), klast = ze + NF - 2;
    load_x(x0, k0 - 1);
    load_x(x1, k0);
    load_x(xn, k0 + 1);
    load_k(kf, k0);
    if constexpr (RESID) load_e(exf, k0);
    if constexpr (ADD) load_e(exf, k0 - (NF - 1));
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        tm[f][r] = tc[f][r] = T2{(T)0, (T)0};
        kq[f][r] = (T)0;
      }
#pragma unroll
    for (int f = 0; f < NF; ++f) {  // edges for the first plane: the input's, zeros above
      edge(0, f)[ew] = f == 0 ? x1[0] : T2{(T)0, (T)0};
      edge(0, f)[ew + 64] = f == 0 ? x1[R - 1] : T2{(T)0, (T)0};
    }
    // all of the prologue's loads have landed: the loop head's waits then count the loop's own
    // memory instructions alone
    __builtin_amdgcn_s_waitcnt(0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    // four planes per trip (register queues rotate by renaming); planes past klast load
    // nothing from memory that is used and store nothing
    for (int kk = k0; kk <= klast; kk += 4) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = kk + u;
        const int par = u & 1;
        // kappa and the extra stream of this plane (loaded one plane ago), then the next loads
#pragma unroll
        for (int f = NF - 1; f > 0; --f)
#pragma unroll
          for (int r = 0; r < R; ++r) kq[f][r] = kq[f - 1][r];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          kq[0][r] = kf[r];
          if constexpr (RESID || ADD) ex[r] = exf[r];
        }
        load_x(xf, k + 2);
        load_k(kf, k + 1);
        if constexpr (RESID) load_e(exf, k + 1);
        if constexpr (ADD) load_e(exf, k + 1 - (NF - 1));
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's edge rows are written
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_barrier();
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        T2 t[R];
        level(RESID ? zr : cr[0], RESID ? zi : ci[0], k, edge(par, 0), x1, x0, xn, kq[0], t);
        edge(par ^ 1, 0)[ew] = xn[0];
        edge(par ^ 1, 0)[ew + 64] = xn[R - 1];
        if constexpr (RESID) {
          // t = (A - z0) y / sh2: |f - (A - z) y|^2 = |f - sh2 t + (z - z0) y|^2 at plane k,
          // then the first factor's own diagonal
          const bool zok = k >= zb && k < ze;
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const double rr = (double)ex[r].x - g.s_h2 * (double)t[r].x + pd.zz_re * (double)x1[r].x - pd.zz_im * (double)x1[r].y;
            const double ri = (double)ex[r].y - g.s_h2 * (double)t[r].y + pd.zz_re * (double)x1[r].y + pd.zz_im * (double)x1[r].x;
            acc += (zok && core[r]) ? rr * rr + ri * ri : 0.0;
            t[r].x = fma_(br, x1[r].x, fma_(-bi, x1[r].y, t[r].x));
            t[r].y = fma_(br, x1[r].y, fma_(bi, x1[r].x, t[r].y));
          }
        }
        ghosts(k, t);
#pragma unroll
        for (int f = 1; f < NF; ++f) {
          edge(par ^ 1, f)[ew] = t[0];
          edge(par ^ 1, f)[ew + 64] = t[R - 1];
          T2 o[R];
          level(cr[f], ci[f], k - f, edge(par, f), tc[f], tm[f], t, kq[f], o);
          if (f < NF - 1) ghosts(k - f, o);  // (the last level's values are stored where inside only)
#pragma unroll
          for (int r = 0; r < R; ++r) {
            tm[f][r] = tc[f][r];
            tc[f][r] = t[r];
            t[r] = o[r];
          }
        }
        const int km = k - (NF - 1);
        const bool zok = km >= zb && km < ze;
        const uint32_t so = pb * zoff(km) + rb * row0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          T2 o{al_r * t[r].x - al_i * t[r].y, al_r * t[r].y + al_i * t[r].x};
          if constexpr (ADD && sizeof(T) == 4) {
            o.x += fma_(lo_r, t[r].x, -lo_i * t[r].y);
            o.y += fma_(lo_r, t[r].y, lo_i * t[r].x);
          }
          if constexpr (ADD) {
            o.x += ex[r].x;
            o.y += ex[r].y;
          }
          const uint32_t v = (zok && core[r]) ? vx : kOOB;
          store(rO, v, so + r * rb, o);
          if constexpr (DUAL) store(rO2, v, so + r * rb, o);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          x0[r] = x1[r];
          x1[r] = xn[r];
          xn[r] = xf[r];
        }
      }
    }
  }
  if constexpr (RESID) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    double* sh = reinterpret_cast<double*>(lds);
    __syncthreads();
    if (lane == 0) sh[wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      double v = 0.0;
      for (int w = 0; w < W; ++w) v += sh[w];
      a.partial[(size_t)s * (q.gx * q.gy * q.nzc) + b] = v;
    }
  }
}

}  // namespace zrows
}  // namespace hfci
