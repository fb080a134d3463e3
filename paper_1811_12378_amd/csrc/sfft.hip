// S x = F^H Lambda F x of the Fourier-spectral operator in three passes over memory, for grids
// whose sides have no prime factor above 7 and whose planes (and z-columns, 64 at a time) fit in
// LDS: the transforms over y and x of a plane; forward over z, Lambda, inverse over z; the
// inverse over x and y, whose last stage goes on to the factor of the fixed-point step (w_out =
// a (A - z0) w + b w with its options) instead of storing S w.
// What bounds it: memory traffic.  The library's transforms run an axis or two per pass with
// transposes between (8 passes), Lambda and the factor read and write the vectors once more
// each, and the vectors of systems still iterating were gathered first.  Shifted solves of 16
// complex64 systems on 128^3 points 10.4 -> 5.1 ms (32 systems 18.8 -> 8.7).  A plane fills most
// of a CU's LDS there, so one block of 16 waves runs per CU and its loads, stages and stores do
// not overlap: 45 us per plane pass (mean over the shrinking batch) for 35 us of the z pass.
//
// In-place decimation-in-frequency stages forward leave the frequencies in digit-reversed
// places, decimation-in-time stages backward take them from there, so nothing is reordered;
// Lambda is looked up by place (params: SpecFft::lam).  The lanes of a wave are 64 lines of the
// other axis, so a stage's indices and twiddles are the wave's (scalar), the loads of the first
// stage and the stores of the last are coalesced, and with an odd row pitch no LDS access
// meets a bank twice (planes with a short side: see thin).  Twiddles are rounded from double.
#include <algorithm>
#include <type_traits>

#include "kernels.h"

namespace hfci {
namespace {

template <typename T> struct V2;
template <> struct V2<float> { using t = float2; };
template <> struct V2<double> { using t = double2; };

template <typename T>
struct Cp {
  T x, y;
};
template <typename T>
__device__ __forceinline__ Cp<T> operator+(Cp<T> a, Cp<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T>
__device__ __forceinline__ Cp<T> operator-(Cp<T> a, Cp<T> b) { return {a.x - b.x, a.y - b.y}; }
template <bool CONJ, typename T>
__device__ __forceinline__ Cp<T> mul(Cp<T> a, Cp<T> w) {
  if (CONJ) return {a.x * w.x + a.y * w.y, a.y * w.x - a.x * w.y};
  return {a.x * w.x - a.y * w.y, a.x * w.y + a.y * w.x};
}
// times -i (forward) or i (inverse)
template <bool INV, typename T>
__device__ __forceinline__ Cp<T> rot(Cp<T> a) {
  if (INV) return {-a.y, a.x};
  return {a.y, -a.x};
}

// cosines and sines of 2 pi k / R
template <int R> struct Unit;
template <> struct Unit<3> {
  static constexpr double c[3] = {1.0, -0.5, -0.5};
  static constexpr double s[3] = {0.0, 0.86602540378443864676, -0.86602540378443864676};
};
template <> struct Unit<5> {
  static constexpr double c[5] = {1.0, 0.30901699437494742410, -0.80901699437494742410, -0.80901699437494742410,
                                  0.30901699437494742410};
  static constexpr double s[5] = {0.0, 0.95105651629515357212, 0.58778525229247312917, -0.58778525229247312917,
                                  -0.95105651629515357212};
};
template <> struct Unit<7> {
  static constexpr double c[7] = {1.0, 0.62348980185873353053, -0.22252093395631440429, -0.90096886790241912624,
                                  -0.90096886790241912624, -0.22252093395631440429, 0.62348980185873353053};
  static constexpr double s[7] = {0.0, 0.78183148246802980871, 0.97492791218182360702, 0.43388373911755812048,
                                  -0.43388373911755812048, -0.97492791218182360702, -0.78183148246802980871};
};

// y_p = sum_k x_k exp(-+ 2 pi i p k / R), in place
template <int R, bool INV, typename T>
__device__ __forceinline__ void dft(Cp<T> (&v)[R]) {
  if constexpr (R == 2) {
    const Cp<T> a = v[0];
    v[0] = a + v[1];
    v[1] = a - v[1];
  } else if constexpr (R == 4) {
    const Cp<T> a = v[0] + v[2], b = v[0] - v[2], c = v[1] + v[3], d = rot<INV>(v[1] - v[3]);
    v[0] = a + c;
    v[1] = b + d;
    v[2] = a - c;
    v[3] = b - d;
  } else if constexpr (R == 8) {
    Cp<T> e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft<4, INV>(e);
    dft<4, INV>(o);
    const T h = (T)0.70710678118654752440;
    const Cp<T> r1 = rot<INV>(o[1]), r3 = rot<INV>(o[3]);
    o[1] = {h * (o[1].x + r1.x), h * (o[1].y + r1.y)};
    o[2] = rot<INV>(o[2]);
    o[3] = {h * (r3.x - o[3].x), h * (r3.y - o[3].y)};
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      v[p] = e[p] + o[p];
      v[p + 4] = e[p] - o[p];
    }
  } else {
    constexpr int H = (R - 1) / 2;
    Cp<T> t[H], u[H];
    Cp<T> s0 = v[0];
#pragma unroll
    for (int k = 0; k < H; ++k) {
      t[k] = v[k + 1] + v[R - 1 - k];
      u[k] = rot<INV>(v[k + 1] - v[R - 1 - k]);
      s0 = s0 + t[k];
    }
    const Cp<T> x0 = v[0];
    v[0] = s0;
#pragma unroll
    for (int p = 1; p <= H; ++p) {
      Cp<T> a = x0, b{(T)0, (T)0};
#pragma unroll
      for (int k = 0; k < H; ++k) {
        const T c = (T)Unit<R>::c[p * (k + 1) % R], s = (T)Unit<R>::s[p * (k + 1) % R];
        a.x += c * t[k].x;
        a.y += c * t[k].y;
        b.x += s * u[k].x;
        b.y += s * u[k].y;
      }
      v[p] = a + b;
      v[R - p] = a - b;
    }
  }
}

// a sink that takes the R values of a butterfly together
template <class S, class = void>
struct AllAtOnce : std::false_type {};
template <class S>
struct AllAtOnce<S, std::void_t<typename S::AllTag>> : std::true_type {};

// One stage over `lines` lines of n values split into blocks of L: forward the DFT of R values
// m = L / R apart, then the twiddles exp(-2 pi i j p / L); inverse the reverse.  MID: the last
// forward stage (L = R), a factor per place, the first inverse stage.
// PACK: up to 32 lines, and a wave takes 64 / lines butterflies of every line at once (indices and
// twiddles are then the lane's).
enum StageKind { FWD, INV, MID };
template <int R, StageKind KIND, typename T, bool PACK, class Ld, class St>
__device__ __forceinline__ void stage_r(int n, int L, int lines, int wave, int nw, int lane,
                                        const typename V2<T>::t* __restrict__ tw, const double* __restrict__ lam,
                                        Ld ld, St st) {
  const int m = L / R, nb = n / R, step = n / L;
  const int per = PACK ? 64 / lines : 1, g = PACK ? lane / lines : 0, l0 = PACK ? lane - g * lines : lane;
  for (int j0 = wave * per; j0 < nb; j0 += nw * per) {  // uniform over the wave
    const int jj = j0 + g;
    if (PACK && (g >= per || jj >= nb)) continue;
    const int q = jj / m, j = jj - q * m, base = q * L + j;
    Cp<T> w[R];
    double f[R];
#pragma unroll
    for (int p = 0; p < R; ++p) {
      if (KIND == MID) {
        f[p] = lam[base + p];
      } else if (p > 0) {
        const auto x = tw[step * j * p];
        w[p] = {x.x, x.y};
      }
    }
    for (int l = l0; l < lines; l += 64) {
      Cp<T> v[R];
#pragma unroll
      for (int k = 0; k < R; ++k) v[k] = ld(l, base + k * m);
      if constexpr (KIND == INV) {
#pragma unroll
        for (int p = 1; p < R; ++p) v[p] = mul<true>(v[p], w[p]);
        dft<R, true>(v);
      } else {
        dft<R, false>(v);
        if constexpr (KIND == MID) {
          st.scale(v, f);
          dft<R, true>(v);
        } else {
#pragma unroll
          for (int p = 1; p < R; ++p) v[p] = mul<false>(v[p], w[p]);
        }
      }
      if constexpr (AllAtOnce<St>::value) {
        st.all(l, base, m, v);
      } else {
#pragma unroll
        for (int k = 0; k < R; ++k) st(l, base + k * m, v[k]);
      }
    }
  }
}
template <StageKind KIND, typename T, bool PACK, class Ld, class St>
__device__ __forceinline__ void stage_p(int r, int n, int L, int lines, int wave, int nw, int lane,
                                        const typename V2<T>::t* __restrict__ tw, const double* __restrict__ lam, Ld ld,
                                        St st) {
  switch (r) {
    case 2: return stage_r<2, KIND, T, PACK>(n, L, lines, wave, nw, lane, tw, lam, ld, st);
    case 3: return stage_r<3, KIND, T, PACK>(n, L, lines, wave, nw, lane, tw, lam, ld, st);
    case 4: return stage_r<4, KIND, T, PACK>(n, L, lines, wave, nw, lane, tw, lam, ld, st);
    case 5: return stage_r<5, KIND, T, PACK>(n, L, lines, wave, nw, lane, tw, lam, ld, st);
    case 7: return stage_r<7, KIND, T, PACK>(n, L, lines, wave, nw, lane, tw, lam, ld, st);
    default: return stage_r<8, KIND, T, PACK>(n, L, lines, wave, nw, lane, tw, lam, ld, st);
  }
}
// THIN: kernels for planes with a side of few points (thin), which share a wave's lanes
constexpr int kThin = 32;
template <StageKind KIND, typename T, bool THIN, class Ld, class St>
__device__ __forceinline__ void stage(int r, int n, int L, int lines, int wave, int nw, int lane,
                                      const typename V2<T>::t* __restrict__ tw, const double* __restrict__ lam, Ld ld,
                                      St st) {
  if (THIN && lines <= kThin) return stage_p<KIND, T, true>(r, n, L, lines, wave, nw, lane, tw, lam, ld, st);
  stage_p<KIND, T, false>(r, n, L, lines, wave, nw, lane, tw, lam, ld, st);
}

template <typename T>
struct LdsAt {  // value idx of line l at l * ls + idx * is
  typename V2<T>::t* s;
  int ls, is;
  __device__ Cp<T> operator()(int l, int idx) const {
    const auto v = s[l * ls + idx * is];
    return {v.x, v.y};
  }
  __device__ void operator()(int l, int idx, Cp<T> v) const {
    auto& o = s[l * ls + idx * is];
    o.x = v.x;
    o.y = v.y;
  }
};

extern __shared__ double2 sfft_lds[];

// a thin plane from one place to another, point by point and four values per thread at a time
template <class Ld, class St>
__device__ __forceinline__ void copy_thin(int nx, int points, int tid, int nt, Ld ld, St st) {
  for (int p = tid; p < points; p += 4 * nt) {
    decltype(ld(0, 0)) t[4];
    auto at = [&](int i) { return min(p + i * nt, points - 1); };
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = ld(at(i) % nx, at(i) / nx);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (p + i * nt < points) st(at(i) % nx, at(i) / nx, t[i]);
  }
}

// y then x of plane blockIdx.x of vector v = blockIdx.y: from in (of system sys[v], if sys) to out
template <typename T, bool THIN>
__global__ __launch_bounds__(THIN ? 512 : 1024) void sfft_plane_fwd_kernel(GridDesc g, SpecFft sf, const typename V2<T>::t* in,
                                                              typename V2<T>::t* out, const int* __restrict__ sys) {
  using T2 = typename V2<T>::t;
  const int nx = g.nx, ny = g.ny, pitch = nx | 1;
  const size_t plane = (size_t)nx * ny, n = plane * g.nz;
  const int v = blockIdx.y;
  const T2* I = in + (size_t)(sys != nullptr ? sys[v] : v) * n + (size_t)blockIdx.x * plane;
  T2* O = out + (size_t)v * n + (size_t)blockIdx.x * plane;
  T2* s = (T2*)sfft_lds;
  const T2* tw = (const T2*)(sizeof(T) == 4 ? (const void*)sf.tw32 : (const void*)sf.tw64);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x / 64;
  const LdsAt<T> byx{s, 1, pitch}, byy{s, pitch, 1};  // lines along y (one per x); lines along x
  int L = ny;
  for (int i = 0; i < sf.y.ns; ++i) {
    if (i == 0)
      stage<FWD, T, THIN>(sf.y.r[0], ny, L, nx, wave, nw, lane, tw + nx, nullptr,
                    [&](int x, int y) {
                      const T2 u = I[(size_t)y * nx + x];
                      return Cp<T>{u.x, u.y};
                    },
                    byx);
    else
      stage<FWD, T, THIN>(sf.y.r[i], ny, L, nx, wave, nw, lane, tw + nx, nullptr, byx, byx);
    L /= sf.y.r[i];
    __syncthreads();
  }
  L = nx;
  for (int i = 0; i < sf.x.ns; ++i) {
    stage<FWD, T, THIN>(sf.x.r[i], nx, L, ny, wave, nw, lane, tw, nullptr, byy, byy);
    L /= sf.x.r[i];
    __syncthreads();
  }
  if constexpr (THIN) {
    copy_thin(nx, nx * ny, threadIdx.x, blockDim.x, [&](int x, int y) { return s[y * pitch + x]; },
              [&](int x, int y, const T2& v) { O[(size_t)y * nx + x] = v; });
    return;
  }
  for (int y = wave; y < ny; y += 4 * nw)
    for (int x = lane; x < nx; x += 64) {
      T2 t[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) t[i] = s[min(y + i * nw, ny - 1) * pitch + x];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (y + i * nw < ny) O[(size_t)(y + i * nw) * nx + x] = t[i];
    }
}

// the sink of the stage with Lambda: mine = s (k_x^2 + k_y^2) of the lane's column, f the places' s k_z^2
template <typename T, class To>
struct Scaled {
  To to;
  double inv_n, mine;
  __device__ void operator()(int l, int idx, Cp<T> v) const { to(l, idx, v); }
  template <int R>
  __device__ void scale(Cp<T> (&v)[R], const double (&f)[R]) const {
#pragma unroll
    for (int p = 0; p < R; ++p) {
      const double w = (mine + f[p]) * inv_n;
      v[p].x = (T)((double)v[p].x * w);
      v[p].y = (T)((double)v[p].y * w);
    }
  }
};

// z forward, Lambda / N, z inverse of COLS columns (places) of a vector, in place: 64, or 32 where
// 64 leave room for one block per CU only (solves of 30 systems: 150 x 64 x 64 complex128 6 % faster
// with 32, 300 x 64 x 64 complex64 6 %; with 64 KB for 64 columns, 128^3 complex64, 3 % slower)
template <typename T, int COLS>
__global__ __launch_bounds__(512) void sfft_z_kernel(GridDesc g, SpecFft sf, typename V2<T>::t* c) {
  using T2 = typename V2<T>::t;
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const size_t plane = (size_t)nx * ny, n = plane * nz;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x / 64;
  constexpr bool PACK = COLS <= 32;
  const int col = blockIdx.x * COLS + lane % COLS;
  const bool ok = col < (int)plane;
  T2* C = c + (size_t)blockIdx.y * n + (ok ? col : 0);
  T2* s = (T2*)sfft_lds;
  const T2* tw = (const T2*)(sizeof(T) == 4 ? (const void*)sf.tw32 : (const void*)sf.tw64) + nx + ny;
  const double* lz = sf.lam + nx + ny;
  const LdsAt<T> lds{s, 1, COLS};
  const double mine = ok ? sf.lam[col % nx] + sf.lam[nx + col / nx] : 0.0;
  const double inv_n = 1.0 / (double)n;
  auto from = [&](int, int z) {
    const T2 u = C[(size_t)z * plane];
    return Cp<T>{u.x, u.y};
  };
  auto to = [&](int, int z, Cp<T> u) {
    if (!ok) return;
    T2 o;
    o.x = u.x;
    o.y = u.y;
    C[(size_t)z * plane] = o;
  };
  const int ns = sf.z.ns;
  if (ns == 1) return stage_p<MID, T, PACK>(sf.z.r[0], nz, nz, COLS, wave, nw, lane, tw, lz, from,
                                   Scaled<T, decltype(to)>{to, inv_n, mine});
  int L = nz;
  for (int i = 0; i < ns - 1; ++i) {
    if (i == 0)
      stage_p<FWD, T, PACK>(sf.z.r[0], nz, L, COLS, wave, nw, lane, tw, lz, from, lds);
    else
      stage_p<FWD, T, PACK>(sf.z.r[i], nz, L, COLS, wave, nw, lane, tw, lz, lds, lds);
    L /= sf.z.r[i];
    __syncthreads();
  }
  stage_p<MID, T, PACK>(sf.z.r[ns - 1], nz, L, COLS, wave, nw, lane, tw, lz, lds,
                Scaled<T, LdsAt<T>>{lds, inv_n, mine});
  for (int i = ns - 2; i >= 0; --i) {
    __syncthreads();
    L *= sf.z.r[i];
    if (i == 0)
      stage_p<INV, T, PACK>(sf.z.r[0], nz, L, COLS, wave, nw, lane, tw, lz, lds, to);
    else
      stage_p<INV, T, PACK>(sf.z.r[i], nz, L, COLS, wave, nw, lane, tw, lz, lds, lds);
  }
}

__device__ __forceinline__ int layer_of(int i, int n, int L) { return max(0, L - min(i, n - 1 - i)); }

constexpr int kPlain = 16;  // S w itself to a.sw, in place

// The factor at points of a plane from S w there (the expressions of spec_factor_kernel); the
// loads of several of a butterfly's points are issued together.
template <typename T, int KIND>
struct Finish {
  using AllTag = void;
  using T2 = typename V2<T>::t;
  static constexpr bool PLAIN = KIND == kPlain;
  static constexpr bool RESID = !PLAIN && (KIND & kFacResid) != 0, ADD = !PLAIN && (KIND & kFacAdd) != 0,
                        DUAL = !PLAIN && (KIND & kFacDual) != 0;
  const T2 *W, *F, *Y1;
  const T* K;
  T2 *O, *O2;
  GridDesc g;
  int dk;
  T car, cai, cbr, cbi, z0r, z0i;
  double zzr, zzi;
  double* acc;

  template <int R>
  __device__ __forceinline__ void all(int x, int y0, int m, const Cp<T> (&sw)[R]) const {
    constexpr int G = sizeof(T) == 8 ? 2 : R > 4 ? 4 : R;  // loads in flight, by registers
    const int dx = max(layer_of(x, g.nx, g.damp_cells), dk);
#pragma unroll
    for (int i0 = 0; i0 < R; i0 += G) {
      T2 w[G], e[G], f[G];
      T kap[G];
#pragma unroll
      for (int q = 0; q < G; ++q) {
        if (i0 + q >= R) continue;
        const unsigned p = (unsigned)(y0 + (i0 + q) * m) * g.nx + x;
        if constexpr (!PLAIN) {
          w[q] = W[p];
          kap[q] = K[p];
        }
        if constexpr (ADD) e[q] = Y1[p];
        if constexpr (RESID) f[q] = F[p];
      }
#pragma unroll
      for (int q = 0; q < G; ++q) {
        const int i = i0 + q;
        if (i >= R) continue;
        const unsigned p = (unsigned)(y0 + i * m) * g.nx + x;
        T2 o;
        if constexpr (PLAIN) {
          o.x = sw[i].x;
          o.y = sw[i].y;
        } else {
          const int d = max(dx, layer_of(y0 + i * m, g.ny, g.damp_cells));
          const T dmp = (T)((double)(d * d) * g.damp_scale), dr = kap[q] + z0r;
          const T ox = sw[i].x - (dr * w[q].x - z0i * w[q].y) + dmp * w[q].y;
          const T oy = sw[i].y - (dr * w[q].y + z0i * w[q].x) - dmp * w[q].x;
          o.x = car * ox - cai * oy + cbr * w[q].x - cbi * w[q].y;
          o.y = car * oy + cai * ox + cbr * w[q].y + cbi * w[q].x;
          if constexpr (ADD) {
            o.x += e[q].x;
            o.y += e[q].y;
          }
          if constexpr (RESID) {
            const double rx = (double)f[q].x - (double)ox + zzr * (double)w[q].x - zzi * (double)w[q].y;
            const double ry = (double)f[q].y - (double)oy + zzr * (double)w[q].y + zzi * (double)w[q].x;
            *acc += rx * rx + ry * ry;
          }
        }
        O[p] = o;
        if constexpr (DUAL) O2[p] = o;
      }
    }
  }
};

// inverse over x and y of plane blockIdx.x of vector blockIdx.y at a.sw, then the factor of its
// system
template <typename T, int KIND, bool THIN>
__global__ __launch_bounds__(THIN ? 512 : 1024) void sfft_plane_inv_kernel(GridDesc g, SpecFft sf, const T* __restrict__ K,
                                                              SpecArgs<typename V2<T>::t> a,
                                                              const int* __restrict__ sys) {
  using T2 = typename V2<T>::t;
  using Fin = Finish<T, KIND>;
  __shared__ double sh[16];
  const int nx = g.nx, ny = g.ny, pitch = nx | 1, k = blockIdx.x;
  const size_t plane = (size_t)nx * ny, n = plane * g.nz;
  const int v = blockIdx.y, sid = !Fin::PLAIN && sys != nullptr ? sys[v] : v;
  T2* C = const_cast<T2*>(a.sw) + (size_t)v * n + (size_t)k * plane;
  T2* s = (T2*)sfft_lds;
  const T2* tw = (const T2*)(sizeof(T) == 4 ? (const void*)sf.tw32 : (const void*)sf.tw64);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x / 64;
  const LdsAt<T> byx{s, 1, pitch}, byy{s, pitch, 1};
  if constexpr (THIN) {
    copy_thin(nx, nx * ny, threadIdx.x, blockDim.x, [&](int x, int y) { return C[(size_t)y * nx + x]; },
              [&](int x, int y, const T2& v) { s[y * pitch + x] = v; });
  } else {
    for (int y = wave; y < ny; y += 4 * nw)
      for (int x = lane; x < nx; x += 64) {
        T2 t[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = C[(size_t)min(y + i * nw, ny - 1) * nx + x];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (y + i * nw < ny) s[(y + i * nw) * pitch + x] = t[i];
      }
  }
  int L = 1;
  for (int i = sf.x.ns - 1; i >= 0; --i) {
    __syncthreads();
    L *= sf.x.r[i];
    stage<INV, T, THIN>(sf.x.r[i], nx, L, ny, wave, nw, lane, tw, nullptr, byy, byy);
  }
  double acc = 0.0;
  Fin fin{};
  fin.g = g;
  fin.acc = &acc;
  if constexpr (Fin::PLAIN) {
    fin.O = C;
  } else {
    const int pole = sid / a.nrhs;
    const FactorCoef cf = a.coef[(size_t)pole * a.cstride + a.k];
    const PoleDev pd = a.poles[pole];
    const size_t off = (size_t)sid * n + (size_t)k * plane;
    fin.car = (T)cf.a_re, fin.cai = (T)cf.a_im, fin.cbr = (T)cf.b_re, fin.cbi = (T)cf.b_im;
    fin.z0r = (T)pd.z0_re, fin.z0i = (T)pd.z0_im;
    fin.zzr = pd.zz_re, fin.zzi = pd.zz_im;
    fin.W = a.win + off;
    fin.K = K + (size_t)k * plane;
    fin.O = a.wout + off;
    fin.dk = layer_of(k, g.nz, g.damp_cells);
    if (Fin::RESID) fin.F = a.f + (size_t)(sid % a.nrhs) * n + (size_t)k * plane;
    if (Fin::ADD) fin.Y1 = a.y1 + off;
    if (Fin::DUAL) fin.O2 = a.wout2 + off;
  }
  L = 1;
  for (int i = sf.y.ns - 1; i >= 0; --i) {
    __syncthreads();
    L *= sf.y.r[i];
    if (i == 0)
      stage<INV, T, THIN>(sf.y.r[0], ny, L, nx, wave, nw, lane, tw + nx, nullptr, byx, fin);
    else
      stage<INV, T, THIN>(sf.y.r[i], ny, L, nx, wave, nw, lane, tw + nx, nullptr, byx, byx);
  }
  if constexpr (Fin::RESID) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    if (lane == 0) sh[wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0;
      for (int w = 0; w < nw; ++w) t += sh[w];
      a.partial[(size_t)sid * gridDim.x + k] = t;
    }
  }
}

template <typename T>
size_t plane_lds(const GridDesc& g) { return (size_t)g.ny * (g.nx | 1) * 2 * sizeof(T); }
// Whether a wave's lanes are shared between butterflies.  With few lines most lanes idle otherwise: 30
// complex64 systems of 300 x 24 x 24 points (z, y, x) took 1.32 times the library's time, now 0.81 of it.
// In complex128 the lanes' own twiddles cost registers: from 9 lines on the idle lanes cost less
// (30 systems of 128 x 128 x 12: 1.15 of the library's time with, 0.9 without; 64 x 4 x 256 0.86 with,
// 1.75 without), unless there are too few blocks to fill the chip anyway (six of 36 x 128 x 16: 0.74 with,
// 0.88 without).  The results have the same bits either way.
template <typename T>
bool thin(const GridDesc& g, int nvec) {
  return std::min(g.nx, g.ny) <= (sizeof(T) == 4 || (long)g.nz * nvec <= 384 ? kThin : 8);
}
// Two blocks per CU where the planes leave room for them; in a thin plane as many waves as its
// busiest stage has work for, up to eight (idle ones would hold the registers of other blocks: 30
// complex128 systems of 64 x 4 x 256 points took 1.45 times the library's time in blocks of eight waves,
// 0.86 in blocks of four).
template <typename T>
int plane_threads(const GridDesc& g, const SpecFft& sf, int nvec) {
  if (!thin<T>(g, nvec)) return plane_lds<T>(g) > 52 * 1024 ? 1024 : 512;
  int waves = 1;
  auto axis = [&](const AxisStages& a, int n, int lines) {
    const int per = lines <= kThin ? 64 / lines : 1;
    for (int i = 0; i < a.ns; ++i) waves = std::max(waves, (n / a.r[i] + per - 1) / per);
  };
  axis(sf.x, g.nx, g.ny);
  axis(sf.y, g.ny, g.nx);
  return 64 * std::min(waves, 8);
}

template <typename T, int KIND>
void launch_inv(hipStream_t st, const GridDesc& g, const SpecFft& sf, const T* K,
                const SpecArgs<typename V2<T>::t>& a, const int* sys, int nvec) {
  const dim3 grid(g.nz, nvec), block(plane_threads<T>(g, sf, nvec));
  if (thin<T>(g, nvec))
    hipLaunchKernelGGL((sfft_plane_inv_kernel<T, KIND, true>), grid, block, plane_lds<T>(g), st, g, sf, K, a, sys);
  else
    hipLaunchKernelGGL((sfft_plane_inv_kernel<T, KIND, false>), grid, block, plane_lds<T>(g), st, g, sf, K, a, sys);
}

}  // namespace

bool sfft_stages(int n, AxisStages& a) {
  a.ns = 0;
  while (n > 1) {
    int r = 0;
    // 8s first; a remaining 2 * 8 as 4 * 4
    for (int c : {8, 7, 5, 4, 3, 2})
      if (n % c == 0 && !(c == 8 && n % 16 == 0 && n % 64 != 0 && n % 32 != 0)) {
        r = c;
        break;
      }
    if (r == 0 || a.ns == kAxisStages) return false;
    a.r[a.ns++] = r;
    n /= r;
  }
  return a.ns > 0;
}

// the plane beside the 128 bytes of the residual's sums; 64 columns
bool sfft_fits(const GridDesc& g, bool f64) {
  const size_t lim = 156 * 1024, e = f64 ? 16 : 8;
  return (size_t)g.ny * (g.nx | 1) * e <= lim && (size_t)g.nz * 64 * e <= lim;
}

template <typename T2>
void launch_sfft_fwd(hipStream_t st, const GridDesc& g, const SpecFft& sf, const T2* in, T2* out, const int* sys,
                     int nvec) {
  using T = decltype(T2::x);
  const dim3 grid(g.nz, nvec), block(plane_threads<T>(g, sf, nvec));
  if (thin<T>(g, nvec))
    hipLaunchKernelGGL((sfft_plane_fwd_kernel<T, true>), grid, block, plane_lds<T>(g), st, g, sf, in, out, sys);
  else
    hipLaunchKernelGGL((sfft_plane_fwd_kernel<T, false>), grid, block, plane_lds<T>(g), st, g, sf, in, out, sys);
  const size_t plane = (size_t)g.nx * g.ny, column = g.nz * sizeof(T2);
  if (64 * column > 72 * 1024)
    hipLaunchKernelGGL((sfft_z_kernel<T, 32>), dim3((unsigned)((plane + 31) / 32), nvec), dim3(512), 32 * column, st, g, sf,
                       out);
  else
    hipLaunchKernelGGL((sfft_z_kernel<T, 64>), dim3((unsigned)((plane + 63) / 64), nvec), dim3(512), 64 * column, st, g, sf,
                       out);
}
template void launch_sfft_fwd<float2>(hipStream_t, const GridDesc&, const SpecFft&, const float2*, float2*, const int*,
                                      int);
template void launch_sfft_fwd<double2>(hipStream_t, const GridDesc&, const SpecFft&, const double2*, double2*,
                                       const int*, int);

template <typename T2>
void launch_sfft_inv(hipStream_t st, const GridDesc& g, const SpecFft& sf, T2* c, int nvec) {
  using T = decltype(T2::x);
  SpecArgs<T2> a{};
  a.sw = c;
  launch_inv<T, kPlain>(st, g, sf, nullptr, a, nullptr, nvec);
}
template void launch_sfft_inv<float2>(hipStream_t, const GridDesc&, const SpecFft&, float2*, int);
template void launch_sfft_inv<double2>(hipStream_t, const GridDesc&, const SpecFft&, double2*, int);

template <typename T2>
bool launch_sfft_factor(hipStream_t st, const GridDesc& g, const SpecFft& sf, const void* K, int kind,
                        const SpecArgs<T2>& a, const int* sys, int nvec) {
  using T = decltype(T2::x);
  const T* kp = (const T*)K;
  switch (kind) {
    case 0: launch_inv<T, 0>(st, g, sf, kp, a, sys, nvec); return true;
    case kFacResid: launch_inv<T, kFacResid>(st, g, sf, kp, a, sys, nvec); return true;
    case kFacAdd: launch_inv<T, kFacAdd>(st, g, sf, kp, a, sys, nvec); return true;
    case kFacResid | kFacAdd: launch_inv<T, kFacResid | kFacAdd>(st, g, sf, kp, a, sys, nvec); return true;
    case kFacDual: launch_inv<T, kFacDual>(st, g, sf, kp, a, sys, nvec); return true;
    default: return false;
  }
}
template bool launch_sfft_factor<float2>(hipStream_t, const GridDesc&, const SpecFft&, const void*, int,
                                         const SpecArgs<float2>&, const int*, int);
template bool launch_sfft_factor<double2>(hipStream_t, const GridDesc&, const SpecFft&, const void*, int,
                                          const SpecArgs<double2>&, const int*, int);

}  // namespace hfci
