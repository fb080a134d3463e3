// 3x3x3 "same" convolutions and the elementwise ops of the learned preconditioner
// (a small 3D U-Net), for gfx950: BF16 activations and weights, FP32 accumulation on
// the matrix cores.
//
// Layout: activations are channels-last, element (voxel v, channel c) of a view at
// p[v * cs + off + c]; a "view" lets a convolution read or write a channel slice of a
// wider buffer, so the U-Net's skip concatenations never copy.  Weights are
// [27 taps][Cout][Cin] (tap = (dz+1)*9 + (dy+1)*3 + (dx+1)), so that the Cin values a
// lane feeds to one MFMA are contiguous.
//
// Implicit GEMM: D[co][v] += sum_{tap, ci} W[tap][co][ci] * X[v + off_tap][ci], one
// v_mfma_f32_16x16x32_bf16 (Cin % 32 == 0) or v_mfma_f32_16x16x16_bf16 per (tap, 32- or
// 16-channel chunk, 16 outputs, 16 voxels).  Lane l supplies row (column) l % 16 and the
// k-range [KB*(l/16), KB*(l/16)+KB) of A (B); the accumulator holds rows 4*(l/16)+r, column
// l%16.
//
// The backward data pass is the same kernel applied to the output gradient with the
// tap-flipped, Cin/Cout-transposed weights; the weight gradient is a GEMM over voxels
// (k = voxel) whose per-block partial sums are reduced in a fixed order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <stdexcept>
#include <type_traits>

#include "netkern.h"

namespace hfci {
namespace {

typedef __bf16 b8v __attribute__((ext_vector_type(8)));
typedef __bf16 b4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest even
  return (uint16_t)(u >> 16);
}

struct Coord {
  int z, y, x;
};
__device__ __forceinline__ Coord coord_of(long v, const Dims& d) {
  Coord c;
  c.x = (int)(v % d.x);
  const long r = v / d.x;
  c.y = (int)(r % d.y);
  c.z = (int)(r / d.y);
  return c;
}

struct Frag {  // v_mfma_f32_16x16x32_bf16: 8 bf16 per lane
  __device__ static b8v load(const uint16_t* p) { return __builtin_bit_cast(b8v, *reinterpret_cast<const uint4*>(p)); }
  __device__ static b8v zero() { return __builtin_bit_cast(b8v, make_uint4(0, 0, 0, 0)); }
  __device__ static f4v mma(b8v a, b8v b, f4v c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
};

// exchanges the odd rows (16 lanes each) of a with the even rows of b, or (32) the upper half of a
// with the lower half of b
template <int N>
__device__ __forceinline__ void swap_rows(uint32_t& a, uint32_t& b) {
  const auto r = N == 16 ? __builtin_amdgcn_permlane16_swap(a, b, false, false)
                         : __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}

// 3x3x3 "same" convolution as a z-marching implicit GEMM.  A block owns a TX x TY voxel tile of
// each plane of a z-chunk and takes its input planes in turn: the tile with its one-voxel halo
// sits in LDS, the next plane's loads are issued before a plane's products and written there
// after them.  A fragment of 16 voxels read from LDS serves the three output planes that use it
// (taps dz = -1, 0, 1 of planes p + 1, p, p - 1, one accumulator each).  A wave owns MB blocks of
// 16 voxels along x and CTW x 16 output channels; the weights are operand A (cout x cin), the
// input B (cin x voxels), so a lane of the accumulator holds four output channels of one voxel,
// stored as 8 bytes.
// 16 and 48 input channels (PAIR): one instruction takes two consecutive 16-channel steps, lanes
// 0-31 the first and 32-63 the second; the instruction sums the first half of k before the
// second, so the result has the bits of two 16x16x16 instructions (which take as long each).
// The odd step out has zeros in lanes 32-63 of both operands.
// Each output sums its products in the order (tap, channels) in one accumulator.
// Weights (three fragments per step and 16 outputs): in registers where all of a wave's fit; for
// 48 -> 16 and 32 -> 32, which leave room for them, in LDS; for 64 and 96 channels a third
// (dz = -1) in LDS and the rest through L1, from where they are the bound (96 -> 32 on 128^3
// voxels: 480 us all through L1, 387 us with the third; the products alone 150 us).
// UP > 0: the first UP input channels are the nearest-neighbour x2 up-sampling of `up` (half
// the grid), read in place; the others are `in`.
// SMALL: 16 x 4 tiles, where the large ones would leave CUs without a block.
// Measured on a 256^3 grid, a block of 64 voxels that read every tap from memory (or one
// 3-plane ring with a loop over taps, 16 and 48 channels) before, this now: 16 -> 16 988 -> 258 us
// (4.2 TB/s), 48 -> 16 2488 -> 600 us and its up-sampling pass 900 us gone (66% of the matrix
// cores' cycles), at 128^3 96 -> 32 and 32 -> 32 1122 (mean) -> 387 and 124 us, 16 -> 32 357 -> 76 us,
// at 64^3 64 -> 64 and 32 -> 64 306 (mean) -> 82 and 50 us.
template <int CIN, int COUT, bool SMALL>
struct ConvCfg {
  static constexpr bool PAIR = CIN % 32 != 0;
  static constexpr int CT = COUT / 16;
  // products of 32 per output, plane and dz; 16-channel steps are (dy, dx, channels)
  static constexpr int NC = PAIR ? CIN / 16 : CIN / 32, NJ = 9 * NC, NS = PAIR ? (NJ + 1) / 2 : NJ;
  // waves: WG groups of output channels times WV groups of voxels
  static constexpr int WG = SMALL && CT == 6 ? 2 : CT;
  static constexpr int TX = SMALL ? 16 : 32, TY = SMALL || (CIN == 32 && CT >= 4) ? 4 : 8;
  static constexpr int MB = SMALL ? (CT == 3 ? 1 : WG) : CIN == 64 && CT == 4 ? 8 : 4;
  static constexpr int WV = TX * TY / 16 / MB, NW = WG * WV, CTW = CT / WG;
  // channels per voxel in LDS: 2 (mod 4) pieces of 16 bytes apart, reads meet no bank twice
  static constexpr int CP = PAIR ? CIN : CIN + 16;
  static constexpr int LX = TX + 2, LY = TY + 2, kPlane = LX * LY * CP;
  // weights: dz < LDZ in LDS; all taps in registers (WREG: up to 108 of a lane's 256, 60 of 168)
  static constexpr int LDZ = CIN == 48 || (CIN == 32 && CT == 2 && !SMALL) ? 3 : CIN >= 64 && !SMALL ? 1 : 0;
  static constexpr bool WREG = !LDZ && 3 * NS * CTW * 4 <= (NW > 8 ? 60 : 108);
  static constexpr bool ROLL = !WREG && LDZ < 3;  // weights through L1: a loop over dy
  static constexpr int kFrags = LDZ * NS * CT;
  static constexpr int PARTS = CIN / 8, kItems = LX * LY * PARTS, NT = 64 * NW, PER = (kItems + NT - 1) / NT;
  static constexpr int NBX = TX / 16;  // blocks per row
  static constexpr int blk(int m) { return (m / NBX * LX + m % NBX * 16) * CP; }
  static_assert(MB % NBX == 0 && WG * CTW == CT && WV * MB * 16 == TX * TY && MB >= 1, "waves cover the tile");
  static_assert(!ROLL || !PAIR, "paired steps keep their weights in registers or LDS");
  // LDS offset of 16-channel (32-channel) step j within a tile
  static constexpr int off(int j) {
    return (j / NC / 3 * LX + j / NC % 3) * CP + j % NC * (PAIR ? 16 : 32);
  }
};

// What becomes of a finished output plane: stored; stored and 2x2x2 averaged (a wave's blocks are
// two rows of two, a lane's x-neighbour is the next lane, and the z-chunks are even); or, 16
// outputs, fed to the head, whose two values replace it (the four lanes with a voxel's channels
// exchange their blocks, so that each has all channels of one voxel).  Both sum in the order of
// pool_kernel and head_fwd_kernel.  As passes of their own they read what the convolution has
// just written: on a 256^3 grid 118 us for the head and 134 us (mean) for each of the averages;
// here the convolutions take 50, 40 and 3 us longer, a forward pass 2.38 -> 2.01 ms.
enum Tail { STORE, POOL, HEAD };

template <int CIN, int COUT, int UP, bool SMALL, Tail TAIL>
__global__ __launch_bounds__((ConvCfg<CIN, COUT, SMALL>::NT), 2) void zconv_kernel(
    Dims d, View in, View up, const uint16_t* __restrict__ w, const float* __restrict__ bias, int relu, View out,
    int zlen, ConvTail tail) {
  using C = ConvCfg<CIN, COUT, SMALL>;
  using F = Frag;
  struct Acc {
    f4v v[C::MB][C::CTW];
  };
  __shared__ __align__(16) uint16_t pl[C::kPlane];
  __shared__ __align__(16) uint16_t wl[C::LDZ ? C::kFrags * 512 : 8];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int gx = (d.x + C::TX - 1) / C::TX, gy = (d.y + C::TY - 1) / C::TY;
  const int bid = blockIdx.x;
  const int x0 = bid % gx * C::TX, y0 = bid / gx % gy * C::TY;
  const int zb = bid / (gx * gy) * zlen, ze = min(d.z, zb + zlen);
  const int row = lane & 15, kq = lane >> 4;
  const int wg = wave % C::WG, wv = wave / C::WG;
  // fragment of the weights for (dz, step s, 16 outputs t): a lane's 8 channels of one output
  auto wfrag = [&](int dz, int st, int t, int l) {
    const int r = l & 15, k = l >> 4;
    int j = st, ch = k * 8;
    if (C::PAIR) {
      j = 2 * st + k / 2;
      ch = k % 2 * 8;
      if (j >= C::NJ) return F::zero();
    }
    const int tap = dz * 9 + j / C::NC;
    return F::load(w + ((size_t)tap * COUT + t * 16 + r) * CIN + j % C::NC * (C::PAIR ? 16 : 32) + ch);
  };
  if constexpr (C::LDZ > 0)
    for (int i = tid; i < C::kFrags * 64; i += C::NT)
      *reinterpret_cast<b8v*>(wl + i * 8) = wfrag(i / 64 / (C::NS * C::CT), i / 64 / C::CT % C::NS, i / 64 % C::CT, i & 63);

  // this thread's 16-byte pieces of a plane: where they come from (in pieces; -1: zeros) and go
  const Dims e{d.z / 2, d.y / 2, d.x / 2};
  int src[C::PER];
  bool coarse[C::PER];
#pragma unroll
  for (int i = 0; i < C::PER; ++i) {
    const int c = tid + i * C::NT;
    const int vox = c / C::PARTS, part = c % C::PARTS;
    const int xg = x0 - 1 + vox % C::LX, yg = y0 - 1 + vox / C::LX;
    const bool ok = c < C::kItems && xg >= 0 && xg < d.x && yg >= 0 && yg < d.y;
    coarse[i] = UP > 0 && part * 8 < UP;
    src[i] = !ok ? -1
             : coarse[i] ? ((yg / 2) * e.x + xg / 2) * (up.cs / 8) + up.off / 8 + part
                         : (yg * d.x + xg) * (in.cs / 8) + in.off / 8 + part - UP / 8;
  }
  // (loads of valid addresses only, without branches: pieces outside the grid become zeros in put)
  uint4 v[C::PER];
  bool zok = false;
  auto fetch = [&](int zp) {
    zok = zp >= 0 && zp < d.z;  // uniform
    zp = min(max(zp, 0), d.z - 1);
    const uint4* f = reinterpret_cast<const uint4*>(in.p + (long)zp * d.y * d.x * in.cs);
    const uint4* g = UP > 0 ? reinterpret_cast<const uint4*>(up.p + (long)(zp / 2) * e.y * e.x * up.cs) : f;
#pragma unroll
    for (int i = 0; i < C::PER; ++i) v[i] = (coarse[i] ? g : f)[max(src[i], 0)];
  };
  auto put = [&] {
#pragma unroll
    for (int i = 0; i < C::PER; ++i) {
      const int c = tid + i * C::NT;
      const bool ok = zok && src[i] >= 0;
      if (c < C::kItems)
        *reinterpret_cast<uint4*>(pl + c / C::PARTS * C::CP + c % C::PARTS * 8) =
            make_uint4(ok ? v[i].x : 0, ok ? v[i].y : 0, ok ? v[i].z : 0, ok ? v[i].w : 0);
    }
  };
  fetch(zb - 1);

  b8v wr[C::WREG ? 3 : 1][C::WREG ? C::NS : 1][C::CTW];
  if constexpr (C::WREG)
#pragma unroll
    for (int dz = 0; dz < 3; ++dz)
#pragma unroll
      for (int st = 0; st < C::NS; ++st)
#pragma unroll
        for (int t = 0; t < C::CTW; ++t) wr[dz][st][t] = wfrag(dz, st, wg * C::CTW + t, lane);
  f4v bv[C::CTW];
#pragma unroll
  for (int t = 0; t < C::CTW; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) bv[t][r] = bias ? bias[(wg * C::CTW + t) * 16 + 4 * kq + r] : 0.f;

  // the wave's blocks of 16 voxels: block m is NBX * 16 voxels of a row along, then rows down
  const int cx = row, cy = wv * (C::MB / C::NBX);
  const int base = (cy * C::LX + cx) * C::CP + (C::PAIR ? kq % 2 : kq) * 8;
  const int hi = C::PAIR ? kq / 2 : 0;  // lanes of a pair's second step
  const int xo = x0 + cx, yo = y0 + cy;
  const long ostep = (long)d.x * out.cs, oplane = d.y * ostep;
  uint16_t* op = out.p + zb * oplane + yo * ostep + (long)xo * out.cs + out.off + wg * C::CTW * 16 + 4 * kq;
  // output planes are finished in turn
  int zo = zb;
  float ps[TAIL == POOL ? 2 : 1][4];  // sums of an even plane
  auto store = [&](const Acc& a) {
    b4v hb[C::MB][C::CTW];
#pragma unroll
    for (int m = 0; m < C::MB; ++m) {
      uint16_t* o = op + m / C::NBX * ostep + m % C::NBX * 16 * out.cs;
#pragma unroll
      for (int t = 0; t < C::CTW; ++t) {
        f4v h = a.v[m][t] + bv[t];
        if (relu)
#pragma unroll
          for (int r = 0; r < 4; ++r) h[r] = fmaxf(h[r], 0.f);
        hb[m][t] = __builtin_convertvector(h, b4v);  // to nearest even
        if (TAIL != HEAD && xo + m % C::NBX * 16 < d.x && yo + m / C::NBX < d.y)
          *reinterpret_cast<b4v*>(o + t * 16) = hb[m][t];
      }
    }
    op += oplane;
    if constexpr (TAIL == POOL) {
      static_assert(C::NBX == 2 && C::MB == 4 && C::CTW == 1, "a wave has two rows of two blocks");
      const bool odd = zo & 1;  // uniform
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        b4v pv;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float s = odd ? ps[q][r] : 0.f;
#pragma unroll
          for (int y = 0; y < 2; ++y) {
            const float x = (float)hb[2 * y + q][0][r];
            s += x;
            s += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, true));  // lane ^ 1
          }
          ps[q][r] = s;
          pv[r] = (__bf16)(0.125f * s);
        }
        if (odd && !(row & 1) && xo + q * 16 < d.x && yo < d.y)
          *reinterpret_cast<b4v*>(tail.pool.p +
                                  (((long)(zo / 2) * e.y + yo / 2) * e.x + xo / 2 + q * 8) * tail.pool.cs +
                                  tail.pool.off + wg * 16 + 4 * kq) = pv;
      }
    }
    if constexpr (TAIL == HEAD) {
      static_assert(C::MB == 4 && COUT == 16, "four lanes exchange four blocks");
      uint32_t u[4][2];  // [block][channel pair], then [channels 4 i on][channel pair] of block kq
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const uint2 x = __builtin_bit_cast(uint2, hb[m][0]);
        u[m][0] = x.x;
        u[m][1] = x.y;
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        swap_rows<32>(u[0][i], u[2][i]);
        swap_rows<32>(u[1][i], u[3][i]);
        swap_rows<16>(u[0][i], u[1][i]);
        swap_rows<16>(u[2][i], u[3][i]);
      }
      float o0 = tail.hb[0], o1 = tail.hb[1];
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        const uint32_t p = u[c / 4][c / 2 % 2];
        const float x = __uint_as_float(c % 2 ? p & 0xffff0000u : p << 16);
        o0 += tail.hw[c] * x;
        o1 += tail.hw[16 + c] * x;
      }
      const int xv = xo + kq % C::NBX * 16, yv = yo + kq / C::NBX;
      if (xv < d.x && yv < d.y) {
        float* o = tail.o + 2 * (((long)zo * d.y + yv) * d.x + xv);
        o[0] = o0;
        o[1] = o1;
      }
    }
    ++zo;
  };

  // products of the plane in LDS for the output planes in mask (bit dz + 1), dz = -1 starts at 0
  auto products = [&](auto mask, Acc& a0, Acc& a1, Acc& a2) {
    constexpr int M = decltype(mask)::value;
    if constexpr (M & 1)
#pragma unroll
      for (int m = 0; m < C::MB; ++m)
#pragma unroll
        for (int t = 0; t < C::CTW; ++t) a0.v[m][t] = f4v{0.f, 0.f, 0.f, 0.f};
    // operands of a step are loaded one step ahead, and no further: registers
    constexpr int N = C::ROLL ? C::NS / 3 : C::NS;
    b8v xb[2][C::MB], wa[2][C::WREG ? 1 : 3][C::CTW];
#pragma unroll(C::ROLL ? 1 : 3)
    for (int dy = 0; dy < (C::ROLL ? 3 : 1); ++dy) {
      int wo = dy * 3 * COUT * CIN;
      if constexpr (C::ROLL) asm volatile("" : "+s"(wo));  // keeps the loads of weights in the loop
      auto operands = [&](int st) {
#pragma unroll
        for (int m = 0; m < C::MB; ++m) {
          b8v& x = xb[st & 1][m];
          if constexpr (C::PAIR) {
            const int j = 2 * st, step = j + 1 < C::NJ ? C::off(j + 1) - C::off(j) : 0;
            x = F::load(pl + base + hi * step + C::blk(m) + C::off(j));
            if (j + 1 == C::NJ) x = hi ? F::zero() : x;
          } else {
            x = F::load(pl + base + dy * C::LX * C::CP + C::blk(m) + C::off(st));
          }
        }
        if constexpr (!C::WREG)
#pragma unroll
          for (int dz = 0; dz < 3; ++dz)
#pragma unroll
            for (int t = 0; t < C::CTW; ++t)
              if (M >> dz & 1)
                wa[st & 1][dz][t] =
                    dz < C::LDZ ? F::load(wl + (((dz * C::NS + dy * N + st) * C::CT + wg * C::CTW + t) * 64 + lane) * 8)
                            : F::load(w + wo + (wg * C::CTW * 16 + row) * CIN + kq * 8 +
                                      ((dz * 9 + st / C::NC) * COUT + t * 16) * CIN + st % C::NC * 32);
      };
      operands(0);
#pragma unroll
      for (int st = 0; st < N; ++st) {
        if (st + 1 < N) operands(st + 1);
#pragma unroll
        for (int dz = 0; dz < 3; ++dz) {
          if (!(M >> dz & 1)) continue;
          Acc& a = dz == 0 ? a0 : dz == 1 ? a1 : a2;
#pragma unroll
          for (int t = 0; t < C::CTW; ++t)
#pragma unroll
            for (int m = 0; m < C::MB; ++m)
              a.v[m][t] = F::mma(C::WREG ? wr[C::WREG ? dz : 0][C::WREG ? st : 0][t] : wa[st & 1][C::WREG ? 0 : dz][t], xb[st & 1][m], a.v[m][t]);
        }
        // no load further ahead: registers (32 channels fit)
        if (CIN != 32) __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // plane p: its products, the output plane that is done with it, and plane p + 1 into LDS
  auto plane = [&](auto mask, int p, Acc& a0, Acc& a1, Acc& a2) {
    constexpr int M = decltype(mask)::value;
    if (M != 4) fetch(p + 1);
    products(mask, a0, a1, a2);
    if (M & 4) store(a2);
    if (M != 4) {
      __syncthreads();  // every wave is done with plane p
      put();
      __syncthreads();
    }
  };
  using std::integral_constant;
  constexpr integral_constant<int, 1> first{};
  constexpr integral_constant<int, 2> only{};
  constexpr integral_constant<int, 3> second{};
  constexpr integral_constant<int, 4> last{};
  constexpr integral_constant<int, 6> before{};
  constexpr integral_constant<int, 7> full{};
  Acc a, b, c;  // the roles of dz = -1, 0, 1 go round
  put();
  __syncthreads();
  plane(first, zb - 1, b, c, a);
  if (ze - zb == 1) {
    plane(only, zb, a, b, c);
    plane(last, ze, c, a, b);
    return;
  }
  plane(second, zb, a, b, c);
  int p = zb + 1;
  for (; p + 2 < ze - 1; p += 3) {
    plane(full, p, c, a, b);
    plane(full, p + 1, b, c, a);
    plane(full, p + 2, a, b, c);
  }
  for (; p < ze - 1; ++p) {
    plane(full, p, c, a, b);
    b = a;
    a = c;
  }
  plane(before, p, c, a, b);
  plane(last, p + 1, b, c, a);
}

// Weight and bias gradient of one layer: dw[tap][co][ci] = sum over voxels of dz[v][co] *
// x[v + off_tap][ci] and db[co] = sum of dz[v][co], as per-block partial sums.
// A GEMM whose k index runs over voxels, so both operands are needed with the voxels of a
// channel side by side while memory is channels-last.  A block stages a 32 x 4 x tz voxel
// tile of dz and the same tile of 16 input channels with its halo in LDS, transposed to
// [channel][row][x] (two x-neighbours packed per 4-byte write), and its nine waves take one
// (dz, dy) pair of taps each: per row of 32 voxels one 16x16x32 MFMA per tap and 16 output
// channels, the taps dx = -1, 0, 1 from one set of LDS reads shifted by 16 bits in registers.
// So memory is read about once per 16 input channels (the halo comes from L2), and the
// accumulators stay in registers over all tiles of a block.  Rows are 48 values (x at 8, so
// that 16-byte reads are aligned), a channel's rows are padded to an odd multiple of 64 bytes
// (the 16 channels of a read then spread over the banks).
// What it replaces (2-byte gathers per lane and tap from channels-last memory, one tap per
// block) took 994 us for a 16 -> 16 layer on 64^3 voxels and 1321 us for the 48 -> 16 one,
// plus 90 us per layer for the bias sums.
constexpr int WGX = 32, WGY = 4, WGZ = 4;            // voxel tile
constexpr int WGR = (WGY + 2) * (WGZ + 2);           // rows of the input tile with halo
constexpr int WGXP = 48, WGX0 = 8;                   // values per input row, position of x = 0
constexpr int WGXS = WGR * WGXP + 32;                // values per input channel (3520 bytes)
constexpr int WGDS = WGY * WGZ * WGX + 32;           // values per dz channel (1088 bytes)
constexpr int WGNT = 9 * 64;
static_assert((WGXS * 2 / 64) % 2 == 1 && (WGDS * 2 / 64) % 2 == 1, "channel strides spread over the banks");

template <int CT>
__global__ __launch_bounds__(WGNT) void conv_wgrad_kernel(Dims d, View x, View dz, int cin, int tz, int ntiles,
                                                          float* __restrict__ part, float* __restrict__ bpart) {
  __shared__ __align__(16) uint16_t xs[16 * WGXS];
  __shared__ __align__(16) uint16_t ds[CT * 16 * WGDS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = lane & 15, kq = lane >> 4;
  const int ci0 = blockIdx.y * 16;
  const int tx = (d.x + WGX - 1) / WGX, ty = (d.y + WGY - 1) / WGY;
  const int tdz = wave / 3, tdy = wave % 3;  // this wave's taps: offsets (tdz - 1, tdy - 1, *)
  f4v acc[3][CT], bacc[CT];
#pragma unroll
  for (int t = 0; t < CT; ++t) {
    bacc[t] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 3; ++i) acc[i][t] = f4v{0.f, 0.f, 0.f, 0.f};
  }
  // eight channels of voxels (xg, xg + 1) of a view into eight rows' 4-byte words, zeros
  // outside the grid
  auto stage = [&](const View& v, int c0, int zg, int yg, int xg, uint16_t* dst, int stride) {
    uint4 a = make_uint4(0, 0, 0, 0), b = a;
    if (zg >= 0 && zg < d.z && yg >= 0 && yg < d.y) {
      const uint16_t* p = v.p + (((long)zg * d.y + yg) * d.x + xg) * v.cs + v.off + c0;
      if (xg >= 0 && xg < d.x) a = *reinterpret_cast<const uint4*>(p);
      if (xg + 1 >= 0 && xg + 1 < d.x) b = *reinterpret_cast<const uint4*>(p + v.cs);
    }
    const uint32_t aw[4] = {a.x, a.y, a.z, a.w}, bw[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      *reinterpret_cast<uint32_t*>(dst + (2 * k) * stride) = __builtin_amdgcn_perm(bw[k], aw[k], 0x05040100u);
      *reinterpret_cast<uint32_t*>(dst + (2 * k + 1) * stride) = __builtin_amdgcn_perm(bw[k], aw[k], 0x07060302u);
    }
  };
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int x0 = (tile % tx) * WGX, y0 = (tile / tx) % ty * WGY, z0 = tile / (tx * ty) * tz;
    // input: rows (lz, ly) of the tile with halo, voxel pairs at x0 - 2 + 2 i for i < 18
    for (int i = tid; i < 2 * (tz + 2) * (WGY + 2) * 18; i += WGNT) {
      const int pr = i % 18, r = i / 18 % ((tz + 2) * (WGY + 2)), half = i / (18 * (tz + 2) * (WGY + 2));
      stage(x, ci0 + half * 8, z0 - 1 + r / (WGY + 2), y0 - 1 + r % (WGY + 2), x0 - 2 + 2 * pr,
            xs + half * 8 * WGXS + r * WGXP + WGX0 - 2 + 2 * pr, WGXS);
    }
    for (int i = tid; i < CT * 2 * tz * WGY * 16; i += WGNT) {
      const int pr = i % 16, r = i / 16 % (tz * WGY), oct = i / (16 * tz * WGY);
      const int zg = z0 + r / WGY;
      stage(dz, oct * 8, zg, y0 + r % WGY, x0 + 2 * pr, ds + oct * 8 * WGDS + r * WGX + 2 * pr, WGDS);
    }
    __syncthreads();
    for (int r = 0; r < tz * WGY; ++r) {
      const uint16_t* xp = xs + row * WGXS + ((r / WGY + tdz) * (WGY + 2) + r % WGY + tdy) * WGXP + WGX0 + 8 * kq;
      const uint4 c = *reinterpret_cast<const uint4*>(xp);
      const uint32_t lo = *reinterpret_cast<const uint32_t*>(xp - 2), hi = *reinterpret_cast<const uint32_t*>(xp + 8);
      const uint32_t s1 = __builtin_amdgcn_alignbit(c.y, c.x, 16), s2 = __builtin_amdgcn_alignbit(c.z, c.y, 16),
                     s3 = __builtin_amdgcn_alignbit(c.w, c.z, 16);
      const b8v bm = __builtin_bit_cast(b8v, make_uint4(__builtin_amdgcn_alignbit(c.x, lo, 16), s1, s2, s3));
      const b8v b0 = __builtin_bit_cast(b8v, c);
      const b8v bp = __builtin_bit_cast(b8v, make_uint4(s1, s2, s3, __builtin_amdgcn_alignbit(hi, c.w, 16)));
#pragma unroll
      for (int t = 0; t < CT; ++t) {
        const b8v a = Frag::load(ds + (t * 16 + row) * WGDS + r * WGX + 8 * kq);
        acc[0][t] = Frag::mma(a, bm, acc[0][t]);
        acc[1][t] = Frag::mma(a, b0, acc[1][t]);
        acc[2][t] = Frag::mma(a, bp, acc[2][t]);
        if (wave == 4 && ci0 == 0) {  // the centre pair's wave also sums dz (a product with ones)
          const uint32_t one = 0x3f803f80u;
          bacc[t] = Frag::mma(a, __builtin_bit_cast(b8v, make_uint4(one, one, one, one)), bacc[t]);
        }
      }
    }
    __syncthreads();
  }
  // accumulator: rows (output channels) 4 kq + r, column (input channel) row
  const int cout = CT * 16;
  float* out = part + (size_t)blockIdx.x * 27 * cout * cin;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        out[((size_t)((tdz * 3 + tdy) * 3 + i) * cout + t * 16 + 4 * kq + r) * cin + ci0 + row] = acc[i][t][r];
  if (wave == 4 && ci0 == 0 && row == 0)
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) bpart[(size_t)blockIdx.x * cout + t * 16 + 4 * kq + r] = bacc[t][r];
}

// sum over chunks, fixed order: out[i] = sum_c part[c][i].  A block
// takes 64 values of a job; 16 waves sum every 16th chunk each, then the 16 sums in order (one thread
// per value over all chunks left most of the chip idle: 22 us per layer on 64^3 voxels).
__global__ __launch_bounds__(1024) void sum_chunks_kernel(SumJobs jobs) {
  __shared__ float sh[16][64];
  int j = 0;
  while (j + 1 < jobs.n && (int)blockIdx.x >= jobs.j[j + 1].blk0) ++j;  // uniform
  const SumJob job = jobs.j[j];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = ((int)blockIdx.x - job.blk0) * 64 + lane;
  float s = 0.f;
  if (i < job.len)
    for (int c = wave; c < job.nchunk; c += 16) s += job.part[(size_t)c * job.len + i];
  sh[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && i < job.len) {
    s = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) s += sh[w][lane];
    job.out[i] = s;
  }
}

// W'[tap][ci][co] = W[26 - tap][co][ci]  (bf16), for the backward data pass
__global__ void flip_transpose_kernel(const uint16_t* __restrict__ w, int cout, int cin, uint16_t* __restrict__ wt) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long n = 27L * cout * cin;
  if (i >= n) return;
  const int tap = (int)(i / ((long)cin * cout));
  const int rem = (int)(i % ((long)cin * cout));
  const int ci = rem / cout, co = rem % cout;
  wt[i] = w[((size_t)(26 - tap) * cout + co) * cin + ci];
}

__global__ void f32_to_bf16_kernel(const float* __restrict__ a, long n, uint16_t* __restrict__ b) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = f2bf(a[i]);
}

// The elementwise passes take 8 channels (16 bytes) per thread; views are multiples of 8 wide.
struct alignas(16) Piece {
  uint16_t h[8];
};
__device__ __forceinline__ Piece piece_at(const View& v, long vox, int part) {
  return *reinterpret_cast<const Piece*>(v.p + vox * v.cs + v.off + 8 * part);
}
__device__ __forceinline__ void put_piece(const View& v, long vox, int part, const Piece& x) {
  *reinterpret_cast<Piece*>(v.p + vox * v.cs + v.off + 8 * part) = x;
}
// the coarse voxel above fine voxel v
__device__ __forceinline__ long parent_of(long v, const Dims& d) {
  const Coord f = coord_of(v, d);
  return ((long)(f.z / 2) * (d.y / 2) + f.y / 2) * (d.x / 2) + f.x / 2;
}
// sums of the 8 fine voxels below coarse voxel vc, in the order z, y, x
__device__ __forceinline__ void sum_children(const Dims& d, const View& in, long vc, int part, float (&s)[8]) {
  const Coord q = coord_of(vc, Dims{d.z / 2, d.y / 2, d.x / 2});
#pragma unroll
  for (int c = 0; c < 8; ++c) s[c] = 0.f;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const long v = ((long)(2 * q.z + (k >> 2)) * d.y + 2 * q.y + ((k >> 1) & 1)) * d.x + 2 * q.x + (k & 1);
    const Piece x = piece_at(in, v, part);
#pragma unroll
    for (int c = 0; c < 8; ++c) s[c] += bf2f(x.h[c]);
  }
}

// relu backward: dzo[v][c] = dh[v][c] if post[v][c] > 0 else 0
__global__ void relu_mask_kernel(View dh, View post, int parts, long nvox, View dzo) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nvox * parts) return;
  const long v = i / parts;
  const int part = (int)(i % parts);
  const Piece pv = piece_at(post, v, part);
  Piece x = piece_at(dh, v, part);
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const bool pos = (pv.h[c] & 0x8000u) == 0 && (pv.h[c] & 0x7fffu) != 0;
    x.h[c] = pos ? x.h[c] : (uint16_t)0;
  }
  put_piece(dzo, v, part, x);
}

// 2x2x2 average pooling (fine dims d, coarse dims d/2)
__global__ void pool_kernel(Dims d, View in, int parts, long n, View out) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float s[8];
  sum_children(d, in, i / parts, (int)(i % parts), s);
  Piece x;
#pragma unroll
  for (int c = 0; c < 8; ++c) x.h[c] = f2bf(0.125f * s[c]);
  put_piece(out, i / parts, (int)(i % parts), x);
}

// adjoint of pooling: out[v][c] = in[parent(v)][c] / 8 + addend[v][c]  (fine dims d)
__global__ void pool_back_kernel(Dims d, View in, int parts, long n, View out, View addend) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const long v = i / parts;
  const int part = (int)(i % parts);
  const Piece a = piece_at(in, parent_of(v, d), part), b = piece_at(addend, v, part);
  Piece x;
#pragma unroll
  for (int c = 0; c < 8; ++c) x.h[c] = f2bf(0.125f * bf2f(a.h[c]) + bf2f(b.h[c]));
  put_piece(out, v, part, x);
}

// nearest-neighbour x2 up-sampling (fine dims d)
__global__ void up_kernel(Dims d, View in, int parts, long n, View out) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const long v = i / parts;
  put_piece(out, v, (int)(i % parts), piece_at(in, parent_of(v, d), (int)(i % parts)));
}

// adjoint of up-sampling: out[vc][c] = sum of the 8 children (coarse dims d/2)
__global__ void up_back_kernel(Dims d, View in, int parts, long n, View out) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float s[8];
  sum_children(d, in, i / parts, (int)(i % parts), s);
  Piece x;
#pragma unroll
  for (int c = 0; c < 8; ++c) x.h[c] = f2bf(s[c]);
  put_piece(out, i / parts, (int)(i % parts), x);
}

// 1x1x1 head 16 -> 2 channels: o[v][k] = b[k] + sum_c W[k][c] h[v][c]  (FP32 out)
__global__ void head_fwd_kernel(View h, long nvox, const float* __restrict__ W, const float* __restrict__ b,
                                float* __restrict__ o) {
  const long v = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= nvox) return;
  float o0 = b[0], o1 = b[1];
  for (int c = 0; c < 16; ++c) {
    const float x = bf2f(h.p[v * h.cs + h.off + c]);
    o0 += W[c] * x;
    o1 += W[16 + c] * x;
  }
  o[2 * v] = o0;
  o[2 * v + 1] = o1;
}

// head backward: dh[v][c] = sum_k dout[v][k] W[k][c] (bf16); partial dW/db per block.  A thread
// keeps its 34 sums over the voxels it takes; one reduction per block (a tree through LDS for
// each of the 34 and every 256 voxels: 36 us on 64^3 voxels).
constexpr int kHeadBlocks = 512;
__global__ __launch_bounds__(256) void head_back_kernel(View h, long nvox, const float* __restrict__ W,
                                                        const float* __restrict__ dout, View dh,
                                                        float* __restrict__ part /* [blk][34] */) {
  __shared__ float sh[4][34];
  float s[34];
#pragma unroll
  for (int k = 0; k < 34; ++k) s[k] = 0.f;
  for (long v = (long)blockIdx.x * 256 + threadIdx.x; v < nvox; v += (long)gridDim.x * 256) {
    const float g0 = dout[2 * v], g1 = dout[2 * v + 1];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const Piece x = piece_at(h, v, p);
      Piece y;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const float f = bf2f(x.h[c]);
        s[8 * p + c] += g0 * f;
        s[16 + 8 * p + c] += g1 * f;
        y.h[c] = f2bf(g0 * W[8 * p + c] + g1 * W[16 + 8 * p + c]);
      }
      put_piece(dh, v, p, y);
    }
    s[32] += g0;
    s[33] += g1;
  }
#pragma unroll
  for (int k = 0; k < 34; ++k) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s[k] += __shfl_down(s[k], o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][k] = s[k];
  }
  __syncthreads();
  if (threadIdx.x < 34)
    part[(size_t)blockIdx.x * 34 + threadIdx.x] =
        (sh[0][threadIdx.x] + sh[1][threadIdx.x]) + (sh[2][threadIdx.x] + sh[3][threadIdx.x]);
}

__global__ void adam_kernel(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, long n, float lr, float b1, float b2, float eps, float c1,
                            float c2, uint16_t* __restrict__ pb) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  p[i] = pi;
  if (pb) pb[i] = f2bf(pi);
}

unsigned blocks_for(long n, int t = 256) { return (unsigned)((n + t - 1) / t); }

template <int CIN, int COUT, int UP, bool SMALL, Tail TAIL>
void run_tiles(hipStream_t s, Dims d, View in, View up, const uint16_t* w, const float* bias, bool relu, View out,
               int zlen, const ConvTail& tail) {
  using C = ConvCfg<CIN, COUT, SMALL>;
  const long cols = (long)((d.x + C::TX - 1) / C::TX) * ((d.y + C::TY - 1) / C::TY);
  hipLaunchKernelGGL((zconv_kernel<CIN, COUT, UP, SMALL, TAIL>), dim3((unsigned)(cols * ((d.z + zlen - 1) / zlen))),
                     dim3(C::NT), 0, s, d, in, up, w, bias, relu ? 1 : 0, out, zlen, tail);
}

// z-chunk: as long as leaves two blocks per CU, for each chunk reads two planes more
template <int CIN, int COUT, bool SMALL>
long conv_blocks(Dims d, int& zlen) {
  using C = ConvCfg<CIN, COUT, SMALL>;
  const long cols = (long)((d.x + C::TX - 1) / C::TX) * ((d.y + C::TY - 1) / C::TY);
  zlen = 64;
  while (zlen > (SMALL ? 1 : 4) && cols * ((d.z + zlen - 1) / zlen) < 512) zlen /= 2;
  return cols * ((d.z + zlen - 1) / zlen);
}

template <int CIN, int COUT, int UP>
void run_conv(hipStream_t s, Dims d, View in, View up, const uint16_t* w, const float* bias, bool relu, View out) {
  int zlen;
  if (conv_blocks<CIN, COUT, false>(d, zlen) >= 256)
    return run_tiles<CIN, COUT, UP, false, STORE>(s, d, in, up, w, bias, relu, out, zlen, ConvTail{});
  conv_blocks<CIN, COUT, true>(d, zlen);
  run_tiles<CIN, COUT, UP, true, STORE>(s, d, in, up, w, bias, relu, out, zlen, ConvTail{});
}

// tile depth and blocks per 16 input channels of the weight gradient: tiles of four planes,
// fewer where that leaves the chip idle (one plane on the coarsest grids), and blocks enough
// for about one and a half per CU, each summing several tiles (a block's partial sums are
// 27 x cout x 16 values: more blocks cost more in the final sum than they gain)
struct WgradPlan {
  int tz, ntiles, nblk;
};
WgradPlan wgrad_plan(Dims d, int cin) {
  WgradPlan p;
  const long txy = (long)((d.x + WGX - 1) / WGX) * ((d.y + WGY - 1) / WGY);
  p.tz = WGZ;
  while (p.tz > 1 && txy * ((d.z + p.tz - 1) / p.tz) * (cin / 16) < 256) p.tz /= 2;
  p.ntiles = (int)(txy * ((d.z + p.tz - 1) / p.tz));
  const int want = (384 + cin / 16 - 1) / (cin / 16);
  p.nblk = p.ntiles < want ? p.ntiles : want;
  return p;
}

}  // namespace

// The layers of the network and, with the channels exchanged, their backward data passes; every
// view's channel stride and offset are multiples of 8, its base 16-byte aligned.
void launch_conv_fwd(hipStream_t s, Dims d, View in, int cin, const uint16_t* w, const float* bias, bool relu,
                     View out, int cout, View up, int cup) {
  const int key = cin * 1000 + cout;
  if (cup > 0) {
    if (key == 96032 && cup == 64) return run_conv<96, 32, 64>(s, d, in, up, w, bias, relu, out);
    if (key == 48016 && cup == 32) return run_conv<48, 16, 32>(s, d, in, up, w, bias, relu, out);
  } else {
    switch (key) {
      case 16016: return run_conv<16, 16, 0>(s, d, in, up, w, bias, relu, out);
      case 16032: return run_conv<16, 32, 0>(s, d, in, up, w, bias, relu, out);
      case 16048: return run_conv<16, 48, 0>(s, d, in, up, w, bias, relu, out);
      case 32016: return run_conv<32, 16, 0>(s, d, in, up, w, bias, relu, out);
      case 32032: return run_conv<32, 32, 0>(s, d, in, up, w, bias, relu, out);
      case 32064: return run_conv<32, 64, 0>(s, d, in, up, w, bias, relu, out);
      case 32096: return run_conv<32, 96, 0>(s, d, in, up, w, bias, relu, out);
      case 64032: return run_conv<64, 32, 0>(s, d, in, up, w, bias, relu, out);
      case 64064: return run_conv<64, 64, 0>(s, d, in, up, w, bias, relu, out);
    }
  }
  throw std::logic_error("internal: unsupported convolution");
}

// a small tile's wave lacks the neighbours: there pooling and head stay passes of their own
template <int CH>
bool run_pooled(hipStream_t s, Dims d, View in, const uint16_t* w, const float* bias, View out, const ConvTail& tail) {
  int zlen;
  if (conv_blocks<CH, CH, false>(d, zlen) < 256) return false;
  run_tiles<CH, CH, 0, false, POOL>(s, d, in, in, w, bias, true, out, zlen, tail);
  return true;
}

void launch_conv_pool(hipStream_t s, Dims d, View in, int ch, const uint16_t* w, const float* bias, View out,
                      View pool) {
  ConvTail tail;
  tail.pool = pool;
  if (ch == 16 ? run_pooled<16>(s, d, in, w, bias, out, tail) : run_pooled<32>(s, d, in, w, bias, out, tail)) return;
  launch_conv_fwd(s, d, in, ch, w, bias, true, out, ch);
  launch_pool(s, d, out, ch, pool);
}

void launch_conv_head(hipStream_t s, Dims d, View in, const uint16_t* w, const float* bias, View h, const float* W,
                      const float* b, float* o) {
  int zlen;
  if (conv_blocks<16, 16, false>(d, zlen) >= 256) {
    ConvTail tail;
    tail.hw = W;
    tail.hb = b;
    tail.o = o;
    return run_tiles<16, 16, 0, false, HEAD>(s, d, in, in, w, bias, true, h, zlen, tail);
  }
  launch_conv_fwd(s, d, in, 16, w, bias, true, h, 16);
  launch_head_fwd(s, h, (long)d.x * d.y * d.z, W, b, o);
}

void launch_conv_wgrad(hipStream_t s, Dims d, View x, int cin, View dz, int cout, float* part, float* dw, float* db,
                       SumJobs& sums) {
  const WgradPlan p = wgrad_plan(d, cin);
  const dim3 g(p.nblk, cin / 16);
  float* bpart = part + (size_t)p.nblk * 27 * cout * cin;
  switch (cout / 16) {
    case 1: hipLaunchKernelGGL((conv_wgrad_kernel<1>), g, dim3(WGNT), 0, s, d, x, dz, cin, p.tz, p.ntiles, part, bpart); break;
    case 2: hipLaunchKernelGGL((conv_wgrad_kernel<2>), g, dim3(WGNT), 0, s, d, x, dz, cin, p.tz, p.ntiles, part, bpart); break;
    case 4: hipLaunchKernelGGL((conv_wgrad_kernel<4>), g, dim3(WGNT), 0, s, d, x, dz, cin, p.tz, p.ntiles, part, bpart); break;
    default: break;
  }
  sums.add(part, dw, p.nblk, 27 * cout * cin);
  sums.add(bpart, db, p.nblk, cout);
}

void SumJobs::add(const float* part, float* out, int nchunk, int len) {
  const int b = n == 0 ? 0 : j[n - 1].blk0 + (j[n - 1].len + 63) / 64;
  j[n++] = SumJob{part, out, nchunk, len, b};
}

void launch_sums(hipStream_t s, const SumJobs& sums) {
  const SumJob& last = sums.j[sums.n - 1];
  hipLaunchKernelGGL(sum_chunks_kernel, dim3(last.blk0 + (last.len + 63) / 64), dim3(1024), 0, s, sums);
}

long wgrad_part_floats(Dims d, int cin, int cout) {
  return (long)wgrad_plan(d, cin).nblk * (27L * cin * cout + cout);
}

void launch_flip_transpose(hipStream_t s, const uint16_t* w, int cout, int cin, uint16_t* wt) {
  const long n = 27L * cout * cin;
  hipLaunchKernelGGL(flip_transpose_kernel, dim3(blocks_for(n)), dim3(256), 0, s, w, cout, cin, wt);
}

void launch_f32_to_bf16(hipStream_t s, const float* a, long n, uint16_t* b) {
  hipLaunchKernelGGL(f32_to_bf16_kernel, dim3(blocks_for(n)), dim3(256), 0, s, a, n, b);
}

void launch_relu_mask(hipStream_t s, View dh, View post, int C, long nvox, View dz) {
  hipLaunchKernelGGL(relu_mask_kernel, dim3(blocks_for(nvox * (C / 8))), dim3(256), 0, s, dh, post, C / 8, nvox, dz);
}

void launch_pool(hipStream_t s, Dims d, View in, int C, View out) {
  const long n = (long)(d.x / 2) * (d.y / 2) * (d.z / 2) * (C / 8);
  hipLaunchKernelGGL(pool_kernel, dim3(blocks_for(n)), dim3(256), 0, s, d, in, C / 8, n, out);
}

void launch_pool_back(hipStream_t s, Dims d, View in, int C, View out, View addend) {
  const long n = (long)d.x * d.y * d.z * (C / 8);
  hipLaunchKernelGGL(pool_back_kernel, dim3(blocks_for(n)), dim3(256), 0, s, d, in, C / 8, n, out, addend);
}

void launch_up(hipStream_t s, Dims d, View in, int C, View out) {
  const long n = (long)d.x * d.y * d.z * (C / 8);
  hipLaunchKernelGGL(up_kernel, dim3(blocks_for(n)), dim3(256), 0, s, d, in, C / 8, n, out);
}

void launch_up_back(hipStream_t s, Dims d, View in, int C, View out) {
  const long n = (long)(d.x / 2) * (d.y / 2) * (d.z / 2) * (C / 8);
  hipLaunchKernelGGL(up_back_kernel, dim3(blocks_for(n)), dim3(256), 0, s, d, in, C / 8, n, out);
}

void launch_head_fwd(hipStream_t s, View h, long nvox, const float* W, const float* b, float* o) {
  hipLaunchKernelGGL(head_fwd_kernel, dim3(blocks_for(nvox)), dim3(256), 0, s, h, nvox, W, b, o);
}

static unsigned head_blocks(long nvox) { return (unsigned)std::min<long>((nvox + 255) / 256, kHeadBlocks); }
long head_part_floats(long nvox) { return (long)head_blocks(nvox) * 34; }

void launch_head_back(hipStream_t s, View h, long nvox, const float* W, const float* dout, View dh, float* part,
                      float* dWb /* [34]: dW (32) then db (2) */, SumJobs& sums) {
  const unsigned nb = head_blocks(nvox);
  hipLaunchKernelGGL(head_back_kernel, dim3(nb), dim3(256), 0, s, h, nvox, W, dout, dh, part);
  sums.add(part, dWb, (int)nb, 34);
}

void launch_adam(hipStream_t s, float* p, const float* g, float* m, float* v, long n, float lr, float b1, float b2,
                 float eps, int step, uint16_t* pb) {
  const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
  hipLaunchKernelGGL(adam_kernel, dim3(blocks_for(n)), dim3(256), 0, s, p, g, m, v, n, lr, b1, b2, eps, c1, c2, pb);
}

}  // namespace hfci
