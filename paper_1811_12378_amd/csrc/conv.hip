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
// Implicit GEMM: output tile = 16 voxels x 16 output channels per wavefront,
//   D[v][co] += sum_{tap, ci} X[v + off_tap][ci] * W[tap][co][ci],
// one v_mfma_f32_16x16x32_bf16 (Cin % 32 == 0) or v_mfma_f32_16x16x16_bf16 per
// (tap, 32- or 16-channel chunk, Cout tile).  Lane l supplies row (l % 16) and the
// k-range [KB*(l/16), KB*(l/16)+KB) of A (voxels x channels) and column (l % 16) of B;
// the accumulator holds rows 4*(l/16)+r, column l%16.  Voxels are numbered linearly
// (x fastest), so any grid shape fills the waves.
//
// The backward data pass is the same kernel applied to the output gradient with the
// tap-flipped, Cin/Cout-transposed weights; the weight gradient is a GEMM over voxels
// (k = voxel) whose per-chunk partial sums are reduced in a fixed order.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "netkern.h"

namespace hfci {
namespace {

typedef short s4v __attribute__((ext_vector_type(4)));
typedef __bf16 b8v __attribute__((ext_vector_type(8)));
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

template <int KB>
struct Frag;
template <>
struct Frag<4> {  // 16x16x16: 4 bf16 per lane
  using T = s4v;
  __device__ static T load(const uint16_t* p) {
    const uint2 u = *reinterpret_cast<const uint2*>(p);
    T r;
    r[0] = (short)(u.x & 0xffff);
    r[1] = (short)(u.x >> 16);
    r[2] = (short)(u.y & 0xffff);
    r[3] = (short)(u.y >> 16);
    return r;
  }
  __device__ static T zero() { return T{0, 0, 0, 0}; }
  __device__ static f4v mma(T a, T b, f4v c) { return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0); }
};
template <>
struct Frag<8> {  // 16x16x32: 8 bf16 per lane
  using T = b8v;
  __device__ static T load(const uint16_t* p) {
    const uint4 u = *reinterpret_cast<const uint4*>(p);
    return __builtin_bit_cast(T, u);
  }
  __device__ static T zero() { return __builtin_bit_cast(T, make_uint4(0, 0, 0, 0)); }
  __device__ static f4v mma(T a, T b, f4v c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
};

// Forward 3x3x3 convolution: one block = 64 consecutive voxels (4 waves x 16);
// each wave produces all Cout channels of its 16 voxels.  CT = Cout / 16 tiles.
template <int KB, int CT>
__global__ __launch_bounds__(256) void conv_fwd_kernel(Dims d, View in, int cin, const uint16_t* __restrict__ w,
                                                       const float* __restrict__ bias, int relu, View out) {
  using F = Frag<KB>;
  constexpr int KC = 4 * KB;  // channels per MFMA
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long nvox = (long)d.x * d.y * d.z;
  const long v0 = (long)blockIdx.x * 64 + wave * 16;
  const int row = lane & 15, kq = lane >> 4;
  const long va = v0 + row;  // voxel whose A-row this lane supplies
  const bool va_ok = va < nvox;
  const Coord ca = coord_of(va_ok ? va : 0, d);
  const int cout = CT * 16;
  f4v acc[CT];
#pragma unroll
  for (int t = 0; t < CT; ++t) acc[t] = f4v{0.f, 0.f, 0.f, 0.f};
  for (int tap = 0; tap < 27; ++tap) {
    const int dz = tap / 9 - 1, dy = (tap / 3) % 3 - 1, dx = tap % 3 - 1;
    const int zz = ca.z + dz, yy = ca.y + dy, xx = ca.x + dx;
    const bool ok = va_ok && zz >= 0 && zz < d.z && yy >= 0 && yy < d.y && xx >= 0 && xx < d.x;
    const long vin = ok ? ((long)zz * d.y + yy) * d.x + xx : 0;
    const uint16_t* ap = in.p + vin * in.cs + in.off + kq * KB;
    const uint16_t* wp = w + (size_t)tap * cout * cin + (size_t)row * cin + kq * KB;
    for (int c0 = 0; c0 < cin; c0 += KC) {
      const typename F::T a = ok ? F::load(ap + c0) : F::zero();
#pragma unroll
      for (int t = 0; t < CT; ++t) {
        const typename F::T b = F::load(wp + (size_t)t * 16 * cin + c0);
        acc[t] = F::mma(a, b, acc[t]);
      }
    }
  }
  // accumulator: rows (voxels) 4*kq + r, column (channel) row
#pragma unroll
  for (int t = 0; t < CT; ++t) {
    const int co = t * 16 + row;
    const float bv = bias ? bias[co] : 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const long v = v0 + kq * 4 + r;
      if (v < nvox) {
        float val = acc[t][r] + bv;
        if (relu) val = fmaxf(val, 0.f);
        out.p[v * out.cs + out.off + co] = f2bf(val);
      }
    }
  }
}

// 16 -> 16 channel layers (the full-resolution level of the U-Net) as a z-marching
// implicit GEMM.  A block owns a 64 x 4 voxel tile of each plane of a z-chunk; the input
// tile with its one-voxel halo (66 x 6 voxels x 16 channels) of planes z-1, z, z+1 sits
// in a 3-plane LDS ring and the 27 x 16 x 16 weights in LDS, so every input voxel is read
// from memory about once per chunk instead of once per tap.  Wave w computes row y0+w:
// four 16-voxel blocks, one MFMA per (tap, block) with the weights as A (cout x cin) and
// the input as B (cin x voxels), so the accumulator of lane l holds output channels
// 4(l/16)..4(l/16)+3 of voxel l%16 and is stored as one 8-byte write.
constexpr int ZCX = 64, ZCY = 4, ZLX = ZCX + 2, ZLY = ZCY + 2;

__global__ __launch_bounds__(256) void zconv16_kernel(Dims d, View in, const uint16_t* __restrict__ w,
                                                      const float* __restrict__ bias, int relu, View out, int zlen) {
  __shared__ __align__(16) uint16_t ring[3][ZLY][ZLX][16];
  __shared__ __align__(16) uint16_t ws[27][16][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int gx = (d.x + ZCX - 1) / ZCX, gy = (d.y + ZCY - 1) / ZCY;
  const int b = blockIdx.x;
  const int bx = b % gx, by = (b / gx) % gy, zc = b / (gx * gy);
  const int x0 = bx * ZCX, y0 = by * ZCY;
  const int zb = zc * zlen, ze = min(d.z, zb + zlen);
  for (int i = threadIdx.x; i < 27 * 16 * 16 / 8; i += 256)
    reinterpret_cast<uint4*>(&ws[0][0][0])[i] = reinterpret_cast<const uint4*>(w)[i];
  // plane zp of the input tile into ring slot zp mod 3 (zeros outside the grid)
  auto load_plane = [&](int zp) {
    uint4* dst = reinterpret_cast<uint4*>(&ring[(zp + 3) % 3][0][0][0]);
    for (int c = threadIdx.x; c < ZLY * ZLX * 2; c += 256) {
      const int vox = c >> 1, half = c & 1;
      const int lx = vox % ZLX, ly = vox / ZLX;
      const int xg = x0 - 1 + lx, yg = y0 - 1 + ly;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (zp >= 0 && zp < d.z && xg >= 0 && xg < d.x && yg >= 0 && yg < d.y)
        v = *reinterpret_cast<const uint4*>(in.p + (((long)zp * d.y + yg) * d.x + xg) * in.cs + in.off + half * 8);
      dst[c] = v;
    }
  };
  if (zb >= ze) return;
  load_plane(zb - 1);
  load_plane(zb);
  const int row = lane & 15, kq = lane >> 4;
  const int yo = y0 + wave;
  float bv[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) bv[r] = bias ? bias[4 * kq + r] : 0.f;
  for (int z = zb; z < ze; ++z) {
    load_plane(z + 1);
    __syncthreads();
    f4v acc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int tap = 0; tap < 27; ++tap) {
      const int dz = tap / 9 - 1, dy = (tap / 3) % 3 - 1, dx = tap % 3 - 1;
      const s4v wa = *reinterpret_cast<const s4v*>(&ws[tap][row][4 * kq]);
      const uint16_t(*pl)[ZLX][16] = ring[(z + dz + 3) % 3];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const s4v xb = *reinterpret_cast<const s4v*>(&pl[wave + 1 + dy][q * 16 + row + 1 + dx][4 * kq]);
        acc[q] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wa, xb, acc[q], 0, 0, 0);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int xo = x0 + q * 16 + row;
      if (xo < d.x && yo < d.y) {
        uint16_t h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float v = acc[q][r] + bv[r];
          if (relu) v = fmaxf(v, 0.f);
          h[r] = f2bf(v);
        }
        const uint2 pk = make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16));
        *reinterpret_cast<uint2*>(out.p + (((long)z * d.y + yo) * d.x + xo) * out.cs + out.off + 4 * kq) = pk;
      }
    }
    __syncthreads();
  }
}

// 48 -> 16 channel layer (the full-resolution decoder's first convolution, on the
// concatenation of the upsampled coarse features and the skip connection) as a z-marching
// implicit GEMM.  As zconv16, but the 48-channel planes are too large for a 64 x 4 tile to
// leave room for two blocks per CU: a block owns a 32 x 4 tile, its input planes (34 x 6
// voxels with the halo, 48 channels padded to 56 per voxel, so 16-byte rows stay aligned)
// sit in a 3-plane LDS ring (68.5 KB), and the weights (27 x 16 x 48, the same for every
// block) are read through the L1 cache.  Wave w computes row y0 + w: two 16-voxel blocks,
// one 16x16x16 MFMA per (tap, 16-channel chunk, block), weights as A and input as B.
constexpr int ZDX = 32, ZDY = 4, ZDLX = ZDX + 2, ZDLY = ZDY + 2, ZDC = 48, ZDCP = 56;

__global__ __launch_bounds__(256) void zconv48_kernel(Dims d, View in, const uint16_t* __restrict__ w,
                                                      const float* __restrict__ bias, int relu, View out, int zlen) {
  __shared__ __align__(16) uint16_t ring[3][ZDLY][ZDLX][ZDCP];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int gx = (d.x + ZDX - 1) / ZDX, gy = (d.y + ZDY - 1) / ZDY;
  const int b = blockIdx.x;
  const int bx = b % gx, by = (b / gx) % gy, zc = b / (gx * gy);
  const int x0 = bx * ZDX, y0 = by * ZDY;
  const int zb = zc * zlen, ze = min(d.z, zb + zlen);
  if (zb >= ze) return;
  constexpr int PARTS = ZDC / 8;  // 16-byte pieces per voxel
  auto load_plane = [&](int zp) {
    uint16_t(*dst)[ZDLX][ZDCP] = ring[(zp + 3) % 3];
    for (int c = threadIdx.x; c < ZDLY * ZDLX * PARTS; c += 256) {
      const int vox = c / PARTS, part = c % PARTS;
      const int lx = vox % ZDLX, ly = vox / ZDLX;
      const int xg = x0 - 1 + lx, yg = y0 - 1 + ly;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (zp >= 0 && zp < d.z && xg >= 0 && xg < d.x && yg >= 0 && yg < d.y)
        v = *reinterpret_cast<const uint4*>(in.p + (((long)zp * d.y + yg) * d.x + xg) * in.cs + in.off + part * 8);
      *reinterpret_cast<uint4*>(&dst[ly][lx][part * 8]) = v;
    }
  };
  load_plane(zb - 1);
  load_plane(zb);
  const int row = lane & 15, kq = lane >> 4;
  const int yo = y0 + wave;
  float bv[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) bv[r] = bias ? bias[4 * kq + r] : 0.f;
  for (int z = zb; z < ze; ++z) {
    load_plane(z + 1);
    __syncthreads();
    f4v acc[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) acc[q] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int tap = 0; tap < 27; ++tap) {
      const int dz = tap / 9 - 1, dy = (tap / 3) % 3 - 1, dx = tap % 3 - 1;
      const uint16_t(*pl)[ZDLX][ZDCP] = ring[(z + dz + 3) % 3];
      const uint16_t* wp = w + ((size_t)tap * 16 + row) * ZDC + 4 * kq;
#pragma unroll
      for (int c = 0; c < ZDC / 16; ++c) {
        const s4v wa = Frag<4>::load(wp + 16 * c);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const s4v xb = *reinterpret_cast<const s4v*>(&pl[wave + 1 + dy][q * 16 + row + 1 + dx][16 * c + 4 * kq]);
          acc[q] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wa, xb, acc[q], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int xo = x0 + q * 16 + row;
      if (xo < d.x && yo < d.y) {
        uint16_t h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float v = acc[q][r] + bv[r];
          if (relu) v = fmaxf(v, 0.f);
          h[r] = f2bf(v);
        }
        const uint2 pk = make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16));
        *reinterpret_cast<uint2*>(out.p + (((long)z * d.y + yo) * d.x + xo) * out.cs + out.off + 4 * kq) = pk;
      }
    }
    __syncthreads();
  }
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
        const b8v a = Frag<8>::load(ds + (t * 16 + row) * WGDS + r * WGX + 8 * kq);
        acc[0][t] = Frag<8>::mma(a, bm, acc[0][t]);
        acc[1][t] = Frag<8>::mma(a, b0, acc[1][t]);
        acc[2][t] = Frag<8>::mma(a, bp, acc[2][t]);
        if (wave == 4 && ci0 == 0) {  // the centre pair's wave also sums dz (a product with ones)
          const uint32_t one = 0x3f803f80u;
          bacc[t] = Frag<8>::mma(a, __builtin_bit_cast(b8v, make_uint4(one, one, one, one)), bacc[t]);
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
// takes 64 values; 16 waves sum every 16th chunk each, then the 16 sums in order (one thread
// per value over all chunks left most of the chip idle: 22 us per layer on 64^3 voxels).
__global__ __launch_bounds__(1024) void sum_chunks_kernel(const float* __restrict__ part, int nchunk, long len,
                                                          float* __restrict__ out) {
  __shared__ float sh[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long i = (long)blockIdx.x * 64 + lane;
  float s = 0.f;
  if (i < len)
    for (int c = wave; c < nchunk; c += 16) s += part[(size_t)c * len + i];
  sh[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && i < len) {
    s = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) s += sh[w][lane];
    out[i] = s;
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

// relu backward: dzo[v][c] = dh[v][c] if post[v][c] > 0 else 0
__global__ void relu_mask_kernel(View dh, View post, int C, long nvox, View dzo) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nvox * C) return;
  const long v = i / C;
  const int c = (int)(i % C);
  const uint16_t pv = post.p[v * post.cs + post.off + c];
  const bool pos = (pv & 0x8000u) == 0 && (pv & 0x7fffu) != 0;
  dzo.p[v * dzo.cs + dzo.off + c] = pos ? dh.p[v * dh.cs + dh.off + c] : (uint16_t)0;
}

// 2x2x2 average pooling (fine dims d, coarse dims d/2)
__global__ void pool_kernel(Dims d, View in, int C, View out) {
  const Dims e{d.z / 2, d.y / 2, d.x / 2};
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long n = (long)e.x * e.y * e.z * C;
  if (i >= n) return;
  const int c = (int)(i % C);
  const long vc = i / C;
  const Coord q = coord_of(vc, e);
  float s = 0.f;
  for (int k = 0; k < 8; ++k) {
    const long v = ((long)(2 * q.z + (k >> 2)) * d.y + 2 * q.y + ((k >> 1) & 1)) * d.x + 2 * q.x + (k & 1);
    s += bf2f(in.p[v * in.cs + in.off + c]);
  }
  out.p[vc * out.cs + out.off + c] = f2bf(0.125f * s);
}

// adjoint of pooling: out[v][c] (+)= in[parent(v)][c] / 8  (fine dims d)
__global__ void pool_back_kernel(Dims d, View in, int C, View out, View addend) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long n = (long)d.x * d.y * d.z * C;
  if (i >= n) return;
  const int c = (int)(i % C);
  const long v = i / C;
  const Coord f = coord_of(v, d);
  const long vc = ((long)(f.z / 2) * (d.y / 2) + f.y / 2) * (d.x / 2) + f.x / 2;
  float s = 0.125f * bf2f(in.p[vc * in.cs + in.off + c]);
  if (addend.p) s += bf2f(addend.p[v * addend.cs + addend.off + c]);
  out.p[v * out.cs + out.off + c] = f2bf(s);
}

// nearest-neighbour x2 up-sampling (fine dims d)
__global__ void up_kernel(Dims d, View in, int C, View out) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long n = (long)d.x * d.y * d.z * C;
  if (i >= n) return;
  const int c = (int)(i % C);
  const long v = i / C;
  const Coord f = coord_of(v, d);
  const long vc = ((long)(f.z / 2) * (d.y / 2) + f.y / 2) * (d.x / 2) + f.x / 2;
  out.p[v * out.cs + out.off + c] = in.p[vc * in.cs + in.off + c];
}

// adjoint of up-sampling: out[vc][c] = sum of the 8 children (coarse dims d/2)
__global__ void up_back_kernel(Dims d, View in, int C, View out) {
  const Dims e{d.z / 2, d.y / 2, d.x / 2};
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long n = (long)e.x * e.y * e.z * C;
  if (i >= n) return;
  const int c = (int)(i % C);
  const long vc = i / C;
  const Coord q = coord_of(vc, e);
  float s = 0.f;
  for (int k = 0; k < 8; ++k) {
    const long v = ((long)(2 * q.z + (k >> 2)) * d.y + 2 * q.y + ((k >> 1) & 1)) * d.x + 2 * q.x + (k & 1);
    s += bf2f(in.p[v * in.cs + in.off + c]);
  }
  out.p[vc * out.cs + out.off + c] = f2bf(s);
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

// head backward: dh[v][c] = sum_k dout[v][k] W[k][c] (bf16); partial dW/db per block
__global__ __launch_bounds__(256) void head_back_kernel(View h, long nvox, const float* __restrict__ W,
                                                        const float* __restrict__ dout, View dh,
                                                        float* __restrict__ part /* [blk][34] */) {
  __shared__ float sh[256];
  const long v = (long)blockIdx.x * 256 + threadIdx.x;
  float g0 = 0.f, g1 = 0.f;
  float x[16];
  if (v < nvox) {
    g0 = dout[2 * v];
    g1 = dout[2 * v + 1];
    for (int c = 0; c < 16; ++c) {
      x[c] = bf2f(h.p[v * h.cs + h.off + c]);
      dh.p[v * dh.cs + dh.off + c] = f2bf(g0 * W[c] + g1 * W[16 + c]);
    }
  } else {
    for (int c = 0; c < 16; ++c) x[c] = 0.f;
  }
  for (int k = 0; k < 34; ++k) {
    float val;
    if (k < 16) val = g0 * x[k];
    else if (k < 32) val = g1 * x[k - 16];
    else val = k == 32 ? g0 : g1;
    sh[threadIdx.x] = val;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
      __syncthreads();
    }
    if (threadIdx.x == 0) part[(size_t)blockIdx.x * 34 + k] = sh[0];
    __syncthreads();
  }
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

void launch_sum_chunks(hipStream_t s, const float* part, int nchunk, long len, float* out) {
  hipLaunchKernelGGL(sum_chunks_kernel, dim3(blocks_for(len, 64)), dim3(1024), 0, s, part, nchunk, len, out);
}

template <int KB>
void fwd_dispatch(hipStream_t s, Dims d, View in, int cin, const uint16_t* w, const float* bias, int relu, View out,
                  int cout) {
  const long nvox = (long)d.x * d.y * d.z;
  const dim3 g((unsigned)((nvox + 63) / 64));
  switch (cout / 16) {
    case 1: hipLaunchKernelGGL((conv_fwd_kernel<KB, 1>), g, dim3(256), 0, s, d, in, cin, w, bias, relu, out); break;
    case 2: hipLaunchKernelGGL((conv_fwd_kernel<KB, 2>), g, dim3(256), 0, s, d, in, cin, w, bias, relu, out); break;
    case 3: hipLaunchKernelGGL((conv_fwd_kernel<KB, 3>), g, dim3(256), 0, s, d, in, cin, w, bias, relu, out); break;
    case 4: hipLaunchKernelGGL((conv_fwd_kernel<KB, 4>), g, dim3(256), 0, s, d, in, cin, w, bias, relu, out); break;
    case 6: hipLaunchKernelGGL((conv_fwd_kernel<KB, 6>), g, dim3(256), 0, s, d, in, cin, w, bias, relu, out); break;
    default: break;
  }
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

bool conv_shape_ok(int cin, int cout) {
  auto ok = [](int c) { return c == 16 || c == 32 || c == 48 || c == 64 || c == 96; };
  return ok(cin) && (cout == 16 || cout == 32 || cout == 48 || cout == 64 || cout == 96);
}

void launch_conv_fwd(hipStream_t s, Dims d, View in, int cin, const uint16_t* w, const float* bias, bool relu,
                     View out, int cout) {
  // the 16 -> 16 layers take the z-marching kernel when the views allow 16-byte vector
  // access (channel stride and offset multiples of 8)
  if (cin == 16 && cout == 16 && in.cs % 8 == 0 && in.off % 8 == 0 && out.cs % 4 == 0 && out.off % 4 == 0) {
    const int gx = (d.x + ZCX - 1) / ZCX, gy = (d.y + ZCY - 1) / ZCY;
    int zlen = 32;
    while (zlen > 4 && (long)gx * gy * ((d.z + zlen - 1) / zlen) < 2048) zlen /= 2;
    const unsigned nb = (unsigned)((long)gx * gy * ((d.z + zlen - 1) / zlen));
    hipLaunchKernelGGL(zconv16_kernel, dim3(nb), dim3(256), 0, s, d, in, w, bias, relu ? 1 : 0, out, zlen);
    return;
  }
  // the 48 -> 16 layer likewise (16-byte loads of the input, 8-byte stores of the output)
  if (cin == ZDC && cout == 16 && in.cs % 8 == 0 && in.off % 8 == 0 && out.cs % 4 == 0 && out.off % 4 == 0) {
    const int gx = (d.x + ZDX - 1) / ZDX, gy = (d.y + ZDY - 1) / ZDY;
    int zlen = 32;
    while (zlen > 4 && (long)gx * gy * ((d.z + zlen - 1) / zlen) < 2048) zlen /= 2;
    const unsigned nb = (unsigned)((long)gx * gy * ((d.z + zlen - 1) / zlen));
    hipLaunchKernelGGL(zconv48_kernel, dim3(nb), dim3(256), 0, s, d, in, w, bias, relu ? 1 : 0, out, zlen);
    return;
  }
  if (cin % 32 == 0)
    fwd_dispatch<8>(s, d, in, cin, w, bias, relu ? 1 : 0, out, cout);
  else
    fwd_dispatch<4>(s, d, in, cin, w, bias, relu ? 1 : 0, out, cout);
}

void launch_conv_wgrad(hipStream_t s, Dims d, View x, int cin, View dz, int cout, float* part, float* dw, float* db) {
  const WgradPlan p = wgrad_plan(d, cin);
  const dim3 g(p.nblk, cin / 16);
  float* bpart = part + (size_t)p.nblk * 27 * cout * cin;
  switch (cout / 16) {
    case 1: hipLaunchKernelGGL((conv_wgrad_kernel<1>), g, dim3(WGNT), 0, s, d, x, dz, cin, p.tz, p.ntiles, part, bpart); break;
    case 2: hipLaunchKernelGGL((conv_wgrad_kernel<2>), g, dim3(WGNT), 0, s, d, x, dz, cin, p.tz, p.ntiles, part, bpart); break;
    case 4: hipLaunchKernelGGL((conv_wgrad_kernel<4>), g, dim3(WGNT), 0, s, d, x, dz, cin, p.tz, p.ntiles, part, bpart); break;
    default: break;
  }
  launch_sum_chunks(s, part, p.nblk, 27L * cout * cin, dw);
  launch_sum_chunks(s, bpart, p.nblk, cout, db);
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
  hipLaunchKernelGGL(relu_mask_kernel, dim3(blocks_for(nvox * C)), dim3(256), 0, s, dh, post, C, nvox, dz);
}

void launch_pool(hipStream_t s, Dims d, View in, int C, View out) {
  const long n = (long)(d.x / 2) * (d.y / 2) * (d.z / 2) * C;
  hipLaunchKernelGGL(pool_kernel, dim3(blocks_for(n)), dim3(256), 0, s, d, in, C, out);
}

void launch_pool_back(hipStream_t s, Dims d, View in, int C, View out, View addend) {
  const long n = (long)d.x * d.y * d.z * C;
  hipLaunchKernelGGL(pool_back_kernel, dim3(blocks_for(n)), dim3(256), 0, s, d, in, C, out, addend);
}

void launch_up(hipStream_t s, Dims d, View in, int C, View out) {
  const long n = (long)d.x * d.y * d.z * C;
  hipLaunchKernelGGL(up_kernel, dim3(blocks_for(n)), dim3(256), 0, s, d, in, C, out);
}

void launch_up_back(hipStream_t s, Dims d, View in, int C, View out) {
  const long n = (long)(d.x / 2) * (d.y / 2) * (d.z / 2) * C;
  hipLaunchKernelGGL(up_back_kernel, dim3(blocks_for(n)), dim3(256), 0, s, d, in, C, out);
}

void launch_head_fwd(hipStream_t s, View h, long nvox, const float* W, const float* b, float* o) {
  hipLaunchKernelGGL(head_fwd_kernel, dim3(blocks_for(nvox)), dim3(256), 0, s, h, nvox, W, b, o);
}

long head_part_floats(long nvox) { return ((nvox + 255) / 256) * 34; }

void launch_head_back(hipStream_t s, View h, long nvox, const float* W, const float* dout, View dh, float* part,
                      float* dWb /* [34]: dW (32) then db (2) */) {
  const unsigned nb = blocks_for(nvox);
  hipLaunchKernelGGL(head_back_kernel, dim3(nb), dim3(256), 0, s, h, nvox, W, dout, dh, part);
  launch_sum_chunks(s, part, (int)nb, 34L, dWb);
}

void launch_adam(hipStream_t s, float* p, const float* g, float* m, float* v, long n, float lr, float b1, float b2,
                 float eps, int step, uint16_t* pb) {
  const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
  hipLaunchKernelGGL(adam_kernel, dim3(blocks_for(n)), dim3(256), 0, s, p, g, m, v, n, lr, b1, b2, eps, c1, c2, pb);
}

}  // namespace hfci
