// Internal interface of the learned-preconditioner kernels (conv.hip, netprep.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace hfci {

struct Dims {
  int z, y, x;
};

// Channels-last BF16 view: element (voxel v, channel c) at p[v * cs + off + c].
struct View {
  uint16_t* p;
  int cs, off;
};

// what a convolution does with a finished output plane besides (or instead of) storing it
struct ConvTail {
  View pool{nullptr, 0, 0};
  const float *hw = nullptr, *hb = nullptr;
  float* o = nullptr;
};
// cup > 0: the first cup input channels are the x2 up-sampling of `up` (half the grid), the
// others `in`
void launch_conv_fwd(hipStream_t s, Dims d, View in, int cin, const uint16_t* w, const float* bias, bool relu,
                     View out, int cout, View up = View{nullptr, 0, 0}, int cup = 0);
// ch -> ch (16 or 32) ReLU layer and the 2x2x2 average of its output (even sides)
void launch_conv_pool(hipStream_t s, Dims d, View in, int ch, const uint16_t* w, const float* bias, View out,
                      View pool);
// 16 -> 16 ReLU layer and the head; h, its output, may be left unwritten
void launch_conv_head(hipStream_t s, Dims d, View in, const uint16_t* w, const float* bias, View h, const float* W,
                      const float* b, float* o);
// The sums over blocks of every gradient of a backward pass, one launch (a launch for each of the
// 21 cost 6.6 us): out[i] = sum over chunks of part[chunk][i], len values; job j's blocks start
// at blk0.  The kernels that write the partials add theirs; each keeps its own part until then.
struct SumJob {
  const float* part;
  float* out;
  int nchunk, len, blk0;
};
struct SumJobs {
  SumJob j[21];
  int n = 0;
  void add(const float* part, float* out, int nchunk, int len);
};
void launch_sums(hipStream_t s, const SumJobs& sums);
long wgrad_part_floats(Dims d, int cin, int cout);
// weight gradient dw [27][cout][cin] and bias gradient db [cout] (part: wgrad_part_floats)
void launch_conv_wgrad(hipStream_t s, Dims d, View x, int cin, View dz, int cout, float* part, float* dw, float* db,
                       SumJobs& sums);
void launch_flip_transpose(hipStream_t s, const uint16_t* w, int cout, int cin, uint16_t* wt);
void launch_f32_to_bf16(hipStream_t s, const float* a, long n, uint16_t* b);
void launch_relu_mask(hipStream_t s, View dh, View post, int C, long nvox, View dz);
void launch_pool(hipStream_t s, Dims d, View in, int C, View out);
void launch_pool_back(hipStream_t s, Dims d, View in, int C, View out, View addend);
void launch_up(hipStream_t s, Dims d, View in, int C, View out);
void launch_up_back(hipStream_t s, Dims d, View in, int C, View out);
void launch_head_fwd(hipStream_t s, View h, long nvox, const float* W, const float* b, float* o);
long head_part_floats(long nvox);
void launch_head_back(hipStream_t s, View h, long nvox, const float* W, const float* dout, View dh, float* part,
                      float* dWb, SumJobs& sums);
void launch_adam(hipStream_t s, float* p, const float* g, float* m, float* v, long n, float lr, float b1, float b2,
                 float eps, int step, uint16_t* pb);

// netprep.hip: network input/output conversions and the loss
// x16[v] = (Re, Im)(phase * r[v]) / scale, kch[v], 0 ... (16 channels), over a crop of the full grid
void launch_prep_input_c64(hipStream_t s, Dims full, Dims crop, int oz, int oy, int ox, const float2* r,
                           const float* kch, float ph_re, float ph_im, const double* scale, uint16_t* x16);
void launch_prep_target_c64(hipStream_t s, Dims full, Dims crop, int oz, int oy, int ox, const float2* e,
                            float ph_re, float ph_im, const double* scale, float* t);
void launch_prep_input_c128(hipStream_t s, long n, const double2* r, const float* kappa, float inv_s_h2,
                            const double* scale, uint16_t* x16);
void launch_output_c128(hipStream_t s, long n, const float* o, const double* scale, double2* z);
// sum of |r|^2 over a crop (complex64) or a full vector (complex128), into partials
int rms_blocks(long n);
void launch_sumsq_crop_c64(hipStream_t s, Dims full, Dims crop, int oz, int oy, int ox, const float2* r,
                           double* part);
void launch_sumsq_c128(hipStream_t s, long n, const double2* r, double* part);
// scale = sqrt(sum / count) (or 1 if zero) from partials
void launch_finish_rms(hipStream_t s, const double* part, int nblk, double count, double* scale);
// kind 0: relative squared loss |o - t|^2 / |t|^2, dout = 2 (o - t) / |t|^2;
// kind 1: scale- and phase-invariant loss 1 - |<o,t>|^2 / (|o|^2 |t|^2) of the complex field.
// sums[0] receives the loss; part needs 4 * rms_blocks(2 * nvox) doubles, sums 5.
void launch_loss(hipStream_t s, long nvox, const float* o, const float* t, double* part, double* sums, float* dout,
                 int kind);
// residual loss (kind 2): p = Ahat o on the box d, the kind-1 loss of p against v, and
// dout = Ahat dL/dp (Ahat is real and symmetric); Ahat = (6 - kch) - sum of the six
// neighbours (zero outside), kch from x16's third channel; p, dp: scratch [n][2]
void launch_residual_loss(hipStream_t s, Dims d, const uint16_t* x16, const float* o, const float* v, double* part,
                          double* sums, float* dout, float* p, float* dp);

}  // namespace hfci
