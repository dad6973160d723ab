// Shared declarations of the gfx950 kernels and their host launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "k_order.h"

namespace gan {

// bf16 storage: upper half of an fp32, round-to-nearest-even on conversion.
struct bf16_t {
  unsigned short v;
};

__host__ __device__ inline float to_float(float x) { return x; }
__host__ __device__ inline float to_float(bf16_t x) {
  union { unsigned u; float f; } c;
  c.u = (unsigned)x.v << 16;
  return c.f;
}
__host__ __device__ inline unsigned short f32_to_bf16_bits(float f) {
  union { unsigned u; float f; } c;
  c.f = f;
  unsigned u = c.u;
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;   // NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
template <typename T> __host__ __device__ inline T from_float(float f);
template <> __host__ __device__ inline float from_float<float>(float f) { return f; }
// On the device the conversion is the hardware's (v_cvt_pk_bf16_f32, round to nearest even like the function above);
// the software rounding costs six vector instructions per element, which made several kernels instruction-bound.
#if defined(__HIP_DEVICE_COMPILE__)
typedef float gan_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 gan_bf16x2 __attribute__((ext_vector_type(2)));
__host__ __device__ inline unsigned pack2_bf16(float lo, float hi) {
  const gan_f32x2 v = {lo, hi};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, gan_bf16x2));
}
template <> __host__ __device__ inline bf16_t from_float<bf16_t>(float f) {
  bf16_t r;
  r.v = __builtin_bit_cast(unsigned short, (__bf16)f);
  return r;
}
#else
__host__ __device__ inline unsigned pack2_bf16(float lo, float hi) { return (unsigned)f32_to_bf16_bits(lo) | ((unsigned)f32_to_bf16_bits(hi) << 16); }
template <> __host__ __device__ inline bf16_t from_float<bf16_t>(float f) {
  bf16_t r;
  r.v = f32_to_bf16_bits(f);
  return r;
}
#endif

// A host launcher that finds its assumptions violated records the reason and launches nothing; the library call in
// progress then returns an error status with this text (nothing in the library ends the process).
void launch_fail(const char* msg);
const char* take_launch_error();   // the first reason recorded on this thread since the last call, or nullptr

// Block tiles of the forward-type GEMM kernel (rows x columns): conv_gemm.hip
enum ConvTile { TILE_BIG = 0, TILE_MID = 1, TILE_SMALL = 2, TILE_NARROW = 3, TILE_TINY = 4, TILE_PAIR = 5, TILE_DEEP = 6 };
enum Epilogue { EPI_NONE = 0, EPI_ACT_BWD = 1, EPI_DROP_BWD = 2, EPI_BN = 3, EPI_BIAS_ACT = 4 };
enum Act { ACT_RELU = 0, ACT_LRELU = 1 };

// Arguments of the grouped implicit-GEMM forward-type kernel (down / up / dense).
struct ConvArgs {
  const void* A;         // gathered activations (storage type)
  const void* W;         // weights of model 0, K-contiguous: [tap][N][C] (storage type); fp32 convolutions with w_plane: [3][tap][N][C] bf16, the
                         // parts of launch_split_weights, planes w_plane elements apart
  long long w_plane;     // 0: W in the storage type
  const float* w_raw;    // the fp32 weights of model 0 themselves, element (tap, n, c) at tap * w_nstride * C + n * raw_n + c * raw_k
  long long raw_stride;  //   (elements between models), for tiles that have no split (see Split8)
  int raw_n, raw_k;
  void* Out;             // output activations (storage type)
  const void* Aux;       // EPI_ACT_BWD, EPI_DROP_BWD: saved forward output at the output position (storage type)
  float* stat_partial;   // if set: per sub-tile (the row block of one wave row of the tile; conv_stat_split of them per tile) the
                         // column sums of the output and of its squared deviations from the sub-tile's column mean,
                         // [(((phase * nseg + segment) * ub_tiles + tile) * split + block) * N + col][2], for the BatchNorm that follows
  int w_nstride;         // rows per tap in the weight block (>= N)
  const int* offs;       // [L+1] sample offsets of the models inside one segment
  const int* tpre;       // [L+1] prefix of M-tiles per model for this geometry
  const int* tmodel;     // model of every M-tile of this geometry (NULL: found by bisection in tpre)
  long long w_stride;    // elements between two models' weight blocks
  int L;                 // models
  int seg_first, nseg;   // segments to process: rows of segment s start at sample s*seg_samples
  int seg_samples;
  int C, N;              // channels per tap of A, output channels
  int Hin;               // side of the gathered tensor
  int Hr;                // side of the row space (rows per sample = Hr*Hr)
  int ub_tiles;          // launched upper bound of M-tiles per (segment, phase)
  ConvTile tile;         // its height is what the prefix array was built for
  int hr_shift;          // log2(Hr) or -1 (filled by the launcher)
  float slope;           // EPI_ACT_BWD, EPI_DROP_BWD: derivative on the non-positive side; EPI_BN, EPI_BIAS_ACT: factor there
  // EPI_BN: BatchNorm with known statistics (gamma (x - mean) / sqrt(var + eps) + beta) and the activation (slope below zero) of every
  // output; column col is channel col % bn_C.  Vectors of model 0; strides between models.
  const float *bn_mean, *bn_var, *bn_gamma, *bn_beta;
  const float* bn_bias;  // [N] added first, then a ReLU (a layer whose activation comes before its BatchNorm), or NULL; EPI_BIAS_ACT: [N] added
  long long bn_rstride, bn_pstride;
  int bn_C;
  float bn_eps;
  float drop_scale;      // EPI_DROP_BWD: 1 / (1 - p); where the saved output is +0 the element was dropped (see dropped())
};

// Arguments of the grouped weight-gradient kernel: dW[tap][cb][cs] = sum_rows big(tap)[cb] * small[cs].
struct WgradArgs {
  const void* Big;       // tensor gathered through the taps, side 2*Hs, channels Cb (ntaps == 1: read row by row)
  const void* Small;     // tensor indexed directly by row, side Hs, channels Cs
  float* dW;             // fp32 output of model 0: [ntaps][Cb][Cs]
  const int* offs;       // [L+1]
  const int* order;      // [L] models by decreasing row count, or NULL: which model a group of blocks takes (the
                         //     big models start first and the XCDs get equal shares; no effect on the results)
  long long dw_stride;   // elements between two models' blocks
  int L, nseg, seg_samples;
  int Cb, Cs, Hs;
  int ntaps;             // 16 (conv) or 1 (dense)
  int ksplit;            // >= 1: the rows of each segment are shared by this many blocks, each writing its own
  long long split_stride;//        partial block dW + split * split_stride (the caller adds them in order)
  int hs_shift;          // log2(Hs) or -1 (filled by the launcher)
  unsigned rps_inv, hs_inv;   // sides that are no power of two: reciprocals of Hs*Hs and Hs (filled by the launcher; 0: divide)
};

// Dropout writes +0 where it drops; a kept value that is or rounds to zero is stored as -0.  The backward pass reads the mask
// off the stored tensor.
__host__ __device__ inline float kept_nonzero(float v) { return v == 0.f ? -0.f : v; }
__host__ __device__ inline bf16_t kept_nonzero(bf16_t v) { v.v = v.v == 0 ? 0x8000 : v.v; return v; }
__device__ inline bool dropped(float saved) { return __float_as_uint(saved) == 0; }

// Position class of pixel (y, x) of an Hs-sided map under a k4 s2 p1 filter, by which of its taps lie outside: first, inner and
// last pixel along either axis.
__device__ inline int pos_class(int y, int x, int Hs) {
  return (y == 0 ? 0 : (y == Hs - 1 ? 2 : 1)) * 3 + (x == 0 ? 0 : (x == Hs - 1 ? 2 : 1));
}

// Whether the tap k (one axis) of the pixels of class cls along it (0 first, 1 inner, 2 last) lies inside the map.
__device__ inline bool tap_inside(int cls, int k) { return !((cls == 0 && k == 0) || (cls == 2 && k == 3)); }
// what the sixteen taps of a constant map add up to at a class of positions, as the storage type holds it
template <typename T>
__device__ inline float label_class_sum(const float (&v)[16], int cls) {
  float s = 0.f;
#pragma unroll
  for (int tap = 0; tap < 16; ++tap)
    if (tap_inside(cls / 3, tap >> 2) && tap_inside(cls % 3, tap & 3)) s += v[tap];
  return to_float(from_float<T>(s));
}

template <typename T> void launch_conv(int mode, int epi, const ConvArgs& a, hipStream_t st);
template <typename T> void launch_wgrad(const WgradArgs& a, hipStream_t st);
// names of the kernel instantiations the two launchers pick (per-kernel timing)
const char* conv_variant_name(int esize, int mode, int epi, const ConvArgs& a);
const char* wgrad_variant_name(int esize, const WgradArgs& a);
// output tiles per model of the weight-gradient launch for this layer shape (esize: bytes per stored element)
int wgrad_tiles_per_model(int esize, int ntaps, int Cb, int Cs);

// The forward-type kernel's tile for a launch shape (esize: bytes per stored element; groups: output phases x segments), its
// rows, and its row blocks with BatchNorm partial sums of their own.
ConvTile conv_choose_tile(int esize, int n_out, double rows_per_model, int n_models, int groups);
ConvTile conv_tile_of_rows(int esize, int rows, int n_out);
int conv_tile_rows(int esize, ConvTile t);
int conv_stat_split(int esize, ConvTile t, bool split_weights);      // split_weights: fp32 convolutions, see ConvArgs

}  // namespace gan
