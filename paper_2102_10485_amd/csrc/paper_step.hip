// Kernels of the training step for the networks exactly as the paper's Tables 1 and 2 print them (Section 4), next to
// what the k4 s2 p1 engine already provides:
//   D block: Conv k3 s2 p1 (+bias) -> LeakyReLU -> Dropout(0.25) [-> BatchNorm(eps 0.8)]  -- the convolution runs on
//            the engine as a k4 s2 p1 one whose fourth tap row and column are zero, channel counts padded to 64;
//            bias, activation and dropout are one pass over its output, BatchNorm takes its statistics from the
//            stored tensor (they cannot come from the GEMM: the activation and the dropout sit in between);
//   G input: Linear (+bias) -> ReLU -> BatchNorm(eps 1e-5)                                 -- bias and ReLU in the GEMM (EPI_BIAS_ACT);
//   G last : Conv k3 s1 p1 (+bias) -> tanh onto the image, and its two gradients: conv3_mfma.hip.
// All sums run in a fixed order (thread-strided partial sums, then ordered merges), so a model's result does not depend
// on what else is in the launch.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.h"

namespace gan {

__device__ inline void philox4(unsigned c0, unsigned c1, unsigned c2, unsigned c3, unsigned k0, unsigned k1, unsigned (&out)[4]) {
  // Philox-4x32-10 (Salmon et al., SC'11), all four output words; same definition as in paper_layers.hip
  constexpr unsigned M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) { k0 += W0; k1 += W1; }
    const unsigned long long p0 = (unsigned long long)M0 * c0, p1 = (unsigned long long)M1 * c2;     // one wide multiply each
    const unsigned hi0 = (unsigned)(p0 >> 32), lo0 = (unsigned)p0, hi1 = (unsigned)(p1 >> 32), lo1 = (unsigned)p1;
    const unsigned n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
  }
  out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// the four output words that hold the keep-decisions of elements lin .. lin + 3 (lin a multiple of 4) of a
// [n][C][H][W]-indexed tensor, or the one of element lin (any lin): see gan_op_dropout in gan.h
__device__ inline void dropout_words(const PointArgs& a, int l, unsigned long long lin, int pass_id, unsigned step, unsigned (&w)[4]) {
  philox4((unsigned)(lin >> 2), (unsigned)(lin >> 34), (unsigned)(a.layer + 256 * pass_id), step, a.seed_lo, a.seed_hi ^ (unsigned)l, w);
}

// x <- dropout(act(x + bias)).  The backward pass has no kernel of its own: the mask and the activation's sign are read off the
// stored result (see dropped()) by the kernels that produce the gradient -- the BatchNorm's backward apply, and for the first block the
// data-gradient GEMM's epilogue.  (As a pass over the gradient that evaluated the generator again: 550 us per step with 100 models
// of 64 32x32x3 samples in bf16, 10.08 -> 9.49 ms.)
template <typename T>
__device__ inline float point_value(const PointArgs& a, float v, const float* bias, int c) {
  if (bias) v += bias[c];
  return v > 0.f ? v : v * a.slope;
}
template <typename T>
__global__ __launch_bounds__(256) void point_kernel(PointArgs a) {
  const int j = blockIdx.x, sidx = blockIdx.y;
  if (j >= a.offs[a.L]) return;
  const int l = a.sample_model[j];
  const int seg = a.seg_first + sidx;
  const int n_local = j - a.offs[l];
  const unsigned step = a.steps ? (unsigned)(a.steps[l] + a.step_add) : 0u;
  const int pass_id = a.pass_of_seg[sidx];
  const long long base = ((long long)seg * a.seg_samples + j) * a.HW * a.Cpad;
  T* x = static_cast<T*>(a.x) + base;
  const float* bias = a.bias ? a.bias + (long long)l * a.pstride : nullptr;
  if (a.thr > 0 && (a.HW & 3) == 0) {
    // A thread takes four consecutive pixels of a channel: consecutive element indices, one generator evaluation.  With an even
    // number of channels it takes two of them, in accesses of two elements (one at a time, the step of 100 such pairs takes 9465 us against 9380).
    const auto groups = [&](auto width) __attribute__((always_inline)) {
      constexpr int W = decltype(width)::value;
      struct alignas(W * sizeof(T)) Group { T v[W]; };
      const int CG = a.C / W, total = (a.HW >> 2) * CG;
      const int dp = 256 / CG, dc = 256 - dp * CG;       // (pixel, channel) carried along instead of divided out
      int pix = (int)threadIdx.x / CG, c = (int)threadIdx.x - pix * CG;      // groups of four pixels, of W channels
      for (int t = threadIdx.x; t < total; t += 256, pix += dp, c += dc) {
        if (c >= CG) { c -= CG; ++pix; }
        Group* const at = reinterpret_cast<Group*>(x + pix * 4 * a.Cpad + W * c);
        const int row = a.Cpad / W;                      // Cpad is a multiple of 64
        Group in[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) in[k] = at[k * row];
        unsigned w[W][4];
#pragma unroll
        for (int q = 0; q < W; ++q) dropout_words(a, l, ((unsigned long long)n_local * a.C + W * c + q) * a.HW + pix * 4, pass_id, step, w[q]);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
#pragma unroll
          for (int q = 0; q < W; ++q) {
            const float v = point_value<T>(a, to_float(in[k].v[q]), bias, W * c + q);
            in[k].v[q] = (w[q][k] >> 8) >= a.thr ? kept_nonzero(from_float<T>(v * a.scale)) : from_float<T>(0.f);
          }
          at[k * row] = in[k];
        }
      }
    };
    if ((a.C & 1) == 0) groups(std::integral_constant<int, 2>{});
    else groups(std::integral_constant<int, 1>{});
    return;
  }
  const int dp = 256 / a.C, dc = 256 - dp * a.C;
  int pix = (int)threadIdx.x / a.C, c = (int)threadIdx.x - pix * a.C;
  const int total = a.HW * a.C;
  for (int t = threadIdx.x; t < total; t += 256, pix += dp, c += dc) {
    if (c >= a.C) { c -= a.C; ++pix; }
    const int o = pix * a.Cpad + c;
    T v = from_float<T>(point_value<T>(a, to_float(x[o]), bias, c));
    if (a.thr > 0) {
      const unsigned long long lin = ((unsigned long long)n_local * a.C + c) * a.HW + pix;
      unsigned w[4];
      dropout_words(a, l, lin, pass_id, step, w);
      const unsigned sel = (unsigned)lin & 3u;
      const unsigned wd = sel == 0 ? w[0] : (sel == 1 ? w[1] : (sel == 2 ? w[2] : w[3]));
      v = (wd >> 8) >= a.thr ? kept_nonzero(from_float<T>(point_value<T>(a, to_float(x[o]), bias, c) * a.scale)) : from_float<T>(0.f);
    }
    x[o] = v;
  }
}
template <typename T> void launch_point_fwd(const PointArgs& a, hipStream_t st) {
  if (a.n == 0 || a.nseg == 0) return;
  hipLaunchKernelGGL((point_kernel<T>), dim3((unsigned)a.n, (unsigned)a.nseg), dim3(256), 0, st, a);
}
template void launch_point_fwd<float>(const PointArgs&, hipStream_t);
template void launch_point_fwd<bf16_t>(const PointArgs&, hipStream_t);

// Rows of (segment, model): samples offs[l] .. offs[l+1] of segment seg, HW rows each, Cpad channels per row.
// Block = PS_CH channels of one (segment,) model: PS_CH / EPV channel lanes of 16 bytes x NTH * EPV / PS_CH row lanes; every row
// lane adds its rows (rl, rl + RL, ...) in order, then the lanes are added in order, a few to a thread and then these sums --
// whole 16-byte loads of 64 or 128 contiguous bytes per row instead of one element per thread.
// What bounds it is how many rows a block has on their way: a model's rows belong to one block (its sums do not depend on other models'
// samples then), a hundred models of 64 channels are 200 blocks, and with 256 threads they left most of the chip's loads unused.
// 64 rows of a sample, a hundred models of 64 samples in bf16, us with 256 and with 1024 threads: column sums (two segments) 68 and 27, statistics (one
// segment) 55 and 25; 16 rows 20 and 11, 14 and 10.  Statistics of 4 rows: 7.5 and 11, so 256 threads there; column sums of 4 rows: 6.9 and 7.8,
// but for one model of 150 samples 8.0 and 7.2, of 1000 samples 26 and 21, for eight of 100 7.7 and 6.1, so 1024.  (Statistics that kept a lane's
// first sixteen rows in registers between the passes: 62 registers spilled, 73 us for 61.)
// One row a sample (G's linear layer, whose 8192 columns are blocks enough): 256 threads.  The number follows from the layer's shape alone.
constexpr int PS_CH = 32;                     // channels per block
template <typename T> struct PsVec { static constexpr int N = 16 / (int)sizeof(T); };
template <typename T> __device__ inline void ps_load(const T* p, float (&v)[PsVec<T>::N]) {
  const uint4 t = *reinterpret_cast<const uint4*>(p);
  if constexpr (sizeof(T) == 2) {
    v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
    v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
    v[4] = __uint_as_float(t.z << 16); v[5] = __uint_as_float(t.z & 0xffff0000u);
    v[6] = __uint_as_float(t.w << 16); v[7] = __uint_as_float(t.w & 0xffff0000u);
  } else {
    v[0] = __uint_as_float(t.x); v[1] = __uint_as_float(t.y); v[2] = __uint_as_float(t.z); v[3] = __uint_as_float(t.w);
  }
}
// sum over the row lanes, in lane order, of every lane's EPV values; result for channel cx (< PS_CH) in the threads
// with threadIdx.x < PS_CH
template <int NTH, int EPV>
__device__ inline float ps_lanes_sum(const float (&v)[EPV], float* sh, int cl, int rl) {
  constexpr int PER = EPV, GROUPS = NTH / PS_CH;     // NTH * EPV / PS_CH lanes: PER of them to each group of threads
  __syncthreads();                                   // the buffer's previous use is over
#pragma unroll
  for (int e = 0; e < EPV; ++e) sh[rl * PS_CH + cl * EPV + e] = v[e];
  __syncthreads();
  const int c = (int)threadIdx.x % PS_CH, g = (int)threadIdx.x / PS_CH;
  float s = 0.f;
#pragma unroll
  for (int k = 0; k < PER; ++k) s += sh[(g * PER + k) * PS_CH + c];
  sh[g * PER * PS_CH + c] = s;                       // (this thread alone reads and writes the group's lanes of its channel)
  __syncthreads();
  s = 0.f;
  if ((int)threadIdx.x < PS_CH)
    for (int k = 0; k < GROUPS; ++k) s += sh[k * PER * PS_CH + threadIdx.x];
  return s;
}

// dbias[l][c] = sum over the segments and rows of g (the segments are added in order inside the block)
template <typename T, int NTH>
__global__ __launch_bounds__(NTH) void col_sum_kernel(PointArgs a, float* __restrict__ out, long long out_stride) {
  constexpr int EPV = PsVec<T>::N, CG = PS_CH / EPV, RL = NTH / CG;
  __shared__ float sh[RL * PS_CH];
  const int cl = threadIdx.x % CG, rl = threadIdx.x / CG;
  const int cblocks = (a.C + PS_CH - 1) / PS_CH;     // (padded channels have no bias)
  const int c0 = (blockIdx.x % cblocks) * PS_CH;
  const int l = blockIdx.x / cblocks;
  const int cnt = a.offs[l + 1] - a.offs[l];
  if (cnt == 0) return;
  const long long rows = (long long)cnt * a.HW;
  const bool live = c0 + cl * EPV < a.Cpad;          // Cpad is a multiple of 8: a 16-byte group is inside or outside
  float tot = 0.f;
  for (int s = 0; s < a.nseg; ++s) {
    const T* g = static_cast<const T*>(a.x) + ((long long)(a.seg_first + s) * a.seg_samples + a.offs[l]) * a.HW * a.Cpad + c0 + cl * EPV;
    float acc[EPV];
#pragma unroll
    for (int e = 0; e < EPV; ++e) acc[e] = 0.f;
    if (live)
#pragma unroll 4
      for (long long r = rl; r < rows; r += RL) {
        float v[EPV];
        ps_load<T>(g + r * a.Cpad, v);
#pragma unroll
        for (int e = 0; e < EPV; ++e) acc[e] += v[e];
      }
    tot += ps_lanes_sum<NTH, EPV>(acc, sh, cl, rl);
  }
  const int c = c0 + (int)threadIdx.x;
  if ((int)threadIdx.x < PS_CH && c < a.C) out[(long long)l * out_stride + c] = tot;
}
template <typename T> void launch_col_sum(const PointArgs& a, float* out, long long out_stride, hipStream_t st) {
  if (a.nseg == 0 || a.L == 0 || a.C == 0) return;
  if (a.Cpad % 8 != 0) return launch_fail("column sums: the channel count of a row must be a multiple of 8");
  const dim3 grid((unsigned)(a.L * ((a.C + PS_CH - 1) / PS_CH)));
  if (a.HW > 1) hipLaunchKernelGGL((col_sum_kernel<T, 1024>), grid, dim3(1024), 0, st, a, out, out_stride);
  else hipLaunchKernelGGL((col_sum_kernel<T, 256>), grid, dim3(256), 0, st, a, out, out_stride);
}
template void launch_col_sum<float>(const PointArgs&, float*, long long, hipStream_t);
template void launch_col_sum<bf16_t>(const PointArgs&, float*, long long, hipStream_t);

// Batch statistics of a stored tensor per (segment, model, channel): mean, biased variance (from the deviations, second
// pass), 1 / sqrt(var + eps); written where the BatchNorm passes expect them ([(segment) * L + model][C]).
// Of channels from `real` on, which are padding and hold zeros, nothing is read.
template <typename T, int NTH>
__global__ __launch_bounds__(NTH) void bn_stats_direct_kernel(NormArgs a, int real) {
  constexpr int EPV = PsVec<T>::N, CG = PS_CH / EPV, RL = NTH / CG;
  __shared__ float sh[RL * PS_CH];
  __shared__ float mean_sh[PS_CH];
  const int cl = threadIdx.x % CG, rl = threadIdx.x / CG;
  const int cblocks = (a.C + PS_CH - 1) / PS_CH;
  const int c0 = (blockIdx.x % cblocks) * PS_CH;
  const int l = (blockIdx.x / cblocks) % a.L;
  const int sidx = blockIdx.x / (cblocks * a.L);
  const int cnt = a.offs[l + 1] - a.offs[l];
  if (cnt == 0) return;
  const long long all = (long long)cnt * a.rps, rows = c0 + cl * EPV < real ? all : 0;       // of the model; those this lane has a part of
  const T* x = static_cast<const T*>(a.x) + ((long long)(a.seg_first + sidx) * a.seg_samples + a.offs[l]) * a.rps * a.C + c0 + cl * EPV;
  float acc[EPV], mean[EPV], v[EPV];
#pragma unroll
  for (int e = 0; e < EPV; ++e) acc[e] = 0.f;
#pragma unroll 4
  for (long long r = rl; r < rows; r += RL) {
    ps_load<T>(x + r * a.C, v);
#pragma unroll
    for (int e = 0; e < EPV; ++e) acc[e] += v[e];
  }
  const float s1 = ps_lanes_sum<NTH, EPV>(acc, sh, cl, rl);
  if ((int)threadIdx.x < PS_CH) mean_sh[threadIdx.x] = s1 / (float)all;
  __syncthreads();
#pragma unroll
  for (int e = 0; e < EPV; ++e) { mean[e] = mean_sh[cl * EPV + e]; acc[e] = 0.f; }
#pragma unroll 4
  for (long long r = rl; r < rows; r += RL) {
    ps_load<T>(x + r * a.C, v);
#pragma unroll
    for (int e = 0; e < EPV; ++e) { const float d = v[e] - mean[e]; acc[e] += d * d; }
  }
  const float s2 = ps_lanes_sum<NTH, EPV>(acc, sh, cl, rl);
  const int c = c0 + (int)threadIdx.x;
  if ((int)threadIdx.x < PS_CH && c < a.C) {
    const float var = s2 / (float)all;
    const long long o = (long long)((a.seg_first + sidx) * a.L + l) * a.C + c;
    a.mean[o] = mean_sh[threadIdx.x];
    a.var[o] = var;
    a.rstd[o] = 1.0f / sqrtf(var + a.eps);
  }
}
template <typename T> void launch_bn_stats_direct(const NormArgs& a, int real, hipStream_t st) {
  const long long tot = (long long)a.nseg * a.L * ((a.C + PS_CH - 1) / PS_CH);
  if (tot == 0) return;
  if (a.C % 8 != 0) return launch_fail("batch statistics: the channel count of a row must be a multiple of 8");
  if (a.rps >= 16) hipLaunchKernelGGL((bn_stats_direct_kernel<T, 1024>), dim3((unsigned)tot), dim3(1024), 0, st, a, real);
  else hipLaunchKernelGGL((bn_stats_direct_kernel<T, 256>), dim3((unsigned)tot), dim3(256), 0, st, a, real);
}
template void launch_bn_stats_direct<float>(const NormArgs&, int, hipStream_t);
template void launch_bn_stats_direct<bf16_t>(const NormArgs&, int, hipStream_t);

}  // namespace gan
