// The strided convolutions that read an image of 1..4 channels: D's first layer, and the gradients of G's last transposed
// convolution, whose output gradient is such an image.  k4 s2 p1, Cs = 64 or 128 feature channels.
//   out[pixel][cs]  = act(sum over (tap, c) of patch(pixel)[tap][c] * w[tap][c][cs] + add[position class][cs])
//   dw[tap][c][cs]  = sum over pixels of patch(pixel)[tap][c] * dy[pixel][cs]
// Both are contractions over 16 taps of a few channels, bound by the feature tensor that they write or read once.  No patch matrix
// exists: an image tile lies in LDS with P = 2, 4 or 8 values a pixel (the channels, a one inside the image, zeros), and the operand reads
// pick the patches out of it.  Forward: a lane's eight values of K are neighbouring pixels of a tile row, 16 bytes.  Weight gradient: the
// transposing LDS read takes an address of 8 bytes per lane, so that its rows are pixels and its columns the (tap, channel) of the patch.
//
// A one-hot label map is a constant plane.  Forward, it and the bias are a row per position class (3 x 3: which taps lie outside), from which
// the accumulators start.  Its gradient is that of the ones inside the image, and the bias's is the same at a tap that is never outside.
// One pair over many labels takes its label maps' gradients from class sums instead (launch_class_sums).
//
// fp32 storage: the tile, the weights and dy are split into three bf16 parts (split_mfma.h).
//
// What it replaced: patch matrices in memory, written by one kernel and read as the operand of a row-by-row GEMM and weight gradient.  us, before
// -> now.  A hundred 32x32 pairs of 64 samples, 128 channels, bf16: both segments 388 -> 217 (now 4.4 TB/s of the 0.96 GB that have to move; 179
// without the image's loads, 107 without the stores), one 129 -> 112, their weight gradients 320 -> 258 and 243 -> 106, which now includes the bias;
// eight 64x64 pairs, 64 channels, 191 -> 88, 51 -> 40, 112 -> 79, 122 -> 44; twenty 32x32 pairs in fp32 184 -> 108, 68 -> 55, 144 -> 133, 105 -> 74; ten
// 28x28 pairs in fp32 93 -> 45, 31 -> 25, 69 -> 51, 62 -> 29.  Whole steps: +10 % (ten 28x28 pairs, bf16) to +2 % (twenty 32x32 pairs, fp32).
#include <algorithm>

#include "image_walk.h"
#include "kernels.h"
#include "lds_copy.h"
#include "split_mfma.h"

namespace gan {

namespace {

constexpr int conv_side_y(int esize) { return esize == 4 ? 8 : 16; }      // outputs along y of a unit, forward (weight gradient: WG_SIDE_Y)
constexpr int ZERO_ROWS = 4;                 // behind the weight gradient's tiles: what pixels outside the map read

// one pixel of the tile: P values, fp32 in three planes `plane` bytes apart
template <typename T, int CB>
__device__ __forceinline__ void put_pixel(unsigned char* at, int plane, const float (&v)[CB], bool in) {
  constexpr int P = img_values(CB);
  float f[P];
#pragma unroll
  for (int i = 0; i < P; ++i) f[i] = i < CB ? v[i] : (i == CB && in ? 1.f : 0.f);
  unsigned q[sizeof(T) == 4 ? 3 : 1][P / 2];
#pragma unroll
  for (int i = 0; i < P / 2; ++i) {
    if constexpr (sizeof(T) == 4) split_pair(f[2 * i], f[2 * i + 1], q[0][i], q[1][i], q[2][i]);
    else q[0][i] = pack2_bf16(f[2 * i], f[2 * i + 1]);
  }
#pragma unroll
  for (int pl = 0; pl < (sizeof(T) == 4 ? 3 : 1); ++pl) {
    unsigned char* const d = at + pl * plane;
    if constexpr (P == 2) *reinterpret_cast<unsigned*>(d) = q[pl][0];
    else if constexpr (P == 4) *reinterpret_cast<uint2*>(d) = make_uint2(q[pl][0], q[pl][1]);
    else *reinterpret_cast<uint4*>(d) = make_uint4(q[pl][0], q[pl][1], q[pl][2], q[pl][3]);
  }
}
// The image under the outputs (y0 .., x0 ..) of a unit: tile pixel (ty, tx) is image pixel (2 y0 - 1 + ty, 2 x0 - 1 + tx), zeros outside.  A thread's
// U pairs of neighbouring pixels are all on their way together (no branch and no conversion between the loads, either of which would wait for
// them), and the tile is written later (put).  own: put also adds up the pixels of the unit's own 2 ph x 2 pw.
template <typename T, int CB, int U>
struct Stager {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  u2 v[U][CB];                                                 // as loaded.  NCHW: channel c of both pixels in v[c]; NHWC: the pair's 2 CB values in a row
  unsigned in;                                                 // bit k: pair k lies inside the image
  bool nchw;
  template <typename F>
  static __device__ __forceinline__ void pairs(const Units& u, int tid, int nt, F&& f) {
    const int per = u.pw + 2, total = (2 * u.ph + 2) * per;
    const float inv = 1.f / (float)per;
    static_for<0, U>([&](auto k) __attribute__((always_inline)) {
      const int q = tid + k.value * nt, ty = (int)(((float)q + 0.5f) * inv);       // (exact: q < 1024)
      f(k, ty, q - ty * per - 1, q < total);
    });
  }
  __device__ __forceinline__ void fetch(const Units& u, const T* img, const float* real, int Hb, int y0, int x0, int tid, int nt) {
    in = 0;
    nchw = img == nullptr;
    const int npix = Hb * Hb;
    const __amdgpu_buffer_rsrc_t rs = buffer_of(nchw ? (const void*)real : (const void*)img, (unsigned)npix * CB * (nchw ? 4u : (unsigned)sizeof(T)));
    const unsigned pixel = nchw ? 4u : (unsigned)sizeof(T) * CB, step = nchw ? 4u * npix : 8u;      // bytes
    pairs(u, tid, nt, [&](auto k, int ty, int pr, bool there) __attribute__((always_inline)) {
      const int iy = 2 * y0 - 1 + ty, ix = 2 * (x0 + pr);
      const bool inside = there && (unsigned)iy < (unsigned)Hb && (unsigned)ix < (unsigned)Hb;
      in |= inside ? 1u << k.value : 0u;
      const unsigned at = (unsigned)(iy * Hb + ix) * pixel;
      static_for<0, CB>([&](auto c) __attribute__((always_inline)) {
        const bool needed = sizeof(T) == 4 || nchw || 2 * c.value < CB;      // (bf16 NHWC: CB words)
        v[k.value][c.value] = __builtin_amdgcn_raw_buffer_load_b64(rs, inside && needed ? at + c.value * step : NO_ROW, 0, 0);
      });
    });
  }
  template <int P, int C, int K> __device__ __forceinline__ float value() const {      // channel C of pixel P of pair K
    constexpr int e = P * CB + C;
    if constexpr (sizeof(T) == 2) {
      const unsigned w = v[K][e / 4][e / 2 % 2], half = e & 1 ? w & 0xffff0000u : w << 16;
      return __uint_as_float(nchw ? v[K][C][P] : half);
    } else {
      return __uint_as_float(nchw ? v[K][C][P] : v[K][e / 2][e % 2]);
    }
  }
  __device__ __forceinline__ void put(unsigned char* tile, int plane, const Units& u, int tid, int nt, double (*own)[CB]) const {
    float sum[CB] = {};                                        // of the unit
    constexpr int PB = 2 * img_values(CB);
    pairs(u, tid, nt, [&](auto k, int ty, int pr, bool there) __attribute__((always_inline)) {
      unsigned char* const at = tile + ty * u.pitch + (2 * pr + 1) * PB;
      const bool inside = (in >> k.value) & 1;
      float a[CB], b[CB];
      static_for<0, CB>([&](auto c) __attribute__((always_inline)) {
        a[c.value] = value<0, c.value, k.value>();
        b[c.value] = value<1, c.value, k.value>();
      });
      if (there && pr >= 0) put_pixel<T, CB>(at, plane, a, inside);
      if (there && pr < u.pw) put_pixel<T, CB>(at + PB, plane, b, inside);
      if (own) {
        const bool mine = there && ty > 0 && ty <= 2 * u.ph && pr >= 0 && pr < u.pw;
        static_for<0, CB>([&](auto c) __attribute__((always_inline)) { sum[c.value] += mine ? a[c.value] + b[c.value] : 0.f; });
      }
    });
    if (own) static_for<0, CB>([&](auto c) __attribute__((always_inline)) { (*own)[c.value] += (double)sum[c.value]; });
  }
};
// pairs of the largest unit
constexpr int unit_pairs(int side_y) { return (2 * side_y + 2) * (IMG_SIDE + 2); }

__device__ inline bool any_not_finite(const floatx16& a) {
  float z = 0.f;
#pragma unroll
  for (int e = 0; e < 16; ++e) z = __builtin_fmaf(a[e], 0.f, z);
  return __ballot(z != z) != 0;
}

// The value of patch column m = tap * P + c at output pixel (y, x), from memory
template <typename T, int CB>
__device__ inline float patch_value(const T* img, const float* real, int Hb, int y, int x, int m) {
  constexpr int P = img_values(CB);
  const int tap = m / P, c = m - tap * P, iy = 2 * y - 1 + (tap >> 2), ix = 2 * x - 1 + (tap & 3);
  if (c > CB || (unsigned)iy >= (unsigned)Hb || (unsigned)ix >= (unsigned)Hb) return 0.f;
  if (c == CB) return 1.f;
  return img ? to_float(img[((long long)iy * Hb + ix) * CB + c]) : real[((long long)c * Hb + iy) * Hb + ix];
}

// ---------------------------------------------------------------------------------------------------------
// Forward: a block per (unit, sample, segment), bound by its stores.  A wave owns 128 bytes of channels (64 in bf16, 32 in fp32), whose weights stay in its registers, and
// multiplies them with 32 pixels at a time; the result's columns are pixels, so that a lane has 16 channels of its pixel from every product.  They
// go through a patch of LDS of the wave's own, so that a store writes whole 128-byte lines of eight pixels (16 bytes a lane straight from the
// registers, 32 or 64 in a row: 294 and 265 us for 217; past the caches 302).
// ---------------------------------------------------------------------------------------------------------
constexpr int OUT_ROW = 128 + 16;            // bytes of a pixel in the patch
template <typename T, int CB, int CS>
__global__ __launch_bounds__(256) void image_conv_kernel(ImageConvArgs a, Units u) {
  constexpr int P = img_values(CB), PB = 2 * P, KS = P, PL = sizeof(T) == 4 ? 3 : 1;
  constexpr int NB = PL == 1 ? 2 : 1, GROUPS = CS / (32 * NB), TURNS = 4 / GROUPS;      // blocks of 32 channels a wave, waves across the channels, and along the pixels
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int per_sample = u.nx * u.ny, j = (int)blockIdx.x / per_sample, unit = (int)blockIdx.x - j * per_sample;
  if (j >= a.offs[a.L]) return;
  const int l = a.sample_model[j], seg = a.seg_first + (int)blockIdx.y;
  const int Hs = a.Hs, Hb = 2 * Hs, plane = (2 * u.ph + 2) * u.pitch;
  const int uy = unit / u.nx, y0 = uy * u.ph, x0 = (unit - uy * u.nx) * u.pw;
  const int ph = min(u.ph, Hs - y0), pw = min(u.pw, Hs - x0), px = ph * pw;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, h = lane >> 5, cg = wave % GROUPS, c0 = cg * 32 * NB;
  const bool nchw = a.real && seg == 0;
  const T* img = nchw ? nullptr : static_cast<const T*>(a.img) + ((long long)seg * a.seg_samples + j) * Hb * Hb * CB;
  const float* real = nchw ? a.real + (long long)a.perm[j] * CB * Hb * Hb : nullptr;
  Stager<T, CB, (unit_pairs(conv_side_y((int)sizeof(T))) + 255) / 256> image;
  image.fetch(u, img, real, Hb, y0, x0, tid, 256);
  // this lane's row of weights: channel 8 h' + e of the first sixteen, of the second, so that the results come out eight channels at a time
  const int e_ = (r >> 3) * 4 + (r & 3), ch = (e_ >> 3) * 16 + ((r >> 2) & 1) * 8 + (e_ & 7);
  u32x4 w[NB][PL][KS];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const T* wr = static_cast<const T*>(a.w) + ((long long)l * CS + c0 + 32 * b + ch) * 16 * P + 8 * h;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const u32x4* q = reinterpret_cast<const u32x4*>(wr + 16 * s);
      if constexpr (PL == 3) {
        const Split8 t = split8(q[0], q[1]);
        w[b][0][s] = t.h; w[b][1][s] = t.m; w[b][2][s] = t.l;
      } else {
        w[b][0][s] = q[0];
      }
    }
  }
  float* const add = reinterpret_cast<float*>(lds + PL * plane);
  unsigned char* const patch = lds + PL * plane + 9 * CS * 4 + wave * (32 * OUT_ROW);
  {
    const float4* src = a.add ? reinterpret_cast<const float4*>(a.add + (long long)(a.sample_slot ? a.sample_slot[j] : l) * 9 * CS) : nullptr;
    const float4* bias = a.bias ? reinterpret_cast<const float4*>(a.bias + l * a.bias_stride) : nullptr;
    const auto in_t = [](float x) { return to_float(from_float<T>(x)); };
    for (int i = tid; i < 9 * CS / 4; i += 256) {
      float4 t = src ? src[i] : make_float4(0.f, 0.f, 0.f, 0.f);
      const float4 q = bias ? bias[i % (CS / 4)] : make_float4(0.f, 0.f, 0.f, 0.f);
      t.x += in_t(q.x); t.y += in_t(q.y); t.z += in_t(q.z); t.w += in_t(q.w);
      reinterpret_cast<float4*>(add)[i] = t;
    }
  }
  image.put(lds, plane, u, tid, 256, nullptr);
  __syncthreads();
  // K-step s, lane half h: pixels of the patch row ky = s (P = 4: columns 2 h, 2 h + 1), 2 s + h (P = 2: all four) or s / 2 (P = 8: column 2 (s % 2) + h)
  const int hoff = P == 2 ? h * u.pitch : (P == 4 ? 2 * h * PB : h * PB);
  T* const out = static_cast<T*>(a.out) + ((long long)seg * a.seg_samples + j) * Hs * Hs * CS + c0;
  const float inv_pw = 1.f / (float)pw;
  const auto row_of = [&](int q) __attribute__((always_inline)) { return (int)(((float)q + 0.5f) * inv_pw); };      // (exact: at most 16 x 16 pixels)
  for (int p0 = wave / GROUPS * 32; p0 < px; p0 += TURNS * 32) {
    const int pc = min(p0 + r, px - 1), yl = row_of(pc), xl = pc - yl * pw, y = y0 + yl, x = x0 + xl;
    const unsigned char* const q = lds + 2 * yl * u.pitch + 2 * xl * PB + hoff;
    const float* const ad = add + pos_class(y, x, Hs) * CS + c0 + h * 8;
    floatx16 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int e = 0; e < 16; e += 4) {
        const float4 t = *reinterpret_cast<const float4*>(ad + 32 * b + (e >> 3) * 16 + (e & 7));
        acc[b][e] = t.x; acc[b][e + 1] = t.y; acc[b][e + 2] = t.z; acc[b][e + 3] = t.w;
      }
    const auto pixels = [&](int s, int pl) __attribute__((always_inline)) {
      const unsigned char* const at = q + pl * plane + (P == 2 ? 2 * s * u.pitch : (P == 4 ? s * u.pitch : (s >> 1) * u.pitch + (s & 1) * 2 * PB));
      if constexpr (P == 2) {                          // 8-byte aligned
        const uint2 lo = *reinterpret_cast<const uint2*>(at), hi = *reinterpret_cast<const uint2*>(at + 8);
        return u32x4{lo.x, lo.y, hi.x, hi.y};
      } else {
        return *reinterpret_cast<const u32x4*>(at);
      }
    };
    if constexpr (PL == 1) {
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const u32x4 f = pixels(s, 0);
#pragma unroll
        for (int b = 0; b < NB; ++b) mma_u4(acc[b], w[b][0][s], f);
      }
    } else {
      floatx16 sum, low = {};                          // (what is added comes first: rounded with the products instead of once more behind them)
#pragma unroll
      for (int e = 0; e < 16; ++e) sum[e] = acc[0][e] * (1.f / SPLIT_UNSCALE);
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const u32x4 fh = pixels(s, 0), fm = pixels(s, 1), fl = pixels(s, 2);
        mma_u4(low, w[0][2][s], fh);
        mma_u4(sum, w[0][0][s], fh);
        mma_u4(low, w[0][0][s], fl);
        mma_u4(low, w[0][1][s], fm);
        mma_u4(low, w[0][1][s], fh);
        mma_u4(low, w[0][0][s], fm);
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) sum[e] = (sum[e] + low[e]) * SPLIT_UNSCALE;
      if (any_not_finite(sum)) {                       // what has no split: these 32 pixels again, value by value
        const T* w0 = static_cast<const T*>(a.w) + ((long long)l * CS + c0 + h * 8) * 16 * P;
        sum = acc[0];
        for (int m = 0; m < 16 * P; ++m) {
          if (m % P >= CB) continue;
          const float v = patch_value<T, CB>(img, real, Hb, y, x, m);
#pragma unroll
          for (int e = 0; e < 16; ++e) sum[e] = __builtin_fmaf(v, to_float(w0[((e >> 3) * 16 + (e & 7)) * 16 * P + m]), sum[e]);
        }
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[0][e] = sum[e];
    }
    // into the patch: pixel r, channels 32 b + 16 g + 8 h .. + 7
#pragma unroll
    for (int b = 0; b < NB; ++b) {
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[b][e] = acc[b][e] > 0.f ? acc[b][e] : acc[b][e] * a.slope;
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        unsigned char* const d = patch + r * OUT_ROW + (32 * b + 16 * g + 8 * h) * (int)sizeof(T);
        if constexpr (PL == 1) {
          *reinterpret_cast<u32x4*>(d) = u32x4{pack2_bf16(acc[b][8 * g], acc[b][8 * g + 1]), pack2_bf16(acc[b][8 * g + 2], acc[b][8 * g + 3]),
                                               pack2_bf16(acc[b][8 * g + 4], acc[b][8 * g + 5]), pack2_bf16(acc[b][8 * g + 6], acc[b][8 * g + 7])};
        } else {
#pragma unroll
          for (int k = 0; k < 8; k += 4)
            *reinterpret_cast<float4*>(d + 4 * k) = make_float4(acc[b][8 * g + k], acc[b][8 * g + k + 1], acc[b][8 * g + k + 2], acc[b][8 * g + k + 3]);
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 8 * i + (lane >> 3), pg = p0 + row, yg = row_of(pg);
      const u32x4 v = *reinterpret_cast<const u32x4*>(patch + row * OUT_ROW + (lane & 7) * 16);
      if (pg < px) *reinterpret_cast<u32x4*>(out + ((y0 + yg) * Hs + x0 + pg - yg * pw) * CS + (lane & 7) * (16 / (int)sizeof(T))) = v;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}
template <typename T, int CB, int CS>
void conv_one(const ImageConvArgs& a, hipStream_t st) {
  const Units u = img_units(a.Hs, CB, conv_side_y((int)sizeof(T)));
  const size_t lds = (size_t)(sizeof(T) == 4 ? 3 : 1) * (2 * u.ph + 2) * u.pitch + 9 * CS * 4 + 4 * 32 * OUT_ROW;
  if (lds > 48 * 1024)   // above the default dynamic limit: ask for it (idempotent, cheap)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&image_conv_kernel<T, CB, CS>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  const long long blocks = (long long)a.n * u.nx * u.ny;
  if (blocks >= (1LL << 31)) return launch_fail("image-side convolution: more blocks than a launch can have");
  hipLaunchKernelGGL((image_conv_kernel<T, CB, CS>), dim3((unsigned)blocks, (unsigned)a.nseg), dim3(256), lds, st, a, u);
}

// ---------------------------------------------------------------------------------------------------------
// Weight gradient: a block takes the samples of one tile of a model (both segments), unit by unit, and leaves partial sums; what adds them
// follows below.  Four waves multiply, each its own 32 feature channels (64 of them: two waves share 32, a K-step of 16 pixels each in turn), so
// that dy needs no barrier: its pixels come into the wave's own ring of LDS (fp32: of registers) K-steps ahead.  A fifth wave stages the next
// unit's image tile meanwhile.
// ---------------------------------------------------------------------------------------------------------
constexpr int wg_ring(int esize) { return esize == 4 ? 3 : 6; }      // K-steps of dy on their way, a wave (bf16: 1 KiB each, fp32: 2)
constexpr int WG_THREADS = 320;
// K-steps (16 pixels) whose products a wave's accumulators add up before they go to sums in memory.  An accumulator that takes a tile's pixels in one chain
// rounds each against all in front of it, and the chains of large tiles were longer than the row splits in whose place the tiles came.  Error against 64-bit sums, one
// chain -> these: twenty 32x32 pairs of 64 samples in fp32 2.2e-7 -> 1.5e-7, a hundred in bf16 4.2e-7 -> 2.9e-7 (the row splits: 0.9 of one chain's).  Both
// weight gradients of a step 195 -> 205 and 350 -> 363 us; with fp32 chains of 15 1.0e-7 and 224 us, with a second set of registers for the sums 0.96e-7
// and, of ten 28x28 pairs, 125 us for 78.
constexpr int wg_chain(int esize) { return esize == 4 ? 48 : 162; }

// EVEN: even_units; every lane's addresses are then its own constants and wave-uniform offsets.  (Registers: held to what the
// launches had without the sums in memory; D's of a hundred 32x32 pairs in bf16 with four waves a SIMD 284 us, with five 257.)
template <typename T, int CB, int CS, bool EVEN>
__global__ __launch_bounds__(WG_THREADS, (CB == 4 ? 1 : sizeof(T) == 2 ? (EVEN ? 5 : 4) : CB == 1 ? 4 : 3)) void image_wgrad_kernel(ImageWgradArgs a, Units u) {
  constexpr int P = img_values(CB), PB = 2 * P, NC = CS / 32, TURNS = 4 / NC, MF = P == 2 ? 1 : P / 2, PL = sizeof(T) == 4 ? 3 : 1;
  constexpr int WG_RING = wg_ring((int)sizeof(T));
  constexpr int RING_BYTES = PL == 1 ? WG_RING * 1024 : 3 * 1024;      // of a wave
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
  const int tile = blockIdx.x;
  if (tile >= a.tpre[a.L]) return;
  const int l = a.tmodel ? a.tmodel[tile] : 0;
  const int per_tile = image_tile(a.tiles, a.offs[l + 1] - a.offs[l]), j0 = a.offs[l] + (tile - a.tpre[l]) * per_tile, j1 = min(a.offs[l + 1], j0 + per_tile);
  const int Hs = a.Hs, Hb = 2 * Hs, npix = Hb * Hb;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int trows = 2 * u.ph + 2, plane = (trows + ZERO_ROWS) * u.pitch, buf = PL * plane;
  unsigned char* const tiles = lds + 4 * RING_BYTES;                   // two
  const UnitAt first = {a.seg_first, j0, 0, 0};
  double own[CB] = {};                                                   // (in fp32 a tile's pixels are chains of hundreds)
  Stager<T, CB, (unit_pairs(WG_SIDE_Y) + 63) / 64> image;
  UnitAt ahead = first;
  int place = a.real ? a.perm[j0] : 0;                                   // of the sample `ahead`, known a unit before it is needed
  const auto fetch = [&]() __attribute__((always_inline)) {
    const bool nchw = a.real && ahead.seg == 0;
    image.fetch(u, nchw ? nullptr : static_cast<const T*>(a.img) + ((long long)ahead.seg * a.seg_samples + ahead.j) * npix * CB,
                nchw ? a.real + (long long)place * CB * npix : nullptr, Hb, ahead.y0, ahead.x0, lane, 64);
    next_unit(ahead, u, Hs, j0, j1);
    if (a.real) place = a.perm[ahead.j];
  };
  const auto put = [&](int i) __attribute__((always_inline)) { image.put(tiles + (i & 1) * buf, plane, u, lane, 64, a.pixel_sums ? &own : nullptr); };
  if (wave == 4) fetch();
  // the rows that pixels outside the map read
  for (int i = tid; i < 2 * PL * ZERO_ROWS * u.pitch / 16; i += WG_THREADS) {
    const int per = ZERO_ROWS * u.pitch / 16, q = i / per;
    *reinterpret_cast<uint4*>(tiles + q * plane + trows * u.pitch + (i - q * per) * 16) = make_uint4(0, 0, 0, 0);
  }

  const int cb = wave % NC, turn = wave / NC % TURNS;
  floatx16 acc[MF] = {}, low[PL == 3 ? MF : 1] = {};
  // ---- dy: lane -> pixel and 16 bytes of this wave's 32 channels, K-steps in the order of the units
  constexpr int LPP = PL == 1 ? 4 : 8, LOADS = PL == 1 ? 1 : 2;        // lanes a pixel, loads a K-step
  int lane_pixel[LOADS];
#pragma unroll
  for (int i = 0; i < LOADS; ++i) lane_pixel[i] = lane / LPP + i * (64 / LPP);
  GradWalk<LOADS, TURNS, EVEN> walk;
  walk.start(u, Hs, first, j1, a.nseg, turn, lane_pixel, CS * (unsigned)sizeof(T), (unsigned)(cb * 32 + lane % LPP * (16 / (int)sizeof(T))) * (unsigned)sizeof(T), wave < 4);
  const int units = walk.units, steps = walk.steps;                    // steps: K-steps of a unit, each of 16 pixels in row order, that this wave takes
  const auto sample_grad = [&]() __attribute__((always_inline)) { return static_cast<const T*>(a.dy) + ((long long)walk.at.seg * a.seg_samples + walk.at.j) * Hs * Hs * CS; };
  const T* dy_sample = sample_grad();
  const unsigned dy_bytes = (unsigned)(Hs * Hs * CS * (int)sizeof(T));
  // ---- operands: lane = 32 kgrp + 16 hb + s reads, for rows 8 kgrp + 4 half + s / 4 of a K-step (pixels), the 8 bytes s % 4 of the 16 columns hb
  const int s16 = lane & 15, hb = (lane >> 4) & 1, kgrp = lane >> 5, frow = 8 * kgrp + (s16 >> 2), sg = s16 & 3;
  // column group 4 hb + sg of fragment t: P = 4: tap (2 t + hb, sg); P = 2: taps (2 hb + sg / 2, 2 (sg % 2) ..); P = 8: half sg % 2 of tap (t, 2 hb + sg / 2)
  const int goff = P == 4 ? hb * u.pitch + sg * PB : (P == 2 ? (2 * hb + (sg >> 1)) * u.pitch + (sg & 1) * 2 * PB : (2 * hb + (sg >> 1)) * PB + (sg & 1) * 8);
  const int tstep = P == 4 ? 2 * u.pitch : u.pitch;
  int py_first[2], px_first[2], py[2], px[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int p = 16 * turn + frow + 4 * i;
    py_first[i] = p / u.pw; px_first[i] = p - py_first[i] * u.pw;
  }
  unsigned char* const ring = lds + wave * RING_BYTES;
  const unsigned ring_lds = (unsigned)(uintptr_t)ring;
  const unsigned char* const bq = ring + frow * 64 + hb * 32 + sg * 8;
  u32x4 v[PL == 3 ? WG_RING : 1][2];
  const auto request = [&](auto slot) __attribute__((always_inline)) {
    if constexpr (PL == 1) {
      load16_to_lds(make_rsrc(dy_sample, walk.live ? dy_bytes : 0), walk.offset(0), walk.uniform, ring_lds + slot.value * 1024);
    } else {
      const __amdgpu_buffer_rsrc_t rs = buffer_of(dy_sample, walk.live ? dy_bytes : 0);
#pragma unroll
      for (int i = 0; i < 2; ++i) v[slot.value][i] = __builtin_amdgcn_raw_buffer_load_b128(rs, walk.offset(i), walk.uniform, 0);
    }
    if (walk.advance()) dy_sample = sample_grad();
  };
  UnitAt cur = first;
  const int even_first = 2 * turn * u.pitch;
  int even_row = even_first;                           // EVEN: tile row of the K-step to multiply, in bytes
  const auto multiply = [&](auto slot, const unsigned char* tb, bool there) __attribute__((always_inline)) {
    u32x4 b[PL], f[MF][PL];
    if constexpr (PL == 1) {
      wait_vm<WG_RING - 1>();
    } else {
      // split into the planes [part][pixel][32 channels], which this wave alone reads and writes
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const Split4 q = split4(v[slot.value][i]);
        unsigned char* const d = ring + (lane / 8 + 8 * i) * 64 + lane % 8 * 8;
        *reinterpret_cast<uint2*>(d) = q.h;
        *reinterpret_cast<uint2*>(d + 1024) = q.m;
        *reinterpret_cast<uint2*>(d + 2048) = q.l;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    const unsigned char* pa[2];
    if constexpr (EVEN) {
#pragma unroll
      for (int i = 0; i < 2; ++i) pa[i] = tb + even_row + 2 * (frow + 4 * i) * PB + goff;
      even_row += 2 * TURNS * u.pitch;
    } else
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const bool ok = py[i] < u.ph && cur.y0 + py[i] < Hs && cur.x0 + px[i] < Hs;
      pa[i] = tb + (ok ? 2 * py[i] * u.pitch + 2 * px[i] * PB : trows * u.pitch) + goff;
      px[i] += walk.dx; py[i] += walk.dy;
      if (px[i] >= u.pw) { px[i] -= u.pw; ++py[i]; }
    }
#pragma unroll
    for (int pl = 0; pl < PL; ++pl) {
      const unsigned char* const q = bq + (PL == 1 ? slot.value * 1024 : pl * 1024);
      const uint2 lo = lds_read_tr16(q), hi = lds_read_tr16(q + 4 * 64);
      b[pl] = u32x4{lo.x, lo.y, hi.x, hi.y};
#pragma unroll
      for (int t = 0; t < MF; ++t) {
        const uint2 p0 = lds_read_tr16(pa[0] + pl * plane + t * tstep), p1 = lds_read_tr16(pa[1] + pl * plane + t * tstep);
        f[t][pl] = u32x4{p0.x, p0.y, p1.x, p1.y};
      }
    }
    if constexpr (PL == 1) {
      __builtin_amdgcn_s_waitcnt(0xc07f);                // lgkmcnt(0): the slot has been read and may be filled again
      asm volatile("" : : : "memory");
      request(slot);
      if (there)
#pragma unroll
        for (int t = 0; t < MF; ++t) mma_u4(acc[t], f[t][0], b[0]);
    } else {
      request(slot);
      if (there)
#pragma unroll
      for (int t = 0; t < MF; ++t) {
        mma_u4(low[t], f[t][2], b[0]);
        mma_u4(acc[t], f[t][0], b[0]);
        mma_u4(low[t], f[t][0], b[2]);
        mma_u4(low[t], f[t][1], b[1]);
        mma_u4(low[t], f[t][1], b[0]);
        mma_u4(low[t], f[t][0], b[1]);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  };
  // ---- what the accumulators have added up goes onto sums of the wave's own in memory and they start at zero again (more), or these are added to them.
  // (its lines are those of the tile's partial sums, as the registers lie, and for the second turn others behind all of those)
  int put_away = 0;                                    // K-steps whose sums lie there
  const auto add_away = [&](auto more) __attribute__((always_inline)) {
    // (addressed from their middle, which immediate offsets reach from; not through a buffer: a store of 16 bytes with a scalar offset is not kept apart from writes
    // to its registers behind it, and lost some)
    float4* const sums = reinterpret_cast<float4*>(a.part + (((long long)turn * gridDim.x + tile) * NC + cb) * (MF * 16 * 64)) + 256 + lane;
    static_for<0, MF>([&](auto t) __attribute__((always_inline)) {
      float4 q[4] = {};
      if (put_away > 0)
#pragma unroll
        for (int k = 0; k < 4; ++k) q[k] = sums[(4 * t.value + k - 4) * 64];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        q[k].x += acc[t.value][4 * k]; q[k].y += acc[t.value][4 * k + 1]; q[k].z += acc[t.value][4 * k + 2]; q[k].w += acc[t.value][4 * k + 3];
        if constexpr (more.value) {
          sums[(4 * t.value + k - 4) * 64] = q[k];
        } else {
          acc[t.value][4 * k] = q[k].x; acc[t.value][4 * k + 1] = q[k].y; acc[t.value][4 * k + 2] = q[k].z; acc[t.value][4 * k + 3] = q[k].w;
        }
      }
      if constexpr (more.value) acc[t.value] = floatx16{};
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  if (wave == 4) {
    put(0);
    if (units > 1) fetch();
    __syncthreads();
    for (int i = 0; i < units; ++i) {
      if (i + 1 < units) put(i + 1);
      if (i + 2 < units) fetch();
      __syncthreads();
    }
  } else {
    static_for<0, WG_RING>([&](auto k) __attribute__((always_inline)) { request(k); });
    __syncthreads();
    int i = 0, s = 0;
#pragma unroll
    for (int k = 0; k < 2; ++k) { py[k] = py_first[k]; px[k] = px_first[k]; }
    // (whole rounds of the ring, whose slots are registers or constant offsets: behind the last unit nothing is multiplied, for which the other tile may never have been written)
    for (int g = 0; g < units * steps; g += WG_RING) {
      if (g - put_away >= wg_chain((int)sizeof(T))) {
        add_away(std::true_type{});
        put_away = g;
      }
      static_for<0, WG_RING>([&](auto k) __attribute__((always_inline)) {
        multiply(k, tiles + (i & 1) * buf, i < units);
        if (++s == steps && i < units) {
          __syncthreads();
          s = 0;
          ++i;
          next_unit(cur, u, Hs, j0, j1);
          even_row = even_first;
#pragma unroll
          for (int q = 0; q < 2; ++q) { py[q] = py_first[q]; px[q] = px_first[q]; }
        }
      });
    }
    if (put_away > 0) add_away(std::false_type{});
  }
  wait_vm<0>();
  __syncthreads();
  // ---- partial sums [tile][16 P][CS]
  float* const part = a.part + (long long)tile * 16 * P * CS;
  if constexpr (PL == 3) {
#pragma unroll
    for (int t = 0; t < MF; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[t][e] = (acc[t][e] + low[t][e]) * SPLIT_UNSCALE;
    bool bad = false;
    if (wave < 4) {
#pragma unroll
      for (int t = 0; t < MF; ++t) bad = any_not_finite(acc[t]) || bad;
    }
    if (bad) {                                         // what has no split: this wave's sums again with the fp32 MFMAs, from memory
#pragma unroll
      for (int t = 0; t < MF; ++t) acc[t] = floatx16{};
      UnitAt q = first;
      for (int i = 0; i < units; ++i, next_unit(q, u, Hs, j0, j1)) {
        const bool nchw = a.real && q.seg == 0;
        const T* img = nchw ? nullptr : static_cast<const T*>(a.img) + ((long long)q.seg * a.seg_samples + q.j) * npix * CB;
        const float* real = nchw ? a.real + (long long)a.perm[q.j] * CB * npix : nullptr;
        const T* dys = static_cast<const T*>(a.dy) + ((long long)q.seg * a.seg_samples + q.j) * Hs * Hs * CS;
        for (int k = 0; k < 16 * steps; k += 2) {      // the pixels of its own K-steps
          const int p = ((k >> 4) * TURNS + turn) * 16 + (k & 15) + kgrp, yl = p / u.pw, y = q.y0 + yl, x = q.x0 + p - yl * u.pw;
          const bool ok = yl < u.ph && y < Hs && x < Hs;
          const float d = ok ? to_float(dys[(long long)(y * Hs + x) * CS + cb * 32 + (lane & 31)]) : 0.f;
#pragma unroll
          for (int t = 0; t < MF; ++t)
            acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(ok ? patch_value<T, CB>(img, real, Hb, y, x, 32 * t + (lane & 31)) : 0.f, d, acc[t], 0, 0, 0);
        }
      }
    }
  }
  if constexpr (TURNS > 1) {                           // the second wave's sums onto the first's (the rings and tiles are free)
    static_assert(TURNS == 2, "two waves");
    float* const sums = reinterpret_cast<float*>(lds) + cb * MF * 16 * 64;
    if (wave < 4 && turn == 1)
#pragma unroll
      for (int t = 0; t < MF; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) sums[(t * 16 + e) * 64 + lane] = acc[t][e];
    __syncthreads();
    if (wave < 4 && turn == 0)
#pragma unroll
      for (int t = 0; t < MF; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] += sums[(t * 16 + e) * 64 + lane];
  }
  if (wave < 4 && turn == 0) {
#pragma unroll
    for (int t = 0; t < MF; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) part[(32 * t + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3)) * CS + cb * 32 + (lane & 31)] = acc[t][e];
  }
  if (wave == 4 && a.pixel_sums) {
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      double s = own[c];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
      if (lane == 0) a.pixel_sums[tile * 4 + c] = (float)s;
    }
  }
}
template <typename T, int CB, int CS>
void wgrad_one(const ImageWgradArgs& a, int tiles, hipStream_t st) {
  const Units u = img_units(a.Hs, CB, WG_SIDE_Y);
  constexpr int PL = sizeof(T) == 4 ? 3 : 1, MF = img_values(CB) == 2 ? 1 : img_values(CB) / 2;
  const size_t lds = std::max<size_t>(4 * (PL == 1 ? wg_ring((int)sizeof(T)) * 1024 : 3 * 1024) + (size_t)2 * PL * (2 * u.ph + 2 + ZERO_ROWS) * u.pitch, CS == 64 ? 2 * MF * 16 * 64 * 4 : 0);
  const bool even = even_units(u, a.Hs, CS);
  const void* const kernel = even ? reinterpret_cast<const void*>(&image_wgrad_kernel<T, CB, CS, true>) : reinterpret_cast<const void*>(&image_wgrad_kernel<T, CB, CS, false>);
  if (lds > 48 * 1024)   // above the default dynamic limit: ask for it (idempotent, cheap)
    (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (even) hipLaunchKernelGGL((image_wgrad_kernel<T, CB, CS, true>), dim3((unsigned)tiles), dim3(WG_THREADS), lds, st, a, u);
  else hipLaunchKernelGGL((image_wgrad_kernel<T, CB, CS, false>), dim3((unsigned)tiles), dim3(WG_THREADS), lds, st, a, u);
}

// The tiles' partial sums of every model, added in a fixed order, where the gradients belong.  A block takes 16 groups of four columns of one
// model; lane group q adds the tiles q, q + 16, ... in turn, eight loads in flight, then the groups' sums, rounded once, are added in order; both in double.
// Blocks behind those: a model's pixel sums (the bias of G's last layer), the label maps' gradients from class sums, the row splits of the linear
// head's weight gradient (a launch of its own takes 4.6 us whatever it does).
__global__ __launch_bounds__(256) void image_wgrad_final_kernel(ImageGradArgs a, int col_blocks, int main_blocks, int sum_blocks, int label_blocks) {
  const int b = (int)blockIdx.x;
  const int P = a.P, Cs = a.Cs;
  if (b < main_blocks) {
    __shared__ float4 red[16][16];
    const int l = b / col_blocks, c = threadIdx.x & 15, q = threadIdx.x >> 4;
    const int t0 = a.tpre[l], t1 = a.tpre[l + 1], i = (b - l * col_blocks) * 16 + c;      // 16 P Cs / 4 is a multiple of 16
    const long long size4 = (long long)16 * P * Cs / 4;
    const float4* p = reinterpret_cast<const float4*>(a.part) + i;
    double d[4] = {0., 0., 0., 0.};
    for (int k0 = t0 + q; k0 < t1; k0 += 8 * 16) {
      float4 t[8];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (k0 + 16 * k < t1) t[k] = p[(long long)(k0 + 16 * k) * size4];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (k0 + 16 * k < t1) { d[0] += t[k].x; d[1] += t[k].y; d[2] += t[k].z; d[3] += t[k].w; }
    }
    red[q][c] = make_float4((float)d[0], (float)d[1], (float)d[2], (float)d[3]);
    __syncthreads();
    if (q > 0) return;
    const int groups = min(16, t1 - t0);
#pragma unroll 4
    for (int g = 1; g < groups; ++g) {
      const float4 t = red[g][c];
      d[0] += t.x; d[1] += t.y; d[2] += t.z; d[3] += t.w;
    }
    const float4 s = make_float4((float)d[0], (float)d[1], (float)d[2], (float)d[3]);
    const int m = 4 * i / Cs, cs = 4 * i - m * Cs, tap = m / P, ch = m - tap * P;
    if (a.k3 && ((tap >> 2) == 3 || (tap & 3) == 3)) return;
    float* const dw = a.dw + (long long)l * a.pstride + ((long long)tap * a.CBT + ch) * Cs + cs;
    if (ch < a.CB) *reinterpret_cast<float4*>(dw) = s;
    if (ch == a.CB) {
      if (a.plane_labels) *reinterpret_cast<float4*>(dw + (long long)(a.L == 1 ? 0 : l) * Cs) = s;
      if (tap == 5 && a.dbias) *reinterpret_cast<float4*>(a.dbias + (long long)l * a.pstride + cs) = s;
    }
    return;
  }
  if (b < main_blocks + sum_blocks) {
    __shared__ double sh[256];
    const int l = b - main_blocks, t0 = a.tpre[l], t1 = a.tpre[l + 1];
    if (t0 == t1) return;
    for (int c = 0; c < a.CB; ++c) {
      double s = 0.;
      for (int t = t0 + (int)threadIdx.x; t < t1; t += 256) s += a.pixel_sums[t * 4 + c];
      sh[threadIdx.x] = s;
      __syncthreads();
      for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
      }
      if (threadIdx.x == 0) a.image_bias[(long long)l * a.pstride + c] = (float)sh[0];
      __syncthreads();
    }
    return;
  }
  if (b >= main_blocks + sum_blocks + label_blocks) {
    const HeadSplits& h = a.head;
    const long long idx = (long long)(b - main_blocks - sum_blocks - label_blocks) * 256 + threadIdx.x;
    if (idx >= (long long)a.L * (h.K + 1)) return;
    const int l = (int)(idx / (h.K + 1)), k = (int)(idx - (long long)l * (h.K + 1));      // (index K: the bias term)
    if (a.tpre[l] == a.tpre[l + 1]) return;              // no samples
    float s = 0.f;
#pragma unroll 8
    for (int sp = 0; sp < h.rsplit; ++sp) s += h.part[((long long)sp * a.L + l) * (h.K + 4) + k];     // loads in flight together, sum in order
    if (k < h.K) h.dw[(long long)l * a.pstride + k] = s;
    else h.db[(long long)l * a.pstride] = s;
    return;
  }
  const int e = (b - main_blocks - sum_blocks) * 256 + (int)threadIdx.x;      // (label, tap, cs), one model
  if (e >= a.labels * 16 * Cs) return;
  const int cs = e % Cs, tap = e / Cs % 16, label = e / (16 * Cs);
  float s = 0.f;
  for (int cls = 0; cls < 9; ++cls)
    if (tap_inside(cls / 3, tap >> 2) && tap_inside(cls % 3, tap & 3)) s += a.label_sums[((long long)label * 9 + cls) * Cs + cs];
  a.dw[((long long)tap * a.CBT + a.CB + label) * Cs + cs] = s;
}

// w[l][cs][tap * P + c] and, behind them, the rows to add: add[table][class][cs] = sum of the label map's taps inside + bias, each as stored
template <typename T>
__global__ __launch_bounds__(256) void pack_image_w_kernel(ImagePackArgs a, int w_blocks) {
  const int P = a.P, Cs = a.Cs;
  if ((int)blockIdx.x < w_blocks) {
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long long)a.L * 16 * P * Cs) return;
    const int m = (int)(idx % (16 * P)), cs = (int)(idx / (16 * P) % Cs), l = (int)(idx / ((long long)16 * P * Cs));
    const int tap = m / P, c = m - tap * P;
    static_cast<T*>(a.packed)[idx] = from_float<T>(c < a.CB ? a.w[(long long)l * a.pstride + ((long long)tap * a.CBT + c) * Cs + cs] : 0.f);
    return;
  }
  const int idx = ((int)blockIdx.x - w_blocks) * 256 + (int)threadIdx.x;
  if (idx >= a.tables * 9 * Cs) return;
  const int cs = idx % Cs, cls = idx / Cs % 9, t = idx / (9 * Cs), l = a.L == 1 ? 0 : t;
  const float* w = a.w + (long long)l * a.pstride;
  float v[16];                                         // (all loads first: the kernel is bound by their latency)
#pragma unroll
  for (int tap = 0; tap < 16; ++tap) v[tap] = w[((long long)tap * a.CBT + a.CB + t) * Cs + cs];
  a.add[idx] = label_class_sum<T>(v, cls);
}

// f(channels of the image, feature channels) as types
template <typename F> bool with_channels(int CB, int Cs, F&& f) {
  const auto cs = [&](auto cb) {
    if (Cs == 64) f(cb, std::integral_constant<int, 64>{}); else f(cb, std::integral_constant<int, 128>{});
  };
  if (Cs != 64 && Cs != 128) return false;
  if (CB == 1) cs(std::integral_constant<int, 1>{});
  else if (CB == 2) cs(std::integral_constant<int, 2>{});
  else if (CB == 3) cs(std::integral_constant<int, 3>{});
  else if (CB == 4) cs(std::integral_constant<int, 4>{});
  else return false;
  return true;
}

}  // namespace

int image_values(int CB) { return img_values(CB); }
long long image_part_floats(int esize, int CB, int Hs, int Cs, int nseg, const ImageTiles& t, long long tiles) {
  const Units u = img_units(Hs, CB, WG_SIDE_Y);
  const int turns = 128 / Cs;
  // (two waves that share 32 channels: the second one's chains go to lines of their own, where a tile has more than one)
  const bool chains = (long long)t.most * nseg * u.nx * u.ny * (((u.ph * u.pw + 15) / 16 + turns - 1) / turns) > wg_chain(esize);
  return tiles * 16 * img_values(CB) * Cs * (chains ? turns : 1);
}

template <typename T> void launch_image_conv(const ImageConvArgs& a, hipStream_t st) {
  if (a.n == 0 || a.nseg == 0) return;
  if (!a.img || !a.w || !a.out || !a.offs || !a.sample_model || (a.real && !a.perm) || a.Hs < 1)
    return launch_fail("image-side convolution: null operand");
  if ((long long)a.Hs * a.Hs * a.Cs * (long long)sizeof(T) >= (1LL << 31)) return launch_fail("image-side convolution: a sample of 2 GiB or larger");
  if (!with_channels(a.CB, a.Cs, [&](auto cb, auto cs) { conv_one<T, cb.value, cs.value>(a, st); }))
    launch_fail("image-side convolution: more than 4 image channels, or feature channels other than 64 / 128");
}
template void launch_image_conv<float>(const ImageConvArgs&, hipStream_t);
template void launch_image_conv<bf16_t>(const ImageConvArgs&, hipStream_t);

template <typename T> void launch_image_wgrad(const ImageWgradArgs& a, int ub_tiles, hipStream_t st) {
  if (ub_tiles == 0 || a.nseg == 0) return;
  if (!a.img || !a.dy || !a.part || !a.offs || !a.tpre || (a.L > 1 && !a.tmodel) || (a.real && !a.perm) || a.tiles.most < 1 || a.tiles.parts < 1 || a.Hs < 1)
    return launch_fail("image-side weight gradient: null operand");
  if ((long long)a.Hs * a.Hs * a.Cs * (long long)sizeof(T) >= (1LL << 31)) return launch_fail("image-side weight gradient: a sample of 2 GiB or larger");
  if (!with_channels(a.CB, a.Cs, [&](auto cb, auto cs) { wgrad_one<T, cb.value, cs.value>(a, ub_tiles, st); }))
    launch_fail("image-side weight gradient: more than 4 image channels, or feature channels other than 64 / 128");
}
template void launch_image_wgrad<float>(const ImageWgradArgs&, int, hipStream_t);
template void launch_image_wgrad<bf16_t>(const ImageWgradArgs&, int, hipStream_t);

void launch_image_wgrad_final(const ImageGradArgs& a, hipStream_t st) {
  if (!a.part || !a.dw || !a.tpre || a.pstride % 4 != 0 || ((uintptr_t)a.dw & 15) != 0 || ((uintptr_t)a.dbias & 15) != 0 || (a.labels > 0 && (!a.label_sums || a.L != 1)))
    return launch_fail("image-side weight gradient: null operand, or gradients that are not 16-byte aligned");
  const int cols = 16 * a.P * a.Cs / 64;
  const long long main_blocks = (long long)a.L * cols, sum_blocks = a.image_bias ? a.L : 0, label_blocks = ((long long)a.labels * 16 * a.Cs + 255) / 256;
  const long long head_blocks = a.head.part ? ((long long)a.L * (a.head.K + 1) + 255) / 256 : 0, blocks = main_blocks + sum_blocks + label_blocks + head_blocks;
  if (blocks >= (1LL << 31)) return launch_fail("image-side weight gradient: more blocks than a launch can have");
  hipLaunchKernelGGL(image_wgrad_final_kernel, dim3((unsigned)blocks), dim3(256), 0, st, a, cols, (int)main_blocks, (int)sum_blocks, (int)label_blocks);
}

template <typename T> void launch_pack_image_w(const ImagePackArgs& a, hipStream_t st) {
  const long long w_blocks = ((long long)a.L * 16 * a.P * a.Cs + 255) / 256, add_blocks = a.add ? ((long long)a.tables * 9 * a.Cs + 255) / 256 : 0;
  if (w_blocks + add_blocks >= (1LL << 31)) return launch_fail("image-side weights: more blocks than a launch can have");
  hipLaunchKernelGGL((pack_image_w_kernel<T>), dim3((unsigned)(w_blocks + add_blocks)), dim3(256), 0, st, a, (int)w_blocks);
}
template void launch_pack_image_w<float>(const ImagePackArgs&, hipStream_t);
template void launch_pack_image_w<bf16_t>(const ImagePackArgs&, hipStream_t);

}  // namespace gan
