// The layers that write an image of 1..4 channels, or sums over one: the transposed convolution onto the image (G's last layer, the data
// gradient of D's first), the class sums that give the label maps of one pair over many labels their gradient, and the sums of an image's pixels.
// The layers that read an image: image_conv.hip.
#include <stdlib.h>

#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "split_mfma.h"

namespace gan {


template <typename T> __device__ inline float ldf(const T* p) { return to_float(*p); }

// Class sums of a layer's output gradient, for one pair's label maps.  First per sample: a block takes one sample
// of one segment and up to 128 channels, a thread 8 channels of every 16th pixel row; inner rows meet in LDS, in a fixed order.
// It reads the tensor once, 16 bytes a lane, and is bound by that.  Then per slot: a block owns 64 sums of a slot; of every 1024 samples
// its sixteen waves take the slot's in turn, eight loads in flight, and the waves' sums meet in LDS in order.  That bounds the chain of
// dependent additions when one label fills the batch (a thread that added all samples of its slot itself: 8x8 images, 40 labels, bf16,
// 20000 samples, 2061 us a step with labels drawn evenly and 5183 with one label; now 1898 and 1994).
template <typename T>
__global__ __launch_bounds__(256) void class_sums_sample_kernel(ClassSumArgs a) {
  __shared__ float inner[16][3][128];
  const int j = blockIdx.x, sidx = blockIdx.y, c0 = blockIdx.z * 128;
  if (j >= a.offs[a.L]) return;
  const int g = threadIdx.x & 15, lane = threadIdx.x >> 4;              // channels c0 + 8 g .., pixel rows lane, lane + 16, ..
  const int c = c0 + 8 * g, H = a.Hs, Cs = a.Cs;
  const bool have = c < Cs;                                             // Cs is a multiple of 64
  const T* dy = static_cast<const T*>(a.dy) + ((long long)(a.seg_first + sidx) * a.seg_samples + j) * H * H * Cs + c;
  float* out = a.part + ((long long)sidx * a.n + j) * 9 * Cs;
  float mid[3][8] = {};
  if (have)
    for (int y = lane; y < H; y += 16) {
      float s[3][8] = {};
      const auto add = [&](int x, int cls) __attribute__((always_inline)) {
        alignas(16) T v[8];
        const uint4* q = reinterpret_cast<const uint4*>(dy + ((long long)y * H + x) * Cs);
        uint4* d = reinterpret_cast<uint4*>(v);
        d[0] = q[0];
        if constexpr (sizeof(T) == 4) d[sizeof(T) / 4] = q[1];
#pragma unroll
        for (int k = 0; k < 8; ++k) s[cls][k] += to_float(v[k]);
      };
      add(0, 0);
#pragma unroll 4
      for (int x = 1; x < H - 1; ++x) add(x, 1);
      if (H > 1) add(H - 1, 2);
      const int row = y == 0 ? 0 : (y == H - 1 ? 2 : 1);
#pragma unroll
      for (int cls = 0; cls < 3; ++cls)
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          if (row == 1) mid[cls][k] += s[cls][k];
          else out[(row * 3 + cls) * Cs + c + k] = s[cls][k];
          if (H == 1) out[(6 + cls) * Cs + c + k] = 0.f;                // no last row
        }
    }
#pragma unroll
  for (int cls = 0; cls < 3; ++cls)
#pragma unroll
    for (int k = 0; k < 8; ++k) inner[lane][cls][8 * g + k] = mid[cls][k];
  __syncthreads();
  for (int t = threadIdx.x; t < 3 * 128; t += 256) {
    const int cls = t >> 7, cc = t & 127;
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) s += inner[r][cls][cc];
    if (c0 + cc < Cs) out[(3 + cls) * Cs + c0 + cc] = s;
  }
}
constexpr int SLOT_T = 1024, SLOT_W = SLOT_T / 64;
__global__ __launch_bounds__(SLOT_T) void class_sums_slot_kernel(ClassSumArgs a) {
  __shared__ int list[SLOT_T];
  __shared__ int wave_n[SLOT_W];
  __shared__ float part[SLOT_W][64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int slot = blockIdx.x, per = 9 * a.Cs, e = blockIdx.y * 64 + lane;      // per is a multiple of 64
  const int n = a.offs[a.L];
  float s = 0.f;
  for (int j0 = 0; j0 < n; j0 += SLOT_T) {
    const int j = j0 + threadIdx.x;
    const bool mine = j < n && a.sample_slot[j] == slot;
    const unsigned long long votes = __ballot(mine);
    if (lane == 0) wave_n[wave] = __popcll(votes);
    __syncthreads();
    int at = 0, total = 0;
#pragma unroll
    for (int w = 0; w < SLOT_W; ++w) {
      if (w < wave) at += wave_n[w];
      total += wave_n[w];
    }
    if (mine) list[at + __popcll(votes & ((1ull << lane) - 1))] = j;
    __syncthreads();
    for (int sidx = 0; sidx < a.nseg; ++sidx) {
      const float* p = a.part + (long long)sidx * a.n * per + e;
#pragma unroll 8
      for (int i = wave; i < total; i += SLOT_W) s += p[(long long)list[i] * per];
    }
    __syncthreads();
  }
  part[wave][lane] = s;
  __syncthreads();
  if (wave == 0) {
    s = part[0][lane];
#pragma unroll
    for (int w = 1; w < SLOT_W; ++w) s += part[w][lane];
    a.sums[(long long)slot * per + e] = s;
  }
}
template <typename T> void launch_class_sums(const ClassSumArgs& a, hipStream_t st) {
  if (a.n < 1 || a.Cs % 64 != 0) return launch_fail("class sums: no samples, or channels that are no multiple of 64");
  hipLaunchKernelGGL((class_sums_sample_kernel<T>), dim3((unsigned)a.n, (unsigned)a.nseg, (unsigned)((a.Cs + 127) / 128)), dim3(256), 0, st, a);
  hipLaunchKernelGGL(class_sums_slot_kernel, dim3((unsigned)a.labels, (unsigned)(9 * a.Cs / 64)), dim3(SLOT_T), 0, st, a);
}
template void launch_class_sums<float>(const ClassSumArgs&, hipStream_t);
template void launch_class_sums<bf16_t>(const ClassSumArgs&, hipStream_t);

// dbias[cb] = sum over the model's image-side pixels (G's last layer): block (chunk of pixels, model) partial
// sums, then one small pass adds the chunks in order.
template <typename T>
__global__ __launch_bounds__(256) void img_bias_partial_kernel(ImgBiasArgs a) {
  __shared__ float red[256];
  const int l = blockIdx.y;
  const int cnt = a.offs[l + 1] - a.offs[l];
  const long long pix = (long long)cnt * a.HW;
  const long long per = (pix + gridDim.x - 1) / gridDim.x;
  const long long p0 = per * blockIdx.x, p1 = min(pix, p0 + per);
  const T* img = static_cast<const T*>(a.img) + (long long)a.offs[l] * a.HW * a.CB;
  for (int cb = 0; cb < a.CB; ++cb) {
    float s = 0.f;
    for (long long i = p0 + threadIdx.x; i < p1; i += 256) s += ldf(img + i * a.CB + cb);
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
      __syncthreads();
    }
    if (threadIdx.x == 0) a.partial[((long long)l * gridDim.x + blockIdx.x) * 4 + cb] = red[0];
    __syncthreads();
  }
}
// one block per model: thread t adds the chunks t, t + 256, ... in turn, then a fixed tree over the threads
__global__ __launch_bounds__(256) void img_bias_final_kernel(ImgBiasArgs a, int chunks) {
  __shared__ float red[256];
  const int l = blockIdx.x;
  if (a.offs[l + 1] == a.offs[l]) return;
  for (int cb = 0; cb < a.CB; ++cb) {
    float s = 0.f;
    for (int k = threadIdx.x; k < chunks; k += 256) s += a.partial[((long long)l * chunks + k) * 4 + cb];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
      __syncthreads();
    }
    if (threadIdx.x == 0) a.dbias[(long long)l * a.pstride + cb] = red[0];
    __syncthreads();
  }
}
// chunks of a model's pixels: enough blocks to fill the chip with few models; a function of the model count only
int img_bias_chunks(int L) { return std::min(std::max(2048 / (L > 0 ? L : 1), 32), 256); }
template <typename T> void launch_img_bias_grad(const ImgBiasArgs& a, hipStream_t st) {
  const int chunks = img_bias_chunks(a.L);
  hipLaunchKernelGGL((img_bias_partial_kernel<T>), dim3(chunks, a.L), dim3(256), 0, st, a);
  hipLaunchKernelGGL(img_bias_final_kernel, dim3(a.L), dim3(256), 0, st, a, chunks);
}
template void launch_img_bias_grad<float>(const ImgBiasArgs&, hipStream_t);
template void launch_img_bias_grad<bf16_t>(const ImgBiasArgs&, hipStream_t);

// ---------------------------------------------------------------------------------------------------------
// Transposed convolution onto the image (or the data gradient of D's first convolution, which is the same
// operation): img[n, 2y+py, 2x+px][cb] = sum over the 4 taps of that phase and cs of feat[n, y+dy, x+dx][cs] * w[tap][cb][cs].
// One product per 8 x 8 patch of feature pixels: R[halo pixel][(tap, image channel)] = F[halo pixel] . w[tap][channel], rows = the
// 100 pixels of the patch with its 1-pixel halo (32 per wave), columns = the 16 CB (tap, channel) pairs, K = the feature
// channels.  A row's features go straight from memory to the lane that multiplies them -- each is used by one wave --, R
// meets in LDS, and an output pixel adds the four entries of the neighbours that hold it.  (Multiplying per output pixel, with
// K = (neighbour, channel), takes 18 MFMAs for these 8, splits every fp32 value nine times, and needs sums across the waves.)
// A block keeps the weights in LDS (fp32: their three bf16 parts) and walks over patches of its sample; the next patch's
// features are on their way while the results of this one are written.  What bounds it is the way of the features through the
// CU and the two barriers per patch.  Per launch, before -> now: 128 channels at side 16, fp32, 1280 samples 238 -> 94 us, bf16, 6400
// samples 187 -> 139 (3.4 TB/s); 64 channels at side 14, fp32, 64 samples 10.2 -> 5.6.
// Epilogue: bias + tanh, or times (1 - y^2).
// ---------------------------------------------------------------------------------------------------------
constexpr int UP_TS = 8;                    // patch side (feature pixels)
constexpr int UP_HALO = UP_TS + 2;
constexpr int UP_RROW = 128 + 4;            // floats per column of R: 128 rows, padded
constexpr int UP_BLOCKS = 2048;             // blocks that fill the chip (see the launcher)

template <typename T, int CS, int CB>
constexpr int up_img_lds() { return 16 * CB * ((sizeof(T) == 4 ? 3 : 1) * (CS * 2 + 16) + UP_RROW * 4); }

// USER: into the caller's images, a channel plane's pixels next to each other (no pass of its own over the images: 37 of 1407 us for
// 6400 samples of 32x32x3).
template <typename T, int CS, int CB, bool USER>
__global__ __launch_bounds__(256) void up_img_kernel(UpImgArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  constexpr int SZ = (int)sizeof(T), NC = 16 * CB, NCT = (NC + 31) / 32, KS = CS / 16;
  constexpr int WROW = CS * 2 + 16, WPLANE = NC * WROW;        // bytes per weight row / part in LDS
  unsigned char* const Wl = lds;
  float* const R = reinterpret_cast<float*>(lds + (SZ == 4 ? 3 : 1) * WPLANE);     // [NC][UP_RROW]
  const int j = blockIdx.y;                                   // routed sample inside the segment
  if (j >= a.offs[a.L]) return;
  const int l = a.sample_model[j];
  const int Hs = a.Hs, Hb = 2 * Hs;
  const long long sample = (long long)a.seg * a.seg_samples + j;
  const int tiles = (Hs + UP_TS - 1) / UP_TS, np = tiles * tiles;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, h = lane >> 5;
  const T* feat = static_cast<const T*>(a.feat) + sample * (long long)Hs * Hs * CS;
  // this lane's halo pixel and its channels 16 k + 8 h .. + 7, k < KS, of one patch
  const int q = wave * 32 + r, qy = q / UP_HALO - 1, qx = q % UP_HALO - 1;
  constexpr int CH = SZ / 2;                                  // 16-byte loads per eight channels
  u32x4 fv[KS][CH];
  const auto load = [&](int p) __attribute__((always_inline)) {
    const int y = p / tiles * UP_TS + qy, x = p % tiles * UP_TS + qx;
    const bool in = q < UP_HALO * UP_HALO && (unsigned)y < (unsigned)Hs && (unsigned)x < (unsigned)Hs;
    const u32x4* src = reinterpret_cast<const u32x4*>(feat + ((long long)y * Hs + x) * CS + 8 * h);
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
      for (int c = 0; c < CH; ++c) fv[k][c] = in ? src[(16 * k * SZ) / 16 + c] : u32x4{0, 0, 0, 0};
  };
  load(blockIdx.x);
  const T* w = static_cast<const T*>(a.w) + (long long)l * a.w_stride;
  for (int i = tid; i < NC * (CS / 8); i += 256) {            // eight channels of a weight row
    const int c = i / (CS / 8), ch = i % (CS / 8), tap = c / CB, cb = c % CB;
    const u32x4* src = reinterpret_cast<const u32x4*>(w + ((long long)tap * a.CBT + cb) * CS + 8 * ch);
    unsigned char* dst = Wl + c * WROW + ch * 16;
    if constexpr (SZ == 2) {
      *reinterpret_cast<u32x4*>(dst) = src[0];
    } else {
      const Split8 s = split8(src[0], src[1]);
      *reinterpret_cast<u32x4*>(dst) = s.h;
      *reinterpret_cast<u32x4*>(dst + WPLANE) = s.m;
      *reinterpret_cast<u32x4*>(dst + 2 * WPLANE) = s.l;
    }
  }
  __syncthreads();
  // columns past the last pair repeat it and are not read
  const unsigned char* wrow[NCT];
#pragma unroll
  for (int t = 0; t < NCT; ++t) wrow[t] = Wl + min(32 * t + r, NC - 1) * WROW + h * 16;
  const auto part = [&](int t, int k, int plane) __attribute__((always_inline)) {
    return *reinterpret_cast<const u32x4*>(wrow[t] + plane * WPLANE + k * 32);
  };
  for (int p = blockIdx.x; p < np; p += gridDim.x) {
    floatx16 acc[NCT] = {}, low[NCT] = {};
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      if constexpr (SZ == 2) {
#pragma unroll
        for (int t = 0; t < NCT; ++t) mma_u4(acc[t], fv[k][0], part(t, k, 0));
      } else {
        const Split8 f = split8(fv[k][0], fv[k][1]);
#pragma unroll
        for (int t = 0; t < NCT; ++t) {
          const Split8 g = {part(t, k, 0), part(t, k, 1), part(t, k, 2)};
          mma_u4(low[t], f.l, g.h);
          mma_u4(acc[t], f.h, g.h);
          mma_u4(low[t], f.h, g.l);
          mma_u4(low[t], f.m, g.m);
          mma_u4(low[t], f.m, g.h);
          mma_u4(low[t], f.h, g.m);
        }
      }
    }
    if constexpr (SZ == 4) {
      float z = 0.f;
#pragma unroll
      for (int t = 0; t < NCT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          acc[t][e] = (acc[t][e] + low[t][e]) * SPLIT_UNSCALE;
          z = __builtin_fmaf(acc[t][e], 0.f, z);
        }
      if (__ballot(z != z)) {                               // what has no split: this wave's rows again with the fp32 MFMAs
#pragma unroll
        for (int t = 0; t < NCT; ++t) {
          acc[t] = floatx16{};
          const int c = min(32 * t + r, NC - 1);
          const T* wc = w + ((long long)(c / CB) * a.CBT + c % CB) * CS + 8 * h;
#pragma unroll
          for (int k = 0; k < KS; ++k)
#pragma unroll
            for (int e = 0; e < 8; ++e)
              acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(fv[k][e / 4][e % 4]), to_float(wc[16 * k + e]), acc[t], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < NCT; ++t)
      if (32 * t + r < NC)
#pragma unroll
        for (int e = 0; e < 16; e += 4)                     // rows 8 (e / 4) + 4 h .. + 3 of this wave
          *reinterpret_cast<float4*>(R + (32 * t + r) * UP_RROW + wave * 32 + 2 * e + 4 * h) =
              make_float4(acc[t][e], acc[t][e + 1], acc[t][e + 2], acc[t][e + 3]);
    if (p + (int)gridDim.x < np) load(p + gridDim.x);
    __syncthreads();
    const int y0 = p / tiles * UP_TS, x0 = p % tiles * UP_TS;
    T* out = static_cast<T*>(a.out);
    const T* aux = static_cast<const T*>(a.aux);
    constexpr int rowlen = 2 * UP_TS * CB;                    // contiguous output elements per patch row
#pragma unroll
    for (int i = tid; i < 2 * UP_TS * rowlen; i += 256) {
      int Yl, Xl, cb;
      if constexpr (USER) {
        cb = i / (4 * UP_TS * UP_TS);
        Yl = i / (2 * UP_TS) % (2 * UP_TS);
        Xl = i % (2 * UP_TS);
      } else {
        const int rem = i % rowlen;
        Yl = i / rowlen;
        Xl = rem / CB;
        cb = rem % CB;
      }
      const int Y = 2 * y0 + Yl, X = 2 * x0 + Xl;
      if (Y >= Hb || X >= Hb) continue;
      const long long o = ((sample * Hb + Y) * Hb + X) * CB + cb;
      // output phase 0 takes the pixel itself through tap 1 and the one before through tap 3, phase 1 the one after through tap 0
      // and the pixel itself through tap 2
      const int py = Yl & 1, px = Xl & 1;
      const float* e0 = R + cb * UP_RROW + (Yl / 2 + 1) * UP_HALO + Xl / 2 + 1;
      const auto at = [&](int ay, int ax) {
        const int ky = ay == 0 ? 1 + py : 3 - 3 * py, kx = ax == 0 ? 1 + px : 3 - 3 * px;
        const int dy = ay == 0 ? 0 : 2 * py - 1, dx = ax == 0 ? 0 : 2 * px - 1;
        return e0[(ky * 4 + kx) * CB * UP_RROW + dy * UP_HALO + dx];
      };
      float v = (at(0, 0) + at(0, 1)) + (at(1, 0) + at(1, 1));
      if constexpr (USER) {
        a.user[(((long long)a.perm[j] * CB + cb) * Hb + Y) * Hb + X] = tanhf(v + a.bias[(long long)l * a.bias_stride + cb]);
        continue;
      }
      if (a.mode == 1) v = tanhf(v + a.bias[(long long)l * a.bias_stride + cb]);
      else if (a.mode == 2) { const float yv = to_float(aux[o]); v *= (1.f - yv * yv); }
      out[o] = from_float<T>(v);
    }
    __syncthreads();
  }
}
template <typename T, int CS, int CB, bool USER> static void up_img_one(const UpImgArgs& a, hipStream_t st) {
  const int tiles = (a.Hs + UP_TS - 1) / UP_TS, np = tiles * tiles;
  // a block per patch while that leaves CUs idle, else several patches per block, for one read of the weights (6400 samples of 4
  // patches: one patch per block 171 us, two 146, four 140; 1024 samples of 16: 89, 86 with two per block, 74 with eight)
  const int blocks = (int)std::min<long long>(np, std::max<long long>(1, (UP_BLOCKS + a.n - 1) / a.n));
  constexpr int lds = up_img_lds<T, CS, CB>();
  if (lds > 48 * 1024)   // above the default dynamic limit: ask for it (idempotent, cheap)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&up_img_kernel<T, CS, CB, USER>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  hipLaunchKernelGGL((up_img_kernel<T, CS, CB, USER>), dim3((unsigned)blocks, (unsigned)a.n), dim3(256), lds, st, a);
}
template <typename T> void launch_up_img(const UpImgArgs& a, hipStream_t st) {
  if (a.n == 0) return;
  if (!a.feat || !a.w || !a.out || a.CB < 1 || a.CB > 4 || (a.Cs != 64 && a.Cs != 128) || (a.mode == 1 && !a.bias) || (a.mode == 2 && !a.aux) ||
      (a.user && (a.mode != 1 || !a.perm)))
    return launch_fail("image-side transposed convolution: null operand, more than 4 image channels, or feature channels other than 64 / 128");
  const auto with_cs = [&](auto cb) {
    if (a.user) {
      if (a.Cs == 64) up_img_one<T, 64, cb.value, true>(a, st); else up_img_one<T, 128, cb.value, true>(a, st);
    } else {
      if (a.Cs == 64) up_img_one<T, 64, cb.value, false>(a, st); else up_img_one<T, 128, cb.value, false>(a, st);
    }
  };
  if (a.CB == 1) with_cs(std::integral_constant<int, 1>{});
  else if (a.CB == 2) with_cs(std::integral_constant<int, 2>{});
  else if (a.CB == 3) with_cs(std::integral_constant<int, 3>{});
  else with_cs(std::integral_constant<int, 4>{});
}
template void launch_up_img<float>(const UpImgArgs&, hipStream_t);
template void launch_up_img<bf16_t>(const UpImgArgs&, hipStream_t);

}  // namespace gan
