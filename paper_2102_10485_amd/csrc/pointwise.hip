// Bandwidth-bound kernels of the training step: label routing, staging, BatchNorm statistics / apply / backward
// fused with the activation, D's linear head and the two logistic costs (Eq. 3, Eq. 4), Adam, layout copies.
// Every reduction has an order that follows from the configuration (models, sizing batch, layer shapes) and the model's own samples, so results are
// deterministic and a model's numbers do not change with what else is in the launch.
#include <algorithm>

#include "kernels.h"
#include "split_mfma.h"

namespace gan {

// ---------------------------------------------------------------------------------------------------------
// routing: stable partition of the flat batch by model
// ---------------------------------------------------------------------------------------------------------

__device__ inline int model_of_label(int y, int L) { return L == 1 ? 0 : y; }

// One block of ROUTE_WAVES waves does the whole partition: wave w owns the w-th run of consecutive samples, 64 at a time.
//   1. per-(wave, model) counts;  2. per model, the exclusive scan over the waves (a wave's samples of a model follow
//   those of the waves before it: stable) and the model's total;  3. model offsets, the tile prefix of every geometry
//   (a wave each, scanned 64 models at a time) and the models' order by size;  4. the scatter: a sample's place among its wave's 64 is the
//   number of lanes before it with the same model, found with one vote per bit of the model's number.
// The tables live in LDS when they fit; otherwise they are the global arrays, which one block may
// use the same way (barriers order its own global accesses).  Bound by latency: 100 models, 6400 samples 39.8 -> 18.5 us, 10 models,
// 1117 samples 11.8 -> 6.7, one model, 64 samples 10.2 -> 4.6 against 256 threads with a run of samples, and a row of the table, each.
constexpr int ROUTE_THREADS = 64 * ROUTE_WAVES;
constexpr int ROUTE_LDS_BYTES = 152 * 1024;
// (the placement is a template parameter so that every access is known to be an LDS or a global one: through
// pointers that may be either, each LDS access took several times as long)
template <typename T>
__device__ inline T staged_noise(const float* __restrict__ noise, const int* __restrict__ label_ids, int src, int k, int zdim, int cond_g) {
  float v = 0.f;
  if (k < zdim) v = noise[(long long)src * zdim + k];
  else if (k < zdim + cond_g) v = (k - zdim == label_ids[src]) ? 1.f : 0.f;
  return from_float<T>(v);
}
// The staging of one model's few rows as a tail of the routing (STAGE_INSIDE): another launch costs more than one block's pass over them.
template <typename T> struct StageTail { const float* noise; T* zin; int zdim, cond_g, kp; };      // noise NULL: none
template <bool in_lds, typename T>
__global__ __launch_bounds__(ROUTE_THREADS) void route_kernel(const int* __restrict__ label_ids, int n, int L, int n_labels, int bits,
                                                              GeomTable geoms, RouteBuffers rb, StageTail<T> tail) {
  extern __shared__ int route_lds[];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  int* cl = in_lds ? route_lds : rb.counts;                    // [L]
  int* ol = in_lds ? route_lds + L : rb.offs;                  // [L + 1]
  int* cnt = in_lds ? route_lds + (2 * L + 1) : rb.cnt;        // [ROUTE_WAVES][L]
  for (int i = t; i < ROUTE_WAVES * L; i += ROUTE_THREADS) cnt[i] = 0;
  __syncthreads();
  int* row = cnt + (long long)wave * L;
  const int share = ((n + ROUTE_WAVES - 1) / ROUTE_WAVES + 63) / 64 * 64;
  const int i0 = min(n, wave * share), i1 = min(n, i0 + share);
  // f(sample, model or -1) for the wave's samples, 64 at a time; eight loads in flight
  const auto for_samples = [&](auto f) {
    for (int b = i0; b < i1; b += 512) {
      int ys[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) ys[k] = b + 64 * k + lane < i1 ? label_ids[b + 64 * k + lane] : -1;
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (b + 64 * k < i1) f(b + 64 * k + lane, ys[k]);
    }
  };
  bool bad = false;
  for_samples([&](int i, int y) {
    if (i >= i1) return;
    if (y < 0 || y >= n_labels) bad = true;
    else atomicAdd(&row[model_of_label(y, L)], 1);
  });
  if (bad) rb.flags[0] = 1;
  __syncthreads();
  for (int l = t; l < L; l += ROUTE_THREADS) {
    int v[ROUTE_WAVES], run = 0;
#pragma unroll
    for (int w = 0; w < ROUTE_WAVES; ++w) v[w] = cnt[(long long)w * L + l];
#pragma unroll
    for (int w = 0; w < ROUTE_WAVES; ++w) {
      cnt[(long long)w * L + l] = run;
      run += v[w];
    }
    cl[l] = run;
    rb.counts[l] = run;
  }
  __syncthreads();
  // table 0: the model offsets; table 1 + g: the tile prefix of geometry g
  for (int g = wave - 1; g < geoms.n; g += ROUTE_WAVES) {
    const int rps = g < 0 ? 1 : geoms.rps[g], tr = g < 0 ? 1 : geoms.tile_rows[g];
    int* dst = g < 0 ? rb.offs : rb.tpre + (long long)g * (L + 1);
    const int sh = (tr & (tr - 1)) == 0 ? __ffs(tr) - 1 : -1;      // tile heights are powers of two
    const int parts = g < 0 ? 0 : geoms.parts[g];
    int run = 0;
    for (int l0 = 0; l0 < L; l0 += 64) {
      const int c = l0 + lane < L ? cl[l0 + lane] * rps + tr - 1 : 0;
      int v;
      if (parts > 0) {
        const int own = l0 + lane < L ? cl[l0 + lane] : 0, per = image_tile(ImageTiles{tr, parts}, own);
        v = own;
        if (per > 1) v = (own + per - 1) / per;
      } else {
        v = sh >= 0 ? c >> sh : c / tr;
      }
      int incl = v;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_up(incl, d, 64);
        if (lane >= d) incl += up;
      }
      if (l0 + lane < L) {
        dst[l0 + lane] = run + incl - v;
        if (in_lds && g < 0) ol[l0 + lane] = run + incl - v;
      }
      run += __shfl(incl, 63, 64);
    }
    if (lane == 0) {
      dst[L] = run;
      if (in_lds && g < 0) ol[L] = run;
    }
  }
  if (rb.order)
    // order[rank of l] = l, rank = number of models with more samples, or as many and a smaller index
    for (int l = wave; l < L; l += ROUTE_WAVES) {
      const int c = cl[l];
      int rank = 0;
      for (int j0 = 0; j0 < L; j0 += 64) {
        const int j = j0 + lane, cj = j < L ? cl[j] : -1;
        rank += __popcll(__ballot(cj > c || (cj == c && j < l)));
      }
      if (lane == 0) rb.order[rank] = l;
    }
  __syncthreads();
  for_samples([&](int i, int y) {
    const bool valid = y >= 0 && y < n_labels;
    const int mdl = valid ? model_of_label(y, L) : 0;
    unsigned long long same = __ballot(valid);
    for (int k = 0; k < bits; ++k) {
      const unsigned long long ones = __ballot((mdl >> k) & 1);
      same &= (mdl >> k) & 1 ? ones : ~ones;
    }
    const int rank = __popcll(same & ((1ull << lane) - 1));
    int base = 0;
    if (valid) base = row[mdl];
    // the next 64 samples find the row moved on: every lane has read before the first of each model writes
    if (in_lds) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); else __threadfence_block();
    __builtin_amdgcn_wave_barrier();
    if (valid && rank == 0) row[mdl] = base + __popcll(same);
    if (in_lds) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); else __threadfence_block();
    __builtin_amdgcn_wave_barrier();
    if (valid) {
      const int pos = ol[mdl] + base + rank;
      rb.perm[pos] = i;
      rb.sample_model[pos] = mdl;
      rb.sample_slot[pos] = (L == 1) ? y : 0;
    }
  });
  if (tail.noise) {
    __syncthreads();
    const int rows = ol[L];
    for (int i = t; i < rows * tail.kp; i += ROUTE_THREADS) {
      const int j = i / tail.kp;
      tail.zin[i] = staged_noise<T>(tail.noise, label_ids, rb.perm[j], i - j * tail.kp, tail.zdim, tail.cond_g);
    }
  }
}

// model of tile t of a geometry
__device__ inline void tile_model(const int* __restrict__ tpre, int L, int* __restrict__ tmodel, int cap, int t) {
  if (t >= tpre[L] || t >= cap) return;
  int lo = 0, hi = L;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (tpre[mid] <= t) lo = mid; else hi = mid;
  }
  tmodel[t] = lo;
}
// Q threads share an element's splits, thread q adding q, q + Q, ..., then the threads' sums are added in order.
template <int Q>
__global__ __launch_bounds__(256) void sum_splits_kernel(const float* __restrict__ part, float* __restrict__ dW, long long dw_stride,
                                                          long long size4, int L, int nsplit) {
  __shared__ float4 sh[Q][256 / Q];
  const int c = threadIdx.x % (256 / Q), q = threadIdx.x / (256 / Q);
  const long long idx = (long long)blockIdx.x * (256 / Q) + c;
  const bool have = idx < size4 * L;
  const int l = have ? (int)(idx / size4) : 0;
  const long long i = idx - (long long)l * size4;
  const float4* p = reinterpret_cast<const float4*>(part) + (long long)l * size4 + i;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  // eight loads in flight, added in order (written out: a loop of fewer trips than it is unrolled by loads one after the other)
  if (have)
    for (int k0 = q; k0 < nsplit; k0 += 8 * Q) {
      float4 t[8];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (k0 + k * Q < nsplit) t[k] = p[(long long)(k0 + k * Q) * L * size4];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (k0 + k * Q < nsplit) { s.x += t[k].x; s.y += t[k].y; s.z += t[k].z; s.w += t[k].w; }
    }
  if constexpr (Q > 1) {
    sh[q][c] = s;
    __syncthreads();
    if (q > 0) return;
#pragma unroll
    for (int k = 1; k < Q; ++k) { const float4 t = sh[k][c]; s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w; }
  }
  if (have) *reinterpret_cast<float4*>(dW + (long long)l * dw_stride + 4 * i) = s;
}
void launch_sum_splits(const float* part, float* dW, long long dw_stride, long long size, int L, int nsplit, hipStream_t st) {
  if (size % 4 != 0 || dw_stride % 4 != 0 || ((uintptr_t)dW & 15) != 0 || ((uintptr_t)part & 15) != 0)
    return launch_fail("sum of row splits: sizes and pointers must be multiples of 16 bytes");
  const long long tot = size / 4 * L;
  if (tot == 0) return;
  // (few elements: four threads each.  16 taps of 64 x 128 in 32 splits 8.0 -> 5.5 us)
  if (split_chains(size * L, nsplit) == 4)
    hipLaunchKernelGGL(sum_splits_kernel<4>, dim3((unsigned)((tot + 63) / 64)), dim3(256), 0, st, part, dW, dw_stride, size / 4, L, nsplit);
  else
    hipLaunchKernelGGL(sum_splits_kernel<1>, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, part, dW, dw_stride, size / 4, L, nsplit);
}

__global__ void tile_prefix_kernel(const int* offs, int L, int rps, int tile_rows, int* tpre) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    int run = 0;
    for (int l = 0; l < L; ++l) {
      tpre[l] = run;
      run += ((offs[l + 1] - offs[l]) * rps + tile_rows - 1) / tile_rows;
    }
    tpre[L] = run;
  }
}
void launch_tile_prefix(const int* offs, int L, int rps, int tile_rows, int* tpre, hipStream_t st) {
  hipLaunchKernelGGL(tile_prefix_kernel, dim3(1), dim3(64), 0, st, offs, L, rps, tile_rows, tpre);
}

// ---------------------------------------------------------------------------------------------------------
// staging: gather through perm, NCHW fp32 -> NHWC storage type; z | one-hot | zero padding
// ---------------------------------------------------------------------------------------------------------

// The blocks behind those of the noise name the model of every tile of every geometry, which needs nothing but the routing either:
// 256 tiles of a geometry each (a launch of its own took 3.4-5 us).
template <typename T>
__global__ __launch_bounds__(256) void stage_noise_kernel(const float* __restrict__ noise, const int* __restrict__ label_ids, int n, int L,
                                                          int zdim, int cond_g, int kp, T* __restrict__ zin, RouteBuffers rb, int noise_blocks,
                                                          int tile_blocks) {
  if ((int)blockIdx.x >= noise_blocks) {
    const int b = (int)blockIdx.x - noise_blocks, g = b / tile_blocks;
    tile_model(rb.tpre + (long long)g * (L + 1), L, rb.tmodel + (long long)g * rb.tmodel_stride, rb.tmodel_stride,
               (b - g * tile_blocks) * 256 + (int)threadIdx.x);
    return;
  }
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;   // (j, k)
  if (idx >= (long long)n * kp) return;
  const int j = (int)(idx / kp), k = (int)(idx - (long long)j * kp);
  if (j >= rb.offs[L]) return;
  zin[idx] = staged_noise<T>(noise, label_ids, rb.perm[j], k, zdim, cond_g);
}

// Elements of one model's noise rows up to which the routing's block stages them itself: four a thread.  2048 elements: 5.6 us for both,
// 4.2 and 3.0 in launches of their own; 8192 elements: 11.5, 4.8 and 3.5.
constexpr int STAGE_INSIDE = 4 * ROUTE_THREADS;
template <typename T>
void launch_route_stage(const int* label_ids, const float* noise, int n, int L, int n_labels, int zdim, int cond_g, int kp, const GeomTable& geoms,
                        const RouteBuffers& rb, T* zin, hipStream_t st) {
  int bits = 0;
  while (bits < 31 && (1 << bits) < L) ++bits;
  const bool inside = L == 1 && (long long)n * kp <= STAGE_INSIDE;
  const StageTail<T> tail = {inside ? noise : nullptr, zin, zdim, cond_g, kp};
  const size_t lds = ((size_t)(2 + ROUTE_WAVES) * L + 1) * 4;
  const auto go = [&](auto kernel, size_t bytes) {
    if (bytes > 48 * 1024)   // above the default dynamic limit: ask for it (idempotent, cheap)
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    hipLaunchKernelGGL(kernel, dim3(1), dim3(ROUTE_THREADS), bytes, st, label_ids, n, L, n_labels, bits, geoms, rb, tail);
  };
  if (lds <= (size_t)ROUTE_LDS_BYTES) go(&route_kernel<true, T>, lds);
  else go(&route_kernel<false, T>, 0);
  if (n == 0 || inside) return;
  const long long noise_blocks = ((long long)n * kp + 255) / 256;
  const int tile_blocks = (rb.tmodel_stride + 255) / 256;
  const long long blocks = noise_blocks + (L > 1 ? (long long)tile_blocks * geoms.n : 0);      // (one model's tiles need no table)
  if (blocks >= (1LL << 31)) return launch_fail("staging: more blocks than a launch can have");
  hipLaunchKernelGGL((stage_noise_kernel<T>), dim3((unsigned)blocks), dim3(256), 0, st, noise, label_ids, n, L, zdim, cond_g, kp, zin, rb,
                     (int)noise_blocks, tile_blocks);
}
template void launch_route_stage<float>(const int*, const float*, int, int, int, int, int, int, const GeomTable&, const RouteBuffers&, float*, hipStream_t);
template void launch_route_stage<bf16_t>(const int*, const float*, int, int, int, int, int, int, const GeomTable&, const RouteBuffers&, bf16_t*, hipStream_t);

// ---------------------------------------------------------------------------------------------------------
// BatchNorm
// ---------------------------------------------------------------------------------------------------------

// Loads 4 consecutive channels as floats.
__device__ inline void load4(const float* p, float (&v)[4]) {
  const float4 t = *reinterpret_cast<const float4*>(p);
  v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
__device__ inline void load4(const bf16_t* p, float (&v)[4]) {
  const uint2 t = *reinterpret_cast<const uint2*>(p);
  v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
  v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
}
__device__ inline void store4(float* p, const float (&v)[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
__device__ inline void store4(bf16_t* p, const float (&v)[4]) {
  uint2 t;
  t.x = pack2_bf16(v[0], v[1]);
  t.y = pack2_bf16(v[2], v[3]);
  *reinterpret_cast<uint2*>(p) = t;
}

// 16 bytes of consecutive channels as floats: 4 (fp32) or 8 (bf16).
template <typename T> struct Vec16 { static constexpr int N = 16 / (int)sizeof(T); };
__device__ inline void loadv(const float* p, float (&v)[4]) { load4(p, v); }
__device__ inline void loadv(const bf16_t* p, float (&v)[8]) {
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  const u4 t = __builtin_nontemporal_load(reinterpret_cast<const u4*>(p));
  v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
  v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
  v[4] = __uint_as_float(t.z << 16); v[5] = __uint_as_float(t.z & 0xffff0000u);
  v[6] = __uint_as_float(t.w << 16); v[7] = __uint_as_float(t.w & 0xffff0000u);
}
// EPV consecutive per-channel parameters (channel counts and the layout of the parameter blocks keep them 16-byte aligned)
template <int N> __device__ inline void load_params(const float* p, float (&v)[N]) {
#pragma unroll
  for (int k = 0; k < N; k += 4) {
    const float4 t = *reinterpret_cast<const float4*>(p + k);
    v[k] = t.x; v[k + 1] = t.y; v[k + 2] = t.z; v[k + 3] = t.w;
  }
}
__device__ inline void store_cached(float* p, const float (&v)[4]) { store4(p, v); }        // (through the caches, for a tensor that is read next)
__device__ inline void store_cached(bf16_t* p, const float (&v)[8]) {
  *reinterpret_cast<uint4*>(p) = make_uint4(pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3]), pack2_bf16(v[4], v[5]), pack2_bf16(v[6], v[7]));
}
__device__ inline void storev(float* p, const float (&v)[4]) { store4(p, v); }
__device__ inline void storev(bf16_t* p, const float (&v)[8]) {
  uint4 t;
  t.x = pack2_bf16(v[0], v[1]);
  t.y = pack2_bf16(v[2], v[3]);
  t.z = pack2_bf16(v[4], v[5]);
  t.w = pack2_bf16(v[6], v[7]);
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  u4 q; q.x = t.x; q.y = t.y; q.z = t.z; q.w = t.w;
  __builtin_nontemporal_store(q, reinterpret_cast<u4*>(p));
}

// mean / var / rstd from what the producing GEMM left per sub-tile and column: (sum, sum of squared deviations from
// the sub-tile's mean); a tile of tile_rows rows is wsplit sub-tiles of tile_rows / wsplit rows, the last ones of a
// model's last tile possibly empty.  Sub-tiles (and output phases, and column runs) of one (segment, model) are added
// in a fixed order in double:  N mean = sum s_t,  N var = sum (M2_t + s_t^2 / n_t) - (sum s_t)^2 / N.
// The GEMM's N columns are `groups` runs of the C channels (the linear layer feeding G's first BatchNorm has one
// run per pixel of the first feature map; the convolutions have one).
// A block = CX channels x SL slices of one model's entries: phase sl % nphase, of that phase every (SL / nphase)-th (sub-tile, column run)
// from sl / nphase on; first of the first segment, then of the second: with both in one block it also updates the running statistics.
// Bound by the latency of the entries' loads, which plain sums leave independent of each other (eight in flight); as a chain of pairwise
// merges in fp32, a division each, the launches of one step took 135 us of a 2774 us step (one 32x32 pair, 1000 images) and 62 of 574
// (one 28x28 pair, 64 images), now 54 and 21.
// Threads of a block: 16 channels x 16 slices as a rule; 64 slices, or 128 of 8 channels, when a model has so many entries that
// sixteen slices would be long and a launch has few blocks (one pair over the whole batch).  The choice follows from
// the configuration (tile bound per model at the sizing batch), never from a call's batch.
template <int SL, int CX>
__global__ __launch_bounds__(SL * CX) void bn_stats_from_partial_kernel(NormArgs a, const float* __restrict__ partial,
                                                                        const int* __restrict__ tpre, int ub_tiles, int nphase,
                                                                        int groups, unsigned groups_inv, int tile_rows, int gemm_rps, int wsplit) {
  constexpr int WAVES = SL * CX / 64;
  __shared__ double sh[2][WAVES][CX][2];
  const int cx = threadIdx.x % CX, sl = threadIdx.x / CX;
  const int cblocks = (a.C + CX - 1) / CX;
  const int c = (blockIdx.x % cblocks) * CX + cx;
  const int l = blockIdx.x / cblocks;
  const int cnt = a.offs[l + 1] - a.offs[l];
  if (cnt == 0) return;                                // block-uniform
  const int rows = cnt * gemm_rps;                     // rows of this model in the GEMM's row space (per phase)
  const int sub_rows = tile_rows / wsplit, nsub = (rows + sub_rows - 1) / sub_rows;      // sub-tiles that hold rows: the others are never written
  const int seq = nsub * groups;                       // entries of a phase, the column runs fastest
  const int ph = sl & (nphase - 1), first = sl / nphase, step = SL / nphase;
  const double inv_sub = 1.0 / (double)sub_rows, inv_last = 1.0 / (double)(rows - (nsub - 1) * sub_rows);
  const long long row_len = (long long)a.C * groups;
  for (int sidx = 0; sidx < a.nseg; ++sidx) {
    const float2* const p = reinterpret_cast<const float2*>(partial) +
                            (((long long)ph * a.nseg + sidx) * ub_tiles * wsplit + (long long)tpre[l] * wsplit) * row_len + min(c, a.C - 1);
    double s = 0, q2 = 0;
    for (int e0 = first; e0 < seq; e0 += 8 * step) {
      float2 v[8];
      int t[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int e = min(e0 + k * step, seq - 1);
        t[k] = groups_inv ? (int)__umulhi((unsigned)e, groups_inv) : e;      // e / groups, or one more
        if (t[k] * groups > e) --t[k];
        v[k] = p[t[k] * row_len + (long long)(e - t[k] * groups) * a.C];
      }
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (e0 + k * step < seq) {
          const double st = v[k].x;
          s += st;
          q2 += (double)v[k].y + st * st * (t[k] + 1 < nsub ? inv_sub : inv_last);
        }
    }
#pragma unroll
    for (int d = CX; d < 64; d <<= 1) {
      s += __shfl_xor(s, d, 64);
      q2 += __shfl_xor(q2, d, 64);
    }
    if ((threadIdx.x & 63) < CX) {
      sh[sidx][threadIdx.x >> 6][cx][0] = s;
      sh[sidx][threadIdx.x >> 6][cx][1] = q2;
    }
  }
  __syncthreads();
  if (sl != 0 || c >= a.C) return;
  const double N = (double)rows * nphase * groups;
  const long long S = (long long)cnt * a.rps;
  const long long ro = (long long)l * a.rstride + c;
  float rm = 0.f, rv = 0.f;
  if (a.fold_running) { rm = a.run_mean[ro]; rv = a.run_var[ro]; }
  for (int sidx = 0; sidx < a.nseg; ++sidx) {
    double s = 0, q2 = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) { s += sh[sidx][w][cx][0]; q2 += sh[sidx][w][cx][1]; }
    const double m = s / N;
    const double dev = (q2 - s * m) / N;
    const float mean = (float)m, var = (float)(dev < 0.0 ? 0.0 : dev);     // (a NaN stays one: fmax would make it 0)
    const long long o = (long long)((a.seg_first + sidx) * a.L + l) * a.C + c;
    a.mean[o] = mean;
    a.var[o] = var;
    a.rstd[o] = 1.0f / sqrtf(var + a.eps);
    rm = (1.f - a.momentum) * rm + a.momentum * mean;
    if (S > 1) rv = (1.f - a.momentum) * rv + a.momentum * var * ((float)S / (float)(S - 1));
  }
  if (a.fold_running) { a.run_mean[ro] = rm; a.run_var[ro] = rv; }     // what bn_running_kernel would do next, without the launch
}
void launch_bn_stats_from_partial(const NormArgs& a, const float* partial, const int* tpre, int ub_tiles, int size_tiles, int nphase,
                                  int groups, int tile_rows, int gemm_rps, int wsplit, hipStream_t st) {
  if ((long long)a.nseg * a.L * a.C == 0) return;
  if (!tpre || !partial) return launch_fail("BatchNorm statistics: no tile prefix array or no partial sums");
  if (a.nseg > 2) return launch_fail("BatchNorm statistics: more than two segments");
  if (wsplit < 1 || tile_rows % wsplit) return launch_fail("BatchNorm statistics: the tile height is not a whole number of sub-tiles");
  if (nphase != 1 && nphase != 4) return launch_fail("BatchNorm statistics: one output phase or four");
  // ceil(2^32 / groups): the high half of its product with an entry's number is the quotient, or one more from number * groups = 2^32 on
  const unsigned inv = groups > 1 ? (unsigned)(((1ULL << 32) + groups - 1) / groups) : 0;
  const auto go = [&](auto kernel, int sl, int cx) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)(a.L * ((a.C + cx - 1) / cx))), dim3(sl * cx), 0, st, a, partial, tpre, ub_tiles, nphase, groups,
                       inv, tile_rows, gemm_rps, wsplit);
  };
  const double entries = (double)size_tiles * wsplit * nphase * groups / a.L;     // per model, at the sizing batch
  if (entries > 1024) go(&bn_stats_from_partial_kernel<128, 8>, 128, 8);
  else if (entries > 128) go(&bn_stats_from_partial_kernel<64, 16>, 64, 16);
  else go(&bn_stats_from_partial_kernel<16, 16>, 16, 16);
}

// running <- (1 - momentum) running + momentum * batch, once per segment in order; unbiased variance stored.
__global__ void bn_running_kernel(NormArgs a) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= a.L * a.C) return;
  const int l = idx / a.C, c = idx - l * a.C;
  const int cnt = a.offs[l + 1] - a.offs[l];
  if (cnt == 0) return;
  const long long S = (long long)cnt * a.rps;
  float rm = a.run_mean[(long long)l * a.rstride + c], rv = a.run_var[(long long)l * a.rstride + c];
  for (int s = 0; s < a.nseg; ++s) {
    const long long o = (long long)((a.seg_first + s) * a.L + l) * a.C + c;
    rm = (1.f - a.momentum) * rm + a.momentum * a.mean[o];
    if (S > 1) rv = (1.f - a.momentum) * rv + a.momentum * a.var[o] * ((float)S / (float)(S - 1));
  }
  a.run_mean[(long long)l * a.rstride + c] = rm;
  a.run_var[(long long)l * a.rstride + c] = rv;
}
void launch_bn_running(const NormArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(bn_running_kernel, dim3((a.L * a.C + 255) / 256), dim3(256), 0, st, a);
}

// Blocks that share a sample in the two apply passes: one, unless the samples alone are too few blocks to fill the chip.
// One 28x28 pair of 64 samples, 12544 values each: 64 blocks take 6.8-7.6 us a pass, 4.0-5.0 us with shared samples.
static unsigned apply_split(const NormArgs& a, int epv) {
  const long long blocks = (long long)a.n * a.nseg, most = ((long long)a.rps * a.C / epv + 255) / 256;
  return (unsigned)std::max(1LL, std::min(1024 / blocks, most));
}
// The rows of a sample that a thread of the apply passes takes, in 16-byte channel groups, cg of them a row.  Its group is fixed when the threads
// of a sample's blocks are a multiple of cg (the usual case), and U rows are then taken at a time, so that their loads are on their way together;
// otherwise the group changes from row to row and its parameters are loaded again.
// Row by row a thread had one or two loads on their way.  A hundred 32x32 pairs in bf16, GB/s: forward 5507 -> 5783, backward 5669 -> 5987; eight 64x64
// pairs 4702 -> 4820, 5021 -> 5120.  (Four rows: the backward pass with an activation in front, PRE, gets slower, 5033 -> 4776 with the whole of the
// tables' networks, so two there.)
template <int U, int NT = 256, typename P, typename R>
__device__ __forceinline__ void walk_rows(int rps, int cg, P&& params, R&& rows) {
  const int step = NT * gridDim.z, total = rps * cg;
  int t = blockIdx.z * NT + threadIdx.x;
  if (t >= total) return;
  if (step % cg == 0) {
    const int dr = step / cg, g = t % cg;
    int r = t / cg;
    params(g);
    for (; r + (U - 1) * dr < rps; r += U * dr) rows(std::integral_constant<int, U>{}, r, dr, g);
    for (; r < rps; r += dr) rows(std::integral_constant<int, 1>{}, r, dr, g);
  } else {
    for (; t < total; t += step) {
      const int r = t / cg, g = t - r * cg;
      params(g);
      rows(std::integral_constant<int, 1>{}, r, 0, g);
    }
  }
}
// y = act(gamma * (x - mean) * rstd + beta).  One block (or gridDim.z of them) per (sample, segment): a thread keeps the parameters of its
// 16 bytes of channels in registers and walks down the sample's rows.
template <typename T>
__global__ __launch_bounds__(256) void bn_apply_kernel(NormArgs a) {
  constexpr int EPV = Vec16<T>::N;
  const int j = blockIdx.x, sidx = blockIdx.y;
  if (j >= a.offs[a.L]) return;
  const int l = a.sample_model[j];
  const int seg = a.seg_first + sidx;
  const int cg = a.C / EPV;                           // channel groups per row
  const long long base = ((long long)seg * a.seg_samples + j) * a.rps * a.C;
  const T* x = static_cast<const T*>(a.x) + base;
  T* y = static_cast<T*>(a.y) + base;
  const long long so = (long long)(seg * a.L + l) * a.C;
  float sc[EPV], mu[EPV], be[EPV];
  walk_rows<4>(a.rps, cg, [&](int g) __attribute__((always_inline)) {
    float rs[EPV];
    load_params(a.gamma + (long long)l * a.pstride + g * EPV, sc);
    load_params(a.rstd + so + g * EPV, rs);
    load_params(a.mean + so + g * EPV, mu);
    load_params(a.beta + (long long)l * a.pstride + g * EPV, be);
#pragma unroll
    for (int k = 0; k < EPV; ++k) sc[k] *= rs[k];
  }, [&](auto count, int r, int dr, int g) __attribute__((always_inline)) {
    constexpr int U = decltype(count)::value;
    float v[U][EPV];
#pragma unroll
    for (int i = 0; i < U; ++i) loadv(x + (long long)(r + i * dr) * a.C + g * EPV, v[i]);
#pragma unroll
    for (int i = 0; i < U; ++i) {
#pragma unroll
      for (int k = 0; k < EPV; ++k) {
        const float u = (v[i][k] - mu[k]) * sc[k] + be[k];
        v[i][k] = u > 0.f ? u : u * a.slope;
      }
      storev(y + (long long)(r + i * dr) * a.C + g * EPV, v[i]);
    }
  });
}
template <typename T> void launch_bn_apply(const NormArgs& a, hipStream_t st) {
  if (a.n == 0 || a.nseg == 0) return;
  hipLaunchKernelGGL((bn_apply_kernel<T>), dim3((unsigned)a.n, (unsigned)a.nseg, apply_split(a, Vec16<T>::N)), dim3(256), 0, st, a);
}
template void launch_bn_apply<float>(const NormArgs&, hipStream_t);
template void launch_bn_apply<bf16_t>(const NormArgs&, hipStream_t);

// sums[g][c] = (sum g, sum g * xhat) with g = dy * act'(u), u = gamma * xhat + beta.
// Stage 1: block (tile of red_rows rows of one model, segment), all channels -> partial[segment][tile][C][2].
// Stage 2: the tiles of a (segment, model) added in a fixed order.
template <typename T>
__global__ __launch_bounds__(256) void bn_bwd_reduce_kernel(NormArgs a, const int* __restrict__ tpre, const int* __restrict__ tmodel,
                                                            int ub_tiles, float* __restrict__ partial) {
  constexpr int EPV = Vec16<T>::N;
  extern __shared__ float red[];                    // [2][RL][C]
  const int tile = blockIdx.x;
  if (tile >= tpre[a.L]) return;
  int lo = 0;
  if (tmodel) {
    lo = tmodel[tile];
  } else {
    int hi = a.L;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (tpre[mid] <= tile) lo = mid; else hi = mid;
    }
  }
  const int l = lo, sidx = blockIdx.y;
  const int seg = a.seg_first + sidx;
  const int cnt = a.offs[l + 1] - a.offs[l];
  const int g = seg * a.L + l;
  const int cg = a.C / EPV;                         // channel lanes (<= 256, a divisor of 256 or not)
  const int RL = 256 / cg;                          // row lanes
  const int cl = threadIdx.x % cg, rl = threadIdx.x / cg;
  const long long rows = (long long)cnt * a.rps;
  const long long r0 = (long long)(tile - tpre[l]) * a.red_rows;
  const long long r1 = min(rows, r0 + a.red_rows);
  const long long base = ((long long)seg * a.seg_samples + a.offs[l]) * a.rps * a.C + cl * EPV;
  const T* x = static_cast<const T*>(a.x) + base;
  const T* dy = static_cast<const T*>(a.dy) + base;
  float mu[EPV], rs[EPV], ga[EPV], be[EPV], sg[EPV], sgx[EPV];
  load_params(a.mean + (long long)g * a.C + cl * EPV, mu);
  load_params(a.rstd + (long long)g * a.C + cl * EPV, rs);
  load_params(a.gamma + (long long)l * a.pstride + cl * EPV, ga);
  load_params(a.beta + (long long)l * a.pstride + cl * EPV, be);
#pragma unroll
  for (int e = 0; e < EPV; ++e) {
    sg[e] = 0.f;
    sgx[e] = 0.f;
  }
  if (rl < RL) {
    // four rows per trip: eight 16-byte loads in flight per thread (the sums stay in row order)
    long long r = r0 + rl;
    for (; r + 3 * RL < r1; r += 4 * RL) {
      float v[4][EPV], d[4][EPV];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        loadv(x + (r + k * RL) * a.C, v[k]);
        loadv(dy + (r + k * RL) * a.C, d[k]);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
          const float xh = (v[k][e] - mu[e]) * rs[e];
          const float u = ga[e] * xh + be[e];
          const float gg = u > 0.f ? d[k][e] : d[k][e] * a.slope;
          sg[e] += gg;
          sgx[e] += gg * xh;
        }
    }
    for (; r < r1; r += RL) {
      float v[EPV], d[EPV];
      loadv(x + r * a.C, v);
      loadv(dy + r * a.C, d);
#pragma unroll
      for (int e = 0; e < EPV; ++e) {
        const float xh = (v[e] - mu[e]) * rs[e];
        const float u = ga[e] * xh + be[e];
        const float gg = u > 0.f ? d[e] : d[e] * a.slope;
        sg[e] += gg;
        sgx[e] += gg * xh;
      }
    }
#pragma unroll
    for (int e = 0; e < EPV; ++e) {
      red[(0 * RL + rl) * a.C + cl * EPV + e] = sg[e];
      red[(1 * RL + rl) * a.C + cl * EPV + e] = sgx[e];
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < 2 * a.C; t += 256) {
    const int w = t / a.C, c = t - w * a.C;
    float acc = 0.f;
    for (int i = 0; i < RL; ++i) acc += red[(w * RL + i) * a.C + c];
    partial[(((long long)sidx * ub_tiles + tile) * a.C + c) * 2 + w] = acc;
  }
}
// (SL slices x 16 channels of one model, slice s adding every SL-th tile from s on: 16, or 64 when a model has many tiles at the sizing
// batch (the call's own batch may not decide, or the order of a model's sums would follow the other models' samples); both segments
// in one block, which with that also adds them up to the parameters' gradients)
template <int SL>
__global__ __launch_bounds__(SL * 16) void bn_bwd_reduce_final_kernel(NormArgs a, const int* __restrict__ tpre, int ub_tiles,
                                                                      const float* __restrict__ partial) {
  __shared__ float sh[2][SL / 4][16][2];
  const int cx = threadIdx.x & 15, sl = threadIdx.x >> 4;
  const int cblocks = (a.C + 15) / 16;
  const int c = (blockIdx.x % cblocks) * 16 + cx;
  const int l = blockIdx.x / cblocks;
  if (a.offs[l + 1] == a.offs[l]) return;              // block-uniform
  const int t0 = tpre[l], t1 = tpre[l + 1];
  for (int sidx = 0; sidx < a.nseg; ++sidx) {
    float s0 = 0.f, s1 = 0.f;
    const float2* const p = reinterpret_cast<const float2*>(partial) + (long long)sidx * ub_tiles * a.C + min(c, a.C - 1);
    for (int t = t0 + sl; t < t1; t += 8 * SL) {       // (eight tiles' loads in flight, added in order)
      float2 e[8];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (t + k * SL < t1) e[k] = p[(long long)(t + k * SL) * a.C];
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (t + k * SL < t1) {
          s0 += e[k].x;
          s1 += e[k].y;
        }
    }
#pragma unroll
    for (int d = 16; d < 64; d <<= 1) {
      s0 += __shfl_xor(s0, d, 64);
      s1 += __shfl_xor(s1, d, 64);
    }
    if ((threadIdx.x & 63) < 16) { sh[sidx][threadIdx.x >> 6][cx][0] = s0; sh[sidx][threadIdx.x >> 6][cx][1] = s1; }
  }
  __syncthreads();
  if (sl != 0 || c >= a.C) return;
  float db = 0.f, dg = 0.f;
  for (int sidx = 0; sidx < a.nseg; ++sidx) {
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int k = 0; k < SL / 4; ++k) { s0 += sh[sidx][k][cx][0]; s1 += sh[sidx][k][cx][1]; }
    const long long o = ((long long)((a.seg_first + sidx) * a.L + l) * a.C + c) * 2;
    a.sums[o] = s0;
    a.sums[o + 1] = s1;
    db += s0;
    dg += s1;
  }
  if (a.param_grads) {
    a.dbeta[(long long)l * a.pstride + c] = db;
    a.dgamma[(long long)l * a.pstride + c] = dg;
  }
}
// Rows a block of the first stage sums: 256, or 64 where those leave the chip short of blocks.  One 32x32 pair of 1000 images, both
// stages, 256 rows against 64: 16000 rows of 512 channels 28 us and 15, 64000 of 256 20 and 21.  By the sizing batch, never a call's.
int bn_red_rows(long long rows, int L) { return rows / 256 + L < 192 ? 64 : 256; }
void launch_bn_bwd_final(const NormArgs& a, const int* tpre, int ub_tiles, const float* partial, hipStream_t st) {
  if (a.nseg == 0 || ub_tiles == 0) return;
  if (!tpre || !partial || a.red_tiles < ub_tiles || a.nseg > 2)
    return launch_fail("BatchNorm backward: no tile prefix array, no partial sums, more tiles than at the sizing batch, or more than two segments");
  const long long tot = (long long)a.L * ((a.C + 15) / 16);
  if (a.red_tiles > 64LL * a.L) hipLaunchKernelGGL(bn_bwd_reduce_final_kernel<64>, dim3((unsigned)tot), dim3(1024), 0, st, a, tpre, ub_tiles, partial);
  else hipLaunchKernelGGL(bn_bwd_reduce_final_kernel<16>, dim3((unsigned)tot), dim3(256), 0, st, a, tpre, ub_tiles, partial);
}
template <typename T>
void launch_bn_bwd_reduce(const NormArgs& a, const int* tpre, const int* tmodel, int ub_tiles, float* partial, hipStream_t st) {
  if (a.nseg == 0 || ub_tiles == 0) return;
  if (!tpre || a.red_rows < 1 || a.nseg > 2) return launch_fail("BatchNorm backward: no tile prefix array, no tile height, or more than two segments");
  const int cg = a.C / Vec16<T>::N;
  if (cg < 1 || cg > 256) return launch_fail("BatchNorm backward: one thread per 16 bytes of a row needs at most 256 of them");
  const size_t lds = (size_t)2 * (256 / cg) * a.C * sizeof(float);
  hipLaunchKernelGGL((bn_bwd_reduce_kernel<T>), dim3(ub_tiles, a.nseg), dim3(256), lds, st, a, tpre, tmodel, ub_tiles, partial);
  launch_bn_bwd_final(a, tpre, ub_tiles, partial, st);
}
template void launch_bn_bwd_reduce<float>(const NormArgs&, const int*, const int*, int, float*, hipStream_t);
template void launch_bn_bwd_reduce<bf16_t>(const NormArgs&, const int*, const int*, int, float*, hipStream_t);

// dx = gamma * rstd * (g - sum_g / S - xhat * sum_gx / S).  Same block shape as the forward pass.
template <typename T, bool PRE>
__global__ __launch_bounds__(256) void bn_bwd_apply_kernel(NormArgs a) {
  constexpr int EPV = Vec16<T>::N;
  const int j = blockIdx.x, sidx = blockIdx.y;
  if (j >= a.offs[a.L]) return;
  const int l = a.sample_model[j];
  const int seg = a.seg_first + sidx;
  const int cg = a.C / EPV;
  const float invS = 1.0f / ((float)(a.offs[l + 1] - a.offs[l]) * (float)a.rps);
  const long long base = ((long long)seg * a.seg_samples + j) * a.rps * a.C;
  const T* x = static_cast<const T*>(a.x) + base;
  const T* dy = static_cast<const T*>(a.dy) + base;
  T* dx = static_cast<T*>(a.y) + base;
  const long long so = (long long)(seg * a.L + l) * a.C;
  float rs[EPV], ga[EPV], mu[EPV], be[EPV], s1[EPV], s2[EPV];
  walk_rows<PRE ? 2 : 4>(a.rps, cg, [&](int g) __attribute__((always_inline)) {
    float ss[2 * EPV];
    load_params(a.rstd + so + g * EPV, rs);
    load_params(a.gamma + (long long)l * a.pstride + g * EPV, ga);
    load_params(a.mean + so + g * EPV, mu);
    load_params(a.beta + (long long)l * a.pstride + g * EPV, be);
    load_params(a.sums + (so + g * EPV) * 2, ss);
#pragma unroll
    for (int k = 0; k < EPV; ++k) {
      s1[k] = ss[2 * k] * invS;
      s2[k] = ss[2 * k + 1] * invS;
    }
  }, [&](auto count, int r, int dr, int g) __attribute__((always_inline)) {
    constexpr int U = decltype(count)::value;
    float v[U][EPV], d[U][EPV];
#pragma unroll
    for (int i = 0; i < U; ++i) {
      loadv(x + (long long)(r + i * dr) * a.C + g * EPV, v[i]);
      loadv(dy + (long long)(r + i * dr) * a.C + g * EPV, d[i]);
    }
#pragma unroll
    for (int i = 0; i < U; ++i) {
#pragma unroll
      for (int k = 0; k < EPV; ++k) {
        const float xh = (v[i][k] - mu[k]) * rs[k];
        const float u = ga[k] * xh + be[k];
        const float gg = u > 0.f ? d[i][k] : d[i][k] * a.slope;
        float o = ga[k] * rs[k] * (gg - s1[k] - xh * s2[k]);
        if (PRE) {
          if (!(v[i][k] > 0.f)) o *= a.pre_slope;
          o = a.pre_drop && dropped(v[i][k]) ? 0.f : o * a.pre_scale;
        }
        v[i][k] = o;
      }
      storev(dx + (long long)(r + i * dr) * a.C + g * EPV, v[i]);
    }
  });
}
template <typename T> void launch_bn_bwd_apply(const NormArgs& a, hipStream_t st) {
  if (a.n == 0 || a.nseg == 0) return;
  const dim3 grid((unsigned)a.n, (unsigned)a.nseg, apply_split(a, Vec16<T>::N));
  if (a.pre_act) hipLaunchKernelGGL((bn_bwd_apply_kernel<T, true>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((bn_bwd_apply_kernel<T, false>), grid, dim3(256), 0, st, a);
}
template void launch_bn_bwd_apply<float>(const NormArgs&, hipStream_t);
template void launch_bn_bwd_apply<bf16_t>(const NormArgs&, hipStream_t);

// ---------------------------------------------------------------------------------------------------------
// D's linear head, the costs, and their gradients
// ---------------------------------------------------------------------------------------------------------

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ inline float softplus_f(float u) { return fmaxf(u, 0.f) + log1pf(expf(-fabsf(u))); }
__device__ inline float sigmoid_f(float u) {
  if (u >= 0.f) return 1.f / (1.f + expf(-u));
  const float e = expf(u);
  return e / (1.f + e);
}

// COST_D (Eq. 3): J_D = scale*mean softplus(-s_real) + scale*mean softplus(s_fake), segments (0, 1).  COST_G (Eq. 4, negated):
// scale*mean softplus(-s_fake') on segment seg_first.
__device__ inline float head_sign(const HeadArgs& a, int seg) { return a.cost == COST_D && seg == 1 ? 1.f : -1.f; }

// BatchNorm and activation of D's last feature map, its linear head and the cost's derivative: a block per (sample, segment) normalises as
// bn_apply_kernel does and multiplies what it stores with the head's weights.  The head read the stored tensor once more and was a launch of its own:
// a hundred 32x32 pairs, bf16, both segments 71 + 49 -> 101 us, one 38 + 27 -> 55; ten 28x28 pairs, fp32, 25 + 16 -> 28 and 14 + 11 -> 17; one 4.2 + 6.0 ->
// 6.4.  The head's weight gradient reads the tensor next, which past the caches takes it longer (ten pairs, bf16, 26 us for 17).
// A sample of few values (a 2 x 2 map of the tables' networks) is one wave's.  Large maps of few samples gain as well, though a sample is one block: the head
// was one wave a sample.  Both passes of a step, 8 samples of 16x16x128 in fp32 48 -> 22, 4 of 16x16x1024 234 -> 112, in bf16 274 -> 85.
template <typename T, int NT>
__global__ __launch_bounds__(NT) void bn_apply_head_kernel(NormArgs a, HeadArgs h) {
  constexpr int EPV = Vec16<T>::N;
  __shared__ float red[NT / 64];
  const int j = blockIdx.x, seg = a.seg_first + (int)blockIdx.y;
  if (j >= a.offs[a.L]) return;
  const int l = a.sample_model[j];
  const long long row = (long long)seg * a.seg_samples + j;
  const T* x = static_cast<const T*>(a.x) + row * h.K;
  T* y = static_cast<T*>(a.y) + row * h.K;
  const float* w = h.w + (long long)l * h.pstride;
  const long long so = (long long)(seg * a.L + l) * a.C;
  float sc[EPV], mu[EPV], be[EPV], acc = 0.f;
  walk_rows<4, NT>(a.rps, a.C / EPV, [&](int g) __attribute__((always_inline)) {
    float rs[EPV];
    load_params(a.gamma + (long long)l * a.pstride + g * EPV, sc);
    load_params(a.rstd + so + g * EPV, rs);
    load_params(a.mean + so + g * EPV, mu);
    load_params(a.beta + (long long)l * a.pstride + g * EPV, be);
#pragma unroll
    for (int k = 0; k < EPV; ++k) sc[k] *= rs[k];
  }, [&](auto count, int r, int dr, int g) __attribute__((always_inline)) {
    constexpr int U = decltype(count)::value;
    float v[U][EPV], ww[U][EPV];
#pragma unroll
    for (int i = 0; i < U; ++i) {
      loadv(x + (long long)(r + i * dr) * a.C + g * EPV, v[i]);
      load_params(w + (long long)(r + i * dr) * a.C + g * EPV, ww[i]);
    }
#pragma unroll
    for (int i = 0; i < U; ++i) {
#pragma unroll
      for (int k = 0; k < EPV; ++k) {
        const float u = (v[i][k] - mu[k]) * sc[k] + be[k];
        v[i][k] = u > 0.f ? u : u * a.slope;
        acc += to_float(from_float<T>(v[i][k])) * ww[i][k];
      }
      store_cached(y + (long long)(r + i * dr) * a.C + g * EPV, v[i]);
    }
  });
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    float sum = red[0];
#pragma unroll
    for (int i = 1; i < NT / 64; ++i) sum += red[i];
    const float logit = sum + h.b[(long long)l * h.pstride], sign = head_sign(h, seg);
    h.logits[row] = logit;
    h.dlogits[row] = h.scale * sign * sigmoid_f(sign * logit) * (1.f / (float)(a.offs[l + 1] - a.offs[l]));
  }
}
template <typename T> void launch_bn_apply_head(const NormArgs& a, const HeadArgs& h, hipStream_t st) {
  if (a.n == 0 || a.nseg == 0) return;
  if (h.K != a.rps * a.C || h.seg_first != a.seg_first || h.nseg != a.nseg || h.seg_samples != a.seg_samples)
    return launch_fail("linear head: its rows are not the normalised tensor's samples");
  const dim3 grid((unsigned)a.n, (unsigned)a.nseg);
  if (h.K / Vec16<T>::N <= 128) hipLaunchKernelGGL((bn_apply_head_kernel<T, 64>), grid, dim3(64), 0, st, a, h);
  else hipLaunchKernelGGL((bn_apply_head_kernel<T, 256>), grid, dim3(256), 0, st, a, h);
}
template void launch_bn_apply_head<float>(const NormArgs&, const HeadArgs&, hipStream_t);
template void launch_bn_apply_head<bf16_t>(const NormArgs&, const HeadArgs&, hipStream_t);

// One block per model: its cost, and the step count of the update that follows.
__device__ inline void head_loss(const HeadArgs& a, int l) {
  __shared__ float red[256];
  const int s0 = a.offs[l], cnt = a.offs[l + 1] - s0;
  if (cnt == 0) { if (threadIdx.x == 0) a.loss[l] = 0.f; return; }
  const float inv = 1.f / (float)cnt;
  float acc = 0.f;
  for (int s = 0; s < a.nseg; ++s) {
    const int seg = a.seg_first + s;
    const float sign = head_sign(a, seg);
    for (int i = threadIdx.x; i < cnt; i += 256) acc += softplus_f(sign * a.logits[(long long)seg * a.seg_samples + s0 + i]);
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    a.loss[l] = a.scale * red[0] * inv;
    // and its bias corrections (a launch of their own took 4.6 us)
    const int t = a.adam_t[l] + 1;
    a.adam_t[l] = t;
    a.adam_bc[2 * l] = (float)(1.0 - pow((double)a.beta1, (double)t));
    a.adam_bc[2 * l + 1] = (float)(1.0 - pow((double)a.beta2, (double)t));
  }
}

// dfeat[row][k] = dlogit[row] * w[model][k]; a thread takes 8 consecutive k of one row (K is a multiple of 8: the
// feature maps have whole 64-channel lines); 32-bit index arithmetic (the launcher checks).
template <typename T>
__device__ inline void head_data(const HeadArgs& a, int sidx, unsigned idx) {
  const unsigned k8 = (unsigned)a.K >> 3;
  const unsigned j = idx / k8;
  if (j >= (unsigned)a.n || (int)j >= a.offs[a.L]) return;
  const int k = (int)(idx - j * k8) * 8;
  const int l = a.sample_model[j];
  const long long r = (long long)(a.seg_first + sidx) * a.seg_samples + j;
  const float d = a.dlogits[r];
  const float* w = a.w + (long long)l * a.pstride + k;
  const float4 w0 = *reinterpret_cast<const float4*>(w), w1 = *reinterpret_cast<const float4*>(w + 4);
  const float v[8] = {d * w0.x, d * w0.y, d * w0.z, d * w0.w, d * w1.x, d * w1.y, d * w1.z, d * w1.w};
  T* dst = static_cast<T*>(a.dfeat) + r * a.K + k;
  if constexpr (sizeof(T) == 2) {
    storev(dst, v);
  } else {
    *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4*>(dst + 4) = make_float4(v[4], v[5], v[6], v[7]);
  }
}

// dw[model][k] = sum_rows dlogit[row] * feat[row][k] ; db = sum_rows dlogit.  Block (k chunk of 1024, model, row split).
template <typename T>
__device__ inline void head_weights(const HeadArgs& a, int kc, int l, int sp) {
  const int s0 = a.offs[l], cnt = a.offs[l + 1] - s0;
  if (cnt == 0) return;
  const int k = kc * 1024 + threadIdx.x * 4;
  const int rsplit = a.rsplit > 1 ? a.rsplit : 1;
  const int per = (cnt + rsplit - 1) / rsplit;
  const int i0 = sp * per, i1 = min(cnt, i0 + per);
  float acc[4] = {0, 0, 0, 0}, accb = 0.f;
  for (int s = 0; s < a.nseg; ++s) {
    const long long r0 = (long long)(a.seg_first + s) * a.seg_samples + s0;
#pragma unroll 8
    for (int i = i0; i < i1; ++i) {               // (eight rows' loads in flight, added in order)
      const float d = a.dlogits[r0 + i];
      accb += d;
      if (k < a.K) {
        float v[4];
        load4(static_cast<const T*>(a.feat) + (r0 + i) * a.K + k, v);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += d * v[e];
      }
    }
  }
  if (rsplit > 1) {
    float* part = a.part + ((long long)sp * a.L + l) * (a.K + 4);
    if (k < a.K) *reinterpret_cast<float4*>(part + k) = make_float4(acc[0], acc[1], acc[2], acc[3]);
    if (kc == 0 && threadIdx.x == 0) part[a.K] = accb;
    return;
  }
  if (k < a.K) *reinterpret_cast<float4*>(a.dw + (long long)l * a.pstride + k) = make_float4(acc[0], acc[1], acc[2], acc[3]);
  if (kc == 0 && threadIdx.x == 0) a.db[(long long)l * a.pstride] = accb;
}

// Everything that needs nothing but the logits and their derivatives, which the forward kernel leaves: the weight gradient's blocks first (they
// take longest), the costs', the data gradient's.  In small configurations every launch is 4 to 6 us whatever it does, and these
// were three: one 28x28 pair 425 -> 417 us a step, ten in bf16 1.8 % less, a hundred 32x32 pairs 0.5 %.
template <typename T>
__global__ __launch_bounds__(256) void head_bwd_kernel(HeadArgs a, int w_blocks, unsigned data_blocks) {
  const int b = (int)blockIdx.x;
  if (b < w_blocks) {
    const int kcs = (a.K + 1023) / 1024, q = b / kcs;
    head_weights<T>(a, b - q * kcs, q % a.L, q / a.L);
  } else if (b < w_blocks + a.L) {
    head_loss(a, b - w_blocks);
  } else {
    const unsigned q = (unsigned)(b - w_blocks - a.L), sidx = q / data_blocks;
    head_data<T>(a, (int)sidx, (q - sidx * data_blocks) * 256u + threadIdx.x);
  }
}
template <typename T> void launch_head_bwd(const HeadArgs& a, bool weights, hipStream_t st) {
  if (a.nseg == 0 || a.L == 0) return;
  const long long tot = (long long)a.n * (a.K / 8), data_blocks = (tot + 255) / 256;
  if (a.K % 8 != 0 || tot + 256 >= (1LL << 32)) return launch_fail("head data gradient: K must be a multiple of 8 and n * K / 8 below 2^32");
  if (weights && a.rsplit > 1 && !a.part) return launch_fail("linear head: no buffer for the row splits");
  const int rsplit = a.rsplit > 1 ? a.rsplit : 1;
  const long long w_blocks = weights ? (long long)((a.K + 1023) / 1024) * a.L * rsplit : 0, blocks = w_blocks + a.L + data_blocks * a.nseg;
  if (blocks >= (1LL << 31)) return launch_fail("linear head: more blocks than a launch can have");
  hipLaunchKernelGGL((head_bwd_kernel<T>), dim3((unsigned)blocks), dim3(256), 0, st, a, (int)w_blocks, (unsigned)data_blocks);
}
template void launch_head_bwd<float>(const HeadArgs&, bool, hipStream_t);
template void launch_head_bwd<bf16_t>(const HeadArgs&, bool, hipStream_t);

// ---------------------------------------------------------------------------------------------------------
// Adam (bias-corrected, epsilon outside the root), all models and tensors of one network in one sweep
// ---------------------------------------------------------------------------------------------------------

// streaming accesses of the optimiser state: every element is touched once per step
__device__ inline float4 ld_stream(const float* p) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  const f4 v = __builtin_nontemporal_load(reinterpret_cast<const f4*>(p));
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ inline void st_stream(float* p, const float4& v) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  f4 t; t.x = v.x; t.y = v.y; t.z = v.z; t.w = v.w;
  __builtin_nontemporal_store(t, reinterpret_cast<f4*>(p));
}
__device__ inline float adam_update1(const AdamArgs& a, float bc1, float bc2, float g, float th, float& m, float& v) {
  m = a.beta1 * m + (1.f - a.beta1) * g;
  v = a.beta2 * v + (1.f - a.beta2) * g * g;
  const float mh = m / bc1, vh = v / bc2;
  return th - a.lr * mh / (sqrtf(vh) + a.eps);
}
__device__ inline void adam_update4(const AdamArgs& a, float bc1, float bc2, const float4& g, float4& th, float4& m, float4& v,
                                    float (&tt)[4]) {
  tt[0] = adam_update1(a, bc1, bc2, g.x, th.x, m.x, v.x);
  tt[1] = adam_update1(a, bc1, bc2, g.y, th.y, m.y, v.y);
  tt[2] = adam_update1(a, bc1, bc2, g.z, th.z, m.z, v.z);
  tt[3] = adam_update1(a, bc1, bc2, g.w, th.w, m.w, v.w);
  th = make_float4(tt[0], tt[1], tt[2], tt[3]);
}

// The ranges between the tiled regions: block `block` of model l's.
template <typename T>
__device__ inline void adam_gap(const AdamArgs& a, const AdamImage& im, int l, int block) {
  if (a.counts[l] == 0) return;
  int r = 0;
  while (r + 1 < a.ngaps && block >= a.gap_blk0[r + 1]) ++r;
  const long long i = a.gap_lo[r] + ((long long)(block - a.gap_blk0[r]) * 256 + threadIdx.x) * 4;
  if (i >= a.gap_hi[r]) return;
  const long long o = (long long)l * a.P + i, in_image = i - im.w;
  const bool image = im.packed && in_image >= 0 && in_image < 16LL * im.CBT * im.Cs;
  int tap = 0, ch = 0, cs = 0;
  if (image) {
    const int row = (int)in_image / im.Cs;
    cs = (int)in_image - row * im.Cs;
    tap = row / im.CBT;
    ch = row - tap * im.CBT;
    if (im.add && ch >= im.CB && (a.L == 1 || ch - im.CB == l)) return;       // adam_label_maps's
  }
  const float4 g = ld_stream(a.g + o);
  float4 th = ld_stream(a.theta + o);
  float4 m = ld_stream(a.m + o);
  float4 v = ld_stream(a.v + o);
  float tt[4];
  adam_update4(a, a.bc[2 * l], a.bc[2 * l + 1], g, th, m, v, tt);
  st_stream(a.theta + o, th);
  st_stream(a.m + o, m);
  st_stream(a.v + o, v);
  if (a.shadow) store4(static_cast<bf16_t*>(a.shadow) + o, tt);
  if (image && ch < im.CB) {
    T* const d = static_cast<T*>(im.packed) + ((long long)l * im.Cs + cs) * 16 * im.P + tap * im.P + ch;
#pragma unroll
    for (int e = 0; e < 4; ++e) d[(long long)e * 16 * im.P] = from_float<T>(tt[e]);
  }
}
// The label map of one table at one feature channel: its sixteen taps, and what they add up to at the nine classes of positions.
template <typename T>
__device__ inline void adam_label_maps(const AdamArgs& a, const AdamImage& im, int idx) {
  if (idx >= im.tables * im.Cs) return;
  const int t = idx / im.Cs, cs = idx - t * im.Cs, l = a.L == 1 ? 0 : t;
  if (a.counts[l] == 0) return;
  const long long o = (long long)l * a.P + im.w + (long long)(im.CB + t) * im.Cs + cs, step = (long long)im.CBT * im.Cs;
  const float bc1 = a.bc[2 * l], bc2 = a.bc[2 * l + 1];
  float th[16];
#pragma unroll
  for (int k0 = 0; k0 < 16; k0 += 8) {                 // eight at a time: all sixteen in flight would take the registers of half the kernel's waves
    float g[8], m[8], v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const long long i = o + (k0 + k) * step;
      g[k] = a.g[i]; th[k0 + k] = a.theta[i]; m[k] = a.m[i]; v[k] = a.v[i];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const long long i = o + (k0 + k) * step;
      const float t = adam_update1(a, bc1, bc2, g[k], th[k0 + k], m[k], v[k]);
      th[k0 + k] = t;
      a.theta[i] = t; a.m[i] = m[k]; a.v[i] = v[k];
      if (a.shadow) static_cast<bf16_t*>(a.shadow)[i] = from_float<bf16_t>(t);
    }
  }
#pragma unroll
  for (int cls = 0; cls < 9; ++cls) im.add[((long long)t * 9 + cls) * im.Cs + cs] = label_class_sum<T>(th, cls);
}

// Four (eight) weights as bf16 parts, the planes `plane` elements apart.
__device__ inline void store_split4(unsigned short* p, long long plane, const float (&t)[4]) {
  unsigned h0, m0, l0, h1, m1, l1;
  split_pair(t[0], t[1], h0, m0, l0);
  split_pair(t[2], t[3], h1, m1, l1);
  *reinterpret_cast<uint2*>(p) = make_uint2(h0, h1);
  *reinterpret_cast<uint2*>(p + plane) = make_uint2(m0, m1);
  *reinterpret_cast<uint2*>(p + 2 * plane) = make_uint2(l0, l1);
}
__device__ inline void store_split8(unsigned short* p, long long plane, const uint4& lo, const uint4& hi) {
  const Split8 s = split8(__builtin_bit_cast(u32x4, lo), __builtin_bit_cast(u32x4, hi));
  *reinterpret_cast<u32x4*>(p) = s.h;
  *reinterpret_cast<u32x4*>(p + plane) = s.m;
  *reinterpret_cast<u32x4*>(p + 2 * plane) = s.l;
}
// One 64 (cb) x 64 (cs) tile of one tap of every model, as in the update below (which splits the weights it writes itself).
__global__ __launch_bounds__(256) void split_weights_kernel(SplitArgs a) {
  __shared__ __attribute__((aligned(16))) float tile[64][68];
  const int tcs_n = a.Cs >> 6, tcb_n = a.Cb >> 6, per = 16 * tcs_n * tcb_n;
  const int l = blockIdx.x / per;
  int q = blockIdx.x - l * per;
  const int tcs = q % tcs_n; q /= tcs_n;
  const int tcb = q % tcb_n, tap = q / tcb_n;
  const float* src = a.src + (long long)l * a.src_stride;
  const int c4 = (threadIdx.x & 15) * 4, r0 = threadIdx.x >> 4;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = r0 + 16 * i;
    const long long o = ((long long)tap * a.Cb + tcb * 64 + row) * a.Cs + tcs * 64 + c4;
    const float4 v = *reinterpret_cast<const float4*>(src + o);
    const float t[4] = {v.x, v.y, v.z, v.w};
    store_split4(a.up + 3 * (long long)l * a.plane + o, a.plane, t);
#pragma unroll
    for (int e = 0; e < 4; ++e) tile[c4 + e][row] = t[e];
  }
  if (!a.down) return;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int cid = threadIdx.x + 256 * i, cs = cid >> 3, ch = (cid & 7) * 8;
    store_split8(a.down + 3 * (long long)l * a.plane + ((long long)tap * a.Cs + tcs * 64 + cs) * a.Cb + tcb * 64 + ch, a.plane,
                 *reinterpret_cast<const uint4*>(&tile[cs][ch]), *reinterpret_cast<const uint4*>(&tile[cs][ch + 4]));
  }
}
void launch_split_weights(const SplitArgs& a, hipStream_t st) {
  if (!a.src || !a.up || a.Cb % 64 || a.Cs % 64 || a.src_stride % 4 || a.plane % 8) return launch_fail("split of the weights: channel counts or strides");
  const long long blocks = (long long)a.L * 16 * (a.Cb / 64) * (a.Cs / 64);
  if (blocks == 0) return;
  if (blocks >= (1LL << 31)) return launch_fail("split of the weights: more blocks than a launch can have");
  hipLaunchKernelGGL(split_weights_kernel, dim3((unsigned)blocks), dim3(256), 0, st, a);
}

// One 64 (cb) x 64 (cs) tile of one tap of a convolution weight: the update, the storage-type copy, and - through
// LDS - the transposed storage-type copy, so that the new weights are read from HBM once.  fp32 storage: both copies as bf16 parts (a
// quarter more to write: twenty 32x32 pairs 665 -> 806 us a step), which spares every GEMM block the split of its columns (8.1 -> 7.1 ms); with few rows
// a model the transposed copy in fp32 alone.
// The tables' discriminator, whose k3 filters of 16 and 32 channels are held as k4 ones of 64: nothing of the fourth taps and of the padded channels
// is read or written (a hundred pairs 136 -> 83 us a launch, and the four launches that cleared their gradients, 37 us, are gone).  The
// same for the padded columns of G's linear layer, 28 of every 128, is slower than updating them: 566 -> 633 us for the holes in the lines.
//
// SPLITS: the gradient comes as the row splits of its product (AdamSplits), which are added here, in split_chains sums, on their way and left in a.g.  A launch
// of its own read the splits, wrote the sum and had it read again: eight 64x64 pairs, 512 and 1024 tiles of 64 x 64, 23 + 31 -> 40 us and 18 + 29 -> 42;
// one 32x32 pair, 128 and 512 tiles, 14 + 9 -> 18 and 18 + 16 -> 29; one 28x28 pair, 32 tiles in 32 splits, 5 + 9 -> 10.
// ROWS: rows (cb) of a tile a block takes; with fewer than all 64 a launch of few tiles has four times the blocks.
__device__ __forceinline__ void add4(float4& s, const float4& t) { s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w; }
template <typename T, int ROWS, bool SPLITS>
__device__ inline void adam_tile(const AdamArgs& a, const AdamSplits& sp, unsigned block) {
  constexpr int TSTRIDE = ROWS * (int)sizeof(T) + 16;          // bytes per transposed row (ROWS cb)
  constexpr int NI = ROWS / 16, SUB = 64 / ROWS;
  __shared__ __attribute__((aligned(16))) unsigned char tile[64 * TSTRIDE];
  const int items = a.tile_count * SUB;                        // of a model
  const int l = (int)(block / (unsigned)items), item = (int)(block - (unsigned)(l * items));
  const bool moves = a.counts[l] != 0;
  if (!moves && !SPLITS) return;
  const int bx = item / SUB + a.tile_first, sub = (item % SUB) * ROWS;
  int r = 0;
  while (r + 1 < a.nregions && bx >= a.reg_tile0[r + 1]) ++r;
  const int Cb = a.reg_cb[r], Cs = a.reg_cs[r];
  const int tcs_n = Cs >> 6, tcb_n = Cb >> 6;
  int q = bx - a.reg_tile0[r];
  const int tcs = q % tcs_n; q /= tcs_n;
  const int tcb = q % tcb_n;
  const int tap = q / tcb_n;
  if (a.k3 && ((tap >> 2) == 3 || (tap & 3) == 3)) return;
  const int cb0 = tcb * 64 + sub, cb_real = a.reg_cb_real[r] - cb0, cs_real = a.reg_cs_real[r] - tcs * 64;      // inside the tile
  const long long base = (long long)l * a.P + a.reg_w[r], part = 3 * (long long)l * a.plane + a.reg_part[r];
  const float bc1 = a.bc[2 * l], bc2 = a.bc[2 * l + 1];
  const int c4 = (threadIdx.x & 15) * 4, r0 = threadIdx.x >> 4;
  const long long in0 = ((long long)tap * Cb + cb0 + r0) * Cs + tcs * 64 + c4, o0 = base + in0;
  float4 gs[NI], ths[NI], ms[NI], vs[NI];      // all loads first: a launch of few tiles is one memory latency, not four
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const long long o = o0 + 16LL * i * Cs;
    if (r0 + 16 * i >= cb_real || c4 >= cs_real) continue;
    if constexpr (!SPLITS) gs[i] = ld_stream(a.g + o);
    ths[i] = ld_stream(a.theta + o);
    ms[i] = ld_stream(a.m + o);
    vs[i] = ld_stream(a.v + o);
  }
  if constexpr (SPLITS) {                                       // (no padding: the caller's regions are whole)
    constexpr int DEEP = NI == 1 ? 12 : 4;                      // splits in flight (sixteen and the four sums would cost the gaps' blocks a fifth of their waves)
    float4 more[4] = {};                                        // (quarter tiles: the other three sums, where there are four)
    const bool four = NI == 1 && sp.chains == 4;
    const long long layer = 16LL * Cb * Cs, step = (long long)a.L * layer;
    const float* const p = sp.part + l * layer + in0;
#pragma unroll
    for (int i = 0; i < NI; ++i) gs[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k0 = 0; k0 < sp.n; k0 += DEEP) {
      float4 t[DEEP][NI];
#pragma unroll
      for (int k = 0; k < DEEP; ++k)
        if (k0 + k < sp.n) {
#pragma unroll
          for (int i = 0; i < NI; ++i) t[k][i] = ld_stream(p + (k0 + k) * step + 16LL * i * Cs);
        }
#pragma unroll
      for (int k = 0; k < DEEP; ++k)
        if (k0 + k < sp.n) {
#pragma unroll
          for (int i = 0; i < NI; ++i)
            if (four && k % 4 > 0) add4(more[k % 4 - 1], t[k][i]); else add4(gs[i], t[k][i]);
        }
    }
    if (four)
#pragma unroll
      for (int k = 0; k < 3; ++k) add4(gs[0], more[k]);
#pragma unroll
    for (int i = 0; i < NI; ++i) st_stream(a.g + o0 + 16LL * i * Cs, gs[i]);
    if (!moves) return;                                         // (the gradient of a model without samples is zero all the same)
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int row = r0 + 16 * i;                                // cb inside the tile
    if (row >= cb_real || c4 >= cs_real) continue;
    const long long o = o0 + 16LL * i * Cs;
    float tt[4];
    adam_update4(a, bc1, bc2, gs[i], ths[i], ms[i], vs[i], tt);
    st_stream(a.theta + o, ths[i]);
    st_stream(a.m + o, ms[i]);
    st_stream(a.v + o, vs[i]);
    if constexpr (sizeof(T) == 2) store4(static_cast<bf16_t*>(a.shadow) + o, tt);
    else if (a.split_u) store_split4(a.split_u + part + (o - base), a.plane, tt);
#pragma unroll
    for (int e = 0; e < 4; ++e) *reinterpret_cast<T*>(tile + (c4 + e) * TSTRIDE + row * (int)sizeof(T)) = from_float<T>(tt[e]);
  }
  __syncthreads();
  for (int cid = threadIdx.x; cid < 8 * ROWS; cid += 256) {       // eight values of a transposed row at a time
    const int cs = cid / (ROWS / 8), ch = cid % (ROWS / 8) * 8;
    const long long o = ((long long)tap * Cs + tcs * 64 + cs) * Cb + cb0 + ch;
    if (ch + 8 > cb_real || cs >= cs_real) {                    // padding, or the last real channels one by one
      for (int k = 0; k < 8 && ch + k < cb_real && cs < cs_real; ++k) {
        const T v = *reinterpret_cast<const T*>(tile + cs * TSTRIDE + (ch + k) * (int)sizeof(T));
        if constexpr (sizeof(T) == 2) {
          static_cast<T*>(a.shadow_t)[base + o + k] = v;
        } else {                                                // (fp32 weights with padding are held split: adam_plan)
          unsigned h, m, l_;
          split_pair(v, 0.f, h, m, l_);
          unsigned short* const d = a.split_d + part + o + k;
          d[0] = (unsigned short)h; d[a.plane] = (unsigned short)m; d[2 * a.plane] = (unsigned short)l_;
        }
      }
      continue;
    }
    const uint4* src = reinterpret_cast<const uint4*>(tile + cs * TSTRIDE + ch * (int)sizeof(T));
    if constexpr (sizeof(T) == 2) *reinterpret_cast<uint4*>(static_cast<T*>(a.shadow_t) + base + o) = src[0];
    else if (a.split_u) store_split8(a.split_d + part + o, a.plane, src[0], src[1]);
    else {
      uint4* dst = reinterpret_cast<uint4*>(static_cast<T*>(a.shadow_t) + (long long)l * a.plane + a.reg_part[r] + o);
      dst[0] = src[0];
      dst[1] = src[1];
    }
  }
}

template <typename T, int ROWS, bool SPLITS>
__global__ __launch_bounds__(256) void adam_tile_kernel(AdamArgs a, AdamSplits sp) { adam_tile<T, ROWS, SPLITS>(a, sp, blockIdx.x); }

// What is left of an update, in one launch: the gaps, with the operand of the image-side layer written from the weights just computed, its label maps, and
// (TILES) the last region in quarter tiles.  Three launches that waited for one another, the operand's reading the weights back: one 28x28 pair 10 + 4 + 3 -> 11 us
// (D) and 10 + 7 + 3 -> 14 (G).  Of large blocks nothing changes (a hundred 32x32 pairs, G's gaps: 566 us, 5.3 TB/s).
template <typename T, bool LABELS, bool TILES, bool SPLITS>
__global__ __launch_bounds__(256) void adam_rest_kernel(AdamArgs a, AdamImage im, AdamSplits sp, unsigned tile_blocks, unsigned gap_blocks) {
  unsigned b = blockIdx.x;
  if constexpr (TILES) {
    if (b < tile_blocks) return adam_tile<T, 16, SPLITS>(a, sp, b);
    b -= tile_blocks;
  }
  if (b < gap_blocks) {
    const unsigned per = (unsigned)a.gap_blk0[a.ngaps];
    return adam_gap<T>(a, im, (int)(b / per), (int)(b % per));
  }
  if constexpr (LABELS) adam_label_maps<T>(a, im, (int)((b - gap_blocks) * 256 + threadIdx.x));
}

// Launches of fewer 64 x 64 tiles than this take them in quarters: whole, they leave CUs without a block, or a second round nearly empty, and the update waits
// for one block's chain of loads, divisions and stores.  Whole tiles and quarters, with splits: 32 tiles 18.3 and 9.9 us, 128 tiles 22.6 and 18.0, 320 18.4
// and 16.3 (bf16), 22.2 and 19.7 to 23.2 (fp32), 512 28.1 and 29.5, 1024 41 and 41; without, 4096 91 and 90.  The launch of the gaps has quarters of as many all the
// same, which cost less than a launch: all four of a 32x32 pair's update launches, with 512 tiles in each network, 87 us in fp32 and 78 in bf16; quarters in both
// places 92 and 80, a launch more in place of the quarters 90 and 85.
constexpr long long ADAM_FEW_TILES = 512;
// Fills the launch geometry: the tiled regions (sorted by offset: the caller's job) and the gaps between them, which
// cover the rest of [0, P).  False (and a launch error) when the regions do not fit the kernels.
bool adam_plan(AdamArgs& a) {
  if (a.nregions < 0 || a.nregions > ADAM_MAX_REGIONS || a.P % 8) {
    launch_fail("Adam: too many weight regions, or a parameter block that is not a multiple of 8");
    return false;
  }
  long long pos = 0;
  a.ngaps = 0;
  a.reg_tile0[0] = 0;
  a.gap_blk0[0] = 0;
  a.tile_first = 0;
  for (int r = 0; r <= a.nregions; ++r) {
    const long long lo = r < a.nregions ? a.reg_w[r] : a.P;
    if (lo < pos || lo % 4) { launch_fail("Adam: weight regions must be sorted and 16-byte aligned"); return false; }
    if (lo > pos) {
      a.gap_lo[a.ngaps] = pos; a.gap_hi[a.ngaps] = lo;
      a.gap_blk0[a.ngaps + 1] = a.gap_blk0[a.ngaps] + (int)((lo - pos + 1023) / 1024);
      ++a.ngaps;
    }
    if (r < a.nregions) {
      if (a.reg_cb[r] % 64 || a.reg_cs[r] % 64 || a.reg_cb_real[r] > a.reg_cb[r] || a.reg_cs_real[r] > a.reg_cs[r] || (a.split_u ? !a.split_d : !a.shadow_t) || a.plane % 8) {
        launch_fail("Adam: tiled regions need channel counts that are multiples of 64");
        return false;
      }
      if (!a.shadow && !a.split_u && (a.reg_cb_real[r] < a.reg_cb[r] || a.reg_cs_real[r] < a.reg_cs[r])) {
        launch_fail("Adam: padded fp32 weights without split copies");
        return false;
      }
      a.reg_tile0[r + 1] = a.reg_tile0[r] + 16 * (a.reg_cb[r] / 64) * (a.reg_cs[r] / 64);
      pos = lo + 16LL * a.reg_cb[r] * a.reg_cs[r];
    }
  }
  return true;
}
// The parts of one update of a planned AdamArgs, in any order after head_bwd_kernel, which advances the step counts and bias
// corrections: the rest (the gaps, if need be with a last region); one tiled region (or all of them, region < 0).  Each element is updated by
// exactly one part.
static bool set_region(AdamArgs& a, int region, const AdamSplits& sp) {
  const int first = region < 0 ? 0 : a.reg_tile0[region];
  const int last = region < 0 ? a.reg_tile0[a.nregions] : a.reg_tile0[region + 1];
  a.tile_first = first;
  a.tile_count = last - first;
  if ((long long)a.tile_count * a.L > 0x7fffffffLL) { launch_fail("Adam: more than 2^31 weight tiles in one launch"); return false; }
  if (sp.n > 1 && (region < 0 || !sp.part || ((uintptr_t)sp.part & 15) != 0 || a.k3 || a.reg_cb_real[region] != a.reg_cb[region] || a.reg_cs_real[region] != a.reg_cs[region])) {
    launch_fail("Adam: row splits are those of one region without padding");
    return false;
  }
  if (sp.chains != 1 && (long long)a.tile_count * a.L > ADAM_FEW_TILES) { launch_fail("Adam: whole tiles add their row splits in one sum"); return false; }
  return true;
}
bool adam_region_joins_rest(const AdamArgs& a, int region) {
  return (long long)(a.reg_tile0[region + 1] - a.reg_tile0[region]) * a.L <= ADAM_FEW_TILES;
}
template <typename T>
void launch_adam_rest(AdamArgs a, const AdamImage& im, int region, const AdamSplits& sp, hipStream_t st) {
  const bool tiles = region >= 0 && region < a.nregions;
  if (im.packed && (im.w % 4 != 0 || im.Cs % 4 != 0 || (im.add && (im.CBT <= im.CB || im.tables < 1)) || 16LL * im.CBT * im.Cs >= (1LL << 31)))
    return launch_fail("Adam: image-side layer");
  if (tiles && (!set_region(a, region, sp) || !adam_region_joins_rest(a, region))) return launch_fail("Adam: a region of too many tiles for the last launch");
  const long long tile_blocks = tiles ? 4LL * a.tile_count * a.L : 0, gap_blocks = a.ngaps > 0 ? (long long)a.gap_blk0[a.ngaps] * a.L : 0;
  const long long label_blocks = im.packed && im.add ? ((long long)im.tables * im.Cs + 255) / 256 : 0, blocks = tile_blocks + gap_blocks + label_blocks;
  if (blocks > 0x7fffffffLL) return launch_fail("Adam: more blocks than a launch can have");
  if (blocks == 0) return;
  const auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, st, a, im, sp, (unsigned)tile_blocks, (unsigned)gap_blocks); };
  const auto with_labels = [&](auto labels) {
    if (!tiles) go(adam_rest_kernel<T, labels.value, false, false>);
    else if (sp.n > 1) go(adam_rest_kernel<T, labels.value, true, true>);
    else go(adam_rest_kernel<T, labels.value, true, false>);
  };
  if (label_blocks > 0) with_labels(std::true_type{}); else with_labels(std::false_type{});
}
template void launch_adam_rest<float>(AdamArgs, const AdamImage&, int, const AdamSplits&, hipStream_t);
template void launch_adam_rest<bf16_t>(AdamArgs, const AdamImage&, int, const AdamSplits&, hipStream_t);
template <typename T>
void launch_adam_region(AdamArgs a, int region, const AdamSplits& sp, hipStream_t st) {
  if (a.nregions == 0 || region >= a.nregions) return;
  if (!set_region(a, region, sp)) return;
  const long long blocks = (long long)a.tile_count * a.L;
  if (blocks == 0) return;
  const bool quarters = blocks < ADAM_FEW_TILES;
  const dim3 grid((unsigned)(quarters ? 4 * blocks : blocks));
  if (quarters) {
    if (sp.n > 1) hipLaunchKernelGGL((adam_tile_kernel<T, 16, true>), grid, dim3(256), 0, st, a, sp);
    else hipLaunchKernelGGL((adam_tile_kernel<T, 16, false>), grid, dim3(256), 0, st, a, sp);
  } else {
    if (sp.n > 1) hipLaunchKernelGGL((adam_tile_kernel<T, 64, true>), grid, dim3(256), 0, st, a, sp);
    else hipLaunchKernelGGL((adam_tile_kernel<T, 64, false>), grid, dim3(256), 0, st, a, sp);
  }
}
template void launch_adam_region<float>(AdamArgs, int, const AdamSplits&, hipStream_t);
template void launch_adam_region<bf16_t>(AdamArgs, int, const AdamSplits&, hipStream_t);

template <typename T>
void launch_adam(AdamArgs a, hipStream_t st) {
  if (!adam_plan(a)) return;
  launch_adam_rest<T>(a, AdamImage{}, -1, AdamSplits{}, st);
  launch_adam_region<T>(a, -1, AdamSplits{}, st);
}
template void launch_adam<float>(AdamArgs, hipStream_t);
template void launch_adam<bf16_t>(AdamArgs, hipStream_t);

template <typename T>
__global__ void cast_shadow_kernel(const float* __restrict__ theta, T* __restrict__ shadow, long long total) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < total) shadow[i] = from_float<T>(theta[i]);
}
template <typename T> void launch_cast_shadow(const float* theta, T* shadow, long long total, hipStream_t st) {
  if (total == 0) return;
  hipLaunchKernelGGL((cast_shadow_kernel<T>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, theta, shadow, total);
}
template void launch_cast_shadow<bf16_t>(const float*, bf16_t*, long long, hipStream_t);
template void launch_cast_shadow<float>(const float*, float*, long long, hipStream_t);

// dst[tap][cs][cb] <- src[tap][cb][cs]; block = 32 x 32 tile, grid (tiles, 16 taps, L)
template <typename T, typename S>
__global__ void transpose_w_kernel(const S* __restrict__ src, T* __restrict__ dst, long long src_stride, long long dst_stride, int Cb, int Cs) {
  __shared__ float tile[32][33];
  const int tb = Cb / 32;
  const int tcs = blockIdx.x / tb, tcb = blockIdx.x - tcs * tb;
  src += (long long)blockIdx.z * src_stride + (long long)blockIdx.y * Cb * Cs;
  dst += (long long)blockIdx.z * dst_stride + (long long)blockIdx.y * Cb * Cs;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 256 threads: 8 rows per pass
  for (int r = ty; r < 32; r += 8) {
    const int cb = tcb * 32 + r, cs = tcs * 32 + tx;
    tile[r][tx] = (cs < Cs) ? to_float(src[(long long)cb * Cs + cs]) : 0.f;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int cs = tcs * 32 + r, cb = tcb * 32 + tx;
    if (cs < Cs) dst[(long long)cs * Cb + cb] = from_float<T>(tile[tx][r]);
  }
}
template <typename T, typename S>
void launch_transpose_w(const S* src, T* dst, long long src_stride, long long dst_stride, int L, int Cb, int Cs, hipStream_t st) {
  dim3 grid((Cb / 32) * ((Cs + 31) / 32), 16, L);
  hipLaunchKernelGGL((transpose_w_kernel<T, S>), grid, dim3(256), 0, st, src, dst, src_stride, dst_stride, Cb, Cs);
}
template void launch_transpose_w<float, float>(const float*, float*, long long, long long, int, int, int, hipStream_t);
template void launch_transpose_w<bf16_t, bf16_t>(const bf16_t*, bf16_t*, long long, long long, int, int, int, hipStream_t);

// ---------------------------------------------------------------------------------------------------------
// Mixture sampling (Eq. 5): class draws from the prior.  The cumulative probabilities come from the host in
// double; the comparison is done in double so that the integer result does not depend on who computes it.
// ---------------------------------------------------------------------------------------------------------
// Cumulative probabilities in device memory, or (up to DRAW_ARGS of them) among the kernel's arguments, from where a block copies them into
// LDS: no copy from the host, before which the host had to wait for the stream (with the shorter routing, 6400 samples of a hundred 32x32
// generators 1165 -> 1114 us)
__global__ __launch_bounds__(256) void draw_labels_kernel(const float* __restrict__ u, const double* __restrict__ cdf_mem, DrawTable table, int K,
                                                          int last, int n, int* __restrict__ labels) {
  __shared__ double sh[DRAW_ARGS];
  if (!cdf_mem) {
    if ((int)threadIdx.x < K) sh[threadIdx.x] = table.cdf[threadIdx.x];
    __syncthreads();
  }
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double ui = (double)u[i];
  const auto search = [&](const double* cdf) {
    int lo = 0, hi = K;               // first k in [0, K) with cdf[k] > ui (cdf is non-decreasing), K if none
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (cdf[mid] > ui) hi = mid; else lo = mid + 1;
    }
    labels[i] = lo < K ? lo : last;
  };
  if (cdf_mem) search(cdf_mem); else search(sh);
}
void launch_draw_labels(const float* u, const double* cdf_mem, const DrawTable& table, int n_labels, int last, int n, int* labels, hipStream_t st) {
  if (n == 0) return;
  if (!cdf_mem && n_labels > DRAW_ARGS) return launch_fail("class draws: more labels than fit the kernel's arguments");
  hipLaunchKernelGGL(draw_labels_kernel, dim3((n + 255) / 256), dim3(256), 0, st, u, cdf_mem, table, n_labels, last, n, labels);
}

// ---------------------------------------------------------------------------------------------------------
// One-way ANOVA of the image intensities by class (Section 4).  Two kernels, double arithmetic, every sum in a fixed
// order: per-lane partial sums, then a tree.
// ---------------------------------------------------------------------------------------------------------
__device__ inline double wave_sum_f64(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
// Means of single channel images, one wave each.  VEC: 16-byte loads, four in flight per lane, no barrier.  Bound by reading the images
// once: 79 MB of 6400 32x32x3 images in 14.2 us when they come from memory (5.6 TB/s), 11.9 when a call before left them in the
// memory-side cache; one block per channel image with 4-byte loads and an eight-step tree over LDS took 31.1 and 24.2.  It is a third
// of the call (33 us on repeated images).
template <bool VEC>
__global__ __launch_bounds__(256) void anova_image_mean_kernel(const float* __restrict__ images, long long count, int HW, double* __restrict__ x) {
  const long long ic = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);      // image * C + channel
  if (ic >= count) return;
  const int lane = threadIdx.x & 63;
  const float* p = images + ic * HW;
  double s = 0.0;
  if (VEC) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4* q = reinterpret_cast<const f4*>(p);
    const int n4 = HW >> 2;
    int i = lane;
    for (; i + 192 < n4; i += 256) {
      f4 v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = __builtin_nontemporal_load(q + i + 64 * k);
#pragma unroll
      for (int k = 0; k < 4; ++k) s += ((double)v[k].x + (double)v[k].y) + ((double)v[k].z + (double)v[k].w);
    }
    for (; i < n4; i += 64) {
      const f4 v = q[i];
      s += ((double)v.x + (double)v.y) + ((double)v.z + (double)v.w);
    }
  } else {
    for (int i = lane; i < HW; i += 64) s += (double)p[i];
  }
  s = wave_sum_f64(s);
  if (lane == 0) x[ic] = s / (double)HW;
}
// One block per label: the sum of its images' means and their number, then the squared deviations from the group mean, over all
// channels.  The kernel is a chain of latencies: the labels, the means of the few that match, two sums across lanes.  So the label's
// images are first gathered into a list in LDS (eight labels a thread, places from ballots, in a fixed order), then four waves share
// the list of one channel, so that a sum over lanes is one butterfly and four values, and up to four means a lane stay in registers for
// the second pass: 6400 images, 100 labels 14.1 -> 6.2 us of a call of 40.1, now 33.1 (before: 1024 threads
// with eight labels each, every sum over all of them, once per channel).  What loses is one label with nearly all of a full trip, whose list
// four waves walk: 8192 images, 34 us of a call against 30.
constexpr int ANOVA_T = 1024, ANOVA_W = ANOVA_T / 64, ANOVA_E = 8, ANOVA_TRIP = ANOVA_E * ANOVA_T, ANOVA_KEEP = 4;
__global__ __launch_bounds__(ANOVA_T) void anova_group_kernel(const int* __restrict__ label_ids, const double* __restrict__ x, int n, int C,
                                                              double* __restrict__ gsum, double* __restrict__ ssw, int* __restrict__ gcnt) {
  __shared__ int list[ANOVA_TRIP];
  __shared__ int votes_n[ANOVA_E * ANOVA_W];
  __shared__ double sh[ANOVA_W];
  const int k = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = wave >> 2, q0 = (wave & 3) * 64 + lane;                // this wave's channel, and its lane's first place in the list
  // the label's images among ANOVA_TRIP from i0 on -> list; returns their number
  const auto gather = [&](int i0) {
    int lab[ANOVA_E];
    unsigned long long votes[ANOVA_E];
#pragma unroll
    for (int e = 0; e < ANOVA_E; ++e) {
      const int i = i0 + ANOVA_T * e + (int)threadIdx.x;
      lab[e] = i < n ? label_ids[i] : -1;
    }
#pragma unroll
    for (int e = 0; e < ANOVA_E; ++e) {
      votes[e] = __ballot(lab[e] == k);
      if (lane == 0) votes_n[e * ANOVA_W + wave] = __popcll(votes[e]);
    }
    __syncthreads();
    // running sums of the 128 counts: two a lane, every wave alike
    const int a = votes_n[2 * lane], b = votes_n[2 * lane + 1];
    int run = a + b;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(run, o, 64);
      if (lane >= o) run += t;
    }
#pragma unroll
    for (int e = 0; e < ANOVA_E; ++e) {
      const int at = e * ANOVA_W + wave;                                // the counts before this one
      const int before = __shfl(run - a - b, at >> 1, 64) + ((at & 1) ? __shfl(a, at >> 1, 64) : 0);
      if (lab[e] == k) list[before + __popcll(votes[e] & ((1ull << lane) - 1))] = i0 + ANOVA_T * e + (int)threadIdx.x;
    }
    const int total = __shfl(run, 63, 64);
    __syncthreads();
    return total;
  };
  static_assert(ANOVA_E * ANOVA_W == 128, "two counts a lane");
  double mean = 0.0;
  double keep[ANOVA_KEEP];
  int total = 0;
  long long all = 0;
  const bool once = n <= ANOVA_TRIP;
  for (int pass = 0; pass < 2; ++pass) {
    double s = 0.0;
    for (int i0 = 0; i0 < n; i0 += ANOVA_TRIP) {
      if (!once || pass == 0) {
        total = gather(i0);
        if (pass == 0) all += total;
      }
      if (c < C) {
        const auto add = [&](double v) {
          const double d = v - mean;
          s += pass ? d * d : d;
        };
        if (!once || pass == 0) {
#pragma unroll
          for (int e = 0; e < ANOVA_KEEP; ++e) keep[e] = q0 + 256 * e < total ? x[(long long)list[q0 + 256 * e] * C + c] : 0.0;
        }
#pragma unroll
        for (int e = 0; e < ANOVA_KEEP; ++e)
          if (q0 + 256 * e < total) add(keep[e]);
#pragma unroll 8
        for (int i = q0 + 256 * ANOVA_KEEP; i < total; i += 256) add(x[(long long)list[i] * C + c]);
      }
      if (!once) __syncthreads();                                       // the list is written again
    }
    s = wave_sum_f64(s);
    if (lane == 0) sh[wave] = s;
    __syncthreads();
    const double t = ((sh[4 * c] + sh[4 * c + 1]) + sh[4 * c + 2]) + sh[4 * c + 3];
    if (!pass) mean = all > 0 ? t / (double)all : 0.0;
    if ((threadIdx.x & 255) == 0 && c < C) (pass ? ssw : gsum)[(long long)k * C + c] = t;
    if (threadIdx.x == 0 && !pass) gcnt[k] = (int)all;
    __syncthreads();                                                    // sh is written again by the second pass
  }
}
// The same without lists, for many images: every thread adds the means of its own images that match, over all channels at once, and keeps
// nothing, so a trip over 8192 labels waits for nobody.  With lists every further trip costs two barriers and is gathered again in the second
// pass, and a long list has four waves of sixteen on it.  us of a call, lists / without (4x4 images, one channel): 65536 images 116 / 69 with
// two labels, 67 / 58 with 100, 186 / 120 with 1000; 32768 67 / 46, 43 / 42, 113 / 94; 16384 43 / 35, 31 / 34, 76 / 81; one trip, 8192
// images, 27 / 30, 23 / 31, 48 / 75.
__global__ __launch_bounds__(ANOVA_T) void anova_group_many_kernel(const int* __restrict__ label_ids, const double* __restrict__ x, int n, int C,
                                                                   double* __restrict__ gsum, double* __restrict__ ssw, int* __restrict__ gcnt) {
  __shared__ double sh[5][ANOVA_W];
  const int k = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double mean[4] = {0.0, 0.0, 0.0, 0.0};
  for (int pass = 0; pass < 2; ++pass) {
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    int cnt = 0;
    for (int i0 = threadIdx.x; i0 < n; i0 += ANOVA_TRIP) {
      int lab[ANOVA_E];
      double v[ANOVA_E][4];
#pragma unroll
      for (int e = 0; e < ANOVA_E; ++e) lab[e] = i0 + ANOVA_T * e < n ? label_ids[i0 + ANOVA_T * e] : -1;
#pragma unroll
      for (int e = 0; e < ANOVA_E; ++e)
        if (lab[e] == k) {
          const double* xi = x + (long long)(i0 + ANOVA_T * e) * C;
#pragma unroll
          for (int c = 0; c < 4; ++c) v[e][c] = c < C ? xi[c] : 0.0;
        }
#pragma unroll
      for (int e = 0; e < ANOVA_E; ++e)
        if (lab[e] == k) {
          ++cnt;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const double d = v[e][c] - mean[c];
            s[c] += pass ? d * d : d;
          }
        }
    }
    // per wave, then the waves' sums by every wave alike (16 lanes of a butterfly): all threads need the mean
    const double all5[5] = {wave_sum_f64(s[0]), wave_sum_f64(s[1]), wave_sum_f64(s[2]), wave_sum_f64(s[3]), wave_sum_f64((double)cnt)};
    if (lane == 0) {
#pragma unroll
      for (int c = 0; c < 5; ++c) sh[c][wave] = all5[c];
    }
    __syncthreads();
    double t[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      t[c] = sh[c][lane & (ANOVA_W - 1)];
#pragma unroll
      for (int o = ANOVA_W / 2; o > 0; o >>= 1) t[c] += __shfl_xor(t[c], o, 64);
    }
    __syncthreads();                                                   // sh is written again by the second pass
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (threadIdx.x == 0 && c < C) (pass ? ssw : gsum)[(long long)k * C + c] = t[c];
      if (!pass) mean[c] = t[4] > 0.0 ? t[c] / t[4] : 0.0;
    }
    if (threadIdx.x == 0 && !pass) gcnt[k] = (int)t[4];
  }
}
void launch_anova(const int* label_ids, const float* images, int n, int n_labels, int C, int HW, double* x, double* gsum,
                  double* ssw, int* gcnt, hipStream_t st) {
  if (n == 0) return;
  const long long count = (long long)n * C;
  const dim3 grid((unsigned)((count + 3) / 4));
  if (HW % 4 == 0 && (reinterpret_cast<uintptr_t>(images) & 15) == 0)
    hipLaunchKernelGGL(anova_image_mean_kernel<true>, grid, dim3(256), 0, st, images, count, HW, x);
  else
    hipLaunchKernelGGL(anova_image_mean_kernel<false>, grid, dim3(256), 0, st, images, count, HW, x);
  // lists for one trip, and for two or three where a label has 2048 images or fewer on average (see the second kernel)
  const bool lists = n <= ANOVA_TRIP || (n <= 3 * ANOVA_TRIP && n <= 2048LL * n_labels);
  hipLaunchKernelGGL(lists ? &anova_group_kernel : &anova_group_many_kernel, dim3(n_labels), dim3(ANOVA_T), 0, st, label_ids, x, n, C, gsum, ssw, gcnt);
}

}  // namespace gan
