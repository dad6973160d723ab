// Grouped implicit-GEMM engine on MFMA for the k4 s2 p1 (transposed) convolutions and the linear layers of all
// per-label models at once.  One launch covers every model (Eq. 5 of the paper makes them independent, so the
// "batch of small GEMMs" is a single grid): an M-tile never crosses a model boundary, and each tile reads its
// own model's weights.
//
// Forward-type kernel (conv_gemm_kernel): C[row][n] = sum_{tap, c} A(row, tap)[c] * W[tap][n][c]
//   down : rows are output pixels of the small tensor, 16 taps gathered from the big tensor at (2y-1+ky, 2x-1+kx)
//   up   : rows are the pixels of one output phase (Y%2, X%2) of the big tensor, 4 taps gathered from the small one
//   dense: one tap, rows are read directly (linear layer)
// Weight-gradient kernel (wgrad_kernel): dW[tap][cb][cs] = sum_rows Big(row, tap)[cb] * Small(row)[cs]; the
//   reduction index is the slow memory index of both operands: tiles go into LDS as they lie in memory, and the operand
//   reads do the transposition.
//
// Both stage K-chunks in LDS and feed v_mfma_f32_32x32x16_bf16 from it (fp32 storage: three bf16 parts a value, six MFMAs a
// product, see Split8); accumulation is fp32 in both cases.
// Forward-type kernel: K-chunks of KB bytes per row travel global -> LDS directly (buffer_load_dwordx4 ... lds, no
// registers in between) into a ring of NST buffers while the MFMAs of the current chunk run.  In bf16 the 256 x 256 tile uses
// KB = 128 with two buffers (one block per CU); the 256 x 128 tile uses KB = 64 with three, which leaves room for two blocks
// per CU, so that one block's epilogue and barriers hide behind the other's MFMAs; the smaller ones: see FwdTiles.
// The 16-byte chunk c of row
// R sits at position c ^ ((R / (256/KB)) % (KB/16)), which keeps both the 1 KiB-per-wave copies and the MFMA operand
// reads conflict-free.
// One barrier per chunk in both, except that the 256 x 256 tiles of the convolutions and of the weight gradient have one per quarter of a
// chunk (their quad_loops), tiles that share pixels one per tap of a stage, and the fp32 weight gradient two per chunk (split_loop).
#include <math.h>
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>

#include "lds_copy.h"
#include "split_mfma.h"
#include <type_traits>

namespace gan {


// Block tile BM x BN computed by WM x WN waves, each (TM*32) x (TN*32); forward kernel: KB bytes of K per LDS row,
// NST buffers.  KS (forward kernel): groups of WM x WN waves that share the tile's reduction, chunk c going to group c % KS; each has a
// ring of buffers of its own, and their sums are added at the end.
// SLOTS > 0, SHARE (forward kernel, MODE_UP): the two taps of a filter row gather the same pixels one column apart, and share one stage of
// them; NST buffers of weights, two of SLOTS pixels.
// QUAD (forward kernel, MODE_DOWN and MODE_UP): a chunk is multiplied in four quarters, half the rows by half the columns, see quad_loop.
template <int BM_, int BN_, int WM_, int WN_, int KB_ = 128, int NST_ = 2, int KS_ = 1, int SLOTS_ = 0, bool QUAD_ = false>
struct Tile {
  static constexpr bool QUAD = QUAD_;
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, KB = KB_, NST = NST_, KS = KS_;
  static constexpr bool SHARE = SLOTS_ > 0;
  // An output pixel's one tap reads the pixel that its neighbour's other tap reads, so a stage holds H + 1 pixels for every H rows of the tile.
  static constexpr int SLOTS = SLOTS_;
  static constexpr int NT = 64 * WM_ * WN_;          // threads of a group
  static constexpr int TM = BM_ / (32 * WM_), TN = BN_ / (32 * WN_);
  static constexpr int CPR = KB_ / 16;               // 16-byte chunks per LDS row
  static constexpr int RPP = NT / CPR;               // tile rows filled per loader pass
  static constexpr int PA = BM_ / RPP, PB = BN_ / RPP;
};
// The forward-type kernel's tiles, by storage type (fp32: see the splits below; they hold two accumulators per element).
template <typename T> struct FwdTiles;
template <> struct FwdTiles<bf16_t> {
  typedef Tile<256, 256, 2, 4, 128, 2> Big;      // 512 threads, wave tile 128 x 64, 128 KiB of LDS
                                                 // (MODE_DENSE, whose reductions are a few chunks)
  typedef Tile<256, 256, 2, 4, 128, 2, 1, 0, true> BigQuad;      // the same in quarters, MODE_DOWN and MODE_UP
  typedef Tile<256, 128, 4, 2, 64, 3> Mid;       // 512 threads, wave tile 64 x 64, 72 KiB of LDS
  typedef Tile<128, 128, 2, 2, 128, 2> Small;    // 256 threads, wave tile 64 x 64 (few rows per model), 64 KiB of LDS
  typedef Small SmallWhole;
  typedef Tile<256, 64, 4, 1, 128, 2> Narrow;    // 256 threads, wave tile 64 x 64, for layers with 64 output channels:
                                                 // 128-byte chunks, two buffers of 40 KiB, so two blocks still share a CU
  typedef Tile<256, 64, 4, 1, 64, 2> NarrowShort;  // the same with two buffers of 20 KiB for MODE_UP and MODE_DENSE: their reductions are
                                                 // short, and what a block waits for before it can multiply weighs more
  typedef Tile<64, 64, 2, 2, 128, 2> Tiny;       // 256 threads, wave tile 32 x 32, 32 KiB of LDS: workloads so small that
                                                 // the larger tiles would leave most of the chip without a block
  // MODE_UP with shared pixels, for sides from 4 up (share_fits): the loop lives on the CU's load path, and a pair of taps brings in half the
  // pixels and a bit.  us: 256 -> 128 channels, side 8, 6400 samples 433 -> 413; 128 -> 64, side 16, 1024 samples 106 -> 91.  MODE_DOWN gained
  // nothing (256x128 78.6 and 79.3, 256x64 77 and 78), nor did side 7, whose runs need padding against bank conflicts (57.7 and 58.8), and on
  // 256x256 tiles the quarters gain more than the sharing did (512 -> 256, side 4, 6400 samples: 372 plain, 365 shared, 331 in quarters).
  typedef Tile<256, 128, 4, 2, 64, 3, 1, 320> MidShare;        // 64 KiB
  typedef Tile<128, 128, 2, 2, 128, 2, 1, 160> SmallShare;     // 72 KiB
  typedef Tile<256, 64, 4, 1, 64, 3, 1, 320> NarrowShare;      // 52 KiB, three blocks per CU
  typedef Tile<64, 64, 2, 2, 128, 2, 2> Pair;    // Tiny with two groups of waves on its reduction: 512 threads, 64 KiB
  typedef Tile<32, 64, 1, 2, 128, 3, 4> Deep;    // 32 x 64 with four groups: 512 threads, 144 KiB, six or more chunks on their way.  Both
                                                 // for launches that a CU gets a block or two of, whose time is that of one block: see TILES
  // Chunk sizes, in TFLOP/s, 128-byte x 2 against 64-byte x 3: 64x64 down 64 -> 128 channels at side 7, one model of 64 samples, 76
  // against 63, 64 -> 64 at side 8, 100 models, 453 against 359; 128x128 down 64 -> 128 at side 7, ten models, 541 against 495.
  // 256x64: up 128 -> 64 at side 16 480 against 582 with 64-byte x 2, up 64 -> 64 at side 8 401 against 438, but down 64 -> 64 at
  // side 8 586 against 422.
};
// fp32: a wave splits the rows it reads (its weights are split once, by the update), so wave tiles are one 32-row block and as wide as the
// tile; two blocks per CU.  20 x 64 samples, us: down 128 -> 256 channels, side 8: 128x128 with 32 x 128 wave tiles 435, 64 x 64 474,
// 32 x 64 (eight waves) 445, 256x128 (eight waves, one block per CU) 490; up 256 -> 128, side 8: 438, 451, 455, 450; with weights split
// by every wave 538 and 486 (64 x 64, the best then).  10 x 128 samples, up 128 -> 64, side 7: 128x64 108, 256x64 (one block per CU) 129, before 113.
// G's linear layer (MODE_DENSE), and convolutions of contexts whose weights the update does not split, read the weights as
// fp32 and split them too: 64 x 64 wave tiles there (SmallWhole).
template <> struct FwdTiles<float> {
  typedef Tile<128, 128, 4, 1, 128, 2> Small;    // 256 threads, wave tile 32 x 128, 80 KiB of LDS
  typedef Tile<128, 128, 2, 2, 128, 2> SmallWhole;
  typedef Tile<128, 64, 4, 1, 128, 2> Narrow;    // 256 threads, wave tile 32 x 64, 56 KiB
  typedef Narrow NarrowShort;
  typedef Tile<64, 64, 2, 2, 128, 2> Tiny;       // 256 threads, wave tile 32 x 32, 40 KiB
  typedef Tile<64, 64, 2, 2, 128, 2, 2> Pair;    // 80 KiB
  typedef Tile<32, 64, 1, 2, 128, 2, 4> Deep;    // 128 KiB
};

// SHARE: the xor of the 16-byte chunks of the pixel p = 0 .. H of a run of H columns.  Sixteen rows that are read together lie in G = 256 / KB
// places of the bank period; what a read of them must not do is meet twice in a place with the same xor, be it the rows' first pixels
// (p = 0 .. H - 1 of each run) or their second ones (1 .. H).  With sides that are multiples of G the pixels of one place have H / G values in turn,
// which p = 0 and p = H, never read together, share.  (The usual xor of the slot number doubled the time of the reads.)
__device__ inline int share_xor(int H, int G, int run, int p) {
  const int per = H / G, k = p / G;
  return run * per + (k >= per ? k - per : k);
}
// whether the kernel can (side, and the slots that a tile of BM rows reads; tiles start at multiples of BM rows)
template <typename TL> static bool share_fits(int H) {
  const int runs = (TL::BM - 1 + (TL::BM % H ? H - 1 : 0)) / H;
  return H % (256 / TL::KB) == 0 && TL::BM + runs + 1 <= TL::SLOTS;
}

// What a tile is to the chooser: its shape, the row blocks with statistics of their own, the blocks of it that a CU holds, and
// the rate a full chip of them reaches against the fastest one of the storage type (0: the storage type has no such tile).  The bf16
// 256x64 line describes Narrow, which MODE_DOWN runs; MODE_DENSE and MODE_UP run NarrowShort and, with sides that allow it, NarrowShare (four and
// three blocks per CU; 582 and 670 TFLOP/s where Narrow reaches 480) and are judged by the same line, so the estimate is too high for them.
// Deep and Pair take launches of at most `most` tiles.  There a launch takes as long as one block, which waits for each chunk, splits it
// (fp32) and multiplies it in turn; more waves on the same tile overlap these.  In us, Tiny / Pair / Deep by the number of 64x64 tiles, fp32:
// down 64 -> 128 channels, side 7: 104 tiles 30.2 / 25.2 / 17.0, 200 31.3 / 26.4 / 31.5, 400 44.1 / 40.4 / 59.5, 800 72.6 / 73.7 / 102;
// up 256 -> 128, side 4: 104 28.3 / 24.1 / 15.7, 408 41.1 / 38.6 / 56.7, 808 70.0 / 72.0 / 98; bf16: down 128 -> 256, side 4: 104 13.3 /
// 11.6 / 9.6, 208 13.8 / 12.2 / 16.8, 408 17.6 / 17.3 / 31.7; up 128 -> 64, side 7: 104 6.5 / 6.6 / 6.3, 400 8.1 / 9.0 / 18.3.
// (Their rates are such that the time of a lone block compares with a lone Tiny's.)
// The bf16 rates were taken when the 256x256 tile multiplied whole chunks, as MODE_DENSE still does.  With chunks in quarters, a hundred models of
// 64 samples, us of 256x256, 128x128 and 64x64: down 128 -> 256 channels, side 8, 367, 498, 714; 256 -> 512, side 4, 338, 421, 632; up 512 -> 256,
// side 4, 351, 414, 662; 128 -> 256, side 8, 438, 506, 730: 128x128 at 0.74 to 0.87, 64x64 at 0.51 to 0.60.  256x128 and 128x128: down 256 -> 128,
// side 8, 450 and 433; up 256 -> 128, side 8, 414 and 460: 0.77 to 0.95 for 256x128.
// So the lines still lie inside what their tiles reach; what differs is the mode, which they do not tell apart.
struct TileInfo { ConvTile id; const char* name; int rows, cols, split, per_cu; double rate; int most; };
template <typename TL> constexpr TileInfo info(ConvTile id, const char* name, int per_cu, double rate, int most = 1 << 30) {
  return {id, name, TL::BM, TL::BN, TL::WM, per_cu, rate, most};
}
static const TileInfo TILES[2][7] = {
    {info<FwdTiles<bf16_t>::Big>(TILE_BIG, "256x256", 1, 1.0), info<FwdTiles<bf16_t>::Mid>(TILE_MID, "256x128", 2, 0.88),
     info<FwdTiles<bf16_t>::Small>(TILE_SMALL, "128x128", 2, 0.77), info<FwdTiles<bf16_t>::Narrow>(TILE_NARROW, "256x64", 2, 0.70),
     info<FwdTiles<bf16_t>::Tiny>(TILE_TINY, "64x64", 5, 0.52),
     info<FwdTiles<bf16_t>::Pair>(TILE_PAIR, "64x64 pair", 2, 0.585, 256), info<FwdTiles<bf16_t>::Deep>(TILE_DEEP, "32x64 deep", 1, 0.36, 256)},
    {{TILE_BIG, "", 0, 0, 0, 0, 0, 0}, {TILE_MID, "", 0, 0, 0, 0, 0, 0},
     info<FwdTiles<float>::Small>(TILE_SMALL, "128x128", 2, 1.0), info<FwdTiles<float>::Narrow>(TILE_NARROW, "128x64", 2, 0.75),
     info<FwdTiles<float>::Tiny>(TILE_TINY, "64x64", 5, 0.64),
     info<FwdTiles<float>::Pair>(TILE_PAIR, "64x64 pair", 2, 0.76, 512), info<FwdTiles<float>::Deep>(TILE_DEEP, "32x64 deep", 1, 0.58, 256)},
};
static const TileInfo& tile_info(int esize, ConvTile t) { return TILES[esize == 4][t]; }
int conv_tile_rows(int esize, ConvTile t) { return tile_info(esize, t).rows; }
int conv_stat_split(int esize, ConvTile t, bool split_weights) {
  if (esize == 4 && t == TILE_SMALL && !split_weights) return FwdTiles<float>::SmallWhole::WM;
  return tile_info(esize, t).split;
}

// The tile with the smallest estimated time for a launch of `groups` row spaces (phases x segments) of rows_per_model rows in
// each of n_models models and n_out output columns: rounds of blocks over the chip's 256 CUs times a block's share of its
// CU, at the tile's rate.  A last round that leaves CUs idle costs as much as a full one, which is what rules out large
// tiles for small launches; blocks beyond the first round of their CU come in wherever one ends, so a partial round is
// counted half a block longer than an even spread.
ConvTile conv_choose_tile(int esize, int n_out, double rows_per_model, int n_models, int groups) {
  const TileInfo* best = nullptr;
  double best_t = 0;
  for (const TileInfo& t : TILES[esize == 4]) {
    if (t.rate == 0) continue;
    if (t.cols > 64 && n_out % t.cols != 0) continue;      // half-filled tiles
    const double tiles = ceil(rows_per_model / t.rows) * n_models * groups * ((n_out + t.cols - 1) / t.cols);
    if (tiles > t.most) continue;
    const double per_round = 256.0 * t.per_cu, full = floor(tiles / per_round), rest = tiles - full * per_round;
    double blocks = full * t.per_cu;                       // blocks one CU works through
    if (rest > 0) blocks += std::min((double)t.per_cu, ceil(rest / 256.0) + (full > 0 ? 0.5 : 0.0));
    const double time = blocks * t.rows * t.cols / t.rate;
    if (!best || time < best_t) { best = &t; best_t = time; }
  }
  return best->id;
}
// the tile of a given height (single-operation tests): with 256 rows the width follows the output channels
ConvTile conv_tile_of_rows(int esize, int rows, int n_out) {
  if (rows == 64) return TILE_TINY;
  if (rows == 128) return TILE_SMALL;
  return n_out <= 64 || esize == 4 ? TILE_NARROW : (n_out % 256 == 0 ? TILE_BIG : TILE_MID);
}

// One K-step (16 bytes of every operand row) of a wave's TM x TN tiles.
template <int TM, int TN>
__device__ __forceinline__ void mma_step(floatx16 (&acc)[TM][TN], const u32x4 (&a)[TM], const u32x4 (&b)[TN], bf16_t) {
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) mma16B(acc[tm][tn], __builtin_bit_cast(uint4, a[tm]), __builtin_bit_cast(uint4, b[tn]), bf16_t());
}
// fp32, one value at a time (tiles with infinities or NaN, see Split8): four k-pairs; lane half h supplies k = 4h + j to
// MFMA j, for A and B alike.  The pair is the outer loop, so that an accumulator comes round only after all the others.
template <int TM, int TN>
__device__ __forceinline__ void mma_step(floatx16 (&acc)[TM][TN], const u32x4 (&a)[TM], const u32x4 (&b)[TN], float) {
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
        acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[tm][j]), __uint_as_float(b[tn][j]), acc[tm][tn], 0, 0, 0);
}

// one row fragment against TN column fragments: h*h into acc, the five smaller products into low
template <int TN>
__device__ __forceinline__ void mma_split(floatx16 (&acc)[TN], floatx16 (&low)[TN], const Split8& a, const Split8 (&b)[TN]) {
#pragma unroll
  for (int t = 0; t < TN; ++t) mma_u4(low[t], a.l, b[t].h);
#pragma unroll
  for (int t = 0; t < TN; ++t) mma_u4(acc[t], a.h, b[t].h);
#pragma unroll
  for (int t = 0; t < TN; ++t) mma_u4(low[t], a.h, b[t].l);
#pragma unroll
  for (int t = 0; t < TN; ++t) mma_u4(low[t], a.m, b[t].m);
#pragma unroll
  for (int t = 0; t < TN; ++t) mma_u4(low[t], a.m, b[t].h);
#pragma unroll
  for (int t = 0; t < TN; ++t) mma_u4(low[t], a.h, b[t].m);
}
// 1 if any of this lane's sums is an infinity or NaN
template <int TM, int TN>
__device__ inline int not_finite(const floatx16 (&acc)[TM][TN]) {
  float z = 0.f;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) z = __builtin_fmaf(acc[i][j][e], 0.f, z);
  return z != z;
}
// the same for the whole block, through a few bytes of LDS that nothing else is using (barriers on both sides)
template <int WAVES>
__device__ inline bool block_any(int flag, unsigned char* lds, int wave) {
  int* const word = reinterpret_cast<int*>(lds);
  const bool mine = __ballot(flag) != 0;
  if ((threadIdx.x & 63) == 0) word[wave] = mine;
  __syncthreads();
  int any = 0;
  for (int w = 0; w < WAVES; ++w) any |= word[w];
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(any) != 0;
}
// the sum of the products of split operands
template <int TM, int TN>
__device__ inline void add_acc(floatx16 (&acc)[TM][TN], const floatx16 (&low)[TM][TN]) {
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = (acc[i][j][e] + low[i][j][e]) * SPLIT_UNSCALE;
}
template <int TM, int TN>
__device__ inline void clear_acc(floatx16 (&acc)[TM][TN]) {
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
}

// One K-chunk of the forward-type kernel: rows KB bytes apart, the 16-byte chunk c of tile row R at position
// c ^ ((R / (256/KB)) % (KB/16)).  Sixteen lanes reading one chunk index of sixteen consecutive rows then touch
// sixteen different 16-byte slots of the 256-byte bank period, and so do the rows one wave-wide copy fills.
template <int KB>
__device__ inline int fwd_swz(int row) { return (row / (256 / KB)) % (KB / 16); }
// The end of a quarter of a chunk (QUAD): the operands requested in it are here, at most N copies are still in flight, and so say all waves.  The
// compiler counts the operands' reads and sees this wait, so that no register is read, moved or used again before its operand is there.
template <int N>
__device__ __forceinline__ void quad_wait() {
  static_assert(N < 16, "the counter's low bits");
  asm volatile("" : : : "memory");
  __builtin_amdgcn_s_waitcnt(0x70 | N);       // vmcnt(N) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" : : : "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// QUAD: the column of the tile that row R of a buffer of weights holds: first the 32 columns of each of the four waves' first blocks, then
// those of their second ones
__device__ inline int quad_col(int R) { return ((R >> 5) & 3) * 64 + (R >> 7) * 32 + (R & 31); }

template <typename T, int TM, int TN, int KB>
__device__ __forceinline__ void tile_mma_fwd(floatx16 (&acc)[TM][TN], const unsigned char* As, const unsigned char* Bs, int wm, int wn,
                                    int lane) {
  const int r = lane & 31, h = lane >> 5;
  const int sw = fwd_swz<KB>(r);   // tile rows start at multiples of 32, a multiple of the swizzle period
  constexpr int NV = KB / 32;
  // `at`: this lane's 16 bytes of K-step 0 in its rows; K-step vs sits there with bit 5 .. flipped by vs (chunk index
  // (2 vs + h) ^ sw = (2 vs) ^ (h ^ sw): no carries).  The reads of K-step vs + 1 are in flight while the MFMAs of K-step vs run (two register
  // sets), which the scheduling barriers keep in this order.
  const unsigned char* const a0 = As + (wm * TM * 32 + r) * KB;
  const unsigned char* const b0 = Bs + (wn * TN * 32 + r) * KB;
  const int at = (h ^ sw) << 4;
  u32x4 a[2][TM], b[2][TN];
  auto fetch = [&](auto vs, auto set) __attribute__((always_inline)) {
    const int k = at ^ (vs.value << 5);
#pragma unroll
    for (int t = 0; t < TM; ++t) a[set.value][t] = *reinterpret_cast<const u32x4*>(a0 + k + t * 32 * KB);
#pragma unroll
    for (int t = 0; t < TN; ++t) b[set.value][t] = *reinterpret_cast<const u32x4*>(b0 + k + t * 32 * KB);
    __builtin_amdgcn_sched_barrier(0);
  };
  fetch(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
  static_for<0, NV>([&](auto vs) __attribute__((always_inline)) {
    constexpr int cur = vs.value & 1;
    if constexpr (vs.value + 1 < NV) fetch(std::integral_constant<int, vs.value + 1>{}, std::integral_constant<int, cur ^ 1>{});
    mma_step(acc, a[cur], b[cur], T());
    __builtin_amdgcn_sched_barrier(0);       // keep these MFMAs in front of the next K-step's wait
  });
}

// The same with the offset of every fragment's row in its stage given (SHARE).
template <typename T, int TM, int TN, int KB>
__device__ __forceinline__ void tile_mma_rows(floatx16 (&acc)[TM][TN], const unsigned (&arow)[TM], unsigned a_stage, const unsigned char* As,
                                              const unsigned char* Bs, int wn, int lane) {
  const int r = lane & 31, h = lane >> 5;
  constexpr int NV = KB / 32;
  const unsigned char* const b0 = Bs + (wn * TN * 32 + r) * KB;
  const int at = (h ^ fwd_swz<KB>(r)) << 4;
  u32x4 a[2][TM], b[2][TN];
  auto fetch = [&](auto vs, auto set) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < TM; ++t) a[set.value][t] = *reinterpret_cast<const u32x4*>(As + ((arow[t] + a_stage) ^ (vs.value << 5)));
#pragma unroll
    for (int t = 0; t < TN; ++t) b[set.value][t] = *reinterpret_cast<const u32x4*>(b0 + (at ^ (vs.value << 5)) + t * 32 * KB);
    __builtin_amdgcn_sched_barrier(0);
  };
  fetch(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
  static_for<0, NV>([&](auto vs) __attribute__((always_inline)) {
    constexpr int cur = vs.value & 1;
    if constexpr (vs.value + 1 < NV) fetch(std::integral_constant<int, vs.value + 1>{}, std::integral_constant<int, cur ^ 1>{});
    mma_step(acc, a[cur], b[cur], T());
    __builtin_amdgcn_sched_barrier(0);       // keep these MFMAs in front of the next K-step's wait
  });
}

// fp32 through splits: two K-steps (16 values of K per row) are one step here; lane half h supplies values 8 h .. 8 h + 7 of the step.
// PRE: the columns are split already, three planes of BN rows of KB / 2 bytes each (swizzled like rows of a bf16 tile).
template <int TM, int TN, int KB, bool PRE, int BN>
__device__ __forceinline__ void tile_mma_split(floatx16 (&acc)[TM][TN], floatx16 (&low)[TM][TN], const unsigned char* As,
                                               const unsigned char* Bs, int wm, int wn, int lane) {
  const int r = lane & 31, h = lane >> 5;
  const int sw = fwd_swz<KB>(r), swb = fwd_swz<KB / 2>(r);
  const unsigned char* const ap = As + (wm * TM * 32 + r) * KB;
  const unsigned char* const bp = Bs + (wn * TN * 32 + r) * (PRE ? KB / 2 : KB);
  static_for<0, KB / 64>([&](auto ps) __attribute__((always_inline)) {
    const int c0 = ((4 * ps.value + 2 * h) ^ sw) * 16, c1 = ((4 * ps.value + 2 * h + 1) ^ sw) * 16;
    Split8 b[TN];
    static_for<0, TN>([&](auto t) __attribute__((always_inline)) {
      if constexpr (PRE) {
        const unsigned char* const q = bp + t.value * 32 * (KB / 2) + ((2 * ps.value + h) ^ swb) * 16;
        b[t.value].h = *reinterpret_cast<const u32x4*>(q);
        b[t.value].m = *reinterpret_cast<const u32x4*>(q + BN * (KB / 2));
        b[t.value].l = *reinterpret_cast<const u32x4*>(q + 2 * BN * (KB / 2));
      } else {
        b[t.value] = split8(*reinterpret_cast<const u32x4*>(bp + t.value * 32 * KB + c0), *reinterpret_cast<const u32x4*>(bp + t.value * 32 * KB + c1));
      }
    });
    static_for<0, TM>([&](auto t) __attribute__((always_inline)) {
      const Split8 a = split8(*reinterpret_cast<const u32x4*>(ap + t.value * 32 * KB + c0), *reinterpret_cast<const u32x4*>(ap + t.value * 32 * KB + c1));
      mma_split(acc[t.value], low[t.value], a, b);
    });
  });
}

__device__ inline void store_out(float* p, float v) { *p = v; }
__device__ inline void store_out(bf16_t* p, float v) { *p = from_float<bf16_t>(v); }

// row of a model -> (sample, y, x); shift form when the side is a power of two
__device__ inline void decode_row(int r, int H, int rps, int sh, int& n, int& y, int& x) {
  if (sh >= 0) {
    n = r >> (2 * sh);
    const int rem = r & (rps - 1);
    y = rem >> sh;
    x = rem & (H - 1);
  } else {
    n = r / rps;
    const int rem = r - n * rps;
    y = rem / H;
    x = rem - y * H;
  }
}
// Row order of the forward-type kernel inside a model: pixel row y slowest, then the sample, then x.  A tile of
// consecutive rows then covers few pixel rows (one, when samples * H is a multiple of the tile height), and the taps
// that fall above or below the map for all of them are skipped as whole K-chunks.  row_block = samples * H.
__device__ inline void decode_row_yfirst(int r, int H, int row_block, int sh, int& n, int& y, int& x) {
  y = r / row_block;
  const int rem = r - y * row_block;
  if (sh >= 0) {
    n = rem >> sh;
    x = rem & (H - 1);
  } else {
    n = rem / H;
    x = rem - n * H;
  }
}
static int log2_or_neg(int v) {
  for (int s = 0; s < 30; ++s)
    if ((1 << s) == v) return s;
  return -1;
}

// Waves a SIMD should hold at least, which bounds the registers.  Wave tiles of 64 x 64: two (fp32 needs about 200 registers for its
// two accumulators; without the bound bf16 takes 171, half of them accumulation registers, and with it 107, four waves).
template <typename T, typename TL> constexpr int waves_per_simd() { return TL::TM * TL::TN == 4 ? 2 : 1; }
// PRE: fp32 convolutions whose weights come split (launch_split_weights), as three bf16 planes
template <typename T, int MODE, int EPI, typename TL, bool PRE>
__global__ __launch_bounds__(TL::NT * TL::KS, (waves_per_simd<T, TL>())) void conv_gemm_kernel(ConvArgs p) {
  constexpr int BM = TL::BM, BN = TL::BN, TM = TL::TM, TN = TL::TN, PA = TL::PA, PB = TL::PB, RPP = TL::RPP;
  constexpr int KB = TL::KB, NST = TL::NST, KS = TL::KS;
  static_assert(!PRE || (sizeof(T) == 4 && MODE != MODE_DENSE), "split weights: fp32 convolutions");
  constexpr int KBB = PRE ? KB / 2 * 3 : KB;                                   // bytes of a column in LDS
  constexpr bool SHARE = TL::SHARE, QUAD = TL::QUAD;
  static_assert(!QUAD || (sizeof(T) == 2 && MODE != MODE_DENSE && KB == 128 && NST == 2 && KS == 1 && !SHARE && TM == 4 && TN == 2 && PA == 4 && PB == 4),
                "quadrants: bf16, 256 x 256");
  static_assert(!SHARE || (sizeof(T) == 2 && MODE == MODE_UP && KS == 1), "shared pixels: bf16, MODE_UP");
  constexpr int SLOTS = TL::SLOTS;
  constexpr int A_RING = SHARE ? 2 * SLOTS * KB : NST * BM * KB;               // of one group
  constexpr int RING = A_RING + NST * BN * KBB;
  constexpr int SMEM_RING = KS * RING;
  constexpr int ROWTAB = BM * 8;                                               // see the epilogue
  constexpr int SMEM_EPI = ROWTAB + (TL::NT / 64) * 32 * (TN * 32 * 4 + 16);
  constexpr int SMEM = SMEM_RING > SMEM_EPI ? SMEM_RING : SMEM_EPI;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[SMEM];
  const int kgrp = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / TL::NT);      // this wave's share of the reduction
  unsigned char* const As = smem + kgrp * RING;        // buffer s at As + s * BM * KB
  unsigned char* const Bs = As + A_RING;               // buffer s at Bs + s * BN * KBB
  constexpr int BK = KB / (int)sizeof(T);              // elements of K per chunk
  constexpr int LINES = 128 / KB;                      // chunks per 128-byte line
  constexpr int EPV = 16 / (int)sizeof(T);
  constexpr int RPB = TL::NT / (KB / 32), PP = BN / RPB;           // PRE: rows of a plane filled per pass, passes per plane
  constexpr int LPT = PA + (PRE ? 3 * PP : PB);        // loads per thread per chunk
  int tid = KS == 1 ? (int)threadIdx.x : (int)threadIdx.x - kgrp * TL::NT, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / TL::WN, wn = wave % TL::WN;

  // ---- which tile: consecutive virtual ids stay on one XCD (block ids are dealt round-robin to the 8 XCDs).
  // Virtual id = ((M-tile * segments + segment) * phases + phase) * N-tiles + N-tile: blocks that run together on
  // an XCD read the same activations (other phase / N-tile) or the same model's weights (other M-tile, segment)
  // out of that XCD's L2.
  constexpr int NPH = (MODE == MODE_UP) ? 4 : 1;
  const int NT = (p.N + BN - 1) / BN;
  const int Ttot = p.tpre[p.L];
  const int total = Ttot * NT * p.nseg * NPH;
  const int per_xcd = (total + 7) >> 3;
  const int slot = blockIdx.x >> 3;
  if (slot >= per_xcd) return;
  const int v = (blockIdx.x & 7) * per_xcd + slot;
  if (v >= total) return;
  const int nt = v % NT;
  const int v1 = v / NT;
  const int phase = v1 % NPH;
  const int v2 = v1 / NPH;
  const int sidx = v2 % p.nseg;
  const int mt = v2 / p.nseg;
  int lo = 0;
  if (p.tmodel) {
    lo = p.tmodel[mt];
  } else {
    int hi = p.L;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (p.tpre[mid] <= mt) lo = mid; else hi = mid;
    }
  }
  const int l = lo;
  const int seg = p.seg_first + sidx;
  const int s0 = p.offs[l], s1 = p.offs[l + 1];
  const int Hr = p.Hr, Hin = p.Hin, C = p.C, N = p.N;
  const int rps = Hr * Hr;
  const int Mrows = (s1 - s0) * rps;
  const int m0 = (mt - p.tpre[l]) * BM;
  const long long sample_base = (long long)seg * p.seg_samples + s0;
  const int py = phase >> 1, px = phase & 1;

  constexpr int SZ = (int)sizeof(T);
  const int cpl = C * SZ / 128;   // 128-byte channel lines per tap
  // Pixel rows this tile covers (rows are ordered y, sample, x) and the taps that are inside the map for at least
  // one of them: a tap row that is outside for the whole tile contributes zeros only and its K-chunks are skipped.
  const int row_block = (s1 - s0) * Hr;
  int cnt_lo = 4, cnt_hi = 4;     // down: valid taps of the classes with ky even / odd ; up: cnt_lo = valid taps
  bool first_gone = false;        // the skipped taps are the first ones of their group (otherwise the last ones)
  if (MODE != MODE_DENSE) {
    // (scalar registers: the divisions are vector instructions, and the K order that follows from them would stay in vector registers)
    const int y_lo = __builtin_amdgcn_readfirstlane(m0 / row_block);
    const int y_hi = __builtin_amdgcn_readfirstlane((min(m0 + BM, Mrows) - 1) / row_block);
    const bool top_only = y_hi == 0, bottom_only = y_lo == Hr - 1;          // only the first / last pixel row
    if (MODE == MODE_DOWN) {
      if (top_only) cnt_lo = 2;                      // ky = 0 reads row -1
      if (bottom_only) cnt_hi = 2;                   // ky = 3 reads row Hin
      first_gone = top_only;
    } else {
      // phase py = 0 gathers rows y and y - 1, py = 1 rows y + 1 and y (tap index a = 0, 1 in this order)
      if (py == 0 && top_only) cnt_lo = 2;           // a = 1 (row y - 1) is gone: the last ones
      if (py == 1 && bottom_only) { cnt_lo = 2; first_gone = true; }   // a = 0 (row y + 1) is gone
    }
  }
  const int chunks_per_tap = cpl * LINES;
  const int nk = (MODE == MODE_DOWN) ? 2 * (cnt_lo + cnt_hi) * chunks_per_tap
                                     : (MODE == MODE_UP ? cnt_lo * chunks_per_tap : C / BK);
  const int wns = p.w_nstride;   // rows per tap in the weight block (N, or more when only some rows are used)
  // this model's slice of the gathered tensor (one segment) and its weight block, as bounds-checked buffers
  const int nsamp = s1 - s0;
  const long long a_elems = (MODE == MODE_DENSE) ? (long long)nsamp * rps * C : (long long)nsamp * Hin * Hin * C;
  const T* a_base = static_cast<const T*>(p.A) + ((MODE == MODE_DENSE) ? sample_base * rps * C : sample_base * (long long)(Hin * Hin) * C);
  // A tap's pixel offset can be negative: the gathered tensor's buffer starts `bias` bytes in front of the slice, and the
  // offsets carry `bias` more (down: in the rows' part, which starts at pixel (-1, -1); up: in the taps' part).  No lane
  // reads in front of the slice: those taps are masked.
  const unsigned px_bytes = (unsigned)(C * SZ), row_bytes = (unsigned)(Hin * C * SZ), wtap_bytes = (unsigned)(wns * C * SZ);
  const unsigned bias = (MODE == MODE_DENSE) ? 0u : row_bytes + px_bytes;
  const int4v a_rsrc = make_rsrc(reinterpret_cast<const unsigned char*>(a_base) - bias, (unsigned long long)a_elems * SZ + bias);
  // PRE: a descriptor for every plane, so that a 32-bit offset need only reach over one of them
  int4v w_rsrc[PRE ? 3 : 1];
  if constexpr (PRE) {
#pragma unroll
    for (int pl = 0; pl < 3; ++pl)
      w_rsrc[pl] = make_rsrc(static_cast<const bf16_t*>(p.W) + (long long)l * p.w_stride + pl * p.w_plane, 32ull * wns * C);
  } else {
    w_rsrc[0] = make_rsrc(static_cast<const T*>(p.W) + (long long)l * p.w_stride, (unsigned long long)(MODE == MODE_DENSE ? 1 : 16) * wns * C * SZ);
  }

  // ---- per-thread load assignment: rows tid/CPR + RPP i, LDS position tid % CPR of the row, which holds the row's
  // 16-byte chunk (tid % CPR) ^ swizzle(row) (RPP is a multiple of the swizzle period, so the same chunk in every
  // pass).  Per row: byte offset of its pixel at tap offset (0, 0), and the set of taps that fall outside the map (all of
  // them for a row past the model's end): a bit turned into a mask and or-ed into the offset sends the lane out of the
  // buffer, so a load costs two vector instructions, one for the weights.
  constexpr int CPR = TL::CPR;
  const int row0 = tid / CPR;
  const int chunk = (tid % CPR) ^ fwd_swz<KB>(row0);
  constexpr int PS = SHARE ? (SLOTS + RPP - 1) / RPP : PA;       // passes over the pixels
  unsigned apix[PS], bcol[PRE ? PP : PB];
  int outside[PS];
  // SHARE: slot t of a stage is pixel p = u % (H + 1), column p - 1 + px, of run u / (H + 1) of H rows, u = t + x0, the first run being the
  // one that the tile's first row lies in, x0 columns behind its start.  Tile row r reads the slots p = x (tap b = 1) and x + 1 (b = 0).
  // Per slot the filter rows whose pixel is outside the map.
  constexpr int G = 256 / KB;
  const int q0 = SHARE ? m0 / Hr : 0, x0 = m0 - q0 * Hr;
  const int need = BM + (BM - 1 + x0) / Hr + 1;                  // slots that the tile's rows read
  unsigned arow[2][TM];
  if constexpr (SHARE) {
    const float inv_run = 1.f / (float)(Hr + 1), inv_n = 1.f / (float)nsamp;
#pragma unroll
    for (int i = 0; i < PS; ++i) {
      const int u = row0 + RPP * i + x0, run = (int)(((float)u + 0.5f) * inv_run), p_ = u - run * (Hr + 1);      // (exact: u < 1024)
      const int q = q0 + run;
      int y = (int)((float)q * inv_n);
      y -= y * nsamp > q ? 1 : 0;
      y += (y + 1) * nsamp <= q ? 1 : 0;
      const int n = q - y * nsamp;
      outside[i] = -1;
      if (y < Hr && (unsigned)(p_ + px - 1) < (unsigned)Hin)
        outside[i] = ~(((unsigned)(y + py) < (unsigned)Hin ? 1 : 0) | ((unsigned)(y + py - 1) < (unsigned)Hin ? 2 : 0));
      const int chunk_ = (tid % CPR) ^ (share_xor(Hr, G, run, p_) & (CPR - 1));
      apix[i] = (unsigned)((((n * Hin + y) * Hin + p_) * C + chunk_ * EPV) * SZ);
    }
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      const int v = x0 + wm * TM * 32 + t * 32 + (lane & 31), run = v / Hr, x = v - run * Hr;
#pragma unroll
      for (int sft = 0; sft < 2; ++sft) {
        const int slot = run * (Hr + 1) + x + sft - x0;
        arow[sft][t] = slot * KB + (((lane >> 5) ^ (share_xor(Hr, G, run, x + sft) & (CPR - 1))) << 4);
      }
    }
  } else
#pragma unroll
  for (int i = 0; i < PA; ++i) {
    const int r = m0 + row0 + RPP * i;
    apix[i] = 0;
    outside[i] = -1;
    if (r < Mrows) {
      if (MODE == MODE_DENSE) {
        apix[i] = (unsigned)((r * C + chunk * EPV) * SZ);
        outside[i] = 0;
      } else {
        int n, y, x;
        decode_row_yfirst(r, Hr, row_block, p.hr_shift, n, y, x);
        const int by = (MODE == MODE_DOWN) ? 2 * y : y, bx = (MODE == MODE_DOWN) ? 2 * x : x;      // (down: + 1)
        apix[i] = (unsigned)((((n * Hin + by) * Hin + bx) * C + chunk * EPV) * SZ);
        int inside = 0;
        if (MODE == MODE_DOWN) {             // tap (ky, kx) is inside iff row by - 1 + ky and column bx - 1 + kx are: separable
          int xm = 0;
#pragma unroll
          for (int k = 0; k < 4; ++k) xm |= ((unsigned)(bx - 1 + k) < (unsigned)Hin ? 1 : 0) << k;
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if ((unsigned)(by - 1 + k) < (unsigned)Hin) inside |= xm << (4 * k);
        } else {
          for (int t = 0; t < 4; ++t) {
            const int iy = by + py - (t >> 1), ix = bx + px - (t & 1);
            if ((unsigned)iy < (unsigned)Hin && (unsigned)ix < (unsigned)Hin) inside |= 1 << t;
          }
        }
        outside[i] = ~inside;
      }
    }
  }
  if constexpr (PRE) {
    static_assert(PP >= 1 && RPB % 16 == 0, "loader shape");
    const int brow0 = tid / (KB / 32), bchunk = (tid % (KB / 32)) ^ fwd_swz<KB / 2>(brow0);
#pragma unroll
    for (int i = 0; i < PP; ++i) {
      const int col = nt * BN + brow0 + RPB * i;
      bcol[i] = col < N ? (unsigned)((col * C + bchunk * 8) * 2) : NO_ROW;
    }
  } else {
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      const int col = nt * BN + (QUAD ? quad_col(row0 + RPP * i) : row0 + RPP * i);
      bcol[i] = col < N ? (unsigned)((col * C + chunk * EPV) * SZ) : NO_ROW;
    }
  }

  const unsigned lds0 = (unsigned)(uintptr_t)As;       // LDS byte address of the buffers
  // The next K-chunk to load
  KOrder<MODE, KB, QUAD> order;
  order.cpl = cpl; order.cnt_lo = cnt_lo; order.cnt_hi = cnt_hi; order.first_gone = first_gone; order.py = py; order.px = px;
  order.row_bytes = row_bytes; order.px_bytes = px_bytes; order.wtap_bytes = wtap_bytes;
  auto load_chunk = [&](int stage, auto split) {       // this group's next chunk, into a buffer
    const unsigned a_dst = lds0 + (stage * BM + wave * (1024 / KB)) * KB;        // + pass * RPP rows
    const unsigned b_dst = lds0 + NST * BM * KB + stage * BN * KBB + wave * 1024;
#pragma unroll
    for (int i = 0; i < PA; ++i)
      load16_to_lds(a_rsrc, apix[i] | (unsigned)__builtin_amdgcn_sbfe(outside[i], order.tap, 1), order.aoff, a_dst + i * RPP * KB);
    if constexpr (PRE && split.value) {
#pragma unroll
      for (int pl = 0; pl < 3; ++pl)
#pragma unroll
        for (int i = 0; i < PP; ++i)
          load16_to_lds(w_rsrc[pl], bcol[i], order.woff >> 1, b_dst + (pl * BN + i * RPB) * (KB / 2));
    } else if constexpr (PRE) {
      // the weights as they are, value by value (tiles that are computed again: rare)
      const float* const raw = p.w_raw + (long long)l * p.raw_stride + (long long)order.wtap * wns * C;
      for (int e = tid; e < BN * CPR; e += TL::NT) {
        const int row = e / CPR, col = nt * BN + row, kk = order.line * 32 + ((e % CPR) ^ fwd_swz<KB>(row)) * 4;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (col < N) {
          const float* const q = raw + (long long)col * p.raw_n + (long long)kk * p.raw_k;
          v = make_float4(q[0], q[p.raw_k], q[2 * (long long)p.raw_k], q[3 * (long long)p.raw_k]);
        }
        *reinterpret_cast<float4*>(Bs + stage * BN * KBB + e * 16) = v;
      }
    } else {
#pragma unroll
      for (int i = 0; i < PB; ++i) load16_to_lds(w_rsrc[0], bcol[i], order.woff, b_dst + i * RPP * KB);
    }
#pragma unroll
    for (int i = 0; i < KS; ++i) order.advance();
  };
  floatx16 acc[TM][TN];

  // Ring of NST buffers: chunk c lives in buffer c % NST.  While chunk c is multiplied, chunks c+1 .. c+NST-1 are on
  // their way; the barrier that ends iteration c tells every wave that chunk c+1 has landed everywhere and that
  // buffer c % NST may be refilled (with chunk c+NST, by the next iteration).
  floatx16 low[TM][TN];
  auto k_loop = [&](auto split) __attribute__((always_inline)) {
    order.start();
    clear_acc(acc);
    if constexpr (split.value) clear_acc(low);
    for (int i = 0; i < kgrp; ++i) order.advance();
    int st_load = 0, st = 0;                           // buffers of the next chunk to load and of the current one
    const int mine = (nk - kgrp + KS - 1) / KS, steps = (nk + KS - 1) / KS;      // this group's chunks; the barriers are everyone's
    for (int c = 0; c < NST - 1 && c < mine; ++c) load_chunk(st_load++, split);
    if (KS > 1 && mine >= NST - 1) wait_vm<(NST - 2) * LPT>(); else wait_vm<0>();
    __syncthreads();
    for (int kc = 0; kc < steps; ++kc) {
      const bool more = kc + NST - 1 < mine;
      if (more) {
        load_chunk(st_load, split);
        st_load = st_load == NST - 1 ? 0 : st_load + 1;
      }
      if (KS == 1 || kc < mine) {
        if constexpr (split.value) tile_mma_split<TM, TN, KB, PRE, BN>(acc, low, As + st * BM * KB, Bs + st * BN * KBB, wm, wn, lane);
        else tile_mma_fwd<T, TM, TN, KB>(acc, As + st * BM * KB, Bs + st * BN * KBB, wm, wn, lane);
      }
      st = st == NST - 1 ? 0 : st + 1;
      if (more) wait_vm<(NST - 2) * LPT>(); else wait_vm<0>();     // chunk kc + 1 has landed; those behind it may stay in flight
      __syncthreads();
    }
  };
  // SHARE: stages of pixels and, two to a stage, chunks of weights.  Stage order, fastest first: the halves of a 128-byte line (KB = 64), the
  // filter rows, which read the same pixels shifted by a row, the channel line.  The next stage's pixels are requested at the start of a stage, its
  // weights NST - 1 chunks ahead.
  struct Stage { int part = 0, j = 0, line = 0; };
  const int frows = cnt_lo >> 1;                       // filter rows a = 0, 1 (y + py - a), or the one that is inside the map
  auto stage_row = [&](const Stage& g) { return frows == 2 ? g.j : (first_gone ? 1 : 0); };
  auto stage_next = [&](Stage& g) {
    if (LINES == 2) {
      g.part ^= 1;
      if (g.part) return;
    }
    if (++g.j < frows) return;
    g.j = 0;
    ++g.line;
  };
  auto load_pixels = [&](const Stage& g, int buf) {
    const int a = stage_row(g);
    const unsigned off = (py - a + 1) * row_bytes + px * px_bytes + g.line * 128 + g.part * KB;
    const unsigned dst = lds0 + buf * SLOTS * KB + wave * 1024;
#pragma unroll
    for (int i = 0; i < PS; ++i)
      if (i < PA || RPP * i + wave * (1024 / KB) < need)          // (a wave's copy fills 1024 / KB slots; the last passes may have none)
        load16_to_lds(a_rsrc, apix[i] | (unsigned)__builtin_amdgcn_sbfe(outside[i], a, 1), off, dst + i * RPP * KB);
  };
  auto load_weights = [&](const Stage& g, int sft, int buf) {
    const int tap = (2 * stage_row(g) + 1 - py) * 4 + 2 * (1 - sft) + 1 - px;
    const unsigned off = tap * wtap_bytes + g.line * 128 + g.part * KB;
    const unsigned dst = lds0 + A_RING + buf * BN * KBB + wave * 1024;
#pragma unroll
    for (int i = 0; i < PB; ++i) load16_to_lds(w_rsrc[0], bcol[i], off, dst + i * RPP * KB);
  };
  auto share_loop = [&]() __attribute__((always_inline)) {
    clear_acc(acc);
    const int stages = nk >> 1;
    Stage ga, gb;                                                 // of the next pixels and of the next weights to load
    int sb = 0, b_load = 0, b_cur = 0;
    auto next_weights = [&]() {
      load_weights(gb, sb, b_load);
      b_load = b_load == NST - 1 ? 0 : b_load + 1;
      sb ^= 1;
      if (!sb) stage_next(gb);
    };
    load_pixels(ga, 0);
    stage_next(ga);
    for (int c = 0; c < NST - 1; ++c) next_weights();             // (a stage has two)
    wait_vm<0>();
    __syncthreads();
    for (int i = 0; i < stages; ++i) {
      const bool more = i + 1 < stages;
      const unsigned a_stage = (i & 1) * (SLOTS * KB);
      // first tap.  More stages: two chunks of weights at least are not loaded yet
      if (NST == 2 || more) next_weights();
      if (more) {
        load_pixels(ga, (i + 1) & 1);
        stage_next(ga);
      }
      tile_mma_rows<T, TM, TN, KB>(acc, arow[0], a_stage, As, Bs + b_cur * BN * KBB, wn, lane);
      b_cur = b_cur == NST - 1 ? 0 : b_cur + 1;
      // the second tap's weights have landed; what was requested after them may stay in flight: later weights and the pixels, PA or more copies
      if (more) wait_vm<(NST - 2) * PB + PA>(); else wait_vm<0>();
      __syncthreads();
      if (more) next_weights();
      tile_mma_rows<T, TM, TN, KB>(acc, arow[1], a_stage, As, Bs + b_cur * BN * KBB, wn, lane);
      b_cur = b_cur == NST - 1 ? 0 : b_cur + 1;
      // the next stage's pixels and first weights have landed
      if (more && NST > 2) wait_vm<PB>(); else wait_vm<0>();
      __syncthreads();
    }
  };
  // QUAD.  With whole chunks in two buffers a buffer is free when its last K-step has been read and has to be full one chunk later, so a chunk took
  // at least as long as its 64 copies: 1100 to 1400 cycles to issue, in which the waves stand in front of the first products, and the slowest one's
  // way to memory, 3500 to 3900 in all (a launch's cycles over the chunks of its rounds of blocks) for 2048 of MFMAs.  Here a wave multiplies half
  // its rows by half its columns at a time, in the order (0, f) (0, s) (1, s) (1, f) with the operands of all four K-steps in registers, f and s
  // being the halves of columns, f = 0 in even chunks and 1 in odd ones.  A quarter needs one half of an operand that the previous ones did not,
  // which is read in the quarter before it; the quarter after that, the half's place in LDS is filled with that of the chunk after the next.  So
  // every half has six quarters and a part of one to arrive in, two copies a wave go out in each, between the products, and one barrier a quarter
  // says both that the next half is here and that the last one is free.  Cycles of a launch, 128 -> 256 channels at side 8, two segments of 6400
  // samples: 1538k -> 1276k, 256 -> 512 at side 4 1391k -> 1146k (matrix pipe busy 0.50 -> 0.60 and 0.52 -> 0.63 of them).  The clock goes down with
  // the power the pipe takes, 2.05 -> 1.8 GHz, which leaves 769 -> 688 and 701 -> 616 us; 512 -> 256 transposed, side 4, one segment 363 -> 331.
  // Issuing the copies in front of the reads or between them, or at a raised wave priority: +-0.5 %.
  auto quad_loop = [&](auto) __attribute__((always_inline)) {      // (a template, so that only the tiles that call it compile it)
    clear_acc(acc);
    order.start();
    const int a_bytes = a_rsrc.z, w_bytes = w_rsrc[0].z;
    int4v ra = a_rsrc, rw = w_rsrc[0];
    int to_load = nk;
    // 128 of 256 registers are accumulators and 96 operands, so the rest is kept few: the masks of taps outside the map, 16 bits a row,
    // of passes i and i + 2 share one, and a lane's four columns, a whole number of columns apart, one offset
    const int out2[2] = {(outside[0] & 0xffff) | (outside[2] << 16), (outside[1] & 0xffff) | (outside[3] << 16)};
    const int lds_wave = __builtin_amdgcn_readfirstlane((int)lds0 + wave * 1024);
    // (the offsets come out of 64-bit multiply-adds, whose upper halves would stay in registers)
    unsigned pix[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) asm volatile("v_mov_b32 %0, %1" : "=v"(pix[i]) : "v"(apix[i]));
    auto load_a = [&](auto half, auto buf) __attribute__((always_inline)) {
      static_for<0, 2>([&](auto i) __attribute__((always_inline)) {
        load16_to_lds_at<buf.value * 32768 + half.value * 8192 + i.value * 16384>(
            ra, pix[half.value + 2 * i.value] | (unsigned)__builtin_amdgcn_sbfe(out2[half.value], order.tap + 16 * i.value, 1), order.aoff, lds_wave);
      });
    };
    auto load_b = [&](auto half, auto buf) __attribute__((always_inline)) {
      static_for<0, 2>([&](auto i) __attribute__((always_inline)) {
        load16_to_lds_at<65536 + buf.value * 32768 + half.value * 16384 + i.value * 8192>(
            rw, bcol[0], order.woff + (unsigned)((half.value * 32 + i.value * 128) * C * SZ), lds_wave);
      });
    };
    auto next_chunk = [&]() __attribute__((always_inline)) {
      const bool more = order.next(to_load);
      ra.z = more ? a_bytes : 0;
      rw.z = more ? w_bytes : 0;
    };
    const int r = lane & 31, h = lane >> 5, sw = fwd_swz<KB>(r);
    const int a0 = (wm * 128 + r) * 128 + ((h ^ sw) << 4), b0 = 65536 + (wn * 32 + r) * 128 + ((h ^ sw) << 4);
    u32x4 a[2][2][4], b[2][4];
    auto read_a = [&](auto half, auto buf, auto k) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
        a[half.value][t][k.value] = *reinterpret_cast<const u32x4*>(smem + (a0 ^ (k.value << 5)) + buf.value * 32768 + half.value * 8192 + t * 4096);
    };
    auto read_b = [&](auto half, auto buf, auto k) __attribute__((always_inline)) {
      b[half.value][k.value] = *reinterpret_cast<const u32x4*>(smem + (b0 ^ (k.value << 5)) + buf.value * 32768 + half.value * 16384);
    };
    const std::integral_constant<int, 0> c0{};
    const std::integral_constant<int, 1> c1{};
    // the first two chunks, and the registers that the first quarter multiplies; the copies of chunk j go out in the order A half 0, first B,
    // second B, A half 1, the first of them a quarter earlier than the others.  (Behind the last chunk the descriptors are empty and the
    // copies write zeros, which nothing multiplies, so that the count in flight stays the same.)
    load_a(c0, c0); load_b(c0, c0); load_b(c1, c0); load_a(c1, c0);
    next_chunk();
    load_a(c0, c1); load_b(c1, c1); load_b(c0, c1); load_a(c1, c1);
    next_chunk();
    quad_wait<12>();
    static_for<0, 4>([&](auto k) __attribute__((always_inline)) { read_a(c0, c0, k); read_b(c0, c0, k); });
    quad_wait<10>();
    load_a(c0, c0);
    // a quarter of a chunk: rows ah, columns bh; reads(k) and loads(k) go between its four K-steps
    auto quarter = [&](auto ah, auto bh, auto&& reads, auto&& loads) __attribute__((always_inline)) {
      static_for<0, 4>([&](auto k) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
          mma16B(acc[ah.value * 2 + t][bh.value], __builtin_bit_cast(uint4, a[ah.value][t][k.value]), __builtin_bit_cast(uint4, b[bh.value][k.value]), bf16_t());
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (k.value < 2) {
          reads(std::integral_constant<int, 2 * k.value>{});
          reads(std::integral_constant<int, 2 * k.value + 1>{});
        }
        if constexpr (k.value == 2) loads();
        __builtin_amdgcn_sched_barrier(0);
      });
    };
    // chunk in buffer BUF, whose first columns are half BUF, its second ones the other half
    auto chunk = [&](auto buf) __attribute__((always_inline)) {
      constexpr int B = buf.value;
      const std::integral_constant<int, B> first{};
      const std::integral_constant<int, 1 - B> second{};
      quarter(c0, first, [&](auto k) __attribute__((always_inline)) { read_b(second, buf, k); }, [&]() __attribute__((always_inline)) { load_b(first, buf); });
      quad_wait<12>();
      quarter(c0, second, [&](auto k) __attribute__((always_inline)) { read_a(c1, buf, k); }, [&]() __attribute__((always_inline)) { load_b(second, buf); });
      quad_wait<12>();
      quarter(c1, second, [&](auto k) __attribute__((always_inline)) { read_a(c0, second, k); }, [&]() __attribute__((always_inline)) { load_a(c1, buf); });
      quad_wait<12>();
      quarter(c1, first, [&](auto k) __attribute__((always_inline)) { read_b(second, second, k); },
              [&]() __attribute__((always_inline)) { next_chunk(); load_a(c0, second); });
      quad_wait<12>();
    };
    for (int c = 0; c < nk; c += 2) {
      chunk(c0);
      chunk(c1);
    }
    wait_vm<0>();
    __syncthreads();
  };
  if constexpr (QUAD) {
    quad_loop(0);
    lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));      // (not kept through the loop)
    tid = wave * 64 + lane;
  } else if constexpr (SHARE) {
    static_assert(NST == 2 || NST == 3, "the waits count for these");
    share_loop();
  } else if constexpr (SZ == 4) {
    k_loop(std::true_type{});
    add_acc(acc, low);
    if (block_any<TL::NT / 64 * KS>(not_finite(acc), smem, kgrp * (TL::NT / 64) + wave)) k_loop(std::false_type{});
  } else {
    k_loop(std::false_type{});
  }

  if constexpr (KS > 1) {
    // the groups' sums, added in order by the first group, which also does the epilogue (the buffers are free now)
    constexpr int PER = TM * TN * 16 * 4;                // bytes per thread
    static_assert((KS - 1) * TL::NT * PER <= SMEM, "the sums fit into the buffers");
    float4* const sums = reinterpret_cast<float4*>(smem);
    if (kgrp > 0) {
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            sums[((kgrp - 1) * (PER / 16) + (tm * TN + tn) * 4 + e) * TL::NT + tid] =
                make_float4(acc[tm][tn][4 * e], acc[tm][tn][4 * e + 1], acc[tm][tn][4 * e + 2], acc[tm][tn][4 * e + 3]);
    }
    __syncthreads();
    if (kgrp == 0) {
#pragma unroll
      for (int g = 1; g < KS; ++g)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
          for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float4 t = sums[((g - 1) * (PER / 16) + (tm * TN + tn) * 4 + e) * TL::NT + tid];
              acc[tm][tn][4 * e] += t.x; acc[tm][tn][4 * e + 1] += t.y; acc[tm][tn][4 * e + 2] += t.z; acc[tm][tn][4 * e + 3] += t.w;
            }
    }
    __syncthreads();
    if (kgrp > 0) return;                              // (no barrier below waits for the waves that have ended)
  }
  // ---- epilogue: output row index of every tile row, through LDS (the buffers are free now)
  long long* orow = reinterpret_cast<long long*>(smem);
  for (int t = tid; t < BM; t += TL::NT) {
    const int r = m0 + t;
    long long o = -1;
    if (r < Mrows) {
      if (MODE == MODE_DENSE) {
        o = sample_base * rps + r;
      } else {
        int n, y, x;
        decode_row_yfirst(r, Hr, row_block, p.hr_shift, n, y, x);
        const int Hb = 2 * Hr;
        if (MODE == MODE_UP) o = ((sample_base + n) * Hb + (2 * y + py)) * Hb + (2 * x + px);
        else o = ((sample_base + n) * Hr + y) * Hr + x;
      }
    }
    orow[t] = o;
  }
  __syncthreads();
  T* __restrict__ Out = static_cast<T*>(p.Out);
  const T* __restrict__ Aux = static_cast<const T*>(p.Aux);
  {
    // Each wave passes its 32 x (TN*32) blocks (fp32) through a private LDS patch so that every lane stores 16
    // contiguous bytes of an output row (full N is a multiple of 64 for these tiles).  The patch belongs to one
    // wave, whose LDS operations execute in order: no block-wide barrier is needed around it.
    constexpr int WCOLS = TN * 32;
    constexpr int PSTRIDE = WCOLS * 4 + 16;                             // bytes per patch row
    constexpr int CPR = WCOLS / EPV;                                    // 16-byte output chunks per patch row
    unsigned char* patch = smem + ROWTAB + wave * (32 * PSTRIDE);       // after the row tables
    static_assert(SMEM >= ROWTAB + (TL::NT / 64) * 32 * PSTRIDE && SMEM_EPI == ROWTAB + (TL::NT / 64) * 32 * PSTRIDE, "patch area");
    const int colw = nt * BN + wn * WCOLS;                              // first column of this wave
    // EPI_BN: the statistics are known before the GEMM runs, so the pass that reads and writes the stored tensor once more, and the
    // launch that prepares its parameters, are not needed (6400 samples of a hundred 32x32 generators, bf16, 1407 -> 1172 us with the
    // images' own pass gone too; sixteen 28x28 digits, fp32, 62 -> 42).  Applied to the accumulators, where a lane has TN columns: in the
    // store loop it has 16 / sizeof(T) of them, whose parameters' registers cost the 256x128 tile its second block per CU (1422 us).
    // EPI_BIAS_ACT: what is stored is what a pass over the stored products would make of them (which are rounded to the storage type first);
    // that pass took 130 us for 6400 samples of 8192 columns in bf16, and the GEMM takes the 87 that it took without this.
    float bn_sc[TN], bn_mu[TN], bn_be[TN], bn_bi[TN];
    if constexpr (EPI == EPI_BIAS_ACT) {
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) bn_bi[tn] = p.bn_bias[(long long)l * p.bn_pstride + min(colw + tn * 32 + (lane & 31), N - 1)];
    }
    if constexpr (EPI == EPI_BN) {
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) {
        const int col = min(colw + tn * 32 + (lane & 31), N - 1), ch = col % p.bn_C;
        const long long po = (long long)l * p.bn_pstride, ro = (long long)l * p.bn_rstride;
        bn_sc[tn] = p.bn_gamma[po + ch] * (1.0f / sqrtf(p.bn_var[ro + ch] + p.bn_eps));
        bn_mu[tn] = p.bn_mean[ro + ch];
        bn_be[tn] = p.bn_beta[po + ch];
        bn_bi[tn] = p.bn_bias ? p.bn_bias[po + col] : 0.f;
      }
    }
    // EPI_ACT_BWD, EPI_DROP_BWD: the saved outputs of a 32-row block are requested while the block in front of it is stored.  Requested in the store
    // loop, each in its row's branch, they were waited for one by one, the whole way to memory every time.  us, two segments: bf16 256 -> 128
    // channels, side 8, 6400 samples 933 -> 873, 128 -> 64, side 16, 1024 samples 249 -> 227, with dropout 64 -> 64, side 8, 6400 samples 280 -> 233;
    // fp32 128 -> 64, side 7, 1280 samples 244 -> 225.  (A second set of registers, for a whole block ahead, costs the 256x128 tile its second
    // block per CU.)
    constexpr bool AUX = EPI == EPI_ACT_BWD || EPI == EPI_DROP_BWD;
    constexpr int PASSES = 32 * CPR / 64;
    uint4 aux[AUX ? PASSES : 1];
    auto request_aux = [&](int tm, int i) __attribute__((always_inline)) {
      const int cid = lane + 64 * i, pr = cid / CPR, col = colw + (cid - pr * CPR) * EPV;
      const long long o = orow[wm * TM * 32 + tm * 32 + pr];
      aux[i] = *reinterpret_cast<const uint4*>(Aux + (o < 0 ? 0 : o) * N + (col < N ? col : 0));      // (any place for what is not stored)
    };
    if constexpr (AUX)
#pragma unroll
      for (int i = 0; i < PASSES; ++i) request_aux(0, i);
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int pr = (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
          float val = acc[tm][tn][e];
          if constexpr (EPI == EPI_BIAS_ACT) {
            val = to_float(from_float<T>(val)) + bn_bi[tn];
            val = val > 0.f ? val : val * p.slope;
          }
          if constexpr (EPI == EPI_BN) {
            if (p.bn_bias) {
              val += bn_bi[tn];
              if (!(val > 0.f)) val *= 0.f;
            }
            val = (val - bn_mu[tn]) * bn_sc[tn] + bn_be[tn];
            if (!(val > 0.f)) val *= p.slope;
          }
          *reinterpret_cast<float*>(patch + pr * PSTRIDE + (tn * 32 + (lane & 31)) * 4) = val;
        }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int i = 0; i < PASSES; ++i) {
        const int cid = lane + 64 * i;
        const int pr = cid / CPR, pc = cid - pr * CPR;
        const long long o = orow[wm * TM * 32 + tm * 32 + pr];
        const int col = colw + pc * EPV;
        if (o >= 0 && col < N) {
          float vf[EPV];
#pragma unroll
          for (int k = 0; k < EPV; k += 4) {
            const float4 t4 = *reinterpret_cast<const float4*>(patch + pr * PSTRIDE + (pc * EPV + k) * 4);
            vf[k] = t4.x; vf[k + 1] = t4.y; vf[k + 2] = t4.z; vf[k + 3] = t4.w;
          }
          if constexpr (AUX) {      // times the activation's derivative (and the dropout), from the saved output
            const T* aa = reinterpret_cast<const T*>(&aux[i]);
#pragma unroll
            for (int k = 0; k < EPV; ++k)
            {
              const float s = to_float(aa[k]);
              if (!(s > 0.f)) vf[k] *= p.slope;
              if (EPI == EPI_DROP_BWD) vf[k] = dropped(s) ? 0.f : vf[k] * p.drop_scale;
            }
          }
          uint4 vraw;
          if constexpr (sizeof(T) == 2) {
            vraw = make_uint4(pack2_bf16(vf[0], vf[1]), pack2_bf16(vf[2], vf[3]), pack2_bf16(vf[4], vf[5]), pack2_bf16(vf[6], vf[7]));
          } else {
            vraw = make_uint4(__float_as_uint(vf[0]), __float_as_uint(vf[1]), __float_as_uint(vf[2]), __float_as_uint(vf[3]));
          }
          {
            typedef unsigned u4 __attribute__((ext_vector_type(4)));
            u4 q; q.x = vraw.x; q.y = vraw.y; q.z = vraw.z; q.w = vraw.w;
            __builtin_nontemporal_store(q, reinterpret_cast<u4*>(Out + o * N + col));      // read next by another kernel, never by this one
          }
        }
        if constexpr (AUX)
          if (tm + 1 < TM) request_aux(tm + 1, i);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
  if (p.stat_partial) {
    // For the BatchNorm that follows.  Every wave's (TM*32)-row block of the tile is a sub-tile of its own: per column
    // the sum s of its fp32 results and the sum M2 of their squared deviations from the sub-tile's column mean, from which the
    // statistics kernel gets the channel's as sum(M2 + s^2 / n) - (sum s)^2 / N, in double (whose bits pay for what cancels).
    // One pass over the accumulators with the sub-tile's first row as the shift K:
    //   sum = K n + sum(x - K),   M2 = sum((x - K)^2) - (sum(x - K))^2 / n
    // (a sample of the column is as good a shift as its mean up to a few units of the last place), no block-wide
    // barrier and nothing shared between the waves, so a wave is done when its own stores and sums are.
    constexpr int SUB = TM * 32;
    const int nvalid = min(max(Mrows - m0 - wm * SUB, 0), SUB);          // valid rows of this wave's sub-tile: a prefix
    const long long tix = (((long long)phase * p.nseg + sidx) * p.ub_tiles + mt) * TL::WM + wm;
    if (nvalid > 0) {
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) {
        const float K = __shfl(acc[0][tn][0], lane & 31, 64);           // row 0 of the sub-tile, this lane's column
        float s1 = 0.f, s2 = 0.f;
        if (nvalid == SUB) {
#pragma unroll
          for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              const float d = acc[tm][tn][e] - K;
              s1 += d;
              s2 += d * d;
            }
        } else {
#pragma unroll
          for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
              const int rr = tm * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
              const float d = acc[tm][tn][e] - K;
              if (rr < nvalid) { s1 += d; s2 += d * d; }
            }
        }
        s1 += __shfl_xor(s1, 32, 64);
        s2 += __shfl_xor(s2, 32, 64);
        const int col = nt * BN + wn * TN * 32 + tn * 32 + (lane & 31);
        if (lane < 32 && col < N) {
          const float nf = (float)nvalid;
          p.stat_partial[(tix * N + col) * 2] = K * nf + s1;
          const float m2 = s2 - s1 * s1 / nf;
          p.stat_partial[(tix * N + col) * 2 + 1] = m2 < 0.f ? 0.f : m2;      // (a NaN, from squares beyond fp32 for one, stays a NaN)
        }
      }
    }
  }
}

template <typename T, int MODE, int EPI, typename TL, bool PRE>
static void launch_one(ConvArgs a, hipStream_t st) {
  a.hr_shift = log2_or_neg(a.Hr);
  const int NT = (a.N + TL::BN - 1) / TL::BN;
  const long long blocks = ((long long)a.ub_tiles * NT * a.nseg * (MODE == MODE_UP ? 4 : 1) + 7) / 8 * 8;
  if (blocks == 0 || a.nseg == 0) return;
  dim3 grid((unsigned)blocks, 1, 1);
  hipLaunchKernelGGL((conv_gemm_kernel<T, MODE, EPI, TL, PRE>), grid, dim3(TL::NT * TL::KS), 0, st, a);
}

template <typename T, int MODE, int EPI, bool PRE>
static void launch_wide(const ConvArgs& a, hipStream_t st) {
  typedef FwdTiles<T> Tiles;
  if constexpr (sizeof(T) == 2 && MODE == MODE_UP) {
    bool done = false;
    const auto shared = [&](ConvTile id, auto tile) {
      if (done || a.tile != id || !share_fits<decltype(tile)>(a.Hr)) return;
      launch_one<T, MODE, EPI, decltype(tile), PRE>(a, st);
      done = true;
    };
    shared(TILE_MID, typename Tiles::MidShare());
    shared(TILE_SMALL, typename Tiles::SmallShare());
    shared(TILE_NARROW, typename Tiles::NarrowShare());
    if (done) return;
  }
  if constexpr (sizeof(T) == 2) {
    if (a.tile == TILE_BIG) return launch_one<T, MODE, EPI, std::conditional_t<MODE != MODE_DENSE, typename Tiles::BigQuad, typename Tiles::Big>, PRE>(a, st);
    if (a.tile == TILE_MID) return launch_one<T, MODE, EPI, typename Tiles::Mid, PRE>(a, st);
  }
  if (a.tile == TILE_SMALL)
    return launch_one<T, MODE, EPI, std::conditional_t<PRE || sizeof(T) == 2, typename Tiles::Small, typename Tiles::SmallWhole>, PRE>(a, st);
  if (a.tile == TILE_NARROW)
    return launch_one<T, MODE, EPI, std::conditional_t<MODE != MODE_DOWN, typename Tiles::NarrowShort, typename Tiles::Narrow>, PRE>(a, st);
  if (a.tile == TILE_TINY) return launch_one<T, MODE, EPI, typename Tiles::Tiny, PRE>(a, st);
  if (a.tile == TILE_PAIR) return launch_one<T, MODE, EPI, typename Tiles::Pair, PRE>(a, st);
  if (a.tile == TILE_DEEP) return launch_one<T, MODE, EPI, typename Tiles::Deep, PRE>(a, st);
  launch_fail("GEMM: a tile that this storage type does not have");
}

template <typename T, int MODE, int EPI>
static void launch_mode(const ConvArgs& a, hipStream_t st) {
  if constexpr (sizeof(T) == 4 && MODE != MODE_DENSE)
    if (a.w_plane != 0) return launch_wide<T, MODE, EPI, true>(a, st);
  launch_wide<T, MODE, EPI, false>(a, st);
}

// The (mode, epilogue, tile) combinations the networks use.
template <typename T>
void launch_conv(int mode, int epi, const ConvArgs& a, hipStream_t st) {
  // the kernel's assumptions, checked before anything is launched
  if (!a.A || !a.W || !a.Out || !a.offs || !a.tpre || a.N < 1 || a.w_nstride < a.N || a.C % (128 / (int)sizeof(T)) != 0 ||
      ((epi == EPI_ACT_BWD || epi == EPI_DROP_BWD) && !a.Aux) ||
      (epi == EPI_BIAS_ACT && !a.bn_bias) || (epi == EPI_BN && (!a.bn_mean || !a.bn_var || !a.bn_gamma || !a.bn_beta || a.bn_C < 1)))
    return launch_fail("GEMM: null operand, or channel counts that are not whole 128-byte lines");
  if (a.tile == TILE_BIG && a.N % 256 != 0) return launch_fail("GEMM: 256 x 256 tiles need whole tiles of columns");
  if (a.N < 64) return launch_fail("GEMM: fewer than 64 output channels (image-side outputs have their own kernel)");
  const bool pre = a.w_plane != 0;
  {
    // the loaders address one model's slice of A and one weight block with 32-bit byte offsets
    const long long side = mode == MODE_DENSE ? a.Hr : a.Hin;
    if (pre && (sizeof(T) != 4 || mode == MODE_DENSE || !a.w_raw || a.w_plane < 16LL * a.w_nstride * a.C || a.w_plane % 8))
      return launch_fail("GEMM: split weights are those of fp32 convolutions");
    if ((long long)a.seg_samples * side * side * a.C * (long long)sizeof(T) >= (1LL << 31) ||
        16LL * a.w_nstride * a.C * (long long)sizeof(T) >= (1LL << 31))
      return launch_fail("GEMM: one segment of the gathered tensor, or one weight block, is 2 GiB or larger");
  }
  if (mode == MODE_DOWN && epi == EPI_NONE) return launch_mode<T, MODE_DOWN, EPI_NONE>(a, st);
  if (mode == MODE_UP && epi == EPI_NONE) return launch_mode<T, MODE_UP, EPI_NONE>(a, st);
  if (mode == MODE_UP && epi == EPI_ACT_BWD) return launch_mode<T, MODE_UP, EPI_ACT_BWD>(a, st);
  if (mode == MODE_UP && epi == EPI_BN) return launch_mode<T, MODE_UP, EPI_BN>(a, st);
  if (mode == MODE_DENSE && epi == EPI_BN) return launch_mode<T, MODE_DENSE, EPI_BN>(a, st);
  if (mode == MODE_UP && epi == EPI_DROP_BWD) return launch_mode<T, MODE_UP, EPI_DROP_BWD>(a, st);
  if (mode == MODE_DENSE && epi == EPI_NONE) return launch_mode<T, MODE_DENSE, EPI_NONE>(a, st);
  if (mode == MODE_DENSE && epi == EPI_BIAS_ACT) return launch_mode<T, MODE_DENSE, EPI_BIAS_ACT>(a, st);
  launch_fail("GEMM: (mode, epilogue) combination without an instantiation");
}
// Name of the kernel instantiation launch_conv picks (for per-kernel timing): mode, epilogue, tile.
const char* conv_variant_name(int esize, int mode, int epi, const ConvArgs& a) {
  static const char* modes[3] = {"down", "up", "dense"};
  static const char* epis[5] = {"", "+actbwd", "+dropbwd", "+bn", "+bias+act"};
  static char names[2][3][5][7][48];
  char* n = names[esize == 4][mode][epi][a.tile];
  if (!n[0]) snprintf(n, 48, "gemm_%s%s<%s>", modes[mode], epis[epi], tile_info(esize, a.tile).name);
  return n;
}
template void launch_conv<float>(int, int, const ConvArgs&, hipStream_t);
template void launch_conv<bf16_t>(int, int, const ConvArgs&, hipStream_t);

// ---------------------------------------------------------------------------------------------------------
// weight gradient
// ---------------------------------------------------------------------------------------------------------

// Which model the i-th group of blocks works on.  Groups are dealt round-robin to the 8 XCDs in rows of eight; with
// the models sorted by decreasing size the rows alternate direction, so that every XCD gets the same share of the
// rows and starts with its largest models.
__device__ inline int wgrad_model(const WgradArgs& p, int i) {
  if (!p.order) return i;
  const int row = i >> 3;
  if ((row & 1) && row * 8 + 8 <= p.L) i = row * 8 + 7 - (i & 7);
  return p.order[i];
}

// Both operands are stored [row][channel] in HBM while the MFMA wants, per lane, consecutive rows (the reduction
// index) of one channel.  The kernel copies K-chunks of WG_KR rows x BM (BN) channels global -> LDS as they are.
// bf16: ds_read_b64_tr_b16 does the transposition on the way to the registers: within each block of 16 lanes, lane i
// receives element i%4 of the 8-byte groups addressed by lanes i/4, 4 + i/4, 8 + i/4, 12 + i/4; pointing lane s of a
// block at row (s/4), channel group (s%4) therefore hands lane i rows 0..3 of channel i.
// fp32: the chunk is split on the way into LDS (split_loop) and its bf16 planes are read like a bf16 chunk; only a tile that is computed
// again with the fp32 MFMAs (infinities, NaN) has the chunk itself there and reads it four bytes at a time, lane r of a half-wave channel r.
// The 16-byte chunk c of row R sits at position c ^ swz(R), so that the rows one read touches fall into different
// bank groups.
template <typename T> constexpr int wg_kr() { return 128 / (int)sizeof(T); }     // rows (reduction index) per chunk: 64 or 32
template <typename T, int ROWB>
__device__ inline int wg_swz(int row) {   // in 16-byte chunks
  if (sizeof(T) == 4) return 8 * (row & 1);
  return ROWB >= 256 ? 4 * (row & 3) : 4 * ((row >> 1) & 1);
}

template <typename T, typename TL>
__global__ __launch_bounds__(TL::NT, (waves_per_simd<T, TL>())) void wgrad_kernel(WgradArgs p) {
  constexpr int SZ = (int)sizeof(T), EPV = 16 / SZ, WG_KR = wg_kr<T>();
  constexpr int BM = TL::BM, BN = TL::BN, TM = TL::TM, TN = TL::TN, NT_ = TL::NT;
  constexpr int RBA = BM * SZ, RBB = BN * SZ;               // bytes per LDS row
  constexpr int CPA = BM / EPV, CPB = BN / EPV;             // 16-byte chunks per row
  constexpr int PA = WG_KR * CPA / NT_, PB = WG_KR * CPB / NT_;
  constexpr int RPA = NT_ / CPA, RPB = NT_ / CPB;           // rows per loader pass (multiples of 4)
  static_assert(WG_KR * CPA % NT_ == 0 && WG_KR * CPB % NT_ == 0 && RPA % 4 == 0 && RPB % 4 == 0, "loader shape");
  constexpr int STAGE_A = WG_KR * RBA, STAGE_B = WG_KR * RBB;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * (STAGE_A + STAGE_B)];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / TL::WN, wn = wave % TL::WN;

  // ---- tile: all tiles of one (model, row split) run on one XCD -- they read the same rows -- and the
  // (model, split) pairs are dealt round-robin to the XCDs
  const int Cb = p.Cb, Cs = p.Cs, Hs = p.Hs;
  const int Mtot = p.ntaps * Cb;
  const int MT = (Mtot + BM - 1) / BM, NTL = (Cs + BN - 1) / BN;
  const int bid = blockIdx.x;
  const int unit = (bid / (8 * MT * NTL)) * 8 + (bid & 7);
  if (unit >= p.L * p.ksplit) return;
  const int l = wgrad_model(p, unit / p.ksplit), split = unit % p.ksplit;
  const int tile = (bid >> 3) % (MT * NTL);
  const int mt = tile / NTL, nt = tile - mt * NTL;
  const int s0 = p.offs[l], s1 = p.offs[l + 1];
  const int rps = Hs * Hs;
  const int R = (s1 - s0) * rps;
  const int Hb = 2 * Hs;
  const int rows_split = ((R + p.ksplit - 1) / p.ksplit + WG_KR - 1) / WG_KR * WG_KR;
  const int r_lo = split * rows_split, r_hi = min(R, r_lo + rows_split);

  // ---- loader: slot = pass * NT + tid is the 16-byte LDS slot; it holds chunk (slot % CP) ^ swz(row) of row slot / CP
  const int rowA0 = tid / CPA, rowB0 = tid / CPB;
  const int chA = (tid % CPA) ^ wg_swz<T, RBA>(rowA0), chB = (tid % CPB) ^ wg_swz<T, RBB>(rowB0);
  const int mA = mt * BM + chA * EPV;                        // first of this thread's channels along M
  const bool okA = mA < Mtot;
  const int tapA = okA ? mA / Cb : 0;
  const int cA = mA - tapA * Cb;
  const int kyA = p.ntaps == 1 ? 1 : (tapA >> 2), kxA = p.ntaps == 1 ? 1 : (tapA & 3);
  const int cB = nt * BN + chB * EPV;
  const bool okB = cB < Cs;
  const unsigned lds0 = (unsigned)(uintptr_t)smem;
  const long long big_per_sample = p.ntaps == 1 ? (long long)rps * Cb : (long long)Hb * Hb * Cb;

  // Chunks start at multiples of WG_KR rows.  With a power-of-two side of at most WG_KR a chunk is a whole number of
  // samples or of pixel rows, so a thread's rows keep their x, their y offset inside the chunk and their sample
  // offset: everything that depends on the row is computed once, and a chunk only adds a wave-uniform offset
  // (sample n0, pixel row y0 of the chunk's first row) and re-tests the vertical border.
  const bool fast = p.ntaps == 1 || (p.hs_shift >= 0 && Hs <= WG_KR);
  // Reduction order "pixel row first" (y, sample, x) for the models whose samples * H rows per pixel row are whole
  // chunks: a chunk then lies inside one pixel row y0, the vertical border test is the same for the whole chunk, and
  // the chunks of the one pixel row whose tap row ky falls outside the map (y0 = 0 for ky = 0, y0 = H - 1 for
  // ky = 3) hold zeros only and are skipped.  The tile's taps share one ky (4 * Cb >= BM).  The choice depends on the
  // model's own sample count only.
  const int rb = (s1 - s0) * Hs;                    // rows per pixel row
  const bool yfirst = p.ntaps == 16 && fast && rb % WG_KR == 0 && 4 * Cb >= BM && Cb % 8 == 0 && (BM % Cb == 0 || Cb % BM == 0);
  const int ky_tile = (mt * BM / Cb) >> 2;
  unsigned fa_off[PA], fb_off[PB];
  int fa_iy[PA];                   // 2 * (y inside the chunk) - 1 + ky ; a large value marks a lane that never loads
#pragma unroll
  for (int i = 0; i < PA; ++i) {
    const int c = rowA0 + i * RPA;
    fa_off[i] = 0;
    fa_iy[i] = 1 << 20;
    if (okA) {
      if (p.ntaps == 1) {
        fa_off[i] = (unsigned)((c * Cb + cA) * SZ);
        fa_iy[i] = 0;
      } else if (yfirst) {
        // row c of a chunk: sample n0 + c / H, x = c % H, pixel row y0 (chunk-uniform)
        const int sh = p.hs_shift;
        const int ni = c >> sh, xi = c & (Hs - 1);
        const int ix = 2 * xi - 1 + kxA;
        if ((unsigned)ix < (unsigned)Hb) {
          fa_iy[i] = kyA - 1;
          fa_off[i] = (unsigned)((((ni * Hb + fa_iy[i]) * Hb + ix) * Cb + cA) * SZ);    // may wrap below zero: masked
        }
      } else if (fast) {
        const int sh = p.hs_shift;
        const int ni = c >> (2 * sh), rem = c & (rps - 1);
        const int yi = rem >> sh, xi = rem & (Hs - 1);
        const int ix = 2 * xi - 1 + kxA;
        if ((unsigned)ix < (unsigned)Hb) {
          fa_iy[i] = 2 * yi - 1 + kyA;
          fa_off[i] = (unsigned)((((ni * Hb + fa_iy[i]) * Hb + ix) * Cb + cA) * SZ);    // may wrap below zero: masked
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < PB; ++i) {
    const int c = rowB0 + i * RPB;
    if (yfirst) fb_off[i] = (unsigned)((((c >> p.hs_shift) * rps + (c & (Hs - 1))) * Cs + cB) * SZ);
    else fb_off[i] = (unsigned)((c * Cs + cB) * SZ);
  }

  // this thread's byte offsets of a chunk, as a_load(pass, offset) and b_load(pass, offset)
  auto chunk_offsets = [&](int k0, auto&& a_load, auto&& b_load) __attribute__((always_inline)) {
    const int left = r_hi - k0;                 // rows of this chunk that exist
    unsigned b_delta = (unsigned)(k0 * Cs * SZ);
    if (fast) {
      unsigned a_delta;
      int y2 = 0;
      if (p.ntaps == 1) {
        a_delta = (unsigned)(k0 * Cb * SZ);
      } else if (yfirst) {
        const int y0 = k0 / rb, n0 = (k0 - y0 * rb) >> p.hs_shift;
        a_delta = (unsigned)(((n0 * Hb + 2 * y0) * Hb) * Cb * SZ);
        y2 = 2 * y0;
        b_delta = (unsigned)(((n0 * Hs + y0) * Hs) * Cs * SZ);
      } else {
        const int n0 = k0 >> (2 * p.hs_shift), y0 = (k0 & (rps - 1)) >> p.hs_shift;
        a_delta = (unsigned)(((n0 * Hb + 2 * y0) * Hb) * Cb * SZ);
        y2 = 2 * y0;
      }
#pragma unroll
      for (int i = 0; i < PA; ++i) {
        const bool ok = rowA0 + i * RPA < left && (unsigned)(fa_iy[i] + y2) < (unsigned)Hb;
        a_load(i, ok ? fa_off[i] + a_delta : NO_ROW);
      }
    } else {
#pragma unroll
      for (int i = 0; i < PA; ++i) {
        const int r = k0 + rowA0 + i * RPA;
        unsigned off = NO_ROW;
        if (r < r_hi && okA) {
          int n, y, x;
          if (p.rps_inv) {                        // r / rps and rem / Hs as products with the rounded-up reciprocals
            n = (int)__umulhi((unsigned)r, p.rps_inv);
            const int rem = r - n * rps;
            y = (int)__umulhi((unsigned)rem, p.hs_inv);
            x = rem - y * Hs;
          } else {
            decode_row(r, Hs, rps, p.hs_shift, n, y, x);
          }
          const int iy = 2 * y - 1 + kyA, ix = 2 * x - 1 + kxA;
          if ((unsigned)iy < (unsigned)Hb && (unsigned)ix < (unsigned)Hb) off = (unsigned)((((n * Hb + iy) * Hb + ix) * Cb + cA) * SZ);
        }
        a_load(i, off);
      }
    }
#pragma unroll
    for (int i = 0; i < PB; ++i) b_load(i, (rowB0 + i * RPB < left && okB) ? fb_off[i] + b_delta : NO_ROW);
  };
  auto a_slice = [&](int seg) { return static_cast<const T*>(p.Big) + ((long long)seg * p.seg_samples + s0) * big_per_sample; };
  auto b_slice = [&](int seg) { return static_cast<const T*>(p.Small) + ((long long)seg * p.seg_samples + s0) * rps * Cs; };
  const unsigned long long a_slice_bytes = (unsigned long long)(s1 - s0) * big_per_sample * SZ, b_slice_bytes = (unsigned long long)R * Cs * SZ;
  auto load_chunk = [&](int seg, int k0, int stage) __attribute__((always_inline)) {
    const int4v a_rsrc = make_rsrc(a_slice(seg), a_slice_bytes), b_rsrc = make_rsrc(b_slice(seg), b_slice_bytes);
    const unsigned a_dst = lds0 + stage * STAGE_A + wave * 1024;
    const unsigned b_dst = lds0 + 2 * STAGE_A + stage * STAGE_B + wave * 1024;
    chunk_offsets(k0, [&](int i, unsigned off) __attribute__((always_inline)) { load16_to_lds(a_rsrc, off, 0u, a_dst + i * NT_ * 16); },
                  [&](int i, unsigned off) __attribute__((always_inline)) { load16_to_lds(b_rsrc, off, 0u, b_dst + i * NT_ * 16); });
  };

  floatx16 acc[TM][TN], low[TM][TN];      // (low: fp32 only)

  // ---- fragment addressing: lane = 32 * kgrp + 16 * hb + s ; it points at row 8*kgrp + 4*half + s/4 of the k-step,
  // channels 16*hb + 4*(s%4) .. +3 of the 32-channel fragment
  const int s16 = lane & 15, hb = (lane >> 4) & 1, kgrp = lane >> 5;
  const int frow = 8 * kgrp + (s16 >> 2);                    // + 16 * kstep + 4 * half
  const int fch = 2 * hb + ((s16 & 3) >> 1);                 // 16-byte chunk inside the 32-channel fragment (0..3)
  const int fbyte = 8 * (s16 & 1);
  const int swzA = wg_swz<T, RBA>(frow), swzB = wg_swz<T, RBB>(frow);   // frow % 4 (and (frow/2) % 2) do not change with kstep or half
  // The reads of step ks + 1 are issued in front of the MFMAs of step ks (two register sets; the scheduling barriers keep
  // the compiler from pulling them together, which left every step waiting for its own reads).
  auto mma_chunk16 = [&](int stage) __attribute__((always_inline)) {
    const unsigned char* As = smem + stage * STAGE_A;
    const unsigned char* Bs = smem + 2 * STAGE_A + stage * STAGE_B;
    uint4 a[2][TM], b[2][TN];
    auto fetch = [&](int ks, int set) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < TM; ++t) {
        const int ch = ((wm * TM + t) * 4 + fch) ^ swzA;
        const unsigned char* q0 = As + (ks * 16 + frow) * RBA + ch * 16 + fbyte;
        const uint2 lo = lds_read_tr16(q0), hi = lds_read_tr16(q0 + 4 * RBA);
        a[set][t] = make_uint4(lo.x, lo.y, hi.x, hi.y);
      }
#pragma unroll
      for (int t = 0; t < TN; ++t) {
        const int ch = ((wn * TN + t) * 4 + fch) ^ swzB;
        const unsigned char* q0 = Bs + (ks * 16 + frow) * RBB + ch * 16 + fbyte;
        const uint2 lo = lds_read_tr16(q0), hi = lds_read_tr16(q0 + 4 * RBB);
        b[set][t] = make_uint4(lo.x, lo.y, hi.x, hi.y);
      }
    };
    fetch(0, 0);
#pragma unroll
    for (int ks = 0; ks < WG_KR / 16; ++ks) {
      if (ks + 1 < WG_KR / 16) fetch(ks + 1, (ks + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) mma16B(acc[tm][tn], a[ks & 1][tm], b[ks & 1][tn], bf16_t());
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // fp32: a step is the row pairs 2 ks, 2 ks + 1 for two values of ks; lane half h reads row 2 ks + h (swz flips with h only)
  auto mma_chunk32 = [&](int stage) __attribute__((always_inline)) {
    const int r = lane & 31, h = lane >> 5;
    const unsigned char* As = smem + stage * STAGE_A + h * RBA + (r & 3) * 4;
    const unsigned char* Bs = smem + 2 * STAGE_A + stage * STAGE_B + h * RBB + (r & 3) * 4;
    const float* ap[TM];
    const float* bp[TN];
#pragma unroll
    for (int t = 0; t < TM; ++t) ap[t] = reinterpret_cast<const float*>(As + ((((wm * TM + t) * 8 + (r >> 2)) ^ (8 * h)) * 16));
#pragma unroll
    for (int t = 0; t < TN; ++t) bp[t] = reinterpret_cast<const float*>(Bs + ((((wn * TN + t) * 8 + (r >> 2)) ^ (8 * h)) * 16));
    float a[2][2][TM], b[2][2][TN];
    auto fetch = [&](int step, int set) __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
#pragma unroll
        for (int t = 0; t < TM; ++t) a[set][q][t] = ap[t][(2 * step + q) * 2 * BM];
#pragma unroll
        for (int t = 0; t < TN; ++t) b[set][q][t] = bp[t][(2 * step + q) * 2 * BN];
      }
    };
    fetch(0, 0);
#pragma unroll
    for (int st = 0; st < WG_KR / 4; ++st) {
      if (st + 1 < WG_KR / 4) fetch(st + 1, (st + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
          for (int tn = 0; tn < TN; ++tn)
            acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[st & 1][q][tm], b[st & 1][q][tn], acc[tm][tn], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // fp32 through splits: the chunk comes into registers, is split there, once a block, and goes to LDS as three planes of bf16 rows, which are then
  // read like a bf16 chunk.  Split by the waves that multiply, every value was split twice in a 128 x 128 tile, and the vector instructions of that took
  // longer (830 cycles a 16-row step) than the MFMAs (770): 128 -> 256 channels, side 8, two segments of 20 x 64 samples 1035 -> 942 us,
  // 256 -> 512, side 4 1060 -> 949; 10 x 128 samples, 64 -> 128, side 7 256 -> 229.  The matrix pipe is busy 0.57 of the
  // time a CU has blocks.  PLANE: bytes of one; buffers are not doubled, the next chunk waits in the registers.
  constexpr int PLANE_A = WG_KR * BM * 2, PLANE_B = WG_KR * BN * 2;
  auto split_loop = [&](auto chunk_row, int per_seg, int nchunks) __attribute__((always_inline)) {
    clear_acc(acc);
    clear_acc(low);
    if (nchunks <= 0) return;
    static_assert(sizeof(T) == 2 || 3 * (PLANE_A + PLANE_B) <= 2 * (STAGE_A + STAGE_B), "the planes fit into the buffers");
    u32x4 va[PA], vb[PB];
    auto fetch = [&](int seg, int k0) __attribute__((always_inline)) {
      const __amdgpu_buffer_rsrc_t ra = buffer_of(a_slice(seg), a_slice_bytes), rb_ = buffer_of(b_slice(seg), b_slice_bytes);
      chunk_offsets(k0, [&](int i, unsigned off) __attribute__((always_inline)) { va[i] = __builtin_amdgcn_raw_buffer_load_b128(ra, off, 0, 0); },
                    [&](int i, unsigned off) __attribute__((always_inline)) { vb[i] = __builtin_amdgcn_raw_buffer_load_b128(rb_, off, 0, 0); });
    };
    // four channels of a row into the three planes
    auto put = [&](unsigned char* plane0, int plane_bytes, int row_bytes, int row, int ch, int swz, const u32x4& v) __attribute__((always_inline)) {
      const Split4 q = split4(v);
      unsigned char* const at = plane0 + row * row_bytes + (((ch >> 1) ^ swz) << 4) + (ch & 1) * 8;
      *reinterpret_cast<uint2*>(at) = q.h;
      *reinterpret_cast<uint2*>(at + plane_bytes) = q.m;
      *reinterpret_cast<uint2*>(at + 2 * plane_bytes) = q.l;
    };
    unsigned char* const Ap = smem;
    unsigned char* const Bp = smem + 3 * PLANE_A;
    auto fragment = [&](const unsigned char* base, int plane_bytes, int row_bytes, int tile32, int swz, int ks) __attribute__((always_inline)) {
      const unsigned char* q = base + (ks * 16 + frow) * row_bytes + ((tile32 * 4 + fch) ^ swz) * 16 + fbyte;
      Split8 v;
      const auto one = [&](u32x4& d, const unsigned char* a) __attribute__((always_inline)) {
        const uint2 lo = lds_read_tr16(a), hi = lds_read_tr16(a + 4 * row_bytes);
        d.x = lo.x; d.y = lo.y; d.z = hi.x; d.w = hi.y;
      };
      one(v.h, q);
      one(v.m, q + plane_bytes);
      one(v.l, q + 2 * plane_bytes);
      return v;
    };
    const int sa = wg_swz<bf16_t, BM * 2>(frow), sb = wg_swz<bf16_t, BN * 2>(frow);
    fetch(0, chunk_row(0));
    int seg = 0, cin = 0;
    for (int c = 0; c < nchunks; ++c) {
      if (c > 0) __syncthreads();                                // the previous chunk has been read
#pragma unroll
      for (int i = 0; i < PA; ++i) put(Ap, PLANE_A, BM * 2, rowA0 + i * RPA, chA, wg_swz<bf16_t, BM * 2>(rowA0 + i * RPA), va[i]);
#pragma unroll
      for (int i = 0; i < PB; ++i) put(Bp, PLANE_B, BN * 2, rowB0 + i * RPB, chB, wg_swz<bf16_t, BN * 2>(rowB0 + i * RPB), vb[i]);
      if (c + 1 < nchunks) {
        if (++cin == per_seg) { cin = 0; ++seg; }
        fetch(seg, chunk_row(cin));
      }
      __syncthreads();
#pragma unroll
      for (int ks = 0; ks < WG_KR / 16; ++ks) {
        Split8 b[TN];
#pragma unroll
        for (int t = 0; t < TN; ++t) b[t] = fragment(Bp, PLANE_B, BN * 2, wn * TN + t, sb, ks);
#pragma unroll
        for (int t = 0; t < TM; ++t) mma_split(acc[t], low[t], fragment(Ap, PLANE_A, BM * 2, wm * TM + t, sa, ks), b);
      }
    }
    __syncthreads();
  };

  // QUAD: the forward-type kernel's quarters, with halves of channels on both sides.  A half of an operand is 64 rows of 128 channels in LDS.
  // Cycles of a launch, 128 -> 256 channels at side 8, two segments of 6400 samples: 1911k -> 1639k, 256 -> 512 at side 4 1674k -> 1472k; clock
  // 2.19 -> 2.04 GHz, 877 -> 817 and 800 -> 780 us (one segment 451 -> 433, 472 -> 446).  What is left there are the stores of dW (256 KiB a
  // tile after 16 to 128 chunks) and the last round of blocks (800 tiles on 256 CUs).
  const int chunks_of_share = r_hi > r_lo ? (r_hi - r_lo + WG_KR - 1) / WG_KR : 0;
  auto quad_loop = [&](int bad0, int nbad, int nchunks) __attribute__((always_inline)) {
    clear_acc(acc);
    if (nchunks <= 0) return;
    const int per_seg = chunks_of_share - nbad, sh = p.hs_shift;
    // ---- loader: rows tid / 16 and + 32 of a chunk, 16 bytes: of A channels 128 (chunk / 8) + 64 half + 8 (chunk % 8), of B 64 (chunk / 4) +
    // 32 half + 8 (chunk % 4) of the tile.  What rows 32 further down and the other half add is wave-uniform.
    const int row = tid >> 4, chunk = (tid & 15) ^ (4 * (row & 3));
    const int m = mt * BM + (chunk >> 3) * 128 + (chunk & 7) * 8, tap = m / Cb, ky = tap >> 2, kx = tap & 3;
    const int ni = yfirst ? row >> sh : row >> (2 * sh), yi = yfirst ? 0 : (row & (rps - 1)) >> sh, xi = row & (Hs - 1);
    const int ix = 2 * xi - 1 + kx;
    const bool whole_rows = !yfirst && rps > 32;                 // 32 rows are some pixel rows of the same sample, otherwise some samples
    const unsigned px = (unsigned)(Cb * SZ), line = (unsigned)Hb * px, bias = line + px;      // (row -1, column -1 have offset 0)
    int iy = (unsigned)ix < (unsigned)Hb ? 2 * yi - 1 + ky : 1 << 20;
    unsigned aoff = (unsigned)(ni * Hb * Hb) * px + (unsigned)(2 * yi + ky) * line + (unsigned)(ix + 1) * px + (unsigned)(m - tap * Cb) * SZ;
    unsigned boff = (unsigned)(((yfirst ? (row >> sh) * rps + xi : row) * Cs + nt * BN + (chunk >> 2) * 64 + (chunk & 3) * 8) * SZ);
    const int rows32 = 32 >> sh;                                 // 32 rows in pixel rows of one sample
    const unsigned a32 = whole_rows ? 2 * rows32 * line : (yfirst ? rows32 : 32 >> (2 * sh)) * (unsigned)(Hb * Hb) * px;
    const unsigned b32 = (unsigned)((yfirst ? rows32 * rps : 32) * Cs * SZ);
    const int dy32 = whole_rows ? 2 * rows32 : 0;
    // ---- the chunk to load next
    const unsigned long long a_bytes = (unsigned long long)(s1 - s0) * big_per_sample * SZ + bias, b_bytes = (unsigned long long)R * Cs * SZ;
    const T* a_base = reinterpret_cast<const T*>(reinterpret_cast<const unsigned char*>(static_cast<const T*>(p.Big) + s0 * big_per_sample) - bias);
    const T* b_base = static_cast<const T*>(p.Small) + (long long)s0 * rps * Cs;
    int4v ra = make_rsrc(a_base, a_bytes), rb_ = make_rsrc(b_base, b_bytes);
    int cin = 0, to_load = __builtin_amdgcn_readfirstlane(nchunks), k0, y0 = 0, rem = 0, left, y2;
    unsigned a_delta, b_delta;
    auto place = [&]() __attribute__((always_inline)) {
      k0 = r_lo + (cin < bad0 ? cin : cin + nbad) * WG_KR;
      if (yfirst) {
        y0 = __builtin_amdgcn_readfirstlane(k0 / rb);
        rem = k0 - y0 * rb;
      }
    };
    auto set = [&]() __attribute__((always_inline)) {
      left = r_hi - k0;
      const int n0 = yfirst ? rem >> sh : k0 >> (2 * sh), y = yfirst ? y0 : (k0 & (rps - 1)) >> sh;
      y2 = 2 * y;
      a_delta = (unsigned)((n0 * Hb + y2) * Hb) * px;
      b_delta = yfirst ? (unsigned)(((n0 * Hs + y0) * Hs) * Cs * SZ) : (unsigned)(k0 * Cs * SZ);
    };
    auto next_chunk = [&]() __attribute__((always_inline)) {
      if (--to_load <= 0) {                                      // behind the last chunk: copies of zeros
        ra.z = rb_.z = 0;
        return;
      }
      if (++cin == per_seg) {
        cin = 0;
        a_base += (long long)p.seg_samples * big_per_sample;
        b_base += (long long)p.seg_samples * rps * Cs;
        ra = make_rsrc(a_base, a_bytes);
        rb_ = make_rsrc(b_base, b_bytes);
        place();
      } else if (cin == bad0 && nbad > 0) {
        place();
      } else {
        k0 += WG_KR;
        rem += WG_KR;
        if (rem == rb) { rem = 0; ++y0; }
      }
      // (kept out of the vector registers, of which none is left)
      cin = __builtin_amdgcn_readfirstlane(cin);
      k0 = __builtin_amdgcn_readfirstlane(k0);
      rem = __builtin_amdgcn_readfirstlane(rem);
      y0 = __builtin_amdgcn_readfirstlane(y0);
      set();
    };
    const int lds_wave = __builtin_amdgcn_readfirstlane((int)lds0 + wave * 1024);
    auto load_a = [&](auto half, auto buf) __attribute__((always_inline)) {
      static_for<0, 2>([&](auto i) __attribute__((always_inline)) {
        const bool ok = row + 32 * i.value < left && (unsigned)(iy + y2 + i.value * dy32) < (unsigned)Hb;
        load16_to_lds_at<buf.value * 32768 + half.value * 16384 + i.value * 8192>(ra, ok ? aoff : NO_ROW, a_delta + i.value * a32 + half.value * 128, lds_wave);
      });
    };
    auto load_b = [&](auto half, auto buf) __attribute__((always_inline)) {
      static_for<0, 2>([&](auto i) __attribute__((always_inline)) {
        load16_to_lds_at<65536 + buf.value * 32768 + half.value * 16384 + i.value * 8192>(rb_, row + 32 * i.value < left ? boff : NO_ROW,
                                                                                        b_delta + i.value * b32 + half.value * 64, lds_wave);
      });
    };
    // ---- operands: rows of 128 channels (256 bytes); the two fragments of a half of A differ in bit 2 of the chunk
    const unsigned char* ap[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) ap[t] = smem + frow * 256 + ((wm * 8 + t * 4 + fch) ^ (4 * (frow & 3))) * 16 + fbyte;
    const unsigned char* const bp = smem + 65536 + frow * 256 + ((wn * 4 + fch) ^ (4 * (frow & 3))) * 16 + fbyte;
    u32x4 a[2][2][4], b[2][4];
    auto fragment = [&](const unsigned char* q) __attribute__((always_inline)) {
      const uint2 lo = lds_read_tr16(q), hi = lds_read_tr16(q + 4 * 256);
      u32x4 v;
      v.x = lo.x; v.y = lo.y; v.z = hi.x; v.w = hi.y;
      return v;
    };
    auto read_a = [&](auto half, auto buf, auto k) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < 2; ++t) a[half.value][t][k.value] = fragment(ap[t] + buf.value * 32768 + half.value * 16384 + k.value * 4096);
    };
    auto read_b = [&](auto half, auto buf, auto k) __attribute__((always_inline)) {
      b[half.value][k.value] = fragment(bp + buf.value * 32768 + half.value * 16384 + k.value * 4096);
    };
    const std::integral_constant<int, 0> c0{};
    const std::integral_constant<int, 1> c1{};
    place();
    set();
    load_a(c0, c0); load_b(c0, c0); load_b(c1, c0); load_a(c1, c0);
    next_chunk();
    load_a(c0, c1); load_b(c1, c1); load_b(c0, c1); load_a(c1, c1);
    next_chunk();
    quad_wait<12>();
    static_for<0, 4>([&](auto k) __attribute__((always_inline)) { read_a(c0, c0, k); read_b(c0, c0, k); });
    quad_wait<10>();
    load_a(c0, c0);
    auto quarter = [&](auto ah, auto bh, auto&& reads, auto&& loads) __attribute__((always_inline)) {
      static_for<0, 4>([&](auto k) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
          mma16B(acc[ah.value * 2 + t][bh.value], __builtin_bit_cast(uint4, a[ah.value][t][k.value]), __builtin_bit_cast(uint4, b[bh.value][k.value]), bf16_t());
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (k.value < 2) {
          reads(std::integral_constant<int, 2 * k.value>{});
          reads(std::integral_constant<int, 2 * k.value + 1>{});
        }
        if constexpr (k.value == 2) loads();
        __builtin_amdgcn_sched_barrier(0);
      });
      quad_wait<12>();
    };
    auto chunk_mma = [&](auto buf) __attribute__((always_inline)) {
      constexpr int B = buf.value;
      const std::integral_constant<int, B> first{};
      const std::integral_constant<int, 1 - B> second{};
      quarter(c0, first, [&](auto k) __attribute__((always_inline)) { read_b(second, buf, k); }, [&]() __attribute__((always_inline)) { load_b(first, buf); });
      quarter(c0, second, [&](auto k) __attribute__((always_inline)) { read_a(c1, buf, k); }, [&]() __attribute__((always_inline)) { load_b(second, buf); });
      quarter(c1, second, [&](auto k) __attribute__((always_inline)) { read_a(c0, second, k); }, [&]() __attribute__((always_inline)) { load_a(c1, buf); });
      quarter(c1, first, [&](auto k) __attribute__((always_inline)) { read_b(second, second, k); },
              [&]() __attribute__((always_inline)) { next_chunk(); load_a(c0, second); });
    };
    for (int c = 0; c < nchunks; c += 2) {
      chunk_mma(c0);
      if (c + 1 == nchunks) break;
      chunk_mma(c1);
    }
    wait_vm<0>();
    __syncthreads();
  };

  // chunks of all segments as one sequence; in pixel-row-first order the chunks [bad0, bad0 + nbad) of every segment
  // (the pixel row whose tap row is outside the map) are left out
  const int per_seg_all = chunks_of_share;
  int bad0 = 0, nbad = 0;
  if (yfirst && per_seg_all > 0 && (ky_tile == 0 || ky_tile == 3)) {
    const int yb = ky_tile == 0 ? 0 : Hs - 1;
    const int lo = max(yb * rb, r_lo), hi = min((yb + 1) * rb, r_hi);      // rows of that pixel row inside this block's share
    if (hi > lo) { bad0 = (lo - r_lo) / WG_KR; nbad = (hi - lo) / WG_KR; } // both multiples of the chunk height
  }
  const int per_seg = per_seg_all - nbad;
  const int nchunks = per_seg * p.nseg;
  auto chunk_row = [&](int cin) { return r_lo + (cin < bad0 ? cin : cin + nbad) * WG_KR; };
  auto row_loop = [&](auto mma_chunk) __attribute__((always_inline)) {
    clear_acc(acc);
    if (nchunks <= 0) return;
    load_chunk(0, chunk_row(0), 0);
    wait_vm<0>();
    __syncthreads();
    int seg = 0, cin = 0;
    for (int c = 0; c < nchunks; ++c) {
      if (c + 1 < nchunks) {
        if (++cin == per_seg) { cin = 0; ++seg; }
        load_chunk(seg, chunk_row(cin), (c + 1) & 1);
      }
      mma_chunk(c & 1);
      wait_vm<0>();
      __syncthreads();
    }
  };
  if constexpr (SZ == 4) {
    split_loop(chunk_row, per_seg, nchunks);
    add_acc(acc, low);
    if (block_any<NT_ / 64>(not_finite(acc), smem, wave)) row_loop(mma_chunk32);
  } else if constexpr (TL::QUAD) {
    quad_loop(bad0, nbad, nchunks);
  } else {
    row_loop(mma_chunk16);
  }

  // Epilogue: each wave passes its 32 x (TN*32) blocks through a private LDS patch (the K buffers are free after the
  // loop's last barrier) so that every lane stores 16 contiguous bytes of a row of dW.
  float* __restrict__ dW = p.dW + (long long)split * p.split_stride + (long long)l * p.dw_stride;
  constexpr int WCOLS = TN * 32;
  constexpr int PSTRIDE = WCOLS * 4 + 16;
  constexpr int CPRW = WCOLS / 4;                                       // 16-byte chunks per patch row
  static_assert((TL::NT / 64) * 32 * PSTRIDE <= 2 * (STAGE_A + STAGE_B), "patch area");
  unsigned char* patch = smem + wave * (32 * PSTRIDE);
  const int colw = nt * BN + wn * WCOLS;
#pragma unroll
  for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int pr = (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
        *reinterpret_cast<float*>(patch + pr * PSTRIDE + (tn * 32 + (lane & 31)) * 4) = acc[tm][tn][e];
      }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 32 * CPRW / 64; ++i) {
      const int cid = lane + 64 * i;
      const int pr = cid / CPRW, pc = cid - pr * CPRW;
      const int m = mt * BM + wm * TM * 32 + tm * 32 + pr;
      const int col = colw + pc * 4;
      if (m < Mtot && col < Cs) {       // Cs is a multiple of 8: a 16-byte chunk is inside or outside
        typedef float f4 __attribute__((ext_vector_type(4)));
        const float4 t = *reinterpret_cast<const float4*>(patch + pr * PSTRIDE + pc * 16);
        f4 q; q.x = t.x; q.y = t.y; q.z = t.z; q.w = t.w;
        __builtin_nontemporal_store(q, reinterpret_cast<f4*>(dW + (long long)m * Cs + col));   // read next by the update kernel
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// Tiles of the weight gradient.  bf16: the largest tile the output fills, because the loop lives on the CU's path from
// L2 (operand bytes per product fall with the tile's sides).  fp32: six times the matrix-pipe time, so
// tiles are small: 128 x 128 with two blocks per CU leaves little of a last round of blocks idle (640 such tiles of 20 models run
// at 126 TFLOP/s, 256 x 128 ones at 90-106, 256 x 64 at 119, all without the scaling of the operands).
typedef Tile<256, 64, 4, 1> TileWg64;     // 64 channels on the N side, bf16
typedef Tile<256, 256, 2, 4> TileWgBig;
typedef Tile<256, 256, 2, 4, 128, 2, 1, 0, true> TileWgQuad;      // in quarters, see quad_loop
typedef Tile<256, 128, 4, 2> TileWgMid;
typedef Tile<128, 128, 2, 2> TileWgF32;
typedef Tile<128, 64, 2, 2> TileWgF32N;

template <typename T, typename TL>
static void launch_wgrad_one(WgradArgs a, hipStream_t st) {
  a.hs_shift = log2_or_neg(a.Hs);
  const int MT = (a.ntaps * a.Cb + TL::BM - 1) / TL::BM, NT = (a.Cs + TL::BN - 1) / TL::BN;
  const long long blocks = ((long long)a.L * a.ksplit + 7) / 8 * 8 * MT * NT;
  if (blocks == 0) return;
  // 32-bit byte offsets inside one model's slice of either operand
  const long long side = a.ntaps == 1 ? a.Hs : 2 * a.Hs, rps = (long long)a.Hs * a.Hs;
  if ((long long)a.seg_samples * side * side * a.Cb * (long long)sizeof(T) >= (1LL << 31) ||
      (long long)a.seg_samples * rps * a.Cs * (long long)sizeof(T) >= (1LL << 31))
    return launch_fail("weight gradient: one segment of an operand is 2 GiB or larger");
  // ceil(2^32 / d): the high half of its product with r is r / d exactly while r * d < 2^32
  a.rps_inv = a.hs_inv = 0;
  if (a.hs_shift < 0 && a.seg_samples * rps * rps < (1LL << 32)) {
    a.rps_inv = (unsigned)(((1ULL << 32) + rps - 1) / rps);
    a.hs_inv = (unsigned)(((1ULL << 32) + a.Hs - 1) / a.Hs);
  }
  if constexpr (std::is_same_v<TL, TileWgBig>) {
    // What the quarters' loader assumes: both halves of a tile's big channels under the same tap, whole tiles, and 32 rows of a chunk a fixed
    // distance from the other 32.  Other shapes have no registers left for their rows.
    if (a.ntaps == 16 && a.Cb % 128 == 0 && a.Cs % 256 == 0 && a.hs_shift >= 0 && a.Hs <= 32) {
      hipLaunchKernelGGL((wgrad_kernel<T, TileWgQuad>), dim3((unsigned)blocks), dim3(TL::NT), 0, st, a);
      return;
    }
  }
  hipLaunchKernelGGL((wgrad_kernel<T, TL>), dim3((unsigned)blocks), dim3(TL::NT), 0, st, a);
}

// Which tile a layer's weight gradient uses, as f(tile, name)
template <typename T, typename F>
static void with_wgrad_tile(int Cs, F&& f) {
  if constexpr (sizeof(T) == 4) {
    if (Cs <= 64) f(TileWgF32N(), "wgrad<128x64>"); else f(TileWgF32(), "wgrad<128x128>");
  } else {
    if (Cs % 256 == 0) f(TileWgBig(), "wgrad<256x256>");
    else if (Cs <= 64) f(TileWg64(), "wgrad<256x64>");
    else f(TileWgMid(), "wgrad<256x128>");
  }
}

template <typename T>
void launch_wgrad(const WgradArgs& a, hipStream_t st) {
  if (!a.Big || !a.Small || !a.dW || !a.offs || a.Cb % 8 || a.Cs % 8 || (a.ntaps != 1 && a.ntaps != 16) || a.ksplit < 1 ||
      (a.ksplit > 1 && a.split_stride <= 0))
    return launch_fail("weight gradient: null operand, channel counts that are not multiples of 8, or a bad row split");
  with_wgrad_tile<T>(a.Cs, [&](auto tile, const char*) { launch_wgrad_one<T, decltype(tile)>(a, st); });
}
int wgrad_tiles_per_model(int esize, int ntaps, int Cb, int Cs) {
  int tiles = 0;
  const auto count = [&](auto tile, const char*) { tiles = (ntaps * Cb + tile.BM - 1) / tile.BM * ((Cs + tile.BN - 1) / tile.BN); };
  if (esize == 4) with_wgrad_tile<float>(Cs, count); else with_wgrad_tile<bf16_t>(Cs, count);
  return tiles;
}
const char* wgrad_variant_name(int esize, const WgradArgs& a) {
  const char* name = "";
  const auto take = [&](auto, const char* n) { name = n; };
  if (esize == 4) with_wgrad_tile<float>(a.Cs, take); else with_wgrad_tile<bf16_t>(a.Cs, take);
  return name;
}
template void launch_wgrad<float>(const WgradArgs&, hipStream_t);
template void launch_wgrad<bf16_t>(const WgradArgs&, hipStream_t);

}  // namespace gan
