// Host launchers of the bandwidth-bound kernels (routing, staging, BatchNorm + activation, the skinny first /
// last layers, losses, Adam).  T is the storage type of activations: float or bf16_t.
#pragma once

#include "common.h"
#include "image_walk.h"

namespace gan {

constexpr int ROUTE_WAVES = 16;     // runs of the flat batch, one wave each
constexpr int MAX_GEOMS = 60;

// One "geometry" = how rows of a layer split into tiles: rows per sample and rows per tile; or, where parts is not 0 (one row a sample), the most of them a
// tile, by ImageTiles.
struct GeomTable {
  int n;
  int rps[MAX_GEOMS];
  int tile_rows[MAX_GEOMS];
  int parts[MAX_GEOMS];
};

struct RouteBuffers {
  int* cnt;           // [ROUTE_WAVES][L] scratch
  int* counts;        // [L]
  int* offs;          // [L+1]
  int* perm;          // [n]
  int* sample_model;  // [n] model of the j-th routed sample
  int* sample_slot;   // [n] label-map slot of the j-th routed sample
  int* tpre;          // [MAX_GEOMS][L+1]
  int* tmodel;        // [MAX_GEOMS][tmodel_stride]: model of every tile of every geometry (built by the staging; one model: not at all)
  int tmodel_stride;
  int* flags;         // [0]: out-of-range label seen
  int* order;         // [L] models by decreasing sample count (ties by index), for kernels whose work per model
                      //     follows the count (may be NULL)
};

// the partition, G's input rows (noise | one-hot label | zeros, kp values a row) in its order, and the model of every tile (rb.tmodel)
template <typename T>
void launch_route_stage(const int* label_ids, const float* noise, int n, int L, int n_labels, int zdim, int cond_g, int kp, const GeomTable& geoms,
                        const RouteBuffers& rb, T* zin, hipStream_t st);

// Batch statistics and the normalise+activate passes.  Groups = (segment, model); rows of group (s, l) are the
// rps rows of each of samples s*seg_samples + offs[l] .. offs[l+1].
struct NormArgs {
  const void* x;            // pre-normalisation tensor [rows][C]
  void* y;                  // apply: activated output ; bwd apply: dx
  const void* dy;           // bwd: gradient w.r.t. the activated output
  float* mean;              // [nseg_total*L][C] (indexed by absolute segment)
  float* var;
  float* rstd;
  float* sums;              // bwd: [seg*L + l][C][2] = (sum g, sum g*xhat)
  const float* gamma;       // model 0; per-model stride pstride
  const float* beta;
  float* dgamma;            // bwd param grads (may be NULL)
  float* dbeta;
  long long pstride;
  float* run_mean;          // model 0, stride rstride (may be NULL)
  float* run_var;
  long long rstride;
  const int* offs;
  const int* counts;
  const int* sample_model;
  int L, C, rps;
  int seg_first, nseg, seg_samples;
  int n;                    // samples per segment passed by the caller (upper bound of offs[L])
  int act;                  // ACT_RELU / ACT_LRELU
  float slope, eps, momentum;
  // bwd apply, networks whose BatchNorm follows an activation: x is that activation's (and dropout's) result, and the gradient goes
  // on through both, to the convolution's output
  int pre_act, pre_drop;    // pre_drop: x is +0 where dropped (see dropped())
  float pre_slope, pre_scale;
  int fold_running;         // statistics from the GEMM's partials: that kernel also updates the running statistics
  int red_rows;             // backward reduction: rows per block (bn_red_rows)
  int red_tiles;            // and its tiles at the sizing batch, which decide how its second stage adds them
  int param_grads;          // backward reduction: its last stage also writes dgamma / dbeta, the segments' sums added in order
};
// statistics from the per-tile column sums a GEMM left behind (stat_partial of ConvArgs)
// (wsplit: sub-tiles per tile, conv_stat_split of the GEMM's tile; size_tiles: the tiles at the sizing batch, which decide the order of the sums)
void launch_bn_stats_from_partial(const NormArgs& a, const float* partial, const int* tpre, int ub_tiles, int size_tiles, int nphase,
                                  int groups, int tile_rows, int gemm_rps, int wsplit, hipStream_t st);
void launch_bn_running(const NormArgs& a, hipStream_t st);
template <typename T> void launch_bn_apply(const NormArgs& a, hipStream_t st);
int bn_red_rows(long long rows, int L);     // rows per block of the backward reduction over `rows` rows of L models (its tile prefix geometry)
template <typename T>
void launch_bn_bwd_reduce(const NormArgs& a, const int* tpre, const int* tmodel, int ub_tiles, float* partial, hipStream_t st);
// its second stage on partial sums [segment][ub_tiles][C][2] of tiles tpre[l] .. tpre[l + 1]
void launch_bn_bwd_final(const NormArgs& a, const int* tpre, int ub_tiles, const float* partial, hipStream_t st);
template <typename T> void launch_bn_bwd_apply(const NormArgs& a, hipStream_t st);

// sums[slot][class][cs] = sum of dy over the samples of the slot (both segments, in order) and the pixels of the class
struct ClassSumArgs {
  const void* dy;           // [rows][Cs] storage type, rows indexed by absolute sample
  float* part;              // scratch [nseg][n][9][Cs]
  float* sums;              // [labels][9][Cs]
  const int* offs;
  const int* sample_slot;
  int L, n, Hs, Cs, labels, seg_first, nseg, seg_samples;
};
template <typename T> void launch_class_sums(const ClassSumArgs& a, hipStream_t st);

// Transposed convolution onto the image side (G's last layer; data gradient of D's first layer).
struct UpImgArgs {
  const void* feat;         // [samples][Hs][Hs][Cs] storage type, indexed by absolute sample
  const void* w;            // model 0 storage-type weights [16][CBT][Cs]; w_stride elements between models
  long long w_stride;
  void* out;                // [samples][2Hs][2Hs][CB] storage type, indexed by absolute sample
  const void* aux;          // mode 2: the saved tanh output, same indexing as out
  const float* bias;        // mode 1: [CB] of model 0, bias_stride between models
  long long bias_stride;
  const int* offs;
  const int* sample_model;
  int L, n, seg, seg_samples;
  int CB, CBT, Cs, Hs;
  int mode;                 // 0: plain ; 1: + bias, tanh ; 2: times (1 - aux^2)
  float* user;              // mode 1: the caller's NCHW fp32 images, written in place of out through perm (or NULL)
  const int* perm;
};
template <typename T> void launch_up_img(const UpImgArgs& a, hipStream_t st);

// The strided convolutions that read an image (image_conv.hip): D's first layer, and the gradients of G's last, whose output gradient is an image.
// Images: NHWC in the storage type, indexed by absolute sample; segment 0 may be the caller's NCHW fp32 batch instead, gathered through perm.
int image_values(int CB);                    // values a pixel has in a tile: 2, 4 or 8; packed weights have 16 times as many a feature channel
struct ImageConvArgs {
  const void* img;
  const float* real;
  const int* perm;
  const void* w;            // [L][Cs][16 P], launch_pack_image_w
  const float* add;         // [tables][9][Cs]: added to the outputs by position class, or NULL
  const float* bias;        // [Cs] of model 0, bias_stride between models, or NULL
  long long bias_stride;
  const int* sample_slot;   // the table of a sample, or NULL: its model's
  void* out;                // [rows][Cs], rows indexed by absolute sample
  const int* offs;
  const int* sample_model;
  int L, n, CB, Hs, Cs, seg_first, nseg, seg_samples;
  float slope;              // factor below zero
};
template <typename T> void launch_image_conv(const ImageConvArgs& a, hipStream_t st);
struct ImageWgradArgs {
  const void* img;
  const float* real;
  const int* perm;
  const void* dy;           // [rows][Cs], rows indexed by absolute sample
  float* part;              // [tiles][16 P][Cs], partial sums of every tile, and scratch behind the launch's tiles: image_part_floats
  float* pixel_sums;        // [tiles][4]: the sums of the image's pixels, or NULL
  const int* offs;
  const int* tpre;          // the prefix array and models of the tiles (tmodel NULL: one model)
  const int* tmodel;
  int L, CB, Hs, Cs, seg_first, nseg, seg_samples;
  ImageTiles tiles;
};
// floats of `part` for up to `tiles` tiles of up to nseg segments
long long image_part_floats(int esize, int CB, int Hs, int Cs, int nseg, const ImageTiles& t, long long tiles);
template <typename T> void launch_image_wgrad(const ImageWgradArgs& a, int ub_tiles, hipStream_t st);
// The row splits of the linear head's weight gradient (HeadArgs, rsplit > 1), which another kernel of D's backward pass adds up along the way
struct HeadSplits {
  const float* part;        // NULL: none
  float *dw, *db;
  int K, rsplit;
};
struct ImageGradArgs {      // the tiles' sums into the gradient blocks
  HeadSplits head;          // (same pstride)
  const float* part;
  const float* pixel_sums;
  const int* tpre;
  float* dw;                // model 0 [16][CBT][Cs]; pstride between models
  float* dbias;             // [Cs], or NULL
  float* image_bias;        // [CB], from the pixel sums, or NULL
  const float* label_sums;  // labels > 0 (one model): [labels][9][Cs], the class sums of the layer's output gradient
  long long pstride;
  int L, CB, CBT, Cs, P, labels;
  int plane_labels;         // the model's one label map has the gradient of the ones
  int k3;                   // the taps of the fourth row and column are no parameters: not written
};
void launch_image_wgrad_final(const ImageGradArgs& a, hipStream_t st);
struct ImagePackArgs {
  const float* w;           // model 0 master weights [16][CBT][Cs]; pstride between models
  void* packed;             // [L][Cs][16 P] storage type
  float* add;               // [tables][9][Cs] (label maps), or NULL
  long long pstride;
  int L, CB, CBT, Cs, P, tables;
};
template <typename T> void launch_pack_image_w(const ImagePackArgs& a, hipStream_t st);

int img_bias_chunks(int L);          // pixel chunks per model of the image-side bias gradient
struct ImgBiasArgs {
  const void* img;          // [pixels][CB] of segment 0
  float* partial;           // [L][img_bias_chunks(L)][4]
  float* dbias;             // model 0, stride pstride
  long long pstride;
  const int* offs;
  int L, CB, HW;
};
template <typename T> void launch_img_bias_grad(const ImgBiasArgs& a, hipStream_t st);

// D's final linear layer (one logit), the two costs, and their gradients.
enum Cost { COST_D = 0, COST_G = 1 };      // the discriminator's, on (real, fake); the generator's, on fake
struct HeadArgs {
  const void* feat;         // [rows][K] last feature map, flattened (h,w,c)
  void* dfeat;              // gradient w.r.t. it
  const float* w;           // model 0 [K] then bias; per-model stride pstride
  const float* b;
  float* dw;
  float* db;
  long long pstride;
  float* logits;            // [nseg_total * seg_samples]
  float* dlogits;
  float* loss;              // [L]
  const int* offs;
  const int* sample_model;
  int L, K, seg_first, nseg, seg_samples, n;
  int* adam_t;              // with the costs: [L] step counts of the update that follows, advanced with the bias corrections adam_bc [L][2]
  float* adam_bc;
  float beta1, beta2;
  Cost cost;
  float scale;
  // weight gradient: rsplit > 1 shares every model's rows among rsplit blocks per K chunk; their partial sums go to
  // part[rsplit][L][K + 4] (the bias term at index K) and are added in order later (HeadSplits)
  float* part;
  int rsplit;
};
// BatchNorm and activation of the last feature map (as launch_bn_apply), the logits and the cost's derivatives by them
template <typename T> void launch_bn_apply_head(const NormArgs& a, const HeadArgs& h, hipStream_t st);
// the costs and the data gradient; weights: the weight gradient too
template <typename T> void launch_head_bwd(const HeadArgs& a, bool weights, hipStream_t st);

constexpr int ADAM_MAX_REGIONS = 8;
struct AdamArgs {
  float* theta; float* m; float* v;
  float* g;                 // read; written where the update adds up row splits
  void* shadow;             // storage-type copy of theta (NULL when the storage type is fp32)
  void* shadow_t;           // storage-type copy with every region below transposed: [tap][cs][cb]
  // fp32 storage, in place of the two copies: the regions, from element reg_part of a plane on, as three bf16 planes, as they are and
  // transposed (launch_split_weights; models 3 * plane elements apart).  Or both NULL, and shadow_t has the regions only, from reg_part on, models
  // plane elements apart.
  unsigned short *split_u, *split_d;
  long long plane;
  long long P;              // elements per model
  int L;
  const int* counts;
  int* t;                   // [L] step counts
  float* bc;                // [L][2] scratch: 1-beta1^t, 1-beta2^t
  float lr, beta1, beta2, eps;
  // Convolution weights [16][Cb][Cs] (Cb, Cs multiples of 64) that need the transposed copy: updated tile by tile.
  // Everything else is the list of gaps between them, updated as flat ranges.
  int nregions;
  long long reg_w[ADAM_MAX_REGIONS], reg_part[ADAM_MAX_REGIONS];
  int reg_cb[ADAM_MAX_REGIONS], reg_cs[ADAM_MAX_REGIONS];
  int reg_cb_real[ADAM_MAX_REGIONS], reg_cs_real[ADAM_MAX_REGIONS];      // channels from here on are padding: zeros that no update moves
  int k3;                                 // the taps of the fourth row and column are no parameters (zeros likewise, whatever their gradients hold)
  int reg_tile0[ADAM_MAX_REGIONS + 1];    // prefix of 64 x 64 tiles (filled by the launcher)
  int ngaps;
  long long gap_lo[ADAM_MAX_REGIONS + 1], gap_hi[ADAM_MAX_REGIONS + 1];
  int gap_blk0[ADAM_MAX_REGIONS + 2];     // prefix of 1024-element blocks (filled by the launcher)
  int tile_first, tile_count;             // the 64 x 64 tiles (per model) of a launch over some of the regions
};
// T: storage type of the shadows.  launch_adam does the whole update; the parts below do it piecewise (plan first).
template <typename T> void launch_adam(AdamArgs a, hipStream_t st);
bool adam_plan(AdamArgs& a);
// The gradient of one region as the row splits of its product, [n][L][16][Cb][Cs], which the update adds up into g on the way (n < 2: g holds it),
// as launch_sum_splits does: chains is split_chains of them.
struct AdamSplits {
  const float* part = nullptr;
  int n = 0, chains = 1;
};
template <typename T> void launch_adam_region(AdamArgs a, int region, const AdamSplits& sp, hipStream_t st);
// The image-side layer among the gaps, whose operand (ImagePackArgs) is written along with its weights.
struct AdamImage {
  long long w = 0;          // its weights [16][CBT][Cs] in a model's block
  void* packed = nullptr;   // NULL: no such layer
  float* add = nullptr;     // [tables][9][Cs], or NULL
  int CB = 0, CBT = 0, Cs = 0, P = 0, tables = 0;
};
bool adam_region_joins_rest(const AdamArgs& a, int region);      // few enough tiles for the launch below
template <typename T> void launch_adam_rest(AdamArgs a, const AdamImage& im, int region, const AdamSplits& sp, hipStream_t st);
template <typename T> void launch_cast_shadow(const float* theta, T* shadow, long long total, hipStream_t st);
// dst[tap][cs][cb] <- src[tap][cb][cs] for every model (src: T or float master)
template <typename T, typename S>
void launch_transpose_w(const S* src, T* dst, long long src_stride, long long dst_stride, int L, int Cb, int Cs, hipStream_t st);

// fp32 weights as three bf16 planes (split_mfma.h): the block src[tap][cb][cs] of every model into up[plane][tap][cb][cs] and, transposed,
// down[plane][tap][cs][cb]; planes `plane`, models src_stride (src) and 3 * plane elements apart.  down may be NULL.
struct SplitArgs {
  const float* src;
  unsigned short *up, *down;
  long long src_stride, plane;
  int L, Cb, Cs;
};
void launch_split_weights(const SplitArgs& a, hipStream_t st);

// How many sums the row splits of `elements` values (of all models) are added in: with four, split k goes to sum k % 4, in order, and the sums are
// added in order.  Of many splits one sum's error is up to twice as large; many elements have few splits.
inline int split_chains(long long elements, int nsplit) { return elements / 4 < 256 * 256 && nsplit >= 16 ? 4 : 1; }
// dW[l * dw_stride + i] = part[(0 * L + l) * size + i] + part[(1 * L + l) * size + i] + ... (nsplit terms, in split_chains sums),
// i < size (a multiple of 4), l < L
void launch_sum_splits(const float* part, float* dW, long long dw_stride, long long size, int L, int nsplit, hipStream_t st);

void launch_tile_prefix(const int* offs, int L, int rps, int tile_rows, int* tpre, hipStream_t st);
// Class draws: labels[i] = first k with cdf[k] > (double)u[i]; if none (rounding), `last` .
// cdf: device memory, or NULL: in the table (at most DRAW_ARGS labels)
constexpr int DRAW_ARGS = 256;
struct DrawTable { double cdf[DRAW_ARGS]; };
void launch_draw_labels(const float* u, const double* cdf_mem, const DrawTable& table, int n_labels, int last, int n, int* labels, hipStream_t st);

// One-way analysis of variance of the per-image channel means by label; all arithmetic in double, fixed order.
//   x[i][c]    = mean over the pixels of channel c of image i (images: NCHW fp32)
//   gsum[k][c] = sum of x over the images of label k, gcnt[k] = their number
//   ssw[k][c]  = sum over the images of label k of (x - gsum/gcnt)^2
// (gsum, ssw and gcnt may be pinned host memory: the kernels only write them)
void launch_anova(const int* label_ids, const float* images, int n, int n_labels, int C, int HW, double* x, double* gsum,
                  double* ssw, int* gcnt, hipStream_t st);

// ---- pieces of the networks as printed in the paper's Tables 1 and 2 (paper_layers.hip) ----
// In-place dropout of an NHWC tensor whose samples are grouped by model (offs[g] .. offs[g+1]): the keep-mask comes
// from Philox-4x32-10 with counter (element index low, high, layer + 256 * pass, step), key (seed low, seed high ^ g),
// element index ((n C + c) H + y) W + x, n counted inside the group; kept values are scaled by 1 / (1 - p).
template <typename T>
void launch_dropout(T* x, const int* offs, int n_groups, int n, int C, int H, int W, float p, unsigned long long seed, int step,
                    int layer, int pass_id, hipStream_t st);
// w4[g][ty*4+tx][cb][cs] = sum of w3[g][ky*3+kx][cb][cs] over ky in S(ty), kx in S(tx), S = {2}, {1,2}, {0,1}, {0}
// (Upsample x2 + Conv k3 s1 p1 == ConvTranspose k4 s2 p1 with these taps); w4t is the same with cb and cs exchanged.
// group g reads w3 + g * w3_stride and writes w4 + g * w4_stride, w4t + g * w4_stride (strides in elements; 0: packed)
template <typename T>
void launch_w3_to_w4(const float* w3, T* w4, T* w4t, int n_groups, int cb, int cs, hipStream_t st, long long w3_stride = 0,
                     long long w4_stride = 0);
void launch_dw4_to_dw3(const float* dw4, float* dw3, int n_groups, int cb, int cs, hipStream_t st, long long dw4_stride = 0,
                       long long dw3_stride = 0);   // the adjoint map

// ---- the training step of the networks as printed in Tables 1 and 2 (paper_step.hip) ----
// One pass over a stored NHWC tensor whose samples are grouped by model: rows of sample j (model-major) are HW pixels
// of Cpad channels, of which the first C are real (the rest is channel padding and is left alone).
struct PointArgs {
  void* x;                  // forward: the layer output, in place ; sums: the tensor
  const float* bias;        // forward: [C] of model 0, pstride between models (may be NULL)
  long long pstride;
  const int* offs;
  const int* sample_model;
  const int* steps;         // dropout: per-model count of iterations taken (NULL when thr == 0)
  int step_add;             // the iteration number is steps[l] + step_add
  int L, n, C, Cpad, HW;
  int seg_first, nseg, seg_samples;
  int pass_of_seg[2];       // dropout: pass id of each processed segment
  int layer;
  unsigned thr;             // ceil(p 2^24); 0: no dropout
  float scale;              // 1 / (1 - p)
  float slope;              // activation: x > 0 ? x : slope x   (1: none)
  unsigned seed_lo, seed_hi;
};
template <typename T> void launch_point_fwd(const PointArgs& a, hipStream_t st);     // x <- dropout(act(x + bias))
// out[l * out_stride + c] = sum over the segments and rows of model l of x[.., c]
template <typename T> void launch_col_sum(const PointArgs& a, float* out, long long out_stride, hipStream_t st);
// batch statistics (mean, biased variance, 1/sqrt(var + eps)) of a stored tensor with C channels per row, of which those from `real` on are padding
template <typename T> void launch_bn_stats_direct(const NormArgs& a, int real, hipStream_t st);

// Conv k3 s1 p1 between Cin feature channels (64 or 128) and CO image channels (1..4), side H, NHWC, rows model-major.
struct Conv3Args {
  const void* in;           // features [samples][H][H][Cin] (segment 0)
  void* out;                // forward: tanh(conv + bias) into segment out_seg of the image buffer
  const void* dout;         // backward: gradient w.r.t. the pre-tanh output, segment out_seg of the image-gradient buffer
  void* din;                // backward: gradient w.r.t. `in`
  const float* w;           // [9][CO][Cin] of model 0, w_stride between models
  long long w_stride;
  const float* bias;        // [CO] of model 0
  long long bias_stride;
  const int* offs;
  const int* sample_model;
  int L, n, H, Cin, CO;
  int out_seg, seg_samples;
  float* user;              // forward: the caller's NCHW fp32 images, written in place of out through perm (or NULL)
  const int* perm;
  // with bn_mean (the backward kernels always): `in` is the tensor in front of the BatchNorm (batch statistics [L][Cin]; gamma, beta of model 0, bn_pstride between models) and
  // the activation (slope below zero) whose result the features are
  const float *bn_mean, *bn_rstd, *bn_gamma, *bn_beta;
  long long bn_pstride;
  float bn_slope;
  float* bn_part;           // data gradient without bn_sums: [n][Cin][2], the sums of every sample that BatchNorm's backward pass wants
  const float* bn_sums;     // [L][Cin][2], their sums by model: with them the data gradient itself
};
template <typename T> void launch_conv3_fwd(const Conv3Args& a, hipStream_t st);
template <typename T> void launch_conv3_dgrad(const Conv3Args& a, hipStream_t st);
// part: [conv3_wgrad_splits(L)][L][9*CO*Cin] scratch ; dw: [9][CO][Cin] of model 0, dw_stride between models
int conv3_wgrad_splits(int L);
template <typename T> void launch_conv3_wgrad(const Conv3Args& a, float* part, float* dw, long long dw_stride, hipStream_t st);

}  // namespace gan
