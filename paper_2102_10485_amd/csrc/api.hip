// Host side of the library: context, arenas, parameter layout, and the launch sequence of one training step
// (Section 2 of the paper: cost of Eq. 3 and Adam on theta_D, then cost of Eq. 4 through the updated D and Adam on
// theta_G, for all label models of Eq. 5 at once).
#include "../../include/gan.h"

#include <math.h>
#include <stdio.h>
#include <string.h>
#include <algorithm>

#include <set>
#include <string>
#include <vector>

#include "anova_host.h"
#include "kernels.h"

using namespace gan;

namespace gan {
static thread_local const char* g_launch_error = nullptr;
void launch_fail(const char* msg) { if (!g_launch_error) g_launch_error = msg; }
const char* take_launch_error() { const char* e = g_launch_error; g_launch_error = nullptr; return e; }
}  // namespace gan

namespace {

inline long long round_up(long long x, long long m) { return (x + m - 1) / m * m; }

constexpr int WG_MAX_KSPLIT = 64;

// A (transposed) convolution between a "big" tensor (Cb channels, side 2*Hs) and a "small" one (Cs, side Hs).
// Internal weight layout [tap][Cb (or CBT)][Cs].
struct ConvLayer {
  int Cb = 0, CBT = 0, Cs = 0, Hs = 0;
  long long w = -1, bias = -1, gamma = -1, beta = -1;   // offsets into the per-model parameter block
  long long rs = -1;                                    // offset into the running-statistics block
  int bnC = 0;                                          // channels normalised after this layer (0: none)
  int nbias = 0;
  // networks as printed in the paper's tables: real (unpadded) channel counts, and for G's blocks the place of the
  // summed-tap k4 weights in the storage-type arenas
  int cs_real = 0, cb_real = 0;
  long long w4 = -1;
  long long part = -1;                                  // fp32 storage, layers on the GEMM engine: offset into a plane of the split weights, or into shadow_d
};

struct Net {
  std::vector<ConvLayer> conv;     // G: transposed convs 1..n_g ; D: convs 1..n_d
  // linear layer: G's input stage (J outputs, Kp padded inputs, followed by BN over C0) / D's head (K inputs)
  long long fc_w = -1, fc_b = -1, fc_gamma = -1, fc_beta = -1, fc_rs = -1;
  int J = 0, Kz = 0, Kp = 0, C0 = 0, h0 = 0, K = 0;
  long long P = 0;                 // internal parameters per model (multiple of 64: keeps 16-byte alignment)
  long long Pext = 0;              // parameters per model in the documented order
  long long nbn = 0;
  std::vector<long long> ext2int;  // documented index -> internal index
  std::vector<long long> bn_ext2int;   // documented running-statistics index -> internal (empty: identical)
  std::vector<int> ext_kind;       // per documented element: 0 weight, 1 gamma, 2 zero-initialised (built-in initialiser)
  // networks as printed in the paper's tables (G): k4 weights with summed taps, [tap][cb][cs] and (bf16 storage) [tap][cs][cb]
  long long fc_bias = -1, P4 = 0;
  void *w4u = nullptr, *w4d = nullptr;
  float *theta = nullptr, *m = nullptr, *v = nullptr, *g = nullptr;
  void *shadow_u = nullptr, *shadow_d = nullptr;   // bf16 storage: copies [tap][cb][cs] and [tap][cs][cb] (fp32: shadow_u is theta)
  // fp32 storage: the weights of the convolutions on the GEMM engine (the k4 weights, where there are any) as three bf16 planes in both
  // layouts, [model][plane][PS] (without presplit: shadow_d, the second layout in fp32, [model][PS])
  long long PS = 0;
  unsigned short *split_u = nullptr, *split_d = nullptr;
  float *run_mean = nullptr, *run_var = nullptr;
  int* t = nullptr;
  float* bc = nullptr;
};

struct ProfEntry { const char* name; hipEvent_t e0, e1; double flops, bytes; };

}  // namespace

struct gan_ctx {
  gan_config cfg;
  hipStream_t st = nullptr;
  bool bf16 = false;
  int L = 0, NB = 0;
  Net G, D;
  GeomTable geoms;
  RouteBuffers rb;                 // the set the launch helpers use (the training step's, except inside gan_generate)
  RouteBuffers rb_gen;             // gan_generate / gan_sample route into this one
  // workspace (storage type unless noted)
  void *zin = nullptr, *xd = nullptr, *dimg = nullptr, *bufA = nullptr, *bufB = nullptr;
  std::vector<void*> gpre, gact, dpre, dact;
  std::vector<float*> g_mean, g_var, g_rstd, g_sums, d_mean, d_var, d_rstd, d_sums;
  float *logits = nullptr, *dlogits = nullptr, *loss_d = nullptr, *loss_g = nullptr;
  // image-side layers: packed weights (and what the label maps and the bias add, by position class), partial weight gradients
  void *wpD = nullptr, *wpG = nullptr;
  float *addD = nullptr, *img_part = nullptr, *img_sums = nullptr, *bias_partial = nullptr, *stat_partial = nullptr;
  ImageTiles img_tiles = {1, 1};   // of their weight gradients
  float* head_part = nullptr;      // row-split partial sums of the linear head's weight gradient (few models only)
  int head_rsplit = 1;
  float* wg_part = nullptr;        // row-split partial weight gradients (few models only)
  bool paper = false;              // the networks as printed in the paper's tables
  bool presplit = false;           // fp32 storage: the convolutions on the GEMM engine read weights that the update has split (see presplit_pays)
  float *dw4 = nullptr, *c3_part = nullptr;   // paper G: k4 weight gradient of one block; row-split partials of the last conv
  int labels = 0;             // > 0: one pair over that many labels, whose maps' gradients come from class sums
  float *label_sums = nullptr, *class_part = nullptr;
  int last_n = -1;
  bool shadows_dirty = true;
  std::string err;
  std::vector<void*> allocs;
  // mixture sampling and ANOVA: buffers allocated at first use
  double* cdf = nullptr;            // [n_labels]
  double* an_x = nullptr;           // [NB*img_c]
  double* an_res = nullptr;         // pinned host memory the kernels write their results to: gsum, ssw [n_labels*img_c], gcnt int [n_labels]
  // profiling
  bool prof = false, prof_detail = false, prof_gemm_only = false;
  std::set<std::string> prof_names;
  std::vector<ProfEntry> prof_entries;
  std::vector<hipEvent_t> event_pool;
  // A second stream (default priority) for the weight gradients and the Adam updates of the convolution weights, which
  // nothing later in the backward chain waits for: they can run beside it and fill the chip where the chain's kernels
  // leave it idle (tile-count tails, bandwidth-bound passes).  Ordering between the two streams is by events.  Off
  // unless the caller asks (gan_use_second_stream): it shortens the largest workload's step by 1.7 %, and every
  // kernel that shares the chip with another one runs longer, which blurs per-kernel timings.
  hipStream_t side = nullptr;
  bool side_on = false;
  std::vector<hipEvent_t> order_events;
  size_t order_next = 0;
  // Replayable steps.  A training step's launches depend on the call's arguments only through the three device
  // pointers and n (everything else the kernels read lives in device tables the step itself rebuilds), so a call that
  // repeats the arguments of a recent call can be captured once into a HIP graph (on `cap`, an internal stream: the
  // caller's may be the legacy default stream, which cannot be captured) and replayed on the caller's stream from
  // then on: one host call instead of a hundred and more.  Off unless the caller asks (gan_use_graphs): on this
  // part the steps are bound by the chain of dependent kernels on the device, not by the host's launch calls, and a
  // replay measured 0-4 % slower than the plain launches in every configuration.
  struct StepGraph { const void *lab, *noise, *real; int n; hipGraphExec_t exec; unsigned long long used; };
  hipStream_t cap = nullptr;
  std::vector<StepGraph> graphs;
  bool graphs_on = false;
  struct StepArgs { const void *lab, *noise, *real; int n; };
  std::vector<StepArgs> seen;      // the last eight distinct argument sets that ran as plain launches
  unsigned long long calls = 0, replays = 0;
  int op_tile_rows = 0;            // single-operation entry points: tile height forced by the caller (0: chosen as in a step)
  int op_segments = 1, op_splits = 1;      // of gan_op_conv_wgrad
};

namespace {

size_t esize(const gan_ctx* c) { return c->bf16 ? 2 : 4; }

gan_status fail(gan_ctx* c, gan_status s, const std::string& msg) {
  if (c) c->err = msg;
  return s;
}

// After a call has enqueued its launches: a refused launch (shape the kernels do not support) or a HIP launch error.
gan_status launch_status(gan_ctx* c) {
  const char* refused = take_launch_error();
  const hipError_t e = hipGetLastError();
  if (refused) return fail(c, GAN_E_SHAPE, refused);
  if (e != hipSuccess) return fail(c, GAN_E_HIP, std::string("launch failed: ") + hipGetErrorString(e));
  return GAN_OK;
}

bool dev_alloc(gan_ctx* c, void** p, size_t bytes) {
  if (bytes == 0) bytes = 16;
  if (hipMalloc(p, bytes) != hipSuccess) { (void)hipGetLastError(); return false; }
  c->allocs.push_back(*p);
  return true;
}

int find_geom(const gan_ctx* c, int rps, int tile_rows, int parts) {
  for (int i = 0; i < c->geoms.n; ++i)
    if (c->geoms.rps[i] == rps && c->geoms.tile_rows[i] == tile_rows && c->geoms.parts[i] == parts) return i;
  return -1;
}
int geom_id(gan_ctx* c, int rps, int tile_rows, int parts = 0) {
  const int g = find_geom(c, rps, tile_rows, parts);
  if (g >= 0) return g;
  if (c->geoms.n >= MAX_GEOMS) return -1;
  c->geoms.rps[c->geoms.n] = rps;
  c->geoms.tile_rows[c->geoms.n] = tile_rows;
  c->geoms.parts[c->geoms.n] = parts;
  return c->geoms.n++;
}
const int* tmodel_of(gan_ctx* c, int rps, int tile_rows, int parts = 0) {
  const int g = find_geom(c, rps, tile_rows, parts);
  return c->L == 1 || g < 0 ? nullptr : c->rb.tmodel + (long long)g * c->rb.tmodel_stride;
}
const int* tpre_of(gan_ctx* c, int rps, int tile_rows, int parts = 0) {
  const int g = find_geom(c, rps, tile_rows, parts);
  if (g < 0) {   // every geometry a launch uses is registered at create; anything else would read an unbuilt prefix
    launch_fail("a launch asked for a tile geometry that was not registered when the context was created");
    return nullptr;   // the launchers refuse a null prefix array
  }
  return c->rb.tpre + (long long)g * (c->L + 1);
}
// the tile of a layer's launch: from the average rows per model at the sizing batch (fixed at create, so the prefix
// arrays built at every routing match)
ConvTile layer_tile(const gan_ctx* c, int mode, int n_out, int rps, int nseg) {
  return conv_choose_tile((int)esize(c), n_out, (double)c->NB * rps / c->L, c->L, nseg * (mode == MODE_UP ? 4 : 1));
}
int ub_tiles(const gan_ctx* c, int n, int rps, int tile_rows) {
  return (int)(((long long)n * rps) / tile_rows) + (n < c->L ? n : c->L);
}

// row blocks of a BatchNorm's backward reduction, from the sizing batch like the tiles
int red_rows(const gan_ctx* c, int rps) { return bn_red_rows((long long)c->NB * rps, c->L); }

// ---- profiling: two events around a launch ------------------------------------------------------------
struct Scope {
  gan_ctx* c; int idx = -1; hipStream_t st;
  // st: the stream the launch goes to (default: the caller's)
  Scope(gan_ctx* c_, const char* name, double flops, double bytes, const char* detail = nullptr, hipStream_t st_ = nullptr)
      : c(c_), st(st_ ? st_ : c_->st) {
    if (!c->prof) return;
    if (c->prof_gemm_only && strncmp(name, "gemm_", 5) != 0 && strncmp(name, "wgrad", 5) != 0) return;
    if (c->prof_detail && detail) name = c->prof_names.insert(std::string(name) + detail).first->c_str();
    ProfEntry e; e.name = name; e.flops = flops; e.bytes = bytes;
    for (hipEvent_t* ev : {&e.e0, &e.e1}) {          // events are reused across profiling sessions
      if (c->event_pool.empty()) hipEventCreateWithFlags(ev, hipEventDisableSystemFence);   // device-side timing only: no system-scope fence
      else { *ev = c->event_pool.back(); c->event_pool.pop_back(); }
    }
    hipEventRecord(e.e0, st);
    c->prof_entries.push_back(e);
    idx = (int)c->prof_entries.size() - 1;
  }
  ~Scope() { if (idx >= 0) hipEventRecord(c->prof_entries[idx].e1, st); }
};

// The stream for work that may run beside the caller's stream (per-launch timing records its events on whichever
// stream a launch goes to, so the timed steps run exactly like the untimed ones).
hipStream_t side_stream(gan_ctx* c) { return (c->side && c->side_on) ? c->side : c->st; }
// whatever is enqueued on `later` from now on starts after everything enqueued on `earlier` so far
void order_after(gan_ctx* c, hipStream_t later, hipStream_t earlier) {
  if (later == earlier) return;
  if (c->order_next == c->order_events.size()) {
    hipEvent_t e;
    if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) return launch_fail("could not create an ordering event");
    c->order_events.push_back(e);
  }
  hipEvent_t e = c->order_events[c->order_next++];
  hipEventRecord(e, earlier);
  hipStreamWaitEvent(later, e, 0);
}

template <typename T> void adam_region_call(gan_ctx* c, const AdamArgs& a, int region, hipStream_t st, const AdamSplits& sp = {});
template <typename T> void pack_image_call(gan_ctx* c, const Net& net);
// a region whose update a backward pass leaves to the last launch of the update, with the row splits of its gradient
struct AdamTail {
  int region = -1;
  AdamSplits splits;
};

double valid_tap_fraction(int Hs) {   // k4 s2 p1: per axis 2 of the 4*Hs (row, tap) pairs fall outside
  const double f = (4.0 * Hs - 2.0) / (4.0 * Hs);
  return f * f;
}

// ---- parameter layout ----------------------------------------------------------------------------------
void build_layout(gan_ctx* c) {
  const gan_config& f = c->cfg;
  {
    Net& G = c->G;
    long long o = 0, ext = 0, r = 0;
    G.Kz = f.z_dim + f.cond_g;
    G.Kp = (int)round_up(G.Kz, 64);
    G.C0 = f.g_ch[0]; G.h0 = f.g_h0; G.J = G.C0 * G.h0 * G.h0;
    G.fc_w = o; o += (long long)G.J * G.Kp;
    G.fc_gamma = o; o += G.C0; G.fc_beta = o; o += G.C0; G.fc_rs = r; r += G.C0;
    o = round_up(o, 8);
    // documented order: fc.w [(c,h,w)][Kz]
    G.ext2int.reserve(1 << 20);
    for (int ch = 0; ch < G.C0; ++ch)
      for (int y = 0; y < G.h0; ++y)
        for (int x = 0; x < G.h0; ++x)
          for (int i = 0; i < G.Kz; ++i)
            G.ext2int.push_back(G.fc_w + ((long long)((y * G.h0 + x) * G.C0 + ch)) * G.Kp + i);
    for (int ch = 0; ch < G.C0; ++ch) G.ext2int.push_back(G.fc_gamma + ch);
    for (int ch = 0; ch < G.C0; ++ch) G.ext2int.push_back(G.fc_beta + ch);
    int h = f.g_h0;
    for (int i = 1; i <= f.n_g; ++i) {
      ConvLayer l;
      l.Cs = f.g_ch[i - 1]; l.Cb = (i < f.n_g) ? f.g_ch[i] : f.img_c; l.CBT = l.Cb; l.Hs = h;
      l.w = o; o += (long long)16 * l.CBT * l.Cs;
      for (int cs = 0; cs < l.Cs; ++cs)
        for (int cb = 0; cb < l.Cb; ++cb)
          for (int tap = 0; tap < 16; ++tap) G.ext2int.push_back(l.w + ((long long)tap * l.CBT + cb) * l.Cs + cs);
      if (i < f.n_g) {
        l.gamma = o; o += l.Cb; l.beta = o; o += l.Cb; l.rs = r; r += l.Cb; l.bnC = l.Cb;
        for (int ch = 0; ch < l.Cb; ++ch) G.ext2int.push_back(l.gamma + ch);
        for (int ch = 0; ch < l.Cb; ++ch) G.ext2int.push_back(l.beta + ch);
      } else {
        l.bias = o; l.nbias = l.Cb; o += l.Cb;
        for (int ch = 0; ch < l.Cb; ++ch) G.ext2int.push_back(l.bias + ch);
      }
      o = round_up(o, 8);
      G.conv.push_back(l);
      h *= 2;
    }
    G.P = round_up(o, 64); G.Pext = (long long)G.ext2int.size(); G.nbn = r; (void)ext;
  }
  {
    Net& D = c->D;
    long long o = 0, r = 0;
    int h = f.img_hw;
    for (int j = 0; j < f.n_d; ++j) {
      ConvLayer l;
      l.Cb = (j == 0) ? f.img_c : f.d_ch[j - 1];
      l.CBT = (j == 0) ? f.img_c + f.cond_d : l.Cb;
      l.Cs = f.d_ch[j]; l.Hs = h / 2;
      l.w = o; o += (long long)16 * l.CBT * l.Cs;
      for (int cs = 0; cs < l.Cs; ++cs)
        for (int cb = 0; cb < l.CBT; ++cb)
          for (int tap = 0; tap < 16; ++tap) D.ext2int.push_back(l.w + ((long long)tap * l.CBT + cb) * l.Cs + cs);
      if (j == 0) {
        l.bias = o; l.nbias = l.Cs; o += l.Cs;
        for (int ch = 0; ch < l.Cs; ++ch) D.ext2int.push_back(l.bias + ch);
      } else {
        l.gamma = o; o += l.Cs; l.beta = o; o += l.Cs; l.rs = r; r += l.Cs; l.bnC = l.Cs;
        for (int ch = 0; ch < l.Cs; ++ch) D.ext2int.push_back(l.gamma + ch);
        for (int ch = 0; ch < l.Cs; ++ch) D.ext2int.push_back(l.beta + ch);
      }
      o = round_up(o, 8);
      D.conv.push_back(l);
      h /= 2;
    }
    const int Cl = f.d_ch[f.n_d - 1];
    D.K = Cl * h * h; D.h0 = h; D.C0 = Cl;
    D.fc_w = o; o += D.K;
    for (int ch = 0; ch < Cl; ++ch)
      for (int y = 0; y < h; ++y)
        for (int x = 0; x < h; ++x) D.ext2int.push_back(D.fc_w + (long long)(y * h + x) * Cl + ch);
    D.fc_b = o; o += 1;
    D.ext2int.push_back(D.fc_b);
    D.P = round_up(o, 64); D.Pext = (long long)D.ext2int.size(); D.nbn = r;
  }
}

// The networks as printed in the paper's Tables 1 and 2.  D's k3 s2 p1 convolutions sit in the engine's k4 layout
// (fourth tap row / column and channel padding are not parameters and stay zero); G's Upsample + k3 blocks keep their
// 3 x 3 weights as parameters and run on k4 weights with summed taps rebuilt after every update.
void build_layout_paper(gan_ctx* c) {
  const gan_config& f = c->cfg;
  auto pad64 = [](int v) { return (int)round_up(v, 64); };
  {
    Net& G = c->G;
    long long o = 0, r = 0, o4 = 0;
    G.Kz = f.z_dim; G.Kp = (int)round_up(G.Kz, 64);
    G.C0 = f.g_ch[0]; G.h0 = f.g_h0; G.J = G.C0 * G.h0 * G.h0;
    G.fc_w = o; o += (long long)G.J * G.Kp;
    G.fc_bias = o; o += G.J;
    G.fc_gamma = o; o += G.C0; G.fc_beta = o; o += G.C0; G.fc_rs = r; r += G.C0;
    o = round_up(o, 8);
    auto ext = [&](long long internal, int kind) { G.ext2int.push_back(internal); G.ext_kind.push_back(kind); };
    for (int ch = 0; ch < G.C0; ++ch)
      for (int y = 0; y < G.h0; ++y)
        for (int x = 0; x < G.h0; ++x)
          for (int i = 0; i < G.Kz; ++i) ext(G.fc_w + ((long long)((y * G.h0 + x) * G.C0 + ch)) * G.Kp + i, 0);
    for (int ch = 0; ch < G.C0; ++ch)
      for (int y = 0; y < G.h0; ++y)
        for (int x = 0; x < G.h0; ++x) ext(G.fc_bias + (long long)(y * G.h0 + x) * G.C0 + ch, 2);
    for (int ch = 0; ch < G.C0; ++ch) ext(G.fc_gamma + ch, 1);
    for (int ch = 0; ch < G.C0; ++ch) ext(G.fc_beta + ch, 2);
    int h = f.g_h0;
    for (int i = 1; i < f.n_g; ++i) {                       // Upsample x2 + Conv k3: 3 x 3 master weights [9][cb][cs]
      ConvLayer l;
      l.Cs = f.g_ch[i - 1]; l.Cb = f.g_ch[i]; l.CBT = l.Cb; l.Hs = h; l.cs_real = l.Cs; l.cb_real = l.Cb;
      l.w = o; o += (long long)9 * l.Cb * l.Cs;
      l.w4 = o4; o4 += (long long)16 * l.Cb * l.Cs;
      for (int co = 0; co < l.Cb; ++co)
        for (int ci = 0; ci < l.Cs; ++ci)
          for (int tap = 0; tap < 9; ++tap) ext(l.w + ((long long)tap * l.Cb + co) * l.Cs + ci, 0);
      l.gamma = o; o += l.Cb; l.beta = o; o += l.Cb; l.rs = r; r += l.Cb; l.bnC = l.Cb;
      for (int ch = 0; ch < l.Cb; ++ch) ext(l.gamma + ch, 1);
      for (int ch = 0; ch < l.Cb; ++ch) ext(l.beta + ch, 2);
      o = round_up(o, 8);
      G.conv.push_back(l);
      h *= 2;
    }
    {                                                       // last: Conv k3 s1 p1 onto the image, [9][img_c][cs]
      ConvLayer l;
      l.Cs = f.g_ch[f.n_g - 1]; l.Cb = f.img_c; l.CBT = l.Cb; l.Hs = h; l.cs_real = l.Cs; l.cb_real = l.Cb;
      l.w = o; o += (long long)9 * l.Cb * l.Cs;
      for (int co = 0; co < l.Cb; ++co)
        for (int ci = 0; ci < l.Cs; ++ci)
          for (int tap = 0; tap < 9; ++tap) ext(l.w + ((long long)tap * l.Cb + co) * l.Cs + ci, 0);
      l.bias = o; l.nbias = l.Cb; o += l.Cb;
      for (int ch = 0; ch < l.Cb; ++ch) ext(l.bias + ch, 2);
      o = round_up(o, 8);
      G.conv.push_back(l);
    }
    G.P = round_up(o, 64); G.Pext = (long long)G.ext2int.size(); G.nbn = r; G.P4 = round_up(o4, 64);
  }
  {
    Net& D = c->D;
    long long o = 0, r = 0;
    auto ext = [&](long long internal, int kind) { D.ext2int.push_back(internal); D.ext_kind.push_back(kind); };
    int h = f.img_hw;
    for (int j = 0; j < f.n_d; ++j) {
      ConvLayer l;
      l.cb_real = (j == 0) ? f.img_c : f.d_ch[j - 1];
      l.cs_real = f.d_ch[j];
      l.Cb = (j == 0) ? f.img_c : pad64(l.cb_real); l.CBT = l.Cb; l.Cs = pad64(l.cs_real); l.Hs = h / 2;
      l.w = o; o += (long long)16 * l.CBT * l.Cs;
      for (int co = 0; co < l.cs_real; ++co)
        for (int ci = 0; ci < l.cb_real; ++ci)
          for (int ky = 0; ky < 3; ++ky)
            for (int kx = 0; kx < 3; ++kx) ext(l.w + ((long long)(ky * 4 + kx) * l.CBT + ci) * l.Cs + co, 0);
      l.bias = o; l.nbias = l.Cs; o += l.Cs;
      for (int ch = 0; ch < l.cs_real; ++ch) ext(l.bias + ch, 2);
      if (j > 0) {
        l.gamma = o; o += l.Cs; l.beta = o; o += l.Cs; l.rs = r; l.bnC = l.Cs;
        for (int ch = 0; ch < l.cs_real; ++ch) ext(l.gamma + ch, 1);
        for (int ch = 0; ch < l.cs_real; ++ch) ext(l.beta + ch, 2);
        for (int ch = 0; ch < l.cs_real; ++ch) D.bn_ext2int.push_back(r + ch);
        r += l.Cs;
      }
      o = round_up(o, 8);
      D.conv.push_back(l);
      h /= 2;
    }
    const ConvLayer& last = D.conv.back();
    D.K = last.Cs * h * h; D.h0 = h; D.C0 = last.Cs;
    D.fc_w = o; o += D.K;
    for (int ch = 0; ch < last.cs_real; ++ch)
      for (int y = 0; y < h; ++y)
        for (int x = 0; x < h; ++x) ext(D.fc_w + (long long)(y * h + x) * last.Cs + ch, 0);
    D.fc_b = o; o += 1;
    ext(D.fc_b, 2);
    D.P = round_up(o, 64); D.Pext = (long long)D.ext2int.size(); D.nbn = r;
  }
}

// whether the GEMM engine runs this convolution (all but the ones next to the image)
bool on_engine(const gan_ctx* c, const Net& n, size_t i) { return &n == &c->G ? i + 1 < n.conv.size() : i > 0; }

// fp32 storage: whether the update writes the convolutions' weights split.  That is 40 bytes an update and weight where the weights and a
// transposed copy are 32, and 6 bytes instead of 4 in every GEMM; it spares the GEMMs splits for every row they multiply.  The line is on the rows a
// weight meets per model at the sizing batch (never a call's).  us a step, split / whole: a hundred 32x32 pairs, 102 rows 11357 / 9945, 205 rows 14830 /
// 14047, 410 rows 21633 / 21364, 819 rows 35735 / 36922; ten of them 102 rows 1694 / 1599, 205 rows 2249 / 2270, 410 rows 3130 / 3255; eight 64x64
// pairs 146 rows 1948 / 1850, 293 rows 2429 / 2487; a thousand 16x16 pairs 43 rows 9219 / 7865, 87 rows 11277 / 10155.  The networks of the
// tables, whose generator's k4 weights are made anew in any case, always have them split.
bool presplit_pays(const gan_ctx* c) {
  if (c->paper) return true;
  double weights = 0, rows = 0;
  for (const Net* n : {&c->G, &c->D})
    for (size_t i = 0; i < n->conv.size(); ++i) {
      const ConvLayer& cl = n->conv[i];
      if (!on_engine(c, *n, i)) continue;
      weights += (double)cl.Cb * cl.Cs;
      rows += (double)cl.Cb * cl.Cs * cl.Hs * cl.Hs;
    }
  return rows * c->NB >= 256.0 * c->L * weights;
}

bool alloc_net(gan_ctx* c, Net& n) {
  const size_t tot = (size_t)c->L * n.P;
  bool ok = dev_alloc(c, (void**)&n.theta, tot * 4) && dev_alloc(c, (void**)&n.m, tot * 4) &&
            dev_alloc(c, (void**)&n.v, tot * 4) && dev_alloc(c, (void**)&n.g, tot * 4) &&
            dev_alloc(c, (void**)&n.run_mean, (size_t)c->L * n.nbn * 4) &&
            dev_alloc(c, (void**)&n.run_var, (size_t)c->L * n.nbn * 4) &&
            dev_alloc(c, (void**)&n.t, (size_t)c->L * 4) && dev_alloc(c, (void**)&n.bc, (size_t)c->L * 8);
  if (!ok) return false;
  if (c->bf16) {
    if (!dev_alloc(c, &n.shadow_u, tot * 2) || !dev_alloc(c, &n.shadow_d, tot * 2)) return false;
    hipMemsetAsync(n.shadow_d, 0, tot * 2, c->st);
  } else {
    for (size_t i = 0; i < n.conv.size(); ++i) {
      ConvLayer& cl = n.conv[i];
      if (!on_engine(c, n, i)) continue;
      cl.part = n.PS;
      n.PS += (long long)16 * cl.Cb * cl.Cs;
    }
    const size_t parts = (size_t)c->L * n.PS * 6;
    if (c->presplit ? !dev_alloc(c, (void**)&n.split_u, parts) || !dev_alloc(c, (void**)&n.split_d, parts)
                    : !dev_alloc(c, &n.shadow_d, (size_t)c->L * n.PS * 4)) return false;
    n.shadow_u = n.theta;
  }
  hipMemsetAsync(n.theta, 0, tot * 4, c->st);
  hipMemsetAsync(n.m, 0, tot * 4, c->st);
  hipMemsetAsync(n.v, 0, tot * 4, c->st);
  hipMemsetAsync(n.g, 0, tot * 4, c->st);
  hipMemsetAsync(n.run_mean, 0, (size_t)c->L * n.nbn * 4, c->st);
  hipMemsetAsync(n.t, 0, (size_t)c->L * 4, c->st);
  hipMemsetAsync(n.bc, 0, (size_t)c->L * 8, c->st);
  return true;
}

// ---- built-in initialiser (host side, documented order; tests overwrite it through gan_set_params) ------
__global__ void init_normal_kernel(float* p, long long count, float std, unsigned long long seed, int inner, int inner_valid) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  if ((int)(i % inner) >= inner_valid) { p[i] = 0.f; return; }
  unsigned long long z = seed + 0x9E3779B97F4A7C15ull * (unsigned long long)(i + 1);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  const float u1 = ((float)(unsigned)(z >> 40) + 1.0f) * (1.0f / 16777217.0f);
  const float u2 = (float)(unsigned)((z >> 8) & 0xffffffu) * (1.0f / 16777216.0f);
  p[i] = std * sqrtf(-2.0f * logf(u1)) * cosf(6.2831853f * u2);
}
__global__ void fill_kernel(float* p, long long count, float v) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = v;
}
void init_normal(gan_ctx* c, float* p, long long count, int inner, int inner_valid, unsigned long long salt) {
  hipLaunchKernelGGL(init_normal_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, c->st, p, count,
                     c->cfg.init_std, c->cfg.seed * 0x100000001B3ull + salt, inner, inner_valid);
}
void fill(gan_ctx* c, float* p, long long count, float v) {
  if (count == 0) return;
  hipLaunchKernelGGL(fill_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, c->st, p, count, v);
}

void builtin_init(gan_ctx* c) {
  unsigned long long salt = 1;
  for (int l = 0; l < c->L; ++l) {
    Net& G = c->G;
    float* th = G.theta + (long long)l * G.P;
    init_normal(c, th + G.fc_w, (long long)G.J * G.Kp, G.Kp, G.Kz, salt++);
    fill(c, th + G.fc_gamma, G.C0, 1.f);
    for (auto& cl : G.conv) {
      init_normal(c, th + cl.w, (long long)16 * cl.CBT * cl.Cs, 1, 1, salt++);
      if (cl.bnC) fill(c, th + cl.gamma, cl.bnC, 1.f);
    }
    Net& D = c->D;
    th = D.theta + (long long)l * D.P;
    for (auto& cl : D.conv) {
      init_normal(c, th + cl.w, (long long)16 * cl.CBT * cl.Cs, 1, 1, salt++);
      if (cl.bnC) fill(c, th + cl.gamma, cl.bnC, 1.f);
    }
    init_normal(c, th + D.fc_w, D.K, 1, 1, salt++);
  }
  fill(c, c->G.run_var, (long long)c->L * c->G.nbn, 1.f);
  fill(c, c->D.run_var, (long long)c->L * c->D.nbn, 1.f);
}

// Built-in initialiser of the networks as printed in the tables: drawn on the host in the documented order and placed
// through the index map, so that padding and the unused fourth taps stay zero.
static float host_normal(unsigned long long& st) {
  auto next = [&]() {
    unsigned long long z = (st += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
  };
  const double u1 = ((double)(next() >> 11) + 1.0) / 9007199254740993.0, u2 = (double)(next() >> 11) / 9007199254740992.0;
  return (float)(sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2));
}
bool builtin_init_paper(gan_ctx* c) {
  unsigned long long st = c->cfg.seed * 0x100000001B3ull + 17;
  for (Net* n : {&c->G, &c->D}) {
    std::vector<float> tmp((size_t)n->P);
    for (int l = 0; l < c->L; ++l) {
      std::fill(tmp.begin(), tmp.end(), 0.f);
      for (long long i = 0; i < n->Pext; ++i) {
        const int kind = n->ext_kind[(size_t)i];
        tmp[(size_t)n->ext2int[(size_t)i]] = kind == 0 ? c->cfg.init_std * host_normal(st) : (kind == 1 ? 1.f : 0.f);
      }
      if (hipMemcpy(n->theta + (long long)l * n->P, tmp.data(), (size_t)n->P * 4, hipMemcpyHostToDevice) != hipSuccess) return false;
    }
  }
  fill(c, c->G.run_var, (long long)c->L * c->G.nbn, 1.f);
  fill(c, c->D.run_var, (long long)c->L * c->D.nbn, 1.f);
  return true;
}

// ---- storage-type copies of the weights ------------------------------------------------------------------

template <typename T>
void refresh_transposes(gan_ctx* c, Net& n) {
  pack_image_call<T>(c, n);                             // the image-side layer
  // layers run by the GEMM engine in "down" form need [tap][cs][cb]
  for (size_t i = 0; i < n.conv.size(); ++i) {
    const ConvLayer& cl = n.conv[i];
    if (!on_engine(c, n, i)) continue;
    Scope s(c, "transpose_w", 0, (double)c->L * 16 * cl.Cb * cl.Cs * 2 * sizeof(T));
    if (c->bf16)
      launch_transpose_w<bf16_t, bf16_t>((const bf16_t*)n.shadow_u + cl.w, (bf16_t*)n.shadow_d + cl.w, n.P, n.P, c->L, cl.Cb, cl.Cs, c->st);
    else if (!c->presplit)
      launch_transpose_w<float, float>(n.theta + cl.w, (float*)n.shadow_d + cl.part, n.P, n.PS, c->L, cl.Cb, cl.Cs, c->st);
    else
      launch_split_weights({n.theta + cl.w, n.split_u + cl.part, n.split_d + cl.part, n.P, n.PS, c->L, cl.Cb, cl.Cs}, c->st);
  }
}
// k4 weights with summed taps of G's Upsample + Conv k3 blocks, from the 3 x 3 master weights
template <typename T>
void paper_rebuild_w4(gan_ctx* c) {
  Net& G = c->G;
  for (size_t i = 0; i + 1 < G.conv.size(); ++i) {
    const ConvLayer& cl = G.conv[i];
    launch_w3_to_w4<T>(G.theta + cl.w, (T*)G.w4u + cl.w4, c->bf16 ? (T*)G.w4d + cl.w4 : nullptr, c->L, cl.Cb, cl.Cs, c->st, G.P, G.P4);
    if (!c->bf16) launch_split_weights({(const float*)G.w4u + cl.w4, G.split_u + cl.part, G.split_d + cl.part, G.P4, G.PS, c->L, cl.Cb, cl.Cs}, c->st);
  }
}
void refresh_shadows(gan_ctx* c) {
  for (Net* n : {&c->G, &c->D}) {
    if (c->bf16) launch_cast_shadow<bf16_t>(n->theta, (bf16_t*)n->shadow_u, (long long)c->L * n->P, c->st);
    if (c->paper && n == &c->G) {
      if (c->bf16) paper_rebuild_w4<bf16_t>(c); else paper_rebuild_w4<float>(c);
      continue;
    }
    if (c->bf16) refresh_transposes<bf16_t>(c, *n); else refresh_transposes<float>(c, *n);
  }
  c->shadows_dirty = false;
}

// ---- launch helpers ---------------------------------------------------------------------------------------
// The weights of a GEMM launch: see ConvArgs.
struct Weights {
  const void* w;
  long long stride, plane = 0;
  const float* raw = nullptr;
  long long raw_stride = 0;
  int raw_n = 0, raw_k = 0;
};
// of a convolution on the engine; up: as G's transposed convolutions and D's data gradients read them
Weights layer_weights(const gan_ctx* c, const Net& net, const ConvLayer& cl, bool up) {
  const bool k4 = cl.w4 >= 0;                          // summed taps (the networks of the tables, G)
  const long long off = k4 ? cl.w4 : cl.w, P = k4 ? net.P4 : net.P;
  if (c->bf16) return {(const bf16_t*)(k4 ? (up ? net.w4u : net.w4d) : (up ? net.shadow_u : net.shadow_d)) + off, P};
  if (!c->presplit) {
    if (up) return {net.theta + cl.w, net.P};
    return {(const float*)net.shadow_d + cl.part, net.PS};
  }
  return {(up ? net.split_u : net.split_d) + cl.part, 3 * net.PS, net.PS, (k4 ? (const float*)net.w4u : net.theta) + off, P, up ? cl.Cs : 1, up ? 1 : cl.Cs};
}
template <typename T>
void conv_call(gan_ctx* c, const char* name, int mode, int epi, const void* A, const Weights& W, void* Out,
               const void* Aux, int C, int N, int Hin, int Hr, int seg_first, int nseg, int n,
               bool stats = false, const NormArgs* known = nullptr, const float* bias = nullptr) {
  ConvArgs a = {};
  a.A = A; a.W = W.w; a.Out = Out; a.Aux = Aux; a.w_nstride = N;
  a.tile = layer_tile(c, mode, N, Hr * Hr, nseg);
  const int tr = conv_tile_rows((int)sizeof(T), a.tile);
  a.offs = c->rb.offs; a.tpre = tpre_of(c, Hr * Hr, tr); a.tmodel = tmodel_of(c, Hr * Hr, tr);
  a.w_stride = W.stride; a.w_plane = W.plane; a.w_raw = W.raw; a.raw_stride = W.raw_stride; a.raw_n = W.raw_n; a.raw_k = W.raw_k;
  a.L = c->L; a.seg_first = seg_first; a.nseg = nseg; a.seg_samples = n;
  a.C = C; a.N = N; a.Hin = Hin; a.Hr = Hr; a.ub_tiles = ub_tiles(c, n, Hr * Hr, tr);
  a.slope = c->cfg.leaky_slope;
  if (epi == EPI_BN) {
    a.bn_mean = known->run_mean; a.bn_var = known->run_var; a.bn_rstride = known->rstride;
    a.bn_gamma = known->gamma; a.bn_beta = known->beta; a.bn_bias = bias; a.bn_pstride = known->pstride;
    a.bn_C = known->C; a.bn_eps = known->eps; a.slope = known->slope;
  }
  if (epi == EPI_BIAS_ACT) { a.bn_bias = bias; a.bn_pstride = known->pstride; a.slope = 0.f; }
  if (epi == EPI_DROP_BWD) a.drop_scale = 1.0f / (1.0f - c->cfg.dropout_p);
  a.stat_partial = stats ? c->stat_partial : nullptr;
  const int ntaps = mode == MODE_DOWN ? 16 : (mode == MODE_UP ? 4 : 1);
  const int phases = mode == MODE_UP ? 4 : 1;
  const double rows = (double)n * nseg * Hr * Hr * phases;
  const double frac = mode == MODE_DENSE ? 1.0 : valid_tap_fraction(Hr);
  const double flops = 2.0 * rows * N * C * ntaps * frac;
  const double in_elems = mode == MODE_DENSE ? rows * C : (double)n * nseg * Hin * Hin * C;
  const double bytes = sizeof(T) * (in_elems + rows * N + (double)c->L * (mode == MODE_DENSE ? 1 : 16) * C * N);
  char detail[64];
  snprintf(detail, sizeof(detail), "[C%d N%d H%d seg%d]", C, N, Hr, nseg);
  (void)name;
  Scope s(c, conv_variant_name((int)sizeof(T), mode, epi, a), flops, bytes, detail);
  launch_conv<T>(mode, epi, a, c->st);
}

// Row splits of a weight-gradient launch whose output tiles alone would leave part of the chip idle: every model's rows
// are shared by this many blocks per tile, whose partial results are added in a fixed order.  The number with the
// smallest estimated time: the products at the rate a full chip reaches, stretched by what the last round of blocks
// leaves idle, plus writing and adding the partial results.  A function of the configuration only -- the number of
// models, the sizing batch and the layer's shape -- never of a call's batch.  Partial results are charged with their writing, their reading and a launch that
// writes the sum.  That launch is left to the linear layers and the tables' networks; where the update adds them up on its way (wgrad_call, leave) a split
// costs that much less than it is charged with, which no number of splits has been measured again for.
int wgrad_ksplit(const gan_ctx* c, int Cb, int Cs, int ntaps, int Hs, int nseg) {
  const double blocks = (double)c->L * wgrad_tiles_per_model((int)esize(c), ntaps, Cb, Cs);
  const double rows = (double)c->NB * nseg * Hs * Hs, out = (double)c->L * ntaps * Cb * Cs * 4;
  // bf16: counted as one block per CU, which the 256x256 and 256x128 tiles are (128 and 96 KiB of LDS); of the 256x64 tile (80 KiB) a CU
  // holds two, which the estimate does not tell apart.  fp32: a CU holds two blocks, which reached 133 TFLOP/s over the chip where single ones reached 99
  // when every wave split what it multiplied (ten models of 128 samples, 64 -> 128 channels at side 7, two segments, 80 tiles); with chunks split once a block
  // 156 and 106: 3 splits 310 us, 4 287, 6 211, 7 279, 8 254, 12 213.  The bf16 256x256 tile in quarters reaches 900 to 1020.  Of 99 shapes, batches and
  // numbers of models two (fp32) and eleven (bf16) would be split otherwise with these rates, ten of the thirteen by a tenth at most, so the rates
  // stand as they were taken.
  const double product = 2.0 * rows * ntaps * Cb * Cs / (c->bf16 ? 900e12 : 133e12), single = c->bf16 ? 1.0 : 1.34;
  const double chunk_rows = 128 / (double)esize(c);
  int best = 1;
  double best_t = 0;
  for (int k = 1; k <= WG_MAX_KSPLIT; ++k) {
    if (k > 1 && rows / nseg / c->L < 2 * chunk_rows * k) break;             // at least two chunks for every block
    const double b = blocks * k, full = (double)(((long long)b + 255) / 256), rounds = full > 1 ? full : single;
    const double t = product * rounds * 256 / b + (k > 1 ? 5e-6 + (2 * k + 1) * out / 4e12 : 0);
    if (k == 1 || t < best_t) { best = k; best_t = t; }
  }
  return best;
}

// A weight gradient into dW, its rows split as wgrad_ksplit says, through c->wg_part.  leave: the splits, which the update of these weights, which has to
// come before the next of these calls, adds up itself.
template <typename T>
void wgrad_call(gan_ctx* c, const void* Big, const void* Small, float* dW, long long stride, int Cb, int Cs, int Hs, int ntaps, int nseg, int n,
                hipStream_t st = nullptr, AdamSplits* leave = nullptr) {
  if (!st) st = c->st;
  WgradArgs a = {};
  a.Big = Big; a.Small = Small; a.dW = dW; a.offs = c->rb.offs; a.order = c->rb.order; a.dw_stride = stride;
  a.L = c->L; a.nseg = nseg; a.seg_samples = n; a.Cb = Cb; a.Cs = Cs; a.Hs = Hs; a.ntaps = ntaps;
  const long long layer = (long long)ntaps * Cb * Cs;
  const int ksplit = a.ksplit = wgrad_ksplit(c, Cb, Cs, ntaps, Hs, nseg);
  if (ksplit > 1) {
    a.dW = c->wg_part; a.dw_stride = layer; a.split_stride = (long long)c->L * layer;
  }
  const double rows = (double)n * nseg * Hs * Hs;
  const double frac = ntaps == 1 ? 1.0 : valid_tap_fraction(Hs);
  const double big_elems = ntaps == 1 ? rows * Cb : (double)n * nseg * 4 * Hs * Hs * Cb;
  const double bytes = sizeof(T) * (big_elems + rows * Cs) + 4.0 * c->L * ntaps * Cb * Cs;
  char detail[64];
  snprintf(detail, sizeof(detail), "[Cb%d Cs%d H%d seg%d]", Cb, Cs, Hs, nseg);
  {
    Scope s(c, wgrad_variant_name((int)sizeof(T), a), 2.0 * rows * Cb * Cs * ntaps * frac, bytes, detail, st);
    launch_wgrad<T>(a, st);
  }
  if (leave) *leave = {c->wg_part, ksplit, split_chains(layer * c->L, ksplit)};
  else if (ksplit > 1) launch_sum_splits(c->wg_part, dW, stride, layer, c->L, ksplit, st);
}

template <typename T>
NormArgs norm_args(gan_ctx* c, Net& net, int C, int rps, long long gamma, long long beta, long long rs, float* mean, float* var,
                   float* rstd, float* sums, int seg_first, int nseg, int n, float slope) {
  NormArgs a;
  memset(&a, 0, sizeof(a));
  a.mean = mean; a.var = var; a.rstd = rstd; a.sums = sums;
  a.gamma = net.theta + gamma; a.beta = net.theta + beta; a.dgamma = net.g + gamma; a.dbeta = net.g + beta;
  a.pstride = net.P;
  a.run_mean = net.run_mean + rs; a.run_var = net.run_var + rs; a.rstride = net.nbn;
  a.offs = c->rb.offs; a.counts = c->rb.counts; a.sample_model = c->rb.sample_model;
  a.L = c->L; a.C = C; a.rps = rps; a.seg_first = seg_first; a.nseg = nseg; a.seg_samples = n; a.n = n;
  a.slope = slope; a.eps = c->cfg.bn_eps; a.momentum = c->cfg.bn_momentum;
  return a;
}

// BatchNorm with batch statistics + activation: x -> y (with running statistics both are part of the GEMM: EPI_BN)
// gemm_mode / gemm_rps describe the GEMM that produced x and left per-tile column sums in c->stat_partial
// the normalised and activated tensor; head: and D's head behind it
template <typename T>
void apply_call(gan_ctx* c, const NormArgs& a, const HeadArgs* head) {
  const double elems = (double)a.n * a.nseg * a.rps * a.C;
  Scope s(c, head ? "bn_apply_head" : "bn_apply", 0, 2 * elems * sizeof(T));
  if (head) launch_bn_apply_head<T>(a, *head, c->st);
  else launch_bn_apply<T>(a, c->st);
}
template <typename T>
void bn_forward(gan_ctx* c, NormArgs a, const void* x, void* y, bool update_running, int gemm_mode, int gemm_rps, int col_groups = 1,
                const HeadArgs* head = nullptr) {      // y NULL: the statistics only
  a.x = x; a.y = y;
  {
    const ConvTile tile = layer_tile(c, gemm_mode, a.C * col_groups, gemm_rps, a.nseg);   // of the GEMM that left the partials (N = C * col_groups)
    const int tr = conv_tile_rows((int)sizeof(T), tile), gemm_phases = gemm_mode == MODE_UP ? 4 : 1;
    a.fold_running = update_running;
    launch_bn_stats_from_partial(a, c->stat_partial, tpre_of(c, gemm_rps, tr), ub_tiles(c, a.n, gemm_rps, tr), ub_tiles(c, c->NB, gemm_rps, tr),
                                 gemm_phases, col_groups, tr, gemm_rps, conv_stat_split((int)sizeof(T), tile, c->presplit && gemm_mode != MODE_DENSE), c->st);
  }
  if (y) apply_call<T>(c, a, head);
}

// dy (w.r.t. the activated output) -> dx (w.r.t. the pre-normalisation tensor), plus dgamma / dbeta
template <typename T>
void bn_backward(gan_ctx* c, NormArgs a, const void* x, const void* dy, void* dx, bool param_grads) {
  a.x = x; a.dy = dy; a.y = dx;
  a.param_grads = param_grads;
  const double elems = (double)a.n * a.nseg * a.rps * a.C;
  {
    Scope s(c, "bn_bwd_reduce", 0, 2 * elems * sizeof(T));
    const int tr = a.red_rows = red_rows(c, a.rps);
    a.red_tiles = ub_tiles(c, c->NB, a.rps, tr);
    launch_bn_bwd_reduce<T>(a, tpre_of(c, a.rps, tr), tmodel_of(c, a.rps, tr), ub_tiles(c, a.n, a.rps, tr), c->stat_partial, c->st);
  }
  Scope s(c, "bn_bwd_apply", 0, 3 * elems * sizeof(T));
  launch_bn_bwd_apply<T>(a, c->st);
}

double img_flops(const ConvLayer& cl, int n, int nseg) {
  return 2.0 * n * nseg * cl.Hs * cl.Hs * 16 * cl.Cb * cl.Cs * valid_tap_fraction(cl.Hs);
}

// transposed conv onto the image side: feat (absolute segment seg) -> out (same segment indexing), or the caller's images
template <typename T>
void up_img_call(gan_ctx* c, Net& net, const ConvLayer& cl, const void* feat, void* out, const void* aux, int mode, int seg, int n,
                 float* user = nullptr) {
  UpImgArgs a;
  memset(&a, 0, sizeof(a));
  a.feat = feat; a.w = (const T*)net.shadow_u + cl.w; a.w_stride = net.P; a.out = out; a.aux = aux;
  a.bias = mode == 1 ? net.theta + cl.bias : nullptr; a.bias_stride = net.P;
  a.offs = c->rb.offs; a.sample_model = c->rb.sample_model; a.L = c->L; a.n = n; a.seg = seg; a.seg_samples = n;
  a.CB = cl.Cb; a.CBT = cl.CBT; a.Cs = cl.Cs; a.Hs = cl.Hs; a.mode = mode; a.user = user; a.perm = c->rb.perm;
  Scope s(c, "up_img", img_flops(cl, n, 1), sizeof(T) * (double)n * cl.Hs * cl.Hs * (cl.Cs + 4.0 * cl.Cb * (mode == 2 ? 2 : 1)));
  launch_up_img<T>(a, c->st);
}

// packed weights of an image-side layer
template <typename T>
void pack_image_call(gan_ctx* c, const Net& net) {
  const bool first = &net == &c->D;                 // (G's last layer: as its gradients read it)
  const ConvLayer& cl = first ? net.conv.front() : net.conv.back();
  ImagePackArgs a = {};
  a.w = net.theta + cl.w; a.packed = first ? c->wpD : c->wpG; a.add = first && cl.CBT > cl.Cb ? c->addD : nullptr;
  a.pstride = net.P; a.L = c->L; a.CB = cl.Cb; a.CBT = cl.CBT; a.Cs = cl.Cs; a.P = image_values(cl.Cb); a.tables = c->labels > 0 ? c->labels : c->L;
  Scope s(c, "pack_w", 0, (double)c->L * cl.Cs * 16 * (4.0 * cl.CBT + a.P * sizeof(T)));
  launch_pack_image_w<T>(a, c->st);
}
// The strided convolution of images: D's first layer (label maps, bias, LeakyReLU), or with `grad` the data gradient of G's last layer from
// the gradient of its images.  real: the caller's batch in place of segment 0.
template <typename T>
void image_conv_call(gan_ctx* c, const ConvLayer& cl, const void* img, const float* real, void* out, bool grad, int seg_first, int nseg, int n) {
  ImageConvArgs a = {};
  a.img = img; a.real = real; a.perm = c->rb.perm; a.w = grad ? c->wpG : c->wpD; a.add = grad || cl.CBT == cl.Cb ? nullptr : c->addD;
  a.bias = grad ? nullptr : c->D.theta + cl.bias; a.bias_stride = c->D.P;
  a.sample_slot = !grad && c->labels > 0 ? c->rb.sample_slot : nullptr;
  a.out = out; a.offs = c->rb.offs; a.sample_model = c->rb.sample_model;
  a.L = c->L; a.n = n; a.CB = cl.Cb; a.Hs = cl.Hs; a.Cs = cl.Cs; a.seg_first = seg_first; a.nseg = nseg; a.seg_samples = n;
  a.slope = grad ? 1.f : c->cfg.leaky_slope;
  const double rows = (double)n * nseg * cl.Hs * cl.Hs;
  Scope s(c, grad ? "image_conv_grad" : "image_conv", img_flops(cl, n, nseg), sizeof(T) * rows * (4.0 * cl.Cb + cl.Cs));
  launch_image_conv<T>(a, c->st);
}
// Its weight gradient, into the network's gradient block: the taps, the label maps and the bias of D's first layer, the taps and the bias of G's last.
template <typename T>
void image_wgrad_call(gan_ctx* c, Net& net, const ConvLayer& cl, const void* img, const float* real, const void* dy, int seg_first, int nseg, int n) {
  const bool first = &net == &c->D;
  ImageWgradArgs a = {};
  a.img = img; a.real = real; a.perm = c->rb.perm; a.dy = dy; a.part = c->img_part; a.pixel_sums = first ? nullptr : c->img_sums;
  a.tiles = c->img_tiles;
  a.offs = c->rb.offs; a.tpre = tpre_of(c, 1, a.tiles.most, a.tiles.parts); a.tmodel = tmodel_of(c, 1, a.tiles.most, a.tiles.parts);
  a.L = c->L; a.CB = cl.Cb; a.Hs = cl.Hs; a.Cs = cl.Cs; a.seg_first = seg_first; a.nseg = nseg; a.seg_samples = n;
  const double rows = (double)n * nseg * cl.Hs * cl.Hs;
  {
    Scope s(c, "image_wgrad", img_flops(cl, n, nseg), sizeof(T) * rows * (4.0 * cl.Cb + cl.Cs));
    launch_image_wgrad<T>(a, (int)image_tile_bound(a.tiles, n, c->L), c->st);
  }
  if (first && c->labels > 0) {
    ClassSumArgs b;
    memset(&b, 0, sizeof(b));
    b.dy = dy; b.part = c->class_part; b.sums = c->label_sums; b.offs = c->rb.offs; b.sample_slot = c->rb.sample_slot;
    b.L = c->L; b.n = n; b.Hs = cl.Hs; b.Cs = cl.Cs; b.labels = c->labels; b.seg_first = seg_first; b.nseg = nseg; b.seg_samples = n;
    Scope s(c, "class_sums", 0, rows * cl.Cs * sizeof(T));
    launch_class_sums<T>(b, c->st);
  }
  ImageGradArgs g = {};
  g.part = c->img_part; g.pixel_sums = a.pixel_sums; g.tpre = a.tpre; g.dw = net.g + cl.w;
  g.dbias = first ? net.g + cl.bias : nullptr; g.image_bias = first ? nullptr : net.g + cl.bias;
  g.k3 = c->paper;
  if (first && c->head_rsplit > 1) g.head = {c->head_part, net.g + net.fc_w, net.g + net.fc_b, net.K, c->head_rsplit};
  g.labels = first ? c->labels : 0; g.label_sums = c->label_sums; g.plane_labels = first && cl.CBT > cl.Cb && c->labels == 0;
  g.pstride = net.P; g.L = c->L; g.CB = cl.Cb; g.CBT = cl.CBT; g.Cs = cl.Cs; g.P = image_values(cl.Cb);
  // the tiles' sums (of as many tiles as evenly spread samples have), the gradients, the head's splits
  const int own = (n + c->L - 1) / c->L, per = image_tile(a.tiles, own);
  const double sums = (double)c->L * 16 * cl.Cs * ((own + per - 1) / per * g.P + cl.CBT), heads = g.head.part ? (double)c->L * (g.head.rsplit + 1) * g.head.K : 0;
  Scope s(c, "image_wgrad_sum", 0, 4.0 * (sums + heads));
  launch_image_wgrad_final(g, c->st);
}

// A pass through D belongs to one of the two costs, and that says which segments it runs over.
struct Segments { int first, count; };
Segments segments_of(Cost cost) { return cost == COST_D ? Segments{0, 2} : Segments{1, 1}; }

// D's linear head
HeadArgs head_args(gan_ctx* c, int n, Cost cost) {
  Net& D = c->D;
  HeadArgs h;
  memset(&h, 0, sizeof(h));
  h.feat = c->dact[D.conv.size() - 1]; h.dfeat = c->bufA; h.w = D.theta + D.fc_w; h.b = D.theta + D.fc_b;
  h.dw = D.g + D.fc_w; h.db = D.g + D.fc_b; h.pstride = D.P; h.logits = c->logits; h.dlogits = c->dlogits;
  h.part = c->head_part; h.rsplit = c->head_rsplit;
  h.offs = c->rb.offs; h.sample_model = c->rb.sample_model; h.L = c->L; h.K = D.K;
  const Segments seg = segments_of(cost);
  h.seg_first = seg.first; h.nseg = seg.count; h.seg_samples = n; h.n = n;
  h.cost = cost;
  h.loss = cost == COST_D ? c->loss_d : c->loss_g;
  h.scale = cost == COST_D ? c->cfg.d_loss_scale : c->cfg.g_loss_scale;
  const Net& net = cost == COST_D ? c->D : c->G;      // whose update follows
  h.adam_t = net.t; h.adam_bc = net.bc; h.beta1 = c->cfg.beta1; h.beta2 = c->cfg.beta2;
  return h;
}

// ---- the networks -------------------------------------------------------------------------------------------
// user: the caller's images (generation), or NULL: into the fake half of D's image buffer
template <typename T>
void g_forward(gan_ctx* c, int n, bool use_running, bool update_running, float* user = nullptr) {
  Net& G = c->G;
  const float relu = 0.f;
  const NormArgs a0 = norm_args<T>(c, G, G.C0, G.h0 * G.h0, G.fc_gamma, G.fc_beta, G.fc_rs, c->g_mean[0], c->g_var[0], c->g_rstd[0],
                                   c->g_sums[0], 0, 1, n, relu);
  conv_call<T>(c, "gemm_dense", MODE_DENSE, use_running ? EPI_BN : EPI_NONE, c->zin, Weights{(const T*)G.shadow_u + G.fc_w, G.P},
               use_running ? c->gact[0] : c->gpre[0], nullptr, G.Kp, G.J, 1, 1, 0, 1, n, !use_running, &a0);
  if (!use_running) bn_forward<T>(c, a0, c->gpre[0], c->gact[0], update_running, MODE_DENSE, 1, G.h0 * G.h0);
  const int nl = (int)G.conv.size();
  for (int i = 0; i + 1 < nl; ++i) {
    const ConvLayer& cl = G.conv[i];
    const NormArgs a = norm_args<T>(c, G, cl.Cb, 4 * cl.Hs * cl.Hs, cl.gamma, cl.beta, cl.rs, c->g_mean[i + 1], c->g_var[i + 1],
                                    c->g_rstd[i + 1], c->g_sums[i + 1], 0, 1, n, relu);
    conv_call<T>(c, "gemm_up", MODE_UP, use_running ? EPI_BN : EPI_NONE, c->gact[i], layer_weights(c, G, cl, true),
                 use_running ? c->gact[i + 1] : c->gpre[i + 1], nullptr, cl.Cs, cl.Cb, cl.Hs, cl.Hs, 0, 1, n, !use_running, &a);
    if (!use_running) bn_forward<T>(c, a, c->gpre[i + 1], c->gact[i + 1], update_running, MODE_UP, cl.Hs * cl.Hs);
  }
  // last transposed conv (+bias, tanh) straight into the fake half of D's image buffer
  const ConvLayer& cl = G.conv[nl - 1];
  // G's samples sit in segment 0, the fake images in segment 1 of D's image buffer: offset the output pointer
  T* fake = (T*)c->xd + (long long)n * 4 * cl.Hs * cl.Hs * cl.Cb;
  up_img_call<T>(c, G, cl, c->gact[nl - 1], fake, nullptr, 1, 0, n, user);
}

template <typename T>
void d_forward(gan_ctx* c, int n, Cost cost, bool update_running, const float* real = nullptr) {
  Net& D = c->D;
  const int seg_first = segments_of(cost).first, nseg = segments_of(cost).count;
  const float slope = c->cfg.leaky_slope;
  image_conv_call<T>(c, D.conv[0], c->xd, real, c->dact[0], false, seg_first, nseg, n);      // first conv (+label maps, bias, LeakyReLU)
  const int nl = (int)D.conv.size();
  const HeadArgs head = head_args(c, n, cost);
  for (int j = 1; j < nl; ++j) {
    const ConvLayer& cl = D.conv[j];
    conv_call<T>(c, "gemm_down", MODE_DOWN, EPI_NONE, c->dact[j - 1], layer_weights(c, D, cl, false), c->dpre[j], nullptr, cl.Cb,
                 cl.Cs, 2 * cl.Hs, cl.Hs, seg_first, nseg, n, true);
    bn_forward<T>(c, norm_args<T>(c, D, cl.Cs, cl.Hs * cl.Hs, cl.gamma, cl.beta, cl.rs, c->d_mean[j], c->d_var[j], c->d_rstd[j],
                                  c->d_sums[j], seg_first, nseg, n, slope),
                  c->dpre[j], c->dact[j], update_running, MODE_DOWN, cl.Hs * cl.Hs, 1, j == nl - 1 ? &head : nullptr);
  }
}

// Backward through D.  param_grads: fill D's gradient block (both segments summed).  to_image: continue down to
// d cost / d fake, multiplied by the tanh derivative, into dimg.
// adam (with param_grads): D's planned update, whose step counts and bias corrections the head's launch here advances, in front of
// every part of it; the update of a convolution's weights is enqueued beside the chain as soon as its gradient is complete and its
// data gradient has read the old ones.
template <typename T>
void d_backward(gan_ctx* c, int n, Cost cost, bool param_grads, bool to_image, const float* real = nullptr, const AdamArgs* adam = nullptr, AdamTail* tail = nullptr) {
  Net& D = c->D;
  const int seg_first = segments_of(cost).first, nseg = segments_of(cost).count;
  hipStream_t side = side_stream(c);
  const float slope = c->cfg.leaky_slope;
  const int nl = (int)D.conv.size();
  {
    Scope s(c, "head_bwd", 0, sizeof(T) * (double)n * nseg * D.K * (param_grads ? 2 : 1));
    launch_head_bwd<T>(head_args(c, n, cost), param_grads, c->st);
  }
  int pending = -1;                // region of D's planned update whose turn comes next
  AdamSplits splits;               // and the row splits of its gradient
  for (int j = nl - 1; j >= 1; --j) {
    const ConvLayer& cl = D.conv[j];
    // in place: the pre-normalisation tensor is not needed again in this step, its gradient takes its place
    void* dx = c->dpre[j];
    bn_backward<T>(c, norm_args<T>(c, D, cl.Cs, cl.Hs * cl.Hs, cl.gamma, cl.beta, cl.rs, c->d_mean[j], c->d_var[j], c->d_rstd[j],
                                   c->d_sums[j], seg_first, nseg, n, slope),
                   c->dpre[j], c->bufA, dx, param_grads);
    if (param_grads) {
      // Beside the chain, in this order: the update of the layer above (its data gradient, which read the old weights,
      // is done; being bandwidth-bound it pairs with the data-gradient GEMM below), then this layer's weight gradient.
      order_after(c, side, c->st);
      if (adam && pending >= 0) adam_region_call<T>(c, *adam, pending, side, splits);
      wgrad_call<T>(c, c->dact[j - 1], dx, D.g + cl.w, D.P, cl.Cb, cl.Cs, cl.Hs, 16, nseg, n, side, adam ? &splits : nullptr);
      pending = j - 1;
    }
    // data gradient; for the first conv's output the LeakyReLU derivative is applied in the epilogue
    conv_call<T>(c, "gemm_up", MODE_UP, j == 1 ? EPI_ACT_BWD : EPI_NONE, dx, layer_weights(c, D, cl, true), c->bufA,
                 j == 1 ? c->dact[0] : nullptr, cl.Cs, cl.Cb, cl.Hs, cl.Hs, seg_first, nseg, n);
  }
  if (param_grads && adam && pending >= 0) {
    if (side == c->st && adam_region_joins_rest(*adam, pending)) {
      *tail = {pending, splits};
    } else {
      order_after(c, side, c->st);
      adam_region_call<T>(c, *adam, pending, side, splits);
    }
  }
  const ConvLayer& c1 = D.conv[0];
  if (param_grads) image_wgrad_call<T>(c, D, c1, c->xd, real, c->bufA, seg_first, nseg, n);
  if (to_image)   // d cost / d fake, times the tanh derivative (fake segment only)
    up_img_call<T>(c, D, c1, c->bufA, c->dimg, c->xd, 2, 1, n);
}

// Backward through G from dimg (fake segment) = d cost / d (pre-tanh output).
template <typename T>
void g_backward(gan_ctx* c, int n, const AdamArgs* adam = nullptr, AdamTail* tail = nullptr) {
  Net& G = c->G;
  hipStream_t side = side_stream(c);
  const int nl = (int)G.conv.size();
  const ConvLayer& last = G.conv[nl - 1];
  const T* dlast = (const T*)c->dimg + (long long)n * 4 * last.Hs * last.Hs * last.Cb;
  image_wgrad_call<T>(c, G, last, dlast, nullptr, c->gact[nl - 1], 0, 1, n);
  image_conv_call<T>(c, last, dlast, nullptr, c->bufA, true, 0, 1, n);
  int pending = -1;
  AdamSplits splits;
  for (int i = nl - 2; i >= 0; --i) {
    const ConvLayer& cl = G.conv[i];
    void* dx = c->gpre[i + 1];     // in place, as in D
    bn_backward<T>(c, norm_args<T>(c, G, cl.Cb, 4 * cl.Hs * cl.Hs, cl.gamma, cl.beta, cl.rs, c->g_mean[i + 1], c->g_var[i + 1],
                                   c->g_rstd[i + 1], c->g_sums[i + 1], 0, 1, n, 0.f),
                   c->gpre[i + 1], c->bufA, dx, true);
    order_after(c, side, c->st);
    if (adam && pending >= 0) adam_region_call<T>(c, *adam, pending, side, splits);      // as in D
    wgrad_call<T>(c, dx, c->gact[i], G.g + cl.w, G.P, cl.Cb, cl.Cs, cl.Hs, 16, 1, n, side, adam ? &splits : nullptr);
    pending = i;
    conv_call<T>(c, "gemm_down", MODE_DOWN, EPI_NONE, dx, layer_weights(c, G, cl, false), c->bufA, nullptr, cl.Cb, cl.Cs,
                 2 * cl.Hs, cl.Hs, 0, 1, n);
  }
  bn_backward<T>(c, norm_args<T>(c, G, G.C0, G.h0 * G.h0, G.fc_gamma, G.fc_beta, G.fc_rs, c->g_mean[0], c->g_var[0], c->g_rstd[0],
                                 c->g_sums[0], 0, 1, n, 0.f),
                 c->gpre[0], c->bufA, c->gpre[0], true);
  // (row-split partial sums share one scratch area with the weight gradients above: same stream)
  order_after(c, side, c->st);
  if (adam && pending >= 0) {
    if (side == c->st && adam_region_joins_rest(*adam, pending) && (splits.n < 2 || wgrad_ksplit(c, G.J, G.Kp, 1, 1, 1) == 1)) *tail = {pending, splits};
    else adam_region_call<T>(c, *adam, pending, side, splits);
  }
  wgrad_call<T>(c, c->gpre[0], c->zin, G.g + G.fc_w, G.P, G.J, G.Kp, 1, 1, 1, n, side);
  order_after(c, c->st, side);
}

// ---- the networks as printed in the paper's Tables 1 and 2 ---------------------------------------------------
PointArgs point_args(gan_ctx* c, void* x, int C, int Cpad, int HW, int seg_first, int nseg, int n) {
  PointArgs a;
  memset(&a, 0, sizeof(a));
  a.x = x; a.offs = c->rb.offs; a.sample_model = c->rb.sample_model; a.L = c->L; a.n = n; a.C = C; a.Cpad = Cpad; a.HW = HW;
  a.seg_first = seg_first; a.nseg = nseg; a.seg_samples = n; a.slope = 1.f; a.scale = 1.f;
  a.seed_lo = (unsigned)(c->cfg.seed & 0xffffffffull); a.seed_hi = (unsigned)(c->cfg.seed >> 32);
  return a;
}
float dropout_scale(const gan_ctx* c) { return 1.0f / (1.0f - c->cfg.dropout_p); }
// dropout of D's block `layer` (1-based) in the passes pass0 (first processed segment) and pass0 + 1
void with_dropout(gan_ctx* c, PointArgs& a, int layer, int pass0, int step_add) {
  const float p = c->cfg.dropout_p;
  if (!(p > 0.f)) return;
  a.thr = (unsigned)ceil((double)p * 16777216.0);
  a.scale = dropout_scale(c);
  a.layer = layer; a.pass_of_seg[0] = pass0; a.pass_of_seg[1] = pass0 + 1;
  a.steps = c->D.t; a.step_add = step_add;
}

// BatchNorm whose batch statistics are taken from the stored tensor (`real` channels and padding); no activation after it
template <typename T>
void bn_forward_direct(gan_ctx* c, NormArgs a, int real, const void* x, void* y, float eps, bool update_running, const HeadArgs* head = nullptr) {
  a.x = x; a.y = y; a.eps = eps; a.slope = 1.f;
  launch_bn_stats_direct<T>(a, real, c->st);
  if (update_running) launch_bn_running(a, c->st);
  apply_call<T>(c, a, head);
}

// G's last convolution reads the block in front of it before its BatchNorm and activation
void paper_last_norm(gan_ctx* c, Conv3Args& a) {
  const Net& G = c->G;
  const int last = (int)G.conv.size() - 1;
  const ConvLayer& cl = G.conv[last - 1];
  a.in = c->gpre[last];
  a.bn_mean = c->g_mean[last]; a.bn_rstd = c->g_rstd[last]; a.bn_gamma = G.theta + cl.gamma; a.bn_beta = G.theta + cl.beta;
  a.bn_pstride = G.P; a.bn_slope = c->cfg.leaky_slope;
}

template <typename T>
void paper_g_forward(gan_ctx* c, int n, bool use_running, bool update_running, float* user = nullptr) {
  Net& G = c->G;
  const gan_config& f = c->cfg;
  NormArgs a0 = norm_args<T>(c, G, G.C0, G.h0 * G.h0, G.fc_gamma, G.fc_beta, G.fc_rs, c->g_mean[0], c->g_var[0], c->g_rstd[0],
                             c->g_sums[0], 0, 1, n, 1.f);
  a0.eps = f.bn_eps_first;
  conv_call<T>(c, "gemm_dense", MODE_DENSE, use_running ? EPI_BN : EPI_BIAS_ACT, c->zin, Weights{(const T*)G.shadow_u + G.fc_w, G.P},
               use_running ? c->gact[0] : c->gpre[0], nullptr, G.Kp, G.J, 1, 1, 0, 1, n, false, &a0, G.theta + G.fc_bias);   // + bias, ReLU
  if (!use_running) bn_forward_direct<T>(c, a0, a0.C, c->gpre[0], c->gact[0], f.bn_eps_first, update_running);
  const int nl = (int)G.conv.size();
  for (int i = 0; i + 1 < nl; ++i) {                   // Upsample x2 + Conv k3 as a k4 s2 p1 transposed convolution
    const ConvLayer& cl = G.conv[i];
    const NormArgs a = norm_args<T>(c, G, cl.Cb, 4 * cl.Hs * cl.Hs, cl.gamma, cl.beta, cl.rs, c->g_mean[i + 1], c->g_var[i + 1],
                                    c->g_rstd[i + 1], c->g_sums[i + 1], 0, 1, n, f.leaky_slope);
    conv_call<T>(c, "gemm_up", MODE_UP, use_running ? EPI_BN : EPI_NONE, c->gact[i], layer_weights(c, G, cl, true),
                 use_running ? c->gact[i + 1] : c->gpre[i + 1], nullptr, cl.Cs, cl.Cb, cl.Hs, cl.Hs, 0, 1, n, !use_running, &a);
    // (the last block's BatchNorm and activation are part of the kernels that read its output)
    if (!use_running) bn_forward<T>(c, a, c->gpre[i + 1], i + 2 < nl ? c->gact[i + 1] : nullptr, update_running, MODE_UP, cl.Hs * cl.Hs);
  }
  const ConvLayer& cl = G.conv[nl - 1];                // Conv k3 s1 p1 (+bias) -> tanh, into the fake half of D's image buffer or the caller's
  Conv3Args a;
  memset(&a, 0, sizeof(a));
  a.in = c->gact[nl - 1]; a.out = c->xd; a.w = G.theta + cl.w; a.w_stride = G.P; a.bias = G.theta + cl.bias; a.bias_stride = G.P;
  a.offs = c->rb.offs; a.sample_model = c->rb.sample_model; a.L = c->L; a.n = n; a.H = cl.Hs; a.Cin = cl.Cs; a.CO = cl.Cb;
  a.out_seg = 1; a.seg_samples = n; a.user = user; a.perm = c->rb.perm;
  if (!use_running) paper_last_norm(c, a);
  Scope s(c, "conv3_img", 2.0 * n * cl.Hs * cl.Hs * 9 * cl.Cs * cl.Cb, sizeof(T) * (double)n * cl.Hs * cl.Hs * (cl.Cs + cl.Cb));
  launch_conv3_fwd<T>(a, c->st);
}

// pass0: dropout pass id of the first processed segment (real 0, fake 1, fake through the updated D 2);
// step_add: 1 before D's update of this iteration, 0 after it (the iteration number is D's step count + step_add)
template <typename T>
void paper_d_forward(gan_ctx* c, int n, Cost cost, bool update_running, int pass0, int step_add, const float* real = nullptr) {
  Net& D = c->D;
  const int seg_first = segments_of(cost).first, nseg = segments_of(cost).count;
  const gan_config& f = c->cfg;
  const ConvLayer& c1 = D.conv[0];
  image_conv_call<T>(c, c1, c->xd, real, c->dact[0], false, seg_first, nseg, n);
  if (f.dropout_p > 0.f) {
    PointArgs a = point_args(c, c->dact[0], c1.cs_real, c1.Cs, c1.Hs * c1.Hs, seg_first, nseg, n);
    with_dropout(c, a, 1, pass0, step_add);
    Scope s(c, "bias_act_dropout", 0, 2.0 * n * nseg * c1.Hs * c1.Hs * c1.cs_real * sizeof(T));
    launch_point_fwd<T>(a, c->st);
  }
  const int nl = (int)D.conv.size();
  const HeadArgs head = head_args(c, n, cost);
  for (int j = 1; j < nl; ++j) {
    const ConvLayer& cl = D.conv[j];
    conv_call<T>(c, "gemm_down", MODE_DOWN, EPI_NONE, c->dact[j - 1], layer_weights(c, D, cl, false), c->dpre[j], nullptr, cl.Cb,
                 cl.Cs, 2 * cl.Hs, cl.Hs, seg_first, nseg, n);
    PointArgs a = point_args(c, c->dpre[j], cl.cs_real, cl.Cs, cl.Hs * cl.Hs, seg_first, nseg, n);
    a.bias = D.theta + cl.bias; a.pstride = D.P; a.slope = f.leaky_slope;
    with_dropout(c, a, j + 1, pass0, step_add);
    { Scope s(c, "bias_act_dropout", 0, 2.0 * n * nseg * cl.Hs * cl.Hs * cl.cs_real * sizeof(T)); launch_point_fwd<T>(a, c->st); }
    bn_forward_direct<T>(c, norm_args<T>(c, D, cl.Cs, cl.Hs * cl.Hs, cl.gamma, cl.beta, cl.rs, c->d_mean[j], c->d_var[j], c->d_rstd[j],
                                         c->d_sums[j], seg_first, nseg, n, 1.f),
                         cl.cs_real, c->dpre[j], c->dact[j], f.bn_eps, update_running, j == nl - 1 ? &head : nullptr);
  }
}

template <typename T>
void paper_d_backward(gan_ctx* c, int n, Cost cost, bool param_grads, bool to_image, const float* real = nullptr) {
  Net& D = c->D;
  const int seg_first = segments_of(cost).first, nseg = segments_of(cost).count;
  const gan_config& f = c->cfg;
  const int nl = (int)D.conv.size();
  {
    Scope s(c, "head_bwd", 0, sizeof(T) * (double)n * nseg * D.K * (param_grads ? 2 : 1));
    launch_head_bwd<T>(head_args(c, n, cost), param_grads, c->st);
  }
  for (int j = nl - 1; j >= 1; --j) {
    const ConvLayer& cl = D.conv[j];
    NormArgs na = norm_args<T>(c, D, cl.Cs, cl.Hs * cl.Hs, cl.gamma, cl.beta, cl.rs, c->d_mean[j], c->d_var[j], c->d_rstd[j],
                               c->d_sums[j], seg_first, nseg, n, 1.f);
    na.eps = f.bn_eps;
    na.pre_act = 1; na.pre_slope = f.leaky_slope; na.pre_drop = f.dropout_p > 0.f; na.pre_scale = dropout_scale(c);
    bn_backward<T>(c, na, c->dpre[j], c->bufA, c->bufB, param_grads);         // -> gradient w.r.t. the convolution's output
    if (param_grads) {
      const PointArgs a = point_args(c, c->bufB, cl.cs_real, cl.Cs, cl.Hs * cl.Hs, seg_first, nseg, n);
      launch_col_sum<T>(a, D.g + cl.bias, D.P, c->st);
      wgrad_call<T>(c, c->dact[j - 1], c->bufB, D.g + cl.w, D.P, cl.Cb, cl.Cs, cl.Hs, 16, nseg, n);
    }
    const int first = f.dropout_p > 0.f ? EPI_DROP_BWD : EPI_ACT_BWD;         // the first block's LeakyReLU and dropout
    conv_call<T>(c, "gemm_up", MODE_UP, j == 1 ? first : EPI_NONE, c->bufB, layer_weights(c, D, cl, true), c->bufA,
                 j == 1 ? c->dact[0] : nullptr, cl.Cs, cl.Cb, cl.Hs, cl.Hs, seg_first, nseg, n);
  }
  const ConvLayer& c1 = D.conv[0];
  if (param_grads) {
    image_wgrad_call<T>(c, D, c1, c->xd, real, c->bufA, seg_first, nseg, n);
  }
  if (to_image) up_img_call<T>(c, D, c1, c->bufA, c->dimg, c->xd, 2, 1, n);
}

template <typename T>
void paper_g_backward(gan_ctx* c, int n) {
  Net& G = c->G;
  const gan_config& f = c->cfg;
  const int nl = (int)G.conv.size();
  const ConvLayer& last = G.conv[nl - 1];
  const T* dlast = (const T*)c->dimg + (long long)n * last.Hs * last.Hs * last.Cb;
  {
    Conv3Args a;
    memset(&a, 0, sizeof(a));
    a.dout = c->dimg; a.din = c->bufB; a.w = G.theta + last.w; a.w_stride = G.P;
    a.offs = c->rb.offs; a.sample_model = c->rb.sample_model; a.L = c->L; a.n = n; a.H = last.Hs; a.Cin = last.Cs; a.CO = last.Cb;
    a.out_seg = 1; a.seg_samples = n;
    paper_last_norm(c, a);
    { Scope s(c, "conv3_img_wgrad", 2.0 * n * last.Hs * last.Hs * 9 * last.Cs * last.Cb, sizeof(T) * (double)n * last.Hs * last.Hs * (last.Cs + last.Cb));
      launch_conv3_wgrad<T>(a, c->c3_part, G.g + last.w, G.P, c->st); }
    ImgBiasArgs b;
    b.img = dlast; b.partial = c->bias_partial; b.dbias = G.g + last.bias; b.pstride = G.P; b.offs = c->rb.offs;
    b.L = c->L; b.CB = last.Cb; b.HW = last.Hs * last.Hs;
    launch_img_bias_grad<T>(b, c->st);
    // the data gradient twice, for the sums of BatchNorm's backward pass and for its result (bufB)
    const ConvLayer& cl = G.conv[nl - 2];
    NormArgs na = norm_args<T>(c, G, cl.Cb, 4 * cl.Hs * cl.Hs, cl.gamma, cl.beta, cl.rs, c->g_mean[nl - 1], c->g_var[nl - 1], c->g_rstd[nl - 1],
                               c->g_sums[nl - 1], 0, 1, n, f.leaky_slope);
    na.param_grads = 1; na.red_tiles = c->NB;
    a.bn_part = c->stat_partial;
    const double flops = 2.0 * n * last.Hs * last.Hs * 9 * last.Cs * last.Cb, elems = (double)n * last.Hs * last.Hs;
    {
      Scope s(c, "conv3_img_dgrad_sums", flops, sizeof(T) * elems * (last.Cs + last.Cb));
      launch_conv3_dgrad<T>(a, c->st);
      launch_bn_bwd_final(na, c->rb.offs, n, c->stat_partial, c->st);
    }
    a.bn_sums = c->g_sums[nl - 1];
    Scope s(c, "conv3_img_dgrad", flops, sizeof(T) * elems * (2 * last.Cs + last.Cb));
    launch_conv3_dgrad<T>(a, c->st);
  }
  for (int i = nl - 2; i >= 0; --i) {
    const ConvLayer& cl = G.conv[i];
    NormArgs na = norm_args<T>(c, G, cl.Cb, 4 * cl.Hs * cl.Hs, cl.gamma, cl.beta, cl.rs, c->g_mean[i + 1], c->g_var[i + 1],
                               c->g_rstd[i + 1], c->g_sums[i + 1], 0, 1, n, f.leaky_slope);
    if (i < nl - 2) bn_backward<T>(c, na, c->gpre[i + 1], c->bufA, c->bufB, true);
    const long long per = (long long)16 * cl.Cb * cl.Cs;
    wgrad_call<T>(c, c->bufB, c->gact[i], c->dw4, per, cl.Cb, cl.Cs, cl.Hs, 16, 1, n);
    launch_dw4_to_dw3(c->dw4, G.g + cl.w, c->L, cl.Cb, cl.Cs, c->st, per, G.P);
    conv_call<T>(c, "gemm_down", MODE_DOWN, EPI_NONE, c->bufB, layer_weights(c, G, cl, false), c->bufA, nullptr, cl.Cb, cl.Cs,
                 2 * cl.Hs, cl.Hs, 0, 1, n);
  }
  NormArgs na = norm_args<T>(c, G, G.C0, G.h0 * G.h0, G.fc_gamma, G.fc_beta, G.fc_rs, c->g_mean[0], c->g_var[0], c->g_rstd[0],
                             c->g_sums[0], 0, 1, n, 1.f);
  na.eps = f.bn_eps_first;
  na.pre_act = 1; na.pre_slope = 0.f; na.pre_scale = 1.f;                     // ReLU derivative from the stored output
  bn_backward<T>(c, na, c->gpre[0], c->bufA, c->bufB, true);
  const PointArgs a = point_args(c, c->bufB, G.J, G.J, 1, 0, 1, n);
  launch_col_sum<T>(a, G.g + G.fc_bias, G.P, c->st);
  wgrad_call<T>(c, c->bufB, c->zin, G.g + G.fc_w, G.P, G.J, G.Kp, 1, 1, 1, n);
}

template <typename T>
void paper_adam_g(gan_ctx* c) {
  Net& G = c->G;
  AdamArgs a = {};
  a.theta = G.theta; a.m = G.m; a.v = G.v; a.g = G.g; a.shadow = c->bf16 ? G.shadow_u : nullptr; a.shadow_t = nullptr;
  a.P = G.P; a.L = c->L; a.counts = c->rb.counts; a.t = G.t; a.bc = G.bc;
  a.lr = c->cfg.lr; a.beta1 = c->cfg.beta1; a.beta2 = c->cfg.beta2; a.eps = c->cfg.adam_eps;
  {
    Scope s(c, "adam", 0, (double)c->L * G.P * (28.0 + (c->bf16 ? 2.0 : 0.0)));
    launch_adam<T>(a, c->st);
  }
  paper_rebuild_w4<T>(c);
}

// The planned update of one network: every convolution weight the GEMM engine also reads in "down" form is a tiled
// region (the update writes that transposed copy too), in layer order; the rest of the block is the gaps.
template <typename T>
AdamArgs adam_args(gan_ctx* c, Net& net) {
  AdamArgs a = {};
  a.theta = net.theta; a.m = net.m; a.v = net.v; a.g = net.g; a.shadow = c->bf16 ? net.shadow_u : nullptr;
  a.P = net.P; a.L = c->L; a.counts = c->rb.counts; a.t = net.t; a.bc = net.bc;
  a.lr = c->cfg.lr; a.beta1 = c->cfg.beta1; a.beta2 = c->cfg.beta2; a.eps = c->cfg.adam_eps;
  a.shadow_t = net.shadow_d; a.split_u = net.split_u; a.split_d = net.split_d; a.plane = net.PS;
  for (size_t i = 0; i < net.conv.size(); ++i) {
    if (!on_engine(c, net, i)) continue;
    const ConvLayer& cl = net.conv[i];
    a.reg_w[a.nregions] = cl.w; a.reg_part[a.nregions] = cl.part; a.reg_cb[a.nregions] = cl.Cb; a.reg_cs[a.nregions] = cl.Cs;
    a.reg_cb_real[a.nregions] = c->paper ? cl.cb_real : cl.Cb; a.reg_cs_real[a.nregions] = c->paper ? cl.cs_real : cl.Cs;
    ++a.nregions;
  }
  a.k3 = c->paper;                                 // (D: its k3 filters are held as k4 ones)
  adam_plan(a);
  return a;
}
// bytes one update moves per element: g, theta, m, v in; theta, m, v out; the storage-type copy (tiled regions: and the transposed
// one; fp32: both as three planes, or with few rows a model the transposed one alone)
inline double adam_bytes_per_element(const gan_ctx* c) { return 28.0 + (c->bf16 ? 2.0 : 0.0); }
// ... of one region: what is moved of it, and, where the update adds up row splits, these and their sum in place of the gradient
double adam_region_bytes(const gan_ctx* c, const AdamArgs& a, int region, const AdamSplits& sp) {
  const double per = adam_bytes_per_element(c) + (c->bf16 ? 2.0 : c->presplit ? 12.0 : 4.0) + (sp.n > 1 ? 4.0 * sp.n : 0.0);
  return (double)c->L * (a.k3 ? 9 : 16) * a.reg_cb_real[region] * a.reg_cs_real[region] * per;
}
template <typename T>
void adam_region_call(gan_ctx* c, const AdamArgs& a, int region, hipStream_t st, const AdamSplits& sp) {
  double bytes = 0;
  for (int r = 0; r < a.nregions; ++r)
    if (region < 0 || r == region) bytes += adam_region_bytes(c, a, r, sp);
  Scope s(c, "adam", 0, bytes, nullptr, st);
  launch_adam_region<T>(a, region, sp, st);
}
// what is left of a planned update once the regions are done (or enqueued beside): the gaps, the operand of the image-side layer, and
// the region that a backward pass has left (AdamTail)
template <typename T>
void adam_rest_call(gan_ctx* c, Net& net, const AdamArgs& a, const AdamTail& tail = {}) {
  double elems = 0;
  for (int r = 0; r < a.ngaps; ++r) elems += (double)(a.gap_hi[r] - a.gap_lo[r]);
  const bool first = &net == &c->D;
  const ConvLayer& cl = first ? net.conv.front() : net.conv.back();
  AdamImage im;
  im.w = cl.w; im.packed = first ? c->wpD : c->wpG; im.add = first && cl.CBT > cl.Cb ? c->addD : nullptr;
  im.CB = cl.Cb; im.CBT = cl.CBT; im.Cs = cl.Cs; im.P = image_values(cl.Cb); im.tables = c->labels > 0 ? c->labels : c->L;
  Scope s(c, "adam", 0, (double)c->L * elems * adam_bytes_per_element(c) + (tail.region >= 0 ? adam_region_bytes(c, a, tail.region, tail.splits) : 0));
  launch_adam_rest<T>(a, im, tail.region, tail.splits, c->st);
}
// the whole update on the caller's stream
template <typename T>
void adam_call(gan_ctx* c, Net& net) {
  const AdamArgs a = adam_args<T>(c, net);
  adam_region_call<T>(c, a, -1, c->st);
  adam_rest_call<T>(c, net, a);
}

template <typename T>
void route_and_stage(gan_ctx* c, const int32_t* label_ids, const float* noise, int n) {
  Scope s(c, "stage", 0, (double)n * c->cfg.z_dim * (4.0 + sizeof(T)));
  launch_route_stage<T>(label_ids, noise, n, c->L, c->cfg.n_labels, c->cfg.z_dim, c->cfg.cond_g, c->G.Kp, c->geoms, c->rb, (T*)c->zin, c->st);
}

template <typename T>
void paper_train_step(gan_ctx* c, const int32_t* label_ids, const float* noise, const float* real, int n) {
  if (c->shadows_dirty) refresh_shadows(c);
  route_and_stage<T>(c, label_ids, noise, n);
  paper_g_forward<T>(c, n, false, true);                               // fake = G(z)
  paper_d_forward<T>(c, n, COST_D, true, 0, 1, real);                   // D(real), D(fake): dropout passes 0 and 1
  paper_d_backward<T>(c, n, COST_D, true, false, real);                 // Eq. 3
  adam_call<T>(c, c->D);
  paper_d_forward<T>(c, n, COST_G, true, 2, 0);                        // updated D on the same fake batch: pass 2
  paper_d_backward<T>(c, n, COST_G, false, true);                      // Eq. 4 (negated: minimised)
  paper_g_backward<T>(c, n);
  paper_adam_g<T>(c);
}

template <typename T>
void train_step(gan_ctx* c, const int32_t* label_ids, const float* noise, const float* real, int n) {
  if (c->paper) return paper_train_step<T>(c, label_ids, noise, real, n);
  if (c->shadows_dirty) refresh_shadows(c);
  route_and_stage<T>(c, label_ids, noise, n);
  g_forward<T>(c, n, false, true);                 // fake = G(z)
  d_forward<T>(c, n, COST_D, true, real);              // D(real), D(fake): separate batch statistics per segment
  c->order_next = 0;
  {
    const AdamArgs aD = adam_args<T>(c, c->D);
    AdamTail tail;
    d_backward<T>(c, n, COST_D, true, false, real, &aD, &tail); // Eq. 3; weight gradients and the convolutions' updates beside the chain
    adam_rest_call<T>(c, c->D, aD, tail);
    order_after(c, c->st, side_stream(c));
  }
  d_forward<T>(c, n, COST_G, true);                // updated D on the same fake batch
  d_backward<T>(c, n, COST_G, false, true);        // Eq. 4 (negated: minimised); only data gradients: theta_D is not G's to move
  {
    const AdamArgs aG = adam_args<T>(c, c->G);
    AdamTail tail;
    g_backward<T>(c, n, &aG, &tail);
    adam_rest_call<T>(c, c->G, aG, tail);
    order_after(c, c->st, side_stream(c));
  }
}

bool check_config_paper(const gan_config* f, std::string& why) {
  if (f->n_g < 2 || f->n_g > GAN_MAX_LAYERS || f->n_d < 2 || f->n_d > GAN_MAX_LAYERS) { why = "n_g, n_d must be in [2, 8]"; return false; }
  if (f->img_c < 1 || f->img_c > 4) { why = "img_c must be in [1, 4]"; return false; }
  if (f->cond_g != 0 || f->cond_d != 0) { why = "the networks of the tables are unconditional: cond_g = cond_d = 0"; return false; }
  if ((f->g_h0 << (f->n_g - 1)) != f->img_hw) { why = "img_hw must equal g_h0 * 2^(n_g - 1)"; return false; }
  if (((f->img_hw >> f->n_d) << f->n_d) != f->img_hw || (f->img_hw >> f->n_d) < 1) { why = "img_hw must be divisible by 2^n_d"; return false; }
  for (int i = 0; i < f->n_g; ++i) if (f->g_ch[i] <= 0 || f->g_ch[i] % 64 || f->g_ch[i] > 1024) { why = "g_ch must be multiples of 64, at most 1024"; return false; }
  for (int i = 0; i < f->n_d; ++i) if (f->d_ch[i] <= 0 || f->d_ch[i] > 1024) { why = "d_ch must be in [1, 1024]"; return false; }
  if (f->g_ch[f->n_g - 1] != 64 && f->g_ch[f->n_g - 1] != 128) { why = "the last generator block must have 64 or 128 channels"; return false; }
  if (f->d_ch[0] > 128) { why = "the first discriminator block supports at most 128 channels"; return false; }
  if ((f->g_ch[0] * f->g_h0 * f->g_h0) % 128) { why = "g_ch[0]*g_h0^2 must be a multiple of 128"; return false; }
  if (f->z_dim < 1 || f->max_total_batch < 1) { why = "bad z_dim / max_total_batch"; return false; }
  if (!(f->dropout_p >= 0.f && f->dropout_p < 1.f) || !(f->bn_eps_first > 0.f) || !(f->bn_eps > 0.f)) { why = "bad dropout_p / epsilon"; return false; }
  return true;
}

bool check_config(const gan_config* f, std::string& why) {
  if (f->n_models < 1 || f->n_labels < 1) { why = "n_models and n_labels must be positive"; return false; }
  if (f->n_models != 1 && f->n_models != f->n_labels) { why = "n_models must be 1 or n_labels"; return false; }
  if (f->precision != GAN_FP32 && f->precision != GAN_BF16_FP32MASTER) { why = "unknown precision"; return false; }
  if (f->family == GAN_FAMILY_PAPER) return check_config_paper(f, why);
  if (f->family != GAN_FAMILY_STRIDED) { why = "unknown network family"; return false; }
  if (f->n_g < 2 || f->n_g > GAN_MAX_LAYERS || f->n_d < 2 || f->n_d > GAN_MAX_LAYERS) { why = "n_g, n_d must be in [2, 8]"; return false; }
  if (f->img_c < 1 || f->img_c > 4) { why = "img_c must be in [1, 4]"; return false; }
  if ((f->g_h0 << f->n_g) != f->img_hw) { why = "img_hw must equal g_h0 * 2^n_g"; return false; }
  if (((f->img_hw >> f->n_d) << f->n_d) != f->img_hw || (f->img_hw >> f->n_d) < 1) { why = "img_hw must be divisible by 2^n_d"; return false; }
  for (int i = 0; i < f->n_g; ++i) if (f->g_ch[i] <= 0 || f->g_ch[i] % 64) { why = "g_ch must be multiples of 64"; return false; }
  for (int i = 0; i < f->n_d; ++i) if (f->d_ch[i] <= 0 || f->d_ch[i] % 64) { why = "d_ch must be multiples of 64"; return false; }
  for (int i = 0; i < f->n_g; ++i) if (f->g_ch[i] > 1024) { why = "at most 1024 channels per layer"; return false; }
  for (int i = 0; i < f->n_d; ++i) if (f->d_ch[i] > 1024) { why = "at most 1024 channels per layer"; return false; }
  if (f->g_ch[f->n_g - 1] > 128 || f->d_ch[0] > 128) { why = "the layers next to the image support 64 or 128 feature channels"; return false; }
  if ((f->g_ch[0] * f->g_h0 * f->g_h0) % 128) { why = "g_ch[0]*g_h0^2 must be a multiple of 128"; return false; }
  if (f->z_dim < 1 || f->cond_g < 0 || f->cond_d < 0 || f->max_total_batch < 1) { why = "bad z_dim / cond / max_total_batch"; return false; }
  if (f->cond_g > f->n_labels || (f->cond_d != 0 && f->cond_d < f->n_labels)) { why = "cond_d must cover every label"; return false; }
  if (f->precision != GAN_FP32 && f->precision != GAN_BF16_FP32MASTER) { why = "unknown precision"; return false; }
  return true;
}

}  // namespace

// ---------------------------------------------------------------------------------------------------------
extern "C" {

gan_status gan_create(const gan_config* cfg, void* hip_stream, gan_ctx** out) {
  if (!cfg || !out || cfg->struct_size != sizeof(gan_config)) return GAN_E_ARG;
  std::string why;
  if (!check_config(cfg, why)) return GAN_E_SHAPE;
  gan_ctx* c = new gan_ctx();
  c->cfg = *cfg;
  c->st = (hipStream_t)hip_stream;
  c->bf16 = cfg->precision == GAN_BF16_FP32MASTER;
  c->L = cfg->n_models; c->NB = cfg->max_total_batch;
  c->geoms.n = 0;
  c->paper = cfg->family == GAN_FAMILY_PAPER;
  if (c->paper) build_layout_paper(c); else build_layout(c);
  c->presplit = !c->bf16 && presplit_pays(c);
  const int L = c->L, NB = c->NB;
  const size_t es = esize(c);
  bool ok = alloc_net(c, c->G) && alloc_net(c, c->D);
  // geometries used by any launch: (rows per sample, tile height) of every GEMM's row space
  {
    auto reg = [&](int rps, int tile_rows) { if (geom_id(c, rps, tile_rows) < 0) ok = false; };
    auto reg_gemm = [&](int mode, int n_out, int rps, int nseg) { reg(rps, conv_tile_rows((int)es, layer_tile(c, mode, n_out, rps, nseg))); };
    reg_gemm(MODE_DENSE, c->G.J, 1, 1);                                         // G's linear layer
    for (size_t i = 0; i + 1 < c->G.conv.size(); ++i) {
      const ConvLayer& cl = c->G.conv[i];
      reg_gemm(MODE_UP, cl.Cb, cl.Hs * cl.Hs, 1);                               // forward
      reg_gemm(MODE_DOWN, cl.Cs, cl.Hs * cl.Hs, 1);                             // data gradient
    }
    c->img_tiles = image_tiles((int)es, NB, L);
    if (geom_id(c, 1, c->img_tiles.most, c->img_tiles.parts) < 0) ok = false;   // the weight gradients of the image-side layers
    for (int nseg = 1; nseg <= 2; ++nseg) {                                     // D runs on one segment and on both
      for (size_t j = 1; j < c->D.conv.size(); ++j) {
        const ConvLayer& cl = c->D.conv[j];
        reg_gemm(MODE_DOWN, cl.Cs, cl.Hs * cl.Hs, nseg);                        // forward
        reg_gemm(MODE_UP, cl.Cb, cl.Hs * cl.Hs, nseg);                          // data gradient
      }
    }
    // row space of every BatchNorm, in the row blocks of its backward reduction
    auto reg_bn = [&](int rps) { reg(rps, red_rows(c, rps)); };
    reg_bn(c->G.h0 * c->G.h0);
    for (size_t i = 0; i + 1 < c->G.conv.size(); ++i) reg_bn(4 * c->G.conv[i].Hs * c->G.conv[i].Hs);
    for (size_t j = 1; j < c->D.conv.size(); ++j) reg_bn(c->D.conv[j].Hs * c->D.conv[j].Hs);
  }
  // two sets of routing buffers: the training step's (what gan_get_losses / gan_get_routing report) and one for
  // gan_generate / gan_sample, so that generating between a step and its queries changes nothing they return
  RouteBuffers& rb = c->rb;
  for (RouteBuffers* r : {&c->rb, &c->rb_gen}) {
    ok = ok && dev_alloc(c, (void**)&r->cnt, (size_t)ROUTE_WAVES * L * 4) && dev_alloc(c, (void**)&r->counts, (size_t)L * 4) &&
         dev_alloc(c, (void**)&r->offs, (size_t)(L + 1) * 4) && dev_alloc(c, (void**)&r->perm, (size_t)NB * 4) &&
         dev_alloc(c, (void**)&r->sample_model, (size_t)NB * 4) && dev_alloc(c, (void**)&r->sample_slot, (size_t)NB * 4) &&
         dev_alloc(c, (void**)&r->tpre, (size_t)MAX_GEOMS * (L + 1) * 4) && dev_alloc(c, (void**)&r->order, (size_t)L * 4);
    int mx = 1;
    for (int g = 0; g < c->geoms.n; ++g)
      mx = std::max(mx, c->geoms.parts[g] > 0 ? (int)image_tile_bound(c->img_tiles, NB, L) : ub_tiles(c, NB, c->geoms.rps[g], c->geoms.tile_rows[g]));
    r->tmodel_stride = mx;
    ok = ok && dev_alloc(c, (void**)&r->tmodel, (size_t)c->geoms.n * mx * 4);
  }
  ok = ok && dev_alloc(c, (void**)&rb.flags, 16);
  c->rb_gen.flags = rb.flags;                  // one sticky out-of-range flag for both
  const long long img_elems = (long long)cfg->img_hw * cfg->img_hw * cfg->img_c;
  long long max_act = img_elems;
  ok = ok && dev_alloc(c, &c->zin, (size_t)NB * c->G.Kp * es) && dev_alloc(c, &c->xd, (size_t)2 * NB * img_elems * es) &&
       dev_alloc(c, &c->dimg, (size_t)2 * NB * img_elems * es);
  // G activations (one segment)
  {
    const int nl = (int)c->G.conv.size();
    c->gpre.resize(nl); c->gact.resize(nl); c->g_mean.resize(nl); c->g_var.resize(nl); c->g_rstd.resize(nl); c->g_sums.resize(nl);
    for (int i = 0; i < nl && ok; ++i) {
      const long long e = i == 0 ? c->G.J : (long long)4 * c->G.conv[i - 1].Hs * c->G.conv[i - 1].Hs * c->G.conv[i - 1].Cb;
      const int C = i == 0 ? c->G.C0 : c->G.conv[i - 1].Cb;
      max_act = e > max_act ? e : max_act;
      ok = dev_alloc(c, &c->gpre[i], (size_t)NB * e * es) && dev_alloc(c, &c->gact[i], (size_t)NB * e * es) &&
           dev_alloc(c, (void**)&c->g_mean[i], (size_t)2 * L * C * 4) && dev_alloc(c, (void**)&c->g_var[i], (size_t)2 * L * C * 4) &&
           dev_alloc(c, (void**)&c->g_rstd[i], (size_t)2 * L * C * 4) && dev_alloc(c, (void**)&c->g_sums[i], (size_t)4 * L * C * 4);
    }
  }
  // D activations (two segments: real, fake)
  {
    const int nl = (int)c->D.conv.size();
    c->dpre.assign(nl, nullptr); c->dact.assign(nl, nullptr);
    c->d_mean.assign(nl, nullptr); c->d_var.assign(nl, nullptr); c->d_rstd.assign(nl, nullptr); c->d_sums.assign(nl, nullptr);
    for (int j = 0; j < nl && ok; ++j) {
      const ConvLayer& cl = c->D.conv[j];
      const long long e = (long long)cl.Hs * cl.Hs * cl.Cs;
      max_act = e > max_act ? e : max_act;
      ok = dev_alloc(c, &c->dact[j], (size_t)2 * NB * e * es);
      if (j > 0)
        ok = ok && dev_alloc(c, &c->dpre[j], (size_t)2 * NB * e * es) && dev_alloc(c, (void**)&c->d_mean[j], (size_t)2 * L * cl.Cs * 4) &&
             dev_alloc(c, (void**)&c->d_var[j], (size_t)2 * L * cl.Cs * 4) && dev_alloc(c, (void**)&c->d_rstd[j], (size_t)2 * L * cl.Cs * 4) &&
             dev_alloc(c, (void**)&c->d_sums[j], (size_t)4 * L * cl.Cs * 4);
    }
  }
  {
    // column sums left by the GEMM in front of every BatchNorm: phases x segments x tiles x sub-tiles (at most 4) x columns x 2
    size_t mx = (size_t)4 * ub_tiles(c, NB, 1, conv_tile_rows((int)es, layer_tile(c, MODE_DENSE, c->G.J, 1, 1))) * c->G.J;
    for (size_t i = 0; i + 1 < c->G.conv.size(); ++i) {
      const ConvLayer& cl = c->G.conv[i];
      const size_t v = (size_t)4 * 4 * ub_tiles(c, NB, cl.Hs * cl.Hs, conv_tile_rows((int)es, layer_tile(c, MODE_UP, cl.Cb, cl.Hs * cl.Hs, 1))) * cl.Cb;
      mx = v > mx ? v : mx;
    }
    for (size_t j = 1; j < c->D.conv.size(); ++j) {
      const ConvLayer& cl = c->D.conv[j];
      for (int nseg = 1; nseg <= 2; ++nseg) {
        const size_t v = (size_t)4 * nseg * ub_tiles(c, NB, cl.Hs * cl.Hs, conv_tile_rows((int)es, layer_tile(c, MODE_DOWN, cl.Cs, cl.Hs * cl.Hs, nseg))) * cl.Cs;
        mx = v > mx ? v : mx;
      }
    }
    // and the BatchNorm backward reduction: segments x row blocks x channels x 2
    {
      const auto red_tiles = [&](int rps) { return ub_tiles(c, NB, rps, red_rows(c, rps)); };
      size_t v = (size_t)red_tiles(c->G.h0 * c->G.h0) * c->G.C0;
      mx = v > mx ? v : mx;
      for (size_t i = 0; i + 1 < c->G.conv.size(); ++i) {
        const ConvLayer& cl = c->G.conv[i];
        v = (size_t)red_tiles(4 * cl.Hs * cl.Hs) * cl.Cb;
        mx = v > mx ? v : mx;
      }
      for (size_t j = 1; j < c->D.conv.size(); ++j) {
        const ConvLayer& cl = c->D.conv[j];
        v = (size_t)2 * red_tiles(cl.Hs * cl.Hs) * cl.Cs;
        mx = v > mx ? v : mx;
      }
    }
    if (c->paper) mx = std::max(mx, (size_t)NB * c->G.conv.back().Cs);        // the same from G's last layer: samples x channels x 2
    ok = ok && dev_alloc(c, (void**)&c->stat_partial, mx * 2 * 4);
  }
  ok = ok && dev_alloc(c, &c->bufA, (size_t)2 * NB * max_act * es) && dev_alloc(c, &c->bufB, (size_t)2 * NB * max_act * es) &&
       dev_alloc(c, (void**)&c->logits, (size_t)2 * NB * 4) && dev_alloc(c, (void**)&c->dlogits, (size_t)2 * NB * 4) &&
       dev_alloc(c, (void**)&c->loss_d, (size_t)L * 4) && dev_alloc(c, (void**)&c->loss_g, (size_t)L * 4);
  {
    const ConvLayer& c1 = c->D.conv[0];
    const ConvLayer& gl = c->G.conv.back();
    if (L == 1 && cfg->cond_d > 1) {
      c->labels = cfg->cond_d;
      ok = ok && dev_alloc(c, (void**)&c->label_sums, (size_t)c->labels * 9 * c1.Cs * 4) && dev_alloc(c, (void**)&c->class_part, (size_t)2 * NB * 9 * c1.Cs * 4);
    }
    const size_t d1 = (size_t)16 * image_values(c1.Cb) * c1.Cs, g1 = c->paper ? 0 : (size_t)16 * image_values(gl.Cb) * gl.Cs, tiles = image_tile_bound(c->img_tiles, NB, L),
                 part = std::max(image_part_floats((int)es, c1.Cb, c1.Hs, c1.Cs, 2, c->img_tiles, tiles), c->paper ? 0 : image_part_floats((int)es, gl.Cb, gl.Hs, gl.Cs, 1, c->img_tiles, tiles));
    ok = ok && dev_alloc(c, &c->wpD, (size_t)L * d1 * es) && dev_alloc(c, &c->wpG, (size_t)L * g1 * es) &&
         dev_alloc(c, (void**)&c->addD, (size_t)(c->labels > 0 ? c->labels : L) * 9 * c1.Cs * 4) &&
         dev_alloc(c, (void**)&c->img_part, part * 4) && dev_alloc(c, (void**)&c->img_sums, tiles * 4 * 4) &&
         dev_alloc(c, (void**)&c->bias_partial, c->paper ? (size_t)L * img_bias_chunks(L) * 4 * 4 : 0);
  }
  {
    // partial blocks of the weight gradients that are split over rows (few models only)
    size_t need = 0;
    auto want = [&](int Cb, int Cs, int ntaps, int Hs, int nseg) {      // as the training step calls wgrad_call
      const int ks = wgrad_ksplit(c, Cb, Cs, ntaps, Hs, nseg);
      if (ks > 1) need = std::max(need, (size_t)ks * L * ntaps * Cb * Cs * 4);
    };
    for (size_t j = 1; j < c->D.conv.size(); ++j) want(c->D.conv[j].Cb, c->D.conv[j].Cs, 16, c->D.conv[j].Hs, 2);
    for (size_t i = 0; i + 1 < c->G.conv.size(); ++i) want(c->G.conv[i].Cb, c->G.conv[i].Cs, 16, c->G.conv[i].Hs, 1);
    want(c->G.J, c->G.Kp, 1, 1, 1);
    c->wg_part = nullptr;
    if (need) ok = ok && dev_alloc(c, (void**)&c->wg_part, need);
    if (c->paper) {
      // G's summed-tap k4 weights (both layouts), the k4 weight gradient of one block, the last conv's row-split partials
      size_t per = 0;
      for (size_t i = 0; i + 1 < c->G.conv.size(); ++i) per = std::max(per, (size_t)16 * c->G.conv[i].Cb * c->G.conv[i].Cs);
      const ConvLayer& last = c->G.conv.back();
      ok = ok && dev_alloc(c, &c->G.w4u, (size_t)L * c->G.P4 * es) && (!c->bf16 || dev_alloc(c, &c->G.w4d, (size_t)L * c->G.P4 * es)) &&
           dev_alloc(c, (void**)&c->dw4, (size_t)L * per * 4) &&
           dev_alloc(c, (void**)&c->c3_part, (size_t)conv3_wgrad_splits(L) * L * 9 * last.Cb * last.Cs * 4);
    }
    // the linear head's weight gradient: blocks of 1024 columns per model, rows split when that leaves the chip idle.  A block is a chain of waits for its
    // rows; 512 and 1024 blocks: twenty 32x32 pairs in fp32 47 and 36 us, ten 28x28 pairs 37 and 28, eight 64x64 pairs in bf16 27 and 19 (2048: 32, 26, 21).
    c->head_rsplit = (int)std::min<long long>(std::max<long long>(1024 / ((long long)L * ((c->D.K + 1023) / 1024)), 1), 64);
    if (c->head_rsplit > 1) ok = ok && dev_alloc(c, (void**)&c->head_part, (size_t)c->head_rsplit * L * (c->D.K + 4) * 4);
  }
  {
    // the GEMM loaders address one segment of any activation tensor with 32-bit byte offsets.  Beside those, a bound that no tensor asks for: the image-side
    // layers count with 16 columns an image channel and 9 a label of one pair, in lines of 64, as when they were patch matrices.  A configuration
    // takes the batches that it took then.
    const ConvLayer& c1 = c->D.conv[0];
    const ConvLayer& gl = c->G.conv.back();
    const long long lim = 1LL << 31, slots = cfg->cond_d > 0 && L == 1 ? cfg->cond_d : 1;
    const long long big = std::max({(long long)NB * max_act * (long long)es, (long long)NB * c1.Hs * c1.Hs * round_up(16 * c1.Cb + 9 * slots + 1, 64) * (long long)es,
                                    c->paper ? 0LL : (long long)NB * gl.Hs * gl.Hs * round_up(16 * gl.Cb, 64) * (long long)es});
    if (big >= lim) {
      for (void* p : c->allocs) (void)hipFree(p);
      delete c;
      return GAN_E_SHAPE;
    }
  }
  if (!ok) {
    for (void* p : c->allocs) (void)hipFree(p);
    delete c;
    return GAN_E_OOM;
  }
  hipMemsetAsync(rb.flags, 0, 16, c->st);
  hipMemsetAsync(rb.counts, 0, (size_t)L * 4, c->st);
  hipMemsetAsync(rb.offs, 0, (size_t)(L + 1) * 4, c->st);
  hipMemsetAsync(c->loss_d, 0, (size_t)L * 4, c->st);
  hipMemsetAsync(c->loss_g, 0, (size_t)L * 4, c->st);
  bool init_ok = true;
  if (c->paper) { hipStreamSynchronize(c->st); init_ok = builtin_init_paper(c); }
  else builtin_init(c);
  if (!init_ok || hipStreamSynchronize(c->st) != hipSuccess || hipGetLastError() != hipSuccess) {
    for (void* p : c->allocs) (void)hipFree(p);
    delete c;
    return GAN_E_HIP;
  }
  if (hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking) != hipSuccess) {
    (void)hipGetLastError();
    c->side = nullptr;                         // everything then runs on the caller's stream
  }
  if (hipStreamCreateWithFlags(&c->cap, hipStreamNonBlocking) != hipSuccess) {
    (void)hipGetLastError();
    c->cap = nullptr;                          // no replayable steps
  }
  c->shadows_dirty = true;
  *out = c;
  return GAN_OK;
}

gan_status gan_destroy(gan_ctx* c) {
  if (!c) return GAN_E_ARG;
  (void)hipStreamSynchronize(c->st);
  if (c->side) { (void)hipStreamSynchronize(c->side); (void)hipStreamDestroy(c->side); }
  for (auto& g : c->graphs) (void)hipGraphExecDestroy(g.exec);
  if (c->cap) (void)hipStreamDestroy(c->cap);
  for (auto& e : c->order_events) hipEventDestroy(e);
  for (auto& e : c->prof_entries) { hipEventDestroy(e.e0); hipEventDestroy(e.e1); }
  for (auto& e : c->event_pool) hipEventDestroy(e);
  for (void* p : c->allocs) (void)hipFree(p);
  if (c->an_res) (void)hipHostFree(c->an_res);
  delete c;
  return GAN_OK;
}

const char* gan_last_error(const gan_ctx* c) { return c ? c->err.c_str() : "null context"; }

gan_status gan_train_step(gan_ctx* c, const int32_t* label_ids, const float* noise, const float* real_batch, int32_t n) {
  if (!c) return GAN_E_ARG;
  if (n < 0 || n > c->NB) return fail(c, GAN_E_ARG, "n out of range [0, max_total_batch]");
  if (n > 0 && (!label_ids || !noise || !real_batch)) return fail(c, GAN_E_ARG, "null input pointer");
  c->last_n = n;
  if (n == 0) {
    hipMemsetAsync(c->rb.counts, 0, (size_t)c->L * 4, c->st);
    hipMemsetAsync(c->rb.offs, 0, (size_t)(c->L + 1) * 4, c->st);
    hipMemsetAsync(c->loss_d, 0, (size_t)c->L * 4, c->st);
    hipMemsetAsync(c->loss_g, 0, (size_t)c->L * 4, c->st);
    return GAN_OK;
  }
  (void)take_launch_error();
  ++c->calls;
  if (c->graphs_on && c->cap && !c->prof) {
    if (c->shadows_dirty) refresh_shadows(c);          // host-side condition: outside anything that is replayed
    gan_ctx::StepGraph* hit = nullptr;
    for (auto& g : c->graphs)
      if (g.lab == label_ids && g.noise == noise && g.real == real_batch && g.n == n) hit = &g;
    bool repeat = false;
    for (auto& a : c->seen) repeat = repeat || (a.lab == label_ids && a.noise == noise && a.real == real_batch && a.n == n);
    if (!hit && !repeat) {
      if (c->seen.size() >= 8) c->seen.erase(c->seen.begin());
      c->seen.push_back({label_ids, noise, real_batch, n});
    }
    if (!hit && repeat) {
      // capture this step's launches (both streams: the second one joins through the ordering events) without running them
      hipStream_t user = c->st;
      hipGraph_t graph = nullptr;
      hipGraphExec_t exec = nullptr;
      bool ok = hipStreamBeginCapture(c->cap, hipStreamCaptureModeRelaxed) == hipSuccess;
      if (ok) {
        c->st = c->cap;
        if (c->bf16) train_step<bf16_t>(c, label_ids, noise, real_batch, n);
        else train_step<float>(c, label_ids, noise, real_batch, n);
        c->st = user;
        ok = hipStreamEndCapture(c->cap, &graph) == hipSuccess && graph != nullptr;
      }
      const char* refused = take_launch_error();
      if (refused) {
        if (graph) (void)hipGraphDestroy(graph);
        (void)hipGetLastError();
        return fail(c, GAN_E_SHAPE, refused);
      }
      ok = ok && hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) == hipSuccess;
      if (graph) (void)hipGraphDestroy(graph);
      if (ok) {
        if (c->graphs.size() >= 8) {                    // keep the eight most recently used
          size_t oldest = 0;
          for (size_t i = 1; i < c->graphs.size(); ++i)
            if (c->graphs[i].used < c->graphs[oldest].used) oldest = i;
          (void)hipGraphExecDestroy(c->graphs[oldest].exec);
          c->graphs.erase(c->graphs.begin() + oldest);
        }
        c->graphs.push_back({label_ids, noise, real_batch, n, exec, c->calls});
        hit = &c->graphs.back();
      } else {
        (void)hipGetLastError();
        c->graphs_on = false;                           // capture is not available here: plain launches from now on
      }
    }
    if (hit) {
      hit->used = c->calls;
      ++c->replays;
      if (hipGraphLaunch(hit->exec, c->st) != hipSuccess) return fail(c, GAN_E_HIP, "graph launch failed");
      return launch_status(c);
    }
  }
  if (c->bf16) train_step<bf16_t>(c, label_ids, noise, real_batch, n);
  else train_step<float>(c, label_ids, noise, real_batch, n);
  return launch_status(c);
}

gan_status gan_use_second_stream(gan_ctx* c, int32_t enable) {
  if (!c) return GAN_E_ARG;
  if (hipStreamSynchronize(c->st) != hipSuccess) return fail(c, GAN_E_HIP, "stream synchronisation failed");
  c->side_on = enable != 0 && c->side != nullptr;
  for (auto& g : c->graphs) (void)hipGraphExecDestroy(g.exec);      // captured with the other setting
  c->graphs.clear();
  c->seen.clear();
  return GAN_OK;
}

gan_status gan_graph_replays(const gan_ctx* c, int64_t* n) {
  if (!c || !n) return GAN_E_ARG;
  *n = (int64_t)c->replays;
  return GAN_OK;
}

gan_status gan_use_graphs(gan_ctx* c, int32_t enable) {
  if (!c) return GAN_E_ARG;
  c->graphs_on = enable != 0 && c->cap != nullptr;
  c->seen.clear();
  return GAN_OK;
}

gan_status gan_generate(gan_ctx* c, const int32_t* label_ids, const float* noise, int32_t n, float* out_images,
                        int32_t use_running_stats) {
  if (!c) return GAN_E_ARG;
  if (n < 0 || n > c->NB) return fail(c, GAN_E_ARG, "n out of range [0, max_total_batch]");
  if (n == 0) return GAN_OK;
  if (!label_ids || !noise || !out_images) return fail(c, GAN_E_ARG, "null pointer");
  if (c->shadows_dirty) refresh_shadows(c);
  (void)take_launch_error();
  const RouteBuffers train_rb = c->rb;         // the launch helpers read c->rb: point them at the generate set
  c->rb = c->rb_gen;
  if (c->bf16) {
    route_and_stage<bf16_t>(c, label_ids, noise, n);
    if (c->paper) paper_g_forward<bf16_t>(c, n, use_running_stats != 0, false, out_images);
    else g_forward<bf16_t>(c, n, use_running_stats != 0, false, out_images);
  } else {
    route_and_stage<float>(c, label_ids, noise, n);
    if (c->paper) paper_g_forward<float>(c, n, use_running_stats != 0, false, out_images);
    else g_forward<float>(c, n, use_running_stats != 0, false, out_images);
  }
  c->rb = train_rb;
  return launch_status(c);
}

gan_status gan_sample(gan_ctx* c, const double* prior, const float* u, const float* noise, int32_t n, float* out_images,
                      int32_t* out_labels, int32_t use_running_stats) {
  if (!c) return GAN_E_ARG;
  if (n < 0 || n > c->NB) return fail(c, GAN_E_ARG, "n out of range [0, max_total_batch]");
  if (!prior) return fail(c, GAN_E_ARG, "null prior");
  const int K = c->cfg.n_labels;
  double total = 0.0;
  int last = -1;
  for (int k = 0; k < K; ++k) {
    if (!(prior[k] >= 0.0)) return fail(c, GAN_E_ARG, "negative (or NaN) prior entry");
    total += prior[k];
    if (prior[k] > 0.0) last = k;
  }
  if (!(total > 0.0)) return fail(c, GAN_E_ARG, "the prior sums to zero");
  if (n == 0) return GAN_OK;
  if (!u || !noise || !out_images || !out_labels) return fail(c, GAN_E_ARG, "null pointer");
  std::vector<double> cdf((size_t)K);
  double cum = 0.0;
  for (int k = 0; k < K; ++k) { cum += prior[k] / total; cdf[(size_t)k] = cum; }
  DrawTable table = {};
  if (K <= DRAW_ARGS) {
    std::copy(cdf.begin(), cdf.end(), table.cdf);
  } else {
    if (!c->cdf && !dev_alloc(c, (void**)&c->cdf, (size_t)K * sizeof(double))) return fail(c, GAN_E_OOM, "cumulative prior");
    if (hipStreamSynchronize(c->st) != hipSuccess ||      // an earlier call may still read the buffer
        hipMemcpy(c->cdf, cdf.data(), (size_t)K * sizeof(double), hipMemcpyHostToDevice) != hipSuccess)
      return fail(c, GAN_E_HIP, "copy of the cumulative prior failed");
  }
  launch_draw_labels(u, K <= DRAW_ARGS ? nullptr : c->cdf, table, K, last, n, out_labels, c->st);
  return gan_generate(c, out_labels, noise, n, out_images, use_running_stats);
}

gan_status gan_anova_f(gan_ctx* c, const int32_t* label_ids, const float* images, int32_t n, double* F) {
  if (!c || !F) return GAN_E_ARG;
  if (n < 0 || n > c->NB) return fail(c, GAN_E_ARG, "n out of range [0, max_total_batch]");
  const gan_config& f = c->cfg;
  const int K = f.n_labels, C = f.img_c, HW = f.img_hw * f.img_hw;
  for (int ch = 0; ch < C; ++ch) F[ch] = 0.0;
  if (n == 0) return fail(c, GAN_E_STATE, "no images");
  if (!label_ids || !images) return fail(c, GAN_E_ARG, "null pointer");
  const size_t kc = (size_t)K * C;
  if (!c->an_x && !dev_alloc(c, (void**)&c->an_x, (size_t)c->NB * C * sizeof(double))) return fail(c, GAN_E_OOM, "analysis-of-variance buffers");
  if (!c->an_res && hipHostMalloc((void**)&c->an_res, 2 * kc * sizeof(double) + (size_t)K * sizeof(int), hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    c->an_res = nullptr;
    return fail(c, GAN_E_OOM, "analysis-of-variance results");
  }
  // the results (a few KB) go straight to the host's memory: one wait instead of one and three synchronous copies
  int* gcnt = reinterpret_cast<int*>(c->an_res + 2 * kc);
  (void)hipGetLastError();      // what an earlier HIP call of the caller's left behind is not this call's failure
  launch_anova(label_ids, images, n, K, C, HW, c->an_x, c->an_res, c->an_res + kc, gcnt, c->st);
  if (hipGetLastError() != hipSuccess || hipStreamSynchronize(c->st) != hipSuccess) return fail(c, GAN_E_HIP, "analysis of variance failed on the device");
  if (!anova_f_from_sums(c->an_res, c->an_res + kc, gcnt, K, C, F))
    return fail(c, GAN_E_STATE, "fewer than two labels present, or not more images than labels");
  return GAN_OK;
}

static gan_status sync(gan_ctx* c) {
  const hipError_t e = hipStreamSynchronize(c->st);
  if (e != hipSuccess) return fail(c, GAN_E_HIP, std::string("stream failed: ") + hipGetErrorString(e));
  return GAN_OK;
}

gan_status gan_get_losses(gan_ctx* c, float* d_loss, float* g_loss, int32_t* counts) {
  if (!c) return GAN_E_ARG;
  gan_status s = sync(c);
  if (s != GAN_OK) return s;
  if (d_loss) hipMemcpy(d_loss, c->loss_d, (size_t)c->L * 4, hipMemcpyDeviceToHost);
  if (g_loss) hipMemcpy(g_loss, c->loss_g, (size_t)c->L * 4, hipMemcpyDeviceToHost);
  if (counts) hipMemcpy(counts, c->rb.counts, (size_t)c->L * 4, hipMemcpyDeviceToHost);
  int flag = 0;
  hipMemcpy(&flag, c->rb.flags, 4, hipMemcpyDeviceToHost);
  if (flag) {
    hipMemset(c->rb.flags, 0, 4);
    return fail(c, GAN_E_LABEL, "a label id outside [0, n_labels) was dropped");
  }
  return GAN_OK;
}

gan_status gan_param_count(const gan_ctx* c, int32_t which, int64_t* per_model) {
  if (!c || !per_model || which < 0 || which > 1) return GAN_E_ARG;
  *per_model = which == 0 ? c->G.Pext : c->D.Pext;
  return GAN_OK;
}
gan_status gan_bn_count(const gan_ctx* c, int32_t which, int64_t* per_model) {
  if (!c || !per_model || which < 0 || which > 1) return GAN_E_ARG;
  const Net& net = which == 0 ? c->G : c->D;
  *per_model = net.bn_ext2int.empty() ? net.nbn : (long long)net.bn_ext2int.size();
  return GAN_OK;
}

static gan_status read_block(gan_ctx* c, int which, int model, const float* dev_base, float* dst, int64_t n) {
  if (!c || !dst || which < 0 || which > 1 || model < 0 || model >= c->L) return GAN_E_ARG;
  Net& net = which == 0 ? c->G : c->D;
  if (n != net.Pext) return fail(c, GAN_E_ARG, "wrong element count");
  gan_status s = sync(c);
  if (s != GAN_OK) return s;
  std::vector<float> tmp((size_t)net.P);
  if (hipMemcpy(tmp.data(), dev_base + (long long)model * net.P, (size_t)net.P * 4, hipMemcpyDeviceToHost) != hipSuccess)
    return fail(c, GAN_E_HIP, "copy failed");
  for (long long i = 0; i < net.Pext; ++i) dst[i] = tmp[(size_t)net.ext2int[(size_t)i]];
  return GAN_OK;
}

gan_status gan_get_params(gan_ctx* c, int32_t which, int32_t model, float* dst, int64_t n) {
  if (!c || which < 0 || which > 1) return GAN_E_ARG;
  return read_block(c, which, model, (which == 0 ? c->G : c->D).theta, dst, n);
}
gan_status gan_get_grads(gan_ctx* c, int32_t which, int32_t model, float* dst, int64_t n) {
  if (!c || which < 0 || which > 1) return GAN_E_ARG;
  return read_block(c, which, model, (which == 0 ? c->G : c->D).g, dst, n);
}
gan_status gan_get_opt_state(gan_ctx* c, int32_t which, int32_t model, float* m, float* v, int64_t* t) {
  if (!c || which < 0 || which > 1 || model < 0 || model >= c->L) return GAN_E_ARG;
  Net& net = which == 0 ? c->G : c->D;
  gan_status s = GAN_OK;
  if (m) s = read_block(c, which, model, net.m, m, net.Pext);
  if (s == GAN_OK && v) s = read_block(c, which, model, net.v, v, net.Pext);
  if (s == GAN_OK && t) {
    s = sync(c);
    int tt = 0;
    hipMemcpy(&tt, net.t + model, 4, hipMemcpyDeviceToHost);
    *t = tt;
  }
  return s;
}

gan_status gan_set_params(gan_ctx* c, int32_t which, int32_t model, const float* src, int64_t n) {
  if (!c || !src || which < 0 || which > 1 || model < 0 || model >= c->L) return GAN_E_ARG;
  Net& net = which == 0 ? c->G : c->D;
  if (n != net.Pext) return fail(c, GAN_E_ARG, "wrong element count");
  gan_status s = sync(c);
  if (s != GAN_OK) return s;
  std::vector<float> tmp((size_t)net.P, 0.f);
  for (long long i = 0; i < net.Pext; ++i) tmp[(size_t)net.ext2int[(size_t)i]] = src[i];
  if (hipMemcpy(net.theta + (long long)model * net.P, tmp.data(), (size_t)net.P * 4, hipMemcpyHostToDevice) != hipSuccess)
    return fail(c, GAN_E_HIP, "copy failed");
  c->shadows_dirty = true;
  return GAN_OK;
}

static gan_status write_block(gan_ctx* c, Net& net, int model, float* dev_base, const float* src) {
  std::vector<float> tmp((size_t)net.P, 0.f);
  for (long long i = 0; i < net.Pext; ++i) tmp[(size_t)net.ext2int[(size_t)i]] = src[i];
  if (hipMemcpy(dev_base + (long long)model * net.P, tmp.data(), (size_t)net.P * 4, hipMemcpyHostToDevice) != hipSuccess)
    return fail(c, GAN_E_HIP, "copy failed");
  return GAN_OK;
}

gan_status gan_set_opt_state(gan_ctx* c, int32_t which, int32_t model, const float* m, const float* v, int64_t t) {
  if (!c || which < 0 || which > 1 || model < 0 || model >= c->L || t < 0 || t > 0x7fffffff) return GAN_E_ARG;
  Net& net = which == 0 ? c->G : c->D;
  gan_status s = sync(c);
  if (s == GAN_OK && m) s = write_block(c, net, model, net.m, m);
  if (s == GAN_OK && v) s = write_block(c, net, model, net.v, v);
  if (s == GAN_OK) {
    const int tt = (int)t;
    if (hipMemcpy(net.t + model, &tt, 4, hipMemcpyHostToDevice) != hipSuccess) return fail(c, GAN_E_HIP, "copy failed");
  }
  return s;
}

static long long bn_ext_count(const Net& net) { return net.bn_ext2int.empty() ? net.nbn : (long long)net.bn_ext2int.size(); }

gan_status gan_set_bn_running(gan_ctx* c, int32_t which, int32_t model, const float* mean, const float* var, int64_t n) {
  if (!c || !mean || !var || which < 0 || which > 1 || model < 0 || model >= c->L) return GAN_E_ARG;
  Net& net = which == 0 ? c->G : c->D;
  if (n != bn_ext_count(net)) return fail(c, GAN_E_ARG, "wrong element count");
  gan_status s = sync(c);
  if (s != GAN_OK) return s;
  std::vector<float> m((size_t)net.nbn, 0.f), v((size_t)net.nbn, 1.f);
  for (long long i = 0; i < n; ++i) {
    const long long k = net.bn_ext2int.empty() ? i : net.bn_ext2int[(size_t)i];
    m[(size_t)k] = mean[i]; v[(size_t)k] = var[i];
  }
  if (hipMemcpy(net.run_mean + (long long)model * net.nbn, m.data(), (size_t)net.nbn * 4, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(net.run_var + (long long)model * net.nbn, v.data(), (size_t)net.nbn * 4, hipMemcpyHostToDevice) != hipSuccess)
    return fail(c, GAN_E_HIP, "copy failed");
  return GAN_OK;
}

gan_status gan_get_bn_running(gan_ctx* c, int32_t which, int32_t model, float* mean, float* var, int64_t n) {
  if (!c || !mean || !var || which < 0 || which > 1 || model < 0 || model >= c->L) return GAN_E_ARG;
  Net& net = which == 0 ? c->G : c->D;
  if (n != bn_ext_count(net)) return fail(c, GAN_E_ARG, "wrong element count");
  gan_status s = sync(c);
  if (s != GAN_OK) return s;
  std::vector<float> m((size_t)net.nbn), v((size_t)net.nbn);
  if (hipMemcpy(m.data(), net.run_mean + (long long)model * net.nbn, (size_t)net.nbn * 4, hipMemcpyDeviceToHost) != hipSuccess ||
      hipMemcpy(v.data(), net.run_var + (long long)model * net.nbn, (size_t)net.nbn * 4, hipMemcpyDeviceToHost) != hipSuccess)
    return fail(c, GAN_E_HIP, "copy failed");
  for (long long i = 0; i < n; ++i) {
    const long long k = net.bn_ext2int.empty() ? i : net.bn_ext2int[(size_t)i];
    mean[i] = m[(size_t)k]; var[i] = v[(size_t)k];
  }
  return GAN_OK;
}

gan_status gan_get_routing(gan_ctx* c, int32_t* perm, int32_t* offs) {
  if (!c) return GAN_E_ARG;
  if (c->last_n < 0) return fail(c, GAN_E_STATE, "no step has been taken");
  gan_status s = sync(c);
  if (s != GAN_OK) return s;
  if (offs) hipMemcpy(offs, c->rb.offs, (size_t)(c->L + 1) * 4, hipMemcpyDeviceToHost);
  if (perm && c->last_n > 0) {
    int nv = 0;
    hipMemcpy(&nv, c->rb.offs + c->L, 4, hipMemcpyDeviceToHost);
    for (int i = 0; i < c->last_n; ++i) perm[i] = -1;
    hipMemcpy(perm, c->rb.perm, (size_t)nv * 4, hipMemcpyDeviceToHost);
  }
  return GAN_OK;
}

gan_status gan_profile_enable(gan_ctx* c, int32_t enable) {
  if (!c) return GAN_E_ARG;
  gan_status s = sync(c);
  if (s != GAN_OK) return s;
  for (auto& e : c->prof_entries) { c->event_pool.push_back(e.e0); c->event_pool.push_back(e.e1); }
  c->prof_entries.clear();
  c->prof = enable != 0;
  c->prof_detail = enable == 2;     // 2: one family per layer shape
  c->prof_gemm_only = enable == 3;  // 3: only the MFMA kernels (fewest events in the stream)
  return GAN_OK;
}

gan_status gan_profile_read(gan_ctx* c, int32_t cap, const char** names, int64_t* launches, double* ms, double* flops,
                            double* bytes, int32_t* n_out) {
  if (!c || !names || !launches || !ms || !flops || !bytes || !n_out || cap < 1) return GAN_E_ARG;
  gan_status s = sync(c);
  if (s != GAN_OK) return s;
  int nf = 0;
  for (auto& e : c->prof_entries) {
    int k = -1;
    for (int i = 0; i < nf; ++i) if (strcmp(names[i], e.name) == 0) { k = i; break; }
    if (k < 0) {
      if (nf >= cap) continue;
      k = nf++;
      names[k] = e.name; launches[k] = 0; ms[k] = 0; flops[k] = 0; bytes[k] = 0;
    }
    float t = 0.f;
    hipEventElapsedTime(&t, e.e0, e.e1);
    launches[k] += 1; ms[k] += t; flops[k] += e.flops; bytes[k] += e.bytes;
  }
  // The MFMA launches of the two streams overlap: the time during which at least one of them ran (union of their
  // intervals on the clock of the first timed launch), with their summed work, as one more family.
  if (nf < cap && !c->prof_entries.empty()) {
    std::vector<std::pair<float, float>> iv;
    double fl = 0, by = 0;
    const hipEvent_t origin = c->prof_entries.front().e0;
    for (auto& e : c->prof_entries) {
      if (strncmp(e.name, "gemm_", 5) != 0 && strncmp(e.name, "wgrad", 5) != 0) continue;
      float t0 = 0.f, t1 = 0.f;
      if (hipEventElapsedTime(&t0, origin, e.e0) != hipSuccess || hipEventElapsedTime(&t1, origin, e.e1) != hipSuccess) continue;
      iv.push_back({t0, t1});
      fl += e.flops; by += e.bytes;
    }
    (void)hipGetLastError();
    if (!iv.empty()) {
      std::sort(iv.begin(), iv.end());
      double busy = 0;
      float lo = iv[0].first, hi = iv[0].second;
      for (auto& x : iv) {
        if (x.first <= hi) hi = std::max(hi, x.second);
        else { busy += hi - lo; lo = x.first; hi = x.second; }
      }
      busy += hi - lo;
      names[nf] = "(mfma busy)"; launches[nf] = (int64_t)iv.size(); ms[nf] = busy; flops[nf] = fl; bytes[nf] = by;
      ++nf;
    }
  }
  *n_out = nf;
  return GAN_OK;
}

// ---- single operations ------------------------------------------------------------------------------------
// enqueue, wait, and report: a refused launch, a launch error, or a failure while running
static gan_status finish_op(gan_ctx* c) {
  const gan_status launched = launch_status(c);
  const gan_status s = sync(c);
  return launched != GAN_OK ? launched : s;
}

static gan_status op_common(gan_ctx* c, const int32_t* offs, int n_groups, int rps, int tile_rows, int** tpre_out) {
  int* tp = nullptr;
  if (hipMalloc((void**)&tp, (size_t)(n_groups + 1) * 4) != hipSuccess) return fail(c, GAN_E_OOM, "tile prefix alloc");
  launch_tile_prefix(offs, n_groups, rps, tile_rows, tp, c->st);
  *tpre_out = tp;
  return GAN_OK;
}

// what the GEMM kernels address with 32-bit byte offsets: one segment of an operand
static bool fits_32bit(long long samples, long long side, long long channels, size_t es) {
  return samples * side * side * channels * (long long)es < (1LL << 31);
}

static gan_status op_conv(gan_ctx* c, int mode, const void* A, const void* W, void* Out, const int32_t* offs, int n_groups,
                          int n_samples, int C, int N, int Hin, int Hr, long long wstride) {
  if (!c || !A || !W || !Out || !offs || n_groups < 1 || n_samples < 0 || Hr < 1) return GAN_E_ARG;
  if (C < 64 || N < 64 || C % 64 || N % 64) return fail(c, GAN_E_SHAPE, "channel counts must be multiples of 64");
  if (!fits_32bit(n_samples, Hin, C, esize(c)) || !fits_32bit(n_samples, 2 * Hr, N, esize(c)) ||
      16LL * C * N * (long long)esize(c) >= (1LL << 31))
    return fail(c, GAN_E_SHAPE, "an operand of 2 GiB or more (the kernels use 32-bit byte offsets)");
  (void)take_launch_error();
  int* tp = nullptr;
  const ConvTile tile = c->op_tile_rows ? conv_tile_of_rows((int)esize(c), c->op_tile_rows, N)
                                        : conv_choose_tile((int)esize(c), N, (double)n_samples * Hr * Hr / n_groups, n_groups, mode == MODE_UP ? 4 : 1);
  const int tr = conv_tile_rows((int)esize(c), tile);
  gan_status s = op_common(c, offs, n_groups, Hr * Hr, tr, &tp);
  if (s != GAN_OK) return s;
  ConvArgs a = {};
  a.A = A; a.W = W; a.Out = Out; a.Aux = nullptr; a.w_nstride = N; a.offs = offs; a.tpre = tp; a.w_stride = wstride; a.L = n_groups;
  unsigned short* parts = nullptr;
  if (!c->bf16) {
    if (hipMalloc((void**)&parts, (size_t)n_groups * wstride * 6) != hipSuccess) {
      (void)hipGetLastError();
      (void)hipFree(tp);
      return fail(c, GAN_E_OOM, "split weights alloc");
    }
    const SplitArgs sp = {(const float*)W, parts, nullptr, wstride, wstride, n_groups, N, C};
    launch_split_weights(sp, c->st);
    a.W = parts; a.w_stride = 3 * wstride; a.w_plane = wstride; a.w_raw = (const float*)W; a.raw_stride = wstride; a.raw_n = C; a.raw_k = 1;
  }
  a.seg_first = 0; a.nseg = 1; a.seg_samples = n_samples; a.C = C; a.N = N; a.Hin = Hin; a.Hr = Hr;
  a.ub_tiles = (int)(((long long)n_samples * Hr * Hr) / tr) + n_groups; a.slope = 0.f; a.tile = tile;
  if (c->bf16) launch_conv<bf16_t>(mode, EPI_NONE, a, c->st); else launch_conv<float>(mode, EPI_NONE, a, c->st);
  s = finish_op(c);
  (void)hipFree(tp);
  if (parts) (void)hipFree(parts);
  return s;
}

gan_status gan_op_tile_rows(gan_ctx* c, int32_t rows) {
  if (!c) return GAN_E_ARG;
  if (rows != 0 && rows != 64 && rows != 128 && rows != 256) return fail(c, GAN_E_ARG, "tile heights are 64, 128 and 256 (0: automatic)");
  c->op_tile_rows = rows;
  return GAN_OK;
}

gan_status gan_op_wgrad_parts(gan_ctx* c, int32_t segments, int32_t splits) {
  if (!c) return GAN_E_ARG;
  if (segments < 1 || segments > 2 || splits < 1 || splits > WG_MAX_KSPLIT) return fail(c, GAN_E_ARG, "one or two segments, and as many row splits as a step may take");
  c->op_segments = segments;
  c->op_splits = splits;
  return GAN_OK;
}

gan_status gan_op_conv_down(gan_ctx* c, const void* big, const void* w_down, void* small_out, const int32_t* offs,
                            int32_t n_groups, int32_t n_samples, int32_t cb, int32_t cs, int32_t hs) {
  return op_conv(c, MODE_DOWN, big, w_down, small_out, offs, n_groups, n_samples, cb, cs, 2 * hs, hs, (long long)16 * cb * cs);
}
gan_status gan_op_conv_up(gan_ctx* c, const void* small_in, const void* w_up, void* big_out, const int32_t* offs,
                          int32_t n_groups, int32_t n_samples, int32_t cb, int32_t cs, int32_t hs) {
  return op_conv(c, MODE_UP, small_in, w_up, big_out, offs, n_groups, n_samples, cs, cb, hs, hs, (long long)16 * cb * cs);
}
gan_status gan_op_conv_wgrad(gan_ctx* c, const void* big, const void* small_in, float* dw, const int32_t* offs,
                             int32_t n_groups, int32_t n_samples, int32_t cb, int32_t cs, int32_t hs) {
  if (!c || !big || !small_in || !dw || !offs || n_groups < 1 || n_samples < 0 || hs < 1) return GAN_E_ARG;
  if (cb < 8 || cs < 8 || (16 * cb) % 128 || cb % 8 || cs % 8) return fail(c, GAN_E_SHAPE, "unsupported channel counts");
  if (!fits_32bit(n_samples, 2 * hs, cb, esize(c)) || !fits_32bit(n_samples, hs, cs, esize(c)))
    return fail(c, GAN_E_SHAPE, "an operand of 2 GiB or more (the kernels use 32-bit byte offsets)");
  (void)take_launch_error();
  WgradArgs a = {};
  a.Big = big; a.Small = small_in; a.dW = dw; a.offs = offs; a.dw_stride = (long long)16 * cb * cs;
  a.L = n_groups; a.nseg = c->op_segments; a.seg_samples = n_samples; a.Cb = cb; a.Cs = cs; a.Hs = hs; a.ntaps = 16; a.ksplit = c->op_splits;
  a.split_stride = n_groups * a.dw_stride;
  if (c->bf16) launch_wgrad<bf16_t>(a, c->st); else launch_wgrad<float>(a, c->st);
  return finish_op(c);
}

// What the two entries below share: the model of every sample, and what the launches need in device memory for as long as they run.
struct ImageOp {
  std::vector<int> offs;
  std::vector<void*> held;
  ~ImageOp() { for (void* p : held) (void)hipFree(p); }
  void* hold(size_t bytes) {
    void* p = nullptr;
    if (hipMalloc(&p, bytes < 16 ? 16 : bytes) != hipSuccess) { (void)hipGetLastError(); return nullptr; }
    held.push_back(p);
    return p;
  }
  int* hold(const std::vector<int>& v) {
    int* p = (int*)hold(v.size() * 4);
    if (p && !v.empty() && hipMemcpy(p, v.data(), v.size() * 4, hipMemcpyHostToDevice) != hipSuccess) return nullptr;
    return p;
  }
};
static gan_status image_op_begin(gan_ctx* c, ImageOp& op, const void* img, const float* nchw, const int32_t* perm, const int32_t* offs, int32_t n_groups,
                                 int32_t n_samples, int32_t cb, int32_t cs, int32_t hs, int32_t maps) {
  if (!c || !offs || n_groups < 1 || n_samples < 1 || (nchw && !perm) || (!img && (!nchw || c->op_segments > 1))) return GAN_E_ARG;
  if (cb < 1 || cb > 4 || (cs != 64 && cs != 128) || hs < 2 || (maps != 0 && maps != n_groups)) return fail(c, GAN_E_SHAPE, "image-side layers: 1 to 4 image channels, 64 or 128 feature channels");
  (void)take_launch_error();
  const gan_status s = sync(c);
  if (s != GAN_OK) return s;
  op.offs.resize(n_groups + 1);
  if (hipMemcpy(op.offs.data(), offs, (size_t)(n_groups + 1) * 4, hipMemcpyDeviceToHost) != hipSuccess) return fail(c, GAN_E_HIP, "copy failed");
  for (int l = 0; l < n_groups; ++l)
    if (op.offs[l] < 0 || op.offs[l] > op.offs[l + 1]) return fail(c, GAN_E_ARG, "sample offsets must not decrease");
  if (op.offs[n_groups] != n_samples) return fail(c, GAN_E_ARG, "n_samples must be offs[n_groups]");
  return GAN_OK;
}
gan_status gan_op_image_conv(gan_ctx* c, const void* img, const float* nchw, const int32_t* perm, const float* w, const float* bias, void* small_out,
                             const int32_t* offs, int32_t n_groups, int32_t n_samples, int32_t cb, int32_t cs, int32_t hs, int32_t maps) {
  ImageOp op;
  if (!w || !small_out) return GAN_E_ARG;
  const gan_status s = image_op_begin(c, op, img, nchw, perm, offs, n_groups, n_samples, cb, cs, hs, maps);
  if (s != GAN_OK) return s;
  std::vector<int> model(n_samples);
  for (int l = 0; l < n_groups; ++l) std::fill(model.begin() + op.offs[l], model.begin() + op.offs[l + 1], l);
  ImagePackArgs p = {};
  p.w = w; p.L = n_groups; p.CB = cb; p.CBT = cb + maps; p.Cs = cs; p.P = image_values(cb); p.pstride = 16LL * p.CBT * cs; p.tables = n_groups;
  p.packed = op.hold((size_t)n_groups * 16 * p.P * cs * esize(c));
  p.add = maps ? (float*)op.hold((size_t)n_groups * 9 * cs * 4) : nullptr;
  ImageConvArgs a = {};
  a.img = img ? img : nchw; a.real = nchw; a.perm = perm; a.w = p.packed; a.add = p.add; a.bias = bias; a.bias_stride = cs; a.out = small_out; a.offs = offs;
  a.sample_model = op.hold(model);
  if (!p.packed || (maps && !p.add) || !a.sample_model) return fail(c, GAN_E_OOM, "image-side operand alloc");
  a.L = n_groups; a.n = n_samples; a.CB = cb; a.Hs = hs; a.Cs = cs; a.nseg = c->op_segments; a.seg_samples = n_samples; a.slope = 1.f;
  if (c->bf16) { launch_pack_image_w<bf16_t>(p, c->st); launch_image_conv<bf16_t>(a, c->st); }
  else { launch_pack_image_w<float>(p, c->st); launch_image_conv<float>(a, c->st); }
  return finish_op(c);
}
gan_status gan_op_image_wgrad(gan_ctx* c, const void* img, const float* nchw, const int32_t* perm, const void* small_in, float* grad, const int32_t* offs,
                              int32_t n_groups, int32_t n_samples, int32_t cb, int32_t cs, int32_t hs, int32_t maps, int32_t size_samples,
                              int32_t size_models) {
  ImageOp op;
  if (!small_in || !grad || size_samples < n_samples || size_models < 1) return GAN_E_ARG;
  const gan_status s = image_op_begin(c, op, img, nchw, perm, offs, n_groups, n_samples, cb, cs, hs, maps);
  if (s != GAN_OK) return s;
  const ImageTiles tiling = image_tiles((int)esize(c), size_samples, size_models);
  const int P = image_values(cb);
  std::vector<int> tpre(1, 0), tmodel;
  for (int l = 0; l < n_groups; ++l) {
    const int own = op.offs[l + 1] - op.offs[l], per = image_tile(tiling, own);
    tmodel.insert(tmodel.end(), (own + per - 1) / per, l);
    tpre.push_back((int)tmodel.size());
  }
  const int tiles = (int)tmodel.size();
  ImageWgradArgs a = {};
  a.img = img ? img : nchw; a.real = nchw; a.perm = perm; a.dy = small_in; a.offs = offs;
  a.part = (float*)op.hold((size_t)image_part_floats((int)esize(c), cb, hs, cs, c->op_segments, tiling, tiles) * 4); a.pixel_sums = (float*)op.hold((size_t)tiles * 4 * 4);
  a.tpre = op.hold(tpre); a.tmodel = op.hold(tmodel);
  if (!a.part || !a.pixel_sums || !a.tpre || !a.tmodel) return fail(c, GAN_E_OOM, "image-side partial sums alloc");
  a.L = n_groups; a.CB = cb; a.Hs = hs; a.Cs = cs; a.nseg = c->op_segments; a.seg_samples = n_samples; a.tiles = tiling;
  ImageGradArgs g = {};
  g.part = a.part; g.pixel_sums = a.pixel_sums; g.tpre = a.tpre; g.L = n_groups; g.CB = cb; g.CBT = cb + maps; g.Cs = cs; g.P = P; g.plane_labels = maps > 0;
  const long long taps = 16LL * g.CBT * cs;
  g.dw = grad; g.dbias = grad + taps; g.image_bias = grad + taps + cs; g.pstride = taps + cs + 4;
  if (c->bf16) launch_image_wgrad<bf16_t>(a, tiles, c->st); else launch_image_wgrad<float>(a, tiles, c->st);
  launch_image_wgrad_final(g, c->st);
  return finish_op(c);
}

gan_status gan_op_split_sum(gan_ctx* c, const float* parts, float* sum, int32_t n_groups, int32_t splits, int32_t cb, int32_t cs) {
  if (!c || !parts || !sum || n_groups < 1 || splits < 2 || splits > WG_MAX_KSPLIT) return GAN_E_ARG;
  if (cb < 64 || cs < 64 || cb % 64 || cs % 64) return fail(c, GAN_E_SHAPE, "channel counts must be multiples of 64");
  (void)take_launch_error();
  AdamArgs a = {};
  const long long layer = 16LL * cb * cs, all = layer * n_groups;
  // an update of zero weights with step counts and corrections of one: theta, m, v, the copies (bf16: two; fp32: one), counts, bc
  float* scratch = nullptr;
  const long long floats = 5 * all + 3LL * n_groups;
  if (hipMalloc((void**)&scratch, (size_t)floats * 4) != hipSuccess) {
    (void)hipGetLastError();
    return fail(c, GAN_E_OOM, "update scratch alloc");
  }
  std::vector<float> ones((size_t)n_groups * 3, 1.f);
  const int one = 1;
  for (int l = 0; l < n_groups; ++l) memcpy(&ones[(size_t)l], &one, 4);
  gan_status s = sync(c);
  if (s == GAN_OK && (hipMemset(scratch, 0, (size_t)floats * 4) != hipSuccess ||
                      hipMemcpy(scratch + 5 * all, ones.data(), ones.size() * 4, hipMemcpyHostToDevice) != hipSuccess)) s = fail(c, GAN_E_HIP, "copy failed");
  if (s == GAN_OK) {
    a.theta = scratch; a.m = scratch + all; a.v = scratch + 2 * all; a.g = sum; a.P = layer; a.plane = layer; a.L = n_groups;
    if (c->bf16) a.shadow = scratch + 3 * all;
    a.shadow_t = scratch + 4 * all;
    a.counts = (const int*)(scratch + 5 * all); a.bc = scratch + 5 * all + n_groups;
    a.lr = 0.f; a.beta1 = 0.5f; a.beta2 = 0.999f; a.eps = 1e-8f;
    a.nregions = 1; a.reg_cb[0] = a.reg_cb_real[0] = cb; a.reg_cs[0] = a.reg_cs_real[0] = cs;
    const AdamSplits sp = {parts, splits, split_chains(all, splits)};
    if (adam_plan(a)) { if (c->bf16) launch_adam_region<bf16_t>(a, 0, sp, c->st); else launch_adam_region<float>(a, 0, sp, c->st); }
    s = finish_op(c);
  }
  (void)hipFree(scratch);
  return s;
}

gan_status gan_op_dropout(gan_ctx* c, void* x, const int32_t* offs, int32_t n_groups, int32_t n_samples, int32_t ch, int32_t h,
                          int32_t w, float p, uint64_t seed, int32_t step, int32_t layer, int32_t pass_id) {
  if (!c || !x || !offs || n_groups < 1 || n_samples < 0 || ch < 1 || h < 1 || w < 1 || step < 0 || layer < 0 || layer > 255 ||
      pass_id < 0)
    return GAN_E_ARG;
  if (!(p >= 0.f && p < 1.f)) return fail(c, GAN_E_ARG, "dropout probability outside [0, 1)");
  (void)take_launch_error();
  if (c->bf16) launch_dropout<bf16_t>(static_cast<bf16_t*>(x), offs, n_groups, n_samples, ch, h, w, p, seed, step, layer, pass_id, c->st);
  else launch_dropout<float>(static_cast<float*>(x), offs, n_groups, n_samples, ch, h, w, p, seed, step, layer, pass_id, c->st);
  return finish_op(c);
}
gan_status gan_op_w3_to_w4(gan_ctx* c, const float* w3, void* w4, void* w4t, int32_t n_groups, int32_t cb, int32_t cs) {
  if (!c || !w3 || !w4 || !w4t || n_groups < 1 || cb < 1 || cs < 1) return GAN_E_ARG;
  (void)take_launch_error();
  if (c->bf16) launch_w3_to_w4<bf16_t>(w3, static_cast<bf16_t*>(w4), static_cast<bf16_t*>(w4t), n_groups, cb, cs, c->st);
  else launch_w3_to_w4<float>(w3, static_cast<float*>(w4), static_cast<float*>(w4t), n_groups, cb, cs, c->st);
  return finish_op(c);
}
gan_status gan_op_dw4_to_dw3(gan_ctx* c, const float* dw4, float* dw3, int32_t n_groups, int32_t cb, int32_t cs) {
  if (!c || !dw4 || !dw3 || n_groups < 1 || cb < 1 || cs < 1) return GAN_E_ARG;
  (void)take_launch_error();
  launch_dw4_to_dw3(dw4, dw3, n_groups, cb, cs, c->st);
  return finish_op(c);
}

}  // extern "C"
