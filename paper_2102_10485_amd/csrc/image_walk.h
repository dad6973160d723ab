// How the image-side weight gradient (image_conv.hip) walks its units, and the byte offsets of the feature gradient's values that it requests on
// the way.  Plain arithmetic, which the host can walk too.
#pragma once

#include "k_order.h"

namespace gan {

constexpr int img_values(int CB) { return CB == 1 ? 2 : (CB < 4 ? 4 : 8); }      // values a pixel has in a tile of CB channels

constexpr int IMG_SIDE = 16;                 // outputs along x of a unit, at most
constexpr int WG_SIDE_Y = 8;                 // along y: the weight gradient, where one wave's registers hold the next unit's image

// Units of a map of side Hs: ph x pw outputs, their tile rows `pitch` bytes apart.  A pitch of 80 to 176 bytes modulo 256 keeps the rows that one
// transposing read touches apart.
struct Units { int pw, ph, nx, ny, pitch; };
inline Units img_units(int Hs, int CB, int side_y) {
  Units u;
  u.nx = (Hs + IMG_SIDE - 1) / IMG_SIDE;
  u.pw = (Hs + u.nx - 1) / u.nx;
  u.ny = (Hs + side_y - 1) / side_y;
  u.ph = (Hs + u.ny - 1) / u.ny;
  u.pitch = ((2 * u.pw + 2) * 2 * img_values(CB) + 15) / 16 * 16;
  while (u.pitch % 256 < 80 || u.pitch % 256 > 176) u.pitch += 16;
  return u;
}
// Units of sixteen columns that the map is a whole number of, so that a K-step of sixteen pixels is a row and those of a wave (each in turn of 128 / CS)
// a fixed distance apart.
inline bool even_units(const Units& u, int Hs, int CS) { return u.pw == 16 && u.nx * u.pw == Hs && u.ny * u.ph == Hs && u.ph % (128 / CS) == 0; }

// Samples of a tile of the weight gradient.  A model's tiles are `parts` of its own samples, of `most` samples at most: at the sizing batch a round of blocks over all
// models (three a CU in bf16, two in fp32), and in calls of fewer samples as many blocks of shorter tiles.  What a model's tiles are follows from its own samples
// and the configuration.  Steps of 64 samples of one pair sized for
// 6400, with tiles of `most` (seven blocks) and with these, us: 28x28 in fp32 728 and 518, in bf16 448 and 369, 32x32 in bf16 1182 and 1093; of eight 64x64 pairs sized
// for 1024 1564 and 1528; steps of the sizing batch as they were.
struct ImageTiles { int most, parts; };
inline ImageTiles image_tiles(int esize, long long size_samples, int L) {
  const int tiles = esize == 4 ? 480 : 700;
  const long long most = (size_samples + tiles - 1) / tiles, parts = tiles / L;
  return ImageTiles{most < 1 ? 1 : (int)most, parts < 1 ? 1 : (int)parts};
}
GAN_HOST_DEVICE_INLINE int image_tile(const ImageTiles& t, int samples) {
  if (samples <= t.parts) return 1;           // (small calls wait for no division)
  const int per = (samples + t.parts - 1) / t.parts;
  return per < t.most ? per : t.most;
}
// no more tiles than this of n samples, however they fall: a model has `parts`, or one more than whole ones of `most`
inline long long image_tile_bound(const ImageTiles& t, long long n, int L) {
  const long long b = (n < L ? n : L) * (long long)t.parts + n / t.most;
  return b < n ? b : n;
}

struct UnitAt { int seg, j, y0, x0; };
// along x, along y, the next sample, the next segment
GAN_DEVICE_INLINE void next_unit(UnitAt& t, const Units& u, int Hs, int j0, int j1) {
  if ((t.x0 += u.pw) < Hs) return;
  t.x0 = 0;
  if ((t.y0 += u.ph) < Hs) return;
  t.y0 = 0;
  if (++t.j < j1) return;
  t.j = j0;
  ++t.seg;
}

constexpr unsigned NO_PIXEL = 0xffffffffu;   // an offset outside every buffer

// One lane's requests of a wave that takes the K-steps turn, turn + TURNS, ... of every unit.  A request is offset(i), its own, plus uniform, the
// wave's, inside the sample (at.seg, at.j), whose buffer is empty behind the last unit (live).
template <int LOADS, int TURNS, bool EVEN>
struct GradWalk {
  Units u;
  int Hs, j0, j1, units, steps;
  unsigned row_bytes, px_bytes, lane_bytes;  // of the map's rows and pixels; of the lane inside its pixel
  int dx, dy;                                // a K-step of this wave further
  int px_first[LOADS], py_first[LOADS];      // the lane's pixel of load i in a unit's first K-step

  UnitAt at;
  int unit, step;
  bool live;
  int px[LOADS], py[LOADS];
  unsigned lane_off[LOADS], uniform;

  // lane_pixel[i]: pixel of load i in a K-step
  GAN_DEVICE_INLINE void start(const Units& units_, int Hs_, const UnitAt& first, int j1_, int nseg, int turn, const int (&lane_pixel)[LOADS],
                               unsigned px_bytes_, unsigned lane_bytes_, bool live_) {
    u = units_; Hs = Hs_; j0 = first.j; j1 = j1_;
    units = (j1 - j0) * u.nx * u.ny * nseg;
    steps = ((u.ph * u.pw + 15) / 16 + TURNS - 1) / TURNS;
    px_bytes = px_bytes_; row_bytes = (unsigned)Hs * px_bytes; lane_bytes = lane_bytes_;
    dx = 16 * TURNS % u.pw; dy = 16 * TURNS / u.pw;
    at = first; unit = step = 0; live = live_;
    uniform = EVEN ? unit_offset() : 0u;
    for (int i = 0; i < LOADS; ++i) {
      const int p = 16 * turn + lane_pixel[i];
      py_first[i] = p / u.pw; px_first[i] = p - py_first[i] * u.pw;
      py[i] = py_first[i]; px[i] = px_first[i];
      lane_off[i] = (unsigned)turn * row_bytes + (unsigned)lane_pixel[i] * px_bytes + lane_bytes;
    }
  }
  GAN_DEVICE_INLINE unsigned unit_offset() const { return (unsigned)at.y0 * row_bytes + (unsigned)at.x0 * px_bytes; }
  GAN_DEVICE_INLINE unsigned offset(int i) const {
    if (EVEN) return lane_off[i];
    const int y = at.y0 + py[i], x = at.x0 + px[i];
    const bool ok = py[i] < u.ph && y < Hs && x < Hs;
    return ok ? (unsigned)(y * Hs + x) * px_bytes + lane_bytes : NO_PIXEL;
  }
  // To the next request; true where it is in another unit.  Behind the last unit the buffer is empty and the wave's offset zero: the range check may
  // subtract it from the buffer's size, and that of a K-step that does not exist would then have wrapped the empty buffer round to a large one.
  GAN_DEVICE_INLINE bool advance() {
    if (!live) return false;
    if (++step < steps) {
      if (EVEN) { uniform += TURNS * row_bytes; return false; }
      for (int i = 0; i < LOADS; ++i) {
        px[i] += dx; py[i] += dy;
        if (px[i] >= u.pw) { px[i] -= u.pw; ++py[i]; }
      }
      return false;
    }
    step = 0;
    for (int i = 0; i < LOADS; ++i) { py[i] = py_first[i]; px[i] = px_first[i]; }
    if (++unit < units) {
      next_unit(at, u, Hs, j0, j1);
      if (EVEN) uniform = unit_offset();
      return true;
    }
    live = false;
    uniform = 0;
    return false;
  }
};

}  // namespace gan
