// The image-side weight gradient's requests of the feature gradient, walked on the host (tests/test_image_walk.py).
#include "../../paper_2102_10485_amd/csrc/image_walk.h"

template <int ESIZE, int CS, bool EVEN>
static void walk(int CB, int Hs, int j0, int j1, int nseg, int wave, int lane, int requests, int* live, int* seg, int* sample, unsigned* offset, unsigned* uniform) {
  constexpr int TURNS = 128 / CS, LPP = ESIZE == 2 ? 4 : 8, LOADS = ESIZE == 2 ? 1 : 2;      // as image_wgrad_kernel has them
  gan::GradWalk<LOADS, TURNS, EVEN> w;
  int pixel[LOADS];
  for (int i = 0; i < LOADS; ++i) pixel[i] = lane / LPP + i * (64 / LPP);
  const int cb = wave % (CS / 32);
  w.start(gan::img_units(Hs, CB, gan::WG_SIDE_Y), Hs, gan::UnitAt{0, j0, 0, 0}, j1, nseg, wave / (CS / 32) % TURNS, pixel, CS * ESIZE, (cb * 32 + lane % LPP * (16 / ESIZE)) * ESIZE, true);
  for (int k = 0; k < requests; ++k) {
    live[k] = w.live; seg[k] = w.at.seg; sample[k] = w.at.j;
    for (int i = 0; i < LOADS; ++i) offset[k * LOADS + i] = w.offset(i);
    uniform[k] = w.uniform;
    w.advance();
  }
}

extern "C" int image_walk_even(int Hs, int CB, int CS) { return gan::even_units(gan::img_units(Hs, CB, gan::WG_SIDE_Y), Hs, CS); }
extern "C" int image_walk_steps(int Hs, int CB, int CS) {      // K-steps of a unit that a wave takes
  const gan::Units u = gan::img_units(Hs, CB, gan::WG_SIDE_Y);
  return ((u.ph * u.pw + 15) / 16 + 128 / CS - 1) / (128 / CS);
}
extern "C" int image_walk_units(int Hs, int CB) { const gan::Units u = gan::img_units(Hs, CB, gan::WG_SIDE_Y); return u.nx * u.ny; }
extern "C" void image_walk(int esize, int CB, int Hs, int CS, int j0, int j1, int nseg, int wave, int lane, int requests, int* live, int* seg, int* sample,
                           unsigned* offset, unsigned* uniform) {
  const bool even = image_walk_even(Hs, CB, CS);
#define GO(E, C) (even ? walk<E, C, true> : walk<E, C, false>)(CB, Hs, j0, j1, nseg, wave, lane, requests, live, seg, sample, offset, uniform)
  if (esize == 2) { if (CS == 64) GO(2, 64); else GO(2, 128); }
  else { if (CS == 64) GO(4, 64); else GO(4, 128); }
}

// tiles of the weight gradient: how many, of counts[0 .. L) samples, in a context sized for `size`; at[0], at[1]: the bound the host launches, the longest tile
extern "C" int image_walk_tiles(int esize, int size, int L, const int* counts, int* at) {
  const gan::ImageTiles t = gan::image_tiles(esize, size, L);
  long long n = 0;
  int tiles = 0;
  at[1] = 0;
  for (int l = 0; l < L; ++l) {
    const int per = gan::image_tile(t, counts[l]);
    tiles += (counts[l] + per - 1) / per;
    if (counts[l] > 0 && per > at[1]) at[1] = per;
    n += counts[l];
  }
  at[0] = (int)gan::image_tile_bound(t, n, L);
  return tiles;
}
