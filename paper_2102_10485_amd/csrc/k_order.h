// The order in which a tile of the forward-type GEMM walks its reduction, chunk by chunk (conv_gemm.hip): which tap a chunk gathers and the
// wave-uniform byte offsets it adds to the rows' and the columns'.  Plain arithmetic, which the host can walk too.
#pragma once

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define GAN_DEVICE_INLINE __device__ __forceinline__
#define GAN_HOST_DEVICE_INLINE __host__ __device__ __forceinline__
#else
#define GAN_DEVICE_INLINE inline
#define GAN_HOST_DEVICE_INLINE inline
#endif

namespace gan {

enum ConvMode { MODE_DOWN = 0, MODE_UP = 1, MODE_DENSE = 2 };

// K order, fastest first: the chunks of one 128-byte line; the taps whose gathers land on the same input pixels
// shifted by one (down: the 4 taps of a (ky%2, kx%2) class, up: the phase's 4 taps), which find their rows in
// L2; the channel line; (down) the class.  Carried along chunk by chunk: decoding the chunk's number took 90 scalar
// instructions a chunk, more issue time than the 8 MFMAs per wave of a 64-byte chunk.
// down: classes 0, 1 hold the taps with ky in {0, 2}, classes 2, 3 those with ky in {1, 3}; a class keeps cnt taps, and the
// two left in a class of two are its kx pair at the one valid ky: ky = 2 (top tile, even class) or 1 (bottom, odd).
// KB: bytes of a chunk.  SCALAR: the counters are put into scalar registers in every step.
template <int MODE, int KB, bool SCALAR>
struct KOrder {
  int cpl;                               // 128-byte channel lines of a tap
  int cnt_lo, cnt_hi;                    // down: valid taps of the classes with ky even / odd; up: cnt_lo = valid taps
  bool first_gone;                       // up: the skipped taps are the first ones of their group
  int py, px;                            // up: the phase
  unsigned row_bytes, px_bytes, wtap_bytes;

  int part, j, line, cls, cnt;           // the chunk
  int tap = 0, wtap = 0;                 // its tap, and the tap's place in the weight block
  unsigned aoff = 0, woff = 0;

  GAN_DEVICE_INLINE void start() {
    part = j = line = cls = 0;
    cnt = MODE == MODE_DENSE ? 1 : cnt_lo;
    set();
  }
  GAN_DEVICE_INLINE void set() {
    if (MODE == MODE_DOWN) {
      const int i = cnt == 4 ? j : j + (cls < 2 ? 2 : 0);
      const int ky = (cls >> 1) + 2 * (i >> 1), kx = (cls & 1) + 2 * (i & 1);
      tap = ky * 4 + kx;
      aoff = ky * row_bytes + kx * px_bytes + line * 128;
      wtap = tap;
      woff = wtap * wtap_bytes + line * 128;
    } else if (MODE == MODE_UP) {
      // phase py = 0 gathers rows y and y - 1 through ky = 1 and 3, py = 1 rows y + 1 and y through ky = 0 and 2; likewise x
      tap = cnt == 4 ? j : j + (first_gone ? 2 : 0);
      const int a = tap >> 1, b = tap & 1;
      aoff = (py - a + 1) * row_bytes + (px - b + 1) * px_bytes + line * 128;
      wtap = (2 * a + 1 - py) * 4 + 2 * b + 1 - px;
      woff = wtap * wtap_bytes + line * 128;
    } else {
      aoff = woff = line * 128;
    }
  }
  GAN_DEVICE_INLINE void advance() {
    if (KB < 128) {
      part ^= 1;
      if (part) { aoff += KB; woff += KB; return; }
    }
    if (++j == cnt) {
      j = 0;
      if (++line == cpl && MODE == MODE_DOWN) {
        line = 0;
        ++cls;
        cnt = cls < 2 ? cnt_lo : cnt_hi;
      }
    }
#if defined(__HIP_DEVICE_COMPILE__)
    if (SCALAR) {
      j = __builtin_amdgcn_readfirstlane(j);
      line = __builtin_amdgcn_readfirstlane(line);
    }
#endif
    set();
  }
  // The next of `left` chunks, for a loop whose copies go on behind the last one: advances and returns true, or stays where it is.  (The range
  // check of a buffer may subtract the scalar offset from the buffer's size; with an offset of a chunk that does not exist, one pixel or one row of
  // weights behind the slice, an empty buffer would then have wrapped round to a large one.)
  GAN_DEVICE_INLINE bool next(int& left) {
    const bool more = --left > 0;
    if (more) advance();
    return more;
  }
};

}  // namespace gan
