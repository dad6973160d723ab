// The forward-type GEMM's reduction order, walked on the host (tests/test_k_order.py).
#include "../../paper_2102_10485_amd/csrc/k_order.h"

template <int MODE>
static void walk(int cpl, int lo, int hi, int first_gone, int py, int px, unsigned row, unsigned pxb, unsigned wtap, int chunks, int states,
                 int* more, int* tap, int* line, unsigned* aoff, unsigned* woff) {
  gan::KOrder<MODE, 128, true> o;
  o.cpl = cpl; o.cnt_lo = lo; o.cnt_hi = hi; o.first_gone = first_gone != 0; o.py = py; o.px = px;
  o.row_bytes = row; o.px_bytes = pxb; o.wtap_bytes = wtap;
  o.start();
  int left = chunks;
  bool is = left > 0;
  for (int i = 0; i < states; ++i) {
    more[i] = is; tap[i] = o.tap; line[i] = o.line; aoff[i] = o.aoff; woff[i] = o.woff;
    is = o.next(left);
  }
}

extern "C" void k_order_walk(int mode, int cpl, int lo, int hi, int first_gone, int py, int px, unsigned row, unsigned pxb, unsigned wtap,
                             int chunks, int states, int* more, int* tap, int* line, unsigned* aoff, unsigned* woff) {
  if (mode == gan::MODE_DOWN) walk<gan::MODE_DOWN>(cpl, lo, hi, first_gone, py, px, row, pxb, wtap, chunks, states, more, tap, line, aoff, woff);
  else walk<gan::MODE_UP>(cpl, lo, hi, first_gone, py, px, row, pxb, wtap, chunks, states, more, tap, line, aoff, woff);
}
