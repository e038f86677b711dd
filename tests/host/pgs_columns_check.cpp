// Host-only walk over every column load of the Gauss-Seidel chains, built and
// run by tests/test_host_library.py: no load may end past the buffer of
// blocked couplings, whose range check does not see the column's offset.
#include <cstdio>

#include "pgs_layout.hpp"

using namespace icr;

static long bad = 0, loads = 0;

// take() as the chains call it: kPgsAhead columns before the first one in use,
// then one for each that is done with
static void walk(PgsColumns cols, int done, size_t bytes) {
  for (int i = 0; i < kPgsAhead + done; ++i) {
    ++loads;
    if (cols.take() + 8ull * kPgsGroup > bytes) ++bad;
  }
}

static void sweep(int nS, size_t bytes) {
  const int nsp = pgs_wave_pad(nS);
  const unsigned stride = 8u * kPgsBlk * (unsigned)nsp;
  for (int w = 0; w < nsp / 64; ++w)
    for (int b = 0; b < nS; b += 64) {
      const int n = nS - b < 64 ? nS - b : 64;
      const PgsColumns cols(8u * kPgsGroup * (unsigned)w + stride * (unsigned)b, stride, n);
      PgsColumns turn = cols;   // the columns in use come in turn
      for (int i = 0; i < n; ++i)
        if (turn.take() != 8u * kPgsGroup * (unsigned)w + stride * (unsigned)(b + i)) ++bad;
      // the solving wave rounds its visits up to whole groups of kPgsAhead
      walk(cols, b == 64 * w ? (n + kPgsAhead - 1) / kPgsAhead * kPgsAhead : n, bytes);
    }
}

int main() {
  for (int nS = 1; nS <= kPgsWaveMax; ++nS) sweep(nS, 8 * pgs_wss_elems(nS));
  for (int nB = 1; nB <= kPgsCoopB; ++nB) sweep(nB, 8 * pgs_coop_blk_elems(nB));
  std::printf("%ld of %ld loads out of place\n", bad, loads);
  return bad != 0;
}
