// Layout of the contact solve's work buffers, for host and device code.
#pragma once
#include <cstddef>

namespace icr {

// Layout of the PGS work buffers: per-contact records of kPgsRecWidth rows,
// the blocked coupling matrix of an active set of up to kPgsWaveMax contacts
// in 3x3 blocks of kPgsBlk doubles, padded to pgs_wave_pad contacts.
constexpr int kPgsRecWidth = 20;
constexpr int kPgsWaveMax = 512;
constexpr int kPgsBlk = 9;
constexpr inline int pgs_wave_pad(int nS) { return 64 * ((nS + 63) / 64); }
// doubles of the blocked coupling matrix of an active set (n_c contacts)
constexpr inline size_t pgs_wss_elems(int nc) {
  return (size_t)(nc < kPgsWaveMax ? nc : kPgsWaveMax) * pgs_wave_pad(nc < kPgsWaveMax ? nc : kPgsWaveMax) * kPgsBlk;
}
// doubles of the prepared records (and gaps) of a first active set
constexpr inline size_t pgs_rec_elems(int nc) { return (size_t)(nc < kPgsWaveMax ? nc : kPgsWaveMax) * kPgsRecWidth; }
// Block Gauss-Seidel over the whole GPU (sets beyond kPgsWaveMax contacts):
// blocks of kPgsCoopB contacts, each block's couplings padded like a wave set.
constexpr int kPgsCoopB = 128;
constexpr int kPgsCoopSync = 256;   // ints of sync words
constexpr inline size_t pgs_coop_blk_elems(int nc) {
  return (size_t)((nc + kPgsCoopB - 1) / kPgsCoopB) * kPgsCoopB * kPgsCoopB * kPgsBlk;
}

// Columns of the blocked couplings that a chain has in flight ahead of the
// one in use, and their byte offsets in turn (one wave's group of rows of a
// block's n >= 1 columns, `stride` apart).  The loads run ahead of the last
// column; from there the walk stays on it, so that no load leaves the buffer
// (a buffer load's scalar offset is no part of its range check).  What such a
// load returns is not used.
constexpr int kPgsAhead = 4;
constexpr int kPgsGroup = 64 * kPgsBlk;   // doubles of a group: 64 rows of one column
struct PgsColumns {
  unsigned off, last, stride;
  constexpr PgsColumns(unsigned first, unsigned stride_, int n)
      : off(first), last(first + stride_ * (unsigned)(n - 1)), stride(stride_) {}
  constexpr unsigned take() {
    const unsigned o = off;
    off = o + stride < last ? o + stride : last;
    return o;
  }
};

}  // namespace icr
