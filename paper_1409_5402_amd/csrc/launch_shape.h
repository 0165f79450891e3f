// Who works on what in the draw kernels: the arithmetic of their launches and loads, without any device code, so that a
// host program can check it for every size.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define SAME_HD __host__ __device__
#else
#define SAME_HD
#endif

namespace same {

constexpr int kMaxBlocks = 32;                  // blocks of topics per task (= lanes of a half-wave)

SAME_HD inline int block_len(int K) { return 4 * ((K + 127) / 128); }
SAME_HD inline int blocks_in_use(int K) { return (K + block_len(K) - 1) / block_len(K); }

// Blocks that all end inside the row: their loads need no bounds.
SAME_HD inline bool blocks_fill_row(int K) { return K % block_len(K) == 0; }

// The first topic that lane hl of a half-wave loads in the scan, for blocks of T topics of which nblk are in use.  Lanes
// past the last block (from 17 on at K = 136, from 25 on at K = 200) load that block once more: a block of their own would lie
// behind the row, and behind the matrix in its last row.  The sums they write are never read.
SAME_HD inline int scan_first_topic(int hl, int T, int nblk) { return (hl < nblk ? hl : nblk - 1) * T; }

}  // namespace same
