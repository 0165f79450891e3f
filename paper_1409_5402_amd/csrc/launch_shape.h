// Who works on what in the draw kernels: the arithmetic of their launches and loads, without any device code, so that a
// host program can check it for every size.
#pragma once
#include <stddef.h>
#include <stdint.h>

#ifdef __HIPCC__
#define SAME_HD __host__ __device__
#else
#define SAME_HD
#endif

namespace same {

constexpr int kWave = 64;                       // lanes per workgroup (one wave)
constexpr int kMaxBlocks = 32;                  // blocks of topics per task (= lanes of a half-wave)

SAME_HD inline int block_len(int K) { return 4 * ((K + 127) / 128); }
SAME_HD inline int blocks_in_use(int K) { return (K + block_len(K) - 1) / block_len(K); }

// Blocks that all end inside the row: their loads need no bounds.
SAME_HD inline bool blocks_fill_row(int K) { return K % block_len(K) == 0; }

// The first topic that lane hl of a half-wave loads in the scan, for blocks of T topics of which nblk are in use.  Lanes
// past the last block (from 17 on at K = 136, from 25 on at K = 200) load that block once more: a block of their own would lie
// behind the row, and behind the matrix in its last row.  The sums they write are never read.
SAME_HD inline int scan_first_topic(int hl, int T, int nblk) { return (hl < nblk ? hl : nblk - 1) * T; }

// Tickets: one counter for every kGroups-th workgroup, zero at launch.  The device does one returning atomic on an
// address in about 16 ns whatever asks for it; with one counter for segments of 512 positions those atomics were the
// whole time of small launches (98,000 tasks: 86 us, 26 without) and a fifth of a launch of 9 million tasks
// (0.567 -> 0.466 ms).  Halving shares need some ten tickets per workgroup, all told, and end with small ones.
constexpr int kShareMin = 64;           // (32 and 128 measured within 1 %)
constexpr int kShareAll = 128;          // up to this many positions per workgroup round 0 covers everything
constexpr int kGroups = 32;             // (8 and 64 measured within 1 %)
constexpr int kCounterStride = 32;      // words between two counters: a cache line each
constexpr int kCounterWords = kGroups * kCounterStride;

struct Shares { int32_t waves, first; };        // workgroups of a launch, positions of a share of round 0
inline Shares shares_for(int64_t n, int64_t resident)
{
    Shares s;
    const int64_t per = (n + resident - 1) / resident;
    if (per <= kShareAll) {                                        // fewer workgroups, none with less than a wave's worth
        s.first = per < kWave ? kWave : (int32_t)per;
        s.waves = (int32_t)((n + s.first - 1) / s.first);
    } else {
        s.first = (int32_t)(per / (2 * kShareMin) * kShareMin);
        s.waves = (int32_t)resident;
    }
    return s;
}
SAME_HD inline int32_t share_of_round(int32_t first, int round)
{
    const int32_t s = round < 31 ? (first >> round) & ~31 : 0;
    return s < kShareMin ? kShareMin : s;
}

// The group of a workgroup: runs of eight neighbours, one on each die, belong to the same group, so that a group's shares
// are not one die's.  All groups have a workgroup only from 8 * kGroups workgroups on, and the shares of a group without one
// would never be drawn: whole_groups is the number of workgroups of a launch that hands out tickets.
SAME_HD inline uint32_t ticket_group(uint32_t block) { return (block >> 3) % kGroups; }
inline int64_t whole_groups(int64_t workgroups)
{
    const int64_t n = workgroups / kGroups * kGroups;
    return n < 8 * kGroups ? 8 * kGroups : n;
}

// The share that ticket t of a group stands for, in a launch of `waves` workgroups (a multiple of kGroups): a group's shares
// are every kGroups-th of a round.  From n on nothing is left.
struct Share { int64_t from; int32_t size; };
SAME_HD inline Share share_of_ticket(uint32_t t, uint32_t group, uint32_t waves, int32_t first, int64_t n)
{
    const uint32_t per_round = waves / kGroups;
    Share s;
    s.from = (int64_t)waves * first;                               // round 1
    s.size = share_of_round(first, 1);
    for (int round = 2; t >= per_round && s.from < n; ++round) {
        s.from += (int64_t)waves * s.size; t -= per_round;
        s.size = share_of_round(first, round);
    }
    s.from += ((int64_t)t * kGroups + group) * s.size;
    return s;
}

// Kernels over rows: workgroup b owns `per_block` of them, the last one the rest.  Numbers of rows reach 2^31 - 1, with the hot
// words' copies behind them 2^31 + 2^13: all of it is unsigned, and no sum here passes 2^32 for per_block below 2^30.
struct Rows { uint32_t from, to; };
SAME_HD inline Rows rows_of_block(uint32_t block, uint32_t per_block, uint32_t rows)
{
    Rows r;
    r.from = block * per_block;
    r.to = r.from + per_block < rows ? r.from + per_block : rows;
    return r;
}
SAME_HD inline uint32_t blocks_of_rows(uint32_t rows, uint32_t per_block) { return (rows + per_block - 1u) / per_block; }

// The next document of a loop in strides; false past the last one.  (d + step itself may pass 2^31.)
SAME_HD inline bool next_document(int32_t& d, int32_t step, int32_t D)
{
    if (d >= D - step) return false;
    d += step;
    return true;
}

// Workgroups of one wave that a compute unit's LDS holds: it has 160 KB and hands it out in pieces of 1280 bytes.  The runtime's
// occupancy query divides without rounding up: it says 15 for the 10,496 bytes of K = 512 where 14 run at once (measured: one more
// takes twice the time; 16 at 10,240 bytes, 14 up to 11,520, 12 up to 12,800).  The last 256 workgroups of such a launch
// began when the others had ended, each with its share of round 0: 270,000 documents 21.7 ms instead of 16.9.
inline int lds_groups(int64_t bytes)
{
    const int64_t pieces = (bytes + 1279) / 1280;
    return (int)(160 * 1024 / 1280 / (pieces > 0 ? pieces : 1));
}

// Workgroups of a draw launch on one compute unit, of the `most` that fit.  Beyond 1024 topics a block is read in several
// batches and a wave's theta row again for every pair of tasks (up to 1024 it stays in registers): the rows of the waves on a
// compute unit have to fit its cache of 32 KB, or every pair fetches a row of up to 8 KB from the next one.  News-shaped
// documents at m = 100, ms per sweep:
//   K = 1100   27,000 documents    sixteen 21.2  eight 13.3  six 13.2  four 15.6
//   K = 1540   27,000              sixteen 28.6  eight 19.2  six 18.4  four 21.0
//   K = 2048    5,000, m = 1       twelve 3.08   eight 3.01  six 2.84  four 2.72
// At K = 1024 fewer are slower: 40,000 documents twelve 6.4, ten 6.8, seven 8.5.
inline int groups_per_unit(int K, int most)
{
    const int fit = K <= 1024 ? most : (32 << 10) / (4 * K);       // 7 down to 4
    return fit < most ? fit : most;
}

// Whether the document of a draw wave's row of counts also has its row of theta in LDS, for the reload of a step's block.
// Sixteen waves' rows of theta and their pieces of phi do not fit the 32 KB of a compute unit's cache for
// long, and every load of a step takes it a cycle per lane; the row costs up to a quarter of the waves and some registers.
// ms per draw without / with, 2 million tokens in documents of 60 tokens from a flat posterior and in documents of 330 with topics formed:
//   up to 287 topics                 K = 260  m = 1 0.278 / 0.297, 0.270 / 0.286   m = 16 0.875 / 0.899, 0.773 / 0.803: never
//   to 512, aligned, whole blocks    K = 300  m = 1 0.291 / 0.284, 0.268 / 0.263   m = 16 0.984 / 0.874, 0.718 / 0.735
//                                    K = 448  m = 16 1.102 / 1.058, 0.814 / 0.787   K = 512  m = 100 3.440 / 3.269, 1.770 / 1.734
//   aligned, the row ends in a block K = 340  m = 1 0.322 / 0.343, 0.294 / 0.299   K = 500  m = 1 0.480 / 0.486, 0.393 / 0.400: never
//   any alignment                    K = 333  m = 1 0.349 / 0.320, 0.320 / 0.301   m = 16 1.202 / 0.989, 0.868 / 0.804
//   to 640, any alignment            K = 601  m = 1 0.650 / 0.586, 0.545 / 0.504   m = 100 5.324 / 4.451, 2.454 / 2.487
//   to 768, aligned                  K = 768  m = 1 0.685 / 0.650, 0.553 / 0.541   m = 16 1.770 / 1.525, 1.100 / 1.016
//           any alignment            K = 701  m = 1 0.686 / 0.653, 0.566 / 0.546   m = 16 1.729 / 1.646, 1.175 / 1.124
//                                    m = 100 5.357 / 5.372, 2.581 / 2.693
//   to 896, aligned                  K = 896  (three waves per SIMD) m = 1 0.857 / 0.785, 0.706 / 0.640   m = 100 6.055 / 5.810, 2.770 / 2.663
//           any alignment            K = 895  m = 1 1.051 / 0.928, 0.858 / 0.771   m = 16 2.274 / 1.992, 1.391 / 1.270
//                                    m = 100 6.396 / 6.075, 2.891 / 2.903
// From 897 topics on a block is more than one batch of loads and a wave would need 16 KB.
SAME_HD constexpr bool theta_rows_some(int quads) { return quads >= 3 && quads <= 7; }
SAME_HD constexpr bool theta_rows_all(int quads, bool aligned) { return quads >= 5 ? quads <= 7 : quads == 4 && !aligned; }
inline bool theta_rows(int K)
{
    const int quads = block_len(K) / 4;
    if (quads == 3 || quads == 4) return K >= 288 && (K % 4 != 0 || blocks_fill_row(K));
    return theta_rows_some(quads);
}

// The topic totals' memory, in 64-bit words: the copies that the documents' workgroups add to, then the totals.  The copies come
// first because they are cleared with 16-byte stores: behind the totals they would start half-way between two for every odd K.
inline int nk_copies_for(int K) { return K <= 128 ? 8 : (K <= 256 ? 4 : (K <= 512 ? 2 : 1)); }
struct TotalsLayout { size_t copies, copy_words, totals, words; };
inline TotalsLayout totals_layout(int K)
{
    const size_t n = (size_t)nk_copies_for(K) * (size_t)K;
    return {0, n, n, n + (size_t)K};
}

// How the totals and theta (update_kernels.h) go over n_dk.  `fold` documents at a time have a multiple of four counts and start on
// a 16-byte boundary, whatever the number of topics: a thread owns the same 16 bytes of every `fold` documents, four topics that
// depend on its unit alone.  Units beyond a workgroup's 256 threads are other workgroups' (turns), split so that few threads
// are left over; groups of `per` threads take `fold` documents each.
struct TotalsSplit { int fold, units, turns, per, groups; };
inline TotalsSplit totals_split(int K)
{
    TotalsSplit s;
    s.fold = K % 4 == 0 ? 1 : (K % 2 == 0 ? 2 : 4);
    s.units = s.fold * K / 4;
    int busy = 0;
    const int least = (s.units + 255) / 256;
    for (int turns = least; turns <= (least > 1 ? least + 3 : 1); ++turns) {
        const int per = (s.units + turns - 1) / turns;
        if (256 / per * per > busy) { busy = 256 / per * per; s.turns = turns; s.per = per; s.groups = 256 / per; }
    }
    return s;
}
struct TotalsBlocks { uint32_t rows, rows_per_block, blocks; };    // rows of `fold` documents; workgroups, all turns
inline TotalsBlocks totals_blocks(const TotalsSplit& s, uint32_t D)
{
    // at least a turn of four rows per thread, and at most some 512 workgroups (64-bit atomics per topic)
    TotalsBlocks b;
    b.rows = D / (uint32_t)s.fold;
    const uint32_t at_once = 4u * (uint32_t)s.groups;
    b.rows_per_block = blocks_of_rows(b.rows, s.turns < 8 ? 512u / (uint32_t)s.turns : 64u);
    if (b.rows_per_block < at_once) b.rows_per_block = at_once;
    b.blocks = blocks_of_rows(b.rows, b.rows_per_block);
    if (b.blocks == 0 && D > 0) b.blocks = 1;                      // fewer documents than one row: the first workgroup's (the rest of D / fold)
    b.blocks *= (uint32_t)s.turns;
    return b;
}

// The pool of chunks that continue full pair-list slots: each of `waves` workgroups owns `share` of its `chunks`, the rest is
// handed out in batches by a counter.  The counter counts batches: a workgroup adds to it once more before it sees that the
// pool is used up, and the Poisson form has a workgroup for every 64 tasks, up to 2^25 of them.  A counter of
// chunks came round from 2^24 workgroups on and handed out chunks that already held other tasks' counts.
constexpr uint32_t kChunkBatch = 256;

// A workgroup's own share, in a launch of n tasks: half a chunk per task, a converged sweep needs less, and at most half the pool.
// (A share of half the pool whatever the launch needs, four chunks per task, left the chunks in use spread over eight times
// the memory, 15 GB for 60 million tasks: the reduction, which follows them in word order, took 6.2 ms, 2.4 ms with chunks
// from the counter alone.  One chunk per task measures the same as a half; batches of 1024 cost the Poisson form a third.)
inline uint32_t chunk_share(uint32_t chunks, int64_t n, int64_t waves)
{
    const int64_t own = n / 2 < (int64_t)(chunks / 2) ? n / 2 : (int64_t)(chunks / 2);
    return (uint32_t)(own / waves);
}

struct Chunks { uint32_t next, end; };          // empty: the pool is used up
SAME_HD inline Chunks chunk_batch(uint32_t taken, uint32_t waves, uint32_t share, uint32_t chunks)
{
    // a pool has fewer than 2^31 chunks and half of it at most is the workgroups' own: no sum below reaches 2^32 before the
    // limit on `taken` ends it.  (A comparison with the number of batches kept two more scalar registers alive: 1 % at K = 256.)
    Chunks c = {0u, 0u};
    const uint32_t next = waves * share + taken * kChunkBatch;
    if (taken < (1u << 31) / kChunkBatch && next < chunks) {
        c.next = next;
        c.end = chunks - next < kChunkBatch ? chunks : next + kChunkBatch;
    }
    return c;
}

// Nonzero number `first + at` of a document of n, past the end its last one.  A document may have all of the 2^31 - 1 nonzeros
// of a matrix, and the E-step loads rounds ahead, up to kVbAhead numbers past the end: they are unsigned.
constexpr uint32_t kVbAhead = 48;       // three rounds of four groups of four
SAME_HD inline uint32_t vb_nonzero(uint32_t first, uint32_t at, uint32_t n) { return first + at < n ? first + at : n - 1u; }

// Whether the normaliser's workgroups share the words out among the dies (sddmm_kernel.h): where phi is several times a die's
// 4 MB of cache and its rows are long enough to outweigh the list of nonzeros that each wave then makes, and documents have
// enough words for an eighth of them to be a run.  ms without / with, 30,000 news-shaped documents:
//   V = 100,000   K = 128 0.178 / 0.212   150 0.261 / 0.276   200 0.361 / 0.326   (100,000 documents) 256 1.46 / 1.20
//   K = 256       V = 30,000 0.344 / 0.302   60,000 0.419 / 0.338   100,000 and documents of 60 tokens 0.098 / 0.110
//   K = 512       V = 8,000 0.611 / 0.488   20,000 0.809 / 0.546        K = 1000   V = 10,000 1.64 / 0.91
constexpr int kSddmmSliced = 176;       // not up to this many topics
inline bool sddmm_sliced(int64_t V, int K, int64_t nnz, int64_t D)
{
    return K > kSddmmSliced && V * K >= 3000000 && nnz >= 65536 && nnz >= 64 * D;
}

// Nonzeros that a wave of the normaliser looks through: enough to share its start, few enough for four waves per SIMD.
constexpr int kSddmmStretch = 512;
inline int sddmm_stretch(bool sliced, int64_t nnz)
{
    if (sliced) return kSddmmStretch;
    int n = 64;
    while (n > 16 && nnz < (int64_t)n * 4096) n /= 2;
    return n;
}

}  // namespace same
