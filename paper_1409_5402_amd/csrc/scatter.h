// What the two draw kernels (multinomial form: draw_kernel.h, Poisson form: poisson_kernel.h) share:
// the launch arguments, the scatter of a task's counts (Algorithm 3, the two accumulation lines) and
// the kernel that adds the recorded (topic, count) pairs to the word rows.
#pragma once
#include "launch_shape.h"
#include "rng_binom.h"

namespace same {

constexpr int kSlotWords = 4;           // words of a pair-list slot: up to 3 (topic, count) pairs and a header
constexpr int kPairWords = 16;          // words of a chunk that continues it: up to 15 pairs and a header
constexpr uint32_t kFirstPair = kPairWords - kSlotWords;   // a slot is filled and written like the last quarter of a chunk
constexpr uint32_t kPairLink = 0x80000000u;   // header bit: slot or chunk is full and the chunk named by the other bits goes on
constexpr int kPairShift = 11;          // a pair is topic | count << 11 (topics < 2048, counts < 2^21)
constexpr int kWalkSteps = 8;           // pmf steps per trip of a draw machine
constexpr float kPieceMean = 32.0f;     // a binomial / Poisson variable whose mean exceeds this is cut into pieces
constexpr int kPoolMin = 8;             // waiting multi-piece variables that trigger a pass shared by the wave

// Variables of several pieces wait for kPoolMin of them, or for kPoolTrips trips: from a flat posterior five of the 64
// lanes waited at any time for eight to gather.  (1, 2, 4, 8 trips: 9.62, 9.59, 9.80, 10.4 ms there against 12.4 without
// the limit; converged 11.02, 10.83, 10.73, 10.73 ms.)
constexpr int kPoolTrips = 4;

struct DrawArgs {
    int64_t         n;          // tasks in this launch
    uint32_t*       counter;    // multinomial form: [kCounterWords] tickets for shares of the positions (zero at launch)
    int32_t         first;      // multinomial form: launch positions of a workgroup's first share
    const int32_t*  heavy;      // multinomial form: [n_heavy] ids of the tasks of at least heavy_from tokens
    int32_t         n_heavy;
    uint32_t        heavy_from;
    const int32_t*  t_doc;      // [n_tasks] document of the task
    const int32_t*  t_word;     // [n_tasks] word of the task
    const uint32_t* t_g;        // [n_tasks] tokens in the task's group
    const int32_t*  order;      // Poisson form: [n_tasks] task id handled at each launch position
    uint32_t*       cost;       // Poisson form: [n_tasks] out: trips this task was busy for (null: not recorded)
    const int64_t*  ids;        // debug launches: task ids to draw instead (else null)
    const float*    theta;      // [D][K]   (unused when weights are uniform)
    const float*    phi;        // [V][K]
    uint32_t*       ndk;        // [D][K]   (debug launches: [n][K] output rows)
    uint32_t*       nwk;        // [V][K] or null
    uint32_t*       pairs;      // [n_slots][kSlotWords] pair list in word order, or null (update nwk directly)
    const int32_t*  t_slot;     // [n_tasks] slot of each task in the pair list, -1 for a task without one
    uint32_t*       chunks;     // [n_chunks][kPairWords] pool of chunks that continue full slots, or null
    uint32_t*       chunk_counter;  // batches taken from the common part of the pool (zero at launch)
    uint32_t        n_chunks;   // chunks in the pool (below 2^31)
    uint32_t        chunk_share;    // chunks that are each workgroup's own; the rest is taken from the counter in batches
    int32_t         K;
    uint32_t        m;          // copies per token (multinomial form)
    float           mf;         // copies per token (Poisson form: any positive real)
    uint32_t        seed_lo, seed_hi, pass;
    int32_t         V;          // rows of nwk that are words; the copies of the hot words' rows follow them
    uint32_t*       hot_used;   // set when a copy of a hot word's row has taken a count (zero at launch)
    const int16_t*  hot_of;     // [V] index of a hot word among the hot words, -1 for the others (null: no hot words)
#ifdef SAME_STATS
    unsigned long long* stats;  // profiling builds only: event counters
#endif
};

#ifdef SAME_STATS
#define SAME_COUNT(a, i, v) do { if ((a).stats) atomicAdd((a).stats + (i), (unsigned long long)(v)); } while (0)
#else
#define SAME_COUNT(a, i, v) do { } while (0)
#endif

// Additions to LDS and to device memory, with the kind of memory in the pointer's type.  Two branches that add to the one and to
// the other through plain pointers become one flat addition to a selected address: a dozen more instructions for the
// address, and whatever waits for LDS next also waits for the additions that went to memory.
__device__ __forceinline__ void add_lds(uint32_t* p, uint32_t v)
{
    __hip_atomic_fetch_add((__attribute__((address_space(3))) uint32_t*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void add_global(uint32_t* p, uint32_t v)
{
    __hip_atomic_fetch_add((__attribute__((address_space(1))) uint32_t*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Rows of [V][K] that very many tasks update at once (the most frequent words: their tasks spread copies
// over many topics, fill their pair-list slot and send the rest straight to the row) are a bottleneck of
// their own: atomics on a handful of lines are served by a handful of memory channels, one after the other.
// Such a word therefore gets kHotCopies private copies of its row behind the matrix; a workgroup adds to the
// copy picked by its index, and the parameter update adds the copies to the word's row and clears them.
constexpr int kHotMax = 256;            // words that may be hot (those holding at least 1/256 of all tokens)
constexpr int kHotCopies = 32;          // copies of a hot word's row

// Where the counts of one task go.  Every placed count goes to the document's row at once (an atomic:
// several waves may hold tasks of one document).  The word's row is updated either the same way or, when
// the launch has a pair list, later by word_reduce (counts_kernel): the task records (topic, count) in its slot of
// the list (slots are in word order), so that the scattered updates of [V][K] become one streaming pass
// with all updates of a row close together.  A slot is four words: three pairs and, last, a header.  A task that
// places more than three pairs continues in chunks of 15 pairs and a header taken from a pool: the header of a full
// slot or chunk names the chunk that follows it, the header of the last one tells its number of pairs.  When the
// pool is used up the remaining counts go straight to the word's row.  The last pairs are kept in three registers that
// shift, and written four words at a time with one 16-byte store: the memory system handles a 16-byte write as fast as
// a 4-byte one.  So a task of up to three pairs costs one scattered 16-byte store, and the pass over the list reads
// 16 bytes for it.  (Slots of 16 words took a second scattered store for the header and 64 bytes to read for every
// task, most of which place one to four pairs.)  Chunks are consecutive for the lanes of a wave: dense stores.

// The last three pairs of a task, the newest in p2: the npairs & 3 of them that are not yet written are among them.
struct Staged {
    uint32_t p0 = 0u, p1 = 0u, p2 = 0u;
    __device__ __forceinline__ void push(uint32_t pair)
    {
        const uint32_t a = p1, b = p2;
        p0 = a; p1 = b; p2 = pair;
    }
};

// The place of the next four pairs is kept as an address: computing it from a slot number again for every store took
// some ten vector instructions in nearly every trip of the draw machine (some lane stores in most).
struct Scatter {
    uint32_t drow;      // row of a.ndk that takes the counts (the document; debug launches: the task's output row)
    uint4* dst;         // where the next four words go, in a slot of the pair list or a chunk; null: the task has no slot
    uint32_t npairs;    // pairs in that chunk (in a slot: kFirstPair more than there are)

    // straight to row w of the word counts, or to this workgroup's copy of it if the word is hot
    __device__ __forceinline__ void emit_row(const DrawArgs& a, int k, uint32_t n, int32_t w) const
    {
        const int hot = a.hot_of ? (int)a.hot_of[w] : -1;
        size_t row = (size_t)w;
        if (hot >= 0) {
            row = (size_t)a.V + (size_t)(blockIdx.x % kHotCopies) * kHotMax + (size_t)hot;
            *a.hot_used = 1u;
        }
        add_global(a.nwk + row * a.K + k, n);
    }
    // the word's half of a count (the caller adds it to the document's row itself)
    __device__ __forceinline__ void emit_word(const DrawArgs& a, int k, uint32_t n, int32_t w, Staged& t)
    {
        if (dst != nullptr && npairs < (uint32_t)(kPairWords - 1)) {
            const uint32_t pair = (uint32_t)k | (n << kPairShift);
            if ((npairs & 3u) == 3u) { *dst = make_uint4(t.p0, t.p1, t.p2, pair); dst += 1; }   // a chunk's pairs 0-3, 4-7 or 8-11
            t.push(pair);
            npairs += 1;
        } else if (a.nwk != nullptr) {
            emit_row(a, k, n, w);                                  // no slot, or full and no chunk to go on with
        }
    }
    __device__ __forceinline__ bool full() const { return dst != nullptr && npairs >= (uint32_t)(kPairWords - 1); }
    // a full slot or chunk (its last three pairs are not yet written) goes on in chunk idx of the pool
    __device__ __forceinline__ void extend(const DrawArgs& a, uint32_t idx, const Staged& t)
    {
        *dst = make_uint4(t.p0, t.p1, t.p2, kPairLink | idx);
        dst = reinterpret_cast<uint4*>(a.chunks + (size_t)idx * kPairWords);
        npairs = 0;
    }
    // the unwritten pairs and the header of the last slot or chunk: how many pairs it holds
    __device__ __forceinline__ void close(bool live, const Staged& t) const
    {
        if (dst != nullptr && live) {
            // the j unwritten pairs come first in their quad; words past the last pair are never read
            const uint32_t q = npairs >> 2, j = npairs & 3u;
            const uint32_t x0 = t.p0, x1 = t.p1, x2 = t.p2;
            const uint32_t w0 = j == 1u ? x2 : (j == 2u ? x1 : x0), w1 = j == 2u ? x2 : x1;
            if (j != 0u || q == 3u) *dst = make_uint4(w0, w1, x2, npairs);   // q = 3: the header shares the last quad
            if (q != 3u) reinterpret_cast<uint32_t*>(dst)[kPairWords - 1 - 4u * q] = npairs;
        }
    }
};

template <bool DEBUG>
__device__ __forceinline__ Scatter make_scatter(const DrawArgs& a, int64_t row, int64_t tau, int32_t d)
{
    Scatter s;
    s.drow = DEBUG ? (uint32_t)row : (uint32_t)d;
    s.dst = nullptr;
    s.npairs = kFirstPair;
    if (!DEBUG && a.pairs != nullptr) {
        const int32_t slot_id = a.t_slot[tau];
        if (slot_id >= 0) s.dst = reinterpret_cast<uint4*>(a.pairs + (size_t)slot_id * kSlotWords);
    }
    return s;
}

// A wave's chunks: its own share of the pool (chunk_share: the counter's atomics are returning ones on one address, 16 ns
// each), then batches from the counter.
struct ChunkSupply {
    uint32_t next, end;     // not yet handed out
    bool dry;               // the pool has none left for this wave
    __device__ __forceinline__ explicit ChunkSupply(const DrawArgs& a)
    {
        next = end = 0u;
        dry = a.chunks == nullptr;
        if (!dry) { next = blockIdx.x * a.chunk_share; end = next + a.chunk_share; }
    }
    // Whole wave: lanes that need one (their slot or chunk is full) go on in a new chunk.
    __device__ __forceinline__ void give(const DrawArgs& a, int lane, Scatter& sc, bool need, const Staged& staged)
    {
        if (dry) return;
        const uint64_t need_mask = __ballot(need);
        if (need_mask == 0) return;
        const uint32_t cnt = (uint32_t)__popcll((unsigned long long)need_mask);
        if (end - next < cnt) {
            uint32_t taken = 0;
            if (lane == 0) taken = atomicAdd(a.chunk_counter, 1u);
            const Chunks c = chunk_batch((uint32_t)__builtin_amdgcn_readfirstlane((int)taken), gridDim.x, a.chunk_share, a.n_chunks);
            next = c.next; end = c.end;
            dry = next == end;
            if (lane == 0) SAME_COUNT(a, 14, 1);                   // batches of chunks taken
        }
        const uint32_t mine = next + (uint32_t)__popcll((unsigned long long)(need_mask & ((1ull << lane) - 1ull)));
        if (need && mine < end) { sc.extend(a, mine, staged); SAME_COUNT(a, 15, 1); }
        next = end - next < cnt ? end : next + cnt;
    }
};

// Adds the recorded pairs to the word rows.  Slots are in word order and exist only for words with
// at least kSlotMinTasks tasks: a workgroup takes kReduceChunk consecutive slots, sums the pairs of
// the first `rows` words it meets in an LDS table and sends the rest straight to [V][K]; the table is
// then added to the rows it stands for.  A range of few words keeps several copies of their rows, one for every so many
// threads and a word apart in the banks: tasks of one word have their large counts at the same topics.  A thread reads
// a slot with one 16-byte load, a chunk with four, and starts with the quad of a chunk picked by its index.  Bound: memory,
// 20 bytes per slot in a stream and a line per chunk.
constexpr int kReduceChunk = 512;       // slots per workgroup of a long list; shorter lists take fewer (reduce_chunk).  2048, 1024 and 512
                                        // measured 0.48, 0.45 and 0.43 ms for 20 million slots of which half go on in a chunk
                                        // (more words than rows in a range send their counts straight to memory)
constexpr int kSlotMinTasks = 2;         // (32 measured 1.5 % slower on the resident matrix and 5 % on a minibatch: the direct
                                        // updates of rare words are atomics on lines that have long left the cache)
constexpr int kReduceThreads = kReduceChunk / 2;    // at most: two slots per thread, the kernel waits on its loads, many waves hide that

struct ReduceArgs {
    const uint32_t* pairs; const uint32_t* chunks; uint32_t n_chunks;
    const int32_t* slot_word; int64_t n;   // [n] slots
    int K, rows, chunk; uint32_t* nwk;
};

// The slots of workgroup `block`; tab: [rows][K + 1] of LDS.
__device__ __forceinline__ void word_reduce(const ReduceArgs& a, uint32_t block, uint32_t* tab)
{
    const uint32_t* __restrict__ pairs = a.pairs;
    const uint32_t* __restrict__ chunks = a.chunks;
    const int32_t* __restrict__ slot_word = a.slot_word;
    uint32_t* __restrict__ nwk = a.nwk;
    const uint32_t n_chunks = a.n_chunks;
    const int64_t n = a.n;
    const int K = a.K, rows = a.rows, chunk = a.chunk;
    const int64_t s0 = (int64_t)block * chunk;
    const int64_t s1 = s0 + chunk < n ? s0 + chunk : n;
    const int32_t w0 = slot_word[s0];
    const int32_t w1 = slot_word[s1 - 1];                          // the last word of the range
    const int stride = K + 1;
    const int words = w1 - w0 < rows ? w1 - w0 + 1 : rows;         // words with rows in the table
    int copies = 1;
    while (2 * copies * words <= rows && copies < 32) copies *= 2;
    const int mine = threadIdx.x & (copies - 1);
    for (int i = threadIdx.x; i < words * copies * stride; i += blockDim.x) tab[i] = 0u;
    __syncthreads();
    for (int64_t s = s0 + threadIdx.x; s < s1; s += blockDim.x) {
        const uint4 slot = reinterpret_cast<const uint4*>(pairs)[s];
        const int32_t w = slot_word[s];
        const bool in_tab = w - w0 < rows;
        uint32_t* in_lds = tab + (in_tab ? ((w - w0) * copies + mine) * stride : 0);
        auto add = [&](uint32_t p) {
            const uint32_t k = p & ((1u << kPairShift) - 1u), n = p >> kPairShift;
            if (in_tab) add_lds(in_lds + k, n); else add_global(nwk + (size_t)w * K + k, n);
        };
        uint32_t head = slot.w;
        {
            const uint32_t cnt = (head & kPairLink) ? 3u : head - kFirstPair;   // 0 to 3
            if (cnt > 0u && cnt <= 3u) add(slot.x);
            if (cnt > 1u && cnt <= 3u) add(slot.y);
            if (cnt == 3u) add(slot.z);
        }
        const uint32_t t = threadIdx.x & 3u;                       // which quad of a chunk this thread starts with
        while ((head & kPairLink) != 0u && (head & ~kPairLink) < n_chunks) {   // the chunks that continue the slot
            const uint4* __restrict__ s4 = reinterpret_cast<const uint4*>(chunks + (size_t)(head & ~kPairLink) * kPairWords);
            uint4 q[4];                                            // the whole chunk: four 16-byte loads in flight
#pragma unroll
            for (uint32_t i = 0; i < 4u; ++i) q[i] = s4[(t + i) & 3u];
            head = t == 0u ? q[3].w : (t == 1u ? q[2].w : (t == 2u ? q[1].w : q[0].w));
            const uint32_t cnt = ((head & kPairLink) != 0u || head > (uint32_t)(kPairWords - 1)) ? (uint32_t)(kPairWords - 1) : head;
#pragma unroll
            for (uint32_t i = 0; i < 4u; ++i) {
                const uint32_t first = 4u * ((t + i) & 3u);        // index of the quad's first pair
                const uint32_t p[4] = {q[i].x, q[i].y, q[i].z, q[i].w};
#pragma unroll
                for (uint32_t j = 0; j < 4u; ++j) if (first + j < cnt) add(p[j]);
            }
        }
    }
    __syncthreads();
    // A word whose slots all lie in this workgroup's range is updated by no other workgroup: the others that reduce own other
    // slots, those of the same launch that work on documents never write n_wk, and the draw has ended.  Its row takes plain
    // additions.  Only the first and the last word of the range may share their rows with the neighbours.
    const bool first_shared = s0 > 0 && slot_word[s0 - 1] == w0;
    const bool last_shared = s1 < n && slot_word[s1] == w1;
    uint32_t* base = nwk + (size_t)w0 * K;                         // row w0 + r, topic k is at base[r*K + k]
    for (int i = threadIdx.x; i < words * K; i += blockDim.x) {
        const int r = i / K, k = i - r * K;
        uint32_t v = 0u;
        for (int c = 0; c < copies; ++c) v += tab[(r * copies + c) * stride + k];
        if (v == 0u) continue;                                     // only rows of real words hold counts
        const int32_t w = w0 + r;
        if ((w == w0 && first_shared) || (w == w1 && last_shared)) atomicAdd(base + i, v);
        else base[i] += v;
    }
}

// Slots per workgroup of 256 threads: one per thread while that is at most 512 workgroups (two per compute unit), else two
// (kReduceChunk).  The table shrinks with it.
inline int reduce_chunk(int64_t n) { int c = 256; while (c < kReduceChunk && (int64_t)c * 512 < n) c *= 2; return c; }
inline int reduce_rows(int K, int chunk) { const int r = 8 * chunk / K; return r < 1 ? 1 : (r > 64 ? 64 : r); }

}  // namespace same
