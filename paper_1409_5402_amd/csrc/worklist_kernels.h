// Device-side construction of the draw work list from a CSC matrix (columns = documents).
//
// A nonzero (d, w, c) stands for c tokens with identical conditionals; its tokens are drawn in
// groups ("tasks") of at most G.  These kernels validate the matrix and produce, without a host
// copy of the matrix: the document of every nonzero, the tasks (document, word, group size) in
// storage order, the first task of every tile of documents, and the slots of the word-ordered pair
// list.  The exclusive sums and the stable sort by word that this takes are kernels of this file too.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "launch_shape.h"

namespace same {

// Filled by the kernels below; first_bad is the smallest (index << 2 | code) over all defects found,
// ~0 if the matrix is sound: code 1 = column pointer decreases (index = document), 2 = word id out
// of range, 3 = count not an integer in [1, 2^24) (index = nonzero).
constexpr int kSizeClasses = 49;           // groups of up to 2^24 tokens
struct BuildStats {
    unsigned long long tokens;
    unsigned long long n_tasks;
    unsigned long long first_bad;
    unsigned long long max_doc_tokens;     // largest number of tokens in one document, and that document
    unsigned long long max_word_tokens;    // largest number of tokens of one word, and that word
    uint32_t max_doc, max_word;
    uint32_t max_group;
    uint32_t n_slots;
    uint32_t n_hot;                        // words holding at least 1/kHotMax of all tokens
    uint32_t n_heavy;                      // tasks of at least heavy_from tokens (wl_heavy)
    uint32_t sizes[kSizeClasses];          // tasks by size class (size_class)
};

// Size class of a group of g tokens: 0 for one token, then two classes per power of two (2, 3, 4-5, 6-7, 8-11, ...).
__host__ __device__ inline int size_class(uint32_t g)
{
    if (g < 2u) return 0;
    int e = 1;
    while ((g >> (e + 1)) != 0u) ++e;
    return 2 * e - 1 + (int)((g >> (e - 1)) & 1u);
}
__host__ __device__ inline uint32_t class_start(int c) { return c == 0 ? 1u : (2u + (uint32_t)((c - 1) & 1)) << ((c - 1) >> 1); }

// The heavy tasks of a matrix: those of the largest size classes, as many whole classes as hold at most 1/kHeavyShare of the
// tasks.  The draw starts with them (draw_kernel.h).  Returns the smallest heavy group; ~0 if there are none.
constexpr uint32_t kHeavyShare = 256;      // (1/16, 1/64, 1/256, 1/1024: from a flat posterior 7.24, 7.30, 7.55, 7.7 ms against 9.4 without a
                                           // list; converged 10.43, 10.21, 10.08, 10.05 ms against 10.05: heavy tasks taken out of their
                                           // documents' order cost row changes and scans of single tasks)
__host__ __device__ inline uint32_t heavy_from(const uint32_t* sizes, unsigned long long n_tasks)
{
    unsigned long long sum = 0ull;
    uint32_t from = ~0u;
    for (int c = kSizeClasses - 1; c > 0; --c) {
        sum += sizes[c];
        if (sum * kHeavyShare > n_tasks) break;
        if (sizes[c]) from = class_start(c);
    }
    return from;
}

__global__ void wl_init_stats(BuildStats* s)
{
    s->tokens = 0ull; s->n_tasks = 0ull; s->first_bad = ~0ull; s->max_group = 0u; s->n_slots = 0u;
    s->max_doc_tokens = 0ull; s->max_word_tokens = 0ull; s->max_doc = ~0u; s->max_word = ~0u; s->n_hot = 0u; s->n_heavy = 0u;
    for (int c = 0; c < kSizeClasses; ++c) s->sizes[c] = 0u;
}

// One pass over the matrix, 16 lanes per document: column pointers, word ids and counts are checked, every nonzero gets
// its document and its number of tasks, every document its token total (only entries that passed are counted; the
// largest values the count matrices can reach are m times the totals).  Ranges are clamped to the matrix, so that broken
// column pointers are reported and not followed.  (A search of the column pointers per nonzero and separate passes for
// the totals of documents and words took 0.32, 0.10 and 0.43 ms for a minibatch of 7.7 million nonzeros.)
// ntask has nnz + 1 entries; the last one is set to 0 so that an exclusive sum over all of them ends with the total.
// Held to 32 registers (the attribute counts half of them): beside a draw of four waves of 120 a SIMD has no more.  us per step of a
// stream at K = 200, documents of 354 tokens, with 34 and 31: 959 and 910; K = 300 and 60 tokens 826 and 768.
constexpr int kDocLanes = 16;
__global__ __launch_bounds__(256) __attribute__((amdgpu_num_vgpr(16))) void wl_scan_docs(const int32_t* __restrict__ colptr, const int32_t* __restrict__ rowidx,
                                                    const float* __restrict__ val, int32_t D, int64_t nnz, int32_t V, uint32_t G,
                                                    int32_t* __restrict__ nz_doc, uint32_t* __restrict__ ntask,
                                                    unsigned long long* __restrict__ doc_tok, BuildStats* s)
{
    __shared__ uint32_t sh_sizes[kSizeClasses];                    // (a sweep's draw beside it may hold all LDS: at K = 256 sixteen
                                                                   // workgroups a compute unit, eight pieces of 1,280 bytes each)
    for (int c = threadIdx.x; c < kSizeClasses; c += 256) sh_sizes[c] = 0u;
    __syncthreads();
    unsigned long long tok = 0ull, tasks = 0ull, doc_max = 0ull;
    uint32_t gmax = 0u, ones = 0u;
    const int sub = threadIdx.x & (kDocLanes - 1);
    const int32_t docs_at_once = (int32_t)(gridDim.x * (256 / kDocLanes));
    if (blockIdx.x == 0 && threadIdx.x == 0) ntask[nnz] = 0u;
    int32_t d = (int32_t)(blockIdx.x * (256 / kDocLanes) + threadIdx.x / kDocLanes);
    if (d < D) do {
        const int64_t c0 = colptr[d], c1 = colptr[d + 1];
        if (c1 < c0 && sub == 0) atomicMin(&s->first_bad, ((unsigned long long)d << 2) | 1ull);
        const int64_t lo = c0 < 0 ? 0 : c0, hi = c1 < nnz ? c1 : nnz;
        unsigned long long mine = 0ull;
        for (int64_t i = lo + sub; i < hi; i += kDocLanes) {
            nz_doc[i] = d;
            const int32_t w = rowidx[i];
            const float c = val[i];
            uint32_t nt = 0u;
            const bool number = c >= 1.0f && c < 16777216.0f;
            if (w < 0 || w >= V) {
                atomicMin(&s->first_bad, ((unsigned long long)i << 2) | 2ull);
            } else if (!number || c != floorf(c)) {
                atomicMin(&s->first_bad, ((unsigned long long)i << 2) | 3ull);
            } else {
                const uint32_t ci = (uint32_t)c;
                nt = (ci + G - 1u) / G;
                tok += ci; tasks += nt; mine += ci;
                gmax = max(gmax, ci < G ? ci : G);
                const uint32_t full = ci / G, rest = ci - full * G;   // the groups: full ones of G tokens and one of the rest
                if (full > 0u) { if (G == 1u) ones += full; else atomicAdd(&sh_sizes[size_class(G)], full); }
                if (rest > 0u) { if (rest == 1u) ones += 1u; else atomicAdd(&sh_sizes[size_class(rest)], 1u); }
            }
            ntask[i] = nt;
        }
        for (int o = kDocLanes / 2; o > 0; o >>= 1) mine += __shfl_xor(mine, o);
        if (sub == 0) doc_tok[d] = mine;
        doc_max = mine > doc_max ? mine : doc_max;
    } while (next_document(d, docs_at_once, D));
    if (ones) atomicAdd(&sh_sizes[0], ones);
    for (int o = 32; o > 0; o >>= 1) {
        tok += __shfl_xor(tok, o); tasks += __shfl_xor(tasks, o);
        gmax = max(gmax, __shfl_xor(gmax, o));
        const unsigned long long other = __shfl_xor(doc_max, o);
        doc_max = other > doc_max ? other : doc_max;
    }
    if ((threadIdx.x & 63) == 0) {
        if (tok) atomicAdd(&s->tokens, tok);
        if (tasks) atomicAdd(&s->n_tasks, tasks);
        if (gmax) atomicMax(&s->max_group, gmax);
        if (doc_max) atomicMax(&s->max_doc_tokens, doc_max);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < kSizeClasses; c += 256) if (sh_sizes[c]) atomicAdd(&s->sizes[c], sh_sizes[c]);
}

// Token totals per word from the tasks in word order: a wave takes 64 consecutive ones, adds up the runs of one word
// lane by lane and sends each run's total with one atomic (the most frequent words would otherwise receive one per
// document on a single address).
__global__ __launch_bounds__(256) void wl_word_tokens(const int32_t* __restrict__ keys, const int32_t* __restrict__ tasks,
                                                      const uint32_t* __restrict__ t_g, int64_t n,
                                                      unsigned long long* __restrict__ word_tok)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const int32_t key = i < n ? keys[i] : -1;
    uint32_t sum = i < n ? t_g[tasks[i]] : 0u;                     // 64 groups of less than 2^24 tokens
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t up = __shfl_up(sum, o);
        const int32_t kup = __shfl_up(key, o);
        if (lane >= o && kup == key) sum += up;
    }
    const int32_t next = __shfl_down(key, 1);
    if (key >= 0 && (lane == 63 || next != key)) atomicAdd(word_tok + key, (unsigned long long)sum);
}

// The same from the nonzeros directly, one atomic each: for a matrix whose pair list did not fit.
__global__ __launch_bounds__(256) void wl_word_tokens_plain(const int32_t* __restrict__ rowidx, const float* __restrict__ val,
                                                            int64_t nnz, unsigned long long* __restrict__ word_tok)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nnz; i += stride)
        atomicAdd(word_tok + rowidx[i], (unsigned long long)val[i]);
}

// The largest word total, and the hot words: those that hold at least one part in hot_max of all tokens (so at most
// hot_max of them).  They are numbered in the order the threads arrive; the numbering only names the copies of their
// rows, no result depends on it.  hot_of[w] = number or -1.
__global__ __launch_bounds__(256) void wl_words(const unsigned long long* __restrict__ word_tok, int32_t V, int32_t hot_max,
                                                int16_t* __restrict__ hot_of, BuildStats* s)
{
    __shared__ unsigned long long sh[256];
    const int32_t w = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    const unsigned long long tot = w < V ? word_tok[w] : 0ull;
    if (w < V) {
        int16_t idx = -1;
        if (tot > 0ull && tot * (unsigned long long)hot_max >= s->tokens) {
            const uint32_t at = atomicAdd(&s->n_hot, 1u);
            if (at < (uint32_t)hot_max) idx = (int16_t)at;
        }
        hot_of[w] = idx;
    }
    sh[threadIdx.x] = tot;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) sh[threadIdx.x] = sh[threadIdx.x] > sh[threadIdx.x + off] ? sh[threadIdx.x] : sh[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0 && sh[0]) atomicMax(&s->max_word_tokens, sh[0]);
}

// The lowest id that attains a maximum (for the error message).
__global__ void wl_argmax(const unsigned long long* __restrict__ tok, int32_t n, const unsigned long long* __restrict__ largest,
                          uint32_t* __restrict__ id)
{
    const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n && tok[i] == *largest) atomicMin(id, (uint32_t)i);
}

// The ids of the heavy tasks (heavy_from).  A workgroup takes kHeavyTile consecutive tasks and reserves the places of its
// heavy ones with one atomic (one per wave was one in 16 ns: 1.2 ms for 7.7 million tasks); inside a tile they keep
// their order, so that neighbours in the list are mostly of one document.  The order only decides when a task is drawn.
constexpr int kHeavyTile = 4096;
__global__ __launch_bounds__(256) void wl_heavy(const uint32_t* __restrict__ t_g, int64_t n, uint32_t capacity, int32_t* __restrict__ heavy,
                                                BuildStats* s)
{
    __shared__ uint32_t from, first, wave_total[4];
    if (threadIdx.x == 0) from = heavy_from(s->sizes, s->n_tasks);
    __syncthreads();
    constexpr int kEach = kHeavyTile / 256;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t i0 = (int64_t)blockIdx.x * kHeavyTile + (int64_t)wv * (kHeavyTile / 4) + lane;
    uint64_t masks[kEach];
    uint32_t total = 0;
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
        const int64_t i = i0 + 64 * j;
        masks[j] = __ballot(i < n && t_g[i < n ? i : 0] >= from);
        total += (uint32_t)__popcll((unsigned long long)masks[j]);
    }
    if (lane == 0) wave_total[wv] = total;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t all = 0;
        for (int v = 0; v < 4; ++v) { const uint32_t t = wave_total[v]; wave_total[v] = all; all += t; }
        first = all ? atomicAdd(&s->n_heavy, all) : 0u;
    }
    __syncthreads();
    uint32_t at = first + wave_total[wv];
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
        const uint32_t mine = at + (uint32_t)__popcll((unsigned long long)(masks[j] & ((1ull << lane) - 1ull)));
        if (((masks[j] >> lane) & 1ull) && mine < capacity) heavy[mine] = (int32_t)(i0 + 64 * j);
        at += (uint32_t)__popcll((unsigned long long)masks[j]);
    }
}

// The tasks of every nonzero, consecutive from tbase[i]; the processing order starts as storage order.
__global__ void wl_expand(const int32_t* __restrict__ nz_doc, const int32_t* __restrict__ rowidx,
                          const float* __restrict__ val, const uint32_t* __restrict__ tbase, int64_t nnz, uint32_t G,
                          int32_t* __restrict__ t_doc, int32_t* __restrict__ t_word, uint32_t* __restrict__ t_g,
                          int32_t* __restrict__ order, uint32_t* __restrict__ cost)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nnz; i += stride) {
        const uint32_t t0 = tbase[i], t1 = tbase[i + 1];
        const int32_t d = nz_doc[i], w = rowidx[i];
        uint32_t left = (uint32_t)val[i];
        for (uint32_t t = t0; t < t1; ++t) {
            const uint32_t g = left < G ? left : G;
            t_doc[t] = d; t_word[t] = w; t_g[t] = g;
            order[t] = (int32_t)t; cost[t] = 0u;
            left -= g;
        }
    }
}

// tile_start[T] = first task of document tile T (tile_docs documents per tile), n_tiles + 1 entries.
__global__ void wl_tiles(const int32_t* __restrict__ colptr, const uint32_t* __restrict__ tbase, int32_t D,
                         int32_t tile_docs, int32_t n_tiles, int32_t* __restrict__ tile_start)
{
    const int32_t T = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (T > n_tiles) return;
    const int64_t d = (int64_t)T * tile_docs;
    tile_start[T] = (int32_t)tbase[colptr[d < D ? d : D]];
}

// ---- Exclusive sum of 32-bit counts.  A workgroup owns a tile of kScanTile consecutive items.  One launch adds up
// every tile, the tile totals are summed the same way (recursively, until one tile is left), and a last launch
// per level writes the items' exclusive sums from the tile's base.  All sums are modulo 2^32 (the callers' totals
// stay below 2^31).
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;                                     // consecutive items per thread
constexpr int kScanTile = kScanThreads * kScanItems;

// sum over the workgroup; every thread receives it
__device__ __forceinline__ uint32_t wl_block_sum(uint32_t v, uint32_t* sh /* [kScanThreads / 64] */)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    uint32_t t = 0;
    for (int i = 0; i < kScanThreads / 64; ++i) t += sh[i];
    __syncthreads();
    return t;
}

__global__ __launch_bounds__(kScanThreads) void wl_tile_sums(const uint32_t* __restrict__ in, size_t n, uint32_t* __restrict__ tile_sum)
{
    __shared__ uint32_t sh[kScanThreads / 64];
    const size_t first = (size_t)blockIdx.x * kScanTile + (size_t)threadIdx.x * kScanItems;
    uint32_t v = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) if (first + j < n) v += in[first + j];
    const uint32_t t = wl_block_sum(v, sh);
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = t;
}

// out[i] = tile_base[tile of i] + sum of the items of the tile before i (tile_base null: zero, a single tile)
__global__ __launch_bounds__(kScanThreads) void wl_tile_scan(const uint32_t* __restrict__ in, size_t n, const uint32_t* __restrict__ tile_base,
                                                            uint32_t* __restrict__ out)
{
    __shared__ uint32_t wave_total[kScanThreads / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const size_t first = (size_t)blockIdx.x * kScanTile + (size_t)threadIdx.x * kScanItems;
    uint32_t x[kScanItems];
    uint32_t mine = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) { x[j] = first + j < n ? in[first + j] : 0u; mine += x[j]; }
    uint32_t incl = mine;                                          // inclusive sum over the wave's lanes
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t up = __shfl_up(incl, o);
        if (lane >= o) incl += up;
    }
    if (lane == 63) wave_total[wv] = incl;
    __syncthreads();
    uint32_t base = tile_base ? tile_base[blockIdx.x] : 0u;
    for (int i = 0; i < wv; ++i) base += wave_total[i];
    uint32_t run = base + incl - mine;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        if (first + j < n) out[first + j] = run;
        run += x[j];
    }
}

// ---- Stable radix sort of (key, value) pairs by 8-bit digits, least significant first.  A workgroup owns a tile of
// kSortTile consecutive items, wave v of it the items [v * 1024, (v + 1) * 1024) of the tile, read 64 at a time (a row).
// Per pass: wl_sort_histogram counts the tile's items per digit into hist[digit][tile]; the exclusive sum of hist
// in that order is where each tile's run of each digit starts in the output; wl_sort_scatter places the items: a
// lane's position is the start of its (digit, tile) run, plus the items of the same digit in the waves before its
// own, in the earlier rows of its wave, and in the lower lanes of its row.  Items keep their order inside a digit:
// the sort is stable, and the passes from the lowest digit up sort by the whole key.
constexpr int kSortThreads = 256;
constexpr int kSortRows = 16;                                     // rows of 64 items per wave
constexpr int kSortTile = kSortThreads * kSortRows;               // 4096 items
constexpr int kSortDigits = 256;
static_assert(kSortThreads == kSortDigits, "thread d of a workgroup owns digit d");

__global__ __launch_bounds__(kSortThreads) void wl_sort_histogram(const int32_t* __restrict__ keys, int64_t n, int shift, uint32_t n_tiles,
                                                                 uint32_t* __restrict__ hist)
{
    __shared__ uint32_t h[kSortDigits];
    h[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t first = (int64_t)blockIdx.x * kSortTile;
    for (int j = 0; j < kSortRows; ++j) {
        const int64_t i = first + (int64_t)j * kSortThreads + threadIdx.x;
        if (i < n) atomicAdd(&h[((uint32_t)keys[i] >> shift) & (kSortDigits - 1)], 1u);
    }
    __syncthreads();
    hist[(size_t)threadIdx.x * n_tiles + blockIdx.x] = h[threadIdx.x];
}

// vals_in null: the value of item i is i (the first pass sorts the identity)
__global__ __launch_bounds__(kSortThreads) void wl_sort_scatter(const int32_t* __restrict__ keys_in, const int32_t* __restrict__ vals_in,
                                                                int64_t n, int shift, uint32_t n_tiles, const uint32_t* __restrict__ start,
                                                                int32_t* __restrict__ keys_out, int32_t* __restrict__ vals_out)
{
    __shared__ uint32_t cnt[kSortThreads / 64][kSortDigits];      // per wave and digit: items, then the next output position
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int v = 0; v < kSortThreads / 64; ++v) cnt[v][threadIdx.x] = 0u;
    __syncthreads();
    const int64_t first = (int64_t)blockIdx.x * kSortTile + (int64_t)wv * (kSortRows * 64) + lane;
    int32_t key[kSortRows], val[kSortRows];
#pragma unroll
    for (int j = 0; j < kSortRows; ++j) {
        const int64_t i = first + (int64_t)j * 64;
        const bool in = i < n;
        key[j] = in ? keys_in[i] : 0;
        val[j] = in ? (vals_in ? vals_in[i] : (int32_t)i) : 0;
        if (in) atomicAdd(&cnt[wv][((uint32_t)key[j] >> shift) & (kSortDigits - 1)], 1u);
    }
    __syncthreads();
    {   // thread d: where the waves' items of digit d start
        uint32_t pos = start[(size_t)threadIdx.x * n_tiles + blockIdx.x];
        for (int v = 0; v < kSortThreads / 64; ++v) { const uint32_t c = cnt[v][threadIdx.x]; cnt[v][threadIdx.x] = pos; pos += c; }
    }
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int j = 0; j < kSortRows; ++j) {
        const bool in = first + (int64_t)j * 64 < n;
        const uint32_t dgt = ((uint32_t)key[j] >> shift) & (kSortDigits - 1);
        uint64_t peers = __ballot(in);                             // the lanes of this row that hold the same digit
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const bool one = (dgt >> bit) & 1u;
            const uint64_t m = __ballot(one);
            peers &= one ? m : ~m;
        }
        if (in) {
            const uint32_t rank = (uint32_t)__popcll((unsigned long long)(peers & below));
            const uint32_t pos = cnt[wv][dgt] + rank;              // every peer reads the position before the first one moves it on
            if (rank == 0u) cnt[wv][dgt] = pos + (uint32_t)__popcll((unsigned long long)peers);
            if ((int64_t)pos < n) {                                // always true; keeps a wrong count from becoming a wild store
                keys_out[pos] = key[j];
                vals_out[pos] = val[j];
            }
        }
    }
}

// wstart[w] = first position of word w in the word-sorted task list (n for words beyond the last), V + 1 entries.
__global__ void wl_word_starts(const int32_t* __restrict__ keys, int32_t n, int32_t V, int32_t* __restrict__ wstart)
{
    const int32_t w = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (w > V) return;
    int32_t lo = 0, hi = n;                                        // first position with keys[pos] >= w
    while (lo < hi) { const int32_t mid = lo + (hi - lo) / 2; if (keys[mid] < w) lo = mid + 1; else hi = mid; }
    wstart[w] = lo;
}

// flag[i] = 1 if the word at sorted position i has at least min_tasks tasks (its tasks get slots).
__global__ void wl_slot_flags(const int32_t* __restrict__ keys, const int32_t* __restrict__ wstart, int64_t n,
                              int32_t min_tasks, uint32_t* __restrict__ flag)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= n; i += stride) {
        if (i == n) { flag[i] = 0u; break; }
        const int32_t w = keys[i];
        flag[i] = (wstart[w + 1] - wstart[w] >= min_tasks) ? 1u : 0u;
    }
}

// Slots in (word, task id) order: pos is the exclusive sum of flag (n + 1 entries, the last = number of slots).
__global__ void wl_slot_scatter(const int32_t* __restrict__ keys, const int32_t* __restrict__ tasks,
                                const uint32_t* __restrict__ flag, const uint32_t* __restrict__ pos, int64_t n,
                                int32_t* __restrict__ t_slot, int32_t* __restrict__ slot_word, BuildStats* s)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        if (flag[i]) { t_slot[tasks[i]] = (int32_t)pos[i]; slot_word[pos[i]] = keys[i]; }
        else t_slot[tasks[i]] = -1;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) s->n_slots = pos[n];
}

}  // namespace same
