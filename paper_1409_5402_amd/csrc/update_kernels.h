// Dense kernels around the draw: zeroing, topic totals, the parameter update of Eq. 6 /
// Algorithm 3 (add priors, normalise phi over words, blend) and the log-likelihood reduction.
// All are plain coalesced streams over [rows][K] matrices; every arithmetic step is one
// binary32 operation (no contraction), in the order stated next to it.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "launch_shape.h"
#include "rng_binom.h"
#include "scatter.h"

namespace same {

// Self-test: reciprocal of every integer in [1, 2^24); the quotients of quot_1 for every operand it is used with; quot_int for
// a seeded numerator over every integer and four over those whose reciprocals round worst; the published Philox known answers.
__global__ void selftest_kernel(unsigned long long* __restrict__ failures)
{
    const uint32_t x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= 1u && x < (1u << 24)) {
        const float fx = (float)x;
        if (inv_int(fx) != 1.0f / fx) atomicAdd(failures, 1ull);
        for (uint32_t i = 0; i < (x < 4096u || x >= (1u << 24) - 4096u ? 64u : 4u); ++i) {
            const float a = -flog(uniform_from_word((x * 64u + i) * 0x9E3779B9u));
            if (quot_int(a, fx) != a / fx) atomicAdd(failures, 1ull);
        }
        float f = __uint_as_float(0x3F800000u | (x & 0x007FFFFFu));    // every mantissa (twice)
        if (f > 1.41421354f) f = f * 0.5f;
        const float a = f - 1.0f, b = f + 1.0f;
        if (quot_1(a, b) != a / b) atomicAdd(failures, 1ull);
    }
    for (uint32_t i = x + 1u; i <= 0x3F000000u; i += gridDim.x * blockDim.x) {   // every binary32 in (0, 1/2]
        const float v = __uint_as_float(i), d1 = 1.0f - v, d2 = 2.0f - v;
        if (quot_1(v, d1) != v / d1 || quot_1(v, d2) != v / d2) atomicAdd(failures, 1ull);
    }
    if (x < 3u) {
        const uint32_t in[3][6] = {{0u, 0u, 0u, 0u, 0u, 0u},
                                   {0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu},
                                   {0x243f6a88u, 0x85a308d3u, 0x13198a2eu, 0x03707344u, 0xa4093822u, 0x299f31d0u}};
        const uint32_t want[3][4] = {{0x6627e8d5u, 0xe169c58du, 0xbc57ac4cu, 0x9b00dbd8u},
                                     {0x408f276du, 0x41c83b0eu, 0xa20bc7c6u, 0x6d5451fdu},
                                     {0xd16cfe09u, 0x94fdccebu, 0x5001e420u, 0x24126ea1u}};
        uint32_t out[4];
        philox4x32_10(in[x][0], in[x][1], in[x][2], in[x][3], in[x][4], in[x][5], out);
        for (int i = 0; i < 4; ++i) if (out[i] != want[x][i]) atomicAdd(failures, 1ull);
    }
}

// Clears up to four arrays in one launch (each aligned to 16 bytes): a launch costs some 4.5 us whatever it does, and a
// sweep needs four things cleared.
struct ClearArgs { uint32_t* p[4]; size_t n[4]; };
__global__ __launch_bounds__(256) void clear_kernel(ClearArgs a)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x, i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const size_t quads = a.n[j] / 4;
        uint4* p = reinterpret_cast<uint4*>(a.p[j]);
        for (size_t i = i0; i < quads; i += stride) p[i] = make_uint4(0u, 0u, 0u, 0u);
        if (i0 < (a.n[j] & 3u)) a.p[j][4 * quads + i0] = 0u;
    }
}

__global__ void zero_u32_kernel(uint32_t* __restrict__ p, size_t n)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0u;
}

__global__ void zero_u64_kernel(unsigned long long* __restrict__ p, size_t n)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0ull;
}

// Re-sorts the processing order of one document tile by descending cost (counting sort over 256
// cost buckets; ties land in arbitrary order, which only affects scheduling, never results).
__global__ __launch_bounds__(256) void reorder_kernel(const int32_t* __restrict__ tile_start,
                                                      const uint32_t* __restrict__ cost,
                                                      int32_t* __restrict__ order)
{
    __shared__ uint32_t bins[256];
    const int t0 = tile_start[blockIdx.x], t1 = tile_start[blockIdx.x + 1];
    bins[threadIdx.x] = 0u;
    __syncthreads();
    for (int i = t0 + (int)threadIdx.x; i < t1; i += 256) atomicAdd(&bins[min(cost[i], 255u)], 1u);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t acc = 0u;
        for (int b = 255; b >= 0; --b) { const uint32_t c = bins[b]; bins[b] = acc; acc += c; }
    }
    __syncthreads();
    for (int i = t0 + (int)threadIdx.x; i < t1; i += 256) {
        const uint32_t pos = atomicAdd(&bins[min(cost[i], 255u)], 1u);
        order[t0 + (int)pos] = i;
    }
}

// How the kernels over [rows][K] matrices share a row's topics out: a thread owns one unit of W consecutive topics (W = 4,
// 16-byte accesses, where K is a multiple of 4, else 1), a workgroup of 256 threads G = 256 / (K / W) rows at a time (one,
// in several turns, where a row has more than 256 units; the sampled phi step does the same with 1024 threads).  What depends on the topic alone is then computed once per
// thread, and no element needs a remainder by K.
template <int W, int THREADS = 256>
struct RowSplit {
    int units, groups, unit, group;
    __device__ __forceinline__ explicit RowSplit(int K)
    {
        units = K / W;
        groups = units >= THREADS ? 1 : THREADS / units;
        unit = groups == 1 ? (int)threadIdx.x : (int)threadIdx.x % units;
        group = groups == 1 ? 0 : (int)threadIdx.x / units;
    }
};
inline int rows_at_once(int K) { const int units = K % 4 == 0 ? K / 4 : K; return units >= 256 ? 1 : 256 / units; }

template <int W>
__device__ __forceinline__ void load_unit(const uint32_t* __restrict__ p, uint32_t (&v)[W])
{
    if constexpr (W == 4) {
        const uint4 q = *reinterpret_cast<const uint4*>(p);
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    } else {
        v[0] = *p;
    }
}

// theta = n_dk / m + alpha   (divide, then add), n elements
__global__ __launch_bounds__(256) void theta_update_kernel(const uint32_t* __restrict__ ndk, float* __restrict__ theta,
                                                          size_t n, float mf, float alpha)
{
    const size_t first = (size_t)blockIdx.x * 256u + threadIdx.x, stride = (size_t)gridDim.x * 256u;
    const size_t quads = n / 4;
    for (size_t i = first; i < quads; i += stride) {
        const uint4 c = reinterpret_cast<const uint4*>(ndk)[i];
        float4 t;
        t.x = (float)c.x / mf + alpha;
        t.y = (float)c.y / mf + alpha;
        t.z = (float)c.z / mf + alpha;
        t.w = (float)c.w / mf + alpha;
        reinterpret_cast<float4*>(theta)[i] = t;
    }
    if (first < (n & 3u)) theta[4 * quads + first] = (float)ndk[4 * quads + first] / mf + alpha;
}

// n_k, the copies of topic k, exact in 64-bit integers (any order gives the same value), and theta.  Every copy is in n_dk and
// in n_wk; the sum is taken over n_dk, which theta reads anyway and which is complete when the draw ends (the sampled form, whose
// theta is another kernel's, takes it over n_wk in gamma_phi_kernel).  A workgroup owns a range of documents, 16-byte accesses at
// every number of topics (totals_split), four in flight per thread, and ends with one 64-bit atomic per topic, on one of a few
// copies of the totals: the 512 of a launch on one address take longer than the rest of it where that is small (K = 64, 50,000
// documents: 18 us a sweep).  Who needs the totals adds the copies up (nk_total), which every workgroup of the phi update
// does: eight copies up to 128 topics, down to one at 1024 (nk_copies_for; with eight there 110 us of 4.6 ms lost).
struct NkCopies { unsigned long long* p; int n; };
__device__ __forceinline__ unsigned long long nk_total(const NkCopies& a, int K, int k)
{
    unsigned long long n = 0;
    if (a.n == 8) {                                                // all loads in flight together
#pragma unroll
        for (int c = 0; c < 8; ++c) n += a.p[(size_t)c * K + k];
    } else {
        for (int c = 0; c < a.n; ++c) n += a.p[(size_t)c * K + k];
    }
    return n;
}
struct ThetaArgs {
    const uint32_t* ndk; float* theta;
    NkCopies nk; uint32_t D; int K; TotalsSplit split; TotalsBlocks blocks;
    float mf, alpha;
};

__device__ __forceinline__ void theta_totals(const ThetaArgs& a, uint32_t block, unsigned long long* tot)   // tot: [K] of LDS
{
    const TotalsSplit& s = a.split;
    const int K = a.K;
    const uint32_t turns = (uint32_t)s.turns, groups = (uint32_t)s.groups;
    for (int k = threadIdx.x; k < K; k += 256) tot[k] = 0ull;
    __syncthreads();
    auto add = [&](int k, unsigned long long v) {
        if (v) __hip_atomic_fetch_add((__attribute__((address_space(3))) unsigned long long*)(tot + k), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    const uint32_t group = threadIdx.x / (uint32_t)s.per;
    const int unit = (int)(block % turns) * s.per + (int)(threadIdx.x % (uint32_t)s.per);
    const size_t row = 4 * (size_t)s.units;                        // counts of `fold` documents
    if (group < groups && unit < s.units) {
        const Rows b = rows_of_block(block / turns, a.blocks.rows_per_block, a.blocks.rows);
        unsigned long long acc[4] = {};
        for (uint32_t r = b.from + group; r < b.to; r += 4u * groups) {
            uint32_t v[4][4];
#pragma unroll
            for (uint32_t j = 0; j < 4u; ++j) {
                const uint32_t rj = r + j * groups;
                load_unit<4>(a.ndk + (rj < b.to ? rj : r) * row + 4 * unit, v[j]);
            }
#pragma unroll
            for (uint32_t j = 0; j < 4u; ++j) {
                const uint32_t rj = r + j * groups;
                if (rj >= b.to) break;
                float x[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) { acc[c] += v[j][c]; x[c] = (float)v[j][c] / a.mf + a.alpha; }
                *reinterpret_cast<float4*>(a.theta + rj * row + 4 * unit) = make_float4(x[0], x[1], x[2], x[3]);
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) add((4 * unit + c) % K, acc[c]);
    }
    if (block == 0) {                                              // the documents that fill no whole row: fewer than `fold`
        const size_t from = a.blocks.rows * row, n = (size_t)a.D * K - from;
        for (size_t i = threadIdx.x; i < n; i += 256) {
            const uint32_t v = a.ndk[from + i];
            add((int)(i % (uint32_t)K), v);
            a.theta[from + i] = (float)v / a.mf + a.alpha;
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < K; k += 256) if (tot[k]) atomicAdd(a.nk.p + (size_t)(block % (uint32_t)a.nk.n) * K + k, tot[k]);
}

// What follows a draw and needs nothing but its counts: the word rows from the pair list, and beside it in the same launch (the
// first t.blocks.blocks workgroups) the topic totals and theta.  One after the other the two took 12 and 11 us of the 72 us of a
// sweep over 4,000 documents at K = 50, 36 and 18 of 460 at 50,000 documents and K = 64; together
// tiny_fit's ten sweeps take 410 instead of 460 us, those five 390 instead of 440, and at K = 1024 the totals' pass over 400 MB
// of n_wk is gone (140 us).
__global__ __launch_bounds__(256) void counts_kernel(ThetaArgs t, ReduceArgs r)
{
    static_assert(kReduceThreads == 256, "workgroups of both kinds");
    extern __shared__ __align__(16) uint32_t counts_lds[];
    if (blockIdx.x < t.blocks.blocks) theta_totals(t, blockIdx.x, reinterpret_cast<unsigned long long*>(counts_lds));
    else                              word_reduce(r, blockIdx.x - t.blocks.blocks, counts_lds);
}

// The copies of a hot word's row (scatter.h): their counts of the W topics from `at` on are added to n and
// the copies are left clear.  True if there were any.
template <int W>
__device__ __forceinline__ bool take_in_copies(uint32_t* __restrict__ nwk, int V, int K, int hot, int hot_max, int hot_copies, int at,
                                               uint32_t (&n)[W])
{
    uint32_t any = 0u;
    uint32_t* first = nwk + ((size_t)V + (size_t)hot) * K + at;
    const size_t step = (size_t)hot_max * K;
    constexpr int kTurn = 8;                                       // copies whose loads are in flight together
    for (int copy = 0; copy < hot_copies; copy += kTurn) {
        uint32_t v[kTurn][W];
#pragma unroll
        for (int j = 0; j < kTurn; ++j) load_unit<W>(first + (size_t)(copy + j) * step, v[j]);
#pragma unroll
        for (int j = 0; j < kTurn; ++j)
            for (int c = 0; c < W; ++c) {
                if (v[j][c]) first[(size_t)(copy + j) * step + c] = 0u;
                n[c] += v[j][c]; any |= v[j][c];
            }
    }
    return any != 0u;
}

// phi_hat = (n_wk/m + beta) / (n_k/m + V*beta);  phi = rho == 1 ? phi_hat : (1-rho)*phi + rho*phi_hat.
// A hot word's row first takes in its copies, which are left clear.
struct PhiArgs {
    uint32_t* nwk; NkCopies copies; unsigned long long* nk; float* phi; const int16_t* hot_of;   // nk: out; hot_of null: no hot words
    const uint32_t* hot_used;              // 0: their copies have taken nothing
    int V, K, hot_max, hot_copies; uint32_t rows_per_block;
    float mf, beta, vbeta, rho;
};

template <int W>
__global__ __launch_bounds__(256) void phi_update_kernel(PhiArgs a)
{
    const RowSplit<W> s(a.K);
    if (s.group >= s.groups) return;
    const Rows b = rows_of_block(blockIdx.x, a.rows_per_block, (uint32_t)a.V);
    const bool copies = a.hot_of != nullptr && *a.hot_used != 0u;
    const float one_minus_rho = 1.0f - a.rho;
    for (int u = s.unit; u < s.units; u += s.groups == 1 ? 256 : s.units) {
        float den[W];
#pragma unroll
        for (int c = 0; c < W; ++c) {
            const unsigned long long n_k = nk_total(a.copies, a.K, W * u + c);
            if (blockIdx.x == 0 && s.group == 0) a.nk[W * u + c] = n_k;
            den[c] = (float)n_k / a.mf + a.vbeta;
        }
        for (uint32_t r = b.from + s.group; r < b.to; r += s.groups) {
            const size_t at = (size_t)r * a.K + W * u;
            uint32_t n[W];
            load_unit<W>(a.nwk + at, n);
            const int hot = copies ? (int)a.hot_of[r] : -1;
            if (hot >= 0 && take_in_copies<W>(a.nwk, a.V, a.K, hot, a.hot_max, a.hot_copies, W * u, n))
                for (int c = 0; c < W; ++c) a.nwk[at + c] = n[c];
            float hat[W];
#pragma unroll
            for (int c = 0; c < W; ++c) {
                const float num = (float)n[c] / a.mf + a.beta;
                hat[c] = num / den[c];
            }
            if (a.rho != 1.0f) {
#pragma unroll
                for (int c = 0; c < W; ++c) {
                    const float keep = one_minus_rho * a.phi[at + c];
                    const float add = a.rho * hat[c];
                    hat[c] = keep + add;
                }
            }
            if constexpr (W == 4) *reinterpret_cast<float4*>(a.phi + at) = make_float4(hat[0], hat[1], hat[2], hat[3]);
            else a.phi[at] = hat[0];
        }
    }
}

// finish(k, sum over b of partial[b][k]) for every topic: 8 topics per workgroup of 256 threads, 32 threads each over every
// 32nd block sum, whose results are added in a fixed order (sums repeat from run to run).  One thread per topic, as it
// was, is a chain of `blocks` dependent loads: 190 to 370 us for 782 to 1563 blocks, 9 us so.
template <class Finish>
__device__ __forceinline__ void column_sums(const double* __restrict__ partial, int blocks, int K, Finish finish)
{
    __shared__ double sh[32][8];
    const int c = threadIdx.x & 7, slice = threadIdx.x >> 3;
    const int k = blockIdx.x * 8 + c;
    double acc = 0.0;
    if (k < K) for (int b = slice; b < blocks; b += 32) acc += partial[(size_t)b * K + k];
    sh[slice][c] = acc;
    __syncthreads();
    if (slice == 0 && k < K) {
        for (int s = 1; s < 32; ++s) acc += sh[s][c];
        finish(k, acc);
    }
}
inline unsigned column_sum_blocks(int K) { return (unsigned)((K + 7) / 8); }

// log of each document's theta total: one wave per document, lanes across topics, in double (a fixed tree)
__global__ __launch_bounds__(256) void doc_log_total_kernel(const float* __restrict__ theta, int D, int K, double* __restrict__ out)
{
    const int lane = threadIdx.x & 63;
    const int d = (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
    if (d >= D) return;                                            // the whole wave
    double s = 0.0;
    for (int k = lane; k < K; k += 64) s += (double)theta[(size_t)d * K + k];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) out[d] = log(s);
}

// Per nonzero: c * (log mu - log theta total), mu from the normaliser (sddmm_kernel.h; a nonzero per thread with a running
// sum over its two rows took 1.82 ms for 6.7 million nonzeros at K = 256, lines of two rows per lane; the normaliser
// kernel and this one 0.60 ms).  Block partial sums (double) go to part[].
__global__ __launch_bounds__(256) void loglik_kernel(int64_t nnz, const int32_t* __restrict__ nz_doc,
                                                     const float* __restrict__ val, const float* __restrict__ mu,
                                                     const double* __restrict__ doc_log_total,
                                                     double* __restrict__ part)
{
    __shared__ double red[256];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    red[threadIdx.x] = i < nnz ? (double)val[i] * (log((double)mu[i]) - doc_log_total[nz_doc[i]]) : 0.0;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

}  // namespace same
