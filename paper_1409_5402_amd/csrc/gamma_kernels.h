// The sampled parameter step (Algorithm 2, third step; Section 3.1) for gfx950: theta and phi drawn
// from their Dirichlet conditionals given the counts of the m copies,
//   theta_d ~ Dirichlet(n_dk + m*alpha),   phi_k ~ Dirichlet over words (n_wk + m*beta),
// as independent Gamma(shape, 1) variables (theta: divided by m and left unnormalised, mean
// n_dk/m + alpha as in the collapsed update; phi: divided by their sum over words).
//
// Gamma variables after Marsaglia and Tsang (ACM TOMS 26, 2000): d = a - 1/3, c = 1/sqrt(9d),
// z standard normal, v = (1 + c z)^3, accept d*v when v > 0 and log u < z^2/2 + d(1 - v + log v),
// tried first as u < 1 - 0.0331 z^4; a shape below one takes Gamma(a+1) * u'^(1/a).  The normal is
// sqrt(-2 log u1) cos(2 pi u2).  Attempt j of element (row, k) uses the Philox block with counter
// (row, k, j, pass word): words 0 and 1 make the normal, word 2 the acceptance uniform, word 3 the
// uniform of the small-shape factor.  After 64 refused attempts the shape itself is the result.
// Logarithm, cosine and exponential are fixed sequences of + - * / in binary32, one rounding each,
// so that every acceptance is decided the same way by any implementation of these steps.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rng_binom.h"
#include "update_kernels.h"

namespace same {

// cos(2 pi u), u in (0,1): quarter turn, then the Taylor polynomial of sine or cosine on [0, pi/2).
__device__ __forceinline__ float cos2pi(float u)
{
    const float t = u * 4.0f;
    const int quarter = (int)t;
    const float x = (t - (float)quarter) * 1.57079637f;
    const float x2 = x * x;
    float sn = 1.60590444e-10f;
    sn = sn * x2; sn = sn + -2.50521079e-08f;
    sn = sn * x2; sn = sn + 2.75573188e-06f;
    sn = sn * x2; sn = sn + -0.000198412701f;
    sn = sn * x2; sn = sn + 0.00833333377f;
    sn = sn * x2; sn = sn + -0.166666672f;
    sn = sn * x2; sn = sn + 1.0f;
    sn = sn * x;
    float cs = -1.14707454e-11f;
    cs = cs * x2; cs = cs + 2.08767570e-09f;
    cs = cs * x2; cs = cs + -2.75573188e-07f;
    cs = cs * x2; cs = cs + 2.48015876e-05f;
    cs = cs * x2; cs = cs + -0.00138888892f;
    cs = cs * x2; cs = cs + 0.0416666679f;
    cs = cs * x2; cs = cs + -0.5f;
    cs = cs * x2; cs = cs + 1.0f;
    const int q = quarter & 3;
    return q == 0 ? cs : q == 1 ? -sn : q == 2 ? -cs : sn;
}

// Gamma(a, 1) for element (row, k) of the stream with the given pass word.
__device__ __forceinline__ float gamma_variable(float a, uint32_t seed_lo, uint32_t seed_hi, uint32_t row,
                                                uint32_t k, uint32_t pass)
{
    const bool small = a < 1.0f;
    const float a1 = small ? a + 1.0f : a;
    const float d = a1 - 0.333333343f;
    const float c = 1.0f / sqrtf(9.0f * d);
    float g = a1;
    uint32_t x[4] = {0u, 0u, 0u, 0u};
    for (uint32_t attempt = 0; attempt < 64u; ++attempt) {
        philox4x32_10(row, k, attempt, pass, seed_lo, seed_hi, x);
        const float l1 = flog(uniform_from_word(x[0]));
        const float r = sqrtf(-2.0f * l1);
        const float z = r * cos2pi(uniform_from_word(x[1]));
        const float u = uniform_from_word(x[2]);
        const float t = 1.0f + c * z;
        if (!(t > 0.0f)) continue;
        float v = t * t;
        v = v * t;
        const float z2 = z * z;
        const float z4 = z2 * z2;
        bool accept = u < 1.0f - 0.0331f * z4;
        if (!accept) {
            const float lhs = flog(u);
            const float inner = (1.0f - v) + flog(v);
            const float rhs = 0.5f * z2 + d * inner;
            accept = lhs < rhs;
        }
        if (accept) { g = d * v; break; }
    }
    if (small) {
        float y = -flog(uniform_from_word(x[3]));
        y = y / a;
        if (y > 200.0f) y = 200.0f;
        g = g * expneg(y);
    }
    return g < 1e-30f ? 1e-30f : g;
}

// theta[d][k] = Gamma(n_dk + m*alpha) / m; rows_per_block documents per workgroup
__global__ __launch_bounds__(256) void gamma_theta_kernel(const uint32_t* __restrict__ ndk, float* __restrict__ theta, int D, int K,
                                                         float mf, float prior, uint32_t seed_lo, uint32_t seed_hi, uint32_t pass,
                                                         uint32_t rows_per_block)
{
    const RowSplit<1> s(K);
    if (s.group >= s.groups) return;
    const Rows b = rows_of_block(blockIdx.x, rows_per_block, (uint32_t)D);
    for (int k = s.unit; k < K; k += s.groups == 1 ? 256 : K)
        for (uint32_t d = b.from + s.group; d < b.to; d += s.groups) {
            const size_t i = (size_t)d * K + k;
            const float a = (float)ndk[i] + prior;
            theta[i] = gamma_variable(a, seed_lo, seed_hi, d, (uint32_t)k, pass) / mf;
        }
}

// phi[w][k] = Gamma(n_wk + m*beta), the sum of each topic over this block's rows (double, in a fixed order) and its copies in
// them, added to the copies of n_k (n_k over n_dk cost a pass over that matrix).  A hot
// word's row first takes in its copies, as in phi_update_kernel.  1024 threads per workgroup: the variables are long
// chains of arithmetic, and the block sums' scratch fixes the number of workgroups, not that of waves.
constexpr int kGammaThreads = 1024;
__global__ __launch_bounds__(kGammaThreads) void gamma_phi_kernel(uint32_t* __restrict__ nwk, const int16_t* __restrict__ hot_of,
                                                                 const uint32_t* __restrict__ hot_used,
                                                                 int hot_max, int hot_copies, float* __restrict__ phi, int V, int K,
                                                                 float prior, uint32_t seed_lo, uint32_t seed_hi, uint32_t pass,
                                                                 uint32_t rows_per_block, double* __restrict__ partial, NkCopies totals)
{
    __shared__ double sh[kGammaThreads];
    __shared__ unsigned long long sh_n[kGammaThreads];
    const RowSplit<1, kGammaThreads> s(K);
    const Rows b = rows_of_block(blockIdx.x, rows_per_block, (uint32_t)V);
    const bool copies = hot_of != nullptr && *hot_used != 0u;
    for (int k = s.unit; k < K; k += s.groups == 1 ? kGammaThreads : K) {
        double acc = 0.0;
        unsigned long long copies_k = 0;                           // the topic's copies in these rows
        if (s.group < s.groups) {
            for (uint32_t r = b.from + s.group; r < b.to; r += s.groups) {
                const size_t i = (size_t)r * K + k;
                uint32_t n[1] = {nwk[i]};
                const int hot = copies ? (int)hot_of[r] : -1;
                if (hot >= 0 && take_in_copies<1>(nwk, V, K, hot, hot_max, hot_copies, k, n)) nwk[i] = n[0];
                copies_k += n[0];
                const float g = gamma_variable((float)n[0] + prior, seed_lo, seed_hi, r, (uint32_t)k, pass);
                phi[i] = g;
                acc += (double)g;
            }
        }
        if (s.groups > 1) {
            sh[threadIdx.x] = acc;
            sh_n[threadIdx.x] = copies_k;
            __syncthreads();
            if (s.group != 0) break;
            for (int g = 1; g < s.groups; ++g) { acc += sh[g * K + k]; copies_k += sh_n[g * K + k]; }
        }
        if (copies_k) atomicAdd(totals.p + (size_t)(blockIdx.x % (uint32_t)totals.n) * K + k, copies_k);
        partial[(size_t)blockIdx.x * K + k] = acc;
    }
}

// total[k] = sum of the block sums (double, in a fixed order), rounded to binary32; and the topic totals from their copies
__global__ __launch_bounds__(256) void gamma_phi_totals_kernel(const double* __restrict__ partial, int blocks, int K, float* __restrict__ total,
                                                              NkCopies copies, unsigned long long* __restrict__ nk)
{
    column_sums(partial, blocks, K, [&](int k, double sum) { total[k] = (float)sum; nk[k] = nk_total(copies, K, k); });
}

__global__ __launch_bounds__(256) void gamma_phi_normalise_kernel(float* __restrict__ phi, int V, int K, const float* __restrict__ total,
                                                                 uint32_t rows_per_block)
{
    const RowSplit<1> s(K);
    if (s.group >= s.groups) return;
    const Rows b = rows_of_block(blockIdx.x, rows_per_block, (uint32_t)V);
    for (int k = s.unit; k < K; k += s.groups == 1 ? 256 : K) {
        const float t = total[k];
        for (uint32_t r = b.from + s.group; r < b.to; r += s.groups) phi[(size_t)r * K + k] = phi[(size_t)r * K + k] / t;
    }
}

}  // namespace same
