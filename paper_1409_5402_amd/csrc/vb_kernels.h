// E-step of online variational Bayes LDA on the normaliser of Algorithm 3 (Section 5.3: the product of two
// dense matrices at the nonzeros of a sparse one is the bottleneck the sampler shares with online variational
// Bayes LDA).  The paper does not print that method; the update below is the published one (Hoffman, Blei and
// Bach, 2010), restated:
//     a_dk = exp(psi(gamma_dk) - psi(sum_k gamma_dk)),   b_wk = exp(psi(lambda_wk) - psi(sum_w lambda_wk)),
//     mu_i = sum_k a_dk b_wk  for nonzero i = (d, w, c),   gamma'_dk = alpha + a_dk sum_{i in d} (c_i / mu_i) b_wk.
// psi and exp are evaluated in double (they are a few per row element and iteration), mu in binary32 with fused
// multiply-adds, the sums over a document's nonzeros and gamma itself in double.  gamma' does not change when a word's row of b is
// multiplied by a constant (mu_i takes the same factor): rows of b are stored divided by their largest entry,
// with the logarithm of that entry beside them, and the normaliser is returned as log mu.
#pragma once
#include "sddmm_kernel.h"
#include "update_kernels.h"

namespace same {

// psi(x) for x > 0: below 6 the recurrence psi(x) = psi(x + 6) - sum_i 1/(x+i), i = 0..5, the sum as one quotient N/D of
// polynomials with positive terms (D = x(x+1)..(x+5), N its derivative), then the asymptotic series
// ln x - 1/(2x) - sum_n B_2n / (2n x^2n) through x^-14 (below 1e-12 there).  Two divisions instead of up to eight.
__device__ __forceinline__ double digamma_d(double x)
{
    double r = 0.0;
    if (x < 6.0) {
        double D = x, N = 1.0;
#pragma unroll
        for (int i = 1; i < 6; ++i) { const double y = x + (double)i; N = __builtin_fma(N, y, D); D = D * y; }
        r = -(N / D);
        x += 6.0;
    }
    const double inv = 1.0 / x;
    const double f = inv * inv;
    const double t = f * (1.0 / 12.0 - f * (1.0 / 120.0 - f * (1.0 / 252.0 - f * (1.0 / 240.0 - f * (1.0 / 132.0
                     - f * (691.0 / 32760.0 - f * (1.0 / 12.0)))))));
    return r + log(x) - 0.5 * inv - t;
}

constexpr int kVbRows = 64;             // rows of lambda per workgroup of the column sums

// partial[blk][k] = sum of lambda[w][k] over the workgroup's rows, in row order, in double
__global__ __launch_bounds__(256) void vb_colsum_kernel(const float* __restrict__ lam, int V, int K,
                                                        double* __restrict__ partial)
{
    const int w0 = blockIdx.x * kVbRows;
    const int w1 = w0 + kVbRows < V ? w0 + kVbRows : V;
    for (int k = threadIdx.x; k < K; k += blockDim.x) {
        double s = 0.0;
        for (int w = w0; w < w1; ++w) s += (double)lam[(size_t)w * K + k];
        partial[(size_t)blockIdx.x * K + k] = s;
    }
}

// psi_total[k] = psi(sum_w lambda[w][k])
__global__ __launch_bounds__(256) void vb_colpsi_kernel(const double* __restrict__ partial, int blocks, int K, double* __restrict__ psi_total)
{
    column_sums(partial, blocks, K, [&](int k, double sum) { psi_total[k] = digamma_d(sum); });
}

// One wave per word: e_k = psi(lambda[w][k]) - psi_total[k] (= E[log beta_kw]); shift[w] = max_k e_k;
// b[w][k] = exp(e_k - shift[w]).  The largest entry of a row is 1: a word's row never underflows as a whole,
// whatever the size of its lambda (psi(0.01) is -100.6, and exp of that is not a binary32 number).
// N: topics per lane (64 N >= K); e_k stays in registers from the maximum to the exponential.
template <int N>
__global__ __launch_bounds__(256) void vb_exp_elog_beta_kernel(const float* __restrict__ lam, int V, int K,
                                                               const double* __restrict__ psi_total,
                                                               float* __restrict__ b, float* __restrict__ shift)
{
    const int lane = threadIdx.x & 63;
    const int w = (int)(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
    if (w >= V) return;                                            // the whole wave
    const float* __restrict__ row = lam + (size_t)w * K;
    double e[N];
    double top = -1.0e300;
#pragma unroll
    for (int c = 0; c < N; ++c) {
        const int k = 64 * c + lane;
        if (k < K) {
            e[c] = digamma_d((double)row[k]) - psi_total[k];
            top = e[c] > top ? e[c] : top;
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        const double other = __shfl_xor(top, o);
        top = other > top ? other : top;
    }
#pragma unroll
    for (int c = 0; c < N; ++c) {
        const int k = 64 * c + lane;
        if (k < K) b[(size_t)w * K + k] = (float)exp(e[c] - top);
    }
    if (lane == 0) shift[w] = (float)top;
}

// A wave per document, one in a workgroup.  A group of LANES lanes (16 up to 64 topics, 32 up to 128, else 64) takes four
// nonzeros per round, CH 16-byte loads of a lane per row of b (K <= 4 LANES CH; ALIGNED: K is a multiple of 4, else a row's
// last load is moved back into it and what it repeats has no weight).  gamma, a and, at the end of an iteration, the groups'
// sums over their nonzeros are in LDS, where a lane owns every 64th topic.
//
// Bound by the rows of b: 69 GB of them for 60,000 news-shaped documents and five iterations at K = 256, of which the second-level
// caches (4 MB a die) miss half, and by the conversions and sums in double behind them (per nonzero and lane at K = 256
// four conversions and four fused additions, beside four in binary32).  The rows of the next round are loaded while a round is
// worked off; every turn issues the same loads, past the document's end with its last nonzero's index and a count of zero, so that
// the wait before a round's arithmetic has a fixed number of younger loads behind it.  The four normalisers of a group end in lanes l & 3 (lane_sum_4): one division serves
// all four.  ms per launch before (all lanes on one nonzero, gamma and sums in registers, LDS off multiples of four) and now, five
// iterations: that case 6.13 and 5.02; 20,000 documents at K = 50 4.61 and 0.40, 128 2.22 and 0.91, 333 26.8 and 2.94, 512 4.20
// and 3.50, 1000 9.31 and 7.69.  (Two to sixteen waves per document, so that its rows might be found in the caches again:
// slower the more there are, 8.9 ms with sixteen; rows kept in registers over the iterations: the constants of the logarithm
// and exponential in double already fill them.)
struct VbArgs {
    const int32_t* colptr; const int32_t* rowidx; const float* val; int32_t D; int K;
    const float* b; const float* shift; float alpha; int iters; float* gamma; float* log_mu;
};
inline size_t vb_lds_bytes(int K, int lanes) { return 8u * ((size_t)(64 / lanes + 1) * K) + 4u * (size_t)K; }

// Four waves per SIMD up to 256 topics (five and six, with 24 registers and more in scratch: 5.99 and 6.83 ms for the case above),
// three up to 512, two up to 1024.
template <int LANES, int CH, bool ALIGNED>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(CH == 1 ? 4 : (CH == 2 ? 3 : (CH == 4 ? 2 : 1))))) void vb_estep_kernel(VbArgs p)
{
    typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));
    constexpr int kGroups = 64 / LANES, kRound = 4 * kGroups;
    extern __shared__ double vb_lds[];
    const int K = p.K, lane = threadIdx.x;
    const int sub = lane & (LANES - 1), grp = lane / LANES;
    double* sums = vb_lds;                                         // [kGroups][K]: the groups' sums over their nonzeros
    double* g = sums + kGroups * K;                                // [K]: gamma, in double from one iteration to the next: the iteration
                                                                   // converges slowly along some directions, and binary32
                                                                   // rounding fed back ten times shows at 1e-5
    float* av = reinterpret_cast<float*>(g + K);                   // [K]: a
    const int32_t d = (int32_t)blockIdx.x;
    const int32_t lo = p.colptr[d];
    const uint32_t n = (uint32_t)(p.colptr[d + 1] - lo);           // the document's nonzeros
    const int32_t* __restrict__ ids = p.rowidx + lo;
    const float* __restrict__ val = p.val + lo;
    float* __restrict__ grow = p.gamma + (size_t)d * K;
    for (int k = lane; k < K; k += 64) g[k] = (double)grow[k];

    int off[CH];                                                   // the lane's topics: CH windows of four inside the row
    bool ok[CH][4];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int k = 4 * (LANES * c + sub);
        off[c] = k < K - 4 ? k : K - 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) ok[c][j] = off[c] + j >= k;
    }
    static_assert(3 * kRound <= kVbAhead, "rounds loaded ahead");
    auto rows = [&](uint32_t first, float4 (&bv)[4][CH], float& cnt) {   // the round that begins with nonzero `first`
        const uint32_t i0 = first + (kGroups > 1 ? 4u * grp : 0u);
#pragma unroll
        for (uint32_t j = 0; j < 4u; ++j) {
            const float* __restrict__ row = p.b + (size_t)ids[vb_nonzero(i0, j, n)] * K;
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                if constexpr (ALIGNED) {
                    bv[j][c] = *reinterpret_cast<const float4*>(row + off[c]);
                } else {
                    const float4_any v = *reinterpret_cast<const float4_any*>(row + off[c]);
                    bv[j][c] = make_float4(v.x, v.y, v.z, v.w);
                }
            }
        }
        const uint32_t i = i0 + (lane & 3);
        cnt = i < n ? val[i] : 0.f;
    };
    for (int it = 0; it < p.iters; ++it) {
        __syncthreads();
        double s = 0.0;
#pragma unroll 1
        for (int k = lane; k < K; k += 64) s += g[k];
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        const double ps = digamma_d(s);
#pragma unroll 1
        for (int k = lane; k < K; k += 64) av[k] = (float)exp(digamma_d(g[k]) - ps);
        __syncthreads();
        float4 a[CH];
        double acc[CH][4];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            a[c].x = ok[c][0] ? av[off[c]] : 0.f;     a[c].y = ok[c][1] ? av[off[c] + 1] : 0.f;
            a[c].z = ok[c][2] ? av[off[c] + 2] : 0.f; a[c].w = ok[c][3] ? av[off[c] + 3] : 0.f;
            acc[c][0] = 0.0; acc[c][1] = 0.0; acc[c][2] = 0.0; acc[c][3] = 0.0;
        }
        auto work = [&](uint32_t first, const float4 (&bv)[4][CH], float cnt) {
            float sj[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                sj[j] = 0.f;
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    if constexpr (ALIGNED) {
                        float x = __builtin_fmaf(a[c].x, bv[j][c].x, sj[j]);
                        x = __builtin_fmaf(a[c].y, bv[j][c].y, x);
                        x = __builtin_fmaf(a[c].z, bv[j][c].z, x);
                        x = __builtin_fmaf(a[c].w, bv[j][c].w, x);
                        sj[j] = ok[c][0] ? x : sj[j];
                    } else {
                        sj[j] = ok[c][0] ? __builtin_fmaf(a[c].x, bv[j][c].x, sj[j]) : sj[j];
                        sj[j] = ok[c][1] ? __builtin_fmaf(a[c].y, bv[j][c].y, sj[j]) : sj[j];
                        sj[j] = ok[c][2] ? __builtin_fmaf(a[c].z, bv[j][c].z, sj[j]) : sj[j];
                        sj[j] = ok[c][3] ? __builtin_fmaf(a[c].w, bv[j][c].w, sj[j]) : sj[j];
                    }
                }
            }
            const float m = lane_sum_4<LANES>(sj, lane);
            const double q = cnt > 0.f ? (double)cnt / (double)m : 0.0;
            const int qlo = __double2loint(q), qhi = __double2hiint(q);
            // Value j's quotient from lane j of every row of 16, the same in all rows of a group.  (Every fourth lane has one, but added
            // up in another order: the document's topics would see different normalisers of one nonzero.)
            auto add = [&](int j, auto ctrl) {
                const double rj = __hiloint2double(__builtin_amdgcn_update_dpp(0, qhi, decltype(ctrl)::value, 0xF, 0xF, true),
                                                   __builtin_amdgcn_update_dpp(0, qlo, decltype(ctrl)::value, 0xF, 0xF, true));
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    acc[c][0] = __builtin_fma(rj, (double)bv[j][c].x, acc[c][0]);
                    acc[c][1] = __builtin_fma(rj, (double)bv[j][c].y, acc[c][1]);
                    acc[c][2] = __builtin_fma(rj, (double)bv[j][c].z, acc[c][2]);
                    acc[c][3] = __builtin_fma(rj, (double)bv[j][c].w, acc[c][3]);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            __builtin_amdgcn_sched_barrier(0);
            add(0, std::integral_constant<int, 0x150>{});
            add(1, std::integral_constant<int, 0x151>{});
            add(2, std::integral_constant<int, 0x152>{});
            add(3, std::integral_constant<int, 0x153>{});
            if (p.log_mu != nullptr && it == p.iters - 1) {
                const uint32_t i = first + 4 * grp + (lane & 3);
                if (sub < 4 && i < n) p.log_mu[lo + i] = logf(m) + (p.shift ? p.shift[ids[i]] : 0.f);
            }
        };
        if (n > 0) {
            float4 b0[4][CH], b1[4][CH];
            float c0, c1;
            rows(0, b0, c0);
            for (uint32_t i = 0; ; i += 2 * kRound) {              // two rounds per turn: no copies between the two sets
                rows(i + kRound, b1, c1);
                __builtin_amdgcn_sched_barrier(0);                 // the next round's loads first, then this round's work
                work(i, b0, c0);
                __builtin_amdgcn_sched_barrier(0);
                if (i + kRound >= n) break;
                rows(i + 2 * kRound, b0, c0);
                __builtin_amdgcn_sched_barrier(0);
                work(i + kRound, b1, c1);
                __builtin_amdgcn_sched_barrier(0);
                if (i + 2 * kRound >= n) break;
            }
        }
        double* mine = sums + grp * K;
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) if (ok[c][j]) mine[off[c] + j] = acc[c][j];
        __syncthreads();
#pragma unroll 1
        for (int k = lane; k < K; k += 64) {
            double total = 0.0;
#pragma unroll
            for (int i = 0; i < kGroups; ++i) total += sums[i * K + k];
            g[k] = __builtin_fma((double)av[k], total, (double)p.alpha);
        }
    }
    for (int k = lane; k < K; k += 64) grow[k] = (float)g[k];       // the lane's own
}

// Fewer than four topics: a wave per document, the same steps with the document's vectors in LDS (gamma and the sums in
// double, a in binary32: 20 K bytes per wave).
__global__ __launch_bounds__(256) void vb_estep_few_kernel(const int32_t* __restrict__ colptr, const int32_t* __restrict__ rowidx,
                                                           const float* __restrict__ val, int32_t D, int K,
                                                           const float* __restrict__ b, const float* __restrict__ shift,
                                                           float alpha, int iters, float* __restrict__ gamma,
                                                           float* __restrict__ log_mu_out)
{
    extern __shared__ double vb_lds[];                             // [waves][g: K doubles][acc: K doubles][a: K floats, padded]
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int32_t d = (int32_t)(blockIdx.x * (blockDim.x >> 6) + wv);
    if (d >= D) return;
    const int per_wave = 2 * K + (K + 1) / 2;                      // doubles
    double* g = vb_lds + (size_t)wv * per_wave;
    double* acc = g + K;
    float* a = reinterpret_cast<float*>(acc + K);
    const int64_t lo = colptr[d], hi = colptr[d + 1];
    float* __restrict__ grow = gamma + (size_t)d * K;
    for (int k = lane; k < K; k += 64) g[k] = (double)grow[k];
    for (int it = 0; it < iters; ++it) {
        double s = 0.0;
        for (int k = lane; k < K; k += 64) s += g[k];
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        const double ps = digamma_d(s);
        for (int k = lane; k < K; k += 64) { a[k] = (float)exp(digamma_d(g[k]) - ps); acc[k] = 0.0; }
        for (int64_t i = lo; i < hi; ++i) {
            const float* __restrict__ p = b + (size_t)rowidx[i] * K;
            float s0 = 0.f;
            for (int k = lane; k < K; k += 64) s0 = __builtin_fmaf(a[k], p[k], s0);
            const float m0 = wave_sum(s0);
            const double r0 = (double)val[i] / (double)m0;
            for (int k = lane; k < K; k += 64) acc[k] = __builtin_fma(r0, (double)p[k], acc[k]);
            if (log_mu_out != nullptr && it == iters - 1 && lane == 0)
                log_mu_out[i] = logf(m0) + (shift ? shift[rowidx[i]] : 0.f);
        }
        for (int k = lane; k < K; k += 64) g[k] = __builtin_fma((double)a[k], acc[k], (double)alpha);
    }
    for (int k = lane; k < K; k += 64) grow[k] = (float)g[k];
}

}  // namespace same
