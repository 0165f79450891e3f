// The normaliser of Algorithm 3 as a kernel of its own (Section 5.3: SDDMM, the product of two dense matrices evaluated at
// the nonzeros of a sparse one): mu[i] = sum_k theta[d][k] * phi[w][k]; and the sums over lanes that it shares with the
// variational E-step.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "launch_shape.h"

namespace same {

template <int CTRL>
__device__ __forceinline__ float dpp_add(float v)
{
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

__device__ __forceinline__ float wave_sum(float v)
{
    v = dpp_add<0xB1>(v);      // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);      // quad_perm [2,3,0,1]
    v = dpp_add<0x141>(v);     // row_half_mirror
    v = dpp_add<0x140>(v);     // row_mirror: every lane of a row of 16 holds the row's sum
    const int b = __float_as_int(v);
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(b, 0)), r1 = __int_as_float(__builtin_amdgcn_readlane(b, 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(b, 32)), r3 = __int_as_float(__builtin_amdgcn_readlane(b, 48));
    return (r0 + r1) + (r2 + r3);
}

// The sums of four values over each group of LANES lanes: lane l returns that of value l & 3.  Two steps inside groups of
// four lanes turn four values per lane into one, the other steps then work on a single value: for 64 lanes 17 vector
// instructions where four sums of their own take 44.
template <int LANES>
__device__ __forceinline__ float lane_sum_4(const float (&v)[4], int lane)
{
    const bool b0 = (lane & 1) != 0, b1 = (lane & 2) != 0;
    auto exchange = [](float keep, float give, auto ctrl) {
        return keep + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(give), decltype(ctrl)::value, 0xF, 0xF, true));
    };
    const float r01 = exchange(b0 ? v[1] : v[0], b0 ? v[0] : v[1], std::integral_constant<int, 0xB1>{});   // lane ^ 1
    const float r23 = exchange(b0 ? v[3] : v[2], b0 ? v[2] : v[3], std::integral_constant<int, 0xB1>{});
    float r = exchange(b1 ? r23 : r01, b1 ? r01 : r23, std::integral_constant<int, 0x4E>{});               // lane ^ 2
    r = dpp_add<0x124>(r);                                         // rotations inside a row of 16 by 4 and 8
    r = dpp_add<0x128>(r);
    if constexpr (LANES >= 32) {
        auto p16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(r), __float_as_uint(r), false, false);     // rows 0 and 1, 2 and 3
        r = __uint_as_float(p16[0]) + __uint_as_float(p16[1]);
    }
    if constexpr (LANES == 64) {
        auto p32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(r), __float_as_uint(r), false, false);     // the halves
        r = __uint_as_float(p32[0]) + __uint_as_float(p32[1]);
    }
    return r;
}

// LANES lanes per nonzero (16 up to 64 topics, 32 up to 128, else 64), CH 16-byte loads of a lane per row (K <= 4 LANES CH).
// ALIGNED: K is a multiple of 4; else a row's last load is moved back into it and what it repeats is left out.
//
// Two things bound this kernel: the vector cache, which hands out 64 bytes a cycle, and what the second-level caches (4 MB on
// each of eight dies) miss, which comes in at some 6.6 TB/s whatever serves it.  Against the first, the theta row stays in
// registers over a run of nonzeros of one document.  Against the second, SLICES = 8: a workgroup takes the nonzeros whose
// word is congruent to its index mod 8, of a stretch of the matrix that seven neighbours look through as well.  Workgroups go
// round the dies in turn, so each die reads an eighth of the rows of phi and its cache holds eight times as many of
// those; theta rows are read eight times, which is little beside a row of phi per nonzero.  (Only time depends on where a
// workgroup runs.)
//
// A wave gathers its nonzeros of the stretch in LDS, then takes up to 64 of one document at a time, in rounds of four per
// group of lanes with the rows of the next round in flight (no conditional load between a load and the sum that waits for
// it: the compiler's wait would cover both).  ms per launch before (a wave per nonzero, both rows loaded for each) and now:
// 22 million news-shaped nonzeros at K = 256 1.77 and 1.20 (19 TB/s of phi rows), 6.7 million at K = 512 1.05 and 0.55, at
// 1000 2.5 and 0.91; 11 million at K = 100 0.62 and 0.23, at 50 0.60 and 0.11; 4.5 million at K = 333 1.18 and 0.34.
struct SddmmArgs {
    const int32_t* nz_doc; const int32_t* rowidx; int64_t nnz; int K;
    const float* theta; const float* phi; float* mu;
    int stretch;                       // nonzeros a wave looks through, at most kSddmmStretch
};
constexpr int kSddmmWaves = 4;         // per workgroup

template <int LANES, int CH, bool ALIGNED, int SLICES>
__global__ __launch_bounds__(64 * kSddmmWaves) void sddmm_kernel(SddmmArgs a)
{
    typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));
    __shared__ int2 list[kSddmmWaves][SLICES > 1 ? kSddmmStretch : 1];      // document and word
    __shared__ uint16_t list_at[kSddmmWaves][SLICES > 1 ? kSddmmStretch : 1];   // place in the stretch
    constexpr int kGroups = 64 / LANES, kRound = 4 * kGroups;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int sub = lane & (LANES - 1), grp = lane / LANES;
    const int K = a.K;
    const int slice = (int)(blockIdx.x % SLICES);
    const int64_t i0 = ((int64_t)(blockIdx.x / SLICES) * kSddmmWaves + wv) * a.stretch;
    if (i0 >= a.nnz) return;                                       // the whole wave
    const int here = a.nnz - i0 < a.stretch ? (int)(a.nnz - i0) : a.stretch;
    int n = here;                                                  // nonzeros to do
    if constexpr (SLICES > 1) {
        n = 0;
        constexpr int kTurns = 4;                                  // turns whose loads are in flight together
        for (int base = 0; base < here; base += 64 * kTurns) {
            int32_t d[kTurns], w[kTurns];
#pragma unroll
            for (int j = 0; j < kTurns; ++j) {
                const int i = base + 64 * j + lane;
                d[j] = a.nz_doc[i0 + (i < here ? i : 0)];
                w[j] = a.rowidx[i0 + (i < here ? i : 0)];
            }
#pragma unroll
            for (int j = 0; j < kTurns; ++j) {
                const int i = base + 64 * j + lane;
                const bool mine = i < here && w[j] % SLICES == slice;
                const uint64_t all = __ballot(mine);
                const int to = n + (int)__popcll((unsigned long long)(all & ((1ull << lane) - 1ull)));
                if (mine) { list[wv][to] = make_int2(d[j], w[j]); list_at[wv][to] = (uint16_t)i; }
                n += (int)__popcll((unsigned long long)all);
            }
        }
        // (a wave reads only what it wrote itself, and LDS serves a wave's accesses in order)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }

    // the lane's topics of every row: CH windows of four, inside the row; what a window repeats has a weight of zero
    int off[CH];
    bool ok[CH][4];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int k = 4 * (LANES * c + sub);
        off[c] = k < K - 4 ? k : K - 4;
#pragma unroll
        for (int j = 0; j < 4; ++j) ok[c][j] = off[c] + j >= k;
    }
    auto window = [&](const float* __restrict__ p) {
        if constexpr (ALIGNED) return *reinterpret_cast<const float4*>(p);
        const float4_any v = *reinterpret_cast<const float4_any*>(p);
        return make_float4(v.x, v.y, v.z, v.w);
    };
    int32_t held = -1;                                             // the document whose theta values t holds
    float4 t[CH];
    for (int e = 0; e < n; ) {
        const int mine = e + lane < n ? e + lane : n - 1;
        int at = mine;
        int32_t my_d, my_w;
        if constexpr (SLICES > 1) {
            const int2 dw = list[wv][mine];
            my_d = dw.x; my_w = dw.y; at = list_at[wv][mine];
        } else {
            my_d = a.nz_doc[i0 + mine]; my_w = a.rowidx[i0 + mine];
        }
        const int32_t doc = __builtin_amdgcn_readfirstlane(my_d);
        const uint64_t other = __ballot(e + lane >= n || my_d != doc);
        const int len = other ? __ffsll((unsigned long long)other) - 1 : 64;   // of this document, from e on
        if (doc != held) {
#pragma unroll
            for (int c = 0; c < CH; ++c) t[c] = window(a.theta + (size_t)doc * K + off[c]);
            held = doc;
        }
        auto rows = [&](int r, float4 (&p)[4][CH]) {               // the rows of round r
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int x = r * kRound + 4 * grp + j, src = x < len ? x : len - 1;
                const int32_t w = LANES == 64 ? __builtin_amdgcn_readlane(my_w, __builtin_amdgcn_readfirstlane(src)) : __shfl(my_w, src);
                const float* __restrict__ row = a.phi + (size_t)w * K;
#pragma unroll
                for (int c = 0; c < CH; ++c) p[j][c] = window(row + off[c]);
            }
        };
        auto sums = [&](int r, const float4 (&p)[4][CH]) {
            float s[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                s[j] = 0.f;
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    if constexpr (ALIGNED) {
                        float x = __builtin_fmaf(t[c].x, p[j][c].x, s[j]);
                        x = __builtin_fmaf(t[c].y, p[j][c].y, x);
                        x = __builtin_fmaf(t[c].z, p[j][c].z, x);
                        x = __builtin_fmaf(t[c].w, p[j][c].w, x);
                        s[j] = ok[c][0] ? x : s[j];
                    } else {
                        s[j] = ok[c][0] ? __builtin_fmaf(t[c].x, p[j][c].x, s[j]) : s[j];
                        s[j] = ok[c][1] ? __builtin_fmaf(t[c].y, p[j][c].y, s[j]) : s[j];
                        s[j] = ok[c][2] ? __builtin_fmaf(t[c].z, p[j][c].z, s[j]) : s[j];
                        s[j] = ok[c][3] ? __builtin_fmaf(t[c].w, p[j][c].w, s[j]) : s[j];
                    }
                }
            }
            const float v = lane_sum_4<LANES>(s, lane);
            const int x = r * kRound + 4 * grp + (lane & 3);
            const int to = __shfl(at, x < len ? x : len - 1);
            if (sub < 4 && x < len) a.mu[i0 + to] = v;
        };
        float4 pa[4][CH], pb[4][CH];
        const int rounds = (len + kRound - 1) / kRound;
        rows(0, pa);
        int r = 0;
        while (r + 2 < rounds) {                                   // pa holds round r; every sum has a round's loads behind it
            rows(r + 1, pb);
            __builtin_amdgcn_sched_barrier(0);
            sums(r, pa);
            __builtin_amdgcn_sched_barrier(0);
            rows(r + 2, pa);
            __builtin_amdgcn_sched_barrier(0);
            sums(r + 1, pb);
            __builtin_amdgcn_sched_barrier(0);
            r += 2;
        }
        if (r + 1 < rounds) {
            rows(r + 1, pb);
            __builtin_amdgcn_sched_barrier(0);
            sums(r, pa);
            sums(r + 1, pb);
        } else {
            sums(r, pa);
        }
        e += len;
    }
}

// Fewer than four topics: a thread per nonzero.
__global__ __launch_bounds__(256) void sddmm_few_kernel(SddmmArgs a)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= a.nnz) return;
    const float* __restrict__ t = a.theta + (size_t)a.nz_doc[i] * a.K;
    const float* __restrict__ p = a.phi + (size_t)a.rowidx[i] * a.K;
    float s = 0.f;
    for (int k = 0; k < a.K; ++k) s = __builtin_fmaf(t[k], p[k], s);
    a.mu[i] = s;
}

}  // namespace same
