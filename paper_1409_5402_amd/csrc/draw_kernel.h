// Draw-and-scatter kernel of the SAME LDA sweep (Algorithm 3, the loop over document-word pairs;
// Section 4, multinomial form of the factored draw) for gfx950.
//
// One wave per workgroup takes 64 draw tasks (a task: a group of tokens of one nonzero) through two
// phases.
//
// Scan (lanes across topics).  Two tasks at a time, one per half-wave: lane l of a half owns block l of
// its task's topics, T = 4*ceil(K/128) consecutive topics (T = 8 at K = 256: the 32 lanes read the
// task's phi row and its document's theta row as two 16-byte loads each), multiplies them
// (w_k = theta[d][k] * phi[w][k]) and adds the block's weights left to right.  The 32 block sums of a
// task go to LDS.  No random numbers are used here and nothing is kept per topic.  (Up to 64 topics four, eight or
// sixteen tasks go at a time, scan_lanes lanes each; at K = 512 and from 897 to 1024 the lanes of a half read consecutive
// 16-byte pieces instead and share the blocks' sums: see COAL below.)
//
// Draw (one lane per task).  A lane first turns its task's block sums into running sums S_0..S_31 (left to
// right, so S_l is the cumulative weight at the end of block l and S_31 = mu, the normaliser of
// Algorithm 3; in LDS word l holds the weight below block l, S_{l-1}).  The cumulative weight at topic k of block l is P_k = S_{l-1} + (running sum inside the
// block): topic k owns the interval (P_{k-1}, P_k] of (0, mu).  The N = m*g copies are N uniform points
// on (0, mu); they are placed from the top, one step per topic that receives copies.  With R copies
// left, all below U:
//   - the highest one sits at y = U * u^(1/R) (one uniform, the R-th root by the fixed log/exp
//     sequences of rng_binom.h);
//   - its block is the first l with S_l >= y (binary search in LDS); the lane reloads that one block's
//     theta and phi values, rebuilds its P_k and takes the first k with P_k >= y;
//   - the other R-1 copies are uniform below y: 1 + Binomial(R-1, (y - P_{k-1}) / y) copies go to k
//     (exact inversion sampler), the rest continue below U = P_{k-1}.
// The work of a task is proportional to the number of topics that receive copies, not to K, and the
// second visit of a row touches only the blocks that receive copies.
//
// Lanes differ in the number of steps and in the length of their pmf walks; the draw therefore runs as a
// per-lane state machine: every trip lets each lane either take its next step or advance its walk by
// a few terms, so lanes with long walks do not hold up lanes with many short steps.  A binomial that
// the sampler cuts into several pieces (independent, one uniform each) is handed to the whole wave,
// one piece per lane.  Two consecutive steps of a task share one Philox block.
#pragma once
#include <type_traits>
#include "launch_shape.h"
#include "scatter.h"

namespace same {

constexpr int kSumStride = kMaxBlocks + 1;      // words between the block sums of two tasks in LDS (more than 64 topics): lanes
                                                // that read the same block of 64 different tasks hit 32 different banks

// Lanes that scan a task, and words between the sums of two tasks in LDS: a power of two that covers the blocks of up to
// 128 topics (blocks of four: one 16-byte load per lane and matrix), 32 beyond, and a padding word.
__host__ __device__ inline int scan_lanes(int K) { return K <= 16 ? 4 : (K <= 32 ? 8 : (K <= 64 ? 16 : kMaxBlocks)); }
__host__ __device__ inline int sum_stride(int K) { return scan_lanes(K) + 1; }

// Rows of document counts a wave keeps in LDS: two up to K = 128, one up to K = 1024 (4 KB at most), none beyond.
// A second row at K = 256 would serve the waves that straddle two documents, but its kilobyte costs two of the
// fifteen waves a compute unit holds, which costs more.
__host__ __device__ inline int doc_rows(int K) { return K <= 128 ? 2 : (K <= 1024 ? 1 : 0); }

// The value of v in the next lower lane (lanes 0, 16, 32, 48 receive 0): a row shift inside the vector ALU.
__device__ __forceinline__ float from_lane_below(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x111, 0xf, 0xf, true));
}

// Position of the highest of R copies uniform on (0, U).
__device__ __forceinline__ float top_position(float U, uint32_t R, float u)
{
    const float a = -flog(u);
    const float z = quot_int(a, (float)R);                         // 2^-24 < a < 17
    const float e = __builtin_fminf(expneg(z), 1.0f);
    float y = (R == 1u) ? U * u : U * e;
    if (!(y > 0.0f)) y = U;
    return y;
}

// Four consecutive floats of a row of K at topic e.  ALIGNED (K is a multiple of 4): one aligned load, zeros from K on.
// Else: one load that needs only the alignment of a float, moved back where it would leave the row; shift_quad then puts
// the four products in their places.
typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));
template <bool ALIGNED, bool WHOLE>
__device__ __forceinline__ float4 load_quad(const float* __restrict__ row, int e, int K)
{
    if constexpr (ALIGNED) {
        return (WHOLE || e < K) ? *reinterpret_cast<const float4*>(row + e) : make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
        const float4_any v = *reinterpret_cast<const float4_any*>(row + (e < K - 4 ? e : K - 4));
        return make_float4(v.x, v.y, v.z, v.w);
    }
}
typedef __attribute__((address_space(3))) float lds_float;
template <bool ALIGNED, bool WHOLE>
__device__ __forceinline__ float4 lds_quad(const lds_float* row, int e, int K)
{
    typedef float f4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) f4 lds_f4;
    typedef __attribute__((address_space(3))) float4_any lds_f4_any;
    if constexpr (ALIGNED) {
        if (!WHOLE && e >= K) return make_float4(0.f, 0.f, 0.f, 0.f);
        const f4 v = *(const lds_f4*)(row + e);
        return make_float4(v.x, v.y, v.z, v.w);
    } else {
        const float4_any v = *(const lds_f4_any*)(row + (e < K - 4 ? e : K - 4));
        return make_float4(v.x, v.y, v.z, v.w);
    }
}
// x holds the values of topics min(e, K-4) ..: moves them so that x[0] is topic e's; topics from K on are zero
template <bool ALIGNED>
__device__ __forceinline__ void shift_quad(float (&x)[4], int e, int K)
{
    if constexpr (!ALIGNED) {
        const int s = e - (K - 4);                                 // places to move by, none if negative
        const bool one = s > 0 && (s & 1) != 0, two = s > 0 && (s & 2) != 0, all = s >= 4;
        x[0] = one ? x[1] : x[0]; x[1] = one ? x[2] : x[1]; x[2] = one ? x[3] : x[2]; x[3] = one ? 0.f : x[3];
        x[0] = two ? x[2] : x[0]; x[1] = two ? x[3] : x[1]; x[2] = two ? 0.f : x[2]; x[3] = two ? 0.f : x[3];
        x[0] = all ? 0.f : x[0]; x[1] = all ? 0.f : x[1]; x[2] = all ? 0.f : x[2]; x[3] = all ? 0.f : x[3];
    }
}

// The first of N ascending values that reaches y, when the last one is known to: its index; prev
// becomes the value before it (it comes in as the value before the first).  A search whose answer stays in registers: at
// N = 8 it takes 3 comparisons and 10 selections where a walk along the values takes 7 and 14.
template <int N>
__device__ __forceinline__ int first_reaching(float (&P)[N], float y, float& prev)
{
    constexpr int M = N <= 4 ? 4 : (N <= 8 ? 8 : (N <= 16 ? 16 : 32));
    int idx = 0;
#pragma unroll
    for (int h = M / 2; h > 0; h >>= 1) {
        const float at = P[h <= N ? h - 1 : 0];
        const bool below = h <= N && !(at >= y);                   // (N is no power of two: the last value stands for the rest)
        prev = below ? at : prev;
        idx = below ? idx + h : idx;
#pragma unroll
        for (int j = 0; j < h - 1; ++j) if (j < N) {
            const float lo = P[j], hi = P[j + h < N ? j + h : N - 1];   // values: selected as elements of the array they become
            P[j] = below ? hi : lo;                                     // a variable index, 25 comparisons at N = 8
        }
    }
    return idx;
}

constexpr int kRecips = 64;     // reciprocals 1/x that a wave keeps in LDS for its pmf walks: a multiple of kWalkSteps

// Idle lanes that make the wave fetch new tasks: kRefillMin; fewer are enough when the last refill is kRefillLateTrips
// trips back, since tasks are then long and a refill is a small part of their cost (from a flat posterior, 83 steps per
// task, 12 of the 64 lanes were idle on average; converged, a refill comes every three trips).
constexpr int kRefillMin = 24;
constexpr int kRefillLate = 8;
constexpr int kRefillLateTrips = 8;
// VEC: K is a multiple of 4 (rows are aligned to 16 bytes), else loads of any alignment (load_quad).  TB: 16-byte loads per
// matrix that a lane has in flight at a time: a block of T = 4 ceil(K / 128) topics is read in T / (4 TB) batches of TB
// loads per matrix.  ONE: a block is a single batch (up to 896 topics: TB = T / 4, 1 to 7; a K of 300, 640, 768 or 896 in
// batches of one load took 1.5 to 3 times as long).  TB = 0: fewer than four topics, element by element.  KC > 0: the
// same kernel with the number of topics a constant (row addresses become shifts, the bounds of the loads vanish).
// COAL (TB = 4: blocks of 16 topics in one batch, or of 32 in two): in the scan a load covers 128 consecutive topics per
// half-wave, four per lane, instead of four topics of every lane's own block: a wave's load touches 8 cache lines, not 32
// or 64, and the cache serves a load one line at a time.  The lanes that hold a block then add its products in the
// same left-to-right order through a chain of lane-to-lane shifts; the block sums are the same bits.  From 897 topics it
// halves the kernel (1.87 -> 0.91 ms at K = 1000, 9000 news-shaped documents, m = 10); at K = 512 it is even with the other
// form and at 385 to 511 topics 8 % slower (0.65 against 0.60 ms), so those use the other one.  The steps' reloads of
// single blocks stay as they are (a lane's block belongs to its own task).
//
// The launch positions (tasks in storage order) are shared out in rounds.  A launch has as many workgroups (of one wave)
// as the device holds at once.  In round 0 every workgroup owns a.first consecutive positions, about half of an equal
// share, without asking; in round r a share has a.first / 2^r positions (at least kShareMin), and a workgroup draws a
// ticket for one when its own positions are used up.  Its lanes take positions as they become free: tasks differ widely
// in the number of steps they need (one for most, a hundred for a few), so a lane that waited for the slowest of 64
// fixed tasks would idle most of the time, and a wave with a fixed share of the matrix would end with one lane busy.
// Whenever kRefillMin lanes are idle the wave stops stepping, gives each idle lane the next position, scans the new tasks
// (two per instruction) and goes on.
//
// Heavy tasks first.  The largest groups of tokens (at most one in 256 tasks) place copies on nearly every topic
// from a flat posterior, 256 steps where a single token takes 83, and a launch ended with a few waves stepping through
// the ones that had been taken last: 1.7 of 9.9 ms for 6 million tasks at K = 256.  The workgroups share a list of them
// out before round 0 and pass over them afterwards.
//
// (How shares and tickets are dealt out: launch_shape.h.)
//
// THETA: the document of the row of counts also has its row of theta in LDS, for the reload of a step's block (theta_rows in
// launch_shape.h).
//
// Waves per SIMD: five for fewer than four topics (60,000 documents of 30 tokens, m = 1 and 100: K = 3 with four 13 and 5 % slower,
// K = 1 12 and 12 %), four where 128 registers hold the kernel, else three, and two where three would keep up to 63 registers and
// 140 bytes a lane in scratch (rows that are not aligned from 641 to 1024 topics, 7 loads per matrix in flight).  ms per draw with
// three / two, documents of 60 tokens from a flat posterior and of 330 with topics formed, m = 16 and then 100: K = 701 1.90 / 1.65,
// 1.32 / 1.12 and 6.23 / 5.37, 3.08 / 2.69; K = 895 3.21 / 1.99, 2.04 / 1.27 and 12.2 / 6.08, 5.52 / 2.90; K = 896 1.80 / 1.69,
// 1.19 / 1.09 and 5.71 / 5.16, 2.59 / 2.36; K = 1001 2.69 / 2.31, 1.49 / 1.43 and 9.23 / 7.37, 3.39 / 3.33, but at m = 1 0.80 / 0.88
// and 0.72 / 0.73.
constexpr int draw_waves(bool uniform, bool vec, int tb, bool one, int kc, bool coal)
{
    if (uniform) return 6;
    if (tb == 0) return 5;
    if (tb <= 3) return 4;
    return (one && tb == 7) || (!vec && ((one && tb == 6) || (coal && kc == 0))) ? 2 : 3;
}
template <bool UNIFORM, bool VEC, bool DEBUG, int TB, bool ONE, int KC = 0, bool COAL = false, bool THETA = false>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(draw_waves(UNIFORM, VEC, TB, ONE, KC, COAL)))) void draw_kernel(DrawArgs a)
{
    extern __shared__ __align__(16) uint32_t lds[];
    constexpr bool SMALL = !UNIFORM && KC == 0 && (TB == 0 || (TB == 1 && ONE));   // up to 128 topics: blocks of four
    const int kStride = UNIFORM ? 1 : (SMALL ? sum_stride(a.K) : kSumStride);      // (weights of one need no sums)
    const float* recips = reinterpret_cast<const float*>(lds);     // [kRecips]: 1, 1/2, 1/3, ...
    float* sums = reinterpret_cast<float*>(lds) + kRecips;         // [64 lanes][kStride]: block sums, then the weight below each block
    uint32_t* acc = lds + kRecips + (kStride - 1);                 // piece totals by owner lane: lane l's is acc[l * kStride],
                                                                   // the word of its row of sums that pads the stride
    const int lane = threadIdx.x;
    const int K = KC > 0 ? KC : a.K;                              // KC: the number of topics where it is known at compile time
    const int T = (TB > 0 && ONE) ? 4 * TB : block_len(K);         // topics per block
    const int nb = (TB > 0 && !ONE) ? T / (4 * (TB > 0 ? TB : 1)) : 1;   // batches of loads per block
    const int nblk = (K + T - 1) / T;                              // blocks in use (<= 32)
    const int half = lane >> 5, hl = lane & 31;
    // Rows of the new document counts kept in LDS while the wave works on their documents (the launch positions are
    // in storage order: the 64 lanes hold tasks of one or two documents at a time).  Counts are added here and
    // reach the matrix in one pass over the row when the wave has left the document; tasks of a document that
    // has no row here add to the matrix at once.
    uint32_t* rows = lds + kRecips + (size_t)kWave * kStride;      // [n_rows][K]
    const int n_rows = DEBUG && !THETA ? 0 : doc_rows(K);          // (DEBUG: for the row of theta alone)
    int tag0 = -1, tag1 = -1;                                      // the documents of rows 0 and 1 (wave-uniform), -1: free
    int myrow = -1;                                                // the row of this lane's document, -1: none
    for (int i = lane; i < n_rows * K; i += kWave) rows[i] = 0u;
    static_assert(!THETA || (ONE && TB >= 3 && !UNIFORM), "theta_rows");
    float* th_row_lds = reinterpret_cast<float*>(rows) + K;        // THETA: [K], theta of that document (one row at these K)
    // the wave's positions not yet handed out
    int32_t next, end;
    bool heavy;                                                    // they are positions of the list of heavy tasks
    {
        const int64_t each = ((int64_t)a.n_heavy + gridDim.x - 1) / gridDim.x;
        const int64_t from = (int64_t)blockIdx.x * each;
        next = (int32_t)(from < a.n_heavy ? from : a.n_heavy);
        end = (int32_t)(from + each < a.n_heavy ? from + each : a.n_heavy);
        heavy = true;
    }
    bool drained = false;                                          // nothing is left to take
    ChunkSupply supply(a);
    acc[lane * kStride] = 0u;
    static_assert(kRecips == kWave, "a reciprocal per lane");
    reinterpret_cast<float*>(lds)[lane] = inv_int((float)(lane + 1));
    __syncthreads();
    const float* my_sums = sums + lane * kStride;

    // ---- the lane's current task
#ifdef SAME_STATS
    uint32_t R_task_g = 0;
#endif
    bool open = false;      // a task was taken and its slot of the pair list is not yet closed
    int32_t d = 0, w = 0;
    // Its rows of theta and phi, as addresses: from d and w they take nine instructions a step (more where K is no constant).
    // Not where the four registers are not to be had without spilling others (rows that are not aligned up to 128 topics: six in scratch
    // with them, K = 125 at m = 100 1.119 and 1.070 ms a sweep), and not at K = 1024 (from a flat posterior
    // at m = 100, documents of 60 and 330 tokens, 6.17 and 6.86 ms with them, 5.90 and 6.67 without).
    constexpr bool kRowAddr = KC == 256 || KC == 512 ||
                              (KC == 0 && ONE && (TB == 0 || (TB == 1 && VEC) || TB == 2 || TB == 4 || (TB == 5 && (VEC || !THETA))));
    const float* th_row = a.theta;
    const float* ph_row = a.phi;
    Scatter sc;
    sc.drow = 0; sc.dst = nullptr; sc.npairs = 0;
    Staged staged;          // its last pairs, on their way to the pair list
    StreamKey key;
    key.seed_lo = a.seed_lo; key.seed_hi = a.seed_hi; key.tau_lo = 0; key.tau_hi = 0; key.pass = a.pass;
    PrimaryPre pre = primary_pre(key);

    // ---- the draw of that task: a per-lane state machine
    uint32_t R = 0;         // copies not yet placed, all of them below U
    float U = 0.0f;
    int top = K;            // the copies left belong to topics below top
    uint32_t step = 0;      // steps taken: the next one uses words 2*(step & 1), +1 of block step >> 1
    uint32_t xs2 = 0, xs3 = 0;   // the second half of the last Philox block, for the odd step
    int st = 0;             // 0: between steps, 1: walking a single-piece binomial,
                            // 3: holds a binomial of several pieces, waiting for the wave to share it
    uint32_t bR = 0, L = 0, bstep = 0;
    float r = 0.f, lq = 0.f, pm = 0.f, cdf = 0.f, u = 0.f;
    float left = 0.f;                                              // the walk: trials not yet counted as successes
    int walked = 0;                                                // and terms added in earlier trips
    bool flip = false;
    int kk = 0;

    int trips = 0;          // trips since the last refill
    int waited = 0;         // trips since a binomial of several pieces has been waiting

    // Adds row i of the LDS counts to the matrix row of document doc and clears it (whole wave).
    auto flush_row = [&](int i, int doc) {
        __syncthreads();
        if (!DEBUG) for (int k = lane; k < K; k += kWave) {
            const uint32_t v = rows[i * K + k];
            if (v) { add_global(a.ndk + (size_t)doc * K + k, v); rows[i * K + k] = 0u; }
        }
        __syncthreads();
    };

    // Theta of document doc beside its LDS counts (whole wave).
    auto load_theta = [&](int doc) {
        if (THETA) {
            const float* __restrict__ t = a.theta + (size_t)doc * K;
            for (int k = lane; k < K; k += kWave) th_row_lds[k] = t[k];
        }
    };

    // Idle lanes take the next positions, the wave scans the new tasks' block sums (two tasks at a time, one
    // per half-wave: lane hl of a half owns block hl), each new lane turns its sums into running sums.
    auto refill = [&](uint64_t idle_mask) {
        const bool idle = (idle_mask >> lane) & 1ull;
        if (idle && open) { sc.close(true, staged); open = false; }
        const int rank = (int)__popcll(idle_mask & ((1ull << lane) - 1ull));
        const int avail = end - next;
        bool take = idle && rank < avail;
        if (take) {
            const int64_t pos = (int64_t)next + rank;
            const int64_t tau = DEBUG ? a.ids[pos] : (heavy ? (int64_t)a.heavy[pos] : pos);
            d = a.t_doc[tau];
            w = a.t_word[tau];
            const uint32_t tokens = a.t_g[tau];
            if (!UNIFORM && kRowAddr) { th_row = a.theta + (size_t)d * K; ph_row = a.phi + (size_t)w * K; }
#ifdef SAME_STATS
            R_task_g = tokens;
#endif
            sc = make_scatter<DEBUG>(a, pos, tau, d);
            key.tau_lo = (uint32_t)tau; key.tau_hi = (uint32_t)((uint64_t)tau >> 32) & 0xFFu;
            pre = primary_pre(key);
            take = heavy || tokens < a.heavy_from;                 // a heavy task has had its turn
            open = take;
            R = take ? a.m * tokens : 0u;
            top = K; step = 0; st = 0;
        }
        const int n_idle = (int)__popcll(idle_mask);
        next += n_idle < avail ? n_idle : avail;
        uint64_t fresh = __ballot(take);
        if (n_rows > 0) {
            // lanes that keep working keep their row; a new task joins the row of its document if there is one;
            // documents that are new to the wave get the rows no lane uses any more, lowest document first
            if (idle) myrow = -1;
            if (take) myrow = d == tag0 ? 0 : ((n_rows > 1 && d == tag1) ? 1 : -1);
            for (int round = 0; round < n_rows; ++round) {
                const uint64_t used0 = __ballot(myrow == 0), used1 = __ballot(myrow == 1);
                const int free_row = used0 == 0 ? 0 : ((n_rows > 1 && used1 == 0) ? 1 : -1);
                const uint64_t rowless = __ballot(take && myrow < 0);
                if (rowless == 0) break;
                const int dn = __builtin_amdgcn_readlane(d, __ffsll((unsigned long long)rowless) - 1);   // the lowest of their documents
                if (free_row < 0) {
                    // one row (n_rows == 1) in use: it goes to the new document if that one now has more lanes than
                    // the row's document has left; the lanes that stay behind add to the matrix directly from here on
                    if (n_rows != 1) break;
                    const int n_new = (int)__popcll((unsigned long long)__ballot(take && myrow < 0 && d == dn));
                    if (n_new <= (int)__popcll((unsigned long long)used0)) break;
                    flush_row(0, tag0);
                    if (myrow == 0) myrow = -1;
                    tag0 = dn;
                    load_theta(dn);
                    if (take && d == dn) myrow = 0;
                    break;
                }
                const int old = free_row == 0 ? tag0 : tag1;
                if (old >= 0) flush_row(free_row, old);
                if (free_row == 0) tag0 = dn; else tag1 = dn;
                load_theta(dn);
                if (take && d == dn) myrow = free_row;
            }
        }
        if (!UNIFORM) {
            const int k0 = scan_first_topic(hl, T, nblk);
            // the next pair of new lanes: one for each half-wave (the last one twice if their number is odd)
            auto pick = [&](uint64_t& rem) {
                const int la = __ffsll((unsigned long long)rem) - 1;
                rem &= rem - 1;
                int lb = la;
                if (rem) { lb = __ffsll((unsigned long long)rem) - 1; rem &= rem - 1; }
                return half ? lb : la;
            };
            if constexpr (SMALL && TB > 0) {
                // Up to 128 topics: scan_lanes lanes of the wave per task, 64 / scan_lanes tasks per load.  The words and
                // documents of the new tasks are brought into the order of their ranks first (a lane of rank r keeps
                // task r's), so that a group of lanes finds its next task by a lane-to-lane read.
                const int per = scan_lanes(K), at_once = kWave / per;
                const int sub = lane & (per - 1), grp = lane / per, n_new = (int)__popcll((unsigned long long)fresh);
                const int at = (int)__popcll((unsigned long long)(fresh & ((1ull << lane) - 1ull)));   // rank among the new tasks
                const int to = (take ? at : 63) * 4;               // lanes without a new task all write to lane 63 ...
                int who = __builtin_amdgcn_ds_permute(to, take ? lane : -1);
                if (n_new < kWave && lane >= n_new) who = 0;       // ... which then has no task of its own
                const int32_t w_r = __shfl(w, who), d_r = __shfl(d, who);
                const int e = 4 * sub;
                auto fetch = [&](int i, float4& p, float4& t, int& src) {
                    int r = i * at_once + grp;
                    r = r < n_new ? r : n_new - 1;                 // past the last one: its task once more
                    const int32_t pw = __shfl(w_r, r), pd = __shfl(d_r, r);
                    src = __shfl(who, r);
                    p = load_quad<VEC, false>(a.phi + (size_t)pw * K, e, K);
                    t = load_quad<VEC, false>(a.theta + (size_t)pd * K, e, K);
                };
                auto total = [&](const float4& p, const float4& t, int src) {
                    float x[4] = {t.x * p.x, t.y * p.y, t.z * p.z, t.w * p.w};
                    shift_quad<VEC>(x, e, K);
                    float rs = 0.0f + x[0];
                    rs = rs + x[1];
                    rs = rs + x[2];
                    rs = rs + x[3];
                    if (sub < nblk) sums[src * kStride + sub] = rs;
                };
                if (n_new > 0) {
                    float4 p0, t0, p1, t1;
                    int s0, s1;
                    const int turns = (n_new + at_once - 1) / at_once;
                    fetch(0, p0, t0, s0);
                    int i = 0;
                    for (; i + 2 < turns; i += 2) {                // the loads of the next turn behind every sum
                        fetch(i + 1, p1, t1, s1);
                        __builtin_amdgcn_sched_barrier(0);
                        total(p0, t0, s0);
                        __builtin_amdgcn_sched_barrier(0);
                        fetch(i + 2, p0, t0, s0);
                        __builtin_amdgcn_sched_barrier(0);
                        total(p1, t1, s1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (i + 1 < turns) {
                        fetch(i + 1, p1, t1, s1);
                        total(p0, t0, s0);
                        total(p1, t1, s1);
                    } else {
                        total(p0, t0, s0);
                    }
                }
            } else if constexpr (TB > 0) {
                // Where every block in use is whole (256 at T = 8, 200 with 25 of them) the loads need no bounds.  Blocks of one batch
                // (ONE) and of two batches of four loads go through the pipeline in run(); blocks of other shapes load
                // the next batch into a second set of registers before the current one is summed (the load there sits
                // under a condition, and the compiler's wait then covers it too: no overlap, rare shapes).
                struct Item { int src, b; bool last, valid; };
                auto advance = [&](Item& it) {                     // the next (pair of tasks, batch) of this refill
                    if (it.valid && !it.last) { it.b += 1; it.last = it.b == nb - 1; return; }
                    if (fresh == 0) { it.valid = false; return; }
                    it.src = pick(fresh); it.b = 0; it.last = nb == 1; it.valid = true;
                };
                auto run = [&](auto whole) {
                    constexpr bool WHOLE = decltype(whole)::value;
                    auto issue = [&](float4* pv, float4* tv, const Item& it) {     // blocks of several batches
                        const int32_t pd = __shfl(d, it.src), pw = __shfl(w, it.src);
                        const int kb = COAL ? 128 * TB * it.b + 4 * hl : k0 + 4 * TB * it.b;
                        constexpr int kStep = COAL ? 128 : 4;      // topics between two loads of a lane
#pragma unroll
                        for (int c = 0; c < TB; ++c) {
                            pv[c] = load_quad<VEC, WHOLE>(a.phi + (size_t)pw * K, kb + kStep * c, K);
                            tv[c] = load_quad<VEC, WHOLE>(a.theta + (size_t)pd * K, kb + kStep * c, K);
                        }
                    };
                    float rs = 0.0f;
                    auto consume = [&](const float4* pv, const float4* tv, const Item& it) {
                        if constexpr (COAL) {
                            // A load covers 128 consecutive topics of the task, four per lane: the kNL lanes that hold a block
                            // add its products left to right, the running sum handed from lane to lane.  Every lane
                            // runs all kNL stages; stage j is meaningful in the block's lane j, and the block's last lane
                            // ends with the same sum, rounded in the same order, as one lane that adds the block alone.
                            constexpr int kNL = ONE ? TB : 2 * TB; // lanes per block of 16 (one batch) or 32 topics (two)
                            static_assert(!COAL || TB == 4, "blocks must not straddle loads");
#pragma unroll
                            for (int c = 0; c < TB; ++c) {
                                float x[4] = {tv[c].x * pv[c].x, tv[c].y * pv[c].y, tv[c].z * pv[c].z, tv[c].w * pv[c].w};
                                shift_quad<VEC>(x, 128 * (TB * it.b + c) + 4 * hl, K);
                                const float x0 = x[0], x1 = x[1], x2 = x[2], x3 = x[3];
                                float s = 0.0f;
#pragma unroll
                                for (int j = 0; j < kNL; ++j) {
                                    const float in = j == 0 ? 0.0f : from_lane_below(s);
                                    s = in + x0;
                                    s = s + x1;
                                    s = s + x2;
                                    s = s + x3;
                                }
                                if ((hl & (kNL - 1)) == kNL - 1)
                                    sums[it.src * kStride + (TB * it.b + c) * (32 / kNL) + hl / kNL] = s;
                            }
                            return;
                        }
#pragma unroll
                        for (int c = 0; c < TB; ++c) {
                            float x[4] = {tv[c].x * pv[c].x, tv[c].y * pv[c].y, tv[c].z * pv[c].z, tv[c].w * pv[c].w};
                            shift_quad<VEC>(x, k0 + 4 * (TB * it.b + c), K);
                            rs = rs + x[0];
                            rs = rs + x[1];
                            rs = rs + x[2];
                            rs = rs + x[3];
                        }
                        if (it.last) { sums[it.src * kStride + hl] = rs; rs = 0.0f; }
                    };
                    // Blocks of one batch, or of two (K = 1024).  The new tasks of a refill are worked off in runs whose
                    // document stays the same (a document's tasks are consecutive): the run's theta values are loaded once,
                    // one set of registers per batch, and the phi loads of the next batch are in flight while a batch is
                    // summed, in two sets used in turn (with two batches per block a set always holds the same batch).
                    // The loop has the same number of loads behind every sum on every path that reaches it: the
                    // compiler's wait then lets the younger loads fly.
                    auto pipeline = [&](auto batches) {
                        constexpr int NB = decltype(batches)::value;   // batches per block: 1 or 2
                        constexpr int N = 2;                       // sets of phi registers
                        constexpr int kStep = COAL ? 128 : 4;      // topics between two loads of a lane
                        constexpr int kBatch = COAL ? 128 * TB : 4 * TB;   // topics between two batches of a lane
                        const int kb0 = COAL ? 4 * hl : k0;
                        float4 pv[N][TB > 0 ? TB : 1], tv[NB][TB > 0 ? TB : 1];
                        int srcs[N];
                        int32_t held = -1;                         // the document whose theta values tv holds
                        int src_cur = 0;
                        const float* __restrict__ row_cur = a.phi; // the phi row of the pair whose batches are being issued
                        auto lane_of = [&](uint64_t m) { return __ffsll((unsigned long long)m) - 1; };
                        auto of_lane = [&](int32_t v, int l0, int l1) {    // v of lane l0 (first half-wave) or l1 (second)
                            const int32_t va = __builtin_amdgcn_readlane(v, l0), vb = __builtin_amdgcn_readlane(v, l1);
                            return half ? vb : va;
                        };
                        // batch i % NB of pair i / NB of the run goes to set i % N: with N = 2 and NB = 1 or 2 the batch
                        // of a set is known at compile time (j % NB)
                        auto issue_phi = [&](float4* p, int& src, int bt) {
                            if (bt == 0) {                         // the next pair of the run
                                const int l0 = lane_of(fresh);
                                fresh &= fresh - 1;
                                const int l1 = fresh ? lane_of(fresh) : l0;
                                fresh &= fresh - 1;
                                src_cur = half ? l1 : l0;
                                row_cur = a.phi + (size_t)of_lane(w, l0, l1) * K;
                            }
                            src = src_cur;
                            const int kb = kb0 + kBatch * bt;
#pragma unroll
                            for (int c = 0; c < TB; ++c)
                                p[c] = load_quad<VEC, WHOLE>(row_cur, kb + kStep * c, K);
                        };
                        auto sum_batch = [&](const float4* p, int src, int bt) {
                            Item it{src, bt, bt == NB - 1, true};
                            consume(p, tv[bt], it);
                        };
                        while (fresh) {
                            const int32_t doc = __builtin_amdgcn_readlane(d, lane_of(fresh));
                            const uint64_t other = fresh & ~__ballot(d == doc);
                            const uint64_t lead = other ? fresh & ((other & (~other + 1ull)) - 1ull) : fresh;
                            const int lanes_in = (int)__popcll((unsigned long long)lead);
                            // pairs inside the document; a lane left over is scanned alone, as its own partner, when
                            // nothing else of its document is left
                            int pairs = lanes_in / 2;
                            uint64_t rest = 0;                     // new lanes set aside while this run is scanned
                            if (pairs == 0) { pairs = 1; rest = fresh & (fresh - 1); fresh &= ~rest; }
                            else {
                                rest = fresh & ~lead;
                                if (lanes_in & 1) rest |= 1ull << (63 - __clzll((unsigned long long)lead));
                                fresh &= ~rest;
                            }
                            const int P = pairs * NB;              // batches of the run
                            if (doc != held) {
                                const float* __restrict__ tp = a.theta + (size_t)doc * K;
#pragma unroll
                                for (int bt = 0; bt < NB; ++bt)
#pragma unroll
                                    for (int c = 0; c < TB; ++c) {
                                        tv[bt][c] = load_quad<VEC, WHOLE>(tp, kb0 + kBatch * bt + kStep * c, K);
                                    }
                                held = doc;
                            }
                            issue_phi(pv[0], srcs[0], 0);          // P >= 1
                            int issued = 1;
                            while (P - issued >= N) {              // whole rounds: every sum has the loads of one batch behind it
#pragma unroll
                                for (int j = 0; j < N; ++j) {
                                    issue_phi(pv[(j + 1) % N], srcs[(j + 1) % N], (j + 1) % NB);
                                    __builtin_amdgcn_sched_barrier(0);     // the loads first, then the sum that waits
                                    sum_batch(pv[j], srcs[j], j % NB);
                                    __builtin_amdgcn_sched_barrier(0);
                                }
                                issued += N;
                            }
                            if (P - issued == 1) {                 // one batch not yet issued: it goes to set 1
                                issue_phi(pv[1], srcs[1], 1 % NB);
                                sum_batch(pv[0], srcs[0], 0);
                                sum_batch(pv[1], srcs[1], 1 % NB);
                            } else {
                                sum_batch(pv[0], srcs[0], 0);
                            }
                            fresh = rest;
                        }
                    };
                    if constexpr (ONE) {
                        pipeline(std::integral_constant<int, 1>{});
                        return;
                    } else if constexpr (TB == 4) {
                        if (nb == 2) {
                            pipeline(std::integral_constant<int, 2>{});
                            return;
                        }
                    }
                    float4 pa[TB > 0 ? TB : 1], ta[TB > 0 ? TB : 1], pb[TB > 0 ? TB : 1], tb[TB > 0 ? TB : 1];
                    Item cur{0, 0, false, false};
                    advance(cur);
                    if (cur.valid) issue(pa, ta, cur);
                    while (cur.valid) {
                        Item nxt = cur;
                        advance(nxt);
                        if (nxt.valid) issue(pb, tb, nxt);
                        consume(pa, ta, cur);
                        if (!nxt.valid) break;
                        cur = nxt;
                        advance(cur);
                        if (cur.valid) issue(pa, ta, cur);
                        consume(pb, tb, nxt);
                    }
                };
                if (KC > 0 || (VEC && !COAL && blocks_fill_row(K))) run(std::true_type{}); else run(std::false_type{});
            } else {   // fewer than four topics
                while (fresh) {
                    const int src = pick(fresh);
                    const int32_t pd = __shfl(d, src), pw = __shfl(w, src);
                    const float* __restrict__ tp = a.theta + (size_t)pd * K;
                    const float* __restrict__ pp = a.phi + (size_t)pw * K;
                    float rs = 0.0f;
                    for (int j = 0; j < T; ++j) if (k0 + j < K) rs = rs + tp[k0 + j] * pp[k0 + j];
                    if (hl < nblk) sums[src * kStride + hl] = rs;
                }
            }
        }
        __syncthreads();
        if (take) {
            float run = 0.0f;
            if (UNIFORM) {
                run = (float)K;                                    // weights of one need no sums
            } else {
                for (int l = 0; l < nblk; ++l) {                   // word l becomes the weight below block l
                    const float b = sums[lane * kStride + l];
                    sums[lane * kStride + l] = run;
                    run = run + b;
                }
                // the steps' search probes up to the next power of two
                if (KC == 0) for (int l = nblk; (l & (l - 1)) != 0; ++l) sums[lane * kStride + l] = run;
            }
            U = run;
        }
    };

    // Up to kWalkSteps terms of the pmf of a binomial of n trials, lane by lane: a lane that has its count drops out (the
    // execution mask costs scalar instructions, selections would cost vector ones) and the wave leaves with its last lane.
    // The terms' reciprocals come from LDS, eight at a time (all the walks of a wave begin at 1).  The trials left are
    // a whole float below 2^24: exact.  With none left the next term is zero, which ends the walk one too late: the
    // caller takes fewer than none for none.  True if the walk goes on.  A term takes seven vector instructions; with
    // its reciprocal computed, successes counted and trials tested it took twelve, twice the cycles.  (Constants for the
    // first eight terms and a table in memory for the others, two copies of the loop, made the kernel 15 % slower.)
    auto walk = [&](float& pm, float& cdf, float& left, float r, float u, int from) {
        float inv[kWalkSteps];
        {
            const int at = from < kRecips ? from : 0;              // a multiple of kWalkSteps
            const float4 v0 = *reinterpret_cast<const float4*>(recips + at), v1 = *reinterpret_cast<const float4*>(recips + at + 4);
            inv[0] = v0.x; inv[1] = v0.y; inv[2] = v0.z; inv[3] = v0.w;
            inv[4] = v1.x; inv[5] = v1.y; inv[6] = v1.z; inv[7] = v1.w;
        }
        if (from >= kRecips) {                                     // rare: a piece has an expectation of 32 at most
#pragma unroll
            for (int i = 0; i < kWalkSteps; ++i) inv[i] = inv_int((float)(from + i + 1));
        }
        bool more = u > cdf;
#pragma unroll
        for (int i = 0; i < kWalkSteps; ++i) {
            if (!more) break;
            SAME_COUNT(a, 4, 1);                                   // pmf terms
            pm = pm * r;
            pm = pm * left;
            pm = pm * inv[i];
            left = left - 1.0f;
            const float next_cdf = cdf + pm;
            more = next_cdf != cdf && u > next_cdf;
            cdf = next_cdf;
        }
        return more && left > 0.0f;
    };

    // Binomials cut into pieces.  The pieces are independent (own uniform each): those of all the
    // lanes in state 3 are numbered consecutively and dealt out over the 64 lanes; every owner
    // receives the total of its pieces through an LDS counter.  Returns the owner's successes.
    auto pool = [&](uint64_t pend) -> uint32_t {
        const uint32_t np = (st == 3) ? (bR + L - 1u) / L : 0u;
        uint32_t total = 0;
        for (uint64_t p = pend; p != 0; p &= p - 1) total += __shfl(np, __ffsll((unsigned long long)p) - 1);
        if (lane == 0) { SAME_COUNT(a, 6, 1); SAME_COUNT(a, 7, total); }
        for (uint32_t base = 0; base < total; base += kWave) {
            const uint32_t p = base + (uint32_t)lane;
            int owner = lane;
            uint32_t first = 0, off = 0;
            for (uint64_t q = pend; q != 0; q &= q - 1) {        // the last owner whose first piece is <= p
                const int src = __ffsll((unsigned long long)q) - 1;
                if (p >= off) { owner = src; first = off; }
                off += __shfl(np, src);
            }
            const uint32_t oR = __shfl(bR, owner), oL = __shfl(L, owner), onp = __shfl(np, owner);
            const float olq = __shfl(lq, owner), orr = __shfl(r, owner), ou = __shfl(u, owner);
            const uint32_t ostep = __shfl(bstep, owner);
            StreamKey okey = key;
            okey.tau_lo = __shfl(key.tau_lo, owner);
            okey.tau_hi = __shfl(key.tau_hi, owner);
            if (p < total) {
                const uint32_t jp = p - first;
                const uint32_t nj = (jp == onp - 1u) ? oR - jp * oL : oL;
                float pmj = expneg((float)nj * olq);               // no success among the piece's trials
                float uj = ou;
                if (jp > 0) {
                    uint32_t xb[4];
                    piece_block(okey, ostep, (jp - 1u) >> 2, xb);
                    const uint32_t sel = (jp - 1u) & 3u;
                    uj = uniform_from_word(sel == 0u ? xb[0] : sel == 1u ? xb[1] : sel == 2u ? xb[2] : xb[3]);
                }
                float cdfj = pmj, leftj = (float)nj;
                for (int from = 0; walk(pmj, cdfj, leftj, orr, uj, from); from += kWalkSteps) { }
                const uint32_t xj = nj - (uint32_t)__builtin_fmaxf(leftj, 0.0f);
                if (xj > 0) add_lds(acc + owner * kStride, xj);
            }
        }
        __syncthreads();
        uint32_t part = 0;
        if (st == 3) { part = acc[lane * kStride]; acc[lane * kStride] = 0u; }
        __syncthreads();
        return part;
    };

    // One trip of the machine for the whole wave.
    auto trip = [&]() {
        if (lane == 0) SAME_COUNT(a, 2, 1);
#ifdef SAME_STATS
        {   // lanes by what they do in this trip: step, walk on, wait for a shared pass, idle
            const uint64_t b_step = __ballot(st == 0 && R > 0), b_walk = __ballot(st == 1), b_wait = __ballot(st == 3);
            if (lane == 0) {
                SAME_COUNT(a, 8, __popcll((unsigned long long)b_step)); SAME_COUNT(a, 9, __popcll((unsigned long long)b_walk));
                SAME_COUNT(a, 10, __popcll((unsigned long long)b_wait));
                SAME_COUNT(a, 11, 64 - __popcll((unsigned long long)(b_step | b_walk | b_wait)));
            }
        }
#endif
        int ek = 0;             // the count this trip settles for this lane: en copies to topic ek
        uint32_t en = 0;
        if (st == 0 && R > 0) {
            SAME_COUNT(a, 1, 1);                                   // steps
            if (!(U > 0.0f)) {                                     // no weight left: a degenerate input
                ek = top > 0 ? top - 1 : 0; en = R;
                R = 0;
            } else {
                uint32_t xa, xb;
                if ((step & 1u) == 0u) {
                    uint32_t x[4];
                    primary_block(key, pre, step >> 1, x);
                    xa = x[0]; xb = x[1]; xs2 = x[2]; xs3 = x[3];
                } else {
                    xa = xs2; xb = xs3;
                }
                const float y = top_position(U, R, uniform_from_word(xa));
                int k;                                             // the step's topic: the first with P_k >= y
                float prev = 0.0f;                                 // P_{k-1}
                if (UNIFORM) {                                     // weights of one: P_k = k + 1, exactly
                    const float c = __builtin_ceilf(y);
                    prev = c - 1.0f;
                    k = (int)prev;
                } else {
                    // the first block whose cumulative weight reaches y (mu >= U >= y; entries past the last block repeat
                    // mu), and prev = the cumulative weight below that block
                    int l = 0;
#pragma unroll
                    for (int h = kMaxBlocks / 2; h > 0; h >>= 1) {
                        if (KC == 0 && h >= nblk) continue;
                        const float v = my_sums[l + h];            // (an address kept in place of l, prev read at the end: K = 1024
                        const bool below = !(v >= y);              // from a flat posterior at m = 100 6.79 in place of 6.17 ms,
                        prev = below ? v : prev;                   // K = 350 with its row of theta 3.36 and 3.19)
                        l = below ? l + h : l;
                    }
                    if (KC == 0) l = min(l, nblk - 1);             // (only negative weights could lead past it)
                    // inside the block: rebuild P_k from the block's weights.  Its last P_k is the block's cumulative
                    // weight, the same sum in the same order, so the search ends inside the block.
                    const int k0 = l * T;
                    const float* __restrict__ th = kRowAddr ? th_row : a.theta + (size_t)d * K;
                    const float* __restrict__ ph = kRowAddr ? ph_row : a.phi + (size_t)w * K;
                    const float base = prev;
                    float rs = 0.0f;
                    if (TB > 0) {
                        auto reload = [&](auto whole) {
                            constexpr bool WHOLE = decltype(whole)::value;
                            constexpr int N = TB > 0 ? 4 * TB : 4;
                            int at = 0;
                            bool found = false;
                            float before = base;                   // P of the topic before the batch
                            for (int b = 0; b < nb; ++b) {
                                const int kb = k0 + N * b;
                                float4 pv[N / 4], tv[N / 4];
#pragma unroll
                                for (int c = 0; c < N / 4; ++c) pv[c] = load_quad<VEC, WHOLE>(ph, kb + 4 * c, K);
                                if (THETA && myrow >= 0) {
                                    const lds_float* tr = (const lds_float*)th_row_lds;
#pragma unroll
                                    for (int c = 0; c < N / 4; ++c) tv[c] = lds_quad<VEC, WHOLE>(tr, kb + 4 * c, K);
                                } else {
#pragma unroll
                                    for (int c = 0; c < N / 4; ++c) tv[c] = load_quad<VEC, WHOLE>(th, kb + 4 * c, K);
                                }
                                float P[N];
#pragma unroll
                                for (int c = 0; c < N / 4; ++c) {
                                    float x[4] = {tv[c].x * pv[c].x, tv[c].y * pv[c].y, tv[c].z * pv[c].z, tv[c].w * pv[c].w};
                                    shift_quad<VEC>(x, kb + 4 * c, K);
                                    rs = rs + x[0]; P[4 * c + 0] = base + rs;
                                    rs = rs + x[1]; P[4 * c + 1] = base + rs;
                                    rs = rs + x[2]; P[4 * c + 2] = base + rs;
                                    rs = rs + x[3]; P[4 * c + 3] = base + rs;
                                }
                                if (ONE) {
                                    at = first_reaching<N>(P, y, prev);
                                } else {
                                    const float last = P[N - 1];
                                    float pb = before;
                                    const int ib = N * b + first_reaching<N>(P, y, pb);
                                    const bool here = !found && (b == nb - 1 || last >= y);
                                    at = here ? ib : at;
                                    prev = here ? pb : prev;
                                    found = found || here;
                                    before = last;
                                }
                            }
                            k = k0 + at;
                        };
                        if (KC > 0 || (VEC && blocks_fill_row(K))) reload(std::true_type{}); else reload(std::false_type{});
                    } else {
                        int at = 0;
                        auto visit = [&](float wk) {
                            rs = rs + wk;
                            const float P = base + rs;
                            const bool below = !(P >= y);
                            at += below ? 1 : 0;
                            prev = below ? P : prev;
                        };
                        for (int j = 0; j < T; ++j) {
                            const int kj = k0 + j;
                            if (kj < K) visit(th[kj] * ph[kj]);
                        }
                        k = k0 + at;
                    }
                }
                k = max(min(k, top - 1), 0);
                SAME_COUNT(a, 3, 1);                               // block reloads
                // the step's topic, its top copy, and the binomial of the copies that share the topic
                const uint32_t Rm = R - 1u;
                const float width = y - prev;
                const float q = width / y;
                kk = k;
                bstep = step;
                U = prev; top = k; step += 1u;
                if (Rm == 0u || !(q > 0.0f)) {
                    ek = k; en = 1u;
                    R = Rm;
                } else if (q >= 1.0f) {
                    ek = k; en = R;
                    R = 0;
                } else {
                    flip = q > 0.5f;
                    const float qq = flip ? 1.0f - q : q;
                    const float s1 = 1.0f - qq;
                    r = quot_1(qq, s1);
                    lq = log1m(qq);
                    bR = Rm;
                    R = Rm;                                        // the binomial's share comes off when it is known
                    u = uniform_from_word(xb);
                    if (((float)Rm * qq) <= kPieceMean) {          // one piece of Rm trials
                        const float pm0 = expneg((float)Rm * lq);
                        walked = 0; left = (float)Rm; pm = pm0; cdf = pm0;
                        st = 1;
                    } else {                                       // pieces of L trials: shared by the wave
                        L = (uint32_t)(kPieceMean / qq);
                        st = 3;
                    }
                }
            }
        }
        {
            const uint64_t pend = __ballot(st == 3);
            const bool share = pend != 0 && (__popcll((unsigned long long)pend) >= kPoolMin || waited >= kPoolTrips ||
                                             !__any(st == 1 || (st == 0 && R > 0)));
            waited = (pend != 0 && !share) ? waited + 1 : 0;
            if (share) {
                const uint32_t part = pool(pend);
                if (st == 3) {
                    const uint32_t nk = flip ? bR - part : part;
                    ek = kk; en = 1u + nk;
                    R -= nk;
                    st = 0;
                    SAME_COUNT(a, 5, 1);
                }
            }
        }
        if (__any(st == 1)) {
            if (lane == 0) SAME_COUNT(a, 12, 1);                       // trips with a walk
            if (st == 1) {
                if (walk(pm, cdf, left, r, u, walked)) {
                    walked += kWalkSteps;
                } else {                                           // the binomial is known
                    const uint32_t rest = (uint32_t)__builtin_fmaxf(left, 0.0f);
                    const uint32_t nk = flip ? rest : bR - rest;
                    ek = kk; en = 1u + nk;
                    R -= nk;
                    st = 0;
                    SAME_COUNT(a, 5, 1);
                }
            }
        }
        if (!DEBUG) supply.give(a, lane, sc, en > 0u && sc.full(), staged);
#ifdef SAME_STATS
        if (en > 0u && sc.full()) {                                // a count that goes straight to the word's row
            const uint32_t g = R_task_g;
            SAME_COUNT(a, 16 + min(5, 31 - __clz((int)max(g, 1u))), 1);
            SAME_COUNT(a, 22 + (w < 16 ? 0 : w < 256 ? 1 : w < 4096 ? 2 : 3), 1);
        }
#endif
        if (en > 0u) {
            if (!DEBUG && myrow >= 0) add_lds(rows + myrow * K + ek, en);
            else add_global(a.ndk + (size_t)sc.drow * K + ek, en);
            sc.emit_word(a, ek, en, w, staged);
        }
    };

    for (;;) {
        const uint64_t idle_mask = __ballot(st == 0 && R == 0);
        const int n_idle = (int)__popcll((unsigned long long)idle_mask);
        if (!drained && (n_idle >= kRefillMin || (n_idle >= kRefillLate && trips >= kRefillLateTrips) || n_idle == kWave)) {
            if (next >= end && heavy) {                            // on to the workgroup's share of round 0
                heavy = false;
                const int64_t from = (int64_t)blockIdx.x * a.first;
                next = (int32_t)(from < a.n ? from : a.n);
                end = (int32_t)(from + a.first < a.n ? from + a.first : a.n);
            }
            if (next >= end) {                                     // the next share (all lanes obtain the same values)
                const int64_t after = (int64_t)gridDim.x * a.first;   // where round 1 begins
                int64_t from = after;
                int32_t size = 0;
                if (after < a.n) {
                    const uint32_t group = ticket_group(blockIdx.x);
                    uint32_t t = 0;                                // this group's ticket
                    if (lane == 0) t = atomicAdd(a.counter + kCounterStride * group, 1u);
                    t = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
                    const Share s = share_of_ticket(t, group, gridDim.x, a.first, a.n);
                    from = s.from; size = s.size;
                }
                drained = from >= a.n;
                next = drained ? 0 : (int32_t)from;
                end = drained ? 0 : (int32_t)(from + size < a.n ? from + size : a.n);
            }
            if (next < end) {
                if (lane == 0) SAME_COUNT(a, 13, 1);               // refills
                refill(idle_mask);
                trips = 0;
                continue;
            }
        }
        if (idle_mask == ~0ull) break;                             // nothing in flight and nothing left to take
        trip();
        trips += 1;
    }
    if (open) sc.close(true, staged);
    if (n_rows > 0 && tag0 >= 0) flush_row(0, tag0);
    if (n_rows > 1 && tag1 >= 0) flush_row(1, tag1);
}

// Registers left for what runs beside a sweep.  Sixteen waves a compute unit are four per SIMD; at 128 registers (what the
// compiler takes if it may) they hold the whole file, and the staging of the next minibatch, whose first upload is a copy kernel where
// the column pointers are short, stands still until the draw ends.  Held to 112 up to 128 topics (where LDS has room too, the matrix
// build's first pass gets in with 64 left) and to 120 up to 384; not the forms of three loads with rows that are not aligned, which
// would keep ten registers in scratch (K = 350 at m = 100 12 % slower).  us per step of a stream, free / held (before the table of
// reciprocals, which took them over the line): documents of 354 tokens from a flat posterior, m = 30, 280e6 / K tokens: K = 50
// 1915 / 1736 (1756), 128 1168 / 1124 (1152), 200 1107 / 910 (952), 250 1013 / 862 (867), 300 946 / 820 (803).  Sweeps by themselves
// are within 1 %, at K = 300 (three registers in scratch) 3 % slower.
// The attribute counts half of the unified file: 56 are 112 registers.
template __attribute__((amdgpu_num_vgpr(56))) __global__ void draw_kernel<false, true, false, 1, true, 0, false, false>(DrawArgs);
template __attribute__((amdgpu_num_vgpr(56))) __global__ void draw_kernel<false, false, false, 1, true, 0, false, false>(DrawArgs);
template __attribute__((amdgpu_num_vgpr(60))) __global__ void draw_kernel<false, true, false, 2, true, 0, false, false>(DrawArgs);
template __attribute__((amdgpu_num_vgpr(60))) __global__ void draw_kernel<false, false, false, 2, true, 0, false, false>(DrawArgs);
template __attribute__((amdgpu_num_vgpr(60))) __global__ void draw_kernel<false, true, false, 3, true, 0, false, false>(DrawArgs);
template __attribute__((amdgpu_num_vgpr(60))) __global__ void draw_kernel<false, true, false, 3, true, 0, false, true>(DrawArgs);

inline size_t draw_lds_bytes(int K, bool uniform, bool theta)
{
    return 4u * ((size_t)kRecips + (size_t)kWave * (size_t)(uniform ? 1 : sum_stride(K)) + (size_t)(doc_rows(K) + (theta ? 1 : 0)) * (size_t)K);
}

}  // namespace same
