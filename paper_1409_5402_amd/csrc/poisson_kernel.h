// Draw-and-scatter kernel of the SAME LDA sweep in the Poisson form (Section 4, second part; the
// sampling line of Algorithm 3 as printed) for gfx950: topic k of a task with Nf = mf * g copies gets
// an independent Poisson(Nf * w_k / mu) count, mu = the running sum of all weights.
//
// Mapping: one wave per workgroup, one lane per draw task.  A lane walks the K topics of its task twice.
//   pass 1  accumulates the running sums P_k = w_0 + ... + w_k left to right
//           (w_k = theta[d][k] * phi[w][k]) up to mu;
//   pass 2  revisits the 16-topic blocks from the last to the first, generates the topics' uniforms
//           (one Philox block per 4 topics) and tests every topic: a topic whose uniform already
//           proves that its count is 0 is dropped; the others are queued in LDS.
// The queue is drained by a per-lane state machine: every trip of the drain loop lets each lane either
// fetch its next queued topic and start its draw, or advance its pmf walk by a few steps, so lanes
// with long walks do not hold up lanes with many short ones.  A rate above 32 is cut into equal
// pieces (independent, one uniform each) that are handed to the whole wave, one piece per lane.
//
// The drop test is conservative and never changes a result.  A Poisson variable of rate
// lambda <= Nf * q (q = w/mu) drawn by inversion is 0 iff u <= exp(-lambda) as the sampler evaluates
// it; that value is >= 1 - Nf*(q + 2^-22).  The test checks q <= 0.499 and
// u + Nf*(q*(1+1e-4) + 1e-6) <= 1 - 1e-4, evaluated without a division (see ZeroTest), which
// implies the former.  A topic of zero weight passes it.
#pragma once
#include "draw_kernel.h"

namespace same {

constexpr int kBlk = 16;                // topics per block of the Poisson kernel's second pass
constexpr int kQCap = 16;               // queued topics per lane between drains (drain when > kQCap - 4; 8, 12 and 16
                                        // measured 3.12, 3.02 and 3.00 ms for 6 million tasks at K = 256)

// How a block's rows are read.  kWhole: K is a multiple of 16, aligned loads.  kQuads: any K from 4 on, loads of any
// alignment that stay inside the row (load_quad); the last block's products are shifted into place.  kFew: element by
// element.  (Every K that is no multiple of 16 was read element by element: 9,000 news-shaped documents, K = 100 1.47 and now
// 0.40 ms per draw, K = 200 3.12 and 0.82, K = 1000 17.7 and 4.1.)
constexpr int kFew = 0, kQuads = 1, kWhole = 2;

// The sixteen theta and phi values of one block, loaded ahead of their use (not kFew).
struct PhiBlock { float4 v[kBlk / 4]; float4 t[kBlk / 4]; };

template <int READ>
__device__ __forceinline__ PhiBlock load_phi(const float* __restrict__ th, const float* __restrict__ ph, int b, int K)
{
    PhiBlock r;
    if (READ != kFew) {
#pragma unroll
        for (int v = 0; v < kBlk / 4; ++v) {
            r.v[v] = load_quad<READ == kWhole, true>(ph, b * kBlk + 4 * v, K);
            r.t[v] = load_quad<READ == kWhole, true>(th, b * kBlk + 4 * v, K);
        }
    }
    return r;
}

// The 16 weights of block b (zero beyond K).
template <int READ>
__device__ __forceinline__ void block_weights(const float* __restrict__ th, const float* __restrict__ ph,
                                              const PhiBlock& pre, int b, int K, float (&wv)[kBlk])
{
    const int k0 = b * kBlk;
    if (READ != kFew) {
#pragma unroll
        for (int v = 0; v < kBlk / 4; ++v) {
            const float4 t = pre.t[v];
            const float4 c = pre.v[v];
            wv[4 * v + 0] = t.x * c.x;
            wv[4 * v + 1] = t.y * c.y;
            wv[4 * v + 2] = t.z * c.z;
            wv[4 * v + 3] = t.w * c.w;
        }
        if (READ == kQuads && k0 + kBlk > K) {                     // the last block (the same for the whole wave)
#pragma unroll
            for (int v = 0; v < kBlk / 4; ++v) {
                float x[4] = {wv[4 * v], wv[4 * v + 1], wv[4 * v + 2], wv[4 * v + 3]};
                shift_quad<false>(x, k0 + 4 * v, K);
                wv[4 * v] = x[0]; wv[4 * v + 1] = x[1]; wv[4 * v + 2] = x[2]; wv[4 * v + 3] = x[3];
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < kBlk; ++j) wv[j] = (k0 + j < K) ? th[k0 + j] * ph[k0 + j] : 0.0f;
    }
}

// The drop test without a division: for q = w/M it checks q <= 0.499 and
// u + Rf*(q*(1+1e-4) + 1e-6) <= 1 - 1e-4, both multiplied through by M > 0
// (the margins cover the few roundings of this evaluation), in one comparison A*w <= d*M:
//   d = (1-1e-4) - Rf*1e-6 - u', with u' = x * 2^-32 rounded, never below u - 2^-24 (x is the raw
//       random word of the topic, u = (2*(x>>9)+1)/2^24; the 2^-24 is taken off in Bp);
//   A = max(Rf*(1+1e-4), 2.0041): since d < 1, A*w <= d*M also gives w/M < 1/2.0041 < 0.499.
// ZeroTest holds the two terms that depend only on the bound Rf.
struct ZeroTest {
    float A, Bp;
    __device__ __forceinline__ explicit ZeroTest(float Rf)
        : A(fmaxf(Rf * 1.0001f, 2.0041f)), Bp((0.9999f - Rf * 1.0e-6f) - 5.9604644775390625e-8f) {}
    // true when the count of a topic of weight wk is certainly 0 for every number of copies <= Rf
    __device__ __forceinline__ bool surely_zero(float wk, float Mk, uint32_t x) const
    {
        const float d = __builtin_fmaf((float)x, -2.3283064365386963e-10f, Bp);
        return A * wk <= d * Mk;
    }
};

// KC: the number of topics where it is known at compile time.  WAVES: the least number per SIMD that the registers are held to
// (1: the compiler's own choice).  The kernel for any multiple of 16 needs 134 registers, three waves; held to the 128 of four
// waves it spills two.  Four waves are the faster form up to 128 topics (K = 64: 0.84 against 0.94 ms for 9000 news-shaped
// documents at 100 copies, 0.90 against 0.97 at 20 from a flat posterior) and up to 256 where many topics receive copies
// (K = 240: 2.51 against 2.60 ms at 100 copies, but 0.94 against 0.91 at 1.5).  Beyond, three: rows of more waves than that push one
// another out of the cache (K = 512 from a flat posterior 4.34 against 4.07 ms, K = 1024 7.21 against 6.47).  K = 256 has 128
// registers by itself (holding it to four waves only changes the schedule: 0.7 % slower), the kernel for any K (kQuads) 125.
template <int READ, bool DEBUG, int KC = 0, int WAVES = 1>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(WAVES))) void poisson_draw_kernel(DrawArgs a)
{
    extern __shared__ __align__(16) uint32_t lds[];
    const int lane = threadIdx.x;
    const int K = KC > 0 ? KC : a.K;
    const int nblk = (K + kBlk - 1) / kBlk;
    constexpr int qw = 2;                                          // words per queue entry: weight, random word with the topic's low bits
    constexpr bool kHigh = KC == 0 || KC > 512;                    // topics may need more than nine bits
    uint32_t* que = lds;                                           // [kQCap][qw][64], a ring per lane
    uint32_t* acc = lds + (size_t)(qw * kQCap) * kWave;            // [64] piece totals by owner lane
    static_assert(kQCap <= 16, "two bits per ring slot in one register");
    uint32_t khi = 0;       // bits 9 and 10 of the topic queued in each ring slot (the entry holds the low nine)

    // lanes past the end take the last task with zero copies: all loads stay valid, nothing is emitted
    const int64_t slot = (int64_t)blockIdx.x * kWave + lane;
    const bool live = slot < a.n;
    const int64_t row = live ? slot : a.n - 1;
    // order holds non-negative 32-bit ids: the high byte of tau is then a constant zero for the whole launch
    const int64_t tau = DEBUG ? a.ids[row] : (int64_t)(uint32_t)a.order[row];
    const int32_t d = a.t_doc[tau];
    const int32_t w = a.t_word[tau];
    const float Nf = live ? a.mf * (float)a.t_g[tau] : 0.0f;
    const float* __restrict__ th = a.theta + (size_t)d * K;
    const float* __restrict__ ph = a.phi + (size_t)w * K;
    Scatter sc = make_scatter<DEBUG>(a, row, tau, d);
    if (!live) sc.dst = nullptr;                                   // (the last task's slot is its own lane's)
    ChunkSupply supply(a);
    Staged staged;
    acc[lane] = 0u;
    // 1/x for x = 1 to 64, the factors of the walks below (three instructions each where computed, a third of a term:
    // poisson_sweep 3.98 and, from the table, 3.78 ms; K = 64 at 100 copies 0.71 and 0.58)
    float* recips = reinterpret_cast<float*>(acc + kWave);
    recips[lane] = inv_int((float)(lane + 1));
    __syncthreads();

    StreamKey key;
    key.seed_lo = a.seed_lo; key.seed_hi = a.seed_hi;
    key.tau_lo = (uint32_t)tau; key.tau_hi = (uint32_t)((uint64_t)tau >> 32) & 0xFFu;
    key.pass = a.pass;
    const PrimaryPre pre = primary_pre(key);

    // ---- pass 1: the normaliser mu (left-to-right running sum)
    float mu = 0.0f;
    {
        float P = 0.0f;
        PhiBlock cur = load_phi<READ>(th, ph, 0, K);
        for (int b = 0; b < nblk; ++b) {
            PhiBlock nxt = cur;
            if (b + 1 < nblk) nxt = load_phi<READ>(th, ph, b + 1, K);
            float wv[kBlk];
            block_weights<READ>(th, ph, cur, b, K, wv);
#pragma unroll
            for (int j = 0; j < kBlk; ++j) P = P + wv[j];
            cur = nxt;
        }
        mu = P;
    }

    // ---- the draws of the queued topics, a per-lane state machine that lives across the whole scan
    int qh = 0, cnt = 0;    // ring queue: position of the oldest entry, entries queued
    int st = 0;             // 0: between draws, 1: walking a single piece,
                            // 3: holds a variable of several pieces, waiting for the wave to share it
    uint32_t np = 0;
    float r = 0.f, pm = 0.f, cdf = 0.f, u = 0.f;
    uint32_t walked = 0;    // terms added so far
    int waited = 0;         // trips since a variable of several pieces has been waiting
    int kk = 0;
    uint32_t busy = 0;      // trips in which this lane had work: its cost for the next ordering

    // Up to kWalkSteps terms of the pmf, lane by lane under the execution mask, as in the multinomial form's walk; x terms have
    // been added before, a multiple of kWalkSteps.  True if the walk goes on.
    auto walk = [&](float& pm, float& cdf, uint32_t& x, float r, float u) {
        float inv[kWalkSteps];
        {
            const uint32_t at = x < (uint32_t)kWave ? x : 0u;
            const float4 v0 = *reinterpret_cast<const float4*>(recips + at), v1 = *reinterpret_cast<const float4*>(recips + at + 4);
            inv[0] = v0.x; inv[1] = v0.y; inv[2] = v0.z; inv[3] = v0.w;
            inv[4] = v1.x; inv[5] = v1.y; inv[6] = v1.z; inv[7] = v1.w;
        }
        if (x >= (uint32_t)kWave) {                                // rare: a piece's rate is 32 at most
#pragma unroll
            for (int i = 0; i < kWalkSteps; ++i) inv[i] = inv_int((float)(x + i + 1));
        }
        bool more = u > cdf;
#pragma unroll
        for (int i = 0; i < kWalkSteps; ++i) {
            if (!more) break;
            SAME_COUNT(a, 4, 1);                                   // walk steps
            x += 1;
            pm = pm * r;
            pm = pm * inv[i];
            const float next = cdf + pm;
            more = next != cdf && u > next;
            cdf = next;
        }
        return more;
    };

    // Variables cut into pieces.  The pieces are independent (own uniform each): those of all the
    // lanes in state 3 are numbered consecutively and dealt out over the 64 lanes; every owner
    // receives the total of its pieces through an LDS counter.
    auto pool = [&](uint64_t pend) -> uint32_t {
        const uint32_t mine = (st == 3) ? np : 0u;
        uint32_t total = 0;
        for (uint64_t p = pend; p != 0; p &= p - 1) total += __shfl(mine, __ffsll((unsigned long long)p) - 1);
        if (lane == 0) { SAME_COUNT(a, 6, 1); SAME_COUNT(a, 7, total); }
        for (uint32_t base = 0; base < total; base += kWave) {
            const uint32_t p = base + (uint32_t)lane;
            int owner = lane;
            uint32_t first = 0, off = 0;
            for (uint64_t q = pend; q != 0; q &= q - 1) {        // the last owner whose first piece is <= p
                const int src = __ffsll((unsigned long long)q) - 1;
                if (p >= off) { owner = src; first = off; }
                off += __shfl(mine, src);
            }
            const float opm = __shfl(pm, owner), orr = __shfl(r, owner), ou = __shfl(u, owner);
            const uint32_t ok = (uint32_t)__shfl(kk, owner);
            StreamKey okey = key;
            okey.tau_lo = __shfl(key.tau_lo, owner);
            okey.tau_hi = __shfl(key.tau_hi, owner);
            if (p < total) {
                const uint32_t jp = p - first;
                float pmj = opm;                                   // the owner's exp(-rate)
                float uj = ou;
                if (jp > 0) {
                    uint32_t xb[4];
                    piece_block(okey, ok, (jp - 1u) >> 2, xb);
                    const uint32_t sel = (jp - 1u) & 3u;
                    uj = uniform_from_word(sel == 0u ? xb[0] : sel == 1u ? xb[1] : sel == 2u ? xb[2] : xb[3]);
                }
                uint32_t xj = 0;
                float cdfj = pmj;
                while (walk(pmj, cdfj, xj, orr, uj)) { }
                if (xj > 0) atomicAdd(acc + owner, xj);
            }
        }
        __syncthreads();
        uint32_t nk = 0;
        if (st == 3) {
            nk = acc[lane];
            acc[lane] = 0u;
            st = 0;
        }
        __syncthreads();
        return nk;
    };

    // One trip of the machine for the whole wave: lanes in state 0 take their next queued topic,
    // shared variables are worked off when enough of them wait or nothing else is in flight,
    // walking lanes advance by kWalkSteps pmf steps.
    auto trip = [&]() {
        if (lane == 0) SAME_COUNT(a, 2, 1);
        busy += (st != 0 || cnt > 0) ? 1u : 0u;
        uint32_t en = 0;        // the count this trip settles for this lane: en copies to topic kk_done
        int kk_done = 0;
        if (st == 0 && cnt > 0) {
            const float wq = __uint_as_float(que[(qh * qw + 0) * kWave + lane]);
            const uint32_t xk = que[(qh * qw + 1) * kWave + lane];
            kk = (int)((xk & 511u) | (kHigh ? ((khi >> (2 * qh)) & 3u) << 9 : 0u));
            u = uniform_from_word(xk);
            qh = (qh + 1 == kQCap) ? 0 : qh + 1;
            --cnt;
            const float scaled = Nf * wq;
            const float lam = scaled / mu;
            if (lam > 0.0f) {
                if (lam <= kPieceMean) {                           // one piece
                    r = lam;
                    const float pm0 = expneg(lam);
                    walked = 0; pm = pm0; cdf = pm0;
                    st = 1;
                } else {                                           // equal pieces: shared by the wave
                    np = (uint32_t)(lam / kPieceMean) + 1u;
                    r = lam / (float)np;
                    pm = expneg(r);
                    st = 3;
                }
            }
        }
        {
            const uint64_t pend = __ballot(st == 3);
            const bool share = pend != 0 && (__popcll((unsigned long long)pend) >= kPoolMin || waited >= kPoolTrips || !__any(st == 1));
            waited = (pend != 0 && !share) ? waited + 1 : 0;
            if (share) { en = pool(pend); kk_done = kk; }
        }
        if (__any(st == 1)) {
            if (st == 1 && !walk(pm, cdf, walked, r, u)) {         // the piece is finished
                en = walked; kk_done = kk;
                st = 0;
            }
        }
        if (!DEBUG) supply.give(a, lane, sc, en > 0u && sc.full(), staged);
        if (en > 0u) {
            SAME_COUNT(a, 5, 1);
            atomicAdd(a.ndk + (size_t)sc.drow * a.K + kk_done, en);
            sc.emit_word(a, kk_done, en, w, staged);
        }
    };

    // ---- pass 2: blocks from last to first
    {
        PhiBlock cur = load_phi<READ>(th, ph, nblk - 1, K);
        const ZeroTest zt(Nf);
        for (int b = nblk - 1; b >= 0; --b) {
            if (!__any(Nf > 0.0f)) break;
            PhiBlock nxt = cur;
            if (b > 0) nxt = load_phi<READ>(th, ph, b - 1, K);
            float wv[kBlk];
            block_weights<READ>(th, ph, cur, b, K, wv);
            cur = nxt;
#pragma unroll
            for (int g = kBlk / 4 - 1; g >= 0; --g) {
                uint32_t x[4];
                primary_block(key, pre, (uint32_t)(b * (kBlk / 4) + g), x);
#pragma unroll
                for (int j = 3; j >= 0; --j) {
                    const int k = b * kBlk + g * 4 + j;
                    const float wk = wv[g * 4 + j];
                    // a zero weight passes the test
                    const bool cand = (READ == kWhole || k < K) && Nf > 0.0f && !zt.surely_zero(wk, mu, x[j]);
                    if (cand) {
                        int e = qh + cnt;
                        e = e >= kQCap ? e - kQCap : e;
                        que[(e * qw + 0) * kWave + lane] = __float_as_uint(wk);
                        que[(e * qw + 1) * kWave + lane] = (x[j] & ~511u) | ((uint32_t)k & 511u);   // the uniform uses the top 23 bits
                        if (kHigh) khi = (khi & ~(3u << (2 * e))) | (((uint32_t)k >> 9) << (2 * e));
                        cnt += 1;
                        SAME_COUNT(a, 1, 1);                       // queued topics
                    }
                }
                // trips are run only while some lane could not take the next four topics
                while (__any(cnt > kQCap - 4)) trip();
            }
        }
    }
    while (__any(st != 0 || cnt > 0)) trip();
    sc.close(live, staged);
    // The ordering key for the next pass: a running mean (weight 1/4 on this pass) predicts a task's next
    // cost a little better than this pass's cost alone.
    if (!DEBUG && live && a.cost) a.cost[tau] = (3u * a.cost[tau] + busy + 2u) >> 2;
}

inline bool poisson_four_waves(int K, float mf) { return K <= 128 || (K <= 256 && mf >= 10.0f); }
inline size_t poisson_lds_bytes() { return 4u * (size_t)kWave * (size_t)(2 * kQCap + 2); }

}  // namespace same
