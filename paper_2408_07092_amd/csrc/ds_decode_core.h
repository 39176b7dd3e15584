// The decode of one layer in one launch (Algorithm 1 steps 1-5): body of k_refine_attend, for label
// caches that the launch scores itself, and for units of one workgroup behind a scoring launch.
//
// A workgroup owns a chunk of a unit's tokens, or the whole unit.
//   1. Its label rows are streamed; every thread keeps the keys of its up to 32 tokens in registers.
//   2. Threshold bin: from the chunk's histogram in LDS (one workgroup per unit), or the chunk
//      histograms meet in the unit's histograms in memory and every workgroup finds the bin there.
//   3. The keys are split into definite tokens (bin above: selected whatever the exact threshold is),
//      candidates (in the bin, one key in a thousand) and the rest; the lists go to LDS.
//   4. Wavefront 0 settles the exact threshold (T, tie cut) -- among the candidates of all of the unit's
//      workgroups, which meet in memory -- while the others stream the definite rows; it then adds
//      the workgroup's selected candidates to the row list and raises a flag.
//   5. The others take the rest of the list; the wavefronts' partials meet in LDS, the workgroups' in memory.
//
// What bounds it: the two streams (label rows, gathered K/V rows) at memory's rate, 6.1 TB/s each on 32 heads
// of 64K tokens, and between, before and behind them a chain of latencies: 2 us to the first scores, 2.3 for the
// unit's threshold bin, 1.3 for the lists, 1.5 for the partial, 2 for the merge.
// Why this split (us per layer, before -> after, 32 heads of 64K tokens unless said otherwise):
//   - A wavefront issues an instruction every 8 clocks at best, two to a SIMD fill that: 512 threads. With 1024, and
//     every wavefront running the list work, one layer of 4K tokens took 12.6, with 512 9.2.
//   - One wavefront does what needs no more; the others never wait at its barriers (31.1 -> 26.5 with the next two).
//   - Bins of 1/128 octave instead of 1/8 (see ds_bins.h): 70 candidates in a unit where there were 1100, so that every workgroup settles
//     the threshold alone; one that did it for the unit held the others up until 10 us after the last had arrived.
//   - No more row loads in flight than memory needs: a workgroup's hand-over queues behind them. Eight rows per slot 34.6,
//     four 33.1, two 32.0 (with the settling workgroup).
//   - Fewer, larger workgroups: 8 per unit instead of 32 meet at the same lines of memory.
// Keys kept in LDS as well, so that candidates' keys need no search in the registers, change nothing (9.0 and 9.0; 14.9 and
// 14.9); rows held back until the candidates have been sent, so that these do not queue, cost 0.6 us at 64K.
#pragma once

#include "ds_attend_core.h"
#include "ds_bins.h"

namespace ds {

constexpr int kKeys = 32;               // tokens of a thread at most
constexpr int kQRow = kD + 8;           // halves from one query row in LDS to the next (spreads the matrix cores' reads over the banks)
constexpr uint32_t kCandLds = 512;      // candidates of a workgroup that LDS holds; the others go through memory
// More candidates than these are settled by the whole workgroup: see wave_settle.  (One workgroup per unit, several.)
constexpr uint32_t kWaveSettlesOwn = 384, kWaveSettlesUnit = 1024;

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
__device__ __forceinline__ uint32_t read_lane(uint32_t x, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)x, l); }
__device__ __forceinline__ uint32_t bits_below(unsigned long long m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
// LDS written by lanes of this wavefront is about to be read by others of it (the wavefront's LDS
// accesses are performed in order; this keeps the compiler from reordering them).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// (__builtin_expect below: what few calls come to lies behind the others' code, whose instructions are fetched anew by every
//  launch: 500 calls of 128 to 5000 tokens take 1.5 % less time than with everything in place.)

// How a label cache's rows are loaded.  SMODE = r: fp16 rows of r channels (a multiple of 4, up to 32),
// in pieces of PE channels; SMODE = -8 / -16: 4-bit codes of up to 8 / 16 channels, 16 bytes = TPL tokens;
// SMODE = 0: the keys that a scoring launch has left, for labels that the launch cannot score (RR: at most).
template <int SMODE>
struct LabelRows {
    static constexpr bool kQ4 = SMODE < 0, kKeysGiven = SMODE == 0;
    static constexpr int RR = kQ4 ? -SMODE : kKeysGiven ? kD : SMODE;
    static constexpr int PE = RR % 8 ? 4 : 8;
    static constexpr int NV = kQ4 || kKeysGiven ? 1 : RR / PE;   // loads of a step
    static constexpr int TPL = kQ4 ? (RR == 8 ? 4 : 2) : 1;      // tokens of a step
    static constexpr int STEPS = kQ4 ? 2 : RR <= 4 || kKeysGiven ? 8 : RR <= 12 ? 4 : 2;  // steps of a batch
    static constexpr int SB = STEPS * TPL;                       // tokens of a batch (two batches are in flight)
    static constexpr bool kPairs = SMODE == 16;
    using Piece = typename std::conditional<kKeysGiven, uint32_t, typename std::conditional<kQ4, uint4,
                  typename std::conditional<PE == 8, half8, half4>::type>::type>::type;
};

// m = 2 m + (a < b), a uniform: a thread's keys against a bound, a bit each, two instructions a key.
__device__ __forceinline__ void push_less(uint32_t &m, uint32_t a, uint32_t b)
{
    asm("v_cmp_lt_u32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(m) : "s"(a), "v"(b) : "vcc");
}

// A wavefront's view of a list of n candidates: up to 64 kHeld of them stay in registers, a lane's
// i-th at index 64 i + lane; a longer list is read again by every pass.  at(i) gives candidate i.
template <int kHeld, class At>
struct HeldCands {
    uint2 e[kHeld];
    uint32_t n;
    At at;
    bool loaded = false;
    __device__ __forceinline__ HeldCands(uint32_t n_, At at_) : n(n_), at(at_) {}
    template <class F>
    __device__ __forceinline__ void each(F f)
    {
        const uint32_t lane = (uint32_t)lane_id();
        for (uint32_t i0 = 0; i0 < n; i0 += 64u * kHeld) {
            if (!loaded) {
#pragma unroll
                for (int x = 0; x < kHeld; ++x) {
                    if (i0 + (uint32_t)(x * 64) >= n) break;
                    e[x] = at(min(i0 + (uint32_t)(x * 64) + lane, n - 1u));
                }
            }
#pragma unroll
            for (int x = 0; x < kHeld; ++x) {
                if (i0 + (uint32_t)(x * 64) >= n) break;
                f(e[x], i0 + (uint32_t)(x * 64) + lane < n);
            }
        }
        loaded = n <= 64u * kHeld;
    }
};

// A candidate's place in the order key descending, token ascending, as a number, larger = earlier: the key less
// lo_key, the key of a bin's first, and the token inverted in its tb bits.
__device__ __forceinline__ unsigned long long place_of(uint2 e, uint32_t lo_key, int tb)
{
    return (unsigned long long)(e.x - lo_key) << tb | (e.y ^ ((1u << tb) - 1u));
}
// Threshold that the places from `place` on pass.
__device__ __forceinline__ void threshold_at(unsigned long long place, uint32_t lo_key, int tb, uint32_t &T, int &tcut)
{
    const uint32_t mask = (1u << tb) - 1u;
    T = lo_key + (uint32_t)(place >> tb);
    tcut = (int)(((uint32_t)place & mask) ^ mask);
}

// Exact k-th key of a unit among its candidates, whose keys less lo_key are below 2^span and whose tokens
// below 2^tb, by one wavefront: the krem-th in the order key descending, token ascending.  No more than 64 are
// ranked among themselves.  Of more, one lane is a radix bin, six bits of the place at a time, as often as
// it takes to be left with 64, or with none but selected ones.  lh: 64 words of LDS; small: room for 64 candidates.
// False when the counts do not add up (a workspace that was not cleared): the workgroup then takes the long way.
// Up to how many candidates it is tried: what its registers hold for a unit's one workgroup (128 units of 6000 tokens, 600 equal
// keys: 21.9 us with a limit of 384, 26.5 with 1024); for several workgroups, whose lists are in memory and whose row
// wavefronts are still busy, some more (32 units of 64K tokens, 550 candidates: 28.4 us with 1024, 30.8 with 384).
template <class Held>
__device__ __forceinline__ bool wave_settle(Held &c, uint32_t krem, uint32_t lo_key, int span, int tb, uint32_t *lh, uint2 *small,
                                            uint32_t &T, int &tcut)
{
    const uint32_t lane = (uint32_t)lane_id();
    uint32_t m = c.n;
    unsigned long long pre = 0;  // the settled bits of the place
    int sh = span + tb;
    while (__builtin_expect(m > 64u && sh > 0, 0)) {
        const int nb = min(sh, 6);
        sh -= nb;
        lh[lane] = 0u;
        wave_lds_sync();
        c.each([&](uint2 e, bool have) {
            const unsigned long long x = (place_of(e, lo_key, tb) ^ pre) >> sh;
            if (have && x >> nb == 0ull) atomicAdd(&lh[63u - (uint32_t)x], 1u);
        });
        wave_lds_sync();
        const uint32_t cnt = lh[lane];
        const uint32_t incl = (uint32_t)wave_inclusive_scan((int)cnt, (int)lane);
        const unsigned long long own = __ballot(incl - cnt < krem && incl >= krem);
        if (own == 0ull) return false;
        const int l = __builtin_ctzll(own);
        pre |= (unsigned long long)(63u - (uint32_t)l) << sh;
        krem -= read_lane(incl - cnt, l);
        m = read_lane(cnt, l);
        if (m == krem) {
            threshold_at(pre, lo_key, tb, T, tcut);
            return true;
        }
        wave_lds_sync();
    }
    if (__builtin_expect(m > 64u, 0)) return false;
    uint2 mine = make_uint2(0u, 0u);
    if (__builtin_expect(m == c.n, 1)) {
        c.each([&](uint2 e, bool have) {
            if (have) mine = e;
        });
    } else {
        uint32_t got = 0;
        c.each([&](uint2 e, bool have) {
            const bool hit = have && (place_of(e, lo_key, tb) ^ pre) >> sh == 0ull;
            const unsigned long long hm = __ballot(hit);
            if (hm) {
                const uint32_t pos = got + bits_below(hm);
                if (hit && pos < 64u) small[pos] = e;
                got += (uint32_t)__builtin_popcountll(hm);
            }
        });
        if (got != m) return false;
        wave_lds_sync();
        if (lane < m) mine = small[lane];
    }
    // (key and inverted token as one number: sorts before <=> larger)
    const unsigned long long me = (unsigned long long)mine.x << 32 | (0xffffffffu - mine.y);
    uint32_t before = 0;
    for (uint32_t j = 0; j < m; ++j)
        before += ((unsigned long long)read_lane((uint32_t)(me >> 32), (int)j) << 32 | read_lane((uint32_t)me, (int)j)) > me ? 1u : 0u;
    const unsigned long long hit = __ballot(lane < m && before + 1u == krem);
    if (hit == 0ull) return false;
    const int l = __builtin_ctzll(hit);
    T = read_lane(mine.x, l);
    tcut = (int)read_lane(mine.y, l);
    return true;
}

// Threshold bin of a complete histogram of kHistBins counts in LDS: the bin holding the kth key from the top
// and the rank inside it, to res.  A thread owns consecutive bins.  Two barriers.
template <int NW>
__device__ __forceinline__ void find_bin(const uint32_t *hist, uint32_t kth, uint32_t *s_w, uint32_t *res)
{
    constexpr int PER = kHistBins / (64 * NW);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t cnt[PER], sum = 0;
#pragma unroll
    for (int i = 0; i < PER / 4; ++i) {
        const uint4 q = reinterpret_cast<const uint4 *>(hist)[kHistBins / 4 - 1 - tid * (PER / 4) - i];
        cnt[4 * i] = q.w; cnt[4 * i + 1] = q.z; cnt[4 * i + 2] = q.y; cnt[4 * i + 3] = q.x;
        sum += (q.w + q.z) + (q.y + q.x);
    }
    const uint32_t incl = (uint32_t)wave_inclusive_scan((int)sum, lane);
    if (lane == 63) s_w[wave] = incl;
    if (tid == 0) { res[0] = 0u; res[1] = 1u; }  // (in range also when the counts do not reach kth)
    __syncthreads();
    const uint32_t x = lane < wave ? s_w[lane] : 0u;  // (NW <= 16 <= a row of lanes)
    uint32_t y = (uint32_t)wave_inclusive_scan((int)x, lane);
    uint32_t before = read_lane(y, 15) + incl - sum;
    if (before < kth && before + sum >= kth) {
        bool done = false;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (!done && before + cnt[i] >= kth) {
                res[0] = (uint32_t)(kHistBins - 1 - tid * PER - i);
                res[1] = kth - before;
                done = true;
            }
            before += cnt[i];
        }
    }
    __syncthreads();
}

// f of each of n candidates, by the whole workgroup; eight loads of a thread are in flight.
template <int WGT, class At, class F>
__device__ __forceinline__ void wg_each(uint32_t n, At at, F f)
{
    for (uint32_t i0 = threadIdx.x; i0 < n; i0 += 8u * WGT) {
        uint2 v[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) v[x] = at(min(i0 + (uint32_t)(x * WGT), n - 1u));
#pragma unroll
        for (int x = 0; x < 8; ++x)
            if (i0 + (uint32_t)(x * WGT) < n) f(v[x]);
    }
}

// wave_settle's task by the whole workgroup, for any number of candidates, ten bits of the place at a time.  Sets T and
// tcut in every thread.  Equal keys, of which there can be thousands, share a radix bin: a wavefront's candidates that
// fall into the first one's are counted with one add (64 adds to one word of LDS wait for each other).
template <int NW, class At>
__device__ __forceinline__ void wg_settle(uint32_t n, At at, uint32_t krem, uint32_t lo_key, int span, int tb, uint32_t *lh,
                                          uint32_t *s_w, uint32_t *s_res, uint32_t &T, int &tcut)
{
    constexpr int WGT = 64 * NW, PER = 1024 / WGT;
    const uint32_t tid = threadIdx.x;
    unsigned long long pre = 0;
    uint32_t rank = krem;
    for (int sh = span + tb; sh > 0;) {
        const int nb = min(sh, 10);
        sh -= nb;
        for (uint32_t i = tid; i < 1024u; i += WGT) lh[i] = 0u;
        __syncthreads();
        wg_each<WGT>(n, at, [&](uint2 e) {
            const unsigned long long p = (place_of(e, lo_key, tb) ^ pre) >> sh;
            if (p >> nb == 0ull) {
                const uint32_t d = (uint32_t)p, d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
                const unsigned long long same = __ballot(d == d0);
                if (d != d0) atomicAdd(&lh[d], 1u);
                else if (bits_below(same) == 0u) atomicAdd(&lh[d0], (uint32_t)__builtin_popcountll(same));
            }
        });
        __syncthreads();
        hist_select<PER, true, NW>([&](int bin) { return lh[bin]; }, rank, s_w, s_res);
        pre |= (unsigned long long)s_res[0] << sh;
        rank = s_res[1];
        const uint32_t m = lh[s_res[0]];
        __syncthreads();
        if (m == rank) break;  // (none but selected ones are left)
    }
    threshold_at(pre, lo_key, tb, T, tcut);
}

// Rows of single heads and pairs.  The RW row wavefronts' 16-lane slots take the list's rows in turn, HB rows a
// slot and round; NB rounds are in flight.
template <int GT, int RW, bool ST, int HB, int NB>
struct VectorRows {
    static constexpr int HR = RW * 4 * HB;
    half8 k[NB][HB], v[NB][HB];
    RowState<GT> st;
    int h, at;  // the next round to fold in is h + at, in k[at], v[at]

    struct Src {
        const char *Ku, *Vu;      // first row of the chunk
        uint32_t row_bytes;
        const uint16_t *sel;
        const _Float16 (*q)[kQRow];
        int place;                // the slot's place among the row wavefronts' slots
    };
    __device__ __forceinline__ int row(const Src &s, int round, int i) const { return round * HR + i * RW * 4 + s.place; }
    __device__ __forceinline__ void load(const Src &s, half8 &kr, half8 &vr, int p)
    {
        const uint32_t off = (uint32_t)s.sel[p] * s.row_bytes + (uint32_t)(threadIdx.x & 15) * 16u;
        kr = row_load<ST>(reinterpret_cast<const half8 *>(s.Ku + off));
        vr = row_load<ST>(reinterpret_cast<const half8 *>(s.Vu + off));
    }
    // the rows of a round that there are; zeros in the place of the others
    __device__ __forceinline__ void issue(const Src &s, half8 (&kr)[HB], half8 (&vr)[HB], int round, int n)
    {
        if ((round + 1) * HR <= n) {
#pragma unroll
            for (int i = 0; i < HB; ++i) load(s, kr[i], vr[i], row(s, round, i));
        } else {
#pragma unroll
            for (int i = 0; i < HB; ++i) {
                kr[i] = (half8)(_Float16)0;
                vr[i] = (half8)(_Float16)0;
                if (row(s, round, i) < n) load(s, kr[i], vr[i], row(s, round, i));
            }
        }
    }
    __device__ __forceinline__ void fold(const Src &s, half8 (&kr)[HB], half8 (&vr)[HB], int round, int n)
    {
        const bool full = (round + 1) * HR <= n;
        const int part = threadIdx.x & 15;
#pragma unroll
        for (int g = 0; g < GT; ++g) {
            const half8 qv = *reinterpret_cast<const half8 *>(&s.q[g][part * 8]);
            float sc4[HB], mx = kNegInf;
#pragma unroll
            for (int i = 0; i < HB; ++i) {
                sc4[i] = row16_sum(dot8(qv, kr[i])) * kScaleLog2;
                if (!full && row(s, round, i) >= n) sc4[i] = kNegInf;
                mx = fmaxf(mx, sc4[i]);
            }
            const float mn = fmaxf(st.m[g], mx);
            if (mn != kNegInf) {
                const float sc = (st.m[g] == kNegInf) ? 0.0f : __builtin_amdgcn_exp2f(st.m[g] - mn);
                st.m[g] = mn;
                st.l[g] *= sc;
#pragma unroll
                for (int j = 0; j < 8; ++j) st.acc[g][j] *= sc;
#pragma unroll
                for (int i = 0; i < HB; ++i) {
                    const float p = __builtin_amdgcn_exp2f(sc4[i] - mn);
                    st.l[g] += p;
#pragma unroll
                    for (int j = 0; j < 8; ++j) st.acc[g][j] = __builtin_fmaf(p, (float)vr[i][j], st.acc[g][j]);
                }
            }
        }
    }
    // the definite rows as far as they fill whole rounds; the last NB of these are still on their way
    __device__ __forceinline__ void definite(const Src &s, int n_def)
    {
        h = 0;
#pragma unroll
        for (int x = 0; x < NB; ++x)
            if ((x + 1) * HR <= n_def) issue(s, k[x], v[x], x, n_def);
        for (;; h += NB) {
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                if ((h + NB + x + 1) * HR > n_def) {
                    at = x;
                    return;
                }
                fold(s, k[x], v[x], h + x, n_def);
                issue(s, k[x], v[x], h + NB + x, n_def);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    // all that is left of the n rows
    __device__ __forceinline__ void rest(const Src &s, int n_def, int n)
    {
        if (h == 0 && at == 0) {
            // (rounds that have not been issued yet: fewer definite rows than fill NB)
#pragma unroll
            for (int x = 0; x < NB; ++x)
                if ((x + 1) * HR > n_def && x * HR < n) issue(s, k[x], v[x], x, n);
        }
        for (;; h += NB) {
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                if (x < at) continue;
                if ((h + x) * HR >= n) return;
                fold(s, k[x], v[x], h + x, n);
                if ((h + NB + x) * HR < n) issue(s, k[x], v[x], h + NB + x, n);
                __builtin_amdgcn_sched_barrier(0);
            }
            at = 0;
        }
    }
};

// Rows of larger query groups on the matrix cores (see attend_rows_mfma): a row wavefront takes 16 rows a
// round.  The K pieces of a tile are dead once its scores are formed, the V pieces once they are folded
// in: the next round's loads are issued into the same registers.
template <int RW>
struct MatrixRows {
    static constexpr int HR = RW * 16;
    half8 kr[4], vr[4];
    MfmaState st;
    int h;
    bool live;  // round h has been issued

    struct Src {
        const char *Ku, *Vu;
        uint32_t row_bytes;
        const uint16_t *sel;
        const _Float16 *q;  // the lane's head's query row, from channel 8 hi on
        float *sc;          // 16 floats of LDS private to the wavefront
        int place;          // the wavefront's place among the row wavefronts
    };
    // (the tile's first row; rows past the end re-read the last one and their scores are masked)
    __device__ __forceinline__ int row0(const Src &s, int round) const { return round * HR + s.place * 16; }
    __device__ __forceinline__ void issue_k(const Src &s, int r0, int n)
    {
        const int lo = threadIdx.x & 15, hi = (threadIdx.x & 63) >> 4;
        const uint32_t off = (uint32_t)s.sel[min(r0 + lo, n - 1)] * s.row_bytes + 16u * (uint32_t)hi;
#pragma unroll
        for (int x = 0; x < 4; ++x) kr[x] = row_load<false>(reinterpret_cast<const half8 *>(s.Ku + off + 64u * x));
    }
    __device__ __forceinline__ void issue_v(const Src &s, int r0, int n)
    {
        const int lo = threadIdx.x & 15, hi = (threadIdx.x & 63) >> 4;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            vr[r] = row_load(reinterpret_cast<const half8 *>(s.Vu + ((uint32_t)s.sel[min(r0 + 4 * hi + r, n - 1)] * s.row_bytes + 16u * (uint32_t)lo)));
    }
    __device__ __forceinline__ void step(const Src &s, int n, bool more)
    {
        const int hi = (threadIdx.x & 63) >> 4, lo = threadIdx.x & 15;
        const int r0 = row0(s, h), r1 = row0(s, h + 1);
        more = more && r1 < n;
        __builtin_amdgcn_sched_barrier(0);
        float4v S = (float4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int x = 0; x < 4; ++x)
            S = __builtin_amdgcn_mfma_f32_16x16x32_f16(kr[x], *reinterpret_cast<const half8 *>(s.q + 32 * x), S, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (more) issue_k(s, r1, n);
        __builtin_amdgcn_sched_barrier(0);
        mfma_fold(S, vr, r0, n, st, s.sc, lo, hi);
        __builtin_amdgcn_sched_barrier(0);
        if (more) issue_v(s, r1, n);
    }
    __device__ __forceinline__ void definite(const Src &s, int n_def)
    {
        h = 0;
        live = HR <= n_def;
        if (!live) return;
        issue_k(s, row0(s, 0), n_def);
        issue_v(s, row0(s, 0), n_def);
        for (; (h + 2) * HR <= n_def; ++h) step(s, n_def, true);
    }
    __device__ __forceinline__ void rest(const Src &s, int n)
    {
        if (!live && row0(s, h) < n) {
            issue_k(s, row0(s, h), n);
            issue_v(s, row0(s, h), n);
        }
        // (the first round after definite() has been issued, but not the one behind it)
        for (; row0(s, h) < n; ++h) step(s, n, true);
    }
};

// Combines the n_ch chunk partials of each of a unit's G heads (see merge_partials): 2 NW groups of 32
// threads, four channels each; gph groups share a head's partials, eight of them in flight, so that the
// dependent batches of loads, a round trip to memory each at the launch's very end, are few (12 units of
// 20K tokens in groups of 7, 10 chunks: one channel to a thread, and seven rounds of heads, took 9 us).
template <int NW>
__device__ __forceinline__ void merge_unit(const float *part_unit, int G, int n_ch, float *out_unit,
                                           float (*red)[kD], float (*red_ml)[2])
{
    constexpr int NG = 2 * NW, kBatch = 8;
    const int tid = threadIdx.x, grp = tid >> 5, d4 = (tid & 31) * 4;
    int gph = 1;
    while (gph * 2 <= n_ch && gph * 2 * min(G, NG) <= NG) gph *= 2;
    const int hpr = NG / gph, hr = grp / gph, sub = grp % gph;
    for (int g0 = 0; g0 < G; g0 += hpr) {
        const int g = g0 + hr;
        float m = kNegInf, l = 0.0f;
        float4 A = make_float4(0.f, 0.f, 0.f, 0.f);
        if (g < G) {
            const float *ph = part_unit + (size_t)g * n_ch * kPartStride;
            for (int c0 = sub; c0 < n_ch; c0 += gph * kBatch) {
                float2 ml[kBatch], lo[kBatch], hi[kBatch];
#pragma unroll
                for (int i = 0; i < kBatch; ++i) {
                    if (c0 + i * gph < n_ch) {
                        const float *pc = ph + (size_t)(c0 + i * gph) * kPartStride;
                        ml[i] = ld_dev(reinterpret_cast<const float2 *>(pc));
                        lo[i] = ld_dev(reinterpret_cast<const float2 *>(pc + 4 + d4));
                        hi[i] = ld_dev(reinterpret_cast<const float2 *>(pc + 6 + d4));
                    } else {
                        ml[i] = make_float2(kNegInf, 0.f);
                        lo[i] = hi[i] = make_float2(0.f, 0.f);
                    }
                }
#pragma unroll
                for (int i = 0; i < kBatch; ++i) {
                    if (ml[i].x != kNegInf) {
                        const float mn = fmaxf(m, ml[i].x);
                        const float so = (m == kNegInf) ? 0.0f : __builtin_amdgcn_exp2f(m - mn);
                        const float sn = __builtin_amdgcn_exp2f(ml[i].x - mn);
                        l = l * so + ml[i].y * sn;
                        A.x = A.x * so + lo[i].x * sn;
                        A.y = A.y * so + lo[i].y * sn;
                        A.z = A.z * so + hi[i].x * sn;
                        A.w = A.w * so + hi[i].y * sn;
                        m = mn;
                    }
                }
            }
        }
        if (gph == 1) {
            if (g < G) *reinterpret_cast<float4 *>(out_unit + (size_t)g * kD + d4) = make_float4(A.x / l, A.y / l, A.z / l, A.w / l);
            continue;
        }
        *reinterpret_cast<float4 *>(&red[grp][d4]) = A;
        if (d4 == 0) {
            red_ml[grp][0] = m;
            red_ml[grp][1] = l;
        }
        __syncthreads();
        for (int i = tid; i < hpr * kD; i += 64 * NW) {
            const int hh = i >> 7, d = i & (kD - 1);
            if (g0 + hh < G) {
                float M = kNegInf, As = 0.0f, Ls = 0.0f;
                for (int x = 0; x < gph; ++x) M = fmaxf(M, red_ml[hh * gph + x][0]);
                for (int x = 0; x < gph; ++x) {
                    const float ms = red_ml[hh * gph + x][0];
                    const float f = (ms == kNegInf) ? 0.0f : __builtin_amdgcn_exp2f(ms - M);
                    As += f * red[hh * gph + x][d];
                    Ls += f * red_ml[hh * gph + x][1];
                }
                out_unit[(size_t)(g0 + hh) * kD + d] = As / Ls;
            }
        }
        __syncthreads();
    }
}

// The wavefronts' states of n_heads heads in wpart[wave][head] = {m, l, -, -, acc[128]} merged in wave
// order: the result to out_direct, or the workgroup's partial to po.  128 threads a head where that takes one
// round of heads, else 32 threads a head, four channels each (the quotients are what costs: with 32 threads
// one layer of 4K tokens 8.83 -> 8.99 us, with 128 eight units of 32K in groups of 8 18.9 -> 19.4).
template <int GH, int NW>
__device__ __forceinline__ void combine_waves(const float (*wpart)[GH][kPartStride], int n_heads, float *po, size_t head_stride,
                                              float *out_direct)
{
    constexpr int CH = GH <= NW / 2 ? 1 : 4, TPH = kD / CH;  // channels of a thread, threads of a head
    const int d = (threadIdx.x % TPH) * CH;
    for (int g = threadIdx.x / TPH; g < n_heads; g += 64 * NW / TPH) {
        float mw[NW], M = kNegInf, Ls = 0.0f, A[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) A[c] = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            mw[w] = wpart[w][g][0];
            M = fmaxf(M, mw[w]);
        }
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float f = (mw[w] == kNegInf) ? 0.0f : __builtin_amdgcn_exp2f(mw[w] - M);
#pragma unroll
            for (int c = 0; c < CH; ++c) A[c] += f * wpart[w][g][4 + d + c];
            Ls += f * wpart[w][g][1];
        }
        if (out_direct) {
#pragma unroll
            for (int c = 0; c < CH; ++c) out_direct[(size_t)g * kD + d + c] = A[c] / Ls;
        } else {
            float *pg = po + (size_t)g * head_stride;
            if constexpr (CH == 1) {
                st_dev(pg + 4 + d, A[0]);
            } else {
#pragma unroll
                for (int c = 0; c < CH; c += 2)
                    st_dev(reinterpret_cast<uint2 *>(pg + 4 + d + c), make_uint2(__float_as_uint(A[c]), __float_as_uint(A[c + 1])));
            }
            if (d == 0) st_dev(reinterpret_cast<uint2 *>(pg), make_uint2(__float_as_uint(M), __float_as_uint(Ls)));
        }
    }
}

template <int GT, int NW>
__device__ __forceinline__ void store_partial(const RowState<GT> &st, float *pool, int n_heads, float *po, size_t head_stride,
                                              float *out_direct)
{
    float(*wpart)[GT][kPartStride] = reinterpret_cast<float(*)[GT][kPartStride]>(pool);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, part = lane & 15;
#pragma unroll
    for (int g = 0; g < GT; ++g) {
        const float mm = rows_max(st.m[g]);
        const float w = (st.m[g] == kNegInf) ? 0.0f : __builtin_amdgcn_exp2f(st.m[g] - mm);
        const float lv = rows_sum(st.l[g] * w);
        float av[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) av[j] = rows_sum(st.acc[g][j] * w);
        if (lane < 16) {
            float4 *to = reinterpret_cast<float4 *>(&wpart[wave][g][4 + part * 8]);
            to[0] = make_float4(av[0], av[1], av[2], av[3]);
            to[1] = make_float4(av[4], av[5], av[6], av[7]);
            if (part == 0) {
                wpart[wave][g][0] = mm;
                wpart[wave][g][1] = lv;
            }
        }
    }
    __syncthreads();
    combine_waves<GT, NW>(wpart, n_heads, po, head_stride, out_direct);
}

// (eight heads at a time, as many as the pool holds)
template <int GT, int NW>
__device__ __forceinline__ void store_partial(const MfmaState &st, float *pool, int n_heads, float *po, size_t head_stride,
                                              float *out_direct)
{
    constexpr int GH = GT < 8 ? GT : 8;
    float(*wpart)[GH][kPartStride] = reinterpret_cast<float(*)[GH][kPartStride]>(pool);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lo = lane & 15, hi = lane >> 4;
    const float lv = rows_sum(st.l);
#pragma unroll
    for (int g0 = 0; g0 < GT; g0 += GH) {
        if (g0 >= n_heads) break;
        if (g0) __syncthreads();
        if (hi == 0 && lo >= g0 && lo < g0 + GH) {
            wpart[wave][lo - g0][0] = st.m;
            wpart[wave][lo - g0][1] = lv;
        }
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int head = 4 * hi + rr - g0;
            if (head >= 0 && head < GH) {
                float4 *to = reinterpret_cast<float4 *>(&wpart[wave][head][4 + 8 * lo]);
                to[0] = make_float4(st.O[0][rr], st.O[1][rr], st.O[2][rr], st.O[3][rr]);
                to[1] = make_float4(st.O[4][rr], st.O[5][rr], st.O[6][rr], st.O[7][rr]);
            }
        }
        __syncthreads();
        combine_waves<GH, NW>(wpart, min(GH, n_heads - g0), po + (size_t)g0 * head_stride, head_stride,
                              out_direct ? out_direct + (size_t)g0 * kD : nullptr);
    }
}

template <int GT, int SMODE, int NW, bool ST, int HB = 4, int NB = 2>
__device__ __forceinline__ void decode_unit(const AttendArgs &a)
{
    using LR = LabelRows<SMODE>;
    constexpr int WGT = 64 * NW, RW = NW - 1;
    constexpr int RR = LR::RR, NV = LR::NV, PE = LR::PE, TPL = LR::TPL, SB = LR::SB, STEPS = LR::STEPS;
    using Piece = typename LR::Piece;
    extern __shared__ __attribute__((aligned(16))) uint32_t dyn_sh[];
    uint16_t *sel = reinterpret_cast<uint16_t *>(dyn_sh);  // ch tokens: definite rows, then selected candidates
    // 16 KiB: the chunk histogram; then radix bins and staged candidates of the settling wavefront;
    // then the wavefronts' partials
    constexpr bool kMatrix = GT > 2;
    constexpr int kPart = NW * (GT < 8 ? GT : 8) * kPartStride, kPool = kPart > kHistBins ? kPart : kHistBins;
    __shared__ __attribute__((aligned(16))) uint32_t pool[kPool];
    __shared__ __attribute__((aligned(16))) uint2 cand_sh[kCandLds], small_sh[64];
    __shared__ __attribute__((aligned(16))) _Float16 qrow_sh[GT > 8 ? GT : 8][kQRow];
    __shared__ uint32_t coarse_sh[256];
    __shared__ uint32_t s_cnt[NW], s_w[NW], s_res[2], s_T[2], s_base, s_nsel, s_n, s_off, s_ready, s_flag, s_ok, s_failed, s_sticky;
    __shared__ float red_ml[2 * NW][2];
    __shared__ __attribute__((aligned(16))) float sc_sh[kMatrix ? NW : 1][16];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int u = blockIdx.y + a.unit0, c = blockIdx.x;
    const int hk = u % a.Hkv;
    const int t0 = c * a.ch, n_tok = min(a.L, t0 + a.ch) - t0;
    const bool single = gridDim.x == 1;
    uint2 *cu = a.cand + (size_t)u * a.L;
    UnitCtl *ctl = a.ctl_rw + u;
    unsigned long long *cand_arrive = reinterpret_cast<unsigned long long *>(&ctl->pad[2]);
    DS_TR(0);
    // The unit's error word, raised by an earlier call or, in this one, by a workgroup that waited in vain for one
    // that starts late.  It can change at any time, so the workgroup goes by thread 0's copy of it, which comes through LDS:
    // wavefronts that left on a value of their own would leave the others with lists half made, and a flag that nobody raises.
    // (Loaded by all: behind a branch of thread 0's the first wavefront waits for it there, before anything else is on its way;
    //  and the copy is read with the first counts, not by itself: 500 calls of 128 to 5000 tokens together 1.9 -> 1.2 % above
    //  those without a copy.)
    const uint32_t sticky = a.ctl[u].err;
    auto raise_err = [&](uint32_t code) {
        uint32_t none = 0u;
        __hip_atomic_compare_exchange_strong(&ctl->err, &none, code, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        s_failed = 1u;
    };
    auto poison_out = [&]() {
        float *ou = a.out + (size_t)u * a.G * kD;
        for (int i = tid; i < a.G * kD; i += WGT) ou[i] = __builtin_nanf("");
    };
    if (tid == 0) s_failed = s_ready = 0u;

    // ---- 1. scores
    // token of key i (from t0), see LabelRows
    auto token_of = [&](int i) {
        if constexpr (LR::kPairs) return i * WGT + wave * 64 + (lane >> 1) + ((lane & 1) ? 32 : 0);
        else if constexpr (LR::kQ4) return (i / TPL) * (WGT * TPL) + tid * TPL + (i % TPL);
        else return i * WGT + tid;
    };
    const int n_pass = (n_tok + WGT * TPL - 1) / (WGT * TPL) * TPL;  // <= kKeys
    Piece v[2][STEPS][NV];
    auto issue = [&](Piece (&vv)[STEPS][NV], int bt) {
#pragma unroll
        for (int x = 0; x < STEPS; ++x) {
            const int i = bt * STEPS + x;
            if constexpr (LR::kKeysGiven) {
                vv[x][0] = (a.keys + (size_t)u * a.key_stride + t0)[min(i * WGT + tid, n_tok - 1)];
            } else if constexpr (LR::kQ4) {
                constexpr int WW = RR / 8;
                const uint32_t *codes = reinterpret_cast<const uint32_t *>(a.label) + ((size_t)u * a.L_max + t0) * WW;
                const int t = min(i * WGT * TPL + tid * TPL, (n_tok - 1) & ~(TPL - 1));
                vv[x][0] = stream_load<ST>(reinterpret_cast<const uint4 *>(codes + (size_t)t * WW));
            } else {
                const _Float16 *lab = a.label + ((size_t)u * a.L_max + t0) * RR;
                if constexpr (LR::kPairs) {
                    // (whole cache lines per load, two tokens' halves per lane: neighbours swap below)
                    const int p0 = 2 * (i * WGT + wave * 64) + lane, p_last = 2 * n_tok - 1;
                    const half8 *pieces = reinterpret_cast<const half8 *>(lab);
                    vv[x][0] = label_load<1, ST>(pieces + min(p0, p_last));
                    vv[x][1] = label_load<1, ST>(pieces + min(p0 + 64, p_last));
                } else {
                    const Piece *row = reinterpret_cast<const Piece *>(lab + (size_t)min(i * WGT + tid, n_tok - 1) * RR);
#pragma unroll
                    for (int j = 0; j < NV; ++j) vv[x][j] = label_load<NV, ST>(row + j);
                }
            }
        }
    };
    // label query of the group; the first two batches of label rows are on their way meanwhile
    // (every wavefront forms it for itself, a channel to a lane: one barrier less than by one of them)
    constexpr int QL = (RR + 63) / 64;
    const bool scaled = LR::kQ4 || (LR::kKeysGiven && a.amax);
    int c_q[QL];
    float a_q[QL], step[QL];
#pragma unroll
    for (int x = 0; x < QL; ++x) {
        const int j = lane + 64 * x;
        c_q[x] = j < a.r ? a.channels[hk * a.r + j] : 0;
        step[x] = scaled && j < a.r ? a.amax[(size_t)u * a.r + j] : 0.0f;
        a_q[x] = 0.0f;
    }
    for (int g0 = 0; g0 < a.G; g0 += 8) {
        const int ng = min(8, a.G - g0);
        if (g0) __syncthreads();
        uint4 qv = make_uint4(0u, 0u, 0u, 0u);
        const int qg = (tid - 128) >> 4, qp = (tid - 128) & 15;
        const bool has_q = tid >= 128 && tid < 256;  // (rows that there are not: zeros)
        if (has_q && qg < ng)
            qv = *reinterpret_cast<const uint4 *>(a.q + ((size_t)u * a.G + g0 + qg) * kD + qp * 8);
        if (g0 == 0) {
            // (no wavefront's label loads before the query's: they share one queue)
            __builtin_amdgcn_s_barrier();
            issue(v[0], 0);
            if (SB < n_pass) issue(v[1], 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < kHistBins / 4 / WGT; ++i)
                reinterpret_cast<uint4 *>(pool)[i * WGT + tid] = make_uint4(0u, 0u, 0u, 0u);
        }
        if (has_q) *reinterpret_cast<uint4 *>(&qrow_sh[qg][qp * 8]) = qv;
        __syncthreads();
#pragma unroll
        for (int x = 0; x < QL; ++x) {
            _Float16 y[8];  // (all eight on their way at once; zeros where there is no head)
#pragma unroll
            for (int g = 0; g < 8; ++g) y[g] = qrow_sh[g][c_q[x]];
#pragma unroll
            for (int g = 0; g < 8; ++g) a_q[x] = a_q[x] + (float)y[g];
        }
    }
#pragma unroll
    for (int x = 0; x < QL; ++x) {
        if (scaled) a_q[x] = a_q[x] * (step[x] / 7.0f);
        if (lane + 64 * x >= a.r) a_q[x] = 0.0f;
    }
    DS_TR(15);
    float qs[LR::kKeysGiven ? 1 : RR], magnitude = 0.0f;  // (the largest of the label query)
    if constexpr (LR::kKeysGiven) {
        magnitude = fmaxf(fabsf(a_q[0]), fabsf(a_q[QL - 1]));
#pragma unroll
        for (int m = 1; m < 16; m *= 2) magnitude = fmaxf(magnitude, __shfl_xor(magnitude, m));
        magnitude = rows_max(magnitude);
    } else {
#pragma unroll
        for (int j = 0; j < RR; ++j) {
            qs[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a_q[0]), j));
            magnitude = fmaxf(magnitude, fabsf(qs[j]));
        }
    }
    const BinScale bins(__builtin_amdgcn_readfirstlane(__float_as_int(magnitude)));
    typedef uint32_t KeyVec __attribute__((ext_vector_type(kKeys)));
    KeyVec key;
    auto nib = [](uint32_t word, int i) { return (float)(((int32_t)(word << (28 - 4 * i))) >> 28); };
    auto score = [&](Piece (&vv)[STEPS][NV], int bt) {
#pragma unroll
        for (int x = 0; x < STEPS; ++x) {
            if constexpr (LR::kPairs) {
                const bool odd = lane & 1;
                const half8 got = swap_pairs(odd ? vv[x][0] : vv[x][1]);
                if (odd) vv[x][0] = got;
                else vv[x][1] = got;
            }
#pragma unroll
            for (int e = 0; e < TPL; ++e) {
                const int i = (bt * STEPS + x) * TPL + e;
                float acc = 0.0f;
                if constexpr (LR::kKeysGiven) {
                } else if constexpr (LR::kQ4) {
                    constexpr int WW = RR / 8;
                    const uint32_t c4[4] = {vv[x][0].x, vv[x][0].y, vv[x][0].z, vv[x][0].w};
#pragma unroll
                    for (int w = 0; w < WW; ++w)
#pragma unroll
                        for (int j = 0; j < 8; ++j) acc = __builtin_fmaf(qs[w * 8 + j], nib(c4[e * WW + w], j), acc);
                } else {
#pragma unroll
                    for (int j = 0; j < NV; ++j)
#pragma unroll
                        for (int f = 0; f < PE; ++f) acc = __builtin_fmaf(qs[j * PE + f], (float)vv[x][j][f], acc);
                }
                key[i] = 0u;  // (past the chunk's end: below every bin's first key that counts)
                if (token_of(i) < n_tok) {
                    uint32_t bits, sgn;
                    if constexpr (LR::kKeysGiven) {
                        key[i] = vv[x][0];
                        sgn = ~(uint32_t)((int32_t)key[i] >> 31);
                        bits = key[i] ^ sgn;
                    } else {
                        // (never -0, which would have to tie with +0: a sum that starts from +0 becomes -0 only where a tiny
                        //  negative number is rounded, and sums of such products are 0 or above 2^-80)
                        bits = __float_as_uint(acc);
                        sgn = (uint32_t)((int32_t)bits >> 31);
                        key[i] = bits ^ (sgn | 0x80000000u);
                    }
                    atomicAdd(&pool[kSideBins + (bins.bin(bits) ^ sgn)], 1u);
                }
            }
        }
    };
#pragma unroll
    for (int bt = 0; bt < kKeys / SB; bt += 2) {
        if (bt * SB >= n_pass) break;
        score(v[0], bt);
        if ((bt + 2) * SB < n_pass) issue(v[0], bt + 2);
        __builtin_amdgcn_sched_barrier(0);
        if ((bt + 1) * SB >= n_pass) break;
        score(v[1], bt + 1);
        if ((bt + 3) * SB < n_pass) issue(v[1], bt + 3);
        __builtin_amdgcn_sched_barrier(0);
    }
    DS_PRIO(3);
    if (tid == 0) s_sticky = sticky;
    __syncthreads();
    DS_TR(11);
    // (whichever workgroup leaves on it writes NaN: without it none of the unit's is the last, which would)
    const uint32_t leave = s_sticky;

    // ---- 2. threshold bin
    uint32_t bstar, krem;
    if (single) {
        find_bin<NW>(pool, (uint32_t)a.k_eff, s_w, s_res);
        if (__builtin_expect(leave != 0u, 0)) {
            poison_out();
            return;
        }
        bstar = s_res[0];
        krem = s_res[1];
    } else {
        // The chunk's coarse counts (16 bins each) are added to the unit's; of the fine ones only those of the
        // three coarse bins round the one that holds the chunk's share of k, and later, where the
        // unit's threshold lies elsewhere, of that one.
        uint32_t *hu = a.hist + (size_t)u * kHistBins;
        uint32_t *cuh = a.coarse + (size_t)u * 256;
        if (__builtin_expect(leave != 0u, 0)) {
            poison_out();
            return;
        }
        if (tid < 256) {
            uint32_t cc = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint4 q = reinterpret_cast<const uint4 *>(pool)[tid * 4 + ((i + tid) & 3)];
                cc += (q.x + q.y) + (q.z + q.w);
            }
            if (cc) atomicAdd(&cuh[tid], cc);
            coarse_sh[tid] = cc;
        }
        __syncthreads();
        if (wave == 0) {
            // lane l owns the coarse bins 255 - 4 l .. 252 - 4 l, from the top
            auto scan = [&](const uint32_t (&cc)[4]) { return (uint32_t)wave_inclusive_scan((int)((cc[0] + cc[1]) + (cc[2] + cc[3])), lane); };
            auto find = [&](const uint32_t (&cc)[4], uint32_t incl, uint32_t want, uint32_t &bin, uint32_t &rank, uint32_t &count) {
                uint32_t before = incl - ((cc[0] + cc[1]) + (cc[2] + cc[3])), at = 0, n = 0, bef = 0;
                bool done = false;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (!done && before < want && before + cc[i] >= want) {
                        at = 255u - 4u * (uint32_t)lane - (uint32_t)i;
                        n = cc[i];
                        bef = before;
                        done = true;
                    }
                    before += cc[i];
                }
                const unsigned long long hit = __ballot(done);
                if (!hit) { bin = 0u; rank = 1u; count = 0xffffffffu; return; }
                const int l = __builtin_ctzll(hit);
                bin = read_lane(at, l);
                rank = want - read_lane(bef, l);
                count = read_lane(n, l);
            };
            uint32_t cb0;
            {
                const uint32_t k_loc = min(max((uint32_t)((float)n_tok * a.k_share), 1u), (uint32_t)n_tok);
                uint32_t cc[4], bin, rank, count;
#pragma unroll
                for (int i = 0; i < 4; ++i) cc[i] = coarse_sh[255 - 4 * lane - i];
                find(cc, scan(cc), k_loc, bin, rank, count);
                cb0 = min(max(bin, 1u) - 1u, 253u);  // fine bins of the coarse bins cb0 .. cb0 + 2
                if (lane < 48) {
                    const uint32_t x = pool[cb0 * 16 + lane];
                    if (x) atomicAdd(&hu[cb0 * 16 + lane], x);
                }
            }
            uint32_t extra = 0xffffffffu;  // another coarse bin whose fine counts have been added
            // (The unit's histograms are complete when the coarse counts add up to L and the fine counts
            //  of the unit's coarse bin to its count: looked at until they are.  An arrival counter
            //  in front of them was one more round trip to memory on every workgroup's path.)
            uint32_t bin = kHistBins - 1, rk = 1;
            for (uint32_t attempt = 0;; ++attempt) {
                uint32_t fv = 0;
                if (lane < 48) fv = ld_dev(hu + cb0 * 16 + lane);
                const uint2 hi2 = ld_dev(reinterpret_cast<const uint2 *>(cuh + 254 - 4 * lane));
                const uint2 lo2 = ld_dev(reinterpret_cast<const uint2 *>(cuh + 252 - 4 * lane));
                const uint32_t cc[4] = {hi2.y, hi2.x, lo2.y, lo2.x};
                const uint32_t incl_c = scan(cc);
                if (read_lane(incl_c, 63) == (uint32_t)a.L) {
                    uint32_t cb, rank, count;
                    find(cc, incl_c, (uint32_t)a.k_eff, cb, rank, count);
                    // lane i < 16: the coarse bin's i-th fine count from the top
                    uint32_t f;
                    if (cb - cb0 < 3u) {
                        f = (uint32_t)__shfl((int)fv, (int)((cb - cb0) * 16u) + 15 - (lane & 15));
                    } else {
                        if (extra != cb && lane < 16) {
                            const uint32_t x = pool[cb * 16 + lane];
                            if (x) atomicAdd(&hu[cb * 16 + lane], x);
                        }
                        extra = cb;
                        f = ld_dev(hu + cb * 16 + 15 - (lane & 15));
                    }
                    if (lane >= 16) f = 0u;
                    const uint32_t incl = (uint32_t)wave_inclusive_scan((int)f, lane);
                    const unsigned long long hit = __ballot(lane < 16 && incl - f < rank && incl >= rank);
                    if (read_lane(incl, 63) == count && hit) {
                        const int l = __builtin_ctzll(hit);
                        bin = cb * 16u + 15u - (uint32_t)l;
                        rk = rank - read_lane(incl - f, l);
                        break;
                    }
                }
                // (counts that never add up: a workspace that was not cleared, or adds that do not arrive)
                if (attempt + 1u >= a.spin_limit) {
                    if (lane == 0) raise_err(9u);
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            if (lane == 0) {
                s_T[0] = bin;
                s_T[1] = rk;
            }
        }
        __syncthreads();
        bstar = s_T[0];
        krem = s_T[1];
    }
    DS_TR(10);

    // ---- 3. lists
    // One look at each key: which of the thread's keys are definite and which are candidates goes into
    // bit masks (bit j <-> key n_seen - 1 - j); the writes walk the set bits, few as they are.
    uint32_t lo_key, hi_key;
    bins.keys((uint32_t)__builtin_amdgcn_readfirstlane((int)bstar), lo_key, hi_key);
    lo_key = max(lo_key, 1u);  // (dead keys are zero)
    const int span = hi_key > lo_key ? 32 - __builtin_clz(hi_key - lo_key) : 0;  // <= 31
    const int tb = 32 - __builtin_clz(max(a.L - 1, 1));  // <= 24
    uint32_t mdef = 0, mcan = 0;
    int n_seen = 0;
#pragma unroll
    for (int g = 0; g < kKeys / SB; ++g) {
        if (g * SB >= n_pass) break;
#pragma unroll
        for (int e = 0; e < SB; ++e) {
            push_less(mdef, hi_key, key[g * SB + e]);
            push_less(mcan, lo_key - 1u, key[g * SB + e]);
        }
        n_seen += SB;
    }
    mcan &= ~mdef;
    const uint32_t mine = (uint32_t)__builtin_popcount(mdef) | (uint32_t)__builtin_popcount(mcan) << 16;
    const uint32_t winc = (uint32_t)wave_inclusive_scan((int)mine, lane);
    if (lane == 63) s_cnt[wave] = winc;
    // groups of more than eight heads: the query rows of a pass (the label query had eight at a time)
    auto load_q16 = [&](int g0) {
        if (tid < 256) {
            const int g = tid >> 4, pp = tid & 15;
            uint4 x = make_uint4(0u, 0u, 0u, 0u);
            if (g0 + g < a.G) x = *reinterpret_cast<const uint4 *>(a.q + ((size_t)u * a.G + g0 + g) * kD + pp * 8);
            *reinterpret_cast<uint4 *>(&qrow_sh[g][pp * 8]) = x;
        }
    };
    if constexpr (GT > 8) load_q16(0);
    __syncthreads();
    uint32_t n_cand;
    int n_def;
    uint32_t early_base = 0, cand_base = 0;  // the workgroup's place in the unit's list
    {
        const uint32_t x = lane < NW ? s_cnt[lane] : 0u;
        const uint32_t incl = (uint32_t)wave_inclusive_scan((int)x, lane);
        const uint32_t total = read_lane(incl, 63), ex = read_lane(incl - x, wave) + winc - mine;
        n_def = (int)(total & 0xffffu);
        n_cand = total >> 16;
        if (!single && tid == 0 && n_cand)
            early_base = (uint32_t)__hip_atomic_fetch_add(cand_arrive, (unsigned long long)n_cand, __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_AGENT);
        uint16_t *dp = sel + (ex & 0xffffu);
        for (; mdef; mdef &= mdef - 1u) *dp++ = (uint16_t)token_of(n_seen - 1 - __builtin_ctz(mdef));
        // (one key in a thousand is a candidate)
        if (__builtin_expect(n_cand > kCandLds, 0)) {
            if (tid == 0) s_base = early_base;
            __syncthreads();
            cand_base = s_base;
            if (cand_base + n_cand > (uint32_t)a.L && tid == 0) raise_err(8u);
        }
        unsigned long long any = __ballot(mcan != 0u);
        if (any) {
            uint32_t cp = read_lane(ex >> 16, 0);
            do {
                // the candidates among the wavefront's keys of one index
                const uint32_t bit = (uint32_t)__builtin_ctz(read_lane(mcan, __builtin_ctzll(any)));
                const int i = n_seen - 1 - (int)bit;
                const uint32_t kk = key[i];
                const bool has = mcan >> bit & 1u;
                const unsigned long long hm = __ballot(has);
                const uint32_t at = cp + bits_below(hm);
                if (has) {
                    const uint2 entry = make_uint2(kk, (uint32_t)(t0 + token_of(i)));
                    if (at < kCandLds) cand_sh[at] = entry;
                    else if (__builtin_expect(cand_base + at < (uint32_t)a.L, 0)) st_dev(cu + cand_base + at, entry);
                    mcan &= ~(1u << bit);
                }
                cp += (uint32_t)__builtin_popcountll(hm);
                any = __ballot(mcan != 0u);
            } while (any);
            if (__builtin_expect(n_cand > kCandLds, 0)) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
    }
    __syncthreads();
    DS_TR(1);

    // ---- 4. wavefront 0: exact threshold and the workgroup's selected candidates; the others: definite rows
    const char *Ku = reinterpret_cast<const char *>(a.K + ((size_t)u * a.L_max + t0) * a.kv_stride);
    const char *Vu = reinterpret_cast<const char *>(a.V + ((size_t)u * a.L_max + t0) * a.kv_stride);
    const uint32_t row_bytes = 2 * a.kv_stride;
    uint32_t *lh = pool;
    // candidate i of this workgroup
    if (n_cand <= kCandLds && wave == 0) cand_base = (uint32_t)__builtin_amdgcn_readfirstlane((int)early_base);
    auto own_cand = [&](uint32_t i) { return i < kCandLds ? cand_sh[i] : ld_dev(cu + min(cand_base + i, (uint32_t)a.L - 1u)); };
    using Rows = typename std::conditional<kMatrix, MatrixRows<RW>, VectorRows<GT, RW, ST, HB, NB>>::type;
    Rows rows;
    typename Rows::Src src;
    src.Ku = Ku;
    src.Vu = Vu;
    src.row_bytes = row_bytes;
    src.sel = sel;
    if constexpr (kMatrix) {
        src.sc = sc_sh[wave];
        src.place = wave - 1;
        src.q = &qrow_sh[lane & (GT > 8 ? 15 : 7)][8 * (lane >> 4)];
    } else {
        src.q = qrow_sh;
        src.place = (wave - 1) * 4 + (lane >> 4);
    }
    rows.st.init();
    HeldCands<2, decltype(own_cand)> own(n_cand, own_cand);
    const bool want_off = !single && a.idx_out;
    if (wave == 0) {
        uint32_t n = n_cand, off = 0;
        bool big = false, ok = true;
        uint32_t T = 0xffffffffu;
        int tcut = -1;
        if (single) {
            big = n > kWaveSettlesOwn || !wave_settle(own, krem, lo_key, span, tb, lh, small_sh, T, tcut);
        } else {
            // the candidates of all of the unit's workgroups meet in its list in memory, and every workgroup
            // settles the threshold by itself
            if (cand_base + n_cand <= (uint32_t)a.L) {
                for (uint32_t i = lane; i < min(n_cand, kCandLds); i += 64) st_dev(cu + cand_base + i, cand_sh[i]);
            } else if (lane == 0) {
                raise_err(8u);
            }
            if (want_off && lane == 0) st_dev(a.ndef + (size_t)u * a.n_ch + c, (uint32_t)n_def);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            uint2 w = make_uint2(0u, 0u);
            if (lane == 0) {
                const unsigned long long t = __hip_atomic_fetch_add(cand_arrive, 1ull << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                w = make_uint2((uint32_t)t, (uint32_t)(t >> 32) + 1u);
            }
            DS_TR(2);
            for (uint32_t it = 0;; ++it) {
                n = (uint32_t)__builtin_amdgcn_readfirstlane((int)w.x);
                if ((uint32_t)__builtin_amdgcn_readfirstlane((int)w.y) == gridDim.x) break;
                if (it >= a.spin_limit) { ok = false; break; }
                __builtin_amdgcn_s_sleep(1);
                w = ld_dev(reinterpret_cast<const uint2 *>(cand_arrive));
            }
            DS_TR(12);
            n = min(n, (uint32_t)a.L);
            if (!ok) {
                if (lane == 0) raise_err(6u);  // (nothing more is selected)
            } else {
                auto unit_at = [&](uint32_t i) { return ld_dev(cu + i); };
                HeldCands<6, decltype(unit_at)> all(n, unit_at);
                uint32_t before = 0;
                if (want_off)
                    for (int i = lane; i < c; i += 64) before += ld_dev(a.ndef + (size_t)u * a.n_ch + i);
                big = n > kWaveSettlesUnit || !wave_settle(all, krem, lo_key, span, tb, lh, small_sh, T, tcut);
                if (want_off && !big) {
                    // selected tokens in front of this chunk
                    all.each([&](uint2 e, bool have) {
                        if (have && (int)e.y < t0 && is_selected(e.x, (int)e.y, T, tcut)) ++before;
                    });
                    off = read_lane((uint32_t)wave_inclusive_scan((int)before, lane), 63);
                }
            }
            DS_TR(14);
        }
        DS_TR(4);
        uint32_t n_sel = 0;
        if (__builtin_expect(!big, 1)) {
            own.each([&](uint2 e, bool have) {
                const bool hit = have && e.y - (uint32_t)t0 < (uint32_t)n_tok && is_selected(e.x, (int)e.y, T, tcut);
                const unsigned long long hm = __ballot(hit);
                if (hm) {
                    if (hit) sel[n_def + (int)n_sel + (int)bits_below(hm)] = (uint16_t)(e.y - (uint32_t)t0);
                    n_sel += (uint32_t)__builtin_popcountll(hm);
                }
            });
        }
        if (lane == 0) {
            s_nsel = n_sel;
            s_n = n;
            s_off = off;
            __hip_atomic_store(&s_ready, big ? 2u : 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        DS_TR(5);
        if (__builtin_expect(a.idx_out && !big, 0)) {
            // the chunk's slice of the index list, in token order: the row list as a bit mask (where the
            // candidates were), its set bits counted; a lane takes consecutive words of it
            uint32_t *words = reinterpret_cast<uint32_t *>(cand_sh);
            int32_t *io = a.idx_out + (size_t)u * a.k;
            const int n_words = (n_tok + 31) >> 5, per = (n_words + 63) >> 6, n_rows = n_def + (int)n_sel;
            wave_lds_sync();
            for (int i = lane; i < n_words; i += 64) words[i] = 0u;
            wave_lds_sync();
            for (int i = lane; i < n_rows; i += 64) atomicOr(&words[sel[i] >> 5], 1u << (sel[i] & 31));
            wave_lds_sync();
            uint32_t mine = 0;
            for (int i = lane * per; i < min(n_words, (lane + 1) * per); ++i) mine += (uint32_t)__builtin_popcount(words[i]);
            uint32_t at = off + (uint32_t)wave_inclusive_scan((int)mine, lane) - mine;
            for (int i = lane * per; i < min(n_words, (lane + 1) * per); ++i)
                for (uint32_t w = words[i]; w; w &= w - 1u, ++at)
                    if (at < (uint32_t)a.k_eff) io[at] = t0 + i * 32 + __builtin_ctz(w);
        }
    } else {
        DS_PRIO(0);
        rows.definite(src, n_def);
        DS_TR1(8);
        DS_PRIO(3);
    }
    // (no barrier: a wavefront goes on as soon as the list is complete; what is already on its way stays so.
    //  The flag comes: wavefront 0 is in the workgroup whenever the others are, waits for other workgroups a bounded
    //  number of times, and raises it on every way out of them.)
    uint32_t ready;
    while ((ready = __hip_atomic_load(&s_ready, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP)) == 0u) __builtin_amdgcn_s_sleep(1);
    ready = (uint32_t)__builtin_amdgcn_readfirstlane((int)ready);
    if (__builtin_expect(ready == 2u, 0)) {
        __syncthreads();
        // (hundreds of candidates: all wavefronts together)
        uint32_t T, n_sel = 0, total;
        int tcut;
        const uint32_t n = s_n;
        auto unit_at = [&](uint32_t i) { return single ? own_cand(i) : ld_dev(cu + i); };
        wg_settle<NW>(n, unit_at, krem, lo_key, span, tb, lh, s_w, s_res, T, tcut);
        if (want_off) {
            uint32_t before = 0;
            for (int i = tid; i < c; i += WGT) before += ld_dev(a.ndef + (size_t)u * a.n_ch + i);
            wg_each<WGT>(n, unit_at, [&](uint2 e) { before += (int)e.y < t0 && is_selected(e.x, (int)e.y, T, tcut) ? 1u : 0u; });
            block_exclusive_scan<NW>(before, s_w, &total);
            if (tid == 0) s_off = total;
        }
        for (uint32_t i0 = 0; i0 < n_cand; i0 += 8u * WGT) {
            uint2 v[8];
            uint32_t hits = 0;
#pragma unroll
            for (int x = 0; x < 8; ++x) v[x] = own_cand(min(i0 + (uint32_t)(x * WGT + tid), n_cand - 1u));
#pragma unroll
            for (int x = 0; x < 8; ++x)
                if (i0 + (uint32_t)(x * WGT + tid) < n_cand && v[x].y - (uint32_t)t0 < (uint32_t)n_tok && is_selected(v[x].x, (int)v[x].y, T, tcut))
                    hits |= 1u << x;
            uint32_t at = (uint32_t)n_def + n_sel + block_exclusive_scan<NW>((uint32_t)__builtin_popcount(hits), s_w, &total);
#pragma unroll
            for (int x = 0; x < 8; ++x)
                if (hits >> x & 1u) sel[at++] = (uint16_t)(v[x].y - (uint32_t)t0);
            n_sel += total;
        }
        if (tid == 0) s_nsel = n_sel;
        __syncthreads();
        if (a.idx_out) {
            const uint32_t off = s_off;
            const int n_rows = n_def + (int)n_sel;
            int32_t *io = a.idx_out + (size_t)u * a.k;
            const int n_words = (n_tok + 31) >> 5;  // <= WGT
            for (int i = tid; i < n_words; i += WGT) pool[i] = 0u;
            __syncthreads();
            for (int i = tid; i < n_rows; i += WGT) atomicOr(&pool[sel[i] >> 5], 1u << (sel[i] & 31));
            __syncthreads();
            uint32_t w = tid < n_words ? pool[tid] : 0u, total;
            uint32_t at = off + block_exclusive_scan<NW>((uint32_t)__builtin_popcount(w), s_w, &total);
            for (; w; w &= w - 1u, ++at)
                if (at < (uint32_t)a.k_eff) io[at] = t0 + tid * 32 + __builtin_ctz(w);
            __syncthreads();
        }
    }
    const int n_rows = n_def + (int)s_nsel;
    if (__builtin_expect(a.idx_out && c == 0 && wave == 0, 0))
        for (int i = a.k_eff + lane; i < a.k; i += 64) a.idx_out[(size_t)u * a.k + i] = -1;

    // ---- 5. the other rows; partial.  (Groups of more than GT heads pass over the rows again.)
    for (int g0 = 0; g0 < a.G; g0 += GT) {
        const int n_heads = min(GT, a.G - g0);
        if (g0) {
            __syncthreads();
            if constexpr (GT > 8) load_q16(g0);
            __syncthreads();
            rows.st.init();
        }
        if (wave != 0) {
            DS_PRIO(2);
            if constexpr (kMatrix) {
                if (g0) {
                    rows.h = 0;
                    rows.live = false;
                }
                rows.rest(src, n_rows);
            } else {
                rows.rest(src, n_def, n_rows);
            }
            DS_TR1(13);
            DS_PRIO(3);
        }
        DS_TR(3);
        store_partial<GT, NW>(rows.st, reinterpret_cast<float *>(pool), n_heads,
                              a.part + (((size_t)u * a.G + g0) * a.n_ch + c) * kPartStride, (size_t)a.n_ch * kPartStride,
                              single ? a.out + ((size_t)u * a.G + g0) * kD : nullptr);
    }
    if (single) return;

    // ---- the unit's last workgroup merges the partials and leaves the control words clean
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
        const uint32_t mine = s_failed ? 0x10000u : 0u;
        const uint32_t t = __hip_atomic_fetch_add(&ctl->arrive_c, 1u + mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_flag = ((t & 0xffffu) == gridDim.x - 1u) ? 1u : 0u;
        s_ok = ((t >> 16) != 0u || mine != 0u) ? 0u : 1u;
    }
    __syncthreads();
    DS_TR(6);
    if (!s_flag) return;
    if (tid == 0) {
        ctl->arrive_c = 0u;
        *cand_arrive = 0ull;
    }
    if (!s_ok) poison_out();
    else
        merge_unit<NW>(a.part + (size_t)u * a.G * a.n_ch * kPartStride, a.G, a.n_ch, a.out + (size_t)u * a.G * kD,
                       reinterpret_cast<float(*)[kD]>(pool), red_ml);
    DS_TR(7);
    uint4 *hu4 = reinterpret_cast<uint4 *>(a.hist + (size_t)u * kHistBins);
    for (int i = tid; i < kHistBins / 4; i += WGT) hu4[i] = make_uint4(0u, 0u, 0u, 0u);
    if (tid < 256) a.coarse[(size_t)u * 256 + tid] = 0u;
}

// The decode kernel.  Four wavefronts per SIMD are what the plans count on (two workgroups of 512 threads
// to a compute unit, 128 registers); groups of more than eight heads need more, and get three (one workgroup of
// 512 threads, or three of 256).
// FORM: 10 wavefronts + rows of a 16-lane slot in flight, two or four (single heads and pairs).
template <int GT, int SMODE, int FORM, bool ST>
__global__ __launch_bounds__(FORM / 10 * 64, GT > 8 ? 3 : 4) void k_refine_attend(AttendArgs a)
{
    decode_unit<GT, SMODE, FORM / 10, ST, 2, FORM % 10 / 2>(a);
}

// The instantiation for labels of this kind (see ra_kernel).
template <int GT>
RaFn decode_fn(int smode, DecodeVariant v);

#ifdef DS_TRACE
template <int GT>
int trace_read(void *dst, size_t bytes);
#endif

// Defines them for heads per pass GT, in a source file of its own each (they compile side by side).
template <int GT, int FORM, bool ST>
static RaFn decode_fn_of(int smode)
{
    switch (smode) {
    case 0: return k_refine_attend<GT, 0, FORM, ST>;
    case 4: return k_refine_attend<GT, 4, FORM, ST>;
    case 8: return k_refine_attend<GT, 8, FORM, ST>;
    case 12: return k_refine_attend<GT, 12, FORM, ST>;
    case 16: return k_refine_attend<GT, 16, FORM, ST>;
    case 20: return k_refine_attend<GT, 20, FORM, ST>;
    case 24: return k_refine_attend<GT, 24, FORM, ST>;
    case 28: return k_refine_attend<GT, 28, FORM, ST>;
    case 32: return k_refine_attend<GT, 32, FORM, ST>;
    case -8: return k_refine_attend<GT, -8, FORM, ST>;
    default: return k_refine_attend<GT, -16, FORM, ST>;
    }
}
#define DS_DEFINE_DECODE_FN(GT)                                                                       \
    template <>                                                                                       \
    RaFn decode_fn<GT>(int smode, DecodeVariant v)                                                    \
    {                                                                                                 \
        if (v == DECODE_NARROW) return decode_fn_of<GT, 42, true>(smode);                             \
        if constexpr (GT <= 2) {                                                                      \
            if (v == DECODE_LIGHT) return decode_fn_of<GT, 84, false>(smode);                         \
            if (v == DECODE_DEEP) return decode_fn_of<GT, 84, true>(smode);                           \
        }                                                                                             \
        return decode_fn_of<GT, 82, true>(smode);                                                     \
    }
#ifdef DS_TRACE
#define DS_DEFINE_TRACE_READ(GT)                                                                      \
    template <>                                                                                       \
    int trace_read<GT>(void *dst, size_t bytes)                                                       \
    {                                                                                                 \
        return (int)hipMemcpyFromSymbol(dst, HIP_SYMBOL(g_trace), bytes, 0, hipMemcpyDeviceToHost);   \
    }
#else
#define DS_DEFINE_TRACE_READ(GT)
#endif

}  // namespace ds
