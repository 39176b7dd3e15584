// Steps 3-5 of Algorithm 1 on gfx950: gather the selected K/V rows as whole
// 256-byte rows and run exact softmax attention over them; the same kernel body
// serves dense decode (all rows of a token chunk) and attention over rows that
// were gathered beforehand.
//
// Work split: one workgroup per (token chunk, unit).  A wavefront loads four
// rows per instruction -- 16 lanes x 16 bytes cover one row -- so each 16-lane
// group ("slot") owns a row at a time and keeps its own online-softmax state
// (running max m, denominator l, 8 output channels per lane).  The 16 slots of
// a workgroup are merged in a fixed order and written as one partial per chunk;
// the last workgroup of a unit to finish combines the chunk partials of its
// heads in a fixed order, so results are bit-reproducible whichever workgroup
// that happens to be.
// Logits are kept in the log2 domain: s2 = (q.k) * log2(e)/sqrt(d), p = 2^(s2-m).
#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>

#include "ds_device.h"

namespace ds {
DS_TRACE_BUFFER
}

#include "ds_decode_core.h"

namespace ds {


constexpr int kRowsPerSlot = 4;   // rows of a 16-lane slot in flight (2: -0.2 us on the 64K workload, 8: +0.5)
// ... on the vector path of the 256-thread variants: five, i.e. rounds of 80 rows.  A chunk of the
// 64K workload has 128 +- 11 selected rows; with rounds of 64 nearly half the workgroups run a
// third, almost empty round (31.1 -> 30.9 us/layer; batch 4 x 16K tokens 30.9 -> 30.5; six rows
// per slot: 31.4).
constexpr int kRowsPerSlotVector = 5;

// MODE 0: rows = tokens of the chunk that pass the selection predicate
// MODE 1: rows = all tokens of the chunk (dense)
// MODE 2: rows = pre-gathered [k][2][d] K|V pairs
template <int GT, int MODE>
__global__ __launch_bounds__(kWG, (GT == 1 ? 8 : 1)) void k_attend(AttendArgs a)
{
    extern __shared__ int sel[];  // ch words: selected tokens of the chunk (sparse mode only)
    __shared__ uint32_t s_w[4], s_flag;
    __shared__ __attribute__((aligned(16))) float red[8][kD];
    __shared__ float red_ml[8][2];
    __shared__ __attribute__((aligned(16))) _Float16 qsh[GT >= 4 ? 1 : GT][kD];
    __shared__ __attribute__((aligned(16))) float sc_sh[4][16];
    __shared__ __attribute__((aligned(16))) float wpart[4][GT][kPartStride];

    const int tid = threadIdx.x;
    const int u = blockIdx.y, c = blockIdx.x;
    const int b = u / a.Hkv, h = u % a.Hkv;
    const int t0 = c * a.ch;
    int n;
    DS_TR(0);
    if (MODE == 0) {
        const int t1 = min(a.L, t0 + a.ch);
        const uint32_t T = a.ctl[u].T;
        const int tcut = a.ctl[u].tcut;
        n = compact_selected(a.keys + (size_t)u * a.key_stride, t0, t1, T, tcut, sel, s_w);
        if (a.idx_out) {
            int32_t *io = a.idx_out + (size_t)u * a.k;
            const uint32_t off = a.offs[(size_t)u * a.n_ch + c];
            for (int i = tid; i < n; i += kWG)
                if (off + i < (uint32_t)a.k_eff) io[off + i] = sel[i];
            if (c == 0)
                for (int i = a.k_eff + tid; i < a.k; i += kWG) io[i] = -1;
        }
    } else if (MODE == 1) {
        n = min(a.L, t0 + a.ch) - t0;
    } else {
        n = min(a.n_rows, t0 + a.ch) - t0;
    }

    DS_TR(1);
    // unit base pointers are uniform; a row is addressed by a 32-bit byte offset from them
    const char *Ku, *Vu;
    uint32_t row_bytes;
    if (MODE == 2) {
        Ku = reinterpret_cast<const char *>(a.K + ((size_t)u * a.k + t0) * 2 * kD);
        Vu = Ku + kD * 2;
        row_bytes = 4 * kD;
    } else {
        Ku = reinterpret_cast<const char *>(a.K + (size_t)u * a.L_max * a.kv_stride);
        Vu = reinterpret_cast<const char *>(a.V + (size_t)u * a.L_max * a.kv_stride);
        row_bytes = 2 * a.kv_stride;
    }

    auto row_of = [&](int ri) { return (MODE == 0) ? sel[ri] : (MODE == 1) ? (t0 + ri) : ri; };
    const bool single = gridDim.x == 1;  // the unit's only workgroup writes the result itself
    for (int g0 = 0; g0 < a.G; g0 += GT) {
        float *po = a.part + (((size_t)u * a.G + g0) * a.n_ch + c) * kPartStride;
        float *od = single ? a.out + ((size_t)u * a.G + g0) * kD : nullptr;
        const _Float16 *q0 = a.q + ((size_t)b * a.Hq + (size_t)h * a.G + g0) * kD;
        __syncthreads();
        if constexpr (GT >= 4) {
            // query group on the matrix cores: up to GT heads share every gathered row
            const int n_heads = min(GT, a.G - g0);
            half8 qreg[4];
            load_q_mfma(q0, n_heads, qreg);
            MfmaState st;
            st.init();
            attend_rows_mfma(Ku, Vu, row_bytes, n, row_of, qreg, st, sc_sh[tid >> 6]);
            DS_TR(2);
            wg_store_partial_mfma<GT>(st, wpart, n_heads, po, (size_t)a.n_ch * kPartStride, od);
        } else {
            if (tid < GT * 16) {
                const int g = tid >> 4, p = tid & 15;
                *reinterpret_cast<uint4 *>(&qsh[g][p * 8]) = *reinterpret_cast<const uint4 *>(q0 + (size_t)g * kD + p * 8);
            }
            __syncthreads();
            RowState<GT> st;
            st.init();
            attend_rows<GT>(Ku, Vu, row_bytes, n, row_of, qsh, st);
            DS_TR(2);
            wg_store_partial<GT>(st, wpart, po, (size_t)a.n_ch * kPartStride, od);
        }
    }

    // ---- last workgroup of the unit: combine the chunk partials of every head of the group
    DS_TR(3);
    if (single) return;
    {
        const bool last = last_arrival(&a.ctl_rw[u].arrive_c, gridDim.x, &s_flag);
        DS_TR(4);
        if (!last) return;
    }
    if (tid == 0) a.ctl_rw[u].arrive_c = 0u;
    // (single heads: eight partials in flight do not fit the 64 registers that eight wavefronts per
    //  SIMD leave, 52 bytes a lane went to scratch; eight groups share a head's partials there anyway)
    merge_partials<(GT == 1 ? 4 : 8)>(a.part + (size_t)u * a.G * a.n_ch * kPartStride, a.G, a.n_ch,
                   a.out + (size_t)u * a.G * kD, red, red_ml, [](int, bool) {});
    DS_TR(5);
}


// ---------------------------------------------------------------- exact threshold + attention behind a scoring launch
// Runs after k_score has left the unit's keys and the threshold bin b* (with the
// rank krem of the k-th key inside it).  Tokens whose key lies in a bin above b*
// are selected whatever the exact threshold turns out to be, so a workgroup
//   1. splits its chunk's keys into definite tokens, candidates (bin b*) and the rest,
//      appends the candidates to the unit's list and arrives at the unit's counter;
//   2. attends the definite rows -- the bulk of the traffic -- straight away;
//   3. picks up the exact k-th key T and the tie cut, appends its selected
//      candidates and attends those;
//   4. writes its partial; the unit's last workgroup merges the partials.
// The workgroup whose arrival completes the unit radix-selects T from the
// candidate list before its own step 2 and publishes (T, tie cut, ready) as one
// 64-bit word, so the refinement hides behind the other workgroups' row traffic.
// Waiting: a workgroup waits only for the publishing workgroup, which is running
// by then and never waits itself; every workgroup of the unit arrives before
// any waits, and workgroups are dispatched in grid order, so all of a unit's
// workgroups get to run as long as one XCD can hold its share (every eighth) of
// the n_ch of them (checked on the host).  Every wait is bounded as well: on expiry the unit's
// error word is raised and the workgroup carries on with a value that keeps all accesses in range.
// (Label caches that the attention launch can score itself take decode_unit instead, see
// ds_decode_core.h.)
// (It serves units of several chunks, of which a scoring launch has many: up to 200 workgroups of a unit
//  meet less often here.  Where decode_unit takes the keys of the scoring launch with so many chunks, four
//  units of 200K tokens scored with 40 channels take 61 -> 82 us.)
template <int GT, bool ST>
__global__ __launch_bounds__(kWG, ST ? (GT == 1 ? 4 : 3) : 2) void k_attend_behind_scoring(AttendArgs a)
{
    constexpr int NW = 4, WGT = 64 * NW;
    extern __shared__ __attribute__((aligned(16))) uint32_t dyn_sh[];  // ch keys | ch 16-bit row list | n_ch counters
    uint32_t *keys_sh = dyn_sh;
    uint16_t *sel = reinterpret_cast<uint16_t *>(dyn_sh + a.ch);
    uint32_t *cnt = dyn_sh + a.ch + a.ch / 2;
    __shared__ uint32_t s_w[NW], s_flag, s_res[2], s_base, s_T[2], s_ok, s_cnt2;
    __shared__ float red_ml[8][2];
    __shared__ __attribute__((aligned(16))) _Float16 qsh[GT >= 4 ? 1 : GT][kD];
    __shared__ __attribute__((aligned(16))) float sc_sh[4][16];
    // 4 KiB serve the radix bins of the refinement, later the merge of the unit's partials; the
    // workgroup's own wavefront partials lie between the two in time and share the space when
    // they are at least that large
    __shared__ __attribute__((aligned(16))) float wpart[NW][GT][kPartStride];
    __shared__ __attribute__((aligned(16))) float red_own[GT >= 2 ? 1 : 8][kD];
    float(*red)[kD] = GT >= 2 ? reinterpret_cast<float(*)[kD]>(&wpart[0][0][0]) : red_own;
    uint32_t *lh = reinterpret_cast<uint32_t *>(&red[0][0]);  // 1024 radix bins

    const int tid = threadIdx.x;
    const int u = blockIdx.y + a.unit0, c = blockIdx.x;
    const int b = u / a.Hkv, h = u % a.Hkv;
    const int t0 = c * a.ch, t1 = min(a.L, t0 + a.ch);
    constexpr int kMaxPass = 8;                              // ch <= 8192
    const int n_pass = (t1 - t0 + WGT * 4 - 1) / (WGT * 4);  // <= kMaxPass
    const uint32_t *ku = a.keys + (size_t)u * a.key_stride;
    uint2 *cu = a.cand + (size_t)u * a.L;
    UnitCtl *ctl = a.ctl_rw + u;
    uint2 *ready = reinterpret_cast<uint2 *>(&ctl->cnt_a);  // {T, tie cut | 1<<31}
    unsigned long long *cand_arrive = reinterpret_cast<unsigned long long *>(&ctl->pad[2]);
    DS_TR(0);
    // A wait for another workgroup that ran out: the unit's error word is raised (it stays up until
    // the workspace is cleared) and the workgroup remembers it for its last arrival, so that the
    // workgroup that would merge the unit writes NaN instead.  A unit whose word is up when the
    // launch starts is not computed at all: its output is NaN again.
    // (One thread reads the word, which can go up at any time, and the whole workgroup goes by that copy.)
    __shared__ uint32_t s_failed, s_sticky;
    auto raise_err = [&](uint32_t code) {
        uint32_t none = 0u;  // (the unit's first code stays)
        __hip_atomic_compare_exchange_strong(&ctl->err, &none, code, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        s_failed = 1u;
    };
    auto poison_out = [&]() {
        float *ou = a.out + (size_t)u * a.G * kD;
        for (int i = tid; i < a.G * kD; i += WGT) ou[i] = __builtin_nanf("");
    };
    if (tid == 0) {
        s_failed = 0u;
        s_sticky = a.ctl[u].err;
    }

    if constexpr (GT <= 2) {
        if (tid < GT * 16) {
            const int g = tid >> 4, p = tid & 15;
            const _Float16 *q0 = a.q + ((size_t)b * a.Hq + (size_t)h * a.G) * kD;
            *reinterpret_cast<uint4 *>(&qsh[g][p * 8]) = *reinterpret_cast<const uint4 *>(q0 + (size_t)g * kD + p * 8);
        }
    }
    // ---- 1. the chunk's keys come from the scoring launch, with the unit's threshold bin;
    // all of the thread's key loads are in flight together; the keys then live in LDS
    const uint32_t bstar = ctl->bstar, krem_unit = ctl->krem;
    uint4 kv[kMaxPass];
#pragma unroll
    for (int p = 0; p < kMaxPass; ++p) {
        const int t = t0 + (p * WGT + tid) * 4;
        kv[p] = make_uint4(0u, 0u, 0u, 0u);
        if (p < n_pass && t < t1) kv[p] = *reinterpret_cast<const uint4 *>(ku + t);
    }
#pragma unroll
    for (int p = 0; p < kMaxPass; ++p) {
        const int lt = (p * WGT + tid) * 4;
        if (p < n_pass && t0 + lt < t1) *reinterpret_cast<uint4 *>(keys_sh + lt) = kv[p];
    }
    // ---- classify the chunk's keys against bin b*
    const uint32_t lo_key = bstar << kKeyShift;
    // own_keys(p): the thread's four keys of pass p (zeros past the end of the chunk)
    auto own_keys = [&](int p, uint32_t (&k4)[4]) {
        const int lt = (p * WGT + tid) * 4;
        k4[0] = k4[1] = k4[2] = k4[3] = 0u;
        if (t0 + lt < t1) {
            const uint4 v = *reinterpret_cast<const uint4 *>(keys_sh + lt);
            k4[0] = v.x; k4[1] = v.y; k4[2] = v.z; k4[3] = v.w;
        }
    };
    int n_def = 0;
    uint32_t n_cand = 0;
    uint32_t early_base = 0;  // (thread 0)
    // Each thread owns n_pass groups of four consecutive keys (group p of thread t: keys
    // 4 (p WGT + t) ..: a wavefront's loads then cover the LDS banks evenly).  One look at each key:
    // which of the thread's keys are definite and which are candidates goes into bit masks, and the
    // writes walk the set bits, few as they are.  Bit 4 p + e of a mask <-> key e of group p, at
    // this place in the chunk:
    auto key_slot = [&](int j) { return ((j >> 2) * WGT + tid) * 4 + (j & 3); };
    uint32_t mdef[2] = {0u, 0u}, mcan[2] = {0u, 0u};
    __syncthreads();  // the keys were stored by other threads
    if (s_sticky != 0u) {
        poison_out();  // (whichever workgroup leaves here: without it none of the unit's is the last, which would write)
        return;
    }
    {
        // Two groups are read at a time, whatever lies past the chunk's end among them, and the
        // masks cut to the chunk afterwards: no bounds in the loop, 32-bit masks at fixed places.
        // (Against a loop over the groups with bounds and 64-bit masks: units of 4K tokens 12.2 -> 11.7 us,
        //  128 units of 32K tokens in groups of 8 46.5 -> 45.7, of 4 with 4-bit labels 40.7 -> 39.8.)
        const uint32_t hi_key = lo_key | ((1u << kKeyShift) - 1u);
#pragma unroll
        for (int w = 0; w < 2; ++w) {
#pragma unroll
            for (int p2 = 0; p2 < 8; p2 += 2) {
                if (w * 8 + p2 >= n_pass) break;
                uint4 kq[2];
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    kq[i] = *reinterpret_cast<const uint4 *>(keys_sh + min(((w * 8 + p2 + i) * WGT + tid) * 4, a.ch - 4));
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const uint32_t k4[4] = {kq[i].x, kq[i].y, kq[i].z, kq[i].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t bit = 1u << ((p2 + i) * 4 + e);
                        mdef[w] |= k4[e] > hi_key ? bit : 0u;
                        mcan[w] |= k4[e] >= lo_key ? bit : 0u;
                    }
                }
            }
        }
        // (the groups before the last pass are whole, the last has what is left of the chunk)
        const int last = 4 * (n_pass - 1);
        const int left = min(max(t1 - t0 - (last * WGT + tid * 4), 0), 4);
        const unsigned long long live = ((1ull << last) << left) - 1ull;
        mdef[0] &= (uint32_t)live;
        mdef[1] &= (uint32_t)(live >> 32);
        mcan[0] &= (uint32_t)live & ~mdef[0];
        mcan[1] &= (uint32_t)(live >> 32) & ~mdef[1];
    }
    {
        const uint32_t packed = (uint32_t)(__builtin_popcount(mdef[0]) + __builtin_popcount(mdef[1])) |
                                (uint32_t)(__builtin_popcount(mcan[0]) + __builtin_popcount(mcan[1])) << 16;
        uint32_t total;
        const uint32_t ex = block_exclusive_scan<NW>(packed, s_w, &total);
        DS_TR(13);
        // the chunk's place in the unit's candidate list is fetched while the lists are written
        if (tid == 0 && (total >> 16))
            early_base = (uint32_t)__hip_atomic_fetch_add(cand_arrive, (unsigned long long)(total >> 16), __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_AGENT);
        n_def = (int)(total & 0xffffu);
        n_cand = total >> 16;
        // the definite rows from the front of the list, the candidates behind them; both in the
        // thread's key order
        int dpos = (int)(ex & 0xffffu);
        int cp = n_def + (int)(ex >> 16);
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            for (uint32_t m = mdef[w]; m; m &= m - 1u) sel[dpos++] = (uint16_t)key_slot(w * 32 + __builtin_ctz(m));
            for (uint32_t m = mcan[w]; m; m &= m - 1u) {
                sel[cp++] = (uint16_t)key_slot(w * 32 + __builtin_ctz(m));
            }
        }
    }
    // where the chunk's i-th candidate waits in the row list: behind the definite rows
    auto cand_slot = [&](uint32_t i) { return n_def + (int)i; };
    if (tid == 0) {
        // candidate count of the unit (low word) and arrivals (high word) share one 64-bit counter
        s_base = early_base;
        if (a.idx_out) st_dev(a.ndef + (size_t)u * a.n_ch + c, (uint32_t)n_def);
    }
    __syncthreads();
    // (a unit has L candidates at most; a base beyond that means the workspace was not cleared)
    const uint32_t base = s_base;
    if (base + n_cand <= (uint32_t)a.L) {
        for (uint32_t i = tid; i < n_cand; i += WGT) {
            const int lt = sel[cand_slot(i)];
            st_dev(cu + base + i, make_uint2(keys_sh[lt], (uint32_t)(t0 + lt)));
        }
    } else if (tid == 0) {
        raise_err(8u);
    }
    DS_TR(1);
    bool have_T = last_arrival_sum(cand_arrive, gridDim.x, &s_flag, &s_base);
    DS_TR(2);
    uint32_t T = 0;
    int tcut = 0x7fffffff;
    if (have_T) {
        // ---- the unit is complete: exact k-th key among the candidates (10 + 10 key bits), ties
        // to the lowest token (4 + 10 + 10 index bits; tokens are below 2^24).  The first 2048
        // candidates (eight per thread) stay in registers; what lies beyond is read again by every
        // pass, eight loads in flight.  (One load at a time, the 4400 candidates of a unit of 256K
        // tokens took 16.5 us of the launch's 55, and every workgroup of the unit waited for them.)
        const uint32_t n = min(s_base, (uint32_t)a.L);  // the completed count came with the arrival
        uint2 ce[8];
        auto read8 = [&](uint2 (&v)[8], uint32_t i0) {
#pragma unroll
            for (int x = 0; x < 8; ++x) v[x] = ld_dev(cu + min(i0 + (uint32_t)(x * WGT), n - 1));
        };
        if (n) read8(ce, tid);
        auto each = [&](auto f) {
#pragma unroll
            for (int x = 0; x < 8; ++x)
                if ((uint32_t)(tid + x * WGT) < n) f(ce[x]);
            for (uint32_t i0 = tid + 8u * WGT; i0 < n; i0 += 8u * WGT) {
                uint2 v[8];
                read8(v, i0);
#pragma unroll
                for (int x = 0; x < 8; ++x)
                    if (i0 + (uint32_t)(x * WGT) < n) f(v[x]);
            }
        };
        if (tid == 0) s_cnt2 = 0u;  // (pass 1 has barriers before its first use)
        DS_TR(8);
        uint32_t krem = krem_unit;
        bool settled = false;
        // Up to 256 candidates (short units, as a rule): one per thread, each counts the candidates
        // that sort before it -- key descending, token ascending -- out of LDS, sixteen per step;
        // the one with krem - 1 before it is the unit's k-th key, and its token is the tie cut.
        constexpr uint32_t kRankAll = 256;
        if (n >= 1u && n <= kRankAll) {
            // (key and inverted token as one 64-bit number: sorts before <=> larger; 0 for the rest)
            unsigned long long *s_c = reinterpret_cast<unsigned long long *>(lh);  // (2 KiB of the radix bins' 4)
            const uint2 me2 = ce[0];
            const unsigned long long me =
                (uint32_t)tid < n ? ((unsigned long long)me2.x << 32) | (unsigned long long)(0xffffffffu - me2.y) : 0ull;
            if (tid < (int)kRankAll) s_c[tid] = me;
            __syncthreads();
            if ((uint32_t)tid < n) {
                uint32_t before = 0;
                for (uint32_t j = 0; j < n; j += 16) {
                    unsigned long long o[16];
#pragma unroll
                    for (int e = 0; e < 16; ++e) o[e] = s_c[j + e];
#pragma unroll
                    for (int e = 0; e < 16; ++e) before += o[e] > me ? 1u : 0u;
                }
                if (before + 1u == krem) {
                    s_T[0] = me2.x;
                    s_T[1] = me2.y;
                }
            }
            __syncthreads();
            // (a rank beyond the list means a workspace that was not cleared: take the long way)
            if (krem >= 1u && krem <= n) {
                T = s_T[0];
                tcut = (int)s_T[1];
                settled = true;
            }
        }
        uint32_t pre22 = 0, n22 = 0xffffffffu;
        if (!settled) {
            svc_radix_pass<1024 / WGT, true, NW>(each, [](uint2) { return true; },
                                    [](uint2 e) { return (e.x >> 10) & 1023u; }, krem, lh, s_w, s_res);
            pre22 = (bstar << 10) | s_res[0];
            krem = s_res[1];
            n22 = lh[s_res[0]];  // candidates that share the k-th key's 22-bit prefix
            __syncthreads();
        }
        DS_TR(14);
        if (!settled && n22 <= 64u) {
            // One or two candidates as a rule: they are ranked among themselves by one wavefront,
            // in the order (key descending, token ascending); the one of rank krem is the unit's
            // k-th key, and its token is the tie cut.
            __shared__ uint2 s_small[64];
            each([&](uint2 e) {
                if ((e.x >> 10) == pre22) {
                    const uint32_t slot = atomicAdd(&s_cnt2, 1u);
                    if (slot < 64u) s_small[slot] = e;
                }
            });
            __syncthreads();
            const uint32_t m = min(s_cnt2, 64u);
            if (tid < 64 && (uint32_t)tid < m) {
                const uint2 mine = s_small[tid];
                uint32_t before = 0;
                for (uint32_t j = 0; j < m; ++j) {
                    const uint2 o = s_small[j];
                    before += (o.x > mine.x || (o.x == mine.x && o.y < mine.y)) ? 1u : 0u;
                }
                if (before + 1u == krem) {
                    s_T[0] = mine.x;
                    s_T[1] = mine.y;
                }
            }
            __syncthreads();
            // (counts that do not add up mean a workspace that was not cleared: take the long way)
            if (m == n22 && krem >= 1u && krem <= m) {
                T = s_T[0];
                tcut = (int)s_T[1];
                settled = true;
            }
        }
        if (!settled) {
            svc_radix_pass<1024 / WGT, true, NW>(each, [&](uint2 e) { return (e.x >> 10) == pre22; },
                                    [](uint2 e) { return e.x & 1023u; }, krem, lh, s_w, s_res);
            T = (pre22 << 10) | s_res[0];
            const uint32_t m_ties = s_res[1];
            const uint32_t n_ties = lh[s_res[0]];
            __syncthreads();
            if (m_ties < n_ties) {
                svc_radix_pass<1, false, NW>(each, [&](uint2 e) { return e.x == T; },
                                         [](uint2 e) { return (e.y >> 20) & 255u; }, m_ties, lh, s_w, s_res);
                uint32_t prefix = s_res[0], want = s_res[1];
                __syncthreads();
                svc_radix_pass<1024 / WGT, false, NW>(each, [&](uint2 e) { return e.x == T && (e.y >> 20) == prefix; },
                                         [](uint2 e) { return (e.y >> 10) & 1023u; }, want, lh, s_w, s_res);
                prefix = (prefix << 10) | s_res[0];
                want = s_res[1];
                __syncthreads();
                svc_radix_pass<1024 / WGT, false, NW>(each, [&](uint2 e) { return e.x == T && (e.y >> 10) == prefix; },
                                         [](uint2 e) { return e.y & 1023u; }, want, lh, s_w, s_res);
                tcut = (int)((prefix << 10) | s_res[0]);
                __syncthreads();
            }
        }
        if (a.idx_out) {
            // selected tokens per chunk = keys above b* + selected candidates; prefix -> offsets
            for (int i = tid; i < a.n_ch; i += WGT) cnt[i] = ld_dev(a.ndef + (size_t)u * a.n_ch + i);
            __syncthreads();
            each([&](uint2 e) {
                if (is_selected(e.x, (int)e.y, T, tcut)) atomicAdd(&cnt[e.y / (uint32_t)a.ch], 1u);
            });
            __syncthreads();
            const int per = (a.n_ch + WGT - 1) / WGT;
            const int c0 = min(a.n_ch, tid * per), c1 = min(a.n_ch, c0 + per);
            uint32_t sum = 0;
            for (int i = c0; i < c1; ++i) sum += cnt[i];
            uint32_t total;
            uint32_t run = block_exclusive_scan<NW>(sum, s_w, &total);
            for (int i = c0; i < c1; ++i) {
                st_dev(a.offs_rw + (size_t)u * a.n_ch + i, run);
                run += cnt[i];
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
        }
        DS_TR(15);
        if (tid == 0) {
            st_dev(ready, make_uint2(T, (uint32_t)tcut | 0x80000000u));
            __hip_atomic_store(cand_arrive, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        DS_TR(9);
    }

    // ---- 2..4 per pass over the query group
    const char *Ku = reinterpret_cast<const char *>(a.K + (size_t)u * a.L_max * a.kv_stride);
    const char *Vu = reinterpret_cast<const char *>(a.V + (size_t)u * a.L_max * a.kv_stride);
    const uint32_t row_bytes = 2 * a.kv_stride;
    int n_sel = 0;
    // First the definite rows that fill whole rounds of the workgroup's wavefronts (64 rows a round,
    // or 4 * RPS per wavefront on the vector path); the rest of them joins the selected candidates in one list, so
    // that at most one round of the workgroup runs partly empty.
    // (the variants for calls that move little data run on a mostly idle device, where a round
    //  trip is all that a round of rows costs: eight rows per slot in flight there)
    constexpr int kRowsInFlight = !ST ? 8 : GT > 2 ? kRowsPerSlot : kRowsPerSlotVector;
    constexpr int kRound = (GT >= 4) ? 64 : 4 * NW * kRowsInFlight;
    const int n_first = (n_def / kRound) * kRound;
    auto row_def = [&](int ri) { return t0 + (int)sel[ri]; };
    auto row_rest = [&](int ri) { return t0 + (int)sel[n_first + ri]; };
    // After the definite rows of the first pass: fetch (T, tie cut), append the selected candidates
    // to the row list and write the chunk's slice of the index list.
    auto settle = [&]() {
        if (!have_T) {
            if (tid == 0) {
                uint2 w = make_uint2(0u, 0u);
                uint32_t ok = 0;
                for (uint32_t it = 0; it < a.spin_limit; ++it) {
                    w = ld_dev(ready);
                    if (w.y & 0x80000000u) { ok = 1u; break; }
                    __builtin_amdgcn_s_sleep(1);
                }
                s_T[0] = w.x;
                s_T[1] = w.y & 0x7fffffffu;
                s_ok = ok;
                if (!ok) raise_err(6u);
            }
            __syncthreads();
            T = s_T[0];
            tcut = (int)s_T[1];
            if (!s_ok) { T = 0xffffffffu; tcut = -1; }  // nothing more is selected
            have_T = true;
        }
        DS_TR(4);
        const uint32_t off = a.idx_out ? ld_dev(a.offs_rw + (size_t)u * a.n_ch + c) : 0u;
        int32_t *io = a.idx_out ? a.idx_out + (size_t)u * a.k : nullptr;
        int all_base = 0;
        // the row list in thread-major order (any fixed order will do); an index list, if wanted,
        // is written in token order by the pass loop further down
        // The chunk's candidates -- already listed, behind the definite rows -- are all there is to
        // look at for the row list: one scan per 256 of them.  The selected ones close up to the
        // definite rows in place (a batch is read before it is written, and what it writes never
        // reaches the next batch).
        for (uint32_t c0 = 0; c0 < n_cand; c0 += WGT) {
            const uint32_t i = c0 + tid;
            int lt = 0;
            bool hit = false;
            if (i < n_cand) {
                lt = sel[cand_slot(i)];
                hit = is_selected(keys_sh[lt], t0 + lt, T, tcut);
            }
            uint32_t total;
            const uint32_t ex = block_exclusive_scan<NW>(hit ? 1u : 0u, s_w, &total);
            if (hit) sel[n_def + n_sel + (int)ex] = (uint16_t)lt;
            n_sel += (int)total;
        }
        // the chunk's slice of the index list, in token order: one scan per 1024 keys
        for (int p = 0; p < (io ? n_pass : 0); ++p) {
            const int lt = (p * WGT + tid) * 4;
            uint32_t k4[4];
            own_keys(p, k4);
            bool fs[4];
            uint32_t mine = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                fs[e] = (t0 + lt + e < t1) && is_selected(k4[e], t0 + lt + e, T, tcut);
                mine += fs[e] ? 1u : 0u;
            }
            uint32_t total;
            const uint32_t ex = block_exclusive_scan<NW>(mine, s_w, &total);
            uint32_t ap = off + (uint32_t)all_base + ex;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (fs[e]) {
                    if (ap < (uint32_t)a.k_eff) io[ap] = t0 + lt + e;
                    ++ap;
                }
            }
            all_base += (int)total;
        }
        if (io && c == 0)
            for (int i = a.k_eff + tid; i < a.k; i += WGT) io[i] = -1;
        __syncthreads();
    };

    for (int g0 = 0; g0 < a.G; g0 += GT) {
        float *po = a.part + (((size_t)u * a.G + g0) * a.n_ch + c) * kPartStride;
        const _Float16 *q0 = a.q + ((size_t)b * a.Hq + (size_t)h * a.G + g0) * kD;
        __syncthreads();
        if constexpr (GT >= 4) {
            const int n_heads = min(GT, a.G - g0);
            half8 qreg[4];
            load_q_mfma(q0, n_heads, qreg);
            MfmaState st;
            st.init();
            // (row loops at the lowest priority, hand-over sections at the highest: a workgroup
            //  that is still making its lists shares the compute unit with two that stream rows)
            DS_PRIO(0);
            attend_rows_mfma<false>(Ku, Vu, row_bytes, n_first, row_def, qreg, st, sc_sh[tid >> 6]);
            DS_PRIO(3);
            if (g0 == 0) { DS_TR(3); settle(); }
            DS_PRIO(2);
            attend_rows_mfma<false>(Ku, Vu, row_bytes, n_def - n_first + n_sel, row_rest, qreg, st, sc_sh[tid >> 6]);
            DS_PRIO(3);
            DS_TR(5);
            wg_store_partial_mfma<GT>(st, wpart, n_heads, po, (size_t)a.n_ch * kPartStride, nullptr);
        } else {
            // (the query rows have been in LDS since the kernel's first steps, barriers passed)
            RowState<GT> st;
            st.init();
            DS_PRIO(0);
            attend_rows<GT, kRowsInFlight, ST>(Ku, Vu, row_bytes, n_first, row_def, qsh, st);
            DS_PRIO(3);
            if (g0 == 0) { DS_TR(3); settle(); }
            DS_PRIO(2);
            attend_rows<GT, kRowsInFlight, ST>(Ku, Vu, row_bytes, n_def - n_first + n_sel, row_rest, qsh, st);
            DS_PRIO(3);
            DS_TR(5);
            wg_store_partial<GT, NW>(st, wpart, po, (size_t)a.n_ch * kPartStride, nullptr);
        }
    }

    // ---- last workgroup of the unit: merge the chunk partials, leave the control words clean
    {
        // (the arrival count in the low half of the word; a workgroup whose wait ran out adds a
        //  mark in the high half, which the last one to arrive sees without another load)
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
    }
    const bool unit_ok = s_ok != 0u;
    if (tid == 0) {
        ctl->arrive_c = 0u;
        ctl->cnt_a = 0u;
        ctl->cnt_b = 0u;
    }
    if (!unit_ok) {
        poison_out();
    } else {
        merge_partials<8>(a.part + (size_t)u * a.G * a.n_ch * kPartStride, a.G, a.n_ch,
                       a.out + (size_t)u * a.G * kD, red, red_ml, [](int, bool) {});
    }
    DS_TR(7);
}

// ---------------------------------------------------------------- launchers
static inline char *wsp(void *ws, size_t off) { return static_cast<char *>(ws) + off; }

// Heads handled per pass over the rows: 1 or 2 on the vector ALUs, 4 / 8 / 16 (padded) on the
// matrix cores; larger groups take several passes of 16.
static int pick_gt(int G)
{
    if (G <= 2) return G;
    if (G <= 4) return 4;
    if (G <= 8) return 8;
    return 16;
}

template <int MODE>
static void launch_attend_mode(int kid, const AttendArgs &a, dim3 grid, size_t shmem, hipStream_t st)
{
    switch (pick_gt(a.G)) {
    case 16: DS_LAUNCH(kid, (k_attend<16, MODE>), grid, dim3(kWG), shmem, st, a); break;
    case 8: DS_LAUNCH(kid, (k_attend<8, MODE>), grid, dim3(kWG), shmem, st, a); break;
    case 4: DS_LAUNCH(kid, (k_attend<4, MODE>), grid, dim3(kWG), shmem, st, a); break;
    case 2: DS_LAUNCH(kid, (k_attend<2, MODE>), grid, dim3(kWG), shmem, st, a); break;
    default: DS_LAUNCH(kid, (k_attend<1, MODE>), grid, dim3(kWG), shmem, st, a); break;
    }
}

hipError_t launch_attend_sparse(const void *q, const void *K, const void *V, void *ws, float *out,
                                int32_t *idx_out, const Plan &p, const ds_shape_t &s,
                                hipStream_t st, int kv_stride)
{
    AttendArgs a{};
    a.q = static_cast<const _Float16 *>(q);
    a.K = static_cast<const _Float16 *>(K);
    a.V = static_cast<const _Float16 *>(V);
    a.keys = reinterpret_cast<const uint32_t *>(wsp(ws, p.off_keys));
    a.ctl = reinterpret_cast<const UnitCtl *>(wsp(ws, p.off_ctl));
    a.ctl_rw = reinterpret_cast<UnitCtl *>(wsp(ws, p.off_ctl));
    a.out = out;
    a.offs = reinterpret_cast<const uint32_t *>(wsp(ws, p.off_offs));
    a.idx_out = idx_out;
    a.part = reinterpret_cast<float *>(wsp(ws, p.off_part));
    a.Hq = s.Hq; a.Hkv = s.Hkv; a.G = p.G; a.L = s.L; a.L_max = s.L_max;
    a.key_stride = p.key_stride; a.ch = p.ch; a.n_ch = p.n_ch; a.k = s.k; a.k_eff = p.k_eff;
    a.n_rows = 0;
    a.kv_stride = kv_stride;
    launch_attend_mode<0>(KID_ATTEND, a, dim3(p.n_ch, p.units), (size_t)p.ch * sizeof(int), st);
    return hipGetLastError();
}

// Whether the attention launch can take this plan's chunks: a workgroup keeps its chunk's keys in registers, or
// (several chunks per unit behind a scoring launch) loads them in at most eight passes of 1024.
bool refine_attend_ok(const Plan &p, bool scores_itself)
{
    return p.ch <= (scores_itself || p.n_ch == 1 ? kDecodeTokens : 8192) && (p.ch & 3) == 0;
}

// ---- the instantiation that serves a launch, by function pointer
struct RaKernel {
    RaFn fn;
    int threads;
    size_t shmem;
};

#ifdef DS_TRACE
static int g_last_decode = 0;
#endif

static RaFn decode_kernel(int gt, int smode, DecodeVariant v)
{
    switch (gt) {
    case 16: return decode_fn<16>(smode, v);
    case 8: return decode_fn<8>(smode, v);
    case 4: return decode_fn<4>(smode, v);
    case 2: return decode_fn<2>(smode, v);
    default: return decode_fn<1>(smode, v);
    }
}

// smode: 0 = keys and threshold bin come from the scoring launch; 4 .. 32 = fp16 labels of that
// many channels scored here; -8 / -16 = 4-bit labels of up to that many channels scored here.
static RaKernel ra_kernel(const Plan &p, const ds_shape_t &s, int smode)
{
    const int gt = pick_gt(p.G);
    if (smode == 0 && p.n_ch > 1) {
        const bool st = decode_bytes(p, s) >= kStreamBytes;
        const size_t shmem = (size_t)p.ch * 6 + (size_t)p.n_ch * 4;
        switch (gt) {
        case 16: return {k_attend_behind_scoring<16, true>, kWG, shmem};
        case 8: return {k_attend_behind_scoring<8, true>, kWG, shmem};
        case 4: return {k_attend_behind_scoring<4, true>, kWG, shmem};
        case 2: return {st ? k_attend_behind_scoring<2, true> : k_attend_behind_scoring<2, false>, kWG, shmem};
        default: return {st ? k_attend_behind_scoring<1, true> : k_attend_behind_scoring<1, false>, kWG, shmem};
        }
    }
    const DecodeVariant v = decode_variant(p, s);
    return {decode_kernel(gt, smode, v), v == DECODE_NARROW ? 256 : 512, (size_t)(p.ch + 7) / 8 * 16};
}

// 0 when the labels cannot be scored in the attention launch
static int ra_smode(const ds_shape_t &s, bool scores_itself, bool q4)
{
    if (!scores_itself) return 0;
    if (q4) return (s.r > 16 || (s.L_max & (s.r > 8 ? 1 : 3))) ? 0 : (s.r > 8 ? -16 : -8);
    return attend_scores_r(s.r) ? s.r : 0;
}

// What the runtime says of a kernel, asked once per (kernel, dynamic LDS): more than 64 KiB of
// dynamic LDS has to be granted first (all that the compute unit has beyond the kernel's static
// arrays); then the number of its workgroups that one compute unit holds at a time.
static int ra_workgroups_per_cu(const RaKernel &k, const DeviceCaps &caps)
{
    const size_t shmem = k.shmem;
    struct Key {
        const void *fn;
        size_t shmem;
        int dev;
        bool operator<(const Key &o) const { return std::tie(fn, shmem, dev) < std::tie(o.fn, o.shmem, o.dev); }
    };
    static std::mutex mu;
    static std::map<Key, int> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    const void *fn = reinterpret_cast<const void *>(k.fn);
    std::lock_guard<std::mutex> lk(mu);
    const Key key{fn, shmem, dev};
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    int per_cu = 0;
    bool ok = true;
    if (shmem > (64u << 10)) {
        hipFuncAttributes fa;
        ok = hipFuncGetAttributes(&fa, fn) == hipSuccess;
        const int room = ok ? caps.lds_per_cu - (int)fa.sharedSizeBytes : 0;
        ok = ok && (size_t)room >= shmem &&
             hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, room) == hipSuccess;
    }
    if (ok && hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, k.threads, shmem) != hipSuccess) per_cu = 0;
    if (!ok) per_cu = 0;
    (void)hipGetLastError();
    cache[key] = per_cu;
    return per_cu;
}

// Whether the device holds, at the same time, all the workgroups that a launch of this plan lets
// wait for each other.  A launch that scores as well waits (for its unit's histogram) for
// workgroups that may not have started: the whole grid has to be resident.  After a scoring
// launch a workgroup waits only for one that is running; workgroups start in grid order and are
// dealt out to the dies in turn, so one die has to hold its share of a unit's workgroups.  A unit
// with a single workgroup waits for nobody.
static bool ra_fits(const RaKernel &k, const Plan &p, int smode)
{
    const DeviceCaps caps = device_caps();
    const int per_cu = ra_workgroups_per_cu(k, caps);
    if (per_cu < 1) return false;
    if (p.n_ch == 1) return true;
    if (smode != 0) return (int64_t)p.n_ch * ((p.units + p.unit_groups - 1) / p.unit_groups) <= (int64_t)per_cu * caps.cus;
    const int dies = std::max(1, caps.xccs);
    return (p.n_ch + dies - 1) / dies <= per_cu * std::max(1, caps.cus / dies);
}

bool refine_attend_fits(const Plan &p, const ds_shape_t &s, bool scores_itself, bool q4)
{
    const int smode = ra_smode(s, scores_itself, q4);
    if (scores_itself && smode == 0) return false;
    return ra_fits(ra_kernel(p, s, smode), p, smode);
}

// score_label: non-null to run the scoring in the same launch (fp16 labels of as many channels as
// attend_scores_r allows; with amax the 4-bit label cache of up to 16 channels, whose token rows
// must be 16-byte loadable: L_max % 4 == 0 for one word per token, L_max % 2 == 0 for two);
// otherwise the keys of a preceding k_score launch are read from the workspace.  channels and amax are
// those of the label query either way.  kNotResident, with nothing enqueued, when the device cannot
// hold the workgroups that would wait for each other.
hipError_t launch_refine_attend(const void *q, const void *K, const void *V, void *ws, float *out,
                                int32_t *idx_out, const Plan &p, const ds_shape_t &s, hipStream_t st,
                                int kv_stride, const int32_t *channels, const float *amax, const void *score_label)
{
    AttendArgs a{};
    a.q = static_cast<const _Float16 *>(q);
    a.K = static_cast<const _Float16 *>(K);
    a.V = static_cast<const _Float16 *>(V);
    a.keys = reinterpret_cast<const uint32_t *>(wsp(ws, p.off_keys));
    a.ctl = reinterpret_cast<const UnitCtl *>(wsp(ws, p.off_ctl));
    a.ctl_rw = reinterpret_cast<UnitCtl *>(wsp(ws, p.off_ctl));
    a.out = out;
    a.cand = reinterpret_cast<uint2 *>(wsp(ws, p.off_cand));
    a.ndef = reinterpret_cast<uint32_t *>(wsp(ws, p.off_ndef));
    a.offs = reinterpret_cast<const uint32_t *>(wsp(ws, p.off_offs));
    a.offs_rw = reinterpret_cast<uint32_t *>(wsp(ws, p.off_offs));
    a.idx_out = idx_out;
    a.part = reinterpret_cast<float *>(wsp(ws, p.off_part));
    a.Hq = s.Hq; a.Hkv = s.Hkv; a.G = p.G; a.L = s.L; a.L_max = s.L_max;
    a.key_stride = p.key_stride; a.ch = p.ch; a.n_ch = p.n_ch; a.k = s.k; a.k_eff = p.k_eff;
    a.spin_limit = tune_get(5) ? (uint32_t)tune_get(5) : 1u << 21;
    a.kv_stride = kv_stride;
    a.label = static_cast<const _Float16 *>(score_label);
    a.channels = channels;
    a.hist = reinterpret_cast<uint32_t *>(wsp(ws, p.off_hist));
    a.coarse = reinterpret_cast<uint32_t *>(wsp(ws, p.off_coarse));
    a.amax = amax;
    a.r = s.r;
    a.k_share = (float)p.k_eff / (float)s.L;
    const int smode = ra_smode(s, score_label != nullptr, amax != nullptr);
    if (score_label && smode == 0) return hipErrorInvalidValue;
    const RaKernel k = ra_kernel(p, s, smode);
    if (!ra_fits(k, p, smode)) return kNotResident;
#ifdef DS_TRACE
    g_last_decode = smode != 0 || p.n_ch == 1 ? pick_gt(p.G) : 0;
#endif
    // (a launch that scores as well may take a share of the units at a time: see make_plan)
    const int groups = smode != 0 ? std::max(1, p.unit_groups) : 1;
    const int per_group = (p.units + groups - 1) / groups;
    for (int u0 = 0; u0 < p.units; u0 += per_group) {
        a.unit0 = u0;
        const dim3 grid(p.n_ch, std::min(per_group, p.units - u0)), block(k.threads);
        void *args[] = {&a};
        hipEvent_t ev_a = nullptr, ev_b = nullptr;
        hipError_t e;
        if (prof_events(KID_REFINE_ATTEND, &ev_a, &ev_b))
            e = hipExtLaunchKernel(reinterpret_cast<const void *>(k.fn), grid, block, args, k.shmem, st, ev_a, ev_b, 0);
        else
            e = hipLaunchKernel(reinterpret_cast<const void *>(k.fn), grid, block, args, k.shmem, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_attend_dense(const void *q, const void *K, const void *V, void *ws, float *out,
                               const DensePlan &p, const ds_shape_t &s, hipStream_t st)
{
    AttendArgs a{};
    a.q = static_cast<const _Float16 *>(q);
    a.K = static_cast<const _Float16 *>(K);
    a.V = static_cast<const _Float16 *>(V);
    a.part = reinterpret_cast<float *>(wsp(ws, p.off_part));
    a.ctl_rw = reinterpret_cast<UnitCtl *>(wsp(ws, p.off_ctl));
    a.out = out;
    a.Hq = s.Hq; a.Hkv = s.Hkv; a.G = p.G; a.L = s.L; a.L_max = s.L_max;
    a.ch = p.ch; a.n_ch = p.n_ch;
    a.kv_stride = kD;
    launch_attend_mode<1>(KID_DENSE, a, dim3(p.n_ch, p.units), 0, st);
    return hipGetLastError();
}

hipError_t launch_attend_rows(const void *q, const void *KV_rows, void *ws, float *out,
                              const DensePlan &p, const ds_shape_t &s, int n_rows, hipStream_t st)
{
    AttendArgs a{};
    a.q = static_cast<const _Float16 *>(q);
    a.K = static_cast<const _Float16 *>(KV_rows);
    a.V = nullptr;
    a.part = reinterpret_cast<float *>(wsp(ws, p.off_part));
    a.ctl_rw = reinterpret_cast<UnitCtl *>(wsp(ws, p.off_ctl));
    a.out = out;
    a.Hq = s.Hq; a.Hkv = s.Hkv; a.G = p.G; a.L = s.L; a.L_max = s.L_max;
    a.ch = p.ch; a.n_ch = p.n_ch; a.k = s.k; a.n_rows = n_rows;
    launch_attend_mode<2>(KID_ATTEND_ROWS, a, dim3(p.n_ch, p.units), 0, st);
    return hipGetLastError();
}

}  // namespace ds

#ifdef DS_TRACE
// the stamps of the last decode launch that scored itself, or else of this file's kernels
extern "C" int ds_trace_read_attend(void *dst, size_t bytes)
{
    switch (ds::g_last_decode) {
    case 16: return ds::trace_read<16>(dst, bytes);
    case 8: return ds::trace_read<8>(dst, bytes);
    case 4: return ds::trace_read<4>(dst, bytes);
    case 2: return ds::trace_read<2>(dst, bytes);
    case 1: return ds::trace_read<1>(dst, bytes);
    default: return (int)hipMemcpyFromSymbol(dst, HIP_SYMBOL(ds::g_trace), bytes, 0, hipMemcpyDeviceToHost);
    }
}
#endif
