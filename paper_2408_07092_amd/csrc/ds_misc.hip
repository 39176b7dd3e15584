// Label-cache maintenance (Sec. 4.2), the host-row gather of the offload
// arrangement (Sec. 5.1) and the read-bandwidth probe.
#include <algorithm>
#include <cmath>

#include "ds_device.h"

namespace ds {

// The label values of K rows are picked by a fixed thread layout: thread tid takes channel j =
// tid mod r of the rows i0 = tid / r, i0 + P, i0 + 2 P, .. with P = 256 / r rows per pass (the last
// 256 - P r threads idle), so that its channel stays in a register and no element costs a division.
// A wavefront's load covers every line of 64 / r rows once.
struct PickLayout {
    int r, P;
    uint32_t inv;  // tid / r == tid * inv >> 16 for every thread of a workgroup and r <= 128
};
static PickLayout pick_layout(int r) { return {r, kWG / r, (65535u + (uint32_t)r) / (uint32_t)r}; }
struct PickLanes {
    int P, j, i0;
    bool on;
    __device__ __forceinline__ explicit PickLanes(const PickLayout &l)
    {
        P = l.P;
        i0 = (int)(threadIdx.x * l.inv >> 16);
        j = (int)threadIdx.x - i0 * l.r;
        on = i0 < P;
    }
};

// label[u, t, j] = K[u, t, channels[h, j]] for t in [t0, t0 + n): a bit copy, `per_wg` tokens to a
// workgroup (kv_stride halves from row to row: d, or 2d when each K row is followed by the
// token's V row); h = blockIdx.y, batch blockIdx.z.  Bound by the read of the K rows' lines: 512 MiB of K,
// 8 channels, in 94 us, where a bare read of them takes 80.  PICK passes of a thread are in flight (see
// launch_label for where one pass, without the streaming mark, is better than eight with it).
template <int PICK, bool ST>
__global__ __launch_bounds__(kWG) void k_label(const uint16_t *__restrict__ K,
                                               const int32_t *__restrict__ channels,
                                               uint16_t *__restrict__ label, int L_max,
                                               PickLayout pl, int t0, int n, int kv_stride, int per_wg)
{
    const PickLanes p(pl);
    if (!p.on) return;
    const int h = blockIdx.y, u = blockIdx.z * gridDim.y + h, r = pl.r;
    const int c = channels[h * r + p.j];
    const int lo = blockIdx.x * per_wg, hi = min(n, lo + per_wg);
    const uint16_t *Ku = K + ((size_t)u * L_max + t0) * kv_stride + c;
    uint16_t *lu = label + ((size_t)u * L_max + t0) * r + p.j;
    if constexpr (PICK == 1) {
        for (int i = lo + p.i0; i < hi; i += p.P) {
            const uint16_t *src = Ku + (size_t)i * kv_stride;
            lu[(size_t)i * r] = ST ? __builtin_nontemporal_load(src) : *src;
        }
        return;
    }
    for (int ib = lo; ib < hi; ib += PICK * p.P) {
        const int i = ib + p.i0;
        uint16_t x[PICK];
#pragma unroll
        for (int e = 0; e < PICK; ++e)
            if (ib + e * p.P < hi) {
                const uint16_t *src = Ku + (size_t)min(i + e * p.P, hi - 1) * kv_stride;
                x[e] = ST ? __builtin_nontemporal_load(src) : *src;
            }
#pragma unroll
        for (int e = 0; e < PICK; ++e)
            if (i + e * p.P < hi) lu[(size_t)(i + e * p.P) * r] = x[e];
    }
}

// Decode-step cache maintenance in one launch (Sec. 4.2: a decode step extends the label cache
// by the new tokens' r selected channels only): the n new tokens' K and V rows go into
// the caches at tokens [t0, t0 + n) and their r label values into the label cache.
// 16 lanes move one 256-byte row.  One token of one unit is all that a decode step has for a workgroup, so the
// launch is latency: channel ids and rows come in with one round trip, and the label values are picked
// out of the K rows in LDS.  (Ids, then rows, then the values out of memory again, found by 64-bit
// divisions: three round trips in a row.)
__global__ __launch_bounds__(kWG) void k_append_kv(const uint4 *__restrict__ k_new,
                                                   const uint4 *__restrict__ v_new, uint4 *K, uint4 *V,
                                                   const int32_t *__restrict__ channels,
                                                   uint16_t *__restrict__ label, int Hkv, int L_max,
                                                   int r, int t0, int n, int kv_stride16)
{
    __shared__ int ch_sh[kD];
    __shared__ __attribute__((aligned(16))) uint16_t rows_sh[16][kD];
    const int tid = threadIdx.x, u = blockIdx.y, h = u % Hkv;
    const int row = tid >> 4, p = tid & 15;
    int c = 0;
    if (tid < r) c = channels[h * r + tid];
    for (int i0 = blockIdx.x * 16; i0 < n; i0 += gridDim.x * 16) {
        const int m = min(16, n - i0);
        if (row < m) {
            const size_t src = ((size_t)u * n + i0 + row) * 16 + p;
            const size_t dst = ((size_t)u * L_max + t0 + i0 + row) * kv_stride16 + p;
            const uint4 k = k_new[src], v = v_new[src];
            *reinterpret_cast<uint4 *>(&rows_sh[row][p * 8]) = k;
            K[dst] = k;
            V[dst] = v;
        }
        if (tid < r) ch_sh[tid] = c;
        __syncthreads();
        uint16_t *lab = label + ((size_t)u * L_max + t0 + i0) * r;
        for (int e = tid; e < m * r; e += kWG) lab[e] = rows_sh[(uint32_t)e / (uint32_t)r][ch_sh[(uint32_t)e % (uint32_t)r]];
        __syncthreads();
    }
}

// ---------------------------------------------------------------- 4-bit label cache (Sec. 4.2)
// The paper says only that the label cache can be kept in 4 bits.  Quantiser used here:
// symmetric, one step per (unit, label channel), fixed at build time:
//   amax[u, j] = max_t |K[u, t, C[j]]|,  code = clamp(rint(x * (7 / amax)), -8, 7),
//   label value = code * (amax / 7); eight two's-complement nibbles per 32-bit word,
//   channel j of a token in bits [4 (j mod 8), +4) of the token's word j / 8.
// A binary16 magnitude orders like its 15 bits and widened to binary32 like those bits, so the
// maximum is an integer atomicMax (exact, order-free).
__device__ __forceinline__ uint32_t q4_code(float x, float inv)
{
    const float y = __builtin_rintf(x * inv);
    const int c = y < -8.0f ? -8 : (y > 7.0f ? 7 : (int)y);
    return (uint32_t)c & 0xfu;
}
__device__ __forceinline__ float q4_inverse(float amax) { return amax > 0.0f ? 7.0f / amax : 0.0f; }

__device__ __forceinline__ float q4_f16(uint16_t v) { return (float)__builtin_bit_cast(_Float16, v); }

// Largest magnitude of the thread's channel over its share of the rows [lo, hi), values to `keep`; eight
// passes of a thread in flight.  With the streaming mark at every size: plain loads take, cold, 1.04 to 1.11
// times as long from 64 MiB of K on with 8 or 16 channels (256 units of 8192 tokens 97 and 106 us; built again and
// again 0.97 to 1.14, just after K was written 0.98 to 1.12), 0.94 to 1.00 times below 32 MiB, 0.5 us at most;
// 64 channels 0.90 to 1.04.
template <class Keep>
__device__ __forceinline__ uint32_t q4_pick(const uint16_t *Kc, const PickLanes &p, int lo, int hi, Keep keep)
{
    constexpr int kPick = 8;
    uint32_t mx = 0u;
    if (p.on)
        for (int i = lo + p.i0; i < hi; i += kPick * p.P) {
            uint16_t x[kPick];
#pragma unroll
            for (int e = 0; e < kPick; ++e)
                x[e] = __builtin_nontemporal_load(Kc + (size_t)min(i + e * p.P, hi - 1) * kD);
#pragma unroll
            for (int e = 0; e < kPick; ++e) {
                mx = max(mx, (uint32_t)(x[e] & 0x7fffu));
                if (i + e * p.P < hi) keep(i + e * p.P, x[e]);
            }
        }
    return __float_as_uint(q4_f16((uint16_t)mx));
}

// Folds every thread's maximum into its channel's of mx_sh (after a barrier).  Powers of two: lanes a
// multiple of r apart hold the same channel, and a wavefront's are folded in registers first (one
// channel: 256 adds to one LDS word otherwise).
__device__ __forceinline__ void q4_fold_max(uint32_t mine, const PickLanes &p, int r, uint32_t *mx_sh)
{
    bool add = p.on;
    if (r <= 32 && (r & (r - 1)) == 0) {
        for (int d = 32; d >= r; d >>= 1) mine = max(mine, (uint32_t)__shfl_xor((int)mine, d));
        add = (threadIdx.x & 63) < (uint32_t)r;
    }
    if (add) atomicMax(&mx_sh[p.j], mine);
}

// Codes of the n tokens whose picked values are in tile_sh ([n][8 W]), words to cu[n][W]; a thread keeps
// its word of a token.  skip_first: token 0's first word is left alone.
__device__ __forceinline__ void q4_code_tile(const uint16_t *tile_sh, const float *inv_sh, int r, const PickLayout &words,
                                             int n, bool skip_first, uint32_t *cu)
{
    const PickLanes q(words);
    const int W = words.r;
    if (!q.on) return;
    for (int i = q.i0; i < n; i += q.P) {
        const half8 v = *reinterpret_cast<const half8 *>(tile_sh + (i * W + q.j) * 8);
        uint32_t word = 0u;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (q.j * 8 + k < r) word |= q4_code((float)v[k], inv_sh[q.j * 8 + k]) << (4 * k);
        if (i + q.j || !skip_first) cu[(size_t)i * W + q.j] = word;
    }
}

// Before k_q4_build and k_q4_amax: amax, and for k_q4_build every unit's counter word (its first word of
// codes), to zero.
__global__ __launch_bounds__(kWG) void k_q4_zero(uint32_t *amax, size_t n, uint32_t *codes, size_t unit_words,
                                                 int units)
{
    const size_t i0 = (size_t)blockIdx.x * kWG + threadIdx.x, step = (size_t)gridDim.x * kWG;
    for (size_t i = i0; i < n; i += step) amax[i] = 0u;
    for (size_t i = i0; i < (size_t)units; i += step) codes[i * unit_words] = 0u;
}

// Builds the 4-bit label cache with one read of the K rows, which bounds it (64 units of 16K tokens,
// 16 channels: 268 MB in 53 us; 32 of 32K 59, with two reads of the rows 86).  A workgroup picks the label values of its tile of
// tokens into LDS, adds its channel maxima to the unit's (amax), arrives at the unit's
// counter and waits for the unit's other workgroups; with the unit's maxima complete it codes the
// tile out of LDS.  The counter (arrivals in the low half, departures in the high half) is the
// unit's first word of codes: it is coded by the last workgroup to depart, when nobody looks
// at the counter any more.  A unit with one workgroup needs none of this: no k_q4_zero, no atomics.
// The wait: make_q4_plan lets workgroups wait only where the device holds a unit's several times over; a
// unit's workgroups are neighbours in the grid and start in grid order, so those that a workgroup
// waits for are running or next in line.  It is bounded all the same, and a workgroup
// whose wait runs out reads the unit's K rows itself for the maxima: slower, the same result.
// (Eight workgroups to a compute unit by registers, so that LDS alone decides how many it holds.)
__global__ __launch_bounds__(kWG, 8) void k_q4_build(const uint16_t *__restrict__ K,
                                                     const int32_t *__restrict__ channels, uint32_t *amax_bits,
                                                     uint32_t *codes, int L_max, PickLayout pl, PickLayout words,
                                                     int L, int tile, uint32_t spin_limit)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t tile_sh[];  // [tile][8 W] picked values
    __shared__ uint32_t mx_sh[kD];
    __shared__ float inv_sh[kD];
    __shared__ uint32_t s_ok, s_last;
    const int tid = threadIdx.x, h = blockIdx.y, u = blockIdx.z * gridDim.y + h, r = pl.r;
    const int W = words.r, stride = 8 * W;
    const PickLanes p(pl);
    const int c = p.on ? channels[h * r + p.j] : 0;
    if (tid < kD) mx_sh[tid] = 0u;
    const uint16_t *Ku = K + (size_t)u * L_max * kD + c;
    const int t0 = blockIdx.x * tile, t1 = min(L, t0 + tile);
    const uint32_t mine = q4_pick(Ku, p, t0, t1, [&](int t, uint16_t x) { tile_sh[(t - t0) * stride + p.j] = x; });
    __syncthreads();
    q4_fold_max(mine, p, r, mx_sh);
    __syncthreads();
    uint32_t *am = amax_bits + (size_t)u * r;
    uint32_t *cu = codes + (size_t)u * L_max * W;
    if (gridDim.x == 1) {
        if (tid < r) {
            am[tid] = mx_sh[tid];
            inv_sh[tid] = q4_inverse(__uint_as_float(mx_sh[tid]));
        }
        __syncthreads();
        q4_code_tile(tile_sh, inv_sh, r, words, t1, false, cu);
        return;
    }
    if (tid < r && mx_sh[tid]) atomicMax(&am[tid], mx_sh[tid]);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
        const uint32_t n_wg = gridDim.x;
        uint32_t ok = ((__hip_atomic_fetch_add(cu, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 0xffffu) + 1u == n_wg);
        for (uint32_t it = 0; !ok && it < spin_limit; ++it) {
            __builtin_amdgcn_s_sleep(1);
            ok = (ld_dev(cu) & 0xffffu) == n_wg;
        }
        s_ok = ok;
        const uint32_t left = __hip_atomic_fetch_add(cu, 1u << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 16;
        s_last = left + 1u == n_wg;
    }
    __syncthreads();
    if (!s_ok) {
        const uint32_t all = q4_pick(Ku, p, 0, L, [](int, uint16_t) {});
        q4_fold_max(all, p, r, mx_sh);
        __syncthreads();
        if (tid < r) inv_sh[tid] = q4_inverse(__uint_as_float(mx_sh[tid]));
    } else if (tid < r) {
        inv_sh[tid] = q4_inverse(__uint_as_float(ld_dev(am + tid)));
    }
    __syncthreads();
    q4_code_tile(tile_sh, inv_sh, r, words, t1 - t0, t0 == 0, cu + (size_t)t0 * W);
    if (s_last && tid == 0) {
        uint32_t word = 0u;
        for (int k = 0; k < 8 && k < r; ++k)
            word |= q4_code(q4_f16(Ku[channels[h * r + k] - c]), inv_sh[k]) << (4 * k);
        cu[0] = word;
    }
}

// The same with two reads of the K rows and nobody waiting: the channel maxima ...
__global__ __launch_bounds__(kWG) void k_q4_amax(const uint16_t *__restrict__ K, const int32_t *__restrict__ channels,
                                                 uint32_t *amax_bits, int L_max, PickLayout pl, int L, int per_wg)
{
    __shared__ uint32_t mx_sh[kD];
    const int tid = threadIdx.x, h = blockIdx.y, u = blockIdx.z * gridDim.y + h, r = pl.r;
    const PickLanes p(pl);
    const int c = p.on ? channels[h * r + p.j] : 0;
    if (tid < kD) mx_sh[tid] = 0u;
    const int lo = blockIdx.x * per_wg;
    const uint32_t mine = q4_pick(K + (size_t)u * L_max * kD + c, p, lo, min(L, lo + per_wg), [](int, uint16_t) {});
    __syncthreads();
    q4_fold_max(mine, p, r, mx_sh);
    __syncthreads();
    if (tid < r && mx_sh[tid]) atomicMax(&amax_bits[(size_t)u * r + tid], mx_sh[tid]);
}

// ... and the codes.
__global__ __launch_bounds__(kWG) void k_q4_code(const uint16_t *__restrict__ K, const int32_t *__restrict__ channels,
                                                 const float *__restrict__ amax, uint32_t *__restrict__ codes, int L_max,
                                                 PickLayout pl, PickLayout words, int L, int tile)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t tile_sh[];  // [tile][8 W] picked values
    __shared__ float inv_sh[kD];
    const int tid = threadIdx.x, h = blockIdx.y, u = blockIdx.z * gridDim.y + h, r = pl.r;
    const int W = words.r, stride = 8 * W;
    const PickLanes p(pl);
    const int c = p.on ? channels[h * r + p.j] : 0;
    if (tid < r) inv_sh[tid] = q4_inverse(amax[(size_t)u * r + tid]);
    const int t0 = blockIdx.x * tile, t1 = min(L, t0 + tile);
    q4_pick(K + (size_t)u * L_max * kD + c, p, t0, t1, [&](int t, uint16_t x) { tile_sh[(t - t0) * stride + p.j] = x; });
    __syncthreads();
    q4_code_tile(tile_sh, inv_sh, r, words, t1 - t0, false, codes + ((size_t)u * L_max + t0) * W);
}

// One thread per (token, word): up to eight codes packed into the word.
__global__ __launch_bounds__(kWG) void k_q4_write(const _Float16 *__restrict__ K,
                                                  const int32_t *__restrict__ channels,
                                                  const float *__restrict__ amax,
                                                  uint32_t *__restrict__ codes, int Hkv, int L_max,
                                                  int r, int t0, int n)
{
    __shared__ int ch_sh[kD];
    __shared__ float inv_sh[kD];
    const int u = blockIdx.y, h = u % Hkv;
    if (threadIdx.x < r) {
        ch_sh[threadIdx.x] = channels[h * r + threadIdx.x];
        inv_sh[threadIdx.x] = q4_inverse(amax[(size_t)u * r + threadIdx.x]);
    }
    __syncthreads();
    const int W = (r + 7) / 8;
    const size_t total = (size_t)n * W;
    for (size_t e = (size_t)blockIdx.x * kWG + threadIdx.x; e < total; e += (size_t)gridDim.x * kWG) {
        const size_t row = (size_t)u * L_max + t0 + e / W;
        const int w = (int)(e % W);
        uint32_t word = 0u;
        for (int i = 0; i < 8 && w * 8 + i < r; ++i)
            word |= q4_code((float)K[row * kD + ch_sh[w * 8 + i]], inv_sh[w * 8 + i]) << (4 * i);
        codes[row * W + w] = word;
    }
}

// ---------------------------------------------------------------- next-layer query prediction (Sec. 5.1)
// q_out[b, n] = sum_m Wq[n, m] * x[b, m], the shape of the step that turns a layer's input
// embedding into an approximate query of the NEXT layer so that its rows can be fetched early.
// Bound by the one read of Wq.  A wavefront owns an output feature n at a time: its 64 lanes
// split m in 16-byte pieces, products are exact (fp16 x fp16) and accumulated in binary32, the
// lanes are summed in a fixed butterfly, the result is rounded once to fp16.  Up to four batch
// rows share a pass over Wq (x sits in LDS); larger batches take several passes.
// Up to PIECES pieces of a row are in flight per lane and the first are asked for before x is staged (a
// piece of two rows in turn at a time: 4096 x 4096 11.6 us, now 8.4; 8192 x 8192 42, now 24).  PIECES goes by
// the row length (launch_predict_query); the order of the sums does not depend on it.
constexpr int kPredBatch = 4;

template <int PIECES, bool ST>
__global__ __launch_bounds__(kWG) void k_predict_query(const _Float16 *__restrict__ x,
                                                       const _Float16 *__restrict__ Wq,
                                                       _Float16 *__restrict__ q_out, int B, int Dm,
                                                       int N, int rows_per_wg)
{
    extern __shared__ __attribute__((aligned(16))) _Float16 x_sh[];  // [min(B, kPredBatch)][Dm]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_lo = blockIdx.x * rows_per_wg, n_hi = min(N, n_lo + rows_per_wg);
    half8 wv[PIECES];
    // (pieces past the end of the row re-read its last one; they are not used)
    auto issue = [&](int n, int m0) {
        const _Float16 *wrow = Wq + (size_t)min(n, N - 1) * Dm;
#pragma unroll
        for (int i = 0; i < PIECES; ++i)
            if (m0 - lane * 8 + i * 512 < Dm) {
                const half8 *src = reinterpret_cast<const half8 *>(wrow + min(m0 + i * 512, Dm - 8));
                wv[i] = ST ? __builtin_nontemporal_load(src) : *src;
            }
    };
    for (int b0 = 0; b0 < B; b0 += kPredBatch) {
        const int nb = min(kPredBatch, B - b0);
        issue(n_lo + wave, lane * 8);
        __syncthreads();
        for (int i = tid * 8; i < nb * Dm; i += kWG * 8)
            *reinterpret_cast<uint4 *>(x_sh + i) = *reinterpret_cast<const uint4 *>(x + (size_t)b0 * Dm + i);
        __syncthreads();
        for (int n = n_lo + wave; n < n_hi; n += 4) {
            float acc[kPredBatch] = {0.0f, 0.0f, 0.0f, 0.0f};
            for (int m0 = lane * 8; m0 - lane * 8 < Dm; m0 += 512 * PIECES) {
                if (m0 >= 512 * PIECES || n != n_lo + wave) issue(n, m0);
#pragma unroll
                for (int i = 0; i < PIECES; ++i) {
                    const int m = m0 + i * 512;
                    if (m >= Dm) continue;
#pragma unroll
                    for (int b = 0; b < kPredBatch; ++b) {
                        if (b < nb) {
                            const half8 xv = *reinterpret_cast<const half8 *>(x_sh + b * Dm + m);
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const half2v a2 = {wv[i][2 * e], wv[i][2 * e + 1]};
                                const half2v b2 = {xv[2 * e], xv[2 * e + 1]};
                                acc[b] = __builtin_amdgcn_fdot2(a2, b2, acc[b], false);
                            }
                        }
                    }
                }
            }
#pragma unroll
            for (int b = 0; b < kPredBatch; ++b) {
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) acc[b] += __shfl_xor(acc[b], o);
                if (lane == 0 && b < nb) q_out[(size_t)(b0 + b) * N + n] = (_Float16)acc[b];
            }
        }
    }
}

// rows[u, i, 0, :] = K_host[u, idx[u, i], :], rows[u, i, 1, :] = V_host[...]:
// 16 lanes move one 256-byte row; K_host / V_host are pinned host memory read
// over the host link by the kernel itself.  Bound by the link (about 55 GB/s), which 0.5 to 0.75 MiB
// of loads in flight keep full.  More in flight only fills the queues that the other streams'
// kernels share: with a workgroup for every 16 rows the query prediction of the next layer took
// 200 us beside the gather and the gather 340; with 64 workgroups 109 and 304, with 24 of them 33
// and 302, with 12 21 and 315 (alone: 20).
constexpr int kGatherRows = 4;   // rows of a 16-lane slot in flight
constexpr int kGatherWgs = 24;   // 24 x 16 slots x 4 rows of 512 bytes: 768 KiB
constexpr int kGatherFew = 512;  // up to this many rows: k_gather_few
// So few rows that their loads are all in flight anyway: a slot per row, nothing to divide or to loop
// over (8 units of 64 rows 7.4 us, with the loop 8.1; one of 16 2.7 and 2.9; from 1024 rows on the loop is
// faster, 12.1 against 13.2).
__global__ __launch_bounds__(kWG) void k_gather_few(const uint4 *__restrict__ Kh, const uint4 *__restrict__ Vh,
                                                    const int32_t *__restrict__ idx, uint4 *__restrict__ rows,
                                                    int L_max, int k)
{
    const int u = blockIdx.y;
    const int i = blockIdx.x * 16 + (threadIdx.x >> 4), p = threadIdx.x & 15;
    if (i >= k) return;
    const int tok = idx[(size_t)u * k + i];
    uint4 kv = make_uint4(0, 0, 0, 0), vv = kv;
    if (tok >= 0) {
        const size_t src = ((size_t)u * L_max + tok) * 16 + p;
        kv = Kh[src];
        vv = Vh[src];
    }
    const size_t dst = ((size_t)u * k + i) * 32 + p;
    rows[dst] = kv;
    rows[dst + 16] = vv;
}

__global__ __launch_bounds__(kWG) void k_gather_host(const uint4 *__restrict__ Kh,
                                                     const uint4 *__restrict__ Vh,
                                                     const int32_t *__restrict__ idx,
                                                     uint4 *__restrict__ rows, int L_max, int k, int total)
{
    const int p = threadIdx.x & 15, step = gridDim.x * 16;
    for (int i0 = blockIdx.x * 16 + (threadIdx.x >> 4); i0 < total; i0 += step * kGatherRows) {
        uint4 kv[kGatherRows], vv[kGatherRows];
#pragma unroll
        for (int e = 0; e < kGatherRows; ++e) {
            const int i = i0 + e * step;
            kv[e] = vv[e] = make_uint4(0, 0, 0, 0);
            const int tok = i < total ? idx[i] : -1;
            if (tok >= 0) {
                const size_t src = ((size_t)(i / k) * L_max + tok) * 16 + p;
                kv[e] = Kh[src];
                vv[e] = Vh[src];
            }
        }
#pragma unroll
        for (int e = 0; e < kGatherRows; ++e) {
            const int i = i0 + e * step;
            if (i >= total) break;
            rows[(size_t)i * 32 + p] = kv[e];
            rows[(size_t)i * 32 + p + 16] = vv[e];
        }
    }
}

// Plain streaming read: every workgroup reads 64 KiB as 16-byte loads marked as streaming (the
// mark is worth about 10 % on reads far larger than the caches), sixteen per thread in flight
// (eight leave about 8 % of the rate on the table).
constexpr int kProbeLoads = 16;
__global__ __launch_bounds__(kWG) void k_probe(const uint4 *__restrict__ src, size_t n16,
                                               uint32_t *sink)
{
    const size_t base = (size_t)blockIdx.x * (kWG * kProbeLoads) + threadIdx.x;
    uint4 v[kProbeLoads];
#pragma unroll
    for (int i = 0; i < kProbeLoads; ++i) {
        const size_t e = base + (size_t)i * kWG;
        v[i] = (e < n16) ? stream_load(src + e) : make_uint4(0, 0, 0, 0);
    }
    uint32_t x = 0;
#pragma unroll
    for (int i = 0; i < kProbeLoads; ++i) x ^= v[i].x ^ v[i].y ^ v[i].z ^ v[i].w;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x ^= __shfl_xor(x, o);
    if ((threadIdx.x & 63) == 0 && x != 0x9e3779b9u) atomicXor(&sink[blockIdx.x & 1023], x);
}

hipError_t launch_label(const void *K, const int32_t *channels, void *label, const ds_shape_t &s,
                        int t0, int n, hipStream_t st, int kv_stride)
{
    if (n <= 0) return hipSuccess;
    const PickLayout pl = pick_layout(s.r);
    // How many rows a workgroup takes, and how, goes by the size of the K rows.  Measured cold (several
    // K in turn), just after a kernel has written K (with that write), and with K built again and again, 1
    // to 512 units of 1 to 131072 tokens, 1 to 128 channels; us, cold where nothing else is said:
    // - One pass at a time and many workgroups, whose wavefronts hide the latency: until there are 4
    //   per compute unit below 48 MiB, 16 below 100, 64 above.  (Eight passes in flight and 4 workgroups:
    //   8 units of 8192 tokens, 64 channels 8.2 against 5.9; 32 of 32K, 24 channels 71 against 57, of which 66 with
    //   one pass but 4 workgroups; one unit of 128K, 24 channels 8.5 with 4 workgroups, 11.6 with 64.)
    // - From 200 MiB on and below 64 channels, eight passes in flight with the streaming mark (256 units
    //   of 8192, 24 channels 116 against 138; 32 of 32K, 8 channels 46 against 48, written just before 137
    //   against 156).  Below that the mark loses where the memory-side cache (256 MiB) holds K: 256 units of
    //   2500 tokens, 16 channels, built again 35 against 26; at 256 MiB still 45 against 42.
    const int64_t units = (int64_t)s.B * s.Hkv, bytes = units * n * kv_stride * 2, mib = 1 << 20;
    const bool stream = bytes >= 200 * mib && s.r < 64;
    const int64_t want = (bytes < 48 * mib ? 4ll : bytes < 100 * mib ? 16ll : 64ll) * device_caps().cus;
    const int round = (stream ? 8 : 1) * pl.P;
    int per_wg = round * std::max(1, 256 / round);
    while (per_wg > pl.P && units * ((n + per_wg - 1) / per_wg) < want) per_wg = (per_wg + 1) / 2;
    // (equal shares: 300 tokens in pieces of 256 would be one long and one short)
    const int n_wg = (n + per_wg - 1) / per_wg;
    per_wg = (n + n_wg - 1) / n_wg;
    const dim3 grid((n + per_wg - 1) / per_wg, s.Hkv, s.B);
    const auto *Kh = static_cast<const uint16_t *>(K);
    auto *lh = static_cast<uint16_t *>(label);
    if (stream)
        DS_LAUNCH(KID_LABEL, (k_label<8, true>), grid, dim3(kWG), 0, st, Kh, channels, lh, s.L_max, pl, t0, n, kv_stride, per_wg);
    else
        DS_LAUNCH(KID_LABEL, (k_label<1, false>), grid, dim3(kWG), 0, st, Kh, channels, lh, s.L_max, pl, t0, n, kv_stride, per_wg);
    return hipGetLastError();
}

void make_q4_plan(const ds_shape_t &s, Q4Plan *p)
{
    const DeviceCaps caps = device_caps();
    const int64_t units = (int64_t)s.B * s.Hkv, tokens = units * s.L;
    const int W = (s.r + 7) / 8, P = std::min(kWG / s.r, 32);  // rows of a pass (few channels: as far as it matters)
    const size_t token_lds = 16 * (size_t)W;
    const int most = (int)(kQ4TileLds / token_lds);            // tokens of the largest tile
    // One workgroup per unit: up to four rounds of eight passes, where one read of the rows by one
    // workgroup is over before several have met (us, 32 units: 300 tokens of 8 channels 8.9 -> 5.5, of 16 9.0 -> 6.4;
    // 1024 tokens of 8 channels 9.4 against 9.3; 500 of 24, six rounds, 1.27 times as long); all that fit the LDS when the
    // units fill the device (256 units of 2500 tokens, 8 channels 34.0 -> 31.9).
    if (s.L <= most && (s.L <= 32 * P || units >= caps.cus)) {
        *p = {1, s.L, 1, 0, 0};
        return;
    }
    // A workgroup's tile: its rounds of loads cost about 1.2 us each, its atomics on the unit's words 0.15 us
    // one after the other, and the sum is least at the root of tokens times rows of a pass -- half of that
    // on an idle device, more where other units' workgroups hide the rounds.  (0.5 / 1 / 2 / 4 times
    // as many tokens: 1.01 / 1.05 / 1.2 / 1.5 times the best below 50K tokens in all; 512 units of 500 to
    // 2500 tokens, 16 channels and more 1.7 / 1.15 / 1.0 / 1.1.)
    const double root = std::sqrt((double)s.L * P);
    const double share = tokens < 49152 ? 0.5 : units * 2 >= caps.cus ? 1.5 : 1.0;
    const int tile = std::min(most, std::max(4 * P, (int)(share * root)));
    const int n = (s.L + tile - 1) / tile;
    // One read and a wait for the unit's other workgroups, or two reads without.  The read that is saved
    // has to be worth the second counter and the atomics that queue on a unit's words (two reads
    // against one: 8 units of 8192 tokens 8 channels 11.9 against 11.6, 16 channels 11.9 against 12.8; 32 of
    // 8192 with 16 channels 26 against 20; with 128 channels, 64 workgroups of 128 atomics each, 46 against
    // 60; one unit of 32K, 8 channels 11 against 13).  And a device has to hold a unit's workgroups four times over, in each
    // of its dies: with that, calls on several streams at once, each with one unit partly started, all get on.
    const int held = (int)std::min<size_t>(8, (size_t)caps.lds_per_cu / (tile * token_lds + kQ4StaticLds));
    const int dies = std::max(1, caps.xccs);
    const bool fits = 4 * ((n + dies - 1) / dies) <= held * std::max(1, caps.cus / dies);
    if (units >= 4 && tokens >= (W == 1 ? 8192 : 49152) && n <= 128 && n * W <= 400 && fits) {
        const int even = (s.L + n - 1) / n;
        *p = {2, even, (s.L + even - 1) / even, 0, 0};
        return;
    }
    // Two reads.  The maxima by shares of half the root (no counter and no wait: atomics cost less; an
    // eighth / a quarter / half / once / twice: one unit of 32K tokens, 8 channels 12.0 / 10.7 / 11.1 / 13.4 / 17.6 us); the codes by a round of
    // eight passes, or four with 64 channels and more (512 units of 2500, 128 channels 1.16 times as long by one).
    const int per = std::min(s.L, std::max(4 * P, (int)(root / 2)));
    const int n_max = (s.L + per - 1) / per;
    int code = std::min(most, s.r >= 64 && tokens >= 60000 ? 32 * P : 8 * P);
    while ((s.L + code - 1) / code > (1 << 23) && code * 2 <= most) code *= 2;  // (grid limit: 2^32 threads)
    code = std::min(code, s.L);
    *p = {3, code, (s.L + code - 1) / code, per, n_max};
}

hipError_t launch_q4_build(const void *K, const int32_t *channels, float *amax, void *codes,
                           const ds_shape_t &s, hipStream_t st)
{
    const int W = (s.r + 7) / 8;
    const size_t n_amax = (size_t)s.B * s.Hkv * s.r;
    const PickLayout pl = pick_layout(s.r), words = pick_layout(W);
    const auto *Kh = static_cast<const uint16_t *>(K);
    auto *am = reinterpret_cast<uint32_t *>(amax), *cw = static_cast<uint32_t *>(codes);
    Q4Plan p;
    make_q4_plan(s, &p);
    const size_t lds = (size_t)p.tile * 16 * W;
    if (p.launches > 1)
        hipLaunchKernelGGL(k_q4_zero, dim3((unsigned)std::min<size_t>((n_amax + kWG - 1) / kWG, 1024)), dim3(kWG), 0, st,
                           am, n_amax, cw, (size_t)s.L_max * W, p.launches == 2 ? s.B * s.Hkv : 0);
    if (p.launches < 3) {
        DS_LAUNCH(KID_Q4_BUILD, k_q4_build, dim3(p.n_wg, s.Hkv, s.B), dim3(kWG), lds, st, Kh, channels, am, cw,
                  s.L_max, pl, words, s.L, p.tile, tune_get(5) ? (uint32_t)tune_get(5) : 1u << 14);
    } else {
        DS_LAUNCH(KID_Q4_AMAX, k_q4_amax, dim3(p.n_max, s.Hkv, s.B), dim3(kWG), 0, st, Kh, channels, am, s.L_max, pl,
                  s.L, p.per_wg);
        DS_LAUNCH(KID_Q4_CODE, k_q4_code, dim3(p.n_wg, s.Hkv, s.B), dim3(kWG), lds, st, Kh, channels,
                  static_cast<const float *>(amax), cw, s.L_max, pl, words, s.L, p.tile);
    }
    return hipGetLastError();
}

hipError_t launch_q4_write(const void *K, const int32_t *channels, const float *amax, void *codes,
                           const ds_shape_t &s, int t0, int n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const size_t total = (size_t)n * ((s.r + 7) / 8);
    size_t blocks = (total + kWG - 1) / kWG;
    if (blocks > 4096) blocks = 4096;
    DS_LAUNCH(KID_Q4_WRITE, k_q4_write, dim3((unsigned)blocks, s.B * s.Hkv), dim3(kWG), 0, st,
              static_cast<const _Float16 *>(K), channels, amax, static_cast<uint32_t *>(codes), s.Hkv,
              s.L_max, s.r, t0, n);
    return hipGetLastError();
}

hipError_t launch_predict_query(const void *x, const void *Wq, void *q_out, int B, int Dm, int N,
                                hipStream_t st)
{
    // a row per wavefront up to four workgroups per compute unit; every workgroup re-reads x once
    // per batch pass
    int rows_per_wg = (N + 1023) / 1024;
    rows_per_wg = (rows_per_wg + 3) & ~3;
    const int blocks = (N + rows_per_wg - 1) / rows_per_wg;
    const size_t shmem = (size_t)std::min(B, kPredBatch) * Dm * sizeof(_Float16);
    // Pieces in flight: all of a row of up to 2048 elements, where more code for a row than it has only
    // costs (512 x 512 2.85 us with one, 3.2 with eight), four up to 4096 (4096 x 4096 8.4, with eight 8.5; batch 8
    // 16.9 and 18.4), eight beyond (8192 x 8192 24.2 and 25.0).
    // The streaming mark where Wq is no small part of what the memory-side cache holds and is not read
    // over and over, once per four rows of a batch (8192 x 8192 24.2 us with it, 26.2 without, batch 8 68.7 and 70.9, batch
    // 64 493 and 485; 4096 x 4096 8.8 and 8.4, in the cache 6.0 and 5.2, batch 64 112 and 100).
    const bool mark = B <= 4 * kPredBatch && (size_t)N * Dm * 2 >= (64u << 20);
    auto go = [&](auto kernel) {
        DS_LAUNCH(KID_PREDICT, kernel, dim3((unsigned)blocks), dim3(kWG), shmem, st, static_cast<const _Float16 *>(x),
                  static_cast<const _Float16 *>(Wq), static_cast<_Float16 *>(q_out), B, Dm, N, rows_per_wg);
    };
    if (Dm > 4096) mark ? go(k_predict_query<8, true>) : go(k_predict_query<8, false>);
    else if (Dm > 1024) mark ? go(k_predict_query<4, true>) : go(k_predict_query<4, false>);
    else if (Dm > 512) mark ? go(k_predict_query<2, true>) : go(k_predict_query<2, false>);
    else mark ? go(k_predict_query<1, true>) : go(k_predict_query<1, false>);
    return hipGetLastError();
}

hipError_t launch_append_kv(const void *k_new, const void *v_new, void *K, void *V,
                            const int32_t *channels, void *label, const ds_shape_t &s, int t0, int n,
                            int kv_stride, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    size_t blocks = ((size_t)n + 15) / 16;
    if (blocks > 2048) blocks = 2048;
    DS_LAUNCH(KID_APPEND_KV, k_append_kv, dim3((unsigned)blocks, s.B * s.Hkv), dim3(kWG), 0, st,
              static_cast<const uint4 *>(k_new), static_cast<const uint4 *>(v_new),
              static_cast<uint4 *>(K), static_cast<uint4 *>(V), channels,
              static_cast<uint16_t *>(label), s.Hkv, s.L_max, s.r, t0, n, kv_stride / 8);
    return hipGetLastError();
}

hipError_t launch_gather_host(const void *Kh, const void *Vh, const int32_t *idx, void *rows,
                              const ds_shape_t &s, hipStream_t st)
{
    const int total = s.B * s.Hkv * s.k;
    if (total <= kGatherFew) {
        DS_LAUNCH(KID_GATHER_HOST, k_gather_few, dim3((s.k + 15) / 16, s.B * s.Hkv), dim3(kWG), 0, st,
                  static_cast<const uint4 *>(Kh), static_cast<const uint4 *>(Vh), idx, static_cast<uint4 *>(rows),
                  s.L_max, s.k);
        return hipGetLastError();
    }
    DS_LAUNCH(KID_GATHER_HOST, k_gather_host, dim3(std::min(kGatherWgs, (total + 15) / 16)), dim3(kWG), 0, st,
                       static_cast<const uint4 *>(Kh), static_cast<const uint4 *>(Vh), idx,
                       static_cast<uint4 *>(rows), s.L_max, s.k, total);
    return hipGetLastError();
}

hipError_t launch_probe(const void *src, size_t bytes, uint32_t *sink, hipStream_t st)
{
    const size_t n16 = bytes / 16;
    const size_t blocks = (n16 + kWG * kProbeLoads - 1) / (kWG * kProbeLoads);
    DS_LAUNCH(KID_PROBE, k_probe, dim3((unsigned)blocks), dim3(kWG), 0, st,
                       static_cast<const uint4 *>(src), n16, sink);
    return hipGetLastError();
}

}  // namespace ds
