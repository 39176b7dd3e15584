// C-ABI layer of libdsattn: argument validation, launch plans / workspace
// layout, the host-side offline calibration and the per-kernel event timing.
// No kernel code lives here; every device step is enqueued through the
// launchers declared in ds_internal.h.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <vector>

#include <hip/hip_runtime.h>

#include "ds_internal.h"

// Scratch of ds_sparse_decode_static: device memory that the library itself holds, one copy per
// GPU from the moment the code object is loaded there until the process ends.  In host code the
// array's name is only a handle for hipGetSymbolAddress; kernels get the resolved address.
#define DS_STATIC_SCRATCH_BYTES (32u << 20)
static __device__ __align__(256) unsigned char scratch[DS_STATIC_SCRATCH_BYTES];

namespace ds {

// ---------------------------------------------------------------- knobs
// (process-wide, for sweeps and tests; atomic so that a set in one thread and plans made in
//  another do not race -- a plan reads each knob once)
static std::atomic<int> g_tune[6];
int tune_get(int knob) { return (knob >= 0 && knob < 6) ? g_tune[knob].load(std::memory_order_relaxed) : 0; }

// ---------------------------------------------------------------- device
static thread_local const DeviceCaps *t_pretend = nullptr;
static thread_local DeviceCaps t_pretend_caps;

void device_caps_pretend(const DeviceCaps *caps)
{
    if (caps) {
        t_pretend_caps = *caps;
        t_pretend = &t_pretend_caps;
    } else {
        t_pretend = nullptr;
    }
}

DeviceCaps device_caps()
{
    if (t_pretend) return *t_pretend;
    static std::mutex mu;
    static DeviceCaps cache[64];
    static bool have[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        (void)hipGetLastError();  // no device: the plan of an MI355X
        return DeviceCaps();
    }
    std::lock_guard<std::mutex> lk(mu);
    if (!have[dev]) {
        DeviceCaps c;
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) c.cus = v;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeNumberOfXccs, dev) == hipSuccess && v > 0) c.xccs = v;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) == hipSuccess && v > 0)
            c.lds_per_cu = v;
        (void)hipGetLastError();
        cache[dev] = c;
        have[dev] = true;
    }
    return cache[dev];
}

// ---------------------------------------------------------------- plans
static size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

static bool shape_ok(const ds_shape_t &s, bool need_rk)
{
    if (s.B < 1 || s.Hq < 1 || s.Hkv < 1 || s.d != kD) return false;
    if (s.Hq % s.Hkv != 0) return false;
    if (s.L < 1 || s.L > s.L_max) return false;
    if (need_rk && (s.r < 1 || s.r > s.d || s.k < 1)) return false;
    if ((int64_t)s.B * s.Hkv > 65535) return false;  // units ride on gridDim.y
    if ((int64_t)s.L_max * kD * 2 > 0xffffffffll) return false;  // rows are addressed by 32-bit byte offsets
    if (need_rk && (int64_t)std::min(s.k, s.L) * kD * 4 > 0xffffffffll) return false;
    return true;
}

// Workspace of a decode that scores itself with several workgroups per unit: room for the partials and counters of
// as many chunks as this many tokens make, which is also the most that choose_chunks may pick.  What a caller sees
// of it is ds_workspace_bytes and which shapes the static scratch takes, so it is a rule by itself and not
// the number that the launch ends up with: chunks for w = 4 workgroups to a compute unit (groups of three heads and
// more: 3), or fewer, until w times 6 bytes a token and about 26 KiB (groups: the wavefronts' partials) are within the
// compute unit's LDS; in up to four shares of the units where even one workgroup each is too many.
// 0: no such number; the room is then that of the chunks behind a scoring launch.
static int room_chunk(int units, int L, int G, const DeviceCaps &caps)
{
    const bool single = G <= 2;
    const int gt = G <= 4 ? 4 : G <= 8 ? 8 : 16;
    const size_t fixed = single ? 26u << 10 : 512 + 3072 + 4 * (size_t)std::max(kHistBins, 4 * gt * kPartStride);
    for (int g = 1; g <= 4; ++g) {
        const int units_g = (units + g - 1) / g;
        for (int w = single ? 4 : 3; w >= 1; --w) {
            const int n = std::min((caps.cus * w) / units_g, kMaxChunks);
            if (n < (single ? 2 : 1)) continue;
            const int c = std::max(single ? 1024 : 2048, (((L + n - 1) / n) + 63) & ~63);
            const size_t lds = (size_t)c * 6 + (size_t)((L + c - 1) / c) * 4 + fixed;
            if (c <= (single ? 16384 : 8192) && lds * w <= (size_t)caps.lds_per_cu) return c;
        }
    }
    return 0;
}

// Chunks of a decode launch that scores itself with several workgroups per unit, whose whole grid has to be
// resident: two workgroups of 512 threads to a compute unit by registers and LDS; for groups of more than
// eight heads, whose kernels take more registers, one, or three of 256 threads and half the tokens.
// The number of chunks per unit with the least estimated time, and in how many launches of a share of the units each:
//   - the busiest compute unit's tokens, scored and their rows attended: about 53 GB/s (48 bytes a token with 8
//     channels and a sixteenth of the rows: 0.9 us a thousand) by one workgroup, 61 by two, whose idle
//     stretches fill each other's (128 single heads of 32K tokens 43.6 us with one, 42.8 with two; 96 of 30K, one
//     35.7, two 32.1; but 32 of 64K 26.9 and 28.3);
//   - 0.25 us for each of a unit's workgroups, which meet at the same few lines of memory (one unit of 256K tokens
//     39.7 us with 256 chunks, 28.0 with 128, 21.9 with 64; 32 units of 16K 21.7 with 2, 18.5 with 4, 17.7 with 8,
//     20.8 with 16);
//   - 10 us for every launch.
// At most n_room chunks, for which the workspace has room.
static bool choose_chunks(int units, int L, int G, double token_bytes, int cus, int n_room, int *ch, int *groups)
{
    const double us = std::max(0.5e-3, token_bytes * 0.01875e-3);
    // (more than one is measured on a whole MI355X only: a part of one plans one)
    const int per_cu = cus < 128 ? 1 : G > 8 ? 3 : 2;
    double best = 0.0;
    bool found = false;
    for (int g = 1; g <= 3; ++g) {
        const int u = (units + g - 1) / g, n_max = std::min(n_room, per_cu * cus / u);
        const int n0 = std::max(2, (L + kDecodeTokens - 1) / kDecodeTokens);
        for (int n = n0; n <= std::min(n_max, n0 + 64); ++n) {
            const int c = (((L + n - 1) / n) + 63) & ~63, n_ch = (L + c - 1) / c;
            const int on_cu = (int)(((int64_t)u * n_ch + cus - 1) / cus);
            if (c > (G > 8 && on_cu > 1 ? kDecodeTokens / 2 : kDecodeTokens)) continue;
            const double cost = g * (10.0 + c * us * (on_cu == 1 ? 1.0 : on_cu == 2 ? 1.73 : 2.5) + 0.25 * n_ch);
            if (!found || cost < best) {
                best = cost;
                *ch = c;
                *groups = g;
                found = true;
            }
        }
    }
    return found;
}

// (4-bit labels, a quarter of it or a half, are counted as if they were fp16: the lines of decode_variant lie better for
//  them that way.  With their own size, 120 random shapes of 16 to 44 MiB lost the streaming mark and took 1.01 of the
//  time, 0.89 to 1.06; nine with few units 0.985.)
size_t decode_bytes(const Plan &p, const ds_shape_t &s)
{
    return (size_t)p.units * ((size_t)s.L * s.r * 2 + (size_t)p.k_eff * 2 * kD * 2);
}

// The variant of the attention kernel.
//   - 256 threads where single-workgroup units outnumber two to a compute unit (groups of more than eight heads:
//     one), of which four fit at once (1024 single heads of 1000 tokens 16.8 us with 512 threads, 12.9 with 256; of
//     2048 22.5 and 19.8; 256 units of 1000 7.7 and 7.8);
//   - single heads and pairs, one workgroup per unit and units for less than three quarters of the device: four
//     rows per slot in flight instead of two (128 units of 6000 tokens 14.5 -> 13.8 us, of 8192 18.0 -> 17.0; 256 of 8192
//     22.4 -> 22.9);
//   - without the streaming mark below 16 MiB, and where so few units read less than 32 MiB, of which the memory-side
//     cache holds several layers (eight layers of 128 units of 4096 tokens 12.4 -> 11.0 us a layer, of 64 of 6144 13.2 ->
//     11.6; 128 of 6000 14.0 either way; 160 of 6144 14.8 -> 15.6, 128 of 8192 17.0 -> 17.9).
DecodeVariant decode_variant(const Plan &p, const ds_shape_t &s)
{
    const int64_t wgs = (int64_t)p.n_ch * ((p.units + p.unit_groups - 1) / p.unit_groups);
    if (wgs > (p.G > 8 ? 1 : 2) * (int64_t)p.cus && p.ch <= kDecodeTokens / 2) return DECODE_NARROW;
    const size_t bytes = decode_bytes(p, s);
    const bool few = p.n_ch == 1 && (int64_t)p.units * 4 < 3 * (int64_t)p.cus;
    if (bytes < (few ? 2 : 1) * kStreamBytes) return DECODE_LIGHT;
    return few ? DECODE_DEEP : DECODE_WIDE;
}

bool make_plan(const ds_shape_t &s, Plan *p, PlanFor purpose, bool q4)
{
    if (!shape_ok(s, true)) return false;
    const DeviceCaps caps = device_caps();
    p->cus = caps.cus;
    p->units = s.B * s.Hkv;
    p->G = s.Hq / s.Hkv;
    p->k_eff = std::min(s.k, s.L);
    const int64_t tokens = (int64_t)p->units * s.L;

    int sc = tune_get(0);
    // fewer, larger workgroups: every workgroup pays an arrival atomic and a histogram flush
    if (sc == 0) {
        sc = (tokens >= (1 << 21)) ? 4096 : (tokens >= (1 << 20)) ? 2048 : 1024;
        // enough units to fill the device on their own: one workgroup scores a whole short unit
        // and takes the threshold bin from its own histogram, with no traffic between workgroups
        if (p->units >= caps.cus && s.L <= 8192) sc = (s.L + 255) & ~255;
    }
    p->sc_chunk = sc;
    p->n_sc = (s.L + sc - 1) / sc;

    // Launch shape of ds_sparse_decode: units of more than 8K tokens refine the threshold behind
    // the attention (one launch where it can score as well, else two).  Short units get one workgroup each, which
    // refines and attends the whole unit and writes the result itself (and scores it too when the label
    // cache allows it): everything between workgroups -- keys in memory,
    // histograms, arrival counting, partials -- costs more than it spreads at that size.  "Short"
    // is 4K tokens; 8K when there are enough units (256) to fill the device; 16K, what a workgroup's registers
    // hold, for single heads or pairs that it scores itself, with 192 units or more.
    // Units of 4K to 8K tokens that are too few for that take the long units'
    // path when the attention launch can score, with one workgroup or several (see below); what is
    // left refines the threshold in the scoring launch's tail.
    const bool one_wg_units =
        purpose != PLAN_SELECT &&
        (s.L <= 4096 || (p->units >= caps.cus && s.L <= 8192) ||
         (purpose == PLAN_DECODE_SCORING && p->units >= caps.cus * 3 / 4 && p->G <= 2 && s.L <= 16384));
    p->refine_attend = purpose != PLAN_SELECT &&
                       (tune_get(3) == 4 ||
                        (tune_get(3) == 0 && (s.L > (1 << 13) || one_wg_units ||
                                            (purpose == PLAN_DECODE_SCORING && s.L > (1 << 12)))));
    int ch = tune_get(1), ch_room = 0;
    p->chunks_score = false;
    p->unit_groups = 1;
    if (ch == 0 && p->refine_attend && !one_wg_units && purpose == PLAN_DECODE_SCORING)
        ch = room_chunk(p->units, s.L, p->G, caps);  // (choose_chunks below decides about the launch)
    if (ch != 0) {
        // (set by the knob, or the workspace's room)
    } else if (p->refine_attend && one_wg_units) {
        ch = (s.L + 255) & ~255;
    } else if (p->refine_attend) {
        // every workgroup resident at once (registers allow four per CU on the vector path, three on
        // the matrix cores) when chunks of up to 4096 / 6144 tokens allow it
        if (p->G <= 2) {
            // Behind a scoring launch: a second round of workgroups for the few that do not fit costs far
            // more than chunks of twice the size (scores from K rows, 17 single heads of 64K tokens, 1088
            // workgroups 104.4 us, 544 93.3; 48 of 32K 113.0 and 103.6; pairs 107.0 and 95.1; 64
            // fp16 channels 78.9 and 67.9; below that line 40 single heads of 16K tokens in 640 or 320, 59.7 and 59.0).
            ch = 1024;
            while (ch < 4096 && (int64_t)p->units * ((s.L + ch - 1) / ch) > 6 * caps.cus) ch *= 2;
            ch_room = ch;  // (the workspace keeps the room of six per CU)
            while (ch < 4096 && (int64_t)p->units * ((s.L + ch - 1) / ch) > 4 * caps.cus) ch *= 2;
        } else {
            ch = 2048;
            while (ch < 6144 && ch < s.L && (int64_t)p->units * ((s.L + ch - 1) / ch) > 3 * caps.cus) ch += 256;
        }
    } else {
        ch = (tokens >= (1 << 21)) ? 2048 : (tokens >= (1 << 20)) ? 1024 : (tokens >= (1 << 18)) ? 512 : 256;
        if (p->G >= 4 && ch < 4096) ch *= 2;  // a query group writes G partials per chunk
        while ((s.L + ch - 1) / ch > kMaxChunks && ch < 4096) ch *= 2;
        // The matrix-core attention holds three workgroups per CU (768 on the device).  A launch
        // slightly over that runs a nearly empty second round: grow the chunks to fit in one.
        if (p->G >= 4)
            while ((int64_t)p->units * ((s.L + ch - 1) / ch) > 3 * caps.cus && ch < 6144 && ch < s.L) ch += 256;
    }
    // One workgroup also takes a unit of up to 6K tokens, and with half as many units as compute units
    // one of up to 8K, when it can score it: what passes between several costs more than one compute
    // unit's rate (about 33 GB/s) over a sixteenth of so many rows.  Several against one, us per
    // layer: single heads, 8 channels, 32 units of 5000 tokens 17.7 -> 15.0, 128 of 6016 22.7 -> 18.7,
    // 128 of 8192 25.1 -> 21.6; 16 channels 19.5 -> 18.7, 24.1 -> 21.5, 27.5 -> 25.7; groups of 4 and 8,
    // 8 to 64 units of 6016 20.1 .. 22.2 -> 19.4 .. 21.0, 128 of 8192 25.4 -> 24.8.  On the other side
    // of the line: 64 single heads of 8192 tokens 20.8 -> 20.5 and with 16 channels 22.2 -> 24.0, 32
    // to 64 groups of 4 21.3 -> 23.8, 128 single heads of 10240 with 16 channels 30.0 -> 30.1; 680 rows,
    // 80 single heads of 5445 22.0 -> 24.7.  Pairs gain less: 64 units of 6016 20.8 -> 21.6, 128
    // 23.6 -> 22.0, 128 of 8192 26.3 -> 26.9.
    // Where heads share a unit, wide label rows (more than 12 fp16 channels, two words of 4-bit codes) move the
    // line: one / several for groups of 4 with 16 channels 0.97 at 5000 tokens, 1.01 at 5632, 1.02 to 1.04 at 6144 (8 to 32
    // units), 4-bit 0.94, 0.99, 1.00; 128 units with 24 channels 0.90 at 6144, 0.95 at 7000, 1.02 at 8192, 4-bit 0.92, 1.02,
    // 1.05; pairs 4-bit 0.98 at 5632, 1.02 at 6144.  Single heads of up to 24 channels stay below 1 (64 units of 6144, 4-bit of
    // 16 channels: 1.02).
    // (The workspace keeps the room of the plan with several.)
    const int n_ws = (s.L + (ch_room ? ch_room : ch) - 1) / (ch_room ? ch_room : ch);
    const bool half_full = p->units * 2 >= caps.cus;
    const bool wide = s.r > (q4 ? 8 : 12);
    const int one_wg_tokens = p->G == 1   ? (half_full ? 8192 : 6144)
                              : p->G == 2 ? (half_full ? (wide ? 5632 : 6144) : 0)
                              : half_full ? (wide ? 6656 : 8192)
                                          : (wide ? 5376 : 6144);
    // Units that fill the device by themselves take one as long as it can hold them, groups as single heads and
    // pairs do above: 192 units of 9000 tokens in groups of 4 27.1 -> 23.2 us, 256 of 16000 38.1 -> 34.9, 512 of 9000 53.7 -> 36.4,
    // 1024 of 12000 139.6 -> 87.2.
    const bool many_groups = p->G > 2 && p->units * 4 >= caps.cus * 3 && s.L > 8192 && s.L <= kDecodeTokens;
    if (n_ws > 1 && p->refine_attend && purpose == PLAN_DECODE_SCORING && tune_get(1) == 0 &&
        (many_groups || (s.L <= one_wg_tokens && p->k_eff <= one_wg_tokens / 16))) {
        ch = (s.L + 255) & ~255;
        p->unit_groups = 1;
    } else if (n_ws > 1 && p->refine_attend && purpose == PLAN_DECODE_SCORING && tune_get(1) == 0) {
        if (!choose_chunks(p->units, s.L, p->G, (q4 ? (s.r + 7) / 8 * 4.0 : 2.0 * s.r) + 512.0 * p->k_eff / s.L, caps.cus, n_ws, &ch, &p->unit_groups))
            return make_plan(s, p, PLAN_DECODE, q4);  // (no launch that scores itself fits at once)
        p->chunks_score = true;
    }
    p->ch = ch;
    p->n_ch = (s.L + ch - 1) / ch;
    if (n_ws > kMaxChunks) return false;
    p->key_stride = (s.L + 3) & ~3;

    size_t off = 0;
    p->off_ctl = off;   off = align_up(off + (size_t)p->units * sizeof(UnitCtl), 256);
    p->off_hist = off;  off = align_up(off + (size_t)p->units * kHistBins * 4, 256);
    p->off_coarse = off; off = align_up(off + (size_t)p->units * 256 * 4, 256);
    p->off_keys = off;  off = align_up(off + (size_t)p->units * p->key_stride * 4, 256);
    p->off_cand = off;  off = align_up(off + (size_t)p->units * s.L * 8, 256);
    p->off_ndef = off;  off = align_up(off + (size_t)p->units * n_ws * 4, 256);
    p->off_offs = off;  off = align_up(off + (size_t)p->units * n_ws * 4, 256);
    p->off_part = off;  off = align_up(off + (size_t)p->units * p->G * n_ws * kPartStride * 4, 256);
    p->total = off;
    return true;
}

// Workspace of a dense plan with n_ch chunks per unit: the same control prefix (records +
// histograms) as the sparse plan, so that sparse and dense calls may alternate on one workspace
// without disturbing each other's zeroed counters, and a partial per chunk and head.
static size_t dense_part_offset(int units)
{
    size_t off = align_up((size_t)units * sizeof(UnitCtl), 256);
    off = align_up(off + (size_t)units * kHistBins * 4, 256);
    return align_up(off + (size_t)units * 256 * 4, 256);
}
static size_t dense_total(int units, int G, int64_t n_ch)
{
    return align_up(dense_part_offset(units) + (size_t)units * G * n_ch * kPartStride * 4, 256);
}

size_t dense_room(const ds_shape_t &s, int n_tokens)
{
    const int units = s.B * s.Hkv;
    const int64_t tokens = (int64_t)units * n_tokens;
    const int ch = tune_get(2) ? tune_get(2) : tokens >= (1 << 20) ? 1024 : tokens >= (1 << 18) ? 256 : 64;
    return dense_total(units, s.Hq / s.Hkv, (n_tokens + ch - 1) / ch);
}

bool make_dense_plan(const ds_shape_t &s, int n_tokens, DensePlan *p, size_t workspace_bytes)
{
    if (!shape_ok(s, false) || n_tokens < 1) return false;
    p->units = s.B * s.Hkv;
    p->G = s.Hq / s.Hkv;
    int ch = tune_get(2);
    const size_t room = workspace_bytes >= dense_room(s, n_tokens) ? workspace_bytes : SIZE_MAX;
    if (ch == 0) {
        // Chunks per unit: the number with the least estimated time, of 1, 2, 3, 4, 6, 8, 12 .. and those
        // that fill the device w = 1/4, 1/2, 1 .. 8 times (chunks of 32 tokens at least, up to eight
        // workgroups per compute unit).  The estimate, in rows of a compute unit, which streams
        // about 46 of them per us:
        //   - the busiest compute unit's rows, in whole rounds of 64 where heads share them, and not
        //     fewer than the average one's (memory's rate) -- except where single heads and pairs have
        //     fewer than 512 rows per compute unit: those wait for latency, which two workgroups on a
        //     compute unit hide from each other;
        //   - a start and an end of each workgroup: 300 on the matrix cores, 60 on the vector path;
        //     groups of more than 16 heads pass over the rows, and pay both, once per 16 heads;
        //   - the merge by the unit's last workgroup: 75, and 110 for each of its dependent batches of
        //     loads (merge_partials: eight groups of threads share the heads of a round, each with eight
        //     partials in flight, four for single heads).
        // Over 649 shapes (1 to 512 units in groups of 1 to 64, 130 to 65536 tokens) the choice is 0.8 %
        // from the best of 23 chunk counts, 3 % at the 90th percentile.  Against chunks of 64 / 256 / 1024
        // tokens by the number of tokens alone: 32 units of 32K tokens in groups of 4 105 -> 83 us, 12
        // units of 20K in groups of 7 116 -> 27, 8 units of 32K in groups of 8 66 -> 33, 32 single heads of
        // 64K 179 -> 153, one unit of 2K in groups of 64 77 -> 50 (with 64 chunks 123); on the other side
        // 200 units of 8K in groups of 4, 143 -> 151.
        // A workspace that has dense_room() but not the chosen plan's takes the best of those that fit it:
        // one sized for more tokens of the same heads serves every shorter call.
        const int cus = device_caps().cus, G = p->G;
        const int64_t units = p->units;
        const bool matrix = G > 2;
        const int passes = (G + 15) / 16;
        const int gph = G > 4 ? 1 : G > 2 ? 2 : G == 2 ? 4 : 8, partials = gph * (G == 1 ? 4 : 8), heads = 8 / gph;
        double best = 0.0;
        auto consider = [&](int64_t n_want) {
            const int64_t nw = std::min<int64_t>(std::max<int64_t>(n_want, 1), std::max(1, n_tokens / 32));
            const int64_t c = ((n_tokens + nw - 1) / nw + 15) & ~15ll, n = (n_tokens + c - 1) / c;
            if ((n > 1 && units * n > 8ll * cus) || dense_total(p->units, G, n) > room) return;
            const int64_t busiest = (units * n + cus - 1) / cus;
            double rows = (double)busiest * (G > 1 ? (c + 63) & ~63ll : c);
            if (matrix || units * n_tokens >= 512ll * cus) rows = std::max(rows, (double)units * n_tokens / cus);
            else if (busiest > 1) rows *= 0.5;
            const double merge = n > 1 ? 75.0 + 110.0 * ((G + heads - 1) / heads) * ((n + partials - 1) / partials) : 0.0;
            const double cost = passes * (rows + busiest * (matrix ? 300.0 : 60.0)) + merge;
            // (of two equals the one with fewer chunks)
            if (ch == 0 || cost < best || (cost == best && c > ch)) {
                best = cost;
                ch = (int)c;
            }
        };
        for (int64_t n = 1; n <= 8ll * cus; n *= 2) {
            consider(n);
            consider(n + n / 2);
        }
        for (int w4 = 1; w4 <= 32; w4 += w4 < 4 ? w4 : 4) consider((int64_t)w4 * cus / 4 / units);
    }
    p->ch = ch;
    p->n_ch = (n_tokens + ch - 1) / ch;
    p->off_ctl = 0;
    p->off_part = dense_part_offset(p->units);
    p->total = dense_total(p->units, p->G, p->n_ch);
    return true;
}

// ---------------------------------------------------------------- per-kernel event timing
static const char *const kKernelNames[KID_COUNT] = {
    "k_init", "k_score", "k_cand", "k_attend", "k_compact", "k_dense",
    "k_attend_rows", "k_label", "k_gather_host", "k_probe",
    "k_refine_attend", "k_append_kv", "k_q4_build", "k_q4_write", "k_predict_query", "k_q4_amax", "k_q4_code"};

struct ProfRec { int id; hipEvent_t a, b; };
static std::mutex g_prof_mu;
static bool g_prof_on = false;
static std::vector<ProfRec> g_prof_recs;
static std::vector<hipEvent_t> g_prof_pool;

static hipEvent_t prof_event()
{
    if (!g_prof_pool.empty()) {
        hipEvent_t e = g_prof_pool.back();
        g_prof_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

bool prof_events(int id, hipEvent_t *start, hipEvent_t *stop)
{
    if (!g_prof_on) return false;
    std::lock_guard<std::mutex> lk(g_prof_mu);
    hipEvent_t a = prof_event();
    if (!a) return false;
    hipEvent_t b = prof_event();
    if (!b) { g_prof_pool.push_back(a); return false; }
    g_prof_recs.push_back({id, a, b});
    *start = a;
    *stop = b;
    return true;
}

}  // namespace ds

using namespace ds;

// ---------------------------------------------------------------- helpers
static bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

#define DS_TRY(expr)                                  \
    do {                                              \
        if ((expr) != hipSuccess) return DS_ERR_HIP;  \
    } while (0)

extern "C" {

const char *ds_strerror(ds_status_t status)
{
    switch (status) {
    case DS_OK: return "ok";
    case DS_ERR_NULL: return "required pointer is NULL";
    case DS_ERR_SHAPE: return "invalid shape or size argument";
    case DS_ERR_ALIGN: return "pointer is not sufficiently aligned";
    case DS_ERR_WORKSPACE: return "workspace is too small (static-scratch call: the shape needs more than ds_static_scratch_bytes())";
    case DS_ERR_UNSUPPORTED: return "configuration not supported";
    case DS_ERR_HIP: return "HIP runtime reported an error";
    }
    return "unknown status";
}

int ds_version(void) { return 112; }

ds_status_t ds_calibrate_channels(const uint16_t *q_calib, const uint16_t *k_calib, int32_t N,
                                  int32_t Hq, int32_t Hkv, int32_t d, int32_t r,
                                  ds_calib_mode_t mode, int32_t *channels_out)
{
    if (!q_calib || !k_calib || !channels_out) return DS_ERR_NULL;
    if (N < 1 || Hq < 1 || Hkv < 1 || d < 1 || r < 1 || r > d || Hq % Hkv != 0) return DS_ERR_SHAPE;
    if (mode != DS_CALIB_Q && mode != DS_CALIB_K && mode != DS_CALIB_QK) return DS_ERR_SHAPE;
    const int G = Hq / Hkv;
    // |x| of a binary16 bit pattern, widened through binary32 bit assembly
    auto habs = [](uint16_t h) -> double {
        const uint32_t e = (h >> 10) & 0x1f, m = h & 0x3ff;
        if (e == 0) return std::ldexp((double)m, -24);
        if (e == 31) return m ? NAN : INFINITY;
        return std::ldexp((double)(m | 0x400), (int)e - 25);
    };
    std::vector<double> mq(d), mk(d), w(d);
    std::vector<int32_t> order(d);
    for (int h = 0; h < Hkv; ++h) {
        std::fill(mq.begin(), mq.end(), 0.0);
        std::fill(mk.begin(), mk.end(), 0.0);
        for (int n = 0; n < N; ++n) {
            for (int g = 0; g < G; ++g) {
                const uint16_t *row = q_calib + ((size_t)n * Hq + (size_t)h * G + g) * d;
                for (int c = 0; c < d; ++c) mq[c] += habs(row[c]);
            }
            const uint16_t *krow = k_calib + ((size_t)n * Hkv + h) * d;
            for (int c = 0; c < d; ++c) mk[c] += habs(krow[c]);
        }
        for (int c = 0; c < d; ++c) {
            const double a = mq[c] / ((double)N * G), b = mk[c] / (double)N;
            w[c] = mode == DS_CALIB_Q ? a : mode == DS_CALIB_K ? b : a * b;
            order[c] = c;
        }
        std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) { return w[x] > w[y]; });
        std::sort(order.begin(), order.begin() + r);
        std::copy(order.begin(), order.begin() + r, channels_out + (size_t)h * r);
    }
    return DS_OK;
}

static ds_status_t check_label_args(const void *K, const int32_t *channels, void *label,
                                    const ds_shape_t *s)
{
    if (!K || !channels || !label || !s) return DS_ERR_NULL;
    if (s->B < 1 || s->Hkv < 1 || s->d != kD || s->r < 1 || s->r > s->d || s->L_max < 1)
        return DS_ERR_SHAPE;
    if ((int64_t)s->B * s->Hkv > 65535) return DS_ERR_SHAPE;
    if (!aligned(K, 256) || !aligned(label, 16)) return DS_ERR_ALIGN;
    return DS_OK;
}

ds_status_t ds_build_label(const void *K, const int32_t *channels, void *label,
                           const ds_shape_t *shape, void *stream)
{
    ds_status_t st = check_label_args(K, channels, label, shape);
    if (st != DS_OK) return st;
    if (shape->L < 1 || shape->L > shape->L_max) return DS_ERR_SHAPE;
    DS_TRY(launch_label(K, channels, label, *shape, 0, shape->L, (hipStream_t)stream));
    return DS_OK;
}

ds_status_t ds_append_label(const void *K, const int32_t *channels, void *label,
                            const ds_shape_t *shape, int32_t t0, int32_t n_new, void *stream)
{
    ds_status_t st = check_label_args(K, channels, label, shape);
    if (st != DS_OK) return st;
    if (t0 < 0 || n_new < 0 || (int64_t)t0 + n_new > shape->L_max) return DS_ERR_SHAPE;
    DS_TRY(launch_label(K, channels, label, *shape, t0, n_new, (hipStream_t)stream));
    return DS_OK;
}

ds_status_t ds_build_label_q4(const void *K, const int32_t *channels, void *label_q4, float *amax,
                              const ds_shape_t *shape, void *stream)
{
    if (!amax) return DS_ERR_NULL;
    ds_status_t st = check_label_args(K, channels, label_q4, shape);
    if (st != DS_OK) return st;
    if (shape->L < 1 || shape->L > shape->L_max) return DS_ERR_SHAPE;
    if (!aligned(amax, 4)) return DS_ERR_ALIGN;
    DS_TRY(launch_q4_build(K, channels, amax, label_q4, *shape, (hipStream_t)stream));
    return DS_OK;
}

ds_status_t ds_append_label_q4(const void *K, const int32_t *channels, void *label_q4,
                               const float *amax, const ds_shape_t *shape, int32_t t0,
                               int32_t n_new, void *stream)
{
    if (!amax) return DS_ERR_NULL;
    ds_status_t st = check_label_args(K, channels, label_q4, shape);
    if (st != DS_OK) return st;
    if (t0 < 0 || n_new < 0 || (int64_t)t0 + n_new > shape->L_max) return DS_ERR_SHAPE;
    DS_TRY(launch_q4_write(K, channels, amax, label_q4, *shape, t0, n_new, (hipStream_t)stream));
    return DS_OK;
}

ds_status_t ds_build_label_kv(const void *KV, const int32_t *channels, void *label,
                              const ds_shape_t *shape, void *stream)
{
    ds_status_t st = check_label_args(KV, channels, label, shape);
    if (st != DS_OK) return st;
    if (shape->L < 1 || shape->L > shape->L_max) return DS_ERR_SHAPE;
    DS_TRY(launch_label(KV, channels, label, *shape, 0, shape->L, (hipStream_t)stream, 2 * kD));
    return DS_OK;
}

ds_status_t ds_append_kv(const void *k_new, const void *v_new, void *K, void *V,
                         const int32_t *channels, void *label, const ds_shape_t *shape, int32_t t0,
                         int32_t n_new, ds_kv_layout_t layout, void *stream)
{
    if (!k_new || !v_new) return DS_ERR_NULL;
    if (layout != DS_KV_SPLIT && layout != DS_KV_INTERLEAVED) return DS_ERR_SHAPE;
    if (layout == DS_KV_SPLIT && !V) return DS_ERR_NULL;
    ds_status_t st = check_label_args(K, channels, label, shape);
    if (st != DS_OK) return st;
    if (t0 < 0 || n_new < 0 || (int64_t)t0 + n_new > shape->L_max) return DS_ERR_SHAPE;
    if (!aligned(k_new, 16) || !aligned(v_new, 16) || (layout == DS_KV_SPLIT && !aligned(V, 256)))
        return DS_ERR_ALIGN;
    const bool il = layout == DS_KV_INTERLEAVED;
    void *Vp = il ? static_cast<void *>(static_cast<char *>(K) + kD * 2) : V;
    DS_TRY(launch_append_kv(k_new, v_new, K, Vp, channels, label, *shape, t0, n_new, il ? 2 * kD : kD,
                            (hipStream_t)stream));
    return DS_OK;
}

size_t ds_workspace_bytes(const ds_shape_t *shape)
{
    if (!shape) return 0;
    Plan p;
    DensePlan dp, rp;
    size_t need = 0;
    for (PlanFor purpose : {PLAN_SELECT, PLAN_DECODE, PLAN_DECODE_SCORING}) {
        if (make_plan(*shape, &p, purpose)) {
            need = std::max(need, p.total);
            if (make_dense_plan(*shape, p.k_eff, &rp)) need = std::max({need, rp.total, dense_room(*shape, p.k_eff)});
        }
    }
    if (make_dense_plan(*shape, shape->L, &dp)) need = std::max({need, dp.total, dense_room(*shape, shape->L)});
    return need;
}

ds_status_t ds_workspace_init(void *workspace, size_t workspace_bytes, void *stream)
{
    if (!workspace) return DS_ERR_NULL;
    if (workspace_bytes == 0 || workspace_bytes % 16 != 0) return DS_ERR_SHAPE;
    if (!aligned(workspace, 16)) return DS_ERR_ALIGN;
    DS_TRY(launch_init(workspace, workspace_bytes, (hipStream_t)stream));
    return DS_OK;
}

ds_status_t ds_workspace_errors(const void *workspace, size_t workspace_bytes, const ds_shape_t *shape,
                                void *stream, int32_t *n_failed, int32_t *first_code)
{
    if (!workspace || !shape) return DS_ERR_NULL;
    Plan p;
    if (!shape_ok(*shape, true)) return DS_ERR_SHAPE;
    if (!make_plan(*shape, &p, PLAN_DECODE)) return DS_ERR_UNSUPPORTED;
    const size_t bytes = (size_t)p.units * sizeof(UnitCtl);
    if (workspace_bytes < p.off_ctl + bytes) return DS_ERR_WORKSPACE;
    std::vector<UnitCtl> ctl((size_t)p.units);
    if (hipMemcpyAsync(ctl.data(), static_cast<const char *>(workspace) + p.off_ctl, bytes, hipMemcpyDeviceToHost,
                       (hipStream_t)stream) != hipSuccess ||
        hipStreamSynchronize((hipStream_t)stream) != hipSuccess)
        return DS_ERR_HIP;
    int32_t n = 0, first = 0;
    for (const UnitCtl &c : ctl)
        if (c.err) {
            if (!n) first = (int32_t)c.err;
            ++n;
        }
    if (n_failed) *n_failed = n;
    if (first_code) *first_code = first;
    return DS_OK;
}

static ds_status_t select_common(const void *q, const void *label, const int32_t *channels,
                                 void *workspace, size_t workspace_bytes, const ds_shape_t *shape,
                                 Plan *p, PlanFor purpose = PLAN_SELECT, bool q4 = false)
{
    if (!q || !label || !channels || !workspace || !shape) return DS_ERR_NULL;
    if (!shape_ok(*shape, true)) return DS_ERR_SHAPE;
    if (!make_plan(*shape, p, purpose, q4)) return DS_ERR_UNSUPPORTED;
    if (!aligned(q, 16) || !aligned(label, 16) || !aligned(workspace, 16)) return DS_ERR_ALIGN;
    if (workspace_bytes < p->total) return DS_ERR_WORKSPACE;
    return DS_OK;
}

static ds_status_t enqueue_select(const void *q, const void *label, const int32_t *channels,
                                  void *ws, const Plan &p, const ds_shape_t &s, bool want_offsets,
                                  hipStream_t st, ScoreSrc src = ScoreSrc())
{
    // Units of up to 8K tokens: the scoring launch's last workgroup per unit also settles the
    // exact threshold (knob 4 = 1 forces the separate candidate launch, 2 forces the tail).
    const int mode = tune_get(4);
    const bool tail_refine = mode == 2 || (mode == 0 && s.L <= (1 << 13));
    DS_TRY(launch_score(q, label, channels, ws, p, s, true, tail_refine, want_offsets, st, src));
    if (!tail_refine) DS_TRY(launch_cand(ws, p, s, want_offsets, st));
    return DS_OK;
}

static bool label_may_score(const ds_shape_t &s, ScoreSrcKind kind)
{
    // the attention launch can score as well when the labels are plain fp16 of a multiple of 4 channels
    // up to 32 (with a scoring launch against without: 12 channels, 12 units of 20K tokens in groups
    // of 7 29.4 -> 25.3 us, 32 units of 64K tokens 44.3 -> 34.1; 24 channels, 128 units of 4K tokens
    // 24.2 -> 18.3; 4 channels, 32 units of 2K tokens 15.4 -> 10.6), or 4-bit codes of up to 16
    // channels in rows that 16-byte loads can take (knob 4 = 1 keeps the separate scoring launch)
    return tune_get(4) != 1 && ((kind == SRC_LABEL && attend_scores_r(s.r)) ||
                                (kind == SRC_Q4 && s.r <= 16 && (s.L_max & (s.r > 8 ? 1 : 3)) == 0));
}

// Whether the attention launch of a decode call scores as well: a unit with one workgroup always
// can; several workgroups per unit wait for each other before all of them have started, so the
// whole grid has to be resident at once -- as choose_chunks made it, or, with another number of chunks (knob 1; a
// part of a device), single heads and pairs at four workgroups per compute unit, what the 256-thread form allows.
// Knob 4 = 2 forces it, 1 forbids it.  (The launcher checks the grid against the occupancy the runtime reports.)
static bool plan_scores_itself(const Plan &p, bool may_score)
{
    return may_score && (p.n_ch == 1 || tune_get(4) == 2 ||
                         (tune_get(4) == 0 && p.G <= 2 &&
                          (int64_t)((p.units + p.unit_groups - 1) / p.unit_groups) * p.n_ch <= 4 * (int64_t)p.cus) ||
                         (tune_get(4) == 0 && p.chunks_score));
}

// ds_sparse_decode with the scores taken from the label cache, from the K rows themselves or from
// the 4-bit label cache (`label` is then that source's array).
static ds_status_t sparse_decode_impl(const void *q, const void *label, const void *K, const void *V,
                                      const int32_t *channels, float *out, int32_t *idx_out,
                                      void *workspace, size_t workspace_bytes,
                                      const ds_shape_t *shape, void *stream, ScoreSrc src,
                                      int kv_stride = kD, bool clear_first = false)
{
    if (!K || !V || !out) return DS_ERR_NULL;
    Plan p;
    bool may_score = shape && label_may_score(*shape, src.kind);
    ds_status_t rc;
    if (may_score && src.kind == SRC_LABEL && shape->r != 8 && shape->r != 16) {
        // (the workspace that a call needs is that of the plan with a scoring launch; the other
        //  plan is taken when it fits too)
        rc = select_common(q, label, channels, workspace, workspace_bytes, shape, &p, PLAN_DECODE);
        if (rc != DS_OK) return rc;
        Plan ps;
        may_score = make_plan(*shape, &ps, PLAN_DECODE_SCORING) && ps.total <= workspace_bytes;
        if (may_score) p = ps;
    } else {
        rc = select_common(q, label, channels, workspace, workspace_bytes, shape, &p,
                           may_score ? PLAN_DECODE_SCORING : PLAN_DECODE, src.kind == SRC_Q4);
        if (rc != DS_OK) return rc;
    }
    if (!aligned(K, 256) || !aligned(V, 256) || !aligned(out, 16) || (idx_out && !aligned(idx_out, 16)))
        return DS_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    // (a workspace shared by calls of different shapes: counters, histograms and error words start
    //  from zero whatever the last call left there -- a fill kernel, so that the call can be captured)
    if (clear_first) DS_TRY(launch_init(workspace, p.off_keys, st));
    // a workgroup that may score its tokens itself: one launch, keys never leave its registers
    // ... and so can several workgroups per unit (their chunk histograms meet in memory, where each finds
    // the threshold bin) as long as the whole grid is resident at once
    bool scores_itself = plan_scores_itself(p, may_score);
    const bool q4 = src.kind == SRC_Q4;
    if (p.refine_attend && refine_attend_ok(p, scores_itself)) {
        // (the runtime's occupancy figure for the kernel decides whether the workgroups that wait
        //  for each other are all resident; if not, the separate scoring launch needs less room,
        //  and the three launches below need none)
        if (scores_itself && !refine_attend_fits(p, *shape, true, q4)) {
            scores_itself = false;
            Plan ps;  // (chunks for the scoring launch's sake; a knob's chunks stay)
            if (p.chunks_score && make_plan(*shape, &ps, PLAN_DECODE, q4) && ps.total <= workspace_bytes) p = ps;
        }
        if (scores_itself) {
            DS_TRY(launch_refine_attend(q, K, V, workspace, out, idx_out, p, *shape, st, kv_stride, channels, src.amax,
                                        label));
            return DS_OK;
        }
        // otherwise scoring leaves keys and the threshold bin; one more launch settles the exact
        // threshold behind the attention over the rows that are selected either way
        if (refine_attend_ok(p, false) && refine_attend_fits(p, *shape, false, q4)) {
            DS_TRY(launch_score(q, label, channels, workspace, p, *shape, p.n_ch > 1, false, false, st, src));
            DS_TRY(launch_refine_attend(q, K, V, workspace, out, idx_out, p, *shape, st, kv_stride, channels, src.amax,
                                        nullptr));
            return DS_OK;
        }
    }
    rc = enqueue_select(q, label, channels, workspace, p, *shape, idx_out != nullptr, st, src);
    if (rc != DS_OK) return rc;
    DS_TRY(launch_attend_sparse(q, K, V, workspace, out, idx_out, p, *shape, st, kv_stride));
    return DS_OK;
}

ds_status_t ds_pretend_device(int32_t cus, int32_t xccs, int32_t lds_per_cu)
{
    if (cus == 0 && xccs == 0 && lds_per_cu == 0) {
        device_caps_pretend(nullptr);
        return DS_OK;
    }
    if (cus < 1 || xccs < 1 || cus % xccs != 0 || lds_per_cu < (64 << 10)) return DS_ERR_SHAPE;
    DeviceCaps c;
    c.cus = cus;
    c.xccs = xccs;
    c.lds_per_cu = lds_per_cu;
    device_caps_pretend(&c);
    return DS_OK;
}

ds_status_t ds_plan_describe(const ds_shape_t *shape, int32_t label_kind, int32_t out[8])
{
    if (!shape || !out) return DS_ERR_NULL;
    if (label_kind < 0 || label_kind > 2 || !shape_ok(*shape, true)) return DS_ERR_SHAPE;
    const ScoreSrcKind kind = static_cast<ScoreSrcKind>(label_kind);
    const bool may_score = label_may_score(*shape, kind);
    Plan p;
    if (!make_plan(*shape, &p, may_score ? PLAN_DECODE_SCORING : PLAN_DECODE, kind == SRC_Q4)) return DS_ERR_UNSUPPORTED;
    const bool si = plan_scores_itself(p, may_score);
    const bool ra = p.refine_attend && refine_attend_ok(p, si);
    const int planned = !ra ? 3 : si ? p.unit_groups : 2;
    int actual = -1;
    int n_dev = 0;
    if (hipGetDeviceCount(&n_dev) == hipSuccess && n_dev > 0) {
        actual = 3;
        if (ra) {
            const bool q4 = kind == SRC_Q4;
            if (si && refine_attend_fits(p, *shape, true, q4)) actual = p.unit_groups;
            else if (refine_attend_ok(p, false) && refine_attend_fits(p, *shape, false, q4)) actual = 2;
        }
    }
    (void)hipGetLastError();
    out[0] = planned;
    out[1] = actual;
    out[2] = p.ch;
    out[3] = p.n_ch;
    out[4] = p.units * p.n_ch;
    out[5] = p.cus;
    out[6] = si ? 1 : 0;
    out[7] = p.G;
    return DS_OK;
}

ds_status_t ds_sparse_decode(const void *q, const void *label, const void *K, const void *V,
                             const int32_t *channels, float *out, int32_t *idx_out,
                             void *workspace, size_t workspace_bytes, const ds_shape_t *shape,
                             void *stream)
{
    return sparse_decode_impl(q, label, K, V, channels, out, idx_out, workspace, workspace_bytes, shape,
                              stream, ScoreSrc());
}

// Address of this device's copy of the static scratch array, resolved once per device.
static ds_status_t static_scratch(void **ptr)
{
    static std::mutex mu;
    static void *per_device[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return DS_ERR_HIP;
    if (dev < 0 || dev >= 64) return DS_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lk(mu);
    if (!per_device[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return DS_ERR_HIP;
        per_device[dev] = p;
    }
    *ptr = per_device[dev];
    return DS_OK;
}

size_t ds_static_scratch_bytes(void) { return DS_STATIC_SCRATCH_BYTES; }

ds_status_t ds_static_init(void)
{
    void *p = nullptr;
    return static_scratch(&p);
}

ds_status_t ds_sparse_decode_static(const void *q, const void *label, const void *K, const void *V,
                                    const int32_t *channels, float *out, int32_t *idx_out,
                                    const ds_shape_t *shape, void *stream)
{
    if (!q || !label || !K || !V || !channels || !out || !shape) return DS_ERR_NULL;
    void *ws = nullptr;
    ds_status_t rc = static_scratch(&ws);
    if (rc != DS_OK) return rc;
    // shapes whose scratch layout is larger than the array come back as DS_ERR_WORKSPACE
    return sparse_decode_impl(q, label, K, V, channels, out, idx_out, ws, DS_STATIC_SCRATCH_BYTES, shape,
                              stream, ScoreSrc(), kD, true);
}

ds_status_t ds_sparse_decode_nolabel(const void *q, const void *K, const void *V,
                                     const int32_t *channels, float *out, int32_t *idx_out,
                                     void *workspace, size_t workspace_bytes,
                                     const ds_shape_t *shape, void *stream)
{
    ScoreSrc src;
    src.kind = SRC_K_ROWS;
    return sparse_decode_impl(q, K, K, V, channels, out, idx_out, workspace, workspace_bytes, shape,
                              stream, src);
}

ds_status_t ds_sparse_decode_q4(const void *q, const void *label_q4, const float *amax, const void *K,
                                const void *V, const int32_t *channels, float *out,
                                int32_t *idx_out, void *workspace, size_t workspace_bytes,
                                const ds_shape_t *shape, void *stream)
{
    if (!amax) return DS_ERR_NULL;
    if (!aligned(amax, 4)) return DS_ERR_ALIGN;
    ScoreSrc src;
    src.kind = SRC_Q4;
    src.amax = amax;
    return sparse_decode_impl(q, label_q4, K, V, channels, out, idx_out, workspace, workspace_bytes,
                              shape, stream, src);
}

ds_status_t ds_sparse_decode_kv(const void *q, const void *label, const void *KV,
                                const int32_t *channels, float *out, int32_t *idx_out,
                                void *workspace, size_t workspace_bytes, const ds_shape_t *shape,
                                void *stream)
{
    if (!KV) return DS_ERR_NULL;
    // a row is addressed by a 32-bit byte offset inside its unit: 512-byte steps here
    if (shape && (int64_t)shape->L_max * 4 * kD > 0xffffffffll) return DS_ERR_SHAPE;
    const void *V = static_cast<const char *>(KV) + kD * 2;
    return sparse_decode_impl(q, label, KV, V, channels, out, idx_out, workspace, workspace_bytes, shape,
                              stream, ScoreSrc(), 2 * kD);
}

ds_status_t ds_select(const void *q, const void *label, const int32_t *channels, int32_t *idx_out,
                      void *workspace, size_t workspace_bytes, const ds_shape_t *shape, void *stream)
{
    if (!idx_out) return DS_ERR_NULL;
    Plan p;
    ds_status_t rc = select_common(q, label, channels, workspace, workspace_bytes, shape, &p);
    if (rc != DS_OK) return rc;
    if (!aligned(idx_out, 16)) return DS_ERR_ALIGN;
    hipStream_t st = (hipStream_t)stream;
    rc = enqueue_select(q, label, channels, workspace, p, *shape, true, st);
    if (rc != DS_OK) return rc;
    DS_TRY(launch_compact(workspace, idx_out, p, *shape, st));
    return DS_OK;
}

ds_status_t ds_dense_decode(const void *q, const void *K, const void *V, float *out,
                            void *workspace, size_t workspace_bytes, const ds_shape_t *shape,
                            void *stream)
{
    if (!q || !K || !V || !out || !workspace || !shape) return DS_ERR_NULL;
    if (!shape_ok(*shape, false)) return DS_ERR_SHAPE;
    DensePlan p;
    if (!make_dense_plan(*shape, shape->L, &p, workspace_bytes)) return DS_ERR_UNSUPPORTED;
    if (!aligned(K, 256) || !aligned(V, 256) || !aligned(q, 16) || !aligned(out, 16) ||
        !aligned(workspace, 16))
        return DS_ERR_ALIGN;
    if (workspace_bytes < p.total) return DS_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    DS_TRY(launch_attend_dense(q, K, V, workspace, out, p, *shape, st));
    return DS_OK;
}

ds_status_t ds_predict_query(const void *x, const void *Wq, void *q_out, int32_t B, int32_t Dm,
                             int32_t N, void *stream)
{
    if (!x || !Wq || !q_out) return DS_ERR_NULL;
    // 16-byte pieces of a row; x for up to four batch rows has to fit the 64 KiB of LDS asked for
    if (B < 1 || N < 1 || Dm < 8 || Dm % 8 != 0 || Dm > 8192) return DS_ERR_SHAPE;
    if (!aligned(x, 16) || !aligned(Wq, 16) || !aligned(q_out, 2)) return DS_ERR_ALIGN;
    DS_TRY(launch_predict_query(x, Wq, q_out, B, Dm, N, (hipStream_t)stream));
    return DS_OK;
}

ds_status_t ds_gather_rows_host(const void *K_host, const void *V_host, const int32_t *idx,
                                void *KV_rows, const ds_shape_t *shape, void *stream)
{
    if (!K_host || !V_host || !idx || !KV_rows || !shape) return DS_ERR_NULL;
    if (!shape_ok(*shape, true)) return DS_ERR_SHAPE;
    if (!aligned(K_host, 256) || !aligned(V_host, 256) || !aligned(KV_rows, 256) || !aligned(idx, 4))
        return DS_ERR_ALIGN;
    DS_TRY(launch_gather_host(K_host, V_host, idx, KV_rows, *shape, (hipStream_t)stream));
    return DS_OK;
}

ds_status_t ds_attend_rows(const void *q, const void *KV_rows, float *out, void *workspace,
                           size_t workspace_bytes, const ds_shape_t *shape, void *stream)
{
    if (!q || !KV_rows || !out || !workspace || !shape) return DS_ERR_NULL;
    if (!shape_ok(*shape, true)) return DS_ERR_SHAPE;
    const int n_rows = std::min(shape->k, shape->L);
    DensePlan p;
    if (!make_dense_plan(*shape, n_rows, &p, workspace_bytes)) return DS_ERR_UNSUPPORTED;
    if (!aligned(KV_rows, 256) || !aligned(q, 16) || !aligned(out, 16) || !aligned(workspace, 16))
        return DS_ERR_ALIGN;
    if (workspace_bytes < p.total) return DS_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    DS_TRY(launch_attend_rows(q, KV_rows, workspace, out, p, *shape, n_rows, st));
    return DS_OK;
}

ds_status_t ds_probe_stream_read(const void *src, size_t bytes, uint32_t *sink, void *stream)
{
    if (!src || !sink) return DS_ERR_NULL;
    if (bytes == 0 || bytes % 16 != 0 || bytes / 16 / (kWG * 8) > 0x7fffffffull) return DS_ERR_SHAPE;
    if (!aligned(src, 16) || !aligned(sink, 4)) return DS_ERR_ALIGN;
    DS_TRY(launch_probe(src, bytes, sink, (hipStream_t)stream));
    return DS_OK;
}

int ds_profile_kernel_count(void) { return KID_COUNT; }

const char *ds_profile_kernel_name(int id)
{
    return (id >= 0 && id < KID_COUNT) ? kKernelNames[id] : "";
}

ds_status_t ds_profile_enable(int on)
{
    std::lock_guard<std::mutex> lk(g_prof_mu);
    g_prof_on = on != 0;
    return DS_OK;
}

ds_status_t ds_profile_reset(void)
{
    std::lock_guard<std::mutex> lk(g_prof_mu);
    for (auto &r : g_prof_recs) {
        g_prof_pool.push_back(r.a);
        g_prof_pool.push_back(r.b);
    }
    g_prof_recs.clear();
    return DS_OK;
}

ds_status_t ds_profile_read(int id, double *total_ms, int64_t *launches)
{
    if (!total_ms || !launches) return DS_ERR_NULL;
    if (id < 0 || id >= KID_COUNT) return DS_ERR_SHAPE;
    std::lock_guard<std::mutex> lk(g_prof_mu);
    double tot = 0.0;
    int64_t n = 0;
    for (auto &r : g_prof_recs) {
        if (r.id != id) continue;
        if (hipEventSynchronize(r.b) != hipSuccess) return DS_ERR_HIP;
        float ms = 0.0f;
        if (hipEventElapsedTime(&ms, r.a, r.b) != hipSuccess) return DS_ERR_HIP;
        tot += ms;
        ++n;
    }
    *total_ms = tot;
    *launches = n;
    return DS_OK;
}

ds_status_t ds_tune_set(int knob, int value)
{
    if (knob < 0 || knob > 5) return DS_ERR_SHAPE;
    if (value < 0) return DS_ERR_SHAPE;
    if (value != 0) {
        if (knob == 0 && (value % 256 != 0 || value > (1 << 20))) return DS_ERR_SHAPE;
        if (knob == 1 && (value % 64 != 0 || value > 16384)) return DS_ERR_SHAPE;
        if (knob == 2 && (value % 16 != 0 || value > (1 << 20))) return DS_ERR_SHAPE;
        if (knob == 3 && value != 1 && value != 4) return DS_ERR_SHAPE;
        if (knob == 4 && value > 2) return DS_ERR_SHAPE;
    }
    g_tune[knob].store(value, std::memory_order_relaxed);
    return DS_OK;
}

int ds_tune_get(int knob) { return tune_get(knob); }

}  // extern "C"
