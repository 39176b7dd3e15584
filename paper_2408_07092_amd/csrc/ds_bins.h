// First-level bins of the decode launch: where a score is counted, and which keys a bin holds.
//
// A bin of either sign is 1/128 octave wide over 10 octaves around the label query's largest value, which
// every workgroup of a unit knows, and 1/16 octave over the 38 octaves round these; what lies beyond -- of fp16
// labels, 0 and sums that cancel to nearly that -- is in the end bins.  Any non-decreasing map of scores to bins
// keeps the selection exact; this one keeps the threshold's bin small: a thousandth of a unit's keys as a rule (70 of 64K
// tokens), a hundredth where the fine bins end (label channels of K that are below 1/20 or beyond 50).
// (us per layer: with bins of 1/8 octave throughout, the top 12 bits of the key; with 1/128 octave over 16 octaves and nothing
//  beyond; with these.  Label channels of K of ordinary size, 32 heads of 4K tokens 11.6, 8.2, 8.2, of 64K 29.3, 25.4, 25.3, 256 of 16K with
//  16 channels 50.2, 45.3, 45.2; a thousandth of it 11.5, 36.5, 10.2 -- 29.2, 103, 28.4 -- 50.6, 169, 47.6.)
#pragma once

#include <stdint.h>

namespace ds {

constexpr uint32_t kSideBins = 2048;                       // of either sign
constexpr uint32_t kFineOctaves = 10, kFineBins = kFineOctaves * 128;
constexpr uint32_t kCoarseBins = kSideBins - 1u - kFineBins;  // 767: 48 octaves less one bin

// A score is placed by x = exponent and upper 7 bits of its mantissa (128 steps an octave): its bin is the steps
// that x lies above the fine octaves' first, at most kFineBins, and the sixteenths of an octave that it lies above
// the coarse ones' first, at most kCoarseBins.  (So every ninth number among the fine bins stays unused.)
struct BinScale {
    uint32_t fine0, coarse0;  // steps, sixteenths of octaves
    uint32_t fine1, coarse1;  // their last (in vector registers)

    // magnitude: bits of the label query's largest value, sign clear.  Fine from an eighth of its octave on.
    __host__ __device__ explicit BinScale(int magnitude)
    {
        const int e = (magnitude >> 23 & 255) - 3, first = e < 0 ? 0 : e > 244 ? 244 : e;
        fine0 = (uint32_t)first << 7;
        coarse0 = first < 22 ? 0u : (uint32_t)(first - 22) << 4;
        fine1 = fine0 + kFineBins;
        coarse1 = coarse0 + kCoarseBins;
#ifdef __HIP_DEVICE_COMPILE__
        asm("" : "+v"(fine1), "+v"(coarse1));  // (else copied there for every score: an instruction has one scalar operand)
#endif
    }
    // x, but no less than lo and no more than hi (one instruction, which a compiler that does not know lo <= hi needs two for)
    __host__ __device__ static uint32_t within(uint32_t x, uint32_t lo, uint32_t hi)
    {
#ifdef __HIP_DEVICE_COMPILE__
        asm("v_med3_u32 %0, %0, %1, %2" : "+v"(x) : "s"(lo), "v"(hi));
        return x;
#else
        return x < lo ? lo : x < hi ? x : hi;
#endif
    }
    // bits: of the score, its sign is ignored
    __host__ __device__ uint32_t bin(uint32_t bits) const
    {
        return within(bits >> 16 & 0x7fffu, fine0, fine1) + within(bits >> 19 & 0xfffu, coarse0, coarse1) - (fine0 + coarse0);
    }
    // keys (see score_key) of bin b of both signs, 0 <= b < 2 kSideBins: [lo, hi]
    __host__ __device__ void keys(uint32_t b, uint32_t &lo, uint32_t &hi) const
    {
        const bool neg = b < kSideBins;
        const int m = neg ? (int)(kSideBins - 1u - b) : (int)(b - kSideBins);
        // t: from the first fine bin on; a coarse bin is eight steps wide, a fine one one step
        const int t = m + (int)coarse0 - (int)(fine0 >> 3), t1 = (int)kFineBins / 8 * 9;
        const bool fine = t >= 0 && t < t1;
        const int x = (int)fine0 + (fine ? t - (t * 7282 >> 16) : t < 0 ? 8 * t : 8 * t - (8 * t1 - (int)kFineBins));  // (t / 9)
        const uint32_t a = m == 0 ? 0u : (uint32_t)(x < 0x7fff ? x : 0x7fff) << 16;
        const uint32_t z = m == (int)kSideBins - 1 ? 0x7fffffffu : ((uint32_t)(x + (fine ? 1 : 8)) << 16) - 1u;
        lo = neg ? ~(0x80000000u | z) : 0x80000000u | a;
        hi = neg ? ~(0x80000000u | a) : 0x80000000u | z;
    }
};

}  // namespace ds
