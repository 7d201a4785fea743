// wave.h -- 64-lane wave primitives shared by the layout kernels (gfx950).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ep {

// Mask of lanes whose `valid` is set and whose expert id equals this lane's in its low NB
// bits: per bit, the lanes that agree with this lane are ~(ballot ^ own bit).
template <int NB>
__device__ __forceinline__ uint64_t match_bits(int e, bool valid) {
    const uint64_t v = __ballot(valid);
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int own = (e << (31 - b)) >> 31;  // all ones when the bit is set
        const uint64_t bal = __ballot(own != 0);
        lo &= ~((uint32_t)bal ^ (uint32_t)own);
        hi &= ~((uint32_t)(bal >> 32) ^ (uint32_t)own);
    }
    return ((uint64_t)hi << 32) | lo;
}

// The same over nbits bits (wave-uniform, at most 11); unrolled steps, so that the ballots
// of one match overlap.
__device__ __forceinline__ uint64_t match_expert(int e, bool valid, int nbits) {
    if (nbits <= 4)
        return match_bits<4>(e, valid);
    if (nbits <= 6)
        return match_bits<6>(e, valid);
    if (nbits <= 8)
        return match_bits<8>(e, valid);
    return match_bits<11>(e, valid);
}

// Number of lanes of `m` below this lane.
__device__ __forceinline__ int lanes_below(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Inclusive prefix sum over the 64 lanes of a wave with DPP row shifts and broadcasts.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 -> rows 1,3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 -> rows 2,3
    return v;
}

// ---- LDS histograms: C counters per bin (C a power of two up to 16), lane l adding to
// counter l % C of its bin.  The counters of a bin are neighbouring words, so lanes that
// count the same bin use different LDS banks and at most 64 / C lanes of an instruction
// share a word, however skewed the counts are.  Measured on MI355X, cycles of a wave's add
// of 64 ids, 16 copies, three quarters of the ids the same: 8.4; with the copies as rows of
// counters a multiple of 32 words apart, which puts a bin's copies in one bank, 50.9.
__device__ __forceinline__ int hist_index(int bin, int copies, int lane) { return bin * copies + (lane & (copies - 1)); }

// Sum of a bin's C counters; neighbouring lanes start at different quarters of their bins
// (C = 16), so that their 16-byte reads spread over the banks.
__device__ __forceinline__ int hist_sum(const int *hist, int bin, int copies, int lane) {
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    int s = 0;
    if (copies >= 4) {
        const i32x4 *q = reinterpret_cast<const i32x4 *>(hist + bin * copies);
        const int quads = copies / 4;
        for (int i = 0; i < quads; ++i) {
            const i32x4 v = q[(i + (lane >> 2)) & (quads - 1)];
            s += (v[0] + v[1]) + (v[2] + v[3]);
        }
    } else {
        for (int c = 0; c < copies; ++c)
            s += hist[bin * copies + c];
    }
    return s;
}

}  // namespace ep
