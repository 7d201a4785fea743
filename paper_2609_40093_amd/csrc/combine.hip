// combine.hip -- gate-weighted top-k combine for gfx950:
//   out[t][:] = sum_{j<k} w[t*k+j] * recv[slot_pos[t*k+j]][:]
// The returned contributions of a token are added on the GPU that owns the token
// (Sec. 4.3 of the paper: a DMA engine cannot add, so the reduction stays on the GPU),
// which also returns the rows to token order.
//
// Arithmetic: fp32 accumulator, fused multiply-add per slot in order j = 0..k-1 starting
// from +0, then one round-to-nearest-even conversion to bf16 (v_cvt_pk_bf16_f32), or the
// fp32 accumulator itself.  HBM-bound: k row reads and one row write per token.
//
// Mapping: one wave per (token, column chunk); the k slot positions and gates are
// wave-uniform scalar loads.  Slots are taken KC at a time (all k at once up to 8).  Where
// every slot of a batch has a row, all KC*U row loads are issued before the FMAs and
// nothing is conditional.  Otherwise (a window layout: most slots name other ranks'
// experts) only the rows that exist are read, in slot order, up to four at a time; a slot
// without a row adds nothing.  Reading row 0 for such slots instead, with its bits masked,
// took 19.7 us at 2048 gathered tokens of 14 KiB rows with one slot of 8 in the window
// (this: 10.5 us, 5.6 TB/s) and 155 us at 65536 tokens of 4 KiB rows (85 us, 6.3 TB/s).
// A lane loads what makes one 16-byte vector of the output, so the stores of a wave are
// contiguous also for fp32 results (16-byte loads and two stores 32 bytes apart per lane:
// 31.5 us at 2047 tokens, top-4 of 10 KiB rows to fp32; this: 19.6 us, 6.4 TB/s).
// In EXACT instances (rows a whole number of chunks) no lane carries a bounds mask.
// Rows are read once: loads are non-temporal.  Stores are device-scope write-through
// buffer stores when the output is small (write_through_below) and non-temporal from there
// up (RowStore); from 128 MiB up the call runs as launches of about 64 MiB of output
// each (see the launcher).
#include "ep_internal.h"

namespace ep {
namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const bf16x2 b = __builtin_convertvector(f32x2{lo, hi}, bf16x2);
    return __builtin_bit_cast(uint32_t, b);
}

// What one lane moves of a row per load: enough input elements for one 16-byte vector of
// the output (8 bf16, or 4 bf16 widened to fp32), so that a wave's stores are contiguous
// kilobytes for both output types.
template <bool F32_OUT>
struct Unit {
    typedef u32x4 In;
    static constexpr int kWords = 4;
};
template <>
struct Unit<true> {
    typedef uint32_t In __attribute__((ext_vector_type(2)));
    static constexpr int kWords = 2;
};

// Adds N rows (the slots of the N lowest bits of `slots`, which are cleared) to acc, in
// slot order, every load of the N rows issued before the first FMA.
template <int N, int U, bool F32_OUT, bool EXACT>
__device__ __forceinline__ void add_slots(float (&acc)[U][2 * Unit<F32_OUT>::kWords],
                                          const typename Unit<F32_OUT>::In *recv, const int32_t *sp, const float *wt,
                                          uint32_t &slots, int32_t v0, int lane, int32_t V) {
    constexpr int kW = Unit<F32_OUT>::kWords;
    typename Unit<F32_OUT>::In d[N][U];
    float g[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int j = __builtin_ctz(slots);
        slots &= slots - 1;
        const typename Unit<F32_OUT>::In *src = recv + (int64_t)sp[j] * V;
        g[i] = wt[j];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t v = v0 + u * kWave + lane;
            d[i][u] = __builtin_nontemporal_load(src + (EXACT ? v : min(v, V - 1)));
        }
    }
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < kW; ++q) {
                acc[u][2 * q] = __builtin_fmaf(g[i], bf16_lo(d[i][u][q]), acc[u][2 * q]);
                acc[u][2 * q + 1] = __builtin_fmaf(g[i], bf16_hi(d[i][u][q]), acc[u][2 * q + 1]);
            }
}

// FIXED_K: k == KC (one batch of slots, its bounds known at compile time).  SEL: the
// receive buffer is chosen by a round counter in device memory (graph-replayed rounds);
// without it the kernel loads nothing before the slot positions.  V: units per row.
template <int U, int KC, bool F32_OUT, bool EXACT, bool FIXED_K, bool SEL, bool WT>
__global__ __launch_bounds__(256) void combine_kernel(const void *__restrict__ recv_rows,
                                                      const int32_t *__restrict__ slot_pos,
                                                      const float *__restrict__ topk_w, uint32_t T,
                                                      int32_t V, FastDiv chunks, int32_t k,
                                                      void *__restrict__ out, int64_t max_rows,
                                                      RoundSel sel) {
    typedef typename Unit<F32_OUT>::In In;
    constexpr int kW = Unit<F32_OUT>::kWords;
    const int lane = threadIdx.x & (kWave - 1);
    if (SEL && (__hip_atomic_load(sel.round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 1u))
        recv_rows = sel.alt;
    const In *recv = static_cast<const In *>(recv_rows);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t item = blockIdx.x * (blockDim.x / kWave) + wave;
    const uint32_t t = chunks.div(item);
    if (t >= T)
        return;
    const int32_t v0 = (int32_t)(item - t * chunks.d) * (U * kWave);
    const int32_t kk = FIXED_K ? KC : k;

    float acc[U][2 * kW];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < 2 * kW; ++q)
            acc[u][q] = 0.0f;

    for (int32_t j0 = 0; j0 < kk; j0 += KC) {
        const int32_t *sp = slot_pos + (int64_t)t * kk + j0;  // wave-uniform: scalar loads
        const float *wt = topk_w + (int64_t)t * kk + j0;
        int32_t p[KC];
        uint32_t slots = 0;  // the batch's slots that have a row
#pragma unroll
        for (int j = 0; j < KC; ++j) {
            p[j] = FIXED_K || j0 + j < kk ? sp[FIXED_K ? j : min(j, kk - j0 - 1)] : -1;
            slots |= p[j] >= 0 && p[j] < max_rows ? 1u << j : 0u;
        }
        if (slots == (1u << KC) - 1u) {
            // every slot has a row: all loads, then the gates (needed only by the FMAs)
            In d[KC][U];
            float g[KC];
#pragma unroll
            for (int j = 0; j < KC; ++j) {
                const In *src = recv + (int64_t)p[j] * V;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int32_t v = v0 + u * kWave + lane;
                    d[j][u] = __builtin_nontemporal_load(src + (EXACT ? v : min(v, V - 1)));
                }
            }
#pragma unroll
            for (int j = 0; j < KC; ++j)
                g[j] = wt[j];
#pragma unroll
            for (int j = 0; j < KC; ++j)
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int q = 0; q < kW; ++q) {
                        acc[u][2 * q] = __builtin_fmaf(g[j], bf16_lo(d[j][u][q]), acc[u][2 * q]);
                        acc[u][2 * q + 1] = __builtin_fmaf(g[j], bf16_hi(d[j][u][q]), acc[u][2 * q + 1]);
                    }
            continue;
        }
        // only the slots with a row, in slot order, up to four at a time (the count is
        // wave-uniform, so each step's loads are all in flight together)
        while (KC > 4 && __builtin_popcount(slots) >= 4)
            add_slots<4, U, F32_OUT, EXACT>(acc, recv, sp, wt, slots, v0, lane, V);
        switch (__builtin_popcount(slots)) {
        case 3: add_slots<3, U, F32_OUT, EXACT>(acc, recv, sp, wt, slots, v0, lane, V); break;
        case 2: add_slots<2, U, F32_OUT, EXACT>(acc, recv, sp, wt, slots, v0, lane, V); break;
        case 1: add_slots<1, U, F32_OUT, EXACT>(acc, recv, sp, wt, slots, v0, lane, V); break;
        default: break;
        }
    }

    // the token's output row: V 16-byte vectors
    const RowStore<WT ? kStoreWT : kStoreNT> dst((u32x4 *)out + (int64_t)t * V, (uint32_t)V * 16u);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int32_t v = v0 + u * kWave + lane;
        if (!EXACT && v >= V)
            continue;
        u32x4 r;
        if constexpr (F32_OUT)
            r = u32x4{__float_as_uint(acc[u][0]), __float_as_uint(acc[u][1]), __float_as_uint(acc[u][2]),
                      __float_as_uint(acc[u][3])};
        else
            r = u32x4{pack_bf16x2(acc[u][0], acc[u][1]), pack_bf16x2(acc[u][2], acc[u][3]),
                      pack_bf16x2(acc[u][4], acc[u][5]), pack_bf16x2(acc[u][6], acc[u][7])};
        dst.put(r, (uint32_t)v);
    }
}

// Output bytes below which stores write through.  Such stores make the combine itself 1-9%
// faster at any size, but from about 44 MiB of output on the next pack pays for what they
// leave behind.  Measured on MI355X over whole passes (layout, pack, combine; buffers
// rotated past the memory-side cache), write-through / non-temporal: 27 MiB (top-8 of 14 KiB
// rows) 95.3 / 97.2 us, 35 MiB (top-2 of 8 KiB rows) 41.3 / 43.0, 41 MiB (top-8 of 14 KiB) 143.5 /
// 144.8, 42 MiB (top-2 of 8 KiB) 50.5 / 50.6, 47 MiB (top-8 of 14 KiB) 180 / 167.7, 50 MiB (top-2
// of 8 KiB) 65.5 / 58.4, 57 MiB (top-8 of 14 KiB) 211 / 191 (the pack 112 / 92).
constexpr int64_t kCombineWriteThroughBelow = 44ll << 20;
// After the one-kernel dispatch, whose row loads are non-temporal, the line lies higher for bf16
// results.  Write-through / non-temporal, rows in no cache: top-2 of 14 KiB rows 47 MiB 49.9 / 53.0
// us, 56 MiB 59.8 / 64.1; of 8 KiB 59 MiB 64.5 / 69.1; of 4 KiB 50 MiB 58.6 / 61.9; top-1 of 14 KiB 56
// MiB 39.1 / 43.4, of 8 KiB 59 MiB 42.6 / 47.1, 82 MiB 58.8 / 65.5; with the rows just written, top-2
// 56 MiB 74.9 / 78.5, top-1 82 MiB 85.5 / 83.3, 93 MiB 100 / 92.
constexpr int64_t kFusedWriteThroughBelow = 88ll << 20;
inline int64_t write_through_below(Slots expect, bool out_f32) {
    return expect == Slots::kFused && !out_f32 ? kFusedWriteThroughBelow : kCombineWriteThroughBelow;
}
// From 128 MiB of output up the combine runs as several launches over consecutive token
// ranges of about 64 MiB of output each (measured on MI355X, top-8 of 14 KiB rows, 32K
// tokens, non-temporal stores: one launch 747 us, 2 / 4 / 8 / 16 / 32 / 64 launches 733 /
// 727 / 718 / 719 / 748 / 801 us, and the layer's pack after it unchanged; the
// write-through stores of the smaller outputs made the following pack slower when applied
// to such launches).
constexpr int64_t kCombineSplitAbove = 128ll << 20;
constexpr int64_t kCombineLaunchBytes = 64ll << 20;

// LDS a workgroup reserves (and does not use) to limit the workgroups per compute unit, so
// that 80 to 128 KiB of row loads are in flight on each: a wave has loads_512 * 512 bytes in
// flight (five slots in one-unit chunks, at most 5 KiB a wave, are not limited).  More waves at
// once spread the reads over more rows and HBM pages.  A kernel on another stream gets in the
// sooner for it, though it finds little LDS free, because the waves' slots and registers stay
// free: beside the combine of 16384 tokens, top-8 of 14 KiB rows (370 us), limited / not, four
// 512 x 2048 x 4096 products end after 273 / 428 us, a layout after 30 / 96; full-chip products (4096^3)
// and the combine together take as long either way (1137 / 1138 us; 8 KiB rows 1014 / 1004, top-6 of 8192
// tokens 531 / 520).
// Measured on MI355X over whole passes, non-temporal regime, 4-wave workgroups per compute
// unit (none: as many as fit):
//   8 loads of 1 KiB (top-8, 14 KiB rows): 32768 tokens, skewed routing none / 4 / 3 / 2 1487 /
//     1477 / 1448 / 1466 us (the combine 722 -> 685, 6.2 TB/s), uniform 1554 / 1563 / 1545 / 1565;
//     4000 tokens, skewed 183.5 / 182.3 / 178.7 / 183.2;
//   16 (top-8, 8 KiB rows), 16384 tokens: 442.6 / 442.1 / 440.4 / 435.1;
//   14, 12, 10 (top-7, 6, 5, 14 KiB rows), 8192 tokens, none / 2: 359 / 352, 313.8 / 308.1, 266.8 /
//     262.5; 6 (top-6, 5776 B rows): none / 4 / 2 261 / 256 / 263.
// Up to four slots it measured no better (top-4: 491.6 / 490.8 / 491.5 / 494.4).
uint32_t reserved_lds(int32_t k, int loads_512) {
    if (k <= 4)
        return 0;
    const int groups = std::max(2, (48 + loads_512 / 2) / loads_512);  // 96 KiB over 4 waves, rounded
    if (groups > 4)
        return 0;
    return groups == 4 ? 40u << 10 : (groups == 3 ? 52u << 10 : 64u << 10);  // of 160 KiB
}

struct CombineCall {
    Slots expect;
    const void *recv;
    const int32_t *slot_pos;
    const float *topk_w;
    int64_t T;
    int32_t V, k;  // V: units (16-byte output vectors) per row
    void *out;
    int64_t max_rows;
    RoundSel sel;
};

// Launches one call as its token ranges.
template <int U, int KC, bool F32_OUT, bool EXACT, bool FIXED_K, bool SEL>
hipError_t launch_ranges(const CombineCall &c, hipStream_t stream) {
    constexpr int kWaves = 4;  // per workgroup
    const FastDiv chunks = fast_div((uint32_t)((c.V + U * kWave - 1) / (U * kWave)));
    const int64_t row_bytes = (int64_t)c.V * 16;
    const int64_t out_bytes = c.T * row_bytes;
    // token ranges of the launches: one below kCombineSplitAbove bytes of output or with
    // few rows to read, else about kCombineLaunchBytes each; never more items than FastDiv
    // divides
    const bool few_rows = c.max_rows <= c.T * c.k / 2;
    const int64_t launches = out_bytes < kCombineSplitAbove || few_rows
                                 ? 1
                                 : std::min<int64_t>(c.T, (out_bytes + kCombineLaunchBytes - 1) / kCombineLaunchBytes);
    const int64_t per = std::min<int64_t>((c.T + launches - 1) / launches, (INT32_MAX - kWaves) / chunks.d);
    if (per < 1)
        return hipErrorInvalidValue;
    const bool wt = out_bytes < write_through_below(c.expect, F32_OUT);
    const uint32_t lds = c.expect != Slots::kSome && !wt ? reserved_lds(c.k, (F32_OUT ? 1 : 2) * U * KC) : 0;
    (void)hipGetLastError();  // drop an error left by an earlier, already reported call
    const TraceSlot ts = trace_acquire();  // one pair of events around every launch of the call
    for (int64_t t0 = 0; t0 < c.T; t0 += per) {
        const int64_t n = std::min(per, c.T - t0);
        const dim3 grid((unsigned)((n * chunks.d + kWaves - 1) / kWaves)), block(kWaves * kWave);
        const hipEvent_t start = t0 == 0 ? ts.start : nullptr, stop = t0 + n == c.T ? ts.stop : nullptr;
        auto go = [&](auto kern) {
            hipExtLaunchKernelGGL(kern, grid, block, lds, stream, start, stop, 0, c.recv, c.slot_pos + t0 * c.k,
                                  c.topk_w + t0 * c.k, (uint32_t)n, c.V, chunks, c.k,
                                  static_cast<void *>(static_cast<char *>(c.out) + t0 * row_bytes), c.max_rows, c.sel);
        };
        wt ? go(combine_kernel<U, KC, F32_OUT, EXACT, FIXED_K, SEL, true>)
           : go(combine_kernel<U, KC, F32_OUT, EXACT, FIXED_K, SEL, false>);
    }
    const hipError_t err = hipGetLastError();
    if (err == hipSuccess)
        trace_submit("combine", ts);
    return err;
}

// Picks the instance for batches of KC slots.  U units per lane for bf16 results, 2U for
// fp32 results, whose units hold half as many elements of a row.
template <int U, int KC, bool FIXED_K>
hipError_t launch_u(const CombineCall &c, bool out_f32, bool exact, hipStream_t stream) {
    if (exact)
        return out_f32 ? launch_ranges<2 * U, KC, true, true, FIXED_K, false>(c, stream)
                       : launch_ranges<U, KC, false, true, FIXED_K, false>(c, stream);
    if constexpr (U == 1)  // the others are only used for whole rows
        return out_f32 ? launch_ranges<2, KC, true, false, FIXED_K, false>(c, stream)
                       : launch_ranges<1, KC, false, false, FIXED_K, false>(c, stream);
    return hipErrorInvalidValue;
}

// Chunk length, measured on MI355X (2000 tokens of 14 KiB rows, 4000 of 8 KiB, 9001 of
// 4112 B; bf16 and fp32 results): two-unit chunks where they cover the row exactly, within
// 1.5% of one-unit chunks or ahead of them for every k; one-unit chunks for other rows
// (4112 B rows, fp32: top-4 36.4 against 37.8 us, top-8 65.7 against 69.7) and for k >= 8
// with rows of at least 12 KiB (2% ahead at 32768 tokens); four for top-4 to bf16 where
// they are exact (25.4 against 26.0 us).  A batch of exactly k slots (k <= 8) beats batches
// of four and the rest (top-6, 4112 B rows: 43.4 against 44.9 us, fp32 53.9 against 61.8).
template <int KC, bool FIXED_K>
hipError_t launch_k(const CombineCall &c, int32_t H, bool out_f32, hipStream_t stream) {
    if constexpr (KC == 4)
        if (!out_f32 && H % 2048 == 0)
            return launch_u<4, KC, FIXED_K>(c, out_f32, true, stream);
    if (H % 1024 == 0 && !(KC == 8 && H >= 6144))
        return launch_u<2, KC, FIXED_K>(c, out_f32, true, stream);
    return launch_u<1, KC, FIXED_K>(c, out_f32, H % 512 == 0, stream);
}

// One pass of the per-sender accumulation (a combine that reduces each sender's returned
// rows as they land).  For a token and a set M of senders, p_M is the length of the
// longest prefix of its k slots whose rows all come from senders in M (a slot without a
// row belongs to every prefix; a row's sender is the rank segment holding it, rows past
// the last segment count as the last sender's).  Pass i adds the slots [p_prev, p_cur)
// for M = masks[i], masks[i + 1] -- in slot order, to the fp32 partial kept in `acc` (from
// +0 unless an earlier pass added a row of this token), by the very FMAs of
// combine_kernel -- and writes a token whose prefix is complete to `out`.  Sets only
// grow, so every slot is added once and in slot order: the result equals combine_kernel's
// bit for bit whatever order the senders arrive in.  A slot without a row is skipped:
// combine_kernel skips it too.  One wave per (token,
// 64-vector chunk).
template <bool F32_OUT>
__global__ __launch_bounds__(256) void accumulate_kernel(const u32x4 *__restrict__ recv,
                                                         const int32_t *__restrict__ slot_pos,
                                                         const float *__restrict__ topk_w, int64_t T, int32_t V,
                                                         int32_t chunks, int32_t k,
                                                         const int32_t *__restrict__ rank_offsets, int32_t R,
                                                         const uint32_t *__restrict__ masks, int32_t i,
                                                         float *__restrict__ acc, void *__restrict__ out,
                                                         int64_t max_rows) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t item = (int64_t)blockIdx.x * (blockDim.x / kWave) + wave;
    const int64_t t = item / chunks;
    if (t >= T)
        return;
    const int32_t v = (int32_t)(item - t * chunks) * kWave + lane;
    const bool vin = v < V;
    const int32_t ro = lane <= R ? rank_offsets[lane] : INT32_MAX;  // lane r: first row of rank r
    const uint32_t prev = masks[i], cur = masks[i + 1];
    const int32_t *sp = slot_pos + t * k;
    auto sender = [&](int64_t p) {  // the segment holding row p (wave-uniform p)
        return min((int)__popcll(__ballot(ro <= p)) - 1, R - 1);
    };
    int32_t pp = -1, pc = k;
    bool added_before = false;  // a row of this token went into acc in an earlier pass
    for (int32_t j = 0; j < k; ++j) {  // wave-uniform
        const int64_t p = sp[j];
        if (p < 0 || p >= max_rows)
            continue;
        const int r = sender(p);
        if (pp < 0) {
            if ((prev >> r) & 1u)
                added_before = true;
            else
                pp = j;
        }
        if (!((cur >> r) & 1u)) {
            pc = j;
            break;
        }
    }
    if (pp < 0) {  // every row of the token was in before this pass
        if (i != 0)
            return;    // written by an earlier pass
        pp = k;        // a token without rows: written by pass 0, as +0 (combine_kernel's sum)
    } else if (pc == pp) {
        return;
    }
    const int64_t o = t * V + (vin ? v : 0);
    float a[8];
    if (added_before && vin) {
        const u32x4 lo = reinterpret_cast<const u32x4 *>(acc)[2 * o];
        const u32x4 hi = reinterpret_cast<const u32x4 *>(acc)[2 * o + 1];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            a[q] = __uint_as_float(lo[q]);
            a[4 + q] = __uint_as_float(hi[q]);
        }
    } else {
#pragma unroll
        for (int q = 0; q < 8; ++q)
            a[q] = 0.0f;
    }
    for (int32_t j = pp; j < pc; ++j) {
        const int64_t p = sp[j];
        if (p < 0 || p >= max_rows)
            continue;
        const float g = topk_w[t * k + j];
        const u32x4 d = __builtin_nontemporal_load(recv + p * V + (vin ? v : 0));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            a[2 * q] = __builtin_fmaf(g, bf16_lo(d[q]), a[2 * q]);
            a[2 * q + 1] = __builtin_fmaf(g, bf16_hi(d[q]), a[2 * q + 1]);
        }
    }
    if (!vin)
        return;
    if (pc == k) {
        if constexpr (F32_OUT) {
            u32x4 *dst = (u32x4 *)out + 2 * o;
            __builtin_nontemporal_store(u32x4{__float_as_uint(a[0]), __float_as_uint(a[1]), __float_as_uint(a[2]),
                                              __float_as_uint(a[3])}, dst);
            __builtin_nontemporal_store(u32x4{__float_as_uint(a[4]), __float_as_uint(a[5]), __float_as_uint(a[6]),
                                              __float_as_uint(a[7])}, dst + 1);
        } else {
            const u32x4 r = {pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(a[4], a[5]),
                             pack_bf16x2(a[6], a[7])};
            __builtin_nontemporal_store(r, (u32x4 *)out + o);
        }
    } else {
        u32x4 *dst = reinterpret_cast<u32x4 *>(acc) + 2 * o;
        dst[0] = u32x4{__float_as_uint(a[0]), __float_as_uint(a[1]), __float_as_uint(a[2]), __float_as_uint(a[3])};
        dst[1] = u32x4{__float_as_uint(a[4]), __float_as_uint(a[5]), __float_as_uint(a[6]), __float_as_uint(a[7])};
    }
}

}  // namespace

hipError_t launch_combine(const void *recv, const int32_t *slot_pos, const float *topk_w,
                          int64_t T, int32_t H, int32_t k, void *out, bool out_f32,
                          int64_t max_rows, hipStream_t stream, Slots expect, RoundSel sel) {
    if (T == 0)
        return hipSuccess;
    const CombineCall c{expect, recv, slot_pos, topk_w, T, out_f32 ? H / 4 : H / 8, k, out, max_rows, sel};
    // Graph-replayed rounds: the general instance reading the round, for every k and row length:
    // PCIe bounds a round (with an instance per k before / this, compute-unit and SDMA legs: top-8 of
    // 14 KiB rows, 256 tokens 1178 / 1168 and 1129 / 1128 us, top-2 of 8 KiB, 4096 tokens 2533 / 2536 and
    // 2563 / 2560, top-2 of 2 KiB, 128 tokens 49.8 / 49.2 and 140 / 140).
    if (sel.round)
        return out_f32 ? launch_ranges<4, 8, true, false, false, true>(c, stream)
                       : launch_ranges<2, 8, false, false, false, true>(c, stream);
    switch (k) {
    case 1: return launch_k<1, true>(c, H, out_f32, stream);
    case 2: return launch_k<2, true>(c, H, out_f32, stream);
    case 3: return launch_k<3, true>(c, H, out_f32, stream);
    case 4: return launch_k<4, true>(c, H, out_f32, stream);
    case 5: return launch_k<5, true>(c, H, out_f32, stream);
    case 6: return launch_k<6, true>(c, H, out_f32, stream);
    case 7: return launch_k<7, true>(c, H, out_f32, stream);
    case 8: return launch_k<8, true>(c, H, out_f32, stream);
    default:
        // Rows that are no whole number of two-unit chunks: two units all the same where that
        // leaves a wave per SIMD and more.  Measured on MI355X, one-unit / two-unit chunks: top-24, 4001
        // tokens of 2064 B rows 41.0 / 39.7 us, 2000 of 5776 B 53.3 / 51.5, top-64, 1500 of 5136 B 91.0 /
        // 88.5, top-16, 1000 of 6000 B 20.1 / 19.7; 500 of 1040 B 4.7 / 5.7, top-96, 500 of 3088 B 25.9 /
        // 29.6; fp32 results 42.7 / 46.8, 55.8 / 53.8, 93.5 / 93.5.
        if (!out_f32 && H % 1024 != 0 && H > 512 && H < 6144 && T * ((H + 1023) / 1024) >= 1536)
            return launch_ranges<2, 8, false, false, false, false>(c, stream);
        return launch_k<8, false>(c, H, out_f32, stream);
    }
}

hipError_t launch_accumulate(const void *recv, const int32_t *slot_pos, const float *topk_w, int64_t T, int32_t H,
                             int32_t k, const int32_t *rank_offsets, int32_t R, const uint32_t *masks, int32_t i,
                             float *acc, void *out, bool out_f32, int64_t max_rows, hipStream_t stream) {
    if (T <= 0)
        return hipSuccess;
    if (!recv || !slot_pos || !topk_w || !rank_offsets || !masks || !acc || !out || H % 8 != 0 || R < 1 ||
        R > 32 || i < 0)
        return hipErrorInvalidValue;
    const int32_t V = H / 8;
    const int32_t chunks = (V + kWave - 1) / kWave;
    const int64_t blocks = (T * chunks + 3) / 4;
    if (blocks > INT32_MAX)
        return hipErrorInvalidValue;
    (void)hipGetLastError();
    TraceSlot ts = trace_acquire();
    if (out_f32)
        hipExtLaunchKernelGGL(accumulate_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, stream, ts.start,
                              ts.stop, 0, (const u32x4 *)recv, slot_pos, topk_w, T, V, chunks, k, rank_offsets, R,
                              masks, i, acc, out, max_rows);
    else
        hipExtLaunchKernelGGL(accumulate_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, stream, ts.start,
                              ts.stop, 0, (const u32x4 *)recv, slot_pos, topk_w, T, V, chunks, k, rank_offsets, R,
                              masks, i, acc, out, max_rows);
    hipError_t err = hipGetLastError();
    if (err == hipSuccess)
        trace_submit("accumulate", ts);
    return err;
}

}  // namespace ep
