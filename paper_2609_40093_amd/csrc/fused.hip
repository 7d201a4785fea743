// fused.hip -- dispatch layout and pack in one kernel, for small expert counts.
//
// The layout (a stable counting sort of the T*k routing entries by expert, Sec. 4.3 of
// the paper) and the pack (each destination's rows gathered into one contiguous segment,
// Sec. 2.2) otherwise run as two kernels, and the layout's workgroups exchange their
// per-expert totals through memory.  With few experts every workgroup can afford to count
// all entries itself; that removes the exchange and the kernel boundary between layout
// and pack.  A workgroup of W waves owns W*tpw consecutive tokens (a run of tpw per
// wave); W is 4, 8 or 16 by the number of routing entries (each workgroup counts all of
// them, so fewer, larger workgroups for more entries; more, smaller ones for few -- less
// of the kernel waits on its last workgroups).  Below 1024 tokens a row is split over S
// waves instead (each moves 1/S of it; W = m*S for m tokens, one per S waves), so that
// the stores of few tokens still reach every compute unit:
//   A. each wave issues the loads of its first ids, then those of its first token row
//      (they do not depend on the layout; vector loads complete in order, so the ids
//      come first);
//   B. the workgroup counts all T*k entries (16-byte loads of 4 ids) with LDS atomic
//      adds into histograms of 16 neighbouring counters per expert, chosen by lane (wave.h),
//      the entries before its own range apart (vector and LDS work only: a ballot per id
//      would queue every wave of the compute unit on its one scalar unit);
//   C. the totals' exclusive scan (DPP; a lane per expert, or four consecutive experts
//      per lane above 64 experts) gives the expert offsets; workgroup 0 stores the
//      counts, offsets and rank counts/offsets;
//   D. wave 0 ranks the workgroup's own entries in flat order (ballot match-any and a
//      masked popcount, as the layout kernel does: stable), stores slot_pos / row_src and
//      keeps the rows in LDS;
//   E. each wave stores its tokens' rows (or its part of one) to their k packed rows (loads
//      and stores non-temporal; U groups of 64 16-byte vectors, one per lane, all loads in
//      flight together).  For k <= 2 the workgroup's rows are all in before it stores.
// One more workgroup checks the routing (an id outside [0,E), an expert twice in one token
// row) and stores the status word: in every workgroup beside the counting, with the 16
// copies as rows of counters in one LDS bank, the kernel took 9.0 us at 256 tokens, top-8 of
// 256 experts, 14 KiB rows (now 7.4), 20.4 at 2048 tokens, top-8 of 128, 4 KiB rows (16.7), 12.6
// at 8192 tokens, top-2 of 256, 1 KiB rows (8.6).
// Row loads: cached ones are found again only by a program that packs the same rows twice
// without writing them (8192 tokens, top-1 of 4 KiB rows: 23.6 us a layer against 26.6).  Where
// the rows have just been written, or are in no cache, they make the combine after the dispatch
// slower; written, packed and combined, cached / non-temporal: 1024 tokens, top-1 of 8 KiB rows 13.1
// / 12.2 us, 4096 tokens, top-2 of 8 KiB 44.8 / 43.4, 16384 tokens, top-1 of 8 KiB 148 / 134, 2048
// tokens, top-8 of 4 KiB 35.0 / 34.9.
// Rows in before stores (k <= 2, where reads are a third to a half of the traffic): the
// counting takes less time than the device's row loads, so a workgroup that stores at once
// mixes its writes with the others' reads.  Without / with the wait, layers with rows in no
// cache: 4096 tokens, top-2 of 8 KiB 34.6 / 33.7 us, top-1 of 256 experts 25.1 / 23.2, 1024 tokens,
// top-1 of 8 KiB 9.6 / 9.3; for more slots it is slower (1024 tokens, top-4 of 14 KiB 26.6 / 27.1).
// The outputs equal those of the layout kernel followed by the pack kernel, bit for bit.
// Workgroups never wait on each other, so nothing needs them resident together.
//
// Limits (the host falls back to the two kernels outside them): E <= 256 (four experts
// per lane in step C), k in {1, 2, 4, 8} (a token row inside one 4-id load, or two for
// top-8), T*k <= 65536 for E <= 64 and k <= 4, else T*k <= 16384 for rows up to 8 KiB and
// 8192 for longer ones (every workgroup reads and counts every id before its stores:
// beyond that the layout kernel's exchange of totals costs less), rows of 1, 2, 4, 8, 14
// or 16 groups (H = 512 * groups), under 136 MiB packed for k = 2 and under 120 for k = 4 and 8,
// a 16-byte aligned routing array.  The split runs of fewer than 1024 tokens keep the same limits.
#include "ep_internal.h"
#include "wave.h"

namespace ep {
namespace {

constexpr int kFMaxThreads = 16 * kWave;    // largest workgroup (16 waves)
constexpr int kFNarrowE = 64;                // experts with one lane each in step C
constexpr int kFMaxE = 4 * kWave;            // experts with four per lane (wide instances)
constexpr int64_t kFMaxSlots = 65536;        // T*k: every workgroup reads every id
// T*k for E > 64 or k = 8 (measured on MI355X: at 16384 ids the one kernel still wins
// with 4 KiB rows, 20-24 against 23-29 us, and loses with 14 KiB rows, 56 against 55 us)
constexpr int64_t kFMaxSlotsWide = 16384;    // rows of at most 8 KiB
constexpr int64_t kFMaxSlotsWideLong = 8192; // longer rows
// Bytes packed from which the two steps as their own kernels win (their pack gives every slot
// its own wave).  Measured on MI355X, whole passes, one kernel / two.  k >= 4: 64 MiB, top-8 of 4
// KiB rows 29.9 / 34.9 us; 112 MiB, top-8 of 14 KiB 50.6 / 52.6; 128 MiB, top-4 of 4 KiB 64.4 / 60.4,
// of 8 KiB 59.2 / 58.7.  k = 2, rows in no cache, and just written (the pack's cached row loads then
// cost what they cost the combine here, above): 128 MiB of 8 KiB rows 68.4 / 69.9, 84.6 / 89.9; 137
// MiB of 14 KiB 75.3 / 73.8, 91.2 / 94.5; 141 MiB of 8 KiB 79.5 / 77.0, 96.1 / 98.6; 160 MiB of 4 KiB
// 88.5 / 85.4, 111.4 / 109.3; 256 MiB of 4 KiB 153 / 136, 187 / 190; of 8 KiB 151 / 137, 180 / 189.
// k = 1 has no such limit.
constexpr int64_t kFMaxBytes = 120ll << 20, kFMaxBytesTop2 = 136ll << 20;
constexpr int kFMaxOwn = 256;                // entries one workgroup owns (LDS rows)
constexpr int kFOwnRounds = kFMaxOwn / kWave;
constexpr int kFBatch = 4;                   // 16-byte id loads in flight per lane
constexpr int kFMaxWaves = 4096;             // waves in flight over the device (16 per CU)
constexpr int64_t kFSplitBelow = 1024;       // tokens below which rows are split over waves

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

// Does a token row inside a 4-id group name an expert twice?  Ids outside [0,E) are not
// compared (they are errors of their own).
template <int K>
__device__ __forceinline__ bool row_repeats(i32x4 v, int E) {
    auto ok = [E](int id) { return (unsigned)id < (unsigned)E; };
    if constexpr (K == 2)
        return (ok(v[0]) && v[0] == v[1]) || (ok(v[2]) && v[2] == v[3]);
    else if constexpr (K == 4)
        return (ok(v[0]) && (v[0] == v[1] || v[0] == v[2] || v[0] == v[3])) ||
               (ok(v[1]) && (v[1] == v[2] || v[1] == v[3])) || (ok(v[2]) && v[2] == v[3]);
    else
        return false;
}

// Loads the 4-id groups qw + b*threads + lane of a batch: every load is issued (an index
// past the last whole group rereads that group; the caller masks it by index), so the
// compiler can count the loads in flight and wait for the ids alone.
__device__ __forceinline__ void load_ids(const i32x4 *q, int64_t full, int64_t qw, int lane, int threads,
                                         i32x4 *v) {
#pragma unroll
    for (int b = 0; b < kFBatch; ++b)
        v[b] = q[min(qw + (int64_t)b * threads + lane, full - 1)];
}

constexpr int kFCopies = 16;  // counters per bin of the LDS histograms (hist_index)

// Counts one id into an LDS histogram of ME + 1 bins; bin ME takes ids that name no expert.
template <int ME>
__device__ __forceinline__ void count_id(int id, bool in, int E, int *hist, int lane) {
    const int bin = in && (unsigned)id < (unsigned)E ? id : ME;
    atomicAdd(&hist[hist_index(bin, kFCopies, lane)], 1);
}

// Does any id of `a` (in [0,E)) equal one of `b`?  (The two halves of a top-8 row.)
__device__ __forceinline__ bool halves_repeat(i32x4 a, i32x4 b, int E) {
    bool r = false;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        r |= (unsigned)a[i] < (unsigned)E && (a[i] == b[0] || a[i] == b[1] || a[i] == b[2] || a[i] == b[3]);
    return r;
}

// The routing errors of all entries (an id outside [0,E), an expert twice in one token row),
// stored to the status word by one workgroup.  A thread holds whole rows: one 4-id group,
// or two neighbouring ones for top-8.
template <int K>
__device__ __forceinline__ void check_routing(const FusedArgs &a, int *s_err, int tid, int threads) {
    constexpr int kPer = K == 8 ? 2 : 1, kBatch = 4;  // groups per unit, units in flight
    if (tid == 0)
        *s_err = 0;
    __syncthreads();
    const i32x4 *q = reinterpret_cast<const i32x4 *>(a.topk_idx);
    const int64_t slots = a.T * K;
    const int32_t units = (int32_t)(slots / (4 * kPer));
    bool bad = false, dup = false;
    auto bad_id = [&](int id) { return (unsigned)id >= (unsigned)a.E; };
    for (int32_t u0 = tid; u0 < units; u0 += kBatch * threads) {
        i32x4 v[kBatch][kPer];
#pragma unroll
        for (int b = 0; b < kBatch; ++b)  // a unit past the last reads it again
#pragma unroll
            for (int h = 0; h < kPer; ++h)
                v[b][h] = q[(int64_t)min(u0 + b * threads, units - 1) * kPer + h];
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
#pragma unroll
            for (int h = 0; h < kPer; ++h) {
                dup |= row_repeats<K == 8 ? 4 : K>(v[b][h], a.E);
                bad |= bad_id(v[b][h][0]) || bad_id(v[b][h][1]) || bad_id(v[b][h][2]) || bad_id(v[b][h][3]);
            }
            if constexpr (K == 8)
                dup |= halves_repeat(v[b][0], v[b][1], a.E);
        }
    }
    const int64_t i = (int64_t)units * 4 * kPer + tid;  // the last 1..3 ids (whole rows: k <= 2)
    if (i < slots) {
        const int id = a.topk_idx[i];
        bad |= bad_id(id);
        if (K == 2 && tid == 0)
            dup |= !bad_id(id) && id == a.topk_idx[i + 1];  // the tail is one row
    }
    const uint32_t err = (__ballot(bad) ? kRoutingIdOutOfRange : 0u) | (__ballot(dup) ? kRoutingDuplicate : 0u);
    if ((tid & (kWave - 1)) == 0 && err)
        atomicOr(s_err, (int)err);
    __syncthreads();
    if (tid == 0)
        *a.status = (uint32_t)*s_err;
}

// MULTI: more ids than one batch of the workgroup's loads (the count loops).  Instances
// without the loop have only straight-line loads, so the compiler's waits stay exact and
// no wave waits for its token row before the count's barrier.  WIDE: more than 64
// experts (four per lane in step C).  U: groups per wave (the row's, or 1/split of them).
template <int U, int K, bool MULTI, bool WIDE>
__global__ __launch_bounds__(kFMaxThreads) void layout_pack_kernel(FusedArgs a, int32_t tpw, int32_t split) {
    constexpr int ME = WIDE ? kFMaxE : kFNarrowE;  // counters per copy
    constexpr int kHist = kFCopies * (ME + 1);
    __shared__ __align__(16) int s_rest[kHist];  // entries from this workgroup's on
    __shared__ __align__(16) int s_pre[kHist];   // entries before this workgroup's
    __shared__ int s_base[ME];
    __shared__ int s_off[WIDE ? ME + 1 : 1];
    __shared__ int s_pos[kFMaxOwn];
    __shared__ int s_err;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const int threads = blockDim.x, waves = threads / kWave;
    if (blockIdx.x == gridDim.x - 1)
        return check_routing<K>(a, &s_err, tid, threads);
    const int64_t slots = a.T * K;
    const int runs = waves / split;  // token runs of tpw tokens (split == 1: one per wave)
    const int64_t tok0 = (int64_t)blockIdx.x * runs * tpw;  // runs*tpw*K: a multiple of 4
    const int64_t tok1 = min(a.T, tok0 + (int64_t)runs * tpw);
    const int32_t col = (w % split) * U * kWave;  // this wave's first vector of a row
    const int64_t ent0 = tok0 * K, ent1 = tok1 * K;
    const int32_t V = a.H / 8;
    const u32x4 *x = static_cast<const u32x4 *>(a.x);
    const i32x4 *q = reinterpret_cast<const i32x4 *>(a.topk_idx);
    const int64_t full = slots / 4;  // whole 4-id groups; the 0..3 ids after them are the tail
    const int64_t stride = (int64_t)threads * kFBatch;

    // A. first ids, the own entries' ids (step D), then this wave's first token row (a
    //    wave past the workgroup's last token loads that token instead, storing nothing)
    i32x4 v[kFBatch];
    int64_t qw = (int64_t)w * kWave;
    if (full > 0)
        load_ids(q, full, qw, lane, threads, v);
    int own_id[kFOwnRounds];
#pragma unroll
    for (int r = 0; r < kFOwnRounds; ++r)
        own_id[r] = a.topk_idx[min(ent0 + r * kWave + lane, ent1 - 1)];  // masked by index in step D
    // the 0..3 ids after the whole 4-id groups (wave 0 counts them): loaded here, with the
    // rest, so that no load is left after the count (a load there would make every wave
    // wait for its token row before the count's barrier)
    const int64_t ti = full * 4 + lane;
    const int tail_id = a.topk_idx[min(ti, slots - 1)];
    const int64_t wtok = tok0 + (int64_t)(w / split) * tpw;
    u32x4 d[U];
    {
        const u32x4 *src = x + min(wtok, tok1 - 1) * V + col + lane;
#pragma unroll
        for (int u = 0; u < U; ++u)
            d[u] = __builtin_nontemporal_load(src + u * kWave);
    }
    for (int i = tid; i < kHist / 4; i += threads) {
        reinterpret_cast<i32x4 *>(s_rest)[i] = i32x4{0, 0, 0, 0};
        reinterpret_cast<i32x4 *>(s_pre)[i] = i32x4{0, 0, 0, 0};
    }
    __syncthreads();

    // B. count all entries into the LDS counters
    auto count_batch = [&](int64_t qb) {
#pragma unroll
        for (int b = 0; b < kFBatch; ++b) {
            const int64_t g = qb + (int64_t)b * threads;  // this round's first group
            if (g >= full)
                break;
            const int64_t qi = g + lane;
            // entries before this workgroup's: whole 4-id groups (ent0 is a multiple of 4)
            int *hist = qi * 4 < ent0 ? s_pre : s_rest;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                count_id<ME>(v[b][c], qi < full, a.E, hist, lane);
        }
    };
    // the first batch outside the loop: its wait leaves the token row's loads in flight
    if (qw < full)
        count_batch(qw);
    if (MULTI) {
        for (qw += stride; qw < full; qw += stride) {  // wave-uniform
            load_ids(q, full, qw, lane, threads, v);
            count_batch(qw);
        }
    }
    if (w == 0 && ti < slots)  // the tail: 1..3 ids
        count_id<ME>(tail_id, true, a.E, ti < ent0 ? s_pre : s_rest, lane);
    __syncthreads();
    if (WIDE) {  // fold the counters on every wave: totals to s_off, entries before to s_base
        for (int e = tid; e < a.E; e += threads) {
            const int p = hist_sum(s_pre, e, kFCopies, lane);
            s_base[e] = p;
            s_off[e] = p + hist_sum(s_rest, e, kFCopies, lane);
        }
        __syncthreads();
    }

    if (w == 0 && WIDE) {
        // C (wide). Lane l holds experts 4l..4l+3: their totals, one scan of the lanes'
        // sums, the offsets of each expert kept in LDS (read back by other lanes of this
        // wave only, in program order)
        int tot[4], pre[4], sum = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = 4 * lane + q;
            pre[q] = e < a.E ? s_base[e] : 0;
            tot[q] = e < a.E ? s_off[e] : 0;
            sum += tot[q];
        }
        const int incl = wave_inclusive_scan(sum);
        const int total = __shfl(incl, kWave - 1);
        int run = incl - sum;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = 4 * lane + q;
            if (e < a.E) {
                s_off[e] = run;
                s_base[e] = run + pre[q];
            }
            run += tot[q];
        }
        if (lane == 0)
            s_off[a.E] = total;
        __builtin_amdgcn_wave_barrier();  // the reads below follow every lane's writes
        if (blockIdx.x == 0) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (4 * lane + q < a.E)
                    a.expert_counts[4 * lane + q] = tot[q];
            const int L = a.E / a.R;
            for (int e = lane; e <= a.E; e += kWave)
                a.expert_offsets[e] = s_off[e];
            for (int r = lane; r <= a.R; r += kWave) {
                a.rank_offsets[r] = s_off[r * L];
                if (r < a.R)
                    a.rank_counts[r] = s_off[(r + 1) * L] - s_off[r * L];
            }
            if (lane == 0 && a.epoch_word)
                *a.epoch_word = a.epoch;
        }
    } else if (w == 0) {
        // C. totals, offsets; workgroup 0 stores the layout's counts and the status
        const int pre = lane < a.E ? hist_sum(s_pre, lane, kFCopies, lane) : 0;
        const int tot = lane < a.E ? pre + hist_sum(s_rest, lane, kFCopies, lane) : 0;
        const int incl = wave_inclusive_scan(tot);
        const int excl = incl - tot;
        const int total = __shfl(incl, kWave - 1);
        if (lane < a.E)
            s_base[lane] = excl + pre;
        if (blockIdx.x == 0) {
            if (lane < a.E)
                a.expert_counts[lane] = tot;
            if (lane <= a.E)  // lane E (< 64) holds the total too; E == 64 is stored below
                a.expert_offsets[lane] = excl;
            // rank r's first row: the exclusive offset of expert r*L (the total for r = R)
            const int L = a.E / a.R;
            auto offset_of = [&](int e) {
                const int v = __shfl(excl, min(e, kWave - 1));
                return e >= a.E ? total : v;
            };
            const int lo = offset_of(min(lane, a.R) * L);
            const int hi = offset_of(min(lane + 1, a.R) * L);
            if (lane < a.R)
                a.rank_counts[lane] = hi - lo;
            if (lane <= a.R)
                a.rank_offsets[lane] = lo;
            if (lane == 0) {
                if (a.E == kWave)
                    a.expert_offsets[kWave] = total;
                if (a.R == kWave)
                    a.rank_offsets[kWave] = total;
                if (a.epoch_word)
                    *a.epoch_word = a.epoch;
            }
        }
    }
    if (w == 0) {
        // D. rank the own entries in flat order (s_base as step C left it, written by this
        //    wave)
#pragma unroll
        for (int r = 0; r < kFOwnRounds; ++r) {
            const int64_t i = ent0 + r * kWave + lane;
            if (ent0 + r * kWave >= ent1)
                break;
            const int id = i < ent1 ? own_id[r] : -1;
            const bool valid = i < ent1 && (unsigned)id < (unsigned)a.E;
            const uint64_t m = match_expert(id, valid, a.nbits);
            int pos = -1;
            if (valid) {
                const int below = lanes_below(m);
                const int b = s_base[id];
                pos = b + below;
                if (below == 0)
                    s_base[id] = b + (int)__popcll(m);
            }
            if (i < ent1) {
                if ((uint64_t)(uint32_t)pos >= (uint64_t)slots)
                    pos = -1;  // cannot happen with consistent counts; keeps every store in bounds
                a.slot_pos[i] = pos;
                if (pos >= 0 && a.row_src)
                    a.row_src[pos] = (int32_t)i;
                s_pos[i - ent0] = pos;
            }
        }
    }
    if (K <= 2)
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): this wave's row is in
    __syncthreads();

    // E. store each token row (this wave's part of it) to its k packed rows
    u32x4 *packed = static_cast<u32x4 *>(a.packed);
    for (int j0 = 0; j0 < tpw; ++j0) {
        const int64_t t = wtok + j0;
        if (t >= tok1)
            break;
        if (j0 > 0) {
            const u32x4 *src = x + t * V + col + lane;
#pragma unroll
            for (int u = 0; u < U; ++u)
                d[u] = __builtin_nontemporal_load(src + u * kWave);
        }
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int64_t p = s_pos[(t - tok0) * K + j];
            if (p < 0 || p >= a.max_rows)
                continue;
            const RowStore<kStoreNT> dst(packed + p * V + col, (uint32_t)(V - col) * 16u);
#pragma unroll
            for (int u = 0; u < U; ++u)
                dst.put(d[u], u * kWave + lane);
        }
    }
}

template <int U, int K, bool MULTI, bool WIDE>
void launch_one(const FusedArgs &a, int32_t tpw, int32_t split, unsigned blocks, int threads, hipStream_t stream,
                TraceSlot ts) {
    hipExtLaunchKernelGGL((layout_pack_kernel<U, K, MULTI, WIDE>), dim3(blocks + 1), dim3(threads), 0, stream,
                          ts.start, ts.stop, 0, a, tpw, split);  // the last workgroup checks the routing
}

// Launches top-K's instance.  MULTI: whether the limits let these sizes have more ids than one
// batch of loads covers.
template <int U, int K, bool MULTI>
hipError_t launch_top(const FusedArgs &a, int32_t tpw, int32_t split, unsigned blocks, int threads,
                      hipStream_t stream, TraceSlot ts) {
    const bool multi = a.T * a.k > (int64_t)threads * kFBatch * 4;  // one batch: kFBatch 4-id groups per thread
    const bool wide = a.E > kFNarrowE;
    if (multi && (wide || !MULTI))
        return hipErrorInvalidValue;  // excluded by the limits
    if (wide)
        launch_one<U, K, false, true>(a, tpw, split, blocks, threads, stream, ts);
    else if (!multi)
        launch_one<U, K, false, false>(a, tpw, split, blocks, threads, stream, ts);
    else if constexpr (MULTI)
        launch_one<U, K, true, false>(a, tpw, split, blocks, threads, stream, ts);
    return hipSuccess;
}

// Picks the instance: the count loop only where one batch of loads does not cover every
// id (1024 threads x 16 ids: never within the limits of more than 64 experts or top-8, nor with
// so few bytes packed as top-2 may have in rows of 14 groups and top-4 in rows of 8), four
// experts per lane above 64 experts.
template <int U>
hipError_t launch_k(const FusedArgs &a, int32_t tpw, int32_t split, unsigned blocks, int threads, hipStream_t stream,
                    TraceSlot ts) {
    static_assert(kFMaxBytesTop2 / (14 * 1024) <= 16384 && kFMaxBytes / (8 * 1024) <= 16384, "see above");
    switch (a.k) {
    case 1: return launch_top<U, 1, true>(a, tpw, split, blocks, threads, stream, ts);
    case 2: return launch_top<U, 2, (U < 14)>(a, tpw, split, blocks, threads, stream, ts);
    case 4: return launch_top<U, 4, (U < 8)>(a, tpw, split, blocks, threads, stream, ts);
    default: return launch_top<U, 8, false>(a, tpw, split, blocks, threads, stream, ts);
    }
}

// Workgroups of one call.  Below kFSplitBelow tokens a row is split over the fewest waves
// S (dividing its G groups, with an instance for G/S groups) that make the call at least
// kFSplitBelow waves, else over the most; a workgroup holds m tokens (m*S waves: at least
// 4, and enough threads that one batch of id loads covers every id; at most 16; m*k a
// multiple of 4, since step B splits the ids before the workgroup's own at whole 4-id
// groups).  Split
// rows measured on MI355X, 256 experts top-8, 14 KiB rows: 256 tokens 9.8 against 11.4 us,
// 512 tokens 16.1 against 16.9 us.  Otherwise 4, 8 or 16 waves by the entries (4 or 8
// win up to 8192 entries, 16 above), with tpw tokens per wave so that the workgroups hold
// at most kFMaxWaves waves.  Top-1 takes 8 waves once they still give every compute unit a
// workgroup: more rows are then in before a store (4096 tokens of 8 KiB rows, layers with 4 / 8
// waves 24.4 / 23.7 us, fresh rows the same; 2048 tokens 14.2 / 14.2, fresh rows 19.4 / 19.2; 1024
// tokens 9.3 / 9.8).
struct FusedGeom {
    int32_t split = 1, waves = 4, tpw = 1;
    int64_t blocks = 0;
};

FusedGeom fused_geometry(int64_t T, int32_t k, int G) {
    FusedGeom g;
    const int64_t slots = T * k;
    const int64_t ids_per_wave = (int64_t)kWave * kFBatch * 4;  // one batch of 16-byte id loads
    if (T < kFSplitBelow) {
        int split = 1;
        for (int d : {2, 4, 7, 8, 14, 16}) {
            const int u = G % d == 0 ? G / d : 0;
            if (u == 1 || u == 2 || u == 4 || u == 8) {
                split = d;
                if (T * d >= kFSplitBelow)
                    break;
            }
        }
        if (split > 1) {
            int64_t m = split >= 4 ? 1 : 4 / split;
            m = std::max<int64_t>(m, (slots + split * ids_per_wave - 1) / (split * ids_per_wave));
            const int64_t q = k < 4 ? 4 / k : 1;  // m*k a multiple of 4
            m = (m + q - 1) / q * q;
            if (m * split <= 16) {
                g.split = split;
                g.waves = (int32_t)(m * split);
                g.tpw = 1;
                g.blocks = (T + m - 1) / m;
                return g;
            }
        }
    }
    g.waves = (k == 1 ? slots < 8 * 256 : slots <= 4096) ? 4 : (slots <= 8192 ? 8 : 16);
    const int64_t max_blocks = kFMaxWaves / g.waves;
    const int64_t per_block_min = (T + max_blocks - 1) / max_blocks;
    g.tpw = (int32_t)((per_block_min + g.waves - 1) / g.waves);
    g.blocks = (T + (int64_t)g.waves * g.tpw - 1) / ((int64_t)g.waves * g.tpw);
    return g;
}

}  // namespace

bool fused_layout_pack_fits(int64_t T, int32_t k, int32_t E, int32_t H, const void *topk_idx) {
    if (T < 1 || E < 1 || E > kFMaxE || k > E || !(k == 1 || k == 2 || k == 4 || k == 8))
        return false;
    const int64_t wide_limit = H <= 4096 ? kFMaxSlotsWide : kFMaxSlotsWideLong;
    if (T * k > (E > kFNarrowE || k == 8 ? wide_limit : kFMaxSlots))
        return false;
    if (H % 512 != 0)
        return false;
    if (k > 1 && T * k * (int64_t)H * 2 >= (k == 2 ? kFMaxBytesTop2 : kFMaxBytes))
        return false;
    const int G = H / 512;
    return (G == 1 || G == 2 || G == 4 || G == 8 || G == 14 || G == 16) &&
           reinterpret_cast<uintptr_t>(topk_idx) % 16 == 0;
}

hipError_t launch_layout_pack(const FusedArgs &a, hipStream_t stream) {
    if (!fused_layout_pack_fits(a.T, a.k, a.E, a.H, a.topk_idx) || a.R < 1 || a.E % a.R != 0)
        return hipErrorInvalidValue;
    const int G = a.H / 512;
    const FusedGeom g = fused_geometry(a.T, a.k, G);
    if ((int64_t)(g.waves / g.split) * g.tpw * a.k > kFMaxOwn || g.blocks > INT32_MAX)
        return hipErrorInvalidValue;  // excluded by the limits above
    (void)hipGetLastError();  // drop an error left by an earlier, already reported call
    TraceSlot ts = trace_acquire();
    const unsigned nb = (unsigned)g.blocks;
    const int threads = g.waves * kWave;
    hipError_t err;
    switch (G / g.split) {  // groups per wave
    case 1: err = launch_k<1>(a, g.tpw, g.split, nb, threads, stream, ts); break;
    case 2: err = launch_k<2>(a, g.tpw, g.split, nb, threads, stream, ts); break;
    case 4: err = launch_k<4>(a, g.tpw, g.split, nb, threads, stream, ts); break;
    case 8: err = launch_k<8>(a, g.tpw, g.split, nb, threads, stream, ts); break;
    case 14: err = launch_k<14>(a, g.tpw, g.split, nb, threads, stream, ts); break;
    default: err = launch_k<16>(a, g.tpw, g.split, nb, threads, stream, ts); break;
    }
    if (err != hipSuccess)
        return err;  // nothing was launched (unreachable within the limits)
    err = hipGetLastError();
    if (err == hipSuccess)
        trace_submit("layout_pack", ts);
    return err;
}

}  // namespace ep
