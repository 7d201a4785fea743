// pack.hip -- dispatch pack for gfx950: packed[slot_pos[t*k+j]][:] = x[t][:].
//
// A DMA engine moves only contiguous regions, so the rows a destination needs are first
// gathered into one contiguous segment per destination (Sec. 2.2 of the paper).  The
// kernel is HBM-bound: it reads each token row once and writes it k times.
//
// Mapping: a row of V 16-byte vectors is G groups of 64 (one vector per lane); a wave moves
// one chunk of U groups (all its loads in flight together) of one (token, slot): a single
// destination row.  Consecutive lanes touch consecutive 16-byte pieces: every load and store
// is a fully coalesced 1 KiB wave access.  The k waves of a chunk sit in one workgroup (up
// to 16): its loads after the first come from L2 (cached loads), and each wave feeds one
// write stream instead of k (against one wave storing its chunk k times, MI355X, inputs
// outside the memory-side cache: 3001 tokens, top-3 of 12 KiB rows 22.1 against 29.5 us, 6.7
// TB/s; top-2 of 4112 B rows, 4001 tokens 9.3 against 10.7 us).  Whole layouts of top-1 and small
// ones of top-2 take a wave per (token, chunk) instead (pack_token_waves).
// Rows that are no whole number of 128-byte lines: groups are counted from the line that
// holds the destination row's start, so that only the row's first and last stores touch
// partly filled lines, and only those lanes are masked (5003 tokens, top-6 of 5776 B rows:
// 38.4 against 42.7 us with groups counted from the row's start, whose every store splits two
// lines).
// Chunk: the largest divisor of G of at most 16 groups (16 KiB): a whole row for rows up to
// 16 KiB; long exact chunks measured faster than 4-group chunks and than 16-group chunks
// with guarded tails.  Rows with no divisor of 4 to 16 groups (G a prime above 16, 34, 51) use
// 16-group chunks whose last may be shorter.
// Stores: see pack_policy.  Rows carry no reuse across workgroups, so the
// workgroup-to-XCD placement needs no remapping.
#include "ep_internal.h"

namespace ep {
namespace {

struct PackGeom {
    int32_t V;          // 16-byte vectors per row
    int32_t gpc;        // groups per chunk (<= the kernel's U)
    int32_t G;          // groups of 64 vectors per row
    uint32_t lead_mask; // 7 where rows are no whole number of 128-byte lines, else 0
    FastDiv chunks;     // chunks per row
    FastDiv k;          // top-k
};

// How a row's groups meet its ends.
enum Edge {
    kWhole,    // rows are whole groups and chunks whole numbers of U groups
    kPartial,  // chunks whole numbers of U groups; the row's first and last groups may be
               // partly filled
    kRagged,   // the last chunk may have fewer groups, too
};

// The chunk of U groups number `chunk` of a row, one 16-byte vector of each group per lane.
// Groups are counted from `lead` vectors before the destination row's start, where a 128-byte
// line starts, so that every store but the row's first and last covers whole lines.
template <int U, int EDGE>
struct Chunk {
    const int32_t lane, g0, lead, ng, V;
    __device__ __forceinline__ Chunk(const PackGeom &pg, int32_t chunk, int lane, int32_t lead)
        : lane(lane), g0(chunk * pg.gpc), lead(EDGE == kWhole ? 0 : lead),
          ng(EDGE == kRagged ? min(pg.gpc, pg.G - g0) : U), V(pg.V) {}
    // this lane's vector of group u (outside the row at its ends).  Written so that every
    // load's address is computed apart from the others' (lane < 64: an OR): the loads of a
    // wave then issue in pairs some ten instructions apart, among those of the other waves of
    // the workgroup, which read the same row.  Addresses as one base and constant offsets,
    // all loads back to back, measured 7% slower: the prefill pack (top-8 of 14 KiB rows)
    // 815 against 757 us, 12000 tokens 295 against 274 (4 KiB and 8 KiB rows the same).
    __device__ __forceinline__ int32_t vector(int u) const { return (((g0 + u) * kWave) | lane) - lead; }
    // whether group u may reach past the row's ends: in the first group, and in the last two
    // (the row's end moves back by up to seven lanes with the lead)
    static constexpr bool edge(int u) { return EDGE == kRagged || (EDGE == kPartial && (u == 0 || u >= U - 2)); }
    // vector of the row that this lane loads for group u: always inside the row
    __device__ __forceinline__ int32_t load_index(int u) const {
        const int32_t v = vector(EDGE == kRagged ? min(u, ng - 1) : u);
        return edge(u) ? max(0, min(v, V - 1)) : v;
    }
    __device__ __forceinline__ bool store_ok(int u) const {
        return !edge(u) || (u < ng && (uint32_t)vector(u) < (uint32_t)V);
    }
    template <class Store>
    __device__ __forceinline__ void store(const u32x4 (&d)[U], u32x4 *row) const {
        if constexpr (EDGE == kWhole) {  // constant offsets from the chunk's start
            const Store dst(row + g0 * kWave, (uint32_t)(V - g0 * kWave) * 16u);
#pragma unroll
            for (int u = 0; u < U; ++u)
                dst.put(d[u], u * kWave + lane);
        } else {
            const Store dst(row, (uint32_t)V * 16u);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (store_ok(u))
                    dst.put(d[u], vector(u));
        }
    }
};

// The arrays are arguments of their own (restrict-qualified: the positions are then scalar
// loads; with vector loads the 32768-token, top-8 pack of 14 KiB rows took 804 us, so 752).
struct PackArgs {
    uint32_t T;  // tokens of this launch
    int32_t k;
    PackGeom geom;
    int64_t max_rows;
    uint32_t *epoch_word;
    uint32_t epoch;
    RoundSel sel;
    bool fence_system;
    // Before anything else: the round's epoch, and the buffer it selects.
    __device__ __forceinline__ u32x4 *begin(u32x4 *packed) const {
        if (epoch_word && blockIdx.x == 0 && threadIdx.x == 0)
            *epoch_word = epoch;
        if (sel.round && (__hip_atomic_load(sel.round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 1u))
            return static_cast<u32x4 *>(const_cast<void *>(sel.alt));
        return packed;
    }
};

// One wave per (token, chunk, slot), the k waves of a chunk adjacent: each wave writes a
// single destination row.  ONCE: k == 1, the row is read once (non-temporal loads).
template <int U, int EDGE, int SP, bool ONCE>
__global__ __launch_bounds__(1024) void pack_kernel(const u32x4 *__restrict__ x,
                                                    const int32_t *__restrict__ slot_pos,
                                                    u32x4 *__restrict__ packed_rows, PackArgs a) {
    u32x4 *const packed = a.begin(packed_rows);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t item = blockIdx.x * (blockDim.x / kWave) + wave;
    const uint32_t tc = ONCE ? item : a.geom.k.div(item), j = ONCE ? 0 : item - tc * a.k;
    const uint32_t t = a.geom.chunks.div(tc);
    if (t >= a.T)
        return;
    const int64_t p = slot_pos[(int64_t)t * a.k + j];
    if (p < 0 || p >= a.max_rows)
        return;
    u32x4 *const row = packed + p * a.geom.V;
    const int32_t lead = (int32_t)((uint32_t)(reinterpret_cast<uint64_t>(row) >> 4) & a.geom.lead_mask);
    const Chunk<U, EDGE> c(a.geom, (int32_t)(tc - t * a.geom.chunks.d), threadIdx.x & (kWave - 1), lead);
    const u32x4 *src = x + (int64_t)t * c.V;
    u32x4 d[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const u32x4 *v = src + c.load_index(u);
        d[u] = ONCE ? __builtin_nontemporal_load(v) : *v;
    }
    c.template store<RowStore<SP>>(d, row);
    if (a.fence_system)
        __threadfence_system();
}

// One wave per (token, chunk): the chunk is loaded once (non-temporal), before the positions
// are known, and stored to its token's rows.  Whole groups only (pack_token_waves).
template <int U, int SP>
__global__ __launch_bounds__(256) void pack_token_kernel(const u32x4 *__restrict__ x,
                                                         const int32_t *__restrict__ slot_pos,
                                                         u32x4 *__restrict__ packed_rows, PackArgs a) {
    u32x4 *const packed = a.begin(packed_rows);
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t item = blockIdx.x * (blockDim.x / kWave) + wave;
    const uint32_t t = a.geom.chunks.div(item);
    if (t >= a.T)
        return;
    const int32_t v0 = (int32_t)(item - t * a.geom.chunks.d) * (U * kWave);
    const u32x4 *src = x + (int64_t)t * a.geom.V + v0 + lane;
    u32x4 d[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
        d[u] = __builtin_nontemporal_load(src + u * kWave);
    const int32_t *sp = slot_pos + (int64_t)t * a.k;
    for (int32_t j = 0; j < a.k; ++j) {
        const int64_t p = sp[j];
        if (p < 0 || p >= a.max_rows)
            continue;
        const RowStore<SP> dst(packed + p * a.geom.V + v0, (uint32_t)(a.geom.V - v0) * 16u);
#pragma unroll
        for (int u = 0; u < U; ++u)
            dst.put(d[u], u * kWave + lane);
    }
    if (a.fence_system)
        __threadfence_system();
}

struct PackPtrs {
    const u32x4 *x;
    const int32_t *slot_pos;
    u32x4 *packed;
};

template <int U, int EDGE, int SP>
void launch_pack_u(dim3 grid, dim3 block, hipStream_t stream, TraceSlot ts, const PackPtrs &p,
                   const PackArgs &a, bool token_waves) {
    if constexpr (EDGE == kWhole)
        if (token_waves) {
            hipExtLaunchKernelGGL((pack_token_kernel<U, SP>), grid, block, 0, stream, ts.start, ts.stop, 0, p.x,
                                  p.slot_pos, p.packed, a);
            return;
        }
    if (a.k == 1)
        hipExtLaunchKernelGGL((pack_kernel<U, EDGE, SP, true>), grid, block, 0, stream, ts.start, ts.stop, 0, p.x,
                              p.slot_pos, p.packed, a);
    else
        hipExtLaunchKernelGGL((pack_kernel<U, EDGE, SP, false>), grid, block, 0, stream, ts.start, ts.stop, 0, p.x,
                              p.slot_pos, p.packed, a);
}

constexpr int kMaxU = 16;  // longest chunk: 16 KiB

// Launches the instance for chunks of `u` whole groups (0: the ragged instance).
template <int SP, int U = kMaxU>
void launch_chunk(int u, bool partial, dim3 grid, dim3 block, hipStream_t stream, TraceSlot ts,
                  const PackPtrs &p, const PackArgs &a, bool token_waves) {
    if (u == 0)
        return launch_pack_u<kMaxU, kRagged, SP>(grid, block, stream, ts, p, a, token_waves);
    if (u != U) {
        if constexpr (U > 1)
            launch_chunk<SP, U - 1>(u, partial, grid, block, stream, ts, p, a, token_waves);
        return;
    }
    if (partial)
        launch_pack_u<U, kPartial, SP>(grid, block, stream, ts, p, a, token_waves);
    else
        launch_pack_u<U, kWhole, SP>(grid, block, stream, ts, p, a, token_waves);
}

// Store policy of a launch whose slots' rows of row_bytes make up `bytes` bytes, by the time of
// whole passes (layout, pack, combine), since what a policy leaves in the caches is paid for by
// the next kernel.  Measured on MI355X, non-temporal / kStoreWT / kStoreWTStream:
//   rows of whole 64-byte pieces: 52 MiB of 2 KiB rows 33.9 / 38.2 / 33.8 us, 268 MiB of 4 KiB
//     rows 109.2 / 121.4 / 108.2; of 14 KiB rows 437 MiB 190.6 / 199 / 190.3, 875 MiB 398 / 388 /
//     391, 1312 MiB 564 / 556 / 553, 2187 MiB 970 / 947 / 960, 3584 MiB 1525 / 1489 / 1484;
//   other rows, whose ends share a cache line with their neighbours': non-temporal at any size.
//     93 MiB of 8208 B rows 54 / 71 / 62; 875 MiB of 14352 B rows 435 / 520 / 484, 2189 MiB 1069 / 1330
//     / 1195; 17 MiB of 5776 B rows (500 tokens, top-6) in no cache 16.4 / 18.9 / 16.9, just written
//     18.7 / 20.7 / 19.2, 24 MiB of 2064 B rows (4001, top-3) 23.7 / 29.1 / 24.9.  Write-through is
//     ahead only where a program packs into the same buffers again at once (14.0 against 14.9, 20.9
//     against 22.5).
// A window layout packs only some of its slots' rows; there the policies are within 1% of each
// other (whole passes, non-temporal / kStoreWTStream: 28 MiB of 224 packed 31.0 / 31.0, 256 of 2048
// MiB 173.1 / 171.1, 448 of 3584 MiB 315.4 / 316.1), so the slots decide there too.
// Rows to host memory (graph rounds) go non-temporal.
int pack_policy(int64_t bytes, int64_t row_bytes, bool to_host) {
    return to_host || row_bytes % 64 != 0 || bytes < (128ll << 20) ? kStoreNT : kStoreWTStream;
}

// Whether a wave takes a token's chunk for all its rows, not for one.  Its loads need not wait
// for a position, but rows of absent slots are read too, so only where every slot is expected
// to have a row.  Measured on MI355X, pack and combine of rows in no cache, a wave per token / per
// slot: top-1 of 12 KiB rows, 2000 tokens 19.6 / 21.0 us (the pack 9.8 / 10.9); top-2 of 12 KiB, 2000
// tokens 26.6 / 29.6, of 14 KiB, 1000 tokens 16.8 / 18.6; whole passes of top-2: of 12 KiB rows 47 MiB
// packed 31.0 / 33.8, 117 MiB 73.6 / 65.0, of 8 KiB 94 MiB (pack and combine) 52.4 / 48.2.  In a window of
// a quarter of the slots the pack alone takes 75 / 42 (top-2, 32768 tokens of 8 KiB rows) and 29 / 16 us
// (top-1, 16384).
bool pack_token_waves(int32_t k, int32_t H, int64_t bytes, Slots expect) {
    return expect != Slots::kSome && H % (8 * kWave) == 0 && (k == 1 || (k == 2 && bytes < (80ll << 20)));
}

}  // namespace

hipError_t launch_pack(const void *x, int64_t T, int32_t H, int32_t k, const int32_t *slot_pos,
                       void *packed, int64_t max_rows, uint32_t *epoch_word, uint32_t epoch,
                       hipStream_t stream, Slots expect, RoundSel sel, bool fence_system) {
    if (T == 0)
        return hipSuccess;
    const int64_t bytes = T * k * (int64_t)H * 2;  // of every slot's row
    const int32_t V = H / 8, lead_mask = V % 8 ? 7 : 0, G = (V + lead_mask + kWave - 1) / kWave;
    // chunk length: the largest divisor of G, no short chunks for long rows (0: ragged)
    int u = std::min(G, kMaxU);
    while (G % u != 0)
        --u;
    if (u < std::min(G, 4))
        u = 0;
    const bool token_waves = u != 0 && pack_token_waves(k, H, bytes, expect);  // exact chunks
    const int32_t slot_waves = token_waves ? 1 : k;                            // per chunk of a token
    // few tokens: shorter chunks, so that the launch keeps about 1024 waves (measured on
    // MI355X, top-2 of 14 KiB rows: 128 tokens 2.8 against 3.8 us, 512 tokens 5.5 against 6.0)
    for (int v = u - 1; v >= 1 && T * slot_waves * (G / u) < 1024; --v)
        if (G % v == 0)
            u = v;
    PackArgs a;
    a.geom.V = V;
    a.geom.G = G;
    a.geom.lead_mask = (uint32_t)lead_mask;
    a.geom.gpc = u ? u : kMaxU;
    a.geom.chunks = fast_div((uint32_t)((G + a.geom.gpc - 1) / a.geom.gpc));
    a.geom.k = fast_div((uint32_t)k);
    a.k = k;
    a.max_rows = max_rows;
    a.epoch_word = epoch_word;
    a.epoch = epoch;
    a.sel = sel;
    a.fence_system = fence_system;
    // per-slot waves of one token chunk share its row through L2 only inside one workgroup
    // (consecutive workgroups run on different XCDs, each with its own L2): a workgroup of k
    // waves holds them all, so the row is fetched from HBM once (4-wave workgroups fetched
    // it twice at k = 8; measured on MI355X)
    const int waves = slot_waves >= 2 && slot_waves <= 16 ? slot_waves : 4;
    const int64_t waves_per_token = (int64_t)a.geom.chunks.d * slot_waves;
    // launches of at most 2^31 waves (what FastDiv divides); one for any real layer
    const int64_t per = std::min<int64_t>(T, (INT32_MAX - waves) / waves_per_token);
    if (per < 1)
        return hipErrorInvalidValue;
    (void)hipGetLastError();  // drop an error left by an earlier, already reported call
    const TraceSlot ts = trace_acquire();
    const int policy = pack_policy(bytes, V * 16, sel.round != nullptr);
    for (int64_t t0 = 0; t0 < T; t0 += per) {
        a.T = (uint32_t)std::min(per, T - t0);
        const PackPtrs p{static_cast<const u32x4 *>(x) + t0 * V, slot_pos + t0 * k, static_cast<u32x4 *>(packed)};
        const dim3 grid((unsigned)((a.T * waves_per_token + waves - 1) / waves)), block(waves * kWave);
        TraceSlot part;
        part.start = t0 == 0 ? ts.start : nullptr;
        part.stop = t0 + a.T == T ? ts.stop : nullptr;
        if (policy == kStoreWTStream)
            launch_chunk<kStoreWTStream>(u, V % kWave != 0, grid, block, stream, part, p, a, token_waves);
        else
            launch_chunk<kStoreNT>(u, V % kWave != 0, grid, block, stream, part, p, a, token_waves);
    }
    const hipError_t err = hipGetLastError();
    if (err == hipSuccess)
        trace_submit("pack", ts);
    return err;
}

}  // namespace ep
