// layout.hip -- dispatch layout for gfx950: a stable counting sort of the T*k routing
// entries by expert id (rows grouped by expert, token order kept inside a group, groups
// in expert order, hence contiguous per destination rank).  Sec. 4.3 of the paper groups
// tokens by the experts that consume them; Sec. 4.5 sends each destination only its rows.
// The same kernels group only a window of experts (the receive side of the dense design,
// Sec. 4.2-4.3: a rank groups the tokens it gathered by the experts it owns); entries
// naming other experts get no row and are not errors.
//
// Two ways of counting:
//   histogram  where only totals matter: 16-byte loads of four ids, LDS atomic adds into
//              copies of the per-expert counters chosen by lane (wave.h).  Sums of whole
//              numbers: the order of the adds does not matter.
//   ranked     where an entry's position is needed: inside a wave, the lanes holding the
//              same expert are found with ceil(log2 E) 64-lane ballots ("match any"); a
//              lane's rank among them is a masked popcount (mbcnt).  One leader lane per
//              distinct expert adds the group's size to the wave's counter row in LDS;
//              every lane of the group reads the counter's old value first, so it learns
//              its rank among the wave's earlier entries of that expert at the same time.
//              No atomic decides any position: the result is deterministic.
//
// Few entries: one kernel.  Each workgroup owns a run of the entries, histograms all of
// them (those before its run apart), scans the totals and ranks its own run; one more
// workgroup checks the routing.
// More: two kernels, and no workgroup ever waits for another (so nothing depends on which
// workgroups the device runs at once):
//   count  one workgroup per tile of the routing array: the tile's histogram and routing
//          errors (ids outside [0,E), an expert twice in one token row), to the workspace.
//   rank   several workgroups per tile, each owning a run of it: sums every tile's counts
//          (a thread per run of tiles of an expert's column, 8 loads in flight), which
//          gives the expert totals and the rows of each expert in earlier tiles;
//          histograms the entries of its tile before its run; scans the totals; ranks its
//          run and writes every position: expert offset + rows of the expert in earlier
//          tiles and runs + in earlier waves + the entry's rank inside its wave.
// The first workgroup also writes the counts, offsets and status.  The kernel boundary
// orders the count kernel's stores before the rank kernel's loads: no fence, atomic or
// counter in memory is involved, so a layout captured in a graph replays as it runs.
// What bounds a layout is the length of its chain of dependent steps, and in it the
// instructions per compute unit (four waves of a 16-wave workgroup share a SIMD), not bytes:
// so histograms (about 7 instructions an id) rather than ballots (70 a round) wherever no
// position is needed, the routing checked once, by whole rows in registers, and small
// workgroups spread over every compute unit.  Measured on MI355X, layouts back to back,
// against counting everything with ballots in one 16-wave workgroup per tile: 2048 entries
// of 256 experts 4.6 us (before 7.2), 8188 of 64 5.2 (8.7), 65536 of 128 8.6 (10.8), 262144
// of 256 11.3 (17.0), 1M of 256 17.3 (49).
// Cross-tile traffic: tiles x E words written once, read by every rank workgroup (from L2
// after its XCD's first miss), and tiles error words read by the first.
#include "ep_internal.h"
#include "wave.h"

namespace ep {
namespace {

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

// --------------------------------------------------------------------- histogram

constexpr int kHistBatch = 4;    // 16-byte id loads in flight per thread

// Counters per expert: 16 up to 256 experts, 4 up to 512, else one (LDS).
__host__ __device__ constexpr int hist_copies(int E) { return E <= 256 ? 16 : (E <= 512 ? 4 : 1); }

// The 4-id groups a thread takes together, loaded ahead of their use.  PAIRS: the thread's
// groups are neighbours two by two (a top-8 token row each), else a workgroup's threads take
// neighbouring groups.
struct IdBatch {
    i32x4 v[kHistBatch];
};

template <bool PAIRS>
__device__ __forceinline__ uint32_t batch_group(uint32_t gw, int b, int threads) {  // lane 0's
    return gw + (PAIRS ? (b / 2) * 2 * threads + b % 2 : b * threads);
}

// Loads a batch from the array's first `full` groups (entries 4g..4g+3 of group g; a group
// past them rereads the last; full > 0).
template <bool PAIRS>
__device__ __forceinline__ void load_batch(const LayoutArgs &a, uint32_t gw, uint32_t full, int lane, int threads,
                                           IdBatch &ids) {
    const bool aligned = (reinterpret_cast<uintptr_t>(a.topk_idx) & 15) == 0;
#pragma unroll
    for (int b = 0; b < kHistBatch; ++b) {
        const uint32_t g = batch_group<PAIRS>(gw, b, threads) + (PAIRS ? 2 : 1) * lane;
        const int32_t *p = a.topk_idx + 4 * (int64_t)min(g, full - 1);
        if (aligned)
            ids.v[b] = *reinterpret_cast<const i32x4 *>(p);
        else
            ids.v[b] = i32x4{p[0], p[1], p[2], p[3]};
    }
}

// Lane 0's first group of [begin, end) for the wave of thread tid.
template <bool PAIRS>
__device__ __forceinline__ uint32_t first_group(uint32_t begin, int tid) {
    return begin / 4 + (PAIRS ? 2 : 1) * (tid & ~(kWave - 1));
}

// The first batch of visit_ids over [begin, end), loaded by the caller as early as it can.
template <bool PAIRS>
__device__ __forceinline__ void first_batch(const LayoutArgs &a, uint32_t begin, uint32_t end, int tid, int threads,
                                            IdBatch &ids) {
    if (end / 4 > begin / 4)
        load_batch<PAIRS>(a, first_group<PAIRS>(begin, tid), end / 4, tid & (kWave - 1), threads, ids);
}

__device__ __forceinline__ bool same_id(const LayoutArgs &a, int x, int y) {
    return x == y && (unsigned)x < (unsigned)a.all_E;
}

// Does any expert appear twice among the N ids of a token row?  (Ids outside [0, E) are
// errors of their own; the equality of the raw ids is tested first, rows that pass it are
// rare.)
template <int N>
__device__ __forceinline__ bool row_repeats(const LayoutArgs &a, const int (&id)[N]) {
    bool equal = false, dup = false;
#pragma unroll
    for (int x = 0; x < N; ++x)
#pragma unroll
        for (int y = x + 1; y < N; ++y)
            equal |= id[x] == id[y];
    if (equal) {
#pragma unroll
        for (int x = 0; x < N; ++x)
#pragma unroll
            for (int y = x + 1; y < N; ++y)
                dup |= same_id(a, id[x], id[y]);
    }
    return dup;
}

// Goes over the ids of the entries [begin, end).
// COUNT: counts them by expert, those before `split` into hist_pre, the rest into hist_all,
//   each E + 1 bins of hist_copies(E) counters in LDS, zeroed by the caller; bin E takes the
//   ids outside the window (no branch per id).
// CHECK: ORs their routing errors into err.  K: top-k when it is 1, 2, 4 or 8 (whole token
//   rows in a thread's groups; 8 with PAIRS), else 0 (repeated experts: check_rows).
// begin and split are multiples of 64, end too unless it is the array's.  ids: the first
// batch.
template <int K, bool PAIRS, bool COUNT, bool CHECK>
__device__ __forceinline__ void visit_ids(const LayoutArgs &a, uint32_t begin, uint32_t end, uint32_t split, int tid,
                                          int threads, int *hist_pre, int *hist_all, uint32_t &err, IdBatch &ids) {
    static_assert(!CHECK || PAIRS == (K == 8), "a top-8 row is a pair of groups");
    const int lane = tid & (kWave - 1);
    const int copies = hist_copies(a.E);
    bool bad = false, dup = false;
    auto visit = [&](int id, bool in, int *hist) {
        if (CHECK)
            bad |= in && (unsigned)id >= (unsigned)a.all_E;
        if (COUNT) {
            const int bin = (int)min((uint32_t)(in ? id - a.e_lo : -1), (uint32_t)a.E);
            atomicAdd(&hist[hist_index(bin, copies, lane)], 1);
        }
    };
    const uint32_t full = end / 4, step = threads * kHistBatch;  // whole 4-id groups
    for (uint32_t gw = first_group<PAIRS>(begin, tid); gw < full; gw += step) {  // wave-uniform
        IdBatch next;
        if (gw + step < full)
            load_batch<PAIRS>(a, gw + step, full, lane, threads, next);
#pragma unroll
        for (int b = 0; b < kHistBatch; ++b) {
            const uint32_t g0 = batch_group<PAIRS>(gw, b, threads), g = g0 + (PAIRS ? 2 : 1) * lane;
            if (g0 >= full)
                break;
            const bool in = g < full;
            const i32x4 v = ids.v[b];
            if (CHECK && in) {
                if (K == 2)
                    dup |= row_repeats<2>(a, {v[0], v[1]}) || row_repeats<2>(a, {v[2], v[3]});
                if (K == 4)
                    dup |= row_repeats<4>(a, {v[0], v[1], v[2], v[3]});
                if (K == 8 && b % 2 == 1) {  // the array holds whole rows: the pair is in together
                    const i32x4 u = ids.v[b - b % 2];
                    dup |= row_repeats<8>(a, {u[0], u[1], u[2], u[3], v[0], v[1], v[2], v[3]});
                }
            }
            int *hist = 4 * g < split ? hist_pre : hist_all;
#pragma unroll
            for (int c = 0; c < 4; ++c)
                visit(v[c], in, hist);
        }
        ids = next;
    }
    const uint32_t i = full * 4 + tid;  // the last 0..3 entries of the array
    if (i < end) {
        const int id = a.topk_idx[i];
        if (CHECK && K == 2 && tid == 0)
            dup |= same_id(a, id, a.topk_idx[i + 1]);  // an odd number of rows ends with one
        visit(id, true, i < split ? hist_pre : hist_all);
    }
    if (CHECK)
        err |= (bad ? kRoutingIdOutOfRange : 0u) | (dup ? kRoutingDuplicate : 0u);
}

// Routing check of general rows (K = 0): whether a token row that starts in [begin, end) names
// an expert twice (its last ids may lie past end: the array holds whole rows).  Three ways,
// whose cost per id hardly grows with k:
//   k < 8     a thread holds a row;
//   k <= 64   a wave holds as many whole rows as it has lanes for, finds the lanes with equal
//             ids by ballots and keeps those of its own row;
//   longer    a wave marks a row's experts in a bitmap (`seen`: an LDS word per thread).
// Measured on MI355X, whole layouts of 128 experts, against comparing each id with the row's
// earlier ones, loaded again: 4000 entries of top-16 6.2 us (10.9), top-32 6.2 (24.5), top-64 6.2
// (38.1), top-96 6.2 (52.9); 400000 entries of top-16 16.0 (22.7), top-64 16.3 (58.0), top-96 15.1
// (79.7); of 64 experts, top-6 12.3 (15.0), top-7 12.5 (16.0), where ballots take 14.4.
template <int N>
__device__ __forceinline__ bool rows_repeat(const LayoutArgs &a, uint32_t row, uint32_t row_end, uint32_t step) {
    bool dup = false;
    for (; row < row_end; row += step) {
        int id[N];
#pragma unroll
        for (int j = 0; j < N; ++j)
            id[j] = a.topk_idx[row * N + j];
        dup |= row_repeats<N>(a, id);
    }
    return dup;
}
constexpr int kCheckBatch = 4;  // id loads in flight per lane
__device__ __forceinline__ bool rows_repeat_ballots(const LayoutArgs &a, uint32_t begin_row, uint32_t row_end, int tid,
                                                    int threads) {
    const int lane = tid & (kWave - 1);
    const uint32_t k = a.k_div.d, rows = kWave / k;  // whole rows of a wave
    const uint32_t mine = a.k_div.div(lane), slot = lane - mine * k, step = threads / kWave * rows;
    const uint64_t row_lanes = (k == kWave ? ~0ull : (1ull << k) - 1) << (lane - slot);
    const int bits = a.all_E > 1 ? 32 - __builtin_clz(a.all_E - 1) : 0;
    bool dup = false;
    for (uint32_t r = begin_row + tid / kWave * rows; r < row_end; r += kCheckBatch * step) {  // wave-uniform
        int id[kCheckBatch];
#pragma unroll
        for (int b = 0; b < kCheckBatch; ++b) {
            const uint32_t row = r + b * step + mine;
            id[b] = mine < rows && row < row_end ? a.topk_idx[row * k + slot] : -1;
        }
#pragma unroll
        for (int b = 0; b < kCheckBatch; ++b) {
            if (r + b * step >= row_end)
                break;
            const bool ok = (unsigned)id[b] < (unsigned)a.all_E;
            dup |= ok && __popcll(match_expert(id[b], ok, bits) & row_lanes) > 1;
        }
    }
    return dup;
}
__device__ __forceinline__ bool rows_repeat_bitmap(const LayoutArgs &a, uint32_t begin_row, uint32_t row_end, int tid,
                                                   int threads, uint32_t *seen) {
    const int lane = tid & (kWave - 1);
    const uint32_t k = a.k_div.d;
    uint32_t *map = seen + (tid & ~(kWave - 1));  // this wave's
    bool dup = false;
    for (uint32_t r = begin_row + tid / kWave; r < row_end; r += threads / kWave) {  // wave-uniform
        map[lane] = 0;
        __builtin_amdgcn_wave_barrier();  // a wave's LDS operations complete in order
        const int32_t *ids = a.topk_idx + r * k;
        int next = ids[lane];
        for (uint32_t c = lane; c - lane < k; c += kWave) {
            const int id = next;
            next = c + kWave < k ? ids[c + kWave] : -1;
            if ((unsigned)id < (unsigned)a.all_E)
                dup |= (atomicOr(&map[id / 32], 1u << (id % 32)) >> (id % 32)) & 1u;
        }
        __builtin_amdgcn_wave_barrier();
    }
    return dup;
}
__device__ __forceinline__ bool check_rows(const LayoutArgs &a, uint32_t begin, uint32_t end, int tid, int threads,
                                           uint32_t *seen) {
    const uint32_t k = a.k_div.d;
    auto first_row = [&](uint32_t entry) {  // of the rows that start at `entry` or later
        const uint32_t q = a.k_div.div(entry);
        return q + (q * k != entry ? 1u : 0u);
    };
    const uint32_t r0 = first_row(begin), r1 = first_row(end);
    switch (k) {
    case 3: return rows_repeat<3>(a, r0 + tid, r1, threads);
    case 5: return rows_repeat<5>(a, r0 + tid, r1, threads);
    case 6: return rows_repeat<6>(a, r0 + tid, r1, threads);
    case 7: return rows_repeat<7>(a, r0 + tid, r1, threads);
    }
    return k <= kWave ? rows_repeat_ballots(a, r0, r1, tid, threads)
                      : rows_repeat_bitmap(a, r0, r1, tid, threads, seen);
}
// LDS words of `seen`.
__host__ __device__ constexpr int seen_ints(int k, int threads) { return k > kWave ? threads : 0; }
static_assert(kMaxExperts <= 32 * kWave, "a wave's bitmap holds every expert");

// ORs the workgroup's routing errors into the LDS word *flags.
__device__ __forceinline__ void gather_errors(uint32_t err, int lane, int *flags) {
    const uint32_t wave_err = (__ballot(err & kRoutingIdOutOfRange) ? kRoutingIdOutOfRange : 0u) |
                              (__ballot(err & kRoutingDuplicate) ? kRoutingDuplicate : 0u);
    if (wave_err && lane == 0)
        atomicOr(flags, (int)wave_err);
}

// ------------------------------------------------------------------------ ranked

// Counting one round: returns the entry's rank among this wave's entries of its expert so
// far (-1 when it does not name a grouped expert) and bumps the wave's counter row.
__device__ __forceinline__ int rank_entry(const LayoutArgs &a, int id, bool in_range, int *cnt) {
    const int e = id - a.e_lo;
    const bool valid = in_range && (unsigned)e < (unsigned)a.E;
    const uint64_t m = match_expert(e, valid, a.nbits);
    int rank = -1;
    if (valid) {
        const int below = lanes_below(m);
        const int old = cnt[e];
        rank = old + below;
        if (below == 0)
            cnt[e] = old + (int)__popcll(m);
    }
    return rank;
}

__device__ __forceinline__ void write_position(const LayoutArgs &a, uint32_t i, int pos) {
    // positions are < T*k by construction; the check keeps every store inside the arrays
    // whatever the workspace held
    if ((uint32_t)pos >= (uint32_t)a.slots)
        pos = -1;
    a.slot_pos[i] = pos;
    if (pos >= 0 && a.row_src)
        a.row_src[pos] = (int32_t)i;
}

// Counts a wave's run, the entries [run.begin, run.end) in up to `rounds` rounds of 64, into
// its counter row cnt [E] (zeroed by the caller).  Cached runs (ids in registers) keep each
// entry's in-wave rank in rank[] for the positions.
__device__ __forceinline__ void count_run(const LayoutArgs &a, EntryRange run, int rounds, int lane, int *cnt,
                                          const int (&ids)[kLayoutRankCache], int (&rank)[kLayoutRankCache]) {
    if (rounds <= kLayoutRankCache) {
#pragma unroll
        for (int r = 0; r < kLayoutRankCache; ++r) {
            if (r >= rounds || run.begin + r * kWave >= run.end)
                break;
            rank[r] = rank_entry(a, ids[r], run.begin + r * kWave + lane < run.end, cnt);
        }
    } else {
        int next = run.begin + lane < run.end ? a.topk_idx[run.begin + lane] : -1;
        for (int r = 0; r < rounds; ++r) {
            const uint32_t i = run.begin + r * kWave + lane;
            if (i - lane >= run.end)
                break;
            const int id = next;
            next = r + 1 < rounds && i + kWave < run.end ? a.topk_idx[i + kWave] : -1;
            (void)rank_entry(a, id, i < run.end, cnt);
        }
    }
}

// Writes the run's positions from base[E] (the wave's first row per expert) and the ranks
// kept by count_run (cached runs) or found again (longer runs).
__device__ __forceinline__ void write_run(const LayoutArgs &a, EntryRange run, int rounds, int lane, int *base,
                                          const int (&ids)[kLayoutRankCache], const int (&rank)[kLayoutRankCache]) {
    if (rounds <= kLayoutRankCache) {
#pragma unroll
        for (int r = 0; r < kLayoutRankCache; ++r) {
            const uint32_t i = run.begin + r * kWave + lane;
            if (r >= rounds || i - lane >= run.end)
                break;
            if (i < run.end)
                write_position(a, i, rank[r] >= 0 ? base[ids[r] - a.e_lo] + rank[r] : -1);
        }
    } else {
        int next = run.begin + lane < run.end ? a.topk_idx[run.begin + lane] : -1;
        for (int r = 0; r < rounds; ++r) {
            const uint32_t i = run.begin + r * kWave + lane;
            if (i - lane >= run.end)
                break;
            const int id = next;
            next = r + 1 < rounds && i + kWave < run.end ? a.topk_idx[i + kWave] : -1;
            const int pos = rank_entry(a, id, i < run.end, base);  // base row + rank so far
            if (i < run.end)
                write_position(a, i, pos);
        }
    }
}

// Exclusive scan of tot[0..E) into offs[0..E] (offs[E] = total) by the whole workgroup:
// each thread scans a contiguous run of experts, the runs' sums are scanned across it.
template <int W>
__device__ void scan_experts(int E, const int *tot, int *offs, int *wave_sum, int tid) {
    constexpr int kThreads = W * kWave;
    const int lane = tid & (kWave - 1), w = tid / kWave;
    const int per = (E + kThreads - 1) / kThreads;
    const int first = tid * per;
    int s = 0;
    for (int c = 0; c < per; ++c)
        if (first + c < E)
            s += tot[first + c];
    const int incl = wave_inclusive_scan(s);
    if (lane == kWave - 1)
        wave_sum[w] = incl;
    __syncthreads();
    int carry = 0, total = 0;
#pragma unroll
    for (int v = 0; v < W; ++v) {
        carry += v < w ? wave_sum[v] : 0;
        total += wave_sum[v];
    }
    int run = carry + incl - s;
    for (int c = 0; c < per; ++c)
        if (first + c < E) {
            offs[first + c] = run;
            run += tot[first + c];
        }
    if (tid == 0)
        offs[E] = total;
    __syncthreads();
}

// Writes the expert counts and offsets and the rank counts and offsets.
template <int W>
__device__ void write_totals(const LayoutArgs &a, const int *tot, const int *offs, int tid) {
    constexpr int kThreads = W * kWave;
    const int E = a.E;
    for (int e = tid; e < E; e += kThreads) {
        a.expert_counts[e] = tot[e];
        a.expert_offsets[e] = offs[e];
    }
    for (int r = tid; r < a.R; r += kThreads) {  // rank r: experts [r * L, (r + 1) * L)
        a.rank_offsets[r] = offs[r * a.L];
        a.rank_counts[r] = offs[(r + 1) * a.L] - offs[r * a.L];
    }
    if (tid == 0) {
        a.expert_offsets[E] = offs[E];
        a.rank_offsets[a.R] = offs[E];
    }
}

constexpr int kTableBatch = 8;  // loads of tile counts in flight per thread

// N neighbouring counts of one tile.
template <int N>
struct Counts {
    int32_t v[N];
};

// Every tile's counts, added per expert into tot[e] (all tiles) and pre[e] (tiles before
// `tile`), LDS counters zeroed by the caller.  A thread sums N neighbouring columns over a
// run of tiles.
template <int W, int N>
__device__ __forceinline__ void sum_columns(const LayoutArgs &a, int tiles, int tile, int tid, int *tot, int *pre) {
    constexpr int kThreads = W * kWave;
    const int E = a.E, cols = E / N;
    const FastDiv by_cols = N == 1 ? a.e_div : a.e4_div;
    const int groups = max(1, min(tiles, (int)by_cols.div(kThreads)));
    const int per = (tiles + groups - 1) / groups;
    for (int q = tid; q < groups * cols; q += kThreads) {
        const int g = (int)by_cols.div(q), e = (q - g * cols) * N;
        const int t_end = min(tiles, (g + 1) * per);
        int s[N], b[N];
#pragma unroll
        for (int c = 0; c < N; ++c)
            s[c] = b[c] = 0;
        for (int t0 = g * per; t0 < t_end; t0 += kTableBatch) {
            Counts<N> held[kTableBatch];
#pragma unroll
            for (int u = 0; u < kTableBatch; ++u)  // a tile past the end is read again, masked below
                held[u] = *reinterpret_cast<const Counts<N> *>(
                    __builtin_assume_aligned(a.tile_counts + (int64_t)min(t0 + u, t_end - 1) * E + e, 4 * N));
#pragma unroll
            for (int u = 0; u < kTableBatch; ++u) {
                const int in = t0 + u < t_end ? ~0 : 0, before = t0 + u < min(tile, t_end) ? ~0 : 0;
#pragma unroll
                for (int c = 0; c < N; ++c) {
                    s[c] += held[u].v[c] & in;
                    b[c] += held[u].v[c] & before;
                }
            }
        }
#pragma unroll
        for (int c = 0; c < N; ++c) {
            if (s[c])
                atomicAdd(&tot[e + c], s[c]);
            if (b[c])
                atomicAdd(&pre[e + c], b[c]);
        }
    }
}

// Count kernel: the tile's counts and error bits, for the rank kernel.
template <int K>
__global__ __launch_bounds__(1024) void layout_count_kernel(LayoutArgs a, uint32_t tile_entries) {
    extern __shared__ __align__(16) int hist[];  // E + 1 bins of counters, the error bits, check_rows' words
    const int tid = threadIdx.x, threads = blockDim.x, E = a.E;
    const int words = hist_copies(E) * (E + 1);
    const uint32_t begin = blockIdx.x * tile_entries, end = min(begin + tile_entries, (uint32_t)a.slots);
    IdBatch ids;
    first_batch<K == 8>(a, begin, end, tid, threads, ids);
    for (int i = tid; i <= words; i += threads)
        hist[i] = 0;
    __syncthreads();
    uint32_t err = 0;
    visit_ids<K, K == 8, true, true>(a, begin, end, 0, tid, threads, hist, hist, err, ids);
    if (K == 0 && check_rows(a, begin, end, tid, threads, reinterpret_cast<uint32_t *>(hist) + words + 1))
        err |= kRoutingDuplicate;
    gather_errors(err, tid & (kWave - 1), &hist[words]);
    __syncthreads();
    for (int e = tid; e < E; e += threads)
        a.tile_counts[(int64_t)blockIdx.x * E + e] = hist_sum(hist, e, hist_copies(E), tid & (kWave - 1));
    if (tid == 0)
        a.tile_errs[blockIdx.x] = (uint32_t)hist[words];
}

// LDS of the rank kernel, in ints: the histogram of the entries before the run (and, ONE,
// of the rest), wave_cnt [W][E], pre [E] and tot [E] where they are not the histograms
// themselves (zeroed up to here), offs [E+1], wave_sum [W], flags.
template <int W, bool ONE>
__host__ __device__ constexpr int rank_zeroed_ints(int E) {
    const int hists = ONE ? 2 : 1, sums = hist_copies(E) > 1 ? 2 : 2 - hists;
    return (hists * hist_copies(E) * (E + 1) + (W + sums) * E + 3) / 4 * 4;
}
template <int W, bool ONE>
constexpr size_t rank_lds_bytes(int E) {
    return sizeof(int) * ((size_t)rank_zeroed_ints<W, ONE>(E) + (E + 1) + W + 1);
}

// Rank kernel.  Grid: x the runs of a tile (W waves x `rounds` rounds x 64 entries each),
// y the tiles.  ONE: the whole layout in this kernel (one tile, no count kernel): each
// workgroup histograms every entry, and one more workgroup at the end of the grid checks
// the routing and writes the status.  K as in visit_ids.
template <int W, bool ONE, int K>
__global__ __launch_bounds__(W * 64) void layout_rank_kernel(LayoutArgs a, uint32_t tile_entries,
                                                              int32_t run_rounds) {
    constexpr int kThreads = W * kWave;
    const int rounds = ONE ? 1 : run_rounds;
    extern __shared__ __align__(16) int lds[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const uint32_t n = (uint32_t)a.slots, tile = blockIdx.y;
    uint32_t err = 0;
    IdBatch batch;
    if (ONE && blockIdx.x == gridDim.x - 1) {
        int *flags = lds;
        if (tid == 0)
            *flags = 0;
        __syncthreads();
        first_batch<K == 8>(a, 0, n, tid, kThreads, batch);
        visit_ids<K, K == 8, false, true>(a, 0, n, 0, tid, kThreads, nullptr, nullptr, err, batch);
        if (K == 0 && check_rows(a, 0, n, tid, kThreads, reinterpret_cast<uint32_t *>(lds) + 1))
            err |= kRoutingDuplicate;
        gather_errors(err, lane, flags);
        __syncthreads();
        if (tid == 0)
            *a.status = (uint32_t)*flags;
        return;
    }
    const int E = a.E, copies = hist_copies(E);
    const int zeroed = rank_zeroed_ints<W, ONE>(E);
    int *hist_pre = lds, *hist_all = lds + (ONE ? copies * (E + 1) : 0);
    int *wave_cnt = hist_all + copies * (E + 1);  // [W][E]: per-wave counts, then first rows
    int *sums = wave_cnt + W * E;
    int *pre = copies > 1 ? sums : hist_pre;      // [E] rows per expert before this run
    int *tot = copies > 1 ? sums + E : (ONE ? hist_all : sums);  // [E] rows per expert
    int *offs = lds + zeroed;         // [E+1] exclusive expert offsets
    int *wave_sum = offs + E + 1;     // [W] scan carries
    int *flags = wave_sum + W;        // error bits
    const bool first = blockIdx.x == 0 && tile == 0;
    const uint32_t tile_begin = tile * tile_entries;
    const uint32_t own_begin = tile_begin + blockIdx.x * (kThreads * rounds);
    if (own_begin >= min(tile_begin + tile_entries, n) && !first)
        return;  // the last tile may hold fewer runs
    const EntryRange run = layout_wave_run(tile, tile_entries, blockIdx.x, rounds, kThreads, w, n);

    // the ids are loaded up front: the first of those to histogram, and this wave's own
    // (cached runs)
    const uint32_t hist_end = ONE ? n : own_begin;
    first_batch<false>(a, tile_begin, hist_end, tid, kThreads, batch);
    int ids[kLayoutRankCache], rank[kLayoutRankCache];
    if (rounds <= kLayoutRankCache) {
#pragma unroll
        for (int r = 0; r < kLayoutRankCache; ++r) {
            if (r >= rounds)
                break;
            const uint32_t i = run.begin + r * kWave + lane;
            ids[r] = i < run.end ? a.topk_idx[i] : -1;
        }
    }
    for (int i = tid; i < zeroed / 4; i += kThreads)
        reinterpret_cast<i32x4 *>(lds)[i] = i32x4{0, 0, 0, 0};
    if (tid == 0)
        *flags = 0;
    __syncthreads();

    if (!ONE) {
        if ((E & 3) == 0 && (reinterpret_cast<uintptr_t>(a.tile_counts) & 15) == 0)
            sum_columns<W, 4>(a, gridDim.y, tile, tid, tot, pre);
        else
            sum_columns<W, 1>(a, gridDim.y, tile, tid, tot, pre);
        if (first) {
            for (uint32_t t = tid; t < gridDim.y; t += kThreads)
                err |= a.tile_errs[t];
            gather_errors(err, lane, flags);
        }
    }
    visit_ids<0, false, true, false>(a, tile_begin, hist_end, own_begin, tid, kThreads, hist_pre, hist_all, err, batch);
    count_run(a, run, rounds, lane, wave_cnt + w * E, ids, rank);
    __syncthreads();

    if (ONE || (copies > 1 && own_begin > tile_begin))
        for (int e = tid; e < E; e += kThreads) {
            if (copies > 1)
                pre[e] += hist_sum(hist_pre, e, copies, lane);
            if (ONE)
                tot[e] = hist_sum(hist_all, e, copies, lane) + pre[e];
        }
    if (ONE && E > kThreads)  // else scan_experts reads just the column this thread summed
        __syncthreads();
    scan_experts<W>(E, tot, offs, wave_sum, tid);
    if (first) {
        write_totals<W>(a, tot, offs, tid);
        if (!ONE && tid == 0)
            *a.status = (uint32_t)*flags;
    }

    // each wave's first row per expert
    for (int e = tid; e < E; e += kThreads) {
        int c[W];
#pragma unroll
        for (int v = 0; v < W; ++v)
            c[v] = wave_cnt[v * E + e];
        int base = offs[e] + pre[e];
#pragma unroll
        for (int v = 0; v < W; ++v) {
            wave_cnt[v * E + e] = base;
            base += c[v];
        }
    }
    __syncthreads();
    write_run(a, run, rounds, lane, wave_cnt + w * E, ids, rank);
}

template <int W>
void launch_rank(const LayoutArgs &a, const LayoutGeom &g, hipStream_t stream, TraceSlot ts) {
    constexpr int kThreads = W * kWave;
    const uint32_t tile_entries = (uint32_t)(g.waves * kWave * g.rounds);
    const LayoutRuns r = layout_runs(tile_entries, g.tiles, kThreads);
    hipExtLaunchKernelGGL((layout_rank_kernel<W, false, 0>), dim3(r.runs, (unsigned)g.tiles), dim3(kThreads),
                          (uint32_t)rank_lds_bytes<W, false>(a.E), stream, nullptr, ts.stop, 0, a, tile_entries,
                          r.rounds);
}

// The whole layout in one kernel: the runs, and the workgroup that checks the routing.
template <int W, int K>
void launch_one(const LayoutArgs &a, hipStream_t stream, TraceSlot ts) {
    constexpr int kThreads = W * kWave;
    const unsigned runs = (unsigned)std::max<int64_t>(1, (a.slots + kThreads - 1) / kThreads);
    const size_t check_lds = sizeof(int) * (1 + (size_t)seen_ints(a.k, kThreads));
    hipExtLaunchKernelGGL((layout_rank_kernel<W, true, K>), dim3(runs + 1), dim3(kThreads),
                          (uint32_t)std::max(rank_lds_bytes<W, true>(a.E), check_lds), stream, ts.start, ts.stop, 0, a,
                          (uint32_t)a.slots, 1);
}

template <int K>
void launch_layout_k(LayoutArgs &a, hipStream_t stream, TraceSlot ts) {
    if (K != 0 && a.slots <= kLayoutOneKernelIds)
        return launch_one<4, K>(a, stream, ts);
    const LayoutGeom g = layout_geometry(a.slots, a.E);
    if constexpr (K == 0)  // as many threads as fit, for the checks of general rows
        if (g.tiles == 1)
            return g.waves == 16 ? launch_one<16, K>(a, stream, ts) : launch_one<4, K>(a, stream, ts);
    a.e_div = fast_div((uint32_t)a.E);
    a.e4_div = fast_div((uint32_t)std::max(1, a.E / 4));
    const int64_t tile_entries = (int64_t)g.waves * kWave * g.rounds;
    const unsigned count_threads = (unsigned)std::min<int64_t>(1024, std::max<int64_t>(256, tile_entries / 8 / kWave * kWave));
    const size_t count_lds =
        sizeof(int) * ((size_t)hist_copies(a.E) * (a.E + 1) + 1 + seen_ints(a.k, (int)count_threads));
    // both kernels inside one pair of timing events: the layout's time
    hipExtLaunchKernelGGL((layout_count_kernel<K>), dim3((unsigned)g.tiles), dim3(count_threads), (uint32_t)count_lds,
                          stream, ts.start, nullptr, 0, a, (uint32_t)tile_entries);
    if (a.slots > kLayoutWideRank && g.tiles < kLayoutRankGroups && a.E <= 512)
        launch_rank<16>(a, g, stream, ts);
    else
        launch_rank<4>(a, g, stream, ts);
}

}  // namespace

hipError_t launch_layout(LayoutArgs a, hipStream_t stream) {
    a.L = a.E / a.R;
    a.k_div = fast_div((uint32_t)a.k);
    (void)hipGetLastError();  // drop an error left by an earlier, already reported call
    const TraceSlot ts = trace_acquire();
    switch (a.k) {
    case 1: launch_layout_k<1>(a, stream, ts); break;
    case 2: launch_layout_k<2>(a, stream, ts); break;
    case 4: launch_layout_k<4>(a, stream, ts); break;
    case 8: launch_layout_k<8>(a, stream, ts); break;
    default: launch_layout_k<0>(a, stream, ts); break;
    }
    const hipError_t err = hipGetLastError();
    if (err == hipSuccess)
        trace_submit("layout", ts);
    return err;
}

}  // namespace ep
