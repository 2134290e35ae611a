// Rounds by admission over the whole grid, for gfx950: hgm_match and
// hgm_match_batch calls that want only the matching.
//
// The order of the edges is fixed, so the edges whose keys reach a threshold
// form a prefix of it, and an edge of the prefix that holds the maximum at all
// its pins among the prefix's live edges holds it among all live edges: every
// edge left out ranks below it.  So round 0 need not form the maximum over
// every pin.  The rounds start with the top edges and each of the first rounds
// admits the next part of the order; by the time most edges are admitted one
// of their pins is done, which the edge's first pins show.  What reaches the
// maximum, and with it the random reads and device atomics that bound the
// rounds over all edges, falls to 0.29M atomics in the joins of the power-law
// instance (29.8M pins) and 1.6M on the hub-stress one (36M), at the same number
// of rounds; the passes over the weights and the first pins that remain are
// streams.  Per-round counts, priorities redrawn every round
// and a round limit depend on the round an edge is matched in: those calls
// run the rounds of kernels.hip.
//
// A round is two launches:
//   join   the survivors of the last round's live list and the edges admitted
//          this round, those with no done pin, form the round's list and
//          raise best[round & 1] at their pins; best[(round - 1) & 1] goes
//          back to zero at the pins of the last round's list, so no pass over
//          the vertices is needed
//   test   an edge that equals best at all its pins is matched: its bit is
//          set and its pins are marked done
// Each wave owns a range of edge ids and keeps its live edges in its own range
// of the lists: compaction is a ballot, with no barrier and no atomic.  Done
// marks are bits (n / 8 bytes stay in every XCD's L2 beside the streams).
#include "internal.h"
#include "schedule.h"
#include "wave.h"

namespace hgm {
namespace {

constexpr int kWaves = kBlock / kWave;
constexpr int kKeepPins = 8;  // blocks of pins kept in registers (flat_edges)
constexpr int kFill = 16;     // chunks of edges looked at in one step (join_wave)

// Thresholds by sampling, in one workgroup: 256 groups of 16 keys.  The largest
// of each group gives 256 maxima, of which the one of rank r has about
// (1 - r / 256)^(1/16) of all keys below it; the first key of each group
// gives plain quantiles.  Parts of about 1/2700, 1/250, 1/33, 1/10, 1/5 and
// 1/2 of the edges.
constexpr int kSamplesPerGroup = 16;
constexpr int kThresholds = kStagedSteps - 1;
constexpr int kFromMaxima = 3;
// The step at which all edges left are looked at, in order: a tenth is admitted,
// and most of the others have a pin that is done.  Without it each of the last
// three parts gathers its own lines (power-law 400 -> 342 us, hub-stress 505 ->
// 484, RGG 430 -> 418); a step earlier hub-stress takes 8% more, one later
// power-law 2%.
constexpr int kSweep = 4;
__device__ constexpr int kRank[kThresholds] = {1, 16, 98, 25, 51, 128};

template <bool kB>
__device__ __forceinline__ uint64_t staged_key(const Graph &g, const State &s, uint32_t seed,
                                               int e) {
    if constexpr (kB) return s.key[e];
    return ((uint64_t)g.w[e] << 32) | priority_hash(seed, (uint32_t)e);
}

__device__ __forceinline__ uint32_t *done_bits(const State &s) {
    return reinterpret_cast<uint32_t *>(s.done);
}

// Per-wave live counts sit at the front of rec_c, which these rounds do not
// otherwise use; behind those of rec_c[0], the admission step of every edge.
__device__ __forceinline__ uint8_t *step_bytes(const State &s) {
    return reinterpret_cast<uint8_t *>(s.rec_c[0] + (int64_t)s.grid * kWaves);
}

constexpr int kSetupThreads = 1024, kSampleGroups = 256;
constexpr int kSetupParts = kSetupThreads / kSampleGroups;  // threads per sample group

// Rank of group i's key among the 256 groups' (the group decides between equal
// keys: a batch's instances can share one); each of a group's threads compares
// a part of them.
__device__ __forceinline__ int rank_of(const uint64_t *keys, int i, int part) {
    const uint64_t mine = keys[i];
    int rank = 0;
#pragma unroll 8
    for (int q = part; q < kSampleGroups; q += kSetupParts)
        rank += keys[q] > mine || (keys[q] == mine && q < i) ? 1 : 0;
#pragma unroll
    for (int o = 1; o < kSetupParts; o <<= 1) rank += __shfl_xor(rank, o, kWave);
    return rank;
}

// What a workgroup of the setup has seen of v_off (check_bins): the degrees of
// its hot vertices and whether an offset decreases or lies outside [0, kappa].
struct VOffPart {
    unsigned long long hot, bad;
};
__device__ __forceinline__ VOffPart *v_off_parts(const State &s) {
    return reinterpret_cast<VOffPart *>(s.bin_key);
}

// Sparse instances.  Where an edge meets few others, most are matched in the
// first rounds whichever way they are looked at, and the steps cost more than
// they leave out: round 1 then goes on with a later one.  A sample says how many
// others an edge meets (the means do not: with popular vertices the same means
// want every step): the setup reads two pins of up to kMeetEdges edges, one
// from every stretch of ids, and one workgroup puts them in a hash table, where a
// pin that finds its vertex is a hit.  The gathers are spread over workgroups: a
// single one took 28 us for them.
constexpr int kMeetEdges = 4096, kMeetSlots = 12288, kMeetProbes = 8;
constexpr int kFirstWord = 8;  // of hot: the step of round 1

// {two pins} of sampled edge i, -1 where it has fewer.
__device__ __forceinline__ int2 *met_pins(const State &s) {
    return reinterpret_cast<int2 *>(s.rec_key[1]);  // free until round 1's lists
}
__device__ __forceinline__ int met_edges(const Graph &g) {
    return g.m < kMeetEdges ? g.m : kMeetEdges;
}
template <bool kB>
__device__ __forceinline__ void sample_edge(const Graph &g, const State &s, uint32_t seed, int i) {
    const int n = met_edges(g);
    if (i >= n) return;
    const int64_t lo = (int64_t)g.m * i / n, hi = (int64_t)g.m * (i + 1) / n;
    const uint32_t x = priority_hash(seed, 0xedceu + (uint32_t)i);
    const int64_t e = lo + x % (uint32_t)(hi - lo);
    const int64_t base = g.pairs ? 2 * e : g.e_off[e];
    const int len = g.pairs ? 2 : (int)(g.e_off[e + 1] - base);
    const int vb = kB ? g.vbase[e] : 0;
    const uint32_t j = len > 0 ? (x >> 7) % (uint32_t)len : 0;
    int2 v = make_int2(-1, -1);
    if (len > 0) v.x = g.e_pins[base + j] + vb;
    if (len > 1) v.y = g.e_pins[base + ((int)j + 1 < len ? j + 1 : 0)] + vb;
    met_pins(s)[i] = v;
}

// The step of round 1 for `others` met by an edge on average: all edges, half of
// them, a fifth, or the next.  Measured with round 0 at that step, us, graphs of
// 500,000 edges, next step / 4 / 5 / 6 (rounds over all edges): 2 others 291 / 241
// / 219 / 206 (187), 4 256 / 216 / 199 / 205 (180), 8 234 / 193 / 201 / 209 (193);
// of 2M edges 2 476 / 425 / 413 / 474 (368), 4 406 / 355 / 429 / 457, 12 296 / 325 /
// 389; popularity by rank^-0.7, 500,000 edges, 173 others 197 / 254 / 262 / 261.
// With the sample and from round 1 on, without a vertex side: 500,000 edges 2
// others 216, 4 208, 8 194; 2M 2 455, 4 396; 173 others 210 (no step left out,
// 8 to 12 us for the sample).
__device__ __forceinline__ int next_step(float others, int64_t kappa, int next) {
    int step = next;
    if (kappa <= kSparseMiddle)
        step = others <= 1.5f                                ? 6
               : others <= 5.f                               ? 5
               : others <= 14.f || kappa <= kSparseSmall ? 4
                                                              : next;
    else
        step = others <= 3.f ? 5 : others <= 5.f ? 4 : next;
    static_assert(kThresholds == 6, "the steps above");
    return step > next ? step : next;
}

constexpr int kSampleGrid = kMeetEdges / kWave;
__global__ void __launch_bounds__(kWave) k_staged_sample(Graph g, State s, uint32_t seed) {
    sample_edge<false>(g, s, seed, blockIdx.x * kWave + threadIdx.x);
}

// Hashes the sample: one workgroup, between round 0 and the join of round 1 or
// before round 0.  out: {the step, the others met as a float's bits}.
__global__ void __launch_bounds__(kSetupThreads) k_staged_meet(Graph g, State s, int next,
                                                               unsigned long long *out) {
    __shared__ int ids[kMeetSlots];
    __shared__ unsigned int hits;
    constexpr int kOwn = kMeetEdges / kSetupThreads;
    const int tid = threadIdx.x, n = met_edges(g);
    int2 v[kOwn];
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
        const int i = q * kSetupThreads + tid;
        v[q] = i < n ? met_pins(s)[i] : make_int2(-1, -1);
    }
    for (int j = tid; j < kMeetSlots; j += kSetupThreads) ids[j] = -1;
    if (tid == 0) hits = 0;
    __syncthreads();
    unsigned int mine = 0;
    auto put = [&](int x) {
        if (x < 0) return;
        uint32_t h = __umulhi((uint32_t)x * 0x9E3779B1u, (uint32_t)kMeetSlots);
        for (int p = 0; p < kMeetProbes; ++p) {
            const int id = atomicCAS(&ids[h], -1, x);
            if (id == x) ++mine;
            if (id == -1 || id == x) return;
            h = h + 1 < (uint32_t)kMeetSlots ? h + 1 : 0;
        }
    };
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
        put(v[q].x);
        put(v[q].y);
    }
    if (mine) atomicAdd(&hits, mine);
    __syncthreads();
    if (tid == 0) {
        // Two edges share others / m vertices on average, and a shared one is
        // among the sampled pins of both with (2 / size)^2.
        const float size = (float)g.kappa / (float)g.m, over = size > 2.f ? size / 2.f : 1.f;
        const float pairs = 0.5f * (float)n * (float)n;
        const float others = (float)hits / pairs * (float)g.m * over * over;
        const unsigned long long step = (unsigned long long)next_step(others, g.kappa, next);
        s.hot[kFirstWord] = step;
        out[0] = step;
        out[1] = __float_as_uint(others);
    }
}

// Clears the state; workgroup 0 clears the counters and draws the thresholds.
template <bool kB>
__global__ void __launch_bounds__(kSetupThreads) k_staged_setup(Graph g, State s, uint32_t seed,
                                                                uint32_t *bits, int keep_bits,
                                                                int check_bins, int sparse) {
    const int tid = threadIdx.x;
    if (blockIdx.x == 0) {
        for (int j = tid; check_bins && j < s.bin_nb; j += kSetupThreads) s.bin_cursor[j] = 0;
        if (tid < kEndHeader) s.hot[kSub / 2 + tid] = 0;  // the report, without a host slot
        __shared__ uint64_t top[kSampleGroups], one[kSampleGroups];
        constexpr int kOwn = kSamplesPerGroup / kSetupParts;
        const int i = tid / kSetupParts, part = tid % kSetupParts;
        uint64_t key[kOwn], most = 0;
#pragma unroll
        for (int q = 0; q < kOwn; ++q) {
            const uint32_t at = (uint32_t)(q * kSetupThreads + tid);
            const int64_t lo = (int64_t)g.m * at / (kSetupThreads * kOwn);
            const int64_t hi = (int64_t)g.m * (at + 1) / (kSetupThreads * kOwn);
            const uint32_t width = hi > lo ? (uint32_t)(hi - lo) : 1u;
            const int64_t e = lo + priority_hash(seed, 0x5eedu + at) % width;
            key[q] = e < g.m ? staged_key<kB>(g, s, seed, (int)e) : 0;
        }
        if (part == 0) one[i] = key[0];
#pragma unroll
        for (int q = 0; q < kOwn; ++q) most = key[q] > most ? key[q] : most;
#pragma unroll
        for (int o = 1; o < kSetupParts; o <<= 1) {
            const uint64_t other = __shfl_xor((unsigned long long)most, o, kWave);
            most = other > most ? other : most;
        }
        if (part == 0) top[i] = most;
        for (int j = tid; j < s.ring * kSub; j += kSetupThreads)
            s.stats[j / kSub].live[j % kSub] = 0;
        __syncthreads();
        const int r0 = rank_of(top, i, part), r1 = rank_of(one, i, part);
#pragma unroll
        for (int q = 0; q < kThresholds; ++q)
            if (part == 0 && (q < kFromMaxima ? r0 : r1) == kRank[q])
                s.hot[q] = q < kFromMaxima ? top[i] : one[i];
        return;
    }
    if (sparse && tid < kWave)
        for (int i = (blockIdx.x - 1) * kWave + tid; i < kMeetEdges; i += (gridDim.x - 1) * kWave)
            sample_edge<kB>(g, s, seed, i);
    const int64_t stride = (int64_t)(gridDim.x - 1) * kSetupThreads;
    const int64_t at = (int64_t)(blockIdx.x - 1) * kSetupThreads + tid;
    // The arrays start at 256-byte boundaries and are padded to them.
    const int64_t n = g.n;  // up to 2^31 - 1: rounded up in 64 bits
    for (int64_t i = at; i < (n + 1) / 2; i += stride) {
        reinterpret_cast<ulonglong2 *>(s.best[0])[i] = make_ulonglong2(0, 0);
        reinterpret_cast<ulonglong2 *>(s.best[1])[i] = make_ulonglong2(0, 0);
    }
    uint32_t *done = done_bits(s);
    for (int64_t i = at; i < (n + 31) / 32; i += stride) done[i] = 0;
    if (!keep_bits)
        for (int64_t i = at; i < g.words; i += stride) bits[i] = 0;
    if (check_bins) {
        __shared__ unsigned long long hot_sum;
        if (tid == 0) hot_sum = 0;
        __syncthreads();
        unsigned long long hot = 0;
        bool bad = false;
        for (int64_t i = at; i < n; i += stride) {
            const int lo = g.v_off[i], hi = g.v_off[i + 1], deg = hi - lo;
            bad |= lo < 0 || hi < lo || hi > g.kappa;
            if (deg >= s.hot_degree) hot += (unsigned long long)deg;
        }
        if (hot) atomicAdd(&hot_sum, hot);
        const bool any = __syncthreads_or(bad);
        if (tid == 0) v_off_parts(s)[blockIdx.x - 1] = {hot_sum, any ? 1ull : 0ull};
    }
}

// The check that comes with automatic bins, for calls whose rounds do not use
// them: the rounds over all live edges find a v_off that is not the transpose
// when a bin holds more pins than its vertices' degrees add up to.  No bin can
// where every bin's degree sum equals the pins it really has, which this
// counts and k_end compares; where they differ the host runs those rounds and
// returns what they return.  Bins run only where the degrees send round 0 to
// the vertex form, so the pins are left alone elsewhere.
//
// Bound by streaming the pins (4.4 TB/s): hub-stress, 36M pins, 465 -> 506 us;
// 13M uniform pins 354 -> 369, 3.2M 201 -> 213 (230 with 1,024 workgroups, whose
// sums meet at the same few counters); power-law, 30M, the edge form, 341 -> 347
// for the pass over v_off.
constexpr int kCheckThreads = 1024, kCheckGrid = 256, kCheckCopies = 4;
__global__ void __launch_bounds__(kCheckThreads) k_staged_check(Graph g, State s, int parts) {
    __shared__ uint32_t count[kCheckCopies][kBinMaxBins];  // each by some of the waves
    __shared__ unsigned long long hot_sum;
    const int tid = threadIdx.x;
    if (tid == 0) hot_sum = 0;
    __syncthreads();
    unsigned long long hot = 0;
    bool bad = false;
    for (int i = tid; i < parts; i += kCheckThreads) {
        const VOffPart p = v_off_parts(s)[i];
        hot += p.hot;
        bad |= p.bad != 0;
    }
    if (hot) atomicAdd(&hot_sum, hot);
    const bool any = __syncthreads_or(bad);
    const int verdict = 2 * hot_sum >= (unsigned long long)g.kappa ? kBinsUnused
                        : any                                      ? kBinsBadOffsets
                                                                   : kBinsCompare;
    if (blockIdx.x == 0 && tid == 0) *s.piece_count = verdict;
    if (verdict != kBinsCompare) return;
    uint32_t *mine = count[tid / kWave % kCheckCopies];
    for (int j = tid; j < s.bin_nb; j += kCheckThreads)
        for (int w = 0; w < kCheckCopies; ++w) count[w][j] = 0;
    __syncthreads();
    const uint32_t last = (uint32_t)s.bin_nb - 1;
    auto add = [&](int v) { atomicAdd(&mine[min((uint32_t)v >> s.bin_rb, last)], 1u); };
    // 16-byte loads from the first aligned pin on.
    const int64_t head = min((int64_t)((16 - ((uintptr_t)g.e_pins & 15)) / 4 % 4), g.kappa);
    const int4 *quads = reinterpret_cast<const int4 *>(g.e_pins + head);
    const int64_t nq = (g.kappa - head) / 4, tail = head + 4 * nq;
    constexpr int kU = 4;
    const int64_t stride = (int64_t)gridDim.x * kCheckThreads;
    int64_t i = (int64_t)blockIdx.x * kCheckThreads + tid;
    for (; i + (kU - 1) * stride < nq; i += kU * stride) {
        int4 q[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) q[u] = quads[i + u * stride];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            add(q[u].x);
            add(q[u].y);
            add(q[u].z);
            add(q[u].w);
        }
    }
    for (; i < nq; i += stride) {
        const int4 q = quads[i];
        add(q.x);
        add(q.y);
        add(q.z);
        add(q.w);
    }
    if (blockIdx.x == 0) {
        if (tid < head) add(g.e_pins[tid]);
        if (tail + tid < g.kappa) add(g.e_pins[tail + tid]);
    }
    __syncthreads();
    for (int j = tid; j < s.bin_nb; j += kCheckThreads) {
        uint32_t c = 0;
        for (int w = 0; w < kCheckCopies; ++w) c += count[w][j];
        if (c) atomicAdd(&s.bin_cursor[j], c);
    }
}

// Marks every vertex of the instances the solo part has matched.
__global__ void __launch_bounds__(kBlock) k_staged_mark_solo(State s, BatchIn b) {
    uint32_t *done = done_bits(s);
    for (int i = blockIdx.x; i < b.count; i += gridDim.x) {
        const int64_t v0 = b.v_base[i], v1 = b.v_base[i + 1];
        if (v1 - v0 > b.solo_max_verts || solo_size(b.e_base, b.pin_base, i) > b.solo_max_size)
            continue;
        for (int64_t w = (v0 >> 5) + threadIdx.x; w * 32 < v1; w += kBlock) {
            uint32_t m = 0xFFFFFFFFu;
            if (w * 32 < v0) m &= 0xFFFFFFFFu << (v0 & 31);
            if (w * 32 + 32 > v1) m &= 0xFFFFFFFFu >> (32 - (v1 & 31));
            atomicOr(&done[w], m);  // neighbouring instances share words
        }
    }
}

// The live list of wave `wave`: its edge range [lo, lo + per) and its slots.
struct WaveRange {
    int64_t lo;
    int per, wave;
};

__device__ __forceinline__ WaveRange wave_range(const State &s) {
    WaveRange r;
    r.per = s.region / kWaves;
    r.wave = xcd_item(blockIdx.x, gridDim.x) * kWaves + threadIdx.x / kWave;
    r.lo = (int64_t)r.wave * r.per;
    return r;
}

// Live edges of round r, long ones by their weight (its join is finished; every
// lane gets the sum).
__device__ __forceinline__ int64_t live_edges(const State &s, int r) {
    unsigned long long v = s.stats[r % s.ring].live[lane_id()];
    static_assert(kSub == kWave, "one counter per lane");
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return (int64_t)v;
}

// How best[r & 1] goes back to zero before round r + 2 raises it: a round with
// many live edges by one pass over the array, one with few by a store at each
// of its pins; either in the join of round r + 1.  Scattered stores cost as much
// as device atomics (27 G/s).  A long edge adds kLongWeight times its pins to the round's
// count of live edges, instead of 1: a workgroup lowers 2,048 pins in the time
// that the pass takes for about 500 times as many vertices.  (The last rounds'
// workgroup, which also reads the count, leaves such rounds to the grid.)
constexpr unsigned long long kLongWeight = 8;
__device__ __forceinline__ bool clears_by_pass(const Graph &g, int64_t live) {
    return live * 64 >= g.n;
}

// Edges of more pins than a window are left by the waves that meet them to the
// whole workgroup, which takes them one after the other when its waves are
// done (those that find no room stay with their wave).  Bound by latency: two
// dependent reads a step, 2,048 pins in about 2.3 us; one wave needs 10 to 18,
// and such an edge is alone in its chunk.  64 edges of 100,000 pins: 145 ms by
// one wave each 64, 13.3 by short ranges, 6.6 so (the rounds over all edges 55);
// 200,000 small edges and 20 of 300,000 pins: 4.6 -> 1.4 ms (13.1); sixteen
// instances of 20,000 and one of 100,000: 2.7 -> 0.66 ms (0.60).
constexpr int kLong = kWindow, kLongMax = 16;  // kept of each wave
struct LongEdge {
    uint64_t key;
    int e, base, len, vb;
    bool listed;  // in the last round's list
};
struct LongEdges {
    int count[kWaves];
    int kept[kWaves];  // entries of each wave's list (join)
    LongEdge edge[kWaves][kLongMax];
    // By each wave, its own: no barrier.
    __device__ __forceinline__ void reset(int wave) {
        if (lane_id() == 0) count[wave] = 0;
        wave_fence();
    }
    __device__ __forceinline__ bool take(int wave, const LongEdge &x) {
        if (x.len <= kLong) return false;
        const int i = atomicAdd(&count[wave], 1);
        if (i >= kLongMax) return false;
        edge[wave][i] = x;
        return true;
    }
    // After a barrier.
    __device__ __forceinline__ bool any() const {
        int n = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) n |= count[w];
        return n != 0;
    }
    __device__ __forceinline__ int taken(int wave) const {
        return count[wave] < kLongMax ? count[wave] : kLongMax;
    }
};

// The workgroup at the pins of one long edge: look(pin) of kLongU pins a thread
// at a time, then use(pin, looked); whether use held somewhere.  `every`: at
// all pins, else until it holds.  All threads call it and get the answer.
constexpr int kLongU = 8;
template <class Look, class Use>
__device__ __forceinline__ bool long_pins(const int32_t *e_pins, const LongEdge &x, bool every,
                                          Look look, Use use) {
    bool any = false;
    for (int64_t t0 = 0; t0 < x.len; t0 += kLongU * kBlock) {
        int v[kLongU];
        decltype(look(0)) l[kLongU];
#pragma unroll
        for (int u = 0; u < kLongU; ++u) {
            const int64_t t = t0 + u * kBlock + threadIdx.x;
            v[u] = e_pins[x.base + (t < x.len ? t : 0)] + x.vb;
        }
#pragma unroll
        for (int u = 0; u < kLongU; ++u) l[u] = look(v[u]);
#pragma unroll
        for (int u = 0; u < kLongU; ++u)
            if (t0 + u * kBlock + threadIdx.x < x.len) any |= use(v[u], l[u]);
        if (!every && __syncthreads_or(any)) return true;
    }
    return every ? __syncthreads_or(any) : false;
}

// The grid's side of join_wave.
template <bool kPairs, bool kB>
struct GridJoin {
    const Graph &g;
    const State &s;
    const uint32_t *done;
    uint64_t *best, *old;
    uint32_t seed;
    bool lowering;
    LongEdges *longs;
    __device__ __forceinline__ uint32_t done_word(int v) const { return done[v >> 5]; }
    __device__ __forceinline__ void lower(int v) const {
        if (lowering) old[v] = 0;
    }
    // A plain read first skips the atomic where the entry already holds more
    // (best only grows during the pass, a stale read is a lower bound).
    __device__ __forceinline__ uint64_t peek(int v) const {
        return __hip_atomic_load(&best[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ void raise(int v, uint64_t k, uint64_t now) const {
        if (now < k)
            __hip_atomic_fetch_max(&best[v], k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ uint64_t key(int e) const { return staged_key<kB>(g, s, seed, e); }
    __device__ __forceinline__ void place(int e, int &base, int &len, int &vb) const {
        base = kPairs ? 2 * e : g.e_off[e];
        len = kPairs ? 2 : g.e_off[e + 1] - base;
        vb = kB ? g.vbase[e] : 0;
    }
    __device__ __forceinline__ void sort(int e, uint32_t &w, uint64_t &k) const {
        if constexpr (kB)
            k = s.key[e];
        else
            w = g.w[e];
    }
    __device__ __forceinline__ uint64_t exact_sort(int e, uint32_t w) const {
        return (uint64_t)w << 32 | priority_hash(seed, (uint32_t)e);
    }
    __device__ __forceinline__ bool defer(int e, int base, int len, int vb, uint64_t key,
                                          bool listed) const {
        return longs->take(threadIdx.x / kWave, {key, e, base, len, vb, listed});
    }
};

__device__ __forceinline__ WaveLists lists(const State &s, int k) {
    return {s.list[k], s.rec_a[k], s.rec_b[k], s.rec_vb[k], s.rec_key[k]};
}

// Round 0 admits step `first`, round 1 step `second` (-1: as k_staged_meet says),
// and so on.
template <bool kPairs, bool kB>
__global__ void __launch_bounds__(kBlock) k_staged_join(Graph g, State s, int round, int first,
                                                        int second, uint32_t seed) {
    __shared__ WaveScratch scratch[kWaves];
    __shared__ int queue[kWaves][cand_size(kFill)];
    __shared__ LongEdges longs;
    const int wid = threadIdx.x / kWave;
    if (!kPairs) longs.reset(wid);
    const WaveRange range = wave_range(s);
    const int to = round & 1, from = to ^ 1;
    GridJoin<kPairs, kB> m{g, s, done_bits(s), s.best[to], s.best[from], seed, round > 0,
                          &longs};
    if (round > 0 && clears_by_pass(g, live_edges(s, round - 1))) {
        m.lowering = false;
        ulonglong2 *all = reinterpret_cast<ulonglong2 *>(s.best[from]);
        const int64_t stride = (int64_t)gridDim.x * kBlock;
        const int64_t pairs = ((int64_t)g.n + 1) / 2;
        for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < pairs; i += stride)
            all[i] = make_ulonglong2(0, 0);
    }
    const int64_t end = range.lo + range.per < g.m ? range.lo + range.per : g.m;
    if (second < 0 && round > 0) second = (int)s.hot[kFirstWord];
    const int step = round == 0 ? first : second + round - 1;
    const int before = round == 1 ? first : step - 1;  // steps up to it are admitted
    const bool sweep = round > 0 && step >= kSweep && (before < kSweep || round == 1);
    const int kept = join_wave<kPairs, kB, kKeepPins, kStagedSteps, kFill>(
        m, scratch[wid], queue[wid], g.e_pins, lists(s, from), lists(s, to), range.lo, end,
        round > 0 ? s.rec_c[from][range.wave] : 0, round == 0, sweep, before, step, step_bytes(s),
        reinterpret_cast<const uint64_t *>(s.hot));
    // Before the barrier, which waits for what the wave has in flight.
    if (lane_id() == 0) {
        s.rec_c[to][range.wave] = kept;
        if (kept > 0)
            atomicAdd(&s.stats[round % s.ring].live[range.wave % kSub], (unsigned long long)kept);
    }
    if constexpr (!kPairs) {
        if (lane_id() == 0) longs.kept[wid] = kept;
        __syncthreads();
        if (longs.any()) {
            const WaveLists out = lists(s, to);
            for (int w = 0; w < kWaves; ++w)
                for (int i = 0; i < longs.taken(w); ++i) {
                    const LongEdge x = longs.edge[w][i];
                    const bool every = x.listed && m.lowering;
                    const bool dead = long_pins(
                        g.e_pins, x, every, [&](int v) { return m.done_word(v); },
                        [&](int v, uint32_t word) {
                            if (every) m.lower(v);
                            return (bool)((word >> (v & 31)) & 1u);
                        });
                    if (dead) continue;
                    if (threadIdx.x == 0) {
                        const int64_t at =
                            range.lo + (int64_t)w * range.per + longs.kept[w]++;  // wave 0's range
                        out.list[at] = x.e;
                        out.base[at] = x.base;
                        out.len[at] = x.len;
                        if constexpr (kB) out.vb[at] = x.vb;
                        out.key[at] = x.key;
                        atomicAdd(&s.stats[round % s.ring].live[w], kLongWeight * x.len);
                    }
                    long_pins(
                        g.e_pins, x, true, [&](int v) { return m.peek(v); },
                        [&](int v, uint64_t now) {
                            m.raise(v, x.key, now);
                            return false;
                        });
                }
            __syncthreads();
            if (lane_id() == 0) s.rec_c[to][range.wave] = longs.kept[wid];
        }
    }
}

template <bool kPairs, bool kB>
__global__ void __launch_bounds__(kBlock) k_staged_test(Graph g, State s, int round,
                                                        uint32_t *bits) {
    __shared__ WaveScratch scratch[kWaves];
    __shared__ LongEdges longs;
    const int lane = lane_id(), wid = threadIdx.x / kWave;
    if (!kPairs) longs.reset(wid);
    WaveScratch &W = scratch[wid];
    const WaveRange range = wave_range(s);
    const int k = round & 1;
    if (blockIdx.x == 0 && threadIdx.x < kSub)
        s.stats[(round + 1) % s.ring].live[threadIdx.x] = 0;
    const int n = s.rec_c[k][range.wave];
    const uint64_t *best = s.best[k];
    uint32_t *done = done_bits(s);
    auto win = [&](int e) {
        const int bit = kB ? e + g.bitoff[e] : e;
        atomicOr(&bits[bit >> 5], 1u << (bit & 31));
    };
    auto mark = [&](int v) { atomicOr(&done[v >> 5], 1u << (v & 31)); };
    for (int i0 = 0; i0 < n; i0 += kWave) {
        const int i = i0 + lane;
        bool on = i < n;
        int e = 0, base = 0, len = 0, vb = 0;
        uint64_t key = 0;
        if (on) {
            const int64_t at = range.lo + i;
            e = s.list[k][at];
            if constexpr (kPairs) {
                base = 2 * e;
                len = 2;
            } else {
                base = s.rec_a[k][at];
                len = s.rec_b[k][at];
                if constexpr (kB) vb = s.rec_vb[k][at];
            }
            key = s.rec_key[k][at];
        }
        flat_edges<kPairs, kB, kKeepPins>(
            W, g.e_pins, base, len, key, false,
            [&] {
                if (!longs.take(wid, {key, e, base, len, vb, true})) return false;
                on = false;
                return true;
            },
            [&](int v) { return best[v]; },
            [](int, uint64_t key, uint64_t b) { return b != key; },
            [&](bool lost) {
                if (on && !lost) win(e);
                return key;
            },
            NoRead(), [&](int v, uint64_t, int) { mark(v); }, vb);
    }
    if constexpr (!kPairs) {
        __syncthreads();
        if (!longs.any()) return;
        for (int w = 0; w < kWaves; ++w)
            for (int i = 0; i < longs.taken(w); ++i) {
                const LongEdge x = longs.edge[w][i];
                if (long_pins(
                        g.e_pins, x, false, [&](int v) { return best[v]; },
                        [&](int, uint64_t b) { return b != x.key; }))
                    continue;
                if (threadIdx.x == 0) win(x.e);
                long_pins(g.e_pins, x, true, NoRead(), [&](int v, int) {
                    mark(v);
                    return false;
                });
            }
    }
}

}  // namespace

static int setup_grid(const Launch &L) { return L.grid / 4 + 2; }

hipError_t launch_staged_setup(const Launch &L, const Graph &g, const State &s, uint32_t seed,
                               uint32_t *bits, const BatchIn *batch, bool check_bins, bool sparse) {
    const dim3 grid(setup_grid(L)), block(kSetupThreads);
    const int keep = batch && batch->mark_done, check = check_bins ? 1 : 0;
    const int meet = sparse ? 1 : 0;
    if (g.vbase)
        hipLaunchKernelGGL(k_staged_setup<true>, grid, block, 0, L.stream, g, s, seed, bits, keep,
                           0, meet);
    else
        hipLaunchKernelGGL(k_staged_setup<false>, grid, block, 0, L.stream, g, s, seed, bits, keep,
                           check, meet);
    if (keep)
        hipLaunchKernelGGL(k_staged_mark_solo, dim3(L.grid), dim3(kBlock), 0, L.stream, s, *batch);
    return hipGetLastError();
}

hipError_t launch_staged_check(const Launch &L, const Graph &g, const State &s) {
    hipLaunchKernelGGL(k_staged_check, dim3(kCheckGrid), dim3(kCheckThreads), 0, L.stream, g, s,
                       setup_grid(L) - 1);
    return hipGetLastError();
}

hipError_t launch_staged_sample(const Launch &L, const Graph &g, const State &s, uint32_t seed) {
    if (g.vbase) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_staged_sample, dim3(kSampleGrid), dim3(kWave), 0, L.stream, g, s, seed);
    return hipGetLastError();
}

hipError_t launch_staged_meet(const Launch &L, const Graph &g, const State &s, int next,
                              unsigned long long *out) {
    hipLaunchKernelGGL(k_staged_meet, dim3(1), dim3(kSetupThreads), 0, L.stream, g, s, next, out);
    return hipGetLastError();
}

hipError_t launch_staged_join(const Launch &L, const Graph &g, const State &s, int round,
                              int first, int second, uint32_t seed) {
    const dim3 grid(s.grid), block(kBlock);
    if (g.pairs)
        hipLaunchKernelGGL((k_staged_join<true, false>), grid, block, 0, L.stream, g, s, round,
                           first, second, seed);
    else if (g.vbase)
        hipLaunchKernelGGL((k_staged_join<false, true>), grid, block, 0, L.stream, g, s, round,
                           first, second, seed);
    else
        hipLaunchKernelGGL((k_staged_join<false, false>), grid, block, 0, L.stream, g, s, round,
                           first, second, seed);
    return hipGetLastError();
}

hipError_t launch_staged_test(const Launch &L, const Graph &g, const State &s, int round,
                              uint32_t *bits) {
    const dim3 grid(s.grid), block(kBlock);
    if (g.pairs)
        hipLaunchKernelGGL((k_staged_test<true, false>), grid, block, 0, L.stream, g, s, round,
                           bits);
    else if (g.vbase)
        hipLaunchKernelGGL((k_staged_test<false, true>), grid, block, 0, L.stream, g, s, round,
                           bits);
    else
        hipLaunchKernelGGL((k_staged_test<false, false>), grid, block, 0, L.stream, g, s, round,
                           bits);
    return hipGetLastError();
}

}  // namespace hgm
