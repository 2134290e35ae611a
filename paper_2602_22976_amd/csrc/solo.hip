// Instances matched whole by one workgroup, for gfx950.
//
// The same local-max rounds as kernels.hip (paper, Section 4.1), but every
// round of an instance runs inside one workgroup, so a round costs workgroup
// barriers instead of kernel launches.  The done bits of the vertices and
// their maximum keys live in LDS.
//
// The edges are admitted by threshold, the highest keys first (staged.hip says
// why the matching is the same): by the time most edges are admitted their
// pins are done and one read of the done bits in LDS drops them.
//
// Slots.  When an instance has more vertices than LDS holds maxima, vertices
// share slots.  A slot's maximum bounds that of each of its vertices from
// above, so an edge that equals its slots' maxima is a local maximum, and the
// largest live edge always does: sharing can only delay a match by a round,
// never change it.  With small steps few edges are live at a time and the
// visits stay those of unshared maxima (50,000 vertices on 16,384 slots: 24
// rounds instead of 9, 18 thousand edge visits either way).  Maxima outside LDS
// are no choice: even workgroup-scope atomics are performed at the memory side
// here, at 27 G/s for the whole chip (the batch of 4,096 took 5.2 ms).
//
// Calls whose result or counts depend on the round an edge is matched in
// (per-round counts, priorities redrawn every round) have at most one edge per
// thread here and a slot for every vertex.
#include <algorithm>

#include "internal.h"
#include "wave.h"

namespace hgm {
namespace {

constexpr int kSamples = 256;
constexpr int kSteps = 16;  // parts of the order: fifteen thresholds, then the rest
// Rank among the sampled keys of each threshold: parts growing by a third, from
// about a hundredth of the edges.
__device__ constexpr int kRank[kSteps - 1] = {2,  4,  6,  8,  11, 15,  20, 27,
                                              36, 48, 63, 83, 110, 145, 190};
// The parts up to this one, a tenth of the edges, are admitted before the others
// are looked at: by then seven of eight of those have a pin that is done.  (The
// batch: 2.44 ms; 2.48 with one part less, 2.44 and 2.48 with one and two more.
// Parts growing by a half 2.66, by a sixth 2.72: more edges share slots at a
// time, or more rounds.)
constexpr int kSplit = 6;
constexpr int kAdvance = 3;  // parts admitted per round where every vertex has its slot

constexpr int kU = 2;          // edges per lane and step: their loads overlap
constexpr int kGroup = kU * kWave;

// The last rounds keep one live edge per thread and this many pins per thread.
constexpr int kEndPins = 8;

template <int T>
struct SoloShared {
    union {
        int part[T / kWave][kSteps];  // each wave's edges by part: counts, then ends
        struct {  // the last rounds
            uint64_t key[T];
            int start[T];      // first pin of the edge among the gathered pins
            int base[T];       // offset of its pins less start
            uint32_t flag[T];
        } end;
        uint64_t sample[kSamples];
    };
    uint64_t th[kSteps - 1];
    unsigned long long sum[4];    // live pins; matched edges, their weight and pins
    int cnt[T / kWave];           // live edges of each wave's list
    int scan[T / kWave];
    int live[2];                  // live edges by round parity
    int inst;
};

// One instance as a workgroup sees it.
struct Inst {
    int nv, ne;
    const int32_t *e_off, *e_pins;
    const uint32_t *w;
    uint32_t seed;
    uint32_t *bits;
    int64_t words;  // of bits, those of a batch that no edge needs among them
    int64_t at;     // the instance's first slot in the workspace lists
};

__device__ __forceinline__ void add_wave(unsigned long long v, unsigned long long *sum) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    if (lane_id() == 0 && v) atomicAdd(sum, v);
}

// The state of an instance in LDS: done bits, then the slots' maxima.
template <bool kPairs>
struct SoloSide {
    const Inst &I;
    uint32_t *done;
    unsigned long long *max;
    int slots;       // fewer than vertices: shared
    uint32_t seed;   // the round's
    __device__ __forceinline__ uint32_t done_word(int v) const { return done[v >> 5]; }
    __device__ __forceinline__ unsigned long long &slot(int v) const {
        const uint32_t at = __umulhi((uint32_t)v * 0x9E3779B1u, (uint32_t)slots);
        return max[slots < I.nv ? (int)at : v];
    }
    __device__ __forceinline__ void raise(int v, uint64_t k) const {
        atomicMax(&slot(v), (unsigned long long)k);
    }
    __device__ __forceinline__ uint64_t key_of(uint32_t w, int e) const {
        return (uint64_t)w << 32 | priority_hash(seed, (uint32_t)e);
    }
    __device__ __forceinline__ uint64_t key(int e) const { return key_of(I.w[e], e); }
    __device__ __forceinline__ void place(int e, int &base, int &len) const {
        base = kPairs ? 2 * e : I.e_off[e];
        len = kPairs ? 2 : I.e_off[e + 1] - base;
    }
    __device__ __forceinline__ void mark(int v) const { atomicOr(&done[v >> 5], 1u << (v & 31)); }
    __device__ __forceinline__ void win(int e) const {
        atomicOr(&I.bits[e >> 5], 1u << (e & 31));
    }
};

// Lane-per-edge passes over the pins of kU edges per lane (edge u: len[u] pins
// from base[u]): check(pin, key, look(pin)) is asked of the pins until it
// holds (`every`: of all pins), four pins of each edge per step with all loads
// of a step issued before any is used; returns the edges it held for.  Pins
// beyond kLanePins of an edge are left to the whole wave, edge after edge: a
// lane walking thousands of pins would hold its workgroup.  All lanes of the
// wave call it (len 0: no edge).
constexpr int kLanePins = 32;
template <int kU, class Look, class Check>
__device__ __forceinline__ uint32_t lane_pins(const int32_t *e_pins, const int (&base)[kU],
                                              const int (&len)[kU], const uint64_t (&key)[kU],
                                              bool every, Look look, Check check) {
    uint32_t hit = 0;
    int most = 0;
#pragma unroll
    for (int u = 0; u < kU; ++u) most = len[u] > most ? len[u] : most;
    most = most < kLanePins ? most : kLanePins;
    for (int q = 0; q < most; q += 4) {
        int v[kU][4];
        decltype(look(0)) x[kU][4];
        uint32_t open = 0;  // edges with pins in this step
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const bool on = q < len[u] && (every || !(hit >> u & 1));
            open |= on ? 1u << u : 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[u][i] = on && q + i < len[u] ? e_pins[base[u] + q + i] : 0;
        }
        if (!open) break;
#pragma unroll
        for (int u = 0; u < kU; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) x[u][i] = look(v[u][i]);
#pragma unroll
        for (int u = 0; u < kU; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if ((open >> u & 1) && q + i < len[u] && check(v[u][i], key[u], x[u][i]))
                    hit |= 1u << u;
    }
    const int lane = lane_id();
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        unsigned long long more = __ballot(len[u] > kLanePins && (every || !(hit >> u & 1)));
        while (more) {
            const int l = __ffsll(more) - 1;
            more &= more - 1;
            const int b = __shfl(base[u], l, kWave), n = __shfl(len[u], l, kWave);
            const uint64_t k = (uint64_t)__shfl((uint32_t)(key[u] >> 32), l, kWave) << 32 |
                               __shfl((uint32_t)key[u], l, kWave);
            unsigned long long any = 0;
            for (int i0 = kLanePins; i0 < n && (every || !any); i0 += kWave) {
                const int i = i0 + lane, p = i < n ? e_pins[b + i] : 0;
                const auto x = look(p);
                any |= __ballot(i < n && check(p, k, x));
            }
            if (any && lane == l) hit |= 1u << u;
        }
    }
    return hit;
}

// act(pin, key) at every pin of the edges in `on`.
template <int kU, class Act>
__device__ __forceinline__ void lane_act(const int32_t *e_pins, const int (&base)[kU],
                                         const int (&len)[kU], const uint64_t (&key)[kU],
                                         uint32_t on, Act act) {
    int n[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) n[u] = (on >> u & 1) ? len[u] : 0;
    lane_pins<kU>(e_pins, base, n, key, true, NoRead(), [&](int v, uint64_t k, int) {
        act(v, k);
        return false;
    });
}

// A listed edge: its id, pin offset and count, its weight, its first pins.
constexpr int kHead = 4;
struct EdgeHead {
    uint4 edge;
    int4 pin;
};

__device__ __forceinline__ void load_head(const int32_t *e_pins, int len, EdgeHead &h) {
    const int b = (int)h.edge.y;
    h.pin.x = len > 0 ? e_pins[b] : 0;
    h.pin.y = len > 1 ? e_pins[b + 1] : 0;
    h.pin.z = len > 2 ? e_pins[b + 2] : 0;
    h.pin.w = len > 3 ? e_pins[b + 3] : 0;
}

// The same passes for listed edges: their first pins are at hand.
template <int kU, class Look, class Check>
__device__ __forceinline__ uint32_t head_pins(const int32_t *e_pins, const EdgeHead (&h)[kU],
                                              const uint64_t (&key)[kU], uint32_t on, bool every,
                                              Look look, Check check) {
    uint32_t hit = 0;
    decltype(look(0)) x[kU][kHead];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        x[u][0] = look(h[u].pin.x);
        x[u][1] = look(h[u].pin.y);
        x[u][2] = look(h[u].pin.z);
        x[u][3] = look(h[u].pin.w);
    }
    int base[kU], len[kU], most = 0;
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        const int n = (on >> u & 1) ? (int)h[u].edge.z : 0;
        if (n > 0 && check(h[u].pin.x, key[u], x[u][0])) hit |= 1u << u;
        if (n > 1 && check(h[u].pin.y, key[u], x[u][1])) hit |= 1u << u;
        if (n > 2 && check(h[u].pin.z, key[u], x[u][2])) hit |= 1u << u;
        if (n > 3 && check(h[u].pin.w, key[u], x[u][3])) hit |= 1u << u;
        base[u] = (int)h[u].edge.y + kHead;
        len[u] = n > kHead && (every || !(hit >> u & 1)) ? n - kHead : 0;
        most = len[u] > most ? len[u] : most;
    }
    if (__any(most > 0)) hit |= lane_pins<kU>(e_pins, base, len, key, every, look, check);
    return hit;
}

template <int kU, class Act>
__device__ __forceinline__ void head_act(const int32_t *e_pins, const EdgeHead (&h)[kU],
                                         const uint64_t (&key)[kU], uint32_t on, Act act) {
    head_pins<kU>(e_pins, h, key, on, true, NoRead(), [&](int v, uint64_t k, int) {
        act(v, k);
        return false;
    });
}

// The list rounds of an instance of more edges than threads.  Each wave owns a
// range of edge ids, `per` long, and writes records of its edges to its range
// of J.edges: in a first phase of the edges of the first parts, found by their
// weights; when those are admitted, of the others those that are not dead,
// found in one pass over the pins in order.  A phase's records are listed by
// part of the order (the number of thresholds above the key); a round admits a
// part or more, and the live edges stay in the same list, compacted by ballot
// over entries already read.  Ends after a round's test, when every part is
// admitted and at most T edges are listed: returns their number, with *kept
// those of this wave.
//
// Bound by memory.  A part's edges lie far apart: gathered by id as they are
// admitted, each costs a line for its offsets, its weight and its pins.  The
// batch of 4,096 instances with 4.6e8 pins: 3.75 ms so; 2.91 ms with a record of
// every edge sorted first; 2.53 ms in two phases; 2.44 ms with places sorted
// instead of records, by halving (6.6e7 reads and 1.6e7 writes leave L2; the
// pins alone are 1.4e7 lines).  What is left is the pass over the pins and the
// rounds, a chain of memory accesses.
template <int T>
__device__ __forceinline__ int solo_lists(const Inst &I, const SoloJob &J, SoloShared<T> &S,
                                          SoloSide<false> &m, int per, int *kept_out) {
    constexpr int kLast = kSteps - 1, kW = T / kWave;
    static_assert(kW * kWave == T && T % kSamples == 0, "whole waves, whole sample groups");
    const int tid = threadIdx.x, wid = tid / kWave, lane = lane_id();
    int *const part_end = S.part[wid];
    const int lo = wid * per < I.ne ? wid * per : I.ne, end = lo + per < I.ne ? lo + per : I.ne;
    // From the first step that admits at least one edge per thread: a round of
    // fewer costs the same.
    int step = kLast;
    if (I.ne > 2 * T)
        for (int q = kLast - 1; q >= 0; --q)
            if ((int64_t)(kRank[q] + 1) * I.ne >= (int64_t)kSamples * T) step = q;
    if (step < kLast) {
        if (tid < kSamples) {
            const int at = (int)(((int64_t)tid * I.ne) / kSamples);
            const uint32_t width = (uint32_t)(I.ne / kSamples);
            S.sample[tid] = m.key(at + (int)(priority_hash(I.seed, 0x5eedu + tid) % width));
        }
        __syncthreads();
        constexpr int kParts = T / kSamples;  // lanes per sample
        const int i = tid / kParts, part = tid % kParts;
        const uint64_t sample = S.sample[i];
        int rank = 0;
#pragma unroll 8
        for (int q = part; q < kSamples; q += kParts) rank += S.sample[q] > sample ? 1 : 0;
#pragma unroll
        for (int o = 1; o < kParts; o <<= 1) rank += __shfl_xor(rank, o, kWave);
#pragma unroll
        for (int q = 0; q < kLast; ++q)
            if (part == 0 && rank == kRank[q]) S.th[q] = sample;
    } else if (tid < kLast) {
        S.th[tid] = 0;  // no edge is below a threshold
    }
    __syncthreads();
    auto part_of = [&](int e, uint32_t w) -> int {
        const uint64_t k = m.key_of(w, e);
        int part = 0;  // thresholds above the key: they fall
        static_assert(kSteps == 16, "four halvings");
#pragma unroll
        for (int q = 8; q > 0; q >>= 1) part += k < S.th[part + q - 1] ? q : 0;
        return part;
    };
    const int split = step > kSplit ? step : kSplit;  // kLast: one phase
    const uint64_t bound = split < kLast ? S.th[split] : 0;  // of the first phase's keys
    EdgeHead *const edges = reinterpret_cast<EdgeHead *>(J.edges) + I.at + lo;
    uint2 *const picked = J.picked + I.at + lo;  // {id, weight} of the first phase's edges,
    uint32_t *const list = reinterpret_cast<uint32_t *>(picked);  // then places in `edges`
    const int advance = m.slots < I.nv ? 1 : kAdvance;
    auto first = [&](uint32_t w, int e) {
        const uint32_t bw = (uint32_t)(bound >> 32);
        return w == bw ? m.key_of(w, e) >= bound : w > bw;
    };
    int records = 0, kept = 0, before = -1;  // parts up to `before` are admitted
    for (int r = 0, phase = 0;; ++phase) {
        const int old = records;
        if (phase == 0) {
            constexpr int kPickU = 4;
            int count = 0;
            for (int c0 = lo; c0 < end; c0 += kPickU * kWave) {
                uint32_t w[kPickU];
#pragma unroll
                for (int u = 0; u < kPickU; ++u) {
                    const int e = c0 + u * kWave + lane;
                    w[u] = e < end ? I.w[e] : 0;
                }
#pragma unroll
                for (int u = 0; u < kPickU; ++u) {
                    const int e = c0 + u * kWave + lane;
                    const bool take = e < end && first(w[u], e);
                    const uint64_t mask = __ballot(take);
                    if (take) picked[count + bits_below(mask)] = make_uint2((uint32_t)e, w[u]);
                    count += __popcll(mask);
                }
            }
            wave_fence();
            for (int c0 = 0; c0 < count; c0 += kU * kWave) {
                EdgeHead h[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const int i = c0 + u * kWave + lane;
                    const uint2 x = picked[i < count ? i : c0];
                    h[u].edge = make_uint4(x.x, (uint32_t)I.e_off[x.x], (uint32_t)I.e_off[x.x + 1],
                                           x.y);
                }
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    h[u].edge.z -= h[u].edge.y;
                    load_head(I.e_pins, (int)h[u].edge.z, h[u]);
                }
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const int i = c0 + u * kWave + lane;
                    if (i < count) edges[i] = h[u];
                }
            }
            records = count;
        } else {
            for (int c0 = lo; c0 < end; c0 += kU * kWave) {
                EdgeHead h[kU];
                const uint64_t key[kU] = {0};  // not looked at
                uint32_t on = 0;
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const int e = c0 + u * kWave + lane, at = e < end ? e : lo;
                    h[u].edge = make_uint4((uint32_t)e, (uint32_t)I.e_off[at],
                                           (uint32_t)I.e_off[at + 1], I.w[at]);
                }
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    h[u].edge.z -= h[u].edge.y;
                    if ((int)h[u].edge.x < end && !first(h[u].edge.w, (int)h[u].edge.x))
                        on |= 1u << u;
                    load_head(I.e_pins, (on >> u & 1) ? (int)h[u].edge.z : 0, h[u]);
                }
                const uint32_t dead = head_pins<kU>(
                    I.e_pins, h, key, on, false, [&](int v) { return m.done_word(v); },
                    [](int v, uint64_t, uint32_t word) { return (bool)((word >> (v & 31)) & 1u); });
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const bool take = (on & ~dead) >> u & 1;
                    const uint64_t mask = __ballot(take);
                    if (take) edges[records + bits_below(mask)] = h[u];
                    records += __popcll(mask);
                }
            }
        }
        // ---- list them by part, behind the edges still listed
        int next = kept;  // the first entry not admitted
        if (lane < kSteps) part_end[lane] = 0;
        wave_fence();
        for (int pass = 0; pass < 2; ++pass) {
            for (int c0 = old; c0 < records; c0 += kU * kWave) {
                uint4 x[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const int i = c0 + u * kWave + lane;
                    x[u] = edges[i < records ? i : c0].edge;
                }
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const int i = c0 + u * kWave + lane;
                    if (i < records) {
                        const int at = atomicAdd(&part_end[part_of((int)x[u].x, x[u].w)], 1);
                        if (pass) list[at] = (uint32_t)i;
                    }
                }
            }
            wave_fence();
            if (pass == 0) {  // counts to starts; the second pass moves them to the ends
                const int c = lane < kSteps ? part_end[lane] : 0;
                const int begin = next + wave_inclusive_sum(c) - c;
                wave_fence();
                if (lane < kSteps) part_end[lane] = begin;
                wave_fence();
            }
        }
        // ---- the rounds that admit them
        const int last = phase == 0 ? split : kLast;
        for (;; ++r) {
            // ---- join: the survivors of the list, then the round's parts
            if (step > last && before < last) step = last;
            const int listed = kept;
            const int stop = step > last ? next : part_end[step];
            kept = 0;
            for (int i0 = 0; i0 < listed || next < stop;) {
                const bool again = i0 < listed;
                const int from = again ? i0 : next, to = again ? listed : stop;
                EdgeHead h[kU];
                uint32_t at[kU];
                uint64_t key[kU];
                uint32_t on = 0;
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const int i = from + u * kWave + lane;
                    at[u] = list[i < to ? i : from];
                }
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const int i = from + u * kWave + lane;
                    h[u] = edges[at[u]];
                    // A listed empty edge was matched by its test.
                    if (i < to && !(again && h[u].edge.z == 0)) on |= 1u << u;
                    key[u] = m.key_of(h[u].edge.w, (int)h[u].edge.x);
                }
                if (again)
                    i0 += kGroup;
                else
                    next = next + kGroup < stop ? next + kGroup : stop;
                const uint32_t dead = head_pins<kU>(
                    I.e_pins, h, key, on, false, [&](int v) { return m.done_word(v); },
                    [](int v, uint64_t, uint32_t word) { return (bool)((word >> (v & 31)) & 1u); });
                const uint32_t live = on & ~dead;
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const bool l = live >> u & 1;
                    const uint64_t mask = __ballot(l);
                    if (l) list[kept + bits_below(mask)] = at[u];
                    kept += __popcll(mask);
                }
                head_act<kU>(I.e_pins, h, key, live, [&](int v, uint64_t k) { m.raise(v, k); });
            }
            before = step;
            step += advance;
            if (lane == 0 && kept) atomicAdd(&S.live[r & 1], kept);
            __syncthreads();
            const int E = S.live[r & 1];
            // ---- test
            for (int i0 = 0; i0 < kept; i0 += kGroup) {
                EdgeHead h[kU];
                uint64_t key[kU];
                uint32_t on = 0;
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const int i = i0 + u * kWave + lane;
                    h[u] = edges[list[i < kept ? i : i0]];
                    on |= i < kept ? 1u << u : 0;
                    key[u] = m.key_of(h[u].edge.w, (int)h[u].edge.x);
                }
                const uint32_t lost = head_pins<kU>(
                    I.e_pins, h, key, on, false, [&](int v) { return m.slot(v); },
                    [](int, uint64_t k, unsigned long long b) { return b != k; });
                const uint32_t won = on & ~lost;
#pragma unroll
                for (int u = 0; u < kU; ++u)
                    if (won >> u & 1) m.win((int)h[u].edge.x);
                head_act<kU>(I.e_pins, h, key, won, [&](int v, uint64_t) { m.mark(v); });
            }
            __syncthreads();
            if (tid == 0) S.live[r & 1 ^ 1] = 0;
            for (int i = tid; i < m.slots; i += T) m.max[i] = 0;
            if (before >= kLast && E <= T) {
                *kept_out = kept;
                return E;
            }
            __syncthreads();
            if (before >= last && last < kLast) break;
        }
        ++r;
    }
}

// One instance, every round, by T threads.  kMany: it may have more edges than
// threads (calls with exact rounds do not).
template <int T, bool kPairs, bool kMany>
__device__ __forceinline__ void solo_match(const Inst &I, const SoloJob &J, SoloShared<T> &S,
                                           unsigned char *lds) {
    const int tid = threadIdx.x, wid = tid / kWave, lane = lane_id();
    const bool exact = J.exact != 0, rekey = J.reseed != 0;
    const int dwords = (I.nv + 31) >> 5;
    const int room = (J.lds_bytes - (int)solo_done_bytes(I.nv)) / 8;
    SoloSide<kPairs> m{I,
                       reinterpret_cast<uint32_t *>(lds),
                       reinterpret_cast<unsigned long long *>(lds + solo_done_bytes(I.nv)),
                       I.nv < room ? I.nv : room,
                       rekey ? round_seed(I.seed, 0) : I.seed};
    for (int i = tid; i < dwords; i += T) m.done[i] = 0;
    for (int i = tid; i < m.slots; i += T) m.max[i] = 0;
    for (int64_t i = tid; i < I.words; i += T) I.bits[i] = 0;
    if (tid < 2) S.live[tid] = 0;
    if (tid < 4) S.sum[tid] = 0;
    __syncthreads();

    // One live edge per thread.
    bool mine = tid < I.ne, tested = false;
    int e = tid, base = 0, len = 0;
    uint64_t key = 0;
    if (!kMany || I.ne <= T) {
        if (mine) {
            m.place(e, base, len);
            key = m.key(e);
        }
    } else if constexpr (kMany) {
        constexpr int kW = T / kWave;
        static_assert(!kPairs, "batches have no graph layout");
        const int per = ((I.ne + kW - 1) / kW + kWave - 1) / kWave * kWave;
        int kept = 0;
        const int E = solo_lists<T>(I, J, S, m, per, &kept);
        if (lane == 0) S.cnt[wid] = kept;
        __syncthreads();
        mine = tid < E;
        tested = true;
        if (mine) {
            int from = 0, at = tid;
            for (; at >= S.cnt[from]; ++from) at -= S.cnt[from];
            const int64_t i = I.at + (int64_t)from * per;  // the wave's range
            const uint4 x =
                J.edges[2 * (i + reinterpret_cast<const uint32_t *>(J.picked + i)[at])];
            e = (int)x.x;
            base = (int)x.y;
            len = (int)x.z;
            key = m.key_of(x.w, e);
        }
    }

    // The last rounds.  An edge that was tested is dropped first where a pin
    // is done.
    int r = 0;                                  // the round (exact calls)
    unsigned long long tot_m = 0, tot_w = 0;    // thread 0, exact calls
    auto close_round = [&](int E) {             // after a barrier behind the test
        if (exact && tid == 0) {
            if (r < J.row_cap) {
                unsigned long long *row = J.rows + 5 * (int64_t)r;
                row[0] = (unsigned long long)E;
                for (int q = 0; q < 4; ++q) row[q + 1] = S.sum[q];
            }
            if (J.host && r < J.host_rows) {
                unsigned long long *row = J.host + kSoloJobHeader + 5 * (int64_t)r;
                row[0] = (unsigned long long)E;
                for (int q = 0; q < 4; ++q) row[q + 1] = S.sum[q];
            }
            tot_m += S.sum[1];
            tot_w += S.sum[2];
            for (int q = 0; q < 4; ++q) S.sum[q] = 0;
        }
        ++r;
        if (rekey) m.seed = round_seed(I.seed, r);
        tested = true;
    };
    auto count = [&](bool won) {
        if (!exact) return;
        add_wave(won ? 1 : 0, &S.sum[1]);
        add_wave(won ? key >> 32 : 0, &S.sum[2]);
        add_wave(won ? (unsigned long long)len : 0, &S.sum[3]);
    };
    int total;
    const int n = len < kEndPins * T ? len : kEndPins * T + 1;
    const int first = workgroup_scan<T>(mine ? n : 0, S.scan, &total);
    bool alive = mine && (len > 0 || !tested);
    if (total > kEndPins * T) {
        // More pins than the workgroup's registers take: lane per edge.
        const int b1[1] = {base};
        for (;;) {
            const uint64_t k1[1] = {key};
            const int n1[1] = {alive ? len : 0};
            if (tested) {
                const uint32_t dead = lane_pins<1>(
                    I.e_pins, b1, n1, k1, true, [&](int v) { return m.done_word(v); },
                    [&](int v, uint64_t, uint32_t word) {
                        m.slot(v) = 0;
                        return (bool)((word >> (v & 31)) & 1u);
                    });
                alive = alive && !dead && len > 0;
            }
            const int E = __syncthreads_count(alive);
            if (E == 0) break;
            if (rekey && alive) key = m.key_of((uint32_t)(key >> 32), e);
            const uint64_t k2[1] = {key};
            const int n2[1] = {alive ? len : 0};
            lane_act<1>(I.e_pins, b1, n2, k2, 1u, [&](int v, uint64_t k) { m.raise(v, k); });
            if (exact) add_wave((unsigned long long)n2[0], &S.sum[0]);
            __syncthreads();
            const uint32_t lost = lane_pins<1>(
                I.e_pins, b1, n2, k2, false, [&](int v) { return m.slot(v); },
                [](int, uint64_t k, unsigned long long b) { return b != k; });
            const bool won = alive && !lost;
            if (won) m.win(e);
            lane_act<1>(I.e_pins, b1, n2, k2, won ? 1u : 0u, [&](int v, uint64_t) { m.mark(v); });
            count(won);
            __syncthreads();
            close_round(E);
        }
    } else {
        // Every pin in a register of some thread, spread over the workgroup.
        S.end.start[tid] = mine ? first : total;
        S.end.base[tid] = base - first;
        S.end.key[tid] = key;
        S.end.flag[tid] = 0;
        __syncthreads();
        constexpr uint32_t kLost = 1, kDead = 2, kWon = 4;
        int own[kEndPins], v[kEndPins];
        uint32_t open = 0;  // this thread's pins whose edge is alive
#pragma unroll
        for (int i = 0; i < kEndPins; ++i) {
            const int t = i * T + tid;
            own[i] = v[i] = 0;
            if (t < total) {
                int j = 0;  // the last edge that starts at or before t
#pragma unroll
                for (int q = T / 2; q > 0; q >>= 1)
                    if (S.end.start[j + q] <= t) j += q;
                own[i] = j;
                v[i] = I.e_pins[S.end.base[j] + t];
                open |= 1u << i;
            }
        }
        for (;;) {
            if (tested) {
#pragma unroll
                for (int i = 0; i < kEndPins; ++i)
                    if (open >> i & 1) {
                        if (m.done_word(v[i]) >> (v[i] & 31) & 1) atomicOr(&S.end.flag[own[i]], kDead);
                        m.slot(v[i]) = 0;
                    }
                __syncthreads();
#pragma unroll
                for (int i = 0; i < kEndPins; ++i)
                    if ((open >> i & 1) && (S.end.flag[own[i]] & kDead)) open &= ~(1u << i);
                alive = alive && !(S.end.flag[tid] & (kDead | kWon));
                if (rekey && alive)
                    S.end.key[tid] = key = m.key_of((uint32_t)(key >> 32), e);
            }
            const int E = __syncthreads_count(alive);
            if (E == 0) break;
#pragma unroll
            for (int i = 0; i < kEndPins; ++i)
                if (open >> i & 1) m.raise(v[i], S.end.key[own[i]]);
            if (exact) add_wave(alive ? (unsigned long long)len : 0, &S.sum[0]);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kEndPins; ++i)
                if ((open >> i & 1) && m.slot(v[i]) != S.end.key[own[i]])
                    atomicOr(&S.end.flag[own[i]], kLost);
            __syncthreads();
            const bool won = alive && !(S.end.flag[tid] & kLost);
            if (won) m.win(e);
            if (alive) S.end.flag[tid] = won ? kWon : 0;
            count(won);
            __syncthreads();
            close_round(E);
#pragma unroll
            for (int i = 0; i < kEndPins; ++i)
                if ((open >> i & 1) && (S.end.flag[own[i]] & kWon)) m.mark(v[i]);
            __syncthreads();
        }
    }
    if (exact && tid == 0 && J.host) {
        J.host[kSoloJobRounds] = (unsigned long long)r;
        J.host[kSoloJobMatched] = tot_m;
        J.host[kSoloJobWeight] = tot_w;
    }
    if (exact && tid == 0) {
        J.ctl[kSoloJobRounds] = (unsigned long long)r;
        J.ctl[kSoloJobMatched] = tot_m;
        J.ctl[kSoloJobWeight] = tot_w;
    }
}

template <bool kPairs>
__global__ void __launch_bounds__(kSoloOneThreads) k_solo_one(SoloJob J) {
    extern __shared__ __align__(16) unsigned char solo_lds[];
    __shared__ SoloShared<kSoloOneThreads> S;
    const Inst I{J.n, J.m, J.e_off, J.e_pins, J.w, J.seed, J.bits, ((int64_t)J.m + 31) / 32, 0};
    solo_match<kSoloOneThreads, kPairs, false>(I, J, S, solo_lds);
}

// Workgroups take the batch's instances from a counter, in the order that
// k_solo_order wrote: the wide ones first, or (kSmall) those behind them.
template <int T, bool kSmall>
__global__ void __launch_bounds__(T, 4) k_solo_batch(SoloJob J) {
    extern __shared__ __align__(16) unsigned char solo_lds[];
    __shared__ SoloShared<T> S;
    constexpr int kNext = kSmall ? kSoloJobNextSmall : kSoloJobNextWide;
    const int wide = (int)J.ctl[kSoloJobWide];
    const int begin = kSmall ? wide : 0;
    const int n = kSmall ? (int)J.ctl[kSoloJobCount] : wide;
    for (;;) {
        if (threadIdx.x == 0) S.inst = begin + (int)atomicAdd(&J.ctl[kNext], 1ull);
        __syncthreads();
        const int q = S.inst;
        __syncthreads();  // every thread has read the index before it is overwritten
        if (q >= n) break;
        const int i = J.order[q];
        const int64_t v0 = J.v_base[i], e0 = J.e_base[i];
        const Inst I{(int)(J.v_base[i + 1] - v0),
                     (int)(J.e_base[i + 1] - e0),
                     J.e_off + e0 + i,
                     J.e_pins + J.pin_base[i],
                     J.w + e0,
                     J.seeds[i],
                     J.bits + J.word_base[i],
                     J.word_base[i + 1] - J.word_base[i],
                     e0};
        solo_match<T, false, true>(I, J, S, solo_lds);
        __syncthreads();
    }
}

// Lists the batch's solo instances: those too wide for a small workgroup's LDS,
// then the others, each by falling size class (bit length of solo_size), so that
// the longest start first; and counts the instances left to the round kernels.
// One workgroup.
//
// With J.choose the bound on an instance's pins is the default, and the whole
// solo part is left out when its longest instance would outlast the round
// kernels on the whole batch: a workgroup matches about 1e6 pins a millisecond
// after 0.1 ms, the grid's rounds take about 0.15 ms and 1 ms per 6e7 pins, and
// running both parts costs the fixed time of both.  (Instances of up to 7e5
// pins, rounds / here in ms: 400 of them, 4e7 pins, 0.78 / 0.93; 512 0.98 /
// 0.87; 1,500, 1.6e8, 2.60 / 1.17.  Up to 7e4: 256, 4.2e6, 0.23 / 0.28.  Up to
// 2.8e5: 400, 1.9e7, 0.41 / 0.49.  Up to 3.8e4: 2, 4e4, 0.14 / 0.12; 64, 6.8e5,
// 0.14 / 0.12; 1,000, 1.05e7, 0.31 / 0.17.)
//
// An instance with few pins a vertex keeps most of its edges alive, and where
// its vertices share slots it needs many rounds, the more the longer its edges
// are: it takes about as long as one of solo_sparse_pins.  The grid's time on
// such batches goes with the vertices, too, about 30 of them a pin.  (1, 16, 64
// and 256 instances of 100,000 vertices, us, rounds over all edges / here / the
// grid by admission.  1,000 edges of 32 pins: 239 / 620 / 148, 286 / 695 / 208,
// 375 / 706 / 314, 1,067 / 753 / 755.  20,000 edges of 2: 141 / 216 / 185, 199 /
// 229 / 247, 428 / 249 / 478, 1,096 / 383 / 1,603.  30,000 vertices, 15,000 edges
// of 2: 134 / 160 / 165, 184 / 168 / 192, 286 / 180 / 331, 631 / 240 / 894.)
constexpr int kOrderThreads = 1024;
__global__ void __launch_bounds__(kOrderThreads) k_solo_order(SoloJob J) {
    constexpr int kClasses = 128;
    __shared__ int count[kClasses], start[kClasses], rest;
    __shared__ unsigned long long longest, sparse;
    const int tid = threadIdx.x;
    if (tid < kClasses) count[tid] = 0;
    if (tid == 0) {
        rest = 0;
        longest = 0;
        sparse = 0;
    }
    __syncthreads();
    if (J.choose) {
        unsigned long long most = 0, most_sparse = 0;
        for (int i = tid; i < J.count; i += kOrderThreads) {
            const int64_t n = J.v_base[i + 1] - J.v_base[i];
            const int64_t k = solo_size(J.e_base, J.pin_base, i);
            if (k > J.max_size || n > J.max_verts) continue;
            const int64_t p = solo_sparse_pins(n, J.e_base[i + 1] - J.e_base[i],
                                               J.pin_base[i + 1] - J.pin_base[i], J.own_verts);
            most = max(most, (unsigned long long)k);
            most_sparse = max(most_sparse, (unsigned long long)p);
        }
        atomicMax(&longest, most);
        atomicMax(&sparse, most_sparse);
        __syncthreads();
    }
    const int64_t bound = solo_longest(J.pin_base[J.count]);
    const bool none = J.choose && ((int64_t)longest > bound ||
                                   (int64_t)sparse > bound + J.v_base[J.count] / kGridVerts);
    auto size_class = [&](int i) -> int {  // -1: left to the round kernels, -2: nothing to match
        const int64_t n = J.v_base[i + 1] - J.v_base[i];
        const int64_t k = solo_size(J.e_base, J.pin_base, i);
        if (J.e_base[i + 1] == J.e_base[i]) return -2;
        if (none || k > J.max_size || n > J.max_verts) return -1;
        return (n > J.small_verts ? 0 : 64) + (k > 0 ? __clzll(k) : 63);
    };
    for (int i = tid; i < J.count; i += kOrderThreads) {
        const int c = size_class(i);
        if (c >= 0) atomicAdd(&count[c], 1);
        if (c == -1) atomicAdd(&rest, 1);
    }
    __syncthreads();
    if (tid == 0) {
        int at = 0;
        for (int c = 0; c < kClasses; ++c) {
            if (c == 64) J.ctl[kSoloJobWide] = (unsigned long long)at;
            start[c] = at;
            at += count[c];
        }
        J.ctl[kSoloJobNextSmall] = 0;
        J.ctl[kSoloJobNextWide] = 0;
        J.ctl[kSoloJobCount] = (unsigned long long)at;
        J.report[0] = (int64_t)at;
        J.report[1] = (int64_t)rest;
    }
    __syncthreads();
    for (int i = tid; i < J.count; i += kOrderThreads) {
        const int c = size_class(i);
        if (c >= 0) J.order[atomicAdd(&start[c], 1)] = i;
        if (c == -2)  // not listed: any words it has are cleared here
            for (int64_t q = J.word_base[i]; q < J.word_base[i + 1]; ++q) J.bits[q] = 0;
    }
}

template <int T>
constexpr int static_lds() {
    return (int)sizeof(SoloShared<T>) + 256;
}

// LDS that a workgroup of T threads has beside its own variables when
// `per_cu` of them share a compute unit with `lds` bytes.
template <int T>
int room(int lds, int per_cu) {
    const int bytes = lds / per_cu - static_lds<T>();
    return bytes > 0 ? bytes & ~255 : 0;
}

// Most vertices whose done bits and maxima fit `bytes`.
int own_slots(int bytes) {
    const int64_t n = 32 * (int64_t)(bytes - 16) / (4 + 8 * 32);
    return n > 0 ? (int)n : 0;
}

template <bool kPairs>
hipError_t launch_one(hipStream_t stream, const SoloJob &J) {
    static LdsGrant lds;
    const hipError_t rc = lds.ensure(&k_solo_one<kPairs>, J.lds_bytes);
    if (rc != hipSuccess) return rc;
    hipLaunchKernelGGL(k_solo_one<kPairs>, dim3(1), dim3(kSoloOneThreads), J.lds_bytes, stream, J);
    return hipGetLastError();
}

template <int T, bool kSmall>
hipError_t launch_batch(hipStream_t stream, SoloJob J, int workgroups, int lds) {
    static LdsGrant grant;
    J.lds_bytes = lds;
    const hipError_t rc = grant.ensure(&k_solo_batch<T, kSmall>, lds);
    if (rc != hipSuccess) return rc;
    hipLaunchKernelGGL((k_solo_batch<T, kSmall>), dim3(workgroups), dim3(T), lds, stream, J);
    return hipGetLastError();
}

}  // namespace

int solo_wide_own_verts(int lds) { return own_slots(room<kSoloWideThreads>(lds, kSoloWidePerCu)); }

int solo_one_max_verts(int lds, bool exact) {
    const int bytes = room<kSoloOneThreads>(lds, 1);
    return exact ? own_slots(bytes) : 4 * bytes;  // done bits in half of it
}

hipError_t launch_solo_one(hipStream_t stream, SoloJob J, bool pairs, int lds) {
    const int64_t full = solo_done_bytes(J.n) + 8 * (int64_t)J.n;
    J.lds_bytes = (int)std::min<int64_t>(full, room<kSoloOneThreads>(lds, 1));
    return pairs ? launch_one<true>(stream, J) : launch_one<false>(stream, J);
}

hipError_t launch_solo_batch(hipStream_t stream, SoloJob J, int64_t n_total, int cus, int lds) {
    constexpr int kSmall = kSoloSmallThreads, kWide = kSoloWideThreads;
    const int small_lds = room<kSmall>(lds, kSoloSmallPerCu);
    const int wide_lds = room<kWide>(lds, kSoloWidePerCu);
    const int64_t most = n_total < J.max_verts ? n_total : J.max_verts;
    const int64_t full = solo_done_bytes(most) + 8 * most;
    J.small_verts = own_slots(small_lds);
    J.own_verts = solo_wide_own_verts(lds);
    if (J.small_verts <= 0 || solo_done_bytes(most) > wide_lds / 2) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_solo_order, dim3(1), dim3(kOrderThreads), 0, stream, J);
    hipError_t rc = hipGetLastError();
    if (rc == hipSuccess && most > J.small_verts)
        rc = launch_batch<kWide, false>(stream, J, std::min(J.count, kSoloWidePerCu * cus),
                                        (int)std::min<int64_t>(wide_lds, full));
    if (rc == hipSuccess)
        rc = launch_batch<kSmall, true>(stream, J, std::min(J.count, kSoloSmallPerCu * cus),
                                        (int)std::min<int64_t>(small_lds, full));
    return rc;
}

}  // namespace hgm
