// The end of a batch of rounds, for gfx950: the counters that the host reads,
// and the last rounds in one workgroup.
//
// Late rounds have few live edges, and two launches a round then cost far more
// than their work.  After the pass that forms a round's live lists, when at
// most kEdges edges with at most kPins pins are left, one workgroup gathers
// them, numbers their vertices through a hash table in LDS and runs every
// remaining round there: a round is a handful of barriers.  (A workgroup that
// keeps the maxima and the done marks in global memory is no faster than the
// grid: a round is then a chain of memory accesses, too.)  Round by round it
// does what the grid's rounds do, so per-round counts and priorities redrawn
// every round hold.
//
// 20 to 42 us for the last 4 to 8 rounds, where the grid's two kernels take 13
// to 17 us a round plus a read of the counters (two pageable copies and a
// wait, about 25 us, every few rounds).  Calls with statistics before and
// after: 100,000 pins 194 -> 145 us; a graph of 400,000 edges 236 -> 203 us;
// vertex passes, 3.5 M pins 434 -> 383 us; per-round priorities, 4.1 M pins 525
// -> 434 us (runs of one side differ by 17%); 30 M pins by 3%.
#include "internal.h"
#include "wave.h"

namespace hgm {
namespace {

constexpr int kThreads = 1024, kEdges = 2048, kPins = 8192, kSlots = 12288;
constexpr int kPinsPerThread = kPins / kThreads, kEdgesPerThread = kEdges / kThreads;
struct EndShared {
    union {
        unsigned long long best[kSlots];
        int id[kSlots];  // while the vertices are numbered
    };
    uint64_t key[kEdges];
    int start[kEdges];   // first pin of the edge among the gathered pins
    int base[kEdges];    // offset of its pins less start
    int vb[kEdges];
    uint32_t flag[kEdges];
    uint32_t done[kSlots / 32];
    int scan[kThreads / kWave];
    unsigned long long sum[4];  // live pins; matched edges, their weight and pins
};

__device__ __forceinline__ unsigned long long wave_total(unsigned long long v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

template <bool kPairs, bool kB>
__global__ void __launch_bounds__(kThreads) k_end(Graph g, State s, EndArgs a, uint32_t *bits) {
    extern __shared__ __align__(16) unsigned char end_lds[];
    EndShared &S = *reinterpret_cast<EndShared *>(end_lds);
    const int tid = threadIdx.x, wid = tid / kWave, lane = lane_id();
    const int k = a.round & 1;
    static_assert(kSub == kWave, "one counter per lane");
    // The counters of the rounds since the last check, a wave per round.
    if (a.counting) {
        for (int r = a.first + wid; r <= a.round; r += kThreads / kWave) {
            const RoundStats &st = s.stats[r % s.ring];
            const unsigned long long v[5] = {
                wave_total(st.live[lane]), wave_total(st.kappa[lane]), wave_total(st.matched[lane]),
                wave_total(st.weight[lane]), wave_total(st.mpins[lane])};
            if (lane == 0) {
                for (int q = 0; q < 5; ++q) a.report[kEndHeader + 5 * (r - a.first) + q] = v[q];
                if (st.bin_overflow) a.report[kEndOverflow] = 1;
            }
        }
    }
    if (a.check_bins) {
        const int found = *s.piece_count;
        for (int j = tid; found == kBinsCompare && j < s.bin_nb; j += kThreads) {
            const int64_t v0 = (int64_t)j << s.bin_rb, v1 = v0 + ((int64_t)1 << s.bin_rb);
            const int64_t sum = (int64_t)g.v_off[v1 < g.n ? v1 : g.n] - g.v_off[v0];
            if (sum != (int64_t)s.bin_cursor[j]) a.report[kEndOverflow] = 1;
        }
        if (found == kBinsBadOffsets && tid == 0) a.report[kEndOverflow] = 2;
    }
    const unsigned long long live = wave_total(s.stats[a.round % s.ring].live[lane]);
    const bool limit = !a.run || (a.max_rounds > 0 && a.round >= a.max_rounds);
    if (live == 0 || live > (unsigned long long)kEdges || limit) {
        if (tid == 0) {
            a.report[kEndFinished] = live == 0;
            a.report[kEndRounds] = (unsigned long long)a.round;
        }
        return;
    }
    // Gather: each thread takes consecutive lists.
    const int per = (a.lists + kThreads - 1) / kThreads;
    const int w0 = tid * per, w1 = min(w0 + per, a.lists);
    int mine = 0, E;
    for (int w = w0; w < w1; ++w) mine += a.counts[k][w];
    int at = workgroup_scan<kThreads>(mine, S.scan, &E);
    for (int w = w0; w < w1 && mine > 0; ++w) {
        const int n = a.counts[k][w];
        for (int i = 0; i < n; ++i, ++at) {
            const int64_t from = w * a.stride + i;
            const int e = s.list[k][from];
            S.key[at] = s.rec_key[k][from];
            S.base[at] = kPairs ? 2 * e : s.rec_a[k][from];
            S.start[at] = kPairs ? 2 : s.rec_b[k][from];  // the count, until the scan below
            S.vb[at] = kB ? s.rec_vb[k][from] : 0;
            S.flag[at] = (uint32_t)e;
        }
    }
    __syncthreads();
    int e[kEdgesPerThread], len[kEdgesPerThread], pins = 0;
    bool alive[kEdgesPerThread];
#pragma unroll
    for (int q = 0; q < kEdgesPerThread; ++q) {
        const int j = tid * kEdgesPerThread + q;
        alive[q] = j < E;
        e[q] = j < E ? (int)S.flag[j] : 0;
        len[q] = j < E ? S.start[j] : 0;
        pins += len[q] < kPins ? len[q] : kPins + 1;
        pins = pins < kPins ? pins : kPins + 1;
    }
    int total;
    int begin = workgroup_scan<kThreads>(pins, S.scan, &total);
    if (total > kPins) {  // left to the grid's rounds
        if (tid == 0) {
            a.report[kEndFinished] = 0;
            a.report[kEndRounds] = (unsigned long long)a.round;
        }
        return;
    }
#pragma unroll
    for (int q = 0; q < kEdgesPerThread; ++q) {
        const int j = tid * kEdgesPerThread + q;
        if (j < E) {
            S.start[j] = begin;
            S.base[j] -= begin;
            S.flag[j] = 0;
        } else {
            S.start[j] = total;
        }
        begin += len[q];
    }
    for (int i = tid; i < kSlots; i += kThreads) S.id[i] = -1;
    for (int i = tid; i < kSlots / 32; i += kThreads) S.done[i] = 0;
    if (tid < 4) S.sum[tid] = 0;
    // Rounds enqueued behind this kernel find nothing.
    for (int w = w0; w < w1; ++w) {
        a.counts[k][w] = 0;
        a.counts[k ^ 1][w] = 0;
    }
    __syncthreads();
    // This thread's pins: their edge and their vertex's slot.
    int own[kPinsPerThread], v[kPinsPerThread];
#pragma unroll
    for (int i = 0; i < kPinsPerThread; ++i) {
        const int t = i * kThreads + tid;
        own[i] = -1;
        v[i] = 0;
        if (t < total) {
            int j = 0;  // the last edge that starts at or before t (empty ones end where they start)
#pragma unroll
            for (int step = kEdges / 2; step > 0; step >>= 1)
                if (S.start[j + step] <= t) j += step;
            own[i] = j;
            v[i] = g.e_pins[S.base[j] + t] + (kB ? S.vb[j] : 0);
        }
    }
    int slot[kPinsPerThread];
#pragma unroll
    for (int i = 0; i < kPinsPerThread; ++i) {
        slot[i] = 0;
        if (own[i] >= 0) {  // at most kPins of kSlots are taken: a free one is found
            uint32_t h = __umulhi((uint32_t)v[i] * 0x9E3779B1u, (uint32_t)kSlots);
            for (;;) {
                const int id = atomicCAS(&S.id[h], -1, v[i]);
                if (id == -1 || id == v[i]) break;
                h = h + 1 < kSlots ? h + 1 : 0;
            }
            slot[i] = (int)h;
        }
    }
    __syncthreads();
    for (int i = tid; i < kSlots; i += kThreads) S.best[i] = 0;
    __syncthreads();
    constexpr uint32_t kLost = 1, kDead = 2, kWon = 4;
    uint32_t open = 0;  // this thread's pins whose edge is alive
#pragma unroll
    for (int i = 0; i < kPinsPerThread; ++i) open |= own[i] >= 0 ? 1u << i : 0;
    // Counts of the rounds, beside the report's rows (which hold the first):
    // the lists' keys are free once gathered.
    unsigned long long *packed = reinterpret_cast<unsigned long long *>(s.rec_key[k]);
    unsigned long long *weights = reinterpret_cast<unsigned long long *>(s.rec_key[k ^ 1]);
    int r = a.round, live_now = E;
    bool stopped = false;
    for (;;) {
        if (a.counting) {
            unsigned long long kap = 0;
#pragma unroll
            for (int q = 0; q < kEdgesPerThread; ++q) kap += alive[q] ? (unsigned)len[q] : 0;
            kap = wave_total(kap);
            if (lane == 0 && kap) atomicAdd(&S.sum[0], kap);
        }
#pragma unroll
        for (int i = 0; i < kPinsPerThread; ++i)
            if (open >> i & 1) atomicMax(&S.best[slot[i]], (unsigned long long)S.key[own[i]]);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kPinsPerThread; ++i)
            if ((open >> i & 1) && S.best[slot[i]] != S.key[own[i]]) atomicOr(&S.flag[own[i]], kLost);
        __syncthreads();
        unsigned long long nm = 0, wm = 0, pm = 0;
#pragma unroll
        for (int q = 0; q < kEdgesPerThread; ++q) {
            const int j = tid * kEdgesPerThread + q;
            if (alive[q]) {
                if (S.flag[j] & kLost) {
                    S.flag[j] = 0;
                } else {
                    const int bit = kB ? e[q] + g.bitoff[e[q]] : e[q];
                    atomicOr(&bits[bit >> 5], 1u << (bit & 31));
                    S.flag[j] = kWon;
                    alive[q] = false;
                    nm += 1;
                    wm += S.key[j] >> 32;
                    pm += (unsigned)len[q];
                }
            }
        }
        if (a.counting) {
            nm = wave_total(nm);
            wm = wave_total(wm);
            pm = wave_total(pm);
            if (lane == 0 && nm) {
                atomicAdd(&S.sum[1], nm);
                atomicAdd(&S.sum[2], wm);
                atomicAdd(&S.sum[3], pm);
            }
        }
        __syncthreads();
        if (a.counting && tid == 0) {
            const int i = r - a.round, row = r - a.first;
            packed[i] = (unsigned long long)live_now | S.sum[0] << 16 | S.sum[1] << 32 |
                        S.sum[3] << 48;
            weights[i] = S.sum[2];
            if (row < a.rows) {
                unsigned long long *out = a.report + kEndHeader + 5 * row;
                out[0] = (unsigned long long)live_now;
                for (int q = 0; q < 4; ++q) out[q + 1] = S.sum[q];
            }
            for (int q = 0; q < 4; ++q) S.sum[q] = 0;
        }
#pragma unroll
        for (int i = 0; i < kPinsPerThread; ++i)
            if (open >> i & 1) {
                S.best[slot[i]] = 0;
                if (S.flag[own[i]] & kWon) {
                    atomicOr(&S.done[slot[i] >> 5], 1u << (slot[i] & 31));
                    open &= ~(1u << i);
                }
            }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kPinsPerThread; ++i)
            if ((open >> i & 1) && (S.done[slot[i] >> 5] >> (slot[i] & 31) & 1))
                atomicOr(&S.flag[own[i]], kDead);
        __syncthreads();
        ++r;
#pragma unroll
        for (int i = 0; i < kPinsPerThread; ++i)
            if ((open >> i & 1) && (S.flag[own[i]] & kDead)) open &= ~(1u << i);
        static_assert(kEdgesPerThread == 2, "two counts below");
        const uint32_t kseed = a.reseed ? round_seed(a.seed, r) : 0;
#pragma unroll
        for (int q = 0; q < kEdgesPerThread; ++q) {
            const int j = tid * kEdgesPerThread + q;
            alive[q] = alive[q] && !(S.flag[j] & kDead);
            if (a.reseed && alive[q])
                S.key[j] = (S.key[j] >> 32 << 32) | priority_hash(kseed, (uint32_t)e[q]);
        }
        live_now = __syncthreads_count(alive[0]) + __syncthreads_count(alive[1]);
        if (live_now == 0) break;
        if (a.max_rounds > 0 && r >= a.max_rounds) {
            stopped = true;
            break;
        }
    }
    if (tid == 0) {
        a.report[kEndFinished] = stopped ? 0 : 1;
        a.report[kEndRounds] = (unsigned long long)r;
    }
}

template <bool kPairs, bool kB>
hipError_t launch_as(const Launch &L, const Graph &g, const State &s, const EndArgs &a,
                     uint32_t *bits) {
    static LdsGrant lds;
    const hipError_t rc = lds.ensure(&k_end<kPairs, kB>, (int)sizeof(EndShared));
    if (rc != hipSuccess) return rc;
    hipLaunchKernelGGL((k_end<kPairs, kB>), dim3(1), dim3(kThreads), sizeof(EndShared), L.stream, g,
                       s, a, bits);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_end(const Launch &L, const Graph &g, const State &s, const EndArgs &a,
                      uint32_t *bits) {
    if (g.pairs) return launch_as<true, false>(L, g, s, a, bits);
    if (g.vbase) return launch_as<false, true>(L, g, s, a, bits);
    return launch_as<false, false>(L, g, s, a, bits);
}

}  // namespace hgm
