// Wave- and workgroup-level building blocks: the sums and ids that every file
// of kernels uses, then the passes over flattened pins and the join of a wave,
// which are staged.hip's.
#pragma once

#include "internal.h"

namespace hgm {
namespace {

constexpr int kWave = 64;

// v plus the value that DPP control kCtrl reads for this lane (0 where it reads
// none or the row is masked off).
template <int kCtrl, int kRowMask>
__device__ __forceinline__ int dpp_add(int v) {
    return v + __builtin_amdgcn_update_dpp(0, v, kCtrl, kRowMask, 0xF, false);
}

// Inclusive prefix sum over a wave (row shifts by 1, 2, 4, 8, then the
// broadcasts of lanes 15 and 31 into the rows behind them).
__device__ __forceinline__ int wave_inclusive_sum(int v) {
    v = dpp_add<0x111, 0xF>(v);
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    v = dpp_add<0x118, 0xF>(v);
    v = dpp_add<0x142, 0xA>(v);
    v = dpp_add<0x143, 0xC>(v);
    return v;
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Exclusive sum over a workgroup of T threads, with two barriers; tmp: a word a
// wave.
template <int T>
__device__ __forceinline__ int workgroup_scan(int v, int *tmp, int *total) {
    const int wid = threadIdx.x / kWave, incl = wave_inclusive_sum(v);
    if (lane_id() == kWave - 1) tmp[wid] = incl;
    __syncthreads();
    int off = 0, all = 0;
    for (int i = 0; i < T / kWave; ++i) {
        off += i < wid ? tmp[i] : 0;
        all += tmp[i];
    }
    __syncthreads();
    *total = all;
    return off + incl - v;
}

// The work item (edge region or run of vertex chunks) of workgroup b among
// `grid`.  The dispatcher deals workgroups to the chip's 8 XCDs round-robin
// (b on XCD b % 8), and each XCD has its own L2: mapping each XCD's
// workgroups to one contiguous share of the items keeps neighbouring items,
// e.g. the edges and vertices of one instance of a batch, on one L2 instead
// of all eight.  A bijection of [0, grid).
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_item(int b, int grid) {
    const int x = b % kXcds, q = b / kXcds;
    const int per = grid / kXcds, rem = grid % kXcds;
    return x * per + (x < rem ? x : rem) + q;
}

// Bits of m below this lane.
__device__ __forceinline__ int bits_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Orders a wave's own LDS accesses (its lanes exchange values through LDS;
// the hardware keeps a wave's LDS accesses in order, the compiler must too).
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// A wave's scratch for its chunk of 64 edges, the edges with pins numbered
// 0, 1, ... in lane order.
constexpr int kWindow = 2048;  // pins of a chunk flattened at a time
struct WaveScratch {
    uint64_t key[kWave];
    int vb[kWave];                    // vertex base of the edge (batch)
    int rel[kWave];                   // offset of the edge's pins less its start in the chunk
    uint32_t flag[kWave];
    uint32_t bits[kWindow / 32 + 2];  // a bit where an edge's pins start (or a pin is done)
};

// The pins of the wave's 64 edges (lane: n pins from base), flattened over
// the lanes 64 at a time, so that a chunk costs its pins and not 64 times its
// longest edge, and neighbouring lanes read neighbouring pins.  Pin t of the
// chunk belongs to the edge whose start bit is the last at or before t: a
// population count of the start bits below the lane.  Returns the edge's
// number; *total <= kWindow.
__device__ __forceinline__ int flatten(WaveScratch &W, int base, int n, int *total) {
    const int lane = lane_id();
    const int incl = wave_inclusive_sum(n);
    const int start = incl - n;
    const int all = __builtin_amdgcn_readlane(incl, kWave - 1);
    const int ord = bits_below(__ballot(n > 0));
    if (lane * 32 < all) W.bits[lane] = 0;
    if (lane == 0) W.bits[(all + 31) >> 5] = 0;
    W.flag[lane] = 0;
    wave_fence();
    if (n > 0) {
        W.rel[ord] = base - start;
        atomicOr(&W.bits[start >> 5], 1u << (start & 31));
    }
    wave_fence();
    *total = all;
    return ord;
}

// Edge number of pin 64 * blk + lane; `before`: starts in earlier blocks
// (advanced past this one).
__device__ __forceinline__ int flat_edge(const WaveScratch &W, int blk, int &before) {
    const uint64_t m = (uint64_t)W.bits[2 * blk + 1] << 32 | W.bits[2 * blk];
    const int j = before + bits_below(m) + (int)(m >> lane_id() & 1) - 1;
    before += __popcll(m);
    return j;
}

// For the wave's 64 edges (lane: n pins from base): an edge is hit when
// check(pin, key, look(pin)) holds at one of its pins; key = middle(hit) is
// called once per lane; then act(pin, key, peek(pin)) at every pin of the
// edges not hit.  `every` (uniform): check is called at every pin; else an
// edge longer than a window may be left once it is hit.  defer(): whether the
// caller takes the lane's edge (asked where a chunk does not fit the
// registers).  look and peek hold the memory reads: those of all the chunk's
// pins are issued before any is used.  kBase: vb is added to the edge's pins.
// kKeep blocks of 64 pins stay in registers from the check to
// the act (0: none; their ids are read again).  All lanes of the wave call it
// (n = 0: no edge).
template <bool kPairs, bool kBase, int kKeep, class Defer, class Look, class Check, class Middle,
          class Peek, class Act>
__device__ __forceinline__ void flat_edges(WaveScratch &W, const int32_t *e_pins, int base, int n,
                                           uint64_t key, bool every, Defer defer, Look look,
                                           Check check, Middle middle, Peek peek, Act act,
                                           int vb = 0) {
    const int lane = lane_id();
    if constexpr (kPairs) {
        int2 p = make_int2(0, 0);
        if (n > 0) p = *reinterpret_cast<const int2 *>(e_pins + base);
        bool hit = false;
        if (n > 0) {
            const auto x0 = look(p.x), x1 = look(p.y);
            const bool h0 = check(p.x, key, x0), h1 = check(p.y, key, x1);
            hit = h0 || h1;
        }
        key = middle(hit);
        if (n > 0 && !hit) {
            const auto x0 = peek(p.x), x1 = peek(p.y);
            act(p.x, key, x0);
            act(p.y, key, x1);
        }
        return;
    }
    if (kKeep > 0 &&
        __builtin_amdgcn_readlane(wave_inclusive_sum(n), kWave - 1) <= kKeep * kWave) {
        int total;
        const int ord = flatten(W, base, n, &total);
        if (n > 0) {
            W.key[ord] = key;
            if constexpr (kBase) W.vb[ord] = vb;
        }
        wave_fence();
        constexpr int kBlocks = kKeep > 0 ? kKeep : 1;
        int v[kBlocks], j[kBlocks], before = 0;
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
            v[b] = j[b] = 0;
            if (b * kWave < total) {
                j[b] = flat_edge(W, b, before);
                const int t = b * kWave + lane;
                if (t < total) v[b] = e_pins[W.rel[j[b]] + t] + (kBase ? W.vb[j[b]] : 0);
            }
        }
        {
            decltype(look(0)) x[kBlocks];
#pragma unroll
            for (int b = 0; b < kBlocks; ++b)
                if (b * kWave < total) x[b] = look(v[b]);
#pragma unroll
            for (int b = 0; b < kBlocks; ++b)
                if (b * kWave < total && b * kWave + lane < total &&
                    check(v[b], W.key[j[b]], x[b]))
                    W.flag[j[b]] = 1;
        }
        wave_fence();
        const bool hit = n > 0 && W.flag[ord];
        key = middle(hit);
        if (n > 0) W.key[ord] = key;
        wave_fence();
        if (!__any(n > 0 && !hit)) return;
        decltype(peek(0)) x[kBlocks];
        uint32_t on = 0;
#pragma unroll
        for (int b = 0; b < kBlocks; ++b)
            if (b * kWave < total && b * kWave + lane < total && !W.flag[j[b]]) {
                on |= 1u << b;
                x[b] = peek(v[b]);
            }
#pragma unroll
        for (int b = 0; b < kBlocks; ++b)
            if (on >> b & 1) act(v[b], W.key[j[b]], x[b]);
        return;
    }
    if (defer()) n = 0;
    // Window after window, each taking as many pins of every unfinished edge
    // as fit.  use(pin, key, get(pin)): whether the pin hits its edge, which is
    // then finished unless every pin is asked for.
    auto windows = [&](int len, bool every, auto get, auto use) {
        bool hit = false;
        for (int at = 0;;) {
            const unsigned long long open = __ballot(at < len && (every || !hit));
            if (!open) return hit;
            const int take = kWindow / __popcll(open);
            const int left = every || !hit ? len - at : 0, now = left < take ? left : take;
            int total;
            const int ord = flatten(W, base + at, now, &total);
            if (now > 0) {
                W.key[ord] = key;
                if constexpr (kBase) W.vb[ord] = vb;
            }
            wave_fence();
            constexpr int kU = 4;  // blocks whose loads are issued together
            for (int b0 = 0, before = 0; b0 * kWave < total; b0 += kU) {
                int v[kU], j[kU];
                decltype(get(0)) x[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const int t = (b0 + u) * kWave + lane;
                    v[u] = j[u] = 0;
                    if ((b0 + u) * kWave < total) {
                        j[u] = flat_edge(W, b0 + u, before);
                        if (t < total) v[u] = e_pins[W.rel[j[u]] + t] + (kBase ? W.vb[j[u]] : 0);
                    }
                }
#pragma unroll
                for (int u = 0; u < kU; ++u)
                    if ((b0 + u) * kWave < total) x[u] = get(v[u]);
#pragma unroll
                for (int u = 0; u < kU; ++u)
                    if ((b0 + u) * kWave + lane < total && use(v[u], W.key[j[u]], x[u]))
                        W.flag[j[u]] = 1;
            }
            wave_fence();
            hit |= now > 0 && W.flag[ord];
            at += now;
            wave_fence();
        }
    };
    const bool hit = windows(n, every, look, check);
    key = middle(hit);
    windows(hit ? 0 : n, true, peek, [&](int v, uint64_t k, decltype(peek(0)) x) {
        act(v, k, x);
        return false;
    });
}

// Read of nothing, for flat_edges.
struct NoRead {
    __host__ __device__ __forceinline__ int operator()(int) const { return 0; }
};

// The live lists and the edges of one wave.  Edge ids are lo .. end; the
// list slots of the range are the same indices in the list arrays.
struct WaveLists {
    int32_t *list, *base, *len, *vb;  // vb: batch only
    uint64_t *key;
};

// One join for a wave: the survivors of its list `from` (`listed` edges) and
// the edges of its range admitted this round enter the list `to` and raise the
// maxima at their pins.  Returns how many entered.
//
// `step`: the part of the order admitted (kSteps: none), with those behind
// `before`.  In the first round
// the join writes each edge's step, the number of thresholds above its key (so
// that a lower key never has an earlier step, whatever the thresholds), and
// admits the steps up to `step`; later rounds read that byte instead of the
// weight.  The join with `sweep` looks at the first pins of every edge not
// admitted yet and drops the dead ones, so that the steps from it on hold few
// edges.
//
// Edges to look at wait in LDS (cand) until they fill a wave, and one loop
// takes them and the last round's list: flat_edges is inlined once.  (With a
// copy of it behind every place that finds edges the kernel did not fit the
// instruction cache: a round without an edge took 50 us instead of 4.)
//
// M: done_word(v), lower(v), peek(v), raise(v, key, peeked), key(e), place(e,
// base, len, vb), sort(e, w, k) / exact_sort(e, w) (weight or key that the
// thresholds are compared with), defer(e, base, len, vb, key, listed) (true: the
// edge is left to the caller), lowering (whether lower does anything).
// kFill: chunks of 64 edges looked at in one step, at most (a multiple of 4).
constexpr uint8_t kNever = 255;  // step of an edge that was dropped
constexpr int cand_size(int fill) { return (fill + 1) * kWave; }
template <bool kPairs, bool kB, int kKeep, int kSteps, int kFill, class M>
__device__ __forceinline__ int join_wave(M &m, WaveScratch &W, int *cand, const int32_t *e_pins,
                                         const WaveLists &from, const WaveLists &to, int64_t lo,
                                         int64_t end, int listed, bool first_round, bool sweep,
                                         int before, int step, uint8_t *steps,
                                         const uint64_t *thresholds) {
    const int lane = lane_id();
    int queued = 0;
    auto push = [&](int64_t e, bool on) {
        const uint64_t mask = __ballot(on);
        if (on) cand[queued + bits_below(mask)] = (int)e;
        queued += __popcll(mask);
    };
    // Each fill looks at the edges from c0 on, queues those of the round's
    // step and returns how many it looked at.
    auto fill_first = [&](int64_t c0) -> int {
        uint64_t th[kSteps - 1];
#pragma unroll
        for (int q = 0; q < kSteps - 1; ++q) th[q] = thresholds[q];
        constexpr int kU = 4;
        uint32_t w[kU];
        uint64_t k[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t at = c0 + u * kWave + lane;
            w[u] = 0;
            k[u] = 0;
            if (at < end) m.sort((int)at, w[u], k[u]);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t at = c0 + u * kWave + lane;
            int part = 0;
            bool tie = kB;  // the hash is needed only where a weight equals a threshold's
            if constexpr (!kB) {
#pragma unroll
                for (int q = 0; q < kSteps - 1; ++q) {
                    const uint32_t tw = (uint32_t)(th[q] >> 32);
                    part += w[u] < tw ? 1 : 0;
                    tie |= w[u] == tw;
                }
                if (tie) k[u] = m.exact_sort((int)at, w[u]);
            }
            if (tie) {
                part = 0;
#pragma unroll
                for (int q = 0; q < kSteps - 1; ++q) part += k[u] < th[q] ? 1 : 0;
            }
            if (at < end) steps[at] = (uint8_t)part;
            push(at, at < end && part <= step);
        }
        return kU * kWave;
    };
    // Few edges of the step: a lane looks at four per load.
    auto fill_few = [&](int64_t c0) -> int {
        constexpr int kU = kFill / 4;
        uint32_t x[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t at = c0 + 4 * (u * kWave + lane);
            x[u] = at < end ? *reinterpret_cast<const uint32_t *>(steps + at) : ~0u;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t at = c0 + 4 * (u * kWave + lane) + q;
                const int part = (int)(x[u] >> 8 * q & 255);
                push(at, at < end && part > before && part <= step);
            }
        return 4 * kU * kWave;
    };
    // Every edge not admitted yet: the first two pins, then the next four, show
    // that most of them are dead.  Their step becomes kNever.
    auto fill_rest = [&](int64_t c0) -> int {
        constexpr int kU = 4;
        int base[kU], len[kU], vb[kU], p0[kU], p1[kU], part[kU];
        bool on[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t at = c0 + u * kWave + lane;
            part[u] = at < end ? steps[at] : 0;
            on[u] = part[u] > before;
            base[u] = len[u] = vb[u] = 0;
            if (at < end) m.place((int)at, base[u], len[u], vb[u]);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            p0[u] = p1[u] = -1;
            if constexpr (kPairs) {
                if (on[u]) {
                    const int2 p = reinterpret_cast<const int2 *>(e_pins)[base[u] >> 1];
                    p0[u] = p.x;
                    p1[u] = p.y;
                }
            } else {
                if (on[u] && len[u] > 0) p0[u] = e_pins[base[u]] + vb[u];
                if (on[u] && len[u] > 1) p1[u] = e_pins[base[u] + 1] + vb[u];
            }
        }
        uint32_t d0[kU], d1[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            d0[u] = p0[u] >= 0 ? m.done_word(p0[u]) : 0;
            d1[u] = p1[u] >= 0 ? m.done_word(p1[u]) : 0;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u)
            on[u] = on[u] && !((d0[u] >> (p0[u] & 31)) & 1) && !((d1[u] >> (p1[u] & 31)) & 1);
        if constexpr (!kPairs) {
            int p[kU][4];
            uint32_t d[kU][4];
#pragma unroll
            for (int u = 0; u < kU; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    p[u][q] = -1;
                    if (on[u] && len[u] > q + 2) p[u][q] = e_pins[base[u] + q + 2] + vb[u];
                }
#pragma unroll
            for (int u = 0; u < kU; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) d[u][q] = p[u][q] >= 0 ? m.done_word(p[u][q]) : 0;
#pragma unroll
            for (int u = 0; u < kU; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q) on[u] = on[u] && !((d[u][q] >> (p[u][q] & 31)) & 1);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t at = c0 + u * kWave + lane;
            if (part[u] > step && !on[u]) steps[at] = kNever;
            push(at, on[u] && part[u] <= step);
        }
        return kU * kWave;
    };

    if (step >= kSteps) end = lo;
    const bool all = step == kSteps - 1;
    int kept = 0;  // edges entered so far (uniform)
    int64_t c0 = lo;
    for (int i0 = 0;;) {
        int e = 0, base = 0, len = 0, vb = 0;
        uint64_t key = 0;
        bool on;
        const bool listing = i0 < listed;
        if (listing) {
            if (i0 + lane < listed) {
                const int64_t at = lo + i0 + lane;
                e = from.list[at];
                if constexpr (kPairs) {
                    base = 2 * e;
                    len = 2;
                } else {
                    base = from.base[at];
                    len = from.len[at];
                    if constexpr (kB) vb = from.vb[at];
                }
                key = from.key[at];
            }
            on = len > 0;  // an empty edge was matched by its test
            i0 += kWave;
        } else {
            while (queued < kWave && c0 < end) {
                if (first_round && all) {  // every edge, before any is done
                    push(c0 + lane, c0 + lane < end);
                    c0 += kWave;
                } else {
                    c0 += first_round ? fill_first(c0) : sweep ? fill_rest(c0) : fill_few(c0);
                }
            }
            if (queued == 0) break;
            wave_fence();
            const int n = queued < kWave ? queued : kWave;
            queued -= n;
            on = lane < n;
            if (on) {
                e = cand[queued + lane];
                m.place(e, base, len, vb);
                key = m.key(e);
            }
            wave_fence();
        }
        flat_edges<kPairs, kB, kKeep>(
            W, e_pins, base, len, key, listing && m.lowering,
            [&] {
                if (!m.defer(e, base, len, vb, key, listing)) return false;
                on = false;
                return true;
            },
            [&](int v) { return m.done_word(v); },
            [&](int v, uint64_t, uint32_t word) {
                if (listing) m.lower(v);
                return (bool)((word >> (v & 31)) & 1u);
            },
            [&](bool dead) {
                const bool live = on && !dead;
                const uint64_t mask = __ballot(live);
                if (live) {
                    const int64_t at = lo + kept + bits_below(mask);
                    to.list[at] = e;
                    if constexpr (!kPairs) {
                        to.base[at] = base;
                        to.len[at] = len;
                        if constexpr (kB) to.vb[at] = vb;
                    }
                    to.key[at] = key;
                }
                kept += __popcll(mask);
                return key;
            },
            [&](int v) { return m.peek(v); },
            [&](int v, uint64_t k, auto now) { m.raise(v, k, now); }, vb);
    }
    return kept;
}

}  // namespace
}  // namespace hgm
