// Schedule defaults: the values an hgm_opts schedule field of 0 stands for.
// Shared by the host driver (api.hip), which applies them, and the
// autotuner (tune.cpp), which starts its search from them.  Any value gives
// the same matching; these are the fastest measured on the MI355X.
#pragma once

#include <stdint.h>

namespace hgm {

constexpr int kDefaultHubThreshold = 8192;
constexpr int kBlocksPerCu = 8;
// Workgroups of the edge kernels (fixed, device independent, so that the
// workspace size does not depend on the device).  Swept on the MI355X (256
// CUs): one instance runs fastest at 1536 (power-law 1.030 -> 0.945 ms
// against 2048, hub-stress 1.287 -> 1.253, graphs 3-4% faster), a batch's
// round kernels at 4096 (18.3 -> 16.9 ms on 4,096 instances).
constexpr int kEdgeGrid = 1536;
constexpr int kEdgeGridBatch = 4096;
// The test clears the whole next maximum buffer by streaming when a round has
// at least n / kFullClearRatio live pins, else at each pin it visits.
constexpr int kFullClearRatio = 8;
constexpr int kHotDegree = 64;        // AUTO's round-0 form: degree of a hot vertex
constexpr int kFirstBatchPct = 40;    // first batch of rounds: 0.40 log2(kappa)
constexpr int kFirstBatchPctGraph = 35;
// Batches: instances with at most this many pins are matched whole by one
// workgroup each (k_solo) unless the options say otherwise: the batch's
// total pins / kSoloAutoDivisor, clamped to [kSoloAutoMin, kSoloAutoMax].
// One compute unit matches a solo instance at about 1.2e8 pins/s, the round
// kernels the whole batch at about 3e10, so this keeps the longest solo
// instance within about a quarter of the round kernels' time for the batch.
// Measured: 4,096 instances (4.8e8 pins) 16.35 -> 15.85 ms against the
// former fixed 2^20; 1,024 instances (1.2e8 pins) 8.4 -> about 5 ms.
constexpr int64_t kSoloAutoDivisor = 1024;
constexpr int64_t kSoloAutoMin = (int64_t)1 << 12;
constexpr int64_t kSoloAutoMax = (int64_t)1 << 20;
inline int64_t solo_auto_bound(int64_t kappa_total) {
    const int64_t b = kappa_total / kSoloAutoDivisor;
    return b < kSoloAutoMin ? kSoloAutoMin : b > kSoloAutoMax ? kSoloAutoMax : b;
}
// Calls that want only the matching: the solo part takes instances of a batch
// up to kSoloBatchKappa pins.
constexpr int64_t kSoloBatchKappa = (int64_t)1 << 20;
// hgm_match runs an instance of at most 1,024 edges in one workgroup up to these
// many pins.  One workgroup / the grid, us: exact rounds (a slot for every
// vertex) 199 / 409 at 1,000 edges of 131 pins, 525 / 737 at 100 of 1,310.
// Matching only: 28 / 50 for 311 edges; 8,000 pins 40 / 74; 16,000 pins of
// 1,000 edges 82 / 131 and of 100 edges 141 / 119; 32,000 159 / 144; 131,000
// 187 / 140.  Beyond the vertices that have a slot each, 8,192 pins, all that
// the registers hold: 50 / 77 with 50,000 vertices, but 141 / 127 at 16,000
// pins and 3,900 / 123 at 65,000 with 500,000 vertices, whose done bits leave
// fewer slots: there 45 / 68 at 4,000 pins, 161 / 73 at 8,100.
constexpr int64_t kSoloOneExact = (int64_t)1 << 17, kSoloOneKappa = (int64_t)1 << 14;
constexpr int64_t kSoloOneShared = 8192, kSoloOneSharedMany = 4096;
constexpr int kSoloOneManyVerts = 1 << 18;
// An edge-centric round 0 of one instance samples the pins for hubs from this
// many pins, in the setup kernel (Zipf popularity: a call of 4.1 M pins 470 ->
// 380 us; a hub in a quarter of the edges, 4.8 M: 600 -> 480; none, 1.1 M: 3 us
// of 245 for nothing).
constexpr int64_t kHubSampleKappa = (int64_t)1 << 20;
// Rounds over all edges: the last ones run in one workgroup (ending.hip, up to
// 2,048 edges and 8,192 pins) after as many rounds as leave about this many
// live pins (or edges, where those run out first) at the usual shrink per
// round.  A batch that ends a round early costs a second check (about 20 us)
// and one a round late two near-empty launches (about 13 us).
constexpr double kEndingPins = 5000.0;
constexpr double kEndingEdges = 1400.0;
// Rounds by admission: workgroups of the join and the test.  A wave's work
// between two waits grows with its range, and the chip is full with 8 waves a
// compute unit (1024 against 512: 600,000 edges 222 / 208 us, hub-stress, 4M, 470
// / 455, power-law, 5M, and RGG, 6.9M, within 5%); from about 8M edges
// on 16 waves hide more (10M 1,215 / 1,240, 20M 1,750 / 1,805).  At 256 or 1536
// all take longer.
constexpr int kStagedGrid = 512, kStagedGridLarge = 1024;
constexpr int64_t kStagedLargeEdges = (int64_t)1 << 23;
// Rounds by admission, where the mean edge is longer than 8 pins: a wave's range
// shrinks to the pins that it keeps in registers (edges of 258 pins, 2,000 of
// them: 1,023 us with 64 edges a wave, 354 with 4,096 pins, 255 with 512; the
// rounds over all edges 1,115).
constexpr int64_t kStagedWavePins = 512;
// Rounds by admission sample how many others an edge meets (staged.hip) where
// edges are short and the means (pins a vertex times pins an edge) leave room
// for few: kSparseOthersSmall up to kSparseSmall pins, where the sample costs
// what it gains (20,000 edges of 2 pins meeting 8: 106 / 116, 4: 154 / 107),
// kSparseOthers up to kSparseMiddle (500,000 edges meeting 12: 237 / 187),
// kSparseOthersLarge beyond.  Below kSparseSize pins (or edges) every choice is
// a chain of launches.
constexpr int64_t kSparseMean = 8, kSparseSize = 1 << 14, kSparseSmall = 1 << 18,
                  kSparseMiddle = 1 << 21;
constexpr double kSparseOthersSmall = 6.0, kSparseOthers = 14.0, kSparseOthersLarge = 5.0;
// Beyond kSparseAsk pins (or edges) the host waits for the sample (30 us) where
// the means are below the same bounds, and
// runs the rounds over all live edges up to kFewOthers, kFewOthersEdge where
// round 0 has no vertex form, kFewOthersLarge beyond kSparseMiddle pins (none
// without the vertex form).  Admission / over all, us, by others met, wait not
// counted:
//   graphs, 1M pins     1: 306 / 195  2: 291 / 187  4: 256 / 180  6: 248 / 195
//           4M          1: 549 / 411  2: 476 / 368  4: 406 / 361
//           16M         1: 2158 / 1593  2: 1682 / 1307  4: 1252 / 1192
//   edges of 4, 2M      2: 374 / 264  4: 332 / 249  8: 275 / 267
//   no vertex form, 1M  2: 291 / 205  4: 256 / 210; 4M 1: 549 / 476  2: 476 / 434
// and with more than 4 vertices a pin, from kSparseVerts on, the vertex form's
// pass over them costs more (2M pins, 33M vertices 582 / 692).
constexpr int64_t kSparseAsk = 1 << 19, kSparseVerts = 1 << 22;
constexpr double kFewOthers = 6.0, kFewOthersEdge = 4.0, kFewOthersLarge = 4.5;
// Rounds by admission: round 0 starts with the first step expected to admit
// at least this many edges (fewer leave the grid idle for a whole round).
constexpr int64_t kStagedFirstEdges = 1024;
// The last rounds' workgroup follows in the round of the last admission for
// instances of at most this many edges (up to 2^19 edges: one round later, and
// so on).
constexpr int64_t kStagedTailEdges = (int64_t)1 << 15;
// One instance: the tail workgroup (k_tail, state in global memory) takes over
// a round with at most this many live pins (and at most 65536 live edges).  Off
// unless asked for: a round there costs as much as a round of the grid-wide
// kernels (both are a chain of dependent memory accesses).
constexpr int kDefaultTailPins = -1;

}  // namespace hgm
