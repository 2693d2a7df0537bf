// Which kernel instance, split and order of tiles the backprojector (bp.hip) and its adjoint
// (bp_adjoint.hip) take for a plan, and which plans of a batch share a launch.  Host code, apart from
// the order of the tiles.
#pragma once

#include <algorithm>
#include <vector>

#include "kernels.hpp"

namespace kats {
namespace bpdev {

constexpr int kT = kBpTile;               // 16
constexpr int kNT = kT * kT;              // lanes of a tile's workgroup
constexpr unsigned kLdsBytes = 163840;    // per CU and workgroup on gfx950

// Limits of a launch: blocks along z, threads along x (the batches' grids)
constexpr long long kMostLayers = 65535, kMostThreads = (1ll << 32) - 1;

// Tile of block l (0 .. tiles - 1) of layer z of a launch whose layers (slice runs, pitches, parts)
// of tiles_x x tiles_y tiles follow one another; first: the launch's block index of the layer's
// first block.
//
// Blocks go to the eight XCDs in turn, each with an L2 of its own, so with neighbouring tiles side
// by side in the grid every XCD reads the whole filtered window of every layer.  In layers of at least
// `least` tiles (kXcdForward, kXcdAdjoint) the blocks of one XCD take a compact part instead: the tiles are numbered along bands
// of a quarter of the rows, column by column, each quarter of the numbering is cut into eight
// segments, and XCD x takes segment x + z + quarter.  Parts differ in work (corners outside the field
// of view) and an XCD cannot take work from another, hence four quarters a layer, and the turn from
// layer to layer.  512 x 512 x 128: HBM reads of the backprojection 14.2 -> 4.5 GB, whole
// reconstruction 10.46 -> 10.08 ms, whole adjoint 42.5 -> 41.8 ms; 512 x 512 x 10 (network), forward and
// adjoint 2.25 -> 1.90 ms.  Smaller layers read little, and their fewer blocks show what balance is
// lost.  Plain order / this one by tiles, ms:
//   forward   529, one layer (356^2 x 5): 0.329 / 0.336   256: 4.52 / 4.48   361 (301^2 x 77): 3.00 / 3.04   400: 4.87 / 4.83   576: 3.80 / 3.74
//             784: 4.90 / 4.75   1024 (512^2 x 32): 3.29 / 3.20
//   adjoint   256 (sparse): 18.70 / 18.95   400: 14.74 / 14.70   576: 12.88 / 12.98   784: 16.41 / 16.57
//             1024: 11.68 / 11.15
constexpr unsigned kXcdForward = 768, kXcdAdjoint = 1024;      // least tiles
struct TileAt {
    int x, y;
};
__host__ __device__ inline TileAt xcd_tile(unsigned least, int tiles_x, int tiles_y, unsigned l, unsigned z,
                                           unsigned first) {
    const unsigned tiles = (unsigned)tiles_x * (unsigned)tiles_y;
    if (tiles < least) return {(int)(l % (unsigned)tiles_x), (int)(l / (unsigned)tiles_x)};
    const unsigned chunk = (tiles / 4 + 7) / 8 * 8;
    const unsigned c = l / chunk, at = c * chunk;               // chunk: a multiple of 8, so l - at keeps l's XCD
    const unsigned n = tiles - at < chunk ? tiles - at : chunk; // tiles of this chunk
    const unsigned r = (l - at) & 7, i = (l - at) >> 3;         // the i-th block of its XCD in the chunk
    const unsigned turn = (first + z + c) & 7, seg = (r + turn) & 7;
    // blocks of remainder below n % 8 are one more: segments before seg that belong to such
    const unsigned more = (1u << (n & 7)) - 1u;
    const unsigned longer = ((more << turn) | (more >> (8 - turn))) & ((1u << seg) - 1u);
    const unsigned q = at + seg * (n >> 3) + (unsigned)__builtin_popcount(longer) + i;
    const unsigned high = ((unsigned)tiles_y + 3) / 4, band = q / (high * tiles_x), rest = q - band * high * tiles_x;
    const unsigned below = (unsigned)tiles_y - band * high, rows = below < high ? below : high;
    return {(int)(rest / rows), (int)(band * high + rest % rows)};
}

// Kernel instance of a plan: box shape (the first that its largest box fits, kFallback if none
// does) and polynomial degree.  Runs of 8 and 32 slices have the shapes of their usual boxes only.
constexpr int kShapes = 7, kShape48x80 = 3, kFallback = 7;

constexpr int kShapeRows[kShapes] = {32, 64, 64, 48, 64, 48, 48};
constexpr int kShapeCols[kShapes] = {64, 32, 64, 80, 80, 96, 128};

inline int bp_shape(const KParams &k) {
    const bool wide = k.bp_kz == 16;
    const bool has[kShapes] = {k.bp_kz <= 16, wide, k.bp_kz >= 16, wide, wide, wide, wide};
    for (int i = 0; i < kShapes; ++i)
        if (has[i] && k.bp_box_rows <= kShapeRows[i] && k.bp_box_cols <= kShapeCols[i]) return i;
    return kFallback;
}

// Split of a plan's work over workgroups.  A workgroup walks its hull view by view, which takes
// 0.5-0.9 us a view however little there is to do, and a CU holds five of them: a grid with few
// tasks is bound by that chain and leaves CUs idle.  Fewer slices per task make more tasks (each
// repeating the per-view geometry), more teams shorten the chain.  The measure is the reconstructed
// voxels in units of a whole 16 x 16 x 16 task; backprojection whole / halves / halves in 4 teams /
// quarters in 4 teams, us:
//    60 tasks (64^3, 3 pitches)          361 / 231 / 114 /  84
//   105 tasks (169^2 x 15)              1044 / 652 / 298 / 413
//   175 tasks (134^2 x 40)               737 / 495 / 404 / 581
//   302 tasks (262^2 x 18)               711 / 521 / 596 / 757
//   304 tasks (512^2 x 10, network)      601 / 485 / 773 / 870
//   512 tasks (256^2 x 32, boxes 40x79) 1247 / 1462
//   872 tasks (351^2 x 29)               883 / 911
// so wide boxes, whose staging every task repeats, are not halved.
enum { kWhole = 0, kHalves = 1, kHalvesTeams = 2, kQuartersTeams = 3, kThin = 4, kSplits = 5 };
constexpr int kSubs[kSplits] = {1, 2, 2, 4, 1}, kTeams[kSplits] = {1, 1, 4, 4, 1};

// Dynamic LDS: the teams' box buffers, and their sums at the end
inline unsigned bp_bytes(int teams, int pitch, int rows, int kz) {
    const unsigned boxes = (unsigned)teams * 2u * (unsigned)pitch * (unsigned)rows * 4u;
    const unsigned sums = (unsigned)(teams - 1) * (unsigned)kz * kNT * 4u;
    return boxes > sums ? boxes : sums;
}

struct BpClass {
    int shape, split, poly4;
    bool operator==(const BpClass &o) const { return shape == o.shape && split == o.split && poly4 == o.poly4; }
};

inline BpClass kernel_class(const KParams &k) {
    BpClass c;
    c.shape = bp_shape(k);
    c.poly4 = (k.atan_deg >= 0 && k.atan_deg <= 4) ? 1 : 0;
    c.split = kWhole;
    if (k.bp_kz != 16) return c;
    const long long full = k.n_valid / ((long long)kT * kT * 16);
    // Layers and workgroups that have slices.  A team workgroup fills a CU, so a thin volume, which has
    // many workgroups for its voxels, keeps single ones, and whole ones where halves would be empty: of 8
    // slices where no layer has more and the box is the small one.  Backprojection whole / halves /
    // halves in 4 teams / quarters in 4 teams / whole of 8 slices, us, by workgroups that have voxels:
    //   1024 (512^2 x 1)   337 / 320 / 410 / 390 / 302
    //    624 (400^2 x 1)   299 / 288 / 303 / 281 / 269      400^2 x 4  324 / 315 / 346 / 321 / 295
    //    493 (356^2 x 5)   372 / 365 / 391 / 469 / 349
    //    352 (300^2 x 10)  374 / 340 / 377 (whole reconstruction)
    //    348 (300^2 x 2)   271 / 265 / 219 / 203
    //    256 (256^2 x 4)   277 / 248 / 129 / 119            256^2 x 12 459 / 320 / 281 / 342
    const long long last = k.nz - (long long)(k.n_pitches - 1) * k.ns;
    const long long layers = (k.n_pitches - 1) * ((k.ns + 15ll) / 16) + (last + 15) / 16;
    const long long groups = k.n_valid / (kT * kT) * layers / std::max(k.nz, 1);
    const bool many = groups >= 300;
    if (full < 80 && groups < 700) c.split = kQuartersTeams;
    else if (full < 220 && !many) c.split = kHalvesTeams;
    else if (full < 450 && c.shape <= 1 && k.nz > 8 * layers) c.split = kHalves;
    // (the widest shape: 136 floats, 38 rows and more do not fit four times)
    if (kTeams[c.split] > 1 && c.shape < kFallback && bp_bytes(kTeams[c.split], kShapeCols[c.shape] + 8, k.bp_box_rows < 32 ? 32 : k.bp_box_rows, 0) + 64 > kLdsBytes)
        c.split = kHalves;
    // a split whose tasks would pass a launch's limits is left out (a whole one is as large as ever)
    const long long all = (long long)k.n_pitches * k.bp_runs * kSubs[c.split];
    if (all > kMostLayers || all * k.bp_tiles_x * k.bp_tiles_y > kMostThreads / (kNT * kTeams[c.split])) c.split = kWhole;
    if (c.split == kWhole && c.shape == 0 && std::min(k.ns, k.nz) <= 8) c.split = kThin;
    if (c.split != kWhole && c.split != kThin) c.poly4 = 0;    // one instance each: the longer polynomial's further terms are 0
    return c;
}

constexpr int kBatchRound = 1280;          // tasks of one round: five per CU

// The instance of every request of a batch: its own, but a shape with less than a round of tasks (five
// per CU) joins another one, in the first shape that takes both: alone it would end the batch with
// a launch that leaves CUs idle.  Joining costs the other class where the new shape is slower for it,
// so one that changes to another shape than S48x80 (as many workgroups per CU) joins up to two rounds
// of its tasks, and none joins on the HBM path.  Backprojection apart / joined, ms:
//    2048 tasks of 32 x 44 boxes and  512 of 28 x 79, in S48x80        3.49 / 3.00
//    4096                        and  512 of 28 x 79                   5.56 / 5.02
//   10240                        and  512 of 28 x 79                   9.82 / 9.73
//    2048 tasks of 32 x 44       and  512 of 58 x 46, in S64x64        3.88 / 3.83
//    4096                        and  512 of 58 x 46                   5.98 / 6.14
//   10240                        and  768 of 49 x 25                  10.07 / 10.56
//    2048 tasks of 32 x 44       and  512 of 53 x 79, in S64x80        3.84 / 3.80
//    4096                        and  512 of 53 x 79                   5.97 / 6.00
//   10240                        and  512 of 53 x 79                  10.21 / 11.28
//    1536 tasks of 49 x 79       and  512 of 28 x 79, in S64x80        3.88 / 3.10
//     768 tasks of 49 x 25       and  676 of 42 x 103, on the HBM path 2.64 / 3.01
// The shape does not change a result's bits; the split does, so only requests of one split and one
// team join.
inline std::vector<BpClass> batch_classes(const KParams *ks, int n) {
    std::vector<BpClass> cls(n);
    for (int i = 0; i < n; ++i) cls[i] = kernel_class(ks[i]);
    for (int split = 0; split < kSplits; ++split)
        for (int poly4 = 0; poly4 < 2 && kTeams[split] == 1; ++poly4) {
            for (int shape = 0; shape < kShapes; ++shape) {
                long long tasks[kShapes + 1] = {};
                for (int i = 0; i < n; ++i)
                    if (cls[i].split == split && cls[i].poly4 == poly4)
                        tasks[cls[i].shape] += (long long)ks[i].bp_tiles_x * ks[i].bp_tiles_y * ks[i].n_pitches * ks[i].bp_runs * kSubs[split];
                if (tasks[shape] == 0 || tasks[shape] >= kBatchRound) continue;
                // the nearest shape whose class may be joined
                for (int step = 1, joined = kFallback; step < 2 * kShapes && joined == kFallback; ++step) {
                    const int other = shape + (step & 1 ? -(step + 1) / 2 : step / 2);
                    if (other < 0 || other >= kShapes || tasks[other] == 0) continue;
                    auto in = [&](int i) { return cls[i].split == split && cls[i].poly4 == poly4 && (cls[i].shape == shape || cls[i].shape == other); };
                    KParams both = ks[0];
                    both.bp_box_rows = both.bp_box_cols = 0;
                    for (int i = 0; i < n; ++i)
                        if (in(i)) {
                            both.bp_box_rows = std::max(both.bp_box_rows, ks[i].bp_box_rows);
                            both.bp_box_cols = std::max(both.bp_box_cols, ks[i].bp_box_cols);
                        }
                    joined = bp_shape(both);
                    if (joined != other && joined != kShape48x80 && tasks[other] > 2 * kBatchRound) joined = kFallback;
                    if (joined == kFallback) continue;
                    for (int i = 0; i < n; ++i)
                        if (in(i)) cls[i].shape = joined;
                }
            }
        }
    return cls;
}

// Tasks that the views of a (tile, run) hull are split over.  A workgroup walks its hull view by
// view at 3-4 us a view, so few tasks leave CUs idle behind that chain, and a last round of long
// tasks does on larger grids; the boxes' sums meet in g^F-bar anyway.  Whole adjoint by reconstructed
// voxels in units of 16 x 16 x 16 tasks, parts 1 / 4 / 8 / 16 / 32, us:
//      4 (54^2 x 7)             1716 /  571 /  358 /  242 /  187
//     59 (64^3)                 1376 /  458 /  357 /  312 /  281
//    104 (169^2 x 15)           4224 / 1375 / 1290 / 1160 / 1102
//    304 (512^2 x 10, network)  2864 / 2302 / 2228 / 2238 / 2364
//    512 (256^2 x 32)           6023 / 5535 / 5561 / 5601 / 5756
//   1024 (256^2 x 64, sparse)   8265 / 7511 / 7328 / 7325 / 7461
//   8192 (512^2 x 128)         42916 / 42898 (42589 in 2) / 43636
inline int bpT_parts(const KParams &k) {
    const long long full = k.n_valid / ((long long)kT * kT * 16);
    const long long parts = full < 60 ? 32 : (full < 250 ? 16 : (full < 1500 ? 8 : (full < 6000 ? 4 : 2)));
    const long long most = kMostLayers / std::max(1ll, (long long)k.n_pitches * k.bp_runs);
    return (int)std::max(1ll, std::min(parts, most));
}

// Whether the rows' sums are kept in a window common to the wave (WIN) in a plan of more than 32 box
// columns.  It takes half of the LDS atomics' instructions and fewer operations, but its lanes reach one
// column's cells together where the slice-by-slice walk has turned their slices against each other, so
// it pays where boxes are wide for their rows, which keeps the lanes apart; always where an update costs
// more (fixed point: twice the conversions) and in runs of 32 slices, whose walk merges least.  Whole
// adjoint, walk / window, ms:
//     16 slices    20 x 36  1.88 / 1.53    20 x 57  1.68 / 1.31    32 x 44  11.1 / 12.3    32 x 51  11.5 / 11.9
//                  32 x 53  11.7 / 11.8    34 x 43  1.10 / 1.14    40 x 49  4.11 / 4.44    40 x 58  4.38 / 4.54
//                  40 x 62  4.46 / 4.52    40 x 67  5.49 / 5.19    40 x 79  5.58 / 5.19    53 x 66  9.91 / 9.09
//     fixed point  20 x 36  2.43 / 1.35    32 x 33  12.5 / 10.8    32 x 44  12.9 / 10.2    34 x 37  1.38 / 1.02
//                  49 x 39  9.50 / 8.31    40 x 62  5.12 / 4.18    40 x 79  6.49 / 5.34
//     32 slices    20 x 38  3.52 / 1.94    40 x 43  1.99 / 1.36    55 x 44  16.4 / 14.2    65 x 49  5.88 / 5.01
//     8 slices     20 x 47  1.74 / 1.55    22 x 49  3.57 / 4.31    18 x 51  10.8 / 11.6    20 x 57  1.31 / 1.10
// (8 slices: no line through rows and columns separates the two; errors against float64 are the same.)
inline bool bpT_window(const KParams &k, bool fixed_point) {
    if (k.bp_box_cols > 64 || fixed_point || k.bp_kz == 32) return true;
    return k.bp_kz == 8 ? k.bp_box_cols > 50 : 10 * k.bp_box_cols >= 17 * k.bp_box_rows;
}

}  // namespace bpdev
}  // namespace kats
