// Device helpers and the launch arguments shared by the backprojector (bp.hip) and its
// adjoint (bp_adjoint.hip): both walk the same 16 x 16 voxel tiles, slice runs, PI-window
// hulls and footprint boxes of the plan.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>

#include "kernels.hpp"

namespace kats {
namespace bpdev {

__device__ inline int wave_min(int v) {
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ inline int wave_max(int v) {
    for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
    return v;
}

__device__ inline float med3(float x, float lo, float hi) { return __builtin_amdgcn_fmed3f(x, lo, hi); }

// Pointers read from memory (the packed launch's request descriptors) carry no address
// space, so loads through them would be flat (slower, and ordered with LDS traffic);
// every table / g^F / volume access goes through a global-address-space pointer instead.
template <class T>
__device__ inline __attribute__((address_space(1))) T *glb(T *ptr) {
    return (__attribute__((address_space(1))) T *)ptr;
}
// Load of a 4-, 8- or 16-byte value through a global-address-space pointer.
template <class T>
__device__ inline T ldg(const T *ptr) {
    static_assert(sizeof(T) % 4 == 0 && sizeof(T) <= 16, "whole dwords");
    typedef unsigned int W __attribute__((ext_vector_type(sizeof(T) / 4)));
    const W w = *(const __attribute__((address_space(1))) W *)ptr;
    T out;
    __builtin_memcpy(&out, &w, sizeof(T));
    return out;
}

constexpr int kT = kBpTile;       // 16
constexpr int kNT = kT * kT;      // 256 lanes
constexpr int kKG = 4;            // slices per branch group

// The scalars the backprojector needs (a slim kernel argument keeps SGPR pressure low).
struct BpArgs {
    const float4 *view;
    const PiEntry *pi;
    const BpBox *boxes;
    long long n_views, first_view;
    float R, inv_dalpha, col_c, q_scale, row_c, dz, x_first, y_first, dx, dy, scale;
    int nx, ny, nz, ns, Nv, n_lo, W, runs, tiles_x, tiles_y, gf_rows, gf_cols;
    int atan_deg;
    float atan_coef[9];
};

inline BpArgs bp_args(const KParams &k) {
    BpArgs a;
    a.view = k.view;
    a.pi = k.pi;
    a.boxes = k.boxes;
    a.n_views = k.n_views;
    a.first_view = k.first_view;
    a.R = k.R;
    a.inv_dalpha = k.inv_dalpha;
    a.col_c = k.col_c;
    a.q_scale = k.D * k.inv_dw;
    a.row_c = k.row_c;
    a.dz = k.dz;
    a.x_first = k.x_first;
    a.y_first = k.y_first;
    a.dx = k.dx;
    a.dy = k.dy;
    a.scale = k.scale;
    a.nx = k.nx;
    a.ny = k.ny;
    a.nz = k.nz;
    a.ns = k.ns;
    a.Nv = k.Nv;
    a.n_lo = k.n_lo;
    a.W = k.W;
    a.runs = k.bp_runs;
    a.tiles_x = k.bp_tiles_x;
    a.tiles_y = k.bp_tiles_y;
    a.gf_rows = k.gf_rows;
    a.gf_cols = k.gf_cols;
    a.atan_deg = k.atan_deg;
    for (int i = 0; i < 9; ++i) a.atan_coef[i] = k.atan_coef[i];
    return a;
}

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
//   forward   529, one layer (356^2 x 5): 0.340 / 0.354   256: 4.52 / 4.48   361 (301^2 x 77): 3.00 / 3.04   400: 4.87 / 4.83   576: 3.80 / 3.74
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

// A footprint box as stored by the plan: two dwords {r0 | nr << 16, c0 | nc << 16}.
__device__ inline BpBox unpack_box(uint2 w) {
    BpBox b;
    b.r0 = (int16_t)(w.x & 0xffffu);
    b.nr = (int16_t)(w.x >> 16);
    b.c0 = (int16_t)(w.y & 0xffffu);
    b.nc = (int16_t)(w.y >> 16);
    return b;
}

}  // namespace bpdev
}  // namespace kats
