// LDS tile layout of the fused kernels: where a column of a feature-row tile sits in
// LDS and which lanes of a wave are served together.  Plain C++ usable on the host
// and in device code (the host build exists for tests of the set-up logic).
#pragma once
#include <stdint.h>

#include "spdnn_order.h"

namespace spdnn {

// Byte offset inside the LDS tile pair of stage-local column c, buffer 0.  The two
// buffers interleave in chunks of 16 columns (256 bytes = one row of the 64 LDS
// banks), so that a column's 16-byte entry sits in bank quad (c mod 16) in either
// buffer and the second buffer is reached with a constant +256, which fits the
// read instruction's immediate offset.
constexpr int kBufSkew = 256;
SPDNN_HD inline uint32_t tile_offset(uint32_t c) {
    return ((c >> 4) << 9) | ((c & 15u) << 4);
}
// LDS bytes of a tile pair holding `cols` columns.
SPDNN_HD inline uint32_t tile_pair_bytes(uint32_t cols) { return ((cols + 15u) >> 4) << 9; }

// Lanes of a wave that a 16-byte LDS access serves in the same clock (measured on
// gfx950 with a pairwise-conflict probe): the wave's 16 quartets of 4 lanes split
// into four sets, quartets {0,3,5,6}, {1,2,4,7} and the same two shifted by 8.
// lane_of_group(s, i) = i-th lane (0..15) of set s (0..3) within the wave.
SPDNN_HD inline int lane_of_group(int s, int i) {
    const int tbl[2][4] = {{0, 3, 5, 6}, {1, 2, 4, 7}};
    return (tbl[s & 1][i >> 2] + 8 * (s >> 1)) * 4 + (i & 3);
}

// Slot (16-byte entry) of stage-local column c inside the LDS tile.  Staging gives
// lane t of the workgroup columns 4t..4t+3 and writes them with four 16-byte
// stores; for those stores to be conflict-free the 16 lanes of a set must hit 16
// different bank quads (slot mod 16) in each store.  Within every span of 128
// columns (32 lanes) the slot is therefore
//     set-in-half | column-in-lane | quartet's rank in its set | lane-in-quartet,
// a permutation of the span; nothing outside the tile code depends on it.
SPDNN_HD inline uint32_t col_slot(uint32_t c) {
    const uint32_t a = c & 3u, m = (c >> 2) & 3u, q8 = (c >> 4) & 7u, hi = c >> 7;
    const uint32_t gr = (0x73261540u >> (4u * q8)) & 7u;  // quartet -> set*4 + rank
    return (hi << 7) | ((gr >> 2) << 6) | (a << 4) | ((gr & 3u) << 2) | m;
}

// Set (0..3) and rank inside the set (0..15) of lane l of a wave: the inverse of
// lane_of_group.
SPDNN_HD inline uint32_t set_of_lane(uint32_t l) {
    const uint32_t gr = (0x73261540u >> (4u * ((l >> 2) & 7u))) & 7u;  // quartet -> set parity * 4 + rank of quartet
    return ((l >> 5) << 1) | (gr >> 2);
}
SPDNN_HD inline uint32_t rank_in_set(uint32_t l) {
    const uint32_t gr = (0x73261540u >> (4u * ((l >> 2) & 7u))) & 7u;
    return ((gr & 3u) << 2) | (l & 3u);
}
// Balanced layout of a single-stage tile (balance_kernel).  Staging lane t writes its
// columns 4t+a, a = 0..3, with four 16-byte stores; the 16 lanes of a set form, per a,
// a "store group" of 16 columns that must land in 16 different bank quads.  Store group
// g = (wave * 4 + set) * 4 + a owns the 256-byte row g of the tile; inside the row the
// 16 columns may take the 16 quads in any order, and that order is what gets chosen.
SPDNN_HD inline uint32_t store_group(uint32_t c) {  // of stage-local column c
    const uint32_t t = c >> 2;
    return (((t >> 6) << 2) | set_of_lane(t & 63u)) << 2 | (c & 3u);
}

// Networks of at most 4096 neurons keep their rows in LDS from layer to layer (resident_kernel): a pass holds up to
// `planes` tiles of 4 rows, interleaved in chunks of 16 columns like the tile pair above, and a connection's slot is
// kept as its entry code -- the LDS byte address of plane 0's entry, divided by 16 -- so that one shift makes it an
// address.  Four planes of up to 2048 columns or two of up to 4096: 13 bits.
SPDNN_HD inline int res_planes_log2(int nblk) { return nblk <= 2 ? 2 : 1; }
SPDNN_HD inline uint32_t res_code(uint32_t slot, int planes_log2) { return ((slot >> 4) << (4 + planes_log2)) | (slot & 15u); }
SPDNN_HD inline uint32_t res_slot(uint32_t code, int planes_log2) { return ((code >> (4 + planes_log2)) << 4) | (code & 15u); }

// Column windows are cyclic: the window {c_lo, ncols} of a block of output neurons covers the columns
// (c_lo + i) mod N, i < ncols (c_lo, ncols and N multiples of 4).  The strided, modular patterns that the
// challenge networks are built from wrap around the row end; their footprint is narrow only on the circle.
SPDNN_HD inline int win_rel(int c, int c_lo, int N) {  // position of column c inside the window starting at c_lo
    const int r = c - c_lo;
    return r < 0 ? r + N : r;
}
SPDNN_HD inline int win_col(int c_lo, int rel, int N) {  // column at position rel (< N) of that window
    const int c = c_lo + rel;
    return c >= N ? c - N : c;
}
// Smallest cyclic window holding the windows {ax, ay} and {cx, cy} (a length of 0 = empty).
SPDNN_HD inline void win_union(int ax, int ay, int cx, int cy, int N, int& ox, int& oy) {
    if (cy == 0) {
        ox = ax;
        oy = ay;
        return;
    }
    if (ay == 0) {
        ox = cx;
        oy = cy;
        return;
    }
    const int d = win_rel(cx, ax, N);       // c starts d columns after a ...
    const int e = d == 0 ? 0 : N - d;       // ... which is the same as a starting e columns after c
    const int span_a = ay > d + cy ? ay : d + cy;
    const int span_c = cy > e + ay ? cy : e + ay;
    if (span_a <= span_c) {
        ox = ax;
        oy = span_a;
    } else {
        ox = cx;
        oy = span_c;
    }
    if (oy >= N) {
        ox = 0;
        oy = N;
    }
}

// Tile of the two-rows-per-entry kernel (fused_row2_kernel): an entry is 8 bytes, the two rows'
// values of one column, at byte 8 * row2_pos(c) for stage-local column c.  Staging lane t owns columns
// 4t..4t+3 and writes them with 8-byte stores, one per column; a ds_write_b64 / ds_read_b64 is served
// half a wave (32 lanes) at a time from 32 pairs of banks, so within every span of 128 columns
// (32 lanes) the entries are transposed: column-in-lane | lane-in-half-wave.  An entry's bank pair is
// row2_pos(c) mod 32 = (c >> 2) mod 32.
SPDNN_HD inline uint32_t row2_pos(uint32_t c) { return (c & ~127u) | ((c & 3u) << 5) | ((c >> 2) & 31u); }

// Which output neurons a 4096-neuron unit of fused_row2_kernel owns.  A unit is 4096 >> seg_log2 segments of
// (1 << seg_log2) neighbouring neurons, one segment every seg_stride neurons: unit u takes the neurons
// k * seg_stride + (u << seg_log2) + i, i < (1 << seg_log2), k < (4096 >> seg_log2), and local index
// p = (k << seg_log2) + i counts them in ascending order.  seg_log2 = 12 is the plain unit of 4096 neighbours;
// with smaller segments the units interleave, so that the neurons of a strided pattern which read the same
// few columns (j, j + stride, j + 2 stride, ... all read j + k stride) land in one unit.  Needs
// seg_stride << (12 - seg_log2) == N; segments are at least 64 neurons, so a wave's outputs stay contiguous.
constexpr int kSegLog2Min = 6, kSegLog2Max = 12;
SPDNN_HD inline int unit_neuron(int u, int p, int seg_log2, int seg_stride) {
    return (p >> seg_log2) * seg_stride + (u << seg_log2) + (p & ((1 << seg_log2) - 1));
}

}  // namespace spdnn
