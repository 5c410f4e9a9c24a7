// Host build of the connection-ordering routine (spdnn_order.h), of the tile
// layout functions (spdnn_layout.h) and of other host logic (spdnn_cut.h, spdnn_profile.h), so that
// it can be tested without a GPU.  Not used by the inference path.
#include "spdnn_cut.h"
#include "spdnn_layout.h"
#include "spdnn_order.h"
#include "spdnn_profile.h"

extern "C" {

// quads: [16][32] quad (0..15) of every connection of 16 neighbouring neurons, 255 = absent.
// step_of: [16][32] out, step at which connection k of lane l is placed (255 if absent).
// nsteps: number of steps (>= the largest number of connections of any lane).
// N: columns of the row, which say whether there are steps that read a quad twice.
// Returns the cost (sum over steps of the largest quad multiplicity).
int spdnn_order_row_host(const uint8_t* quads, uint8_t* step_of, int nsteps, int N) {
    spdnn::OrderScratch S;
    uint8_t placed[16][32];
    for (int i = 0; i < 16 * 32; ++i) {
        step_of[i] = 255;
        (&placed[0][0])[i] = 255;
    }
    spdnn::order_group(
        S, nsteps, spdnn::reads_twice(N), [&](int l, int k) -> unsigned { return quads[l * 32 + k]; },
        [&](int l, int step, int k) {
            step_of[l * 32 + k] = (uint8_t)step;
            placed[l][step] = quads[l * 32 + k];
        });
    return spdnn::order_cost([&](int l, int step) -> unsigned { return placed[l][step]; });
}

// The same for rows of one stage.
int spdnn_order_group_host(const uint8_t* quads, uint8_t* step_of, int nsteps) { return spdnn_order_row_host(quads, step_of, nsteps, 1024); }

int spdnn_spread_step_host(int step, int nsteps, int half) { return spdnn::spread_step(step, nsteps, half); }

// Cost of the order as given (connection k at step k).
int spdnn_order_cost_host(const uint8_t* quads) {
    return spdnn::order_cost([&](int l, int step) -> unsigned { return quads[l * 32 + step]; });
}

// pairs: [32][32] bank pair (0..31) of every connection of 32 neighbouring neurons.
// step_of: [32][32] out, step at which connection k of lane l is placed.
// Returns the cost (sum over the 32 steps of the largest pair multiplicity), -1 if a lane got two
// connections in one step or a connection was never placed.
int spdnn_order_group32_host(const uint8_t* pairs, uint8_t* step_of) {
    static spdnn::Order32Scratch S;
    uint8_t at[32][32];  // pair used by lane l at step s
    for (int i = 0; i < 32 * 32; ++i) {
        step_of[i] = 255;
        (&at[0][0])[i] = 255;
    }
    bool bad = false;
    spdnn::order_group32(
        S, [&](int l, int k) -> unsigned { return pairs[l * 32 + k]; },
        [&](int l, int step, int k) {
            if (k < 0 || k > 31 || step_of[l * 32 + k] != 255 || at[l][step] != 255) {
                bad = true;
                return;
            }
            step_of[l * 32 + k] = (uint8_t)step;
            at[l][step] = pairs[l * 32 + k];
        });
    if (bad) return -1;
    int total = 0;
    for (int step = 0; step < 32; ++step) {
        int m[32] = {0}, mx = 0;
        for (int l = 0; l < 32; ++l) {
            if (at[l][step] == 255) return -1;
            if (++m[at[l][step]] > mx) mx = m[at[l][step]];
        }
        total += mx;
    }
    return total;
}

// Tile layout functions, one call per value.
uint32_t spdnn_tile_offset_host(uint32_t slot) { return spdnn::tile_offset(slot); }
uint32_t spdnn_tile_pair_bytes_host(uint32_t cols) { return spdnn::tile_pair_bytes(cols); }
int spdnn_lane_of_group_host(int set, int rank) { return spdnn::lane_of_group(set, rank); }
uint32_t spdnn_set_of_lane_host(uint32_t lane) { return spdnn::set_of_lane(lane); }
uint32_t spdnn_rank_in_set_host(uint32_t lane) { return spdnn::rank_in_set(lane); }
uint32_t spdnn_col_slot_host(uint32_t c) { return spdnn::col_slot(c); }
uint32_t spdnn_store_group_host(uint32_t c) { return spdnn::store_group(c); }
uint32_t spdnn_row2_pos_host(uint32_t c) { return spdnn::row2_pos(c); }
int spdnn_unit_neuron_host(int u, int p, int seg_log2, int seg_stride) { return spdnn::unit_neuron(u, p, seg_log2, seg_stride); }
void spdnn_win_union_host(int ax, int ay, int cx, int cy, int N, int* out) { spdnn::win_union(ax, ay, cx, cy, N, out[0], out[1]); }
int spdnn_win_rel_host(int c, int c_lo, int N) { return spdnn::win_rel(c, c_lo, N); }
int spdnn_win_col_host(int c_lo, int rel, int N) { return spdnn::win_col(c_lo, rel, N); }

// Workgroup cut of a general layer (spdnn_cut.h).  ptr: N + 1 row pointers; qw: 2 * (N / 4) ints, lowest and
// highest column of every four neurons; out: room for cap pairs {first neuron, number of neurons}.  Returns the
// number of workgroups, or -1 if there are more than cap.
int spdnn_cut_workgroups_host(const int32_t* ptr, const int32_t* qw, int N, int P, int nblk, int G, int32_t* out, int cap) {
    const std::vector<spdnn::NeuronRange> cut = spdnn::cut_workgroups(ptr, qw, N, P, nblk, G);
    if ((int)cut.size() > cap) return -1;
    for (size_t i = 0; i < cut.size(); ++i) {
        out[2 * i] = cut[i].first;
        out[2 * i + 1] = cut[i].count;
    }
    return (int)cut.size();
}

// Neurons by length (spdnn_cut.h).  perm: nlanes entries, nch: nlanes / 64.
void spdnn_order_by_length_host(const int32_t* ptr, int N, int nlanes, int waves, uint16_t* perm, uint32_t* nch) {
    std::vector<uint16_t> p;
    std::vector<uint32_t> c;
    spdnn::order_by_length(ptr, N, nlanes, waves, p, c);
    std::copy(p.begin(), p.end(), perm);
    std::copy(c.begin(), c.end(), nch);
}
double spdnn_uneven_chunks_host(const int32_t* ptr, int N, const uint32_t* nch, int groups, int waves) {
    return spdnn::uneven_chunks(ptr, N, std::vector<uint32_t>(nch, nch + groups), waves);
}
// runs: n triples {first layer, one past the last, a layer's own kernel?} (spdnn_profile.h).
void spdnn_take_host_counts_host(const int32_t* runs, int n, const int* host_counts, int* rows) {
    std::vector<spdnn::LayerRun> r;
    for (int i = 0; i < n; ++i) r.push_back({runs[3 * i], runs[3 * i + 1], runs[3 * i + 2] != 0});
    spdnn::take_host_counts(r.data(), r.size(), host_counts, rows);
}
uint32_t spdnn_res_code_host(uint32_t slot, int planes_log2) { return spdnn::res_code(slot, planes_log2); }
uint32_t spdnn_res_slot_host(uint32_t code, int planes_log2) { return spdnn::res_slot(code, planes_log2); }

}  // extern "C"
