// Launch geometry that integers alone decide, for the launchers and kernels and for checks on the host.
#pragma once
#include <stddef.h>
#include <stdint.h>

#define SNN_LDS_PER_CU (160 * 1024)

// ---- sequential forward part of masked layers, by column (k_layer_seq_col) ------------------------
// Wavefronts per slice of 64 neurons (eight batch elements each), the places of the spikes that a launch of `steps` steps
// exchanges, a cache line per step, slice and wavefront (bytes), and the LDS of a workgroup.
#define SNN_COL_LINE 128 // bytes of a cache line
#define SNN_COL_GROUP 8  // entries per group of loads; columns are padded to whole groups
#define SNN_COL_LDS_MAX ((size_t)34816) // of the stage launch (k_fwd_stage_col), whose currents want as much
constexpr int seq_col_waves_of(int B) { return B <= 8 ? 1 : B <= 16 ? 2 : 4; }
constexpr size_t seq_col_places(int N, int B, int steps) { return (size_t)steps * ((N + 63) / 64) * seq_col_waves_of(B) * SNN_COL_LINE; }
constexpr size_t seq_col_lds(int N) { return (size_t)4 * (64 * ((N + 63) / 64) + 64); }
// Whether a masked matrix of N x N is also kept by column: 32 MB dense-stored and more, where the kernel can run, ...
inline bool csr_by_column(int N, int B) {
  return (size_t)N * N * sizeof(float) >= ((size_t)32 << 20) && B <= 32 && seq_col_lds(N) <= SNN_COL_LDS_MAX;
}
// ... and with `groups` groups of 64 columns in all: no more than two of five synapses exist (beyond, the walk over the dense-stored matrix is
// ahead but for a few percent) and padding takes no more than the entries do.
inline bool csr_column_form(int N, size_t nnz, size_t groups) {
  return nnz * 5 <= (size_t)N * N * 2 && groups * SNN_COL_GROUP * 64 <= 2 * nnz + (size_t)((N + 63) / 64) * SNN_COL_GROUP * 64;
}
// The layers of a launch: synapses, entries of the fullest slice of 64 columns (whole groups), activity (< 0: not known).
struct MaskedLayer { int N; size_t nnz; int longest; double rate; };
// Is the walk by column the faster one for a launch over these layers?  Estimates of a step, in us.  By column every wavefront passes
// its slice's entries whatever the activity, and all wait for the fullest slice.  By row (`rows`, or else the walk over the dense-stored
// matrix, whichever would run) a workgroup passes the active presynaptic neurons, over compressed rows one entry per lane and sub-range of 512 columns
// at a time -- a row with more entries there costs much more --, over the dense-stored matrix bound by its bytes, of all layers and
// batch elements, where it is larger than the caches (13 TB/s, 27 where the batch elements share its rows), or by its rows one after the other.
// Forward passes over 64 steps, ms by column / rows /
// dense-stored:
//   8192, batch 32       density 0.05  4 %  2.7 / 2.3 / 2.6    19 %  2.9 / 6.8 / 9.2     0.1  8 %  4.5 / 4.6 / 4.9    18 %  4.7 / 8.8 / 9.1
//                        0.3           8 % 11.7 /  31 / 4.8    38 % 11.9 / 103 / 8.1     0.9  4 %  32 / 65 / 2.6
//   4 x 8192, batch 32   0.1           4 %   17 / 12 / 18      19 %   17 / 31 / 43       0.3 19 %  35 / 176 / 44       0.5 34 %  52 / 455 / 49
//   2 x 8192, batch 8    0.1           4 %  6.8 / 4.4 / 5.1    11 %  6.9 / 9.7 / 8.5     0.3 11 %  18 / 73 / 8.4
//   3 x 4096, batch 32   0.1           4 %  8.3 / 5.8 / 2.6    15 %  8.4 / 13 / 4.3      0.3 15 %  19 / 74 / 4.3
//   3 x 4096, batch 32, density 0.1 and one neuron with every synapse  15 %  53 / 13 / 4.3
// An activity that is not known: the walk by row.
inline bool seq_by_column(const MaskedLayer *layers, int n, int B, bool rows) {
  double col = 0.0, row = 0.0, dense = 0.0, rows_of_one = 0.0;
  for (int i = 0; i < n; ++i) {
    const MaskedLayer &l = layers[i];
    if (l.rate < 0.0 || l.longest <= 0) return false;
    const double active = l.rate * l.N, e = 512.0 * (double)l.nnz / ((double)l.N * l.N); // a row's entries in a sub-range
    const double per_row = e <= 40.0 ? 0.06 : e <= 60.0 ? 0.06 + 0.002 * (e - 40.0) : 0.0054 * e - 0.15;
    const double c = 0.065 * l.longest, r = 3.0 + active * (per_row < 0.06 ? 0.06 : per_row);
    col = c > col ? c : col;
    row = r > row ? r : row;
    const double bytes = (double)l.N * sizeof(float), rate = l.rate < 0.2 ? 0.0 : l.rate - 0.2;
    const double tb_s = bytes * l.N < 2e8 ? 100.0 : rate > 0.18 ? 27.0 : 13.0 + 75.0 * rate;
    const double chain = active * (l.N > 4096 ? 0.04 : 0.015);
    dense += active * bytes * B / (1e6 * tb_s);
    rows_of_one = chain > rows_of_one ? chain : rows_of_one;
  }
  if (dense < rows_of_one) dense = rows_of_one;
  return n > 0 && 11.0 + col < 0.95 * (rows ? 11.0 + row : 8.0 + dense);
}

// ---- inter-layer products of the adjoint pass -----------------------------------------------------
// N neurons below, K above: split into three bf16 parts (k_up_split) or on the fp32 matrix cores.  The same kernel for every number of
// rows: they differ in the last bits, and gradients must not depend on how the time axis is cut.  From 1024 neurons the split one is
// not slower by more than a percent (training steps of 96 steps, two layers, fp32 / split: 1024 neurons, batch 4 / 16 / 64 1.89 / 2.00 / 2.49 and
// 1.89 / 2.00 / 2.43 ms; 1500-1100, batch 8 / 24 2.41 / 2.69 and 2.42 / 2.64; 2048, batch 64 5.54 and 5.27; 4096, batch 4, 48 steps
// 4.76 and 4.82); with two fp16 parts, half the products, 512 and 700 neurons gained nothing below batch 64.
inline bool split_product(int N, int K) { return N >= 1024 && K >= 1024; }
#define UPS_SLAB_BYTES 96 // 16 elements of a row of a split matrix: the high, the middle and the low parts
constexpr size_t split_row_bytes(int K) { return (size_t)(K + 31) / 32 * (2 * UPS_SLAB_BYTES); } // whole blocks of 32 elements

// ---- weight gradients of large matrices -----------------------------------------------------------
// Tiles of 256 x 64 of a network's matrices (k_dw_split), and where that kernel takes its weight gradients: by the shapes and the batch
// alone, as it differs from the others in the last bits.  Training steps of 96 steps in chunks of 32, us with the better of k_dw_tile and
// k_dw_mfma / with k_dw_split, at 3 % and 45 % activity:
//   3 x 512 (90 tiles)    batch 16 1427 / 1459, 1890 / 1910    32 1606 / 1588, 2046 / 2027
//   2 x 700 (124)         batch 16 1672 / 1699, 2311 / 2333    32 1800 / 1783, 2455 / 2444
//   3 x 640 (173)         batch  8 1830 / 1873, 2473 / 2509    12 1918 / 1903, 2571 / 2548    32 2163 / 2058, 2811 / 2704
//   3 x 1024 (372)        batch  8 2070 / 2092, 3257 / 3202    12 2234 / 2200, 3456 / 3306    32 2577 / 2471, 4019 / 3666
//   2048 (328)            batch  8 1498 / 1539, 2737 / 2659    12 1566 / 1577, 2882 / 2735    32 1727 / 1712, 3437 / 3079
inline int dw_split_tiles(int n_pre, int n_post) { return ((n_pre + 255) / 256) * ((n_post + 63) / 64); }
// octets of batch elements per step: two, or whole parts of four
constexpr int dw_split_octets(int B) { return B <= 16 ? 2 : (B + 31) / 32 * 4; }
#define SNN_DW_STEPS_LEAST 16 // steps of its workspace that a context has whatever the budget (see snn_bptt)
inline bool dw_split_pays(int tiles, int B) { return tiles >= 150 && B >= 12 && B <= 64; }
// Of a masked recurrent matrix of such a network: the dense gradients here rather than the existing synapses' by k_dw_csr, which has few
// workgroups (256 rows x 512 columns, a compute unit each) where a layer is not wide.  Training steps of 96 steps (64 from 4096
// neurons, 32 of 8192) in chunks of 32, density 0.1, us by synapse / dense, batch 16, activity about 0, 4 and 15 to 30 %:
//   3 x 1536 3126 / 2826, 3606 / 3066, 4262 / 3873    2 x 2048 2640 / 2473, 2976 / 2666, 3535 / 3212    4 x 2048 4471 / 4290, 5330 / 4845, 7155 / 6575
//   2 x 3000 5508 / 5483, 6861 / 6765, 8895 / 8570    2 x 4096 4737 / 4826, 6347 / 6335, 8577 / 8441    8192 2337 / 2754, 2922 / 3269, 4091 / 4399
// (the same at batch 12 and 32 and at density 0.05: 2 x 3000 4934 / 4934, 6006 / 5892, 6545 / 6242).
inline bool dw_split_masked(int N) { return N <= 3072; }

// ---- sequential forward part of layers of 257..1024 neurons (k_layer_seq_lds) --------------------
// Columns per slice, wavefronts per workgroup, groups of batch elements per job, slices per unit, units (job, group); entries of a
// list of active neurons; dynamic LDS of a workgroup.
struct SeqLdsPlan { int lpb, waves, groups, slices, units, lcap; size_t lds; };
// What of a compute unit's LDS the launch may ask for: the kernel's static part has the rest.
constexpr size_t SEQ_LDS_DYNAMIC = SNN_LDS_PER_CU - 64;
// The plan for `jobs` layers of at most N neurons and a batch of B where `slots` workgroups fit a die; as few wavefronts per
// workgroup as let all units be resident.  posts: entries for the numbers of the dies.  false: no such plan.
inline bool seq_lds_geometry(int N, int B, int jobs, int slots, int posts, SeqLdsPlan *p) {
  p->lpb = N <= 512 ? 64 : 32;
  p->slices = (N + p->lpb - 1) / p->lpb;
  if (p->slices > slots) return false;
  const int per_wave = 64 / p->lpb, units_max = slots / p->slices * 8;
  for (p->waves = 4; p->waves <= 16; p->waves *= 2) {
    p->groups = (B + p->waves * per_wave - 1) / (p->waves * per_wave);
    p->units = jobs * p->groups;
    if (p->units > units_max || p->units * p->slices > posts) continue;
    const size_t weights = (size_t)(N + 1) * p->lpb * sizeof(float), lists = (size_t)p->waves * per_wave * sizeof(uint16_t);
    const size_t room = (SEQ_LDS_DYNAMIC - weights) / lists;
    p->lcap = (int)((size_t)N + 56 < room ? (size_t)N + 56 : room) & ~7;
    if (p->lcap < 256 + 48) continue; // a quarter of the widest layer, whole groups, the reads ahead, the spare entry
    p->lds = weights + lists * p->lcap;
    return true;
  }
  return false;
}

// ---- register-stationary chain (layers of up to 256 neurons) --------------------------------------
// Byte offsets of weight [q][i] of an N x N matrix for a buffer load: per lane, and per row in the scalar one, which the
// compiler's contract leaves out of the bounds check.  Columns past the layer's width are outside the buffer by their lane's
// offset and read 0; rows past it are the last row again, their spikes are 0.  (The instance for NW has N > NW - 32.)
constexpr uint32_t BUFFER_OUTSIDE = 0x80000000u;
constexpr uint32_t seq_rs_lane_offset(int N, int i) { return i < N ? (uint32_t)i * 4u : BUFFER_OUTSIDE; }
constexpr uint32_t seq_rs_row_offset(int N, int NW, int q) { return (uint32_t)((q <= NW - 32 || q < N ? q : N - 1) * N) * 4u; }

// ---- currents by lists of active neurons or on the matrix cores (k_currents_lists, k_currents_mfma) ------------------
// lanes per row of k_currents_lists (four columns each): the widest slice of columns that fits the LDS for P presynaptic neurons
constexpr size_t list_lds(int P, int lpt) { return (size_t)(P + 1) * 4 * lpt * sizeof(float); }
constexpr int list_lanes(int P) {
  for (int lpt = 16; lpt >= 1; lpt /= 2)
    if (list_lds(P, lpt) + 512 <= SNN_LDS_PER_CU) return lpt;
  return 0;
}
// One matrix of a launch: presynaptic neurons, columns, (t, b) rows, activity of the presynaptic layer.
struct ListsCost { int P, N; long long rows; double rate; };
// Estimated times of a launch over these matrices, in us.  Matrix cores: every presynaptic neuron that is active in any of 16 rows
// takes part for all of them (29 ns per neuron, 16 rows and 64 columns on each of 1024 SIMDs), a workgroup's chain of them is
// the least.  Lists: a workgroup per compute unit passes over its rows, 61 ns per active neuron and full pass (the LDS rate; 2 and
// 2.6 times that for slices of eight and four columns, whose rows meet the same banks) and 3.5 us to begin with.
inline void currents_mfma_us(const ListsCost *m, int n, int slices, double *work, double *chain) {
  for (int i = 0; i < n; ++i) {
    double silent = 1.0 - m[i].rate; // no spike in 16 rows
    for (int k = 0; k < 4; ++k) silent *= silent;
    const double some = 1.0 - silent, c = m[i].P * (0.36 + 0.64 * some) * 0.032;
    *work += (double)m[i].rows * slices * m[i].N * m[i].P * (1.0 + 1.8 * some) * 1e-8;
    *chain = c > *chain ? c : *chain;
  }
}
inline double currents_lists_walk_us(const ListsCost *m, int n) { // one launch per width of slice
  double us = 0.0;
  for (int lpt = 16; lpt >= 1; lpt /= 2) {
    const long long per_pass = 16 * 64 / lpt;
    long long units = 0, groups = 0;
    for (int i = 0; i < n; ++i)
      if (list_lanes(m[i].P) == lpt) units += (m[i].N + 4 * lpt - 1) / (4 * lpt);
    if (!units) continue;
    double longest = 0.0;
    for (int i = 0; i < n; ++i)
      if (list_lanes(m[i].P) == lpt) {
        const long long passes = (m[i].rows + per_pass - 1) / per_pass, most = 256 / units;
        const long long splits = most < 1 ? 1 : passes < most ? passes : most;
        groups += (m[i].N + 4 * lpt - 1) / (4 * lpt) * splits;
        const double lds = lpt == 1 ? 2.6 : lpt == 2 ? 2.0 : 1.0, full = (double)m[i].rows / (double)(passes * per_pass);
        const double t = (double)((passes + splits - 1) / splits) * (0.061 * m[i].P * m[i].rate * lds * full + 3.5);
        longest = t > longest ? t : longest;
      }
    us += 5.0 + longest * (double)((groups + 255) / 256);
  }
  return us;
}
// Are lists the faster way for a launch over `in` (the feed-forward parts) and `rec` (the recurrent parts of a recompute), `slices`
// times those rows?  They have to be a tenth better: over 152 measured launches (one and two layers of 300..2800 neurons, batch
// 16 to 64, 4..48 % activity) the choice then costs at most 4 % against the better of the two.  One bound on the activity cannot do that:
// the two meet at 38 % for 2048 neurons, 20 % for 1500, 8 % for 2800, and below 4 % where a launch is too small to pay for its
// lists (512 neurons at batch 16: 27 us against 54).
inline bool currents_by_lists(const ListsCost *in, int n_in, const ListsCost *rec, int n_rec, int slices) {
  const double lists = slices * (5.0 + currents_lists_walk_us(in, n_in) + currents_lists_walk_us(rec, n_rec));
  double work = 0.0, chain = 0.0; // one launch for both
  currents_mfma_us(in, n_in, slices, &work, &chain);
  currents_mfma_us(rec, n_rec, slices, &work, &chain);
  return 1.1 * lists < 10.0 + (work > chain ? work : chain);
}
