// How a masked layer's rows are dealt to workgroups and wavefronts in the chip-wide adjoint over compressed rows
// (k_adj_rec_csrw).  Plain integer functions, for the kernel and for checks on the host.
#pragma once

// rows of a row block when n_rb blocks are launched for N rows (the last one that owns rows may own fewer)
constexpr int csrw_block_rows(int N, int n_rb) { return (N + n_rb - 1) / n_rb; }
// Row blocks that take part.  Rounding up to whole rows leaves blocks at the end without any (N = 1100, n_rb = 128: five).
// They must not take part: the exchange clears entries on the evidence that who wrote a step's values had read the
// step before, and a workgroup that writes nothing is waited for by nobody.
constexpr int csrw_active_blocks(int N, int n_rb) { return (N + csrw_block_rows(N, n_rb) - 1) / csrw_block_rows(N, n_rb); }
// rows of each of a block's sixteen wavefronts
constexpr int csrw_wave_rows(int N, int n_rb) { return (csrw_block_rows(N, n_rb) + 15) / 16; }
