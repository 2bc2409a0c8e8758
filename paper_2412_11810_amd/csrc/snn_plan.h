// Launch geometry that integers alone decide, for the launchers and kernels and for checks on the host.
#pragma once
#include <stddef.h>
#include <stdint.h>

#define SNN_LDS_PER_CU (160 * 1024)

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
