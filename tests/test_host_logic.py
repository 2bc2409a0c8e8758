"""Host-side logic of the GPU library (no GPU needed): the shared library loads and exports every
symbol the header declares, its schedule generator reproduces the order of Fig. 1 and the
oracle's own execution order, and its state-slot / byte accounting follows the paper's closed forms."""
import math
import os
import re
import subprocess

import numpy as np
import pytest

import oracle
import paper_2412_11810_amd as snn

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GOLD = os.path.join(ROOT, "tests", "golden")


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "snn.h")).read()
    declared = set(re.findall(r"^(?:snn_status|size_t|int32_t|int64_t|const char \*|void)\s*(snn_[a-z_]+)\(", header, re.M))
    assert declared == set(snn.EXPORTS)
    L = snn.lib()
    for name in declared:
        assert hasattr(L, name), name


def test_schedule_matches_fig1_double_panel():
    gold = []
    for line in open(os.path.join(GOLD, "fig1_double_schedule.txt")):
        line = line.strip()
        if line and not line.startswith("#"):
            p = line.split()
            gold.append((p[0], int(p[1]), int(p[2]) if len(p) > 2 else 0))
    ops = [o for o in snn.snn_schedule(snn.SNN_DOUBLE, 11, 6, 3) if o[0] != "SAVE_REMOTE"]
    assert ops == gold


@pytest.mark.parametrize("strategy,T,C,F", [
    (snn.SNN_STANDARD, 23, 0, 0), (snn.SNN_CHUNK, 23, 0, 5), (snn.SNN_CHUNK, 24, 0, 6), (snn.SNN_CHUNK, 7, 0, 7),
    (snn.SNN_REMOTE, 23, 4, 0), (snn.SNN_REMOTE, 9, 9, 0), (snn.SNN_DOUBLE, 23, 7, 3), (snn.SNN_DOUBLE, 50, 20, 6),
    (snn.SNN_DOUBLE, 31, 10, 10), (snn.SNN_DOUBLE, 17, 17, 1), (snn.SNN_DOUBLE, 40, 9, 2),
    (snn.SNN_HIER, 50, 2, 5), (snn.SNN_HIER, 23, 3, 4), (snn.SNN_HIER, 40, 1, 10), (snn.SNN_HIER, 30, 8, 5)])
def test_schedule_equals_oracle_execution_order(strategy, T, C, F):
    """The library's schedule generator and the oracle were written separately; both must walk the
    same checkpoints in the same order."""
    rng = np.random.default_rng(0)
    r = oracle.bptt(3, [4], 2, [rng.standard_normal((3, 4))], [rng.standard_normal((4, 4))],
                    rng.standard_normal((4, 2)), (rng.random((T, 1, 3)) < 0.3).astype(np.uint8), [0],
                    strategy=strategy, coarse=C, fine=F, want_events=True)
    assert snn.snn_schedule(strategy, T, C, F) == r.events


@pytest.mark.parametrize("T,C,F", [(64, 16, 4), (4096, 64, 8), (100, 25, 5), (1000, 32, 6), (100000, 316, 18)])
def test_state_slots_follow_closed_forms(T, C, F):
    cd = lambda a, b: -(-a // b)
    assert snn.snn_state_slots(snn.SNN_STANDARD, T) == (T, 0)                        # M_Base
    assert snn.snn_state_slots(snn.SNN_CHUNK, T, 0, F) == (F + cd(T, F), 0)          # M_Standard
    # host tier: the paper's count plus 9 staging slots (second prefetch slot, eight D2H staging slots: the
    # layers of the forward pass run two tiles apart, up to seven segment ends are being assembled at once)
    assert snn.snn_state_slots(snn.SNN_REMOTE, T, C, 0) == (C + 1 + 9, cd(T, C))     # M_Remote
    assert snn.snn_state_slots(snn.SNN_DOUBLE, T, C, F) == (F + cd(C, F) + 9, cd(T, C))  # M_Double


def test_hierarchical_slots():
    """M_Hier = chunk + nb_local (paper) plus the ring positions that keep the pipelined forward pass
    and the host transfers from colliding: (1 + ceil(6/nb_local)) more batches."""
    cd = lambda a, b: -(-a // b)
    for T, NL, F in [(1000, 4, 25), (4096, 8, 64), (100, 1, 10), (100, 2, 10)]:
        n_ckpt = cd(T, F)
        extra = (1 + cd(6, NL)) * NL
        assert snn.snn_state_slots(snn.SNN_HIER, T, NL, F) == (F + NL + extra, (cd(n_ckpt, NL) - 1) * NL)


def test_default_intervals_are_square_roots():
    assert snn.snn_state_slots(snn.SNN_CHUNK, 4096) == (64 + 64, 0)                  # chunk = sqrt(T) = 64
    n, r = snn.snn_state_slots(snn.SNN_DOUBLE, 4096)
    assert (n, r) == (8 + 8 + 9, 64)                                                 # C = 64, F = 8
    n, r = snn.snn_state_slots(snn.SNN_DOUBLE, 100000)
    assert r == math.ceil(100000 / 317)                                              # ceil(sqrt(1e5)) = 317


def test_bytes_required_accounting():
    cfg = snn.make_config(700, [256, 256], 20, 1000, 32)
    Ms = 4 * 32 * 512
    spikes = 8 * 1001 * 32 * (11 + 4 + 4)
    for strat, C, F in [(snn.SNN_STANDARD, 0, 0), (snn.SNN_CHUNK, 0, 32), (snn.SNN_REMOTE, 32, 0), (snn.SNN_DOUBLE, 100, 10)]:
        slots, _ = snn.snn_state_slots(strat, 1000, C, F)
        chunk = {snn.SNN_STANDARD: 1000, snn.SNN_CHUNK: 32, snn.SNN_REMOTE: 32, snn.SNN_DOUBLE: 10}[strat]
        assert snn.snn_bytes_required(cfg, strat, 1000, C, F) == slots * Ms + spikes + max(min(chunk, 256) * 32 * (3 * 20 + 512) * 4, 64 * 32 * (8 * 20 + 2 * 512) * 4)
    # invalid intervals
    assert snn.snn_bytes_required(cfg, snn.SNN_DOUBLE, 1000, 10, 20) == 0
    assert snn.snn_state_slots(snn.SNN_CHUNK, 10, 0, 11) == (0, 0)


def test_double_local_memory_grows_like_fourth_root():
    """With C = sqrt(T) and F = sqrt(C), Double keeps 2 T^(1/4) states resident (Discussion; Fig. 1 label)."""
    for T in (256, 4096, 65536):
        Cc = int(round(T ** 0.5))
        Ff = int(round(Cc ** 0.5))
        assert snn.snn_state_slots(snn.SNN_DOUBLE, T, Cc, Ff)[0] - 9 == 2 * round(T ** 0.25)


def test_suggested_intervals_fit_the_budget_and_grow_with_it():
    """snn_suggest_intervals: the plan it returns fits the budget, a larger budget never shortens the chunk, no
    budget gives the 256-step cap, and a budget below the memory-minimal plan is an error (paper Section
    "Hyperparameter Study": memory is smallest at the square-root intervals)."""
    cfg = snn.make_config(700, [256, 256], 20, 4096, 32)
    T = 4096
    for strat in (snn.SNN_CHUNK, snn.SNN_REMOTE, snn.SNN_DOUBLE, snn.SNN_HIER):
        C0, F0 = snn.snn_suggest_intervals(cfg, strat, T, 0)
        chunk0 = C0 if strat == snn.SNN_REMOTE else F0
        assert chunk0 == 256
        floor_plan = {snn.SNN_CHUNK: (0, 64), snn.SNN_REMOTE: (1, 0), snn.SNN_DOUBLE: (1, 1), snn.SNN_HIER: (8, 64)}[strat]
        least = snn.snn_bytes_required(cfg, strat, T, *floor_plan)
        with pytest.raises(snn.SnnError) as e:
            snn.snn_suggest_intervals(cfg, strat, T, least - 1)
        assert e.value.status == snn.SNN_E_BUDGET
        prev = 0
        for extra_mb in (0, 1, 2, 4, 8, 16, 64):
            budget = least + extra_mb * (1 << 20)
            C, F = snn.snn_suggest_intervals(cfg, strat, T, budget)
            assert 0 < snn.snn_bytes_required(cfg, strat, T, C, F) <= budget
            chunk = C if strat == snn.SNN_REMOTE else F
            assert chunk >= prev
            prev = chunk
            if strat == snn.SNN_DOUBLE:
                assert C % F == 0 or C == T
                # one more fine checkpoint would not fit (or the segment already spans the sequence)
                assert C == T or snn.snn_bytes_required(cfg, strat, T, min(C + F, T), F) > budget
    assert snn.snn_suggest_intervals(cfg, snn.SNN_STANDARD, T, 0) == (0, 0)
    with pytest.raises(snn.SnnError):
        snn.snn_suggest_intervals(cfg, snn.SNN_STANDARD, T, 1 << 20)


def test_bench_refuses_more_than_one_gpu():
    """bench.py measures one GPU: asking for more exits with a message, before anything touches a device."""
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode != 0
    assert "one GPU" in (r.stderr + r.stdout)


def test_synthetic_inputs_are_seeded_and_shaped():
    """The shared input generator: same seed, same arrays; shapes and rates as the workload says; the forced spike
    trains of the micro-benchmark hit their rate."""
    import synth
    w = synth.config(1, T=40, B=4)
    a, b = synth.generate(w), synth.generate(w)
    assert np.array_equal(a["in_spikes"], b["in_spikes"]) and np.array_equal(a["W_rec"][1], b["W_rec"][1])
    assert a["in_spikes"].shape == (40, 4, 700) and a["in_spikes"].dtype == np.uint8
    assert a["W_in"][0].shape == (700, 256) and a["W_out"].shape == (256, 20) and a["labels"].shape == (4,)
    assert abs(float(a["in_spikes"].mean()) - w.p_in) < 0.005
    m = synth.generate(synth.Workload("masked", 10, (64, 64), 3, T=5, B=2, p_in=0.1, rec_density=0.25, seed=5))
    assert m["rec_mask"] is not None and abs(float(m["rec_mask"][0].mean()) - 0.25) < 0.05
    assert np.all(m["W_rec"][0][m["rec_mask"][0] == 0] == 0.0)
    h = synth.forced_spike_trains(synth.config(1, T=200, B=8), [0.05, 0.2])
    assert h[0].shape == (200, 8, 256) and abs(float(h[0].mean()) - 0.05) < 0.005 and abs(float(h[1].mean()) - 0.2) < 0.01


def test_row_blocks_of_the_chip_wide_adjoint_over_compressed_rows(tmp_path):
    """Every row block that takes part in that kernel's exchange owns at least one row -- a workgroup that reads the
    exchange without writing to it is waited for by nobody and may find entries cleared that it has not read -- the blocks
    cover every row once, and their sixteen wavefronts cover a block."""
    src = tmp_path / "split.cpp"
    src.write_text("""
#include <cstdio>
#include "snn_split.h"
int main() {
  int idle = 0;
  for (int N = 1025; N <= 8192; ++N)
    for (int n_rb = 8; n_rb <= 256; n_rb += 8) {
      const int R = csrw_block_rows(N, n_rb), nw = csrw_wave_rows(N, n_rb), act = csrw_active_blocks(N, n_rb);
      if (nw > 64) continue; // the launcher does not run these
      idle += act < n_rb;
      bool ok = act >= 1 && act <= n_rb && 16 * nw >= R && act * R >= N;
      for (int rb = 0; ok && rb < act; ++rb) ok = rb * R < N;
      if (!ok) { std::printf("N = %d, n_rb = %d: %d blocks of %d rows\\n", N, n_rb, act, R); return 1; }
    }
  std::printf("%d\\n", idle);
  return csrw_active_blocks(1100, 128) == 123 ? 0 : 1;
}
""")
    exe = tmp_path / "split"
    csrc = os.path.join(ROOT, "paper_2412_11810_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-I", csrc, str(src), "-o", str(exe)], check=True)
    got = subprocess.run([str(exe)], capture_output=True, text=True)
    assert got.returncode == 0, got.stdout
    assert int(got.stdout) > 0  # shapes that leave blocks without rows are among them


def test_lds_of_the_sequential_forward_part(tmp_path):
    """Every plan of the sequential part of 257..1024 neurons stays within what the launch may ask for, has lists that hold a
    quarter of the widest layer with the reads ahead, and places its workgroups; widths whose list just reaches the end of
    the LDS (835, 836, 1013) still have one."""
    src = tmp_path / "plan.cpp"
    src.write_text("""
#include <cstdio>
#include "snn_plan.h"
int main() {
  int plans = 0, tight = 0;
  for (int N = 257; N <= 1024; ++N)
    for (int jobs = 1; jobs <= 4; ++jobs)
      for (int B = 1; B <= 1024; ++B) {
        SeqLdsPlan p{};
        if (!seq_lds_geometry(N, B, jobs, 32, 256, &p)) continue;
        const int per_wave = 64 / p.lpb;
        const size_t lists = (size_t)p.waves * per_wave * p.lcap * 2, weights = (size_t)(N + 1) * p.lpb * 4;
        const bool ok = p.lds == weights + lists && p.lds <= SEQ_LDS_DYNAMIC && p.lcap >= 256 + 48 && p.lcap % 8 == 0 &&
                        p.waves <= 16 && p.groups * p.waves * per_wave >= B && p.units == jobs * p.groups &&
                        p.slices * p.lpb >= N && (p.units + 7) / 8 * p.slices <= 32 && p.units * p.slices <= 256;
        if (!ok) { std::printf("N = %d, %d jobs, B = %d: %zu bytes, lists of %d\\n", N, jobs, B, p.lds, p.lcap); return 1; }
        ++plans;
        tight += p.lcap < N + 48;
      }
  std::printf("%d %d\\n", plans, tight);
  SeqLdsPlan p{};
  return seq_lds_geometry(835, 33, 4, 32, 256, &p) && seq_lds_geometry(836, 129, 1, 32, 256, &p) && seq_lds_geometry(1013, 65, 1, 32, 256, &p) ? 0 : 1;
}
""")
    exe = tmp_path / "plan"
    csrc = os.path.join(ROOT, "paper_2412_11810_amd", "csrc")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", csrc, str(src), "-o", str(exe)], check=True)
    got = subprocess.run([str(exe)], capture_output=True, text=True)
    assert got.returncode == 0, got.stdout
    plans, tight = map(int, got.stdout.split())
    assert 0 < tight < plans  # lists shorter than their layer are among them


def test_weights_of_the_register_stationary_chain_stay_in_the_matrix(tmp_path):
    """Every load of the chain's prologue is of a weight of the matrix (rows past the layer's width: the last one's), or its lane's
    offset alone lies outside the buffer: nothing may count on the scalar offset being part of the bounds check."""
    src = tmp_path / "rs.cpp"
    src.write_text("""
#include <cstdio>
#include "snn_plan.h"
int main() {
  for (int N = 1; N <= 256; ++N) {
    const int NW = (N + 31) / 32 * 32;
    for (int q = 0; q < NW; ++q)
      for (int i = 0; i < 256; ++i) {
        const uint32_t lane = seq_rs_lane_offset(N, i), row = seq_rs_row_offset(N, NW, q), bytes = (uint32_t)(N * N) * 4u;
        const int r = q < N ? q : N - 1;
        const bool ok = row < bytes && (i < N ? (uint64_t)lane + row == (uint64_t)(r * N + i) * 4u : lane >= BUFFER_OUTSIDE);
        if (!ok) { std::printf("N = %d, row %d, column %d\\n", N, q, i); return 1; }
      }
  }
}
""")
    exe = tmp_path / "rs"
    csrc = os.path.join(ROOT, "paper_2412_11810_amd", "csrc")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", csrc, str(src), "-o", str(exe)], check=True)
    got = subprocess.run([str(exe)], capture_output=True, text=True)
    assert got.returncode == 0, got.stdout


# Recompute currents of 192 steps, measured: inputs (5 % active), layers, batch, activity of the layers, us on the matrix cores, us by lists
MEASURED_CURRENTS = [
    (64, (300,), 16, (0.037,), 17, 49),
    (64, (512,), 16, (0.037,), 27, 54),
    (64, (1024,), 16, (0.452,), 116, 152),
    (64, (1500,), 16, (0.046,), 150, 134),
    (64, (2048,), 16, (0.043,), 290, 152),
    (64, (2048,), 16, (0.457,), 443, 478),
    (64, (2800,), 16, (0.044,), 539, 452),
    (64, (300,), 64, (0.457,), 54, 113),
    (64, (512,), 64, (0.037,), 76, 74),
    (64, (512,), 64, (0.428,), 107, 140),
    (64, (800,), 64, (0.051,), 168, 134),
    (64, (800,), 64, (0.452,), 234, 367),
    (64, (1024,), 64, (0.154,), 301, 230),
    (64, (1024,), 64, (0.452,), 352, 452),
    (64, (1500,), 64, (0.047,), 525, 323),
    (64, (1500,), 64, (0.483,), 745, 1257),
    (64, (2048,), 64, (0.245,), 1303, 985),
    (64, (2550,), 64, (0.043,), 1572, 763),
    (64, (2550,), 64, (0.447,), 2412, 3540),
    (64, (2800,), 64, (0.161,), 2545, 3167),
    (64, (2800,), 64, (0.451,), 3003, 7806),
    (64, (1024, 2048), 16, (0.044, 0.046), 428, 261),
    (64, (1024, 2048), 16, (0.451, 0.471), 675, 796),
    (2000, (512,), 32, (0.041,), 208, 91),
    (2000, (512,), 32, (0.435,), 204, 125),
    (4000, (400,), 32, (0.048,), 591, 144),
    (4000, (400,), 32, (0.467,), 585, 170),
]


def test_choice_between_lists_and_matrix_cores_follows_the_measured_times(tmp_path):
    """The estimate that picks the kernel of a launch's currents costs at most 5 % against the better of the two at every measured
    point, on both sides of where they meet."""
    calls = []
    for n_in, hidden, B, rate, _, _ in MEASURED_CURRENTS:
        pre, r_in = (n_in,) + hidden[:-1], (0.05,) + rate[:-1]
        mat = lambda P, r: "{" + ", ".join("{%d, %d, %d, %g}" % (p, n, 64 * B, q) for p, n, q in zip(P, hidden, r)) + "}"
        calls.append("{ const ListsCost a[] = %s, b[] = %s; std::puts(currents_by_lists(a, %d, b, %d, 3) ? \"1\" : \"0\"); }"
                     % (mat(pre, r_in), mat(hidden, rate), len(hidden), len(hidden)))
    src = tmp_path / "choice.cpp"
    src.write_text('#include <cstdio>\n#include "snn_plan.h"\nint main() {\n' + "\n".join(calls) + "\n}\n")
    exe = tmp_path / "choice"
    csrc = os.path.join(ROOT, "paper_2412_11810_amd", "csrc")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", csrc, str(src), "-o", str(exe)], check=True)
    picked = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()
    assert len(picked) == len(MEASURED_CURRENTS) and {"0", "1"} == set(picked)
    for choice, (n_in, hidden, B, rate, mfma, lists) in zip(picked, MEASURED_CURRENTS):
        took = lists if choice == "1" else mfma
        assert took <= 1.05 * min(mfma, lists), (n_in, hidden, B, rate, choice)


# Forward passes over 64 steps with the sequential parts by column, over compressed rows and over the dense-stored matrix: layers, neurons,
# batch, density, one neuron has every synapse, activity, ms of the three
MEASURED_WALKS = [
    (1, 8192, 32, 0.03, False, 0.017, 1.89, 1.50, 1.23),
    (1, 8192, 32, 0.03, False, 0.042, 1.94, 2.33, 2.61),
    (1, 8192, 32, 0.03, False, 0.082, 2.01, 3.59, 4.84),
    (1, 8192, 32, 0.03, False, 0.189, 2.11, 6.84, 9.17),
    (1, 8192, 32, 0.03, False, 0.384, 2.14, 12.07, 8.19),
    (1, 8192, 32, 0.1, False, 0.018, 4.41, 1.71, 1.24),
    (1, 8192, 32, 0.1, False, 0.042, 4.46, 2.84, 2.63),
    (1, 8192, 32, 0.1, False, 0.083, 4.54, 4.61, 4.90),
    (1, 8192, 32, 0.1, False, 0.182, 4.66, 8.81, 9.07),
    (1, 8192, 32, 0.1, False, 0.379, 4.66, 15.83, 8.13),
    (1, 8192, 32, 0.2, False, 0.017, 8.01, 4.58, 1.23),
    (1, 8192, 32, 0.2, False, 0.042, 8.04, 9.87, 2.62),
    (1, 8192, 32, 0.2, False, 0.082, 8.13, 18.26, 4.85),
    (1, 8192, 32, 0.2, False, 0.181, 8.22, 30.89, 9.21),
    (1, 8192, 32, 0.2, False, 0.377, 8.24, 59.21, 8.10),
    (1, 8192, 32, 0.3, False, 0.018, 11.64, 7.68, 1.24),
    (1, 8192, 32, 0.3, False, 0.041, 11.67, 16.73, 2.58),
    (1, 8192, 32, 0.3, False, 0.081, 11.72, 31.34, 4.80),
    (1, 8192, 32, 0.3, False, 0.184, 11.83, 54.36, 9.24),
    (1, 8192, 32, 0.3, False, 0.379, 11.86, 103.17, 8.13),
    (1, 8192, 32, 0.1, True, 0.186, 34.82, 9.08, 9.09),
    (4, 8192, 32, 0.03, False, 0.005, 10.23, 7.63, 8.90),
    (4, 8192, 32, 0.03, False, 0.038, 10.23, 10.64, 17.74),
    (4, 8192, 32, 0.03, False, 0.187, 10.39, 23.62, 43.45),
    (4, 8192, 32, 0.03, False, 0.335, 10.43, 33.19, 49.32),
    (4, 8192, 32, 0.03, False, 0.443, 10.47, 39.84, 58.02),
    (4, 8192, 32, 0.1, False, 0.005, 16.95, 7.92, 8.89),
    (4, 8192, 32, 0.1, False, 0.039, 16.96, 12.18, 17.85),
    (4, 8192, 32, 0.1, False, 0.192, 17.05, 30.53, 43.37),
    (4, 8192, 32, 0.1, False, 0.335, 16.98, 43.26, 49.32),
    (4, 8192, 32, 0.1, False, 0.446, 16.97, 51.93, 58.86),
    (4, 8192, 32, 0.2, False, 0.005, 25.98, 11.47, 8.92),
    (4, 8192, 32, 0.2, False, 0.040, 26.20, 32.09, 18.09),
    (4, 8192, 32, 0.2, False, 0.185, 26.29, 99.99, 43.94),
    (4, 8192, 32, 0.2, False, 0.336, 26.39, 146.89, 49.29),
    (4, 8192, 32, 0.2, False, 0.445, 26.40, 187.21, 58.74),
    (4, 8192, 32, 0.3, False, 0.005, 34.71, 15.35, 8.89),
    (4, 8192, 32, 0.3, False, 0.039, 34.84, 51.39, 18.06),
    (4, 8192, 32, 0.3, False, 0.191, 35.05, 175.74, 43.83),
    (4, 8192, 32, 0.3, False, 0.336, 35.14, 255.55, 49.38),
    (4, 8192, 32, 0.3, False, 0.443, 35.07, 324.87, 57.60),
    (4, 8192, 32, 0.1, True, 0.187, 93.44, 30.06, 43.60),
    (2, 8192, 8, 0.03, False, 0.010, 3.28, 2.89, 3.61),
    (2, 8192, 8, 0.03, False, 0.042, 3.33, 3.50, 5.13),
    (2, 8192, 8, 0.03, False, 0.117, 3.41, 7.45, 8.56),
    (2, 8192, 8, 0.03, False, 0.264, 3.54, 14.36, 13.72),
    (2, 8192, 8, 0.03, False, 0.423, 3.58, 20.36, 18.36),
    (2, 8192, 8, 0.1, False, 0.010, 6.76, 2.96, 3.61),
    (2, 8192, 8, 0.1, False, 0.041, 6.82, 4.35, 5.08),
    (2, 8192, 8, 0.1, False, 0.114, 6.90, 9.66, 8.45),
    (2, 8192, 8, 0.1, False, 0.268, 7.01, 19.55, 13.88),
    (2, 8192, 8, 0.1, False, 0.427, 7.01, 27.73, 18.49),
    (2, 8192, 8, 0.2, False, 0.010, 12.10, 6.02, 3.58),
    (2, 8192, 8, 0.2, False, 0.042, 12.16, 16.15, 5.11),
    (2, 8192, 8, 0.2, False, 0.115, 12.25, 41.67, 8.44),
    (2, 8192, 8, 0.2, False, 0.264, 12.36, 83.81, 13.76),
    (2, 8192, 8, 0.2, False, 0.419, 12.36, 121.15, 18.25),
    (2, 8192, 8, 0.3, False, 0.010, 17.43, 10.09, 3.62),
    (2, 8192, 8, 0.3, False, 0.041, 17.46, 27.85, 5.09),
    (2, 8192, 8, 0.3, False, 0.114, 17.52, 73.02, 8.42),
    (2, 8192, 8, 0.3, False, 0.267, 17.68, 149.61, 13.90),
    (2, 8192, 8, 0.3, False, 0.415, 17.78, 209.56, 18.18),
    (2, 8192, 8, 0.1, True, 0.113, 51.69, 9.68, 8.41),
    (3, 4096, 32, 0.03, False, 0.007, 4.33, 3.22, 1.91),
    (3, 4096, 32, 0.03, False, 0.040, 4.34, 5.01, 2.66),
    (3, 4096, 32, 0.03, False, 0.150, 4.44, 9.89, 4.32),
    (3, 4096, 32, 0.03, False, 0.313, 4.48, 16.62, 6.34),
    (3, 4096, 32, 0.03, False, 0.436, 4.48, 21.68, 7.88),
    (3, 4096, 32, 0.1, False, 0.007, 8.24, 3.37, 1.93),
    (3, 4096, 32, 0.1, False, 0.040, 8.28, 5.76, 2.63),
    (3, 4096, 32, 0.1, False, 0.150, 8.37, 12.50, 4.33),
    (3, 4096, 32, 0.1, False, 0.311, 8.42, 21.66, 6.33),
    (3, 4096, 32, 0.1, False, 0.432, 8.42, 28.54, 7.89),
    (3, 4096, 32, 0.2, False, 0.007, 13.66, 4.88, 1.97),
    (3, 4096, 32, 0.2, False, 0.041, 13.72, 15.31, 2.69),
    (3, 4096, 32, 0.2, False, 0.150, 13.79, 43.86, 4.38),
    (3, 4096, 32, 0.2, False, 0.307, 13.86, 80.51, 6.26),
    (3, 4096, 32, 0.2, False, 0.431, 13.80, 110.51, 7.87),
    (3, 4096, 32, 0.3, False, 0.007, 18.99, 6.56, 1.96),
    (3, 4096, 32, 0.3, False, 0.040, 19.13, 25.00, 2.69),
    (3, 4096, 32, 0.3, False, 0.149, 19.14, 74.46, 4.32),
    (3, 4096, 32, 0.3, False, 0.314, 19.20, 141.87, 6.39),
    (3, 4096, 32, 0.3, False, 0.438, 19.16, 195.07, 7.90),
    (3, 4096, 32, 0.1, True, 0.149, 53.16, 12.61, 4.27),
    (1, 4096, 16, 0.03, False, 0.017, 1.15, 0.99, 0.45),
    (1, 4096, 16, 0.03, False, 0.041, 1.16, 1.38, 0.59),
    (1, 4096, 16, 0.03, False, 0.083, 1.18, 2.00, 0.83),
    (1, 4096, 16, 0.03, False, 0.188, 1.22, 3.50, 1.37),
    (1, 4096, 16, 0.03, False, 0.375, 1.28, 6.16, 2.17),
    (1, 4096, 16, 0.1, False, 0.017, 2.46, 1.09, 0.44),
    (1, 4096, 16, 0.1, False, 0.041, 2.48, 1.63, 0.59),
    (1, 4096, 16, 0.1, False, 0.081, 2.52, 2.46, 0.83),
    (1, 4096, 16, 0.1, False, 0.184, 2.54, 4.60, 1.35),
    (1, 4096, 16, 0.1, False, 0.388, 2.60, 8.54, 2.22),
    (1, 4096, 16, 0.3, False, 0.017, 6.01, 3.84, 0.45),
    (1, 4096, 16, 0.3, False, 0.041, 6.02, 8.11, 0.59),
    (1, 4096, 16, 0.3, False, 0.081, 6.05, 15.63, 0.83),
    (1, 4096, 16, 0.3, False, 0.183, 6.07, 31.86, 1.33),
    (1, 4096, 16, 0.3, False, 0.373, 6.12, 59.95, 2.16),
    (1, 4096, 16, 0.1, True, 0.182, 17.57, 4.61, 1.34),
]


def test_choice_of_the_walk_of_masked_layers_follows_the_measured_times(tmp_path):
    """By column only where that is the faster walk: never more than 3 % slower than the one that runs else, and rarely the slower choice."""
    calls, expect = [], []
    for L, N, B, density, full, rate, col, rows, dense in MEASURED_WALKS:
        longest = N if full else -(-int(density * N + 2.6 * (N * density * (1 - density)) ** 0.5) // 8) * 8
        for walk, other in ((1, rows), (0, dense)):
            for n in {1, L}:
                one = "{%d, %d, %d, %g}" % (N, int(density * N * N), longest, rate)
                calls.append("{ const MaskedLayer l[] = {%s}; std::puts(seq_by_column(l, %d, %d, %d) ? \"1\" : \"0\"); }"
                             % (", ".join([one] * n), n, B, walk))
                expect.append((n == L, col, other, (L, N, B, density, full, rate, walk)))
    calls.append("{ const MaskedLayer l[] = {{8192, 6710886, 896, 0.3}, {8192, 6710886, 896, -1.0}};"
                 " std::puts(seq_by_column(l, 1, 32, 1) && !seq_by_column(l, 2, 32, 1) && !seq_by_column(l, 0, 32, 1) ? \"1\" : \"0\"); }")
    src = tmp_path / "walk.cpp"
    src.write_text('#include <cstddef>\n#include <cstdint>\n#include <cstdio>\n#include "snn_plan.h"\nint main() {\n' + "\n".join(calls) + "\n}\n")
    exe = tmp_path / "walk"
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2412_11810_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    picked = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()
    assert picked.pop() == "1" and len(picked) == len(expect) and {"0", "1"} == set(picked)
    slower = 0
    for choice, (all_layers, col, other, what) in zip(picked, expect):
        if choice == "1":
            assert col <= 1.03 * other, (what, col, other)
        elif all_layers:
            slower += other > 1.15 * col
    assert slower <= len(MEASURED_WALKS) // 20


# Training steps, us: inputs, layers, batch, with k_dw_split, with the better of the other two (both at 3 % and at 45 % activity)
MEASURED_GRADIENTS = [
    (300, (1024, 1024), 12, 1901, 1911),
    (300, (1024, 1024), 12, 2808, 2874),
    (300, (1024, 1024), 32, 2028, 2119),
    (300, (1024, 1024), 32, 2985, 3230),
    (300, (1024, 1024), 64, 2303, 2492),
    (300, (1024, 1024), 64, 3452, 3855),
    (512, (640, 640, 640), 12, 1903, 1918),
    (512, (640, 640, 640), 12, 2548, 2571),
    (512, (640, 640, 640), 32, 2058, 2163),
    (512, (640, 640, 640), 32, 2704, 2811),
    (512, (640, 640, 640), 64, 2439, 2674),
    (512, (640, 640, 640), 64, 3249, 3477),
    (200, (900, 900, 900), 12, 2140, 2188),
    (200, (900, 900, 900), 12, 3055, 3175),
    (200, (900, 900, 900), 32, 2385, 2490),
    (200, (900, 900, 900), 32, 3327, 3615),
    (200, (900, 900, 900), 64, 3005, 3214),
    (200, (900, 900, 900), 64, 4269, 4785),
    (700, (1024, 1024, 1024), 12, 2200, 2234),
    (700, (1024, 1024, 1024), 12, 3306, 3456),
    (700, (1024, 1024, 1024), 32, 2471, 2577),
    (700, (1024, 1024, 1024), 32, 3666, 4019),
    (700, (1024, 1024, 1024), 64, 3080, 3331),
    (700, (1024, 1024, 1024), 64, 4795, 5417),
    (512, (2048,), 12, 1577, 1566),
    (512, (2048,), 12, 2735, 2882),
    (512, (2048,), 32, 1712, 1727),
    (512, (2048,), 32, 3079, 3437),
    (512, (2048,), 64, 2055, 2091),
    (512, (2048,), 64, 3987, 4654),
    (300, (1100, 1100), 12, 2189, 2207),
    (300, (1100, 1100), 12, 3167, 3258),
    (300, (1100, 1100), 32, 2410, 2513),
    (300, (1100, 1100), 32, 3583, 3816),
    (300, (1100, 1100), 64, 3112, 3270),
    (300, (1100, 1100), 64, 4864, 5344),
    (512, (2048, 2048), 12, 2998, 3000),
    (512, (2048, 2048), 12, 5055, 5413),
    (512, (2048, 2048), 32, 3464, 3526),
    (512, (2048, 2048), 32, 6071, 6884),
    (512, (2048, 2048), 64, 4710, 4829),
    (512, (2048, 2048), 64, 8993, 10554),
]
# ... of masked networks (layers of that width): batch, activity, dense gradients by k_dw_split, per existing synapse
MEASURED_MASKED = [
    (2048, 12, 0.006, 2441, 2601),
    (2048, 12, 0.040, 2615, 2893),
    (2048, 12, 0.154, 3174, 3444),
    (2048, 32, 0.006, 2995, 3229),
    (2048, 32, 0.040, 3208, 3641),
    (2048, 32, 0.154, 3905, 4513),
    (1536, 12, 0.000, 2799, 3085),
    (1536, 12, 0.043, 3008, 3511),
    (1536, 12, 0.252, 3744, 4124),
    (1536, 32, 0.000, 3467, 3946),
    (1536, 32, 0.043, 3785, 4581),
    (1536, 32, 0.252, 4869, 5563),
    (2048, 12, 0.000, 4287, 4480),
    (2048, 12, 0.042, 4765, 5202),
    (2048, 12, 0.306, 6350, 6894),
    (2048, 32, 0.000, 5528, 5864),
    (2048, 32, 0.042, 6358, 7044),
    (2048, 32, 0.307, 8969, 10072),
    (3000, 12, 0.006, 5224, 5292),
    (3000, 12, 0.039, 6516, 6691),
    (3000, 12, 0.150, 8281, 8682),
    (3000, 32, 0.006, 6980, 7327),
    (3000, 32, 0.039, 8270, 8710),
    (3000, 32, 0.152, 10312, 10983),
    (4096, 12, 0.020, 2206, 2149),
    (4096, 12, 0.040, 2696, 2641),
    (4096, 12, 0.083, 3674, 3662),
    (4096, 32, 0.020, 2709, 2673),
    (4096, 32, 0.040, 3230, 3206),
    (4096, 32, 0.083, 4268, 4319),
    (4096, 12, 0.006, 4632, 4538),
    (4096, 12, 0.039, 6186, 6150),
    (4096, 12, 0.154, 8207, 8321),
    (4096, 32, 0.006, 6285, 6202),
    (4096, 32, 0.040, 8021, 7964),
    (4096, 32, 0.155, 10268, 10553),
    (8192, 12, 0.020, 2674, 2272),
    (8192, 12, 0.042, 3210, 2818),
    (8192, 12, 0.087, 4313, 3995),
    (8192, 32, 0.020, 3455, 3018),
    (8192, 32, 0.042, 4133, 3702),
    (8192, 32, 0.087, 5489, 5154),
]
# ... layers, batch, inter-layer products by k_up_split, on the fp32 matrix cores
MEASURED_PRODUCTS = [
    ((1024, 1024), 4, 1892, 1893),
    ((1024, 1024), 8, 1950, 1953),
    ((1024, 1024), 16, 1996, 1999),
    ((1024, 1024), 24, 2108, 2104),
    ((1024, 1024), 64, 2426, 2485),
    ((1500, 1100), 4, 2316, 2314),
    ((1500, 1100), 8, 2416, 2413),
    ((1500, 1100), 16, 2481, 2491),
    ((1500, 1100), 24, 2638, 2685),
    ((1500, 1100), 64, 3558, 3651),
    ((2048, 2048), 4, 3085, 3084),
    ((2048, 2048), 8, 3336, 3328),
    ((2048, 2048), 16, 3364, 3406),
    ((2048, 2048), 24, 3700, 3805),
    ((2048, 2048), 64, 5267, 5535),
    ((1024, 1024, 1024), 4, 6735, 6781),
    ((1024, 1024, 1024), 8, 7234, 7264),
    ((1024, 1024, 1024), 16, 7328, 7328),
    ((1024, 1024, 1024), 24, 8005, 8040),
    ((1024, 1024, 1024), 64, 11823, 12331),
    ((3000, 3000), 4, 59411, 59266),
    ((3000, 3000), 8, 59721, 59783),
    ((3000, 3000), 16, 59181, 59382),
    ((3000, 3000), 24, 59699, 59904),
    ((3000, 3000), 64, 62410, 62888),
    ((4096, 4096), 4, 4815, 4758),
    ((4096, 4096), 8, 4925, 4958),
    ((4096, 4096), 16, 4996, 5039),
    ((4096, 4096), 24, 6801, 6924),
    ((4096, 4096), 64, 11371, 11953),
]


def test_choice_of_the_split_kernels_follows_the_measured_times(tmp_path):
    """Shapes and batch alone decide (these kernels differ from the others in the last bits): where the split ones run they cost at most
    3 % in any measured step, and a masked matrix takes the better way but for 3 %."""
    calls = []
    for n_in, hidden, B, _, _ in MEASURED_GRADIENTS:
        mats = list(zip((n_in,) + hidden[:-1], hidden)) + [(n, n) for n in hidden] + [(hidden[-1], 20)]
        calls.append("dw_split_pays(%s, %d)" % (" + ".join("dw_split_tiles(%d, %d)" % m for m in mats), B))
    calls += ["dw_split_masked(%d)" % m[0] for m in MEASURED_MASKED]
    calls += ["split_product(%d, %d)" % m[0][:2] for m in MEASURED_PRODUCTS]
    calls += ["dw_split_pays(150, 11)", "dw_split_pays(149, 32)", "dw_split_pays(1000, 65)", "split_product(1023, 4096)", "split_product(4096, 1023)"]
    src = tmp_path / "split.cpp"
    src.write_text('#include <cstddef>\n#include <cstdint>\n#include <cstdio>\n#include "snn_plan.h"\nint main() {\n'
                   + "\n".join("std::puts(%s ? \"1\" : \"0\");" % c for c in calls) + "\n}\n")
    exe = tmp_path / "split"
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2412_11810_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    picked = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()
    assert picked[-5:] == ["0"] * 5
    measured = ([(True, m[-2], m[-1], m) for m in MEASURED_GRADIENTS] + [(None, m[-2], m[-1], m) for m in MEASURED_MASKED]
                + [(True, m[-2], m[-1], m) for m in MEASURED_PRODUCTS])
    for choice, (must, split, other, what) in zip(picked, measured):
        assert must is None or choice == "1", what
        assert (split if choice == "1" else other) <= 1.03 * min(split, other), what
