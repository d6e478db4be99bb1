// Latency evaluator for one kernel launch, in the shape of the paper's Eq. 1
// (L = N_wave x L_warp, N_wave = N_warp / Occupancy, L_warp = N_instruction x CPI),
// re-derived for a bandwidth-bound part: the wave-rounds term is kept, and a
// streaming floor (bytes / achievable HBM bandwidth) is added because on MI355X these
// kernels run at the memory roofline, not at the instruction-issue limit.
#pragma once
#include <cstdint>
#include <vector>

namespace fs {

struct DeviceModel {
  // MI355X (gfx950) public figures
  uint32_t n_cu = 256;
  uint32_t simd_per_cu = 4;
  uint32_t max_waves_per_simd = 8;
  uint32_t vgpr_per_simd_lane = 512;
  uint32_t vgpr_granule = 8;
  uint32_t lds_per_cu = 160 * 1024;
  double clock_hz = 2.4e9;
  double hbm_peak_Bps = 8.0e12;
  // measured / calibrated on one MI355X: every candidate of about 1900 row patterns (rows of 16 to 131072 elements, three
  // dtypes, 0.2 MB to 2 GB) timed; over 1000 of them the candidate ranked first is on average 3.6 % behind the fastest one.
  // With terms that only knew rows of whole 128-byte lines it was 6.3 % over 400 of them: attention rows of 392 16-bit
  // elements ran on 8 lanes in 48.8 us where 64 lanes take 32.4.
  double stream_fraction = 0.84;     // one-shot kernels with three or more independent streams, fraction of hbm_peak
                                     // (the grid-stride copy kernel reaches 0.78)
  double mem_latency_s = 1.2e-6;     // loaded HBM round trip seen by a wave
  double launch_s = 2.2e-6;          // fixed cost of one kernel: dispatch, first load round trip, drain
  double kernel_fixed_s = 1.6e-6;    // the part of it that the evaluator's other terms do not cover
  double queue_latency_s = 0.17e-6;  // latency that bytes in flight have to cover for the full streaming rate
  double l2_Bps = 20.0e12;           // aggregate cache bandwidth for re-read operands
  double last_level_cache_bytes = 256.0 * 1024 * 1024;   // memory-side cache in front of HBM
  double last_level_reread = 0.45;   // time of a re-read that the memory-side cache still holds, relative to HBM (measured)
  // column sums, fitted to every candidate of bias + GELU, LayerNorm and RMS norm backward patterns like the rest: over the
  // first 170 of them the candidate ranked first was 3.7 % behind the fastest one on average, 7.3 % without these terms
  double cu_Bps = 3.3e10;            // what one compute unit streams at most (a loop over rows on few workgroups)
  double partial_weight = 2.4;       // a byte of partial sums, relative to a streamed one (a burst at the end, then a re-read)
  double flush_step_s = 9e-9, flush_value_s = 14e-9, flush_block_s = 30e-9;   // per value: each lane fold, LDS + store; store alone
  double fold_s = 3.0e-6, fold_batch_s = 0.1e-6;   // the fold launch, and per 512 rows of partial sums
  double lds_Bps = 60.0e12;          // aggregate LDS bandwidth
  // One workgroup barrier incl. the LDS round trip and the wait for the slowest wave: by itself, and where every SIMD has
  // wavefronts of its own to wait for (LayerNorm of 72 rows x 1888: wave form 4.7 us, block form 3.8; of 3000 x 1000: 7.9, 8.4).
  double barrier_idle_s = 0.15e-6, barrier_s = 0.65e-6;
  double first_load_s = 0.6e-6;      // a software-pipelined loop over rows: the part of the first row's load latency that shows
  double cycles_valu = 4.0;          // issue cycles of one wave-wide VALU op on a 16-lane SIMD
  double cycles_trans = 16.0;        // quarter-rate transcendental
  double cycles_xlane = 12.0;        // DPP / permute step incl. its dependency stall
};
const DeviceModel& device();

// What one candidate kernel does, as the enumerator describes it.
struct KernelCost {
  double hbm_bytes = 0;                 // bytes that must cross HBM
  double cache_bytes = 0;               // re-reads served by L1/L2
  double lds_traffic_bytes = 0;
  double elems = 0;
  double valu_per_elem = 0;             // plain VALU ops per element
  double trans_per_elem = 0;            // quarter-rate ops per element
  double waves = 0;                     // wavefronts launched
  int32_t waves_per_block = 4;
  double bytes_in_flight_per_lane = 16; // independent load bytes a lane has outstanding
  double rows_per_wave_loop = 1;        // sequential trips of the kernel's outer loop per wave
  double dep_phases = 1;                // dependent global-memory phases per trip (a part of one: partly hidden)
  bool first_load = false;              // the first trip's loads are waited for before the loop
  int32_t xlane_steps = 0;              // cross-lane steps per trip
  int32_t barriers = 0;                 // workgroup barriers per trip
  int32_t vgpr_estimate = 32;
  int32_t lds_bytes_per_block = 0;
  double lane_utilisation = 1.0;        // fraction of lanes holding data
  double access_run_bytes = 0;          // contiguous bytes one row group touches per load (0 = long)
  bool on_grid = false;                 // rows start anywhere, but accesses are aligned but for a row's first and last (row_on_grid())
  bool off_words = false;               // accesses of a workgroup's row start off a 4-byte boundary
  double row_bytes = 0;                 // from one row to the next, in the narrowest row operand (0 = not row by row)
  double stream_penalty = 0;            // the streaming rate falls to 1 / (1 + this) for reasons of the kernel's own
  double store_run_bytes = 0;           // contiguous run written by one store instruction group (0 = long)
  double preamble_instr = 40;           // VALU instructions a wave runs before it can issue its first load
  double serial_tail_s = 0;             // what no other wavefront covers: a lane's own chain from its loads to its stores
  double partial_bytes = 0;             // column sums: partial sums written by the workgroups and read by the fold launch
  double flush_values = 0;              // column sums: values of every lane that leave it at the end of its rows
  double fold_rows = 0;                 // column sums: rows of partial sums
  double flush_steps = -1;              // ... lane-to-lane folds before that (-1: a workgroup per row, no fold)
};

struct CostResult {
  double seconds = 0;
  int32_t waves_per_simd = 0;
  int32_t vgprs = 0;
};
CostResult evaluate(const KernelCost& k, int32_t vgprs_compiled);
// Several kernels without loops over rows or column sums as one launch with the registers of the hungriest.
KernelCost together(const std::vector<const KernelCost*>& members);

}  // namespace fs
