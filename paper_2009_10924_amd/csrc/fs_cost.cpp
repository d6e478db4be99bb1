#include "fs_cost.hpp"

#include <algorithm>
#include <cmath>

namespace fs {

const DeviceModel& device() {
  static const DeviceModel d;
  return d;
}

// What the streaming rate is divided by for the runs in which rows are accessed, see evaluate().
static double run_derating(const KernelCost& k) {
  double f = 1.0;
  if (k.access_run_bytes > 0 && k.access_run_bytes < 128) f *= 1.0 + (128.0 / k.access_run_bytes - 1.0);
  if (k.access_run_bytes > 0 && k.row_bytes > 0 && std::fmod(k.row_bytes, 128.0) != 0.0) {
    // (fitted for each of the three kinds of loop; a workgroup that works through several rows finds the line that two of
    // them share in its caches more often, and column sums are bound by other things first.  Rows of an odd number of 16-bit
    // elements: 94 such softmaxes timed in every shape, the one taken was 3.8 % behind the fastest, 2.7 % with weights of their own)
    const double shared_lines = k.rows_per_wave_loop <= 1 ? (k.off_words ? 2.2 : k.on_grid ? (k.barriers == 0 ? 0.9 : 1.3) : 1.65) : k.partial_bytes > 0 ? 0.3 : 1.07;
    f *= 1.0 + shared_lines * std::min(4.0, 128.0 / k.access_run_bytes);
  }
  return f;
}

KernelCost together(const std::vector<const KernelCost*>& members) {
  KernelCost t;
  t.hbm_bytes = t.elems = t.waves = 0;
  double valu = 0, trans = 0, bif = 0, lanes = 0, xlane = 0, barriers = 0;
  t.vgpr_estimate = 0;
  for (const KernelCost* m : members) {
    t.hbm_bytes += m->hbm_bytes * run_derating(*m);
    t.cache_bytes += m->cache_bytes;
    t.elems += m->elems;
    t.waves += m->waves;
    valu += m->valu_per_elem * m->elems;
    trans += m->trans_per_elem * m->elems;
    bif += m->bytes_in_flight_per_lane * m->waves;
    lanes += m->elems / std::max(0.05, m->lane_utilisation);
    xlane += m->xlane_steps * m->waves;
    barriers += m->barriers * m->waves;
    t.vgpr_estimate = std::max(t.vgpr_estimate, m->vgpr_estimate);
    t.lds_bytes_per_block = std::max(t.lds_bytes_per_block, m->lds_bytes_per_block);
    t.serial_tail_s = std::max(t.serial_tail_s, m->serial_tail_s);
  }
  t.valu_per_elem = valu / t.elems;
  t.trans_per_elem = trans / t.elems;
  t.bytes_in_flight_per_lane = bif / t.waves;
  t.lane_utilisation = t.elems / lanes;
  t.xlane_steps = (int32_t)std::lround(xlane / t.waves);
  t.barriers = (int32_t)std::lround(barriers / t.waves);
  return t;
}

CostResult evaluate(const KernelCost& k, int32_t vgprs_compiled) {
  const DeviceModel& d = device();
  CostResult r;
  r.vgprs = vgprs_compiled > 0 ? vgprs_compiled : k.vgpr_estimate;

  // Occupancy from registers, LDS and workgroup shape (Section 4.3).
  const uint32_t vg = std::max<uint32_t>(d.vgpr_granule, (r.vgprs + d.vgpr_granule - 1) / d.vgpr_granule * d.vgpr_granule);
  uint32_t occ = std::min<uint32_t>(d.max_waves_per_simd, d.vgpr_per_simd_lane / vg);
  const uint32_t wpb = std::max(1, k.waves_per_block);
  uint32_t blocks_per_cu = occ * d.simd_per_cu / wpb;
  if (k.lds_bytes_per_block > 0) blocks_per_cu = std::min<uint32_t>(blocks_per_cu, d.lds_per_cu / (uint32_t)k.lds_bytes_per_block);
  blocks_per_cu = std::max<uint32_t>(1, blocks_per_cu);
  const double waves_per_cu = std::min<double>(occ * d.simd_per_cu, (double)blocks_per_cu * wpb);
  r.waves_per_simd = (int32_t)std::max(1.0, std::floor(waves_per_cu / d.simd_per_cu));

  // N_wave: rounds of resident wavefronts.
  const double capacity = waves_per_cu * d.n_cu;
  const double resident = std::min(k.waves, capacity);
  const double rounds_exact = std::max(1.0, k.waves / capacity);
  const double rounds = std::ceil(rounds_exact - 1e-9);

  // L_warp: one trip of a wave = dependent memory phases + its instruction stream while
  // sharing the SIMD with the other resident waves.
  const double util = std::max(0.05, k.lane_utilisation);
  const double elems_per_wave_trip = k.elems / std::max(1.0, k.waves * k.rows_per_wave_loop);
  const double wave_instr = elems_per_wave_trip / 64.0 / util;
  const double cycles = wave_instr * (k.valu_per_elem * d.cycles_valu + k.trans_per_elem * d.cycles_trans) +
                        k.xlane_steps * d.cycles_xlane;
  const double simd_share = std::max(1.0, resident / (d.n_cu * d.simd_per_cu));
  // two or three waves on a SIMD do not cover each other's instruction latencies
  const double issue_stall = r.waves_per_simd < 4 ? 1.0 + 0.6 * (4 - r.waves_per_simd) : 1.0;
  const double t_issue = cycles * simd_share * issue_stall / d.clock_hz;
  const double t_barrier = d.barrier_idle_s + (d.barrier_s - d.barrier_idle_s) * std::min(1.0, resident / (d.n_cu * d.simd_per_cu));
  const double t_trip = k.dep_phases * d.mem_latency_s + k.barriers * t_barrier + t_issue;
  const double t_latency = rounds * (k.rows_per_wave_loop * t_trip + (k.first_load ? d.first_load_s : 0.0));

  // Streaming floor.  Achievable bandwidth = the measured copy rate, derated for
  //   * bytes in flight (Little's law),
  //   * short contiguous runs per access (a row group of L lanes touches L*16 bytes): below a 128-byte line each
  //     access wastes part of one, and where rows are no multiple of a line apart every run ends inside lines that
  //     the next access touches again,
  //   * lanes that hold padding (their clamped loads still occupy the memory pipeline),
  //   * a last, partly filled round of wavefronts.
  const double in_flight = resident * 64.0 * k.bytes_in_flight_per_lane * util;
  double bw = std::min(d.hbm_peak_Bps * d.stream_fraction, in_flight / d.queue_latency_s);
  bw /= run_derating(k);
  bw /= 1.0 + k.stream_penalty;
  if (k.store_run_bytes > 0 && k.store_run_bytes < 512) bw *= 0.97;
  bw /= 1.0 + (k.on_grid ? 0.3 : 0.12) * (1.0 / util - 1.0);
  bw /= 1.0 + 0.25 * (rounds / rounds_exact - 1.0);
  if (occ < 4) bw /= 1.0 + 0.04 * (4.0 - occ);   // few waves per SIMD: a wave's own stalls are not covered
  const double t_hbm = (k.hbm_bytes + d.partial_weight * k.partial_bytes) / bw;
  const double t_cache = k.cache_bytes / d.l2_Bps;
  const double t_lds = k.lds_traffic_bytes / d.lds_Bps;
  const double t_alu = k.elems / util / 64.0 * (k.valu_per_elem * d.cycles_valu + k.trans_per_elem * d.cycles_trans) /
                       (d.n_cu * d.simd_per_cu) / d.clock_hz;
  // every extra round of a kernel that runs in few rounds pays a ramp of its own;
  // so does a wave that has to wait for its index arithmetic before its first load
  const double t_ramp = std::min(rounds - 1.0, 2.0) * 0.25 * d.mem_latency_s +
                        k.preamble_instr * d.cycles_valu * simd_share / d.clock_hz;

  // The wave-rounds term and the streaming floor overlap only partly: a wave that is
  // computing is not loading, and only the other waves of its SIMD can fill the gap.
  // (re-reads that the caches serve share the memory pipeline with the stream but mostly fill its gaps: a quarter
  // of their own time shows, measured on the patterns with per-column operands)
  const double t_stream = std::max(t_hbm + 0.25 * t_cache + t_lds, t_alu);
  double t_body = std::max(t_latency, t_stream) + 0.10 * std::min(t_latency, t_stream);
  double t_sums = 0;
  if (k.partial_bytes > 0) {
    const double cus = std::min<double>(d.n_cu, std::max(1.0, k.waves / wpb));
    t_body = std::max(t_body, (k.hbm_bytes + k.partial_bytes) / cus / d.cu_Bps);
    t_sums = rounds * k.flush_values * (k.flush_steps < 0 ? d.flush_block_s : d.flush_value_s + k.flush_steps * d.flush_step_s) + d.fold_s +
             d.fold_batch_s * std::ceil(k.fold_rows / 512.0);
  }
  r.seconds = d.kernel_fixed_s + t_body + t_ramp + t_sums + k.serial_tail_s;
  return r;
}

}  // namespace fs
