// What the host prepares for an update's launches, from plain values: the layout
// of its scratch and the descriptor that the kernels read.  No device call.
#pragma once

#include <algorithm>
#include <cstring>

#include "brmppi_internal.h"
#include "served_core.h"

namespace brm {

// rollout launch shape: block size and variant (0 = one lane per sample,
// in-kernel noise; 1 = one lane, precomputed noise; 2 / 3 / 4 = two / four /
// eight lanes per sample, precomputed noise; 5 .. 7 chosen here, not settable: see
// variant_in_kernel and drawn_fits).  No shape changes any result bit.
struct LaunchShape {
  uint32_t block = 0;    // 0: not set
  int variant = 0;
};

// The shape of a plain solve that is neither tuned nor forced.  Blocks of 256:
// the dispatcher spreads a block's waves over its CU's SIMDs, and two blocks of
// two waves can land on the same two (65536 samples, 32 rows, one lane: 610 us
// at 128 threads, 330 at 256).  Lanes: as many as put one wave on each of the
// 1024 SIMDs (65536 lanes), since a wave issues at most one instruction every
// 4 cycles whatever else its SIMD holds; beyond that a lane keeps at most
// eight rows, because the one- and two-lane forms with more rows run out of
// registers.  Measured (us a solve, T = 40; 2/8/16/32 rows; two, four, eight
// lanes): 12000 samples 59 59 72 / 74 67 76 / 95 77 88 / 132 98 100; 20011
// samples 64 75 95 / 82 86 99 / 102 101 113 / 140 127 131; 32768 samples 69 80
// 117 / 85 90 117 / 108 106 136 / 150 136 163; 65536 samples with one lane and
// precomputed normals 84 / 165 / 643 / 293, with four lanes 120 / 136 / 175 / 251.
// Without guidance the lanes share the stage costs, which the collision penalty
// makes the largest part: 20011 samples, two / four / eight lanes 47 / 47 / 50,
// with the penalty over 24 obstacles 70 / 63 / 62; 65536 with one / four 62 / 76 and
// 108 / 107.
// Normals in HBM or drawn by the rollout (variant_in_kernel).  With eight rows the
// one-lane form with precomputed normals spills, most of all with moving obstacles
// or discs (65536 samples, T = 110: eight at rest 466, moving 1277, four around two
// discs 1481; drawn 292, 320, 591; four lanes 339, 368, 511): four lanes up to three
// quarters of a wave per SIMD (49152 samples, T = 60: 146, drawn 174; 57344: 177 and
// 174), drawn beyond.  Elsewhere the buffer pays until its traffic outweighs the
// draws: without guidance at 128 MB, where normals and applied inputs leave the
// last-level cache together (40000 samples, T = 200, 96 MB: 133 and 130 drawn;
// 32768, T = 400, 157 MB: 268 and 218; 131072, T = 110, 173 MB: 203 and 141); with the
// penalty, whose rows four lanes share, only with more than a wave per SIMD
// (131072 samples, T = 40, 63 MB: 24 obstacles 173 and 128; 65536, T = 110, 87 MB: 214
// and 219); with 16 rows around the rear axle from 512 MB and many waves on (65536
// samples, T = 110, 605 MB: 467 and 352; 131072, T = 40, 440 MB: 331 and 344; 40000,
// T = 200, 672 MB: 560 and 582; around four discs 65536, T = 110: 734 and 708, 100000,
// T = 200: 2128 and 2401).
inline LaunchShape default_shape(int bucket, uint32_t S, size_t noise_bytes, bool penalty, bool rear_axle) {
  LaunchShape s;
  s.block = 256;
  bool drawn = false;      // normals drawn by the rollout
  if (S <= 8192) {
    s.variant = 4;
  } else if (bucket == 0 && penalty) {
    s.variant = S <= 24576 ? 4 : 3;
    drawn = S > 65536 && noise_bytes > size_t(48) << 20;
  } else if (bucket == 32) {
    s.variant = S <= 24576 ? 4 : 3;
  } else if (bucket == 16) {
    s.variant = 3;
    drawn = rear_axle && S > 49152 && noise_bytes > size_t(512) << 20;
  } else if (bucket == 8) {
    s.variant = S > 16384 && S <= 32768 ? 2 : 3;
    drawn = S > 49152;
  } else {
    s.variant = S <= 16384 ? 3 : (S <= 32768 ? 2 : 1);
    drawn = bucket == 0 && noise_bytes > size_t(128) << 20;
  }
  if (drawn) s.variant = variant_in_kernel(bucket);
  return s;
}

// Whether k_rollout_drawn takes the place of the noise kernel and the rollout of
// eight lanes (fused: the bytes of its epilogue, 0 for none): up to a block per CU (a
// second one on a CU would wait for the first's LDS), tiles that reduce themselves, a
// horizon whose epilogue fits.  It saves a launch and the wait between the two, 2 to 6 us
// at up to 2048 samples and 4 to 14 at 8192 (drawn / two launches: 256 samples, 24 steps,
// 8 rows 40 / 43 us; 8192, 50 steps, 8 rows 57 / 63; 8192, 130 steps, 16 rows 121 / 132),
// and each run beyond the first costs it a pair of barriers and a draw that nothing
// hides, 2 to 3 us: with few samples, whose noise kernel is short, many runs lose (256
// samples, 32 rows: 40 steps, two runs 63 / 64; 60, three 82 / 79; 162, 14 181 / 160; 2048
// samples: 100 steps, seven 123 / 123; 162, 14 183 / 172; 8192 samples: 14 185 / 192).
constexpr uint32_t kDrawnBlocks = 256;   // eight groups at most
inline bool drawn_fits(int n_cu, int bucket, const LaunchShape& s, uint32_t S, uint32_t T, size_t fused) {
  return s.variant == 4 && s.block == 256 && S <= kDrawnTile * std::min<uint32_t>((uint32_t)n_cu, kDrawnBlocks) &&
         T <= kInlineSteps && fused > 0 && drawn_lds(bucket, T, fused).runs <= 2 + S / 256;
}

// what stays on the device for a controller between its updates
struct Resident {
  float* unom = nullptr;      // nominal sequence, 3T floats
  double* plant = nullptr;    // state, 8 doubles
  float4* path = nullptr;
  uint32_t n_path = 0;
  float ds = 0.0f;
  brmppi_params params{};     // used by problems whose params pointer is NULL
};

// layout of one instance's scratch inside a block (off_out: [stats(4) | u_new(3T)]
// for the plain and closed-loop paths; batches pack their outputs elsewhere)
struct ScratchLayout {
  size_t off_ustar, off_J, off_wpart, off_rpart, off_upart, off_urow, off_out, off_noise, bytes;
  uint32_t S_pad, n_wchunk, n_rgroup, n_normals;  // n_normals > 0: a noise buffer is included
  uint32_t n_units;
  uint32_t rows_item;   // rows of one reduce work item
};

// counters: the instance's, then one per group (fused epilogue), each on its
// own 128-B line so that the groups' atomics do not contend
inline size_t counter_bytes(uint32_t n_groups) {
  return round_up(sizeof(uint32_t) * kCtrStride * (1 + (size_t)n_groups), 256);
}

// units: with the partials of tiles that reduce themselves
inline ScratchLayout scratch_layout(uint32_t S, uint32_t T, uint32_t noise_normals = 0,
                                    uint32_t rows_item = kRowsPerPass, bool units = true) {
  ScratchLayout L;
  L.n_normals = noise_normals;
  L.S_pad = (uint32_t)round_up(S, 256);
  L.n_wchunk = (S + kWChunk - 1) / kWChunk;
  L.n_units = (S + kUnit - 1) / kUnit;
  L.rows_item = rows_item;
  L.n_rgroup = (3 * T + rows_item - 1) / rows_item;
  size_t o = 0;
  L.off_ustar = o;
  o = round_up(o + (size_t)3 * T * L.S_pad * sizeof(float), 256);
  L.off_J = o;
  o = round_up(o + (size_t)L.S_pad * sizeof(float), 256);
  L.off_wpart = o;
  o = round_up(o + (size_t)L.n_wchunk * sizeof(float4), 256);
  L.off_rpart = o;
  o = round_up(o + (size_t)L.n_wchunk * 3 * T * sizeof(float), 256);
  L.off_upart = o;
  o = round_up(o + (units ? (size_t)L.n_units * sizeof(float4) : 0), 256);
  L.off_urow = o;
  o = round_up(o + (units ? (size_t)L.n_units * 3 * T * sizeof(float) : 0), 256);
  L.off_out = o;
  o = round_up(o + (size_t)(4 + 3 * T) * sizeof(float), 256);
  L.off_noise = o;
  o = round_up(o + (size_t)noise_normals * T * L.S_pad * sizeof(float), 256);
  L.bytes = o;
  return L;
}

// an instance of a batch: reduced by k_reduce, no unit partials
inline ScratchLayout batch_scratch(uint32_t S, uint32_t T, uint32_t rows_item) {
  return scratch_layout(S, T, 0, rows_item, false);
}

// Device bytes that one request is counted with in a served batch: scratch,
// descriptor, tiles, work items and alignment slack.  What a batch takes stays below
// this at any launch shape: its smallest tiles, of 16 samples (block 64, four lanes),
// need less than the unit partials that it does not have.
inline size_t request_footprint(uint32_t S, uint32_t T) {
  const ScratchLayout L = scratch_layout(S, T);
  const size_t tiles = (S + 63) / 64;
  const size_t items = L.n_wchunk + (size_t)L.n_wchunk * L.n_rgroup;
  return L.bytes + sizeof(SolveDesc) + (tiles + items) * 8 + sizeof(float) * (4 + 6 * (size_t)T) + 8 * 256;
}

// base: the instance's scratch; unom_dev: device copy of p.u_nom when the
// caller supplied one; counter: a zeroed u32; out: [stats(4) | u_new(3T)]
// fused: the rollout reduces its own tiles (counter must be followed by
// n_wchunk zeroed group counters); ustar_global: the applied inputs are also
// written to HBM (always when k_reduce reduces)
inline void fill_desc(SolveDesc& d, const brmppi_problem& p, const Resident& c, const ScratchLayout& L, char* base,
                      uint32_t seed_offset, const float* unom_dev, uint32_t* counter, float* out, bool fused = false,
                      bool ustar_global = true) {
  std::memset(&d, 0, sizeof(d));
  d.prm = p.params ? *p.params : c.params;
  d.lambda = p.lambda;
  d.inv_lambda = 1.0f / p.lambda;
  for (int k = 0; k < 8; ++k) d.x0[k] = p.x0[k];
  d.t0 = p.t0;
  d.ds = c.ds;
  d.inv_ds = 1.0f / c.ds;
  d.S = p.S;
  d.T = p.T;
  d.n_obs = p.n_obs * n_discs(d.prm);      // obstacle rows
  d.n_objects = p.n_obs;
  d.flags = p.flags;
  d.bucket = (uint32_t)bucket_for(d.n_obs, p.flags);
  d.n_path = c.n_path;
  d.instance = p.instance;
  const uint64_t seed = p.seed + seed_offset;
  d.seed_lo = (uint32_t)(seed & 0xffffffffu);
  d.seed_hi = (uint32_t)(seed >> 32);
  d.S_pad = L.S_pad;
  d.n_wchunk = L.n_wchunk;
  d.n_rgroup = L.n_rgroup;
  d.n_ritems = L.n_wchunk * L.n_rgroup;
  d.rows_item = L.rows_item;
  d.x0_resident = (p.flags & BRMPPI_X0_RESIDENT) ? 1u : 0u;
  d.path = c.path;
  d.u_nom_in = (p.u_nom && unom_dev) ? unom_dev : c.unom;
  d.u_nom_out = c.unom;
  d.u_star = reinterpret_cast<float*>(base + L.off_ustar);
  d.J = reinterpret_cast<float*>(base + L.off_J);
  d.wpart = reinterpret_cast<float4*>(base + L.off_wpart);
  d.rpart = reinterpret_cast<float*>(base + L.off_rpart);
  d.counter = counter;
  d.n_units = L.n_units;
  d.upart = reinterpret_cast<float4*>(base + L.off_upart);
  d.urow = reinterpret_cast<float*>(base + L.off_urow);
  d.fused = fused ? 1u : 0u;
  d.ustar_global = (!fused || ustar_global) ? 1u : 0u;
  d.gctr = fused ? counter + kCtrStride : nullptr;
  d.stats = out;
  d.u_new = out + 4;
  d.plant_x = c.plant;
  d.n_normals = (p.flags & BRMPPI_GUIDANCE_OFF) ? 3u : 5u + d.n_obs;
  d.noise = L.n_normals ? reinterpret_cast<float*>(base + L.off_noise) : nullptr;
  uint32_t kind = kRowsStatic;
  for (uint32_t i = 0; i < p.n_obs; ++i) {
    const brmppi_obstacle& o = p.obs[i];
    d.obs[i] = o;
    if (o.e == 4.0f) kind = kRowsE4;
    else if ((o.vx != 0.0f || o.vy != 0.0f) && kind == kRowsStatic) kind = kRowsMoving;
  }
  d.row_kind = footprint_is_rear_axle(d.prm) ? kind : (uint32_t)kRowsDisc;
}

// An update for the launch shapes to be timed on: `bucket` ellipses at rest on
// both sides of a straight path (bucket 0: no guidance).
struct TuneUpdate {
  brmppi_problem p{};
  brmppi_obstacle obs[BRMPPI_MAX_OBS]{};
  TuneUpdate(int bucket, uint32_t S, uint32_t T, const brmppi_params& prm) {
    p.S = S;
    p.T = T;
    p.x0[2] = 1.0f;
    p.lambda = 1.0f;
    p.params = &prm;
    p.obs = obs;
    p.n_obs = (uint32_t)bucket;
    p.flags = bucket == 0 ? BRMPPI_GUIDANCE_OFF : 0u;
    for (int o = 0; o < bucket; ++o) {
      obs[o].cx = 2.0f + 1.5f * o;
      obs[o].cy = (o % 2) ? 2.5f : -2.5f;
      obs[o].mx = 0.6f;
      obs[o].my = 0.4f;
      obs[o].heading = 0.3f * o;
      obs[o].e = 2.0f;
    }
  }
  TuneUpdate(const TuneUpdate&) = delete;
  TuneUpdate& operator=(const TuneUpdate&) = delete;
};

}  // namespace brm
