// What the host prepares for an update's launches, from plain values: the layout
// of its scratch and the descriptor that the kernels read.  No device call.
#pragma once

#include <cstring>

#include "brmppi_internal.h"
#include "served_core.h"

namespace brm {

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

inline ScratchLayout scratch_layout(uint32_t S, uint32_t T, uint32_t noise_normals = 0,
                                    uint32_t rows_item = kRowsPerPass) {
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
  o = round_up(o + (size_t)L.n_units * sizeof(float4), 256);
  L.off_urow = o;
  o = round_up(o + (size_t)L.n_units * 3 * T * sizeof(float), 256);
  L.off_out = o;
  o = round_up(o + (size_t)(4 + 3 * T) * sizeof(float), 256);
  L.off_noise = o;
  o = round_up(o + (size_t)noise_normals * T * L.S_pad * sizeof(float), 256);
  L.bytes = o;
  return L;
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
