// CPU test of the rules by which the host prepares a launch
// (paper_2508_05773_amd/csrc/launch_plan.h, brmppi_internal.h), over all the sizes that they
// accept.  Built and run by tests/test_launch_plan_host.py under AddressSanitizer +
// UndefinedBehaviorSanitizer.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "launch_plan.h"

using namespace brm;

#define CHECK(c)                                                                \
  do {                                                                          \
    if (!(c)) {                                                                 \
      std::fprintf(stderr, "CHECK failed at line %d: %s\n", __LINE__, #c);      \
      std::abort();                                                             \
    }                                                                           \
  } while (0)

// k_rollout_drawn reads the normals of step tau + 1 in every step tau, also in the
// last of a run: every such read lies inside the launch's LDS, and outside the
// epilogue's part, which other waves write meanwhile.
static void drawn_reads_in_range() {
  for (int bucket : {0, 2, 8, 16, 32}) {
    for (uint32_t T = 1; T <= kInlineSteps; ++T) {
      for (uint32_t groups = 1; groups <= 8; ++groups) {
        const size_t fused = fused_lds_bytes(kDrawnTile, T, groups);
        if (fused > kFusedLdsMax) continue;
        const DrawnLds l = drawn_lds(bucket, T, fused);
        CHECK(l.run >= 2 && l.run % 2 == 0);
        CHECK(l.bytes + kDrawnStatic <= kCuLds);
        CHECK(l.bytes >= l.epilogue + fused && l.epilogue >= l.path + sizeof(float4) * kPathWin);
        CHECK(l.path % 16 == 0 && l.epilogue % 16 == 0);
        // as the kernel walks the horizon: runs of l.run steps, the last one shorter
        for (uint32_t tau0 = 0; tau0 < T; tau0 += l.run) {
          const uint32_t end = tau0 + l.run < T ? tau0 + l.run : T;
          for (uint32_t tau = tau0; tau < end; ++tau) {
            const size_t at = (size_t)(tau + 1 - tau0) * drawn_slot(bucket);   // the slot read in step tau
            CHECK(at + drawn_slot(bucket) <= l.bytes);
            CHECK(at + drawn_slot(bucket) <= l.epilogue);
            // what a step uses was drawn in its own run
            CHECK((size_t)(tau - tau0 + 1) * drawn_slot(bucket) <= l.path);
          }
        }
      }
    }
  }
}

// a one-disc parameter set
static brmppi_params rear_axle() {
  brmppi_params P{};
  P.n_disc_tractor = 1;
  return P;
}

// The update that the launch shapes are timed on: every row that the kernels stage
// (obstacle r % n_objects around disc r / n_objects) is one that its descriptor has.
static void tune_update_rows() {
  const brmppi_params P = rear_axle();
  std::vector<char> mem(1 << 18);
  for (int bucket : {0, 2, 8, 16, 32}) {
    const TuneUpdate t(bucket, 64, 4, P);
    const ScratchLayout L = scratch_layout(64, 4, bucket ? 5 + bucket : 3);
    CHECK(L.bytes <= mem.size());
    Resident c;
    uint32_t counter[2 * kCtrStride] = {};
    float out[4 + 12], unom[12] = {};
    c.unom = unom;
    c.ds = 0.1f;
    SolveDesc d;
    fill_desc(d, t.p, c, L, mem.data(), 0, nullptr, counter, out, true, false);
    CHECK(d.n_obs == (uint32_t)bucket && d.n_objects == (uint32_t)bucket);
    CHECK(d.bucket == (uint32_t)bucket && d.row_kind == kRowsStatic);
    CHECK(d.u_nom_in == unom && d.noise && d.gctr == counter + kCtrStride);
    for (uint32_t r = 0; r < d.n_obs; ++r) {
      CHECK(r / d.n_objects < n_discs(d.prm));
      const brmppi_obstacle& o = d.obs[r % d.n_objects];
      CHECK(o.mx > 0 && o.my > 0 && (o.e == 2.0f || o.e == 4.0f));
    }
  }
}

// The default shape over its whole range: one that the bucket's kernels have, and
// not the one-lane form with precomputed normals where it spills (8 to 32 rows).
static void default_shapes() {
  for (int bucket : {0, 2, 8, 16, 32}) {
    const uint32_t K = bucket ? 5u + (uint32_t)bucket : 3u;
    for (uint32_t S = 1; S <= BRMPPI_MAX_S; S = S < 64 ? S + 1 : S + S / 9) {
      for (uint32_t T : {1u, 20u, 48u, 110u, 216u, 512u}) {
        for (int k = 0; k < 4; ++k) {
          const size_t noise = (size_t)K * T * round_up(S, 256) * sizeof(float);
          const LaunchShape s = default_shape(bucket, S, noise, k & 1, k & 2);
          CHECK(s.block == 256);
          CHECK(variant_pre(s.variant) || s.variant == variant_in_kernel(bucket));
          CHECK(bucket < 8 || s.variant != 1);
          if (S <= 8192) CHECK(s.variant == 4);
          // as few waves as to leave SIMDs idle: several lanes a sample
          if (S <= 16384 && variant_pre(s.variant)) CHECK(variant_lanes(s.variant) >= 4);
        }
      }
    }
  }
}

// k_rollout_drawn is taken only where its launch is valid, and not with more runs than
// its samples pay for.
static void drawn_rule() {
  for (int bucket : {0, 2, 8, 16, 32}) {
    for (uint32_t S = 1; S <= 9000; S += 1 + S / 7) {
      for (uint32_t T = 1; T <= BRMPPI_MAX_T; ++T) {
        size_t fused = fused_lds_bytes(kDrawnTile, T, (S + kWChunk - 1) / kWChunk);
        if (fused > kFusedLdsMax) fused = 0;
        const bool fits = drawn_fits(256, bucket, LaunchShape{256, 4}, S, T, fused);
        if (fits) CHECK(S <= 8192 && T <= kInlineSteps && drawn_lds(bucket, T, fused).runs <= 2 + S / 256);
        if (S <= 8192 && T <= 20) CHECK(fits);
        if (S > 8192 || T > kInlineSteps) CHECK(!fits);
        CHECK(!drawn_fits(256, bucket, LaunchShape{256, 3}, S, T, fused) && !drawn_fits(256, bucket, LaunchShape{64, 4}, S, T, fused));
        if (S > 4096) CHECK(!drawn_fits(128, bucket, LaunchShape{256, 4}, S, T, fused));
      }
    }
  }
  CHECK(drawn_fits(256, 32, LaunchShape{256, 4}, 8192, 162, fused_lds_bytes(kDrawnTile, 162, 8)));
  CHECK(!drawn_fits(256, 32, LaunchShape{256, 4}, 256, 162, fused_lds_bytes(kDrawnTile, 162, 1)));
}

// A served request is counted with the bytes of 64-sample tiles, and a batch of it takes no
// more of the arena at any tile size.
static void request_footprints() {
  CHECK(request_footprint(1000, 30) == 390536);   // with tiles of 64 samples
  CHECK(request_footprint(32768, 100) == 40758064);
  for (uint32_t S = 1; S <= BRMPPI_MAX_S; S = S < 64 ? S + 1 : S + S / 9) {
    for (uint32_t T = 1; T <= BRMPPI_MAX_T; T += 1 + T / 5) {
      for (uint32_t tile : {16u, 32u, 64u, 256u}) {
        const ScratchLayout L = batch_scratch(S, T, kRowsPerPass);
        size_t o = round_up(sizeof(SolveDesc), 256);                 // the parts of a batch, each aligned
        o = round_up(o + sizeof(Tile) * ((S + tile - 1) / tile), 256);
        o = round_up(o + sizeof(Item) * (size_t)L.n_wchunk * L.n_rgroup, 256);
        o = round_up(o + sizeof(float) * 3 * T, 256);
        o = round_up(o + sizeof(uint32_t), 256);
        CHECK(o + L.bytes <= request_footprint(S, T));
      }
    }
  }
}

int main() {
  drawn_reads_in_range();
  tune_update_rows();
  default_shapes();
  drawn_rule();
  request_footprints();
  std::printf("launch plan: all checks passed\n");
  return 0;
}
