// CPU test of the rules by which the host prepares a launch
// (paper_2508_05773_amd/csrc/brmppi_internal.h), over all the sizes that they
// accept.  Built and run by tests/test_launch_plan_host.py under AddressSanitizer +
// UndefinedBehaviorSanitizer.
#include <cstdio>
#include <cstdlib>

#include "brmppi_internal.h"

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

int main() {
  drawn_reads_in_range();
  std::printf("launch plan: all checks passed\n");
  return 0;
}
