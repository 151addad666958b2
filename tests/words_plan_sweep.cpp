// CPU check of the work lists of the digit-word product (csrc/bbmm_plan.h, lay_out_triangle with whole panels and bounded pieces):
// every step of every panel, the blocks on the diagonal included, is dealt out once, no piece is longer than the
// accumulators allow, every workgroup has work, and slots are in range and used once.  Row chunks of the product from whole words
// (wide_split) are no longer than the accumulators allow and few enough for their partial results.
#include <cstdio>
#include <cstdlib>
#include <set>
#include <utility>

#include "bbmm_plan.h"

using namespace bbmm_plan;

static long long checks = 0;

static void require(bool ok, const char* what, int np, int want) {
  if (!ok) {
    std::fprintf(stderr, "FAILED %s: np %d, %d workgroups\n", what, np, want);
    std::exit(1);
  }
  ++checks;
}

int main() {
  const int W = 512, kMax = 2046;
  for (int np : {1024, 1280, 1536, 2304, 5120, 9216, 10240, 20224, 50176, 100096, 200192})
    for (int want : {1, 8, 256, 304}) {
      TriHost L;
      require(lay_out_triangle(np, W, want, L, kMax, true) == nullptr, "list", np, want);
      int S = (np + W - 1) / W;
      std::set<std::pair<int, int>> seen, slots;
      require(L.wgs[0] >= 1 && L.wgs[0] <= want && L.wgs[1] == 0, "workgroups", np, want);
      for (int w = 0; w < L.wgs[0]; ++w) {
        require(L.first[0][w] < L.first[0][w + 1], "a workgroup without work", np, want);
        for (int i = L.first[0][w]; i < L.first[0][w + 1]; ++i) {
          const MmPiece& p = L.pieces[i];
          require(p.strip >= 0 && p.strip < S && p.row_begin % 16 == 0 && p.row_begin >= 0 && p.row_begin < p.row_end &&
                      p.row_end <= std::min(np, (p.strip + 1) * W) && p.row_end - p.row_begin <= 16 * kMax, "piece", np, want);
          require(p.slot >= 0 && p.slot < L.cnt[p.strip] && slots.insert({p.strip, p.slot}).second, "slot", np, want);
          for (int j = p.row_begin / 16; j < p.row_end / 16; ++j) require(seen.insert({p.strip, j}).second, "step twice", np, want);
        }
      }
      size_t steps = 0;
      for (int P = 0; P < S; ++P) {
        steps += std::min(np, (P + 1) * W) / 16;
        require(L.tot[P] == L.cnt[P] + S - 1 - P && L.tot[P] <= L.max_slots, "tot", np, want);
      }
      require(seen.size() == steps, "steps missing", np, want);
    }
  for (int np = 256; np <= 300000; np += 256)
    for (int cus : {8, 104, 256, 304}) {
      int ns = wide_split(np, cus, kMax), per = (np / 16 + ns - 1) / ns;
      require(ns >= 1 && ns <= kMaxSplit && per <= kMax, "row chunks", np, cus);
    }
  std::printf("OK %lld checks\n", checks);
  return 0;
}
