// CPU check of the addresses of the digit product's record copies (csrc/bbmm_plan.h): the ring of k_mm_otf_dig is
// walked request by request, over chunk lengths, input dimensions and block widths, and every byte that a wave
// asks for has to lie in the buffer that the library allocates, also for the last chunk.
#include <cstdio>
#include <cstdlib>

#include "bbmm_plan.h"

using namespace bbmm_plan;

static long long checks = 0;

static void require(bool ok, const char* what, int KK, int ng, int nk, int k) {
  if (!ok) {
    std::fprintf(stderr, "FAILED %s: KK %d ng %d, chunk of %d records, record %d\n", what, KK, ng, nk, k);
    std::exit(1);
  }
  ++checks;
}

int main() {
  for (int KK : {1, 2, 4})
    for (int ng : {2, 4, 6, 8, 9, 12, 16})
      for (int before : {0, 2, 382})                  // records in front of the chunk
        for (int nk : {2, 4, 6, 8, 10, 64, 2046}) {
          const int ring = dig_ring(KK, ng), bytes = dig_record_bytes(KK, ng);
          const long long base = (long long)before * bytes, end = dig_buffer_bytes(before + nk, KK, ng);
          auto request = [&](int k) {
            for (int c = 0; c < dig_copies(KK, ng); ++c)
              for (int wave = 0; wave < 4; ++wave) {
                long long a = base + dig_copy_offset(KK, ng, k, nk, c) + wave * 1024;
                require(a >= base && a + 1024 <= end, "copy outside the buffer", KK, ng, nk, k);
                if (k < nk && c * 4 + wave < dig_pieces(KK, ng))
                  require(a == base + (long long)k * bytes + (c * 4 + wave) * 1024, "piece of another record", KK, ng, nk, k);
              }
          };
          for (int k = 0; k < ring - 1; ++k) request(k);           // prologue
          for (int k = 1; k < nk; ++k) request(k + ring - 2);      // step k
          require(dig_slot_bytes(KK, ng) >= bytes && dig_slot_bytes(KK, ng) * ring <= 160 * 1024, "ring", KK, ng, nk, 0);
        }
  std::printf("OK %lld checks\n", checks);
  return 0;
}
