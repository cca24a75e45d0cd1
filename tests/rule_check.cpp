// Host-only checks of the tile rules (tests/test_tile_rules.py) over the shapes that the library accepts (sides up to 2^20): a
// product's partial sums fit the scratch whenever the largest tiles' do, and the choices at and around the rules' lines.  Prints
// "rules ok" and exits 0 when every check holds.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "tilerule.hpp"

using namespace qp;

static int failures = 0;
#define CHECK(c)                                                        \
  do {                                                                  \
    if (!(c)) {                                                         \
      std::fprintf(stderr, "FAIL %s:%d: %s\n", __FILE__, __LINE__, #c); \
      ++failures;                                                       \
    }                                                                   \
  } while (0)

// workgroups of the default configuration of a direct FP32 or FP64 product
static int64_t blocks(Prec p, int cfg, int64_t M, int64_t N) {
  auto up = [](int64_t x, int64_t b) { return (x + b - 1) / b; };
  if (cfg == kNarrowConfig) return up(M, 16);
  if (p == P_F64) return cfg == 6 ? up(M, 64) * up(N, 128) : up(M, 32) * up(N, 32);
  return cfg == 5 ? up(M, 64) * up(N, 64) : up(M, 32) * up(N, 32);
}

static void partials_fit() {
  std::vector<int64_t> sides = {1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 100, 127, 128, 129, 255, 256, 600, 1000, 1024, 2049, 4096,
                                8191, 16384, 24001, 40000, 65536, 100001, 262144, 524288, 1000001, 1048575, 1048576};
  for (int64_t M : sides)
    for (int64_t N : sides)
      for (int64_t K : sides) {
        for (Prec p : {P_F64, P_F32}) {
          const int cfg = default_config(p, M, N, K, K, N);
          if (blocks(p, p == P_F64 ? 6 : 5, M, N) <= kMaxPartials) CHECK(blocks(p, cfg, M, N) <= kMaxPartials);
        }
        for (Prec p : {P_F64E, P_F32E}) {
          if (!eight_takes(p, 0, M, N, K)) continue;
          const int cfg = default_config(p, M, N, K, K, N);
          CHECK(cfg >= 0 && cfg < 3 && eight_takes(p, cfg, M, N, K));
        }
      }
}

static void lines() {
  const int64_t big = 1 << 20;
  // updates whose 32 x 32 tiles would be more than the scratch holds, or whose offsets do not fit 32 bits
  CHECK(default_config(P_F32, big, 600, 600, 600, 600) == 5);
  CHECK(default_config(P_F32, big, 600, 100, 100, 600) == 5);
  CHECK(default_config(P_F32, 24001, 24001, 24001, 24001, 24001) == 5);
  CHECK(default_config(P_F64, big, 600, 600, 600, 600) == 6);
  CHECK(default_config(P_F64, 20001, 20001, 20001, 20001, 20001) == 6);
  CHECK(default_config(P_F32, 2049, 2047, 2045, 1 << 17, 2047) == 5);  // a stride of 2^17
  // off whole tiles 32 x 32 ones, whole ones as before
  CHECK(default_config(P_F32, 2049, 2047, 2045, 2045, 2047) == 6);
  CHECK(default_config(P_F64, 2049, 2047, 2045, 2045, 2047) == 1);
  CHECK(default_config(P_F32, 4096, 4096, 4096, 4096, 4096) == 5);
  CHECK(default_config(P_F64, 4096, 4096, 4096, 4096, 4096) == 6);
  CHECK(default_config(P_F32, 1024, 1024, 1024, 1024, 1024) == 6);
  // few columns
  CHECK(default_config(P_F64, 4096, 16, 4096, 4096, 16) == kNarrowConfig && default_config(P_F64, 1, 1, 1, 1, 1) == kNarrowConfig);
  CHECK(default_config(P_F64, 4097, 16, 4096, 4096, 16) == 1 && default_config(P_F64, 100000, 16, 512, 512, 16) == 1);
  CHECK(default_config(P_F32, 238, 3, 238, 238, 3) == 6 && default_config(P_F32, 100000, 16, 512, 512, 16) == 6);
  CHECK(default_config(P_F64, 4096, 17, 4096, 4096, 17) == 1);
  // FP64 off whole tiles: by rounds
  CHECK(default_config(P_F64, 4096, 4096, 4104, 4104, 4096) == 6);
  CHECK(default_config(P_F64, 4096, 4032, 4096, 4096, 4032) == 6);
  CHECK(default_config(P_F64, 4096, 2000, 2048, 2048, 2000) == 6);
  CHECK(default_config(P_F64, 4096, 4160, 4096, 4096, 4160) == 1);
  CHECK(default_config(P_F64, 4100, 4100, 4100, 4100, 4100) == 1);
  CHECK(default_config(P_F64, 3000, 3000, 3000, 3000, 3000) == 1);
  // the register tiles of FP32 end at kRegsMaxK
  CHECK(eight_takes(P_F32E, 2, 300, 300, kRegsMaxK) && !eight_takes(P_F32E, 2, 300, 300, kRegsMaxK + 1));
  CHECK(eight_takes(P_F64E, 2, 300, 300, kRegsMaxK + 1));
}

int main() {
  partials_fit();
  lines();
  if (failures == 0) std::printf("rules ok\n");
  return failures == 0 ? 0 : 1;
}
