// Which tile configuration a product takes: rules on sizes, types and strides alone (no device code).
#pragma once

#include <cstdint>

namespace qp {

// P_BF16X3: FP32 storage, each product as three BF16 products of split operands (hi.hi + hi.lo + lo.hi)
// P_F64E, P_F32E: FP64 / FP32 with eight real products per quaternion product (qgemm8_kern.hpp); inside the solvers only
enum Prec : int { P_F64 = 0, P_F32 = 1, P_BF16 = 2, P_BF16X3 = 3, P_F64E = 4, P_F32E = 5 };

// The FP64 form for at most 16 columns (qgemm_narrow_kernel), outside the tables; its number in the product statistics
constexpr int kNarrowConfig = 63;

// It is taken while its workgroups of 16 rows are one round of the 256 compute units.  In a second round 32 x 32 tiles, one
// of which a unit still has, are faster (FP64, us: 512 x 16 x 512 75 against 88, 401 x 1 x 401 46 against 73, 4096 x 16 x 4096 567
// against 704; but 8192 x 16 x 8192 2258 against 1399, 100000 x 16 x 512 1817 against 873).
constexpr int64_t kNarrowRows = 4096;

constexpr int64_t kMaxSide = int64_t(1) << 20;  // rows and columns of a matrix that the library accepts

// Largest number of workgroups (pairs of partial sums) of a product with a reduction; the context's scratch has this room
constexpr int64_t kMaxPartials = int64_t(1) << 19;

// The register tiles of the FP32 eight-product form do not flush their sums: each of their four waves sums a quarter of k.
constexpr int64_t kRegsMaxK = 2048;

// whether kLoadElems' lane offsets in a plane of A (M rows) and a step of B (bk rows) fit 32 bits
inline bool element_offsets(int64_t M, int64_t lda, int64_t bk, int64_t ldb) {
  return M * lda < (int64_t(1) << 28) && bk * ldb < (int64_t(1) << 28);
}

// The tile that takes the least time by a model of rounds: with `cap` workgroups resident on the chip, every full round costs
// full x K microseconds and the last, partial one `part` x K if it leaves at most one workgroup per unit.  Measured, FP64 (us):
//   K = 300, 300 x 300:    64 x 64 90    32 x 32 34    16 x 16 19     (direct form 55)
//   K = 1000, 500 x 500:   64 x 64 267   32 x 32 100   16 x 16 94     (170)
//   K = 700, 700 x 700:    64 x 64 197   32 x 32 128   16 x 16 142    (208)
//   K = 1000, 1000 x 1000: 64 x 64 300   32 x 32 346   16 x 16 377    (565)
//   K = 4096, 4096 x 4096: 64 x 64 16830 32 x 32 19400                (30600; 65.3 TFLOP/s of MFMA work)
// and FP32: 300^3 48 / 22 / 12 (41), 700^3 107 / 72 / 76 (138), 1000^3 162 / 195 / 234 (320), 4096^3 8720 / 10320 (15920).
// (The register tiles' caps belong to the fit: they are two and three workgroups a unit, where three and five fit.)
struct Cost {
  int64_t tile, cap;
  double full, part, fixed;
};
inline const Cost& cost_of(Prec p, int cfg) {
  static constexpr Cost k64[3] = {{64, 256, 0.27, 0.27, 12}, {32, 512, 0.17, 0.094, 6}, {16, 512, 0.046, 0.025, 3}};
  static constexpr Cost k32[3] = {{64, 256, 0.14, 0.14, 10}, {32, 512, 0.095, 0.057, 5}, {16, 768, 0.041, 0.017, 3}};
  return (p == P_F64E ? k64 : k32)[cfg];
}
inline int64_t tiles_of(const Cost& c, int64_t M, int64_t N) { return ((M + c.tile - 1) / c.tile) * ((N + c.tile - 1) / c.tile); }
inline bool takes(Prec p, int cfg, int64_t K) { return !(p == P_F32E && cost_of(p, cfg).tile == 16 && K > kRegsMaxK); }
inline double launch_time(Prec p, int cfg, int64_t M, int64_t N, int64_t K) {
  const Cost& c = cost_of(p, cfg);
  const int64_t tiles = tiles_of(c, M, N), rest = tiles % c.cap;
  return (double)K * ((double)(tiles / c.cap) * c.full + (rest == 0 ? 0.0 : rest <= 256 ? c.part : c.full)) + c.fixed;
}

// The launches of a configuration: its own tiles over all rows, or, where the model gives less, over the rows of its full
// rounds, and smaller tiles over the rows that would be its nearly empty last round (N = M = K = 1536: 576 tiles of 64 x 64,
// 2.25 rounds of 256; the FP32 solve of 2048 x 1536, whose products these are, 19.1 -> 16.1 ms).
struct Split {
  int64_t rows;  // of the configuration's own launch
  int tail;      // configuration of the others
  double time;
};
inline Split split_of(Prec p, int cfg, int64_t M, int64_t N, int64_t K) {
  Split best{M, -1, launch_time(p, cfg, M, N, K)};
  const Cost& c = cost_of(p, cfg);
  const int64_t tn = (N + c.tile - 1) / c.tile, rounds = tiles_of(c, M, N) / c.cap;
  const int64_t rows = rounds > 0 ? rounds * c.cap / tn * c.tile : 0;
  if (rows == 0 || rows >= M) return best;
  const double own = launch_time(p, cfg, rows, N, K);
  for (int t = cfg + 1; t < 3; ++t) {
    if (!takes(p, t, K)) continue;
    const double time = own + launch_time(p, t, M - rows, N, K);
    if (time < 0.97 * best.time) best = Split{rows, t, time};
  }
  return best;
}

inline int64_t eight_blocks(Prec p, int cfg, int64_t M, int64_t N, int64_t K) {
  const Split sp = split_of(p, cfg, M, N, K);
  return tiles_of(cost_of(p, cfg), sp.rows, N) + (sp.tail < 0 ? 0 : tiles_of(cost_of(p, sp.tail), M - sp.rows, N));
}

// whether a configuration may be used for a shape: K within its limit, its partial sums within the scratch
inline bool eight_takes(Prec p, int cfg, int64_t M, int64_t N, int64_t K) {
  return takes(p, cfg, K) &&
         (((M + 15) / 16) * ((N + 15) / 16) <= kMaxPartials ||  // the smallest tiles, more than any launches together have
          eight_blocks(p, cfg, M, N, K) <= kMaxPartials);
}

inline int eight_default(Prec p, int64_t M, int64_t N, int64_t K) {
  int best = 0;
  double best_t = 0.0;
  for (int i = 0; i < 3; ++i) {
    if (!eight_takes(p, i, M, N, K)) continue;
    const double t = split_of(p, i, M, N, K).time;
    if (i == 0 || t < best_t) {
      best = i;
      best_t = t;
    }
  }
  return best;
}

// Measured on MI355X: the 64 x 64 double-buffered tiles win once there are >= 4 of them per compute unit,
// the 32 x 32 ones below that (fewer tiles leave compute units idle in the last wave); for FP64 the 64 x 128
// double-buffered tiles (8 waves of 32 x 32, twice the MFMA work per K-step barrier) beat 64 x 64 there
// (4096^3: 30.8 vs 31.3 ms; 128 x 64 with the same waves 36.6 ms).  BF16 from 1024 tiles
// of 64 x 64: the staged form with its operand tiles loaded straight into LDS; split BF16: 128 x 128 tiles
// from 256 of them (one workgroup of 16 waves per CU), 64 x 64 below.  FP32 and FP64 products of other sizes than whole
// tiles load element by element, and there the FP32 32 x 32 tiles win at every size: they keep two workgroups per unit and
// waste less at the edges (2049 x 2047 x 2045: 2.20 ms against 2.62, 4096 x 4096 x 4104: 16.24 against 16.35, 4097^3: 16.9
// against 17.3).  In FP64 the rounds decide, of 512 resident 32 x 32 tiles at 0.245 us per k or 256 of 64 x 128 at 0.93:
// 2049 x 2047 x 2045 4.39 ms against 5.82, 4096 x 4160 x 4096 32.7 against 34.8, but 4096 x 4096 x 4104 32.9 against 30.6,
// 4096 x 4032 x 4096 31.7 against 30.9, 4096 x 2000 x 2048 8.22 against 7.74.  All that holds as long as they load element by
// element, and while their partial sums fit the scratch; beyond (rows x stride from 2^28 on, more than 2^19 tiles) the
// large tiles stay.
inline int default_config(Prec p, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb) {
  if (p == P_F64E || p == P_F32E) return eight_default(p, M, N, K);
  const int64_t b64 = ((M + 63) / 64) * ((N + 63) / 64);
  const bool whole = M % 64 == 0 && N % (p == P_F64 ? 128 : 64) == 0 && K % 16 == 0;
  const bool small = ((M + 31) / 32) * ((N + 31) / 32) <= kMaxPartials && element_offsets(M, lda, 16, ldb);
  if (p == P_F64) {
    if (N <= 16 && M <= kNarrowRows) return kNarrowConfig;
    const int64_t r32 = (((M + 31) / 32) * ((N + 31) / 32) + 511) / 512, r128 = (((M + 63) / 64) * ((N + 127) / 128) + 255) / 256;
    return b64 >= 1024 && (whole || !small || 0.93 * (double)r128 <= 0.245 * (double)r32) ? 6 : 1;
  }
  if (p == P_BF16) return b64 >= 1024 ? 11 : b64 >= 256 ? 0 : 1;
  if (p == P_BF16X3) return ((M + 127) / 128) * ((N + 127) / 128) >= 256 ? 4 : 3;
  return b64 >= 1024 && (whole || !small) ? 5 : 6;
}

}  // namespace qp
