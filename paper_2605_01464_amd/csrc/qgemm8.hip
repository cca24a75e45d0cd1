// Launches of the eight-product form (qgemm8_kern.hpp): configuration tables and the choice between them.
#include <algorithm>
#include <vector>

#include "qgemm8_kern.hpp"

namespace qp {

template <class MM, int BM, int BN, int WM, int WN, int PF, int FLUSH, int MINW>
__global__ void __launch_bounds__(64 * WM * WN, MINW) qgemm8_kernel(GemmParams<typename MM::T> P) {
  using C = Gemm8Cfg<MM, BM, BN, WM, WN>;
  __shared__ __attribute__((aligned(16))) typename MM::T smem[2 * C::STAGE];
  __shared__ double red_lds[C::NW][2];
  double s_d = 0.0, s_x = 0.0;
  int tm, tn;
  tile_of_block(blockIdx.x, P.tiles_m * P.tiles_n, P.tiles_m, P.tiles_n, tm, tn);
  gemm8_tile<MM, BM, BN, WM, WN, PF, FLUSH>(P, P.tm0 + tm, tn, smem, s_d, s_x);
  store_partials<C::NW>(P.partial, s_d, s_x, red_lds, threadIdx.x & 63, threadIdx.x >> 6, threadIdx.x);
}

template <class MM, int TM, int TN, int NWV, int PF, int MINW>
__global__ void __launch_bounds__(64 * NWV, MINW) qgemm8_regs_kernel(GemmParams<typename MM::T> P) {
  __shared__ __attribute__((aligned(16))) typename MM::T smem[NWV * 4 * 256 * TM * TN];
  __shared__ double red_lds[NWV][2];
  double s_d = 0.0, s_x = 0.0;
  int tm, tn;
  tile_of_block(blockIdx.x, P.tiles_m * P.tiles_n, P.tiles_m, P.tiles_n, tm, tn);
  gemm8_regs_tile<MM, TM, TN, NWV, PF>(P, P.tm0 + tm, tn, smem, s_d, s_x);
  store_partials<NWV>(P.partial, s_d, s_x, red_lds, threadIdx.x & 63, threadIdx.x >> 6, threadIdx.x);
}

// rows of the output that a launch computes (`first` a multiple of the tile's)
struct Rows {
  int64_t first, count;
};

template <class MM, int BM, int BN, int WM, int WN, int PF, int FLUSH, int MINW>
static int64_t launch8(const GemmParams<typename MM::T>& P0, Rows rows, hipStream_t s) {
  using C = Gemm8Cfg<MM, BM, BN, WM, WN>;
  GemmParams<typename MM::T> P = P0;
  P.tm0 = (int)(rows.first / BM);
  P.tiles_m = (int)((rows.count + BM - 1) / BM);
  P.tiles_n = (P.N + BN - 1) / BN;
  const int64_t nt = (int64_t)P.tiles_m * P.tiles_n;
  if (nt == 0) return 0;
  hipLaunchKernelGGL((qgemm8_kernel<MM, BM, BN, WM, WN, PF, FLUSH, MINW>), dim3((unsigned)nt), dim3(C::NT), 0, s, P);
  QP_HIP(hipGetLastError());
  return nt;
}

template <class MM, int TM, int TN, int NWV, int PF, int MINW>
static int64_t launch8_regs(const GemmParams<typename MM::T>& P0, Rows rows, hipStream_t s) {
  GemmParams<typename MM::T> P = P0;
  P.tm0 = (int)(rows.first / (16 * TM));
  P.tiles_m = (int)((rows.count + 16 * TM - 1) / (16 * TM));
  P.tiles_n = (P.N + 16 * TN - 1) / (16 * TN);
  const int64_t nt = (int64_t)P.tiles_m * P.tiles_n;
  if (nt == 0) return 0;
  hipLaunchKernelGGL((qgemm8_regs_kernel<MM, TM, TN, NWV, PF, MINW>), dim3((unsigned)nt), dim3(64 * NWV), 0, s, P);
  QP_HIP(hipGetLastError());
  return nt;
}

template <class T>
struct Entry8 {
  TileConfig cfg;
  int64_t (*fn)(const GemmParams<T>&, Rows, hipStream_t);
};

// Three tiles each: 64 x 64 (8 waves, one workgroup per compute unit) and 32 x 32 (4 waves, two per unit) through LDS, and
// 16 x 16 in registers (4 waves, each every fourth block of k; 131 and 92 registers, three workgroups per unit in FP64 and five
// in FP32).
static const std::vector<Entry8<double>>& f64_table8() {
  static const std::vector<Entry8<double>> t = {
      {{0, 64, 64, 8, 512, "f64x8_64x64_w2x4"}, launch8<MM16D, 64, 64, 2, 4, 2, 0, 2>},
      {{1, 32, 32, 8, 256, "f64x8_32x32_w2x2"}, launch8<MM16D, 32, 32, 2, 2, 2, 0, 2>},
      {{2, 16, 16, 8, 256, "f64x8_16x16_regs4"}, launch8_regs<MM16D, 1, 1, 4, 1, 3>},
  };
  return t;
}

// FP32 sums over k are flushed every 128 k, as in the direct form.  The register form does not flush: each wave sums a
// quarter of k, which kRegsMaxK (tilerule.hpp) keeps at 512, the 128 dependent MFMAs that the direct form's 128 k take.
static const std::vector<Entry8<float>>& f32_table8() {
  static const std::vector<Entry8<float>> t = {
      {{0, 64, 64, 16, 1024, "f32x8_64x64_w4x4"}, launch8<MM16F, 64, 64, 4, 4, 1, 128, 4>},
      {{1, 32, 32, 16, 256, "f32x8_32x32_w2x2"}, launch8<MM16F, 32, 32, 2, 2, 2, 128, 2>},
      {{2, 16, 16, 16, 256, "f32x8_16x16_regs4"}, launch8_regs<MM16F, 1, 1, 4, 1, 4>},
  };
  return t;
}

const std::vector<TileConfig>& eight_configs(Prec p) {
  auto list = [](const auto& table) {
    std::vector<TileConfig> v;
    for (auto& e : table) v.push_back(e.cfg);
    return v;
  };
  static const std::vector<TileConfig> c64 = list(f64_table8()), c32 = list(f32_table8());
  return p == P_F64E ? c64 : c32;
}

template <class T>
static int64_t launch_split(Prec p, const std::vector<Entry8<T>>& table, const GemmParams<T>& P, int cfg, hipStream_t s) {
  const Split sp = split_of(p, cfg, P.M, P.N, P.K);
  const int64_t n = table[cfg].fn(P, Rows{0, sp.rows}, s);
  if (sp.tail < 0) return n;
  GemmParams<T> Q = P;
  if (Q.partial) Q.partial += 2 * n;
  return n + table[sp.tail].fn(Q, Rows{sp.rows, P.M - sp.rows}, s);
}

// Rows on 16-byte boundaries, lane offsets within a plane that fit 32 bits, and a K from which on the form's rounding error is
// the smaller one (FP32, sequential sums, iid planes: 1.12e-7 against the direct form's 1.08e-7 at K = 8, 1.69e-7 against
// 2.09e-7 at K = 32).  And an output whose partial sums fit the scratch, at least by the largest tiles.
bool eight_fits(Prec p, const QView& A, const QView& B, int64_t M, int64_t N, int64_t K) {
  const int64_t es = p == P_F64E ? 8 : 4, va = 16 / es;
  auto al = [&](const QView& v) { return (reinterpret_cast<uintptr_t>(v.p) & 15) == 0 && v.ld % va == 0 && v.ps % va == 0; };
  return al(A) && al(B) && M * A.ld * es < (int64_t(1) << 31) && 16 * B.ld * es < (int64_t(1) << 31) && K >= 16 &&
         eight_takes(p, 0, M, N, K);
}

int64_t f64x8_launch(const GemmParams<double>& P, int cfg, hipStream_t s) { return launch_split(P_F64E, f64_table8(), P, cfg, s); }
int64_t f32x8_launch(const GemmParams<float>& P, int cfg, hipStream_t s) { return launch_split(P_F32E, f32_table8(), P, cfg, s); }

}  // namespace qp
