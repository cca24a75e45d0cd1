// Quaternion GEMM kernels for gfx950 (CDNA4): FP32 and FP64 MFMA, with fused epilogues.
//
// Work decomposition
//   * one workgroup computes a BM x BN tile of all four output planes;
//   * per K-step of BK it stages the four A planes (BM x BK, stored k-major so that a fragment
//     read is 32/16 consecutive words) and the four B planes (BK x BN) in LDS, prefetching the
//     next K-step into registers while the MFMAs run on the current one;
//   * each wave owns a (BM/WM) x (BN/WN) sub-tile as MFMA blocks; for every fragment set it issues
//     the 16 signed plane products of the Hamilton product (a sign flip of an A fragment is one
//     VALU op, so the 4x-expanded real representation never exists anywhere);
//   * the epilogue applies up to three output combinations and optional reductions.
// Block ids are remapped so that the workgroups resident on one XCD (the hardware deals ids
// round-robin over the 8 XCDs) take neighbouring tiles, grouped 8 tile-rows at a time, to share
// that XCD's L2.
#include <algorithm>
#include <mutex>
#include <vector>

#include "qgemm_kern.hpp"

namespace qp {

// A workgroup computes tiles blockIdx.x, blockIdx.x + gridDim.x, ... (one tile when the grid covers
// them all).  With a grid that is a multiple of 8, every tile a workgroup visits maps to the same XCD
// range, so the XCD-aware order is kept.
// WALK = false: one tile per workgroup.  WALK = true: tiles blockIdx.x, blockIdx.x + gridDim.x, ...
// (a separate instantiation, so that the loop's live state does not raise the register count, and
// with it lower the occupancy, of the one-tile form).  With a grid that is a multiple of 8, every tile a
// workgroup visits maps to the same XCD range, so the XCD-aware order is kept.  LM (the operand load
// mode) and DB as in gemm_tile.
template <class MM, int BM, int BN, int BK, int WM, int WN, int FLUSH, bool DB, int LM, bool WALK, int MINW>
__global__ void __launch_bounds__(64 * WM * WN, MINW) qgemm_kernel(GemmParams<typename MM::T> P) {
  using C = GemmCfg<MM, BM, BN, BK, WM, WN>;
  __shared__ __attribute__((aligned(16))) typename MM::T smem[DB ? 2 * C::SMEM : C::SMEM];
  __shared__ double red_lds[C::NW][2];
  const int nt = P.tiles_m * P.tiles_n;
  double s_d = 0.0, s_x = 0.0;
  if constexpr (WALK) {
    for (int t = blockIdx.x; t < nt; t += gridDim.x) {
      int tm, tn;
      tile_of_block(t, nt, P.tiles_m, P.tiles_n, tm, tn);
      gemm_tile<MM, BM, BN, BK, WM, WN, FLUSH, LM, DB>(P, tm, tn, smem, s_d, s_x);
    }
  } else {
    int tm, tn;
    tile_of_block(blockIdx.x, nt, P.tiles_m, P.tiles_n, tm, tn);
    gemm_tile<MM, BM, BN, BK, WM, WN, FLUSH, LM, DB>(P, tm, tn, smem, s_d, s_x);
  }
  store_partials<C::NW>(P.partial, s_d, s_x, red_lds, threadIdx.x & 63, threadIdx.x >> 6, threadIdx.x);
}

// Products of at most 16 columns (a filter's output, the right-hand sides of a Krylov step).  Under 32 x 32 tiles a product of
// 238 rows is 8 workgroups whose waves each issue all 16 plane products of their K chain.  Here a workgroup has 16 rows and its
// wave p forms output plane p alone, the four plane products of each k in the same order, so the results are the 32 x 32
// configuration's bit for bit from a quarter of its MFMAs.  What bounds it is that chain of dependent MFMAs, at 95 ns each (238
// x 3 x 238) to 140 (4096 x 16 x 4096) several times the instruction's own latency: the rest goes to addresses, masks and
// signs formed for every element.  Fragments come straight from global memory, PF = 3 blocks of k ahead (6: 30 and 49 us where 3
// has 29 and 46).  238 x 3 x 238: 45 -> 29 us; 401 x 1 x 401: 74 -> 46 us.  FP64 only: in FP32 the 32 x 32 tiles, which load element
// by element there, are as fast or faster (512 x 16 x 512 46 us against 62, 8192 x 16 x 8192 676 against 1903, 238 x 3 x 238 24.5
// against 23.2).
template <class MM, int PF>
__global__ void __launch_bounds__(256, 1) qgemm_narrow_kernel(GemmParams<typename MM::T> P) {
  using T = typename MM::T;
  constexpr int VA = V16<T>::n, KB = VA * MM::KS;
  static_assert(MM::BLK == 16 && MM::NR == 4, "16 x 16 MFMA");
  __shared__ double red_lds[4][2];
  const int tid = threadIdx.x, lane = tid & 63, p = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = MM::fr(lane), fk = MM::fk(lane), m0 = blockIdx.x * 16;
  const int64_t ra = (int64_t)min(m0 + fr, P.M - 1) * P.lda;
  const int cb = min(fr, P.N - 1);
  const int nb = (P.K + KB - 1) / KB;
  // block b of KB k: plane q of A and plane p ^ q of B.  Every load is issued, from an address clamped into the matrix (no
  // branch, so that the wait for one block does not wait for those behind it); what lies outside is zeroed when used.
  T a[PF][4][VA], w[PF][4][VA];
  auto load = [&](int b, T (&av)[4][VA], T (&bv)[4][VA]) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < VA; ++e) {
      const int64_t k = min(b * KB + VA * fk + e, P.K - 1);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        av[q][e] = gload(P.A, q * P.psa + ra + k);
        bv[q][e] = gload(P.B, (p ^ q) * P.psb + k * P.ldb + cb);
      }
    }
  };
  // signs of the plane products a_q b_{p ^ q} of output plane p
  const bool n1 = p == 0 || p == 2, n2 = p == 0 || p == 3, n3 = p == 0 || p == 1;
  typename MM::Acc acc;
#pragma unroll
  for (int r = 0; r < MM::NR; ++r) acc[r] = T(0);
  const T s1 = n1 ? T(-1) : T(1), s2 = n2 ? T(-1) : T(1), s3 = n3 ? T(-1) : T(1);
  if (nb > 0) {
#pragma unroll
    for (int d = 0; d < PF; ++d) load(d, a[d], w[d]);
  }
  for (int b0 = 0; b0 < nb; b0 += PF) {
#pragma unroll
    for (int d = 0; d < PF; ++d) {
      // blocks beyond K (the last group's) multiply zeros
#pragma unroll
      for (int e = 0; e < VA; ++e) {
        const bool in = (b0 + d) * KB + VA * fk + e < P.K;
        T x[4], y[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          x[q] = in ? a[d][q][e] : T(0);
          y[q] = in ? w[d][q][e] : T(0);
        }
        acc = MM::mma(x[0], y[0], acc);
        acc = MM::mma(s1 * x[1], y[1], acc);
        acc = MM::mma(s2 * x[2], y[2], acc);
        acc = MM::mma(s3 * x[3], y[3], acc);
      }
      load(b0 + d + PF, a[d], w[d]);
    }
  }
  double s_d = 0.0, s_x = 0.0;
  T inv[MM::NR][3];
#pragma unroll
  for (int r = 0; r < MM::NR; ++r) epilogue_inputs_overlap(P, p, m0 + MM::crow(lane, r), MM::ccol(lane), inv[r]);
#pragma unroll
  for (int r = 0; r < MM::NR; ++r)
    epilogue_apply(P, p, m0 + MM::crow(lane, r), MM::ccol(lane), acc[r], inv[r], s_d, s_x);
  store_partials<4>(P.partial, s_d, s_x, red_lds, lane, p, tid);
}

namespace {
struct DevLimits {
  int cus = 0;
  int lds = 0;  // bytes of LDS per compute unit
};

DevLimits dev_limits() {
  static std::mutex mu;
  static std::vector<DevLimits> cache;
  int dev = 0;
  QP_HIP(hipGetDevice(&dev));
  std::lock_guard<std::mutex> g(mu);
  if ((int)cache.size() <= dev) cache.resize(dev + 1);
  DevLimits& d = cache[dev];
  if (d.cus == 0) {
    QP_HIP(hipDeviceGetAttribute(&d.cus, hipDeviceAttributeMultiprocessorCount, dev));
    QP_HIP(hipDeviceGetAttribute(&d.lds, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev));
  }
  return d;
}
}  // namespace

LaunchShape launch_shape(int64_t tiles, int per_cu, int occ, size_t static_lds) {
  LaunchShape ls;
  ls.grid = tiles;
  if (per_cu <= 0 || tiles == 0) return ls;
  const DevLimits d = dev_limits();
  const int c = std::max(1, std::min(per_cu, occ));
  int64_t cap = (int64_t)d.cus * c;
  if (cap >= 8) cap &= ~(int64_t)7;
  if (tiles <= cap) return ls;
  ls.grid = cap;
  // reserve LDS so that at most c workgroups fit on a compute unit (kept within the 64 KiB a
  // workgroup may take without opting in)
  if (d.lds > 0) {
    const size_t target = (size_t)((double)d.lds / (c + 0.5));
    if (target > static_lds) ls.dyn_lds = std::min<size_t>(target, 65536) - static_lds;
  }
  return ls;
}

// Deterministic sum of `count` (d, x) pairs: one workgroup, fixed strided order, fixed tree.
__global__ void __launch_bounds__(256) reduce_pairs_kernel(const double* __restrict__ partial, int64_t count,
                                                           double* __restrict__ red) {
  __shared__ double s0[256], s1[256];
  double a0 = 0.0, a1 = 0.0;
  for (int64_t i = threadIdx.x; i < count; i += 256) {
    a0 += partial[2 * i];
    a1 += partial[2 * i + 1];
  }
  s0[threadIdx.x] = a0;
  s1[threadIdx.x] = a1;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      s0[threadIdx.x] += s0[threadIdx.x + w];
      s1[threadIdx.x] += s1[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    red[0] = s0[0];
    red[1] = s1[0];
  }
}

void reduce_pairs(const double* partial, int64_t count, double* red, hipStream_t stream) {
  hipLaunchKernelGGL(reduce_pairs_kernel, dim3(1), dim3(256), 0, stream, partial, count, red);
  QP_HIP(hipGetLastError());
}

// ------------------------------------------------------------------------------------------------
// configuration table and dispatch
// ------------------------------------------------------------------------------------------------
// Resident workgroups per compute unit and static LDS bytes of a kernel (queried once).
struct KernelLimits {
  int occ = 1;
  size_t lds = 0;
};

template <class K>
static KernelLimits kernel_limits(K kern, int threads) {
  KernelLimits k;
  int occ = 0;
  QP_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, threads, 0));
  hipFuncAttributes fa{};
  QP_HIP(hipFuncGetAttributes(&fa, reinterpret_cast<const void*>(kern)));
  k.occ = std::max(occ, 1);
  k.lds = fa.sharedSizeBytes;
  return k;
}

// Launches the configuration; returns the number of workgroups (partial sums) launched.  PER_CU as
// TileConfig::per_cu.  The operand load mode is the fastest one that the shape and the views allow: kLoadElems takes any
// product that is not of whole, aligned tiles, but for offsets beyond 32 bits and the FP64 tiles that have fewer elements
// than threads (FP32, 1345 x 777 x 1001: 343 us against 533 with kLoadScalar; 1344 x 776 x 1000: 340 against 393 with
// kLoadVec, whose chunks are masked one by one; 513 x 511 x 509: 79 against 112; 500^3 47 against 65).  FP64 gains less, 1-3 %
// (1000^3 538 us against 555, 5000 x 500 x 5000 6.39 ms against 6.57), and loses 1-7 % where a unit has one workgroup to wait for
// its loads (500^3 91.2 us against 89.0, 5000 x 28 x 5000 881 against 819): kLoadVec stays for up to one tile a unit.
// MINW: waves per SIMD the register allocation must leave room for (launch bound).
template <class MM, int BM, int BN, int BK, int WM, int WN, int FLUSH, bool DB, int MINW, bool WALK, int LM>
static void launch_mode(const GemmParams<typename MM::T>& P, int64_t grid, size_t dyn_lds, hipStream_t s) {
  using C = GemmCfg<MM, BM, BN, BK, WM, WN>;
  hipLaunchKernelGGL((qgemm_kernel<MM, BM, BN, BK, WM, WN, FLUSH, DB, LM, WALK, MINW>), dim3((unsigned)grid), dim3(C::NT),
                     dyn_lds, s, P);
}

template <class MM, int BM, int BN, int BK, int WM, int WN, int FLUSH, bool DB, int MINW, bool WALK>
static void launch_any_mode(const GemmParams<typename MM::T>& P, int64_t grid, size_t dyn_lds, hipStream_t s) {
  using C = GemmCfg<MM, BM, BN, BK, WM, WN>;
  constexpr bool ELEMS = BM * BK % C::NT == 0 && BK * BN % C::NT == 0;
  if (P.vec && P.M % BM == 0 && P.N % BN == 0 && P.K % BK == 0)
    launch_mode<MM, BM, BN, BK, WM, WN, FLUSH, DB, MINW, WALK, kLoadAligned>(P, grid, dyn_lds, s);
  else if (ELEMS && element_offsets(P.M, P.lda, BK, P.ldb) && !(sizeof(typename MM::T) == 8 && P.vec && grid <= 256))
    launch_mode<MM, BM, BN, BK, WM, WN, FLUSH, DB, MINW, WALK, ELEMS ? kLoadElems : kLoadScalar>(P, grid, dyn_lds, s);
  else if (P.vec)
    launch_mode<MM, BM, BN, BK, WM, WN, FLUSH, DB, MINW, WALK, kLoadVec>(P, grid, dyn_lds, s);
  else
    launch_mode<MM, BM, BN, BK, WM, WN, FLUSH, DB, MINW, WALK, kLoadScalar>(P, grid, dyn_lds, s);
  QP_HIP(hipGetLastError());
}

template <class MM, int BM, int BN, int BK, int WM, int WN, int FLUSH, bool DB, int PER_CU, int MINW = 1>
static int64_t launch_cfg(const GemmParams<typename MM::T>& P0, hipStream_t s) {
  using C = GemmCfg<MM, BM, BN, BK, WM, WN>;
  GemmParams<typename MM::T> P = P0;
  P.tiles_m = (P.M + BM - 1) / BM;
  P.tiles_n = (P.N + BN - 1) / BN;
  const int64_t nt = (int64_t)P.tiles_m * P.tiles_n;
  if (nt == 0) return 0;
  if constexpr (PER_CU > 0) {
    static const KernelLimits kl =
        kernel_limits(qgemm_kernel<MM, BM, BN, BK, WM, WN, FLUSH, DB, kLoadAligned, true, MINW>, C::NT);
    const LaunchShape ls = launch_shape(nt, PER_CU, kl.occ, kl.lds);
    if (ls.grid < nt) {
      launch_any_mode<MM, BM, BN, BK, WM, WN, FLUSH, DB, MINW, true>(P, ls.grid, ls.dyn_lds, s);
      return ls.grid;
    }
  }
  launch_any_mode<MM, BM, BN, BK, WM, WN, FLUSH, DB, MINW, false>(P, nt, 0, s);
  return nt;
}

using F32Launch = int64_t (*)(const GemmParams<float>&, hipStream_t);
using F64Launch = int64_t (*)(const GemmParams<double>&, hipStream_t);

struct F32Entry {
  TileConfig cfg;
  F32Launch fn;
};
struct F64Entry {
  TileConfig cfg;
  F64Launch fn;
};

// FP32 configurations accumulate in two levels (flush every 128 k); FP64 needs no flush.
// "_db": double-buffered LDS staging; "_cuC": C workgroups per compute unit walking the tiles.
static const std::vector<F32Entry>& f32_table() {
  static const std::vector<F32Entry> t = {
      {{0, 64, 64, 16, 256, "f32_64x64x16_w2x2_mfma32"}, launch_cfg<MM32F, 64, 64, 16, 2, 2, 128, false, 0>},
      {{1, 32, 32, 16, 256, "f32_32x32x16_w2x2_mfma16"}, launch_cfg<MM16F, 32, 32, 16, 2, 2, 128, false, 0>},
      {{2, 128, 64, 16, 256, "f32_128x64x16_w2x2_mfma32"}, launch_cfg<MM32F, 128, 64, 16, 2, 2, 128, false, 0>},
      {{3, 64, 128, 16, 256, "f32_64x128x16_w2x2_mfma32"}, launch_cfg<MM32F, 64, 128, 16, 2, 2, 128, false, 0>},
      {{4, 64, 64, 16, 256, "f32_64x64x16_w2x2_mfma16"}, launch_cfg<MM16F, 64, 64, 16, 2, 2, 128, false, 0>},
      {{5, 64, 64, 16, 256, "f32_64x64x16_w2x2_mfma32_db"}, launch_cfg<MM32F, 64, 64, 16, 2, 2, 128, true, 0>},
      {{6, 32, 32, 16, 256, "f32_32x32x16_w2x2_mfma16_db"}, launch_cfg<MM16F, 32, 32, 16, 2, 2, 128, true, 0>},
      {{7, 64, 64, 16, 1024, "f32_64x64x16_w4x4_mfma16_db"}, launch_cfg<MM16F, 64, 64, 16, 4, 4, 128, true, 0>},
      {{8, 32, 32, 16, 256, "f32_32x32x16_w2x2_mfma16_db_cu3", 3}, launch_cfg<MM16F, 32, 32, 16, 2, 2, 128, true, 3>},
  };
  return t;
}

static const std::vector<F64Entry>& f64_table() {
  static const std::vector<F64Entry> t = {
      {{0, 64, 64, 8, 256, "f64_64x64x8_w2x2_mfma16"}, launch_cfg<MM16D, 64, 64, 8, 2, 2, 0, false, 0>},
      {{1, 32, 32, 16, 256, "f64_32x32x16_w2x2_mfma16"}, launch_cfg<MM16D, 32, 32, 16, 2, 2, 0, false, 0>},
      {{2, 64, 64, 8, 1024, "f64_64x64x8_w4x4_mfma16"}, launch_cfg<MM16D, 64, 64, 8, 4, 4, 0, false, 0>},
      {{3, 32, 32, 16, 256, "f64_32x32x16_w2x2_mfma16_db"}, launch_cfg<MM16D, 32, 32, 16, 2, 2, 0, true, 0>},
      {{4, 64, 64, 8, 1024, "f64_64x64x8_w4x4_mfma16_db"}, launch_cfg<MM16D, 64, 64, 8, 4, 4, 0, true, 0>},
      {{5, 128, 64, 8, 512, "f64_128x64x8_w4x2_mfma16_db"}, launch_cfg<MM16D, 128, 64, 8, 4, 2, 0, true, 0>},
      {{6, 64, 128, 8, 512, "f64_64x128x8_w2x4_mfma16_db"}, launch_cfg<MM16D, 64, 128, 8, 2, 4, 0, true, 0>},
  };
  return t;
}

const std::vector<TileConfig>& bf16_configs();    // qgemm_bf16.hip
const std::vector<TileConfig>& bf16x3_configs();  // qgemm_bf16.hip
const std::vector<TileConfig>& eight_configs(Prec p);  // qgemm8.hip

const std::vector<TileConfig>& tile_configs(Prec p) {
  static std::vector<TileConfig> f32, f64;
  if (f32.empty()) {
    for (auto& e : f32_table()) f32.push_back(e.cfg);
    for (auto& e : f64_table()) f64.push_back(e.cfg);
  }
  if (p == P_BF16) return bf16_configs();
  if (p == P_BF16X3) return bf16x3_configs();
  if (p == P_F64E || p == P_F32E) return eight_configs(p);
  return p == P_F64 ? f64 : f32;
}

static int64_t blocks_for(const TileConfig& c, int64_t M, int64_t N) {
  return ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
}

int64_t qgemm_blocks(Prec p, int cfg, int64_t M, int64_t N) {
  const auto& t = tile_configs(p);
  return blocks_for(t.at(cfg), M, N);
}

template <class T>
static GemmParams<T> make_params(const QView& A, const QView& B, int64_t M, int64_t N, int64_t K,
                                 const Epilogue& e, double* partial) {
  GemmParams<T> P{};
  P.A = static_cast<const T*>(A.p);
  P.lda = A.ld;
  P.psa = A.ps;
  P.B = static_cast<const T*>(B.p);
  P.ldb = B.ld;
  P.psb = B.ps;
  P.M = (int)M;
  P.N = (int)N;
  P.K = (int)K;
  P.nout = e.nout;
  P.nin = e.nin;
  P.ref = e.ref;
  constexpr int VA = V16<T>::n;
  auto al = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  P.vec = al(A.p) && al(B.p) && A.ld % VA == 0 && B.ld % VA == 0 && A.ps % VA == 0 && B.ps % VA == 0;
  for (int t = 0; t < 3; ++t) {
    P.out[t] = t < e.nout ? static_cast<T*>(e.out[t].p) : nullptr;
    P.ldo[t] = e.out[t].ld;
    P.pso[t] = e.out[t].ps;
    P.in[t] = t < e.nin ? static_cast<const T*>(e.in[t].p) : nullptr;
    P.ldi[t] = e.in[t].ld;
    P.psi[t] = e.in[t].ps;
    P.ca[t] = (T)e.a[t];
    P.cg[t] = (T)e.g[t];
    for (int u = 0; u < 3; ++u) P.cb[t][u] = (T)e.b[t][u];
  }
  P.partial = e.reduce ? partial : nullptr;
  P.reduce = e.reduce ? 1 : 0;
  return P;
}

int64_t bf16_launch(const GemmParams<float>& P, int cfg, hipStream_t s, GemmScratch& scratch);  // qgemm_bf16.hip
int64_t bf16_blocks(int cfg, int64_t M, int64_t N);
int64_t bf16x3_launch(const GemmParams<float>& P, int cfg, hipStream_t s, GemmScratch& scratch);
int64_t bf16x3_blocks(int cfg, int64_t M, int64_t N);
int64_t f64x8_launch(const GemmParams<double>& P, int cfg, hipStream_t s);  // qgemm8.hip
int64_t f32x8_launch(const GemmParams<float>& P, int cfg, hipStream_t s);

// an upper bound of the workgroups a configuration launches (a per-CU configuration launches at most this many)
static int64_t config_blocks(Prec p, int cfg, int64_t M, int64_t N, int64_t K) {
  if (cfg == kNarrowConfig) return (M + 15) / 16;
  if (p == P_BF16) return bf16_blocks(cfg, M, N);
  if (p == P_BF16X3) return bf16x3_blocks(cfg, M, N);
  if (p == P_F64E || p == P_F32E) return eight_blocks(p, cfg, M, N, K);
  return blocks_for(tile_configs(p)[cfg], M, N);
}

const char* config_name(Prec p, int cfg) {
  if (cfg == kNarrowConfig && p == P_F64) return "f64_16x16_narrow";
  const auto& t = tile_configs(p);
  return cfg >= 0 && cfg < (int)t.size() ? t[cfg].name : "";
}

bool config_takes(Prec p, int cfg, int64_t M, int64_t N, int64_t K) {
  if (cfg == kNarrowConfig && (N > 16 || p != P_F64)) return false;
  if (p == P_F64E || p == P_F32E) return eight_takes(p, cfg, M, N, K);
  return config_blocks(p, cfg, M, N, K) <= kMaxPartials;
}

void qgemm(Prec p, const QView& A, const QView& B, int64_t M, int64_t N, int64_t K, const Epilogue& epi,
           double* red, GemmScratch& scratch, hipStream_t stream, int cfg) {
  if (M < 0 || N < 0 || K < 0) throw Error(-1, "qgemm: negative size");
  if (epi.nout < 1 || epi.nout > 3 || epi.nin < 0 || epi.nin > 3) throw Error(-1, "qgemm: bad epilogue");
  if (epi.reduce && (!red || epi.ref >= epi.nin)) throw Error(-1, "qgemm: bad reduction");
  if (cfg < 0) cfg = default_config(p, M, N, K, A.ld, B.ld);
  const auto& cfgs = tile_configs(p);
  const bool narrow = cfg == kNarrowConfig && p == P_F64 && N <= 16;
  if (cfg >= (int)cfgs.size() && !narrow) throw Error(-1, "qgemm: bad tile config");
  if (epi.reduce && config_blocks(p, cfg, M, N, K) > scratch.capacity / 2) throw Error(-1, "qgemm: reduction scratch too small");
  double* partial = epi.reduce ? scratch.partial : nullptr;
  int64_t launched = 0;
  if ((p == P_F64E || p == P_F32E) && !(eight_fits(p, A, B, M, N, K) && eight_takes(p, cfg, M, N, K))) throw Error(-1, "qgemm: operands of the eight-product form");
  if (narrow) {
    launched = M == 0 || N == 0 ? 0 : (M + 15) / 16;
    if (launched > 0) {
      hipLaunchKernelGGL((qgemm_narrow_kernel<MM16D, 3>), dim3((unsigned)launched), dim3(256), 0, stream,
                         make_params<double>(A, B, M, N, K, epi, partial));
      QP_HIP(hipGetLastError());
    }
  } else if (p == P_F64E) {
    launched = f64x8_launch(make_params<double>(A, B, M, N, K, epi, partial), cfg, stream);
  } else if (p == P_F32E) {
    launched = f32x8_launch(make_params<float>(A, B, M, N, K, epi, partial), cfg, stream);
  } else if (p == P_F64) {
    launched = f64_table()[cfg].fn(make_params<double>(A, B, M, N, K, epi, partial), stream);
  } else if (p == P_F32) {
    launched = f32_table()[cfg].fn(make_params<float>(A, B, M, N, K, epi, partial), stream);
  } else if (p == P_BF16) {
    launched = bf16_launch(make_params<float>(A, B, M, N, K, epi, partial), cfg, stream, scratch);
  } else {
    launched = bf16x3_launch(make_params<float>(A, B, M, N, K, epi, partial), cfg, stream, scratch);
  }
  if (epi.reduce) reduce_pairs(partial, launched, red, stream);
}

}  // namespace qp
