// Quaternion products with eight real products per quaternion product (FP64 and FP32 MFMA).
//
// The Hamilton product is a bilinear map of rank 8 (T. D. Howell & J. C. Lafon, "The complexity of the quaternion
// product", 1975).  With the eight sums of four values
//     S0..S7(x) = x3 + x1, x3 - x1, x0 - x2, x0 + x2, x3 - x2, x0 + x1, x0 - x1, x3 + x2
// of x = (a0, a1, a2, a3) on the left (L_i) and of x = (b3, b2, b0, b1) on the right (R_i),
//     P0 = L0 R0, P1 = L1 R1, P2 = L2 R3, P3 = L3 R2, P4 = L4 R6, P5 = L5 R7, P6 = L6 R5, P7 = L7 R4,
//     2 c_0 = -P0 + P1 + P2 - P3 - 2 P4,    2 c_2 = P0 + P1 - P2 - P3 + 2 P6,
//     2 c_1 = -P0 + P1 - P2 + P3 + 2 P5,    2 c_3 = P0 + P1 + P2 + P3 - 2 P7,
// so a product of matrices takes 16 M N K real operations on the matrix cores instead of 32, for 8 (M K + K N)
// additions of operand elements and 16 per output element.  Each of the eight sums over k has a quarter of the
// terms that an output plane's sum has in the direct form, at twice their size: its rounding error is about half the
// direct form's, and an output, built from five of them, ends with about 0.7 of it (iid planes, FP32, sequential sums:
// 5.8e-7 against 8.2e-7 at K = 512; from K of about 12 on it is the smaller one).  Real matrices, and complex
// ones (planes s and x), stay exactly real and complex.  What the form does not keep is the direct form's bound plane
// by plane: its error is relative to the norm of all four planes.  An infinity, too, spreads as a NaN, and sums
// overflow within a factor of two of the type's range.  The solvers use it, on operands they have checked (finite, of a
// norm far inside the range, with planes of like size: planes.hpp); products that a caller asks for by themselves keep the
// direct form.
#pragma once

#include "qgemm_kern.hpp"

namespace qp {

// sum i of four values, and the order of B's planes and sums (above)
template <class T>
__device__ __forceinline__ T sum8(int i, T x0, T x1, T x2, T x3) {
  return i == 0 ? x3 + x1 : i == 1 ? x3 - x1 : i == 2 ? x0 - x2 : i == 3 ? x0 + x2 : i == 4 ? x3 - x2 : i == 5 ? x0 + x1
         : i == 6 ? x0 - x1 : x3 + x2;
}
__device__ constexpr int b_plane(int q) { return q == 0 ? 3 : q == 1 ? 2 : q == 2 ? 0 : 1; }
__device__ constexpr int b_sum(int t) { return t < 2 ? t : t == 2 ? 3 : t == 3 ? 2 : t == 4 ? 6 : t == 5 ? 7 : t == 6 ? 5 : 4; }
// the four planes from the eight products
template <class T>
__device__ __forceinline__ void planes_of(const T (&P)[8], T (&c)[4]) {
  const T e = P[1] - P[0], f = P[2] - P[3], g = P[0] + P[1], d = P[2] + P[3];
  c[0] = T(0.5) * (e + f) - P[4];
  c[1] = T(0.5) * (e - f) + P[5];
  c[2] = T(0.5) * (g - d) + P[6];
  c[3] = T(0.5) * (g + d) - P[7];
}

// ------------------------------------------------------------------------------------------------
// Tiles staged through LDS, from operands whose rows are 16-byte aligned.  A thread loads the four planes of one 16-byte chunk
// and writes its eight sums to LDS, so the waves run eight plain products: the sums share the matrix core's FP64 unit, and
// formed here, once per staged element, they take a third of the additions that forming them per fragment takes.
//
// The K loop is one software pipeline over the products t of the steps s: the fragments of product t + PD are read behind the
// MFMAs of product t; the sums of step s + 1 are written to the other stage behind products 1..4 of step s, after which the
// loads of step s + 1 + PF go out; the one barrier of a step stands before the first read from the new stage, PD products
// before the step's end.  PF = 2 holds two steps of loads in registers: the loads behind products 5..7 alone hide about 400
// cycles, less than one takes.  Where the registers have room for it (all but the 16-wave FP32 tile, at 115 of 128): 32 x 32
// tiles at 4096^3 FP64 20.15 -> 19.3 ms, FP32 10.77 -> 10.32; 500 x 500 x 1000 108 -> 100 and 64.6 -> 61.4 us; 64 x 64 FP64 at
// 4096^3 16.98 -> 16.83 ms.
// ------------------------------------------------------------------------------------------------
template <class MM, int BM, int BN, int WM, int WN>
struct Gemm8Cfg {
  using T = typename MM::T;
  static constexpr int NW = WM * WN, NT = 64 * NW;
  static constexpr int VA = V16<T>::n, BK = VA * MM::KS;  // k of a step: one 16-byte fragment read (VA MFMAs)
  static constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 16, TN = WTN / 16;
  static constexpr int ACH = BM * BK / VA, BCH = BK * BN / VA;  // chunks of a step, A's first
  static constexpr int NC = (ACH + BCH + NT - 1) / NT;
  static constexpr int SUM = (BM + BN) * BK, STAGE = 8 * SUM;  // elements of one sum (A's rows, then B's) and of one stage
  // column chunks of 16 columns, and the number of such groups that fill the banks (256 bytes) or the row
  static constexpr int FLIP = sizeof(T), FLIPS = 16 / FLIP < BN / 16 ? 16 / FLIP : BN / 16;
  static_assert(MM::BLK == 16 && BK * sizeof(T) == 64, "a row of A's step is four chunks");
  static_assert(TM >= 1 && TN >= 1 && BM % (16 * WM) == 0 && BN % (16 * WN) == 0, "wave tile");
  static_assert(ACH % 64 == 0 && (BN & (BN - 1)) == 0, "chunks");
};

template <class MM, int BM, int BN, int WM, int WN, int PF, int FLUSH>
__device__ __forceinline__ void gemm8_tile(const GemmParams<typename MM::T>& P, int tm, int tn, typename MM::T* smem,
                                           double& s_d, double& s_x) {
  using C = Gemm8Cfg<MM, BM, BN, WM, WN>;
  using T = typename MM::T;
  using Acc = typename MM::Acc;
  using VG = typename V16<T>::nat;
  constexpr int VA = C::VA, BK = C::BK, NC = C::NC, NB = 4, PD = 2;
  static_assert(PF == 1 || PF == 2, "steps in flight");
  static_assert(FLUSH % BK == 0, "flush interval is a whole number of steps");
  const int m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w % WM, wn = w / WM;
  const int fr = MM::fr(lane), fk = MM::fk(lane);
  const int ns = (P.K + BK - 1) / BK;

  // Chunk u of a thread: c = tid + u NT, of A (row c / 4, k chunk c % 4) or of B (row k, column chunk); a wave's chunks are
  // of one operand.  Rows of A and columns of B outside the matrix are loaded from clamped addresses (what they give only
  // reaches outputs that are not written).  A load's address is a uniform base plus the lane's offset (below 2^31 bytes).
  auto is_a = [&](int u) { return w * 64 + u * C::NT < C::ACH; };
  auto active = [&](int u) { return (C::ACH + C::BCH) % C::NT == 0 || w * 64 + u * C::NT < C::ACH + C::BCH; };
  unsigned voff[NC];  // element offset of the chunk in step 0
  int kk[NC];         // the chunk's first k (A) or row (B) within a step
  int dst[NC];        // its place in a stage's first sum
#pragma unroll
  for (int u = 0; u < NC; ++u) {
    const int c = tid + u * C::NT;
    if (is_a(u)) {
      const int row = c / 4, ch = c % 4;
      kk[u] = ch * VA;
      voff[u] = (unsigned)min(m0 + row, P.M - 1) * (unsigned)P.lda + kk[u];
      dst[u] = row * BK + (ch ^ ((row >> 1) & 3)) * VA;
    } else {
      const int cb = c - C::ACH, k = cb / (BN / VA) % BK, jc = cb % (BN / VA);
      kk[u] = k;
      voff[u] = (unsigned)k * (unsigned)P.ldb + min(n0 + jc * VA, ((P.N - 1) / VA) * VA);
      dst[u] = BM * BK + k * BN + (jc ^ (k / VA % C::FLIPS * C::FLIP)) * VA;
    }
  }
  VG gs[PF][NC][4];  // the steps in flight (`load`, `mask` and `put` take the step's slot)
  auto load = [&](int s, int d) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NC; ++u) {
      if (!active(u)) continue;
      const bool a = is_a(u);
      const int sc = min(s, ns - 1);  // a step beyond the last loads the last one (and is masked)
      const T* const base = (a ? P.A : P.B) + (int64_t)sc * (a ? BK : BK * P.ldb);
      const int64_t ps = a ? P.psa : P.psb;
      unsigned v = voff[u];
      if ((sc + 1) * BK > P.K) {  // chunks (A) or rows (B) beyond the last k: the last one (`over` is at most kk)
        const int over = sc * BK + kk[u] - (a ? ((P.K - 1) / VA) * VA : P.K - 1);
        v -= (unsigned)max(over, 0) * (a ? 1u : (unsigned)P.ldb);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const char* const pl = reinterpret_cast<const char*>(base + (a ? q : b_plane(q)) * ps);
        gs[d][u][q] = gload(reinterpret_cast<const VG*>(pl + (uint32_t)(v * (unsigned)sizeof(T))), 0);
      }
    }
  };
  // elements of step s whose k lies outside the matrix become zeros
  auto mask = [&](int s, int d) __attribute__((always_inline)) {
    if ((s + 1) * BK <= P.K) return;
#pragma unroll
    for (int u = 0; u < NC; ++u)
#pragma unroll
      for (int e = 0; e < VA; ++e) {
        const bool in = s * BK + kk[u] + (is_a(u) ? e : 0) < P.K;
#pragma unroll
        for (int q = 0; q < 4; ++q) gs[d][u][q][e] = in ? gs[d][u][q][e] : T(0);
      }
  };
  // sums t and t + 1 of the loaded step
  auto put = [&](T* st, int t, int d) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < NC; ++u) {
      if (!active(u)) continue;
      const VG(&g)[4] = gs[d][u];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        VG v;
#pragma unroll
        for (int e = 0; e < VA; ++e) v[e] = sum8(t + h, g[0][e], g[1][e], g[2][e], g[3][e]);
        *reinterpret_cast<VG*>(st + dst[u] + (t + h) * C::SUM) = v;
      }
    }
  };

  Acc acc[8][C::TM][C::TN];
  constexpr int FM = FLUSH > 0 ? C::TM : 1, FN = FLUSH > 0 ? C::TN : 1;
  Acc tot[4][FM][FN];  // with a flush interval: the planes' running totals
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j)
#pragma unroll
      for (int r = 0; r < MM::NR; ++r) {
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[t][i][j][r] = T(0);
        if constexpr (FLUSH > 0)
#pragma unroll
          for (int p = 0; p < 4; ++p) tot[p][i][j][r] = T(0);
      }
  auto flush = [&]() __attribute__((always_inline)) {
    if constexpr (FLUSH > 0) {
#pragma unroll
      for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j)
#pragma unroll
          for (int r = 0; r < MM::NR; ++r) {
            T P8[8], c4[4];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
              P8[t] = acc[t][i][j][r];
              acc[t][i][j][r] = T(0);
            }
            planes_of(P8, c4);
#pragma unroll
            for (int p = 0; p < 4; ++p) tot[p][i][j][r] += c4[p];
          }
    }
  };

  // fragments: lane group fk takes k chunk fk of its row of A from one 16-byte read, and those k's rows of B
  struct Frag {
    VG a[C::TM];
    T b[C::TN][VA];
  };
  int fa[C::TM], fb[C::TN];
#pragma unroll
  for (int i = 0; i < C::TM; ++i) {
    const int row = wm * C::WTM + 16 * i + fr;
    fa[i] = row * BK + (fk ^ ((row >> 1) & 3)) * VA;
  }
#pragma unroll
  for (int j = 0; j < C::TN; ++j) {
    const int col = wn * C::WTN + 16 * j + fr;
    fb[j] = BM * BK + VA * fk * BN + ((col / VA) ^ (fk % C::FLIPS * C::FLIP)) * VA + col % VA;
  }
  Frag f[NB];
  auto read = [&](const T* st, int t) __attribute__((always_inline)) {
    Frag& x = f[t % NB];
#pragma unroll
    for (int i = 0; i < C::TM; ++i) x.a[i] = *reinterpret_cast<const VG*>(st + fa[i] + t * C::SUM);
#pragma unroll
    for (int j = 0; j < C::TN; ++j)
#pragma unroll
      for (int e = 0; e < VA; ++e) x.b[j][e] = st[fb[j] + b_sum(t) * C::SUM + e * BN];
  };

  __syncthreads();  // the caller may have used the LDS just before
  if (ns > 0) {
    load(0, 0);
    mask(0, 0);
#pragma unroll
    for (int t = 0; t < 8; t += 2) put(smem, t, 0);
#pragma unroll
    for (int d = 1; d <= PF; ++d) load(d, d % PF);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < PD; ++t) read(smem, t);
  }
  auto step = [&](int s, int h) __attribute__((always_inline)) {  // h: the step's stage
    T* const st = smem + h * C::STAGE;
    T* const nx = smem + (h ^ 1) * C::STAGE;
    const int d = (h + 1) % PF;  // the slot of step s + 1
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      if (t == 8 - PD) {
        // every wave has written its sums of step s + 1 and read its last fragments of step s
        __builtin_amdgcn_s_waitcnt(0xC07F);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
      read(t + PD < 8 ? st : nx, (t + PD) % 8);
      if (t == 0) mask(s + 1, d);
      if (t >= 1 && t <= 4) put(nx, 2 * (t - 1), d);
      if (t == 5) load(s + 1 + PF, d);
#pragma unroll
      for (int e = 0; e < VA; ++e)
#pragma unroll
        for (int i = 0; i < C::TM; ++i)
#pragma unroll
          for (int j = 0; j < C::TN; ++j) acc[t][i][j] = MM::mma(f[t % NB].a[i][e], f[t % NB].b[j][e], acc[t][i][j]);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (FLUSH > 0) {
      if (((s + 1) * BK) % FLUSH == 0 || s + 1 == ns) flush();
    }
  };
  if constexpr (PF == 1) {
    for (int s = 0; s < ns; ++s) step(s, s & 1);
  } else {  // the slots need a fixed stage per copy of the step
    for (int s = 0; s < ns; s += 2) {
      step(s, 0);
      if (s + 1 < ns) step(s + 1, 1);
    }
  }

  // ---------------------------------------------------------------- epilogue
#pragma unroll
  for (int i = 0; i < C::TM; ++i)
#pragma unroll
    for (int j = 0; j < C::TN; ++j) {
      const int rb = m0 + wm * C::WTM + i * 16, cb = n0 + wn * C::WTN + j * 16;
      T c4[MM::NR][4];
#pragma unroll
      for (int r = 0; r < MM::NR; ++r) {
        if constexpr (FLUSH > 0) {
#pragma unroll
          for (int p = 0; p < 4; ++p) c4[r][p] = tot[p][i][j][r];
        } else {
          T P8[8];
#pragma unroll
          for (int t = 0; t < 8; ++t) P8[t] = acc[t][i][j][r];
          planes_of(P8, c4[r]);
        }
      }
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        T inv[MM::NR][3];
#pragma unroll
        for (int r = 0; r < MM::NR; ++r) epilogue_inputs_overlap(P, p, rb + MM::crow(lane, r), cb + MM::ccol(lane), inv[r]);
#pragma unroll
        for (int r = 0; r < MM::NR; ++r)
          epilogue_apply(P, p, rb + MM::crow(lane, r), cb + MM::ccol(lane), c4[r][p], inv[r], s_d, s_x);
      }
    }
  __syncthreads();  // the staging LDS is reused by whatever runs next in this workgroup
}

// ------------------------------------------------------------------------------------------------
// Tiles in registers.  Small outputs leave most compute units idle under 32 x 32 tiles, and a lone workgroup per
// unit waits for its loads and barriers.  Here a workgroup owns one TM x TN group of 16 x 16 blocks and its NWV waves
// each take every NWV-th block of KB k of the whole tile: nothing is shared between waves, so operands go from global memory
// straight to registers in MFMA layout (no LDS, no barrier in the K loop), the sums are formed there, and the waves'
// planes meet once in LDS, where each thread sums its outputs in wave order and writes them.
// ------------------------------------------------------------------------------------------------
template <class MM, int TM, int TN, int NWV, int PF>
__device__ __forceinline__ void gemm8_regs_tile(const GemmParams<typename MM::T>& P, int tm, int tn, typename MM::T* smem,
                                                double& s_d, double& s_x) {
  using T = typename MM::T;
  using Acc = typename MM::Acc;
  using VG = typename V16<T>::nat;
  constexpr int VA = V16<T>::n, KB = VA * MM::KS, BM = 16 * TM, BN = 16 * TN;
  static_assert(MM::BLK == 16 && MM::NR == 4, "16 x 16 MFMA");
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = MM::fr(lane), fk = MM::fk(lane);
  const int m0 = tm * BM, n0 = tn * BN;
  Acc acc[8][TM][TN];
#pragma unroll
  for (int t = 0; t < 8; ++t)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < MM::NR; ++r) acc[t][i][j][r] = T(0);

  // Block `kb` of the wave's share starts at k = (kb NWV + w) KB.  Every load is issued, PF blocks ahead, from an address clamped
  // into the matrix: under a branch the wait for one block would be one for the blocks behind it too.  Addresses are a uniform
  // base (plane and block) and a lane offset that only the last block changes.  (Rows and columns outside the matrix only reach
  // outputs that are not written.)
  const int nb = (P.K + KB - 1) / KB, mine = (nb - w + NWV - 1) / NWV;
  unsigned ra[TM], cb[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) ra[i] = (unsigned)min(m0 + 16 * i + fr, P.M - 1) * (unsigned)P.lda;
#pragma unroll
  for (int j = 0; j < TN; ++j) cb[j] = (unsigned)min(n0 + 16 * j + fr, P.N - 1);
  T a[PF][TM][4][VA], b[PF][TN][4][VA];
  auto load = [&](int kb, int d) __attribute__((always_inline)) {
    const int k0 = min((kb * NWV + w) * KB, (nb - 1) * KB);
    unsigned ka = VA * fk, kr[VA];
#pragma unroll
    for (int e = 0; e < VA; ++e) kr[e] = VA * fk + e;
    if (k0 + KB > P.K) {
      ka = min(ka, (unsigned)(((P.K - 1) / VA) * VA - k0));
#pragma unroll
      for (int e = 0; e < VA; ++e) kr[e] = min(kr[e], (unsigned)(P.K - 1 - k0));
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const char* const pa = reinterpret_cast<const char*>(P.A + q * P.psa + k0);
      const char* const pb = reinterpret_cast<const char*>(P.B + q * P.psb + (int64_t)k0 * P.ldb);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const VG v = gload(reinterpret_cast<const VG*>(pa + (uint32_t)((ra[i] + ka) * (unsigned)sizeof(T))), 0);
#pragma unroll
        for (int e = 0; e < VA; ++e) a[d][i][q][e] = v[e];
      }
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < VA; ++e)
          b[d][j][q][e] = gload(
              reinterpret_cast<const T*>(pb + (uint32_t)((kr[e] * (unsigned)P.ldb + cb[j]) * (unsigned)sizeof(T))), 0);
    }
  };
  auto block = [&](int kb, int d) __attribute__((always_inline)) {
    const int k0 = (kb * NWV + w) * KB;
    if (k0 + KB > P.K) {  // zeros outside
#pragma unroll
      for (int e = 0; e < VA; ++e) {
        const bool in = k0 + VA * fk + e < P.K;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
          for (int i = 0; i < TM; ++i) a[d][i][q][e] = in ? a[d][i][q][e] : T(0);
#pragma unroll
          for (int j = 0; j < TN; ++j) b[d][j][q][e] = in ? b[d][j][q][e] : T(0);
        }
      }
    }
    T l[TM][VA][8], r8[TN][VA][8];
#pragma unroll
    for (int e = 0; e < VA; ++e)
#pragma unroll
      for (int t = 0; t < 8; ++t) {
#pragma unroll
        for (int i = 0; i < TM; ++i) l[i][e][t] = sum8(t, a[d][i][0][e], a[d][i][1][e], a[d][i][2][e], a[d][i][3][e]);
#pragma unroll
        for (int j = 0; j < TN; ++j)
          r8[j][e][t] = sum8(b_sum(t), b[d][j][b_plane(0)][e], b[d][j][b_plane(1)][e], b[d][j][b_plane(2)][e],
                             b[d][j][b_plane(3)][e]);
      }
    load(kb + PF, d);
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
      for (int e = 0; e < VA; ++e)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[t][i][j] = MM::mma(l[i][e][t], r8[j][e][t], acc[t][i][j]);
  };
  if (mine > 0) {
#pragma unroll
    for (int d = 0; d < PF; ++d) load(d, d);
  }
  for (int kb = 0; kb < mine; kb += PF) {
#pragma unroll
    for (int d = 0; d < PF; ++d)
      if (d == 0 || kb + d < mine) block(kb + d, d);
  }

  // each wave's planes to LDS as [wave][plane][BM][BN]
  constexpr int TILE = 4 * BM * BN;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < MM::NR; ++r) {
        T P8[8], c4[4];
#pragma unroll
        for (int t = 0; t < 8; ++t) P8[t] = acc[t][i][j][r];
        planes_of(P8, c4);
#pragma unroll
        for (int p = 0; p < 4; ++p)
          smem[w * TILE + (p * BM + 16 * i + MM::crow(lane, r)) * BN + 16 * j + MM::ccol(lane)] = c4[p];
      }
  constexpr int NT = 64 * NWV, NU = TILE / NT;
  static_assert(NU * NT == TILE, "whole outputs per thread");
  T inv[NU][3];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int e = tid + u * NT;
    epilogue_inputs_overlap(P, e / (BM * BN), m0 + (e / BN) % BM, n0 + e % BN, inv[u]);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int e = tid + u * NT;
    T v = smem[e];
#pragma unroll
    for (int g = 1; g < NWV; ++g) v += smem[g * TILE + e];
    epilogue_apply(P, e / (BM * BN), m0 + (e / BN) % BM, n0 + e % BN, v, inv[u], s_d, s_x);
  }
}

}  // namespace qp
