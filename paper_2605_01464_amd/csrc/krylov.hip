// Global quaternion FOM / GMRES.  The Krylov basis V_0, V_1, ... of n x m quaternion matrices is
// orthonormal in <X, Y> = Re tr(X^H Y), which is the real dot product of the four stacked planes, so
// every basis operation is a dense real vector operation over L = 4 n m doubles: the basis lives in one
// device array [k][4][n][m] (each V_j also a quaternion-matrix view for the products), the projections
// are one dot kernel over all previous V_i and one fused multi-axpy (classical Gram-Schmidt, applied
// twice), and only the small Hessenberg matrix and its Givens rotations are handled on the host.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <vector>

#include "krylov.hpp"

namespace qp {

namespace {

// out[i] = <V_i, W> for i < nvec (one workgroup per i, fixed-order reduction)
__global__ void __launch_bounds__(256) dots_kernel(const double* __restrict__ V, int64_t L, const double* __restrict__ W,
                                                   int nvec, double* __restrict__ out) {
  __shared__ double red[256];
  const int i = blockIdx.x;
  if (i >= nvec) return;
  const double* v = V + (int64_t)i * L;
  double acc = 0.0;
  for (int64_t e = threadIdx.x; e < L; e += 256) acc += v[e] * W[e];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[i] = red[0];
}

// W[e] += sign * sum_i h[i] V_i[e]   (i < nvec, in index order).
//
// The sum of an element is one chain of nvec multiply-adds, whose order fixes the result: its length (1000 steps of a Krylov
// run: 4 us) is the floor, and with one thread per element fetching its own operands every step waited for memory (118 us on
// average at L = 2856 and 1088 steps).  Here a workgroup has 16 elements: its 256 threads fetch CH vectors' 128-byte
// pieces at a time, a chunk ahead, into LDS, and 16 lanes run the chains from there (average 118 -> 10 us).
// Vectors of more than kChunked elements have enough threads with one element each, in the same order (below).
constexpr int64_t kChunked = 16384;
constexpr int AX_E = 16, AX_CH = 128, AX_U = AX_CH * AX_E / 256;
__global__ void __launch_bounds__(256) multi_axpy_kernel(const double* __restrict__ V, int64_t L,
                                                         const double* __restrict__ h, int nvec, double sign,
                                                         double* __restrict__ W) {
  __shared__ double vs[2][AX_CH * AX_E], hs[2][AX_CH];
  const int tid = threadIdx.x;
  const int64_t e0 = (int64_t)blockIdx.x * AX_E;
  const int64_t e = min(e0 + (tid % AX_E), L - 1);
  double r[AX_U], rh = 0.0;
  auto load = [&](int i0) {
#pragma unroll
    for (int u = 0; u < AX_U; ++u) r[u] = V[(int64_t)min(i0 + tid / AX_E + u * (256 / AX_E), nvec - 1) * L + e];
    if (tid < AX_CH) rh = h[min(i0 + tid, nvec - 1)];
  };
  auto store = [&](int b) {
#pragma unroll
    for (int u = 0; u < AX_U; ++u) vs[b][tid + u * 256] = r[u];
    if (tid < AX_CH) hs[b][tid] = rh;
  };
  double acc = 0.0;
  if (nvec > 0) {
    load(0);
    store(0);
  }
  __syncthreads();
  for (int i0 = 0, b = 0; i0 < nvec; i0 += AX_CH, b ^= 1) {
    const bool more = i0 + AX_CH < nvec;
    if (more) load(i0 + AX_CH);
    if (tid < AX_E) {
      const int n = min(AX_CH, nvec - i0);
      const double* v = vs[b] + tid;
      int i = 0;
      for (; i + 16 <= n; i += 16) {
        double x[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) x[u] = v[(i + u) * AX_E];
#pragma unroll
        for (int u = 0; u < 16; ++u) acc = fma(hs[b][i + u], x[u], acc);
      }
      for (; i < n; ++i) acc = fma(hs[b][i], v[i * AX_E], acc);
    }
    if (more) store(b ^ 1);  // last read two chunks ago, behind a barrier
    __syncthreads();
  }
  if (tid < AX_E && e0 + tid < L) W[e0 + tid] = fma(sign, acc, W[e0 + tid]);
}

// The same with one element a thread, U vectors' loads in flight.  What bounds it is memory, where a chunk's 128 rows of the kernel
// above are loaded for 16 elements however few vectors there are (us, chunks against this; L = 16384: 3.2 against 2.7 at 1 vector,
// 24.8 against 48 at 1000; L = 32768: 4.4 / 2.7 and 47 / 52; L = 262144: 22 / 2.7 and 492 / 331; L = 1048576: 80 / 4.3 and 666 /
// 440 at 300).  U = 8 hides the latency of fewer elements (L = 65536: 89 us at 1000 vectors, 234 with U = 2), U = 2 keeps more pages
// open from 2^18 on (L = 1048576: 176 us at 128 vectors, 212 with U = 8).
constexpr int64_t kLongVector = int64_t(1) << 18;
template <int U>
__global__ void __launch_bounds__(256) multi_axpy_long_kernel(const double* __restrict__ V, int64_t L,
                                                              const double* __restrict__ h, int nvec, double sign,
                                                              double* __restrict__ W) {
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < L; e += (int64_t)gridDim.x * 256) {
    double acc = 0.0;
#pragma unroll U
    for (int i = 0; i < nvec; ++i) acc = fma(h[i], V[(int64_t)i * L + e], acc);
    W[e] = fma(sign, acc, W[e]);
  }
}

// hn[0] = ||W||_F^2 in dots_kernel's order, Y = W / ||W||_F, and the step's 2 nvec projections and hn to `host` (pinned).
// Every workgroup forms the norm for itself (the vector is at most kFusedNorm doubles long).
constexpr int64_t kFusedNorm = 16384;
__global__ void __launch_bounds__(256) norm_scale_kernel(const double* __restrict__ W, int64_t L, const double* __restrict__ h,
                                                         int nh, double* __restrict__ host, double* __restrict__ Y) {
  __shared__ double red[256];
  double acc = 0.0;
  for (int64_t e = threadIdx.x; e < L; e += 256) acc += W[e] * W[e];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  const double n2 = red[0];
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < nh; i += 256) host[i] = h[i];
    if (threadIdx.x == 0) host[nh] = n2;
  }
  const double a = 1.0 / sqrt(n2);
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < L; e += (int64_t)gridDim.x * 256) Y[e] = a * W[e];
}

// The same from a norm formed by dots_kernel (longer vectors).
__global__ void __launch_bounds__(256) scale_by_norm_kernel(const double* __restrict__ W, int64_t L, const double* __restrict__ h,
                                                            int nh, double* __restrict__ host, double* __restrict__ Y) {
  const double n2 = h[nh];
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i <= nh; i += 256) host[i] = h[i];
  const double a = 1.0 / sqrt(n2);
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < L; e += (int64_t)gridDim.x * 256) Y[e] = a * W[e];
}

// Y = a X
__global__ void __launch_bounds__(256) scale_kernel(const double* __restrict__ X, int64_t L, double a,
                                                    double* __restrict__ Y) {
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < L; e += (int64_t)gridDim.x * 256) Y[e] = a * X[e];
}

unsigned blocks_for(int64_t L) { return (unsigned)std::min<int64_t>((L + 255) / 256, 2048); }

void multi_axpy(const double* V, int64_t L, const double* h, int nvec, double sign, double* W, hipStream_t s) {
  if (L <= kChunked)
    hipLaunchKernelGGL(multi_axpy_kernel, dim3((unsigned)((L + AX_E - 1) / AX_E)), dim3(256), 0, s, V, L, h, nvec, sign, W);
  else if (L < kLongVector)
    hipLaunchKernelGGL(multi_axpy_long_kernel<8>, dim3(blocks_for(L)), dim3(256), 0, s, V, L, h, nvec, sign, W);
  else
    hipLaunchKernelGGL(multi_axpy_long_kernel<2>, dim3(blocks_for(L)), dim3(256), 0, s, V, L, h, nvec, sign, W);
  QP_HIP(hipGetLastError());
}

// The context's pinned columns, grown on demand, and events.
double* krylov_columns(Ctx& c, size_t doubles, int events) {
  if (c.krylov_cap < doubles) {
    if (c.krylov_buf) (void)hipHostFree(c.krylov_buf);
    c.krylov_buf = nullptr;
    c.krylov_cap = 0;
    if (hipHostMalloc(&c.krylov_buf, sizeof(double) * doubles, hipHostMallocDefault) != hipSuccess) {
      (void)hipGetLastError();
      c.krylov_buf = nullptr;
      throw Error(QPINV_ENOMEM, "krylov: pinned allocation of " + std::to_string(sizeof(double) * doubles) + " bytes failed");
    }
    c.krylov_cap = doubles;
  }
  while ((int)c.krylov_events.size() < events) {
    hipEvent_t e;
    QP_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    c.krylov_events.push_back(e);
  }
  return c.krylov_buf;
}

// a dense n x m view of slot j of the basis array
Mat slot(double* base, int64_t j, int64_t n, int64_t m) {
  Mat v;
  v.v.p = base + j * 4 * n * m;
  v.v.rows = n;
  v.v.cols = m;
  v.v.ld = m;
  v.v.ps = n * m;
  v.rows = n;
  v.cols = m;
  v.dtype = QPINV_F64;
  return v;
}

// C = A B + beta * In (FP64 product)
void product(Ctx& c, const Mat& A, const Mat& B, const Mat& C, hipStream_t s, const Mat* In = nullptr,
             double a = 1.0, double beta = 0.0) {
  Epilogue e;
  e.nout = 1;
  e.out[0] = C.v;
  e.a[0] = a;
  if (In) {
    e.nin = 1;
    e.in[0] = In->v;
    e.b[0][0] = beta;
  }
  gemm(c, P_F64, A, B, e, s);
}

}  // namespace

KrylovResult gl_krylov(Ctx& c, int method, const Mat& A, const Mat& B, const Mat* M, const Mat& X, double tol,
                       int max_iter, double* history, int history_cap, hipStream_t s) {
  const int64_t n = A.rows, m = B.cols, L = 4 * n * m;
  KrylovResult res;
  // device work: basis (max_iter + 1 slots), the product temporaries, residual, projections
  double* V = static_cast<double*>(c.ws.get("krylov_basis", sizeof(double) * (size_t)(L * (max_iter + 1))));
  double* T = static_cast<double*>(c.ws.get("krylov_tmp", sizeof(double) * (size_t)(4 * L)));
  double* dh = static_cast<double*>(c.ws.get("krylov_h", sizeof(double) * (size_t)(2 * (max_iter + 2) + 1)));
  const Mat W = slot(T, 0, n, m), AV = slot(T, 1, n, m), R0 = slot(T, 2, n, m), Xt = slot(T, 3, n, m);
  std::vector<double> hh(2 * (max_iter + 2) + 1);
  auto fetch = [&](int count) {
    QP_HIP(hipMemcpyAsync(hh.data(), dh, sizeof(double) * count, hipMemcpyDeviceToHost, s));
    QP_HIP(hipStreamSynchronize(s));
  };
  auto dot_self = [&](const double* x) {
    hipLaunchKernelGGL(dots_kernel, dim3(1), dim3(256), 0, s, x, L, x, 1, dh);
    QP_HIP(hipGetLastError());
    fetch(1);
    return hh[0];
  };

  // R_0 = B - A X_0 and the initial residual of the iterated system Z_0 = M R_0 (or R_0)
  product(c, A, X, R0, s, &B, -1.0, 1.0);
  const double r0 = std::sqrt(dot_self(static_cast<double*>(R0.v.p)));
  const Mat Z0 = M ? W : R0;
  if (M) product(c, *M, R0, W, s);
  const double beta = M ? std::sqrt(dot_self(static_cast<double*>(W.v.p))) : r0;
  if (beta == 0.0) {
    res.true_rr = 0.0;
    return res;
  }
  hipLaunchKernelGGL(scale_kernel, dim3(blocks_for(L)), dim3(256), 0, s, static_cast<const double*>(Z0.v.p), L,
                     1.0 / beta, V);
  QP_HIP(hipGetLastError());

  // Hessenberg columns (host), Givens rotations, rotated right-hand side
  std::vector<std::vector<double>> H;  // H[j] = column j (rotated: R's column), length j + 2
  std::vector<double> cs, sn, g(1, beta);
  int k = 0;
  // coefficients y of X_k = X_0 + sum_i y_i V_i after k steps
  auto coefficients = [&](int kk) {
    // back substitution column by column (H[l] is contiguous)
    std::vector<double> y(g.begin(), g.begin() + kk);
    // GMRES: upper-triangular R y = g (the rotated Hessenberg).  FOM: H_k y = beta e_1; the first k - 1 rotations bring the
    // square Hessenberg to R with its last diagonal entry taken before the last rotation (c rho), and beta e_1 to g with its
    // last entry taken before the last rotation (g / c).
    const double c_last = method == 1 ? 1.0 : cs[kk - 1];
    for (int l = kk - 1; l >= 0; --l) {
      y[l] = l == kk - 1 ? (y[l] / c_last) / (c_last * H[l][l]) : y[l] / H[l][l];
      for (int i = 0; i < l; ++i) y[i] -= H[l][i] * y[l];
    }
    return y;
  };
  // Xdst = X_0 + sum_i y_i V_i (X holds X_0 until the end)
  auto form = [&](int kk, const Mat& Xdst) {
    const std::vector<double> y = coefficients(kk);
    QP_HIP(hipMemcpyAsync(dh, y.data(), sizeof(double) * kk, hipMemcpyHostToDevice, s));
    if (Xdst.v.p != X.v.p)
      QP_HIP(hipMemcpyAsync(Xdst.v.p, X.v.p, sizeof(double) * (size_t)L, hipMemcpyDeviceToDevice, s));
    multi_axpy(V, L, dh, kk, 1.0, static_cast<double*>(Xdst.v.p), s);
    QP_HIP(hipStreamSynchronize(s));  // y (host) is read by the copy
  };
  // RR = ||B - A Xs||_F / ||B - A X_0||_F
  auto true_residual = [&](const Mat& Xs) {
    product(c, A, Xs, AV, s, &B, -1.0, 1.0);
    return std::sqrt(dot_self(static_cast<double*>(AV.v.p))) / r0;
  };
  // Step j on the stream: W = A V_j (or M A V_j), classical Gram-Schmidt twice (h = V^T W, W -= V h), V_{j+1} = W / ||W||.
  // Nothing in it waits for the host, which reads the new Hessenberg column from pinned memory up to kAhead steps behind: the
  // rotations and the stopping test of one step run while the next ones do.  The steps in flight at the end are dropped (they
  // touch only W, AV and basis slots that X does not use), so they are as many as the run is long enough for: kAheadTime of them
  // for every step done, a third of a step at 238 x 3 (66 us) and a fortieth of one of a millisecond, whose host part is nothing.
  // (Five steps at 238 x 3 take 469 us with none in flight and 436 with three from the start; a preconditioned run that ends after
  // one step at 4096 x 16 takes 5.5 ms, and 12.1 with three from the start.)
  constexpr int kAhead = 3, kRing = kAhead + 1;
  constexpr double kAheadTime = 25e-6;
  const int64_t ring = 2 * (int64_t)max_iter + 1;
  double* const columns = krylov_columns(c, (size_t)(ring * kRing), kRing);
  auto enqueue = [&](int j) {
    const Mat Vj = slot(V, j, n, m);
    if (M) {
      product(c, A, Vj, AV, s);
      product(c, *M, AV, W, s);
    } else {
      product(c, A, Vj, W, s);
    }
    double* w = static_cast<double*>(W.v.p);
    for (int pass = 0; pass < 2; ++pass) {
      double* hp = dh + pass * (j + 1);
      hipLaunchKernelGGL(dots_kernel, dim3(j + 1), dim3(256), 0, s, V, L, w, j + 1, hp);
      QP_HIP(hipGetLastError());
      multi_axpy(V, L, hp, j + 1, -1.0, w, s);
    }
    double* host = columns + (j % kRing) * ring;
    double* next = V + (int64_t)(j + 1) * L;
    if (L <= kFusedNorm) {
      hipLaunchKernelGGL(norm_scale_kernel, dim3(blocks_for(L)), dim3(256), 0, s, w, L, dh, 2 * (j + 1), host, next);
    } else {
      hipLaunchKernelGGL(dots_kernel, dim3(1), dim3(256), 0, s, w, L, w, 1, dh + 2 * (j + 1));
      QP_HIP(hipGetLastError());
      hipLaunchKernelGGL(scale_by_norm_kernel, dim3(blocks_for(L)), dim3(256), 0, s, w, L, dh, 2 * (j + 1), host, next);
    }
    QP_HIP(hipGetLastError());
    QP_HIP(hipEventRecord(c.krylov_events[j % kRing], s));
  };
  res.status = QPINV_ENOTCONVERGED;
  int queued = 0;
  using Clock = std::chrono::steady_clock;
  Clock::time_point first;  // when the first step had ended
  for (int j = 0; j < max_iter; ++j) {
    int ahead = 0;
    if (j == 1) first = Clock::now();
    if (j > 1) {
      const double step = std::chrono::duration<double>(Clock::now() - first).count() / (j - 1);
      ahead = (int)std::min<double>(kAhead, j * kAheadTime / step);
    }
    while (queued < max_iter && queued <= j + ahead) enqueue(queued++);
    QP_HIP(hipEventSynchronize(c.krylov_events[j % kRing]));
    const double* hh = columns + (j % kRing) * ring;
    std::vector<double> col(j + 2, 0.0);
    for (int i = 0; i <= j; ++i) col[i] = hh[i] + hh[j + 1 + i];
    const double hn = std::sqrt(hh[2 * (j + 1)]);
    col[j + 1] = hn;
    H.push_back(col);
    // apply the previous rotations to the new column, then zero its subdiagonal entry
    std::vector<double>& hc = H.back();
    for (int i = 0; i < j; ++i) {
      const double t = cs[i] * hc[i] + sn[i] * hc[i + 1];
      hc[i + 1] = -sn[i] * hc[i] + cs[i] * hc[i + 1];
      hc[i] = t;
    }
    const double rho = std::hypot(hc[j], hc[j + 1]);
    const double cj = rho > 0.0 ? hc[j] / rho : 1.0, sj = rho > 0.0 ? hc[j + 1] / rho : 0.0;
    cs.push_back(cj);
    sn.push_back(sj);
    hc[j] = rho;  // the rotated column: R's column j
    hc[j + 1] = 0.0;
    g.push_back(-sj * g[j]);
    g[j] = cj * g[j];
    k = j + 1;
    // GMRES residual |g_{j+1}|; the FOM residual is larger by 1 / |c_j| (Saad, Prop. 6.9)
    const double res_g = std::fabs(g[j + 1]);
    const double res_k = method == 0 ? (std::fabs(cj) > 0.0 ? res_g / std::fabs(cj) : INFINITY) : res_g;
    res.rr = res_k / beta;
    if (history && j < history_cap) history[j] = res.rr;
    bool stop = hn == 0.0;
    if (res.rr <= tol) {
      // the stopping test is on the original system's residual; with M it is checked from here on
      if (!M) {
        stop = true;
      } else {
        form(k, Xt);
        stop = stop || true_residual(Xt) <= tol;
      }
    }
    if (stop) {
      res.status = QPINV_OK;
      break;
    }
  }
  res.iters = k;

  form(k, X);
  res.true_rr = true_residual(X);
  return res;
}

}  // namespace qp
