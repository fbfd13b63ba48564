// Symmetric eigendecomposition in float64 by the cyclic Jacobi method (Golub
// and Van Loan, "Matrix Computations", the cyclic Jacobi algorithm and its
// parallel ordering).  Used once per build on the m x m second-moment matrix of
// the sampled residuals, whose top-r eigenvectors are the left singular vectors
// Proposition 3.1 asks for.
//
// Up to kHostDim a host core does it, row by row: the matrix sits in its L1,
// while the GPU pays a barrier per step and a round trip per sweep (a whole
// build of 2,000 points: m = 4 370 us with the host's, 496 with the GPU's; 32 526
// and 704; 48 788 and 814; 64 1,737 and 1,061).  Beyond, the GPU with the
// round-robin order of pivots.
//
// A sweep is m - 1 steps; a step rotates m / 2 disjoint pairs (p, q), so its
// rotations are independent and the matrix falls into 2 x 2 blocks, each
// updated from both sides by one thread.  Up to kLdsDim the matrix stays in
// the LDS of one workgroup for a whole sweep (the upper triangle, 1,024
// threads); beyond, each step is one launch over tiles of blocks, from one
// copy of the matrix to the other.  The rotations of a sweep are recorded and
// then applied to the rows of V, which are independent: one workgroup per row
// keeps it in LDS over all steps.  The LDS traffic of the matrix bounds the
// small case (64 KB read and written per step); the launches the large one.
// Measured, against the same rotations one pair after another on a host core:
// m = 128 in 2.5 ms (20 ms), m = 512 about 40 ms (15.5 s), m = 960 about
// 110 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <numeric>
#include <vector>

#include "abi_util.h"
#include "device_common.h"
#include "internal.h"

namespace finger {

namespace {

constexpr int kHostDim = 48;      // largest m solved on the host
constexpr int kLdsDim = 140;      // largest m whose matrix fits one CU's LDS
constexpr int kMaxSweeps = 60;
constexpr int kTile = 32;         // pairs per tile side of a large step

// pair i of step t: players 1 .. m-1 rotate past player 0
__device__ __forceinline__ void pair_of(int m, int t, int i, int& p, int& q) {
  const int n1 = m - 1;
  const int a = i == 0 ? 0 : 1 + (i - 1 + t) % n1;
  const int b = 1 + (m - 2 - i + t) % n1;
  p = a < b ? a : b;
  q = a < b ? b : a;
}

// the rotation that zeroes a_pq: cot(2 phi) = (a_qq - a_pp) / (2 a_pq), and
// tan(phi) the root of t^2 + 2 theta t - 1 = 0 of smaller size
__device__ __forceinline__ void rotation(double app, double aqq, double apq, double& t, double& c, double& s) {
  if (apq == 0.0) {
    t = 0.0;
    c = 1.0;
    s = 0.0;
    return;
  }
  const double theta = (aqq - app) / (2.0 * apq);
  t = (theta >= 0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
  c = 1.0 / sqrt(t * t + 1.0);
  s = t * c;
}

// [x y; z w] <- Ji^T [x y; z w] Jj with J = [c s; -s c]
__device__ __forceinline__ void rotate_block(double& x, double& y, double& z, double& w, double ci, double si, double cj,
                                             double sj) {
  const double x1 = cj * x - sj * y, y1 = sj * x + cj * y;
  const double z1 = cj * z - sj * w, w1 = sj * z + cj * w;
  x = ci * x1 - si * z1;
  z = si * x1 + ci * z1;
  y = ci * y1 - si * w1;
  w = si * y1 + ci * w1;
}

// sum of v over the block (fixed order); every thread gets it
__device__ __forceinline__ double block_sum(double v, double* red) {
  const int t = threadIdx.x;
  red[t] = v;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (t < w) red[t] += red[t + w];
    __syncthreads();
  }
  const double s = red[0];
  __syncthreads();
  return s;
}

// norms[0] = sum of squares above the diagonal, norms[1] = of all entries
__global__ void __launch_bounds__(1024) k_jacobi_norms(const double* A, int m, double* norms) {
  __shared__ double red[1024];
  double off = 0.0, diag = 0.0;
  for (int64_t i = threadIdx.x; i < (int64_t)m * m; i += 1024) {
    const int r = (int)(i / m), c = (int)(i % m);
    const double v = A[i];
    if (c > r) off += v * v;
    else if (c == r) diag += v * v;
  }
  off = block_sum(off, red);
  diag = block_sum(diag, red);
  if (threadIdx.x == 0) {
    norms[0] = off;
    norms[1] = 2.0 * off + diag;
  }
}

__global__ void k_jacobi_symmetrize(const double* M, int m, double* A, double* V) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)m * m) return;
  const int r = (int)(i / m), c = (int)(i % m);
  A[i] = r == c ? M[i] : 0.5 * (M[i] + M[(int64_t)c * m + r]);
  V[i] = r == c ? 1.0 : 0.0;
}

// one sweep with the matrix in LDS (entries above and on the diagonal)
__global__ void __launch_bounds__(1024) k_jacobi_sweep(double* A, int m, double2* rot, double* norms) {
  extern __shared__ __align__(16) char smem[];
  double* S = reinterpret_cast<double*>(smem);                 // [m][m]
  double2* cs = reinterpret_cast<double2*>(S + (int64_t)m * m);  // [m / 2] (c, s)
  int2* pq = reinterpret_cast<int2*>(cs + m / 2);              // [m / 2]
  const int t = threadIdx.x, h = m / 2;
  for (int i = t; i < m * m; i += 1024) S[i] = A[i];
  __syncthreads();
  // unordered pairs of pairs: (i, i + d mod h), d = 1 .. h / 2
  const int blocks = h * (h - 1) / 2;
  auto at = [&](int a, int b) -> double& { return a < b ? S[a * m + b] : S[b * m + a]; };
  for (int step = 0; step < m - 1; ++step) {
    if (t < h) {
      int p, q;
      pair_of(m, step, t, p, q);
      double app = S[p * m + p], aqq = S[q * m + q], apq = S[p * m + q], tn, c, s;
      rotation(app, aqq, apq, tn, c, s);
      S[p * m + p] = app - tn * apq;
      S[q * m + q] = aqq + tn * apq;
      S[p * m + q] = 0.0;
      cs[t] = make_double2(c, s);
      pq[t] = make_int2(p, q);
      rot[(int64_t)step * h + t] = make_double2(c, s);
    }
    __syncthreads();
    for (int b = t; b < blocks; b += 1024) {
      const int d = b / h + 1, i = b % h;
      const int j = i + d < h ? i + d : i + d - h;
      const int2 a = pq[i], e = pq[j];
      const double2 ri = cs[i], rj = cs[j];
      double &x = at(a.x, e.x), &y = at(a.x, e.y), &z = at(a.y, e.x), &w = at(a.y, e.y);
      double xv = x, yv = y, zv = z, wv = w;
      rotate_block(xv, yv, zv, wv, ri.x, ri.y, rj.x, rj.y);
      x = xv;
      y = yv;
      z = zv;
      w = wv;
    }
    __syncthreads();
  }
  for (int i = t; i < m * m; i += 1024) {
    const int r = i / m, c = i % m;
    A[i] = at(r, c);
  }
  double off = 0.0, diag = 0.0;
  for (int i = t; i < m * m; i += 1024) {
    const int r = i / m, c = i % m;
    const double v = S[i];
    if (c > r) off += v * v;
    else if (c == r) diag += v * v;
  }
  __syncthreads();
  double* red = S;  // the matrix is written out
  off = block_sum(off, red);
  diag = block_sum(diag, red);
  if (t == 0) {
    norms[0] = off;
    norms[1] = 2.0 * off + diag;
  }
}

// one step of a large matrix: a tile of 32 x 32 blocks (i, j) per workgroup,
// from A to B; the tiles of the first column record the rotations
__global__ void __launch_bounds__(256) k_jacobi_step(const double* __restrict__ A, double* __restrict__ B, int m, int step,
                                                     double2* __restrict__ rot) {
  __shared__ double2 cs[2][kTile];
  __shared__ double tn[kTile];
  __shared__ int2 pq[2][kTile];
  const int t = threadIdx.x, h = m / 2;
  const int i0 = blockIdx.y * kTile, j0 = blockIdx.x * kTile;
  if (t < 2 * kTile) {
    const int side = t / kTile, k = t % kTile, i = (side == 0 ? i0 : j0) + k;
    if (i < h) {
      int p, q;
      pair_of(m, step, i, p, q);
      double tt, c, s;
      rotation(A[(int64_t)p * m + p], A[(int64_t)q * m + q], A[(int64_t)p * m + q], tt, c, s);
      cs[side][k] = make_double2(c, s);
      pq[side][k] = make_int2(p, q);
      if (side == 0) tn[k] = tt;
      if (side == 0 && blockIdx.x == 0) rot[(int64_t)step * h + i] = make_double2(c, s);
    }
  }
  __syncthreads();
  for (int b = t; b < kTile * kTile; b += 256) {
    const int ki = b / kTile, kj = b % kTile;
    const int i = i0 + ki, j = j0 + kj;
    if (i >= h || j >= h) continue;
    const int2 a = pq[0][ki], e = pq[1][kj];
    const int64_t xx = (int64_t)a.x * m + e.x, xy = (int64_t)a.x * m + e.y;
    const int64_t yx = (int64_t)a.y * m + e.x, yy = (int64_t)a.y * m + e.y;
    double x = A[xx], y = A[xy], z = A[yx], w = A[yy];
    if (i == j) {
      const double apq = y;
      x -= tn[ki] * apq;
      w += tn[ki] * apq;
      y = 0.0;
      z = 0.0;
    } else {
      rotate_block(x, y, z, w, cs[0][ki].x, cs[0][ki].y, cs[1][kj].x, cs[1][kj].y);
    }
    B[xx] = x;
    B[xy] = y;
    B[yx] = z;
    B[yy] = w;
  }
}

// V <- V J for every rotation of a sweep, one workgroup per row
__global__ void __launch_bounds__(256) k_jacobi_rows(double* V, int m, const double2* rot) {
  extern __shared__ __align__(16) char smem[];
  double* v = reinterpret_cast<double*>(smem);
  double* row = V + (int64_t)blockIdx.x * m;
  const int h = m / 2;
  for (int i = threadIdx.x; i < m; i += blockDim.x) v[i] = row[i];
  __syncthreads();
  for (int step = 0; step < m - 1; ++step) {
    for (int i = threadIdx.x; i < h; i += blockDim.x) {
      int p, q;
      pair_of(m, step, i, p, q);
      const double2 r = rot[(int64_t)step * h + i];
      const double x = v[p], y = v[q];
      v[p] = r.x * x - r.y * y;
      v[q] = r.y * x + r.x * y;
    }
    __syncthreads();
  }
  for (int i = threadIdx.x; i < m; i += blockDim.x) row[i] = v[i];
}

// A (m x m, row-major): the eigenvalues on its diagonal on return; V: the
// eigenvectors in its columns.
void jacobi_host(double* A, int m, double* V) {
  for (int i = 0; i < m; ++i)
    for (int j = 0; j < m; ++j) V[i * m + j] = i == j ? 1.0 : 0.0;
  // symmetrize exactly
  for (int i = 0; i < m; ++i)
    for (int j = i + 1; j < m; ++j) A[i * m + j] = A[j * m + i] = 0.5 * (A[i * m + j] + A[j * m + i]);
  double total = 0.0;
  for (int i = 0; i < m * m; ++i) total += A[i] * A[i];
  for (int sweep = 0; sweep < kMaxSweeps; ++sweep) {
    double off = 0.0;
    for (int p = 0; p < m; ++p)
      for (int q = p + 1; q < m; ++q) off += A[p * m + q] * A[p * m + q];
    if (off <= 1e-30 * total || off == 0.0) break;
    for (int p = 0; p < m - 1; ++p) {
      for (int q = p + 1; q < m; ++q) {
        const double apq = A[p * m + q];
        if (apq == 0.0) continue;
        const double theta = (A[q * m + q] - A[p * m + p]) / (2.0 * apq);
        const double t = (theta >= 0 ? 1.0 : -1.0) / (std::fabs(theta) + std::sqrt(theta * theta + 1.0));
        const double c = 1.0 / std::sqrt(t * t + 1.0), s = t * c;
        auto turn = [&](double& x, double& y) {
          const double x0 = x, y0 = y;
          x = c * x0 - s * y0;
          y = s * x0 + c * y0;
        };
        for (int k = 0; k < m; ++k) turn(A[k * m + p], A[k * m + q]);  // A <- A J
        for (int k = 0; k < m; ++k) turn(A[p * m + k], A[q * m + k]);  // A <- J^T A
        A[p * m + q] = A[q * m + p] = 0.0;
        for (int k = 0; k < m; ++k) turn(V[k * m + p], V[k * m + q]);  // V <- V J
      }
    }
  }
}

// the same on the GPU
int jacobi_device(const double* M_dev, int m, double* Ah, double* Vh, hipStream_t s) {
  using namespace abi;
  const size_t mm = (size_t)m * m;
  const int h = m / 2;
  DevBuf<double> A, B, V, norms;
  DevBuf<double2> rot;
  int st;
  if ((st = dev_alloc(reinterpret_cast<void**>(&A.p), mm * 8, "eigensolver")) != FINGER_OK) return st;
  if ((st = dev_alloc(reinterpret_cast<void**>(&V.p), mm * 8, "eigensolver")) != FINGER_OK) return st;
  if ((st = dev_alloc(reinterpret_cast<void**>(&rot.p), (size_t)(m - 1) * h * 16, "eigensolver")) != FINGER_OK) return st;
  if ((st = dev_alloc(reinterpret_cast<void**>(&norms.p), 16, "eigensolver")) != FINGER_OK) return st;
  const bool lds = m <= kLdsDim;
  if (!lds && (st = dev_alloc(reinterpret_cast<void**>(&B.p), mm * 8, "eigensolver")) != FINGER_OK) return st;
  const int lds_bytes = std::max((int)(mm * 8 + (size_t)h * 24), 1024 * 8);
  if (lds)
    HIPCHK(hipFuncSetAttribute(reinterpret_cast<const void*>(k_jacobi_sweep), hipFuncAttributeMaxDynamicSharedMemorySize,
                               lds_bytes));
  hipLaunchKernelGGL(k_jacobi_symmetrize, dim3((unsigned)((mm + 255) / 256)), dim3(256), 0, s, M_dev, m, A.p, V.p);
  hipLaunchKernelGGL(k_jacobi_norms, dim3(1), dim3(1024), 0, s, A.p, m, norms.p);
  HIPCHK(hipGetLastError());
  double n2[2];
  double *cur = A.p, *other = B.p;
  for (int sweep = 0;; ++sweep) {
    HIPCHK(hipMemcpyAsync(n2, norms.p, 16, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    if (n2[0] <= 1e-30 * n2[1] || n2[0] == 0.0 || sweep == kMaxSweeps) break;
    if (lds) {
      hipLaunchKernelGGL(k_jacobi_sweep, dim3(1), dim3(1024), lds_bytes, s, cur, m, rot.p, norms.p);
    } else {
      const unsigned tiles = (unsigned)((h + kTile - 1) / kTile);
      for (int step = 0; step < m - 1; ++step) {
        hipLaunchKernelGGL(k_jacobi_step, dim3(tiles, tiles), dim3(256), 0, s, cur, other, m, step, rot.p);
        std::swap(cur, other);
      }
      hipLaunchKernelGGL(k_jacobi_norms, dim3(1), dim3(1024), 0, s, cur, m, norms.p);
    }
    hipLaunchKernelGGL(k_jacobi_rows, dim3((unsigned)m), dim3(h >= 256 ? 256 : 64 * ((h + 63) / 64)), (size_t)m * 8, s,
                       V.p, m, rot.p);
    HIPCHK(hipGetLastError());
  }
  HIPCHK(hipMemcpyAsync(Ah, cur, mm * 8, hipMemcpyDeviceToHost, s));
  HIPCHK(hipMemcpyAsync(Vh, V.p, mm * 8, hipMemcpyDeviceToHost, s));
  HIPCHK(hipStreamSynchronize(s));
  return FINGER_OK;
}

}  // namespace

// m even (every supported length is a multiple of 4)
int eigh_jacobi(const double* M_dev, int m, double* evals, double* Vout, hipStream_t s) {
  using namespace abi;
  const size_t mm = (size_t)m * m;
  std::vector<double> Ah, Vh;
  std::vector<int> order;
  try {
    Ah.resize(mm);
    Vh.resize(mm);
    order.resize((size_t)m);
  } catch (const std::bad_alloc&) {
    return fail(FINGER_ENOMEM, "host copy of the eigenvectors");
  }
  if (m <= kHostDim) {
    HIPCHK(hipMemcpyAsync(Ah.data(), M_dev, mm * 8, hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    jacobi_host(Ah.data(), m, Vh.data());
  } else {
    const int st = jacobi_device(M_dev, m, Ah.data(), Vh.data(), s);
    if (st != FINGER_OK) return st;
  }
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(),
                   [&](int a, int b) { return Ah[(size_t)a * m + a] > Ah[(size_t)b * m + b]; });
  for (int i = 0; i < m; ++i) {
    const int src = order[i];
    evals[i] = Ah[(size_t)src * m + src];
    // sign: the entry of largest magnitude (first on ties) is positive
    int jmax = 0;
    for (int k = 1; k < m; ++k)
      if (std::fabs(Vh[(size_t)k * m + src]) > std::fabs(Vh[(size_t)jmax * m + src])) jmax = k;
    const double sgn = Vh[(size_t)jmax * m + src] < 0 ? -1.0 : 1.0;
    for (int k = 0; k < m; ++k) Vout[(size_t)i * m + k] = sgn * Vh[(size_t)k * m + src];
  }
  return FINGER_OK;
}

}  // namespace finger
