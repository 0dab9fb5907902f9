// lre_project.hip -- step (iii) of LRE: the density matrix closest to mu.
//
// Sec. II, step (iii): mu from eq. (4) can have negative eigenvalues; the estimate is
// the physical state closest to it, computed with the fast algorithm the paper cites
// (Smolin, Gambetta and Smith 2012): eigendecompose mu, move the spectrum onto the
// probability simplex (negative eigenvalues removed, their mass shared equally over
// the eigenvalues kept), reassemble.
//   n <= 6: everything in one workgroup (jacobi_project_kernel).
//   n = 7, 8: reduction to tridiagonal form in one workgroup (hetrd_kernel), rocSOLVER's
//     divide and conquer on the tridiagonal matrix, and one wave per eigenvector for the
//     back-transformation (unmtr_kernel).
//   n >= 9: rocSOLVER's divide-and-conquer Hermitian solver (zheevd).
// Above 6 qubits the reassembly V diag(lambda) V^H is a rocBLAS zgemm -- dense O(d^3) work,
// bound by FP64 matrix throughput; the spectrum step and the column scaling are kernels of
// this file.
//
// Layout: mu and rho are row-major complex128 [d][d].  Read column-major, the row-major
// buffer of a Hermitian matrix is its conjugate; the projection commutes with complex
// conjugation, so running the column-major solver and product on the buffers as they
// are yields rho row-major.
#include <hip/hip_runtime.h>
#include <rocblas/rocblas.h>
#include <rocsolver/rocsolver.h>

#include "lre.h"
#include "lre_internal.hpp"
#include "lre_kernels.hpp"

namespace {

using lre_detail::DeviceGuard;

size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

// Words beside the solver's info: hetrd_kernel's power of two, whether something is not finite.
constexpr int kInfoSolver = 0, kInfoExp = 1, kInfoBad = 2, kInfoWords = 3;

struct ProjLayout {
  size_t a, b, w, e, lam, info, total;
};

ProjLayout proj_layout(int n) {
  const size_t d = (size_t)1 << n;
  ProjLayout L{};
  size_t off = 0;
  L.a = off; off += align256(16 * d * d);     // eigenvectors (the solver works in place)
  L.b = off; off += align256(16 * d * d);     // eigenvectors scaled by the new spectrum
  L.w = off; off += align256(8 * d);          // eigenvalues of mu, ascending
  L.e = off; off += align256(8 * d);          // solver scratch (off-diagonal)
  L.lam = off; off += align256(8 * d);        // projected spectrum
  L.info = off; off += align256(kInfoWords * sizeof(rocblas_int));
  L.total = off;
  return L;
}

constexpr int kJacobiN = 6;   // mu and its eigenvectors (2 x 64 KiB) fit the LDS
// One CU against a launch per column and step, whole calls: n = 7 1.53 ms (library 3.05),
// n = 8 3.69 (7.45); its time grows by 8 a qubit, the library's by 2 (n = 9: 13.8 ms).
constexpr int kHetrdN = 8;

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 conj2(double2 a) { return make_double2(a.x, -a.y); }
// c + a b, c + a conj(b)
__device__ __forceinline__ double2 cfma(double2 a, double2 b, double2 c) {
  return make_double2(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
__device__ __forceinline__ double2 cfmac(double2 a, double2 b, double2 c) { return cfma(a, conj2(b), c); }

// Spectrum step on ascending eigenvalues w[0..d): the first i >= 0 with w[i] + a_i / (d - i)
// >= 0, a_i the sum of the i below it, is the smallest kept; those below become 0 and the
// kept ones are raised by a_i / (d - i).  One block: every thread sums a run of the values,
// the runs' sums are scanned, and the smallest i is found by a minimum over the block.  (One
// thread walking the list took 42 us at d = 256.)  Returns i and sets shift.
constexpr int kSpectrumThreads = 1024;

template <int THREADS>
__device__ __forceinline__ int spectrum_cut(const double* w, int d, int tid, double* run, int* first, double& shift) {
  const int per = (d + THREADS - 1) / THREADS;
  const int i0 = tid * per < d ? tid * per : d, i1 = i0 + per < d ? i0 + per : d;
  double s = 0.0;
  for (int i = i0; i < i1; ++i) s += w[i];
  run[tid] = s;
  if (tid == 0) *first = d;
  __syncthreads();
  for (int o = 1; o < THREADS; o <<= 1) {
    const double v = tid >= o ? run[tid - o] : 0.0;
    __syncthreads();
    run[tid] += v;
    __syncthreads();
  }
  double a = tid > 0 ? run[tid - 1] : 0.0;
  for (int i = i0; i < i1; ++i) {
    if (w[i] + a / (double)(d - i) >= 0.0) {
      atomicMin(first, i);
      break;
    }
    a += w[i];
  }
  __syncthreads();
  const int cut = *first;
  __syncthreads();
  // the sum below the cut, from the thread whose run holds it
  if (cut < d && cut >= i0 && cut < i1) {
    double b = tid > 0 ? run[tid - 1] : 0.0;
    for (int i = i0; i < cut; ++i) b += w[i];
    run[0] = b / (double)(d - cut);
  }
  __syncthreads();
  shift = run[0];
  return cut;
}

// A solver failure (info), or eigenvalues that are not finite, raise FLAG_EIG and leave lambda = 0.
// own: w are those of hetrd_kernel's matrix (its power of two).
__global__ __launch_bounds__(kSpectrumThreads) void spectrum_kernel(double* __restrict__ w, double* __restrict__ lam,
                                                                    rocblas_int* __restrict__ info, bool own, int d,
                                                                    uint32_t* __restrict__ flags,
                                                                    double* __restrict__ eig_out) {
  __shared__ double run[kSpectrumThreads];
  __shared__ int first, bad;
  const int tid = threadIdx.x;
  if (tid == 0) bad = info[kInfoSolver] != 0 || (own && info[kInfoBad] != 0);
  __syncthreads();
  const int ex = own ? info[kInfoExp] : 0;
  for (int j = tid; j < d; j += kSpectrumThreads) {
    if (!isfinite(w[j])) bad = 1;
    else if (ex != 0) w[j] = ldexp(w[j], ex);
  }
  __syncthreads();
  if (tid == 0) info[kInfoBad] = bad;
  if (bad) {                                 // uniform
    if (tid == 0) lre::raise_flag(flags, lre::FLAG_EIG);
    for (int j = tid; j < d; j += kSpectrumThreads) lam[j] = 0.0;
    return;
  }
  double shift;
  const int cut = spectrum_cut<kSpectrumThreads>(w, d, tid, run, &first, shift);
  for (int j = tid; j < d; j += kSpectrumThreads) {
    lam[j] = j < cut ? 0.0 : w[j] + shift;
    if (eig_out) eig_out[j] = w[j];
  }
}

// Step (iii) of n <= 6 qubits in one workgroup: cyclic two-sided Jacobi on mu in LDS.  A round
// takes the d/2 disjoint pairs of a round robin: their rotations are found by d/2 threads, then
// thread (i, j) applies those of pairs i and j to its own 2 x 2 block of mu, and every column
// pair of the eigenvectors is rotated; two barriers a round, d - 1 rounds a sweep, until a
// sweep finds no element above 1e-17 of mu's norm (7 to 10 sweeps).  The lower triangle of mu
// is read (before rho is written: the two may be one buffer).  Then the spectrum step and
// rho = V diag(lambda) V^H, its lower triangle computed and mirrored.  Sums are in a fixed order.
// Bound by the rounds' latency (two barriers, a square root and two divisions, LDS): n = 1 .. 6
// take 25, 33, 61, 129, 310, 1110 us whole calls; the library's solver and the launches around it
// took 126, 141, 247, 607, 987, 1952.
constexpr int kJacobiSweeps = 40;

template <int N>
struct JacobiGeom {
  static constexpr int D = 1 << N, H = D / 2;
  static constexpr int THREADS = H * H < 64 ? 64 : (H * H > 1024 ? 1024 : H * H);
  static constexpr int PER = (D * D + THREADS - 1) / THREADS;
};

template <int N>
__global__ __launch_bounds__(JacobiGeom<N>::THREADS) void jacobi_project_kernel(const double2* mu,
                                                                               double2* rho,
                                                                               double* __restrict__ eig_out,
                                                                               uint32_t* __restrict__ flags) {
  using G = JacobiGeom<N>;
  constexpr int D = G::D, H = G::H, TH = G::THREADS, P = D + 1;
  __shared__ double2 A[D * P], V[D * P];
  __shared__ double2 rot[H];            // S of every pair
  __shared__ double rotc[H], rotd[H];   // c; what the diagonal elements move by
  __shared__ double w[D], lam[D], rotq[D], run[TH];
  __shared__ int rank[D], any, any_round, first;
  const int tid = threadIdx.x;
  auto element = [&](int r, int c) {
    double2 v = r >= c ? mu[r * D + c] : conj2(mu[c * D + r]);
    if (r == c) v.y = 0.0;
    return v;
  };
  // Work on mu times a power of two that brings its largest entry to [1/2, 1), so that squares
  // stay in range.
  double big = 0.0;
  bool finite = true;
  for (int t = tid; t < D * D; t += TH) {
    const double2 v = element(t / D, t % D);
    finite = finite && isfinite(v.x) && isfinite(v.y);
    big = fmax(big, fmax(fabs(v.x), fabs(v.y)));
  }
  run[tid] = finite ? big : INFINITY;
  __syncthreads();
  for (int o = TH / 2; o > 0; o >>= 1) {
    if (tid < o) run[tid] = fmax(run[tid], run[tid + o]);
    __syncthreads();
  }
  big = run[0];
  __syncthreads();
  int e2 = 0;
  if (big < INFINITY) (void)frexp(big, &e2);
  double norm2 = 0.0;
  for (int t = tid; t < D * D; t += TH) {
    const int r = t / D, c = t % D;
    const double2 m = element(r, c), v = make_double2(ldexp(m.x, -e2), ldexp(m.y, -e2));
    A[r * P + c] = v;
    V[r * P + c] = make_double2(r == c ? 1.0 : 0.0, 0.0);
    norm2 += v.x * v.x + v.y * v.y;
  }
  run[tid] = norm2;
  __syncthreads();
  for (int o = TH / 2; o > 0; o >>= 1) {
    if (tid < o) run[tid] += run[tid + o];
    __syncthreads();
  }
  const double thr2 = run[0] * 1e-34;
  __syncthreads();
  // Pair k of round r: the fixed player D - 1 meets r, the others r + k and r - k mod D - 1.
  auto pair_of = [&](int r, int k, int& p, int& q) {
    const int m = D - 1;
    p = k == 0 ? m : (r + k < m ? r + k : r + k - m);
    q = r >= k ? r - k : r - k + m;
  };
  int sweep = big < INFINITY ? 0 : kJacobiSweeps;   // no eigenvalues of what is not finite
  for (; sweep < kJacobiSweeps; ++sweep) {
    if (tid == 0) any = 0;
    for (int r = 0; r < D - 1; ++r) {
      if (tid == 0) any_round = 0;
      __syncthreads();
      if (tid < H) {
        int p, q;
        pair_of(r, tid, p, q);
        const double2 a = A[p * P + q];
        const double m2 = a.x * a.x + a.y * a.y;
        double c = 1.0;
        double2 S = make_double2(0.0, 0.0);
        double move = 0.0;
        if (m2 > thr2) {
          const double m = sqrt(m2);
          const double tau = (A[q * P + q].x - A[p * P + p].x) / (2.0 * m);
          const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
          c = 1.0 / sqrt(1.0 + t * t);
          const double s = t * c / m;
          S = make_double2(s * a.x, s * a.y);
          move = t * m;
          any = 1;
          any_round = 1;
        }
        rot[tid] = S;
        rotc[tid] = c;
        rotd[tid] = move;
      }
      __syncthreads();
      if (any_round) {
        for (int t = tid; t < H * H; t += TH) {
          const int i = t / H, j = t % H;
          int pi, qi, pj, qj;
          pair_of(r, i, pi, qi);
          pair_of(r, j, pj, qj);
          const double ci = rotc[i], cj = rotc[j];
          const double2 Si = rot[i], Sj = rot[j];
          auto right = [&](double2 x, double2 y, double2& x2, double2& y2) {   // columns (p, q) times J
            const double2 u = cmul(conj2(Sj), y), v = cmul(Sj, x);
            x2 = make_double2(cj * x.x - u.x, cj * x.y - u.y);
            y2 = make_double2(cj * y.x + v.x, cj * y.y + v.y);
          };
          double2 b00, b01, b10, b11;
          right(A[pi * P + pj], A[pi * P + qj], b00, b01);
          right(A[qi * P + pj], A[qi * P + qj], b10, b11);
          auto left = [&](double2 x, double2 y, double2& x2, double2& y2) {    // J^H times rows (p, q)
            const double2 u = cmul(Si, y), v = cmul(conj2(Si), x);
            x2 = make_double2(ci * x.x - u.x, ci * x.y - u.y);
            y2 = make_double2(ci * y.x + v.x, ci * y.y + v.y);
          };
          double2 a00, a01, a10, a11;
          left(b00, b10, a00, a10);
          left(b01, b11, a01, a11);
          if (i == j) {
            a00 = make_double2(A[pi * P + pi].x - rotd[i], 0.0);
            a11 = make_double2(A[qi * P + qi].x + rotd[i], 0.0);
            if (Si.x != 0.0 || Si.y != 0.0) a01 = a10 = make_double2(0.0, 0.0);
          }
          A[pi * P + pj] = a00;
          A[pi * P + qj] = a01;
          A[qi * P + pj] = a10;
          A[qi * P + qj] = a11;
        }
        for (int t = tid; t < D * H; t += TH) {
          const int k = t / H, j = t % H;
          int p, q;
          pair_of(r, j, p, q);
          const double c = rotc[j];
          const double2 S = rot[j], x = V[k * P + p], y = V[k * P + q];
          const double2 u = cmul(conj2(S), y), v = cmul(S, x);
          V[k * P + p] = make_double2(c * x.x - u.x, c * x.y - u.y);
          V[k * P + q] = make_double2(c * y.x + v.x, c * y.y + v.y);
        }
      }
      __syncthreads();
    }
    const int more = any;
    __syncthreads();
    if (!more) break;
  }
  if (sweep == kJacobiSweeps) {           // uniform
    if (tid == 0) lre::raise_flag(flags, lre::FLAG_EIG);
    for (int t = tid; t < D * D; t += TH) rho[t] = make_double2(0.0, 0.0);
    return;
  }
  // The rotations' rounding leaves the columns of V off unit length and the diagonal off the
  // eigenvalues by some 1e-15 of the norm: columns to unit length, eigenvalues as the
  // quotients v^H mu v, whose error is the square of v's (lam holds them, by column).
  for (int i = tid; i < D; i += TH) {
    double s = 0.0;
#pragma unroll 2
    for (int r = 0; r < D; ++r) s += V[r * P + i].x * V[r * P + i].x + V[r * P + i].y * V[r * P + i].y;
    rotq[i] = 1.0 / sqrt(s);
  }
  for (int t = tid; t < D * D; t += TH) {        // mu again (the rounds are over)
    const double2 m = element(t / D, t % D);
    A[(t / D) * P + t % D] = make_double2(ldexp(m.x, -e2), ldexp(m.y, -e2));
  }
  __syncthreads();
  for (int t = tid; t < D * D; t += TH) {
    const int r = t / D, c = t % D;
    V[r * P + c].x *= rotq[c];
    V[r * P + c].y *= rotq[c];
  }
  __syncthreads();
  static_assert(TH % D == 0, "a thread's elements are of one eigenvector");
  double2 mv[G::PER];
  double quotient = 0.0;
#pragma unroll
  for (int q = 0; q < G::PER; ++q) {             // (row r, eigenvector i): conj(v_r) (mu v)_r
    const int t = tid + q * TH, r = t / D, i = t % D;
    mv[q] = make_double2(0.0, 0.0);
    if (t >= D * D) continue;
#pragma unroll 2
    for (int k = 0; k < D; ++k) mv[q] = cfma(A[r * P + k], V[k * P + i], mv[q]);
    const double2 v = V[r * P + i];
    quotient += v.x * mv[q].x + v.y * mv[q].y;
  }
  run[tid] = quotient;
  __syncthreads();
  for (int i = tid; i < D; i += TH) {            // in a fixed order: two runs give the same bits
    double q = 0.0;
    for (int k = i; k < TH; k += D) q += run[k];
    lam[i] = q;
  }
  __syncthreads();
  // The vectors' own error grows with the root of the rotations: at 6 qubits, some 500 a column,
  // rho is further off than by the library's solver (mean 2.5e-15 against 2.0e-15; at 5
  // qubits 1.8e-15 against 2.0e-15).  One correction to first order, V += V E with
  // E_ij = v_i^H (mu v_j - lambda_j v_j) / (lambda_j - lambda_i), for pairs 1e-6 of the norm apart
  // or more (E^2 is then below the rounding; closer ones do not matter to rho).
  if constexpr (N >= 6) {
    static_assert(G::PER * TH == D * D, "an element a thread and step");
#pragma unroll
    for (int q = 0; q < G::PER; ++q) {
      const int t = tid + q * TH, r = t / D, i = t % D;
      const double2 v = V[r * P + i];
      A[r * P + i] = make_double2(fma(-lam[i], v.x, mv[q].x), fma(-lam[i], v.y, mv[q].y));
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < G::PER; ++q) {
      const int t = tid + q * TH, i = t / D, j = t % D;
      double2 s = make_double2(0.0, 0.0);
#pragma unroll 2
      for (int k = 0; k < D; ++k) s = cfma(conj2(V[k * P + i]), A[k * P + j], s);
      const double gap = lam[j] - lam[i];
      const double inv = gap * gap > thr2 * 1e22 ? 1.0 / gap : 0.0;
      mv[q] = make_double2(s.x * inv, s.y * inv);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < G::PER; ++q) A[(tid + q * TH) / D * P + (tid + q * TH) % D] = mv[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < G::PER; ++q) {
      const int t = tid + q * TH, r = t / D, j = t % D;
      mv[q] = make_double2(0.0, 0.0);
#pragma unroll 2
      for (int k = 0; k < D; ++k) mv[q] = cfma(V[r * P + k], A[k * P + j], mv[q]);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < G::PER; ++q) {
      const int t = tid + q * TH;
      double2& v = V[t / D * P + t % D];
      v = make_double2(v.x + mv[q].x, v.y + mv[q].y);
    }
    __syncthreads();
  }
  for (int i = tid; i < D; i += TH) {
    const double x = lam[i];                     // (scaled: the order is the same)
    int k = 0;
#pragma unroll 4
    for (int j = 0; j < D; ++j) {
      const double y = lam[j];
      k += y < x || (y == x && j < i);
    }
    rank[i] = k;
    w[k] = ldexp(x, e2);
  }
  __syncthreads();
  double shift;
  const int cut = spectrum_cut<TH>(w, D, tid, run, &first, shift);
  for (int i = tid; i < D; i += TH) {
    const int k = rank[i];
    lam[i] = k < cut ? 0.0 : w[k] + shift;   // by column of V
    if (eig_out) eig_out[i] = w[i];
  }
  __syncthreads();
  for (int t = tid; t < D * D; t += TH) {
    const int r = t / D, c = t % D;
    if (r < c) continue;
    double2 s = make_double2(0.0, 0.0);
#pragma unroll 2
    for (int k = 0; k < D; ++k) {
      const double l = lam[k];
      const double2 x = V[r * P + k];
      s = cfmac(make_double2(l * x.x, l * x.y), V[c * P + k], s);
    }
    if (r == c) s.y = 0.0;
    rho[t] = s;
    if (r > c) rho[c * D + r] = conj2(s);
  }
}

template <int N>
void launch_jacobi(const double2* mu, double2* rho, double* eig, uint32_t* flags, hipStream_t st) {
  hipLaunchKernelGGL((jacobi_project_kernel<N>), dim3(1), dim3(JacobiGeom<N>::THREADS), 0, st, mu, rho, eig, flags);
}

// Sum over the wave of four values; lanes 0, 32, 16, 48 hold the sums of a, b, c, d (each in
// all 16 lanes from there).
__device__ __forceinline__ double swap_add32(double x, double y) {
  const uint64_t u = __double_as_longlong(x), v = __double_as_longlong(y);
  const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)v, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(v >> 32), false, false);
  return __longlong_as_double(((uint64_t)hi[0] << 32) | lo[0]) + __longlong_as_double(((uint64_t)hi[1] << 32) | lo[1]);
}
__device__ __forceinline__ double swap_add16(double x, double y) {
  const uint64_t u = __double_as_longlong(x), v = __double_as_longlong(y);
  const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)v, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(v >> 32), false, false);
  return __longlong_as_double(((uint64_t)hi[0] << 32) | lo[0]) + __longlong_as_double(((uint64_t)hi[1] << 32) | lo[1]);
}
template <int CTRL>
__device__ __forceinline__ double dpp_add(double x) {
  const uint64_t u = __double_as_longlong(x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
  return x + __longlong_as_double(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double row_sum16(double x) {      // over 16 lanes, in all of them
  x = dpp_add<lre::kDppMirror>(x);
  x = dpp_add<lre::kDppHalfMirror>(x);
  x = dpp_add<lre::kDppQuadXor2>(x);
  return dpp_add<lre::kDppQuadXor1>(x);
}
__device__ __forceinline__ double wave_sum4(double a, double b, double c, double d) {
  return row_sum16(swap_add16(swap_add32(a, b), swap_add32(c, d)));
}

// The Hermitian matrix given by the upper triangle (column-major) of `in`: its lower triangle.
// (The triangle the library's solver is given for the other sizes.)
__global__ __launch_bounds__(256) void lower_copy_kernel(const double2* __restrict__ in, double2* __restrict__ out, int d) {
  __shared__ double2 t[16][17];
  const int x = threadIdx.x % 16, y = threadIdx.x / 16;
  const int bc = blockIdx.x * 16, br = blockIdx.y * 16;          // out: rows br.., columns bc..
  if (br < bc) return;
  t[y][x] = in[(int64_t)(br + y) * d + bc + x];                  // (row bc + x, column br + y)
  __syncthreads();
  out[(int64_t)(bc + y) * d + br + x] = conj2(t[x][y]);
}

// Householder reduction of a Hermitian D x D matrix (column-major, lower triangle) to
// tridiagonal form in one workgroup: A = Q T Q^H, Q = H_0 H_1 ..., H_i = I - tau v v^H with
// v = (0 .. 0, 1, column i of A from row i + 2 on) and tau on A's diagonal; diagonal and
// subdiagonal of T in dg and e.  Column step i: the
// rank-2 update of step i - 1 is applied to column i, which gives the reflector v; one pass
// over the trailing lower triangle then applies the update to it and forms A v: a wave takes
// two columns at a time, lanes along the rows, so that each element is read and written once
// and serves both its column's dot product and its row's sum.  One pass and five barriers a
// step, all within one CU, against five launches a step in the library.  Every sum is taken in a
// fixed order (each wave's row sums of A v in LDS of their own, 64 KiB at n = 8).  Bound by the one
// CU: per step some 4.4k cycles of binary64 arithmetic, 5k of L2 traffic and the barriers'
// serial parts: 2.10 ms at n = 8 (8 us a step; the library: 28), 0.54 at n = 7.  512 threads with
// the next columns loaded ahead: 2.72 ms.
constexpr int kHetrdThreads = 1024;

template <int D>
__global__ __launch_bounds__(kHetrdThreads) void hetrd_kernel(double2* __restrict__ A, double* __restrict__ dg,
                                                              double* __restrict__ e,
                                                              rocblas_int* __restrict__ info) {
  constexpr int CH = D / 64, WAVES = kHetrdThreads / 64;
  __shared__ double2 vP[D], wP[D], vN[D];     // previous step's v and w, this step's v
  __shared__ double ydot[2][D];               // A v: the columns' dot products
  __shared__ double2 yrow[WAVES][D];          // and the rows' sums over each wave's columns
  __shared__ double red[WAVES][2], redm[WAVES];
  __shared__ double2 alpha_s;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Sum of (x, y) over the block, in every thread.
  auto block_sum = [&](double x, double y) {
    const double s = wave_sum4(x, y, 0.0, 0.0);
    if (lane == 0) red[wave][0] = s;
    if (lane == 32) red[wave][1] = s;
    __syncthreads();
    return make_double2(row_sum16(red[lane & 15][0]), row_sum16(red[lane & 15][1]));
  };
  static_assert(WAVES == 16, "a row of lanes takes the waves' sums");
  // Largest m of the block (m >= 0), in every thread.
  auto block_max = [&](double m) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
    if (lane == 0) redm[wave] = m;
    __syncthreads();
    for (int k = 0; k < WAVES; ++k) m = fmax(m, redm[k]);
    return m;
  };
  if (tid < D) vP[tid] = wP[tid] = make_double2(0.0, 0.0);
  __syncthreads();
  for (int i = 0; i < D; ++i) {
    // column i under the previous update; its reflector
    double2 x = make_double2(0.0, 0.0);
    if (tid < D && tid >= i) {
      x = A[tid + (int64_t)i * D];
      const double2 v = vP[tid], w = wP[tid], vi = vP[i], wi = wP[i];
      x = cfmac(make_double2(-v.x, -v.y), wi, x);
      x = cfmac(make_double2(-w.x, -w.y), vi, x);
      if (tid == i) dg[i] = x.x;
      if (tid == i + 1) alpha_s = x;
    }
    if (i == D - 1) break;                     // uniform
    auto tail2 = [&] { return block_sum(tid < D && tid > i + 1 ? x.x * x.x + x.y * x.y : 0.0, 0.0).x; };
    double n2 = tail2();
    double2 al = alpha_s;
    // Squares near the ends of the type's range, or none (uniform): the column times a power of
    // two that brings its largest entry to [1/2, 1).  The reflector is the same, beta scales.
    int ex = 0;
    const double all2 = al.x * al.x + al.y * al.y + n2;
    if (!(all2 > 1e-280 && all2 < 1e280)) {
      const double big = block_max(tid < D && tid > i ? fmax(fabs(x.x), fabs(x.y)) : 0.0);
      if (big > 0.0 && big < INFINITY) {
        (void)frexp(big, &ex);
        x = make_double2(ldexp(x.x, -ex), ldexp(x.y, -ex));
        al = make_double2(ldexp(al.x, -ex), ldexp(al.y, -ex));
        n2 = tail2();
      }
    }
    double beta = al.x;
    double2 tau = make_double2(0.0, 0.0), scale = make_double2(0.0, 0.0);
    if (n2 != 0.0 || al.y != 0.0) {
      beta = sqrt(al.x * al.x + al.y * al.y + n2);
      if (al.x >= 0.0) beta = -beta;
      tau = make_double2((beta - al.x) / beta, -al.y / beta);
      const double dx = al.x - beta, q = 1.0 / (dx * dx + al.y * al.y);
      scale = make_double2(dx * q, -al.y * q);
    }
    if (tid < D) {
      double2 v = make_double2(0.0, 0.0);
      if (tid == i + 1) v.x = 1.0;
      else if (tid > i + 1) {
        v = cmul(x, scale);
        A[tid + (int64_t)i * D] = v;
      }
      vN[tid] = v;
    }
    if (tid == 0) {
      e[i] = ldexp(beta, ex);
      A[i + (int64_t)i * D] = tau;
    }
    __syncthreads();

    // one pass over the trailing lower triangle
    double2 v0[CH], v1[CH], ya[CH];
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      v0[j] = vP[64 * j + lane];
      v1[j] = vN[64 * j + lane];
      ya[j] = make_double2(0.0, 0.0);
    }
    // Two columns c0, c0 + WAVES at a time.
    auto load2 = [&](int c0, double2 (&a)[2][CH]) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int c = c0 + k * WAVES;
#pragma unroll
        for (int j = 0; j < CH; ++j) {
          a[k][j] = make_double2(0.0, 0.0);
          if (c < D && 64 * j + 63 >= c && 64 * j + lane >= c) a[k][j] = A[64 * j + lane + (int64_t)c * D];
        }
      }
    };
    auto work2 = [&](int c0, const double2 (&a)[2][CH]) __attribute__((always_inline)) {
      double2 dot[2] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int c = c0 + k * WAVES;
        if (c >= D) continue;                  // uniform
        const double2 wc = wP[c], vc = vP[c], nc = vN[c];
#pragma unroll
        for (int j = 0; j < CH; ++j) {
          if (64 * j + 63 < c) continue;       // uniform
          const int r = 64 * j + lane;
          if (r >= c) {
            double2 t = cfmac(make_double2(-v0[j].x, -v0[j].y), wc, a[k][j]);
            const double2 wr = wP[r];
            t = cfmac(make_double2(-wr.x, -wr.y), vc, t);
            if (r == c) t.y = 0.0;
            A[r + (int64_t)c * D] = t;
            dot[k] = cfma(conj2(t), v1[j], dot[k]);
            if (r > c) ya[j] = cfma(t, nc, ya[j]);
          }
        }
      }
      const double s = wave_sum4(dot[0].x, dot[0].y, dot[1].x, dot[1].y);
      // lane 0: dot[0].x, 32: dot[0].y, 16: dot[1].x, 48: dot[1].y
      const int cl = c0 + ((lane & 16) ? WAVES : 0);
      if ((lane & 15) == 0 && cl < D) ydot[(lane & 32) ? 1 : 0][cl] = s;
    };
    for (int c0 = i + 1 + wave; c0 < D; c0 += 2 * WAVES) {
      double2 a[2][CH];
      load2(c0, a);
      work2(c0, a);
    }
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      if (64 * j + 63 > i) yrow[wave][64 * j + lane] = ya[j];    // uniform
    }
    __syncthreads();
    // w = tau y - (1/2) tau (tau y)^H v v
    double2 xt = make_double2(0.0, 0.0), vt = make_double2(0.0, 0.0);
    if (tid < D && tid > i) {
      vt = vN[tid];
      double2 y = make_double2(ydot[0][tid], ydot[1][tid]);
#pragma unroll
      for (int k = 0; k < WAVES; ++k) {         // in a fixed order: two runs give the same bits
        const double2 p = yrow[k][tid];
        y.x += p.x;
        y.y += p.y;
      }
      xt = cmul(tau, y);
    }
    const double2 dp = block_sum(xt.x * vt.x + xt.y * vt.y, xt.x * vt.y - xt.y * vt.x);   // conj(x) v
    const double2 half = cmul(make_double2(-0.5 * tau.x, -0.5 * tau.y), dp);
    if (tid < D) {
      vP[tid] = vt;
      wP[tid] = cfma(half, vt, xt);
    }
    __syncthreads();
  }
  // T times a power of two that brings its largest entry to [1/2, 1), which the spectrum step takes
  // back: the library's solver has absolute thresholds (a matrix of 2^-90 had eigenvalues off by
  // 1 % of their size).  What is not finite has no eigenvalues: zeros,
  // for matrix and reflectors.
  __syncthreads();
  const double td = tid < D ? dg[tid] : 0.0, te = tid < D - 1 ? e[tid] : 0.0;
  const double big = block_max(isfinite(td) && isfinite(te) ? fmax(fabs(td), fabs(te)) : INFINITY);
  int ex = 0;
  if (big < INFINITY) (void)frexp(big, &ex);
  if (tid == 0) {
    info[kInfoExp] = ex;
    info[kInfoBad] = big < INFINITY ? 0 : 1;
  }
  if (big < INFINITY && ex == 0) return;     // uniform
  if (tid < D) dg[tid] = big < INFINITY ? ldexp(td, -ex) : 0.0;
  if (tid < D - 1) e[tid] = big < INFINITY ? ldexp(te, -ex) : 0.0;
  if (big < INFINITY) return;
  for (int t = tid; t < D * D; t += kHetrdThreads) A[t] = make_double2(0.0, 0.0);
}

// B = Q B for the reflectors hetrd_kernel leaves in A: a wave takes a column of B into
// registers (lanes along the rows) and applies H_(D-2) .. H_0 to it; the reflectors come from
// L2, kAhead steps before their use.  Columns are independent, so no barrier at all; bound by
// a step's serial chain (dot product, its sum over the wave, update): 96 us at n = 8, where
// the library's blocked form took some 700.  (The library's blocked
// form divides by tau and returns NaN where a reflector is the identity, as for diagonal mu.)
template <int D>
__global__ __launch_bounds__(64) void unmtr_kernel(const double2* __restrict__ A, double2* __restrict__ B) {
  constexpr int CH = D / 64, kAhead = 4;
  const int lane = threadIdx.x;
  double2* col = B + (int64_t)blockIdx.x * D;
  double2 b[CH], v[kAhead][CH], tau[kAhead];
#pragma unroll
  for (int j = 0; j < CH; ++j) b[j] = col[64 * j + lane];
  auto load = [&](int i, double2 (&x)[CH], double2& t) __attribute__((always_inline)) {
    const int ic = i < 0 ? 0 : i;
#pragma unroll
    for (int j = 0; j < CH; ++j) x[j] = A[64 * j + lane + ic * D];
    t = A[ic + ic * D];
  };
#pragma unroll
  for (int k = 0; k < kAhead; ++k) load(D - 2 - k, v[k], tau[k]);
  for (int i0 = D - 2; i0 >= 0; i0 -= kAhead) {
#pragma unroll
    for (int k = 0; k < kAhead; ++k) {
      const int i = i0 - k;
      if (i >= 0) {                              // uniform
        double2 x[CH], dot = make_double2(0.0, 0.0);
#pragma unroll
        for (int j = 0; j < CH; ++j) {
          const int r = 64 * j + lane;
          x[j] = r > i + 1 ? v[k][j] : make_double2(r == i + 1 ? 1.0 : 0.0, 0.0);
          dot = cfma(conj2(x[j]), b[j], dot);
        }
        const double s = wave_sum4(dot.x, dot.y, 0.0, 0.0);
        const double2 f = cmul(make_double2(-tau[k].x, -tau[k].y), make_double2(__shfl(s, 0), __shfl(s, 32)));
#pragma unroll
        for (int j = 0; j < CH; ++j) b[j] = cfma(f, x[j], b[j]);
      }
      load(i - kAhead, v[k], tau[k]);
    }
  }
  // to unit length: the solver's vectors and the reflectors' rounding are off by some 1e-15
  double n2 = 0.0;
#pragma unroll
  for (int j = 0; j < CH; ++j) n2 += b[j].x * b[j].x + b[j].y * b[j].y;
  const double unit = 1.0 / sqrt(__shfl(wave_sum4(n2, 0.0, 0.0, 0.0), 0));
#pragma unroll
  for (int j = 0; j < CH; ++j) col[64 * j + lane] = make_double2(b[j].x * unit, b[j].y * unit);
}

template <int D>
void launch_hetrd(double2* A, double* dg, double* e, rocblas_int* info, hipStream_t st) {
  hipLaunchKernelGGL((hetrd_kernel<D>), dim3(1), dim3(kHetrdThreads), 0, st, A, dg, e, info);
}

template <int D>
void launch_unmtr(const double2* A, double2* B, hipStream_t st) {
  hipLaunchKernelGGL((unmtr_kernel<D>), dim3(D), dim3(64), 0, st, A, B);
}

// b[:, j] = a[:, j] * lam[j] (column-major d x d).  Eigenvectors that are not finite are a failure
// of the solver as well.
__global__ __launch_bounds__(256) void scale_columns_kernel(const double2* __restrict__ a,
                                                            const double* __restrict__ lam,
                                                            double2* __restrict__ b, int n,
                                                            rocblas_int* __restrict__ info,
                                                            uint32_t* __restrict__ flags) {
  const int64_t d = (int64_t)1 << n;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= d * d) return;
  const double s = lam[i >> n];
  const double2 v = a[i];
  b[i] = make_double2(v.x * s, v.y * s);
  if (!(isfinite(v.x) && isfinite(v.y))) {
    info[kInfoBad] = 1;
    lre::raise_flag(flags, lre::FLAG_EIG);
  }
}

// rho = 0 after a failure (the product of a failed solver's vectors need not be).
__global__ __launch_bounds__(256) void clear_failed_kernel(double2* __restrict__ rho, int64_t elems,
                                                           const rocblas_int* __restrict__ info) {
  if (info[kInfoBad] == 0) return;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < elems; i += (int64_t)gridDim.x * 256)
    rho[i] = make_double2(0.0, 0.0);
}

}  // namespace

namespace lre_detail {

void destroy_blas(void* handle) {
  if (handle) (void)rocblas_destroy_handle(static_cast<rocblas_handle>(handle));
}

}  // namespace lre_detail

extern "C" {

size_t lre_project_workspace_bytes(int n) {
  if (n < 1 || n > LRE_MAX_QUBITS) return 0;
  return proj_layout(n).total;
}

lre_status lre_project(lre_ctx* ctx, int n, const void* mu, void* rho, double* eigvals, void* workspace,
                       size_t workspace_bytes, void* stream) {
  if (!ctx || !mu || !rho || !workspace || n < 1 || n > LRE_MAX_QUBITS) return LRE_E_ARG;
  if (((uintptr_t)mu & 15u) || ((uintptr_t)rho & 15u) || ((uintptr_t)workspace & 255u) ||
      ((uintptr_t)eigvals & 7u))
    return LRE_E_ARG;
  const ProjLayout L = proj_layout(n);
  if (workspace_bytes < L.total) return LRE_E_WORKSPACE;
  DeviceGuard g(ctx->device);
  if (!g.ok) return LRE_E_HIP;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (n <= kJacobiN) {
    const auto* m = static_cast<const double2*>(mu);
    auto* r = static_cast<double2*>(rho);
    switch (n) {
      case 1: launch_jacobi<1>(m, r, eigvals, ctx->flags, st); break;
      case 2: launch_jacobi<2>(m, r, eigvals, ctx->flags, st); break;
      case 3: launch_jacobi<3>(m, r, eigvals, ctx->flags, st); break;
      case 4: launch_jacobi<4>(m, r, eigvals, ctx->flags, st); break;
      case 5: launch_jacobi<5>(m, r, eigvals, ctx->flags, st); break;
      default: launch_jacobi<6>(m, r, eigvals, ctx->flags, st); break;
    }
    return hipGetLastError() == hipSuccess ? LRE_OK : LRE_E_HIP;
  }
  if (!ctx->blas) {
    rocblas_handle h = nullptr;
    if (rocblas_create_handle(&h) != rocblas_status_success) return LRE_E_HIP;
    ctx->blas = h;
  }
  rocblas_handle h = static_cast<rocblas_handle>(ctx->blas);
  if (rocblas_set_stream(h, st) != rocblas_status_success) return LRE_E_HIP;

  const int d = 1 << n;
  char* ws = static_cast<char*>(workspace);
  auto* A = reinterpret_cast<rocblas_double_complex*>(ws + L.a);
  auto* B = reinterpret_cast<rocblas_double_complex*>(ws + L.b);
  auto* W = reinterpret_cast<double*>(ws + L.w);
  auto* E = reinterpret_cast<double*>(ws + L.e);
  auto* lam = reinterpret_cast<double*>(ws + L.lam);
  auto* info = reinterpret_cast<rocblas_int*>(ws + L.info);

  auto* V = A;                                  // eigenvectors
  auto* scaled = B;                             // and scaled by the new spectrum
  if (n <= kHetrdN) {
    auto* a2 = reinterpret_cast<double2*>(A);
    auto* b2 = reinterpret_cast<double2*>(B);
    hipLaunchKernelGGL(lower_copy_kernel, dim3((unsigned)(d / 16), (unsigned)(d / 16)), dim3(256), 0, st,
                       static_cast<const double2*>(mu), a2, d);
    if (n == 7) launch_hetrd<128>(a2, W, E, info, st);
    else launch_hetrd<256>(a2, W, E, info, st);
    if (hipGetLastError() != hipSuccess) return LRE_E_HIP;
    // eigenvectors of the tridiagonal matrix into B, then Q times them
    if (rocsolver_zstedc(h, rocblas_evect_tridiagonal, d, W, E, B, d, info) != rocblas_status_success)
      return LRE_E_HIP;
    if (n == 7) launch_unmtr<128>(a2, b2, st);
    else launch_unmtr<256>(a2, b2, st);
    V = B;
    scaled = A;
  } else if (hipMemcpyAsync(A, mu, (size_t)16 * d * d, hipMemcpyDeviceToDevice, st) != hipSuccess ||
             rocsolver_zheevd(h, rocblas_evect_original, rocblas_fill_upper, d, A, d, W, E, info) !=
             rocblas_status_success) {
    return LRE_E_HIP;
  }
  hipLaunchKernelGGL(spectrum_kernel, dim3(1), dim3(kSpectrumThreads), 0, st, W, lam, info, n <= kHetrdN, d,
                     ctx->flags, eigvals);
  const int64_t elems = (int64_t)d * d;
  hipLaunchKernelGGL(scale_columns_kernel, dim3((unsigned)((elems + 255) / 256)), dim3(256), 0, st,
                     reinterpret_cast<const double2*>(V), lam, reinterpret_cast<double2*>(scaled), n, info,
                     ctx->flags);
  if (hipGetLastError() != hipSuccess) return LRE_E_HIP;
  const rocblas_double_complex one = {1.0, 0.0}, zero = {0.0, 0.0};
  if (rocblas_zgemm(h, rocblas_operation_none, rocblas_operation_conjugate_transpose, d, d, d, &one, scaled, d, V,
                    d, &zero, static_cast<rocblas_double_complex*>(rho), d) != rocblas_status_success)
    return LRE_E_HIP;
  hipLaunchKernelGGL(clear_failed_kernel, dim3(256), dim3(256), 0, st, static_cast<double2*>(rho), elems,
                     static_cast<const rocblas_int*>(info));
  return hipGetLastError() == hipSuccess ? LRE_OK : LRE_E_HIP;
}

}  // extern "C"
