// lre_povm.hpp -- gfx950 kernels for LRE with the reduced measurement set of Sec. VI:
// one informationally complete set of four operators E_j per qubit (the same on every
// qubit), measured as 4^n product outcomes j = sum_k j_k 4^{n-k}.
//
// With G[j][a] = Tr(E_j sigma_a) (4 x 4), every Gamma^(j) is a tensor product of the
// one-qubit rows G[j_k][.] / sqrt 2, so X^T X = 2^-n (x)_k G^T G is a tensor product of
// dense 4 x 4 blocks (not diagonal as for the Pauli bases) and eq. (3) becomes
//   e = 2^{n/2} theta = ((x)_k M) p,   M = 2 (G^T G)^{-1} G^T,   p = c / N.
// The paper counts this as O(8^n) work; applied as n mode products of M it is
// O(n 4^n): every pass below applies M to a few digit positions of the 4^n vector,
// held in registers or LDS, and the last pass divides by N.  Passes work in place on
// the coefficient array (each block writes exactly the elements it read).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lre_kernels.hpp"

namespace lre {

// M from G (row-major 4 x 4) by Gauss-Jordan elimination with partial pivoting on
// G^T G in binary64; a (nearly) singular G^T G raises FLAG_ARG and leaves M = 0.
// Also clears the 64-bit total N that the first pass accumulates.  One wave: lane 8 r + c
// (of the first 32) holds element (r, c) of [G^T G | 1], rows move by lane shuffles (one thread with the
// matrix in scratch memory took 6.9 us).
static __global__ __launch_bounds__(64) void povm_setup_kernel(const double* __restrict__ G, double* __restrict__ M,
                                                               unsigned long long* __restrict__ total,
                                                               uint32_t* __restrict__ flags) {
  const int lane = threadIdx.x, r = (lane >> 3) & 3, c = lane & 7;
  if (lane == 0) *total = 0ull;
  const double g = G[lane & 15];               // (j, c) at lane 4 j + c
  double a = 0.0;
#pragma unroll
  for (int j = 0; j < 4; ++j) a += __shfl(g, 4 * j + r) * __shfl(g, 4 * j + (c & 3));
  double scale = c < 4 ? fabs(a) : 0.0;
  if (c >= 4) a = r == c - 4 ? 1.0 : 0.0;
#pragma unroll
  for (int o = 1; o < 32; o <<= 1) scale = fmax(scale, __shfl_xor(scale, o));
  bool ok = scale > 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    int piv = k;
    double best = fabs(__shfl(a, 9 * k));
#pragma unroll
    for (int q = k + 1; q < 4; ++q) {
      const double v = fabs(__shfl(a, 8 * q + k));
      if (v > best) { best = v; piv = q; }
    }
    ok = ok && best > 1e-12 * scale;
    a = __shfl(a, 8 * (r == k ? piv : (r == piv ? k : r)) + c);
    const double top = __shfl(a, 8 * k + c) / __shfl(a, 9 * k);   // row k, scaled
    const double f = __shfl(a, 8 * r + k);
    a = r == k ? top : a - f * top;
  }
  // M row i: 2 (G^T G)^{-1} G^T, lane 4 i + j
  const int i = (lane >> 2) & 3, j = lane & 3;
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) s += __shfl(a, 8 * i + k + 4) * __shfl(g, 4 * j + k);
  if (lane < 16) M[lane] = ok ? 2.0 * s : 0.0;
  if (!ok && lane == 0) raise_flag(flags, FLAG_ARG);
}

// N for the last of several passes.  Empty data (N = 0) is an error, as an empty basis is for
// the Pauli measurements; block 0 reports it.
__device__ __forceinline__ double povm_total(const unsigned long long* __restrict__ total,
                                             uint32_t* __restrict__ flags) {
  const unsigned long long N = *total;
  if (N == 0ull && blockIdx.x == 0 && threadIdx.x == 0) raise_flag(flags, FLAG_EMPTY);
  return (double)N;
}

// y <- M y on one digit: 4 values.
__device__ __forceinline__ void povm_apply1(const double (&m)[16], double* y, int stride) {
  const double y0 = y[0], y1 = y[stride], y2 = y[2 * stride], y3 = y[3 * stride];
#pragma unroll
  for (int r = 0; r < 4; ++r)
    y[r * stride] = m[4 * r] * y0 + m[4 * r + 1] * y1 + m[4 * r + 2] * y2 + m[4 * r + 3] * y3;
}

// y <- (M (x) ... (x) M) y on the F digits of a register block of 4^F values.
template <int F>
__device__ __forceinline__ void povm_apply_regs(const double (&m)[16], double* y) {
#pragma unroll
  for (int d = 0; d < F; ++d) {
    const int st = 1 << (2 * d);
#pragma unroll
    for (int base = 0; base < (1 << (2 * F)); ++base) {
      if ((base >> (2 * d)) & 3) continue;
      povm_apply1(m, y + base, st);
    }
  }
}

__device__ __forceinline__ void povm_load_m(const double* __restrict__ M, double (&m)[16]) {
#pragma unroll
  for (int k = 0; k < 16; ++k) m[k] = M[k];
}

// LDS index of tile element i: one pad slot every 16, so that the 16-value groups of
// the first stage (16 consecutive elements per thread) fall on different banks.
__device__ __forceinline__ constexpr int povm_pad(int i) { return i + (i >> 4); }

// J <= 5 qubits, the only pass: the 4^J counts in LDS, the J digits transformed two at a time
// in registers (one at a time for an odd J), then divided by their sum N and written to coef.
template <int J>
__global__ __launch_bounds__(256) void povm_low_kernel(const uint16_t* __restrict__ counts, double* __restrict__ coef,
                                                       const double* __restrict__ M, uint32_t* __restrict__ flags) {
  constexpr int T = 1 << (2 * J);
  __shared__ double tile[T + T / 16 + 1];
  __shared__ uint64_t part[4];
  double m[16];
  povm_load_m(M, m);
  uint64_t sum = 0;
  for (int i = threadIdx.x; i < T; i += 256) {
    const uint32_t c = counts[i];
    tile[povm_pad(i)] = (double)c;
    sum += c;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
  __syncthreads();
  const uint64_t bsum = part[0] + part[1] + part[2] + part[3];
  if (threadIdx.x == 0 && bsum == 0) raise_flag(flags, FLAG_EMPTY);
#pragma unroll
  for (int d = 0; d < J; d += 2) {
    const int nd = (J - d) >= 2 ? 2 : 1;          // digits in this stage
    const int G = T >> (2 * nd);                  // groups of 4^nd values
    for (int g = threadIdx.x; g < G; g += 256) {
      // element index: digits d, d+1 vary; the others come from g
      const int lo = g & ((1 << (2 * d)) - 1);
      const int hi = g >> (2 * d);
      const int i0 = (hi << (2 * (d + nd))) | lo;
      double y[16];
      const int st = 1 << (2 * d);
      if (nd == 2) {
#pragma unroll
        for (int k = 0; k < 16; ++k) y[k] = tile[povm_pad(i0 + (k & 3) * st + (k >> 2) * 4 * st)];
        povm_apply_regs<2>(m, y);
#pragma unroll
        for (int k = 0; k < 16; ++k) tile[povm_pad(i0 + (k & 3) * st + (k >> 2) * 4 * st)] = y[k];
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) y[k] = tile[povm_pad(i0 + k * st)];
        povm_apply1(m, y, 1);
#pragma unroll
        for (int k = 0; k < 4; ++k) tile[povm_pad(i0 + k * st)] = y[k];
      }
    }
    __syncthreads();
  }
  const double N = (double)bsum;
  for (int i = threadIdx.x; i < T; i += 256) coef[i] = tile[povm_pad(i)] / N;
}

// First pass for J = 6 and 7 digits: 4^J / 16 threads, tiles blockIdx.x, + gridDim.x, ...
// A thread takes 16 consecutive counts (two 16-byte loads; those of the block's next tile are
// loaded ahead) through the two lowest digits in registers; two further pairs of digits
// (J = 6: one) pass through LDS, and the last stage, two digits (J = 7: one) of 16 values a
// thread, stores straight to coef, consecutive threads to consecutive elements.  The barriers
// leave loads and stores in flight.  The block adds its counts to N (FINAL: its sum is N, and
// it divides).  Bound by memory: n = 12, J = 7: 41 us, 4.1 TB/s of reads and writes (tiles of
// 6 digits converted into LDS and written from there: 60 us, 2.8 TB/s).
template <int J>
struct PovmTileGeom {
  static constexpr int T = 1 << (2 * J), TH = T / 16;
};

template <int J, bool FINAL>
__global__ __launch_bounds__(PovmTileGeom<J>::TH) void povm_tile_kernel(const uint16_t* __restrict__ counts,
                                                                       double* __restrict__ coef,
                                                                       const double* __restrict__ M,
                                                                       unsigned long long* __restrict__ total,
                                                                       uint32_t* __restrict__ flags, int tiles) {
  static_assert(J == 6 || J == 7, "the stages below");
  constexpr int T = PovmTileGeom<J>::T, TH = PovmTileGeom<J>::TH;
  __shared__ double tile[T + T / 16];
  __shared__ uint64_t part[TH / 64];
  const int t = threadIdx.x;
  double m[16];
  povm_load_m(M, m);
  uint64_t sum = 0;
  uint4 raw[2];
  auto load = [&](int b) __attribute__((always_inline)) {
    const uint4* __restrict__ p = reinterpret_cast<const uint4*>(counts + (int64_t)b * T) + 2 * t;
    raw[0] = p[0];
    raw[1] = p[1];
  };
  load(blockIdx.x);
  for (int b = blockIdx.x; b < tiles; b += gridDim.x) {
    double y[16];
    uint32_t s = 0;
    const uint32_t w[8] = {raw[0].x, raw[0].y, raw[0].z, raw[0].w, raw[1].x, raw[1].y, raw[1].z, raw[1].w};
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint32_t lo = w[k] & 0xFFFFu, hi = w[k] >> 16;
      y[2 * k] = (double)lo;
      y[2 * k + 1] = (double)hi;
      s += lo + hi;
    }
    sum += s;
    if (b + (int)gridDim.x < tiles) load(b + gridDim.x);
    povm_apply_regs<2>(m, y);
    if (b != (int)blockIdx.x) lds_barrier();     // the previous tile's last stage has read
#pragma unroll
    for (int k = 0; k < 16; ++k) tile[17 * t + k] = y[k];
    lds_barrier();
    // digits 2, 3 (and 4, 5 of 7): in place
#pragma unroll
    for (int d = 2; d < (J == 7 ? 6 : 4); d += 2) {
      const int st = 1 << (2 * d);
      const int i0 = ((t >> (2 * d)) << (2 * d + 4)) | (t & (st - 1));
#pragma unroll
      for (int k = 0; k < 16; ++k) y[k] = tile[povm_pad(i0) + k * povm_pad(st)];
      povm_apply_regs<2>(m, y);
#pragma unroll
      for (int k = 0; k < 16; ++k) tile[povm_pad(i0) + k * povm_pad(st)] = y[k];
      lds_barrier();
    }
    double N = 1.0;
    if constexpr (FINAL) {                       // one tile, one block
      uint64_t all = sum;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) all += __shfl_xor(all, o, 64);
      if ((t & 63) == 0) part[t >> 6] = all;
      __syncthreads();
      all = 0;
      for (int k = 0; k < TH / 64; ++k) all += part[k];
      if (t == 0 && all == 0) raise_flag(flags, FLAG_EMPTY);
      N = (double)all;
    }
    double* __restrict__ out = coef + (int64_t)b * T;
    if constexpr (J == 6) {
#pragma unroll
      for (int k = 0; k < 16; ++k) y[k] = tile[povm_pad(t) + k * povm_pad(TH)];
      povm_apply_regs<2>(m, y);
    } else {                                     // y[4 q + k]: element t + TH q + 4 TH k
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int k = 0; k < 4; ++k) y[4 * q + k] = tile[povm_pad(t) + (q + 4 * k) * povm_pad(TH)];
        povm_apply1(m, y + 4 * q, 1);
      }
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int i = t + TH * (J == 6 ? k : (k >> 2) + 4 * (k & 3));
      out[i] = FINAL ? y[k] / N : y[k];
    }
  }
  if constexpr (!FINAL) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if ((t & 63) == 0) part[t >> 6] = sum;
    __syncthreads();
    if (t == 0) {
      uint64_t all = 0;
      for (int k = 0; k < TH / 64; ++k) all += part[k];
      atomicAdd(total, (unsigned long long)all);
    }
  }
}

// The last five digits lo .. lo + 4 (2 <= lo <= 9) of the vector, in place: tiles of 16 consecutive low
// indices (one 128-byte line a row) x the 1024 values of the five digits, 128 KiB of LDS, tiles
// blockIdx.x, + gridDim.x, ...  A thread loads 16 rows of one column straight into the first
// two digits' registers (the block's next tile is loaded ahead), the next two digits pass
// through LDS and the fifth, divided by N, stores to coef.  Bound by memory: n = 12, one
// pass of 49 us, 5.5 TB/s, where passes of 4 and 2 digits took 43 + 45.
constexpr int kPovmWideCols = 16;

// Rows of one half-wave's access differ in one digit bit: it picks the half of the banks.
__device__ __forceinline__ constexpr int povm_wide_row(int row) {
  return row ^ ((row >> 2 ^ row >> 4 ^ row >> 6 ^ row >> 8) & 1);
}

// Slots of rows base + k for the constants k of one stage (no bit of k set in base but bit 0):
// povm_wide_row is linear over the bits, so two addresses serve, picked by its bit 0 at k.
struct PovmWideSlots {
  int e0, e1;
  __device__ __forceinline__ PovmWideSlots(int base, int col)
      : e0(povm_wide_row(base) * kPovmWideCols + col), e1((povm_wide_row(base) ^ 1) * kPovmWideCols + col) {}
  __device__ __forceinline__ int operator()(int k) const {
    return ((povm_wide_row(k) & 1) ? e1 : e0) + (k & ~1) * kPovmWideCols;
  }
};

static __global__ __launch_bounds__(1024) void povm_high5_kernel(double* __restrict__ coef, int lo, const double* __restrict__ M,
                                                         const unsigned long long* __restrict__ total,
                                                         uint32_t* __restrict__ flags, int64_t tiles) {
  __shared__ double blk[1024 * kPovmWideCols];
  double m[16];
  povm_load_m(M, m);
  const double N = povm_total(total, flags);
  const int64_t L = (int64_t)1 << (2 * lo);
  const int gshift = 2 * lo - 4;                       // log2 of the tiles per high index
  const int col = threadIdx.x % kPovmWideCols, o = threadIdx.x / kPovmWideCols;   // o: 64 values
  // Addresses: a uniform part and a 32-bit byte offset per thread.
  auto tile_base = [&](int64_t b) __attribute__((always_inline)) {
    return reinterpret_cast<char*>(coef + (b >> gshift) * (L << 10) + (b & (((int64_t)1 << gshift) - 1)) * kPovmWideCols);
  };
  const uint32_t Lb = (uint32_t)(L * 8);
  const uint32_t off_in = (uint32_t)(((int64_t)o * 16 * L + col) * 8), off_out = (uint32_t)(((int64_t)o * L + col) * 8);
  const PovmWideSlots s0(16 * o, col), s2(((o >> 4) << 8) | (o & 15), col), s4(o, col);
  double pre[16];
  auto load = [&](int64_t b) __attribute__((always_inline)) {
    uint32_t off = off_in;
    asm volatile("" : "+v"(off));                      // not sixteen offsets kept over the loop
#pragma unroll
    for (int k = 0; k < 16; ++k) pre[k] = *reinterpret_cast<const double*>(tile_base(b) + (off + k * Lb));
  };
  load(blockIdx.x);
  for (int64_t b = blockIdx.x; b < tiles; b += gridDim.x) {
    double y[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) y[k] = pre[k];
    povm_apply_regs<2>(m, y);                          // rows 16 o + k: digits 0, 1
    if (b + gridDim.x < tiles) load(b + gridDim.x);
    if (b != (int64_t)blockIdx.x) lds_barrier();       // the previous tile's last stage has read
#pragma unroll
    for (int k = 0; k < 16; ++k) blk[s0(k)] = y[k];
    lds_barrier();
    // digits 2, 3
#pragma unroll
    for (int k = 0; k < 16; ++k) y[k] = blk[s2(16 * k)];
    povm_apply_regs<2>(m, y);
#pragma unroll
    for (int k = 0; k < 16; ++k) blk[s2(16 * k)] = y[k];
    lds_barrier();
    uint32_t off = off_out;
    asm volatile("" : "+v"(off));
#pragma unroll
    for (int q = 0; q < 4; ++q) {                      // digit 4: rows o + 64 q + 256 k
      double z[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) z[k] = blk[s4(64 * q + 256 * k)];
      povm_apply1(m, z, 1);
#pragma unroll
      for (int k = 0; k < 4; ++k) *reinterpret_cast<double*>(tile_base(b) + (off + (64 * q + 256 * k) * Lb)) = z[k] / N;
    }
  }
}

// Four digits lo .. lo + 3 (lo >= 3) of the vector, in place: a block holds 32
// consecutive low indices (columns) x the 256 values of the four digits in LDS (64 KiB,
// two blocks per compute unit), transforms them two digits at a time in registers;
// FINAL divides by N.
constexpr int kPovmCols = 32;
constexpr int kPovmHighThreads = 512;

template <bool FINAL>
__global__ __launch_bounds__(kPovmHighThreads) void povm_high4_kernel(double* __restrict__ coef, int n, int lo,
                                                                      const double* __restrict__ M,
                                                                      const unsigned long long* __restrict__ total,
                                                                      uint32_t* __restrict__ flags) {
  constexpr int TH = kPovmHighThreads, RPP = TH / kPovmCols;   // rows of 256 loaded per pass
  __shared__ double blk[256 * kPovmCols];
  double m[16];
  povm_load_m(M, m);
  const int64_t L = (int64_t)1 << (2 * lo);            // low indices
  const int64_t colgroups = L / kPovmCols;
  const int64_t hi = blockIdx.x / colgroups;
  const int64_t c0 = (blockIdx.x % colgroups) * kPovmCols;
  double* __restrict__ base = coef + hi * (L << 8) + c0;
  const int col = threadIdx.x % kPovmCols, r0 = threadIdx.x / kPovmCols;
  double v[256 / RPP];
#pragma unroll
  for (int k = 0; k < 256 / RPP; ++k) v[k] = base[(int64_t)(r0 + RPP * k) * L + col];
#pragma unroll
  for (int k = 0; k < 256 / RPP; ++k) blk[(r0 + RPP * k) * kPovmCols + col] = v[k];
  __syncthreads();
#pragma unroll
  for (int stage = 0; stage < 2; ++stage) {
    // units: (column, the other two digits) = 32 x 16, one per thread
    for (int u = threadIdx.x; u < kPovmCols * 16; u += TH) {
      const int c = u % kPovmCols, other = u / kPovmCols;
      double y[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const int d = stage == 0 ? (other << 4) | k : (k << 4) | other;
        y[k] = blk[d * kPovmCols + c];
      }
      povm_apply_regs<2>(m, y);
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const int d = stage == 0 ? (other << 4) | k : (k << 4) | other;
        blk[d * kPovmCols + c] = y[k];
      }
    }
    __syncthreads();
  }
  const double N = FINAL ? povm_total(total, flags) : 1.0;
#pragma unroll
  for (int k = 0; k < 256 / RPP; ++k) {
    const int d = r0 + RPP * k;
    base[(int64_t)d * L + col] = FINAL ? blk[d * kPovmCols + col] / N : blk[d * kPovmCols + col];
  }
}

// F <= 3 digits lo .. lo + F - 1 in registers, one thread per column (every other
// digit), in place; FINAL divides by N.
template <int F, bool FINAL>
__global__ __launch_bounds__(256) void povm_reg_kernel(double* __restrict__ coef, int n, int lo,
                                                       const double* __restrict__ M,
                                                       const unsigned long long* __restrict__ total,
                                                       uint32_t* __restrict__ flags) {
  const int64_t L = (int64_t)1 << (2 * lo);
  const int64_t cols = ((int64_t)1 << (2 * (n - F)));
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= cols) return;
  double m[16];
  povm_load_m(M, m);
  const int64_t low = t & (L - 1), hi = t >> (2 * lo);
  double* __restrict__ p = coef + hi * (L << (2 * F)) + low;
  double y[1 << (2 * F)];
#pragma unroll
  for (int k = 0; k < (1 << (2 * F)); ++k) y[k] = p[(int64_t)k * L];
  povm_apply_regs<F>(m, y);
  const double N = FINAL ? povm_total(total, flags) : 1.0;
#pragma unroll
  for (int k = 0; k < (1 << (2 * F)); ++k) p[(int64_t)k * L] = FINAL ? y[k] / N : y[k];
}

}  // namespace lre
