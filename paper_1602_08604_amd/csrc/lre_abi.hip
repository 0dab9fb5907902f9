// lre_abi.hip -- the C ABI declared in include/lre.h: argument checks, pass planning,
// workspace layout and kernel launches.  All arithmetic runs in lre_kernels.hpp.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "lre.h"
#include "lre_internal.hpp"
#include "lre_kernels.hpp"
#include "lre_povm.hpp"
#include "lre_tile.hpp"

using namespace lre;
using lre_detail::aligned;
using lre_detail::DeviceGuard;
using lre_detail::record_stage;


// Workspace of lre_estimate_noalloc: one copy per device, held until the process
// ends.  Host code never passes this name to a kernel (on the host it is a stand-in,
// not a device address); it uses the per-device address lre_create resolves with
// hipGetSymbolAddress, kept in lre_ctx::scratch.
static __device__ __align__(256) char scratch[LRE_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int kMaxQ1 = 7;     // qubits folded by the int8-MFMA counts pass and lre_signed_sums
constexpr int kSmallN = 5;    // up to this many qubits one workgroup does everything
constexpr int kMaxTail = 4;   // qubits folded by the pass that ends a plan (fold_tail_kernel)
constexpr int kRhoJ = 6;      // qubits of the low step-(ii) transform
// Step (ii) goes through a complex128 intermediate of 4^n entries only beyond 12 qubits
// (up to 10 the LDS tiles, at 11 and 12 the real-arithmetic tiles need none).
constexpr bool rho_needs_tmp(int n) { return n > kRhoJ + 6; }

enum class Ty : int { U32 = 0, F64 = 1 };

size_t ty_size(Ty t) { return t == Ty::U32 ? 4 : 8; }
size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

struct Plan {
  int n = 0;
  bool per_basis = false;
  bool mfma = false;         // counts pass on int8 MFMA
  int q1 = 0;                // qubits folded by the counts pass
  int chunks = 1;            // MFMA form: tiles per counts-pass block, one row group's
  int64_t runs = 1;          // tiles (MFMA form: blocks) along a row
  int64_t per_block = 0;     // tiles per counts-pass block (0: one, or the MFMA form)
  int64_t blocks1 = 0;       // counts-pass blocks
  int64_t parts = 0;         // row-sum parts, of 3^q1 words
  Ty t1 = Ty::U32;           // counts-pass accumulator / output type
  int npass = 0;             // later passes
  int F[4] = {0};
  Ty tout[4] = {Ty::U32};
  size_t off_a = 0, off_b = 0, off_rowpart = 0, off_nb = 0, off_tmp = 0, total = 0;
};

// Partial sums after folding f qubits are bounded by 3^f * (basis total).
Ty int_type_for(int folded, uint64_t shots) {
  long double bound = (long double)shots;
  for (int i = 0; i < folded; ++i) bound *= 3.0L;
  return bound <= (long double)INT32_MAX ? Ty::U32 : Ty::F64;
}

// Qubits the counts pass folds (n > kSmallN): enough that the passes after it stay short,
// as long as its workgroups fill the chip.
int counts_qubits(int n, bool mfma) {
  if (mfma) return kMaxQ1;
  return n <= 8 ? 5 : (n == 9 ? 6 : 7);
}

bool make_plan_form(int n, uint64_t shots, uint32_t flags, bool mfma, Plan& P) {
  P = Plan();
  P.n = n;
  P.per_basis = shots == 0;
  P.mfma = mfma;
  const size_t tmp = (!(flags & LRE_NO_RHO) && rho_needs_tmp(n)) ? (size_t)ipow4(n) * 16 : 0;
  if (n <= kSmallN) {
    P.total = 256;
    return true;
  }
  P.q1 = counts_qubits(n, mfma);
  const int64_t row_groups = ipow3(n - P.q1);
  if (mfma) {
    const int64_t tiles_per_row = (int64_t)1 << (n - kMaxQ1);
    int64_t chunks = 1;
    while (chunks * 2 <= tiles_per_row && chunks < 16 &&
           row_groups * (tiles_per_row / (chunks * 2)) >= 1024)
      chunks *= 2;
    P.chunks = (int)chunks;
    P.runs = tiles_per_row / chunks;
    P.blocks1 = P.parts = row_groups * P.runs;
  } else {
    // outcomes of a tile: 2^q1, or the 64 of a sub-tile where a tile folds fewer than 6 bits
    P.runs = (int64_t)1 << (n - (P.q1 < 6 ? 6 : P.q1));
    const int64_t tiles = row_groups * P.runs;
    P.blocks1 = P.parts = tiles;
    if (P.q1 > 5) {
      // Blocks of equal numbers of tiles: one per workgroup the chip holds, or, where that
      // makes 24 tiles each, blocks of 8, so that unequal speeds even out and neighbouring
      // blocks read near each other (step (i) alone, n = 13: 6.67 ms against 6.79 at 23 tiles;
      // n = 12 with totals: 1320 us against 1340 at 31; without, 15 tiles: 1085 against 1093).
      const int64_t slots = P.per_basis ? 256 : 512;
      P.per_block = tiles >= 24 * slots ? 8 : (tiles + slots - 1) / slots;
      P.blocks1 = (tiles + P.per_block - 1) / P.per_block;
      P.parts = row_groups + P.blocks1;
    }
  }
  P.t1 = P.per_basis ? Ty::F64 : int_type_for(P.q1, shots);

  // Later passes: up to 4 remaining qubits in one pass; more (n >= 12) as 4 with LDS
  // accumulators, then the remaining 1..3 in registers, which reads and writes far less
  // than 3 + 2 + 2 (53 GB instead of 70 GB of partials at n = 14).
  const int h = n - P.q1;
  if (h > kMaxTail) {
    P.npass = 2;
    P.F[0] = 4;
    P.F[1] = h - 4;
  } else if (h > 0) {
    P.npass = 1;
    P.F[0] = h;
  }
  int folded = P.q1;
  Ty prev = P.t1;
  for (int k = 0; k < P.npass; ++k) {
    folded += P.F[k];
    Ty t = P.per_basis ? Ty::F64 : int_type_for(folded, shots);
    if (prev == Ty::F64) t = Ty::F64;
    P.tout[k] = t;
    prev = t;
  }

  // Workspace: partial buffers A (counts pass) and B (first of two later passes).
  const size_t sizeA = P.npass > 0 ? (size_t)(ipow3(h) << h) * (size_t)ipow4(P.q1) * ty_size(P.t1) : 0;
  const int h2 = h - P.F[0];
  const size_t sizeB =
      P.npass > 1 ? (size_t)(ipow3(h2) << h2) * (size_t)ipow4(n - h2) * ty_size(P.tout[0]) : 0;
  const size_t rowpart = (size_t)P.parts * (size_t)ipow3(P.q1) * 4;

  size_t off = 0;
  P.off_a = off; off += align256(sizeA);
  P.off_b = off; off += align256(sizeB);
  P.off_rowpart = off; off += align256(rowpart);
  P.off_nb = off; off += align256(P.per_basis ? (size_t)ipow3(n) * 4 : 0);
  if (tmp && tmp <= sizeA) P.off_tmp = P.off_a;        // partials are dead by then
  else if (tmp && tmp <= sizeB) P.off_tmp = P.off_b;
  else { P.off_tmp = off; off += align256(tmp); }
  P.total = off;
  return true;
}

bool make_plan(int n, uint64_t shots, uint32_t flags, Plan& P) {
  if (n < 1 || n > LRE_MAX_QUBITS) return false;
  // A workspace serves both forms of the counts pass, whichever it was sized for.
  Plan other;
  const bool mfma = (flags & LRE_WHT_MFMA) && n >= kMaxQ1;
  if (n >= kMaxQ1) make_plan_form(n, shots, flags, !mfma, other);
  make_plan_form(n, shots, flags, mfma, P);
  P.total = std::max(P.total, other.total);
  return true;
}

// Blocks of `kernel` the device holds at once (compute units x resident blocks per
// unit); a persistent grid of this size has no second wave of blocks.
// lds_bytes: the kernel's static LDS, which bounds the count to 160 KiB per unit.
template <class K>
int64_t resident_blocks(K kernel, int threads, int64_t lds_bytes) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    cus = 256;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || per_cu <= 0)
    per_cu = 1;
  const int64_t by_lds = std::max<int64_t>(1, (160 * 1024) / std::max<int64_t>(1, lds_bytes));
  return (int64_t)cus * std::min<int64_t>(per_cu, by_lds);
}

// ---- launch helpers -------------------------------------------------------------

// A counts pass: nseg segments (blockIdx.y), counts advancing by seg_counts per segment,
// out by seg_out elements and rowpart by seg_row words.
struct Fold1Args {
  const uint16_t* counts;
  int n, chunks;
  int lrow;             // log2 of the row stride of counts (n for a whole instance)
  const uint32_t* nb;   // per-basis totals (NULL: formed in the pass, kept in nb_own)
  uint32_t* nb_own;
  void* out;
  uint32_t* rowpart;
  uint64_t shots;
  int64_t tiles, per_block, blocks;
  int nseg;
  int64_t seg_counts, seg_out, seg_row;
  hipStream_t st;
};

template <int LV, bool PB, typename Acc, bool NT>
void launch_tile(const Fold1Args& a) {
  const dim3 grid((unsigned)a.blocks, (unsigned)a.nseg);
  if constexpr (LV == 0)
    hipLaunchKernelGGL((counts_subtile_kernel<PB, Acc>), grid, dim3(256), 0, a.st, a.counts, a.n, a.lrow, a.nb,
                       a.nb_own, static_cast<Acc*>(a.out), a.rowpart, a.seg_counts, a.seg_out, a.seg_row);
  else
    hipLaunchKernelGGL((counts_tile_kernel<LV, PB, Acc, NT>), grid, dim3(512), 0, a.st, a.counts, a.n, a.lrow, a.tiles,
                       a.per_block, a.nb, static_cast<Acc*>(a.out), a.rowpart, a.seg_counts, a.seg_out, a.seg_row);
}

template <int LV, bool NT>
void tile_uniform(Ty t, const Fold1Args& a) {
  if (t == Ty::U32) launch_tile<LV, false, uint32_t, NT>(a);
  else launch_tile<LV, false, double, NT>(a);
}

// Partials of uniform shots beyond 1 GiB (n = 13 and 14) are out of the 256 MB cache before they
// are read again: with the nontemporal hint whole calls take n = 13 7.32 instead of 7.39 ms, n = 14
// 39.3 instead of 40.9; n = 12, 0.5 GB, 1190 instead of 1155 us.
template <int LV>
void tile_lv(Ty t, bool pb, const Fold1Args& a) {
  if (pb) return launch_tile<LV, true, double, tile_nt(LV, true)>(a);
  if constexpr (LV == 2)
    if ((size_t)a.seg_out * ty_size(t) > (size_t)1 << 30) return tile_uniform<LV, true>(t, a);
  tile_uniform<LV, tile_nt(LV, false)>(t, a);
}

bool fold1(int q, Ty t, bool pb, const Fold1Args& a) {
  switch (q) {
    case 5: tile_lv<0>(t, pb, a); return true;
    case 6: tile_lv<1>(t, pb, a); return true;
    case 7: tile_lv<2>(t, pb, a); return true;
    default: return false;
  }
}

template <typename Acc, bool PB, Out M>
void launch_fold1_mfma(const Fold1Args& a) {
  constexpr int TH = sizeof(Acc) == 8 ? 512 : 256;
  hipLaunchKernelGGL((fold_counts_mfma_kernel<TH, Acc, PB, M>), dim3((unsigned)a.blocks), dim3(TH), 0,
                     a.st, a.counts, a.n, a.chunks, a.nb, a.out, a.rowpart, a.shots, a.lrow);
}

bool fold1_mfma(Ty t, bool pb, Out m, const Fold1Args& a) {
  if (pb) {
    if (m == Out::Partial) launch_fold1_mfma<double, true, Out::Partial>(a);
    else if (m == Out::CoefPerBasis) launch_fold1_mfma<double, true, Out::CoefPerBasis>(a);
    else return false;
    return true;
  }
  if (t == Ty::U32) {
    switch (m) {
      case Out::Partial: launch_fold1_mfma<uint32_t, false, Out::Partial>(a); return true;
      case Out::CoefUniform: launch_fold1_mfma<uint32_t, false, Out::CoefUniform>(a); return true;
      case Out::PauliT: launch_fold1_mfma<uint32_t, false, Out::PauliT>(a); return true;
      default: return false;
    }
  }
  switch (m) {
    case Out::Partial: launch_fold1_mfma<double, false, Out::Partial>(a); return true;
    case Out::CoefUniform: launch_fold1_mfma<double, false, Out::CoefUniform>(a); return true;
    case Out::PauliT: launch_fold1_mfma<double, false, Out::PauliT>(a); return true;
    default: return false;
  }
}

// A later pass folding F qubits of [3^h][2^h][4^l], nseg segments (blockIdx.y); chk: row
// totals to check in the same launch (nbases 0: none).
struct FoldArgs {
  const void* in;
  void* out;
  int n, h, l;
  uint64_t shots;
  int nseg;
  int64_t seg_in, seg_out;
  RowCheck chk;
  hipStream_t st;
};

template <int F, typename Tin, typename Acc, Out M>
void launch_tail(const FoldArgs& a) {
  using G = FoldTailGeom<F>;
  const int64_t blocks = (ipow3(a.h - F) << (a.h - F)) * (ipow4(a.l) / G::COLS);
  const int64_t checks = (a.chk.nbases + G::THREADS - 1) / G::THREADS;
  hipLaunchKernelGGL((fold_tail_kernel<F, Tin, Acc, M>), dim3((unsigned)(blocks + checks), (unsigned)a.nseg),
                     dim3(G::THREADS), 0, a.st, static_cast<const Tin*>(a.in), a.out, a.n, a.h, a.l, a.shots, blocks,
                     a.seg_in, a.seg_out, a.chk);
}

template <int F, typename Tin, typename Acc>
void tail_m(Out m, const FoldArgs& a) {
  switch (m) {
    case Out::Partial: launch_tail<F, Tin, Acc, Out::Partial>(a); break;
    case Out::CoefUniform: launch_tail<F, Tin, Acc, Out::CoefUniform>(a); break;
    case Out::CoefPerBasis: launch_tail<F, Tin, Acc, Out::CoefPerBasis>(a); break;
    case Out::PauliT: launch_tail<F, Tin, Acc, Out::PauliT>(a); break;
  }
}

template <int F>
bool tail_f(Ty tin, Ty tacc, Out m, const FoldArgs& a) {
  if (tin == Ty::U32 && tacc == Ty::U32) tail_m<F, uint32_t, uint32_t>(m, a);
  else if (tin == Ty::U32) tail_m<F, uint32_t, double>(m, a);
  else if (tacc == Ty::F64) tail_m<F, double, double>(m, a);
  else return false;
  return true;
}

// Element i of an output of mode M.
template <typename Acc, Out M>
void* elem_at(void* out, int64_t i) {
  if constexpr (M == Out::Partial) return static_cast<Acc*>(out) + i;
  else return static_cast<double*>(out) + i;     // coefficients and T: 8 bytes
}

template <int F, typename Tin, typename Acc, Out M>
void launch_foldk(const FoldArgs& a) {
  const int64_t ncols = (ipow3(a.h - F) << (a.h - F)) * ipow4(a.l);
  for (int s = 0; s < a.nseg; ++s)
    hipLaunchKernelGGL((fold_partial_kernel<F, Tin, Acc, M>), dim3((unsigned)((ncols + 255) / 256)), dim3(256), 0, a.st,
                       static_cast<const Tin*>(a.in) + s * a.seg_in, elem_at<Acc, M>(a.out, s * a.seg_out), a.n, a.h,
                       a.l, a.shots, ncols);
}

template <typename Tin, typename Acc>
void launch_fold4(const FoldArgs& a) {
  // Persistent blocks: as many as the device holds at once, each walking
  // groups with a stride of the grid.
  const int64_t groups = (ipow3(a.h - 4) << (a.h - 4)) * (((int64_t)1 << (2 * a.l)) / kF4Cols);
  const int64_t cap = resident_blocks(fold_partial4_kernel<Tin, Acc>, 64 * kF4Waves,
                                      (int64_t)256 * kF4Cols * (int64_t)sizeof(Acc));
  const int64_t blocks = groups < cap ? groups : cap;
  for (int s = 0; s < a.nseg; ++s)
    hipLaunchKernelGGL((fold_partial4_kernel<Tin, Acc>), dim3((unsigned)blocks), dim3(64 * kF4Waves), 0, a.st,
                       static_cast<const Tin*>(a.in) + s * a.seg_in, static_cast<Acc*>(a.out) + s * a.seg_out, a.h,
                       a.l);
}

// The two passes of a plan with more than kMaxTail qubits left: large instances, a launch
// per segment.
template <typename Tin, typename Acc>
bool two_pass_t(int F, bool last, Out m, const FoldArgs& a) {
  if (!last) {
    launch_fold4<Tin, Acc>(a);
    return F == 4;
  }
  auto run = [&](auto fc) {
    constexpr int FF = decltype(fc)::value;
    switch (m) {
      case Out::Partial: launch_foldk<FF, Tin, Acc, Out::Partial>(a); break;
      case Out::CoefUniform: launch_foldk<FF, Tin, Acc, Out::CoefUniform>(a); break;
      case Out::CoefPerBasis: launch_foldk<FF, Tin, Acc, Out::CoefPerBasis>(a); break;
      case Out::PauliT: launch_foldk<FF, Tin, Acc, Out::PauliT>(a); break;
    }
  };
  if (F == 1) run(std::integral_constant<int, 1>{});
  else if (F == 2) run(std::integral_constant<int, 2>{});
  else if (F == 3) run(std::integral_constant<int, 3>{});
  else return false;
  return true;
}

bool two_pass(int F, bool last, Ty tin, Ty tacc, Out m, const FoldArgs& a) {
  if (tin == Ty::U32 && tacc == Ty::U32) return two_pass_t<uint32_t, uint32_t>(F, last, m, a);
  if (tin == Ty::U32) return two_pass_t<uint32_t, double>(F, last, m, a);
  return tacc == Ty::F64 && two_pass_t<double, double>(F, last, m, a);
}

bool fold_tail(int F, Ty tin, Ty tacc, Out m, const FoldArgs& a) {
  switch (F) {
    case 1: return tail_f<1>(tin, tacc, m, a);
    case 2: return tail_f<2>(tin, tacc, m, a);
    case 3: return tail_f<3>(tin, tacc, m, a);
    case 4: return tail_f<4>(tin, tacc, m, a);
    default: return false;
  }
}

// Persistent high transform: as many blocks as the LDS lets the device hold.
template <int H, typename OutT>
void launch_rho_high2(const double2* tmp, void* rho, int n, hipStream_t st) {
  using G = RhoHigh2Geom<H>;
  const int64_t items = ((int64_t)1 << H) * G::D * (G::D / G::XB);
  const int64_t blocks =
      std::min<int64_t>(items, resident_blocks(rho_high2_kernel<H, OutT>, 256, 2LL * G::NH * G::SP * 8));
  hipLaunchKernelGGL((rho_high2_kernel<H, OutT>), dim3((unsigned)blocks), dim3(256), 0, st, tmp, rho, n, items);
}

template <int H, int JB, typename OutT>
void launch_rho_real(const double* coef, void* rho, hipStream_t st) {
  using G = RhoRealGeom<H, JB>;
  const int64_t blocks = std::min<int64_t>(
      G::UNITS, resident_blocks(rho_real_tile_kernel<H, JB, OutT>, 512, (int64_t)G::NVP * 8));
  hipLaunchKernelGGL((rho_real_tile_kernel<H, JB, OutT>), dim3((unsigned)blocks), dim3(512), 0, st, coef, rho);
}

template <typename OutT>
void launch_rho(const Plan& P, const double* coef, void* rho, char* ws, hipStream_t st) {
  const int n = P.n;
  if (n < kRhoJ) {
    switch (n) {
#define LRE_RHO_SMALL(J) \
  case J: hipLaunchKernelGGL((rho_low_kernel<J, true, OutT>), dim3(1), dim3(256), 0, st, coef, rho, n); break;
      LRE_RHO_SMALL(1) LRE_RHO_SMALL(2) LRE_RHO_SMALL(3) LRE_RHO_SMALL(4) LRE_RHO_SMALL(5)
#undef LRE_RHO_SMALL
    }
    return;
  }
  if (n - kRhoJ <= 4) {
    // up to 4 high qubits: units (x_hi, 8 x_lo) from coefficients to mu in LDS
    const dim3 grid((unsigned)((int64_t)8 << (n - kRhoJ)));
    switch (n - kRhoJ) {
      case 0: hipLaunchKernelGGL((rho_tile_kernel<0, OutT>), grid, dim3(512), 0, st, coef, rho); break;
      case 1: hipLaunchKernelGGL((rho_tile_kernel<1, OutT>), grid, dim3(512), 0, st, coef, rho); break;
      case 2: hipLaunchKernelGGL((rho_tile_kernel<2, OutT>), grid, dim3(512), 0, st, coef, rho); break;
      case 3: hipLaunchKernelGGL((rho_tile_kernel<3, OutT>), grid, dim3(512), 0, st, coef, rho); break;
      default: hipLaunchKernelGGL((rho_tile_kernel<4, OutT>), grid, dim3(512), 0, st, coef, rho); break;
    }
    return;
  }
  if (n - kRhoJ <= 6) {
    // 5 or 6 high qubits: real-arithmetic units (x_hi, 8 or 4 x_lo), no intermediate
    if (n - kRhoJ == 5) launch_rho_real<5, 3, OutT>(coef, rho, st);
    else launch_rho_real<6, 2, OutT>(coef, rho, st);
    return;
  }
  double2* tmp = reinterpret_cast<double2*>(ws + P.off_tmp);
  const int64_t nblk = ipow4(n - kRhoJ);
  const int64_t low_blocks = std::min<int64_t>(nblk, resident_blocks(rho_low6_kernel, 256, 4096 * 8));
  hipLaunchKernelGGL(rho_low6_kernel, dim3((unsigned)low_blocks), dim3(256), 0, st, coef, tmp, nblk);
  // 7..9 high qubits: two register phases with one LDS transpose
  switch (n - kRhoJ) {
    case 7: launch_rho_high2<7, OutT>(tmp, rho, n, st); break;
    case 8: launch_rho_high2<8, OutT>(tmp, rho, n, st); break;
    default: launch_rho_high2<9, OutT>(tmp, rho, n, st); break;   // n = 15 (streamed estimates)
  }
}


// Row sums of `nbases` rows of 2^lrow counts (lrow >= 6) into nb.
void launch_row_sums(int64_t nbases, int lrow, const uint16_t* counts, uint32_t* nb, hipStream_t st) {
  const int lr = std::min(6, lrow - 3);
  auto go = [&](auto kernel, int R) {
    const int64_t per_block = (256 >> lr) * R;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((nbases + per_block - 1) / per_block)), dim3(256), 0, st, counts, lrow,
                       nbases, nb);
  };
  switch (lrow) {
    case 6: go(row_sums_kernel<3, 4, 2>, 4); break;
    case 7: go(row_sums_kernel<4, 4, 2>, 4); break;
    case 8: go(row_sums_kernel<5, 4, 2>, 4); break;
    case 9: go(row_sums_kernel<6, 4, 1>, 4); break;
    case 10: go(row_sums_kernel<6, 4, 2>, 4); break;
    case 11: go(row_sums_kernel<6, 2, 4>, 2); break;
    default: hipLaunchKernelGGL(row_sums_wide_kernel, dim3((unsigned)nbases), dim3(256), 0, st, counts, lrow, nb);
  }
}

// What the passes of step (i) read and write.  nseg segments of the counts (a streamed
// slab's) run in the same launches: segment s reads counts + s * seg_counts, writes its
// row-sum parts at rowpart + s * seg_row and its final sums at final_out + s * seg_final
// elements; its partials are the s-th of bufA's and bufB's.
struct PassIO {
  const uint16_t* counts;
  int lrow;                // log2 of the row stride of counts
  const uint32_t* nb;      // per-basis totals
  uint32_t* nb_own = nullptr;   // the counts pass is to form them (= nb)
  uint32_t* rowpart;
  void* final_out;
  void* bufA;
  void* bufB;
  int nseg = 1;
  int64_t seg_counts = 0, seg_row = 0, seg_final = 0;
  RowCheck chk{};          // checked with the last pass (nbases 0: not)
  void* rho = nullptr;     // not NULL (fuses_rho): step (ii) with the last pass, into rho
  bool fp32 = false;
};

template <int H, typename Tin, typename Acc, Out M>
void launch_tail_rho(const FoldArgs& a, void* rho, bool fp32) {
  const dim3 grid((unsigned)((8 << H) + (a.chk.nbases + 511) / 512));
  const Tin* in = static_cast<const Tin*>(a.in);
  double* coef = static_cast<double*>(a.out);
  if (fp32)
    hipLaunchKernelGGL((tail_rho_kernel<H, Tin, Acc, M, float>), grid, dim3(512), 0, a.st, in, coef, rho, a.shots, a.chk);
  else
    hipLaunchKernelGGL((tail_rho_kernel<H, Tin, Acc, M, double>), grid, dim3(512), 0, a.st, in, coef, rho, a.shots, a.chk);
}

// The last pass and step (ii) of n = 6 .. 8 qubits in one launch or two: a unit of 8 qubits reads up to
// 216 partials a thread, which takes 7.6 us from integers (two launches: 4.0 + 4.0 and a
// gap, 12.1 -> 11.1 us a call) but 11.8 from binary64 (13.1 -> 17.4 a call); up to 7 qubits
// at most 36 (n = 7 12.1 -> 8.9 us a call, binary64 12.3 -> 9.9).
bool fuses_rho(const Plan& P) {
  return !P.mfma && P.q1 == 5 && (P.n <= 7 || (P.n == 8 && P.t1 == Ty::U32));
}

template <int H>
void tail_rho_h(Ty tin, Ty tout, Out m, const FoldArgs& a, void* rho, bool fp32) {
  if constexpr (H < 2) {
    if (m == Out::CoefPerBasis) return launch_tail_rho<H, double, double, Out::CoefPerBasis>(a, rho, fp32);
    if (tin == Ty::F64) return launch_tail_rho<H, double, double, Out::CoefUniform>(a, rho, fp32);
  }
  if (tout == Ty::F64) launch_tail_rho<H, uint32_t, double, Out::CoefUniform>(a, rho, fp32);
  else launch_tail_rho<H, uint32_t, uint32_t, Out::CoefUniform>(a, rho, fp32);
}

bool tail_rho(Ty tin, Ty tout, Out m, const FoldArgs& a, void* rho, bool fp32) {
  switch (a.n) {
    case 6: tail_rho_h<0>(tin, tout, m, a, rho, fp32); return true;
    case 7: tail_rho_h<1>(tin, tout, m, a, rho, fp32); return true;
    case 8: tail_rho_h<2>(tin, tout, m, a, rho, fp32); return true;
  }
  return false;
}

// The counts pass (n > kSmallN) and the later passes, into final_out with final mode `fm`.
lre_status run_passes(lre_ctx* ctx, const Plan& P, const PassIO& io, uint64_t shots, Out fm, hipStream_t st) {
  const int n = P.n;
  int h = n - P.q1, l = P.q1;
  const bool single = P.npass == 0;
  Fold1Args a1{};
  a1.counts = io.counts;
  a1.n = n;
  a1.chunks = P.chunks;
  a1.lrow = io.lrow;
  a1.nb = io.nb_own ? nullptr : io.nb;
  a1.nb_own = io.nb_own;
  a1.out = single ? io.final_out : io.bufA;
  a1.rowpart = io.rowpart;
  a1.shots = shots;
  a1.tiles = ipow3(n - P.q1) * P.runs;
  a1.per_block = P.per_block;
  a1.blocks = P.blocks1;
  a1.nseg = io.nseg;
  a1.seg_counts = io.seg_counts;
  a1.seg_out = (ipow3(h) << h) * ipow4(l);
  a1.seg_row = io.seg_row;
  a1.st = st;
  const bool ok = P.mfma ? io.nseg == 1 && fold1_mfma(P.t1, P.per_basis, single ? fm : Out::Partial, a1)
                         : !single && fold1(P.q1, P.t1, P.per_basis, a1);
  if (!ok) return LRE_E_UNSUPPORTED;
  if (hipGetLastError() != hipSuccess) return LRE_E_HIP;
  record_stage(ctx, 1, st);

  Ty tin = P.t1;
  for (int k = 0; k < P.npass; ++k) {
    const bool last = k + 1 == P.npass;
    FoldArgs a{};
    a.in = k == 0 ? io.bufA : io.bufB;
    a.out = last ? io.final_out : io.bufB;
    a.n = n;
    a.h = h;
    a.l = l;
    a.shots = shots;
    a.nseg = io.nseg;
    a.seg_in = (ipow3(h) << h) * ipow4(l);
    h -= P.F[k];
    l += P.F[k];
    a.seg_out = last ? io.seg_final : (ipow3(h) << h) * ipow4(l);
    if (P.npass == 1) a.chk = io.chk;
    a.st = st;
    const bool done = io.rho ? tail_rho(tin, P.tout[k], fm, a, io.rho, io.fp32)
                      : P.npass == 1 ? fold_tail(P.F[k], tin, P.tout[k], fm, a)
                                   : two_pass(P.F[k], last, tin, P.tout[k], fm, a);
    if (!done) return LRE_E_UNSUPPORTED;
    if (hipGetLastError() != hipSuccess) return LRE_E_HIP;
    tin = P.tout[k];
  }
  if (P.npass != 1 && io.chk.nbases) {
    hipLaunchKernelGGL(check_rows_kernel, dim3((unsigned)((io.chk.nbases + 255) / 256)), dim3(256), 0, st, io.chk);
    if (hipGetLastError() != hipSuccess) return LRE_E_HIP;
  }
  return LRE_OK;
}

// An instance of n <= kSmallN qubits: everything in one launch.  fm: what `out` receives.
template <int N, bool PB, Out M, bool RHO, typename OutT>
void launch_small(const uint16_t* counts, uint64_t shots, const uint32_t* nb, void* out, void* rho, uint32_t* flags,
                  hipStream_t st) {
  hipLaunchKernelGGL((small_estimate_kernel<N, PB, M, RHO, OutT>), dim3(1), dim3(256), 0, st, counts, shots, nb, out,
                     rho, flags);
}

template <int N>
void small_n(Out fm, const uint16_t* counts, uint64_t shots, const uint32_t* nb, void* out, void* rho, bool fp32,
             uint32_t* flags, hipStream_t st) {
  if (fm == Out::PauliT) launch_small<N, false, Out::PauliT, false, double>(counts, shots, nb, out, rho, flags, st);
  else if (fm == Out::CoefUniform) {
    if (!rho) launch_small<N, false, Out::CoefUniform, false, double>(counts, shots, nb, out, rho, flags, st);
    else if (fp32) launch_small<N, false, Out::CoefUniform, true, float>(counts, shots, nb, out, rho, flags, st);
    else launch_small<N, false, Out::CoefUniform, true, double>(counts, shots, nb, out, rho, flags, st);
  } else {
    if (!rho) launch_small<N, true, Out::CoefPerBasis, false, double>(counts, shots, nb, out, rho, flags, st);
    else if (fp32) launch_small<N, true, Out::CoefPerBasis, true, float>(counts, shots, nb, out, rho, flags, st);
    else launch_small<N, true, Out::CoefPerBasis, true, double>(counts, shots, nb, out, rho, flags, st);
  }
}

lre_status run_small(lre_ctx* ctx, int n, Out fm, const uint16_t* counts, uint64_t shots, const uint32_t* nb,
                     void* out, void* rho, bool fp32, hipStream_t st) {
  switch (n) {
    case 1: small_n<1>(fm, counts, shots, nb, out, rho, fp32, ctx->flags, st); break;
    case 2: small_n<2>(fm, counts, shots, nb, out, rho, fp32, ctx->flags, st); break;
    case 3: small_n<3>(fm, counts, shots, nb, out, rho, fp32, ctx->flags, st); break;
    case 4: small_n<4>(fm, counts, shots, nb, out, rho, fp32, ctx->flags, st); break;
    default: small_n<5>(fm, counts, shots, nb, out, rho, fp32, ctx->flags, st); break;
  }
  return hipGetLastError() == hipSuccess ? LRE_OK : LRE_E_HIP;
}

// Step (i) of an instance of n > kSmallN qubits into `final_out` (coef or T) with final
// mode `fm`.
lre_status run_step1(lre_ctx* ctx, const Plan& P, const uint16_t* counts, uint64_t shots,
                     const uint32_t* nb_in, void* final_out, Out fm, char* ws, hipStream_t st, void* rho = nullptr,
                     bool fp32 = false) {
  const int64_t nbases = ipow3(P.n);
  PassIO io{};
  io.rho = rho;
  io.fp32 = fp32;
  io.counts = counts;
  io.lrow = P.n;
  io.nb = P.per_basis ? nb_in : nullptr;
  if (P.per_basis && !nb_in) {
    uint32_t* nb = reinterpret_cast<uint32_t*>(ws + P.off_nb);
    if (!P.mfma && P.q1 == 5) io.nb_own = nb;                // summed by the counts pass
    else launch_row_sums(nbases, P.n, counts, nb, st);
    io.nb = nb;
  }
  io.rowpart = reinterpret_cast<uint32_t*>(ws + P.off_rowpart);
  io.final_out = final_out;
  io.bufA = ws + P.off_a;
  io.bufB = ws + P.off_b;
  io.chk = RowCheck{io.rowpart, ipow3(P.q1), P.runs, P.per_block, nbases, io.nb,
                    P.per_basis ? (uint64_t)0 : shots, ctx->flags, 1, 0, 0, 0};
  return run_passes(ctx, P, io, shots, fm, st);
}

// Steps (i) and (ii) of one instance into caller-given workspace (lre_estimate).
lre_status estimate_impl(lre_ctx* ctx, int n, const uint16_t* counts, uint64_t shots,
                         const uint32_t* n_per_basis, double* coef, void* rho, void* workspace,
                         size_t workspace_bytes, uint32_t flags, void* stream) {
  if (!ctx || !counts || !coef || n < 1 || n > LRE_MAX_QUBITS) return LRE_E_ARG;
  if (flags & ~(LRE_NO_RHO | LRE_RHO_FP32 | LRE_WHT_MFMA)) return LRE_E_ARG;
  if (!aligned(counts, 16) || !aligned(coef, 8)) return LRE_E_ARG;
  const bool want_rho = !(flags & LRE_NO_RHO);
  if (want_rho && (!rho || !aligned(rho, 16))) return LRE_E_ARG;
  Plan P;
  if (!make_plan(n, shots, flags, P)) return LRE_E_ARG;
  if (P.total && (!workspace || !aligned(workspace, 256))) return LRE_E_ARG;
  if (workspace_bytes < P.total) return LRE_E_WORKSPACE;
  DeviceGuard g(ctx->device);
  if (!g.ok) return LRE_E_HIP;
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);

  record_stage(ctx, 0, st);
  const Out fm = P.per_basis ? Out::CoefPerBasis : Out::CoefUniform;
  if (n <= kSmallN) {
    const lre_status s = run_small(ctx, n, fm, counts, shots, n_per_basis, coef, want_rho ? rho : nullptr,
                                   (flags & LRE_RHO_FP32) != 0, st);
    for (int k = 1; k < 4; ++k) record_stage(ctx, k, st);
    return s;
  }
  const bool fused = want_rho && fuses_rho(P);
  const lre_status s = run_step1(ctx, P, counts, shots, n_per_basis, coef, fm, ws, st, fused ? rho : nullptr,
                                 (flags & LRE_RHO_FP32) != 0);
  if (s != LRE_OK) return s;
  record_stage(ctx, 2, st);
  if (want_rho && !fused) {
    if (flags & LRE_RHO_FP32) launch_rho<float>(P, coef, rho, ws, st);
    else launch_rho<double>(P, coef, rho, ws, st);
    if (hipGetLastError() != hipSuccess) return LRE_E_HIP;
  }
  record_stage(ctx, 3, st);
  return LRE_OK;
}

}  // namespace

extern "C" {

const char* lre_status_str(lre_status s) {
  switch (s) {
    case LRE_OK: return "ok";
    case LRE_E_ARG: return "invalid argument";
    case LRE_E_WORKSPACE: return "workspace too small";
    case LRE_E_HIP: return "HIP runtime error";
    case LRE_E_SHOTS: return "a basis row does not sum to its declared total";
    case LRE_E_EMPTY_BASIS: return "a basis has zero counts";
    case LRE_E_UNSUPPORTED: return "unsupported request";
    case LRE_E_TIMEOUT: return "a batched run's bounded wait expired";
    case LRE_E_EIG: return "the eigendecomposition of step (iii) did not converge";
  }
  return "unknown status";
}

lre_status lre_create(lre_ctx** out, int hip_device) {
  if (!out) return LRE_E_ARG;
  *out = nullptr;
  DeviceGuard g(hip_device);
  if (!g.ok) return LRE_E_HIP;
  lre_ctx* c = new (std::nothrow) lre_ctx;
  if (!c) return LRE_E_HIP;
  c->device = hip_device;
  c->flags = nullptr;
  c->n_stage_events = 0;
  for (auto& e : c->stage_events) e = nullptr;
  if (hipMalloc(&c->flags, 64) != hipSuccess) { delete c; return LRE_E_HIP; }
  void* mirror = nullptr;
  if (hipHostMalloc(&mirror, 64, hipHostMallocMapped | hipHostMallocPortable) != hipSuccess) {
    (void)hipFree(c->flags);
    delete c;
    return LRE_E_HIP;
  }
  std::memset(mirror, 0, 64);
  c->host_flags = static_cast<volatile uint32_t*>(mirror);
  void* mirror_dev = nullptr;
  uint64_t block[8] = {0};
  if (hipHostGetDevicePointer(&mirror_dev, mirror, 0) == hipSuccess) block[1] = reinterpret_cast<uint64_t>(mirror_dev);
  if (!mirror_dev || hipMemcpy(c->flags, block, sizeof block, hipMemcpyHostToDevice) != hipSuccess) {
    (void)hipFree(c->flags);
    (void)hipHostFree(mirror);
    delete c;
    return LRE_E_HIP;
  }
  // This device's copy of the static scratch array (device `hip_device` is current).
  void* sp = nullptr;
  const hipError_t se = hipGetSymbolAddress(&sp, HIP_SYMBOL(scratch));
  c->scratch_status = (int)se;
  c->scratch = se == hipSuccess ? static_cast<char*>(sp) : nullptr;
  *out = c;
  return LRE_OK;
}

void lre_destroy(lre_ctx* ctx) {
  if (!ctx) return;
  DeviceGuard g(ctx->device);
  (void)hipFree(ctx->flags);
  (void)hipHostFree(const_cast<uint32_t*>(ctx->host_flags));
  lre_detail::destroy_blas(ctx->blas);
  delete ctx;
}

size_t lre_workspace_bytes(int n, uint64_t shots, uint32_t flags) {
  Plan P;
  if (!make_plan(n, shots, flags, P)) return 0;
  return P.total;
}

lre_status lre_estimate(lre_ctx* ctx, int n, const uint16_t* counts, uint64_t shots,
                        const uint32_t* n_per_basis, double* coef, void* rho, void* workspace,
                        size_t workspace_bytes, uint32_t flags, void* stream) {
  return estimate_impl(ctx, n, counts, shots, n_per_basis, coef, rho, workspace, workspace_bytes, flags,
                       stream);
}

lre_status lre_estimate_noalloc(lre_ctx* ctx, int n, const uint16_t* counts, uint64_t shots,
                                const uint32_t* n_per_basis, double* coef, void* rho, uint32_t flags,
                                void* stream) {
  if (!ctx || n < 1 || n > LRE_MAX_QUBITS) return LRE_E_ARG;
  if (lre_workspace_bytes(n, shots, flags) > (size_t)LRE_NOALLOC_SCRATCH_BYTES) return LRE_E_WORKSPACE;
  if (!ctx->scratch) return LRE_E_HIP;
  return estimate_impl(ctx, n, counts, shots, n_per_basis, coef, rho, ctx->scratch,
                       (size_t)LRE_NOALLOC_SCRATCH_BYTES, flags, stream);
}

lre_status lre_set_stage_events(lre_ctx* ctx, void* const* events, int count) {
  if (!ctx || count < 0 || count > 4 || (count > 0 && !events)) return LRE_E_ARG;
  ctx->n_stage_events = events ? count : 0;
  for (int k = 0; k < 4; ++k)
    ctx->stage_events[k] = (events && k < count) ? static_cast<hipEvent_t>(events[k]) : nullptr;
  return LRE_OK;
}

lre_status lre_check(lre_ctx* ctx, void* stream) {
  if (!ctx) return LRE_E_ARG;
  DeviceGuard g(ctx->device);
  if (!g.ok) return LRE_E_HIP;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (hipStreamSynchronize(st) != hipSuccess) return LRE_E_HIP;
  uint32_t any = 0, raised[16], f = 0;
  for (int k = 0; k < 16; ++k) any |= ctx->host_flags[k];
  if (!any) return LRE_OK;
  // Mirror first: a bit raised meanwhile then leaves at worst a mirror word without its bit.
  // If a copy fails, the bits are still raised on the device, whose kernels set the mirror
  // for a new bit only: the words are set again, for the next check.
  for (int k = 0; k < 16; ++k) raised[k] = __atomic_exchange_n(ctx->host_flags + k, 0u, __ATOMIC_RELAXED);
  const uint32_t zero = 0;
  if (hipMemcpy(&f, ctx->flags, sizeof f, hipMemcpyDeviceToHost) != hipSuccess ||
      (f && hipMemcpy(ctx->flags, &zero, sizeof zero, hipMemcpyHostToDevice) != hipSuccess)) {
    for (int k = 0; k < 16; ++k)
      if (raised[k]) ctx->host_flags[k] = 1;
    return LRE_E_HIP;
  }
  if (f & FLAG_WAIT) return LRE_E_TIMEOUT;
  if (f & FLAG_EIG) return LRE_E_EIG;
  if (f & FLAG_ARG) return LRE_E_ARG;
  if (f & FLAG_EMPTY) return LRE_E_EMPTY_BASIS;
  if (f & FLAG_SHOTS) return LRE_E_SHOTS;
  return LRE_OK;
}

lre_status lre_pauli_sums(lre_ctx* ctx, int n, const uint16_t* counts, uint64_t shots, int64_t* T,
                          void* workspace, size_t workspace_bytes, uint32_t flags, void* stream) {
  if (!ctx || !counts || !T || n < 1 || n > LRE_MAX_QUBITS || shots == 0) return LRE_E_ARG;
  if (flags & ~(LRE_NO_RHO | LRE_RHO_FP32 | LRE_WHT_MFMA)) return LRE_E_ARG;
  if (!aligned(counts, 16) || !aligned(T, 8)) return LRE_E_ARG;
  Plan P;
  if (!make_plan(n, shots, flags | LRE_NO_RHO, P)) return LRE_E_ARG;
  if (P.total && (!workspace || !aligned(workspace, 256))) return LRE_E_ARG;
  if (workspace_bytes < P.total) return LRE_E_WORKSPACE;
  DeviceGuard g(ctx->device);
  if (!g.ok) return LRE_E_HIP;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (n <= kSmallN) return run_small(ctx, n, Out::PauliT, counts, shots, nullptr, T, nullptr, false, st);
  return run_step1(ctx, P, counts, shots, nullptr, T, Out::PauliT, static_cast<char*>(workspace), st);
}

lre_status lre_signed_sums(lre_ctx* ctx, int n, const uint16_t* counts, const int64_t* bases,
                           int64_t num_bases, int32_t* out, uint32_t flags, void* stream) {
  if (!ctx || !counts || !bases || !out || n < 1 || n > LRE_MAX_QUBITS || num_bases < 0)
    return LRE_E_ARG;
  if (flags & ~(LRE_WHT_MFMA)) return LRE_E_ARG;
  if ((flags & LRE_WHT_MFMA) && n < 6) return LRE_E_UNSUPPORTED;
  if (!aligned(counts, 16) || !aligned(out, 4) || !aligned(bases, 8)) return LRE_E_ARG;
  if (num_bases == 0) return LRE_OK;
  if (num_bases > INT32_MAX) return LRE_E_ARG;
  DeviceGuard g(ctx->device);
  if (!g.ok) return LRE_E_HIP;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const size_t lds = (size_t)4 << n;
  if (flags & LRE_WHT_MFMA) {
    hipLaunchKernelGGL(signed_sums_mfma_kernel, dim3((unsigned)num_bases), dim3(256), lds, st, counts, n, bases, out,
                       ctx->flags);
    return hipGetLastError() == hipSuccess ? LRE_OK : LRE_E_HIP;
  }
  const int q = n < kMaxQ1 ? n : kMaxQ1;
  switch (q) {
#define LRE_SS(Q)                                                                                  \
  case Q:                                                                                          \
    hipLaunchKernelGGL(signed_sums_kernel<Q>, dim3((unsigned)num_bases), dim3(256), lds, st, counts, n, \
                       bases, out, ctx->flags);                                                    \
    break;
    LRE_SS(1) LRE_SS(2) LRE_SS(3) LRE_SS(4) LRE_SS(5) LRE_SS(6) LRE_SS(7)
#undef LRE_SS
  }
  return hipGetLastError() == hipSuccess ? LRE_OK : LRE_E_HIP;
}


// ---------------------------------------------------------------------------------
// Streamed estimation (lre_stream_*): slabs of 3^(n-h) consecutive bases, each cut
// into 2^h outcome segments run as (n-h)-qubit instances, the top h qubits folded into
// the caller's coefficient array, which accumulates until lre_stream_finish.

}  // extern "C"

struct lre_stream {
  lre_ctx* ctx = nullptr;
  int n = 0, h = 0, np = 0;
  uint64_t shots = 0;
  uint32_t flags = 0;
  Plan P;                     // plan of one (n-h)-qubit segment (no rho), final sums raw
  Ty tV = Ty::F64;            // type of the segments' final sums
  int64_t slabs = 0;          // 3^h
  std::vector<uint8_t> pushed;
  int64_t npushed = 0;
  double* coef = nullptr;     // accumulator / output, set by lre_stream_begin
  int par = 1;                // segments per launch
  size_t off_a = 0, off_b = 0, off_nb = 0, off_V = 0, off_rowpart = 0, off_stage = 0, off_tmp = 0, total = 0;
  size_t seg_rowpart = 0;     // bytes of one segment's row-sum parts
  size_t stage_bytes = 0;
  hipEvent_t copied = nullptr;
};

namespace {

lre_status stream_ws_check(const lre_stream* S, void* ws, size_t ws_bytes) {
  if (!ws || !aligned(ws, 256)) return LRE_E_ARG;
  if (ws_bytes < S->total) return LRE_E_WORKSPACE;
  return LRE_OK;
}

template <int H>
void launch_top_fold(const lre_stream* S, const void* V, uint32_t atop, hipStream_t st) {
  const int64_t ncols = ipow4(S->np);
  const dim3 grid((unsigned)((ncols + 255) / 256));
  if (S->tV == Ty::U32)
    hipLaunchKernelGGL((stream_top_fold_kernel<H, uint32_t>), grid, dim3(256), 0, st, (const uint32_t*)V, S->coef,
                       ncols, atop);
  else
    hipLaunchKernelGGL((stream_top_fold_kernel<H, double>), grid, dim3(256), 0, st, (const double*)V, S->coef,
                       ncols, atop);
}

// One slab already in device memory: totals, the 2^h segments, the row check, the fold
// of the top qubits into the accumulator.
lre_status stream_slab(lre_stream* S, int64_t slab, const uint16_t* counts, const uint32_t* nb_in, char* ws,
                       hipStream_t st) {
  const Plan& P = S->P;
  const int np = S->np, n = S->n, h = S->h;
  const int64_t nbases = ipow3(np);
  PassIO io{};
  io.lrow = n;
  io.nb = P.per_basis ? nb_in : nullptr;
  if (P.per_basis && !nb_in) {
    uint32_t* nb = reinterpret_cast<uint32_t*>(ws + S->off_nb);
    launch_row_sums(nbases, n, counts, nb, st);
    io.nb = nb;
  }
  io.bufA = ws + S->off_a;
  io.bufB = ws + S->off_b;
  io.nseg = S->par;
  io.seg_counts = (int64_t)1 << np;
  io.seg_row = (int64_t)(S->seg_rowpart / 4);
  io.seg_final = ipow4(np);
  const size_t vbytes = (size_t)ipow4(np) * ty_size(S->tV);
  const RowCheck chk{reinterpret_cast<const uint32_t*>(ws + S->off_rowpart), ipow3(P.q1), P.runs, P.per_block, nbases,
                     io.nb, P.per_basis ? (uint64_t)0 : S->shots, S->ctx->flags, 1 << h, io.seg_row, 0, 0};
  // With all segments in one launch the last pass can check the slab's rows (n = 12, h = 2:
  // 10 us a slab by itself).
  if (S->par == 1 << h) io.chk = chk;
  for (int sg = 0; sg < (1 << h); sg += S->par) {
    io.counts = counts + ((int64_t)sg << np);
    io.rowpart = reinterpret_cast<uint32_t*>(ws + S->off_rowpart + (size_t)sg * S->seg_rowpart);
    io.final_out = ws + S->off_V + (size_t)sg * vbytes;
    const lre_status s = run_passes(S->ctx, P, io, S->shots, Out::Partial, st);
    if (s != LRE_OK) return s;
  }
  if (S->par != 1 << h)
    hipLaunchKernelGGL(check_rows_kernel, dim3((unsigned)((nbases + 255) / 256)), dim3(256), 0, st, chk);
  // Letters of the top qubits: digit p of the slab index (base 3) is qubit h - p.
  uint32_t atop = 0;
  int64_t t = slab;
  for (int p = 0; p < h; ++p) {
    atop |= (uint32_t)(t % 3 + 1) << (2 * p);
    t /= 3;
  }
  const void* V = ws + S->off_V;
  switch (h) {
    case 1: launch_top_fold<1>(S, V, atop, st); break;
    case 2: launch_top_fold<2>(S, V, atop, st); break;
    case 3: launch_top_fold<3>(S, V, atop, st); break;
    case 4: launch_top_fold<4>(S, V, atop, st); break;
    case 5: launch_top_fold<5>(S, V, atop, st); break;
    default: launch_top_fold<6>(S, V, atop, st); break;
  }
  return hipGetLastError() == hipSuccess ? LRE_OK : LRE_E_HIP;
}

lre_status stream_take_slab(lre_stream* S, int64_t slab) {
  if (!S->coef) return LRE_E_ARG;                       // lre_stream_begin first
  if (slab < 0 || slab >= S->slabs || S->pushed[(size_t)slab]) return LRE_E_ARG;
  S->pushed[(size_t)slab] = 1;
  ++S->npushed;
  return LRE_OK;
}

}  // namespace

extern "C" {

lre_status lre_stream_create(lre_ctx* ctx, int n, int h, uint64_t shots, uint32_t flags, lre_stream** out) {
  if (!out) return LRE_E_ARG;
  *out = nullptr;
  if (!ctx || n > LRE_STREAM_MAX_QUBITS || h < 1 || h > 6 || n - h < 8 || n - h > LRE_MAX_QUBITS)
    return LRE_E_ARG;
  if (flags & ~(LRE_NO_RHO | LRE_RHO_FP32 | LRE_WHT_MFMA | LRE_STREAM_HOST)) return LRE_E_ARG;
  lre_stream* S = new (std::nothrow) lre_stream;
  if (!S) return LRE_E_HIP;
  S->ctx = ctx;
  S->n = n;
  S->h = h;
  S->np = n - h;
  S->shots = shots;
  S->flags = flags;
  if (!make_plan(S->np, shots, (flags & LRE_WHT_MFMA) | LRE_NO_RHO, S->P)) {
    delete S;
    return LRE_E_ARG;
  }
  S->tV = S->P.npass ? S->P.tout[S->P.npass - 1] : S->P.t1;
  S->slabs = ipow3(h);
  try {
    S->pushed.assign((size_t)S->slabs, 0);
  } catch (...) {   // host memory
    delete S;
    return LRE_E_HIP;
  }
  const size_t segs = (size_t)1 << h;
  S->seg_rowpart = align256((size_t)S->P.parts * (size_t)ipow3(S->P.q1) * 4);
  // Segments of a slab run side by side as far as their partials stay within 4 GiB (one
  // launch of a small segment does not fill the chip); the MFMA form takes one at a time.
  const int hs = S->np - S->P.q1, h2 = hs - S->P.F[0];
  const size_t sizeA = S->P.npass ? (size_t)(ipow3(hs) << hs) * (size_t)ipow4(S->P.q1) * ty_size(S->P.t1) : 0;
  const size_t sizeB =
      S->P.npass > 1 ? (size_t)(ipow3(h2) << h2) * (size_t)ipow4(S->np - h2) * ty_size(S->P.tout[0]) : 0;
  if (!S->P.mfma)
    while (S->par < (int)segs && (sizeA + sizeB) * 2 * (size_t)S->par <= (size_t)4 << 30) S->par *= 2;
  size_t off = 0;
  S->off_a = off; off += align256(sizeA * (size_t)S->par);
  S->off_b = off; off += align256(sizeB * (size_t)S->par);
  S->off_nb = off; off += align256(S->P.per_basis ? (size_t)ipow3(S->np) * 4 : 0);
  S->off_V = off; off += align256(segs * (size_t)ipow4(S->np) * ty_size(S->tV));
  S->off_rowpart = off; off += segs * S->seg_rowpart;
  S->stage_bytes = (size_t)ipow3(S->np) << n;
  S->stage_bytes *= 2;
  if (flags & LRE_STREAM_HOST) {
    S->off_stage = off;
    off += align256(S->stage_bytes);
    off += align256(S->P.per_basis ? (size_t)ipow3(S->np) * 4 : 0);   // staged N_b
  }
  // step (ii)'s intermediate reuses the (then dead) segment buffers
  const size_t tmp = (flags & LRE_NO_RHO) ? 0 : (size_t)ipow4(n) * 16;
  S->off_tmp = 0;
  S->total = off > tmp ? off : tmp;
  DeviceGuard g(ctx->device);
  if (!g.ok || hipEventCreateWithFlags(&S->copied, hipEventDisableTiming) != hipSuccess) {
    delete S;
    return LRE_E_HIP;
  }
  *out = S;
  return LRE_OK;
}

size_t lre_stream_workspace_bytes(const lre_stream* S) { return S ? S->total : 0; }

lre_status lre_stream_begin(lre_stream* S, double* coef, void* workspace, size_t workspace_bytes, void* stream) {
  if (!S || !coef || !aligned(coef, 8)) return LRE_E_ARG;
  const lre_status c = stream_ws_check(S, workspace, workspace_bytes);
  if (c != LRE_OK) return c;
  DeviceGuard g(S->ctx->device);
  if (!g.ok) return LRE_E_HIP;
  S->coef = coef;
  std::fill(S->pushed.begin(), S->pushed.end(), 0);
  S->npushed = 0;
  // the accumulator starts at zero (a fill kernel: capturable, no memset node)
  const int64_t count = ipow4(S->n);             // >= 4^9
  hipLaunchKernelGGL(stream_clear_kernel, dim3((unsigned)(count / kClearBlock)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), coef);
  return hipGetLastError() == hipSuccess ? LRE_OK : LRE_E_HIP;
}

lre_status lre_stream_push(lre_stream* S, int64_t slab, const uint16_t* counts, const uint32_t* n_per_basis,
                           void* workspace, size_t workspace_bytes, void* stream) {
  if (!S || !counts || !aligned(counts, 16)) return LRE_E_ARG;
  if (n_per_basis && !aligned(n_per_basis, 4)) return LRE_E_ARG;
  lre_status c = stream_ws_check(S, workspace, workspace_bytes);
  if (c != LRE_OK) return c;
  if ((c = stream_take_slab(S, slab)) != LRE_OK) return c;
  DeviceGuard g(S->ctx->device);
  if (!g.ok) return LRE_E_HIP;
  return stream_slab(S, slab, counts, S->P.per_basis ? n_per_basis : nullptr, static_cast<char*>(workspace),
                     static_cast<hipStream_t>(stream));
}

lre_status lre_stream_push_host(lre_stream* S, int64_t slab, const uint16_t* counts, const uint32_t* n_per_basis,
                                void* workspace, size_t workspace_bytes, void* stream) {
  if (!S || !counts) return LRE_E_ARG;
  if (!(S->flags & LRE_STREAM_HOST)) return LRE_E_ARG;
  lre_status c = stream_ws_check(S, workspace, workspace_bytes);
  if (c != LRE_OK) return c;
  if (slab < 0 || slab >= S->slabs || S->pushed[(size_t)slab] || !S->coef) return LRE_E_ARG;
  DeviceGuard g(S->ctx->device);
  if (!g.ok) return LRE_E_HIP;
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  uint16_t* stage = reinterpret_cast<uint16_t*>(ws + S->off_stage);
  uint32_t* nb_stage = nullptr;
  // The staging buffer is reused by every slab: the copy is ordered after the previous
  // slab's kernels on the same stream.
  if (hipMemcpyAsync(stage, counts, S->stage_bytes, hipMemcpyHostToDevice, st) != hipSuccess) return LRE_E_HIP;
  if (S->P.per_basis && n_per_basis) {
    nb_stage = reinterpret_cast<uint32_t*>(ws + S->off_stage + align256(S->stage_bytes));
    if (hipMemcpyAsync(nb_stage, n_per_basis, (size_t)ipow3(S->np) * 4, hipMemcpyHostToDevice, st) != hipSuccess)
      return LRE_E_HIP;
  }
  if (hipEventRecord(S->copied, st) != hipSuccess) return LRE_E_HIP;
  if ((c = stream_take_slab(S, slab)) != LRE_OK) return c;
  c = stream_slab(S, slab, stage, nb_stage, ws, st);
  if (c != LRE_OK) return c;
  // the caller may reuse its host buffers once the copies are done (the slab's kernels
  // keep running)
  return hipEventSynchronize(S->copied) == hipSuccess ? LRE_OK : LRE_E_HIP;
}

lre_status lre_stream_finish(lre_stream* S, void* rho, void* workspace, size_t workspace_bytes, void* stream) {
  if (!S || !S->coef) return LRE_E_ARG;
  if (S->npushed != S->slabs) return LRE_E_ARG;
  const bool want_rho = !(S->flags & LRE_NO_RHO);
  if (want_rho && (!rho || !aligned(rho, 16))) return LRE_E_ARG;
  const lre_status c = stream_ws_check(S, workspace, workspace_bytes);
  if (c != LRE_OK) return c;
  DeviceGuard g(S->ctx->device);
  if (!g.ok) return LRE_E_HIP;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int64_t count = ipow4(S->n);
  hipLaunchKernelGGL(stream_finish_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, S->coef, S->n,
                     S->P.per_basis ? (uint64_t)0 : S->shots, count);
  if (hipGetLastError() != hipSuccess) return LRE_E_HIP;
  if (want_rho) {
    Plan R;
    R.n = S->n;
    R.off_tmp = S->off_tmp;
    if (S->flags & LRE_RHO_FP32) launch_rho<float>(R, S->coef, rho, static_cast<char*>(workspace), st);
    else launch_rho<double>(R, S->coef, rho, static_cast<char*>(workspace), st);
    if (hipGetLastError() != hipSuccess) return LRE_E_HIP;
  }
  S->coef = nullptr;
  return LRE_OK;
}

void lre_stream_destroy(lre_stream* S) {
  if (!S) return;
  {
    DeviceGuard g(S->ctx->device);
    if (S->copied) (void)hipEventDestroy(S->copied);
  }
  delete S;
}


// ---------------------------------------------------------------------------------
// Reduced measurement set (Sec. VI): 4^n product operators of one informationally
// complete 4-operator set per qubit.

size_t lre_povm_workspace_bytes(int n, uint32_t flags) {
  if (n < 1 || n > LRE_MAX_QUBITS) return 0;
  const size_t head = 256;   // M (16 binary64) and the 64-bit total N
  const size_t tmp = (!(flags & LRE_NO_RHO) && rho_needs_tmp(n)) ? (size_t)ipow4(n) * 16 : 0;
  return head + align256(tmp);
}

}  // extern "C"

namespace {

// Digits of the first pass and of the next one.  Up to 7 in the first: all of n <= 7; 6 for
// n = 8 .. 10, whose tiles of 7 would leave most CUs idle (n = 10: 23.6 us against 17.8, all
// passes), 7 from there on, which saves a pass or thins the last one (n = 11: 34.5 us against 36.8;
// n = 12: 94 as 7 + 5, 117 as 6 + 4 + 2; n = 14: 2.18 ms as 7 + 4 + 3, 2.27 as 6 + 4 + 4).
int povm_first_digits(int n) { return n <= 7 ? n : (n <= 10 ? 6 : 7); }

// Digits of a pass over `left` digits from lo on: 4, or what is left.  5 only as the last pass
// (n = 12, as 7 + 5): where digits remain after it, its 128 KiB tiles cost more than the later
// pass gains (n = 13: 576 us as 7 + 5 + 1, 542 as 7 + 4 + 2; n = 14: 2387 us as 7 + 5 + 2, 2175 as
// 7 + 4 + 3).  (32-bit offsets in povm_high5_kernel: lo <= 9.)
int povm_next_digits(int left, int lo) { return left == 5 && lo <= 9 ? 5 : (left >= 4 ? 4 : left); }

template <int J, bool FINAL>
void launch_povm_tiles(const uint16_t* counts, double* coef, const double* M, unsigned long long* total,
                       uint32_t* flags, int tiles, hipStream_t st) {
  using G = PovmTileGeom<J>;
  const int blocks = (int)std::min<int64_t>(
      tiles, resident_blocks(povm_tile_kernel<J, FINAL>, G::TH, (G::T + G::T / 16) * 8 + G::TH / 8));
  hipLaunchKernelGGL((povm_tile_kernel<J, FINAL>), dim3((unsigned)blocks), dim3(G::TH), 0, st, counts, coef, M, total,
                     flags, tiles);
}

void launch_povm_high5(double* coef, int lo, const double* M, const unsigned long long* total, uint32_t* flags,
                       int64_t tiles, hipStream_t st) {
  const int64_t blocks =
      std::min<int64_t>(tiles, resident_blocks(povm_high5_kernel, 1024, 1024LL * kPovmWideCols * 8));
  hipLaunchKernelGGL(povm_high5_kernel, dim3((unsigned)blocks), dim3(1024), 0, st, coef, lo, M, total, flags, tiles);
}

}  // namespace

extern "C" {

lre_status lre_povm_estimate(lre_ctx* ctx, int n, const uint16_t* counts, const double* G, double* coef, void* rho,
                             void* workspace, size_t workspace_bytes, uint32_t flags, void* stream) {
  if (!ctx || !counts || !G || !coef || n < 1 || n > LRE_MAX_QUBITS) return LRE_E_ARG;
  if (flags & ~(LRE_NO_RHO | LRE_RHO_FP32)) return LRE_E_ARG;
  if (!aligned(counts, 16) || !aligned(G, 8) || !aligned(coef, 8)) return LRE_E_ARG;
  const bool want_rho = !(flags & LRE_NO_RHO);
  if (want_rho && (!rho || !aligned(rho, 16))) return LRE_E_ARG;
  const size_t need = lre_povm_workspace_bytes(n, flags);
  if (!workspace || !aligned(workspace, 256)) return LRE_E_ARG;
  if (workspace_bytes < need) return LRE_E_WORKSPACE;
  DeviceGuard g(ctx->device);
  if (!g.ok) return LRE_E_HIP;
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  double* M = reinterpret_cast<double*>(ws);
  unsigned long long* total = reinterpret_cast<unsigned long long*>(ws + 128);
  const int64_t count = ipow4(n);

  record_stage(ctx, 0, st);
  hipLaunchKernelGGL(povm_setup_kernel, dim3(1), dim3(64), 0, st, G, M, total, ctx->flags);
  record_stage(ctx, 1, st);

  // Passes over the digits, lowest first; the first also sums the counts into N, the last
  // divides by N.
  const int J = povm_first_digits(n);
  const int tiles = (int)(count >> (2 * J));
  const bool only = J == n;
  switch (J) {
#define LRE_POVM_LOW(JJ)                                                                                          \
  case JJ:                                                                                                        \
    hipLaunchKernelGGL((povm_low_kernel<JJ>), dim3(1), dim3(256), 0, st, counts, coef, (const double*)M, ctx->flags); \
    break;
    LRE_POVM_LOW(1) LRE_POVM_LOW(2) LRE_POVM_LOW(3) LRE_POVM_LOW(4) LRE_POVM_LOW(5)
#undef LRE_POVM_LOW
    case 6:
      if (only) launch_povm_tiles<6, true>(counts, coef, M, total, ctx->flags, tiles, st);
      else launch_povm_tiles<6, false>(counts, coef, M, total, ctx->flags, tiles, st);
      break;
    default:
      if (only) launch_povm_tiles<7, true>(counts, coef, M, total, ctx->flags, tiles, st);
      else launch_povm_tiles<7, false>(counts, coef, M, total, ctx->flags, tiles, st);
  }
  for (int lo = J; lo < n;) {
    const int F = povm_next_digits(n - lo, lo);
    const bool last = n - lo == F;
    const double* Mc = M;
    const unsigned long long* tot = total;
    const int64_t cols = count >> (2 * F);
    const dim3 grid((unsigned)((cols + 255) / 256));
    switch (F) {
      case 5:
        launch_povm_high5(coef, lo, Mc, tot, ctx->flags, cols / kPovmWideCols, st);
        break;
      case 4:
        if (last)
          hipLaunchKernelGGL((povm_high4_kernel<true>), dim3((unsigned)(cols / kPovmCols)), dim3(kPovmHighThreads), 0,
                             st, coef, n, lo, Mc, tot, ctx->flags);
        else
          hipLaunchKernelGGL((povm_high4_kernel<false>), dim3((unsigned)(cols / kPovmCols)), dim3(kPovmHighThreads), 0,
                             st, coef, n, lo, Mc, tot, ctx->flags);
        break;
      case 3: hipLaunchKernelGGL((povm_reg_kernel<3, true>), grid, dim3(256), 0, st, coef, n, lo, Mc, tot, ctx->flags); break;
      case 2: hipLaunchKernelGGL((povm_reg_kernel<2, true>), grid, dim3(256), 0, st, coef, n, lo, Mc, tot, ctx->flags); break;
      default: hipLaunchKernelGGL((povm_reg_kernel<1, true>), grid, dim3(256), 0, st, coef, n, lo, Mc, tot, ctx->flags); break;
    }
    lo += F;
  }
  if (hipGetLastError() != hipSuccess) return LRE_E_HIP;
  record_stage(ctx, 2, st);
  if (want_rho) {
    Plan R;
    R.n = n;
    R.off_tmp = 256;
    if (flags & LRE_RHO_FP32) launch_rho<float>(R, coef, rho, ws, st);
    else launch_rho<double>(R, coef, rho, ws, st);
    if (hipGetLastError() != hipSuccess) return LRE_E_HIP;
  }
  record_stage(ctx, 3, st);
  return LRE_OK;
}

}  // extern "C"
