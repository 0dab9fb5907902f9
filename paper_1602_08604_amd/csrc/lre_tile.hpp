// lre_tile.hpp -- gfx950 counts pass in sub-tiles folded through LDS, the later pass that
// ends a small plan, and the one-workgroup path of at most 5 qubits.
//
// Counts pass.  A sub-tile is 3^5 rows (the letters of the 5 lowest qubits) x 64 outcomes
// (the bits of the 6 lowest): 128 bytes of each row.  Three stages:
//   1. a thread (lam = outcome bits 3-5, rs = letters of qubits 2-4) holds 9 rows x 8
//      outcomes, transforms outcome bits 0-2 in registers, folds qubits 0 and 1 and
//      stores 32 values, [letters of qubits 0, 1][Walsh bit 2], to V;
//   2. a thread (letters of qubits 0, 1; outcome bits 4, 5; basis letter of qubit 4) reads
//      its 3 x 3 x 2 x 2 values of qubits 2 and 3 from V, folds both and stores 16 to W;
//   3. a thread owns 4 of the 4^5 Pauli indices of the sub-tile (the letters of qubit 4),
//      folds qubit 4 from W, and folds the qubits above with accumulators in registers:
//      the sub-tiles of 5 + LV qubits follow one another, letter of the top qubit outermost
//      and its outcome bits innermost, so a letter's odd part is final as soon as it is
//      formed and only the identity letter is kept.
// Every value passes LDS twice, each time as a plain store and load (no atomics), and no
// stage has a chain longer than one thread's fold, so a small instance is not one workgroup's
// serial walk: n = 7 (per-basis totals from the rows) 49.8 -> 10.6 us a call, n = 8 33 -> 11.3,
// n = 10 66 -> 52.7.  At n >= 12 the pass is bound by memory: with 10 % (n = 12) to 19 % (n = 13,
// binary64) of its traffic being writes the device moves 5.2 TB/s (loads alone: 7.0 and 6.4),
// n = 12 927 -> 904 us, n = 13 6.40 -> 6.13 ms.
#pragma once
#include "lre_kernels.hpp"

namespace lre {

constexpr int kTileRows = 243;      // 3^5 rows of a sub-tile
constexpr int kTileUnits = 216;     // stage-1 threads: 27 row sets x 8 lanes of 8 outcomes
constexpr int kTileVP = 218;        // stride of V's 32 codes (26 mod 32: stage 2 reads 16 codes
                                    // x 2 neighbours at a time, all on different banks)
constexpr int kTileUnits2 = 192;    // stage-2 threads: 16 codes x 2 x (3 letters x 2 outcomes)
constexpr int kTileWP = 208;        // stride of W's 16 codes (16 mod 32: stage 3 reads two)
constexpr int kTileV = 32 * kTileVP, kTileW = 16 * kTileWP;

// Qubits folded and outcomes covered by a tile of level LV.
template <int LV>
struct TileGeom {
  static constexpr int Q = 5 + LV;
  static constexpr int NROWS = (int)ipow3(Q);
  static constexpr int WB = LV <= 1 ? 6 : 5 + LV;        // log2 of the outcomes of a tile
  static constexpr int NL = (int)ipow3(LV);              // row blocks of 243 rows
  static constexpr int NS = 1 << (WB - 6);               // 64-outcome columns
};

typedef uint32_t tile_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t tile_u32x2 __attribute__((ext_vector_type(2)));

// A pointer every lane of the wave holds, moved to scalar registers.
template <typename T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<T*>(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const void* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(uniform_ptr(static_cast<const char*>(p))), 0,
                                           __builtin_amdgcn_readfirstlane(bytes), 0x00027000);
}

// The three stages of a sub-tile.  Elem: double (per-basis totals) or int32_t (a sub-tile's
// sums of at most 243 x 64 counts fit).
template <bool PB>
struct TileStages {
  using Elem = std::conditional_t<PB, double, int32_t>;

  // Stage 1 of thread t < kTileUnits.
  struct Rows {
    uint32_t raw[9][4];
    Elem L1[4][2];
    uint32_t rtot;           // lane lam: the total of row lam (r < 8)
    uint32_t rtot8;          // the total of row 8
  };

  // Byte offset of thread t's rows in the sub-tile.  The waves' threads beyond kTileUnits go
  // through stage 1 with the others, on rows out of the descriptor's range (zeros, no traffic)
  // and with the spare columns of V: around a branch, the compiler would have to count the
  // loads it may have skipped and wait for nearly all that are in flight.
  static __device__ __forceinline__ int row_offset(int t, int rowbytes) {
    return t < kTileUnits ? (t >> 3) * 9 * rowbytes + (t & 7) * 16 : 0x40000000;
  }

  static __device__ __forceinline__ void load_row(Rows& R, __amdgpu_buffer_rsrc_t rsrc, int voff, int rowbytes, int r) {
    const tile_u32x4 u = __builtin_amdgcn_raw_buffer_load_b128(
        rsrc, voff, __builtin_amdgcn_readfirstlane(r * rowbytes), 2 /* nt */);
    R.raw[r][0] = u.x; R.raw[r][1] = u.y; R.raw[r][2] = u.z; R.raw[r][3] = u.w;
  }

  static __device__ __forceinline__ void load_rows(Rows& R, __amdgpu_buffer_rsrc_t rsrc, int voff, int rowbytes) {
#pragma unroll
    for (int r = 0; r < 9; ++r) load_row(R, rsrc, voff, rowbytes, r);
  }

  // Rows 3 D1 .. 3 D1 + 2 into Vt = V + (place of t); each row's registers take the row of
  // the sub-tile behind `next` as soon as it has been transformed.
  template <int D1>
  static __device__ __forceinline__ void stage1(Rows& R, Elem* Vt, const double* inv9, int lam,
                                                __amdgpu_buffer_rsrc_t next, int voff, int rowbytes) {
    if constexpr (D1 == 0) {
      R.rtot = 0;
#pragma unroll
      for (int a = 0; a < 4; ++a) R.L1[a][0] = R.L1[a][1] = Elem(0);
    }
    Elem L0[4] = {Elem(0), Elem(0), Elem(0), Elem(0)};         // [m1 + 2 m2]
    double inv[3];
    if constexpr (PB) {
#pragma unroll
      for (int d0 = 0; d0 < 3; ++d0) inv[d0] = inv9[3 * D1 + d0];
    }
#pragma unroll
    for (int d0 = 0; d0 < 3; ++d0) {
      const int r = 3 * D1 + d0;
      int32_t x[8];
      unpack_raw<8>(R.raw[r], x);
      wht_regs<3>(x);
      // Not earlier: the old row's registers would still be in use and the loop would
      // copy all 36 of them.
      __builtin_amdgcn_sched_barrier(0);
      load_row(R, next, voff, rowbytes, r);
      const uint32_t tot = lane_sum<3>((uint32_t)x[0]);
      if (r < 8) R.rtot = lam == r ? tot : R.rtot;
      else R.rtot8 = tot;
      Elem y[8];
      if constexpr (PB) {
#pragma unroll
        for (int v = 0; v < 8; ++v) y[v] = (double)x[v] * inv[d0];
      } else {
#pragma unroll
        for (int v = 0; v < 8; ++v) y[v] = x[v];
      }
#pragma unroll
      for (int mr = 0; mr < 4; ++mr) {
        const int m1 = mr & 1, m2 = mr >> 1;
        L0[mr] += y[2 * mr];
        if (m1 == 0) R.L1[d0 + 1][m2] += y[2 * mr + 1];
        else Vt[(d0 + 1 + 4 * (D1 + 1) + 16 * m2) * kTileVP] = y[2 * mr + 1];
      }
      // The row's values end here: without this the sums of three rows are formed together
      // and hold their terms (99 registers instead of 52 for one sub-tile of integers).
#pragma unroll
      for (int mr = 0; mr < 4; ++mr) asm volatile("" : "+v"(L0[mr]));
      asm volatile("" : "+v"(R.L1[d0 + 1][0]), "+v"(R.L1[d0 + 1][1]));
    }
#pragma unroll
    for (int mr = 0; mr < 4; ++mr) {
      const int m1 = mr & 1, m2 = mr >> 1;
      if (m1 == 0) R.L1[0][m2] += L0[mr];
      else Vt[(4 * (D1 + 1) + 16 * m2) * kTileVP] = L0[mr];
    }
    if constexpr (D1 == 2) {
#pragma unroll
      for (int a0 = 0; a0 < 4; ++a0)
#pragma unroll
        for (int m2 = 0; m2 < 2; ++m2) Vt[(a0 + 16 * m2) * kTileVP] = R.L1[a0][m2];
    }
  }

  // The 9 rows' totals into rt (LDS): set (first tile of the rows) or added.
  static __device__ __forceinline__ void row_totals(const Rows& R, uint32_t* rt, int lam, bool set) {
    if (set) {
      rt[lam] = R.rtot;
      if (lam == 0) rt[8] = R.rtot8;
    } else {
      atomicAdd(&rt[lam], R.rtot);
      if (lam == 0) atomicAdd(&rt[8], R.rtot8);
    }
  }

  // Place of stage-1 thread t in V: outcome bit 5 lowest, then bits 3 and 4.
  static __device__ __forceinline__ int place(int t) {
    return t < kTileUnits ? (t & ~7) | ((t >> 2) & 1) | ((t & 3) << 1) : kTileUnits + (t & 1);
  }
  // Its rows' places among the 243.
  static __device__ __forceinline__ int row_of(int t) { return (t < kTileUnits ? t >> 3 : 0) * 9; }

  // Stage 2 of thread u < kTileUnits2 = code + 16 s5 + 32 (s4 + 2 d4).
  static __device__ __forceinline__ void stage2(const Elem* V, Elem* W, int u) {
    const int q = u >> 5;
    const Elem* const V2 = V + (u & 15) * kTileVP + ((u >> 4) & 1) + 4 * (q & 1) + 72 * (q >> 1);
    Elem* const W2 = W + u;
    Elem I2[4];                                                 // letter I of qubit 2, per a3
#pragma unroll
    for (int d2 = 0; d2 < 3; ++d2) {
#pragma unroll
      for (int m2 = 0; m2 < 2; ++m2) {
        Elem e[3], o[3];
#pragma unroll
        for (int d3 = 0; d3 < 3; ++d3) {
          const Elem a = V2[16 * m2 * kTileVP + 8 * d2 + 24 * d3], b = V2[16 * m2 * kTileVP + 8 * d2 + 24 * d3 + 2];
          e[d3] = a + b;
          o[d3] = a - b;
        }
        const Elem r[4] = {e[0] + e[1] + e[2], o[0], o[1], o[2]};
#pragma unroll
        for (int a3 = 0; a3 < 4; ++a3) {
          if (m2 == 1) W2[(d2 + 1 + 4 * a3) * kTileWP] = r[a3];
          else if (d2 == 0) I2[a3] = r[a3];
          else I2[a3] += r[a3];
        }
      }
    }
#pragma unroll
    for (int a3 = 0; a3 < 4; ++a3) W2[4 * a3 * kTileWP] = I2[a3];
  }

  // Stage 3 of thread t < 256 = code + 16 a2 + 64 a3: T[s5] of Pauli indices t + 256 a4.
  static __device__ __forceinline__ void stage3(const Elem* W, int t, Elem (&T0)[4], Elem (&T1)[4]) {
    const Elem* const W3 = W + (t >> 4) * kTileWP + (t & 15);
    auto fold = [&](const Elem* w, Elem (&T)[4]) __attribute__((always_inline)) {
      Elem e[3];
#pragma unroll
      for (int d4 = 0; d4 < 3; ++d4) {
        const Elem a = w[64 * d4], b = w[64 * d4 + 32];
        e[d4] = a + b;
        T[d4 + 1] = a - b;
      }
      T[0] = e[0] + e[1] + e[2];
    };
    fold(W3, T0);
    fold(W3 + 16, T1);
  }
};

// A row total's reciprocal, correctly rounded (0 for an empty basis, which the row check
// flags).
__device__ __forceinline__ double tile_reciprocal(uint32_t N) { return N ? 1.0 / (double)N : 0.0; }

// Whether partials are stored with the nontemporal hint, unless the launch says so: binary64
// partials of 7-qubit tiles, which are read again only after more than the caches hold (plain
// stores: n = 13 6.99 instead of 6.84 ms).
constexpr bool tile_nt(int lv, bool pb) { return pb && lv >= 2; }

template <bool NT, typename Acc>
__device__ __forceinline__ void tile_put(__amdgpu_buffer_rsrc_t rsrc, int t, int i, Acc v) {
  const int soff = __builtin_amdgcn_readfirstlane(i * (int)sizeof(Acc));
  if constexpr (sizeof(Acc) == 4) {
    __builtin_amdgcn_raw_buffer_store_b32((uint32_t)v, rsrc, t * 4, soff, NT ? 2 : 0);
  } else {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(tile_u32x2, v), rsrc, t * 8, soff, NT ? 2 : 0);
  }
}

// Row totals inside the sub-tile pass: load k (of 8) of thread t takes row (t >> 3) + 32 k.  Byte
// offset of the thread's part of the address; the uniform part 32 k rows + the column is added
// to it.  Rows beyond the 243 get an offset out of range by itself: whether the range check
// of a raw buffer counts the uniform part too is not the same in all descriptions of it.
__host__ __device__ constexpr int subtile_total_offset(int t, int k, int rowbytes) {
  return (t >> 3) + 32 * k < kTileRows ? (t >> 3) * rowbytes + (t & 7) * 16 : 0x40000000;
}

// One sub-tile per workgroup of 256 threads, 5 qubits folded (plans too small to fill the
// chip with anything larger): blockIdx.x = (b_hi, 64-outcome column), blockIdx.y = segment (a
// streamed slab's outcome segment; counts advance by seg_counts, out and rowpart by seg_out
// elements and seg_row words).
// out: [3^(n-5)][2^(n-5)][4^5] partial sums; rowpart: [block][243] row sums of the block.
// nb: per-basis totals (PB), of which every row's reciprocal is formed here; NULL (one
// segment, lrow = n): every workgroup sums its rows over all their outcomes, which its 2^(n-6)
// neighbours also read, and column 0 writes the sums to nb_own for the row check.  (By a
// launch of its own: n = 7 3.3 us of 17.)
template <bool PB, typename Acc>
__global__ __launch_bounds__(256) void counts_subtile_kernel(const uint16_t* __restrict__ counts, int n, int lrow,
                                                             const uint32_t* __restrict__ nb,
                                                             uint32_t* __restrict__ nb_own, Acc* __restrict__ out,
                                                             uint32_t* __restrict__ rowpart, int64_t seg_counts,
                                                             int64_t seg_out, int64_t seg_row) {
  using S = TileStages<PB>;
  using Elem = typename S::Elem;
  __shared__ Elem V[kTileV], W[kTileW];
  __shared__ uint32_t rs_acc[kTileRows];
  __shared__ double invt[PB ? kTileRows : 1];
  const int tid = threadIdx.x, lam = tid & 7;
  const int64_t b_hi = blockIdx.x >> (n - 6), col = blockIdx.x & ((1 << (n - 6)) - 1);
  const int rowbytes = 2 << lrow;
  const bool on1 = tid < kTileUnits;
  typename S::Rows R;
  const int voff = S::row_offset(tid, rowbytes);
  const auto src = tile_rsrc(counts + blockIdx.y * seg_counts + ((b_hi * kTileRows) << lrow) + (col << 6),
                             (kTileRows - 1) * rowbytes + 128);
  const auto none = tile_rsrc(counts, 0);
  S::load_rows(R, src, voff, rowbytes);
  if constexpr (PB) {
    if (nb) {
      if (tid < kTileRows) invt[tid] = tile_reciprocal(nb[b_hi * kTileRows + tid]);
    } else {
      const auto rows = tile_rsrc(counts + ((b_hi * kTileRows) << lrow), kTileRows * rowbytes);
      uint32_t sum[8] = {0, 0, 0, 0, 0, 0, 0, 0};              // rows (tid >> 3) + 32 k, from 243 on zeros
      for (int c = 0; c < (1 << (n - 6)); ++c) {
        tile_u32x4 u[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
          u[k] = __builtin_amdgcn_raw_buffer_load_b128(
              rows, subtile_total_offset(tid, k, rowbytes), __builtin_amdgcn_readfirstlane(32 * k * rowbytes + c * 128), 0);
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
          for (int e = 0; e < 4; ++e) sum[k] += (u[k][e] & 0xFFFFu) + (u[k][e] >> 16);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const uint32_t tot = lane_sum<3>(sum[k]);
        const int r = (tid >> 3) + 32 * k;
        if (lam == 0 && r < kTileRows) {
          invt[r] = tile_reciprocal(tot);
          if (col == 0) nb_own[b_hi * kTileRows + r] = tot;
        }
      }
    }
    lds_barrier();
  }
  {
    Elem* const Vt = V + S::place(tid);
    const double* const inv9 = invt + (PB ? S::row_of(tid) : 0);
    S::template stage1<0>(R, Vt, inv9, lam, none, voff, rowbytes);
    S::template stage1<1>(R, Vt, inv9, lam, none, voff, rowbytes);
    S::template stage1<2>(R, Vt, inv9, lam, none, voff, rowbytes);
    if (on1) S::row_totals(R, rs_acc + S::row_of(tid), lam, true);
  }
  lds_barrier();
  if (tid < kTileUnits2) S::stage2(V, W, tid);
  lds_barrier();
  Elem T0[4], T1[4];
  S::stage3(W, tid, T0, T1);
  const auto o = tile_rsrc(out + blockIdx.y * seg_out + (((b_hi << (n - 5)) + 2 * col) << 10), 2048 * (int)sizeof(Acc));
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    tile_put<false>(o, tid, 256 * k, (Acc)T0[k]);
    tile_put<false>(o, tid, 1024 + 256 * k, (Acc)T1[k]);
  }
  uint32_t* __restrict__ rp = rowpart + blockIdx.y * seg_row + (int64_t)blockIdx.x * kTileRows;
  if (tid < kTileRows) rp[tid] = rs_acc[tid];
}

// What the tiles kernel asks about tile t of its block.
// One instance, or the segments of a slab: tiles ordered (b_hi, tile of the row).
template <int LV, typename Acc>
struct InstanceTiles {
  using G = TileGeom<LV>;
  const uint16_t* counts_;
  const uint32_t* nb_;
  Acc* out_;
  uint32_t* rowpart_;
  int64_t t0;
  int n, lrow, lgT;        // lgT: log2 of the tiles of a row
  __device__ __forceinline__ int64_t group(int t) const { return (t0 + t) >> lgT; }
  __device__ __forceinline__ int64_t tile_of_row(int t) const { return (t0 + t) & (((int64_t)1 << lgT) - 1); }
  __device__ __forceinline__ const uint16_t* counts(int t) const {
    return counts_ + ((group(t) * G::NROWS) << lrow) + (tile_of_row(t) << G::WB);
  }
  __device__ __forceinline__ int rowbytes(int) const { return 2 << lrow; }
  __device__ __forceinline__ const uint32_t* nb(int t) const { return nb_ + group(t) * G::NROWS; }
  __device__ __forceinline__ Acc* out(int t) const {
    return out_ + (((group(t) << (n - G::Q)) + tile_of_row(t)) << (2 * G::Q));
  }
  __device__ __forceinline__ bool first_of_row(int t) const { return t == 0 || group(t) != group(t - 1); }
  __device__ __forceinline__ uint32_t* part(int t) const { return rowpart_ + (group(t) + blockIdx.x) * G::NROWS; }
};

// The tiles of many instances, from a table (batched estimation).
struct TileEntry {
  const uint16_t* counts;      // first row and outcome
  int64_t out, nb;             // byte offset in the workspace of its partial sums; totals: an
  int32_t group, lrow;         // offset too, or (nb_abs) an address
  int32_t nb_abs, pad;
};

template <int LV, typename Acc>
struct BatchTiles {
  using G = TileGeom<LV>;
  // The block's first tile; in the constant address space, so that entries come through
  // scalar loads (a vector load's wait would cover every row in flight).
  const __attribute__((address_space(4))) TileEntry* e;
  char* ws;
  uint32_t* rowpart_;
  __device__ __forceinline__ const uint16_t* counts(int t) const { return e[t].counts; }
  __device__ __forceinline__ int rowbytes(int t) const { return 2 << e[t].lrow; }
  __device__ __forceinline__ const uint32_t* nb(int t) const {
    return reinterpret_cast<const uint32_t*>(e[t].nb_abs ? reinterpret_cast<char*>(e[t].nb) : ws + e[t].nb);
  }
  __device__ __forceinline__ Acc* out(int t) const { return reinterpret_cast<Acc*>(ws + e[t].out); }
  __device__ __forceinline__ bool first_of_row(int t) const { return t == 0 || e[t].group != e[t - 1].group; }
  __device__ __forceinline__ uint32_t* part(int t) const {
    return rowpart_ + ((int64_t)e[t].group + blockIdx.x) * G::NROWS;
  }
};

// Tiles of 5 + LV qubits (LV = 1, 2), 512 threads: waves 0-3 run stage 1 of one sub-tile
// while waves 4-7 run stages 2 and 3 of the one before (V double-buffered), so one's loads
// and transforms overlap the other's LDS traffic and stores; a SIMD holds a wave of each
// kind.  Two barriers per sub-tile: at its end, and between stages 2 and 3, which waves 0-3
// meet after two thirds of their rows.  The rows of sub-tile j + 2 are loaded as those
// of j are used, into the same registers.  Only waves 4-7 store to memory, so no load's wait
// covers a store.
// Binary64 sub-tiles take the LDS of a CU (one workgroup), integers half of it.
template <int LV, bool PB>
struct TileLds {
  using Elem = typename TileStages<PB>::Elem;
  Elem V[2 * kTileV];
  Elem W[kTileW];
  double invt[PB ? 2 * kTileRows : 1];
  uint32_t rs_acc[TileGeom<LV>::NROWS];
};

// The nt tiles of `tiles`, in sequence.  out of a tile: [4^Q] partial sums; part: [3^Q], the
// row sums over the block's tiles of one row group.  NT: partials stored with the nontemporal hint.
template <int LV, bool PB, typename Acc, bool NT, class Tiles>
__device__ __forceinline__ void counts_tiles_block(const Tiles& tiles, int nt, TileLds<LV, PB>& lds) {
  static_assert(LV == 1 || LV == 2, "levels above the sub-tile");
  using G = TileGeom<LV>;
  using S = TileStages<PB>;
  using Elem = typename S::Elem;
  const int nsteps = nt * G::NL * G::NS;                       // sub-tiles
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Elem* const W = lds.W;

  if (wave < 4) {
    // ---- stage 1
    const int tid = threadIdx.x, lam = tid & 7;
    const bool on1 = tid < kTileUnits;
    typename S::Rows R[2];
    // The sub-tile loaded next: tile at, row block alblk, column as.
    int at = 0, alblk = 0, as = 0;
    const uint16_t* abase = uniform_ptr(tiles.counts(0));
    int arow = __builtin_amdgcn_readfirstlane(tiles.rowbytes(0));
    int voff = S::row_offset(tid, arow);
    auto next_rsrc = [&]() __attribute__((always_inline)) {
      const char* p = reinterpret_cast<const char*>(abase) + (int64_t)alblk * kTileRows * arow + as * 128;
      return tile_rsrc(p, at < nt ? (kTileRows - 1) * arow + 128 : 0);
    };
    auto advance = [&]() __attribute__((always_inline)) {
      if (++as == G::NS) {
        as = 0;
        if (++alblk == G::NL) {
          alblk = 0;
          if (++at < nt) {
            abase = uniform_ptr(tiles.counts(at));
            arow = __builtin_amdgcn_readfirstlane(tiles.rowbytes(at));
            voff = S::row_offset(tid, arow);
          }
        }
      }
    };
    S::load_rows(R[0], next_rsrc(), voff, arow);
    advance();
    S::load_rows(R[1], next_rsrc(), voff, arow);
    advance();
    lds_barrier();                                             // reciprocals of the first rows
    int ct = 0, clblk = 0, cs = 0, rho = 0;                    // the sub-tile in hand; row blocks so far
    bool first = true;                                         // its tile is the block's first of its rows
    auto step = [&](typename S::Rows& Rj, int buf) __attribute__((always_inline)) {
      Elem* const Vt = lds.V + buf * kTileV + S::place(tid);
      const double* const inv9 = lds.invt + (PB ? (rho & 1) * kTileRows + S::row_of(tid) : 0);
      const auto next = next_rsrc();
      S::template stage1<0>(Rj, Vt, inv9, lam, next, voff, arow);
      S::template stage1<1>(Rj, Vt, inv9, lam, next, voff, arow);
      lds_barrier();
      S::template stage1<2>(Rj, Vt, inv9, lam, next, voff, arow);
      if (on1) S::row_totals(Rj, lds.rs_acc + clblk * kTileRows + S::row_of(tid), lam, cs == 0 && first);
      lds_barrier();
      advance();
      if (++cs == G::NS) {
        cs = 0;
        ++rho;
        if (++clblk == G::NL) {
          clblk = 0;
          if (++ct < nt) first = tiles.first_of_row(ct);
        }
      }
    };
    int j = 0;
    for (; j + 1 < nsteps; j += 2) {
      step(R[0], 0);
      step(R[1], 1);
    }
    if (j < nsteps) step(R[0], 0);
    lds_barrier();
    lds_barrier();
  } else {
    // ---- stages 2 and 3 of the sub-tile before
    const int tid = threadIdx.x - 256;
    // Totals of row block r of the block's sequence.
    auto load_nb = [&](int r) __attribute__((always_inline)) {
      if constexpr (!PB) return 0u;
      const int t = r / G::NL;
      return t < nt && tid < kTileRows ? tiles.nb(t)[(r % G::NL) * kTileRows + tid] : 0u;
    };
    auto set_inv = [&](int r, uint32_t N) __attribute__((always_inline)) {
      if (PB && tid < kTileRows) lds.invt[(r & 1) * kTileRows + tid] = tile_reciprocal(N);
    };
    set_inv(0, load_nb(0));
    uint32_t nbn = load_nb(1);
    lds_barrier();
    int rho = 0;                                               // row block of the sub-tile processed
    if constexpr (G::NS == 1) {                                // sub-tile 1 has other rows already
      set_inv(1, nbn);
      nbn = load_nb(2);
    }
    lds_barrier();
    lds_barrier();
    int j = 0;
    Elem T0[4], T1[4];
    // Stages 2 and 3 of sub-tile j (column s); the reciprocals the sub-tile after next needs.
    auto stages = [&](int s) __attribute__((always_inline)) {
      if (tid < kTileUnits2) S::stage2(lds.V + (j & 1) * kTileV, W, tid);
      if (s == 0) {
        const int r = rho + (G::NS == 1 ? 2 : 1);
        set_inv(r, nbn);
        nbn = load_nb(r + 1);
      }
      lds_barrier();
      S::stage3(W, tid, T0, T1);
      if (s == G::NS - 1) ++rho;
      ++j;
    };
    Acc i5S[4], i5D[4];          // identity letter of qubit 5 (LV 2: even and odd in outcome bit 6)
    Acc i6[4][4];                // LV 2: identity letter of qubit 6, per letter of qubit 5
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      i5S[k] = i5D[k] = Acc(0);
#pragma unroll
      for (int q = 0; q < 4; ++q) i6[q][k] = Acc(0);
    }
    for (int t = 0; t < nt; ++t) {
      const auto o = tile_rsrc(tiles.out(t), (1 << (2 * G::Q)) * (int)sizeof(Acc));
      // The totals of the rows just finished go out with the block's last tile of them.
      const bool last = t + 1 == nt || tiles.first_of_row(t + 1);
      uint32_t* const part = uniform_ptr(tiles.part(t));
      auto flush = [&](int lblk) __attribute__((always_inline)) {
        if (last && tid < kTileRows) part[lblk * kTileRows + tid] = lds.rs_acc[lblk * kTileRows + tid];
      };
      if constexpr (LV == 1) {
        StaticFor<0, 3>::run([&](auto lc) __attribute__((always_inline)) {
          constexpr int l5 = decltype(lc)::value;
          stages(0);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            tile_put<NT>(o, tid, 1024 * (l5 + 1) + 256 * k, (Acc)(T0[k] - T1[k]));
            i5S[k] += (Acc)(T0[k] + T1[k]);
          }
          flush(l5);
          if constexpr (l5 == 2) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              tile_put<NT>(o, tid, 256 * k, i5S[k]);
              i5S[k] = Acc(0);
            }
          }
          lds_barrier();
        });
      } else {
        for (int l6 = 0; l6 < 3; ++l6) {
          StaticFor<0, 3>::run([&](auto lc) __attribute__((always_inline)) {
            constexpr int l5 = decltype(lc)::value;
            Acc hS[4], hD[4];                                  // outcome bit 6 = 0
            stages(0);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              hS[k] = (Acc)(T0[k] + T1[k]);
              hD[k] = (Acc)(T0[k] - T1[k]);
            }
            lds_barrier();
            stages(1);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const Acc Sk = (Acc)(T0[k] + T1[k]), Dk = (Acc)(T0[k] - T1[k]);
              tile_put<NT>(o, tid, 4096 * (l6 + 1) + 1024 * (l5 + 1) + 256 * k, hD[k] - Dk);
              i5S[k] += hS[k] + Sk;
              i5D[k] += hS[k] - Sk;
              i6[l5 + 1][k] += hD[k] + Dk;
            }
            flush(3 * l6 + l5);
            if constexpr (l5 == 2) {
#pragma unroll
              for (int k = 0; k < 4; ++k) {
                tile_put<NT>(o, tid, 4096 * (l6 + 1) + 256 * k, i5D[k]);
                i6[0][k] += i5S[k];
                i5S[k] = i5D[k] = Acc(0);
              }
              if (l6 == 2) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                  for (int k = 0; k < 4; ++k) {
                    tile_put<NT>(o, tid, 1024 * q + 256 * k, i6[q][k]);
                    i6[q][k] = Acc(0);
                  }
              }
            }
            lds_barrier();
          });
        }
      }
    }
  }
}

// blockIdx.x: `per_block` consecutive tiles of an instance; blockIdx.y: segment, as for the
// sub-tile kernel.  out: [3^(n-Q)][2^(n-Q)][4^Q]; rowpart: [b_hi + block][3^Q].
template <int LV, bool PB, typename Acc, bool NT>
__global__ __launch_bounds__(512, PB ? 2 : 4) void counts_tile_kernel(
    const uint16_t* __restrict__ counts, int n, int lrow, int64_t tiles, int64_t per_block,
    const uint32_t* __restrict__ nb, Acc* __restrict__ out, uint32_t* __restrict__ rowpart, int64_t seg_counts,
    int64_t seg_out, int64_t seg_row) {
  __shared__ TileLds<LV, PB> lds;
  InstanceTiles<LV, Acc> T;
  T.counts_ = counts + blockIdx.y * seg_counts;
  T.nb_ = nb;
  T.out_ = out + blockIdx.y * seg_out;
  T.rowpart_ = rowpart + blockIdx.y * seg_row;
  T.t0 = blockIdx.x * per_block;
  T.n = n;
  T.lrow = lrow;
  T.lgT = n - TileGeom<LV>::WB;
  counts_tiles_block<LV, PB, Acc, NT>(T, (int)(tiles - T.t0 < per_block ? tiles - T.t0 : per_block), lds);
}

// The same over a table of tiles; part of a block's row group: [group + block][3^Q].
template <int LV, bool PB, typename Acc>
__global__ __launch_bounds__(512, PB ? 2 : 4) void batch_tiles_kernel(const TileEntry* __restrict__ table, int tiles,
                                                                      int per_block, char* __restrict__ ws,
                                                                      uint32_t* __restrict__ rowpart) {
  __shared__ TileLds<LV, PB> lds;
  const int t0 = (int)blockIdx.x * per_block;
  const BatchTiles<LV, Acc> T{(const __attribute__((address_space(4))) TileEntry*)(table + t0), ws, rowpart};
  counts_tiles_block<LV, PB, Acc, tile_nt(LV, PB)>(T, tiles - t0 < per_block ? tiles - t0 : per_block, lds);
}

// Row totals: where the parts of basis row group g = b / rows are.  per_block > 0: part
// group0 + g + w for every block w of the counts pass that held one of the group's `runs`
// tiles (the instance's first tile is tile0); else parts g * runs .. + runs - 1.  seg_row:
// words between the parts of the nseg segments.
struct RowCheck {
  const uint32_t* rowpart;
  int64_t rows, runs, per_block, nbases;
  const uint32_t* nb;
  uint64_t shots;
  uint32_t* flags;
  int nseg;
  int64_t seg_row;
  int64_t group0, tile0;
};

__device__ __forceinline__ void check_row_total(const RowCheck& c, int64_t b) {
  const int64_t g = (uint32_t)b / (uint32_t)c.rows, j = (uint32_t)b % (uint32_t)c.rows;
  int64_t p0 = g * c.runs, p1 = p0 + c.runs;
  if (c.per_block > 0) {
    const uint32_t w0 = (uint32_t)(c.tile0 + p0) / (uint32_t)c.per_block;
    const uint32_t w1 = (uint32_t)(c.tile0 + p1 - 1) / (uint32_t)c.per_block;
    p0 = c.group0 + g + w0;
    p1 = c.group0 + g + w1 + 1;
  }
  uint64_t tot = 0;
  for (int s = 0; s < c.nseg; ++s)
    for (int64_t p = p0; p < p1; ++p) tot += c.rowpart[s * c.seg_row + p * c.rows + j];
  const uint64_t want = c.shots ? c.shots : (uint64_t)c.nb[b];
  if (tot != want) raise_flag(c.flags, FLAG_SHOTS);
  if (!c.shots && want == 0) raise_flag(c.flags, FLAG_EMPTY);
}

static __global__ __launch_bounds__(256) void check_rows_kernel(RowCheck c) {
  const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (b < c.nbases) check_row_total(c, b);
}

// ---------------------------------------------------------------------------------
// Later pass folding F <= 4 qubits without atomics: a thread folds the two lowest of the F
// for one column and one (letters, outcomes) of the others (36 loads, all independent),
// the 6^(F-2) x 16 values of a column meet in LDS and a thread per (column, code) folds
// the rest.  COLS consecutive columns a_l per block.  Blocks from fold_blocks on check the
// row totals instead (launched with the pass: one launch less for a small instance).
template <int F>
struct FoldTailGeom {
  static constexpr int COLS = F == 4 ? 16 : (F == 3 ? 32 : 64);
  static constexpr int SUB = F <= 2 ? 1 : (F == 3 ? 6 : 36);   // threads per column
  static constexpr int THREADS = COLS * SUB;
};

// x / den, correctly rounded, by the reciprocal rc = 1 / den (correctly rounded too): x rc is
// off by less than two units, one correction by the exact remainder makes it faithful, and
// the second rounds it correctly (Markstein).  Finite x and positive den away from the
// limits of the type's range, as sums of counts and 3^k N are.
__device__ __forceinline__ double tail_quotient(double x, double den, double rc) {
  double q = x * rc;
  q = fma(fma(-q, den, x), rc, q);
  return fma(fma(-q, den, x), rc, q);
}

// The divisors 3^(n - w) (times the shots) of the weights w = wl + k, k <= K: powers and
// reciprocals once a thread instead of a loop and a division an output (small plans' last pass:
// n = 7 5.6 -> 3.8 us, n = 8 5.7 -> 4.0, n = 10 10.9 -> 9.7; the larger ones are bound by memory).
template <int K, Out MODE>
struct TailDivisors {
  double den[K + 1], rc[K + 1];
  __device__ __forceinline__ TailDivisors(int n, int wl, uint64_t shots) {
    if constexpr (MODE == Out::CoefUniform || MODE == Out::CoefPerBasis) {
      double p = pow3d(n - wl - K);
#pragma unroll
      for (int k = K; k >= 0; --k) {
        den[k] = MODE == Out::CoefUniform ? p * (double)shots : p;
        rc[k] = 1.0 / den[k];
        p *= 3.0;
      }
    }
  }
};

// Block `blk`; mid: LDS of SUB x 16 x COLS values (F > 2).  Every thread of the block calls
// this.  The batch's tail stage runs F = 3 in workgroups of 256: threads from THREADS on have no
// (letters, outcomes) of their own and only meet the barrier.
template <int F, typename Tin, typename Acc, Out MODE>
__device__ __forceinline__ void fold_tail_block(const Tin* __restrict__ in, void* __restrict__ out, int n, int h, int l,
                                                uint64_t shots, int64_t blk, int tid, Acc* __restrict__ mid) {
  using G = FoldTailGeom<F>;
  constexpr int COLS = G::COLS, F1 = F < 2 ? F : 2, N1 = 1 << (2 * F1);
  const int64_t L = (int64_t)1 << (2 * l);
  const int64_t per_outer = L / COLS;
  const int64_t bs = blk / per_outer;
  const int64_t a_l = (blk % per_outer) * COLS + tid % COLS;
  const int q = tid / COLS;
  const int64_t rowstride = ((int64_t)1 << h) * L;

  // Final value of folded code a, k of whose letters are not the identity: divided by
  // 3^(n-w) (and the shots) unless partial.
  const TailDivisors<F, MODE> div(n, MODE == Out::Partial ? 0 : pauli_weight((uint64_t)a_l), shots);
  auto put = [&](int a, double den, double rc, Acc v) __attribute__((always_inline)) {
    if constexpr (MODE == Out::Partial) static_cast<Acc*>(out)[((bs << (2 * F)) + a) * L + a_l] = v;
    else if constexpr (MODE == Out::PauliT) static_cast<int64_t*>(out)[(int64_t)a * L + a_l] = acc_to_i64(v);
    else static_cast<double*>(out)[(int64_t)a * L + a_l] = tail_quotient(acc_to_double(v), den, rc);
  };

  if (tid < G::THREADS) {
    const int dq = q >> (F > 2 ? F - 2 : 0), sq = q & ((1 << (F > 2 ? F - 2 : 0)) - 1);
    const Tin* __restrict__ p =
        in + fold_in_offset<F>(h, l, (bs << (2 * l)) + a_l, dq * (int)ipow3(F1), sq << F1);
    Acc o[N1];
#pragma unroll
    for (int a = 0; a < N1; ++a) o[a] = Acc(0);
    StaticFor<0, (int)ipow3(F1)>::run([&](auto bc) __attribute__((always_inline)) {
      constexpr int beta = decltype(bc)::value;
      Acc x[1 << F1];
#pragma unroll
      for (int sg = 0; sg < (1 << F1); ++sg) x[sg] = in_to_acc<Tin, Acc>(p[beta * rowstride + sg * L]);
      wht_regs<F1>(x);
      StaticFor<0, (1 << F1)>::run([&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value;
        constexpr int a = fold_index(beta, m, F1);
        o[a] += x[m];
      });
    });
    if constexpr (F <= 2) {
#pragma unroll
      for (int a = 0; a < N1; ++a) {
        const int k = __builtin_popcount((a | (a >> 1)) & 0x5);
        put(a, div.den[k], div.rc[k], o[a]);
      }
    } else {
#pragma unroll
      for (int a = 0; a < 16; ++a) mid[(q * 16 + a) * COLS + tid % COLS] = o[a];
    }
  }
  if constexpr (F > 2) {
    const int col = tid % COLS;
    __syncthreads();
    // column t % COLS = tid % COLS
    for (int t = tid < G::THREADS ? tid : 16 * COLS; t < 16 * COLS; t += G::THREADS) {
      const int code = t / COLS;
      const Acc* __restrict__ m0 = mid + code * COLS + col;
      constexpr int F2 = F - 2, N2 = 1 << (2 * F2);
      Acc r[N2];
#pragma unroll
      for (int a = 0; a < N2; ++a) r[a] = Acc(0);
      StaticFor<0, (int)ipow3(F2)>::run([&](auto bc) __attribute__((always_inline)) {
        constexpr int beta = decltype(bc)::value;
        Acc x[1 << F2];
#pragma unroll
        for (int sg = 0; sg < (1 << F2); ++sg) x[sg] = m0[(((beta << F2) | sg) * 16) * COLS];
        wht_regs<F2>(x);
        StaticFor<0, (1 << F2)>::run([&](auto mc) __attribute__((always_inline)) {
          constexpr int m = decltype(mc)::value;
          constexpr int a = fold_index(beta, m, F2);
          r[a] += x[m];
        });
      });
      // of the code's two letters
      const int kc = __popc((uint32_t)(code | (code >> 1)) & 0x5u);
#pragma unroll
      for (int a = 0; a < N2; ++a) {
        const int k = __builtin_popcount((a | (a >> 1)) & 0x5);
        put(code + 16 * a, kc == 0 ? div.den[k] : (kc == 1 ? div.den[k + 1] : div.den[k + 2]),
            kc == 0 ? div.rc[k] : (kc == 1 ? div.rc[k + 1] : div.rc[k + 2]), r[a]);
      }
    }
  }
}

template <int F, typename Tin, typename Acc, Out MODE>
__global__ __launch_bounds__(FoldTailGeom<F>::THREADS) void fold_tail_kernel(
    const Tin* __restrict__ in, void* __restrict__ out, int n, int h, int l, uint64_t shots, int64_t fold_blocks,
    int64_t seg_in, int64_t seg_out, RowCheck chk) {
  using G = FoldTailGeom<F>;
  __shared__ Acc mid[F > 2 ? G::SUB * 16 * G::COLS : 1];
  if ((int64_t)blockIdx.x >= fold_blocks) {
    const int64_t b = ((int64_t)blockIdx.x - fold_blocks) * G::THREADS + threadIdx.x;
    if (blockIdx.y == 0 && b < chk.nbases) check_row_total(chk, b);   // all segments' parts
    return;
  }
  constexpr int64_t kOutBytes = MODE == Out::Partial ? sizeof(Acc) : 8;
  fold_tail_block<F, Tin, Acc, MODE>(in + blockIdx.y * seg_in, static_cast<char*>(out) + blockIdx.y * seg_out * kOutBytes,
                                     n, h, l, shots, blockIdx.x, threadIdx.x, mid);
}

// ---------------------------------------------------------------------------------
// The last pass and step (ii) of n = 6 + H <= 8 qubits in one launch, a unit of rho_tiles per
// workgroup: every coefficient belongs to exactly one unit (its x pattern), so a unit folds
// its own coefficients from the counts pass's partials [3^(H+1)][2^(H+1)][4^5], writes them
// to coef and, through V, to mu.  Thread t takes letters t & 63 of qubits 0..2 and
// z bits t >> 6 of qubits 3..5 (one wave), all 2^H z patterns of the qubits above, whose x
// pattern X says which of their 6 inputs matter: all for I and Z, those of X and Y otherwise.
// Bound by the loads' latency, once per letter of qubit 5 (the sched_barrier keeps a letter's
// loads together: 0.9 us of a call of 7 qubits); n = 7 4.9 us where the two launches took 3.8 + 3.3
// and the gap between them, n = 8 (integers) 7.6 against 4.0 + 4.0.
template <int H, int X, typename Tin, typename Acc>
__device__ __forceinline__ void tail_unit_fold(const Tin* __restrict__ p, int letter5, Acc (&out)[1 << H]) {
  constexpr int h = H + 1, ND = (int)ipow3(H), NS = 1 << H;
#pragma unroll
  for (int z = 0; z < NS; ++z) out[z] = Acc(0);
  const int first = letter5 ? letter5 - 1 : 0, last = letter5 ? letter5 : 3;
  for (int d5 = first; d5 < last; ++d5) {
    Tin y[ND][NS][2];
    StaticFor<0, ND>::run([&](auto dc) __attribute__((always_inline)) {
      constexpr int d = decltype(dc)::value;
      constexpr bool used = !((X & 1) && d % 3 == 2) && !((X & 2) && d / 3 == 2);
#pragma unroll
      for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int s5 = 0; s5 < 2; ++s5)
          y[d][s][s5] = used ? p[((((d * 3 + d5) << h) | (2 * s + s5)) << 10)] : Tin(0);
    });
    __builtin_amdgcn_sched_barrier(0);                         // every load in flight at once
    StaticFor<0, ND>::run([&](auto dc) __attribute__((always_inline)) {
      constexpr int d = decltype(dc)::value;
      Acc v[NS];
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const Acc a = in_to_acc<Tin, Acc>(y[d][s][0]), b = in_to_acc<Tin, Acc>(y[d][s][1]);
        v[s] = letter5 ? a - b : a + b;
      }
      wht_regs<H>(v);
      StaticFor<0, NS>::run([&](auto zc) __attribute__((always_inline)) {
        constexpr int z = decltype(zc)::value;
        constexpr int a0 = (X & 1) ? ((z & 1) ? 2 : 1) : ((z & 1) ? 3 : 0);
        constexpr int a1 = (X & 2) ? ((z & 2) ? 2 : 1) : ((z & 2) ? 3 : 0);
        if constexpr ((a0 == 0 || a0 == d % 3 + 1) && (H < 2 || a1 == 0 || a1 == d / 3 + 1)) out[z] += v[(X | z) & (NS - 1)];
      });
    });
  }
}

template <int H, typename Tin, typename Acc, Out MODE, typename OutT>
__global__ __launch_bounds__(512, 2) void tail_rho_kernel(const Tin* __restrict__ in, double* __restrict__ coef,
                                                       void* __restrict__ rho, uint64_t shots, RowCheck chk) {
  static_assert(H <= 2, "n <= 8");
  constexpr int n = 6 + H, NZ = 1 << H, UNITS = 8 << H;
  __shared__ double V[RhoTileGeom<H>::NV];
  const int t = threadIdx.x;
  if (blockIdx.x >= UNITS) {
    const int64_t b = ((int64_t)blockIdx.x - UNITS) * 512 + t;
    if (b < chk.nbases) check_row_total(chk, b);
    return;
  }
  const uint32_t x_hi = blockIdx.x >> 3, xb = blockIdx.x & 7u;
  const uint32_t zh3 = (uint32_t)__builtin_amdgcn_readfirstlane(t >> 6);
  const uint32_t a5 = letters_of<3>(xb, zh3);                  // letters of qubits 3..5
  const uint32_t low = ((a5 & 15u) << 6) | (uint32_t)(t & 63);
  const int letter5 = (int)(a5 >> 4);
  Acc out[NZ];
  const Tin* __restrict__ p = in + low;
  if constexpr (H == 0) tail_unit_fold<H, 0>(p, letter5, out);
  if constexpr (H == 1) {
    if (x_hi == 0) tail_unit_fold<H, 0>(p, letter5, out);
    else tail_unit_fold<H, 1>(p, letter5, out);
  }
  if constexpr (H == 2) {
    if (x_hi == 0) tail_unit_fold<H, 0>(p, letter5, out);
    else if (x_hi == 1) tail_unit_fold<H, 1>(p, letter5, out);
    else if (x_hi == 2) tail_unit_fold<H, 2>(p, letter5, out);
    else tail_unit_fold<H, 3>(p, letter5, out);
  }
  const TailDivisors<H, MODE> div(n, pauli_weight((uint64_t)low) + (letter5 ? 1 : 0), shots);
#pragma unroll
  for (int z = 0; z < NZ; ++z) {
    const int k = __popc(x_hi | (uint32_t)z);                  // letters of the qubits above that are not I
    double den = div.den[0], rc = div.rc[0];
#pragma unroll
    for (int q = 1; q <= H; ++q)
      if (k == q) { den = div.den[q]; rc = div.rc[q]; }
    const double e = tail_quotient(acc_to_double(out[z]), den, rc);
    coef[((int64_t)letters_of<H>(x_hi, (uint32_t)z) << 12) | (a5 << 6) | (uint32_t)(t & 63)] = e;
    V[z * 512 + t] = e;
  }
  lds_barrier();
  rho_tile_unit<H, OutT, 512>(rho, blockIdx.x, t, V);
}

// ---------------------------------------------------------------------------------
// Totals of `rows` consecutive rows of 2^lrow counts (lrow >= 3): 2^LR lanes per row, R
// rows per lane group and K loads of each issued before any is summed.
template <int LR, int R, int K = 2>
__device__ __forceinline__ void row_sums_block(const uint16_t* __restrict__ counts, int lrow, int64_t rows,
                                               uint32_t* __restrict__ nb, int64_t blk) {
  constexpr int LPR = 1 << LR, GROUPS = 256 / LPR;
  const int lane = threadIdx.x % LPR, grp = threadIdx.x / LPR;
  const int per = 1 << (lrow - 3 - LR);                       // 16-byte loads per lane and row
  const int64_t b0 = (blk * GROUPS + grp) * R;
  const tile_u32x4* __restrict__ base = reinterpret_cast<const tile_u32x4*>(counts);
  uint32_t sum[R];
#pragma unroll
  for (int r = 0; r < R; ++r) sum[r] = 0;
  for (int k = 0; k < per; k += K) {
    tile_u32x4 w[R][K];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int j = 0; j < K; ++j)
        w[r][j] = (b0 + r < rows && k + j < per)
                      ? __builtin_nontemporal_load(base + ((b0 + r) << (lrow - 3)) + (k + j) * LPR + lane)
                      : tile_u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int j = 0; j < K; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[r] += (w[r][j][e] & 0xFFFFu) + (w[r][j][e] >> 16);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
#pragma unroll
    for (int o = LPR / 2; o > 0; o >>= 1) sum[r] += __shfl_xor(sum[r], o, 64);
    if (lane == 0 && b0 + r < rows) nb[b0 + r] = sum[r];
  }
}

template <int LR, int R, int K>
__global__ __launch_bounds__(256) void row_sums_kernel(const uint16_t* __restrict__ counts, int lrow, int64_t rows,
                                                       uint32_t* __restrict__ nb) {
  row_sums_block<LR, R, K>(counts, lrow, rows, nb, blockIdx.x);
}

// The same for lrow >= 12, one row per workgroup of 256 and one load in flight per thread: 4 KiB
// runs, which DRAM serves better than a wave's 1 KiB (n = 12: 594 us, 7.3 TB/s, against 651 to
// 664; two loads in flight: 625).
static __global__ __launch_bounds__(256) void row_sums_wide_kernel(const uint16_t* __restrict__ counts, int lrow,
                                                                   uint32_t* __restrict__ nb) {
  const tile_u32x4* __restrict__ row =
      reinterpret_cast<const tile_u32x4*>(counts) + ((int64_t)blockIdx.x << (lrow - 3)) + threadIdx.x;
  __shared__ uint32_t part[4];
  uint32_t sum = 0;
#pragma unroll 1
  for (int k = 0; k < (1 << (lrow - 11)); ++k) {
    const tile_u32x4 w = __builtin_nontemporal_load(row + k * 256);
#pragma unroll
    for (int e = 0; e < 4; ++e) sum += (w[e] & 0xFFFFu) + (w[e] >> 16);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x == 0) nb[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// ---------------------------------------------------------------------------------
// An instance of N <= 5 qubits in one workgroup and one launch: a thread per basis row
// sums, checks and transforms its row (2^N counts in registers), the identity letters are
// summed qubit by qubit in place in LDS, and the coefficients, divided, go to memory and to
// step (ii).  Sums are held in binary64; with uniform shots they are integers below 2^53,
// so the coefficients are the same correctly rounded quotients as on the other paths.
// MODE: what `out` receives (PauliT: no rho).
// S, E: LDS of SmallLds<N>.
template <int N>
struct SmallLds {
  static constexpr int B = (int)ipow3(N), D = 1 << N, DP = D + 1, NA = 1 << (2 * N);
  // the rows' sums, then step (ii)'s two planes
  static constexpr int S = B * DP > 2 * RhoLowLds<N>::SIZE ? B * DP : 2 * RhoLowLds<N>::SIZE;
  static constexpr int E = NA;
};

template <int N, bool PB, Out MODE, bool RHO, typename OutT>
__device__ __forceinline__ void small_estimate_block(const uint16_t* __restrict__ counts, uint64_t shots,
                                                     const uint32_t* __restrict__ nb_in, void* __restrict__ out,
                                                     void* __restrict__ rho, uint32_t* __restrict__ flags, int tid,
                                                     double* __restrict__ S, double* __restrict__ E) {
  constexpr int B = SmallLds<N>::B, D = SmallLds<N>::D, NA = SmallLds<N>::NA, DP = SmallLds<N>::DP;
  if (tid < B) {
    int32_t x[D];
    const uint32_t* __restrict__ p = reinterpret_cast<const uint32_t*>(counts) + tid * (D / 2);
    if constexpr (D >= 8) {
#pragma unroll
      for (int k = 0; k < D / 8; ++k) {
        const uint4 u = reinterpret_cast<const uint4*>(p)[k];
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
        unpack_raw<8>(w, x + 8 * k);
      }
    } else {
#pragma unroll
      for (int k = 0; k < D / 2; ++k) {
        const uint32_t u = p[k];
        x[2 * k] = (int32_t)(u & 0xffffu);
        x[2 * k + 1] = (int32_t)(u >> 16);
      }
    }
    wht_regs<N>(x);
    const uint32_t tot = (uint32_t)x[0];
    double inv = 1.0;
    if constexpr (PB) {
      const uint32_t want = nb_in ? nb_in[tid] : tot;
      if (tot != want) raise_flag(flags, FLAG_SHOTS);
      if (want == 0) raise_flag(flags, FLAG_EMPTY);
      inv = want ? 1.0 / (double)want : 0.0;
    } else {
      if ((uint64_t)tot != shots) raise_flag(flags, FLAG_SHOTS);
    }
#pragma unroll
    for (int m = 0; m < D; ++m) S[tid * DP + m] = PB ? (double)x[m] * inv : (double)x[m];
  }
  __syncthreads();
  // Identity letter of qubit k: rows with letter 0 there collect the other two letters',
  // for the Walsh indices even in bit k.
#pragma unroll
  for (int k = 0; k < N; ++k) {
    constexpr int I = (B / 3) * (D / 2);
    const int p3 = (int)ipow3(k);
    for (int t = tid; t < I; t += 256) {
      const int mi = t % (D / 2), bi = t / (D / 2);
      const int m = ((mi >> k) << (k + 1)) | (mi & ((1 << k) - 1));
      const int b = (bi / p3) * 3 * p3 + bi % p3;
      S[b * DP + m] += S[(b + p3) * DP + m] + S[(b + 2 * p3) * DP + m];
    }
    __syncthreads();
  }
  for (int a = tid; a < NA; a += 256) {
    int b = 0, m = 0;
#pragma unroll
    for (int k = N - 1; k >= 0; --k) {
      const int d = (a >> (2 * k)) & 3;
      b = 3 * b + (d ? d - 1 : 0);
      m = 2 * m + (d != 0);
    }
    const double v = S[b * DP + m];
    const int w = pauli_weight((uint64_t)a);
    if constexpr (MODE == Out::PauliT) {
      static_cast<int64_t*>(out)[a] = (int64_t)v;
    } else {
      const double e = MODE == Out::CoefUniform ? v / (pow3d(N - w) * (double)shots) : v / pow3d(N - w);
      static_cast<double*>(out)[a] = e;
      if constexpr (RHO) E[a] = e;
    }
  }
  if constexpr (RHO) {
    __syncthreads();                       // S is dead, E complete
    rho_low_block<N, true, OutT, 256>(E, rho, N, 0, tid, S, S + RhoLowLds<N>::SIZE);
  }
}

template <int N, bool PB, Out MODE, bool RHO, typename OutT>
__global__ __launch_bounds__(256) void small_estimate_kernel(const uint16_t* __restrict__ counts, uint64_t shots,
                                                             const uint32_t* __restrict__ nb_in,
                                                             void* __restrict__ out, void* __restrict__ rho,
                                                             uint32_t* __restrict__ flags) {
  __shared__ double S[SmallLds<N>::S];
  __shared__ double E[RHO ? SmallLds<N>::E : 1];
  small_estimate_block<N, PB, MODE, RHO, OutT>(counts, shots, nb_in, out, rho, flags, threadIdx.x, S, E);
}

}  // namespace lre
