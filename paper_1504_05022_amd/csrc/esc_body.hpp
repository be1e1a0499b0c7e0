// Expand-sort-compress of up to G*K products per row by an aligned group of
// G lanes of a wavefront (K products per lane), shared by the per-bin
// kernels and the batched per-class kernels.  See esc.hip.
#pragma once

#include "common.hpp"
#include "internal.hpp"

namespace spg {

constexpr int ESC_NT = 256;

template <typename T, int G, int K, typename Key> struct EscShape {
  static constexpr int U = G * K;
  static constexpr int RPB = ESC_NT / G;  // rows per work-group pass
  static constexpr int KB = sizeof(Key) > 4 ? static_cast<int>(sizeof(Key)) : 4;
  static constexpr int HW = (U + 31) / 32;  // words of the run-start mask
  static constexpr size_t a_bytes = static_cast<size_t>(RPB) * U * KB;
  static constexpr size_t b_bytes = static_cast<size_t>(RPB) * U * sizeof(T);
  static constexpr size_t lds_bytes = a_bytes + b_bytes + static_cast<size_t>(RPB) * HW * 4;
};

// A row's G lanes never leave their wavefront (G <= 64) and
// its LDS is its own, so only wavefront-level ordering is needed: the
// wavefronts of a work-group do not wait for each other.  LDS per row: region
// A holds one word per run (non-empty b_j* row), the B index of product l of
// the run less l, and later the sorted keys; region B holds a_ij of each run
// and later the product values; a bit mask holds where the runs start.  A
// group's lanes share one wavefront, so all reads of the first use precede
// the writes of the second in program order.
//
// The run of product l is the number of run starts in products 1 .. l: a
// count of mask bits below the lane, two VALU instructions per product, where
// a segmented max-scan over the products took about twenty and a second
// trip through LDS.
// The rows of a wavefront (64 / G of them, one per group of G lanes) with at
// most G * K products each; the LDS regions are laid out for KL >= K products
// per lane.
template <typename T, int G, int K, int KL, typename Key>
DEVI void esc_rows_k(const EscArgs<T> &a, const RowRec &rw, int64_t out, unsigned char *lds) {
  using Sh = EscShape<T, G, KL, Key>;
  constexpr int UL = G * KL;
  constexpr int U = G * K;
  constexpr int LOGU = ceil_log2(U);
  constexpr Key KMAX = KeyMax<Key>::v;
  const int grp = threadIdx.x / G;
  const int pos = threadIdx.x & (G - 1);
  int32_t *roff = reinterpret_cast<int32_t *>(lds + grp * UL * Sh::KB);
  Key *sk = reinterpret_cast<Key *>(lds + grp * UL * Sh::KB);
  T *ra = reinterpret_cast<T *>(lds + Sh::a_bytes) + grp * UL;
  T *pv = ra;
  uint32_t *hd = reinterpret_cast<uint32_t *>(lds + Sh::a_bytes + Sh::b_bytes) + grp * Sh::HW;
  const int u = rw.u;

  for (int w = pos; w < Sh::HW; w += G) hd[w] = 0u;
  wave_sync();
  // runs: entry e of the row contributes products [P[e]-P[e0], P[e+1]-P[e0]),
  // which start at B's entry bst[e]; the loads of G entries are issued
  // together (clamped, not branched on).  Differences of P fit its low words.
  const int g0 = lane() & ~(G - 1);
  constexpr uint64_t GMASK = G == 64 ? ~0ull : (1ull << (G & 63)) - 1ull;
  const GLOBAL_AS uint32_t *gP = as_global(reinterpret_cast<const uint32_t *>(a.P));
  int nrun = 0;
  uint32_t pbase = 0;
  for (int32_t x0 = 0; x0 < rw.ne; x0 += G) {
    const uint32_t e = static_cast<uint32_t>(rw.e0 + (x0 + pos < rw.ne ? x0 + pos : rw.ne - 1));
    const uint32_t p0 = gP[2 * static_cast<uint64_t>(e)];
    const uint32_t p1 = gP[2 * static_cast<uint64_t>(e) + 2];
    const int32_t b0 = as_global(a.bst)[e];
    const T av = as_global(a.aval)[e];
    if (x0 == 0) pbase = static_cast<uint32_t>(__shfl(static_cast<int>(p0), g0, WAVE));
    const int32_t q0 = static_cast<int32_t>(p0 - pbase);
    const bool some = x0 + pos < rw.ne && p1 != p0;
    const uint64_t mine = (__ballot(some) >> g0) & GMASK;
    if (some) {
      const int r = nrun + __popcll(mine & ((1ull << pos) - 1ull));
      roff[r] = b0 - q0;
      ra[r] = av;
      if (q0 > 0) atomicOr(&hd[(q0 - 1) >> 5], 1u << ((q0 - 1) & 31));
    }
    nrun += __popcll(mine);
  }
  wave_sync();

  // every load of the row is issued before any is used: positions past the
  // end load B's entry 0 (a row with products implies that B has one) and
  // are then ignored.  Product kk * G + pos: consecutive lanes read
  // consecutive entries of each b_j* row.
  int32_t bc[K];
  T bv[K], av[K];
#pragma unroll
  for (int kk = 0; kk < K; ++kk) {
    bc[kk] = 0;
    bv[kk] = T(0);
    av[kk] = T(0);
  }
  if (u > 0) {
    int below = 0;  // run starts in the mask words before this one
#pragma unroll
    for (int kk = 0; kk < K; ++kk) {
      const int l = kk * G + pos;
      int r;
      if constexpr (G == 64) {
        const uint32_t lo = hd[2 * kk], hi = hd[2 * kk + 1];
        r = below + static_cast<int>(
                        __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u)));
        below += __popc(lo) + __popc(hi);
      } else {
        const uint32_t w = hd[kk * G / 32];
        r = below + __popc(w & ((1u << (l & 31)) - 1u));
        if ((kk + 1) * G % 32 == 0) below += __popc(w);
      }
      const uint32_t g = static_cast<uint32_t>(roff[r] + l);
      const uint32_t bidx = l < u ? g : 0u;
      av[kk] = ra[r];
      bc[kk] = as_global(a.bcol)[bidx];
      bv[kk] = as_global(a.bval)[bidx];
    }
  }
  Key key[K];
  T prod[K];
#pragma unroll
  for (int kk = 0; kk < K; ++kk) {
    const int l = kk * G + pos;
    const bool ok = l < u;
    prod[kk] = ok ? av[kk] * bv[kk] : T(0);
    key[kk] = ok ? ((static_cast<Key>(bc[kk]) << LOGU) | static_cast<Key>(l)) : KMAX;
  }
  wave_sync();  // pv takes the place of ra
#pragma unroll
  for (int kk = 0; kk < K; ++kk) {
    const int l = kk * G + pos;
    if (l < u) pv[l] = prod[kk];
  }

  group_bitonic_sort<G, K, Key>(key);
  wave_sync();  // every product is in pv

  // compress: fold every column's products in expansion order (registers),
  // stage the distinct columns in LDS, store them with consecutive lanes
  int32_t *sc = reinterpret_cast<int32_t *>(sk);
  const int total = fold_runs<T, G, K, Key>(key, u, pv, sc, pv, 0);
  if (u > 0) {
    GLOBAL_AS int32_t *dc = as_global_mut(a.ct_col) + out;
    GLOBAL_AS T *dv = as_global_mut(a.ct_val) + out;
    for (int x = pos; x < total; x += G) {
      dc[x] = sc[x];
      dv[x] = pv[x];
    }
    if (pos == 0) as_global_mut(a.rownnz)[rw.row] = total;
  }
  wave_sync();
}

// One pass of a work-group over the rows recs[base .. base + RPB) (those
// below nrows).
//
// A wavefront whose rows all leave part of the capacity unused takes fewer
// products per lane: every step's cost, the sorting network's above all, is
// proportional to K.  Rows of a bin of 257 .. 512 products spread evenly need
// 6.5 of the 8 on average.
template <typename T, int G, int K, typename Key>
DEVI void esc_rows(const EscArgs<T> &a, const RowRec *recs, const int64_t base,
                   const int64_t nrows, unsigned char *lds) {
  const int64_t r = base + threadIdx.x / G;
  RowRec rw{0, 0, 0, 0};
  if (r < nrows) {
    const GLOBAL_AS int32_t *g = as_global(reinterpret_cast<const int32_t *>(recs + r));
    rw.row = g[0];
    rw.u = g[1];
    rw.e0 = g[2];
    rw.ne = g[3];
  }
  // rows of this launch have 1 <= u <= G * K by binning; the check keeps
  // every LDS and global index in range even if that were violated
  if (rw.u > G * K) rw.u = rw.ne = 0;
  if constexpr (G == WAVE) {
    rw.row = __builtin_amdgcn_readfirstlane(rw.row);
    rw.u = __builtin_amdgcn_readfirstlane(rw.u);
    rw.e0 = __builtin_amdgcn_readfirstlane(rw.e0);
    rw.ne = __builtin_amdgcn_readfirstlane(rw.ne);
  }
  const int64_t out = rw.u > 0 ? as_global(a.cto)[rw.row] : 0;
  if constexpr (sizeof(Key) == 4 && K == 8) {
    if (!__any(rw.u > G * 5)) return esc_rows_k<T, G, 5, K, Key>(a, rw, out, lds);
    if (!__any(rw.u > G * 6)) return esc_rows_k<T, G, 6, K, Key>(a, rw, out, lds);
    if (!__any(rw.u > G * 7)) return esc_rows_k<T, G, 7, K, Key>(a, rw, out, lds);
  }
  if constexpr (sizeof(Key) == 4 && K == 16) {
    if (!__any(rw.u > G * 10)) return esc_rows_k<T, G, 10, K, Key>(a, rw, out, lds);
    if (!__any(rw.u > G * 12)) return esc_rows_k<T, G, 12, K, Key>(a, rw, out, lds);
  }
  esc_rows_k<T, G, K, K, Key>(a, rw, out, lds);
}

}  // namespace spg
