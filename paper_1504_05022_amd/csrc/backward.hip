// Backward of C = A*B for L = <dC, C> on the fixed patterns of A and B:
//   dA_ij = sum over stored b_jk of dC_ik * b_jk       ((dC B^T) on S(A))
//   dB_jk = sum over stored a_ij of a_ij * dC_ik       ((A^T dC) on S(B))
// Every (i, k) reached lies in S(C) because S(C) is the structural product.
// Both are gathers (no floating-point atomics).  dA, and the products
// a_ij dC_ik of dB, come from a product-parallel pass over A; dB then adds
// those products per b_jk over A's transposed pattern (rows of each column in
// ascending order).  Without room for the products, dB is gathered per row
// of B with binary searches in C.  dB sums run in the order of the
// definition (ascending i) from +0.0; a dA sum adds blocks of 64 products as
// a tree across the lanes, block by block (a fixed order).
#include "common.hpp"
#include "internal.hpp"
#include "launch_rules.hpp"

namespace spg {

DEVI int32_t find_col(const int32_t *col, int32_t lo, int32_t hi, int32_t c) {
  while (lo < hi) {
    const int32_t mid = (lo + hi) >> 1;
    if (col[mid] < c)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

template <typename T>
__global__ __launch_bounds__(256) void k_grad_b(const int64_t *tptr, const int32_t *trow,
                                                const int32_t *tpos, const T *aval,
                                                const int32_t *brp, const int32_t *bcol,
                                                int64_t kb, const int32_t *crp,
                                                const int32_t *ccol, const T *dc, T *dB) {
  const int64_t j = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) / WAVE;
  if (j >= kb) return;
  const int64_t t0 = tptr[j], t1 = tptr[j + 1];
  for (int32_t q = brp[j] + lane(); q < brp[j + 1]; q += WAVE) {
    const int32_t c = bcol[q];
    T s = T(0);
    for (int64_t d = t0; d < t1; ++d) {
      const int32_t i = trow[d];
      const int32_t pc = find_col(ccol, crp[i], crp[i + 1], c);
      s = s + aval[tpos[d]] * dc[pc];
    }
    dB[q] = s;
  }
}

// ---------------------------------------------------------------------------
// Product-parallel form.  One wavefront per chunk of BW_CH consecutive
// entries of A, 64 entries at a time, whose products it takes in expansion
// order, one per lane: consecutive lanes read consecutive entries of b_j* and
// write consecutive products of W.  For product q of entry e = (i, j),
// y = dC_ik is looked up -- by its rank in an LDS bitmap of the row's columns
// when C has few columns, else by a binary search in c_i*, whose first steps
// go over samples of the rows in LDS (every step in global memory: 168 us wide,
// then 136; 512 / 2048 samples 138 / 138) -- and
//   dA_e = sum of y * b_jk        (a segmented scan across the lanes)
//   W[P_e + q] = a_ij * y         (q = position of b_jk in b_j*)
// where P_e is the product offset of entry e from stage 1.  W holds every
// product a_ij dC_ik of the dB sums; k_grad_b_sum adds them per b_jk over
// A's transposed pattern (ascending i).
//
// The entry of a product comes from a bit mask of the entries' first
// products (LDS, BW_WIN products at a time) and a count of the bits below the
// lane, so the lanes stay full whatever the row lengths of B.
//
// What bounds it: latency and the B rows gathered past the L2 (one 128-byte
// line or two per b_j* and array); the VALU is busy 58% of the time where B is
// narrow.  One lane per entry of A, as before, left ragged rows waiting on their longest entry and
// touched 64 lines per load: 2374 us where B is narrow (A 300000^2 with 6M
// entries x B 300000x4096, 32 per row, binary32; now 1046), 1389 us where it
// is wide (A 50000^2 with 600k entries x B 50000^2, 12 per row, binary64; now
// 119).  The chunk's rows are found by the whole wavefront (wave_row_of; a
// bisection by one lane: 1187 and 136).  Few entries per chunk spread the long
// tail of a product; with the bitmap a row cut by a chunk is mapped
// twice, so chunks are longer there (64 / 128 / 256 entries 1128 / 1098 / 1112
// us narrow, 64 / 128 136 / 163 wide, each when measured).  A small A takes
// smaller chunks (grad_chunk).  Overlapping the next group's
// loads of B with this group's dC costs more in resident wavefronts than it
// hides (1371).
constexpr int BW_WIN = 2048;  // products whose entry starts the bit mask covers
template <bool DENSE> constexpr int bw_ch() { return DENSE ? 128 : 64; }
// blocks of 64 products whose loads are in flight together (narrow: 3 / 4 / 6
// blocks 1333 / 1257 / 1187 us; wide: 134 / 128 / 119)
constexpr int BW_U = 6;
// consecutive entries of a row of C per lane when its columns are mapped: a
// lane joins the bits that fall into one word, so that few lanes meet on one
// (one entry per lane: 1100 us narrow, now 1046; 2 / 8 per lane 1083 / 1170),
// and passes of loads in flight when they are sampled
constexpr int BW_SC = 4;
// columns of the bitmap: 1 KB of it and 512 bytes of ranks per wavefront,
// where a dense copy of a dC row of 4096 columns took 16 KB and left 9
// wavefronts per CU (the same time, but only up to 2048 binary64 columns)
constexpr int BW_MAP = 8192;
constexpr int BW_MW = BW_MAP / 32 / WAVE;  // its words per lane

// Last row i of [lo, hi) with arp[i] <= e (arp[lo] <= e): the row that holds
// entry e, empty rows skipped.
DEVI int32_t row_of(const int32_t *arp, int32_t lo, int32_t hi, int64_t e) {
  while (hi - lo > 1) {
    const int32_t mid = lo + ((hi - lo) >> 1);
    if (arp[mid] <= e)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// The same by a whole wavefront for one e.
DEVI int32_t wave_row_of(const int32_t *arp, int32_t lo, int32_t hi, int64_t e) {
  return static_cast<int32_t>(wave_last(lo, hi, [&](int64_t i) { return arp[i] <= e; }));
}

// Sums of the lanes from the last segment head at or below each lane (dist
// lanes down; 64 or more: none in the wavefront) up to the lane itself.
template <typename T> DEVI T segment_scan(T v, int dist) {
  const int ln = lane();
  T y = dpp_move<DPP_ROW_SHR + 1, 0xF>(v, T(0));
  v = v + (dist >= 1 ? y : T(0));
  y = dpp_move<DPP_ROW_SHR + 2, 0xF>(v, T(0));
  v = v + (dist >= 2 ? y : T(0));
  y = dpp_move<DPP_ROW_SHR + 4, 0xF>(v, T(0));
  v = v + (dist >= 4 ? y : T(0));
  y = dpp_move<DPP_ROW_SHR + 8, 0xF>(v, T(0));
  v = v + (dist >= 8 ? y : T(0));
  y = dpp_move<DPP_ROW_BCAST15, 0xA>(v, T(0));
  v = v + (dist > (ln & 15) ? y : T(0));
  y = dpp_move<DPP_ROW_BCAST31, 0xC>(v, T(0));
  v = v + (dist > (ln & 31) ? y : T(0));
  return v;
}

// wide C: columns of the batch's rows of C that are held in LDS, for the first
// steps of the searches
constexpr int BW_SAMPLES = 1024;

template <typename T, bool DENSE> struct GradTable {
  alignas(16) uint32_t bits[DENSE ? BW_MAP / 32 : 4];  // columns of one row of C
  uint16_t rank[DENSE ? BW_MAP / 32 : 1];              // columns before each word
  uint32_t head[BW_WIN / 32];  // bit x: an entry starts at product x + 1 of the window
  int32_t off[WAVE];           // entry with products: index in B of the window's product 0
  uint32_t ent[WAVE];          // its lane (entry of the batch)
  int32_t row[WAVE];           // dense: its row
  T av[WAVE];
  int32_t c0[DENSE ? 1 : WAVE], c1[DENSE ? 1 : WAVE];  // its row of C, less cs
  int32_t sample[DENSE ? 1 : BW_SAMPLES];  // every 2^sh-th column of the batch's rows of C
};

constexpr int BW_NT = 256;  // four independent wavefronts

template <typename T, bool DENSE>
__global__ __launch_bounds__(BW_NT) void k_grad_entries(
    const int32_t *arp, const T *aval, int64_t m, int64_t nnz,
    const int64_t *P, const int32_t *bst, const int32_t *bcol, const T *bval, const int32_t *crp,
    const int32_t *ccol, const T *dc, T *dA, T *W, int ch) {
  constexpr int NWV = BW_NT / WAVE;
  __shared__ GradTable<T, DENSE> tabs[NWV];
  const int w = threadIdx.x / WAVE;
  const int ln = lane();
  GradTable<T, DENSE> &tb = tabs[w];
  const int64_t e0 = (static_cast<int64_t>(blockIdx.x) * NWV + w) * ch;
  if (e0 >= nnz) return;  // uniform across the wavefront; no work-group barriers here
  const int64_t e1 = e0 + ch < nnz ? e0 + ch : nnz;
  // its rows [row_lo, row_hi), mostly within 64: their starts one per lane
  const int32_t row_lo = wave_row_of(arp, 0, static_cast<int32_t>(m), e0);
  const int32_t ahead = m - row_lo < WAVE ? static_cast<int32_t>(m) - row_lo : WAVE;
  const int32_t start = arp[row_lo + (ln < ahead ? ln : 0)];
  const int32_t rows = __popcll(__ballot(ln < ahead && start < e1));
  int32_t row_hi = row_lo + rows;
  if (rows == WAVE) row_hi = wave_row_of(arp, row_hi - 1, static_cast<int32_t>(m), e1 - 1) + 1;
  int32_t mapped = -1;  // row in the bitmap
  int32_t mapped_c0 = 0;  // its first entry of C
  const uint64_t le_mask = ~0ull >> (WAVE - 1 - ln);
  for (int64_t eb = e0; eb < e1; eb += WAVE) {
    const int nb = static_cast<int>(e1 - eb < WAVE ? e1 - eb : WAVE);
    const bool in = ln < nb;
    const int64_t e = in ? eb + ln : e1 - 1;
    const int32_t q0 = bst[e];
    const T av = aval[e];
    const int64_t Pb = P[eb];
    const int64_t pre = P[e] - Pb;
    const int64_t len = P[e + 1] - Pb - pre;
    const int64_t tot = P[eb + nb] - Pb;
    int32_t row = row_lo;
    if (row_hi - row_lo <= WAVE) {
      for (int r = 1; r < rows; ++r)
        row += __builtin_amdgcn_readlane(start, r) <= static_cast<int32_t>(e) ? 1 : 0;
    } else {
      row = row_of(arp, row_lo, row_hi, e);
    }
    const int32_t c0 = crp[row], c1 = crp[row + 1];
    const bool some = in && len > 0;
    const int c = __popcll(__ballot(some) & (le_mask >> 1));  // entries with products below
    // wide C: the batch's rows of C begin at entry cs; samples 2^sh apart
    const int32_t cs = __builtin_amdgcn_readfirstlane(c0);
    int sh = 0;
    wave_sync();  // the previous batch's table is dead
    if (some) {
      tb.ent[c] = ln;
      tb.row[c] = row;
      tb.av[c] = av;
      if (!DENSE) {
        tb.c0[c] = c0 - cs;
        tb.c1[c] = c1 - cs;
      }
    }
    if (!DENSE && tot > 0) {
      const int32_t L = __builtin_amdgcn_readlane(c1, nb - 1) - cs;
      const int32_t most =
          tot < WAVE ? WAVE : tot < BW_SAMPLES ? static_cast<int32_t>(tot) : BW_SAMPLES;
      while (((L - 1) >> sh) >= most) ++sh;
      const int32_t last = (L - 1) >> sh;
      for (int32_t xs = 0; xs <= last; xs += BW_SC * WAVE) {
        int32_t cc[BW_SC];
#pragma unroll
        for (int p = 0; p < BW_SC; ++p) {
          const int32_t x = xs + p * WAVE + ln;
          cc[p] = ccol[cs + ((x < last ? x : last) << sh)];
        }
#pragma unroll
        for (int p = 0; p < BW_SC; ++p) {
          const int32_t x = xs + p * WAVE + ln;
          if (x <= last) tb.sample[x] = cc[p];
        }
      }
    }
    if (dA && in && len == 0) dA[e] = T(0);
    T carry = T(0);  // running sum of the entry left open by the previous block
    for (int64_t xw = 0; xw < tot; xw += BW_WIN) {
      const int wl = static_cast<int>(tot - xw < BW_WIN ? tot - xw : BW_WIN);
      const int64_t d = pre - xw;  // this entry's first product in the window
      tb.head[ln] = 0u;
      wave_sync();
      if (some) {
        tb.off[c] = static_cast<int32_t>(q0 - d);  // used when the entry reaches the window
        if (d >= 1 && d <= BW_WIN)
          atomicOr(&tb.head[(d - 1) >> 5], 1u << ((d - 1) & 31));
      }
      // entries that start at or before the window's first product, less
      // one: the entry of that product; whether it is the entry's first
      int base = __popcll(__ballot(some && d <= 0)) - 1;
      uint64_t starts = __any(some && d == 0) ? 1ull : 0ull;
      wave_sync();
      // groups of BW_U blocks whose loads are in flight together
      struct Group {
        int ce[BW_U];
        int32_t kk[BW_U];
        T bv[BW_U];
        uint64_t hm[BW_U];
      };
      auto load_group = [&](int x0, Group &g) {
#pragma unroll
        for (int u = 0; u < BW_U; ++u) {
          const int xb = x0 + u * WAVE;
          const int wd = xb < BW_WIN ? xb / 32 : 0;
          const uint32_t lo = __builtin_amdgcn_readfirstlane(tb.head[wd]);
          const uint32_t hi = __builtin_amdgcn_readfirstlane(tb.head[wd + 1]);
          const bool ok = xb + ln < wl;
          g.hm[u] = (static_cast<uint64_t>(hi) << 32) | lo;
          g.ce[u] = ok ? base + static_cast<int>(__builtin_amdgcn_mbcnt_hi(
                                    hi, __builtin_amdgcn_mbcnt_lo(lo, 0u)))
                       : 0;
          base += __popcll(g.hm[u]);
          // clamped, not branched around: the loads of a group stay in
          // flight together (B has entries whenever A's have products)
          const int32_t bx = ok ? tb.off[g.ce[u]] + xb + ln : 0;
          g.kk[u] = bcol[bx];
          g.bv[u] = bval[bx];
        }
      };
      for (int x0 = 0; x0 < wl; x0 += BW_U * WAVE) {
        Group cur;
        load_group(x0, cur);
        int32_t at[BW_U];  // where C holds the products' columns
        if (DENSE) {
#pragma unroll
          for (int u = 0; u < BW_U; ++u) {
            at[u] = 0;
            if (x0 + u * WAVE >= wl) continue;
            const bool ok = x0 + u * WAVE + ln < wl;
            const int32_t r = tb.row[cur.ce[u]];
            uint64_t todo = __ballot(ok);
            while (todo) {  // the rows among the block's products, in order
              const int32_t rc = __builtin_amdgcn_readlane(r, __builtin_ctzll(todo));
              if (rc != mapped) {
                uint4 *bw = reinterpret_cast<uint4 *>(tb.bits);
                static_assert(BW_MW == 4, "one 16-byte word group per lane");
                wave_sync();  // the previous row's lookups are done
                bw[ln] = make_uint4(0u, 0u, 0u, 0u);
                wave_sync();
                const int hl = __builtin_ctzll(__ballot(some && row == rc));
                const int32_t m0 = __builtin_amdgcn_readlane(c0, hl);
                const int32_t m1 = __builtin_amdgcn_readlane(c1, hl);
                for (int32_t xs = m0; xs < m1; xs += BW_SC * WAVE) {
                  int32_t cc[BW_SC];
                  const int32_t x = xs + ln * BW_SC;
#pragma unroll
                  for (int p = 0; p < BW_SC; ++p) cc[p] = ccol[x + p < m1 ? x + p : m1 - 1];
                  if (x < m1) {
                    int32_t wd = cc[0] >> 5;
                    uint32_t mk = 1u << (cc[0] & 31);
#pragma unroll
                    for (int p = 1; p < BW_SC; ++p) {
                      const bool next = cc[p] >> 5 != wd;
                      if (next) atomicOr(&tb.bits[wd], mk);
                      mk = (next ? 0u : mk) | 1u << (cc[p] & 31);
                      wd = cc[p] >> 5;
                    }
                    atomicOr(&tb.bits[wd], mk);
                  }
                }
                mapped = rc;
                mapped_c0 = m0;
                wave_sync();
                const uint4 b4 = bw[ln];
                const int n0 = __popc(b4.x), n1 = n0 + __popc(b4.y), n2 = n1 + __popc(b4.z);
                const int n3 = n2 + __popc(b4.w);
                const int before = group_incl_sum<WAVE>(n3) - n3;
                uint16_t *rk = tb.rank + BW_MW * ln;
                rk[0] = static_cast<uint16_t>(before);
                rk[1] = static_cast<uint16_t>(before + n0);
                rk[2] = static_cast<uint16_t>(before + n1);
                rk[3] = static_cast<uint16_t>(before + n2);
                wave_sync();
              }
              const bool mine = ok && r == rc;
              if (mine) {
                const int wd = cur.kk[u] >> 5;
                at[u] = mapped_c0 + tb.rank[wd] +
                        __popc(tb.bits[wd] & ((1u << (cur.kk[u] & 31)) - 1u));
              }
              todo &= ~__ballot(mine);
            }
          }
        } else {
          // lower bounds of the BW_U columns in their rows of C, one step of
          // every search at a time (their loads are in flight together): the
          // first sample of the row that is not below, then the entries
          // between it and the sample before
          int32_t lo[BW_U], hi[BW_U], a0[BW_U], a1[BW_U];
          int32_t most = 0;
          const int32_t up = (1 << sh) - 1;
#pragma unroll
          for (int u = 0; u < BW_U; ++u) {
            const bool ok = x0 + u * WAVE + ln < wl;
            a0[u] = ok ? tb.c0[cur.ce[u]] : 0;
            a1[u] = ok ? tb.c1[cur.ce[u]] : 0;
            lo[u] = (a0[u] + up) >> sh;
            hi[u] = (a1[u] + up) >> sh;
            most = max(most, hi[u] - lo[u]);
          }
          while (__any(most > 0)) {
            int32_t mc[BW_U];
#pragma unroll
            for (int u = 0; u < BW_U; ++u) {
              const int32_t mid = (lo[u] + hi[u]) >> 1;
              mc[u] = tb.sample[lo[u] < hi[u] ? mid : 0];
            }
            most = 0;
#pragma unroll
            for (int u = 0; u < BW_U; ++u) {
              const int32_t mid = (lo[u] + hi[u]) >> 1;
              const bool open = lo[u] < hi[u], below = mc[u] < cur.kk[u];
              lo[u] = open && below ? mid + 1 : lo[u];
              hi[u] = open && !below ? mid : hi[u];
              most = max(most, hi[u] - lo[u]);
            }
          }
          most = 0;
#pragma unroll
          for (int u = 0; u < BW_U; ++u) {
            const int32_t t = lo[u] << sh;
            lo[u] = cs + max(a0[u], t - up);
            hi[u] = cs + min(a1[u], t);
            most = max(most, hi[u] - lo[u]);
          }
          while (__any(most > 0)) {
            int32_t mc[BW_U];
#pragma unroll
            for (int u = 0; u < BW_U; ++u) {
              const int32_t mid = lo[u] + ((hi[u] - lo[u]) >> 1);
              mc[u] = lo[u] < hi[u] ? ccol[mid] : 0;
            }
            most = 0;
#pragma unroll
            for (int u = 0; u < BW_U; ++u) {
              if (lo[u] < hi[u]) {
                const int32_t mid = lo[u] + ((hi[u] - lo[u]) >> 1);
                if (mc[u] < cur.kk[u])
                  lo[u] = mid + 1;
                else
                  hi[u] = mid;
              }
              most = max(most, hi[u] - lo[u]);
            }
          }
#pragma unroll
          for (int u = 0; u < BW_U; ++u) at[u] = x0 + u * WAVE + ln < wl ? lo[u] : 0;
        }
        T y[BW_U];
#pragma unroll
        for (int u = 0; u < BW_U; ++u) y[u] = dc[at[u]];  // (C has entries when A's have products)
#pragma unroll
        for (int u = 0; u < BW_U; ++u) {
          const int xb = x0 + u * WAVE;
          if (xb >= wl) continue;
          const bool ok = xb + ln < wl;
          if (W && ok) W[Pb + xw + xb + ln] = tb.av[cur.ce[u]] * y[u];
          if (dA) {
            const uint64_t heads = (cur.hm[u] << 1) | starts;
            starts = cur.hm[u] >> 63;
            const uint64_t mine = heads & le_mask;
            const int dist = mine ? ln - (63 - __builtin_clzll(mine)) : WAVE;
            T v = segment_scan<T>(ok ? y[u] * cur.bv[u] : T(0), dist);
            if (!mine) v = v + carry;
            const bool tail = ((cur.hm[u] >> ln) & 1ull) || xw + xb + ln == tot - 1;
            if (ok && tail) dA[eb + tb.ent[cur.ce[u]]] = v;
            const uint64_t open = ~cur.hm[u] >> 63;
            const T last = __shfl(v, WAVE - 1, WAVE);
            carry = open ? last : T(0);
          }
        }
      }
      wave_sync();  // the window's table is rewritten
    }
  }
}

// dB_jk = sum over A's column j (ascending i) of the products a_ij dC_ik in W.
// BW_SUB lanes per row of B (each lane sums its own entries, so rows share a
// wavefront without any ordering between them).  Bound by the gathers of W
// past the L2 (128 bytes per entry of A and row of B: 710 MB, 266 us for the
// narrow B above; 27 us for the wide one).  The lanes fetch the product
// offsets of BW_SUB entries of A's column together and share them through
// LDS (each lane fetching those of the next BW_SU products itself, three
// dependent loads per BW_SU: 284 and 35 us); then BW_SU products are in flight
// per lane (16: the same).  16 lanes: 471 and 27 us, 64: 269 narrow.
constexpr int BW_SUB = 32;
constexpr int BW_SU = 8;

template <typename T>
__global__ __launch_bounds__(256) void k_grad_b_sum(const int64_t *tptr, const int32_t *tpos,
                                                    const int64_t *P, const int32_t *brp,
                                                    int64_t kb, const T *W, T *dB) {
  __shared__ int64_t offs[256];
  const int64_t j = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) / BW_SUB;
  if (j >= kb) return;  // the lanes of a group together; no work-group barriers here
  const int l = lane() & (BW_SUB - 1);
  int64_t *off = offs + (threadIdx.x - l);
  const int64_t t0 = tptr[j], t1 = tptr[j + 1];
  const int32_t q0 = brp[j], q1 = brp[j + 1];
  for (int32_t qb = q0; qb < q1; qb += BW_SUB) {
    const int32_t q = qb + l;
    const GLOBAL_AS T *Wq = as_global(W) + (q < q1 ? q - q0 : 0);
    T s = T(0);
    for (int64_t db = t0; db < t1; db += BW_SUB) {
      const int n = static_cast<int>(t1 - db < BW_SUB ? t1 - db : BW_SUB);
      wave_sync();  // the previous offsets are read
      off[l] = P[tpos[db + (l < n ? l : n - 1)]];
      wave_sync();
      for (int d = 0; d < n; d += BW_SU) {
        T v[BW_SU];  // entries past the end reread the last one and are not added
#pragma unroll
        for (int u = 0; u < BW_SU; ++u) v[u] = Wq[off[d + u < n ? d + u : n - 1]];
#pragma unroll
        for (int u = 0; u < BW_SU; ++u) s = d + u < n ? s + v[u] : s;
      }
    }
    if (q < q1) dB[q] = s;
  }
}

template <typename T>
void launch_grad_entries(const int32_t *arp, const T *aval, int64_t m, int64_t nnz,
                         const int64_t *P, const int32_t *bst, int64_t products,
                         const int32_t *bcol, const T *bval, int64_t n, const int32_t *crp,
                         const int32_t *ccol, const T *dc, T *dA, T *W, hipStream_t s) {
  if (nnz <= 0) return;
  const int ch = grad_chunk(n <= BW_MAP ? bw_ch<true>() : bw_ch<false>(), nnz, products);
  const int64_t per = int64_t(BW_NT / WAVE) * ch;
  hipLaunchKernelGGL((n <= BW_MAP ? k_grad_entries<T, true> : k_grad_entries<T, false>),
                     dim3((nnz + per - 1) / per), dim3(BW_NT), 0, s, arp, aval, m, nnz, P, bst, bcol,
                     bval, crp, ccol, dc, dA, W, ch);
}

template <typename T>
void launch_grad_b_sum(const int64_t *tptr, const int32_t *tpos, const int64_t *P,
                       const int32_t *brp, int64_t kb, const T *W, T *dB, hipStream_t s) {
  if (kb <= 0) return;
  hipLaunchKernelGGL((k_grad_b_sum<T>), dim3((kb * BW_SUB + 255) / 256), dim3(256), 0, s, tptr,
                     tpos, P, brp, kb, W, dB);
}

template void launch_grad_entries<float>(const int32_t *, const float *, int64_t,
                                         int64_t, const int64_t *, const int32_t *, int64_t,
                                         const int32_t *, const float *, int64_t,
                                         const int32_t *, const int32_t *, const float *, float *,
                                         float *, hipStream_t);
template void launch_grad_entries<double>(const int32_t *, const double *,
                                          int64_t, int64_t, const int64_t *, const int32_t *,
                                          int64_t, const int32_t *, const double *, int64_t,
                                          const int32_t *, const int32_t *, const double *,
                                          double *, double *, hipStream_t);
template void launch_grad_b_sum<float>(const int64_t *, const int32_t *, const int64_t *,
                                      const int32_t *, int64_t, const float *, float *, hipStream_t);
template void launch_grad_b_sum<double>(const int64_t *, const int32_t *, const int64_t *,
                                      const int32_t *, int64_t, const double *, double *, hipStream_t);

// Column counts of A.
__global__ void k_col_count(const int32_t *acol, int64_t nnz, int32_t *cnt) {
  const int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e < nnz) atomicAdd(&cnt[acol[e]], 1);
}

// Scatter (row, position) of every entry into its column's segment, in any
// order; k_col_sort restores ascending rows.  One wavefront per chunk of
// TS_CH consecutive entries (rows found by one binary search per wavefront,
// then walked per lane), TS_U entries per lane whose column loads and slot
// atomics are in flight together.
constexpr int TS_U = 4;
constexpr int TS_CH = WAVE * TS_U;

__global__ __launch_bounds__(256) void k_col_scatter(const int32_t *arp, const int32_t *acol,
                                                     int64_t m, int64_t nnz, const int64_t *tptr,
                                                     int32_t *fill, int32_t *trow,
                                                     int32_t *tpos) {
  const int64_t e0 = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) / WAVE * TS_CH;
  if (e0 >= nnz) return;  // uniform across the wavefront
  int64_t lo = 0, hi = m;  // the row holding e0: last i with arp[i] <= e0
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (arp[mid] <= e0)
      lo = mid;
    else
      hi = mid;
  }
  int64_t e[TS_U], row[TS_U];
  int32_t col[TS_U], slot[TS_U];
  int64_t i = lo;
#pragma unroll
  for (int u = 0; u < TS_U; ++u) {
    e[u] = e0 + u * WAVE + lane();
    if (e[u] < nnz)
      while (arp[i + 1] <= e[u]) ++i;  // entries ascend with u, so rows do too
    row[u] = i;
  }
#pragma unroll
  for (int u = 0; u < TS_U; ++u) col[u] = e[u] < nnz ? acol[e[u]] : 0;
#pragma unroll
  for (int u = 0; u < TS_U; ++u) slot[u] = e[u] < nnz ? atomicAdd(&fill[col[u]], 1) : 0;
#pragma unroll
  for (int u = 0; u < TS_U; ++u) {
    if (e[u] < nnz) {
      const int64_t d = tptr[col[u]] + slot[u];
      trow[d] = static_cast<int32_t>(row[u]);
      tpos[d] = static_cast<int32_t>(e[u]);
    }
  }
}

// Insertion sort of every column segment by row (rows are distinct).
__global__ void k_col_sort(const int64_t *tptr, int64_t k, int32_t *trow, int32_t *tpos) {
  const int64_t j = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (j >= k) return;
  const int64_t a = tptr[j], b = tptr[j + 1];
  for (int64_t x = a + 1; x < b; ++x) {
    const int32_t r = trow[x], p = tpos[x];
    int64_t y = x - 1;
    while (y >= a && trow[y] > r) {
      trow[y + 1] = trow[y];
      tpos[y + 1] = tpos[y];
      --y;
    }
    trow[y + 1] = r;
    tpos[y + 1] = p;
  }
}

void launch_transpose_pattern(const int32_t *arp, const int32_t *acol, int64_t m, int64_t k,
                              int64_t nnz, int32_t *cnt, int64_t *tptr, int32_t *trow,
                              int32_t *tpos, int64_t *part, hipStream_t s) {
  launch_zero(cnt, static_cast<size_t>(k) * 4, s);
  if (nnz > 0)
    hipLaunchKernelGGL(k_col_count, dim3((nnz + 255) / 256), dim3(256), 0, s, acol, nnz, cnt);
  scan_i32(cnt, k, tptr, part, s);
  launch_zero(cnt, static_cast<size_t>(k) * 4, s);
  if (nnz > 0) {
    const int64_t waves = (nnz + TS_CH - 1) / TS_CH;
    hipLaunchKernelGGL(k_col_scatter, dim3((waves * WAVE + 255) / 256), dim3(256), 0, s, arp,
                       acol, m, nnz, tptr, cnt, trow, tpos);
  }
  if (k > 0)
    hipLaunchKernelGGL(k_col_sort, dim3((k + 255) / 256), dim3(256), 0, s, tptr, k, trow, tpos);
}

// ------------------------------------------------ transposed pattern by parts
//
// Stable and without global atomics, for plans, which can afford the space:
// A's entries are partitioned by groups of W columns (tiles of TP_TILE
// entries, one count per tile and group, one scan), then every group is
// partitioned by column by one work-group.  Both steps keep the order of the
// entries, so a column's positions ascend, and with them its rows, without
// a sort.  A wavefront places 64 entries at a time: entries of one bucket find
// each other by one ballot per key bit, and a counter per wavefront and
// bucket gives their place.
//
// 6M entries in 300000 columns: counting 204, slot atomics and scatter 292,
// per-column insertion sorts 294 us before; now 165 us in all (73 to partition,
// 73 to order the groups).
constexpr int TP_NT = 256;
constexpr int TP_NW = TP_NT / WAVE;
constexpr int TP_WAVE_ENTRIES = 2048;
constexpr int TP_TILE = TP_NW * TP_WAVE_ENTRIES;
constexpr int TP_GROUPS = 1024;     // column groups at most (16 KB of counters)
constexpr int TP_WIDTH_LOG = 11;    // columns per group at most (32 KB of counters)
constexpr int TP_GROUP_ENTRIES = 8192;  // entries per group aimed at

struct TpEntry {
  int32_t e, col;
};

// Place of this lane's entry (bucket b < 2^bits; ok: there is one) after the
// entries of its bucket before it; advances the bucket's counter.
DEVI int32_t tp_place(bool ok, uint32_t b, int bits, int32_t *cur) {
  uint64_t same = __ballot(ok);
  for (int k = 0; k < bits; ++k) {
    const bool bit = (b >> k) & 1u;
    const uint64_t m = __ballot(ok && bit);
    same &= bit ? m : ~m;
  }
  const uint64_t below = same & ((1ull << lane()) - 1ull);
  int32_t at = 0;
  if (ok) at = cur[b] + __popcll(below);
  wave_sync();
  if (ok && (same >> lane()) == 1ull) cur[b] = at + 1;  // the bucket's last lane
  wave_sync();
  return at;
}

// Entries of every column group in every tile: table[group * tiles + tile].
__global__ __launch_bounds__(TP_NT) void k_tp_count(const int32_t *acol, int64_t nnz, int wlog,
                                                    int groups, int32_t *table) {
  __shared__ int32_t cnt[TP_GROUPS];
  for (int g = threadIdx.x; g < groups; g += TP_NT) cnt[g] = 0;
  __syncthreads();
  const int64_t e0 = static_cast<int64_t>(blockIdx.x) * TP_TILE;
  int32_t c[TP_TILE / TP_NT];
#pragma unroll
  for (int j = 0; j < TP_TILE / TP_NT; ++j) {
    const int64_t e = e0 + j * TP_NT + threadIdx.x;
    c[j] = acol[e < nnz ? e : nnz - 1];
  }
#pragma unroll
  for (int j = 0; j < TP_TILE / TP_NT; ++j)
    if (e0 + j * TP_NT + threadIdx.x < nnz) atomicAdd(&cnt[c[j] >> wlog], 1);
  __syncthreads();
  for (int g = threadIdx.x; g < groups; g += TP_NT)
    table[static_cast<int64_t>(g) * gridDim.x + blockIdx.x] = cnt[g];
}

// Entries to their column groups, in order (off: scanned table).
__global__ __launch_bounds__(TP_NT) void k_tp_part(const int32_t *acol, int64_t nnz, int wlog,
                                                   int groups, int gbits, const int64_t *off,
                                                   TpEntry *out) {
  __shared__ int32_t cur[TP_NW][TP_GROUPS];
  const int w = threadIdx.x / WAVE;
  for (int g = threadIdx.x; g < TP_NW * TP_GROUPS; g += TP_NT) (&cur[0][0])[g] = 0;
  __syncthreads();
  const int64_t e0 = static_cast<int64_t>(blockIdx.x) * TP_TILE + w * TP_WAVE_ENTRIES;
  constexpr int ROWS = TP_WAVE_ENTRIES / WAVE;
  int32_t c[ROWS];
#pragma unroll
  for (int j = 0; j < ROWS; ++j) {
    const int64_t e = e0 + j * WAVE + lane();
    c[j] = acol[e < nnz ? e : nnz - 1];
  }
#pragma unroll
  for (int j = 0; j < ROWS; ++j)
    if (e0 + j * WAVE + lane() < nnz) atomicAdd(&cur[w][c[j] >> wlog], 1);
  __syncthreads();
  for (int g = threadIdx.x; g < groups; g += TP_NT) {
    int32_t at = static_cast<int32_t>(off[static_cast<int64_t>(g) * gridDim.x + blockIdx.x]);
#pragma unroll
    for (int q = 0; q < TP_NW; ++q) {
      const int32_t n = cur[q][g];
      cur[q][g] = at;
      at += n;
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < ROWS; ++j) {
    const int64_t e = e0 + j * WAVE + lane();
    const bool ok = e < nnz;
    const int32_t at = tp_place(ok, static_cast<uint32_t>(c[j]) >> wlog, gbits, cur[w]);
    if (ok) out[at] = TpEntry{static_cast<int32_t>(e), c[j]};
  }
}

// One work-group per column group: its columns' pointers, and its entries by
// column, in order.
__global__ __launch_bounds__(TP_NT) void k_tp_columns(const TpEntry *in, const int64_t *off,
                                                      int64_t tiles, int64_t k, int wlog,
                                                      int64_t *tptr, int32_t *tpos) {
  extern __shared__ int32_t cur[];  // [TP_NW][width]
  __shared__ int64_t sm[TP_NT / WAVE + 1];
  const int width = 1 << wlog;
  const int w = threadIdx.x / WAVE;
  const int64_t g = blockIdx.x;
  const int64_t s0 = off[g * tiles], s1 = off[(g + 1) * tiles];
  for (int x = threadIdx.x; x < TP_NW * width; x += TP_NT) cur[x] = 0;
  __syncthreads();
  // a quarter of the group per wavefront
  const int64_t per = (s1 - s0 + TP_NW * WAVE - 1) / (TP_NW * WAVE) * WAVE;
  const int64_t w0 = s0 + w * per < s1 ? s0 + w * per : s1;
  const int64_t w1 = w0 + per < s1 ? w0 + per : s1;
  int32_t *mine = cur + w * width;
  for (int64_t x = w0 + lane(); x < w1; x += WAVE) atomicAdd(&mine[in[x].col & (width - 1)], 1);
  __syncthreads();
  int64_t base = s0;
  for (int c0 = 0; c0 < width; c0 += TP_NT) {
    const int c = c0 + threadIdx.x;
    int64_t n = 0, tot;
    if (c < width)
      for (int q = 0; q < TP_NW; ++q) n += cur[q * width + c];
    const int64_t at = base + block_excl_sum<TP_NT>(n, sm, tot);
    if (c < width) {
      int32_t run = static_cast<int32_t>(at);
      for (int q = 0; q < TP_NW; ++q) {
        const int32_t x = cur[q * width + c];
        cur[q * width + c] = run;
        run += x;
      }
      if ((g << wlog) + c < k) tptr[(g << wlog) + c] = at;
    }
    base += tot;
  }
  if (threadIdx.x == 0 && ((g + 1) << wlog) >= k) tptr[k] = s1;
  __syncthreads();
  // the next round's entry is loaded while the current one is placed
  TpEntry next{0, 0};
  if (w0 + lane() < w1) next = in[w0 + lane()];
  for (int64_t x0 = w0; x0 < w1; x0 += WAVE) {
    const TpEntry en = next;
    const int64_t xn = x0 + WAVE + lane();
    if (xn < w1) next = in[xn];
    const bool ok = x0 + lane() < w1;
    const int32_t at = tp_place(ok, static_cast<uint32_t>(en.col) & (width - 1), wlog, mine);
    if (ok) tpos[at] = en.e;
  }
}

// Row of every position of the transposed pattern.
__global__ void k_tp_rows(const int32_t *arp, int64_t m, const int32_t *tpos, int64_t nnz,
                          int32_t *trow) {
  const int64_t d = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (d < nnz) trow[d] = row_of(arp, 0, static_cast<int32_t>(m), tpos[d]);
}

bool transpose_parts(int64_t k, int64_t nnz, TransposeParts &tp) {
  if (k <= 0 || nnz <= 0) return false;
  tp.wlog = 0;
  while (tp.wlog < TP_WIDTH_LOG && (int64_t(2) << tp.wlog) <= k * TP_GROUP_ENTRIES / nnz) ++tp.wlog;
  auto groups = [&] { return (k + (int64_t(1) << tp.wlog) - 1) >> tp.wlog; };
  while (tp.wlog < TP_WIDTH_LOG && groups() > TP_GROUPS) ++tp.wlog;
  if (groups() > TP_GROUPS) return false;  // beyond 2M columns
  tp.groups = groups();
  tp.tiles = (nnz + TP_TILE - 1) / TP_TILE;
  return true;
}

void launch_transpose_parts(const TransposeParts &tp, const int32_t *acol, int64_t k, int64_t nnz,
                            void *entries, int32_t *table, int64_t *off, int64_t *part,
                            int64_t *tptr, int32_t *tpos, hipStream_t s) {
  TpEntry *en = static_cast<TpEntry *>(entries);
  const int groups = static_cast<int>(tp.groups);
  hipLaunchKernelGGL(k_tp_count, dim3(tp.tiles), dim3(TP_NT), 0, s, acol, nnz, tp.wlog, groups,
                     table);
  scan_i32(table, tp.groups * tp.tiles, off, part, s);
  hipLaunchKernelGGL(k_tp_part, dim3(tp.tiles), dim3(TP_NT), 0, s, acol, nnz, tp.wlog, groups,
                     ceil_log2(groups), off, en);
  hipLaunchKernelGGL(k_tp_columns, dim3(tp.groups), dim3(TP_NT),
                     (sizeof(int32_t) * TP_NW) << tp.wlog, s, en, off, tp.tiles, k, tp.wlog, tptr,
                     tpos);
}

void launch_transpose_rows(const int32_t *arp, int64_t m, const int32_t *tpos, int64_t nnz,
                           int32_t *trow, hipStream_t s) {
  if (nnz > 0)
    hipLaunchKernelGGL(k_tp_rows, dim3((nnz + 255) / 256), dim3(256), 0, s, arp, m, tpos, nnz,
                       trow);
}

template <typename T>
void launch_grad_b(const int64_t *tptr, const int32_t *trow, const int32_t *tpos, const T *aval,
                   const int32_t *brp, const int32_t *bcol, int64_t kb, const int32_t *crp,
                   const int32_t *ccol, const T *dc, T *dB, hipStream_t s) {
  if (kb <= 0) return;
  hipLaunchKernelGGL((k_grad_b<T>), dim3((kb * WAVE + 255) / 256), dim3(256), 0, s, tptr, trow,
                     tpos, aval, brp, bcol, kb, crp, ccol, dc, dB);
}

template void launch_grad_b<float>(const int64_t *, const int32_t *, const int32_t *,
                                   const float *, const int32_t *, const int32_t *, int64_t,
                                   const int32_t *, const int32_t *, const float *, float *,
                                   hipStream_t);
template void launch_grad_b<double>(const int64_t *, const int32_t *, const int32_t *,
                                    const double *, const int32_t *, const int32_t *, int64_t,
                                    const int32_t *, const int32_t *, const double *, double *,
                                    hipStream_t);

}  // namespace spg
