// Stages 1-2 of the SpGEMM framework (Section 3.1): per-row upper bounds
// (Algorithm 2) through a device prefix scan, binning (Algorithm 3) as a
// per-work-group histogram, a scan and a scatter, and the hybrid sizes
// of the temporary matrix C~.  Also the reduce-then-scan primitive used by
// every stage.
#include <cstddef>

#include "common.hpp"
#include "internal.hpp"

namespace spg {

constexpr int SCAN_NT = 256;
constexpr int SCAN_IPT = 16;
constexpr int SCAN_TILE = SCAN_NT * SCAN_IPT;

int64_t scan_part_len(int64_t n) { return (n + SCAN_TILE - 1) / SCAN_TILE + 1; }

// brp[j] and brp[j + 1] in one load (4-byte alignment is enough).
struct __attribute__((packed, aligned(4))) RowBounds {
  int32_t begin, end;
};
// Length of b_{acol[e]*}.  Phase 1 of the scan gathers the row bounds, keeps
// where the row starts (bst) and leaves the length, 32 bits, inside the
// tile's own part of the output, where phase 3 (TileLenFn) reads it before
// it writes: gathering the bounds twice was L2-request bound (3.2M entries:
// 20 + 21 us; with the kept lengths 22 + 10).
DEVI int64_t scan_tile_base(int64_t e) { return e / SCAN_TILE * SCAN_TILE; }
// (KEEP false: a scan of one tile, which needs no lengths kept.)
template <bool KEEP> struct RowLenFn {
  const int32_t *acol;
  const int32_t *brp;
  int32_t *bst;
  int64_t *out;
  DEVI void keep(int64_t e, const RowBounds &r) const {
    bst[e] = r.begin;
    if (!KEEP) return;
    const int64_t base = scan_tile_base(e);
    reinterpret_cast<int32_t *>(out + base)[e - base] = r.end - r.begin;
  }
  DEVI int64_t operator()(int64_t e) const {
    const RowBounds r = *reinterpret_cast<const RowBounds *>(brp + acol[e]);
    keep(e, r);
    return static_cast<int64_t>(r.end) - r.begin;
  }
};
struct TileLenFn {
  const int64_t *out;
  DEVI int64_t operator()(int64_t e) const {
    const int64_t base = scan_tile_base(e);
    return reinterpret_cast<const int32_t *>(out + base)[e - base];
  }
};
struct I64Fn {
  const int64_t *v;
  DEVI int64_t operator()(int64_t e) const { return v[e]; }
};
struct I32Fn {
  const int32_t *v;
  DEVI int64_t operator()(int64_t e) const { return v[e]; }
};
struct PieceFn {
  const Piece *p;
  DEVI int64_t operator()(int64_t e) const { return p[e].cnt; }
};

// Elements base + j * SCAN_NT + t of a tile.  A whole tile's loads carry no
// bounds checks, so that they are in flight together (a checked load is
// waited for before the next is issued: 29 against 12 us for the two
// dependent loads of 3.2M row lengths); the last tile checks.
template <typename F>
DEVI void scan_tile_load(const F &f, int64_t n, int64_t base, int64_t (&v)[SCAN_IPT]) {
  if (base + SCAN_TILE <= n) {
#pragma unroll
    for (int j = 0; j < SCAN_IPT; ++j) v[j] = f(base + j * SCAN_NT + threadIdx.x);
  } else {
#pragma unroll
    for (int j = 0; j < SCAN_IPT; ++j) {
      const int64_t e = base + j * SCAN_NT + threadIdx.x;
      v[j] = e < n ? f(e) : 0;
    }
  }
}

// Row lengths of a whole tile: all columns, then all row bounds, then the
// stores (which the compiler may not move loads across).
template <bool KEEP>
DEVI void scan_tile_load(const RowLenFn<KEEP> &f, int64_t n, int64_t base,
                         int64_t (&v)[SCAN_IPT]) {
  if (base + SCAN_TILE <= n) {
    int32_t c[SCAN_IPT];
    RowBounds r[SCAN_IPT];
#pragma unroll
    for (int j = 0; j < SCAN_IPT; ++j) c[j] = f.acol[base + j * SCAN_NT + threadIdx.x];
#pragma unroll
    for (int j = 0; j < SCAN_IPT; ++j) r[j] = *reinterpret_cast<const RowBounds *>(f.brp + c[j]);
#pragma unroll
    for (int j = 0; j < SCAN_IPT; ++j) {
      f.keep(base + j * SCAN_NT + threadIdx.x, r[j]);
      v[j] = static_cast<int64_t>(r[j].end) - r[j].begin;
    }
  } else {
#pragma unroll
    for (int j = 0; j < SCAN_IPT; ++j) {
      const int64_t e = base + j * SCAN_NT + threadIdx.x;
      v[j] = e < n ? f(e) : 0;
    }
  }
}

// Phase 1: sum of every tile.
template <typename F>
__global__ __launch_bounds__(SCAN_NT) void k_scan_reduce(F f, int64_t n, int64_t *part) {
  __shared__ int64_t sm[SCAN_NT / WAVE + 1];
  const int64_t base = static_cast<int64_t>(blockIdx.x) * SCAN_TILE;
  int64_t v[SCAN_IPT];
  scan_tile_load(f, n, base, v);
  int64_t s = 0;
#pragma unroll
  for (int j = 0; j < SCAN_IPT; ++j) s += v[j];
  int64_t tot;
  block_excl_sum<SCAN_NT>(s, sm, tot);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// Phase 2: exclusive scan of the tile sums by one work-group; part[nb] gets
// the grand total.
__global__ __launch_bounds__(SCAN_NT) void k_scan_part(int64_t *part, int64_t nb) {
  __shared__ int64_t sm[SCAN_NT / WAVE + 1];
  int64_t carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += SCAN_NT) {
    const int64_t b = b0 + threadIdx.x;
    int64_t v = b < nb ? part[b] : 0;
    int64_t tot;
    int64_t ex = block_excl_sum<SCAN_NT>(v, sm, tot);
    if (b < nb) part[b] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) part[nb] = carry;
}

// Phase 3: rescan every tile from its offset.  Loads and stores are
// coalesced (consecutive threads, consecutive elements); the tile goes
// through LDS so that thread t can scan its IPT consecutive elements
// t*IPT .. t*IPT+IPT-1 (one pad word per IPT elements keeps that access
// spread over the banks).
DEVI int scan_lds_ix(int i) { return i + i / SCAN_IPT; }

// SELF: `part` holds the raw tile sums and every work-group adds up those
// of the tiles before it (fine for a few thousand tiles; saves the launch of
// phase 2); otherwise `part` is phase 2's exclusive scan.
struct NoEnd {
  DEVI void operator()(int64_t) const {}
};
template <typename F, bool SELF, typename End>
__global__ __launch_bounds__(SCAN_NT) void k_scan_down(F f, int64_t n, const int64_t *part,
                                                       int64_t nb, int64_t *out, End end) {
  __shared__ int64_t sm[SCAN_NT / WAVE + 1];
  __shared__ int64_t tile[SCAN_TILE + SCAN_TILE / SCAN_IPT];
  const int t = threadIdx.x;
  const int64_t base = static_cast<int64_t>(blockIdx.x) * SCAN_TILE;
  int64_t offset = 0;
  if constexpr (SELF) {
    int64_t ps = 0;
    for (int64_t b = t; b < static_cast<int64_t>(blockIdx.x); b += SCAN_NT) ps += part[b];
    block_excl_sum<SCAN_NT>(ps, sm, offset);
  } else {
    offset = part[blockIdx.x];
  }
  int64_t v[SCAN_IPT];
  scan_tile_load(f, n, base, v);
#pragma unroll
  for (int j = 0; j < SCAN_IPT; ++j) tile[scan_lds_ix(j * SCAN_NT + t)] = v[j];
  __syncthreads();
  int64_t s = 0;
#pragma unroll
  for (int j = 0; j < SCAN_IPT; ++j) {
    v[j] = tile[scan_lds_ix(t * SCAN_IPT + j)];
    s += v[j];
  }
  int64_t tot;
  int64_t ex = block_excl_sum<SCAN_NT>(s, sm, tot) + offset;
#pragma unroll
  for (int j = 0; j < SCAN_IPT; ++j) {
    tile[scan_lds_ix(t * SCAN_IPT + j)] = ex;  // the slots this thread read
    ex += v[j];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < SCAN_IPT; ++j) {
    const int i = j * SCAN_NT + t;
    const int64_t e = base + i;
    if (e < n) out[e] = tile[scan_lds_ix(i)];
  }
  // `end` gets the total from one thread
  if constexpr (SELF) {
    if (blockIdx.x == nb - 1 && t == 0) {
      out[n] = offset + tot;
      end(offset + tot);
    }
  } else {
    if (blockIdx.x == 0 && t == 0) {
      out[n] = part[nb];
      end(part[nb]);
    }
  }
}

// tiles up to which a work-group of phase 3 sums the earlier tile sums itself
constexpr int64_t SCAN_SELF_MAX_TILES = 4096;

// Scans f; phase 1 sums `f`, phase 3 reads `down`, and a scan of one tile is
// one launch over `one` (no earlier tiles to sum).
template <typename F, typename G, typename H, typename End>
static void scan_with(F f, G down, H one, End end, int64_t n, int64_t *out, int64_t *part,
                      hipStream_t s) {
  const int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
  if (nb <= 1) {
    hipLaunchKernelGGL((k_scan_down<H, true, End>), dim3(1), dim3(SCAN_NT), 0, s, one, n, part,
                       int64_t(1), out, end);
    return;
  }
  hipLaunchKernelGGL((k_scan_reduce<F>), dim3(nb), dim3(SCAN_NT), 0, s, f, n, part);
  if (nb <= SCAN_SELF_MAX_TILES) {
    hipLaunchKernelGGL((k_scan_down<G, true, End>), dim3(nb), dim3(SCAN_NT), 0, s, down, n, part,
                       nb, out, end);
    return;
  }
  hipLaunchKernelGGL(k_scan_part, dim3(1), dim3(SCAN_NT), 0, s, part, nb);
  hipLaunchKernelGGL((k_scan_down<G, false, End>), dim3(nb), dim3(SCAN_NT), 0, s, down, n, part,
                     nb, out, end);
}
template <typename F>
static void scan_plain(F f, int64_t n, int64_t *out, int64_t *part, hipStream_t s) {
  scan_with(f, f, f, NoEnd{}, n, out, part, s);
}

void scan_row_lengths(const int32_t *acol, const int32_t *brp, int64_t n, int64_t *out,
                      int32_t *bst, int64_t *part, hipStream_t s) {
  scan_with(RowLenFn<true>{acol, brp, bst, out}, TileLenFn{out},
            RowLenFn<false>{acol, brp, bst, out}, NoEnd{}, n, out, part, s);
}
void scan_i64(const int64_t *v, int64_t n, int64_t *out, int64_t *part, hipStream_t s) {
  scan_plain(I64Fn{v}, n, out, part, s);
}
void scan_i32(const int32_t *v, int64_t n, int64_t *out, int64_t *part, hipStream_t s) {
  scan_plain(I32Fn{v}, n, out, part, s);
}
void scan_piece_counts(const Piece *pieces, int64_t n, int64_t *out, int64_t *part,
                       hipStream_t s) {
  scan_plain(PieceFn{pieces}, n, out, part, s);
}

// ------------------------------------------------------------ validation

// One thread per row: row_ptr monotone and bounded, columns in range and
// strictly increasing.  Any violation sets sum->err.
__global__ void k_validate(const int32_t *rp, const int32_t *ci, int64_t rows, int64_t cols,
                           int64_t nnz, Summary *sum) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i > rows) return;
  bool bad = false;
  if (i == 0 && rp[0] != 0) bad = true;
  if (i == rows && rp[rows] != nnz) bad = true;
  if (i < rows) {
    const int32_t a = rp[i], b = rp[i + 1];
    if (b < a || a < 0 || b > nnz) {
      bad = true;
    } else {
      int64_t prev = -1;
      for (int32_t p = a; p < b; ++p) {
        const int32_t c = ci[p];
        if (c < 0 || c >= cols || c <= prev) {
          bad = true;
          break;
        }
        prev = c;
      }
    }
  }
  if (bad) atomicOr(&sum->err, 1);
}

void launch_validate(const int32_t *rp, const int32_t *ci, int64_t rows, int64_t cols,
                     int64_t nnz, Summary *sum, hipStream_t s) {
  const int64_t nb = (rows + 1 + 255) / 256;
  hipLaunchKernelGGL(k_validate, dim3(nb), dim3(256), 0, s, rp, ci, rows, cols, nnz, sum);
}

// --------------------------------------------------------------- binning

// A work-group takes RPT * 256 consecutive rows.  The bin histogram of every
// work-group (k_row_stats), one exclusive scan per bin over the work-groups
// (k_bin_scan) and a scatter (k_bin_scatter) give every bin its rows, in
// work-group order; inside a work-group the order of a bin's rows is that of
// the LDS counter and has no meaning.  Small products do all of it in one
// work-group and one launch (k_rows_small): their launches cost more than
// the work (four launches of about 4 us each and the gaps between them for
// 2000 rows, against one of 8).
constexpr int BIN_NT = 256;

// What row i, with ne entries of A from e0, adds to the long-row planning sums
// (v: see kBlockStats).
DEVI void long_sums(int64_t i, int64_t ui, int bin, int32_t e0, int32_t ne, const RowStatsArgs &a,
                    int64_t (&v)[kBlockStats]) {
  v[0] = v[0] > ui ? v[0] : ui;
  if (bin != LONG_BIN) return;
  const int64_t rmax = ui < a.ncols ? ui : a.ncols;
  int64_t segp;
  int32_t nseg, shift, npiece;
  long_row_plan(ui, a.ncols, a.lp, segp, nseg, shift, npiece);
  v[1] += ui;
  v[2] += rmax;
  v[3] += nseg;
  v[4] += npiece;
  if (nseg > 1) {
    v[5] += ui;
    v[6] += static_cast<int64_t>(nseg) * (npiece + 1);
    v[8] += rmax;
  } else if (ui <= kOneShot) {
    v[5] += rmax;  // one-tile row: its result has a place of its own
  } else if (rmax > a.long_slot) {
    int64_t cap = a.long_slot;
    while (cap < rmax) cap *= 2;
    v[7] += cap;
  }
  const int64_t segr = segp < a.ncols ? segp : a.ncols;
  if (segr > a.l1cap - kLongTile) v[9] += segr * nseg;
  const WinPlan wp = win_plan(ui, a.ncols, a.vbytes);
  v[10] += wp.nitem;
  v[11] += wp.nseg;
  v[12] += wp.table;
  v[13] += wp.partial;
  v[14] += wp.dslots;
  v[15] += wp.mode == WIN_NONE ? 1 : 0;
  // the lengths of four of its rows of B: of every sixteenth long row, spread by
  // its index, and of the longest (of all: 23.8 us for 300000 rows, now 22.5)
  if (wp.mode == WIN_DD &&
      (ne >= 1024 || (static_cast<uint32_t>(i) * 0x9e3779b1u) >> 28 == 0)) {
    int wide = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t e = e0 + (static_cast<int64_t>(ne) * (2 * k + 1) >> 3);
      wide += a.P[e + 1] - a.P[e] > 32 ? 1 : 0;
    }
    v[16] += ne;
    v[17] += static_cast<int64_t>(ne) * wide;
  }
}

// Whether every long row is a direct dense row (win_plan).
DEVI bool narrow_b(const RowStatsArgs &a) {
  return a.ncols <= (int64_t(1) << win_dense_log(a.vbytes));
}

// Work-group totals of the planning sums; the result of sum k is returned to
// thread k (< kBlockStats), others get 0.  Only the maximum is reduced where
// no thread has a long row, and the sums for dense windows only where B is
// narrow.  Contains barriers.
template <int NT> DEVI int64_t block_stats(const int64_t (&v)[kBlockStats], bool any_long,
                                           bool narrow,
                                           int64_t (&red)[NT / WAVE][kBlockStats]) {
  const int w = threadIdx.x / WAVE;
  const bool wl = __any(any_long);
#pragma unroll
  for (int k = 0; k < kBlockStats; ++k) {
    if ((k > 0 && !wl) || (k >= kNarrowStats && !narrow)) {
      if (lane() == 0) red[w][k] = 0;
      continue;
    }
    int64_t x = v[k];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const int64_t y = __shfl_xor(x, o, WAVE);
      x = k == 0 ? (x > y ? x : y) : x + y;
    }
    if (lane() == 0) red[w][k] = x;
  }
  __syncthreads();
  int64_t x = 0;
  if (threadIdx.x < kBlockStats) {
    const int k = threadIdx.x;
    for (int q = 0; q < NT / WAVE; ++q)
      x = k == 0 ? (x > red[q][k] ? x : red[q][k]) : x + red[q][k];
  }
  return x;
}

// The summary's words from the work-group's totals: bin_off[0..NBINS],
// stats[0..], sum_u and sum_h; to the host's slot if there is one, else to
// `sum`.  One wavefront writes it, so that its token follows its words.
DEVI void write_summary(const int64_t *bin_off, const int64_t *stats, int64_t sum_u, int64_t sum_h,
                        Summary *sum, HostSlot *slot, uint64_t token) {
  constexpr int N = sizeof(Summary) / 8;
  static_assert(sizeof(Summary) % 8 == 0 && N <= HostSlot::kWords && N <= WAVE,
                "the summary must fit a slot");
  static_assert(offsetof(Summary, sum_u) == 0 && offsetof(Summary, sum_h) == 8 &&
                    offsetof(Summary, max_u) == 16 && offsetof(Summary, bin_off) == 24 &&
                    offsetof(Summary, sum_u_long) == 24 + 8 * (NBINS + 1) &&
                    offsetof(Summary, err) == 24 + 8 * (NBINS + 1) + 8 * (kBlockStats - 1),
                "word order");
  const int k = threadIdx.x;
  if (k >= WAVE) return;
  int64_t x = 0;  // the last word: no error
  if (k == 0) x = sum_u;
  else if (k == 1) x = sum_h;
  else if (k == 2) x = stats[0];
  else if (k < 3 + NBINS + 1) x = bin_off[k - 3];
  else if (k < 3 + NBINS + 1 + kBlockStats - 1) x = stats[k - (3 + NBINS + 1) + 1];
  if (!slot) {
    if (k < N) reinterpret_cast<int64_t *>(sum)[k] = x;
    return;
  }
  if (k < N)
    __hip_atomic_store(&slot->word[k], static_cast<uint64_t>(x), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
  __threadfence_system();
  if (k == 0)
    __hip_atomic_store(&slot->token, token, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

DEVI int64_t tilde_size(int64_t ui, int bin, const RowStatsArgs &a) {
  return bin == LONG_BIN ? static_cast<int64_t>(a.long_slot) : ui;
}

// Exclusive prefix of the bin totals cnt[0..NBINS) by the first wavefront
// into off[0..NBINS]; the caller synchronizes.
DEVI void bin_offsets(const int64_t *cnt, int64_t *off) {
  if (threadIdx.x >= WAVE) return;
  const int64_t c = lane() < NBINS ? cnt[lane()] : 0;
  const int64_t inc = group_incl_sum<WAVE>(c);
  if (lane() < NBINS) off[lane()] = inc - c;
  if (lane() == NBINS - 1) off[NBINS] = inc;
}

// Stage 1 result per row, and per work-group its bin histogram, its part of
// nnz(C~) and the planning sums (all laid out by kind, then work-group).
template <int RPT>
__global__ __launch_bounds__(BIN_NT) void k_row_stats(RowStatsArgs a) {
  __shared__ int32_t cnt[NBINS];
  __shared__ int64_t red[BIN_NT / WAVE][kBlockStats];
  __shared__ int64_t sm[BIN_NT / WAVE + 1];
  const int t = threadIdx.x;
  if (t < NBINS) cnt[t] = 0;
  __syncthreads();
  int64_t v[kBlockStats] = {};
  int64_t h = 0;
  bool any_long = false;
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    const int64_t i = (static_cast<int64_t>(blockIdx.x) * RPT + r) * BIN_NT + t;
    if (i >= a.m) continue;
    const int32_t e0 = a.arp[i], e1 = a.arp[i + 1];
    const int64_t ui = a.P[e1] - a.P[e0];
    const int bin = bin_of(ui, a.be);
    a.u[i] = ui;
    if (ui == 0) a.rownnz[i] = 0;
    h += tilde_size(ui, bin, a);
    any_long |= bin == LONG_BIN;
    atomicAdd(&cnt[bin], 1);
    long_sums(i, ui, bin, e0, e1 - e0, a, v);
  }
  int64_t hs;
  block_excl_sum<BIN_NT>(h, sm, hs);
  const int64_t st = block_stats<BIN_NT>(v, any_long, narrow_b(a), red);  // (its barrier orders cnt too)
  const int64_t nb = gridDim.x, b = blockIdx.x;
  if (t < NBINS) a.hist[t * nb + b] = cnt[t];
  if (t == 0) a.hpart[b] = hs;
  if (t < kBlockStats) a.bpart[t * nb + b] = st;
}

// One work-group per bin (exclusive scan of its counts over the row
// work-groups, total to tot[bin]), one for nnz(C~), one per planning sum.
__global__ __launch_bounds__(BIN_NT) void k_bin_scan(int32_t *hist, int64_t *hpart,
                                                     const int64_t *bpart, int64_t nb,
                                                     int64_t *tot) {
  __shared__ int64_t sm[BIN_NT / WAVE + 1];
  const int c = blockIdx.x;
  const int t = threadIdx.x;
  int64_t carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += BIN_NT) {
    const int64_t b = b0 + t;
    int64_t x = 0, all;
    if (c < NBINS)
      x = b < nb ? hist[c * nb + b] : 0;
    else if (c == NBINS)
      x = b < nb ? hpart[b] : 0;
    else
      x = b < nb ? bpart[(c - NBINS - 1) * nb + b] : 0;
    if (c == NBINS + 1) {  // the largest u
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const int64_t y = __shfl_xor(x, o, WAVE);
        x = x > y ? x : y;
      }
      if (lane() == 0) sm[t / WAVE] = x;
      __syncthreads();
      for (int w = 0; w < BIN_NT / WAVE; ++w) carry = carry > sm[w] ? carry : sm[w];
      __syncthreads();
      continue;
    }
    const int64_t ex = carry + block_excl_sum<BIN_NT>(x, sm, all);
    if (c < NBINS) {
      if (b < nb) hist[c * nb + b] = static_cast<int32_t>(ex);
    } else if (c == NBINS) {
      if (b < nb) hpart[b] = ex;
    }
    carry += all;
  }
  if (t == 0) tot[c] = carry;
}

// Rows into their bins, C~ offsets; the first work-group writes the summary
// (unless k_summary does).
template <int RPT>
__global__ __launch_bounds__(BIN_NT) void k_bin_scatter(RowStatsArgs a) {
  __shared__ int64_t off[NBINS + 1];
  __shared__ int32_t cnt[NBINS];
  __shared__ int64_t sm[BIN_NT / WAVE + 1];
  const int t = threadIdx.x;
  const int64_t nb = gridDim.x, b = blockIdx.x;
  bin_offsets(a.tot, off);
  if (t < NBINS) cnt[t] = a.hist[t * nb + b];
  int64_t ho = a.hpart[b];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    const int64_t i = (b * RPT + r) * BIN_NT + t;
    const bool valid = i < a.m;
    const int64_t ui = valid ? a.u[i] : 0;
    const int bin = bin_of(ui, a.be);
    int64_t all;
    const int64_t ex = block_excl_sum<BIN_NT>(valid ? tilde_size(ui, bin, a) : 0, sm, all);
    if (valid) {
      a.cto[i] = ho + ex;
      const int32_t e0 = a.arp[i];
      const RowRec rec{static_cast<int32_t>(i),
                       static_cast<int32_t>(ui < INT32_MAX ? ui : INT32_MAX), e0,
                       a.arp[i + 1] - e0};
      const int64_t pos = off[bin] + atomicAdd(&cnt[bin], 1);
      a.binlist[pos] = rec.row;
      a.recs[pos] = rec;
    }
    ho += all;
  }
  if (b == 0) {
    const int64_t sum_h = a.tot[NBINS];
    if (t == 0) a.cto[a.m] = sum_h;
    if (!a.whole)
      write_summary(off, a.tot + NBINS + 1, a.P[a.nnz], sum_h, a.sum, a.slot, a.token);
  }
}

// The summary once every work-group of k_bin_scatter is done.
__global__ __launch_bounds__(WAVE) void k_summary(RowStatsArgs a) {
  __shared__ int64_t off[NBINS + 1];
  bin_offsets(a.tot, off);
  __syncthreads();
  write_summary(off, a.tot + NBINS + 1, a.P[a.nnz], a.tot[NBINS], a.sum, a.slot, a.token);
}

// Everything after stage 1's scan for up to ROWS_SMALL rows.
constexpr int SMALL_NT = 1024;
constexpr int SMALL_RPT = 4;
constexpr int64_t ROWS_SMALL = SMALL_NT * SMALL_RPT;

__global__ __launch_bounds__(SMALL_NT) void k_rows_small(RowStatsArgs a) {
  __shared__ int64_t off[NBINS + 1], tot[NBINS], stats[kBlockStats];
  __shared__ int32_t cnt[NBINS], cur[NBINS];
  __shared__ int64_t red[SMALL_NT / WAVE][kBlockStats];
  __shared__ int64_t sm[SMALL_NT / WAVE + 1];
  const int t = threadIdx.x;
  if (t < NBINS) cnt[t] = cur[t] = 0;
  __syncthreads();
  int64_t v[kBlockStats] = {};
  bool any_long = false;
  int32_t e0[SMALL_RPT], ne[SMALL_RPT];
  int64_t u[SMALL_RPT];
  int bin[SMALL_RPT];
#pragma unroll
  for (int r = 0; r < SMALL_RPT; ++r) {
    const int64_t i = r * SMALL_NT + t;
    u[r] = 0;
    bin[r] = -1;
    if (i >= a.m) continue;
    e0[r] = a.arp[i];
    ne[r] = a.arp[i + 1] - e0[r];
    u[r] = a.P[e0[r] + ne[r]] - a.P[e0[r]];
    bin[r] = bin_of(u[r], a.be);
    a.u[i] = u[r];
    if (u[r] == 0) a.rownnz[i] = 0;
    any_long |= bin[r] == LONG_BIN;
    atomicAdd(&cnt[bin[r]], 1);
    long_sums(i, u[r], bin[r], e0[r], ne[r], a, v);
  }
  const int64_t st = block_stats<SMALL_NT>(v, any_long, narrow_b(a), red);  // (its barrier orders cnt too)
  if (t < kBlockStats) stats[t] = st;
  if (t < NBINS) tot[t] = cnt[t];
  __syncthreads();
  bin_offsets(tot, off);
  __syncthreads();
  int64_t ho = 0;
#pragma unroll
  for (int r = 0; r < SMALL_RPT; ++r) {
    const int64_t i = r * SMALL_NT + t;
    int64_t all;
    if (r * SMALL_NT >= a.m) break;  // uniform
    const int64_t ex =
        block_excl_sum<SMALL_NT>(bin[r] >= 0 ? tilde_size(u[r], bin[r], a) : 0, sm, all);
    if (bin[r] >= 0) {
      a.cto[i] = ho + ex;
      const RowRec rec{static_cast<int32_t>(i),
                       static_cast<int32_t>(u[r] < INT32_MAX ? u[r] : INT32_MAX), e0[r], ne[r]};
      const int64_t pos = off[bin[r]] + atomicAdd(&cur[bin[r]], 1);
      a.binlist[pos] = rec.row;
      a.recs[pos] = rec;
    }
    ho += all;
  }
  if (t == 0) a.cto[a.m] = ho;
  if (a.whole) {
    __threadfence();
    __syncthreads();
  }
  write_summary(off, stats, a.P[a.nnz], ho, a.sum, a.slot, a.token);
}

// rows per thread of the binning kernels: enough that a bin's scan over the
// work-groups stays short (1024 of them at 262144 rows; four rows per thread
// beyond)
int64_t bin_blocks(int64_t m) {
  const int rpt = m > 262144 ? 4 : 1;
  const int64_t nb = (m + BIN_NT * rpt - 1) / (BIN_NT * rpt);
  return nb > 0 ? nb : 1;
}

void launch_binning(const RowStatsArgs &a, hipStream_t s) {
  if (a.m <= ROWS_SMALL) {
    hipLaunchKernelGGL(k_rows_small, dim3(1), dim3(SMALL_NT), 0, s, a);
    return;
  }
  const int64_t nb = bin_blocks(a.m);
  if (a.m > 262144)
    hipLaunchKernelGGL(k_row_stats<4>, dim3(nb), dim3(BIN_NT), 0, s, a);
  else
    hipLaunchKernelGGL(k_row_stats<1>, dim3(nb), dim3(BIN_NT), 0, s, a);
  hipLaunchKernelGGL(k_bin_scan, dim3(NBINS + 1 + kBlockStats), dim3(BIN_NT), 0, s, a.hist,
                     a.hpart, a.bpart, nb, a.tot);
  if (a.m > 262144)
    hipLaunchKernelGGL(k_bin_scatter<4>, dim3(nb), dim3(BIN_NT), 0, s, a);
  else
    hipLaunchKernelGGL(k_bin_scatter<1>, dim3(nb), dim3(BIN_NT), 0, s, a);
  if (a.whole) hipLaunchKernelGGL(k_summary, dim3(1), dim3(WAVE), 0, s, a);
}

__global__ void k_zero(uint32_t *p, int64_t n) {
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    p[i] = 0u;
}

void launch_zero(void *p, size_t bytes, hipStream_t s) {
  const int64_t n = static_cast<int64_t>((bytes + 3) / 4);
  if (n <= 0) return;
  int64_t nb = (n + 255) / 256;
  if (nb > 4096) nb = 4096;
  hipLaunchKernelGGL(k_zero, dim3(nb), dim3(256), 0, s, static_cast<uint32_t *>(p), n);
}

__global__ void k_set_pool(Pool *dst, Pool value) { *dst = value; }

void launch_set_pool(Pool *dst, Pool value, hipStream_t s) {
  hipLaunchKernelGGL(k_set_pool, dim3(1), dim3(1), 0, s, dst, value);
}

// The status of compute, by one thread: to the host's slot if there is one
// (the words, then the token that announces them), else to `st`.
struct StatusEnd {
  const Pool *pool;          // nullptr: no merge method
  const LongCounters *cnt;
  ComputeStatus *st;
  HostSlot *slot;
  uint64_t token;
  DEVI void operator()(int64_t nnz) const {
    ComputeStatus v;
    v.nnz_c = nnz;
    v.fail_count = pool ? pool->fail_count : 0u;
    v.fail2 = pool ? pool->fail2 : 0u;
    v.pool_used = pool ? pool->used : 0ull;
    v.left = cnt ? cnt->l3 : 0u;
    v.pad = 0u;
    if (!slot) {
      *st = v;
      return;
    }
    constexpr int N = sizeof(ComputeStatus) / 8;
    uint64_t w[N];
    __builtin_memcpy(w, &v, sizeof(v));
#pragma unroll
    for (int k = 0; k < N; ++k)
      __hip_atomic_store(&slot->word[k], w[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&slot->token, token, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
};

// Words to pinned host memory, then the token that announces them (one
// work-group).
__global__ __launch_bounds__(256) void k_publish(const uint64_t *src, int64_t words, uint64_t *dst,
                                                 uint64_t *at, uint64_t token) {
  for (int64_t k = threadIdx.x; k < words; k += 256)
    __hip_atomic_store(&dst[k], src[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_store(at, token, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

void launch_publish(const uint64_t *src, int64_t words, uint64_t *dst, uint64_t *at,
                    uint64_t token, hipStream_t s) {
  hipLaunchKernelGGL(k_publish, dim3(1), dim3(256), 0, s, src, words, dst, at, token);
}

__global__ void k_status(const int64_t *rowoff, int64_t m, StatusEnd end) { end(rowoff[m]); }

void launch_status(const int64_t *rowoff, int64_t m, const Pool *pool, const LongCounters *cnt,
                   ComputeStatus *st, HostSlot *slot, uint64_t token, hipStream_t s) {
  hipLaunchKernelGGL(k_status, dim3(1), dim3(1), 0, s, rowoff, m,
                     StatusEnd{pool, cnt, st, slot, token});
}

void scan_rows_status(const int64_t *v, int64_t n, int64_t *out, int64_t *part, const Pool *pool,
                      const LongCounters *cnt, ComputeStatus *st, HostSlot *slot, uint64_t token,
                      hipStream_t s) {
  const I64Fn f{v};
  scan_with(f, f, f, StatusEnd{pool, cnt, st, slot, token}, n, out, part, s);
}

}  // namespace spg
