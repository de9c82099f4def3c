// Index reordering for the TT embedding bag (paper Sections III-C, III-E, III-G).
//
// The paper elects one thread per (i1,i2) prefix with an atomic compare-and-swap
// on a flag array and hands out reuse-buffer slots with an atomic counter.  Here
// the same information -- which prefix products and which rows are distinct --
// comes from a stable LSD radix sort of the lookups by row followed by a
// head-flag scan, so slots are the ranks in sorted order (deterministic), no
// flag array of size N/n3 is needed, and equal rows / prefixes are contiguous
// for the segmented reductions of the backward pass.
//
// All counts stay on the device: later kernels read U_r / U_p from plan->counts.
#include "tt_internal.h"

namespace {

// ------------------------------------------------------------------ key extraction
// Errors only the device can see.  They are reported with atomics on the plan's status word, so
// they are checked in the SECOND kernel of the plan (the first one initialises that word).
__device__ __forceinline__ void check_offsets(const TTDev &d, int l) {
  const int64_t *__restrict__ offsets = d.offsets;
  const int num_bags = d.num_bags;
  if (l > num_bags) return;
  bool bad;
  if (l < num_bags) bad = offsets[l] > offsets[l + 1] || offsets[l] < 0;
  else bad = offsets[num_bags] != (long long)d.nnz || offsets[0] != 0;
  if (bad) atomicOr(&d.plan.counts[4], 2);
}

// A table without lookups, alone or in a batch: no tile of it checks the offsets or writes the groupings,
// which are empty (every range of every segment array is [0, 0)).
template <bool BATCHED>
__global__ void k_empty_plan(TTArg<BATCHED> a) {
  const TTDev &d = a.get();
  if (d.nnz != 0) return;  // uniform
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  check_offsets(d, u);
  if (u <= d.sh.n3) d.plan.i3_seg[u] = 0;
  if (u <= d.sh.n2) d.plan.i2_seg[u] = 0;
  if (u <= d.sh.n1) d.plan.i1_seg[u] = 0;
}

// ------------------------------------------------------------------ LSD radix pass
#define TT_SORT_MAX_PASSES 4  // 31 key bits in digits of at most 10 bits
// The three sorts of a plan: 0 = lookups by row, 1 = distinct rows by i3, 2 = distinct prefixes
// by i2.  (a) buffers hold the final result, (b) buffers are their ping-pong partners.
struct SortBufs {
  int32_t *ka, *va, *kb, *vb;
  const int32_t *count_ptr;  // nullptr: `count` holds the number of keys
  int ntiles, count;
  __device__ __forceinline__ int keys() const { return count_ptr ? *count_ptr : count; }
};
// `which` has to be a plain kernel argument: a variant that took it from the workgroup index (two
// sorts in one launch) was compiled to code that left one pointer of sort 2 at sort 1's value.
__device__ __forceinline__ SortBufs sort_bufs(const TTDev &d, int which) {
  SortBufs b;
  if (which == 0) {
    b.ka = d.plan.sorted_row; b.va = d.plan.perm; b.kb = d.tmp.keys_alt; b.vb = d.tmp.vals_alt;
    b.count_ptr = nullptr; b.count = d.nnz; b.ntiles = d.sort_tiles;
  } else if (which == 1) {
    b.ka = d.plan.i3_of_sorted; b.va = d.plan.rows_by_i3; b.kb = d.tmp.k3_alt; b.vb = d.tmp.v3_alt;
    b.count_ptr = d.plan.counts + 0; b.count = 0;
    b.ntiles = (int)((d.plan.max_rows + TT_SORT_TILE - 1) / TT_SORT_TILE);
  } else {
    b.ka = d.tmp.k2; b.va = d.plan.prefs_by_i2; b.kb = d.tmp.k2_alt; b.vb = d.tmp.v2_alt;
    b.count_ptr = d.plan.counts + 1; b.count = 0;
    b.ntiles = (int)((d.plan.max_prefixes + TT_SORT_TILE - 1) / TT_SORT_TILE);
  }
  return b;
}

// ---- building blocks of the stable counting sorts, for workgroups of NT threads ----------------
// Lanes of the wavefront whose digit (below 2^bits) equals this lane's; invalid lanes match nothing.
// Written without branches per bit: the mask of a bit, or its complement, by an exclusive or.
__device__ __forceinline__ unsigned long long wave_match(int digit, int bits, bool valid) {
  const unsigned long long all = __ballot(valid);
  unsigned lo = (unsigned)all, hi = (unsigned)(all >> 32);
#pragma unroll
  for (int b = 0; b < TT_SORT_MAX_BITS; ++b) {
    if (b >= bits) break;  // uniform
    const unsigned inv = ((unsigned)(digit >> b) & 1u) - 1u;  // 0 where the bit is set, all ones where not
    const unsigned long long m = __ballot((digit >> b) & 1);
    lo &= (unsigned)m ^ inv;
    hi &= (unsigned)(m >> 32) ^ inv;
  }
  return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ unsigned long long lanes_below() {
  const int lane = threadIdx.x & (TT_WAVE - 1);
  return lane == 0 ? 0ull : (~0ull >> (TT_WAVE - lane));
}

// LDS of one tile's ranking.  Wavefront w of a workgroup owns the tile's keys [w*64*ITEMS, ...) and
// ranks them in rounds of 64 (position order), keeping running counts per digit in its own row of
// wave_cnt.  Equal digits keep their order: tiles in order, wavefronts in order, rounds in order,
// lanes in order.
template <int NT>
struct RankLds {
  int wave_cnt[NT / TT_WAVE][1 << TT_SORT_MAX_BITS];
  int gofs[1 << TT_SORT_MAX_BITS];  // output position of the first key of (digit, this tile)
  int tmp[NT / TT_WAVE + 1];
};
// rank[i] = keys with the same digit before key i in its wavefront's range.  The first lane of a group
// of equal digits advances the count with an atomic addition that returns the old value: the wavefront's
// LDS operations execute in order, so the rounds follow each other without waiting for the values,
// which are handed to the group's other lanes at the end.
template <int NT, int ITEMS>
__device__ __forceinline__ void rank_rounds(RankLds<NT> &L, const int (&digit)[ITEMS], const bool (&valid)[ITEMS], int bits,
                                            int (&rank)[ITEMS]) {
  const int lane = threadIdx.x & (TT_WAVE - 1);
  int *row = L.wave_cnt[threadIdx.x / TT_WAVE];  // this wavefront's own row
  for (int b = lane; b < (1 << bits); b += TT_WAVE) row[b] = 0;
  tt_wave_lds_order();
  int leader[ITEMS], old[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const unsigned long long mask = wave_match(digit[i], bits, valid[i]);
    leader[i] = valid[i] ? __ffsll(mask) - 1 : lane;
    rank[i] = __popcll(mask & lanes_below());
    old[i] = 0;
    if (valid[i] && lane == leader[i]) old[i] = atomicAdd(&row[digit[i]], __popcll(mask));
  }
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) rank[i] += __shfl(old[i], leader[i]);
}
// After the rounds (and a barrier): counts per wavefront -> their bases inside the tile's run of a
// digit.  Returns the tile's count of digit `bin`.
template <int NT>
__device__ __forceinline__ int rank_bases(RankLds<NT> &L, int bin) {
  int run = 0;
#pragma unroll
  for (int w = 0; w < NT / TT_WAVE; ++w) {
    const int c = L.wave_cnt[w][bin];
    L.wave_cnt[w][bin] = run;
    run += c;
  }
  return run;
}

// Turns the ranking's counts into output positions: gofs = digits below (exclusive scan of tot) + earlier
// tiles (pre), wave_cnt = the wavefronts' bases.  seg(bin, ex) sees the exclusive scan.  Ends with a barrier.
template <int NT, class Seg>
__device__ __forceinline__ void digit_offsets(RankLds<NT> &L, int nbins, const int *tot, const int *pre, Seg seg) {
  constexpr int PER = (1 << TT_SORT_MAX_BITS) / NT;
  int c[PER], sum = 0, total;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int bin = threadIdx.x * PER + k;
    c[k] = bin < nbins ? tot[bin] : 0;
    sum += c[k];
  }
  int ex = tt_block_excl_scan_n<NT>(sum, L.tmp, &total);
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int bin = threadIdx.x * PER + k;
    if (bin < nbins) {
      rank_bases(L, bin);
      L.gofs[bin] = ex + pre[bin];
      seg(bin, ex);
    }
    ex += c[k];
  }
  __syncthreads();
}

// Columns of a [tile][bin] count matrix: per bin the total over all tiles (tot) and over the tiles
// before `tile` (pre), added up by this workgroup itself, an int4 of four bins and a share of the
// rows per thread.  nbins is a power of two, at least 4.  With super != nullptr, row j of it holds the
// sum of the TT_SUPER_TILES tiles of group j: the rows to read are then the groups and the tiles of the
// own group (335 k keys: 41 rows instead of 328), so a workgroup's share of the scan stays one memory round
// trip where reading every tile took three.
template <int NT>
__device__ __forceinline__ void column_sums(const int32_t *__restrict__ hist, const int32_t *__restrict__ super, int ntiles,
                                            int tile, int nbins, int *tot, int *pre) {
  for (int b = threadIdx.x; b < nbins; b += NT) { tot[b] = 0; pre[b] = 0; }
  __syncthreads();
  const int nq = nbins / 4, parts = NT / nq;  // (at most 1024 bins: two parts or more)
  const int q = threadIdx.x & (nq - 1), part = threadIdx.x / nq;
  // rows 0 .. whole-1 count for tot (and for pre below own_whole), rows whole .. rows-1 for pre only
  const int group = tile / TT_SUPER_TILES;
  const int whole = super ? (ntiles + TT_SUPER_TILES - 1) / TT_SUPER_TILES : ntiles, own_whole = super ? group : tile;
  const int rows = super ? whole + tile % TT_SUPER_TILES : whole;
  const int32_t *__restrict__ first = super ? super : hist, *__restrict__ second = hist + (size_t)group * TT_SUPER_TILES * nbins;
  int4 s = make_int4(0, 0, 0, 0), p = make_int4(0, 0, 0, 0);
#pragma unroll 8
  for (int t = part; t < rows; t += parts) {  // independent loads: eight in flight
    const int4 v = *reinterpret_cast<const int4 *>((t < whole ? first + (size_t)t * nbins : second + (size_t)(t - whole) * nbins) + 4 * q);
    const int ms = t < whole ? -1 : 0, mp = t < own_whole || t >= whole ? -1 : 0;
    s.x += v.x & ms; s.y += v.y & ms; s.z += v.z & ms; s.w += v.w & ms;
    p.x += v.x & mp; p.y += v.y & mp; p.z += v.z & mp; p.w += v.w & mp;
  }
  if (part < rows) {
    atomicAdd(&tot[4 * q], s.x); atomicAdd(&tot[4 * q + 1], s.y); atomicAdd(&tot[4 * q + 2], s.z); atomicAdd(&tot[4 * q + 3], s.w);
    atomicAdd(&pre[4 * q], p.x); atomicAdd(&pre[4 * q + 1], p.y); atomicAdd(&pre[4 * q + 2], p.z); atomicAdd(&pre[4 * q + 3], p.w);
  }
  __syncthreads();
}
// (nullptr: a table of the batch that is short itself has no group rows, it adds up its few tiles)
__device__ __forceinline__ int32_t *super_rows(const TTDev &d, int slot) {
  if (d.sort_tiles <= TT_SCAN_TILES_MAX) return nullptr;
  return d.tmp.super + (size_t)slot * (d.sort_tiles / TT_SUPER_TILES + 1) * ((size_t)1 << TT_SORT_MAX_BITS);
}
// A tile's counts h[] -> its row of the [tile][bin] matrix, and into its group's row.
__device__ __forceinline__ void write_counts(const int *h, int nbins, int32_t *__restrict__ hist, int32_t *super, int tile, int nt) {
  for (int b = threadIdx.x; b < nbins; b += nt) {
    hist[(size_t)tile * nbins + b] = h[b];
    if (super && h[b] != 0) atomicAdd(super + (size_t)(tile / TT_SUPER_TILES) * nbins + b, h[b]);
  }
}

// How a scatter finds its offsets: it adds up the counts of all tiles, of groups of tiles (main sort only:
// the first kernel clears the group rows), or a launch of its own has scanned every column.
enum { SCAN_TILES = 0, SCAN_SUPER = 1, SCAN_LAUNCH = 2 };
#define TT_SCAN_SUPER_MAX 1024   // tiles

// ------------------------------------------------------------------ kernels of the main sort
// First kernel of a plan.  Workgroup 0 initialises the counters; every workgroup takes one sort
// tile of lookups: validate, apply the optional bijection, emit (row, position) and the bag holding
// the position, and, in sorts of few tiles, count the first radix digit of the tile's keys (so
// that the first sort pass needs no histogram launch).  An invalid lookup gets the sentinel key n1*n2*n3.
template <bool BATCHED>
__global__ void __launch_bounds__(TT_SORT_THREADS)
k_extract_keys(TTArg<BATCHED> a, int in_a, int bits, int scan) {
  const TTDev &d = a.get();
  const int64_t *__restrict__ indices = d.indices, *__restrict__ offsets = d.offsets,
                *__restrict__ remap = d.remap;
  const int nnz = d.nnz, num_bags = d.num_bags, sentinel = d.sh.sentinel;
  const long long num_rows = d.sh.num_rows;
  int32_t *__restrict__ keys = in_a ? d.plan.sorted_row : d.tmp.keys_alt;
  int32_t *__restrict__ vals = in_a ? d.plan.perm : d.tmp.vals_alt;
  int32_t *__restrict__ bag_tmp = d.tmp.bag_tmp, *__restrict__ hist = d.tmp.hist;
  if (blockIdx.x == 0) {
    if (threadIdx.x < 16) d.plan.counts[threadIdx.x] = (threadIdx.x == 3) ? nnz : 0;
    // a table without lookups has no workgroup that would write the terminal segment entries
    if (threadIdx.x == 16) d.plan.row_seg[0] = 0;
    if (threadIdx.x == 17) d.plan.pref_seg[0] = 0;
  }
  if ((int)blockIdx.x >= d.sort_tiles) return;  // uniform: a table of the batch with fewer tiles
  __shared__ int h[1 << TT_SORT_MAX_BITS];
  const int nbins = 1 << bits;
  if (scan == SCAN_SUPER) {  // group rows of every pass and grouping: the tiles add into them
    const int words = d.sort_tiles <= TT_SCAN_TILES_MAX ? 0 : TT_SUPER_SLOTS * (d.sort_tiles / TT_SUPER_TILES + 1) << TT_SORT_MAX_BITS;
    for (int e = blockIdx.x * TT_SORT_THREADS + threadIdx.x; e < words; e += d.sort_tiles * TT_SORT_THREADS) d.tmp.super[e] = 0;
  } else {
    for (int b = threadIdx.x; b < nbins; b += TT_SORT_THREADS) h[b] = 0;
  }
  __syncthreads();
  // the thread's lookups go through every step together, so that their loads overlap
  long long row[TT_SORT_ITEMS];
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i) {
    const int l = blockIdx.x * TT_SORT_TILE + i * TT_SORT_THREADS + threadIdx.x;
    row[i] = l < nnz ? indices[l] : -1;
  }
  if (remap) {
#pragma unroll
    for (int i = 0; i < TT_SORT_ITEMS; ++i)
      if (row[i] >= 0 && row[i] < num_rows) row[i] = remap[row[i]];
  }
  // largest b in [0, num_bags) with offsets[b] <= l  (empty bags share an offset and lose)
  int lo[TT_SORT_ITEMS], hi[TT_SORT_ITEMS];
  bool searching = false;
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i) {
    const int l = blockIdx.x * TT_SORT_TILE + i * TT_SORT_THREADS + threadIdx.x;
    lo[i] = 0; hi[i] = num_bags;
    if (nnz == num_bags && l < nnz && offsets[l] == (long long)l && offsets[l + 1] > (long long)l) {
      lo[i] = l; hi[i] = l + 1;  // bag b starts at lookup b (every earlier bag holds one lookup): no search
    }
    if (l >= nnz) hi[i] = lo[i] + 1;  // no lookup: nothing to find
    searching |= hi[i] - lo[i] > 1;
  }
  // Multi-lookup bags.  The tile's lookups are consecutive, so their bags start at the bag of the
  // tile's first lookup: the workgroup finds that bag with a 512-ary search (two rounds of one probe
  // per thread for 260 000 bags, instead of eighteen dependent halving steps per thread), stages the
  // next TT_SORT_TILE + 1 offsets in LDS and every thread bisects there.  Only a thread whose bag lies
  // beyond the staged window (more than a tile's worth of bags, i.e. runs of empty bags) goes on
  // halving in memory.  With offsets that are not monotone the searches still stay inside
  // [0, num_bags]; the offsets check reports them.
  __shared__ long long s_off[TT_SORT_TILE + 1];
  __shared__ int s_cnt[TT_SORT_THREADS / TT_WAVE], s_any;
  if (threadIdx.x == 0) s_any = 0;
  __syncthreads();
  if (searching) s_any = 1;
  __syncthreads();
  if (s_any) {  // uniform
    const long long first = (long long)blockIdx.x * TT_SORT_TILE;
    int wlo = 0, whi = num_bags;  // the bag of lookup `first` is in [wlo, whi)
    while (whi - wlo > 1) {       // uniform
      const int step = (whi - wlo + TT_SORT_THREADS) / (TT_SORT_THREADS + 1);  // probes wlo + (t+1)*step, t = thread
      const long long q = (long long)wlo + (long long)(threadIdx.x + 1) * step;
      const bool le = q < whi && offsets[q] <= first;
      const unsigned long long m = __ballot(le);
      if ((threadIdx.x & (TT_WAVE - 1)) == 0) s_cnt[threadIdx.x / TT_WAVE] = __popcll(m);
      __syncthreads();
      int cnt = 0;
#pragma unroll
      for (int w = 0; w < TT_SORT_THREADS / TT_WAVE; ++w) cnt += s_cnt[w];
      __syncthreads();
      // monotone offsets: the probes that are <= first are the first `cnt` ones
      const long long nlo = (long long)wlo + (long long)cnt * step, nhi = nlo + step;
      wlo = (int)nlo;
      whi = nhi < whi ? (int)nhi : whi;
    }
    const int wcount = (num_bags + 1 - wlo) < (TT_SORT_TILE + 1) ? (num_bags + 1 - wlo) : (TT_SORT_TILE + 1);
    for (int e = threadIdx.x; e < wcount; e += TT_SORT_THREADS) s_off[e] = offsets[wlo + e];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TT_SORT_ITEMS; ++i) {
      const int l = blockIdx.x * TT_SORT_TILE + i * TT_SORT_THREADS + threadIdx.x;
      if (hi[i] - lo[i] <= 1) continue;
      if (s_off[wcount - 1] <= (long long)l && wlo + wcount - 1 < num_bags) {
        lo[i] = wlo + wcount - 1;  // beyond the window: go on in memory
        continue;
      }
      int a = 0, b = wcount - 1;  // s_off[a] <= l is assumed, the answer is in [a, b)
      if (s_off[b] <= (long long)l) b = wcount;  // the last bag of the table
      while (b - a > 1) {
        const int mid = (a + b) >> 1;
        if (s_off[mid] <= (long long)l) a = mid; else b = mid;
      }
      lo[i] = wlo + a < num_bags ? wlo + a : num_bags - 1;
      hi[i] = lo[i] + 1;
    }
    searching = false;
#pragma unroll
    for (int i = 0; i < TT_SORT_ITEMS; ++i) searching |= hi[i] - lo[i] > 1;
  }
  while (searching) {  // one halving step for each of the thread's lookups per round
    searching = false;
#pragma unroll
    for (int i = 0; i < TT_SORT_ITEMS; ++i) {
      const int l = blockIdx.x * TT_SORT_TILE + i * TT_SORT_THREADS + threadIdx.x;
      if (hi[i] - lo[i] > 1) {
        const int mid = (lo[i] + hi[i]) >> 1;
        if (offsets[mid] <= (long long)l) lo[i] = mid; else hi[i] = mid;
        searching |= hi[i] - lo[i] > 1;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i) {
    const int l = blockIdx.x * TT_SORT_TILE + i * TT_SORT_THREADS + threadIdx.x;
    if (l >= nnz) continue;
    const bool ok = row[i] >= 0 && row[i] < num_rows;
    const int key = ok ? (int)row[i] : sentinel;
    keys[l] = key;
    vals[l] = l;
    if (scan != SCAN_SUPER) atomicAdd(&h[key & (nbins - 1)], 1);
    bag_tmp[l] = lo[i];
  }
  if (scan == SCAN_SUPER) return;  // uniform: the first digit is counted by a launch of its own
  __syncthreads();
  write_counts(h, nbins, hist, nullptr, blockIdx.x, TT_SORT_THREADS);
}

template <bool BATCHED>
__global__ void __launch_bounds__(TT_SORT_THREADS)
k_radix_hist(TTArg<BATCHED> a, int which, int in_a, int shift, int bits, int pass, int scan) {
  const TTDev &d = a.get();
  const SortBufs sb = sort_bufs(d, which);
  const int ntiles = sb.ntiles;
  if ((int)blockIdx.x >= ntiles) return;  // uniform: this table has fewer tiles than the widest
  const int32_t *__restrict__ keys = in_a ? sb.ka : sb.kb;
  int32_t *__restrict__ hist = d.tmp.hist + pass * ((size_t)1 << TT_SORT_MAX_BITS) * ((size_t)d.sort_tiles + 1);
  __shared__ int h[1 << TT_SORT_MAX_BITS];
  const int nbins = 1 << bits, tile = blockIdx.x, count = sb.keys();
  const int base = tile * TT_SORT_TILE;
  int key[TT_SORT_ITEMS];
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i) {
    const int pos = base + i * TT_SORT_THREADS + threadIdx.x;
    key[i] = pos < count ? keys[pos] : 0;
  }
  for (int b = threadIdx.x; b < nbins; b += TT_SORT_THREADS) h[b] = 0;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i)
    if (base + i * TT_SORT_THREADS + (int)threadIdx.x < count) atomicAdd(&h[(key[i] >> shift) & (nbins - 1)], 1);
  __syncthreads();
  write_counts(h, nbins, hist, scan == SCAN_SUPER ? super_rows(d, pass) : nullptr, tile, TT_SORT_THREADS);
}

// One workgroup per bin: exclusive scan of that bin's per-tile counts (a column of the [tile][bin]
// matrix), in place.  Only launched for sorts of many tiles; short sorts let every scatter
// workgroup add up its own column prefixes (one launch less per pass).
template <bool BATCHED>
__global__ void __launch_bounds__(TT_BLOCK)
k_radix_binscan(TTArg<BATCHED> a, int which, int nbins, int pass) {
  const TTDev &d = a.get();
  const int ntiles = sort_bufs(d, which).ntiles;
  int32_t *__restrict__ bin_total = d.tmp.bin_total;
  __shared__ int tmp[TT_BLOCK / TT_WAVE + 1];
  int32_t *col = d.tmp.hist + pass * ((size_t)1 << TT_SORT_MAX_BITS) * ((size_t)d.sort_tiles + 1) + blockIdx.x;
  int carry = 0;
  for (int base = 0; base < ntiles; base += TT_BLOCK) {
    int t = base + threadIdx.x;
    int v = t < ntiles ? col[(size_t)t * nbins] : 0, total;
    int ex = tt_block_excl_scan(v, tmp, &total);
    if (t < ntiles) col[(size_t)t * nbins] = carry + ex;
    carry += total;
  }
  if (threadIdx.x == 0) bin_total[blockIdx.x] = carry;
}

// Stable scatter of one pass.  Latency bound: a chain of loads, ranking rounds and barriers per workgroup, so
// a tile is two rounds of 512 keys (tile of 1024 keys on 512 threads / 2048 / 4096: 7.7 / 9.3 / 15 us at 65 k
// keys), and keys and payloads are requested first and land while the offsets are computed.
template <bool BATCHED>
__global__ void __launch_bounds__(TT_SORT_THREADS)
k_radix_scatter(TTArg<BATCHED> a, int which, int in_a, int shift, int bits, int scan, int status, int pass) {
  const TTDev &d = a.get();
  const SortBufs sb = sort_bufs(d, which);
  const int ntiles = sb.ntiles;
  if (status) {  // first pass of the main sort: this launch also covers the bag offsets
#pragma unroll
    for (int i = 0; i < TT_SORT_ITEMS; ++i)
      check_offsets(d, blockIdx.x * TT_SORT_TILE + i * TT_SORT_THREADS + threadIdx.x);
  }
  if ((int)blockIdx.x >= ntiles) return;  // uniform
  const int32_t *__restrict__ keys_in = in_a ? sb.ka : sb.kb, *__restrict__ vals_in = in_a ? sb.va : sb.vb;
  int32_t *__restrict__ keys_out = in_a ? sb.kb : sb.ka, *__restrict__ vals_out = in_a ? sb.vb : sb.va;
  const int32_t *__restrict__ hist = d.tmp.hist + pass * ((size_t)1 << TT_SORT_MAX_BITS) * ((size_t)d.sort_tiles + 1),
                *__restrict__ bin_total = d.tmp.bin_total;
  __shared__ RankLds<TT_SORT_THREADS> L;
  __shared__ int tot[1 << TT_SORT_MAX_BITS], pre[1 << TT_SORT_MAX_BITS];
  const int nbins = 1 << bits, tile = blockIdx.x, count = sb.keys();
  const int base = tile * TT_SORT_TILE;
  if (base >= count) return;  // uniform for the workgroup
  const int lane = threadIdx.x & (TT_WAVE - 1), wave = threadIdx.x / TT_WAVE;
  int keys_r[TT_SORT_ITEMS], vals_r[TT_SORT_ITEMS], rank[TT_SORT_ITEMS];
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i) {
    const int pos = base + (wave * TT_SORT_ITEMS + i) * TT_WAVE + lane;
    keys_r[i] = pos < count ? keys_in[pos] : 0;
    vals_r[i] = pos < count ? vals_in[pos] : 0;
    if (status && pos < count && keys_r[i] == d.sh.sentinel) atomicOr(&d.plan.counts[4], 1);  // an index was out of range
  }
  if (scan != SCAN_LAUNCH) {
    column_sums<TT_SORT_THREADS>(hist, scan == SCAN_SUPER ? super_rows(d, pass) : nullptr, ntiles, tile, nbins, tot, pre);
  } else {
    for (int b = threadIdx.x; b < nbins; b += TT_SORT_THREADS) {
      tot[b] = bin_total[b];
      pre[b] = hist[(size_t)tile * nbins + b];
    }
  }
  int digit[TT_SORT_ITEMS];
  bool valid[TT_SORT_ITEMS];
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i) {
    valid[i] = base + (wave * TT_SORT_ITEMS + i) * TT_WAVE + lane < count;
    digit[i] = (keys_r[i] >> shift) & (nbins - 1);
  }
  rank_rounds(L, digit, valid, bits, rank);
  __syncthreads();
  digit_offsets(L, nbins, tot, pre, [](int, int) {});
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i) {
    if (valid[i]) {
      const int dst = L.gofs[digit[i]] + L.wave_cnt[wave][digit[i]] + rank[i];
      keys_out[dst] = keys_r[i];
      vals_out[dst] = vals_r[i];
    }
  }
}
// ------------------------------------------------------------------ distinct rows / prefixes
#define TT_UNIQ_SELF_SCAN_TILES 1024  // up to this many tiles k_uniq_emit does without k_uniq_scan

// Run heads of the sorted keys: hr = position s starts a row, hp = it starts a prefix.  prev: the
// key in front of it (ignored at s == 0).
__device__ __forceinline__ void head_flags(const TTShape &sh, int s, int key, int prev, bool valid, bool &hr, bool &hp) {
  hr = valid && (s == 0 || prev != key);
  hp = hr && (s == 0 || tt_div(prev, sh.mul3, sh.sh3) != tt_div(key, sh.mul3, sh.sh3));
}

template <bool BATCHED>
__global__ void __launch_bounds__(TT_SORT_THREADS)
k_uniq_reduce(TTArg<BATCHED> a) {
  const TTDev &d = a.get();
  const int nnz = d.nnz, sentinel = d.sh.sentinel, ntiles = d.sort_tiles;
  if ((int)blockIdx.x >= ntiles) return;  // uniform
  const int32_t *__restrict__ keys = d.plan.sorted_row;
  __shared__ int s_sum[TT_SORT_THREADS / TT_WAVE][2];
  const int wave = threadIdx.x / TT_WAVE;
  int key[TT_SORT_ITEMS], prev[TT_SORT_ITEMS];
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i) {
    const int s = blockIdx.x * TT_SORT_TILE + i * TT_SORT_THREADS + threadIdx.x;
    key[i] = s < nnz ? keys[s] : sentinel;
    prev[i] = s < nnz && s > 0 ? keys[s - 1] : 0;
  }
  int sr = 0, sp = 0;
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i) {
    const int s = blockIdx.x * TT_SORT_TILE + i * TT_SORT_THREADS + threadIdx.x;
    bool hr, hp;
    head_flags(d.sh, s, key[i], prev[i], key[i] != sentinel, hr, hp);
    sr += __popcll(__ballot(hr));
    sp += __popcll(__ballot(hp));
  }
  if ((threadIdx.x & (TT_WAVE - 1)) == 0) { s_sum[wave][0] = sr; s_sum[wave][1] = sp; }
  __syncthreads();
  if (threadIdx.x < 2) {
    int sum = 0;
#pragma unroll
    for (int w = 0; w < TT_SORT_THREADS / TT_WAVE; ++w) sum += s_sum[w][threadIdx.x];
    d.tmp.tile_sums[threadIdx.x * ntiles + blockIdx.x] = sum;
  }
}

// Exclusive scan of the tiles' sums in place; only launched above TT_UNIQ_SELF_SCAN_TILES tiles.
template <bool BATCHED>
__global__ void __launch_bounds__(TT_BLOCK)
k_uniq_scan(TTArg<BATCHED> a) {
  const TTDev &d = a.get();
  const int ntiles = d.sort_tiles;
  __shared__ int tmp[TT_BLOCK / TT_WAVE + 1];
  for (int c = 0; c < 2; ++c) {
    int32_t *row = d.tmp.tile_sums + (size_t)c * ntiles;
    int carry = 0;
    for (int base = 0; base < ntiles; base += TT_BLOCK) {
      int t = base + threadIdx.x;
      int v = t < ntiles ? row[t] : 0, total;
      int ex = tt_block_excl_scan(v, tmp, &total);
      if (t < ntiles) row[t] = carry + ex;
      carry += total;
    }
  }
}

// Distinct rows and prefixes at their positions, per tile of sorted lookups.  With `self_scan` the
// tile sums are the raw ones of k_uniq_reduce: every workgroup adds up those of the earlier tiles
// itself (one launch less than scanning them first).  The thread of the last valid lookup writes the totals.
// grouped = 1: the workgroup also counts its distinct rows per i3 and its prefixes per i2 ([tile][bin]
// matrices for k_group), and i1_seg is filled here: prefixes come in i1 order.
// grouped = 0: the keys of the two separate grouping sorts are emitted (a3 / a2: which of their
// ping-pong buffers the sorts start from).
template <bool BATCHED>
__global__ void __launch_bounds__(TT_SORT_THREADS)
k_uniq_emit(TTArg<BATCHED> a, int a3, int a2, int self_scan, int grouped, int bits3, int bits2, int scan) {
  const TTDev &d = a.get();
  const TTShape &sh = d.sh;
  const int nnz = d.nnz, sentinel = sh.sentinel, ntiles = d.sort_tiles;
  if ((int)blockIdx.x >= ntiles) return;  // uniform
  const int32_t *__restrict__ keys = d.plan.sorted_row, *__restrict__ perm = d.plan.perm,
                *__restrict__ bag_tmp = d.tmp.bag_tmp, *__restrict__ tile_sums = d.tmp.tile_sums;
  int32_t *__restrict__ bag_of_sorted = d.plan.bag_of_sorted,
          *__restrict__ slot_of_sorted = d.plan.slot_of_sorted,
          *__restrict__ lookup2row = d.plan.lookup2row, *__restrict__ uniq_row = d.plan.uniq_row,
          *__restrict__ row_seg = d.plan.row_seg, *__restrict__ row2pref = d.plan.row2pref,
          *__restrict__ uniq_pref = d.plan.uniq_pref, *__restrict__ pref_seg = d.plan.pref_seg,
          *__restrict__ i1_seg = d.plan.i1_seg, *__restrict__ counts = d.plan.counts;
  int32_t *__restrict__ k3 = a3 ? d.plan.i3_of_sorted : d.tmp.k3_alt;
  int32_t *__restrict__ v3 = a3 ? d.plan.rows_by_i3 : d.tmp.v3_alt;
  int32_t *__restrict__ k2 = a2 ? d.tmp.k2 : d.tmp.k2_alt;
  int32_t *__restrict__ v2 = a2 ? d.plan.prefs_by_i2 : d.tmp.v2_alt;
  constexpr int NW = TT_SORT_THREADS / TT_WAVE;
  __shared__ int s_sum[NW][2], s_base[2], s_none;
  __shared__ int h3[1 << TT_SORT_MAX_BITS], h2[1 << TT_SORT_MAX_BITS];
  const int lane = threadIdx.x & (TT_WAVE - 1), wave = threadIdx.x / TT_WAVE, tile = blockIdx.x;
  const int first = tile * TT_SORT_TILE + wave * TT_SORT_ITEMS * TT_WAVE + lane;  // + i * 64: a wavefront's keys are contiguous
  // Every load of the kernel comes before its first store: loads and stores complete in issue order here,
  // so a load behind a store waits for the store.
  int key[TT_SORT_ITEMS], prev[TT_SORT_ITEMS], next[TT_SORT_ITEMS], l[TT_SORT_ITEMS], bag[TT_SORT_ITEMS];
  // sums of the earlier tiles: wavefront 0 the rows', wavefront 1 the prefixes' (requested first: loads
  // return in order)
  int before = 0;
  if (wave < 2) {
    if (self_scan) {
      for (int t = lane; t < tile; t += TT_WAVE) before += tile_sums[wave * ntiles + t];
    } else if (lane == 0) {
      before = tile_sums[wave * ntiles + tile];
    }
  }
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i) {
    const int s = first + i * TT_WAVE;
    key[i] = s < nnz ? keys[s] : sentinel;
    prev[i] = s < nnz && s > 0 ? keys[s - 1] : 0;
    next[i] = s + 1 < nnz ? keys[s + 1] : sentinel;
    l[i] = s < nnz ? perm[s] : 0;
  }
  const bool past = first - lane >= nnz;  // (uniform per wavefront)
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i) bag[i] = past ? 0 : bag_tmp[l[i]];
  if (wave < 2) {
    before = tt_wave_incl_scan(before);
    if (lane == TT_WAVE - 1) {
      s_base[wave] = before;
      d.tmp.tile_base[wave * (ntiles + 1) + tile] = before;
    }
  }
  if (grouped) {
    for (int b = threadIdx.x; b < (1 << TT_SORT_MAX_BITS); b += TT_SORT_THREADS) h3[b] = h2[b] = 0;
  }
  bool hr[TT_SORT_ITEMS], hp[TT_SORT_ITEMS];
  unsigned long long mr[TT_SORT_ITEMS], mp[TT_SORT_ITEMS];
  int sr = 0, sp = 0;
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i) {
    head_flags(sh, first + i * TT_WAVE, key[i], prev[i], key[i] != sentinel, hr[i], hp[i]);
    mr[i] = __ballot(hr[i]);
    mp[i] = __ballot(hp[i]);
    sr += __popcll(mr[i]);
    sp += __popcll(mp[i]);
  }
  if (lane == 0) { s_sum[wave][0] = sr; s_sum[wave][1] = sp; }
  if (threadIdx.x == 0) s_none = tile == 0 && key[0] == sentinel;
  __syncthreads();
  int er = s_base[0], ep = s_base[1];
  const bool none = s_none;
#pragma unroll
  for (int w = 0; w < NW; ++w)
    if (w < wave) { er += s_sum[w][0]; ep += s_sum[w][1]; }
  const unsigned long long upto = lanes_below() | (1ull << lane);
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i) {
    const int s = first + i * TT_WAVE;
    const int slot = er + __popcll(mr[i] & upto) - 1, q = ep + __popcll(mp[i] & upto) - 1;  // inclusive counts - 1
    er += __popcll(mr[i]);
    ep += __popcll(mp[i]);
    if (s >= nnz) continue;
    const bool valid = key[i] != sentinel;
    bag_of_sorted[s] = bag[i];
    slot_of_sorted[s] = valid ? slot : -1;
    lookup2row[l[i]] = valid ? slot : -1;
    if (!valid) continue;
    const int pref = tt_div(key[i], sh.mul3, sh.sh3);
    if (hr[i]) {
      const int i3 = key[i] - pref * sh.n3;
      uniq_row[slot] = key[i];
      row_seg[slot] = s;
      row2pref[slot] = q;
      if (grouped) {
        atomicAdd(&h3[i3], 1);
      } else {
        k3[slot] = i3;
        v3[slot] = slot;
      }
    }
    if (hp[i]) {
      const int i1 = tt_div(pref, sh.mul2, sh.sh2), i2 = pref - i1 * sh.n2;
      uniq_pref[q] = pref;
      pref_seg[q] = slot;
      if (grouped) {
        atomicAdd(&h2[i2], 1);
        const int i1_prev = s == 0 ? -1 : tt_div(tt_div(prev[i], sh.mul3, sh.sh3), sh.mul2, sh.sh2);
        for (int t = i1_prev + 1; t <= i1; ++t) i1_seg[t] = q;
      } else {
        k2[q] = i2;
        v2[q] = q;
      }
    }
    if (next[i] == sentinel) {  // the last valid lookup: the totals
      counts[0] = slot + 1;
      counts[1] = q + 1;
      counts[2] = s + 1;
      row_seg[slot + 1] = s + 1;
      pref_seg[q + 1] = slot + 1;
      if (grouped)
        for (int t = tt_div(pref, sh.mul2, sh.sh2) + 1; t <= sh.n1; ++t) i1_seg[t] = q + 1;
    }
  }
  if (grouped) {
    if (none)  // uniform: no valid lookup at all, every i1 range is empty
      for (int t = threadIdx.x; t <= sh.n1; t += TT_SORT_THREADS) i1_seg[t] = 0;
    __syncthreads();
    const size_t hist_stride = ((size_t)1 << TT_SORT_MAX_BITS) * ((size_t)ntiles + 1);
    write_counts(h3, 1 << bits3, d.tmp.hist, scan == SCAN_SUPER ? super_rows(d, 4) : nullptr, tile, TT_SORT_THREADS);
    write_counts(h2, 1 << bits2, d.tmp.hist + hist_stride, scan == SCAN_SUPER ? super_rows(d, 5) : nullptr, tile, TT_SORT_THREADS);
  }
}

// ------------------------------------------------------------------ groupings by i3 / i2 / i1
// seg[t] = first position of the sorted keys whose key is >= t, for t = 0..nkeys: the thread of
// position u fills the entries between its predecessor's key and its own (one memory round trip
// per thread instead of a binary search), the thread of the last position also the tail.
__device__ __forceinline__ void seg_starts(const int32_t *__restrict__ keys, int div, int count, int nkeys,
                                           int32_t *__restrict__ seg, int u) {
  if (count == 0) {
    if (u <= nkeys) seg[u] = 0;
    return;
  }
  if (u >= count) return;
  const int key = keys[u] / div, prev = u > 0 ? keys[u - 1] / div : -1;
  for (int t = prev + 1; t <= key; ++t) seg[t] = u;
  if (u == count - 1)
    for (int t = key + 1; t <= nkeys; ++t) seg[t] = count;
}

template <bool BATCHED>
__global__ void k_seg_bounds(TTArg<BATCHED> a) {
  const TTDev &d = a.get();
  const int32_t *__restrict__ counts = d.plan.counts;
  const int ur = counts[0], up = counts[1];
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  seg_starts(d.plan.i3_of_sorted, 1, ur, d.sh.n3, d.plan.i3_seg, u);
  seg_starts(d.tmp.k2, 1, up, d.sh.n2, d.plan.i2_seg, u);
  seg_starts(d.plan.uniq_pref, d.sh.n2, up, d.sh.n1, d.plan.i1_seg, u);
  if (u < up) {  // what the matrix-core kernels need to know about the u-th prefix in i2 order
    const int q = d.plan.prefs_by_i2[u], u0 = d.plan.pref_seg[q];
    reinterpret_cast<int4 *>(d.plan.pref_meta)[u] = make_int4(d.plan.uniq_pref[q] / d.sh.n2, u0, d.plan.pref_seg[q + 1] - u0, q);
  }
}

// ------------------------------------------------------------------ groupings in one launch
// Workgroups [0, tiles): the distinct rows of a tile of sorted lookups, stably sorted by i3 ->
// rows_by_i3, i3_of_sorted, i3_seg.  Workgroups [tiles, 2 * tiles): its distinct prefixes by i2 ->
// prefs_by_i2, i2_seg and the packed records the matrix-core kernels read (pref_meta).  k_uniq_emit has
// left the [tile][bin] counts and the tiles' first slots, so each workgroup ranks its own items only.
// (Each role is its own code path with its own buffers: no buffer is chosen from the workgroup index.)
struct GroupLds {
  RankLds<TT_SORT_THREADS> rank;
  int tot[1 << TT_SORT_MAX_BITS], pre[1 << TT_SORT_MAX_BITS];
};
// pref_seg: the prefixes' first row slots, loaded with the items (nullptr for the rows).
template <class KeyOf, class Place, class Seg>
__device__ __forceinline__ void group_tile(GroupLds &G, const int32_t *__restrict__ src, const int32_t *__restrict__ pref_seg,
                                           const int32_t *__restrict__ hist, const int32_t *__restrict__ super, int ntiles,
                                           int tile, int lo, int hi, int bits,
                                           KeyOf key_of, Place place, Seg seg) {
  constexpr int NT = TT_SORT_THREADS;
  RankLds<NT> &L = G.rank;
  const int nbins = 1 << bits, lane = threadIdx.x & (TT_WAVE - 1), wave = threadIdx.x / TT_WAVE;
  if (lo >= hi && tile != 0) return;  // uniform: nothing to place (tile 0 still writes the segment starts)
  int item[TT_SORT_ITEMS], key[TT_SORT_ITEMS], rank[TT_SORT_ITEMS], u0[TT_SORT_ITEMS], u1[TT_SORT_ITEMS];
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i) {
    const int pos = lo + (wave * TT_SORT_ITEMS + i) * TT_WAVE + lane;
    item[i] = pos < hi ? src[pos] : 0;
    u0[i] = pref_seg && pos < hi ? pref_seg[pos] : 0;
    u1[i] = pref_seg && pos < hi ? pref_seg[pos + 1] : 0;
  }
  column_sums<NT>(hist, super, ntiles, tile, nbins, G.tot, G.pre);
  bool valid[TT_SORT_ITEMS];
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i) {
    valid[i] = lo + (wave * TT_SORT_ITEMS + i) * TT_WAVE + lane < hi;
    key[i] = valid[i] ? key_of(item[i]) : 0;
  }
  rank_rounds(L, key, valid, bits, rank);
  __syncthreads();
  digit_offsets(L, nbins, G.tot, G.pre, [&](int bin, int ex) { if (tile == 0) seg(bin, ex); });
#pragma unroll
  for (int i = 0; i < TT_SORT_ITEMS; ++i) {
    const int pos = lo + (wave * TT_SORT_ITEMS + i) * TT_WAVE + lane;
    if (pos < hi) place(L.gofs[key[i]] + L.wave_cnt[wave][key[i]] + rank[i], pos, item[i], key[i], u0[i], u1[i]);
  }
}

template <bool BATCHED>
__global__ void __launch_bounds__(TT_SORT_THREADS)
k_group(TTArg<BATCHED> a, int tiles, int bits3, int bits2, int scan) {
  const TTDev &d = a.get();
  const int32_t *__restrict__ counts = d.plan.counts, *__restrict__ tile_base = d.tmp.tile_base;
  const int n2 = d.sh.n2, n3 = d.sh.n3, ntiles = d.sort_tiles;
  const unsigned mul3 = d.sh.mul3, sh3 = d.sh.sh3, mul2 = d.sh.mul2, sh2 = d.sh.sh2;
  __shared__ GroupLds G;
  if ((int)blockIdx.x < tiles) {
    const int tile = blockIdx.x;
    if (tile >= ntiles) return;
    const int lo = tile_base[tile], hi = tile + 1 < ntiles ? tile_base[tile + 1] : counts[0];
    int32_t *__restrict__ rows_by_i3 = d.plan.rows_by_i3, *__restrict__ i3_of_sorted = d.plan.i3_of_sorted,
            *__restrict__ i3_seg = d.plan.i3_seg;
    group_tile(G, d.plan.uniq_row, (const int32_t *)nullptr, d.tmp.hist, scan == SCAN_SUPER ? super_rows(d, 4) : nullptr, ntiles, tile,
               lo, hi, bits3,
               [&](int row) { return row - tt_div(row, mul3, sh3) * n3; },
               [&](int dst, int pos, int, int key, int, int) { rows_by_i3[dst] = pos; i3_of_sorted[dst] = key; },
               [&](int bin, int start) { if (bin <= n3) i3_seg[bin] = start; });
  } else {
    const int tile = (int)blockIdx.x - tiles;
    if (tile >= ntiles) return;
    const int lo = tile_base[ntiles + 1 + tile], hi = tile + 1 < ntiles ? tile_base[ntiles + 1 + tile + 1] : counts[1];
    int32_t *__restrict__ prefs_by_i2 = d.plan.prefs_by_i2, *__restrict__ i2_seg = d.plan.i2_seg;
    int4 *__restrict__ pref_meta = reinterpret_cast<int4 *>(d.plan.pref_meta);
    const int32_t *hist2 = d.tmp.hist + ((size_t)1 << TT_SORT_MAX_BITS) * ((size_t)ntiles + 1);
    group_tile(G, d.plan.uniq_pref, d.plan.pref_seg, hist2, scan == SCAN_SUPER ? super_rows(d, 5) : nullptr, ntiles, tile,
               lo, hi, bits2,
               [&](int pref) { return pref - tt_div(pref, mul2, sh2) * n2; },
               [&](int dst, int pos, int pref, int, int u0, int u1) {
                 prefs_by_i2[dst] = pos;  // i1, first distinct-row slot, distinct rows, prefix slot:
                 pref_meta[dst] = make_int4(tt_div(pref, mul2, sh2), u0, u1 - u0, pos);
               },
               [&](int bin, int start) { if (bin <= n2) i2_seg[bin] = start; });
  }
}

// ------------------------------------------------------------------ short batches: the plan in one launch
// Up to TT_SMALL_MAX_LOOKUPS lookups.  One workgroup builds the whole plan with the batch in LDS: bags by marking every bag's first lookup and
// a running maximum, the radix passes as LDS exchanges, run heads, both groupings.  What a short batch
// costs in the multi-launch plan is its chain of nine dependent launches of 3 to 7 us each (20 lookups: 38 us);
// here the chain is barriers (7.9 us; 256 lookups: 8.2 us).  One compute unit alone, it is bound by the issue of
// its ranking rounds: at 4096 lookups it takes 36 us, no less than the launches, hence the limit.
template <int NT, int ITEMS>
struct SmallLds {
  static constexpr int CAP = NT * ITEMS;
  RankLds<NT> rank;
  int key[CAP];             // sorted keys; afterwards the distinct rows
  int bag[CAP];             // bag of each lookup; while the prefixes are grouped, their first row slots
  int pref[CAP + 1];        // distinct prefixes
  unsigned short pos[CAP];  // payload of the sort: lookup position
  __align__(16) int tiny[2][NT == TT_WAVE ? NT : 4];  // keys of tiny_pass
  int wave_sum[NT / TT_WAVE][2];
  int total[2];
};

// One LDS counting-sort pass over `count` keys held one per (thread, item): ranks key[i] = its digit,
// then place(i, dst) for every valid item.  seg(bin, start) receives the start of every digit's run.
template <int NT, int ITEMS, class Place, class Seg>
__device__ __forceinline__ void small_pass(RankLds<NT> &L, const int (&digit)[ITEMS], int count, int bits, Place place, Seg seg) {
  const int nbins = 1 << bits, lane = threadIdx.x & (TT_WAVE - 1), wave = threadIdx.x / TT_WAVE;
  constexpr int PER = (1 << TT_SORT_MAX_BITS) / NT;
  int rank[ITEMS];
  bool valid[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) valid[i] = (wave * ITEMS + i) * TT_WAVE + lane < count;
  rank_rounds(L, digit, valid, bits, rank);
  __syncthreads();
  int c[PER], sum = 0, total;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int bin = threadIdx.x * PER + k;
    c[k] = bin < nbins ? rank_bases(L, bin) : 0;
    sum += c[k];
  }
  int ex = tt_block_excl_scan_n<NT>(sum, L.tmp, &total);
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int bin = threadIdx.x * PER + k;
    if (bin < nbins) {
      L.gofs[bin] = ex;
      seg(bin, ex);
    }
    ex += c[k];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (valid[i]) place(i, L.gofs[digit[i]] + L.wave_cnt[wave][digit[i]] + rank[i]);
  __syncthreads();
}

// The same for at most NT keys, one per thread: a key's position is the number of keys in front of it,
// counted over all of them (LDS broadcasts), and a run starts at the lower bound of its digit.
// `keys`, `sorted`: LDS, NT + 3 entries.
template <int NT, class Place, class Seg>
__device__ __forceinline__ void tiny_pass(int *keys, int *sorted, unsigned key, int count, int nseg, Place place, Seg seg) {
  const int i = threadIdx.x;
  keys[i] = (int)key;
  __syncthreads();
  if (i < count) {
    int dst = 0;
#pragma unroll 4
    for (int j = 0; j < count; j += 4) {
      const int4 k = *reinterpret_cast<const int4 *>(keys + j);
      const unsigned kk[4] = {(unsigned)k.x, (unsigned)k.y, (unsigned)k.z, (unsigned)k.w};
#pragma unroll
      for (int u = 0; u < 4; ++u) dst += (j + u < count && kk[u] < key + (j + u < i ? 1u : 0u)) ? 1 : 0;
    }
    sorted[dst] = (int)key;
    place(0, dst);
  }
  __syncthreads();
  for (int t = i; t < nseg; t += NT) {
    int lo = 0, hi = count;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (sorted[mid] < t) lo = mid + 1; else hi = mid;
    }
    seg(t, lo);
  }
}

template <bool BATCHED, int NT, int ITEMS>
__global__ void __launch_bounds__(NT)
k_plan_small(TTArg<BATCHED> a, int key_bits, int bits_per_pass, int bits3, int bits2) {
  const TTDev &d = a.get();
  const TTShape &sh = d.sh;
  const int64_t *__restrict__ indices = d.indices, *__restrict__ offsets = d.offsets, *__restrict__ remap = d.remap;
  const int nnz = d.nnz, num_bags = d.num_bags, sentinel = sh.sentinel;
  const int lane = threadIdx.x & (TT_WAVE - 1), wave = threadIdx.x / TT_WAVE;
  constexpr int NW = NT / TT_WAVE;
  __shared__ SmallLds<NT, ITEMS> S;
  __shared__ int s_status;
  const int first = wave * ITEMS * TT_WAVE + lane;  // + i * 64: a wavefront's positions are contiguous
  long long row[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) row[i] = first + i * TT_WAVE < nnz ? indices[first + i * TT_WAVE] : -1;
  if (threadIdx.x == 0) s_status = 0;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) S.bag[first + i * TT_WAVE] = 0;
  __syncthreads();
  // every bag with lookups marks its first one (positions in [0, nnz) only, whatever the offsets hold)
  for (int b = threadIdx.x; b <= num_bags; b += NT) {
    const long long o = offsets[b];
    bool bad;
    if (b < num_bags) {
      const long long o1 = offsets[b + 1];
      bad = o > o1 || o < 0;
      if (o >= 0 && o < o1 && o < nnz) S.bag[o] = b;
    } else {
      bad = o != (long long)nnz || offsets[0] != 0;
    }
    if (bad) atomicOr(&s_status, 2);
  }
  if (remap) {
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if (row[i] >= 0 && row[i] < sh.num_rows) row[i] = remap[row[i]];
  }
  int key[ITEMS], val[ITEMS], digit[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const bool ok = row[i] >= 0 && row[i] < sh.num_rows;
    key[i] = ok ? (int)row[i] : sentinel;
    val[i] = first + i * TT_WAVE;
    if (!ok && val[i] < nnz) atomicOr(&s_status, 1);
  }
  __syncthreads();
  {  // running maximum of the marks: inside the wavefront's range, then over the wavefronts before it
    int run = 0, mark[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      int m = S.bag[first + i * TT_WAVE];
#pragma unroll
      for (int o = 1; o < TT_WAVE; o <<= 1) {
        const int t = __shfl_up(m, o, TT_WAVE);
        if (lane >= o && t > m) m = t;
      }
      m = m > run ? m : run;
      mark[i] = m;
      run = __shfl(m, TT_WAVE - 1, TT_WAVE);
    }
    if (lane == 0) S.wave_sum[wave][0] = run;
    __syncthreads();
    int before = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w)
      if (w < wave && S.wave_sum[w][0] > before) before = S.wave_sum[w][0];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) S.bag[first + i * TT_WAVE] = mark[i] > before ? mark[i] : before;
  }
  // ---- stable sort by row ----
  if constexpr (NT == TT_WAVE) {
    tiny_pass<NT>(S.tiny[0], S.tiny[1], (unsigned)key[0], nnz, 0, [&](int, int dst) { S.key[dst] = key[0]; S.pos[dst] = (unsigned short)val[0]; },
                  [&](int, int) {});
    if (first < nnz) { key[0] = S.key[first]; val[0] = S.pos[first]; }
  } else
  for (int shift = 0; shift < key_bits; shift += bits_per_pass) {
    const int left = key_bits - shift, bits = left < bits_per_pass ? left : bits_per_pass;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) digit[i] = (key[i] >> shift) & ((1 << bits) - 1);
    small_pass<NT, ITEMS>(S.rank, digit, nnz, bits,
                          [&](int i, int dst) { S.key[dst] = key[i]; S.pos[dst] = (unsigned short)val[i]; }, [&](int, int) {});
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if (first + i * TT_WAVE < nnz) { key[i] = S.key[first + i * TT_WAVE]; val[i] = S.pos[first + i * TT_WAVE]; }
  }
  // ---- distinct rows and prefixes ----
  bool hr[ITEMS], hp[ITEMS], last[ITEMS];
  int prev[ITEMS];
  unsigned long long mr[ITEMS], mp[ITEMS];
  int sr = 0, sp = 0;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int s = first + i * TT_WAVE;
    const bool valid = s < nnz && key[i] != sentinel;
    prev[i] = valid && s > 0 ? S.key[s - 1] : 0;
    last[i] = valid && (s == nnz - 1 || S.key[s + 1] == sentinel);
    head_flags(sh, s, key[i], prev[i], valid, hr[i], hp[i]);
    mr[i] = __ballot(hr[i]);
    mp[i] = __ballot(hp[i]);
    sr += __popcll(mr[i]);
    sp += __popcll(mp[i]);
  }
  if (lane == 0) { S.wave_sum[wave][0] = sr; S.wave_sum[wave][1] = sp; }
  if (threadIdx.x < 2) S.total[threadIdx.x] = 0;  // (stays so when no lookup is valid)
  __syncthreads();  // (also: every neighbour key has been read, S.key may take the distinct rows)
  int er = 0, ep = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w)
    if (w < wave) { er += S.wave_sum[w][0]; ep += S.wave_sum[w][1]; }
  const unsigned long long upto = lanes_below() | (1ull << lane);
  int slot_p[ITEMS], slot_u[ITEMS];  // of a prefix head: prefix slot, first row slot
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int s = first + i * TT_WAVE;
    const int slot = er + __popcll(mr[i] & upto) - 1, q = ep + __popcll(mp[i] & upto) - 1;
    er += __popcll(mr[i]);
    ep += __popcll(mp[i]);
    slot_p[i] = -1;
    slot_u[i] = slot;
    if (s >= nnz) continue;
    const bool valid = key[i] != sentinel;
    d.plan.sorted_row[s] = key[i];
    d.plan.perm[s] = val[i];
    d.plan.bag_of_sorted[s] = S.bag[val[i]];
    d.plan.slot_of_sorted[s] = valid ? slot : -1;
    d.plan.lookup2row[val[i]] = valid ? slot : -1;
    if (!valid) continue;
    const int pref = tt_div(key[i], sh.mul3, sh.sh3);
    if (hr[i]) {
      S.key[slot] = key[i];
      d.plan.uniq_row[slot] = key[i];
      d.plan.row_seg[slot] = s;
      d.plan.row2pref[slot] = q;
    }
    if (hp[i]) {
      slot_p[i] = q;
      S.pref[q] = pref;
      d.plan.uniq_pref[q] = pref;
      d.plan.pref_seg[q] = slot;
    }
    if (last[i]) {
      S.total[0] = slot + 1;
      S.total[1] = q + 1;
      d.plan.row_seg[slot + 1] = s + 1;
      d.plan.pref_seg[q + 1] = slot + 1;
      d.plan.counts[2] = s + 1;
    }
  }
  __syncthreads();  // distinct rows, prefixes and totals are in LDS; the bags have been read
  const int ur = S.total[0], up = S.total[1];
  if (threadIdx.x < 16 && (threadIdx.x != 2 || ur == 0))
    d.plan.counts[threadIdx.x] = threadIdx.x == 0 ? ur : threadIdx.x == 1 ? up : threadIdx.x == 3 ? nnz : threadIdx.x == 4 ? s_status : 0;
  if (ur == 0 && threadIdx.x == 0) { d.plan.row_seg[0] = 0; d.plan.pref_seg[0] = 0; }  // no valid lookup
  for (int t = threadIdx.x; t <= sh.n1; t += NT) {  // prefixes are in i1 order: the first one at or above (t, 0)
    int lo = 0, hi = up;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if ((long long)S.pref[mid] < (long long)t * sh.n2) lo = mid + 1; else hi = mid;
    }
    d.plan.i1_seg[t] = lo;
  }
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (slot_p[i] >= 0) S.bag[slot_p[i]] = slot_u[i];
  // ---- groupings ----
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int u = first + i * TT_WAVE;
    digit[i] = 0;
    if (u < ur) {
      const int r = S.key[u];
      digit[i] = r - tt_div(r, sh.mul3, sh.sh3) * sh.n3;
    }
  }
  {
    int32_t *__restrict__ rows_by_i3 = d.plan.rows_by_i3, *__restrict__ i3_of_sorted = d.plan.i3_of_sorted,
            *__restrict__ i3_seg = d.plan.i3_seg;
    auto place = [&](int i, int dst) { rows_by_i3[dst] = first + i * TT_WAVE; i3_of_sorted[dst] = digit[i]; };
    auto seg = [&](int bin, int start) { if (bin <= sh.n3) i3_seg[bin] = start; };
    if constexpr (NT == TT_WAVE) tiny_pass<NT>(S.tiny[0], S.tiny[1], (unsigned)digit[0], ur, sh.n3 + 1, place, seg);
    else small_pass<NT, ITEMS>(S.rank, digit, ur, bits3, place, seg);
  }
  int pref_i1[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int q = first + i * TT_WAVE;
    digit[i] = 0;
    pref_i1[i] = 0;
    if (q < up) {
      const int p = S.pref[q];
      pref_i1[i] = tt_div(p, sh.mul2, sh.sh2);
      digit[i] = p - pref_i1[i] * sh.n2;
    }
  }
  {
    int32_t *__restrict__ prefs_by_i2 = d.plan.prefs_by_i2, *__restrict__ i2_seg = d.plan.i2_seg;
    int4 *__restrict__ pref_meta = reinterpret_cast<int4 *>(d.plan.pref_meta);
    auto place = [&](int i, int dst) {
      const int q = first + i * TT_WAVE, u0 = S.bag[q], u1 = q + 1 < up ? S.bag[q + 1] : ur;
      prefs_by_i2[dst] = q;
      pref_meta[dst] = make_int4(pref_i1[i], u0, u1 - u0, q);
    };
    auto seg = [&](int bin, int start) { if (bin <= sh.n2) i2_seg[bin] = start; };
    if constexpr (NT == TT_WAVE) tiny_pass<NT>(S.tiny[0], S.tiny[1], (unsigned)digit[0], up, sh.n2 + 1, place, seg);
    else small_pass<NT, ITEMS>(S.rank, digit, up, bits2, place, seg);
  }
}

int bit_length(long long v) {
  int b = 0;
  while (v > 0) { ++b; v >>= 1; }
  return b;
}

struct RadixPlan { int passes; int bits_per_pass; };
RadixPlan radix_plan(int key_bits) {
  RadixPlan p;
  p.passes = (key_bits + TT_SORT_MAX_BITS - 1) / TT_SORT_MAX_BITS;
  p.bits_per_pass = p.passes ? (key_bits + p.passes - 1) / p.passes : 0;
  return p;
}

// A sort digit has at least two bits: the [tile][bin] matrices are read as int4.
int sort_bits(int bits) { return bits < 2 ? 2 : bits; }

int scan_mode(int tiles, bool main_sort) {
  if (tiles <= TT_SCAN_TILES_MAX) return SCAN_TILES;
  return main_sort && tiles <= TT_SCAN_SUPER_MAX ? SCAN_SUPER : SCAN_LAUNCH;
}

// One of the three sorts, for every table of the batch, with the same pass structure (so that a
// pass is one launch): key_bits is the widest key of the batch.  The input must sit in the (a)
// buffers when the number of passes is even and in (b) when it is odd; the result lands in (a).
// `status_tiles` > 0 marks the main sort: unless groups of tiles are counted, its first pass finds its
// histogram already there (the kernel that extracted the keys counted the first digit), and its first
// scatter launch is made wide enough to check the bag offsets as well.
tt_status radix_sort(const TTBatch &b, int which, int max_tiles, int key_bits, hipStream_t s, int status_tiles) {
  const RadixPlan rp = radix_plan(key_bits);
  if (max_tiles == 0) return TT_OK;
  int in_a = (rp.passes % 2) == 0;
  int shift = 0;
  for (int p = 0; p < rp.passes; ++p) {
    const int width = (key_bits - shift) < rp.bits_per_pass ? (key_bits - shift) : rp.bits_per_pass, bits = sort_bits(width);
    const bool main_sort = status_tiles > 0;
    const int scan = scan_mode(max_tiles, main_sort);
    const int status = (main_sort && p == 0) ? 1 : 0;
    const int pass = main_sort ? p : 0;
    if (!main_sort || p > 0 || scan == SCAN_SUPER)
      TT_LAUNCH(k_radix_hist, max_tiles, TT_SORT_THREADS, 0, s, b, which, in_a, shift, bits, pass, scan);
    if (scan == SCAN_LAUNCH) TT_LAUNCH(k_radix_binscan, 1 << bits, TT_BLOCK, 0, s, b, which, 1 << bits, pass);
    {
      TTProfScope prof(which == 0 ? &b.host[0].plan : nullptr, TT_KERNEL_SORT_SCATTER, s);
      const int grid = status && status_tiles > max_tiles ? status_tiles : max_tiles;
      TT_LAUNCH(k_radix_scatter, grid, TT_SORT_THREADS, 0, s, b, which, in_a, shift, bits, scan, status, pass);
    }
    shift += width;
    in_a = !in_a;
  }
  return tt_launch_status();
}

}  // namespace

int ttk_radix_passes(int key_bits) { return radix_plan(key_bits).passes; }

tt_status ttk_sort_slot1(const TTDev &d, int key_bits, hipStream_t s) {
  const TTBatch b = {1, &d, nullptr};
  return radix_sort(b, 1, tt_ceil_div(d.plan.max_rows, TT_SORT_TILE), key_bits, s, 0);
}

// The scratch is what the arrays with a place of their own take; batches that fit a fixed scratch depend on it.
size_t tt_sort_tmp_bytes(int64_t nnz, int64_t max_rows, int64_t max_prefixes) {
  const size_t ntiles = (size_t)tt_ceil_div(nnz, TT_SORT_TILE) + 1;
  size_t ints = 3 * (size_t)nnz + 2 * (size_t)max_rows + 3 * (size_t)max_prefixes +
                TT_SORT_MAX_PASSES * ((size_t)1 << TT_SORT_MAX_BITS) * ntiles + ((size_t)1 << TT_SORT_MAX_BITS) +
                2 * ntiles;
  return (ints + 64 * 12) * sizeof(int32_t);
}

TTSortTmp tt_sort_tmp_view(const tt_plan *plan) {
  TTSortTmp t;
  const size_t nnz = (size_t)plan->nnz, mr = (size_t)plan->max_rows,
               mp = (size_t)plan->max_prefixes;
  const size_t ntiles = (size_t)tt_ceil_div(plan->nnz, TT_SORT_TILE) + 1;
  int32_t *p = (int32_t *)plan->sort_tmp;
  auto take = [&](size_t count) {
    int32_t *q = p;
    p += (count + 63) / 64 * 64;  // keep every array 256-byte aligned
    return q;
  };
  t.keys_alt = take(nnz);
  t.vals_alt = take(nnz);
  t.bag_tmp = take(nnz);
  t.k3_alt = take(mr);
  t.v3_alt = take(mr);
  t.k2 = take(mp);
  t.k2_alt = take(mp);
  t.v2_alt = take(mp);
  t.hist = take(TT_SORT_MAX_PASSES * ((size_t)1 << TT_SORT_MAX_BITS) * ntiles);  // one [tile][bin] array per pass
  t.bin_total = take((size_t)1 << TT_SORT_MAX_BITS);
  t.tile_sums = take(2 * ntiles);
  // Two arrays live in space that is free when they are used.  The tiles' first slots (2 * ntiles entries, at least
  // 64 are there) are written after the sort, whose ping-pong keys are dead by then.  The group rows lie at the
  // end of the histograms: a sort of three passes or fewer leaves the last pass's array free, one of
  // four has digits of 8 bits and fills a quarter of it, and from TT_SCAN_TILES_MAX tiles on the rows take less than
  // a third.
  t.tile_base = t.keys_alt;
  const size_t bins = (size_t)1 << TT_SORT_MAX_BITS, tiles = ntiles - 1, groups = tiles / TT_SUPER_TILES + 1;
  t.super = tiles > TT_SCAN_TILES_MAX ? t.hist + TT_SORT_MAX_PASSES * bins * ntiles - TT_SUPER_SLOTS * bins * groups : nullptr;
  return t;
}

tt_status ttk_reorder(const TTBatch &b, hipStream_t s) {
  // main sort: keys in [0, sentinel]
  const int key_bits = bit_length(tt_batch_max(b, [](const TTDev &d) { return (long long)d.sh.sentinel; }));
  const RadixPlan rp0 = radix_plan(key_bits);
  const int in_a = (rp0.passes % 2) == 0;
  const int bits0 = sort_bits(key_bits < rp0.bits_per_pass ? key_bits : rp0.bits_per_pass);
  const int tiles0 = (int)tt_batch_max(b, [](const TTDev &d) { return (long long)d.sort_tiles; });
  const long long n1max = tt_batch_max(b, [](const TTDev &d) { return (long long)d.sh.n1; });
  const long long n2max = tt_batch_max(b, [](const TTDev &d) { return (long long)d.sh.n2; });
  const long long n3max = tt_batch_max(b, [](const TTDev &d) { return (long long)d.sh.n3; });
  // (the values n3, n2 themselves get a bin: its start is the item count)
  const int bits3 = sort_bits(bit_length(n3max)), bits2 = sort_bits(bit_length(n2max));
  const bool narrow = bits3 <= TT_SORT_MAX_BITS && bits2 <= TT_SORT_MAX_BITS;  // groupings of one digit each
  const long long bags = tt_batch_max(b, [](const TTDev &d) { return (long long)d.num_bags; });
  const long long nnz = tt_batch_max(b, [](const TTDev &d) { return (long long)d.nnz; });
  bool any_empty = false;
  for (int t = 0; t < b.T; ++t) any_empty = any_empty || b.host[t].nnz == 0;
  if (narrow && !any_empty && nnz <= TT_SMALL_MAX_LOOKUPS && bags <= TT_SMALL_MAX_BAGS && n1max <= TT_SMALL_MAX_BAGS) {
    const int w = rp0.bits_per_pass;
    // One wavefront needs no barriers but walks everything alone: 20 lookups of n = (200, 250, 200) take it 9.5 us and four
    // wavefronts 10.1, with n1 = 1024 12.8 and 11.2, 60 lookups in 20 bags 13.5 and 10.2, 60 in 1000 bags with n1 = 16000
    // 119 and 37 (and the several launches 86).
    const bool tiny = nnz <= 32 && bags <= 64 && n1max <= 256 && n2max <= 256 && n3max <= 256;
    if (tiny) TT_LAUNCH_T2(k_plan_small, 64, 1, 1, 64, 0, s, b, key_bits, w, bits3, bits2);
    else if (nnz <= 256) TT_LAUNCH_T2(k_plan_small, 256, 1, 1, 256, 0, s, b, key_bits, w, bits3, bits2);
    else if (nnz <= 1024) TT_LAUNCH_T2(k_plan_small, 512, 2, 1, 512, 0, s, b, key_bits, w, bits3, bits2);
    else TT_LAUNCH_T2(k_plan_small, 512, 4, 1, 512, 0, s, b, key_bits, w, bits3, bits2);
    return tt_launch_status();
  }
  // first kernel: counters, keys, bags, histogram of the first digit or cleared group rows
  const int scan = scan_mode(tiles0, true);
  TT_LAUNCH(k_extract_keys, tiles0 > 0 ? tiles0 : 1, TT_SORT_THREADS, 0, s, b, in_a, bits0, scan);
  if (any_empty) {
    const long long cover = tt_batch_max(b, [](const TTDev &d) {
      long long m = d.sh.n1 > d.sh.n2 ? d.sh.n1 : d.sh.n2;
      m = (m > d.sh.n3 ? m : (long long)d.sh.n3) + 1;
      return m > d.num_bags + 1 ? m : (long long)d.num_bags + 1; });
    TT_LAUNCH(k_empty_plan, tt_ceil_div(cover, TT_BLOCK), TT_BLOCK, 0, s, b);
  }
  if (tiles0 == 0) return tt_launch_status();  // no lookups at all: the plan is complete
  // the first scatter pass also checks the bag offsets (one thread per offset)
  tt_status st = radix_sort(b, 0, tiles0, key_bits, s, tt_ceil_div(bags + 1, TT_SORT_TILE));
  if (st != TT_OK) return st;

  // Distinct rows and prefixes, then the groupings: distinct rows by i3, distinct prefixes by i2 (stable),
  // i1 ranges.  Both groupings take one launch when every key fits one digit and each workgroup can add
  // up the [tile][bin] columns itself; two more radix sorts otherwise.
  const bool grouped = narrow && scan != SCAN_LAUNCH;
  const int sb3 = bit_length(n3max - 1), sb2 = bit_length(n2max - 1);  // key widths of the separate grouping sorts
  const int a3 = (radix_plan(sb3).passes % 2) == 0, a2 = (radix_plan(sb2).passes % 2) == 0;
  const int uniq_self = tiles0 <= TT_UNIQ_SELF_SCAN_TILES ? 1 : 0;
  TT_LAUNCH(k_uniq_reduce, tiles0, TT_SORT_THREADS, 0, s, b);
  if (!uniq_self) TT_LAUNCH(k_uniq_scan, 1, TT_BLOCK, 0, s, b);
  TT_LAUNCH(k_uniq_emit, tiles0, TT_SORT_THREADS, 0, s, b, a3, a2, uniq_self, grouped ? 1 : 0, bits3, bits2, scan);
  if (grouped) {
    TT_LAUNCH(k_group, 2 * tiles0, TT_SORT_THREADS, 0, s, b, tiles0, bits3, bits2, scan);
    return tt_launch_status();
  }
  const long long max_rows = tt_batch_max(b, [](const TTDev &d) { return (long long)d.plan.max_rows; });
  const long long max_pref = tt_batch_max(b, [](const TTDev &d) { return (long long)d.plan.max_prefixes; });
  st = radix_sort(b, 1, tt_ceil_div(max_rows, TT_SORT_TILE), sb3, s, 0);
  if (st != TT_OK) return st;
  st = radix_sort(b, 2, tt_ceil_div(max_pref, TT_SORT_TILE), sb2, s, 0);
  if (st != TT_OK) return st;
  // one thread per sorted position (and at least one per segment boundary when a count is zero)
  const long long nmax = tt_batch_max(b, [](const TTDev &d) {
    long long m = d.sh.n1 > d.sh.n2 ? d.sh.n1 : d.sh.n2;
    m = m > d.sh.n3 ? m : (long long)d.sh.n3;
    m += 1;
    return m > d.plan.max_rows ? m : (long long)d.plan.max_rows; });
  TT_LAUNCH(k_seg_bounds, tt_ceil_div(nmax, TT_BLOCK), TT_BLOCK, 0, s, b);
  return tt_launch_status();
}
