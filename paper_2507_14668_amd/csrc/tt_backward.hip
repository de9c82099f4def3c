// Backward pass of the TT embedding bag (paper Section III-D backward equation, Section III-E
// in-advance gradient aggregation) and the gradient-descent core update.
//
// Planned arm:
//   1. merge grad_out over all occurrences of each distinct row (segmented gather-sum);
//   2. per distinct prefix: rebuild P12, and for each distinct row under it form the core-2
//      contribution P12^T g and accumulate the right partial H = sum_rows g G3[i3]^T;
//      then the core-0 contribution H G2[i2]^T;
//   3. reduce the per-row / per-prefix contributions into core-shaped gradients with sorted
//      segmented sums (core 2 by i3, core 0 by i1) and a per-i2 accumulation (core 1).
//   No floating-point atomics: every output element is written once, in a fixed order.
// Naive arm: one workgroup per lookup, full chain, atomicAdd into the core gradients.
#include <type_traits>

#include "tt_internal.h"

namespace {

// ------------------------------------------------------------------ two-stage segmented sum
// Positions 0..M-1 carry a vector src[gidx[pos]][W] and a non-decreasing segment id
// seg_src[pos]/seg_div; seg_off[s]..seg_off[s+1] is the position range of segment s.
// Stage 1 walks fixed chunks of `chunk` positions in order; a segment that lies inside one
// chunk is finished there, otherwise the chunk leaves a partial: slot 0 = run that began before
// the chunk, slot 1 = run that begins in the chunk and continues past its end.
// A position may carry `nsub` consecutive vectors (src[(gidx[pos]*nsub + t)][W], t < nsub),
// which are added in order first.
// Output element e of segment s goes to out[((e/out_inner)*nseg + s)*out_inner + e%out_inner]
// (out_inner = W gives a contiguous [nseg][W] array; out_inner = d3 gives core-2 layout).
template <int VEC>
struct Vec {
  float v[VEC];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int k = 0; k < VEC; ++k) v[k] = 0.f;
  }
  __device__ __forceinline__ void load(const float *p) {
    if (VEC == 4) {
      const float4 t = *reinterpret_cast<const float4 *>(p);
      v[0] = t.x; v[1 % VEC] = t.y; v[2 % VEC] = t.z; v[3 % VEC] = t.w;
    } else {
      v[0] = *p;
    }
  }
  __device__ __forceinline__ void load_stream(const float *p) {  // data read exactly once
    if (VEC == 4) {
      const float4 t = tt_load_stream4(p);
      v[0] = t.x; v[1 % VEC] = t.y; v[2 % VEC] = t.z; v[3 % VEC] = t.w;
    } else {
      v[0] = *p;
    }
  }
  __device__ __forceinline__ void store(float *p) const {
    if (VEC == 4) *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1 % VEC], v[2 % VEC], v[3 % VEC]);
    else *p = v[0];
  }
  // p <- p - lr * v   (the fused core update: the finished gradient slice is never stored)
  __device__ __forceinline__ void store_sgd(float *p, float lr) const {
    Vec old;
    old.load(p);
#pragma unroll
    for (int k = 0; k < VEC; ++k) old.v[k] = fmaf(-lr, v[k], old.v[k]);
    old.store(p);
  }
  __device__ __forceinline__ void add(const Vec &o) {
#pragma unroll
    for (int k = 0; k < VEC; ++k) v[k] += o.v[k];
  }
};

__device__ __forceinline__ size_t seg_out_index(int s, int e, int out_inner, int nseg) {
  const int hi = e / out_inner, lo = e - hi * out_inner;
  return ((size_t)hi * nseg + s) * out_inner + lo;
}

// The three segmented sums of the backward pass, described per table on the device.
enum { SEG_GAGG = 0, SEG_DG3 = 1, SEG_DG1 = 2 };
struct SegView {
  int W;                     // vector width
  const int32_t *count_ptr;  // device: number of positions
  const int32_t *seg_src;
  int seg_div;
  const int32_t *gidx;
  const int32_t *seg_off;
  const float *src;
  int nsub;                  // vectors per position
  float *out;
  int out_inner;
  int nseg;                  // number of segments (output layout / dense zero fill)
  int dense;
  float *partial;
  int fused;                 // out is the core itself: finished sums are applied as out -= lr * sum
  float lr;
  int stream_src;            // every source vector is read once: non-temporal loads
};
__device__ __forceinline__ SegView seg_view(const TTDev &d, int kind) {
  SegView v;
  v.partial = d.plan.partial;
  v.fused = 0; v.lr = d.lr;
  v.stream_src = 1;  // the hand-off buffers are read once; the output gradients only with one lookup per bag
  if (kind == SEG_GAGG) {  // merge grad_out over the occurrences of each distinct row
    v.W = d.sh.D; v.count_ptr = d.plan.counts + 2; v.seg_src = d.plan.slot_of_sorted; v.seg_div = 1;
    v.gidx = d.plan.bag_of_sorted; v.seg_off = d.plan.row_seg; v.src = d.grad_out; v.nsub = 1;
    v.out = d.plan.gagg; v.out_inner = d.sh.D; v.nseg = (int)d.plan.max_rows; v.dense = 0;
    v.stream_src = d.nnz == d.num_bags;
  } else if (kind == SEG_DG3) {  // core 2: per-row contributions of all rows sharing i3
    v.W = d.sh.S3; v.count_ptr = d.plan.counts + 0; v.seg_src = d.plan.i3_of_sorted; v.seg_div = 1;
    v.gidx = d.plan.rows_by_i3; v.seg_off = d.plan.i3_seg; v.src = d.plan.t3buf; v.nsub = 1;
    v.out = d.dg[2]; v.out_inner = d.sh.d3; v.nseg = d.sh.n3; v.dense = 1;
    if (d.fused) { v.out = const_cast<float *>(d.g[2]); v.dense = 0; v.fused = 1; }
  } else {  // core 0: per-prefix contributions of all prefixes sharing i1 (contiguous)
    v.W = d.sh.S1; v.count_ptr = d.plan.counts + 1; v.seg_src = d.plan.uniq_pref; v.seg_div = d.sh.n2;
    v.gidx = nullptr; v.seg_off = d.plan.i1_seg; v.src = d.plan.t1buf; v.nsub = d.strips;
    v.out = d.dg[0]; v.out_inner = d.sh.S1; v.nseg = d.sh.n1; v.dense = 1;
    if (d.fused) { v.out = const_cast<float *>(d.g[0]); v.dense = 0; v.fused = 1; }
  }
  return v;
}

// One launch serves one segmented sum, or two of the same vector width side by side (the first
// `blocks` workgroups the first kind, the rest the second, whose partials follow the first kind's
// in the table's partial buffer).
struct SegLaunch {
  int kind, chunk, blocks;
  int kind_b, chunk_b;  // kind_b < 0: a single sum
  int spread, spread_b; // stage 2 takes a chunk per lane group instead of one per workgroup
};
struct SegPick { int kind, chunk, bid, nblk, spread; size_t poff; };
__device__ __forceinline__ SegPick seg_pick(const SegLaunch &L, const TTDev &d) {
  SegPick p = {L.kind, L.chunk, (int)blockIdx.x, L.kind_b < 0 ? (int)gridDim.x : L.blocks, L.spread, 0};
  if (L.kind_b >= 0 && (int)blockIdx.x >= L.blocks) {
    p.kind = L.kind_b; p.chunk = L.chunk_b; p.spread = L.spread_b; p.bid = (int)blockIdx.x - L.blocks;
    p.nblk = (int)gridDim.x - L.blocks;
    // the first kind's share of this table's partial buffer: two slots per chunk it can have
    const long long cap = L.kind == SEG_GAGG ? d.plan.nnz : (L.kind == SEG_DG3 ? d.plan.max_rows : d.plan.max_prefixes);
    const int W = L.kind == SEG_GAGG ? d.sh.D : (L.kind == SEG_DG3 ? d.sh.S3 : d.sh.S1);
    p.poff = (size_t)((cap + L.chunk - 1) / L.chunk + 1) * 2 * W;
  }
  return p;
}

template <bool BATCHED, int VEC>
__global__ void __launch_bounds__(TT_BLOCK)
k_seg_stage1(TTArg<BATCHED> arg, SegLaunch L, int lanes) {
  const SegPick pk = seg_pick(L, arg.get());
  const int chunk = pk.chunk;
  const SegView sv = seg_view(arg.get(), pk.kind);
  const int W = sv.W, seg_div = sv.seg_div, nsub = sv.nsub, out_inner = sv.out_inner, nseg = sv.nseg;
  const int32_t *__restrict__ seg_src = sv.seg_src, *__restrict__ gidx = sv.gidx;
  const float *__restrict__ src = sv.src;
  float *__restrict__ out = sv.out, *__restrict__ partial = sv.partial + pk.poff;
  const int M = *sv.count_ptr;
  const int nchunks = (M + chunk - 1) / chunk;
  const int fused = sv.fused, stream_src = sv.stream_src;
  const float lr = sv.lr;
  const int groups = blockDim.x / lanes, g = threadIdx.x / lanes, lane = threadIdx.x - g * lanes;
  extern __shared__ float red[];  // [groups][W]
  for (int c = pk.bid * groups + g; c < nchunks; c += pk.nblk * groups) {
    const int lo = c * chunk, hi = lo + chunk, end = hi < M ? hi : M;
    // the `groups` chunks of this workgroup; a segment that starts before and ends after them makes
    // every lane group see the same thing, so `merged` is uniform over the workgroup
    const int block_lo = (c - g) * chunk, block_hi = block_lo + groups * chunk;
    bool merged = false;
    // segment ids just outside the chunk and just outside the workgroup's range (-1 / -2: nothing there)
    const int s_before = lo > 0 ? seg_src[lo - 1] / seg_div : -1;
    const int s_after = hi < M ? seg_src[hi] / seg_div : -2;
    const int s_blk_before = block_lo > 0 ? seg_src[block_lo - 1] / seg_div : -1;
    const int s_blk_after = block_hi < M ? seg_src[block_hi] / seg_div : -2;
    // Where a finished run goes is decided from the segment ids next to the chunk and next to the
    // workgroup's range (ids are non-decreasing), not from the segment's offsets: those would be two
    // dependent loads at every segment change.  `at_end`: the run reaches the chunk's last position.
    // `active`: this lane holds columns of the vector (the flag `merged` is set by idle lanes too: it
    // decides a workgroup barrier).
    auto flush = [&](const Vec<VEC> &acc, int cur, int e, bool active, bool at_end) {
      const bool starts_in = cur != s_before;          // the segment begins inside the chunk
      const bool ends_in = !at_end || cur != s_after;  // ... and ends inside it
      if (starts_in && ends_in) {
        if (active) {
          float *dst = out + seg_out_index(cur, e, out_inner, nseg);
          if (fused) acc.store_sgd(dst, lr); else acc.store(dst);
        }
      } else if (cur == s_blk_before && cur == s_blk_after) {  // it covers the workgroup's whole range:
        if (active) acc.store(red + (size_t)g * W + e);       // one partial for the workgroup, summed below
        merged = true;
      } else if (active) acc.store(partial + ((size_t)c * 2 + (starts_in ? 1 : 0)) * W + e);
    };
    auto load_row = [&](int row, int e, Vec<VEC> &x) {
      if (stream_src) x.load_stream(src + (size_t)row * nsub * W + e);
      else x.load(src + (size_t)row * nsub * W + e);
      for (int t = 1; t < nsub; ++t) {
        Vec<VEC> y;
        y.load(src + ((size_t)row * nsub + t) * W + e);
        x.add(y);
      }
    };
    if (lanes >= TT_SEG_UNROLL) {
      // The lanes of the group fetch the segment ids and gather indices of `lanes` positions at once,
      // one position per lane, and hand them round with lane shuffles: one round trip for the indices
      // of a whole block of positions instead of one in front of every group of gathers.  (Every lane
      // runs every shuffle; positions past the chunk's end carry the id -3 and are skipped.)
      for (int e0 = 0; e0 < W; e0 += lanes * VEC) {
        const int e = e0 + lane * VEC;
        const bool active = e < W;
        Vec<VEC> acc;
        acc.zero();
        int cur = -1;
        for (int sub = lo; sub < hi; sub += lanes) {
          const int mine = sub + lane;
          int my_sg = -3, my_row = 0;
          if (mine < end) {
            my_sg = seg_src[mine] / seg_div;
            my_row = gidx ? gidx[mine] : mine;
          }
          const int cnt = (hi - sub) < lanes ? (hi - sub) : lanes;  // a multiple of TT_SEG_UNROLL
          for (int k = 0; k < cnt; k += TT_SEG_UNROLL) {
            int sg[TT_SEG_UNROLL];
            Vec<VEC> x[TT_SEG_UNROLL];
#pragma unroll
            for (int u = 0; u < TT_SEG_UNROLL; ++u) {
              sg[u] = __shfl(my_sg, k + u, lanes);
              const int row = __shfl(my_row, k + u, lanes);
              if (sg[u] != -3 && active) load_row(row, e, x[u]); else x[u].zero();
            }
#pragma unroll
            for (int u = 0; u < TT_SEG_UNROLL; ++u) {
              if (sg[u] == -3) continue;
              if (sg[u] != cur) {
                if (cur >= 0) flush(acc, cur, e, active, false);
                cur = sg[u];
                acc.zero();
              }
              acc.add(x[u]);
            }
          }
        }
        if (cur >= 0) flush(acc, cur, e, active, true);
      }
    } else {
      for (int e = lane * VEC; e < W; e += lanes * VEC) {
        Vec<VEC> acc;
        acc.zero();
        int cur = -1;
        for (int pos = lo; pos < end; ++pos) {
          const int sgk = seg_src[pos] / seg_div;
          Vec<VEC> x;
          load_row(gidx ? gidx[pos] : pos, e, x);
          if (sgk != cur) {
            if (cur >= 0) flush(acc, cur, e, true, false);
            cur = sgk;
            acc.zero();
          }
          acc.add(x);
        }
        if (cur >= 0) flush(acc, cur, e, true, true);
      }
    }
    if (merged) {  // uniform: the chunks' sums in chunk order -> slot 0 of the workgroup's first chunk
      __syncthreads();
      if (g == 0)
        for (int e = lane * VEC; e < W; e += lanes * VEC) {
          Vec<VEC> acc, x;
          acc.load(red + e);
          for (int k = 1; k < groups; ++k) {
            x.load(red + (size_t)k * W + e);
            acc.add(x);
          }
          acc.store(partial + ((size_t)(c - g) * 2) * W + e);
        }
      __syncthreads();
    }
  }
}

#ifndef TT_SEG2_UNROLL
#define TT_SEG2_UNROLL 8  // partials a lane group of stage 2 keeps in flight
#endif
// Stage 2.  The chunk in which a multi-chunk segment begins owns it and adds its own slot-1 partial and the
// slot-0 partials of the following chunks, in chunk order.  What a workgroup costs is its chain of dependent loads
// (segment id, segment range, partials), whatever it adds.
//   Workgroup per chunk: the shortest chain, as long as the chip holds them in about two rounds.
//   Lane group per chunk (SPREAD, and the kind's `spread`): most owners add two vectors, which a lane group does by itself, so
// that many chunks are through in one round.  Segments of many partials are left to all lane groups of the workgroup; those
// are the hot rows, neighbours in sorted order where ids are not permuted, so the chunks of a workgroup lie a grid
// apart and no workgroup gets many of them.  A kernel of its own: it needs more registers (72 against 46) and a list in LDS.
// Stage 2 of the gradient merge at D = 128, per chunk / spread: 1125 chunks 5.0 / 6.6 us, 4600 8.3 / 9.8, 8192 10.1 / 8.4,
// 10500 13.1 / 11.1, 12800 15.3 / 11.0; the sums are the same bit for bit.
// With `dense`, workgroup (lane group) c also zero-fills segment c if it is empty.
// LDS: red[groups][W], with SPREAD | SegUnits long[groups] | count
#ifndef TT_SEG2_SPREAD_CHUNKS
#define TT_SEG2_SPREAD_CHUNKS 6144  // chunks above which a lane group takes one
#endif
// Partials to add for the segment that chunk c owns: slot 0 of the chunks c+1 .. c1, except that stage 1
// has left ONE partial (in the first chunk) for every run of `groups` chunks handled by one workgroup
// that lies strictly inside the segment: the runs B0 .. B1.  Units in order: single chunks before the
// runs, one per run, single chunks after.
struct SegUnits {
  int seg, c, B0, B1, nh, nm, n;  // n of them
  __device__ __forceinline__ int chunk_of(int u, int groups) const {
    return u < nh ? c + 1 + u : (u < nh + nm ? (B0 + (u - nh)) * groups : (B1 + 1) * groups + (u - nh - nm));
  }
};
static size_t seg2_lds_bytes(int groups, int W, bool spread) {
  return sizeof(float) * (size_t)groups * W + (spread ? sizeof(SegUnits) * (size_t)groups + sizeof(int) : 0);
}
template <bool BATCHED, int VEC, bool SPREAD>
__global__ void __launch_bounds__(TT_BLOCK)
k_seg_stage2(TTArg<BATCHED> arg, SegLaunch L, int lanes) {
  const SegPick pk = seg_pick(L, arg.get());
  const int chunk = pk.chunk;
  const SegView sv = seg_view(arg.get(), pk.kind);
  const int W = sv.W, seg_div = sv.seg_div, out_inner = sv.out_inner, nseg = sv.nseg, dense = sv.dense;
  const int32_t *__restrict__ seg_src = sv.seg_src, *__restrict__ seg_off = sv.seg_off;
  float *__restrict__ out = sv.out;
  const float *__restrict__ partial = sv.partial + pk.poff;
  extern __shared__ float red[];
  const int M = *sv.count_ptr;
  const int nchunks = (M + chunk - 1) / chunk;
  const int groups = blockDim.x / lanes, g = threadIdx.x / lanes, lane = threadIdx.x - g * lanes;
  const int gc = groups * chunk;
  const bool spread = SPREAD && pk.spread;
  const int mine = pk.bid + (spread ? g * pk.nblk : 0);
  if (dense && (spread || g == 0) && mine < nseg && seg_off[mine] == seg_off[mine + 1]) {
    Vec<VEC> z;
    z.zero();
    for (int e = lane * VEC; e < W; e += lanes * VEC)
      z.store(out + seg_out_index(mine, e, out_inner, nseg));
  }
  // Whether a segment starts in chunk c and runs past it, at positions a .. b (most chunks have none, and counting its partials divides).
  auto owns = [&](int c, SegUnits &k, int &a, int &b) __attribute__((always_inline)) {
    const int lo = c * chunk, hi = lo + chunk, end = hi < M ? hi : M;
    k.c = c;
    k.seg = seg_src[end - 1] / seg_div;
    a = seg_off[k.seg]; b = seg_off[k.seg + 1];
    return a >= lo && b > hi;
  };
  auto count = [&](SegUnits &k, int a, int b) __attribute__((always_inline)) {
    const int c1 = (b - 1) / chunk;
    k.B0 = a / gc + 1; k.B1 = (b + gc - 1) / gc - 2;
    k.nh = c1 - k.c; k.nm = 0;
    int nt = 0;
    if (k.B0 <= k.B1) {
      k.nh = k.B0 * groups - (k.c + 1);
      k.nm = k.B1 - k.B0 + 1;
      nt = c1 - (k.B1 + 1) * groups + 1;
    }
    k.n = k.nh + k.nm + nt;
  };
  auto finish = [&](const Vec<VEC> &acc, int s, int e) __attribute__((always_inline)) {
    float *dst = out + seg_out_index(s, e, out_inner, nseg);
    if (sv.fused) acc.store_sgd(dst, sv.lr); else acc.store(dst);
  };
  // One segment by all lane groups: they take the units round-robin, their sums are added in group order.
  auto fold = [&](const SegUnits &k) __attribute__((always_inline)) {
    for (int e = lane * VEC; e < W; e += lanes * VEC) {
      Vec<VEC> acc;
      acc.zero();
      int u = g;
      for (; u + (TT_SEG2_UNROLL - 1) * groups < k.n; u += TT_SEG2_UNROLL * groups) {
        Vec<VEC> x[TT_SEG2_UNROLL];  // independent loads in flight, added in unit order
#pragma unroll
        for (int j = 0; j < TT_SEG2_UNROLL; ++j) x[j].load(partial + ((size_t)k.chunk_of(u + j * groups, groups) * 2) * W + e);
#pragma unroll
        for (int j = 0; j < TT_SEG2_UNROLL; ++j) acc.add(x[j]);
      }
      for (; u < k.n; u += groups) {
        Vec<VEC> x;
        x.load(partial + ((size_t)k.chunk_of(u, groups) * 2) * W + e);
        acc.add(x);
      }
      acc.store(red + (size_t)g * W + e);
    }
    __syncthreads();
    if (g == 0) {
      for (int e = lane * VEC; e < W; e += lanes * VEC) {
        Vec<VEC> acc, x;
        acc.load(partial + ((size_t)k.c * 2 + 1) * W + e);
        for (int j = 0; j < groups; ++j) {
          x.load(red + (size_t)j * W + e);
          acc.add(x);
        }
        finish(acc, k.seg, e);
      }
    }
  };
  if (!spread) {  // uniform
    if (mine >= nchunks) return;
    SegUnits k;
    int a, b;
    if (!owns(mine, k, a, b)) return;
    count(k, a, b);
    fold(k);
    return;
  }
  if constexpr (SPREAD) {
    SegUnits *longs = reinterpret_cast<SegUnits *>(red + (size_t)groups * W);  // segments left to the whole workgroup
    int *nlongs = reinterpret_cast<int *>(longs + groups);
    if (threadIdx.x == 0) *nlongs = 0;
    __syncthreads();
    SegUnits k;
    int a, b;
    if (mine < nchunks && owns(mine, k, a, b)) {
      count(k, a, b);
      if (k.n > TT_SEG2_UNROLL || k.n > groups) {
        if (lane == 0) longs[atomicAdd(nlongs, 1)] = k;  // (segments are independent: their order does not matter)
      } else {
        for (int e = lane * VEC; e < W; e += lanes * VEC) {
          Vec<VEC> acc, x[TT_SEG2_UNROLL];
          acc.load(partial + ((size_t)mine * 2 + 1) * W + e);
#pragma unroll
          for (int u = 0; u < TT_SEG2_UNROLL; ++u)
            if (u < k.n) x[u].load(partial + ((size_t)k.chunk_of(u, groups) * 2) * W + e);
#pragma unroll
          for (int u = 0; u < TT_SEG2_UNROLL; ++u)
            if (u < k.n) acc.add(x[u]);
          finish(acc, k.seg, e);
        }
      }
    }
    __syncthreads();
    const int n = *nlongs;
    for (int i = 0; i < n; ++i) {  // uniform
      fold(longs[i]);
      __syncthreads();
    }
  }
}

// Stage-1 chunk length for `count` positions.  Short chunks give stage 1 more lane groups to hide
// the gather latency with (65 k positions: 8 beats 32 by 2x); long chunks leave stage 2 fewer
// partials to fold for the hottest segment (335 k positions with one segment of 60 k: 32 beats 8).
static int seg_chunk_for(long long count) {
  int c = TT_SEG_MIN_CHUNK;
  while (c < TT_SEG_MAX_CHUNK && (long long)c * 2 * 8192 <= count) c *= 2;
  return c;
}

// Launch shape of one segmented sum over every table of the batch (chunk <= 0: chosen from the count).
struct SegParams { int W, vec, lanes, groups, chunk, nchunks, blocks1, spread; long long blocks2; };
static SegParams seg_params(const TTBatch &b, int kind, int chunk) {
  const TTShape &sh = b.host[0].sh;
  SegParams p;
  p.W = kind == SEG_GAGG ? sh.D : (kind == SEG_DG3 ? sh.S3 : sh.S1);
  const int out_inner = kind == SEG_DG3 ? sh.d3 : p.W;
  bool vec4 = (p.W % 4) == 0 && (out_inner % 4) == 0;
  long long max_count = 0, max_seg = 0;
  for (int t = 0; t < b.T; ++t) {
    const TTDev &d = b.host[t];
    const float *src = kind == SEG_GAGG ? d.grad_out : (kind == SEG_DG3 ? d.plan.t3buf : d.plan.t1buf);
    // the buffer the final stores go to: with the fused update, the core itself
    const float *out = kind == SEG_GAGG ? d.plan.gagg
                                        : (kind == SEG_DG3 ? (d.fused ? d.g[2] : d.dg[2]) : (d.fused ? d.g[0] : d.dg[0]));
    vec4 = vec4 && ((uintptr_t)src % 16) == 0 && ((uintptr_t)out % 16) == 0;
    const long long cnt = kind == SEG_GAGG ? d.nnz : (kind == SEG_DG3 ? d.plan.max_rows : d.plan.max_prefixes);
    const long long nseg = (kind == SEG_GAGG || d.fused) ? 0 : (kind == SEG_DG3 ? d.sh.n3 : d.sh.n1);
    if (cnt > max_count) max_count = cnt;
    if (nseg > max_seg) max_seg = nseg;
  }
  p.chunk = chunk > 0 ? chunk : seg_chunk_for(max_count);
  p.vec = vec4 ? 4 : 1;
  p.lanes = 1;
  while (p.lanes < TT_WAVE && p.lanes * p.vec < p.W) p.lanes <<= 1;
  p.groups = TT_BLOCK / p.lanes;
  p.nchunks = tt_ceil_div(max_count, p.chunk);
  p.blocks1 = tt_ceil_div(p.nchunks, p.groups);
  if (p.blocks1 > 8192) p.blocks1 = 8192;
  p.blocks2 = p.nchunks > max_seg ? p.nchunks : max_seg;  // dense kinds also zero-fill empty segments
  // (the sums of the widest core-0 slices take 64 KB of LDS by themselves, the most that any kernel here asks for)
  p.spread = p.nchunks > TT_SEG2_SPREAD_CHUNKS && seg2_lds_bytes(p.groups, p.W, true) <= 65536;
  if (p.spread) p.blocks2 = tt_ceil_div(p.blocks2, p.groups);
  return p;
}

// One segmented sum, or (kind_b >= 0) two of the same launch shape in the same two launches.
static tt_status seg_launch(const TTBatch &b, const SegParams &pa, int kind, const SegParams *pb, int kind_b,
                            int prof_kernel, hipStream_t s) {
  TTProfScope prof(&b.host[0].plan, prof_kernel, s);  // both stages
  const size_t lds = sizeof(float) * (size_t)pa.groups * pa.W;
  SegLaunch L1 = {kind, pa.chunk, pa.blocks1, pb ? kind_b : -1, pb ? pb->chunk : 0, pa.spread, pb ? pb->spread : 0};
  const long long g1 = pa.blocks1 + (pb ? pb->blocks1 : 0);
  if (g1 > 0) {
    if (pa.vec == 4) TT_LAUNCH_T(k_seg_stage1, 4, g1, TT_BLOCK, lds, s, b, L1, pa.lanes);
    else TT_LAUNCH_T(k_seg_stage1, 1, g1, TT_BLOCK, lds, s, b, L1, pa.lanes);
  }
  SegLaunch L2 = L1;
  L2.blocks = (int)pa.blocks2;
  const long long g2 = pa.blocks2 + (pb ? pb->blocks2 : 0);
  if (g2 > 0) {
    const bool spread = L2.spread || L2.spread_b;
    const size_t lds2 = seg2_lds_bytes(pa.groups, pa.W, spread);
    if (pa.vec == 4 && spread) TT_LAUNCH_T2(k_seg_stage2, 4, true, g2, TT_BLOCK, lds2, s, b, L2, pa.lanes);
    else if (pa.vec == 4) TT_LAUNCH_T2(k_seg_stage2, 4, false, g2, TT_BLOCK, lds2, s, b, L2, pa.lanes);
    else if (spread) TT_LAUNCH_T2(k_seg_stage2, 1, true, g2, TT_BLOCK, lds2, s, b, L2, pa.lanes);
    else TT_LAUNCH_T2(k_seg_stage2, 1, false, g2, TT_BLOCK, lds2, s, b, L2, pa.lanes);
  }
  return tt_launch_status();
}

tt_status seg_sum(const TTBatch &b, int kind, int chunk, int prof_kernel, hipStream_t s) {
  const SegParams p = seg_params(b, kind, chunk);
  return seg_launch(b, p, kind, nullptr, -1, prof_kernel, s);
}

#ifndef TT_SEG_WHOLE_UNROLL
#define TT_SEG_WHOLE_UNROLL TT_SEG_UNROLL  // gathers a lane group of the whole-segment kernel keeps in flight
#endif
// Whole segments: ONE launch for the core-2 and the core-0 reduction.  The first nseg_a * parts_a
// workgroups serve core 2 (rows that share i3: the index split spreads them evenly), the rest core 0,
// `parts` workgroups per segment, each summing its own range of the vector's columns.  Cutting by
// columns gives a long segment more lane groups -- more gathers in flight -- without a second stage:
// a table with few i3 values has few, long core-2 segments, and under a skewed access distribution the
// distinct prefixes pile up under the first few i1 (up to n2 prefixes times the strips each).
// The lane groups of a workgroup take the segment's positions round-robin, TT_SEG_UNROLL gathers in
// flight each, and their sums are added in group order through LDS, so the result does not depend on
// timing.  (The lookups of one hot row can be a fifth of a batch, which is why the gradient merge
// keeps the two-stage sum.)  A long segment is summed by its workgroups alone: correct, only slow.
#ifndef TT_SEG_WHOLE_PARTS
#define TT_SEG_WHOLE_PARTS 8  // column parts of a core-0 segment
#endif
// Column parts per segment and lanes per part.  Core 0: as many parts (at most TT_SEG_WHOLE_PARTS) as leave a
// part 8 lanes wide; core 2 only as many as bring its workgroups to about two per compute unit.  A table's
// own numbers decide, so its sums are the same alone and in a batch.
struct WholeSplit { int parts, lanes; };
__host__ __device__ __forceinline__ WholeSplit whole_split(int W, int vec, int want) {
  WholeSplit w = {1, 1};
  while (w.parts * 2 <= want && w.parts * 2 <= TT_SEG_WHOLE_PARTS && W % (w.parts * 2 * vec) == 0 &&
         W / (w.parts * 2 * vec) >= 8)
    w.parts *= 2;
  while (w.lanes < TT_WAVE && w.lanes * vec < W / w.parts) w.lanes <<= 1;
  return w;
}
__host__ __device__ __forceinline__ int whole_want3(int n3) { return (512 + n3 - 1) / n3; }

// Whether a table's positions go in rounds (below): up to two strips a prefix, and segments that fill a round.  What a round sets up
// costs a short segment more than it saves.  Launches, one position after the other / rounds, distinct rows by i3 (at most) in
// brackets: ranks 32 4.4 / 5.1 us (22), 4.5 / 5.2 (43), 6.6 / 5.9 (47), 6.1 / 5.1 (87), 342 i3 7.2 / 8.0 (23), 8.5 / 8.2 (47);
// one strip, ranks 12 and 20 4.6 / 4.9 (8), 5.0 / 5.3 (16), 5.6 / 4.8 (33), ranks 16 and 4 3.9 / 4.4 (8), 4.7 / 4.7 (30), 6.1 / 5.2 (61).
// Skewed lookups have fewer rows than the capacity that the rule knows: up to 0.8 us lost above the limits, 1 to 9 won from twice them on.
#ifndef TT_SEG_ROUNDS_MIN_1
#define TT_SEG_ROUNDS_MIN_1 32  // positions per segment by capacity: one strip a prefix
#endif
#ifndef TT_SEG_ROUNDS_MIN_2
#define TT_SEG_ROUNDS_MIN_2 45  // ... two
#endif
__host__ __device__ __forceinline__ bool seg_whole_rounds(const TTDev &d) {
  const long long least = d.strips == 1 ? TT_SEG_ROUNDS_MIN_1 : TT_SEG_ROUNDS_MIN_2;
  return d.strips <= 2 && (d.plan.max_rows >= least * d.sh.n3 || d.plan.max_prefixes >= least * d.sh.n1);
}
template <bool BATCHED, int VEC, bool ROUNDS>
__global__ void __launch_bounds__(TT_BLOCK)
k_seg_whole(TTArg<BATCHED> arg, int blocks_a) {
  const TTDev &d = arg.get();
  if (BATCHED && seg_whole_rounds(d) != ROUNDS) return;  // uniform: the other launch serves this table
  const bool second = (int)blockIdx.x >= blocks_a;
  const SegView sv = seg_view(d, second ? SEG_DG1 : SEG_DG3);
  const WholeSplit split = whole_split(sv.W, VEC, second ? TT_SEG_WHOLE_PARTS : whole_want3(d.sh.n3));
  const int parts = split.parts, lanes = split.lanes;
  const int wg = second ? (int)blockIdx.x - blocks_a : (int)blockIdx.x;
  const int s = wg / parts, part = wg - s * parts;
  if (s >= sv.nseg) return;  // uniform: a table of the batch with fewer segments
  const int W = sv.W, nsub = sv.nsub, out_inner = sv.out_inner, nseg = sv.nseg;
  const int Wp = W / parts, e0 = part * Wp;  // this workgroup's columns
  const int32_t *__restrict__ gidx = sv.gidx, *__restrict__ seg_off = sv.seg_off;
  const float *__restrict__ src = sv.src;
  float *__restrict__ out = sv.out;
  const int groups = blockDim.x / lanes, g = threadIdx.x / lanes, lane = threadIdx.x - g * lanes;
  extern __shared__ float red[];  // [groups][Wp]
  const int a = seg_off[s], b = seg_off[s + 1];
  if (a == b) {  // uniform: an empty segment (a slice no lookup touched)
    if (sv.dense && g == 0) {
      Vec<VEC> z;
      z.zero();
      for (int e = lane * VEC; e < Wp; e += lanes * VEC) z.store(out + seg_out_index(s, e0 + e, out_inner, nseg));
    }
    return;
  }
  // Sum of this lane group's positions, columns e ..., NS vectors a position.  A round is a chain of two loads (gather index,
  // vector): the next round's indices are requested with this round's vectors, and the positions left over at the end are one
  // round, not one each.  Whole launches, one left-over position after the other / this: multi-hot at ranks 32 (two strips)
  // 12.5 / 9.4 us, ranks 12 and 20 6.8 / 5.9.
  auto positions = [&](auto ns, int e, Vec<VEC> &acc) {
    constexpr int NS = decltype(ns)::value, U = TT_SEG_WHOLE_UNROLL;
    int row[U];  // -1: past the end
    auto rows_at = [&](int pos) {
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int p = pos + k * groups;
        row[k] = p >= b ? -1 : (gidx ? gidx[p] : p);
      }
    };
    rows_at(a + g);
    for (int pos = a + g; pos < b; pos += U * groups) {
      Vec<VEC> x[U][NS];
#pragma unroll
      for (int k = 0; k < U; ++k) {
#pragma unroll
        for (int t = 0; t < NS; ++t) {
          x[k][t].zero();
          if (row[k] >= 0) x[k][t].load_stream(src + ((size_t)row[k] * NS + t) * W + e0 + e);  // hand-off buffers: read once
        }
      }
      rows_at(pos + U * groups);
#pragma unroll
      for (int k = 0; k < U; ++k)
#pragma unroll
        for (int t = 1; t < NS; ++t) x[k][0].add(x[k][t]);
      // in pairs, then into the running sum: a chain of a quarter of the additions, and of their rounding errors
#pragma unroll
      for (int w = 1; w < U; w <<= 1)
#pragma unroll
        for (int k = 0; k < U; k += 2 * w) x[k][0].add(x[k + w][0]);
      acc.add(x[0][0]);
    }
  };
  // One position after the other.  Four strips a position (ranks 64): sixteen vectors in flight halve the wavefronts a compute unit
  // holds, which costs the many short segments of fused tables more than it gives (nine tables at batch 4096 19.5 us a launch, 25 in rounds
  // of sixteen, 22 in rounds of eight; one table 18.2, 17.6 and 18.8).
  auto load_pos = [&](int pos, int e, Vec<VEC> &x) {
    const int row = gidx ? gidx[pos] : pos;
    x.load_stream(src + (size_t)row * nsub * W + e0 + e);  // hand-off buffers: every vector is read once
    for (int t = 1; t < nsub; ++t) {
      Vec<VEC> y;
      y.load_stream(src + ((size_t)row * nsub + t) * W + e0 + e);
      x.add(y);
    }
  };
  for (int e = lane * VEC; e < Wp; e += lanes * VEC) {
    Vec<VEC> acc;
    acc.zero();
    if constexpr (ROUNDS) {
      if (nsub == 1) positions(std::integral_constant<int, 1>{}, e, acc);  // uniform
      else positions(std::integral_constant<int, 2>{}, e, acc);
    } else {
      int pos = a + g;
      for (; pos + (TT_SEG_WHOLE_UNROLL - 1) * groups < b; pos += TT_SEG_WHOLE_UNROLL * groups) {
        Vec<VEC> x[TT_SEG_WHOLE_UNROLL];
#pragma unroll
        for (int k = 0; k < TT_SEG_WHOLE_UNROLL; ++k) load_pos(pos + k * groups, e, x[k]);
#pragma unroll
        for (int w = 1; w < TT_SEG_WHOLE_UNROLL; w <<= 1)
#pragma unroll
          for (int k = 0; k < TT_SEG_WHOLE_UNROLL; k += 2 * w) x[k].add(x[k + w]);
        acc.add(x[0]);
      }
      for (; pos < b; pos += groups) {
        Vec<VEC> x;
        load_pos(pos, e, x);
        acc.add(x);
      }
    }
    acc.store(red + (size_t)g * Wp + e);
  }
  __syncthreads();
  if (g == 0)
    for (int e = lane * VEC; e < Wp; e += lanes * VEC) {
      // the groups (a power of two of them, four or more), four in pairs and then into the running sum
      Vec<VEC> acc, x[4];
      acc.zero();
      for (int k = 0; k < groups; k += 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j].load(red + (size_t)(k + j) * Wp + e);
        x[0].add(x[1]);
        x[2].add(x[3]);
        x[0].add(x[2]);
        acc.add(x[0]);
      }
      float *dst = out + seg_out_index(s, e0 + e, out_inner, nseg);
      if (sv.fused) acc.store_sgd(dst, sv.lr); else acc.store(dst);
    }
}

#ifndef TT_SEG_WHOLE_MAX_AVG
#define TT_SEG_WHOLE_MAX_AVG 4096  // positions per segment (capacity / segments) up to which whole segments are used
#endif
// ... where the two sums' vectors differ in width: both then go four bytes a lane, and long segments cost more than the
// launches they save.  Whole backward calls, whole segments / two-stage sums, d = 2x4x6, ranks 12, 20.  Every lookup a row of
// its own: 4 i3, rows per i3 500 43.0 / 50.8 us, 1000 61.6 / 56.1, 4000 171 / 108; 30 i3, 1000 0.99 of the two-stage time, 2500
// 1.14; prefixes per i1 1000 49.1 / 57.0, 2000 78.1 / 78.4, 3000 98.8 / 90.0.  Skewed lookups (Zipf exponents 1.05 and 1.2, near-
// cubic tables of 8 k to 1 M rows) have two to five times fewer rows than the capacity that the rule knows: 938 to 2500 per i3
// by capacity are 210 to 620, 50.5 / 62.5 to 119 / 129 us.
static long long seg_mixed_max_rows(int n3) { return n3 < 16 ? 1024 : 3072; }  // rows per i3
#define TT_SEG_MIXED_MAX_PREFS 2048  // prefixes per i1
// ... and where the slices are many: empty ones cost a workgroup per column part (four bytes a lane make many parts).  500
// lookups, d = 4x2x3, ranks 16, 5: 1000 i1 (8000 workgroups) 44.4 / 46.2, 1500 50.9 / 46.8, 100000 1200 / 102; d = 2x4x6,
// ranks 12, 20: 5000 i1 (10000) 40.0 / 46.9, 10000 51.3 / 49.4.
#define TT_SEG_MIXED_MAX_WGS 8192

// The core-2 and core-0 reductions are independent.  With segments of moderate length they take one
// launch of whole-segment workgroups; otherwise the two-stage sum, sharing its launches when their
// vectors have the same width (the smaller one would otherwise pay two launches for a few workgroups).
tt_status seg_sum_dg3_dg1(const TTBatch &b, hipStream_t s) {
  const SegParams p3 = seg_params(b, SEG_DG3, 0), p1 = seg_params(b, SEG_DG1, 0);
  bool whole = true;
  const bool mixed = p3.vec != p1.vec;
  for (int t = 0; t < b.T && whole; ++t) {
    const TTDev &d = b.host[t];
    whole = d.plan.max_rows / d.sh.n3 <= (mixed ? seg_mixed_max_rows(d.sh.n3) : TT_SEG_WHOLE_MAX_AVG) &&
            d.plan.max_prefixes * d.strips / d.sh.n1 <= (mixed ? TT_SEG_MIXED_MAX_PREFS : TT_SEG_WHOLE_MAX_AVG);
  }
  if (whole) {
    // one launch has one vector width (d3 = 6 beside ranks of four, 12 k lookups: 26 us in the four launches of
    // two separate two-stage sums, 7 us here)
    const int vec = mixed ? 1 : p3.vec, W3 = p3.W;
    const WholeSplit w1 = whole_split(p1.W, vec, TT_SEG_WHOLE_PARTS);
    const long long blocks3 = tt_batch_max(b, [=](const TTDev &d) {
      return (long long)d.sh.n3 * whole_split(W3, vec, whole_want3(d.sh.n3)).parts; });
    const long long blocks1 = tt_batch_max(b, [](const TTDev &d) { return (long long)d.sh.n1; }) * w1.parts;
    // floats of LDS: one part's sums per lane group
    const long long lds3 = tt_batch_max(b, [=](const TTDev &d) {
      const WholeSplit w = whole_split(W3, vec, whole_want3(d.sh.n3));
      return (long long)(TT_BLOCK / w.lanes) * (W3 / w.parts); });
    const long long lds1 = (long long)(TT_BLOCK / w1.lanes) * (p1.W / w1.parts);
    const size_t lds = sizeof(float) * (size_t)(lds3 > lds1 ? lds3 : lds1);
    const long long grid = blocks3 + blocks1;
    if (grid <= (mixed ? TT_SEG_MIXED_MAX_WGS : TT_MAX_WORKGROUPS)) {  // (millions of slices: the two-stage sum's workgroups follow the lookups)
      bool rounds = false, single = false;  // (a batch: a launch each that its tables take)
      for (int t = 0; t < b.T; ++t) (seg_whole_rounds(b.host[t]) ? rounds : single) = true;
      if (rounds) {
        if (vec == 4) TT_LAUNCH_T2(k_seg_whole, 4, true, grid, TT_BLOCK, lds, s, b, (int)blocks3);
        else TT_LAUNCH_T2(k_seg_whole, 1, true, grid, TT_BLOCK, lds, s, b, (int)blocks3);
      }
      if (single) {
        if (vec == 4) TT_LAUNCH_T2(k_seg_whole, 4, false, grid, TT_BLOCK, lds, s, b, (int)blocks3);
        else TT_LAUNCH_T2(k_seg_whole, 1, false, grid, TT_BLOCK, lds, s, b, (int)blocks3);
      }
      return tt_launch_status();
    }
  }
  if (p3.W == p1.W && p3.vec == p1.vec && p3.lanes == p1.lanes && p3.blocks1 > 0 && p1.blocks1 > 0)
    return seg_launch(b, p3, SEG_DG3, &p1, SEG_DG1, -1, s);
  tt_status st = seg_launch(b, p3, SEG_DG3, nullptr, -1, -1, s);
  if (st != TT_OK) return st;
  return seg_launch(b, p1, SEG_DG1, nullptr, -1, -1, s);
}

// ------------------------------------------------------------------ per-prefix contractions
// Workgroup per distinct prefix q.
// LDS (floats): g1s[S1] | p12[d1*d2*R2p] | hs[P] | gs[D] | g3s[S3]
template <bool BATCHED>
__global__ void __launch_bounds__(TT_BLOCK)
k_bwd_prefix(TTArg<BATCHED> a) {
  const TTDev &d = a.get();
  const TTShape &sh = d.sh;
  const float *__restrict__ g1 = d.g[0], *__restrict__ g2 = d.g[1], *__restrict__ g3 = d.g[2];
  const int32_t *__restrict__ counts = d.plan.counts, *__restrict__ uniq_pref = d.plan.uniq_pref,
                *__restrict__ pref_seg = d.plan.pref_seg, *__restrict__ uniq_row = d.plan.uniq_row;
  const float *__restrict__ gagg = d.plan.gagg;
  float *__restrict__ t3buf = d.plan.t3buf, *__restrict__ hbuf = d.plan.hbuf,
        *__restrict__ t1buf = d.plan.t1buf;
  extern __shared__ float lds[];
  float *g1s = lds, *p12 = g1s + sh.S1, *hs = p12 + sh.d1 * sh.d2 * sh.R2p, *gs = hs + sh.P,
        *g3s = gs + sh.D;
  const int up = counts[1];
  const int lane = threadIdx.x & (TT_WAVE - 1), wave = threadIdx.x / TT_WAVE;
  for (int q = blockIdx.x; q < up; q += gridDim.x) {
    const int p = uniq_pref[q], i1 = p / sh.n2, i2 = p - i1 * sh.n2;
    for (int e = threadIdx.x; e < sh.S1; e += blockDim.x) g1s[e] = g1[(size_t)i1 * sh.S1 + e];
    for (int o = threadIdx.x; o < sh.P; o += blockDim.x) hs[o] = 0.f;
    __syncthreads();
    // P12[j1][j2][r2] = sum_r1 G1[i1][j1][r1] G2[r1][i2][j2][r2]
    for (int o = threadIdx.x; o < sh.P; o += blockDim.x) {
      const int j1 = o / sh.S2, c = o - j1 * sh.S2;
      const float *col = g2 + (size_t)i2 * sh.S2 + c;
      float acc = 0.f;
      for (int r1 = 0; r1 < sh.R1; ++r1)
        acc = fmaf(g1s[j1 * sh.R1 + r1], col[(size_t)r1 * sh.n2 * sh.S2], acc);
      p12[(j1 * sh.d2 + c / sh.R2) * sh.R2p + c % sh.R2] = acc;
    }
    const int u0 = pref_seg[q], u1 = pref_seg[q + 1];
    for (int u = u0; u < u1; ++u) {
      const int i3 = uniq_row[u] % sh.n3;
      __syncthreads();  // previous row's readers are done; p12 / hs initialisation is visible
      for (int e = threadIdx.x; e < sh.D; e += blockDim.x) gs[e] = gagg[(size_t)u * sh.D + e];
      for (int e = threadIdx.x; e < sh.S3; e += blockDim.x) {
        const int r2 = e / sh.d3, j3 = e - r2 * sh.d3;
        g3s[e] = g3[((size_t)r2 * sh.n3 + i3) * sh.d3 + j3];
      }
      __syncthreads();
      // core-2 contribution of this row: T3[r2][j3] = sum_{j1,j2} P12[j1][j2][r2] g[j1][j2][j3]
      for (int o = threadIdx.x; o < sh.S3; o += blockDim.x) {
        const int r2 = o / sh.d3, j3 = o - r2 * sh.d3;
        float acc = 0.f;
        for (int jj = 0; jj < sh.d1 * sh.d2; ++jj)
          acc = fmaf(p12[jj * sh.R2p + r2], gs[jj * sh.d3 + j3], acc);
        t3buf[(size_t)u * sh.S3 + o] = acc;
      }
      // right partial: H[j1][j2][r2] += sum_j3 g[j1][j2][j3] G3[r2][i3][j3]
      for (int o = threadIdx.x; o < sh.P; o += blockDim.x) {
        const int jj = o / sh.R2, r2 = o - jj * sh.R2;
        float acc = 0.f;
        for (int j3 = 0; j3 < sh.d3; ++j3) acc = fmaf(gs[jj * sh.d3 + j3], g3s[r2 * sh.d3 + j3], acc);
        hs[o] += acc;
      }
    }
    __syncthreads();
    for (int o = threadIdx.x; o < sh.P; o += blockDim.x) hbuf[(size_t)q * sh.P + o] = hs[o];
    // core-0 contribution: T1[j1][r1] = sum_{j2,r2} H[j1][j2][r2] G2[r1][i2][j2][r2]
    // one wavefront per r1: coalesced read of the G2 row, shuffle reduction over (j2,r2)
    for (int r1 = wave; r1 < sh.R1; r1 += blockDim.x / TT_WAVE) {
      const float *rowp = g2 + ((size_t)r1 * sh.n2 + i2) * sh.S2;
      for (int j1 = 0; j1 < sh.d1; ++j1) {
        float part = 0.f;
        for (int c = lane; c < sh.S2; c += TT_WAVE) part = fmaf(hs[j1 * sh.S2 + c], rowp[c], part);
        part = tt_wave_sum(part);
        if (lane == 0) t1buf[(size_t)q * sh.S1 + j1 * sh.R1 + r1] = part;
      }
    }
    __syncthreads();
  }
}

// The same for shapes whose operands are small: one WAVEFRONT per distinct prefix, four per workgroup, no
// barrier on the way; a prefix with more than PW_SOLO_ROWS distinct rows is worked on by all four.
// The work per prefix is a chain of five dependent round trips around a few hundred LDS reads, so what
// counts is how many chains are in flight (sixteen to twenty wavefronts per compute unit) and the number
// of LDS instructions: the core-1 slice is read from memory once (product and T1), j1 and rows come in
// groups of four per 16-byte read, and T1 is a lane (or two, or four) per element, where a wavefront
// reduction per element (six dependent lane exchanges for each of d1*R1 values) was most of the time.
// LDS per wavefront (floats): g1s[R1][j1, padded to fours] | gs[D][4 rows] | g3s[S3][4 rows] | p12[d1*d2*R2p] |
// hs[P] | g2s[R1][S2|1], rounded up to fours
constexpr int PW_WAVES = 4, PW_ROWS = 4, PW_SOLO_ROWS = 16;
struct PrefixWaveLds {
  int gs, g3s, p12, hs, g2s, floats, d1p;
  __host__ __device__ __forceinline__ explicit PrefixWaveLds(const TTShape &sh) {
    d1p = (sh.d1 + 3) & ~3;
    gs = sh.R1 * d1p;
    g3s = gs + PW_ROWS * sh.D;
    p12 = g3s + PW_ROWS * sh.S3;
    hs = p12 + sh.d1 * sh.d2 * sh.R2p;
    g2s = hs + sh.P;
    floats = (g2s + sh.R1 * (sh.S2 | 1) + 3) & ~3;
  }
};
// The rule: four wavefronts' operands fit the 64 KB of LDS a launch gets without asking.  Larger shapes have
// enough work per prefix for a workgroup.  Not how many prefixes there are: a few hundred of one row each are done sooner
// by a workgroup each (whole backward calls, wavefront / workgroup, ranks 12, 20: 64 prefixes 25.0 / 22.0 us, 1536 30.3 / 29.7,
// 2048 33.1 / 37.6; rank 4: 64 24.0 / 21.3, 2048 29.6 / 31.7), but skewed batches have few prefixes with many rows, which a
// workgroup takes one after the other, and the host knows lookups only (Zipf exponent 1.1, passes with reorder, forward and
// update: 363 lookups at rank 8, d = 2x2x4 65.9 / 82.3; 2736, d = 3x5x4 110.7 / 133.1).
static inline bool prefix_wave_fits(const TTShape &sh) {
  return PW_WAVES * (PrefixWaveLds(sh).floats + 1) * (long long)sizeof(float) <= 65536;
}

template <bool BATCHED>
__global__ void __launch_bounds__(TT_WAVE * PW_WAVES)
k_bwd_prefix_wave(TTArg<BATCHED> a) {
  const TTDev &d = a.get();
  const TTShape &sh = d.sh;
  const float *__restrict__ g1 = d.g[0], *__restrict__ g2 = d.g[1], *__restrict__ g3 = d.g[2];
  const int32_t *__restrict__ counts = d.plan.counts, *__restrict__ uniq_pref = d.plan.uniq_pref,
                *__restrict__ pref_seg = d.plan.pref_seg, *__restrict__ uniq_row = d.plan.uniq_row;
  const float *__restrict__ gagg = d.plan.gagg;
  float *__restrict__ t3buf = d.plan.t3buf, *__restrict__ hbuf = d.plan.hbuf, *__restrict__ t1buf = d.plan.t1buf;
  extern __shared__ float lds[];
  __shared__ __align__(16) int s_rows[PW_WAVES];
  const int lane = threadIdx.x & (TT_WAVE - 1), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / TT_WAVE);
  const PrefixWaveLds L(sh);
  float *g1s = lds + wave * L.floats, *gs = g1s + L.gs, *g3s = g1s + L.g3s, *p12 = g1s + L.p12, *hs = g1s + L.hs,
        *g2s = g1s + L.g2s;
  const int up = counts[1], S2p = sh.S2 | 1, JJ = sh.d1 * sh.d2;

  // T1[j1][r1] = sum_c H[j1][c] G2[r1][i2][c] by `threads` threads, `parts` of them per element when the
  // elements would leave most of a wavefront idle (a wavefront then holds 64 / parts elements)
  auto core0 = [&](int q, const float *h, int tid, int threads) __attribute__((always_inline)) {
    const int parts = sh.S1 <= 16 ? 4 : (sh.S1 <= 32 ? 2 : 1), width = TT_WAVE / parts;
    const int part = lane / width, per = (sh.S2 + parts - 1) / parts;
    const int c0 = part * per, c1 = c0 + per < sh.S2 ? c0 + per : sh.S2;
    for (int o0 = tid / TT_WAVE * width; o0 < sh.S1; o0 += threads / parts) {  // uniform per wavefront
      const int o = o0 + (lane & (width - 1)), oc = o < sh.S1 ? o : 0, j1 = oc / sh.R1, r1 = oc - j1 * sh.R1;
      const float *hp = h + j1 * sh.S2, *gp = g2s + r1 * S2p;
      // chains of four products, added in pairs and in blocks of 64: no more rounding than one product per lane and
      // a sum over the lanes
      float sum = 0.f;
      for (int cb = c0; cb < c1; cb += 64) {
        const int end = cb + 64 < c1 ? cb + 64 : c1;
        float block = 0.f;
        int c = cb;
        for (; c + 16 <= end; c += 16) {
          float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int k = 0; k < 16; ++k) acc[k >> 2] = fmaf(hp[c + k], gp[c + k], acc[k >> 2]);
          block += (acc[0] + acc[1]) + (acc[2] + acc[3]);
        }
        if (c + 8 <= end) {
          float acc[2] = {0.f, 0.f};
#pragma unroll
          for (int k = 0; k < 8; ++k) acc[k >> 2] = fmaf(hp[c + k], gp[c + k], acc[k >> 2]);
          block += acc[0] + acc[1];
          c += 8;
        }
        float tail = 0.f;
        for (; c < end; ++c) tail = fmaf(hp[c], gp[c], tail);
        sum += block + tail;
      }
      for (int w = width; w < TT_WAVE; w <<= 1) sum += __shfl_xor(sum, w, TT_WAVE);
      if (part == 0 && o < sh.S1) t1buf[(size_t)q * sh.S1 + o] = sum;
    }
  };
  // NR rows of a batch (one, or up to four of which n exist; the others' values are computed and dropped)
  auto batch_math = [&](auto nr, int ub, int n) __attribute__((always_inline)) {
    constexpr int NR = decltype(nr)::value;
    // T3[r2][j3] = sum_{j1,j2} P12[j1][j2][r2] g[j1][j2][j3]
    for (int o = lane; o < sh.S3; o += TT_WAVE) {
      const int r2 = o / sh.d3, j3 = o - r2 * sh.d3;
      float acc[NR] = {};
#pragma unroll 4
      for (int jj = 0; jj < JJ; ++jj) {
        const float x = p12[jj * sh.R2p + r2], *gp = gs + (jj * sh.d3 + j3) * PW_ROWS;
        if constexpr (NR == 1) {
          acc[0] = fmaf(x, gp[0], acc[0]);
        } else {
          const float4 y = *reinterpret_cast<const float4 *>(gp);
          acc[0] = fmaf(x, y.x, acc[0]); acc[1] = fmaf(x, y.y, acc[1]);
          acc[2] = fmaf(x, y.z, acc[2]); acc[3] = fmaf(x, y.w, acc[3]);
        }
      }
#pragma unroll
      for (int k = 0; k < NR; ++k)
        if (k < n) t3buf[(size_t)(ub + k) * sh.S3 + o] = acc[k];
    }
    // H[j1][j2][r2] += sum_j3 g[j1][j2][j3] G3[r2][i3][j3], row after row
    for (int o = lane; o < sh.P; o += TT_WAVE) {
      const int jj = o / sh.R2, r2 = o - jj * sh.R2;
      const float *gp = gs + jj * sh.d3 * PW_ROWS, *sp = g3s + r2 * sh.d3 * PW_ROWS;
      float acc[NR] = {}, h = hs[o];
#pragma unroll 4
      for (int j3 = 0; j3 < sh.d3; ++j3) {
        if constexpr (NR == 1) {
          acc[0] = fmaf(gp[j3 * PW_ROWS], sp[j3 * PW_ROWS], acc[0]);
        } else {
          const float4 x = *reinterpret_cast<const float4 *>(gp + j3 * PW_ROWS), y = *reinterpret_cast<const float4 *>(sp + j3 * PW_ROWS);
          acc[0] = fmaf(x.x, y.x, acc[0]); acc[1] = fmaf(x.y, y.y, acc[1]);
          acc[2] = fmaf(x.z, y.z, acc[2]); acc[3] = fmaf(x.w, y.w, acc[3]);
        }
      }
#pragma unroll
      for (int k = 0; k < NR; ++k)
        if (k < n) h += acc[k];
      hs[o] = h;
    }
  };
  // product, T3 of the row batches first, first + step, ..., and their right partial in hs
  auto prefix = [&](int q, int u0, int u1, int first, int step) __attribute__((always_inline)) {
    const int p = uniq_pref[q], i1 = tt_div(p, sh.mul2, sh.sh2), i2 = p - i1 * sh.n2;
    int ub = u0 + first * PW_ROWS;
    int id = uniq_row[ub + lane < u1 ? ub + lane : u1 - 1];  // lane k < 4: the batch's k-th row (past the end: the last one)
    for (int e = lane; e < sh.S1; e += TT_WAVE) {
      const int j1 = e / sh.R1;
      g1s[(e - j1 * sh.R1) * L.d1p + j1] = g1[(size_t)i1 * sh.S1 + e];
    }
    for (int c = lane; c < sh.S2; c += TT_WAVE) {
      const float *col = g2 + (size_t)i2 * sh.S2 + c;
      for (int r0 = 0; r0 < sh.R1; r0 += 16) {
        float v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = col[(size_t)(r0 + k < sh.R1 ? r0 + k : r0) * sh.n2 * sh.S2];
#pragma unroll
        for (int k = 0; k < 16; ++k)
          if (r0 + k < sh.R1) g2s[(r0 + k) * S2p + c] = v[k];
      }
    }
    for (int o = lane; o < sh.P; o += TT_WAVE) hs[o] = 0.f;
    tt_wave_lds_order();
    for (int c = lane; c < sh.S2; c += TT_WAVE) {
      const int j2 = c / sh.R2, r2 = c - j2 * sh.R2;
      for (int j0 = 0; j0 < sh.d1; j0 += 4) {  // (the padding columns of g1s are never stored from)
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int r1 = 0; r1 < sh.R1; ++r1) {
          const float x = g2s[r1 * S2p + c];
          const float4 y = *reinterpret_cast<const float4 *>(g1s + r1 * L.d1p + j0);
          acc[0] = fmaf(y.x, x, acc[0]); acc[1] = fmaf(y.y, x, acc[1]);
          acc[2] = fmaf(y.z, x, acc[2]); acc[3] = fmaf(y.w, x, acc[3]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (j0 + j < sh.d1) p12[((j0 + j) * sh.d2 + j2) * sh.R2p + r2] = acc[j];
      }
    }
    for (; ub < u1; ub += step * PW_ROWS) {  // uniform
      const int n = u1 - ub < PW_ROWS ? u1 - ub : PW_ROWS;
      const int i3 = id - tt_div(id, sh.mul3, sh.sh3) * sh.n3, ubn = ub + step * PW_ROWS;
      if (ubn < u1) id = uniq_row[ubn + lane < u1 ? ubn + lane : u1 - 1];
      const float *src[PW_ROWS];
#pragma unroll
      for (int k = 0; k < PW_ROWS; ++k) src[k] = g3 + (size_t)__builtin_amdgcn_readlane(i3, k) * sh.d3;
      for (int e = lane; e < sh.D; e += TT_WAVE) {
        float v[PW_ROWS];
#pragma unroll
        for (int k = 0; k < PW_ROWS; ++k) v[k] = gagg[(size_t)(ub + (k < n ? k : 0)) * sh.D + e];
        *reinterpret_cast<float4 *>(gs + e * PW_ROWS) = make_float4(v[0], v[1], v[2], v[3]);
      }
      for (int e = lane; e < sh.S3; e += TT_WAVE) {
        const int r2 = e / sh.d3;
        const size_t at = (size_t)r2 * sh.n3 * sh.d3 + (e - r2 * sh.d3);
        float v[PW_ROWS];
#pragma unroll
        for (int k = 0; k < PW_ROWS; ++k) v[k] = src[k][at];
        *reinterpret_cast<float4 *>(g3s + e * PW_ROWS) = make_float4(v[0], v[1], v[2], v[3]);
      }
      tt_wave_lds_order();
      if (n == 1) batch_math(std::integral_constant<int, 1>{}, ub, n);
      else batch_math(std::integral_constant<int, PW_ROWS>{}, ub, n);
      tt_wave_lds_order();  // the next batch overwrites gs and g3s
    }
  };

  for (int q0 = blockIdx.x * PW_WAVES; q0 < up; q0 += gridDim.x * PW_WAVES) {  // uniform
    const int q = q0 + wave;
    const int u0 = q < up ? pref_seg[q] : 0, u1 = q < up ? pref_seg[q + 1] : 0;
    const bool solo = u1 - u0 <= PW_SOLO_ROWS;
    if (lane == 0) s_rows[wave] = solo ? 0 : u1 - u0;
    if (solo && u1 > u0) {
      prefix(q, u0, u1, 0, 1);
      for (int o = lane; o < sh.P; o += TT_WAVE) hbuf[(size_t)q * sh.P + o] = hs[o];
      core0(q, hs, lane, TT_WAVE);
    }
    __syncthreads();
    for (int w = 0; w < PW_WAVES; ++w)  // prefixes of many rows: all wavefronts, each on its own copy of the product
      if (s_rows[w] > 0) {
        const int v0 = pref_seg[q0 + w];
        prefix(q0 + w, v0, v0 + s_rows[w], wave, PW_WAVES);
        __syncthreads();
        float *h0 = lds + L.hs;  // the first wavefront's partial takes the sum, in wavefront order
        for (int o = threadIdx.x; o < sh.P; o += TT_WAVE * PW_WAVES) {
          float sum = h0[o];
          for (int v = 1; v < PW_WAVES; ++v) sum += h0[v * L.floats + o];
          h0[o] = sum;
          hbuf[(size_t)(q0 + w) * sh.P + o] = sum;
        }
        __syncthreads();
        core0(q0 + w, h0, threadIdx.x, TT_WAVE * PW_WAVES);
        __syncthreads();  // h0 is rewritten
      }
    __syncthreads();  // s_rows is rewritten
  }
}

// Core-1 gradient: dG2[r1][i2][j2][r2] = sum over the prefixes (i1,i2) of the batch of
// sum_j1 G1[i1][j1][r1] H[(i1,i2)][j1][j2][r2], a product with K = (prefix, j1) for every i2.
// Workgroup (i2, 64 columns, 16 values of r1); K goes through LDS in chunks of 64, whose loads are in
// flight while the previous chunk is multiplied, and every output is one thread's sum in increasing K.
// Latency bound: one dependent plan read and one round trip of loads per chunk.  3000 prefixes of rank 16 under
// 100 i2: 8.9 us (one thread per column that walked the prefixes alone, three dependent loads each: 59.8 us).
#define TT_DG2_C 64
#define TT_DG2_R 16
#define TT_DG2_K 64
#define TT_DG2_ZERO_WGS 8192   // workgroups that clear untouched slices, at most
#define TT_DG2_SPARSE 16384    // workgroups without a prefix from which on they are left out
template <bool BATCHED, bool SPARSE>
__global__ void __launch_bounds__(TT_BLOCK)
k_bwd_dg2(TTArg<BATCHED> a, int first, int zero_wgs, int span, int col_tiles, unsigned dmul, unsigned dsh) {
  const TTDev &d = a.get();
  const TTShape &sh = d.sh;
  const float *__restrict__ g1 = d.g[0], *__restrict__ hbuf = d.plan.hbuf;
  const int4 *__restrict__ pref_meta = reinterpret_cast<const int4 *>(d.plan.pref_meta);
  const int32_t *__restrict__ i2_seg = d.plan.i2_seg;
  float *__restrict__ dg2 = d.fused ? const_cast<float *>(d.g[1]) : d.dg[1];
  const int fused = d.fused;
  const float lr = d.lr;
  // grid.x enumerates (i2 from `first` on, column tile, r1 tile); grid.y is the table in a batched launch.
  // SPARSE, a table most of whose slices no lookup touched: the first zero_wgs workgroups clear those slices, `span` at a
  // time (zero_wgs = 0: nothing to clear), and the others are counted by the prefixes in i2 order, of which the first one of
  // every i2 stands for it.  A workgroup per untouched slice costs more than its zeros: 100 k i2, 500 lookups, rank 1 85.5 us a
  // backward call, 21.1 here (20 k i2 of 256 columns at rank 8: 92.4 and 51.9).
  const int r1_tiles = (sh.R1 + TT_DG2_R - 1) / TT_DG2_R;
  if (SPARSE && (int)blockIdx.x < zero_wgs) {
    for (unsigned lo = blockIdx.x * (unsigned)span; lo < (unsigned)sh.n2; lo += (unsigned)zero_wgs * span) {
      const int m = sh.n2 - (int)lo < span ? sh.n2 - (int)lo : span;
      for (int e = threadIdx.x; e < m * sh.S2; e += TT_BLOCK) {
        const int k = e / sh.S2;
        if (i2_seg[lo + k] == i2_seg[lo + k + 1])
          for (int r1 = 0; r1 < sh.R1; ++r1) dg2[((size_t)r1 * sh.n2 + lo) * sh.S2 + e] = 0.f;
      }
    }
    return;
  }
  const int wg = SPARSE ? blockIdx.x - zero_wgs : blockIdx.x, bz = wg % r1_tiles, by = (wg / r1_tiles) % col_tiles;
  int i2 = first + wg / (r1_tiles * col_tiles);
  if (SPARSE) {
    if (i2 >= d.plan.counts[1]) return;
    const int u = i2, p = d.plan.uniq_pref[d.plan.prefs_by_i2[u]];
    i2 = p - tt_div(p, sh.mul2, sh.sh2) * sh.n2;
    if (i2_seg[i2] != u) return;
  } else if (i2 >= sh.n2) {
    return;
  }
  const int s0 = i2_seg[i2], nq = i2_seg[i2 + 1] - s0;
  if (fused && nq == 0) return;  // untouched slice: nothing to apply
  __shared__ __align__(16) float Hs[TT_DG2_K][TT_DG2_C], Gs[TT_DG2_K][TT_DG2_R];
  __shared__ int s_i1[2][TT_DG2_K], s_q[2][TT_DG2_K], s_j1[2][TT_DG2_K];
  const int c = threadIdx.x % TT_DG2_C, rg = threadIdx.x / TT_DG2_C;  // 4 values of r1 per thread
  const int col = by * TT_DG2_C + c, r1b = bz * TT_DG2_R;
  constexpr int HL = TT_DG2_K * TT_DG2_C / TT_BLOCK, GL = TT_DG2_K * TT_DG2_R / TT_BLOCK;
  TTPairWalk<TT_DG2_K> walk(nq, sh.d1, dmul, dsh);
  auto plan_of = [&](int slot, int n) __attribute__((always_inline)) {  // the walk's chunk (n pairs) -> LDS
    if ((int)threadIdx.x < n) {
      int s, j1;
      walk.pair(threadIdx.x, s, j1);
      const int4 m = pref_meta[s0 + s];
      s_i1[slot][threadIdx.x] = m.x; s_q[slot][threadIdx.x] = m.w; s_j1[slot][threadIdx.x] = j1;
    }
  };
  float h[HL], g[GL];
  auto fetch = [&](int slot, int n) __attribute__((always_inline)) {  // operands of a chunk -> registers (zero past its end)
#pragma unroll
    for (int i = 0; i < HL; ++i) {
      const int kk = rg + i * (TT_BLOCK / TT_DG2_C);
      const bool in = kk < n && col < sh.S2;
      h[i] = in ? hbuf[(size_t)s_q[slot][kk] * sh.P + s_j1[slot][kk] * sh.S2 + col] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < GL; ++i) {
      const int kk = threadIdx.x / TT_DG2_R + i * (TT_BLOCK / TT_DG2_R), r1 = r1b + threadIdx.x % TT_DG2_R;
      const bool in = kk < n && r1 < sh.R1;
      g[i] = in ? g1[(size_t)s_i1[slot][kk] * sh.S1 + s_j1[slot][kk] * sh.R1 + r1] : 0.f;
    }
  };
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  int n = walk.count(), next = 0;  // pairs of the chunk that is multiplied and of the one after it (all uniform)
  if (n > 0) {
    plan_of(0, n);
    __syncthreads();
    fetch(0, n);
    walk.advance();
    next = walk.count();
    plan_of(1, next);
  }
  for (int slot = 0; n > 0; slot ^= 1) {
#pragma unroll
    for (int i = 0; i < HL; ++i) Hs[rg + i * (TT_BLOCK / TT_DG2_C)][c] = h[i];
#pragma unroll
    for (int i = 0; i < GL; ++i) Gs[threadIdx.x / TT_DG2_R + i * (TT_BLOCK / TT_DG2_R)][threadIdx.x % TT_DG2_R] = g[i];
    __syncthreads();  // the chunk and the next one's plan entries are visible
    if (next > 0) fetch(slot ^ 1, next);
    walk.advance();
    const int after = walk.count();
    plan_of(slot, after);  // over this chunk's entries, which were last read before the barrier
#pragma unroll 4
    for (int kk = 0; kk < n; ++kk) {
      const float x = Hs[kk][c];
      const float4 y = *reinterpret_cast<const float4 *>(&Gs[kk][4 * rg]);
      acc[0] = fmaf(y.x, x, acc[0]); acc[1] = fmaf(y.y, x, acc[1]);
      acc[2] = fmaf(y.z, x, acc[2]); acc[3] = fmaf(y.w, x, acc[3]);
    }
    __syncthreads();  // the next chunk overwrites the tiles
    n = next;
    next = after;
  }
  if (col >= sh.S2) return;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int r1 = r1b + 4 * rg + k;
    if (r1 < sh.R1) {
      float *dst = dg2 + ((size_t)r1 * sh.n2 + i2) * sh.S2 + col;
      *dst = fused ? fmaf(-lr, acc[k], *dst) : acc[k];
    }
  }
}

// ------------------------------------------------------------------ naive arm
template <bool BATCHED>
__global__ void k_fill_zero_core(TTArg<BATCHED> a, int k) {
  const TTDev &d = a.get();
  float *__restrict__ p = d.dg[k];
  const size_t count = k == 0 ? (size_t)d.sh.n1 * d.sh.S1
                              : (k == 1 ? (size_t)d.sh.R1 * d.sh.n2 * d.sh.S2 : (size_t)d.sh.n3 * d.sh.S3);
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
       e += (size_t)gridDim.x * blockDim.x)
    p[e] = 0.f;
}

// Workgroup per lookup, no dedup, floating-point atomics into the core gradients.
// LDS: g1s[S1] | p12[d1*d2*R2p] | hs[P] | gs[D] | g3s[S3]
template <bool BATCHED>
__global__ void __launch_bounds__(TT_BLOCK)
k_bwd_naive(TTArg<BATCHED> a) {
  const TTDev &d = a.get();
  const TTShape &sh = d.sh;
  const float *__restrict__ g1 = d.g[0], *__restrict__ g2 = d.g[1], *__restrict__ g3 = d.g[2];
  const int64_t *__restrict__ indices = d.indices, *__restrict__ offsets = d.offsets;
  const int nnz = d.nnz, num_bags = d.num_bags;
  const float *__restrict__ grad_out = d.grad_out;
  float *__restrict__ dg1 = d.dg[0], *__restrict__ dg2 = d.dg[1], *__restrict__ dg3 = d.dg[2];
  extern __shared__ float lds[];
  float *g1s = lds, *p12 = g1s + sh.S1, *hs = p12 + sh.d1 * sh.d2 * sh.R2p, *gs = hs + sh.P,
        *g3s = gs + sh.D;
  const int lane = threadIdx.x & (TT_WAVE - 1), wave = threadIdx.x / TT_WAVE;
  for (int l = blockIdx.x; l < nnz; l += gridDim.x) {
    const long long row = indices[l];
    if (row < 0 || row >= sh.num_rows) continue;  // uniform
    int lo = 0, hi = num_bags;  // bag holding position l
    while (hi - lo > 1) {
      int mid = (lo + hi) >> 1;
      if (offsets[mid] <= (long long)l) lo = mid; else hi = mid;
    }
    const int b = lo;
    const int i3 = (int)(row % sh.n3), p = (int)(row / sh.n3), i1 = p / sh.n2, i2 = p - i1 * sh.n2;
    __syncthreads();
    for (int e = threadIdx.x; e < sh.S1; e += blockDim.x) g1s[e] = g1[(size_t)i1 * sh.S1 + e];
    for (int e = threadIdx.x; e < sh.D; e += blockDim.x) gs[e] = grad_out[(size_t)b * sh.D + e];
    for (int e = threadIdx.x; e < sh.S3; e += blockDim.x) {
      const int r2 = e / sh.d3, j3 = e - r2 * sh.d3;
      g3s[e] = g3[((size_t)r2 * sh.n3 + i3) * sh.d3 + j3];
    }
    __syncthreads();
    for (int o = threadIdx.x; o < sh.P; o += blockDim.x) {
      const int j1 = o / sh.S2, c = o - j1 * sh.S2;
      const float *col = g2 + (size_t)i2 * sh.S2 + c;
      float acc = 0.f;
      for (int r1 = 0; r1 < sh.R1; ++r1)
        acc = fmaf(g1s[j1 * sh.R1 + r1], col[(size_t)r1 * sh.n2 * sh.S2], acc);
      p12[(j1 * sh.d2 + c / sh.R2) * sh.R2p + c % sh.R2] = acc;
      // right partial u[j1][j2][r2] = sum_j3 g[j1][j2][j3] G3[r2][i3][j3]  (o indexes [jj][r2])
      const int jj = o / sh.R2, r2 = o - jj * sh.R2;
      float h = 0.f;
      for (int j3 = 0; j3 < sh.d3; ++j3) h = fmaf(gs[jj * sh.d3 + j3], g3s[r2 * sh.d3 + j3], h);
      hs[o] = h;
    }
    __syncthreads();
    for (int o = threadIdx.x; o < sh.S3; o += blockDim.x) {
      const int r2 = o / sh.d3, j3 = o - r2 * sh.d3;
      float acc = 0.f;
      for (int jj = 0; jj < sh.d1 * sh.d2; ++jj)
        acc = fmaf(p12[jj * sh.R2p + r2], gs[jj * sh.d3 + j3], acc);
      atomicAdd(dg3 + ((size_t)r2 * sh.n3 + i3) * sh.d3 + j3, acc);
    }
    for (int o = threadIdx.x; o < sh.R1 * sh.S2; o += blockDim.x) {
      const int r1 = o / sh.S2, c = o - r1 * sh.S2;
      float acc = 0.f;
      for (int j1 = 0; j1 < sh.d1; ++j1) acc = fmaf(g1s[j1 * sh.R1 + r1], hs[j1 * sh.S2 + c], acc);
      atomicAdd(dg2 + ((size_t)r1 * sh.n2 + i2) * sh.S2 + c, acc);
    }
    for (int r1 = wave; r1 < sh.R1; r1 += blockDim.x / TT_WAVE) {
      const float *rowp = g2 + ((size_t)r1 * sh.n2 + i2) * sh.S2;
      for (int j1 = 0; j1 < sh.d1; ++j1) {
        float part = 0.f;
        for (int c = lane; c < sh.S2; c += TT_WAVE) part = fmaf(hs[j1 * sh.S2 + c], rowp[c], part);
        part = tt_wave_sum(part);
        if (lane == 0) atomicAdd(dg1 + (size_t)i1 * sh.S1 + j1 * sh.R1 + r1, part);
      }
    }
  }
}

// ------------------------------------------------------------------ gradient-descent update
template <bool BATCHED>
__global__ void k_sgd_dense(TTArg<BATCHED> a, int k) {
  const TTDev &d = a.get();
  float *__restrict__ g = const_cast<float *>(d.g[k]);
  const float *__restrict__ dg = d.dg[k];
  const float lr = d.lr;
  const size_t count = k == 0 ? (size_t)d.sh.n1 * d.sh.S1
                              : (k == 1 ? (size_t)d.sh.R1 * d.sh.n2 * d.sh.S2 : (size_t)d.sh.n3 * d.sh.S3);
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < count;
       e += (size_t)gridDim.x * blockDim.x)
    g[e] = fmaf(-lr, dg[e], g[e]);
}

// Workgroup per slice of any of the three cores; untouched slices (empty range) are skipped.
template <bool BATCHED>
__global__ void __launch_bounds__(TT_BLOCK)
k_sgd_touched(TTArg<BATCHED> a) {
  const TTDev &d = a.get();
  const TTShape &sh = d.sh;
  float *__restrict__ g1 = const_cast<float *>(d.g[0]), *__restrict__ g2 = const_cast<float *>(d.g[1]),
        *__restrict__ g3 = const_cast<float *>(d.g[2]);
  const float *__restrict__ dg1 = d.dg[0], *__restrict__ dg2 = d.dg[1], *__restrict__ dg3 = d.dg[2];
  const int32_t *__restrict__ i1_seg = d.plan.i1_seg, *__restrict__ i2_seg = d.plan.i2_seg,
                *__restrict__ i3_seg = d.plan.i3_seg;
  const float lr = d.lr;
  int s = blockIdx.x;
  if (s >= sh.n1 + sh.n2 + sh.n3) return;  // a narrower table of the batch
  if (s < sh.n1) {
    if (i1_seg[s] == i1_seg[s + 1]) return;
    for (int e = threadIdx.x; e < sh.S1; e += blockDim.x) {
      const size_t a = (size_t)s * sh.S1 + e;
      g1[a] = fmaf(-lr, dg1[a], g1[a]);
    }
    return;
  }
  s -= sh.n1;
  if (s < sh.n2) {
    if (i2_seg[s] == i2_seg[s + 1]) return;
    for (int e = threadIdx.x; e < sh.R1 * sh.S2; e += blockDim.x) {
      const int r1 = e / sh.S2, c = e - r1 * sh.S2;
      const size_t a = ((size_t)r1 * sh.n2 + s) * sh.S2 + c;
      g2[a] = fmaf(-lr, dg2[a], g2[a]);
    }
    return;
  }
  s -= sh.n2;
  if (i3_seg[s] == i3_seg[s + 1]) return;
  for (int e = threadIdx.x; e < sh.S3; e += blockDim.x) {
    const int r2 = e / sh.d3, j3 = e - r2 * sh.d3;
    const size_t a = ((size_t)r2 * sh.n3 + s) * sh.d3 + j3;
    g3[a] = fmaf(-lr, dg3[a], g3[a]);
  }
}

size_t bwd_lds_bytes(const TTShape &sh) {
  return sizeof(float) * ((size_t)sh.S1 + (size_t)sh.d1 * sh.d2 * sh.R2p + sh.P + sh.D + sh.S3);
}

long long core_len(const TTShape &sh, int k) {
  if (k == 0) return (long long)sh.n1 * sh.S1;
  if (k == 1) return (long long)sh.R1 * sh.n2 * sh.S2;
  return (long long)sh.n3 * sh.S3;
}

}  // namespace

tt_status ttk_backward_plan(const TTBatch &b, hipStream_t s) {
  const TTShape &sh = b.host[0].sh;
  tt_status st;
  // 1. merge output gradients per distinct row
  if ((st = seg_sum(b, SEG_GAGG, 0, TT_KERNEL_GRAD_MERGE, s)) != TT_OK) return st;
  // 2. per-prefix contractions
  const bool mfma = ttk_batch_mfma(b);
  const long long max_pref = tt_batch_max(b, [](const TTDev &d) { return (long long)d.plan.max_prefixes; });
  if (mfma) {
    if ((st = ttk_backward_mfma(b, s)) != TT_OK) return st;
  } else if (max_pref > 0 && prefix_wave_fits(sh)) {
    const long long wgs = (max_pref + PW_WAVES - 1) / PW_WAVES, blocks = wgs < 4096 ? wgs : 4096;
    TTProfScope prof(&b.host[0].plan, TT_KERNEL_BWD_CONTRACT, s);
    TT_LAUNCH(k_bwd_prefix_wave, blocks, TT_WAVE * PW_WAVES, sizeof(float) * PW_WAVES * PrefixWaveLds(sh).floats, s, b);
  } else if (max_pref > 0) {
    const long long blocks = max_pref < 4096 ? max_pref : 4096;
    TTProfScope prof(&b.host[0].plan, TT_KERNEL_BWD_CONTRACT, s);
    TT_LAUNCH(k_bwd_prefix, blocks, TT_BLOCK, bwd_lds_bytes(sh), s, b);
  }
  // 3. core 1: per-i2 accumulation over prefixes (inside the matrix-core kernel, else here).  It
  //    reads core 0, so with the fused update it has to run before the core-0 reduction below.
  if (!mfma) {
    const int col_tiles = tt_ceil_div(sh.S2, TT_DG2_C), r1_tiles = tt_ceil_div(sh.R1, TT_DG2_R);
    const long long n2max = tt_batch_max(b, [](const TTDev &d) { return (long long)d.sh.n2; });
    unsigned dmul, dsh;
    tt_div_constants(sh.d1, &dmul, &dsh);
    const long long tiles = (long long)col_tiles * r1_tiles, most = TT_MAX_WORKGROUPS / tiles - TT_DG2_ZERO_WGS;
    // untouched slices by the thousands: found by the prefixes (see the kernel)
    const bool sparse = (n2max - max_pref) * tiles >= TT_DG2_SPARSE;
    const bool dense = !b.host[0].fused;  // an untouched slice is written (as zeros) only where the gradient is stored
    const int span = !sparse ? 0 : (sh.S2 >= 2048 ? 1 : 2048 / sh.S2);
    const long long ranges = sparse && dense ? (n2max + span - 1) / span : 0;
    const int zero_wgs = (int)(ranges < TT_DG2_ZERO_WGS ? ranges : TT_DG2_ZERO_WGS);
    // as many a launch as it takes workgroups for: one launch, but for tables of millions of slices
    const long long items = sparse ? max_pref : n2max;
    for (long long at = 0; at < items || (at == 0 && zero_wgs > 0); at += most) {
      const int zw = at == 0 ? zero_wgs : 0;
      const long long part = items - at < most ? items - at : most;
      if (sparse) TT_LAUNCH_T(k_bwd_dg2, true, zw + part * tiles, TT_BLOCK, 0, s, b, (int)at, zw, span, col_tiles, dmul, dsh);
      else TT_LAUNCH_T(k_bwd_dg2, false, part * tiles, TT_BLOCK, 0, s, b, (int)at, 0, 0, col_tiles, dmul, dsh);
    }
  }
  // 4. core 2: sum the per-row contributions of all rows sharing i3; core 0: sum the per-prefix
  //    contributions of all prefixes sharing i1 (contiguous)
  if ((st = seg_sum_dg3_dg1(b, s)) != TT_OK) return st;
  return tt_launch_status();
}

tt_status ttk_backward_naive(const TTBatch &b, hipStream_t s) {
  for (int k = 0; k < 3; ++k) {
    const long long len = tt_batch_max(b, [k](const TTDev &d) { return core_len(d.sh, k); });
    int blocks = tt_ceil_div(len, TT_BLOCK * 4);
    if (blocks > 4096) blocks = 4096;
    TT_LAUNCH(k_fill_zero_core, blocks, TT_BLOCK, 0, s, b, k);
  }
  const long long max_nnz = tt_batch_max(b, [](const TTDev &d) { return (long long)d.nnz; });
  if (max_nnz > 0) {
    const long long blocks = max_nnz < 65536 ? max_nnz : 65536;
    TT_LAUNCH(k_bwd_naive, blocks, TT_BLOCK, bwd_lds_bytes(b.host[0].sh), s, b);
  }
  return tt_launch_status();
}

tt_status ttk_sgd(const TTBatch &b, bool touched_only, hipStream_t s) {
  if (touched_only) {
    const long long slices = tt_batch_max(b, [](const TTDev &d) {
      return (long long)d.sh.n1 + d.sh.n2 + d.sh.n3; });
    TTProfScope prof(&b.host[0].plan, TT_KERNEL_SGD, s);
    TT_LAUNCH(k_sgd_touched, slices, TT_BLOCK, 0, s, b);
  } else {
    for (int k = 0; k < 3; ++k) {
      const long long len = tt_batch_max(b, [k](const TTDev &d) { return core_len(d.sh, k); });
      int blocks = tt_ceil_div(len, TT_BLOCK * 4);
      if (blocks > 4096) blocks = 4096;
      TT_LAUNCH(k_sgd_dense, blocks, TT_BLOCK, 0, s, b, k);
    }
  }
  return tt_launch_status();
}
