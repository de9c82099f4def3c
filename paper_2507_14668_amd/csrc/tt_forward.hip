// Forward pass of the TT embedding bag (paper Section III-B; batch-level reuse, Section III-C).
//
// Planned arm: one workgroup per distinct (i1,i2) prefix forms the prefix product
// P12 = G1[i1] x G2[i2] once in LDS and multiplies it with G3[i3] for every distinct row
// under that prefix; a second kernel sums the rows of each bag (gather-bound).
// Naive arm: one workgroup per bag runs the full three-slice chain for every lookup.
#include "tt_internal.h"

namespace {

// P12[j1][j2][r2] = sum_r1 G1[i1][j1][r1] * G2[r1][i2][j2][r2], written to LDS with row stride
// R2p over (j1,j2).  g1s must already hold the core-0 slice.  Consecutive threads take
// consecutive (j2,r2) so the core-1 reads are coalesced 4-byte streams of S2 floats per r1.
__device__ __forceinline__ void prefix_product(const TTShape &sh, const float *__restrict__ g2,
                                               int i2, const float *g1s, float *p12) {
  for (int o = threadIdx.x; o < sh.P; o += blockDim.x) {
    const int j1 = o / sh.S2, c = o - j1 * sh.S2;
    const float *col = g2 + (size_t)i2 * sh.S2 + c;
    float acc = 0.f;
    for (int r1 = 0; r1 < sh.R1; ++r1)
      acc = fmaf(g1s[j1 * sh.R1 + r1], col[(size_t)r1 * sh.n2 * sh.S2], acc);
    const int jj = j1 * sh.d2 + c / sh.R2, r2 = c % sh.R2;
    p12[jj * sh.R2p + r2] = acc;
  }
}

// row[(j1,j2)][j3] = sum_r2 P12[(j1,j2)][r2] * G3[r2][i3][j3] for output element o < D.
__device__ __forceinline__ float row_element(const TTShape &sh, const float *p12,
                                             const float *g3s, int o) {
  const int jj = o / sh.d3, j3 = o - jj * sh.d3;
  float acc = 0.f;
  for (int r2 = 0; r2 < sh.R2; ++r2) acc = fmaf(p12[jj * sh.R2p + r2], g3s[r2 * sh.d3 + j3], acc);
  return acc;
}

__device__ __forceinline__ void load_g3_slice(const TTShape &sh, const float *__restrict__ g3,
                                              int i3, float *g3s, int tid, int nthreads) {
  for (int e = tid; e < sh.S3; e += nthreads) {
    const int r2 = e / sh.d3, j3 = e - r2 * sh.d3;
    g3s[e] = g3[((size_t)r2 * sh.n3 + i3) * sh.d3 + j3];
  }
}

// LDS layout (floats): g1s[S1] | p12[d1*d2*R2p] | g3s[rows_per_iter * S3]
template <bool BATCHED>
__global__ void __launch_bounds__(TT_BLOCK)
k_fwd_prefix_rows(TTArg<BATCHED> a, int rows_per_iter) {
  const TTDev &d = a.get();
  const TTShape &sh = d.sh;
  const float *__restrict__ g1 = d.g[0], *__restrict__ g2 = d.g[1], *__restrict__ g3 = d.g[2];
  const int32_t *__restrict__ counts = d.plan.counts, *__restrict__ uniq_pref = d.plan.uniq_pref,
                *__restrict__ pref_seg = d.plan.pref_seg, *__restrict__ uniq_row = d.plan.uniq_row;
  float *__restrict__ rowbuf = d.plan.rowbuf;
  extern __shared__ float lds[];
  float *g1s = lds, *p12 = g1s + sh.S1, *g3s = p12 + sh.d1 * sh.d2 * sh.R2p;
  const int up = counts[1];
  for (int q = blockIdx.x; q < up; q += gridDim.x) {
    const int p = uniq_pref[q], i1 = p / sh.n2, i2 = p - i1 * sh.n2;
    for (int e = threadIdx.x; e < sh.S1; e += blockDim.x) g1s[e] = g1[(size_t)i1 * sh.S1 + e];
    __syncthreads();
    prefix_product(sh, g2, i2, g1s, p12);
    __syncthreads();
    const int u0 = pref_seg[q], u1 = pref_seg[q + 1];
    // rows_per_iter rows at a time: thread group `sub` owns row u + sub
    const int sub = threadIdx.x / sh.D, tin = threadIdx.x - sub * sh.D;
    for (int u = u0; u < u1; u += rows_per_iter) {
      if (rows_per_iter == 1) {
        load_g3_slice(sh, g3, uniq_row[u] % sh.n3, g3s, threadIdx.x, blockDim.x);
      } else if (sub < rows_per_iter && u + sub < u1) {
        load_g3_slice(sh, g3, uniq_row[u + sub] % sh.n3, g3s + sub * sh.S3, tin, sh.D);
      }
      __syncthreads();
      if (rows_per_iter == 1) {
        for (int o = threadIdx.x; o < sh.D; o += blockDim.x)
          rowbuf[(size_t)u * sh.D + o] = row_element(sh, p12, g3s, o);
      } else if (sub < rows_per_iter && u + sub < u1) {
        rowbuf[(size_t)(u + sub) * sh.D + tin] = row_element(sh, p12, g3s + sub * sh.S3, tin);
      }
      __syncthreads();
    }
  }
}

#define TT_BAG_BLOCK 64

// VEC consecutive columns of distinct row u (zeros for an invalid lookup, u < 0).
template <int VEC>
__device__ __forceinline__ void load_row_vec(const float *__restrict__ rowbuf, int u, int D, int c,
                                             float (&x)[VEC]) {
  if (u < 0) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) x[v] = 0.f;
  } else if (VEC == 4) {
    const float4 t = *reinterpret_cast<const float4 *>(rowbuf + (size_t)u * D + c);
    x[0] = t.x; x[1 % VEC] = t.y; x[2 % VEC] = t.z; x[3 % VEC] = t.w;
  } else {
    x[0] = rowbuf[(size_t)u * D + c];
  }
}

// out[b][:] = sum over the lookups of bag b of rowbuf[lookup2row[l]][:].
// A group of LANES lanes owns one bag; each lane owns VEC consecutive columns per step.
template <bool BATCHED, int VEC>
__global__ void __launch_bounds__(TT_BLOCK)
k_bag_sum(TTArg<BATCHED> a, int lanes) {
  const TTDev &d = a.get();
  const int D = d.sh.D, num_bags = d.num_bags, nnz = d.nnz;
  const int64_t *__restrict__ offsets = d.offsets;
  const int32_t *__restrict__ lookup2row = d.plan.lookup2row;
  const float *__restrict__ rowbuf = d.plan.rowbuf;
  float *__restrict__ out = d.out;
  const int groups_per_block = blockDim.x / lanes;
  const int g = threadIdx.x / lanes, lane = threadIdx.x - g * lanes;
  const int stride = gridDim.x * groups_per_block;
  int b = blockIdx.x * groups_per_block + g;
  // One-lookup bags (one-hot features), four bags of a lane group at a time: the four chains
  // offsets -> row slot -> row -> store are independent and overlap.  Same arithmetic as the general
  // path below (0 + row), so the result does not depend on which path served a bag.
  for (; b + 3 * stride < num_bags; b += 4 * stride) {
    long long o[4][2];
#pragma unroll
    for (int k = 0; k < 4; ++k) { o[k][0] = offsets[b + k * stride]; o[k][1] = offsets[b + k * stride + 1]; }
    bool single = true;
#pragma unroll
    for (int k = 0; k < 4; ++k) single = single && o[k][0] >= 0 && o[k][0] < nnz && o[k][1] == o[k][0] + 1;
    if (!single) break;  // the general path takes over from bag b (the same for every lane of the group)
    int u[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) u[k] = lookup2row[o[k][0]];
    for (int c = lane * VEC; c < D; c += lanes * VEC) {
      float x[4][VEC];
#pragma unroll
      for (int k = 0; k < 4; ++k) load_row_vec<VEC>(rowbuf, u[k], D, c, x[k]);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float t[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) t[v] = 0.f + (0.f + x[k][v]);
        float *dst = out + (size_t)(b + k * stride) * D + c;
        if (VEC == 4) tt_store_stream4(dst, t[0], t[1 % VEC], t[2 % VEC], t[3 % VEC]);
        else dst[0] = t[0];
      }
    }
  }
  for (; b < num_bags; b += stride) {
    // offsets are clamped to [0, nnz] so that a malformed CSR array cannot index out of bounds
    const long long o0 = offsets[b], o1 = offsets[b + 1];
    const int l0 = o0 < 0 ? 0 : (o0 > nnz ? nnz : (int)o0), l1 = o1 < l0 ? l0 : (o1 > nnz ? nnz : (int)o1);
    for (int c = lane * VEC; c < D; c += lanes * VEC) {
      // two-level sum: blocks of TT_BAG_BLOCK lookups are summed first and then added to the
      // running total, so rounding error grows with len/TT_BAG_BLOCK instead of len
      float tot[VEC];
#pragma unroll
      for (int v = 0; v < VEC; ++v) tot[v] = 0.f;
      for (int base = l0; base < l1; base += TT_BAG_BLOCK) {
        const int stop = base + TT_BAG_BLOCK < l1 ? base + TT_BAG_BLOCK : l1;
        float acc[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
        int l = base;
        for (; l + 4 <= stop; l += 4) {  // four independent gathers in flight
          int u[4];
          float x[4][VEC];
#pragma unroll
          for (int k = 0; k < 4; ++k) u[k] = lookup2row[l + k];
#pragma unroll
          for (int k = 0; k < 4; ++k) load_row_vec<VEC>(rowbuf, u[k], D, c, x[k]);
#pragma unroll
          for (int v = 0; v < VEC; ++v) acc[v] += (x[0][v] + x[1][v]) + (x[2][v] + x[3][v]);
        }
        for (; l < stop; ++l) {
          float x[VEC];
          load_row_vec<VEC>(rowbuf, lookup2row[l], D, c, x);
#pragma unroll
          for (int v = 0; v < VEC; ++v) acc[v] += x[v];
        }
#pragma unroll
        for (int v = 0; v < VEC; ++v) tot[v] += acc[v];
      }
      if (VEC == 4) {
        tt_store_stream4(out + (size_t)b * D + c, tot[0], tot[1 % VEC], tot[2 % VEC], tot[3 % VEC]);
      } else {
        out[(size_t)b * D + c] = tot[0];
      }
    }
  }
}

// Naive arm: workgroup per bag; every lookup recomputes its prefix product and row.
// LDS layout: g1s[S1] | p12[d1*d2*R2p] | g3s[S3]
template <bool BATCHED>
__global__ void __launch_bounds__(TT_BLOCK)
k_fwd_naive(TTArg<BATCHED> a) {
  const TTDev &d = a.get();
  const TTShape &sh = d.sh;
  const float *__restrict__ g1 = d.g[0], *__restrict__ g2 = d.g[1], *__restrict__ g3 = d.g[2];
  const int64_t *__restrict__ indices = d.indices, *__restrict__ offsets = d.offsets;
  const int num_bags = d.num_bags, nnz = d.nnz;
  float *__restrict__ out = d.out;
  extern __shared__ float lds[];
  float *g1s = lds, *p12 = g1s + sh.S1, *g3s = p12 + sh.d1 * sh.d2 * sh.R2p;
  constexpr int MAXO = 4;  // D <= 1024 columns over 256 threads
  for (int b = blockIdx.x; b < num_bags; b += gridDim.x) {
    float acc[MAXO], tot[MAXO];
#pragma unroll
    for (int k = 0; k < MAXO; ++k) acc[k] = tot[k] = 0.f;
    long long l0 = offsets[b], l1 = offsets[b + 1];  // clamped: malformed offsets stay in bounds
    l0 = l0 < 0 ? 0 : (l0 > nnz ? nnz : l0);
    l1 = l1 < l0 ? l0 : (l1 > nnz ? nnz : l1);
    for (long long l = l0; l < l1; ++l) {
      const long long row = indices[l];
      if (((l - l0) % TT_BAG_BLOCK) == 0) {  // two-level sum as in the planned arm
#pragma unroll
        for (int k = 0; k < MAXO; ++k) { tot[k] += acc[k]; acc[k] = 0.f; }
      }
      if (row < 0 || row >= sh.num_rows) continue;  // uniform across the workgroup
      const int i3 = (int)(row % sh.n3), p = (int)(row / sh.n3), i1 = p / sh.n2,
                i2 = p - i1 * sh.n2;
      for (int e = threadIdx.x; e < sh.S1; e += blockDim.x) g1s[e] = g1[(size_t)i1 * sh.S1 + e];
      load_g3_slice(sh, g3, i3, g3s, threadIdx.x, blockDim.x);
      __syncthreads();
      prefix_product(sh, g2, i2, g1s, p12);
      __syncthreads();
#pragma unroll
      for (int k = 0; k < MAXO; ++k) {
        const int o = threadIdx.x + k * TT_BLOCK;
        if (o < sh.D) acc[k] += row_element(sh, p12, g3s, o);
      }
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < MAXO; ++k) {
      const int o = threadIdx.x + k * TT_BLOCK;
      if (o < sh.D) out[(size_t)b * sh.D + o] = tot[k] + acc[k];
    }
  }
}

// Few lookups of a matrix-core shape (d = 4x8x4, ranks R, R), without a plan.  A lane has one column (j2, r2) of the core-1 slices
// and forms P12[j1][j2][r2] = sum_r1 G1[i1][j1][r1] G2[r1][i2][j2][r2]; the wavefront then forms the lookup's 16 columns
// (j1, j3) of each of its j2.  Every sum runs in the order of the planned kernels (the matrix cores add one product after the
// other) and the rows are added as k_bag_sum adds them, so the result is theirs to the bit.
// BAGS: a workgroup has a bag and 64 columns, its wavefronts take the bag's lookups in turn and the sum is formed here: one
// launch.  Otherwise a wavefront has one lookup and 64 columns, the row goes to rowbuf and k_bag_sum follows.
// Latency bound: offsets, index, slices are three dependent round trips; a wavefront requests the next lookup's slices
// before it multiplies the current one's.  A repeated prefix is multiplied again, which limits the number of lookups.
constexpr int DIRECT_WAVES = 8;
template <bool BATCHED, int R, bool BAGS>
__global__ void __launch_bounds__(TT_WAVE * DIRECT_WAVES)
k_fwd_direct(TTArg<BATCHED> a) {
  const TTDev &d = a.get();
  const TTShape &sh = d.sh;
  constexpr int S2 = 8 * R, GROUPS = S2 / TT_WAVE, JW = TT_WAVE / R, NV = 16 * JW;  // NV: columns (j2, j1, j3) of a row here
  static_assert(TT_WAVE % R == 0, "a wavefront holds whole j2");
  const float *__restrict__ g1 = d.g[0], *__restrict__ g2 = d.g[1], *__restrict__ g3 = d.g[2];
  const int64_t *__restrict__ indices = d.indices, *__restrict__ offsets = d.offsets;
  __shared__ __align__(16) float s_p[DIRECT_WAVES][4][TT_WAVE], s_w[DIRECT_WAVES][4][R];  // products [j1][column], core-2 slice [j3][r2]
  __shared__ float s_row[BAGS ? TT_DIRECT_BAG_LOOKUPS : 1][NV];
  const int b = (int)blockIdx.x / GROUPS, grp = (int)blockIdx.x - b * GROUPS;  // bag, or eight lookups
  const int lane = threadIdx.x & (TT_WAVE - 1), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / TT_WAVE);
  const int c = grp * TT_WAVE + lane, r2 = lane & (R - 1);
  int l0 = b * DIRECT_WAVES, l1 = l0 + DIRECT_WAVES < d.nnz ? l0 + DIRECT_WAVES : d.nnz;
  if constexpr (BAGS) {
    // offsets are clamped to [0, nnz] so that a malformed CSR array cannot index out of bounds (nnz <= TT_DIRECT_BAG_LOOKUPS)
    const long long o0 = offsets[b], o1 = offsets[b + 1], nnz = d.nnz;
    l0 = o0 < 0 ? 0 : (o0 > nnz ? (int)nnz : (int)o0);
    l1 = o1 < l0 ? l0 : (o1 > nnz ? (int)nnz : (int)o1);
  }
  const size_t step = (size_t)sh.n2 * S2;
  // the wavefront's lookups, one per lane: l0 + wave, l0 + wave + 8, ... (at most 64 of them)
  const int mine = l0 + wave + DIRECT_WAVES * lane;
  const long long at = mine < l1 ? indices[mine] : -1;
  const int row = at >= 0 && at < sh.num_rows ? (int)at : -1;
  unsigned long long left = __ballot(mine < l1);
  struct Slices { float v[R]; float4 w; int i1, k; };  // this lane's column of core 1, its row of core 2
  auto load = [&](Slices &x) __attribute__((always_inline)) {  // the next lookup (k: of the wavefront)
    x.k = __ffsll(left) - 1;
    left &= left - 1;
    const int r = __builtin_amdgcn_readlane(row, x.k), rc = r < 0 ? 0 : r;  // an invalid lookup reads row 0
    const int p = tt_div(rc, sh.mul3, sh.sh3), i1 = tt_div(p, sh.mul2, sh.sh2), i2 = p - i1 * sh.n2, i3 = rc - p * sh.n3;
    const float *col = g2 + (size_t)i2 * S2 + c;
#pragma unroll
    for (int r1 = 0; r1 < R; ++r1) x.v[r1] = col[(size_t)r1 * step];
    x.w = *reinterpret_cast<const float4 *>(g3 + ((size_t)r2 * sh.n3 + i3) * 4);
    x.i1 = r < 0 ? -1 : i1;
  };
  auto finish = [&](const Slices &x) __attribute__((always_inline)) {
    const float *__restrict__ u = g1 + (size_t)(x.i1 < 0 ? 0 : x.i1) * (4 * R);
    float p[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r1 = 0; r1 < R; ++r1)
#pragma unroll
      for (int j1 = 0; j1 < 4; ++j1) p[j1] = fmaf(u[j1 * R + r1], x.v[r1], p[j1]);
#pragma unroll
    for (int j1 = 0; j1 < 4; ++j1) s_p[wave][j1][lane] = p[j1];
    if (lane < R) { s_w[wave][0][lane] = x.w.x; s_w[wave][1][lane] = x.w.y; s_w[wave][2][lane] = x.w.z; s_w[wave][3][lane] = x.w.w; }
    tt_wave_lds_order();
    if (lane < NV) {
      const float4 *pp = reinterpret_cast<const float4 *>(&s_p[wave][(lane >> 2) & 3][(lane >> 4) * R]),
                   *ww = reinterpret_cast<const float4 *>(s_w[wave][lane & 3]);
      float acc = 0.f;
#pragma unroll
      for (int q = 0; q < R / 4; ++q) {
        const float4 y = pp[q], z = ww[q];
        acc = fmaf(z.x, y.x, acc); acc = fmaf(z.y, y.y, acc); acc = fmaf(z.z, y.z, acc); acc = fmaf(z.w, y.w, acc);
      }
      if constexpr (BAGS) {
        s_row[wave + DIRECT_WAVES * x.k][lane] = x.i1 < 0 ? 0.f : acc;  // an invalid lookup adds zeros
      } else if (x.i1 >= 0) {
        const int j2 = grp * JW + (lane >> 4), j1 = (lane >> 2) & 3, j3 = lane & 3;
        d.plan.rowbuf[(size_t)(l0 + wave) * sh.D + (j1 * 8 + j2) * 4 + j3] = acc;
      }
    }
    tt_wave_lds_order();  // the next lookup overwrites s_p and s_w
  };
  if constexpr (!BAGS) {
    if (left == 0) return;  // uniform per wavefront
    Slices x;
    load(x);
    if (grp == 0 && lane == 0) d.plan.lookup2row[l0 + wave] = x.i1 < 0 ? -1 : l0 + wave;
    finish(x);
    return;
  }
  if (left != 0) {  // uniform per wavefront
    Slices xa, xb;
    load(xa);
    while (true) {  // written out twice so that both sets of slices stay in registers
      bool more = left != 0;
      if (more) load(xb);
      finish(xa);
      if (!more) break;
      more = left != 0;
      if (more) load(xa);
      finish(xb);
      if (!more) break;
    }
  }
  __syncthreads();
  if (threadIdx.x < NV) {
    float tot = 0.f;
    const int len = l1 - l0;
    for (int base = 0; base < len; base += TT_BAG_BLOCK) {
      const int stop = base + TT_BAG_BLOCK < len ? base + TT_BAG_BLOCK : len;
      float sum = 0.f;
      int l = base;
      for (; l + 4 <= stop; l += 4)
        sum += (s_row[l][threadIdx.x] + s_row[l + 1][threadIdx.x]) + (s_row[l + 2][threadIdx.x] + s_row[l + 3][threadIdx.x]);
      for (; l < stop; ++l) sum += s_row[l][threadIdx.x];
      tot += sum;
    }
    const int j2 = grp * JW + (int)threadIdx.x / 16, j1 = (threadIdx.x >> 2) & 3, j3 = threadIdx.x & 3;
    d.out[(size_t)b * sh.D + (j1 * 8 + j2) * 4 + j3] = tot;
  }
}

// The bag sums from bf16 copies of the cores (layouts of k_cores_to_bf16) without a plan.  A workgroup has a bag and 64 columns
// (j2, r2) of core 1, its wavefronts take the bag's lookups in turn.  The product of a lookup is R / 4 MFMAs of sixteen 4x4x4
// blocks (A[m = j1][k = r1], B[k = r1][n = column]: the four r1 of a column are 8 contiguous bytes of the copy), after which a lane
// holds P12[j1 = 0..3] of its column and adds P12[j1] G3[r2][i3][j3] to 16 sums that stay in registers over the bag; the
// sums over r2, across lanes, and over the wavefronts are formed once per bag.  All sums are fp32.
// Bound by the slices a lookup reads, repeated or not (64 KB at ranks 64, out of L1 as fast as out of L2); two columns a lane
// halve the rest (one: 29.8 us for 5161 lookups at ranks 64, two: 23.3; with reorder and planned forward 62).  Errors against 64 bits
// are two thirds of the planned forward's (500 bags of 1 to 20 lookups, ranks 64: 9.7e-8 / 1.59e-7, 2-norm).
typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int BAGB_WAVES = 4, BAGB_COLS = 2, BAGB_BLOCK = 8;  // wavefronts per workgroup, columns per lane, lookups per partial sum
template <bool BATCHED, int R>
__global__ void __launch_bounds__(TT_WAVE * BAGB_WAVES, 4)
k_bag_direct_bf16(TTArg<BATCHED> a) {
  const TTDev &d = a.get();
  const TTShape &sh = d.sh;
  constexpr int CPL = BAGB_COLS, COLS = TT_WAVE * CPL, S2 = 8 * R, GROUPS = S2 / COLS, JW = COLS / R, JL = R / CPL, NV = 16;
  static_assert(COLS % R == 0 && JL >= NV, "a wavefront holds whole j2; NV: sums (j1, j3) of a lane, JL: lanes of a j2");
  const unsigned short *__restrict__ g1 = reinterpret_cast<const unsigned short *>(d.g[0]),
                       *__restrict__ g2 = reinterpret_cast<const unsigned short *>(d.g[1]),
                       *__restrict__ g3 = reinterpret_cast<const unsigned short *>(d.g[2]);
  const int64_t *__restrict__ indices = d.indices, *__restrict__ offsets = d.offsets;
  __shared__ float s_sum[BAGB_WAVES][JW * NV];
  const int b = (int)blockIdx.x / GROUPS, grp = (int)blockIdx.x - b * GROUPS;
  const int lane = threadIdx.x & (TT_WAVE - 1), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / TT_WAVE);
  const int c = grp * COLS + lane * CPL, r2 = (lane * CPL) & (R - 1);
  // offsets are clamped to [0, nnz] so that a malformed CSR array cannot index out of bounds
  const long long o0 = offsets[b], o1 = offsets[b + 1], nnz = d.nnz;
  const int l0 = o0 < 0 ? 0 : (o0 > nnz ? (int)nnz : (int)o0), l1 = o1 < l0 ? l0 : (o1 > nnz ? (int)nnz : (int)o1);
  float acc[NV], tot[NV];  // the running block of BAGB_BLOCK lookups, and the blocks before it: rounding grows with the blocks
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = tot[k] = 0.f;
  int in_block = 0;
  const int64_t *__restrict__ bag = indices + l0;
  const unsigned len = (unsigned)(l1 - l0);  // (unsigned: the last step may end behind 2^31)
  for (unsigned base = wave; base < len; base += BAGB_WAVES * TT_WAVE) {  // uniform per wavefront
    const unsigned mine = base + BAGB_WAVES * lane;  // the wavefront's next 64 lookups, one per lane
    const long long at = mine < len ? bag[mine] : -1;
    const int row = at >= 0 && at < sh.num_rows ? (int)at : -1;  // an invalid lookup adds nothing
    for (unsigned long long left = __ballot(row >= 0); left != 0; left &= left - 1) {
      const int x = __builtin_amdgcn_readlane(row, __ffsll(left) - 1);
      const int p = tt_div(x, sh.mul3, sh.sh3), i1 = tt_div(p, sh.mul2, sh.sh2), i2 = p - i1 * sh.n2, i3 = x - p * sh.n3;
      struct __align__(8 * CPL) Cols { uint2 c[CPL]; };  // four r1 of this lane's columns
      const Cols *col = reinterpret_cast<const Cols *>(g2 + (((size_t)i2 * (R / 4)) * S2 + c) * 4);
      // block q of the A register holds r1 = 4q .. 4q + 3; step q broadcasts it to all blocks
      const uint2 av = *reinterpret_cast<const uint2 *>(g1 + (size_t)i1 * (4 * R) + (lane & 3) * R + 4 * ((lane >> 2) & (R / 4 - 1)));
      const bf16x4 am = *reinterpret_cast<const bf16x4 *>(&av);
      Cols bv[R / 4];
      uint2 w2[CPL];
#pragma unroll
      for (int q = 0; q < R / 4; ++q) bv[q] = col[(size_t)q * (S2 / CPL)];
#pragma unroll
      for (int e = 0; e < CPL; ++e) w2[e] = *reinterpret_cast<const uint2 *>(g3 + ((size_t)(r2 + e) * sh.n3 + i3) * 4);
      __builtin_amdgcn_sched_barrier(0);  // every load is requested before the first product waits
      f32x4 pr[CPL][2];  // per column two chains
#pragma unroll
      for (int e = 0; e < CPL; ++e) pr[e][0] = pr[e][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
      tt_static_for<0, R / 4>([&](auto k) __attribute__((always_inline)) {
        constexpr int q = decltype(k)::value;
#pragma unroll
        for (int e = 0; e < CPL; ++e)
          pr[e][q & 1] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(am, *reinterpret_cast<const bf16x4 *>(&bv[q].c[e]), pr[e][q & 1], 4, q, 0);
      });
#pragma unroll
      for (int e = 0; e < CPL; ++e) {
        const float w[4] = {__uint_as_float(w2[e].x << 16), __uint_as_float(w2[e].x & 0xffff0000u), __uint_as_float(w2[e].y << 16),
                            __uint_as_float(w2[e].y & 0xffff0000u)};
#pragma unroll
        for (int j1 = 0; j1 < 4; ++j1)
#pragma unroll
          for (int j3 = 0; j3 < 4; ++j3) acc[4 * j1 + j3] = fmaf(pr[e][0][j1] + pr[e][1][j1], w[j3], acc[4 * j1 + j3]);
      }
      if (++in_block == BAGB_BLOCK) {  // uniform
        in_block = 0;
#pragma unroll
        for (int k = 0; k < NV; ++k) { tot[k] += acc[k]; acc[k] = 0.f; }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] += tot[k];
  // Over r2, the JL lanes of a j2: a lane hands on the half of its sums that the other one keeps, and ends with one of the 16.
  int idx = 0;
#pragma unroll
  for (int o = 1, half = NV / 2; o < NV; o <<= 1, half >>= 1) {
    const bool up = (lane & o) != 0;
#pragma unroll
    for (int i = 0; i < half; ++i) {
      const float x = acc[i], y = acc[i + half];  // (by value: a choice between elements becomes an index, and a chain of selects)
      acc[i] = (up ? y : x) + __shfl_xor(up ? x : y, o, TT_WAVE);
    }
    idx += up ? half : 0;
  }
#pragma unroll
  for (int o = NV; o < JL; o <<= 1) acc[0] += __shfl_xor(acc[0], o, TT_WAVE);
  if ((lane & (JL - 1)) < NV) s_sum[wave][(lane / JL) * NV + idx] = acc[0];
  __syncthreads();
  if (threadIdx.x < JW * NV) {
    const float sum = (s_sum[0][threadIdx.x] + s_sum[1][threadIdx.x]) + (s_sum[2][threadIdx.x] + s_sum[3][threadIdx.x]);
    const int j2 = grp * JW + (int)threadIdx.x / NV, j1 = (threadIdx.x >> 2) & 3, j3 = threadIdx.x & 3;
    d.out[(size_t)b * sh.D + (j1 * 8 + j2) * 4 + j3] = sum;
  }
}

size_t fwd_lds_bytes(const TTShape &sh, int rows_per_iter) {
  return sizeof(float) * ((size_t)sh.S1 + (size_t)sh.d1 * sh.d2 * sh.R2p +
                          (size_t)rows_per_iter * sh.S3);
}

}  // namespace

tt_status ttk_forward_plan(const TTBatch &b, hipStream_t s) {
  const TTShape &sh = b.host[0].sh;  // d[] and r[] are common to the batch
  const long long max_pref = tt_batch_max(b, [](const TTDev &d) { return (long long)d.plan.max_prefixes; });
  if (max_pref > 0 && ttk_batch_mfma(b)) {
    tt_status st = ttk_forward_mfma(b, s);
    if (st != TT_OK) return st;
  } else if (max_pref > 0) {
    int rows_per_iter = TT_BLOCK / sh.D;
    if (rows_per_iter < 1) rows_per_iter = 1;
    if (rows_per_iter > 8) rows_per_iter = 8;
    const long long blocks = max_pref < 4096 ? max_pref : 4096;
    TTProfScope prof(&b.host[0].plan, TT_KERNEL_FWD_CONTRACT, s);
    TT_LAUNCH(k_fwd_prefix_rows, blocks, TT_BLOCK, fwd_lds_bytes(sh, rows_per_iter), s, b, rows_per_iter);
  }
  return ttk_bag_sum(b, s);
}

tt_status ttk_bag_sum(const TTBatch &b, hipStream_t s) {
  const TTShape &sh = b.host[0].sh;
  const long long max_bags = tt_batch_max(b, [](const TTDev &d) { return (long long)d.num_bags; });
  if (max_bags > 0) {
    bool vec4 = (sh.D % 4) == 0;
    for (int t = 0; t < b.T; ++t) vec4 = vec4 && ((uintptr_t)b.host[t].out % 16) == 0;
    int lanes = 1;
    while (lanes < TT_WAVE && lanes * (vec4 ? 4 : 1) < sh.D) lanes <<= 1;
    const int groups = TT_BLOCK / lanes;
    long long blocks = (max_bags + groups - 1) / groups;
    // a batch of one-lookup bags (as many lookups as bags) lets every lane group take four bags at a time
    bool one_hot = true;
    for (int t = 0; t < b.T; ++t) one_hot = one_hot && b.host[t].nnz == b.host[t].num_bags;
    if (one_hot) blocks = (blocks + 3) / 4;
    if (blocks > 16384) blocks = 16384;
    TTProfScope prof(&b.host[0].plan, TT_KERNEL_BAG_SUM, s);
    if (vec4) TT_LAUNCH_T(k_bag_sum, 4, blocks, TT_BLOCK, 0, s, b, lanes);
    else TT_LAUNCH_T(k_bag_sum, 1, blocks, TT_BLOCK, 0, s, b, lanes);
  }
  return tt_launch_status();
}

tt_status ttk_forward_naive(const TTBatch &b, hipStream_t s) {
  const long long max_bags = tt_batch_max(b, [](const TTDev &d) { return (long long)d.num_bags; });
  if (max_bags == 0) return TT_OK;
  const long long blocks = max_bags < 65536 ? max_bags : 65536;
  TT_LAUNCH(k_fwd_naive, blocks, TT_BLOCK, fwd_lds_bytes(b.host[0].sh, 1), s, b);
  return tt_launch_status();
}

// A plan is a chain of launches (one of 8 to 20 us up to TT_SMALL_MAX_LOOKUPS, nine of 40 us and more above), and what it saves, the
// repeated rows and prefixes, is less than that in a short batch.  Whole calls, reorder + forward / this, in us; rows
// spread over the table / log-uniform / all the same:
//   ranks 32   20 lookups in one bag 18.4 / 5.5     2048 37.5 / 10.7, 35.5 / 10.4, 28.3 / 10.3     16384 75 / 43, 68 / 42, 55 / 38
//   ranks 64   20 lookups in one bag 26.4 / 8.6     2048 50.6 / 26.8, 45.2 / 25.7, 33.1 / 20.2     8192 102 / 86, 80 / 77, 64 / 58
//   (ranks 64, 12000: 118 / 120, 83 / 108, 65 / 83, hence the limits)
// One launch up to TT_DIRECT_BAG_LOOKUPS: 64 lookups in one bag take it 13.2 (ranks 32) and 22.4, the two launches 13.2 and 14.3;
// in 64 bags 4.9 and 6.8, 7.4 and 8.2.  ... and as long as its workgroups, four or eight a bag with lookups or without, are few: 1 /
// 16 / 32 lookups in one launch and in two (7.7 whatever the bags), ranks 32 512 bags 4.9 / 5.5 / 6.7, 768 5.7 / 6.5 / 7.7, 1024
// 6.6 / 7.5 / 8.6, 16384 67 / 69 / 71; ranks 64 96 bags 5.2 / 6.5 / 6.5, 128 5.7 / 8.7 / 11.5, 256 7.6 / 10.6 / 14.5, 16384 300.
#define TT_DIRECT_BAG_MAX_BAGS_32 768
#define TT_DIRECT_BAG_MAX_BAGS_64 96
static bool direct_in_one_launch(const TTDev &d) {
  return d.nnz <= TT_DIRECT_BAG_LOOKUPS && d.num_bags <= (d.sh.R1 == 32 ? TT_DIRECT_BAG_MAX_BAGS_32 : TT_DIRECT_BAG_MAX_BAGS_64);
}
bool ttk_forward_direct_serves(const TTDev &d) {
  // (rowbuf has a row per lookup unless the table itself has fewer)
  return d.mfma && d.nnz <= (d.sh.R1 == 32 ? TT_DIRECT_MAX_LOOKUPS_32 : TT_DIRECT_MAX_LOOKUPS_64) && d.num_bags <= TT_SMALL_MAX_BAGS &&
         (direct_in_one_launch(d) || d.plan.max_rows == d.nnz);
}

tt_status ttk_forward_direct(const TTBatch &b, hipStream_t s) {
  const TTDev &d = b.host[0];
  if (d.num_bags == 0) return TT_OK;
  const int groups = d.sh.S2 / TT_WAVE, nt = TT_WAVE * DIRECT_WAVES;
  if (direct_in_one_launch(d)) {
    if (d.sh.R1 == 32) TT_LAUNCH_T2(k_fwd_direct, 32, true, d.num_bags * groups, nt, 0, s, b);
    else TT_LAUNCH_T2(k_fwd_direct, 64, true, d.num_bags * groups, nt, 0, s, b);
    return tt_launch_status();
  }
  const int wgs = tt_ceil_div(d.nnz, DIRECT_WAVES) * groups;
  if (d.nnz > 0) {
    if (d.sh.R1 == 32) TT_LAUNCH_T2(k_fwd_direct, 32, false, wgs, nt, 0, s, b);
    else TT_LAUNCH_T2(k_fwd_direct, 64, false, wgs, nt, 0, s, b);
  }
  return ttk_bag_sum(b, s);
}

// Nanoseconds per lookup and per bag that this costs (fitted to batches of 100 to 40000 lookups in 500 to 20000 bags), against
// what a plan and the planned forward take at least, with every lookup the same row: 18 us and more up to
// TT_SMALL_MAX_LOOKUPS, 51 us and more above.  Reorder + forward / this, bags of ten, rows spread / log-uniform / all the same:
//   ranks 32   2048 lookups 35 / 5.5, 34 / 5.6, 27 / 5.6   5161 59 / 10.2, 61 / 10.0, 53 / 10.0   40000 87 / 47, 78 / 49, 59 / 46
//   ranks 64   2048 39 / 10.3, 35 / 10.7, 27 / 9.5         5161 67 / 22.6, 63 / 23.3, 52 / 19.5   10000 79 / 37, 67 / 41, 54 / 31
//              20000 97 / 71, 77 / 75, 54 / 59
// One-lookup bags, ranks 64: 5000 62 / 40, 15000 70 / 117; 20000 bags with ten lookups in all: 49 / 86 (ranks 32 50 / 33).
// One or two bags that hold all lookups are chains, of planned row reads or of this.  At ranks 64 a step of this is the longer one:
// one bag 500 lookups 85 / 80, 1500 224 / 234, 5000 717 / 774; two bags 5000 406 / 389, 8000 603 / 621; three 14000 861 / 725.  At
// ranks 32 it is the shorter one (one bag 500 87 / 64, 46000 6219 / 5641).  (A single long bag among many short ones, 8 %
// slower at ranks 64, cannot be told from the sizes.)
bool ttk_bag_direct_bf16_pays(const TTShape &sh, long long nnz, long long bags) {
  if (sh.R1 == 64 && ((bags == 1 && nnz > 1000) || (bags == 2 && nnz > 6000))) return false;
  const long long ns = sh.R1 == 32 ? (19 * nnz + 28 * bags) / 20 : (31 * nnz + 43 * bags) / 10;
  return ns <= (nnz <= TT_SMALL_MAX_LOOKUPS ? 13000 : 45000);
}

tt_status ttk_bag_direct_bf16(const TTBatch &b, hipStream_t s) {
  const TTDev &d = b.host[0];
  if (d.num_bags == 0) return TT_OK;
  const long long wgs = (long long)d.num_bags * (d.sh.S2 / (TT_WAVE * BAGB_COLS));
  if (wgs > TT_MAX_WORKGROUPS) return TT_ERR_INVALID_ARG;
  if (d.sh.R1 == 32) TT_LAUNCH_T(k_bag_direct_bf16, 32, wgs, TT_WAVE * BAGB_WAVES, 0, s, b);
  else TT_LAUNCH_T(k_bag_direct_bf16, 64, wgs, TT_WAVE * BAGB_WAVES, 0, s, b);
  return tt_launch_status();
}
