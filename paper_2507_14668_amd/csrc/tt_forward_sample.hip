// Sample-level reuse forward of the TT embedding bag (paper Section III-B, reuse equation: lookups
// of one bag that share the first two TT indices run one product chain whose third factor is the sum
// of their core-2 slices) on top of the batch-level reuse buffer (Section III-C: one product
// G1[i1] x G2[i2] per distinct prefix of the batch, kept in device memory).
//
//   k_p12_fill   reuse buffer: P12[q][(j1,j2)][r2] for every distinct prefix q of the batch (tables
//                the matrix-core kernels serve fill it with the forward contraction kernel instead)
//   k_bag_chains one wavefront per bag: the bag's lookups are grouped by prefix slot (wavefront
//                ballots, no sorting), each group sums its core-2 slices into S[r2][j3] and adds
//                P12[q] x S to the bag's row, which is written once.  No atomics, no row buffer, no
//                separate bag-sum launch; the price is one read of a whole prefix product per
//                (bag, prefix) group instead of one read of a finished row per lookup.
//   k_bag_chains_4x8x4  the same for the matrix-core shapes, products in registers, several wavefronts per long bag
#include <type_traits>

#include "tt_internal.h"

namespace {

template <bool BATCHED>
__global__ void __launch_bounds__(TT_BLOCK)
k_p12_fill(TTArg<BATCHED> a) {
  const TTDev &d = a.get();
  const TTShape &sh = d.sh;
  const float *__restrict__ g1 = d.g[0], *__restrict__ g2 = d.g[1];
  const int32_t *__restrict__ counts = d.plan.counts, *__restrict__ uniq_pref = d.plan.uniq_pref;
  float *__restrict__ p12buf = d.p12buf;
  extern __shared__ float lds[];
  float *g1s = lds;  // [d1][R1]
  const int up = counts[1];
  for (int q = blockIdx.x; q < up; q += gridDim.x) {
    const int p = uniq_pref[q], i1 = p / sh.n2, i2 = p - i1 * sh.n2;
    __syncthreads();  // the previous prefix's readers of g1s are done
    for (int e = threadIdx.x; e < sh.S1; e += blockDim.x) g1s[e] = g1[(size_t)i1 * sh.S1 + e];
    __syncthreads();
    // consecutive threads take consecutive (j2, r2): coalesced reads of core 1 and writes of P12
    for (int o = threadIdx.x; o < sh.P; o += blockDim.x) {
      const int j1 = o / sh.S2, c = o - j1 * sh.S2;
      const float *col = g2 + (size_t)i2 * sh.S2 + c;
      float acc = 0.f;
      for (int r1 = 0; r1 < sh.R1; ++r1)
        acc = fmaf(g1s[j1 * sh.R1 + r1], col[(size_t)r1 * sh.n2 * sh.S2], acc);
      p12buf[(size_t)q * sh.P + o] = acc;  // o = (j1*d2 + j2)*R2 + r2
    }
  }
}

// NO = outputs per lane (D <= 64 * NO).  LDS per wavefront: the group's prefix product with row
// stride R2 + 1 (lanes of different (j1,j2) on different banks) and the slice sum S[r2][j3].
template <bool BATCHED, int NO>
__global__ void __launch_bounds__(TT_BLOCK)
k_bag_chains(TTArg<BATCHED> a, int lds_per_wave) {
  const TTDev &d = a.get();
  const TTShape &sh = d.sh;
  const float *__restrict__ g3 = d.g[2];
  const float *__restrict__ p12buf = d.p12buf;
  const int64_t *__restrict__ offsets = d.offsets;
  const int32_t *__restrict__ lookup2row = d.plan.lookup2row, *__restrict__ row2pref = d.plan.row2pref,
                *__restrict__ uniq_row = d.plan.uniq_row;
  extern __shared__ float lds[];
  const int lane = threadIdx.x & (TT_WAVE - 1), wave = threadIdx.x / TT_WAVE;
  const int b = blockIdx.x * (blockDim.x / TT_WAVE) + wave;
  if (b >= d.num_bags) return;  // uniform for the wavefront; the kernel has no workgroup barrier
  float *Pw = lds + (size_t)wave * lds_per_wave, *Sw = Pw + sh.d1 * sh.d2 * (sh.R2 + 1);
  const int Rp = sh.R2 + 1;

  int prow[NO], scol[NO];
  float acc[NO];
#pragma unroll
  for (int k = 0; k < NO; ++k) {
    const int o = lane + TT_WAVE * k, jj = o / sh.d3;
    prow[k] = (o < sh.D ? jj : 0) * Rp;
    scol[k] = o < sh.D ? o - jj * sh.d3 : 0;
    acc[k] = 0.f;
  }
  // offsets are clamped to [0, nnz] so that a malformed CSR array cannot index out of bounds
  const long long o0 = offsets[b], o1 = offsets[b + 1], nnz = d.nnz;
  const long long lo = o0 < 0 ? 0 : (o0 > nnz ? nnz : o0), hi = o1 < lo ? lo : (o1 > nnz ? nnz : o1);
  const bool vec4 = (sh.R2 & 3) == 0;  // the buffer is 256-byte aligned and P a multiple of 4 then
  for (long long base = lo; base < hi; base += TT_WAVE) {
    // this lane's lookup: prefix slot and i3 (an invalid lookup has no row slot and takes no part)
    const long long l = base + lane;
    const int u = l < hi ? lookup2row[l] : -1;
    const int q = u >= 0 ? row2pref[u] : -1;
    const int i3 = u >= 0 ? uniq_row[u] - tt_div(uniq_row[u], sh.mul3, sh.sh3) * sh.n3 : 0;
    unsigned long long left = __ballot(q >= 0);
    while (left) {  // uniform: one round per distinct prefix among the 64 lookups
      const int first = __ffsll(left) - 1;
      const int qg = __builtin_amdgcn_readlane(q, first);
      const unsigned long long members = __ballot(q == qg);
      left &= ~members;
      // the group's prefix product: device memory -> LDS
      const float *src = p12buf + (size_t)qg * sh.P;
      if (vec4) {
        for (int e = lane * 4; e < sh.P; e += TT_WAVE * 4) {
          const float4 v = *reinterpret_cast<const float4 *>(src + e);
          const int row = e / sh.R2, c = e - row * sh.R2;
          float *dst = Pw + row * Rp + c;
          dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
        }
      } else {
        for (int e = lane; e < sh.P; e += TT_WAVE) {
          const int row = e / sh.R2;
          Pw[row * Rp + (e - row * sh.R2)] = src[e];
        }
      }
      // S[r2][j3] = sum over the group's lookups, in bag order, of G3[r2][i3][j3]; four lookups per
      // round so that their loads are issued together
      for (int e0 = 0; e0 < sh.S3; e0 += TT_WAVE) {  // uniform trip count: every lane reaches the lane reads
        const int e = e0 + lane < sh.S3 ? e0 + lane : 0, r2 = e / sh.d3, j3 = e - r2 * sh.d3;
        const float *gp = g3 + (size_t)r2 * sh.n3 * sh.d3 + j3;
        float sum = 0.f;
        unsigned long long mm = members;
        while (mm) {
          float v[4];
          bool has[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            has[j] = mm != 0;
            const int m = has[j] ? __ffsll(mm) - 1 : first;
            mm &= mm - 1;  // stays 0 once it is 0
            v[j] = gp[(size_t)__builtin_amdgcn_readlane(i3, m) * sh.d3];
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) sum += has[j] ? v[j] : 0.f;
        }
        if (e0 + lane < sh.S3) Sw[e] = sum;
      }
      tt_wave_lds_order();
#pragma unroll 4
      for (int r2 = 0; r2 < sh.R2; ++r2) {
#pragma unroll
        for (int k = 0; k < NO; ++k) acc[k] = fmaf(Pw[prow[k] + r2], Sw[r2 * sh.d3 + scol[k]], acc[k]);
      }
      tt_wave_lds_order();  // the next group overwrites Pw and Sw
    }
  }
#pragma unroll
  for (int k = 0; k < NO; ++k) {
    const int o = lane + TT_WAVE * k;
    if (o < sh.D) d.out[(size_t)b * sh.D + o] = acc[k];
  }
}

// Bags of the matrix-core shapes (d = 4x8x4, R2 = 32 or 64, core 2 16-byte aligned).  The product of a group
// goes from memory to registers, a float4 along r2 per lane and step: lane = (jj0, r4) holds rows
// jj0 + (64/L)*k, columns 4*r4 .. 4*r4+3 of the product (L = R2/4), and needs the four rows of S with the same
// r2, which it gathers from core 2 itself as float4.  A group of up to REPL lookups is gathered by every row
// of lanes alike; a larger one is dealt to the 64/L rows of lanes, whose sums are added by lane exchanges.
// Sums over r2 across the L lanes are formed once per bag.
// A round is 64 lookups of a wavefront's own bag (WPB = 1), or 256 lookups of the workgroup's bag, whose groups
// belong to the wavefront their prefix slot names (slot mod 4: a prefix is read once per 256 lookups, and the
// hot prefixes, neighbours in slot order, go to different wavefronts); the four results are added in wavefront order.
// Bound by latency: a group is a chain of its product read (R2 = 32: 4 KB, out of the infinity cache) and the
// gathers of its members, and four or five wavefronts per SIMD are in flight (a quarter fewer product reads gave 4 %).
// 2000 bags of 100-300 lookups, Zipf exponent 1.2: 101.5 us (one slice in flight instead of two: 105; a round of 64
// for each wavefront of a shared bag: 110; one wavefront per bag and products through LDS: 256).
template <bool BATCHED, int R2, int WPB>
__global__ void __launch_bounds__(TT_BLOCK, 4)
k_bag_chains_4x8x4(TTArg<BATCHED> a) {
  constexpr int L = R2 / 4, ROWS = TT_WAVE / L, NK = 32 / ROWS, REPL = 6, D = 128, P = 32 * R2;
  constexpr bool PAIR = R2 == 32;
  const TTDev &d = a.get();
  const TTShape &sh = d.sh;
  const float4 *__restrict__ g3 = reinterpret_cast<const float4 *>(d.g[2]);
  const float *__restrict__ p12buf = d.p12buf;
  const int64_t *__restrict__ offsets = d.offsets;
  const int32_t *__restrict__ lookup2row = d.plan.lookup2row, *__restrict__ row2pref = d.plan.row2pref,
                *__restrict__ uniq_row = d.plan.uniq_row;
  __shared__ float s_out[TT_BLOCK / TT_WAVE][D];
  __shared__ int s_list[TT_BLOCK / TT_WAVE][WPB * TT_WAVE];              // i3 of the lookups of a large group
  __shared__ int s_q[WPB == 1 ? 1 : TT_BLOCK], s_i3[WPB == 1 ? 1 : TT_BLOCK];  // the round's lookups
  static_assert(WPB == 1 || WPB == TT_BLOCK / TT_WAVE, "a wavefront per bag, or the workgroup");
  const int lane = threadIdx.x & (TT_WAVE - 1), wave = threadIdx.x / TT_WAVE;
  const int r4 = lane & (L - 1), jj0 = lane / L;
  const int b = WPB == 1 ? (int)blockIdx.x * (TT_BLOCK / TT_WAVE) + wave : (int)blockIdx.x;
  if (b >= d.num_bags) return;  // uniform for the workgroup, or (WPB == 1) for a wavefront that meets no barrier
  float acc[NK][4];
#pragma unroll
  for (int k = 0; k < NK; ++k) acc[k][0] = acc[k][1] = acc[k][2] = acc[k][3] = 0.f;
  // offsets are clamped to [0, nnz] so that a malformed CSR array cannot index out of bounds
  const long long o0 = offsets[b], o1 = offsets[b + 1], nnz = d.nnz;
  const long long lo = o0 < 0 ? 0 : (o0 > nnz ? nnz : o0), hi = o1 < lo ? lo : (o1 > nnz ? nnz : o1);
  const size_t rstep = (size_t)sh.n3;  // float4 between consecutive r2 of core 2
  if (WPB == 1 && lo == hi) {  // uniform: an empty bag has no sums to form
    for (int o = lane; o < D; o += TT_WAVE) d.out[(size_t)b * D + o] = 0.f;
    return;
  }
  for (long long base = lo; base < hi; base += WPB * TT_WAVE) {  // uniform
    // prefix slot and i3 of the round's lookups, lane + 64*j (an invalid lookup has no row slot and takes no part)
    int q[WPB], i3[WPB];
    {
      const long long l = base + (WPB == 1 ? lane : (int)threadIdx.x);
      const int u = l < hi ? lookup2row[l] : -1;
      q[0] = u >= 0 ? row2pref[u] : -1;
      const int row = u >= 0 ? uniq_row[u] : 0;
      i3[0] = row - tt_div(row, sh.mul3, sh.sh3) * sh.n3;
    }
    unsigned long long left[WPB];
    if constexpr (WPB > 1) {
      __syncthreads();  // the previous round has been read
      s_q[threadIdx.x] = q[0];
      s_i3[threadIdx.x] = i3[0];
      __syncthreads();
#pragma unroll
      for (int j = 0; j < WPB; ++j) {
        q[j] = s_q[j * TT_WAVE + lane];
        i3[j] = s_i3[j * TT_WAVE + lane];
        left[j] = __ballot(q[j] >= 0 && (q[j] & (WPB - 1)) == wave);
      }
    } else {
      left[0] = __ballot(q[0] >= 0);
    }
    while (true) {  // uniform: one turn per distinct prefix of this wavefront
      int qg = -1;
#pragma unroll
      for (int j = WPB - 1; j >= 0; --j)
        if (left[j]) qg = __builtin_amdgcn_readlane(q[j], __ffsll(left[j]) - 1);
      if (qg < 0) break;
      const float4 *src = reinterpret_cast<const float4 *>(p12buf + (size_t)qg * P) + lane;
      float4 p[NK];
#pragma unroll
      for (int k = 0; k < NK; ++k) p[k] = src[TT_WAVE * k];
      unsigned long long members[WPB];
      int cnt = 0;
#pragma unroll
      for (int j = 0; j < WPB; ++j) {
        members[j] = __ballot(q[j] == qg);
        left[j] &= ~members[j];
        cnt += __popcll(members[j]);
      }
      float4 s[4];  // rows 4*r4 + i of the summed core-2 slices
#pragma unroll
      for (int i = 0; i < 4; ++i) s[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      // slices of two lookups, all eight loads in flight (R2 = 64 has no registers left for the second four)
      auto add = [&](int m, int m2, bool two) __attribute__((always_inline)) {
        const float4 *gp = g3 + (size_t)(4 * r4) * rstep;
        float4 x[4], y[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = gp[(size_t)i * rstep + m];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (PAIR) y[i] = gp[(size_t)i * rstep + m2];
#pragma unroll
        for (int i = 0; i < 4; ++i) { s[i].x += x[i].x; s[i].y += x[i].y; s[i].z += x[i].z; s[i].w += x[i].w; }
        if (PAIR) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            s[i].x += two ? y[i].x : 0.f; s[i].y += two ? y[i].y : 0.f; s[i].z += two ? y[i].z : 0.f; s[i].w += two ? y[i].w : 0.f;
          }
        }
      };
      if (cnt <= REPL) {  // uniform
#pragma unroll
        for (int j = 0; j < WPB; ++j)
          for (unsigned long long mm = members[j]; mm;) {  // uniform
            const int m = __builtin_amdgcn_readlane(i3[j], __ffsll(mm) - 1);
            mm &= mm - 1;
            if (PAIR && mm) {
              add(m, __builtin_amdgcn_readlane(i3[j], __ffsll(mm) - 1), true);
              mm &= mm - 1;
            } else {
              add(m, m, false);
            }
          }
      } else {
        int before = 0;
#pragma unroll
        for (int j = 0; j < WPB; ++j) {
          if (q[j] == qg) s_list[wave][before + __popcll(members[j] & ((1ull << lane) - 1))] = i3[j];
          before += __popcll(members[j]);
        }
        tt_wave_lds_order();
        for (int m = jj0; m < cnt; m += PAIR ? 2 * ROWS : ROWS) {
          const bool two = PAIR && m + ROWS < cnt;
          add(s_list[wave][m], s_list[wave][two ? m + ROWS : m], two);
        }
        tt_wave_lds_order();  // the next group overwrites the list
#pragma unroll
        for (int o = L; o < TT_WAVE; o <<= 1)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            s[i].x += __shfl_xor(s[i].x, o, TT_WAVE); s[i].y += __shfl_xor(s[i].y, o, TT_WAVE);
            s[i].z += __shfl_xor(s[i].z, o, TT_WAVE); s[i].w += __shfl_xor(s[i].w, o, TT_WAVE);
          }
      }
#pragma unroll
      for (int k = 0; k < NK; ++k) {
        const float pk[4] = {p[k].x, p[k].y, p[k].z, p[k].w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc[k][0] = fmaf(pk[i], s[i].x, acc[k][0]); acc[k][1] = fmaf(pk[i], s[i].y, acc[k][1]);
          acc[k][2] = fmaf(pk[i], s[i].z, acc[k][2]); acc[k][3] = fmaf(pk[i], s[i].w, acc[k][3]);
        }
      }
    }
  }
  // Over r2, the L lanes of a row: in every step a lane hands on the half of its values that the other lane keeps
  // (14 or 30 exchanges; every value at every lane would be 48 or 128), and ends with two columns of the row.
  float v[4 * NK];
#pragma unroll
  for (int k = 0; k < NK; ++k)
#pragma unroll
    for (int j = 0; j < 4; ++j) v[4 * k + j] = acc[k][j];
  int first = 0;
  auto halve = [&](auto lanes_apart, auto values) __attribute__((always_inline)) {
    constexpr int o = decltype(lanes_apart)::value, half = decltype(values)::value / 2;
    const bool up = (r4 & o) != 0;
#pragma unroll
    for (int i = 0; i < half; ++i) {
      const float give = up ? v[i] : v[i + half], keep = up ? v[i + half] : v[i];
      v[i] = keep + __shfl_xor(give, o, TT_WAVE);
    }
    first += up ? half : 0;
  };
  halve(std::integral_constant<int, 1>{}, std::integral_constant<int, 4 * NK>{});
  halve(std::integral_constant<int, 2>{}, std::integral_constant<int, 2 * NK>{});
  halve(std::integral_constant<int, 4>{}, std::integral_constant<int, NK>{});
  if constexpr (L == 16) halve(std::integral_constant<int, 8>{}, std::integral_constant<int, NK / 2>{});
  static_assert(4 * NK / L == 2, "two columns per lane");
  float *mine = s_out[wave] + 4 * (jj0 + ROWS * (first >> 2)) + (first & 3);
  mine[0] = v[0];
  mine[1] = v[1];
  if constexpr (WPB == 1) {
    tt_wave_lds_order();
    for (int o = lane; o < D; o += TT_WAVE) d.out[(size_t)b * D + o] = s_out[wave][o];
  } else {
    __syncthreads();
    if (threadIdx.x < D) {
      float sum = s_out[0][threadIdx.x];
#pragma unroll
      for (int w = 1; w < WPB; ++w) sum += s_out[w][threadIdx.x];
      d.out[(size_t)b * D + threadIdx.x] = sum;
    }
  }
}

}  // namespace

size_t ttk_bag_chains_lds_per_wave(const TTShape &sh) {
  return (size_t)sh.d1 * sh.d2 * (sh.R2 + 1) + sh.S3;
}

tt_status ttk_forward_sample(const TTBatch &b, hipStream_t s) {
  const TTShape &sh = b.host[0].sh;
  // reuse buffer
  if (ttk_batch_mfma(b)) {
    tt_status st = ttk_forward_mfma_p12(b, s);
    if (st != TT_OK) return st;
  } else {
    const long long cap = tt_batch_max(b, [](const TTDev &d) { return (long long)d.plan.max_prefixes; });
    const int grid = (int)(cap < 1 ? 1 : (cap > 8192 ? 8192 : cap));
    TTProfScope prof(&b.host[0].plan, TT_KERNEL_P12_FILL, s);
    TT_LAUNCH(k_p12_fill, grid, TT_BLOCK, sh.S1 * sizeof(float), s, b);
    if (tt_launch_status() != TT_OK) return TT_ERR_HIP;
  }
  if (ttk_batch_mfma(b)) {
    const long long bags = tt_batch_max(b, [](const TTDev &d) { return (long long)d.num_bags; });
    if (bags == 0) return TT_OK;
    // bags of 64 lookups and more on average are shared by a workgroup's four wavefronts (there are few of them, and
    // a wavefront would serve a long chain alone); its wavefronts serve a bag each otherwise, which leaves
    // none of them idle.  The table with the longest bags decides for a batch.
    bool long_bags = false;
    for (int t = 0; t < b.T; ++t) long_bags = long_bags || b.host[t].nnz / TT_WAVE >= b.host[t].num_bags;
    long_bags = long_bags && bags < (1 << 23);  // (a launch has fewer than 2^32 threads)
    const long long grid = long_bags ? bags : (bags + TT_BLOCK / TT_WAVE - 1) / (TT_BLOCK / TT_WAVE);
    TTProfScope prof(&b.host[0].plan, TT_KERNEL_BAG_CHAINS, s);
    if (sh.R2 == 32) {
      if (long_bags) TT_LAUNCH_T2(k_bag_chains_4x8x4, 32, 4, grid, TT_BLOCK, 0, s, b);
      else TT_LAUNCH_T2(k_bag_chains_4x8x4, 32, 1, grid, TT_BLOCK, 0, s, b);
    } else {
      if (long_bags) TT_LAUNCH_T2(k_bag_chains_4x8x4, 64, 4, grid, TT_BLOCK, 0, s, b);
      else TT_LAUNCH_T2(k_bag_chains_4x8x4, 64, 1, grid, TT_BLOCK, 0, s, b);
    }
    return tt_launch_status();
  }
  // bags: as many wavefronts per workgroup (4, 2 or 1) as fit in 64 KB of LDS
  const size_t per_wave = ttk_bag_chains_lds_per_wave(sh);
  int waves = 4;
  while (waves > 1 && waves * per_wave * sizeof(float) > 65536) waves >>= 1;
  if (waves * per_wave * sizeof(float) > 65536) return TT_ERR_SHAPE;
  const long long bags = tt_batch_max(b, [](const TTDev &d) { return (long long)d.num_bags; });
  if (bags == 0) return TT_OK;
  const int grid = tt_ceil_div(bags, waves);
  const size_t lds = waves * per_wave * sizeof(float);
  const int no = tt_ceil_div(sh.D, TT_WAVE);
  TTProfScope prof(&b.host[0].plan, TT_KERNEL_BAG_CHAINS, s);
  if (no <= 1) TT_LAUNCH_T(k_bag_chains, 1, grid, waves * TT_WAVE, lds, s, b, (int)per_wave);
  else if (no <= 2) TT_LAUNCH_T(k_bag_chains, 2, grid, waves * TT_WAVE, lds, s, b, (int)per_wave);
  else if (no <= 4) TT_LAUNCH_T(k_bag_chains, 4, grid, waves * TT_WAVE, lds, s, b, (int)per_wave);
  else if (no <= 8) TT_LAUNCH_T(k_bag_chains, 8, grid, waves * TT_WAVE, lds, s, b, (int)per_wave);
  else TT_LAUNCH_T(k_bag_chains, 16, grid, waves * TT_WAVE, lds, s, b, (int)per_wave);
  return tt_launch_status();
}
