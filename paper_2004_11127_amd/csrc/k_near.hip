// The K nearest columns of every row (arg-K-min, K-min, and the squared
// distance's min and arg-min) for D <= 4 and K <= 64, over the two clouds in
// their spatial order (k_sort.hip).
//
// All pairs of 200 003 x 250 000 points at K = 10 took 8.7 ms on the matrix
// cores, bound by the list insertions; but a row's neighbours lie in the few
// 64-column subtiles around it.  One wave takes R consecutive rows of the
// order: first the subtile at the rows' own place on the curve, then, nearest
// first, those whose bounding box comes as near to some row as that row's K-th
// nearest so far (boxes of 64 subtiles, then of one: a lane tests a box), each
// for the rows that need it.  On a mixture of normals a row meets 6 subtiles;
// tested against the rows' common box and the farthest K-th alone, a wave of
// outliers met 830 and set the time.  Waves that look at too many subtiles give
// their rows up (see Redo).
// 200 003 x 250 000 points, K = 10: 0.37 ms in all; 10^6 x 10^6: 107 -> 2.2 ms.
//
// In a subtile a lane is a column: 64 distances to a row in the direct form
// sum_d (x_d - y_d)^2, the form the result is defined by, so there is nothing
// to re-rank and no limit on the data's extent.  A row's list is one sorted
// (distance, index) entry per lane, so an insertion is a compare, a count and
// a shift by one lane whatever K is (64 nearest of 200 003 x 250 000: 172 -> 1.0
// ms), and the test that keeps columns out uses the exact K-th distance.  Equal
// distances keep the lower index, whatever the order the columns come in.
#include "k_fast_slots.h"

#include <cfloat>
#include <climits>

namespace kred {
namespace {

// Sorted column data: (y_0 .. y_2, index) per column, D = 4 the index apart.
// Padding columns lie at infinity with the index INT_MAX: never nearer, never
// a tie won.
__global__ __launch_bounds__(256) void near_pack_kernel(NearArgs a) {
  const int64_t j = blockIdx.x * (int64_t)256 + threadIdx.x;   // a multiple of 64 columns
  if (a.redo != nullptr && j < 2) a.redo[j] = 0;
  if (j >= (int64_t)a.so.nsub * kSubCols) return;
  const bool ok = j < a.N;
  const int i = ok ? a.so.order_y[j] : INT_MAX;
  float v[4] = {0.0f, 0.0f, 0.0f, 0.0f}, lo[4], hi[4];
#pragma unroll
  for (int d = 0; d < kFastMaxD; ++d) {
    const bool real = d < a.D;
    if (real) v[d] = ok ? a.y[(int64_t)i * a.D + d] : __builtin_inff();
    lo[d] = v[d];
    hi[d] = (ok || !real) ? v[d] : -__builtin_inff();
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      lo[d] = fminf(lo[d], __shfl_xor(lo[d], o));
      hi[d] = fmaxf(hi[d], __shfl_xor(hi[d], o));
    }
  }
  int low = i;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) low = min(low, __shfl_xor(low, o));
  a.cols[j] = float4{v[0], v[1], v[2], a.D == 4 ? v[3] : __int_as_float(i)};
  if (a.D == 4) a.colj[j] = i;
  if ((threadIdx.x & 63) == 0) {
    a.so.box[2 * (j >> 6)] = float4{lo[0], lo[1], lo[2], lo[3]};
    a.so.box[2 * (j >> 6) + 1] = float4{hi[0], hi[1], hi[2], hi[3]};
    a.low[j >> 6] = low;
  }
}

__global__ __launch_bounds__(64) void near_super_kernel(NearArgs a) {
  const int t = blockIdx.x * 64 + threadIdx.x;
  float lo[4], hi[4];
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    lo[d] = __builtin_inff();
    hi[d] = -__builtin_inff();
  }
  if (t < a.so.nsub) {
    const float4 l = a.so.box[2 * t], h = a.so.box[2 * t + 1];
    lo[0] = l.x; lo[1] = l.y; lo[2] = l.z; lo[3] = l.w;
    hi[0] = h.x; hi[1] = h.y; hi[2] = h.z; hi[3] = h.w;
  }
#pragma unroll
  for (int d = 0; d < 4; ++d)
    for (int o = 32; o > 0; o >>= 1) {
      lo[d] = fminf(lo[d], __shfl_xor(lo[d], o));
      hi[d] = fmaxf(hi[d], __shfl_xor(hi[d], o));
    }
  if (threadIdx.x == 0) {
    a.so.sbox[2 * blockIdx.x] = float4{lo[0], lo[1], lo[2], lo[3]};
    a.so.sbox[2 * blockIdx.x + 1] = float4{hi[0], hi[1], hi[2], hi[3]};
  }
}

__device__ __forceinline__ float lane_f(float v, int k) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
}
// the smallest of a non-negative value over the wave
template <int CTRL, int ROWS>
__device__ __forceinline__ int min_step(int v) {
  return min(v, __builtin_amdgcn_update_dpp(v, v, CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ float wave_min(float f) {
  int v = __float_as_int(f);   // orders as the float does
  v = min_step<0x111, 0xf>(v);   // row_shr:1, 2, 4, 8: a row's last lane has the row's
  v = min_step<0x112, 0xf>(v);
  v = min_step<0x114, 0xf>(v);
  v = min_step<0x118, 0xf>(v);
  v = min_step<0x142, 0xa>(v);   // row_bcast:15 and :31: lane 63 has the wave's
  v = min_step<0x143, 0xc>(v);
  return __int_as_float(__builtin_amdgcn_readlane(v, 63));
}
// the value one lane below (lane 0 keeps its own)
__device__ __forceinline__ int from_below(int v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x138, 0xf, 0xf, false);   // wave_shr:1
}

template <int D, int R>
__device__ __forceinline__ void near_rows(const NearArgs& a, int wave, int budget) {
  const int lane = threadIdx.x;
  const int64_t r0 = (int64_t)wave * R;
  const int rows = (int)min((int64_t)R, a.M - r0);
  const int K = a.K;

  // lane l holds row l mod R (a missing row repeats the last); the box of all
  const int64_t mine = a.so.order_x[r0 + min(lane & (R - 1), rows - 1)];
  float xv[D], lo[D], hi[D];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    xv[d] = a.x[mine * D + d];
    lo[d] = hi[d] = xv[d];
    for (int o = R / 2; o > 0; o >>= 1) {
      lo[d] = fminf(lo[d], __shfl_xor(lo[d], o));
      hi[d] = fmaxf(hi[d], __shfl_xor(hi[d], o));
    }
  }
  float xs[R][D];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int d = 0; d < D; ++d) xs[r][d] = lane_f(xv[d], r);

  // a row's list: entry p in lane p, ascending by (distance, index); kth: the
  // K-th distance, the same in every lane
  float ld[R], kth[R];
  int lj[R];
  float mykth = __builtin_inff();   // of the lane's row
#pragma unroll
  for (int r = 0; r < R; ++r) {
    ld[r] = __builtin_inff();
    lj[r] = INT_MAX;
    kth[r] = __builtin_inff();
  }

  // the lane's column, of the subtile at hand and of the two next
  float cy[3][D];
  int cj[3];
  unsigned int need[3];   // the rows that each is for
  auto fetch = [&](int t, float (&to)[D], int& toj) __attribute__((always_inline)) {
    if (t < 0) return;
    const float4 v = a.cols[(int64_t)t * kSubCols + lane];
    const float f[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int d = 0; d < D; ++d) to[d] = f[d];
    toj = D == 4 ? a.colj[(int64_t)t * kSubCols + lane] : __float_as_int(v.w);
  };
  auto distance = [&](int r) __attribute__((always_inline)) {
    float s = 0.0f;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const float t = xs[r][d] - cy[0][d];
      s = __builtin_fmaf(t, t, s);
    }
    return s;
  };
  // the first subtile: its 64 columns sorted into the empty list (a bitonic
  // sort; the rows' sorts are independent and hide each other's latency,
  // where about 28 insertions a row would run one after the other)
  auto fill = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float d = distance(r);
      const bool real = d < __builtin_inff();   // an overflown distance or a NaN is no neighbour
      ld[r] = real ? d : __builtin_inff();
      lj[r] = real ? cj[0] : INT_MAX;
    }
    for (int k = 2; k <= 64; k <<= 1)
      for (int o = k >> 1; o > 0; o >>= 1) {
        const bool low = ((lane & k) == 0) == ((lane & o) == 0);   // keeps the smaller of the pair
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const float d = __shfl_xor(ld[r], o);
          const int j = __shfl_xor(lj[r], o);
          const bool less = (d < ld[r]) | ((d == ld[r]) & (j < lj[r]));
          ld[r] = less == low ? d : ld[r];
          lj[r] = less == low ? j : lj[r];
        }
      }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      kth[r] = lane_f(ld[r], K - 1);
      mykth = (lane & (R - 1)) == r ? kth[r] : mykth;
    }
  };
  auto visit = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (!((need[0] >> r) & 1u)) continue;
      const float s = distance(r);
      // candidates: nearer than the K-th, or as near with a lower index
      if (__builtin_expect(__ballot(s <= kth[r]) != 0, 0)) {
        const int kj = __builtin_amdgcn_readlane(lj[r], K - 1);
        // (FLT_MAX for an open list: an infinite distance is no tie)
        unsigned long long m =
            __ballot(s < kth[r]) | (__ballot(s == fminf(kth[r], FLT_MAX)) & __ballot(cj[0] < kj));
        while (m != 0) {
          const int k = __builtin_ctzll(m);
          m &= m - 1;
          const float d = lane_f(s, k);
          const int j = __builtin_amdgcn_readlane(cj[0], k);
          // entries before (d, j) are the lanes below n
          const int n = __popcll(__ballot(ld[r] < d) | (__ballot(ld[r] == d) & __ballot(lj[r] < j)));
          const float ud = __int_as_float(from_below(__float_as_int(ld[r])));
          const int uj = from_below(lj[r]);
          const bool above = lane > n, here = lane == n;
          ld[r] = above ? ud : ld[r];
          lj[r] = above ? uj : lj[r];
          ld[r] = here ? d : ld[r];
          lj[r] = here ? j : lj[r];
        }
        kth[r] = lane_f(ld[r], K - 1);
        mykth = (lane & (R - 1)) == r ? kth[r] : mykth;
      }
    }
  };
  // squared distance of a box (l, h) and another, a lower bound through its
  // roundings and the distances' own
  auto gap2 = [&](const float (&l)[D], const float (&h)[D], const float (&l2)[D], const float (&h2)[D])
      __attribute__((always_inline)) {
    float s = 0.0f;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const float e = fmaxf(fmaxf(l[d] - h2[d], l2[d] - h[d]), 0.0f);
      s = __builtin_fmaf(e, e, s);
    }
    return s * (1.0f - 1.0f / 65536.0f);
  };
  auto load_box = [&](const float4* b, float (&l)[D], float (&h)[D]) __attribute__((always_inline)) {
    const float4 bl = b[0], bh = b[1];
    const float fl[4] = {bl.x, bl.y, bl.z, bl.w}, fh[4] = {bh.x, bh.y, bh.z, bh.w};
#pragma unroll
    for (int d = 0; d < D; ++d) {
      l[d] = fl[d];
      h[d] = fh[d];
    }
  };
  auto farthest = [&]() __attribute__((always_inline)) {
    float b = kth[0];
#pragma unroll
    for (int r = 1; r < R; ++r) b = fmaxf(b, kth[r]);
    return b;
  };

  // the rows' place among the columns: the last subtile whose first key is below
  // the middle row's (64 probes a step), so of equal columns the lowest come first
  const unsigned int key = a.so.keys_x[r0 + rows / 2];
  int p = 0;
  {
    int end = a.so.nsub;
    while (end - p > 1) {
      const int step = (end - p + 63) / 64;
      const int at = p + lane * step;
      const bool le = at < end && a.so.keys_y[(int64_t)at * kSubCols] < key;
      const int n = __popcll(__ballot(le));
      p += max(n - 1, 0) * step;
      end = min(p + step, end);
    }
  }
  // the other subtiles, nearest first within the nearest 64 of a group of 64
  // times 64: d2, sd2 per lane the distance of its subtile and super, mt, ms
  // those still to come
  int group = 0, base = 0;
  unsigned long long ms = 0, mt = 0;
  float d2 = __builtin_inff(), sd2 = __builtin_inff();
  float bl[D], bh[D];   // the lane's subtile's box
  float bound = __builtin_inff();
  auto next = [&](unsigned int& rows_of) __attribute__((always_inline)) {
    for (;;) {
      if (mt != 0) {
        const float near = wave_min(d2);
        if (near <= bound) {
          const int k = __builtin_ctzll(__ballot(d2 == near) & mt);
          mt &= ~(1ull << k);
          d2 = lane == k ? __builtin_inff() : d2;
          float l[D], h[D];
#pragma unroll
          for (int d = 0; d < D; ++d) {
            l[d] = lane_f(bl[d], k);
            h[d] = lane_f(bh[d], k);
          }
          rows_of = (unsigned int)(__ballot(gap2(l, h, xv, xv) <= mykth) & ((1u << R) - 1u));
          if (rows_of != 0u) return base + k;
          continue;
        }
        mt = 0;
      }
      if (ms != 0) {
        const float near = wave_min(sd2);
        if (near <= bound) {
          const int k = __builtin_ctzll(__ballot(sd2 == near) & ms);
          ms &= ~(1ull << k);
          sd2 = lane == k ? __builtin_inff() : sd2;
          base = ((group - 1) * 64 + k) * 64;
          const int id = base + lane;
          const bool in = id < a.so.nsub && id != p;
          d2 = __builtin_inff();
          if (in) {
            load_box(a.so.box + 2 * id, bl, bh);
            d2 = gap2(bl, bh, lo, hi);
            if (__builtin_expect(bound == 0.0f, 0)) {
              // every row has K columns at its own place: only lower indices still
              // count (a third of 250 000 points at one place: 4.8 ms without)
              int top = 0;
#pragma unroll
              for (int r = 0; r < R; ++r) top = max(top, __builtin_amdgcn_readlane(lj[r], K - 1));
              if (a.low[id] > top) d2 = __builtin_inff();
            }
          }
          mt = __ballot(in);
          continue;
        }
        ms = 0;
      }
      if (group * 64 >= a.so.nsuper) return -1;
      const int id = group * 64 + lane;
      ++group;
      sd2 = __builtin_inff();
      if (id < a.so.nsuper) {
        load_box(a.so.sbox + 2 * id, bl, bh);
        sd2 = gap2(bl, bh, lo, hi);
      }
      ms = __ballot(id < a.so.nsuper);
    }
  };
  // two subtiles' loads are in flight behind the one at hand
  fetch(p, cy[0], cj[0]);
  fill();
  bound = farthest();
  int t1 = next(need[1]), t2 = -1;
  fetch(t1, cy[1], cj[1]);
  if (t1 >= 0) t2 = next(need[2]);
  fetch(t2, cy[2], cj[2]);
  // A wave whose rows look at too many subtiles gives them up: after 64 if many of the
  // boxes at hand still come as near as the K-th nearest, or after the budget.
  int left = budget;
  while (t1 >= 0 && left > 0) {
    --left;
    if (budget != INT_MAX && left == budget - 64 &&
        4 * __popcll(__ballot(sd2 <= bound) & ms) > (R == 1 ? 3 : 1) * min(64, a.so.nsuper - (group - 1) * 64))
      left = 0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      cy[0][d] = cy[1][d];
      cy[1][d] = cy[2][d];
    }
    cj[0] = cj[1];
    cj[1] = cj[2];
    need[0] = need[1];
    need[1] = need[2];
    t1 = t2;
    t2 = -1;
    if (t1 >= 0) t2 = next(need[2]);
    fetch(t2, cy[2], cj[2]);
    visit();
    bound = farthest();
  }
  if (t1 >= 0) {
    // Rows lying apart (where the curve leaves a cluster) do better one at a time; one
    // that three in four of the boxes come near to by itself has no use for the order.
    const int id = (group - 1) * 64 + lane;
    const bool in = id < a.so.nsuper;
    float l[D], h[D];
    load_box(a.so.sbox + 2 * (in ? id : 0), l, h);
    int hopeless = 0;
#pragma unroll
    for (int r = 0; r < R; ++r)
      hopeless += 4 * __popcll(__ballot(in && gap2(l, h, xs[r], xs[r]) <= kth[r])) > 3 * __popcll(__ballot(in));
    int at = 0;
    if (lane == 0) {
      if (hopeless > 0) atomicAdd(&a.redo[0], min(hopeless, rows));
      at = atomicAdd(&a.redo[1], rows);
    }
    at = __builtin_amdgcn_readfirstlane(at);
    if (lane < rows) a.redo[2 + at + lane] = (int)r0 + lane;
    return;
  }

#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (r >= rows) break;
    const int64_t row = __builtin_amdgcn_readlane((int)mine, r);
    if (lane < K) {
      if (a.kvalues) static_cast<float*>(a.out)[row * K + lane] = ld[r];
      else static_cast<int*>(a.out)[row * K + lane] = lj[r] == INT_MAX ? -1 : lj[r];
    }
  }
}

template <int D, int R>
__global__ __launch_bounds__(64) void near_kernel(NearArgs a) {
  near_rows<D, R>(a, blockIdx.x, a.budget);
}

// The rows given up, one at a time; or, if the kernels behind do the call, the columns
// for the fast kernel (in the place of the lists' own scratch).
template <int D>
__global__ __launch_bounds__(64) void near_rest_kernel(NearArgs a) {
  const int rows = a.redo[1];
  if (rows == 0) return;
  if (a.redo[0] >= a.from) {
    if (a.guard == nullptr) return;
    const FastFrame fr = fast_frame(a.guard, a.D, 1.0f, a.limit);
    if (fr.ok) {
      const double qu = fast_quantum(fr.U);
      for (int64_t j = blockIdx.x * (int64_t)64 + threadIdx.x; j < a.N16; j += (int64_t)gridDim.x * 64) {
        __bf16 s[32];
#pragma unroll
        for (int k = 0; k < 32; ++k) s[k] = (__bf16)0.0f;
        float vt[kFastMaxD];
        if (j < a.N) pack_column<D == 4>(a.y, D, 1.0, fr, qu, j, true, 0.0, s, vt);
        uint4 w[4];
        __builtin_memcpy(w, s, 64);
#pragma unroll
        for (int q = 0; q < 4; ++q) a.apk[j * 4 + q] = w[q];
      }
      return;
    }
  }
  for (int w = blockIdx.x; w < rows; w += gridDim.x) near_rows<D, 1>(a, a.redo[2 + w], INT_MAX);
}

template <int D, int R>
hipError_t launch_near_as(const NearArgs& a, hipStream_t s) {
  const unsigned waves = (unsigned)((a.M + R - 1) / R);
  hipLaunchKernelGGL((near_kernel<D, R>), dim3(waves), dim3(64), 0, s, a);
  if (a.redo != nullptr)
    hipLaunchKernelGGL(near_rest_kernel<D>, dim3(std::min(waves, 4096u)), dim3(64), 0, s, a);
  return hipGetLastError();
}
template <int R>
hipError_t launch_near_rows(const NearArgs& a, hipStream_t s) {
  switch (a.D) {
    case 1: return launch_near_as<1, R>(a, s);
    case 2: return launch_near_as<2, R>(a, s);
    case 3: return launch_near_as<3, R>(a, s);
    case 4: return launch_near_as<4, R>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_near(const NearArgs& a, hipStream_t s) {
  const int64_t cols = (int64_t)a.so.nsub * kSubCols;
  hipLaunchKernelGGL(near_pack_kernel, dim3((unsigned)((cols + 255) / 256)), dim3(256), 0, s, a);
  hipLaunchKernelGGL(near_super_kernel, dim3((unsigned)a.so.nsuper), dim3(64), 0, s, a);
  // one row a wave where the rows are few (more waves, each with less to do in
  // turn) or sparse among the columns (the box of several would be wide), else
  // four, which share a subtile's load and box.  us at K = 10, 1 against 4
  // rows: 10^4 x 10^4 points 100 / 147, 2000 x 3 10^5 116 / 356, 200 003 x
  // 250 000 407 / 395, 3 10^5 x 2000 376 / 292 (16 rows 436, 282 at 10^4).
  if (a.M <= 65536 || a.N / 16 >= a.M) return launch_near_rows<1>(a, s);
  return launch_near_rows<4>(a, s);
}

}  // namespace kred
