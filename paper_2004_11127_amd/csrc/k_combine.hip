// Second pass over column-block partials (when the j range was split into C
// blocks to give a small-M problem enough workgroups).  Each partial is the
// reduction of Eq. (2) over one block of columns; this pass applies the same
// reduction across blocks in a fixed order (so results are reproducible run
// to run; several lanes share an element):
//   sum:          a = sum_c a_c  (also the x-gradient sums of the Gaussian
//                 vector-Jacobian product, scaled by -1/sigma^2)
//   log-sum-exp:  (m, s) = (max_c m_c, sum_c s_c 2^(m_c - m)),  a = (m + log2 s) ln 2
//   arg-K-min:    merge the C sorted (distance, index) lists, keep the K first.
// The second pass reads C x M x W floats once; it is HBM-bound.
#include "kred_internal.h"

#include <climits>

namespace kred {
namespace {

// The column blocks of the kernel that ran.
__device__ __forceinline__ int blocks_of(const CombineArgs& a) {
  if (a.guard != nullptr && fast_frame(a.guard, a.D, a.fscale, a.flimit).ok) return a.fast_C;
  return a.C;
}

// Four lanes per output element: lane q of a group sums the blocks c = q,
// q + 4, q + 8, ... in increasing order (four loads in flight), and the group
// then adds its four sums as (s0 + s1) + (s2 + s3).  The order is fixed, so
// results repeat run to run; the group's lanes share their element and leave
// the loop together, so the shuffles see the whole group.  Every lane of the
// group gets the sum.
__device__ __forceinline__ float quad_sum(const float* __restrict__ p, int64_t st, int C) {
  float s = 0.0f;
  int c = threadIdx.x & 3;
  for (; c + 12 < C; c += 16) {
    const float v0 = p[c * st], v1 = p[(c + 4) * st], v2 = p[(c + 8) * st], v3 = p[(c + 12) * st];
    s += v0;
    s += v1;
    s += v2;
    s += v3;
  }
  for (; c < C; c += 4) s += p[c * st];
  s += __shfl_xor(s, 1);
  s += __shfl_xor(s, 2);
  return s;
}

__global__ __launch_bounds__(256) void combine_sum_kernel(CombineArgs a) {
  const int C = blocks_of(a);
  if (C == 1) return;
  const int Ec = min(a.EP, a.E - a.e0);
  const int64_t total = a.M * Ec;
  for (int64_t t = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 2; t < total;
       t += ((int64_t)gridDim.x * blockDim.x) >> 2) {
    const int64_t row = t / Ec;
    const int e = (int)(t - row * Ec);
    const float s = quad_sum(a.part + row * a.EP + e, a.M * a.EP, C);
    if ((threadIdx.x & 3) == 0) static_cast<float*>(a.out)[row * a.E + a.e0 + e] = s;
  }
}

__global__ __launch_bounds__(256) void combine_gradx_kernel(CombineArgs a) {
  const int C = blocks_of(a);
  if (C == 1) return;
  const int W = a.DP + 1;
  const int64_t total = a.M * (1 + a.D);
  for (int64_t t = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 2; t < total;
       t += ((int64_t)gridDim.x * blockDim.x) >> 2) {
    const int64_t row = t / (1 + a.D);
    const int w = (int)(t - row * (1 + a.D));
    const float s = quad_sum(a.part + row * W + w, a.M * W, C);
    if ((threadIdx.x & 3) == 0) static_cast<float*>(a.out)[t] = (w == 0) ? s : -s * a.gscale;
  }
}

// vector-Jacobian product in x: partials are the DP sums G_k; out = -G * gscale
__global__ __launch_bounds__(256) void combine_vjp_kernel(CombineArgs a) {
  const int64_t total = a.M * a.D;
  for (int64_t t = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 2; t < total;
       t += ((int64_t)gridDim.x * blockDim.x) >> 2) {
    const int64_t row = t / a.D;
    const int k = (int)(t - row * a.D);
    const float s = quad_sum(a.part + row * a.DP + k, a.M * a.DP, a.C);
    if ((threadIdx.x & 3) == 0) {
      float* o = static_cast<float*>(a.out) + t;
      const float v = -s * a.gscale;
      *o = a.accumulate ? *o + v : v;
    }
  }
}

// Sixteen lanes per row: lane q folds the blocks q, q + 16, .. into its own
// (m, s), four loads in flight, and the lanes merge by shuffles.  One thread
// per row left all but M / 64 waves idle and took two dependent passes over
// its C pairs: 10^4 rows of 93 blocks took 41 us, now 4.6.
__global__ __launch_bounds__(256) void combine_lse_kernel(CombineArgs a) {
  const int C = blocks_of(a);
  if (C == 1) return;
  const int q = threadIdx.x & 15;
  const float2* part = reinterpret_cast<const float2*>(a.part);
  for (int64_t row = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 4; row < a.M;
       row += ((int64_t)gridDim.x * blockDim.x) >> 4) {
    float m = -__builtin_inff(), s = 0.0f;
    for (int c0 = q; c0 < C; c0 += 64) {
      float2 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        v[u] = c0 + 16 * u < C ? part[(int64_t)(c0 + 16 * u) * a.M + row]
                                 : float2{-__builtin_inff(), 0.0f};
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (v[u].x == -__builtin_inff()) continue;   // an empty block (its sum is 0)
        const float mx = fmaxf(m, v[u].x);
        s = s * __builtin_amdgcn_exp2f(m - mx) + v[u].y * __builtin_amdgcn_exp2f(v[u].x - mx);
        m = mx;
      }
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
      const float m2 = __shfl_xor(m, o), s2 = __shfl_xor(s, o);
      const float mx = fmaxf(m, m2);
      s = (m == -__builtin_inff() ? 0.0f : s * __builtin_amdgcn_exp2f(m - mx)) +
          (m2 == -__builtin_inff() ? 0.0f : s2 * __builtin_amdgcn_exp2f(m2 - mx));
      m = mx;
    }
    if (q == 0) static_cast<float*>(a.out)[row] = (m + __builtin_amdgcn_logf(s)) * kLn2;
  }
}

// (d, j) strictly before (d2, j2) in (distance, index) order.
__device__ __forceinline__ bool before(float d, int j, float d2, int j2) {
  return d < d2 || (d == d2 && j < j2);
}

// The C sorted (distance, index) lists of a row, merged by a group of G lanes:
// each lane holds one list in registers, and KP times the group takes its
// smallest head (a reduction by shuffles) and the lane that held it moves on.
// More lists than lanes go in several batches, the result so far taking the
// place of one list.  What bounds it is latency, so the lists' loads are
// independent and the rows spread over G lanes each: one thread per row took
// 450 us for 20 000 rows of 32 lists of 10 (and 691 us for 10^5 rows of 12),
// these groups 116 and 195.
template <int KP, int G>
__global__ __launch_bounds__(256) void combine_knn_kernel(CombineArgs a) {
  if (redo_skip(a.redo)) return;
  if (a.redo.rows != nullptr && a.guard != nullptr && !fast_frame(a.guard, a.D, a.fscale, a.flimit).ok) return;
  const int C = blocks_of(a);
  if (C == 1) return;
  const int q = threadIdx.x & (G - 1);
  for (int64_t row = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / G; row < a.M;
       row += ((int64_t)gridDim.x * blockDim.x) / G) {
    float rd[KP];   // the result so far, the same in every lane of the group
    int rj[KP];
#pragma unroll
    for (int p = 0; p < KP; ++p) {
      rd[p] = __builtin_inff();
      rj[p] = INT_MAX;
    }
    for (int c0 = 0; c0 < C;) {
      // lane G - 1 takes the result so far (from the second batch on)
      const int lists = c0 == 0 ? G : G - 1;
      float dk[KP];
      int jk[KP];
      const bool own = q < lists && c0 + q < C;
      const float2* src = reinterpret_cast<const float2*>(a.part) +
                          ((int64_t)(own ? c0 + q : 0) * a.M + row) * KP;
#pragma unroll
      for (int p = 0; p < KP; ++p) {
        dk[p] = rd[p];
        jk[p] = rj[p];
        if (own) {
          const float2 v = src[p];
          dk[p] = v.x;
          jk[p] = __float_as_int(v.y);
        } else if (q < lists) {
          dk[p] = __builtin_inff();
          jk[p] = INT_MAX;
        }
      }
#pragma unroll
      for (int p = 0; p < KP; ++p) {
        float d = dk[0];
        int j = jk[0], who = q;
#pragma unroll
        for (int o = G / 2; o > 0; o >>= 1) {
          const float d2 = __shfl_xor(d, o);
          const int j2 = __shfl_xor(j, o), w2 = __shfl_xor(who, o);
          if (before(d2, j2, d, j) || (d2 == d && j2 == j && w2 < who)) {
            d = d2;
            j = j2;
            who = w2;
          }
        }
        rd[p] = d;
        rj[p] = j;
        if (who == q) {
#pragma unroll
          for (int u = 0; u + 1 < KP; ++u) {
            dk[u] = dk[u + 1];
            jk[u] = jk[u + 1];
          }
          dk[KP - 1] = __builtin_inff();
          jk[KP - 1] = INT_MAX;
        }
      }
      c0 += lists;
    }
    // lane p's entry (KP <= G)
    static_assert(KP <= G, "one lane per entry");
    float d = __builtin_inff();
    int j = INT_MAX;
#pragma unroll
    for (int p = 0; p < KP; ++p)
      if (p == q) {
        d = rd[p];
        j = rj[p];
      }
    int rank = q;
    if (a.rx != nullptr) {
      // large-D lists rank by the expanded form, whose error is absolute (about
      // 2^-24 (|x|^2 + |y|^2) per term): the merged candidates get their
      // direct-form distance, accurate relative to itself (exact on integer
      // data), and are ordered again by (distance, index); the unfilled entries
      // (+inf, INT_MAX) stay last
      if (j != INT_MAX) {
        const float* xr = a.rx + row * a.rD;
        const float* yr = a.ry + (int64_t)j * a.rD;
        float s = 0.0f;
        int k = 0;
        for (; k + 8 <= a.rD; k += 8) {
          float xv[8], yv[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            xv[u] = xr[k + u];
            yv[u] = yr[k + u];
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const float t = xv[u] - yv[u];
            s = __builtin_fmaf(t, t, s);
          }
        }
        for (; k < a.rD; ++k) {
          const float t = xr[k] - yr[k];
          s = __builtin_fmaf(t, t, s);
        }
        d = s;
      }
      rank = 0;
#pragma unroll
      for (int p = 0; p < KP; ++p) {
        const float dp = __shfl(d, p, G);
        const int jp = __shfl(j, p, G);
        // (equal entries, the unfilled ones, keep their order)
        rank += (before(dp, jp, d, j) || (dp == d && jp == j && p < q)) ? 1 : 0;
      }
    }
    if (q < KP && rank < a.K) {
      // the expanded form can round a zero distance to a tiny negative value
      if (a.kvalues) static_cast<float*>(a.out)[row * a.K + rank] = fmaxf(d, 0.0f);
      else static_cast<int*>(a.out)[row * a.K + rank] = j == INT_MAX ? -1 : j;   // short (block-sparse) lists
    }
  }
}

// min / max: partials are (sign * value, index) pairs; keep the smallest in
// (value, index) order, so equal values keep the lowest index.
__global__ __launch_bounds__(256) void combine_extreme_kernel(CombineArgs a) {
  const int Ec = min(a.EP, a.E - a.e0);
  const int64_t total = a.M * Ec;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = t / Ec;
    const int e = (int)(t - row * Ec);
    float v = __builtin_inff();
    int j = -1;
    for (int c = 0; c < a.C; ++c) {
      const float* p = a.part + ((int64_t)c * a.M + row) * (2 * a.EP) + 2 * e;
      const int pj = __float_as_int(p[1]);
      if (pj >= 0 && (j < 0 || p[0] < v || (p[0] == v && pj < j))) {
        v = p[0];
        j = pj;
      }
    }
    const int64_t o = row * a.E + a.e0 + e;
    if (a.arg) static_cast<int*>(a.out)[o] = j;
    else static_cast<float*>(a.out)[o] = a.ext_sign * v;
  }
}

unsigned grid_for(int64_t items) {
  const int64_t b = (items + 255) / 256;
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(b, 16384));
}

}  // namespace

hipError_t launch_combine(const CombineArgs& a, hipStream_t s) {
  if (a.M == 0) return hipSuccess;
  if (a.ext) {
    hipLaunchKernelGGL(combine_extreme_kernel, dim3(grid_for(a.M * a.EP)), dim3(256), 0, s, a);
    return hipGetLastError();
  }
  if (a.KP > 0) {
    const dim3 g(grid_for(16 * a.M));
    switch (a.KP) {
#define KRED_COMBINE_KNN(KPV)                                                                  \
  case KPV:                                                                                    \
    hipLaunchKernelGGL((combine_knn_kernel<KPV, 16>), g, dim3(256), 0, s, a);                 \
    break;
      KRED_COMBINE_KNN(1) KRED_COMBINE_KNN(4) KRED_COMBINE_KNN(8) KRED_COMBINE_KNN(10)
      KRED_COMBINE_KNN(12) KRED_COMBINE_KNN(16)
#undef KRED_COMBINE_KNN
      case 64:
        hipLaunchKernelGGL((combine_knn_kernel<64, 64>), dim3(grid_for(64 * a.M)), dim3(256), 0, s, a);
        break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  switch (a.formula) {
    case F_GRADX:
      hipLaunchKernelGGL(combine_gradx_kernel, dim3(grid_for(4 * a.M * (1 + a.D))), dim3(256), 0, s, a);
      break;
    case F_SINKHORN:
    case F_LAPLACE_LSE:
      hipLaunchKernelGGL(combine_lse_kernel, dim3(grid_for(16 * a.M)), dim3(256), 0, s, a);
      break;
    case F_VJP:
      hipLaunchKernelGGL(combine_vjp_kernel, dim3(grid_for(4 * a.M * a.D)), dim3(256), 0, s, a);
      break;
    default:
      hipLaunchKernelGGL(combine_sum_kernel, dim3(grid_for(4 * a.M * a.EP)), dim3(256), 0, s, a);
      break;
  }
  return hipGetLastError();
}

}  // namespace kred
