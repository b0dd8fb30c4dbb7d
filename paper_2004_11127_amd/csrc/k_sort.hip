// Spatial order of the two clouds for the small-D paths: a stable radix sort of
// x and of y along a Hilbert curve over their joint bounding box, so that 64
// consecutive columns (and a workgroup's rows) lie close together and column
// tiles can be left out by their bounding boxes.  (A Morton curve, whose jumps
// stretch the boxes, leaves twice as many subtiles to a group of 16 rows.)
//
// The key of a point has 24 / D bits per axis; three passes of eight
// bits, each a histogram per block of 2048 points, a prefix over the blocks
// of every digit, and a scatter in which each wave ranks its points by ballots,
// so equal keys keep their order and the result is the same on every run.
// Both clouds go through the same launches (blocks of one cloud, then of the
// other), and the first histogram is taken where the keys are made.  Latency
// and launches bound it, so up to 2^17 points a cloud every scatter adds up the blocks
// before its own by itself, and where 16 bits leave few points a cell (D <= 2, the lists
// of 2^15 points at D = 3 and of 2^14 at D = 4) two passes do: four launches instead of
// nine.  us, nine launches and four: 10 nearest of 6000 x 7000 points, D = 2 91 -> 72; of a
// mixture at D = 3, 32 000 x 32 000 129 -> 117, at 65 000 181 -> 184 and at D = 4 258 ->
// 309; gradient of a mixture at D = 3, about 10^5 x 10^5, 3230 -> 3290.  (Histograms of the later passes by
// atomics in the scatter before: 60 us slower at 200 000 points.)  (A
// library sort would clear its counters with memory-set nodes, which a caller
// that captures the reduction in a graph must not get.)
#include "kred_internal.h"

namespace kred {
namespace {

constexpr int kSortBlock = 2048;              // points per workgroup
constexpr int kSortRounds = kSortBlock / 256; // points per lane
constexpr int64_t kSortSmall = 131072;        // points a cloud of the short form

// cell of one coordinate: floor of its share of the box, 24 / D bits
__device__ __forceinline__ unsigned int cell_of(float v, float lo, float inv, int bits) {
  const float top = (float)((1 << bits) - 1);
  return (unsigned int)fminf(fmaxf((v - lo) * inv, 0.0f), top);
}

// Place of a cell along the Hilbert curve (J. Skilling, "Programming the Hilbert
// curve", AIP Conf. Proc. 707, 2004: the axes are brought to the curve's
// transposed bits by exchanges and inversions from the top bit down, then a
// Gray decoding).
__device__ __forceinline__ unsigned int hilbert_key(unsigned int (&q)[kFastMaxD], int D, int bits) {
  if (D == 1) return q[0];
  for (unsigned int top = 1u << (bits - 1); top > 1u; top >>= 1) {
    const unsigned int low = top - 1u;
#pragma unroll
    for (int d = 0; d < kFastMaxD; ++d) {
      if (d >= D) break;
      if (q[d] & top) {
        q[0] ^= low;
      } else {
        const unsigned int t = (q[0] ^ q[d]) & low;
        q[0] ^= t;
        q[d] ^= t;
      }
    }
  }
#pragma unroll
  for (int d = 1; d < kFastMaxD; ++d)
    if (d < D) q[d] ^= q[d - 1];
  unsigned int last = 0u, t = 0u;
#pragma unroll
  for (int d = 0; d < kFastMaxD; ++d)
    if (d < D) last = q[d];
  for (unsigned int top = 1u << (bits - 1); top > 1u; top >>= 1)
    if (last & top) t ^= top - 1u;
  unsigned int key = 0u;
  for (int k = bits - 1; k >= 0; --k)
#pragma unroll
    for (int d = 0; d < kFastMaxD; ++d)
      if (d < D) key = (key << 1) | (((q[d] ^ t) >> k) & 1u);
  return key;
}

// The key's axes.  A cell is the floor of a coordinate's share of the box, unless
// the data leave most cells of that grid empty, which a few far points, clusters far
// apart or a heavy tail bring about: all near points would share a few cells and the
// order would separate nothing (10^5 x 10^5 points, one at 1000 times the cloud's
// extent: 10 nearest 0.26 -> 5.4 ms).  Then the share is of the points instead,
// linear between the sample's quantiles (and the box): monotone, so neighbours along
// the axis stay neighbours.  Emptiness: the box's width times the integral of the
// squared density, 1 for a uniform cloud, about 2.5 for a normal one, 8 where an
// eighth of the cells would be filled.  (Coincident knots don't count: no grid
// separates equal values.)
struct Axis {
  float lo, inv;          // linear: offset and cells per unit
  float knot[kKnots + 2]; // box, quantiles, box
  int share;
};
__device__ __forceinline__ void make_axis(const FastGuard* g, int d, int bits, Axis* ax) {
  // 32 lanes: lane k has the interval between knots k and k + 1
  const int k = threadIdx.x & 31;
  const float lo = fdec(g->lo[d]), hi = fdec(g->hi[d]), w = hi - lo;
  const float q = g->knot[d][k];
  const float len = k < kKnots - 1 ? g->knot[d][k + 1] - q : 0.0f;
  float s = len > 0.0f ? 1.0f / len : 0.0f;
  for (int o = 16; o > 0; o >>= 1) s += __shfl_xor(s, o, 32);
  ax->knot[k + 1] = fminf(fmaxf(q, lo), hi);
  if (k == 0) {
    ax->lo = lo;
    ax->inv = w > 0.0f ? (float)(1 << bits) / w : 0.0f;
    ax->knot[0] = lo;
    ax->knot[kKnots + 1] = hi;
    ax->share = s * w > 8.0f * kKnots * kKnots;
  }
}
__device__ __forceinline__ unsigned int axis_cell(const Axis& ax, float v, int bits) {
  if (!ax.share) return cell_of(v, ax.lo, ax.inv, bits);
  // the last knot at or below v
  int k = 0;
#pragma unroll
  for (int step = 32; step > 0; step >>= 1)
    if (k + step <= kKnots && v >= ax.knot[k + step]) k += step;
  const float a = ax.knot[k], w = ax.knot[k + 1] - a;
  const float t = w > 0.0f ? fminf(fmaxf((v - a) / w, 0.0f), 1.0f) : 0.0f;
  // quantile (k - 1/2) / 32 at knot k, 0 and 1 at the ends
  const float f0 = k == 0 ? 0.0f : (float)k - 0.5f, f1 = k == kKnots ? (float)kKnots : (float)k + 0.5f;
  const float top = (float)((1 << bits) - 1);
  return (unsigned int)fminf(__builtin_fmaf(t, f1 - f0, f0) * ((float)(1 << bits) / kKnots), top);
}

struct SortBlock {
  int cloud;
  int64_t i0, n;   // first point of the block in its cloud, and the cloud's size
  int64_t base;    // the cloud's offset in the concatenated arrays
};
__device__ __forceinline__ SortBlock sort_block(const SortArgs& a) {
  SortBlock b;
  b.cloud = blockIdx.x >= (unsigned)a.nbx;
  b.i0 = (int64_t)(b.cloud ? blockIdx.x - a.nbx : blockIdx.x) * kSortBlock;
  b.n = b.cloud ? a.N : a.M;
  b.base = b.cloud ? a.M : 0;
  return b;
}

// the neighbour lists always read the order (a permutation whatever the data);
// the fast path only where it runs and the order is of use (see sort_useful)
__device__ __forceinline__ bool sort_on(const SortArgs& a) { return a.guard->sorted != 0; }

// The histogram of one 8-bit digit over the block, written for the prefix.
__device__ __forceinline__ void put_counts(const SortArgs& a, const int* h, int cloud) {
  const int nb = cloud ? a.nby : a.nbx;
  const int blk = cloud ? blockIdx.x - a.nbx : blockIdx.x;
  int* c = a.counts + (cloud ? (int64_t)256 * a.nbx : 0);
  c[(int64_t)threadIdx.x * nb + blk] = h[threadIdx.x];
}

__global__ __launch_bounds__(256) void sort_keys_kernel(SortArgs a) {
  const bool on = a.always || sort_useful(a.guard, a.D, a.scale, a.limit, a.min_range);
  if (blockIdx.x == 0 && threadIdx.x == 0) a.guard->sorted = on;
  if (!on) return;
  __shared__ int h[256];
  __shared__ Axis ax[kFastMaxD];
  h[threadIdx.x] = 0;
  const SortBlock b = sort_block(a);
  const int bits = 8 * a.passes / a.D;
  if ((int)threadIdx.x < 32 * a.D) make_axis(a.guard, threadIdx.x >> 5, bits, &ax[threadIdx.x >> 5]);
  __syncthreads();
  const float* pts = b.cloud ? a.y : a.x;
  for (int r = 0; r < kSortRounds; ++r) {
    const int64_t i = b.i0 + r * 256 + threadIdx.x;
    if (i >= b.n) break;
    unsigned int key, q[kFastMaxD];
#pragma unroll
    for (int d = 0; d < kFastMaxD; ++d) {
      if (d >= a.D) break;
      q[d] = axis_cell(ax[d], pts[i * a.D + d], bits);
    }
    key = hilbert_key(q, a.D, bits);
    a.key0[b.base + i] = key;
    atomicAdd(&h[key & 255u], 1);
  }
  __syncthreads();
  put_counts(a, h, b.cloud);
}

__global__ __launch_bounds__(256) void sort_hist_kernel(SortArgs a, const unsigned int* key, int shift) {
  if (!sort_on(a)) return;
  __shared__ int h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const SortBlock b = sort_block(a);
  for (int r = 0; r < kSortRounds; ++r) {
    const int64_t i = b.i0 + r * 256 + threadIdx.x;
    if (i < b.n) atomicAdd(&h[(key[b.base + i] >> shift) & 255u], 1);
  }
  __syncthreads();
  put_counts(a, h, b.cloud);
}

// counts[digit][block] of each cloud becomes the number of its points with the
// digit in an earlier block, one workgroup per (cloud, digit), which also
// leaves the digit's total.
__global__ __launch_bounds__(256) void sort_scan_kernel(SortArgs a) {
  if (!sort_on(a)) return;
  __shared__ int red[4];
  const int cloud = blockIdx.x >> 8, digit = blockIdx.x & 255;
  const int nb = cloud ? a.nby : a.nbx;
  int* c = a.counts + (cloud ? (int64_t)256 * a.nbx : 0) + (int64_t)digit * nb;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int run = 0;
  for (int b0 = 0; b0 < nb; b0 += 256) {
    const int t = b0 + threadIdx.x;
    const int v = t < nb ? c[t] : 0;
    int s = v;
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(s, o);
      if (lane >= o) s += u;
    }
    __syncthreads();
    if (lane == 63) red[wave] = s;
    __syncthreads();
    for (int w = 0; w < wave; ++w) s += red[w];
    if (t < nb) c[t] = run + s - v;
    run += red[0] + red[1] + red[2] + red[3];
  }
  if (threadIdx.x == 0) a.totals[blockIdx.x] = run;
}

// Stable scatter: wave w of the block owns a quarter of its points, in rounds
// of 64; a point's place is its digit's start plus the earlier
// waves' points of that digit, the wave's earlier rounds' and the lower lanes'.
__global__ __launch_bounds__(256) void sort_scatter_kernel(SortArgs a, const unsigned int* key,
                                                           const int* idx, unsigned int* key_out,
                                                           int* idx_out, int shift) {
  if (!sort_on(a)) return;
  __shared__ int base[4][256];
  __shared__ int tot[4];
  const SortBlock b = sort_block(a);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int w = 0; w < 4; ++w) base[w][threadIdx.x] = 0;
  __syncthreads();
  unsigned int k[kSortRounds];
  int v[kSortRounds];
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    const int64_t i = b.i0 + wave * (kSortBlock / 4) + r * 64 + lane;
    const bool ok = i < b.n;
    k[r] = ok ? key[b.base + i] : 0u;
    v[r] = ok ? (idx != nullptr ? idx[b.base + i] : (int)i) : -1;
    if (ok) atomicAdd(&base[wave][(k[r] >> shift) & 255u], 1);
  }
  __syncthreads();
  {
    const int nb = b.cloud ? a.nby : a.nbx;
    const int blk = b.cloud ? blockIdx.x - a.nbx : blockIdx.x;
    const int d = threadIdx.x;
    // the digits below d, then the earlier blocks' points of digit d
    const int* c = a.counts + (b.cloud ? (int64_t)256 * a.nbx : 0) + (int64_t)d * nb;
    int total = 0, before = 0;
    if (a.small) {
#pragma unroll 8
      for (int i = 0; i < nb; ++i) {
        const int n = c[i];
        total += n;
        before += i < blk ? n : 0;
      }
    } else {
      total = a.totals[256 * b.cloud + d];
      before = c[blk];
    }
    int s = total;
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(s, o);
      if (lane >= o) s += u;
    }
    if (lane == 63) tot[wave] = s;
    __syncthreads();
    for (int w = 0; w < wave; ++w) s += tot[w];
    s += before - total;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int n = base[w][d];
      base[w][d] = s;
      s += n;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortRounds; ++r) {
    const bool ok = v[r] >= 0;
    const unsigned int d = (k[r] >> shift) & 255u;
    unsigned long long same = __ballot(ok);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const unsigned long long bit = __ballot((d >> t) & 1u);
      same &= ((d >> t) & 1u) ? bit : ~bit;
    }
    const int below = __popcll(same & ((1ull << lane) - 1ull));
    int at = 0;
    if (ok) at = base[wave][d] + below;
    // the digit's first lane moves the wave's place on, after every lane read it (the
    // fences order the lanes' accesses; a wave's LDS operations run in order, so they
    // cost nothing)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (ok && below == 0) base[wave][d] += __popcll(same);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (ok) {
      key_out[b.base + at] = k[r];
      idx_out[b.base + at] = v[r];
    }
  }
}

}  // namespace

size_t sort_scratch_bytes(int64_t M, int64_t N) {
  const int64_t n = M + N;
  const int64_t nb = (M + kSortBlock - 1) / kSortBlock + (N + kSortBlock - 1) / kSortBlock;
  auto up = [](int64_t b) { return (size_t)((b + 255) / 256 * 256); };
  return 4 * up(n * 4) + up(nb * 256 * 4) + up(512 * 4);
}

// Orders both clouds; a.order_x / a.order_y are set to the permutations
// (sorted place -> index) and the sorted keys of both, inside the scratch.
hipError_t launch_sort(SortArgs& a, void* scratch, hipStream_t s) {
  const int64_t n = a.M + a.N;
  a.nbx = (int)((a.M + kSortBlock - 1) / kSortBlock);
  a.nby = (int)((a.N + kSortBlock - 1) / kSortBlock);
  auto up = [](int64_t b) { return (size_t)((b + 255) / 256 * 256); };
  char* p = static_cast<char*>(scratch);
  unsigned int* k0 = reinterpret_cast<unsigned int*>(p);
  unsigned int* k1 = reinterpret_cast<unsigned int*>(p + up(n * 4));
  int* i0 = reinterpret_cast<int*>(p + 2 * up(n * 4));
  int* i1 = reinterpret_cast<int*>(p + 3 * up(n * 4));
  const int64_t nb = a.nbx + a.nby;
  a.counts = reinterpret_cast<int*>(p + 4 * up(n * 4));
  a.totals = reinterpret_cast<int*>(p + 4 * up(n * 4) + up(nb * 256 * 4));
  a.key0 = k0;
  a.small = a.M <= kSortSmall && a.N <= kSortSmall;
  const int64_t n2 = a.D <= 2 ? (a.always ? 65536 : kSortSmall) : !a.always ? 0 : a.D == 3 ? 32768 : 16384;
  a.passes = a.small && std::max(a.M, a.N) <= n2 ? 2 : 3;
  const dim3 grid((unsigned)nb), block(256);
  hipLaunchKernelGGL(sort_keys_kernel, grid, block, 0, s, a);
  unsigned int* key[2] = {k0, k1};
  int* idx[2] = {i1, i0};
  for (int pass = 0; pass < a.passes; ++pass) {
    if (pass > 0) hipLaunchKernelGGL(sort_hist_kernel, grid, block, 0, s, a, key[pass & 1], 8 * pass);
    if (!a.small) hipLaunchKernelGGL(sort_scan_kernel, dim3(512), block, 0, s, a);
    hipLaunchKernelGGL(sort_scatter_kernel, grid, block, 0, s, a, key[pass & 1],
                       pass > 0 ? idx[pass & 1] : (const int*)nullptr, key[(pass + 1) & 1], idx[(pass + 1) & 1],
                       8 * pass);
  }
  a.order_x = idx[a.passes & 1];
  a.order_y = a.order_x + a.M;
  a.keys_x = key[a.passes & 1];
  a.keys_y = a.keys_x + a.M;
  return hipGetLastError();
}

}  // namespace kred
