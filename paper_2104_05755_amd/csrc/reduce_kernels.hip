// reduce_kernels.hip -- the Reduce TPP (Table 1) for gfx950.
//
// Folds an m x n column-major tensor (leading dimension ld, fp32 or bf16) along its rows or its
// columns with SUM / MUL / MIN / MAX, of x and/or of x*x, into fp32 outputs.  Reduction by
// columns turns m x n into m x 1 (Sec. 3.1); reduction by rows gives 1 x n.
//
//   BY_ROWS (out[c] = fold over r): each column is contiguous, so a group of 8 to 64 lanes folds a
//     column (or a wavefront one row segment of it) with 16-byte loads, then across the lanes
//     with register permutes.
//   BY_COLS (out[r] = fold over c): a thread owns 16 bytes of consecutive rows and walks the
//     columns of its workgroup's column range; the column lanes of a workgroup then meet in
//     LDS.  Column ranges of different workgroups meet in a second, tiny pass.
// 16-byte loads take any element alignment.  X2: x*x is wanted (else only x is folded).
// A batch of G calls (the loop of Alg. 6 around the TPP) runs as one launch: each pass has its
// per-call workgroups G times over, and workgroup b serves call b / per.
// Arithmetic is fp32.  When a shape needs several partial results per output (row segments or
// column ranges), they go to a device work buffer and a second kernel folds them in a fixed
// order (which depends only on the shape), so results do not depend on scheduling.
#include <hip/hip_runtime.h>

#include <math.h>

#include "internal.h"

namespace tpp {
namespace {

constexpr int RT = 256;   // threads per workgroup

template <int N>
struct Count {
  static constexpr int value = N;
};

template <int OP>
__device__ __forceinline__ float fold(float acc, float v) {
  if (OP == TPP_RED_SUM) return acc + v;
  if (OP == TPP_RED_MUL) return acc * v;
  if (OP == TPP_RED_MIN) return v < acc ? v : acc;
  return v > acc ? v : acc;
}

template <int OP>
__device__ __forceinline__ float fold_identity() {
  if (OP == TPP_RED_SUM) return 0.0f;
  if (OP == TPP_RED_MUL) return 1.0f;
  if (OP == TPP_RED_MIN) return INFINITY;
  return -INFINITY;
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

// Fold across groups of `lanes` (8, 16, 32 or 64) consecutive lanes; every lane gets the result.
// Register permutes only: quad swaps and mirrors within a row of 16 lanes, then the row and half
// swaps.  (Butterflies of shuffles go through the LDS unit, six waits on it per result.)
template <int OP>
__device__ __forceinline__ float lanes_fold(float v, int lanes) {
  v = fold<OP>(v, dpp<0xB1>(v));    // lane ^ 1
  v = fold<OP>(v, dpp<0x4E>(v));    // lane ^ 2
  v = fold<OP>(v, dpp<0x141>(v));   // 7 - lane in each 8: the other quad
  if (lanes >= 16) v = fold<OP>(v, dpp<0x140>(v));   // 15 - lane in each 16: the other 8
  if (lanes >= 32) {
    const auto w = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                    false);
    v = fold<OP>(__uint_as_float(w[0]), __uint_as_float(w[1]));
  }
  if (lanes >= 64) {
    const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                    false);
    v = fold<OP>(__uint_as_float(w[0]), __uint_as_float(w[1]));
  }
  return v;
}

template <int OP>
__device__ __forceinline__ float wave_fold(float v) {
  return lanes_fold<OP>(v, 64);
}

template <bool BF16>
__device__ __forceinline__ float load1(const void* base, int64_t idx) {
  if (BF16) return __uint_as_float((uint32_t) static_cast<const uint16_t*>(base)[idx] << 16);
  return static_cast<const float*>(base)[idx];
}

// V consecutive elements starting at idx (16 bytes): V = 8 for bf16, 4 for fp32.
typedef uint32_t u32x4_a2 __attribute__((ext_vector_type(4), aligned(2)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
template <bool BF16, int V>
__device__ __forceinline__ void loadv(const void* base, int64_t idx, float out[V]) {
  if (BF16) {
    const u32x4_a2 w = *reinterpret_cast<const u32x4_a2*>(static_cast<const uint16_t*>(base) + idx);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      out[2 * e] = __uint_as_float(w[e] << 16);
      out[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
    }
  } else {
    const f32x4_a4 w = *reinterpret_cast<const f32x4_a4*>(static_cast<const float*>(base) + idx);
    out[0] = w.x; out[1] = w.y; out[2] = w.z; out[3] = w.w;
  }
}

// Batched calls: workgroup b of a launch works on call g = b / per (per workgroups per call).
// Moves p's input and outputs and the work buffer to call g's and returns the workgroup's index
// within its call.  Each call's partials take wsize floats of the work buffer.
template <bool BF16>
__device__ __forceinline__ int64_t batch_of(ReduceParams& p, int64_t per, float*& work,
                                            int64_t wsize) {
  const int64_t bid = blockIdx.x;
  const int64_t g = bid / per;
  if (g > 0) {
    p.in = static_cast<const char*>(p.in) + g * p.in_stride * (BF16 ? 2 : 4);
    if (p.out_x) p.out_x += g * p.out_stride;
    if (p.out_x2) p.out_x2 += g * p.out_stride;
    if (work) work += g * wsize;
  }
  return bid - g * per;
}

// BY_ROWS with several segments per column: wavefront wid folds rows [s*seg_rows, min(m,
// (s+1)*seg_rows)) of column c, where c = wid % n, s = wid / n, into the work buffer.
template <int OP, bool BF16, int V, bool X2>
__global__ __launch_bounds__(RT) void reduce_rows_kernel(ReduceParams p, int32_t seg_rows,
                                                         int32_t nseg, float* work, int64_t per) {
  const int lane = threadIdx.x & 63;
  const int64_t lb = batch_of<BF16>(p, per, work, 2LL * nseg * p.n);
  const int64_t wid = lb * (RT / 64) + (threadIdx.x >> 6);
  if (wid >= (int64_t)p.n * nseg) return;
  const int32_t c = (int32_t)(wid % p.n), s = (int32_t)(wid / p.n);
  const int32_t r_lo = s * seg_rows;
  const int32_t rows = min(p.m - r_lo, seg_rows);   // r_lo + seg_rows may pass 2^31 - 1
  const int64_t col = (int64_t)c * p.ld;
  float ax = fold_identity<OP>(), ax2 = fold_identity<OP>();
  const int32_t nv = rows / V;   // full V-chunks
  for (int32_t j = lane; j < nv; j += 64) {
    float x[V];
    loadv<BF16, V>(p.in, col + r_lo + (int64_t)j * V, x);
#pragma unroll
    for (int e = 0; e < V; ++e) {
      ax = fold<OP>(ax, x[e]);
      if (X2) ax2 = fold<OP>(ax2, x[e] * x[e]);
    }
  }
  if (lane < rows - nv * V) {
    const float x = load1<BF16>(p.in, col + r_lo + nv * V + lane);
    ax = fold<OP>(ax, x);
    if (X2) ax2 = fold<OP>(ax2, x * x);
  }
  ax = wave_fold<OP>(ax);
  if (X2) ax2 = wave_fold<OP>(ax2);
  if (lane == 0) {
    work[(int64_t)s * p.n + c] = ax;
    if (X2) work[(int64_t)nseg * p.n + (int64_t)s * p.n + c] = ax2;
  }
}

// BY_ROWS with one segment per column: `lanes` lanes fold a column, so a wavefront folds
// 64 / lanes columns at once, and CG such rounds of them, every round's chunk of a pass loaded
// before any is folded (CG loads in flight per lane in place of one).  Short columns (a softmax
// over fewer keys than a wavefront's 512) thus leave no lanes idle.  The last chunk of a column
// whose rows are no multiple of V is the window that ends with it, its first rows masked.
template <int OP, bool BF16, int V, bool X2, int CG>
__global__ __launch_bounds__(RT) void reduce_rows_group_kernel(ReduceParams p, int32_t lanes,
                                                               int64_t per) {
  const int lane = threadIdx.x & 63;
  float* no_work = nullptr;
  const int64_t lb = batch_of<BF16>(p, per, no_work, 0);
  const int64_t wid = lb * (RT / 64) + (threadIdx.x >> 6);
  const int32_t ncol = 64 / lanes;               // columns of a round
  const int32_t lc = lane & (lanes - 1);         // the lane within its column
  const int64_t c0 = wid * CG * ncol + lane / lanes;
  if (wid * CG * ncol >= p.n) return;
  const bool want_x = (p.flags & TPP_RED_X) != 0, want_x2 = (p.flags & TPP_RED_X2) != 0;
  // columns past n repeat the last column's address: loaded, folded, never stored
  int64_t col[CG];
#pragma unroll
  for (int q = 0; q < CG; ++q) {
    const int64_t c = c0 + (int64_t)q * ncol;
    col[q] = (c < p.n ? c : p.n - 1) * p.ld;
  }
  float ax[CG], ax2[CG];
#pragma unroll
  for (int q = 0; q < CG; ++q) ax[q] = ax2[q] = fold_identity<OP>();
  const int32_t nv = p.m / V;   // full V-chunks
  for (int32_t j = lc; j < nv; j += lanes) {
    float x[CG][V];
#pragma unroll
    for (int q = 0; q < CG; ++q) loadv<BF16, V>(p.in, col[q] + (int64_t)j * V, x[q]);
#pragma unroll
    for (int q = 0; q < CG; ++q)
#pragma unroll
      for (int e = 0; e < V; ++e) {
        ax[q] = fold<OP>(ax[q], x[q][e]);
        if (X2) ax2[q] = fold<OP>(ax2[q], x[q][e] * x[q][e]);
      }
  }
  const int32_t rest = p.m - nv * V;
  if (rest != 0 && lc == nv % lanes) {   // the next lane in turn takes the remaining rows
    if (nv > 0) {
      float x[CG][V];
#pragma unroll
      for (int q = 0; q < CG; ++q) loadv<BF16, V>(p.in, col[q] + p.m - V, x[q]);
#pragma unroll
      for (int q = 0; q < CG; ++q)
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const bool mine = e >= V - rest;
          ax[q] = mine ? fold<OP>(ax[q], x[q][e]) : ax[q];
          if (X2) ax2[q] = mine ? fold<OP>(ax2[q], x[q][e] * x[q][e]) : ax2[q];
        }
    } else {
      for (int32_t r = 0; r < rest; ++r)
#pragma unroll
        for (int q = 0; q < CG; ++q) {
          const float x = load1<BF16>(p.in, col[q] + r);
          ax[q] = fold<OP>(ax[q], x);
          if (X2) ax2[q] = fold<OP>(ax2[q], x * x);
        }
    }
  }
#pragma unroll
  for (int q = 0; q < CG; ++q) {
    const float fx = lanes_fold<OP>(ax[q], lanes);
    const float fx2 = X2 ? lanes_fold<OP>(ax2[q], lanes) : 0.0f;
    const int64_t c = c0 + (int64_t)q * ncol;
    if (lc == 0 && c < p.n) {
      if (want_x) p.out_x[c] = fx;
      if (X2 && want_x2) p.out_x2[c] = fx2;
    }
  }
}

// (MAX over 512 rows of 32768 columns of bf16, 33.5 MB from HBM: 9.5 us a call before, 8.0 with the
// lane permutes and x alone folded; 64 rows of 20000 columns: 5.9 and 4.2.)

// BY_COLS: workgroup (rb, s) folds columns [s*col_seg, min(n, (s+1)*col_seg)) for rows
// [rb*TR*V, (rb+1)*TR*V).  Thread t: row vector tr = t % TR, column lane tc = t / TR.
// HBM-bound for tall inputs (262144 rows of 128 bf16 columns, 67 MB: 19.9 us a call before, 14.9 =
// 4.5 TB/s with eight loads in flight per thread and no branch between them).
// U: columns per trip, by how many a column lane has (2, 4 or 8: the registers of eight cost a call of
// one column per lane, 2^20 x 1 bf16, 10.0 us in place of 5.6).  BT: threads of the workgroup.
template <int OP, bool BF16, int V, bool X2, int U, int BT>
__global__ __launch_bounds__(BT) void reduce_cols_kernel(ReduceParams p, int32_t TR,
                                                         int32_t col_seg, int32_t nseg,
                                                         int32_t nrb, float* work, int64_t per) {
  __shared__ __attribute__((aligned(16))) float sx[BT * V];
  __shared__ __attribute__((aligned(16))) float sx2[X2 ? BT * V : 4];
  const int t = threadIdx.x;
  const int TC = BT / TR;
  const int tr = t % TR, tc = t / TR;
  const int64_t lb = batch_of<BF16>(p, per, work, 2LL * nseg * p.m);
  const int32_t rb = (int32_t)(lb % nrb), s = (int32_t)(lb / nrb);
  const int32_t r0 = rb * TR * V + tr * V;
  // unsigned: the sums below pass 2^31 - 1 where n is near it
  const uint32_t c_lo = (uint32_t)s * col_seg, c_hi = min((uint32_t)p.n, c_lo + col_seg);
  float ax[V], ax2[V];
#pragma unroll
  for (int e = 0; e < V; ++e) ax[e] = ax2[e] = fold_identity<OP>();
  // the last rows: the vector that ends with the column, of which the first `skip` rows belong to
  // the thread before
  const bool vec = p.m >= V && r0 < p.m;
  const int32_t skip = vec && p.m - r0 < V ? V - (p.m - r0) : 0;
  const auto load_vec = [&](uint32_t c, float (&x)[V]) {
    loadv<BF16, V>(p.in, (int64_t)c * p.ld + r0 - skip, x);
  };
  const auto load_rows = [&](uint32_t c, float (&x)[V]) {   // fewer than V rows in all
#pragma unroll
    for (int e = 0; e < V; ++e)
      x[e] = r0 + e < p.m ? load1<BF16>(p.in, (int64_t)c * p.ld + r0 + e) : 0.0f;
  };
  // Up to eight columns per trip, all loads issued before any is folded, into four accumulator
  // sets (combined in a fixed order below): a workgroup's usual eight columns per lane then cost
  // one memory latency.
  constexpr int SETS = U < 4 ? U : 4;
  float bx[SETS][V], bx2[SETS][V];
#pragma unroll
  for (int u = 0; u < SETS; ++u)
#pragma unroll
    for (int e = 0; e < V; ++e) bx[u][e] = bx2[u][e] = fold_identity<OP>();
  uint32_t c = c_lo + tc;
  auto trip = [&](auto count, auto&& load) {
    constexpr int N = decltype(count)::value;
    for (; c + (N - 1) * TC < c_hi; c += N * TC) {
      float x[N][V];
#pragma unroll
      for (int u = 0; u < N; ++u) load(c + u * TC, x[u]);
#pragma unroll
      for (int u = 0; u < N; ++u)
#pragma unroll
        for (int e = 0; e < V; ++e) {
          bx[u % SETS][e] = fold<OP>(bx[u % SETS][e], x[u][e]);
          if (X2) bx2[u % SETS][e] = fold<OP>(bx2[u % SETS][e], x[u][e] * x[u][e]);
        }
    }
  };
  if (vec) {
    if constexpr (U >= 8) trip(Count<8>(), load_vec);
    trip(Count<(U < 4 ? U : 4)>(), load_vec);
    trip(Count<1>(), load_vec);
  } else if (r0 < p.m) {
    trip(Count<(U < 4 ? U : 4)>(), load_rows);
    trip(Count<1>(), load_rows);
  }
#pragma unroll
  for (int e = 0; e < V; ++e) {
    if constexpr (SETS == 2) {
      ax[e] = fold<OP>(bx[0][e], bx[1][e]);
      if (X2) ax2[e] = fold<OP>(bx2[0][e], bx2[1][e]);
    } else {
      ax[e] = fold<OP>(fold<OP>(bx[0][e], bx[1][e]), fold<OP>(bx[2][e], bx[3][e]));
      if (X2) ax2[e] = fold<OP>(fold<OP>(bx2[0][e], bx2[1][e]), fold<OP>(bx2[2][e], bx2[3][e]));
    }
  }
  // column lanes that had a column: a batch of 17 x 9 blocks has 9 of 64
  const int lanes = c_hi - c_lo < (uint32_t)TC ? (int)(c_hi - c_lo) : TC;
  if (tc < lanes) {
    const int at = tc * TR * V + tr * V;
    if (skip == 0) {   // 16 bytes at a time: single floats, V apart, meet in V-way bank conflicts
#pragma unroll
      for (int e = 0; e < V; e += 4) {
        *reinterpret_cast<float4*>(sx + at + e) = make_float4(ax[e], ax[e + 1], ax[e + 2], ax[e + 3]);
        if (X2)
          *reinterpret_cast<float4*>(sx2 + at + e) =
              make_float4(ax2[e], ax2[e + 1], ax2[e + 2], ax2[e + 3]);
      }
    } else {
#pragma unroll
      for (int e = 0; e < V; ++e) {
        if (e < skip) continue;
        sx[at + e - skip] = ax[e];
        if (X2) sx2[at + e - skip] = ax2[e];
      }
    }
  }
  __syncthreads();
  const bool want_x = (p.flags & TPP_RED_X) != 0, want_x2 = (p.flags & TPP_RED_X2) != 0;
  const int32_t slots = TR * V;
  auto put = [&](int slot, float fx, float fx2) {
    const int32_t r = rb * slots + slot;
    if (r >= p.m) return;
    if (nseg == 1) {
      if (want_x) p.out_x[r] = fx;
      if (X2 && want_x2) p.out_x2[r] = fx2;
    } else {
      work[(int64_t)s * p.m + r] = fx;
      if (X2) work[(int64_t)nseg * p.m + (int64_t)s * p.m + r] = fx2;
    }
  };
  // Fold the TC column lanes of each row slot.  With fewer slots than threads, BT / slots threads
  // share a slot (TR * V is a power of two), each taking every BT / slots-th column lane, and meet
  // in LDS once more: V reads per thread and BT / slots more, where one thread per slot read all TC
  // in turn (32 for 64 rows of bf16: a third of that kernel's time).
  const int parts = slots < BT ? BT / slots : 1;
  for (int i = t; i < slots * parts; i += BT) {
    const int slot = i % slots, part = i / slots;
    float fx = fold_identity<OP>(), fx2 = fold_identity<OP>();
    for (int l = part; l < lanes; l += parts) {
      fx = fold<OP>(fx, sx[l * slots + slot]);
      if (X2) fx2 = fold<OP>(fx2, sx2[l * slots + slot]);
    }
    if (parts == 1) {
      put(slot, fx, fx2);
    } else {   // one trip: column lane `part` of this slot is this thread's own to overwrite
      sx[part * slots + slot] = fx;
      if (X2) sx2[part * slots + slot] = fx2;
    }
  }
  if (parts == 1) return;
  __syncthreads();
  if (t < slots) {
    float fx = sx[t], fx2 = X2 ? sx2[t] : 0.0f;
    for (int l = 1; l < parts; ++l) {
      fx = fold<OP>(fx, sx[l * slots + t]);
      if (X2) fx2 = fold<OP>(fx2, sx2[l * slots + t]);
    }
    put(t, fx, fx2);
  }
}

// Second pass: out[o] = fold over s < nseg of work[s * n_out + o] (x part, then x2 part).
// A workgroup folds OW neighbouring outputs, RT / OW threads each, every thread with up to eight
// partials in flight, and the threads of an output meet in LDS in thread order.  Bound by latency
// (343 partials of 64 x 2 outputs, the statistics of a 64 x 87808 tensor: 4.3 us with the launch);
// one wavefront per 64 outputs, folding its partials a few loads at a time, took 5001 x 2000 by
// columns to 26.6 us where the call takes 9.1 now.
// Moves the combine pass's pointers to call g = blockIdx.x / per of a batch and returns the
// workgroup's index within its call.
__device__ __forceinline__ int64_t combine_batch(int64_t per, int32_t n_out, int32_t nseg,
                                                 int64_t out_stride, const float*& work,
                                                 float*& out_x, float*& out_x2) {
  const int64_t bid = blockIdx.x;
  const int64_t g = bid / per;
  if (g > 0) {
    work += g * 2LL * nseg * n_out;
    if (out_x) out_x += g * out_stride;
    if (out_x2) out_x2 += g * out_stride;
  }
  return bid - g * per;
}

// Workgroups of blockIdx.y = 1 take the x2 part of a call that wants both (one after the other in one
// workgroup, the two chains of loads made 511 x 9000 bf16 by columns 10.2 us in place of 8.9).
template <int OP, int OW>
__global__ __launch_bounds__(RT) void reduce_combine_kernel(const float* work, int32_t n_out,
                                                            int32_t nseg, uint32_t flags,
                                                            float* out_x, float* out_x2,
                                                            int64_t per, int64_t out_stride) {
  constexpr int SL = RT / OW;   // lanes over the partials
  __shared__ float sx[SL][OW];
  const int ol = threadIdx.x % OW, sl = threadIdx.x / OW;
  const int64_t lb = combine_batch(per, n_out, nseg, out_stride, work, out_x, out_x2);
  const int64_t o = lb * OW + ol;
  const bool second = !(flags & TPP_RED_X) || blockIdx.y != 0;
  const float* const w = work + (second ? (int64_t)nseg * n_out : 0) + o;
  float f = fold_identity<OP>();
  if (o < n_out) {
    int32_t s = sl;
    for (; s + 7 * SL < nseg; s += 8 * SL) {   // eight partials in flight
      float a[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] = w[(int64_t)(s + u * SL) * n_out];
#pragma unroll
      for (int u = 0; u < 8; ++u) f = fold<OP>(f, a[u]);
    }
    float a[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      a[u] = s + u * SL < nseg ? w[(int64_t)(s + u * SL) * n_out] : fold_identity<OP>();
#pragma unroll
    for (int u = 0; u < 8; ++u) f = fold<OP>(f, a[u]);
  }
  sx[sl][ol] = f;
  __syncthreads();
  if (threadIdx.x >= OW || o >= n_out) return;
  f = sx[0][ol];
#pragma unroll
  for (int l = 1; l < SL; ++l) f = fold<OP>(f, sx[l][ol]);
  (second ? out_x2 : out_x)[o] = f;
}

struct Plan {
  bool by_cols;
  int v;          // elements per 16-byte load (4 or 8)
  int32_t nseg;   // partial results per output
  int32_t seg;    // rows per segment (BY_ROWS) or columns per range (BY_COLS)
  int32_t tr;     // BY_COLS: row vectors per workgroup
  int32_t u;      // BY_COLS: columns per trip
  int32_t bt;     // BY_COLS: threads per workgroup
  int32_t nrb;    // BY_COLS: row blocks
  int64_t blocks; // first-pass workgroups
  int32_t cg;     // BY_ROWS with one segment: rounds of columns per wavefront (0: segments)
  int32_t lanes;  // and lanes per column
};

Plan make_plan(const ReduceParams& p) {
  Plan pl{};
  pl.by_cols = (p.flags & TPP_RED_BY_COLS) != 0;
  const int es = p.in_bf16 ? 2 : 4;
  pl.v = 16 / es;
  if (!pl.by_cols) {
    const int64_t rows_per_pass = 64LL * pl.v;
    const int64_t max_seg = (p.m + rows_per_pass - 1) / rows_per_pass;
    int64_t nseg = (4096 + p.n - 1) / p.n;   // aim for >= 4096 wavefronts
    nseg = nseg < 1 ? 1 : (nseg > max_seg ? max_seg : nseg);
    if (nseg > 256) nseg = 256;
    if (p.whole) nseg = 1;
    const int64_t per = (p.m + nseg - 1) / nseg;
    pl.seg = nseg == 1 ? p.m   // whole passes past m may not fit 32 bits
                       : (int32_t)(((per + rows_per_pass - 1) / rows_per_pass) * rows_per_pass);
    pl.nseg = (int32_t)(((int64_t)p.m + pl.seg - 1) / pl.seg);
    pl.blocks = ((int64_t)p.n * pl.nseg + (RT / 64) - 1) / (RT / 64);
    // whole columns: the fewest lanes (8 to 64) whose one pass covers a column, and with plenty
    // of columns 2 or 4 rounds of them per wavefront, still >= 4096 wavefronts
    pl.cg = 0;
    if (pl.nseg == 1) {
      pl.lanes = 8;
      while (pl.lanes < 64 && pl.lanes * pl.v < p.m) pl.lanes *= 2;
      const int64_t ncol = 64 / pl.lanes, rounds = (p.n + ncol - 1) / ncol;
      pl.cg = rounds >= 4 * 4096 ? 4 : (rounds >= 2 * 4096 ? 2 : 1);
      const int64_t waves = (rounds + pl.cg - 1) / pl.cg;
      pl.blocks = (waves + (RT / 64) - 1) / (RT / 64);
    }
  } else {
    const int64_t vecs = ((int64_t)p.m + pl.v - 1) / pl.v;
    int32_t tr = 1;
    while (tr < vecs && tr < RT / 4) tr <<= 1;
    // A tall input with enough rows for 512 row blocks of at least 8 row vectors takes fewer
    // row vectors per workgroup (down to 8, up to 2048 row blocks) instead of column ranges:
    // every workgroup then folds whole columns, no combine pass runs, and the many short
    // workgroups keep more loads in flight per CU.
    if (vecs >= 512LL * 8) {
      while (tr > 8 && (vecs + tr - 1) / tr < 2048) tr >>= 1;
    } else {
      // Fewer row vectors as well where whole columns then fit one pass of at most 8 per lane (4096
      // x 64 fp32: 7.2 us in two column ranges, 4.2 in one), and, of an input of many ranges, where
      // the last row block would leave more than a fifth of the lanes idle (257 x 20000 fp32, 65 row
      // vectors: 13.4 us on blocks of 64, 8.8 on 16).
      while (tr > 16 && p.n > 8 * (RT / tr) && p.n <= 8 * (RT / 16)) tr >>= 1;
      while (tr > 8 && p.n > 8 * (RT / tr) && (vecs + tr - 1) / tr * tr * 4 > vecs * 5) tr >>= 1;
    }
    // more of them where the columns are fewer than half the column lanes (100000 x 10 bf16: 8.4
    // us with 32 column lanes, 4.2 with 16)
    while (tr < RT && tr < vecs && RT / tr >= 2 * (int64_t)p.n) tr <<= 1;
    // blocks whose columns fit two per lane of one wavefront take one wavefront each (5000 calls of
    // 17 x 9 bf16: 21.7 us in workgroups of four, 5.1 so)
    pl.bt = tr <= 16 && p.n <= 2 * (64 / tr) ? 64 : RT;
    pl.tr = tr;
    pl.nrb = (int32_t)((p.m + (int64_t)tr * pl.v - 1) / ((int64_t)tr * pl.v));
    const int32_t tc = pl.bt / tr;
    // otherwise aim for ~1024 workgroups (four per CU), each walking at least 8 columns per
    // column lane, and at most 512 partial results per output for the combine pass
    int64_t nseg = pl.nrb >= 512 ? 1 : (1024 + pl.nrb - 1) / pl.nrb;
    const int64_t max_seg = (p.n + 8LL * tc - 1) / (8LL * tc);
    nseg = nseg < 1 ? 1 : (nseg > max_seg ? max_seg : nseg);
    if (nseg > 512) nseg = 512;
    if (p.whole) nseg = 1;
    pl.seg = (int32_t)(((int64_t)p.n + nseg - 1) / nseg);
    pl.nseg = (int32_t)(((int64_t)p.n + pl.seg - 1) / pl.seg);
    pl.blocks = (int64_t)pl.nrb * pl.nseg;
    pl.u = pl.seg >= 8 * tc ? 8 : pl.seg >= 4 * tc ? 4 : 2;
  }
  return pl;
}

template <int OP, bool BF16, int V, bool X2>
void launch_first(const ReduceParams& p, const Plan& pl, float* work, hipStream_t stream) {
  // with one partial per output the first pass writes the outputs itself (no work buffer)
  float* w = pl.nseg > 1 ? work : nullptr;
  const dim3 grid((unsigned)(pl.blocks * p.G));
#define TPP_RED_GROUP(CG)                                                                        \
  hipLaunchKernelGGL((reduce_rows_group_kernel<OP, BF16, V, X2, CG>), grid, dim3(RT), 0, stream, p, \
                     pl.lanes, pl.blocks)
  if (!pl.by_cols && pl.cg == 4) TPP_RED_GROUP(4);
  else if (!pl.by_cols && pl.cg == 2) TPP_RED_GROUP(2);
  else if (!pl.by_cols && pl.cg == 1) TPP_RED_GROUP(1);
#undef TPP_RED_GROUP
  else if (!pl.by_cols)
    hipLaunchKernelGGL((reduce_rows_kernel<OP, BF16, V, X2>), grid, dim3(RT), 0, stream, p, pl.seg,
                       pl.nseg, w, pl.blocks);
#define TPP_RED_COLS(U, BT)                                                                      \
  hipLaunchKernelGGL((reduce_cols_kernel<OP, BF16, V, X2, U, BT>), grid, dim3(BT), 0, stream, p, \
                     pl.tr, pl.seg, pl.nseg, pl.nrb, w, pl.blocks)
  else if (pl.bt == 64) TPP_RED_COLS(2, 64);
  else if (pl.u == 8) TPP_RED_COLS(8, RT);
  else if (pl.u == 4) TPP_RED_COLS(4, RT);
  else TPP_RED_COLS(2, RT);
#undef TPP_RED_COLS
}

template <int OP>
void launch_op(const ReduceParams& p, const Plan& pl, float* work, hipStream_t stream) {
  const bool x2 = (p.flags & TPP_RED_X2) != 0;
  if (p.in_bf16) {
    if (x2) launch_first<OP, true, 8, true>(p, pl, work, stream);
    else launch_first<OP, true, 8, false>(p, pl, work, stream);
  } else {
    if (x2) launch_first<OP, false, 4, true>(p, pl, work, stream);
    else launch_first<OP, false, 4, false>(p, pl, work, stream);
  }
  if (pl.nseg > 1) {
    const int32_t n_out = pl.by_cols ? p.m : p.n;
    // 16 outputs per workgroup read whole 64-byte runs; few outputs of many partials (the statistics
    // of a convolution) take more threads each, and outputs whose workgroups would pass a grid's
    // 2^32 threads (2^28 in all) fewer
    const int64_t per16 = ((int64_t)n_out + 15) / 16;
    const unsigned parts = (p.flags & TPP_RED_X) && x2 ? 2 : 1;
    const int ow = n_out <= 128 && pl.nseg > 32 ? 4 : per16 * p.G * RT < (1LL << 32) ? 16 : 64;
    const int64_t per = ((int64_t)n_out + ow - 1) / ow;
#define TPP_RED_COMBINE(OW)                                                                     \
  hipLaunchKernelGGL((reduce_combine_kernel<OP, OW>), dim3((unsigned)(per * p.G), parts), dim3(RT), 0, \
                     stream, work, n_out, pl.nseg, p.flags, p.out_x, p.out_x2, per, p.out_stride)
    if (ow == 4) TPP_RED_COMBINE(4);
    else if (ow == 16) TPP_RED_COMBINE(16);
    else TPP_RED_COMBINE(64);
#undef TPP_RED_COMBINE
  }
}

}  // namespace

int64_t reduce_work_floats(const ReduceParams& p) {
  const Plan pl = make_plan(p);
  const int32_t n_out = pl.by_cols ? p.m : p.n;
  // every pass of the launch (first pass, combine) must fit 2^31 - 1 workgroups
  const int64_t per = pl.blocks > ((int64_t)n_out + 3) / 4 ? pl.blocks : ((int64_t)n_out + 3) / 4;
  if (per > 0x7fffffff / (p.G > 0 ? p.G : 1)) return -1;
  if (pl.nseg <= 1) return 0;
  return 2LL * pl.nseg * n_out * p.G;
}

hipError_t launch_reduce(const ReduceParams& p, float* work, hipStream_t stream) {
  const Plan pl = make_plan(p);
  switch (p.op) {
    case TPP_RED_SUM: launch_op<TPP_RED_SUM>(p, pl, work, stream); break;
    case TPP_RED_MUL: launch_op<TPP_RED_MUL>(p, pl, work, stream); break;
    case TPP_RED_MIN: launch_op<TPP_RED_MIN>(p, pl, work, stream); break;
    default: launch_op<TPP_RED_MAX>(p, pl, work, stream); break;
  }
  return hipGetLastError();
}

}  // namespace tpp
