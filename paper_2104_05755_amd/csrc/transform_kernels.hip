// transform_kernels.hip -- the Transform TPP (Table 1; Sec. 3.1): Transpose, VNNI formatting
// ([D1][D0] -> [D1/alpha][D0][alpha], the layout of Sec. 3.2.2) and VNNI to VNNI-transpose.
//
// All three only move entries, so they are bound by HBM traffic: each entry is read once and
// written once.  The paper builds its transposes from register shuffle networks (Sec. 3.3.1);
// here a workgroup stages a 64 x 64 tile in LDS, reading it along the input's contiguous
// direction and writing it along the output's, so both sides are coalesced.
//   - Transpose: 16-byte loads and stores at any alignment; the LDS tile keeps 16-byte chunks
//     XOR-swizzled by column, so the column-wise gathers of the write phase hit distinct banks.
//     Only blocks with an edge below the tile's move entry by entry.
//   - VNNI: no LDS: each thread writes one 16-byte chunk of an output group, gathering its
//     alpha columns with one (16 / alpha)-byte load each, at any alignment (bf16 4097 x 2049
//     16.1 -> 6.6 us against aligned operands only).
//   - VNNI to VNNI-transpose: the tiled kernel with both sides addressed in the VNNI layout,
//     16-byte chunks on whole tiles (at any alignment: bf16 4097 x 2049 20.1 -> 10.3 us against
//     aligned operands only), entry by entry on partial ones.
#include <hip/hip_runtime.h>

#include "brgemm_device.h"
#include "internal.h"

namespace tpp {
namespace {

using dev::gld;
using dev::gst;
using dev::u32x4;

typedef uint32_t u32_a2 __attribute__((aligned(2)));

constexpr int TT = 64;     // tile edge, entries
constexpr int TPB = 256;   // threads per workgroup

template <int ES>
struct Entry;
template <>
struct Entry<2> {
  using T = uint16_t;
};
template <>
struct Entry<4> {
  using T = uint32_t;
};

// 16 bytes from V entries, and entry e of a loaded chunk of `words` 32-bit words.
template <int ES>
__device__ __forceinline__ u32x4 pack16(const typename Entry<ES>::T* v) {
  if constexpr (ES == 4) {
    return (u32x4){v[0], v[1], v[2], v[3]};
  } else {
    return (u32x4){v[0] | ((uint32_t)v[1] << 16), v[2] | ((uint32_t)v[3] << 16),
                   v[4] | ((uint32_t)v[5] << 16), v[6] | ((uint32_t)v[7] << 16)};
  }
}
template <int ES>
__device__ __forceinline__ typename Entry<ES>::T entry_of(const uint32_t* words, int e) {
  if constexpr (ES == 4)
    return words[e];
  else
    return (uint16_t)(words[e >> 1] >> (16 * (e & 1)));
}

// 16 bytes at an entry's own alignment.
template <int ES>
__device__ __forceinline__ u32x4 load16(const void* src) {
  if constexpr (ES == 4)
    return gld<dev::u32x4_a4>(src);
  else
    return gld<dev::u32x4_a2>(src);
}
template <int ES>
__device__ __forceinline__ void store16(void* dst, u32x4 v) {
  if constexpr (ES == 4)
    gst<dev::u32x4_a4>(dst, v);
  else
    gst<dev::u32x4_a2>(dst, v);
}

// Position of entry (c, r) of a staged tile ([c][r], 64 entries per c) with the 16-byte chunks
// of each c XOR-swizzled by c / V: a chunk keeps its 16 bytes together, and V consecutive c of
// one r fall in different chunks.
template <int ES>
__device__ __forceinline__ int tile_pos(int c, int r) {
  constexpr int V = 16 / ES, CH = TT / V;
  return c * TT + (((r / V) ^ ((c / V) % CH)) * V) + r % V;
}

// Index b of a batched launch belongs to call g = b / per (per indices per call), whose blocks
// start g * in_stride and g * out_stride entries on; returns the index within its call.
template <typename T>
__device__ __forceinline__ uint32_t batch_of(const TransformParams& p, uint32_t b, uint32_t per,
                                             const T*& in, T*& out) {
  const uint32_t g = (uint32_t)dev::fdiv(b, p.div_per);   // grids are below 2^31
  in = static_cast<const T*>(p.in) + (int64_t)g * p.in_stride;
  out = static_cast<T*>(p.out) + (int64_t)g * p.out_stride;
  return b - g * per;
}

// The workgroup's tile (r0, c0).  In runs, tiles are numbered along the output's contiguous direction
// and each XCD (workgroup b is on XCD b % 8) takes a contiguous run of them: where rows are no whole
// 128-byte lines, the two tiles that share a line write it into the same L2, which then writes it back
// whole.  Transpose of fp32 4097 x 2049: 15.4 us in launch order along the input, 13.2 with runs per XCD
// along the input, 11.7 so.  Else in launch order along the input (tiles_in_runs).
template <typename T>
__device__ __forceinline__ void tile_of(const TransformParams& p, uint32_t per, const T*& in,
                                        T*& out, int32_t& r0, int32_t& c0) {
  if (p.run == 0) {
    const uint32_t t = batch_of<T>(p, blockIdx.x, per, in, out);
    const uint32_t tn = (uint32_t)dev::fdiv(t, p.div_m);
    r0 = (int32_t)(t - tn * p.tiles_m) * TT;
    c0 = (int32_t)tn * TT;
    return;
  }
  const uint32_t x = blockIdx.x % 8;
  const uint32_t b = x * p.run + min(x, p.rest) + blockIdx.x / 8;
  const uint32_t t = batch_of<T>(p, b, per, in, out);
  const uint32_t tm = (uint32_t)dev::fdiv(t, p.div_n);
  r0 = (int32_t)tm * TT;
  c0 = (int32_t)(t - tm * p.tiles_n) * TT;
}

// Moves the 64 x 64 window at in / out, less the chunks that lie wholly in its first dc columns or
// dr rows (ALL: none).
template <int ES, bool ALL>
__device__ __forceinline__ void move_window(const typename Entry<ES>::T* in,
                                            typename Entry<ES>::T* out, int64_t ld_in,
                                            int64_t ld_out, int dr, int dc,
                                            typename Entry<ES>::T* lds) {
  constexpr int V = 16 / ES, CH = TT / V;
  const int t = threadIdx.x;
  // chunk q: column q / CH, rows (q % CH) * V .. + V - 1 of the window
  constexpr int N = TT * CH / TPB;
  u32x4 x[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int q = i * TPB + t, cc = q / CH, rv = (q % CH) * V;
    if (ALL || (cc + V > dc && rv + V > dr)) x[i] = load16<ES>(in + (int64_t)cc * ld_in + rv);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int q = i * TPB + t, cc = q / CH, rv = (q % CH) * V;
    if (ALL || (cc + V > dc && rv + V > dr))
      *reinterpret_cast<u32x4*>(lds + tile_pos<ES>(cc, rv)) = x[i];
  }
  __syncthreads();
  // chunk q: output column q / CH (an input row), entries (q % CH) * V .. + V - 1
#pragma unroll
  for (int q = t; q < TT * CH; q += TPB) {
    const int rr = q / CH, cv = (q % CH) * V;
    if (ALL || (rr >= dr && cv + V > dc)) {
      typename Entry<ES>::T v[V];
#pragma unroll
      for (int j = 0; j < V; ++j) v[j] = lds[tile_pos<ES>(cv + j, rr)];
      store16<ES>(out + (int64_t)rr * ld_out + cv, pack16<ES>(v));
    }
  }
}

// Transpose: the n x m output's entry (c, r) = in(r, c), per tiles per call.  Memory-bound.  From
// 64 x 64 up every tile is a window of 64 x 64 entries inside the block, moved in 16-byte chunks
// at any alignment: the window of a last, partial tile starts further back, and the chunks that
// lie wholly in the tiles before it are left to them (the rest of a chunk is written twice, with
// the same entries).  Smaller blocks move entry by entry.  Against entry by entry wherever bases
// or leading dimensions are no whole 16-byte units or a tile is partial: fp32 4097 x 2049
// 19.7 -> 11.9 us (5.6 TB/s), bf16 4097 x 4095 31.5 -> 12.7, 512 calls of fp32 65 x 65
// 13.6 -> 6.1, of 64 x 64 (aligned) 4.25 -> 3.9.
template <int ES>
__global__ __launch_bounds__(TPB) void transpose_kernel(TransformParams p, uint32_t per) {
  using T = typename Entry<ES>::T;
  __shared__ __attribute__((aligned(16))) T lds[TT * TT];
  const int t = threadIdx.x;
  const T* in;
  T* out;
  int32_t r0, c0;
  tile_of<T>(p, per, in, out, r0, c0);
  if (p.m >= TT && p.n >= TT) {
    // the tile's window, and the entries of it that an earlier tile moves
    const int32_t rw = min(r0, p.m - TT), cw = min(c0, p.n - TT);
    const int dr = r0 - rw, dc = c0 - cw;
    in += (int64_t)cw * p.ld_in + rw;
    out += (int64_t)rw * p.ld_out + cw;
    if (dr == 0 && dc == 0)
      move_window<ES, true>(in, out, p.ld_in, p.ld_out, 0, 0, lds);
    else
      move_window<ES, false>(in, out, p.ld_in, p.ld_out, dr, dc, lds);
  } else {
    for (int q = t; q < TT * TT; q += TPB) {
      const int cc = q / TT, rr = q % TT;
      if (r0 + rr < p.m && c0 + cc < p.n)
        lds[tile_pos<ES>(cc, rr)] = gld<T>(in + (int64_t)(c0 + cc) * p.ld_in + r0 + rr);
    }
    __syncthreads();
    for (int q = t; q < TT * TT; q += TPB) {
      const int rr = q / TT, cc = q % TT;
      if (r0 + rr < p.m && c0 + cc < p.n)
        gst<T>(out + (int64_t)(r0 + rr) * p.ld_out + c0 + cc, lds[tile_pos<ES>(cc, rr)]);
    }
  }
}

// VNNI to VNNI-transpose: logical tile rows [r0, r0 + 64), columns [c0, c0 + 64) (both multiples
// of alpha, so groups never straddle tiles), staged as lds[c][r].  Reads walk the input's
// contiguous order (c % alpha fastest, then r), writes the output's (r % alpha fastest, then c).
// Whole tiles move 16-byte chunks on both sides: an input chunk is
// V / alpha rows of one group's alpha columns, an output chunk V / alpha columns of one output
// group's alpha rows.  Output rows from m up to the next multiple of alpha are the zero
// completion of the last group (never in a whole tile).
template <int ES, int ALPHA>
__global__ __launch_bounds__(TPB) void vnni_t_kernel(TransformParams p, uint32_t per) {
  using T = typename Entry<ES>::T;
  constexpr int V = 16 / ES, CPG = TT * ALPHA / V;   // 16-byte chunks per group of a tile
  __shared__ T lds[TT][TT + 1];
  const int t = threadIdx.x;
  const T* in;
  T* out;
  int32_t r0, c0;
  tile_of<T>(p, per, in, out, r0, c0);
  if (r0 + TT <= p.m && c0 + TT <= p.n) {
    for (int q = t; q < TT * TT / V; q += TPB) {
      const int gi = q / CPG, j0 = (q % CPG) * V, rr0 = j0 / ALPHA;
      const u32x4 w4 = load16<ES>(in + (int64_t)(c0 / ALPHA + gi) * p.ld_in +
                                  (int64_t)(r0 + rr0) * ALPHA);
      const uint32_t w[4] = {w4[0], w4[1], w4[2], w4[3]};
#pragma unroll
      for (int e = 0; e < V; ++e) lds[gi * ALPHA + e % ALPHA][rr0 + e / ALPHA] = entry_of<ES>(w, e);
    }
    __syncthreads();
    for (int q = t; q < TT * TT / V; q += TPB) {
      const int gi = q / CPG, j0 = (q % CPG) * V, cc0 = j0 / ALPHA;
      T v[V];
#pragma unroll
      for (int e = 0; e < V; ++e) v[e] = lds[cc0 + e / ALPHA][gi * ALPHA + e % ALPHA];
      store16<ES>(out + (int64_t)(r0 / ALPHA + gi) * p.ld_out + (int64_t)(c0 + cc0) * ALPHA,
                  pack16<ES>(v));
    }
    return;
  }
  const int32_t m_pad = (p.m + ALPHA - 1) / ALPHA * ALPHA;
  for (int q = t; q < TT * TT; q += TPB) {
    const int a = q % ALPHA, rr = (q / ALPHA) % TT, cc = (q / (ALPHA * TT)) * ALPHA + a;
    const int32_t r = r0 + rr, c = c0 + cc;
    if (r < p.m && c < p.n)
      lds[cc][rr] = gld<T>(in + (int64_t)(c / ALPHA) * p.ld_in + (int64_t)r * ALPHA + a);
  }
  __syncthreads();
  for (int q = t; q < TT * TT; q += TPB) {
    const int a = q % ALPHA, cc = (q / ALPHA) % TT, rr = (q / (ALPHA * TT)) * ALPHA + a;
    const int32_t r = r0 + rr, c = c0 + cc;
    if (c < p.n && r < m_pad)
      gst<T>(out + (int64_t)(r / ALPHA) * p.ld_out + (int64_t)c * ALPHA + a,
             r < p.m ? lds[cc][rr] : (T)0);
  }
}

// A (16 / ALPHA)-byte load at an entry's own alignment, as 32-bit words.
template <int ES, int BYTES>
__device__ __forceinline__ void load_words(const void* src, uint32_t* w) {
  if constexpr (BYTES == 16) {
    const u32x4 x = load16<ES>(src);
    w[0] = x[0], w[1] = x[1], w[2] = x[2], w[3] = x[3];
  } else if constexpr (BYTES == 8) {
    const dev::u32x2_a2 x = gld<dev::u32x2_a2>(src);
    w[0] = x[0], w[1] = x[1];
  } else {
    w[0] = gld<u32_a2>(src);
  }
}

// VNNI formatting: thread q writes 16-byte chunk q % cpg of output group g = q / cpg (cpg chunks
// cover the group's m * ALPHA entries): entries j0 .. j0 + V - 1, i.e. rows j0 / ALPHA ..
// (j0 + V) / ALPHA - 1 of the group's ALPHA columns.  Columns past n are the zero completion.
template <int ES, int ALPHA>
__global__ __launch_bounds__(TPB) void vnni_kernel(TransformParams p, int64_t cpg, int64_t total,
                                                   uint32_t per) {
  using T = typename Entry<ES>::T;
  constexpr int V = 16 / ES, ROWS = V / ALPHA;
  const T* in;
  T* out;
  const int64_t q = (int64_t)batch_of<T>(p, blockIdx.x, per, in, out) * TPB + threadIdx.x;
  if (q >= total) return;
  const int64_t g = q / cpg;
  const int64_t j0 = (q - g * cpg) * V;
  const int64_t extent = (int64_t)p.m * ALPHA;
  T* o = out + g * p.ld_out + j0;
  if (j0 + V <= extent) {
    const int64_t r0 = j0 / ALPHA;
    T v[V];
#pragma unroll
    for (int a = 0; a < ALPHA; ++a) {
      const int64_t c = g * ALPHA + a;
      uint32_t w[(ROWS * ES + 3) / 4] = {};
      if (c < p.n) load_words<ES, ROWS * ES>(in + c * p.ld_in + r0, w);
#pragma unroll
      for (int e = 0; e < ROWS; ++e) v[e * ALPHA + a] = entry_of<ES>(w, e);
    }
    store16<ES>(o, pack16<ES>(v));
  } else {
    for (int e = 0; e < V && j0 + e < extent; ++e) {
      const int64_t j = j0 + e, r = j / ALPHA, c = g * ALPHA + j % ALPHA;
      gst<T>(o + e, c < p.n ? gld<T>(in + c * p.ld_in + r) : (T)0);
    }
  }
}

// A launch of per workgroups for each of the G calls: at most 2^31 - 1 workgroups in all.
inline bool grid_fits(int64_t per, int64_t G) { return per <= 0x7fffffff / (G > 0 ? G : 1); }

// Whether the tiles go in runs per XCD (see tile_of): always where two tiles share a 128-byte line, and
// otherwise for the sizes that gain by it.  Below the L2s' 32 MiB (in and out) and in blocks one tile wide
// launch order is faster: fp32 1024 x 1024 4.0 us and 4.9 in runs, 65536 x 64 VNNI to VNNI-transpose
// (alpha 2) 5.7 and 6.7.  So it is well past the last-level cache's 256 MiB, where eight distant runs of columns a power of two apart
// meet in the same memory channels: fp32 8192 x 8192 VNNI to VNNI-transpose 112 us (alpha 4), 129 in runs.
// In between: fp32 4096 x 4096 23.5 and 20.1, bf16 8192 x 8192 44.1 and 38.8.
inline bool tiles_in_runs(const TransformParams& p, int64_t es) {
  const auto whole = [&](const void* q, int64_t ld, int64_t stride) {
    return (reinterpret_cast<uintptr_t>(q) | (uintptr_t)(ld * es) | (uintptr_t)(stride * es)) % 128 == 0;
  };
  if (!whole(p.in, p.ld_in, p.in_stride) || !whole(p.out, p.ld_out, p.out_stride)) return true;
  const int64_t bytes = 2 * es * p.m * p.n * p.G;
  return p.m > TT && p.n > TT && bytes >= (32 << 20) && bytes <= (384 << 20);
}

template <int ES>
hipError_t launch_es(TransformParams& p, hipStream_t stream) {
  const int64_t tiles_n = (p.n + TT - 1) / TT;
  const int64_t G = p.G;
  const auto plan = [&](int64_t tiles_m, int64_t per) {   // per * G fits a grid
    p.tiles_n = (uint32_t)tiles_n;
    p.tiles_m = (uint32_t)tiles_m;
    p.div_per = FastDiv(per);
    p.div_n = FastDiv(tiles_n);
    p.div_m = FastDiv(tiles_m);
    const bool runs = tiles_in_runs(p, ES);
    p.run = runs ? (uint32_t)(per * G / 8) : 0;
    p.rest = (uint32_t)(per * G % 8);
  };
  if (p.kind == 0) {
    const int64_t tiles = (p.m + TT - 1) / TT * tiles_n;
    if (!grid_fits(tiles, G)) return hipErrorInvalidConfiguration;
    plan(tiles / tiles_n, tiles);
    hipLaunchKernelGGL(transpose_kernel<ES>, dim3((uint32_t)(tiles * G)), dim3(TPB), 0, stream, p,
                       (uint32_t)tiles);
  } else if (p.kind == 1) {
    constexpr int V = 16 / ES;
    const int64_t cpg = ((int64_t)p.m * p.alpha + V - 1) / V;
    const int64_t total = cpg * ((p.n + p.alpha - 1) / p.alpha);
    const int64_t blocks = (total + TPB - 1) / TPB;
    if (!grid_fits(blocks, G)) return hipErrorInvalidConfiguration;
    plan(1, blocks);
    const dim3 grid((uint32_t)(blocks * G));
    switch (p.alpha) {
      case 1: hipLaunchKernelGGL((vnni_kernel<ES, 1>), grid, dim3(TPB), 0, stream, p, cpg, total, (uint32_t)blocks); break;
      case 2: hipLaunchKernelGGL((vnni_kernel<ES, 2>), grid, dim3(TPB), 0, stream, p, cpg, total, (uint32_t)blocks); break;
      default: hipLaunchKernelGGL((vnni_kernel<ES, 4>), grid, dim3(TPB), 0, stream, p, cpg, total, (uint32_t)blocks); break;
    }
  } else {
    const int64_t m_pad = ((int64_t)p.m + p.alpha - 1) / p.alpha * p.alpha;
    const int64_t tiles = (m_pad + TT - 1) / TT * tiles_n;
    if (!grid_fits(tiles, G)) return hipErrorInvalidConfiguration;
    plan(tiles / tiles_n, tiles);
    const dim3 grid((uint32_t)(tiles * G));
    switch (p.alpha) {
      case 1: hipLaunchKernelGGL((vnni_t_kernel<ES, 1>), grid, dim3(TPB), 0, stream, p, (uint32_t)tiles); break;
      case 2: hipLaunchKernelGGL((vnni_t_kernel<ES, 2>), grid, dim3(TPB), 0, stream, p, (uint32_t)tiles); break;
      default: hipLaunchKernelGGL((vnni_t_kernel<ES, 4>), grid, dim3(TPB), 0, stream, p, (uint32_t)tiles); break;
    }
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_transform(TransformParams& p, hipStream_t stream) {
  return p.es == 2 ? launch_es<2>(p, stream) : launch_es<4>(p, stream);
}

}  // namespace tpp
