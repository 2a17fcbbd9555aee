// embedding_kernels.hip -- the sparse embedding gather-reduce of Alg. 5 for gfx950.
//
// One wavefront per bag.  A table row is split into 16-byte chunks (4 fp32 or 8 bf16 entries, at
// any alignment; a row that is no multiple of them ends with the 16-byte window that ends with it,
// whose first entries the chunk before computes too, to the same bits); lpr lanes cover one row's
// chunks (all of them when the row has at most 64 chunks) and the wavefront's 64 / lpr row slots
// take every slot-th listed index, so one load instruction reads that many rows.  Each slot keeps U
// rows in flight, which plays the part of Alg. 5's unrolled accumulators and next-row prefetch.
// The indices come 64 to a load, a lane each, and reach their slots through shuffles (rows of one or
// two chunks: every slot loads its own).  Lists of a few short rows go an entry per lane.  The slots
// meet through cross-lane shuffles, halving their number each time, and the accumulation order
// depends only on the bag's list, so results do not vary between runs.  The sum is fp32 in
// registers and each output row is stored once.  Rows shorter than a chunk take an entry-per-lane
// kernel.  Indices outside [0, M) add nothing (the table is never read outside its rows).
//
// Bound by HBM on rows of 512 bytes, by the latency of the chain index - row - fold on short ones.
// 16384 bags of 1 to 64 rows, 1M-row tables larger than the last-level cache: 128 fp32 52.2 us with
// an index load in front of every U rows, 47.5 with one per 64; with the next U indices loaded
// behind the rows 58.4.  100 bf16 (not whole chunks) 156 entry by entry, 29.4 in chunks; 16 bf16
// (32 slots, folded one after the other before) 46.5 and 13.7; 13 fp32 72.6 and 15.8.
#include <hip/hip_runtime.h>

#include "brgemm_device.h"
#include "internal.h"

namespace tpp {
namespace {

using namespace dev;

constexpr int ET = 256;   // threads per workgroup: 4 wavefronts, one bag each
constexpr int U = 4;      // rows in flight per row slot

// V entries of a 16-byte chunk, widened to fp32 (bf16: the top half of an fp32, exact).
template <bool W_BF16, int V>
__device__ __forceinline__ void widen16(u32x4 w, float (&x)[V]) {
  if constexpr (W_BF16) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x[2 * e] = __uint_as_float(w[e] << 16);
      x[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = __uint_as_float(w[e]);
  }
}

// N consecutive output entries at o, at any alignment (rounded to bf16 or stored as fp32).
template <bool OUT_BF16, int N>
__device__ __forceinline__ void store_row_part(void* o, const float (&v)[N]) {
  if constexpr (OUT_BF16 && N == 8)
    gst<u32x4_a2>(o, (u32x4){pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                             pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])});
  else if constexpr (OUT_BF16 && N == 4)
    gst<u32x2_a2>(o, (u32x2){pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])});
  else if constexpr (OUT_BF16)
    gst<uint16_t>(o, f32_to_bf16_bits(v[0]));
  else if constexpr (N == 1)
    gst<float>(o, v[0]);
  else
#pragma unroll
    for (int g = 0; g < N / 4; ++g)
      gst<f32x4_a4>(static_cast<float*>(o) + 4 * g,
                    (f32x4){v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]});
}

// Entry `at` of the table, widened to fp32.
template <bool W_BF16>
__device__ __forceinline__ float load_entry(const void* W, int64_t at) {
  return W_BF16 ? bf16_bits_to_f32(gld<uint16_t>(static_cast<const uint16_t*>(W) + at))
                : gld<float>(static_cast<const float*>(W) + at);
}

// 16-byte chunk path: E >= V, any stride and alignment.
// lpr lanes per row (chunks c0 + lane % lpr of a column group), rpw = 64 / lpr row slots.
// FORM, by the row's length: LONG_ROWS; SHORT_ROWS, of at most 64 entries, with a path for lists of a few
// rows; TINY_ROWS, of at most two chunks, whose slots load their own indices as well.  (In one kernel,
// longer rows lose 10 % by the code and registers of the shorter ones' paths.)
enum { LONG_ROWS, SHORT_ROWS, TINY_ROWS };
template <bool W_BF16, bool OUT_BF16, int FORM>
__global__ __launch_bounds__(ET) void embedding_vec_kernel(EmbeddingParams p, int32_t lpr,
                                                           int32_t rpw, int32_t half) {
  constexpr int V = W_BF16 ? 8 : 4;
  constexpr int ES = W_BF16 ? 2 : 4;
  const int lane = threadIdx.x & 63;
  const int64_t b = (int64_t)blockIdx.x * (ET / 64) + (threadIdx.x >> 6);
  if (b >= p.n_bags) return;   // b is the same for the whole wavefront
  const int64_t j0 = p.begin[b], j1 = p.begin[b + 1];
  if (FORM != LONG_ROWS && j1 - j0 <= U) {
    // A few short rows: an entry per lane, every row in flight, nothing to meet (20000 bags of 1 to 3
    // rows of 9 bf16: 12.8 us in chunks, 5.5 so).
    float x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t row = j0 + u < j1 ? gld<int64_t>(p.idx + j0 + u) : -1;
      x[u] = lane < p.E && row >= 0 && row < p.M ? load_entry<W_BF16>(p.W, row * p.ldw + lane) : 0.0f;
    }
    float acc = 0.0f;
#pragma unroll
    for (int u = 0; u < U; ++u) acc += x[u];
    const float v[1] = {acc};
    if (lane < p.E)
      store_row_part<OUT_BF16, 1>(static_cast<char*>(p.out) + (b * p.ldo + lane) * (OUT_BF16 ? 2 : 4), v);
    return;
  }
  const int32_t cpr = (p.E - 1) / V + 1;
  const int r = lane / lpr, cl = lane - (lane / lpr) * lpr;
  const bool slot_ok = r < rpw;
  const int32_t nb = 64 - 64 % rpw;   // indices per block: whole rounds of the slots
  const char* wb = static_cast<const char*>(p.W);
  for (int32_t c0 = 0; c0 < cpr; c0 += lpr) {
    const int32_t c = c0 + cl;
    const bool ok = slot_ok && c < cpr;
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.0f;
    // the first entry of the chunk; the last chunk is the window that ends with the row
    const int32_t e0 = c < p.E / V ? c * V : p.E - V;
    // adds U rows: row_at(u) is the u-th that this lane's slot takes, or one outside the table
    const auto add_rows = [&](auto&& row_at) {
      u32x4 x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t row = row_at(u);
        const bool take = ok && row >= 0 && row < p.M;
        x[u] = take ? (u32x4)gld<u32x4_a2>(wb + (row * p.ldw + e0) * ES) : (u32x4){0u, 0u, 0u, 0u};
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float v[V];
        widen16<W_BF16, V>(x[u], v);
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] += v[e];
      }
    };
    if constexpr (FORM == TINY_ROWS) {
      // 64 indices would fill no more than two rows per slot (one bag of 1000 rows of 4 fp32: 9.5 us
      // from 64 indices at a time, 4.4 so)
      for (int64_t t = j0; t < j1; t += rpw * U) {
        int64_t row[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int64_t at = t + u * rpw + r;
          row[u] = at < j1 ? gld<int64_t>(p.idx + at) : -1;
        }
        add_rows([&](int u) { return row[u]; });
      }
    } else {
      for (int64_t jb = j0; jb < j1; jb += nb) {
        // lane l holds index jb + l; every slot takes its own from there
        const int32_t left = j1 - jb < nb ? (int32_t)(j1 - jb) : nb;
        const int64_t mine = lane < left ? gld<int64_t>(p.idx + jb + lane) : -1;
        for (int32_t t = 0; t < left; t += rpw * U)
          add_rows([&](int u) {
            const int32_t at = t + u * rpw + r;
            const int64_t row = __shfl(mine, at & 63, 64);
            return at < left ? row : -1;
          });
      }
    }
    // slot s adds slot s + h, for h = the half (rounded up to a power of two) of the slots left
    for (int h = half; h > 0; h >>= 1) {
      const bool adds = r < h && r + h < rpw;
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const float t = __shfl(acc[e], lane + h * lpr, 64);
        if (adds) acc[e] += t;
      }
    }
    if (r == 0 && c < cpr) {
      char* ob = static_cast<char*>(p.out) + (b * p.ldo + e0) * (OUT_BF16 ? 2 : 4);
      store_row_part<OUT_BF16, V>(ob, acc);
    }
  }
}

// Entry-per-lane path for rows shorter than a chunk.
template <bool W_BF16, bool OUT_BF16>
__global__ __launch_bounds__(ET) void embedding_elem_kernel(EmbeddingParams p) {
  const int lane = threadIdx.x & 63;
  const int64_t b = (int64_t)blockIdx.x * (ET / 64) + (threadIdx.x >> 6);
  if (b >= p.n_bags) return;
  const int64_t j0 = p.begin[b], j1 = p.begin[b + 1];
  for (int32_t e = lane; e < p.E; e += 64) {
    float acc = 0.0f;
    for (int64_t j = j0; j < j1; ++j) {
      const int64_t row = gld<int64_t>(p.idx + j);
      if (row < 0 || row >= p.M) continue;
      acc += load_entry<W_BF16>(p.W, row * p.ldw + e);
    }
    const float v[1] = {acc};
    char* ob = static_cast<char*>(p.out) + (b * p.ldo + e) * (OUT_BF16 ? 2 : 4);
    store_row_part<OUT_BF16, 1>(ob, v);
  }
}

template <bool W_BF16, bool OUT_BF16>
void launch_typed(const EmbeddingParams& p, dim3 grid, hipStream_t stream) {
  constexpr int V = W_BF16 ? 8 : 4;
  if (p.E >= V) {
    const int32_t cpr = (p.E - 1) / V + 1;
    const int32_t lpr = cpr < 64 ? cpr : 64, rpw = 64 / lpr;
    int32_t half = 0;   // largest power of two below the number of row slots
    for (int32_t h = 1; h < rpw; h *= 2) half = h;
#define TPP_EMBED(FORM)                                                                          \
  hipLaunchKernelGGL((embedding_vec_kernel<W_BF16, OUT_BF16, FORM>), grid, dim3(ET), 0, stream, p, \
                     lpr, rpw, half)
    if (cpr <= 2) TPP_EMBED(TINY_ROWS);
    else if (p.E <= 64) TPP_EMBED(SHORT_ROWS);
    else TPP_EMBED(LONG_ROWS);
#undef TPP_EMBED
  } else {
    hipLaunchKernelGGL((embedding_elem_kernel<W_BF16, OUT_BF16>), grid, dim3(ET), 0, stream, p);
  }
}

}  // namespace

hipError_t launch_embedding(const EmbeddingParams& p, hipStream_t stream) {
  const int64_t blocks = (p.n_bags + ET / 64 - 1) / (ET / 64);
  if (blocks > 0x7fffffff) return hipErrorInvalidConfiguration;
  const dim3 grid((uint32_t)blocks);
  if (p.w_bf16)
    p.out_bf16 ? launch_typed<true, true>(p, grid, stream) : launch_typed<true, false>(p, grid, stream);
  else
    p.out_bf16 ? launch_typed<false, true>(p, grid, stream) : launch_typed<false, false>(p, grid, stream);
  return hipGetLastError();
}

}  // namespace tpp
