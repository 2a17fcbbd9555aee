// brgemm_kernels.hip -- the batch-reduce GEMM TPP kernel family for gfx950 (CDNA4).
//
// Computes, for every instance g of a launch and every (r, c) of its m x n output block,
//     C(r, c) = cvt( act( beta * C(r, c) + sum_i sum_p A_i(r, p) B_i(p, c) + bias[r] ) )
// (Table 3 BRGEMM; Sec. 2.3 variants; the epilogue TPPs of Table 1 / Table 2 fused before the
// single store as Sec. 2.1 principle 5 allows).
//
// Structure, following Alg. 2 re-tiled for the GPU:
//   - a workgroup owns one BM x BN tile of the "virtual C" of its tile group.  For a strided
//     instance grid the virtual C is the (gm*m) x (gn*n) matrix formed by the instances' output
//     blocks side by side, so a tile may fuse several neighbouring instances (they share their
//     A_i rows and B_i columns, as the ib_m / ib_n loops of Alg. 6 do); for an explicit grid the
//     virtual C is one instance's m x n block;
//   - Alg. 2's loops over the pairs i and over k become one flat loop, in steps of BK=64, over
//     stages; each stage copies an A_i panel (BM x 64) and a B_i panel (64 x BN) from HBM into
//     one of two LDS buffers with 16-byte loads, while the MFMAs consume the other buffer;
//   - A is M-contiguous in memory but the MFMA wants 8 consecutive k per lane, so every thread
//     loads an 8x8 bf16 sub-block (8 columns of 8 rows) and transposes it in registers before
//     its LDS store; B is already K-contiguous and is copied as is;
//   - fp32 accumulators stay in registers for the whole reduction (v_mfma_f32_32x32x16_bf16);
//   - the epilogue (beta*C, bias, ReLU / GELU-tanh, fp32 -> bf16) runs on the accumulators and
//     each output element is stored once.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <string>
#include <type_traits>

#include "brgemm_device.h"
#include "internal.h"

namespace tpp {
namespace {

using namespace dev;

// ---------------------------------------------------------------------------------------------
// Epilogue shared by all kernels.  The accumulator layout of a 32x32 MFMA tile: lane l holds
// column l%32, and in register v the row 8*(v/4) + 4*(l/32) + v%4.
// ---------------------------------------------------------------------------------------------
template <bool GENERIC>
__device__ __forceinline__ void store_group(const BrgemmParams& p, const Instance& in, int32_t R0,
                                            int32_t C, const float v_in[4]) {
  // Column C of the virtual C -> element offset in C (relative to the instance base).
  int64_t col_off;
  if (p.fused) {
    if (C >= p.vcols) return;
    const int32_t gi = fdiv(C, p.div_n), c = C - gi * p.n;
    col_off = (int64_t)gi * p.c_step_n + (int64_t)c * p.ldc;
  } else {
    if (C >= p.n) return;
    col_off = (int64_t)C * p.ldc;
  }
  const float* bias = p.bias;
  const bool has_bias = (p.flags & TPP_EPI_BIAS) != 0;
  if (!GENERIC) {
    // Rows of an instance padded to whole groups (p.vm % 4 == 0) and R0 % 4 == 0: the four rows
    // R0..R0+3 belong to one instance; its last group may have fewer than four rows.
    int64_t row_off, bias_idx;
    int32_t nr;
    if (p.fused) {
      if (R0 >= p.vrows) return;
      const int32_t gi = fdiv(R0, p.div_m), r = R0 - gi * p.vm;
      row_off = (int64_t)gi * p.c_step_m + r;
      bias_idx = (int64_t)gi * p.bias_step_m + r;
      nr = p.m - r;
    } else {
      if (R0 >= p.m) return;
      row_off = R0;
      bias_idx = in.bias + R0;
      nr = p.m - R0;
    }
    if (nr < 4) {
      for (int e = 0; e < nr; ++e) {
        const int64_t ei = in.c + row_off + col_off + e;
        float v1[1] = {v_in[e]};
        if (p.beta != 0.0f)
          v1[0] = p.beta * (p.c_bf16 ? bf16_bits_to_f32(static_cast<const uint16_t*>(p.c)[ei])
                                     : static_cast<const float*>(p.c)[ei]) + v1[0];
        if (has_bias) v1[0] += bias[bias_idx + e];
        if (p.flags & EPI_AUX_MASK) epi_aux<1>(p, ei, v1);
        const float o = activate(v1[0], p.flags);
        if (p.c_bf16) static_cast<uint16_t*>(p.c)[ei] = f32_to_bf16_bits(o);
        else static_cast<float*>(p.c)[ei] = o;
      }
      return;
    }
    const int64_t e0 = in.c + row_off + col_off;
    float v[4] = {v_in[0], v_in[1], v_in[2], v_in[3]};
    if (p.c_bf16) {
      uint16_t* cp = static_cast<uint16_t*>(p.c) + e0;
      const bool vec = (reinterpret_cast<uintptr_t>(cp) & 7) == 0;
      if (p.beta != 0.0f) {
        uint32_t h[4];
        if (vec) {
          const uint2 w = *reinterpret_cast<const uint2*>(cp);
          h[0] = w.x & 0xffff; h[1] = w.x >> 16; h[2] = w.y & 0xffff; h[3] = w.y >> 16;
        } else {
          for (int e = 0; e < 4; ++e) h[e] = cp[e];
        }
        for (int e = 0; e < 4; ++e) v[e] = p.beta * bf16_bits_to_f32(h[e]) + v[e];
      }
      if (has_bias)
        for (int e = 0; e < 4; ++e) v[e] += bias[bias_idx + e];
      if (p.flags & EPI_AUX_MASK) epi_aux<4>(p, e0, v);
      uint32_t o[4];
      for (int e = 0; e < 4; ++e) o[e] = f32_to_bf16_bits(activate(v[e], p.flags));
      if (vec) {
        *reinterpret_cast<uint2*>(cp) = make_uint2(o[0] | (o[1] << 16), o[2] | (o[3] << 16));
      } else {
        for (int e = 0; e < 4; ++e) cp[e] = (uint16_t)o[e];
      }
    } else {
      float* cp = static_cast<float*>(p.c) + e0;
      const bool vec = (reinterpret_cast<uintptr_t>(cp) & 15) == 0;
      if (p.beta != 0.0f) {
        if (vec) {
          const float4 w = *reinterpret_cast<const float4*>(cp);
          v[0] = p.beta * w.x + v[0]; v[1] = p.beta * w.y + v[1];
          v[2] = p.beta * w.z + v[2]; v[3] = p.beta * w.w + v[3];
        } else {
          for (int e = 0; e < 4; ++e) v[e] = p.beta * cp[e] + v[e];
        }
      }
      if (has_bias)
        for (int e = 0; e < 4; ++e) v[e] += bias[bias_idx + e];
      if (p.flags & EPI_AUX_MASK) epi_aux<4>(p, e0, v);
      for (int e = 0; e < 4; ++e) v[e] = activate(v[e], p.flags);
      if (vec) {
        *reinterpret_cast<float4*>(cp) = make_float4(v[0], v[1], v[2], v[3]);
      } else {
        for (int e = 0; e < 4; ++e) cp[e] = v[e];
      }
    }
  } else {
    for (int e = 0; e < 4; ++e) {
      const int32_t R = R0 + e;
      int64_t row_off, bias_idx;
      if (p.fused) {
        if (R >= p.vrows) continue;
        const int32_t gi = fdiv(R, p.div_m), r = R - gi * p.vm;
        row_off = (int64_t)gi * p.c_step_m + r;
        bias_idx = (int64_t)gi * p.bias_step_m + r;
      } else {
        if (R >= p.m) continue;
        row_off = R;
        bias_idx = in.bias + R;
      }
      const int64_t ei = in.c + row_off + col_off;
      float v1[1] = {v_in[e]};
      if (p.c_bf16) {
        uint16_t* cp = static_cast<uint16_t*>(p.c) + ei;
        if (p.beta != 0.0f) v1[0] = p.beta * bf16_bits_to_f32(*cp) + v1[0];
        if (has_bias) v1[0] += bias[bias_idx];
        if (p.flags & EPI_AUX_MASK) epi_aux<1>(p, ei, v1);
        *cp = f32_to_bf16_bits(activate(v1[0], p.flags));
      } else {
        float* cp = static_cast<float*>(p.c) + ei;
        if (p.beta != 0.0f) v1[0] = p.beta * *cp + v1[0];
        if (has_bias) v1[0] += bias[bias_idx];
        if (p.flags & EPI_AUX_MASK) epi_aux<1>(p, ei, v1);
        *cp = activate(v1[0], p.flags);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// bf16 kernel family
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t word(const uint4& v, int d) {
  return d == 0 ? v.x : d == 1 ? v.y : d == 2 ? v.z : v.w;
}

// Transpose an 8x8 bf16 sub-block held as 8 k-columns of 8 rows into 8 rows of 8 k, and store
// the rows (16 B each) into the K-contiguous LDS panel.
__device__ __forceinline__ void store_a_transposed(uint16_t* dst_row0, const uint4 col[8]) {
#pragma unroll
  for (int mi = 0; mi < 8; ++mi) {
    const int d = mi >> 1;
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t lo = word(col[2 * e], d), hi = word(col[2 * e + 1], d);
      w[e] = (mi & 1) ? ((lo >> 16) | (hi & 0xffff0000u)) : ((lo & 0xffffu) | (hi << 16));
    }
    *reinterpret_cast<uint4*>(dst_row0 + mi * LDS_ROW) = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// Blocks narrower than one 8-element chunk in m or k: element loads, every row, column and k checked.
template <int BM, int BN, int WAVES_M, int WAVES_N>
__global__ __launch_bounds__(NT) void brgemm_bf16_kernel(BrgemmParams p) {
  constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int KCH = BK / 8;                        // 8-element k chunks per stage
  constexpr int A_SUB = (BM / 8) * KCH;              // 8x8 sub-blocks of the A panel
  constexpr int A_REP = (A_SUB + NT - 1) / NT;
  constexpr int B_CH = BN * KCH;                     // 16-byte chunks of the B panel
  constexpr int B_REP = (B_CH + NT - 1) / NT;
  constexpr int STAGE = (BM + BN) * LDS_ROW;
  static_assert(WAVES_M * WAVES_N * 64 == NT, "4 waves");
  static_assert(TM >= 1 && TN >= 1, "wave tile at least 32x32");

  __shared__ __attribute__((aligned(16))) uint16_t lds[2 * STAGE];

  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave % WAVES_M, wn = wave / WAVES_M;
  const TileCoord tc = decode_tile(p, BM, BN);
  const Instance in = instance_of(p, tc.g);
  const int32_t ksteps = (p.k + BK - 1) / BK;
  const int64_t stages = in.npairs * ksteps;

  // Staging assignments, fixed for the whole reduction.
  int64_t a_off[A_REP][8];
  bool a_ok[A_REP][8];
  int a_kc[A_REP], a_row[A_REP];
#pragma unroll
  for (int rep = 0; rep < A_REP; ++rep) {
    const int q = t + NT * rep;
    a_kc[rep] = q % KCH;
    a_row[rep] = (q / KCH) * 8;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      a_off[rep][e] = 0;
      a_ok[rep][e] = (q < A_SUB) && row_in_a(p, tc.row0 + a_row[rep] + e, a_off[rep][e]);
    }
  }
  int64_t b_off[B_REP];
  bool b_ok[B_REP];
  int b_kc[B_REP], b_col[B_REP];
#pragma unroll
  for (int rep = 0; rep < B_REP; ++rep) {
    const int q = t + NT * rep;
    b_kc[rep] = q % KCH;
    b_col[rep] = q / KCH;
    b_off[rep] = 0;
    b_ok[rep] = (q < B_CH) && col_in_b(p, tc.col0 + b_col[rep], b_off[rep]);
  }

  uint4 a_reg[A_REP][8];
  uint4 b_reg[B_REP];

  auto load_stage = [&](int64_t s) {
    const int64_t i = s / ksteps;
    const int32_t kk = (int32_t)(s - i * ksteps) * BK;
    const uint16_t* pa;
    const uint16_t* pb;
    pair_bases<uint16_t>(p, in, i, pa, pb);
#pragma unroll
    for (int rep = 0; rep < A_REP; ++rep) {
      const int32_t k0 = kk + a_kc[rep] * 8;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        // each of the 8 rows and the k index checked on its own
        uint32_t h[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const bool ok = a_ok[rep][e] && (k0 + j) < p.k;
          h[e] = ok ? pa[a_off[rep][e] + (int64_t)(k0 + j) * p.lda] : 0u;
        }
        a_reg[rep][j] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16),
                                   h[6] | (h[7] << 16));
      }
    }
#pragma unroll
    for (int rep = 0; rep < B_REP; ++rep) {
      const int32_t k0 = kk + b_kc[rep] * 8;
      uint32_t h[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool ok = b_ok[rep] && (k0 + e) < p.k;
        h[e] = ok ? pb[b_off[rep] + k0 + e] : 0u;
      }
      b_reg[rep] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16),
                              h[6] | (h[7] << 16));
    }
  };

  auto store_stage = [&](int buf) {
    uint16_t* As = lds + buf * STAGE;
    uint16_t* Bs = As + BM * LDS_ROW;
#pragma unroll
    for (int rep = 0; rep < A_REP; ++rep) {
      if (t + NT * rep < A_SUB)
        store_a_transposed(As + a_row[rep] * LDS_ROW + a_kc[rep] * 8, a_reg[rep]);
    }
#pragma unroll
    for (int rep = 0; rep < B_REP; ++rep) {
      if (t + NT * rep < B_CH)
        *reinterpret_cast<uint4*>(Bs + b_col[rep] * LDS_ROW + b_kc[rep] * 8) = b_reg[rep];
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[tm][tn][v] = 0.0f;

  const int frag_row = lane & 31;
  const int frag_k = (lane >> 5) * 8;

  if (stages > 0) {
    load_stage(0);
    store_stage(0);
    __syncthreads();
    for (int64_t s = 0; s < stages; ++s) {
      const int buf = (int)(s & 1);
      if (s + 1 < stages) load_stage(s + 1);   // global loads in flight during the MFMAs
      const uint16_t* As = lds + buf * STAGE;
      const uint16_t* Bs = As + BM * LDS_ROW;
#pragma unroll
      for (int kq = 0; kq < BK / 16; ++kq) {
        bf16x8 af[TM], bfr[TN];
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
          af[tm] = *reinterpret_cast<const bf16x8*>(
              As + (wm * WTM + tm * 32 + frag_row) * LDS_ROW + kq * 16 + frag_k);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
          bfr[tn] = *reinterpret_cast<const bf16x8*>(
              Bs + (wn * WTN + tn * 32 + frag_row) * LDS_ROW + kq * 16 + frag_k);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
          for (int tn = 0; tn < TN; ++tn)
            acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[tm], bfr[tn], acc[tm][tn],
                                                                  0, 0, 0);
      }
      if (s + 1 < stages) store_stage(buf ^ 1);
      __syncthreads();
    }
  }

  // Epilogue on the accumulators, one store per output element.
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
      const int32_t C = tc.col0 + wn * WTN + tn * 32 + (lane & 31);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int32_t R0 = tc.row0 + wm * WTM + tm * 32 + q * 8 + (lane >> 5) * 4;
        const float v[4] = {acc[tm][tn][q * 4 + 0], acc[tm][tn][q * 4 + 1],
                            acc[tm][tn][q * 4 + 2], acc[tm][tn][q * 4 + 3]};
        store_group<true>(p, in, R0, C, v);
      }
    }
}

// ---------------------------------------------------------------------------------------------
// bf16 16-byte-load kernel, for m and k of at least 8, any strides and any alignment (a 16-byte
// load takes any element address).  Every 8-element chunk a thread moves is contiguous in one
// block.  FULL: every tile is complete (no row, column or k tail), so the loads carry no bounds
// logic at all; otherwise out-of-range chunks read a clamped, in-range address and k past the end
// is replaced by zeros without branching (rows and columns past the end only reach outputs that
// are not stored).
// RAGGED: m or k is no multiple of 8.  The virtual rows of each instance are padded to whole
// chunks (p.vm of them), so a chunk still lies in one block, and the last chunk of a block's rows
// or k-run reads the 8-element window that ends with the block instead of passing it: a row window
// goes d rows higher in the LDS panel (where it writes the d rows below it once more, the same
// values; the panel has 8 spare rows in front for a tile that starts with such a chunk), a k
// window is shifted down by d elements.  A classifier layer of 1000 outputs on 777 features and
// 1533 tokens (384 tiles of 64 x 64, bound by its chain of 13 stages) took 107 us through the
// element-load kernel above, one stage of element loads at a time, and takes 18 us here.
// ---------------------------------------------------------------------------------------------
// Transpose an 8 x SK bf16 sub-block held as SK k-columns of 8 rows into 8 rows of SK k, and
// store the rows (2*SK bytes each) into the K-contiguous LDS panel.
template <int SK>
__device__ __forceinline__ void store_a_transposed_v(uint16_t* dst_row0, const u32x4 col[SK]) {
#pragma unroll
  for (int mi = 0; mi < 8; ++mi) {
    const int d = mi >> 1;
    uint32_t w[SK / 2];
#pragma unroll
    for (int e = 0; e < SK / 2; ++e) {
      const uint32_t lo = col[2 * e][d], hi = col[2 * e + 1][d];
      w[e] = (mi & 1) ? ((lo >> 16) | (hi & 0xffff0000u)) : ((lo & 0xffffu) | (hi << 16));
    }
    if constexpr (SK == 8)
      *reinterpret_cast<u32x4*>(dst_row0 + mi * LDS_ROW) = (u32x4){w[0], w[1], w[2], w[3]};
    else
      *reinterpret_cast<uint2*>(dst_row0 + mi * LDS_ROW) = make_uint2(w[0], w[1]);
  }
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool FULL, int KIND, bool RAGGED>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void brgemm_bf16_vec_kernel(BrgemmParams p) {
  static_assert(!(FULL && RAGGED), "a ragged block has tails");
  // Register prefetch depth: two stages ahead with one wave per SIMD, one stage ahead with two
  // waves per SIMD (the second wave hides the latency, and the registers are needed for it).
  constexpr int DEPTH = (WAVES_M * WAVES_N > 4) ? 1 : 2;
  constexpr int NTH = 64 * WAVES_M * WAVES_N;        // threads per workgroup
  constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int KCH = BK / 8;                        // 8-element k chunks per stage
  // A moves in 8-row x SK-k sub-blocks; SK = 4 when 8x8 sub-blocks would leave threads idle.
  constexpr int SK = ((BM / 8) * (BK / 8) >= NTH) ? 8 : 4;
  constexpr int KCA = BK / SK;
  constexpr int A_SUB = (BM / 8) * KCA;
  constexpr int A_REP = (A_SUB + NTH - 1) / NTH;
  constexpr int B_CH = BN * KCH;                     // 16-byte chunks of the B panel
  constexpr int B_REP = (B_CH + NTH - 1) / NTH;
  constexpr int GUARD = RAGGED ? 8 * LDS_ROW : 0;    // spare rows in front of the A panel
  constexpr int STAGE = GUARD + (BM + BN) * LDS_ROW;
  constexpr int EP_ROW = WTM + 4;                    // epilogue slab: 32 columns x WTM rows fp32
  static_assert(TM >= 1 && TN >= 1, "wave tile at least 32x32");
  static_assert(WAVES_M * WAVES_N * 32 * EP_ROW * 4 <= 2 * STAGE * 2,
                "epilogue slabs fit in the stage buffers");

  __shared__ __attribute__((aligned(16))) uint16_t lds[2 * STAGE];

  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave % WAVES_M, wn = wave / WAVES_M;
  const TileCoord tc = decode_tile(p, BM, BN);
  const Instance in = instance_of(p, tc.g);
  const int32_t ksteps = (p.k + BK - 1) / BK;
  // The host bounds the stages of stride and offset kind by 2^31; a pointer list may be longer.
  using StageCount = std::conditional_t<KIND == TPP_BR_ADDRESS, int64_t, int32_t>;
  const StageCount stages = (StageCount)(in.npairs * ksteps);

  // Staging assignments, fixed for the whole reduction.  Out-of-range rows / columns keep
  // offset 0 (an in-range address) and a false flag.
  int64_t a_off[A_REP];
  bool a_ok[A_REP];
  int a_kc[A_REP], a_row[A_REP];
#pragma unroll
  for (int rep = 0; rep < A_REP; ++rep) {
    const int q = t + NTH * rep;
    a_kc[rep] = q % KCA;
    a_row[rep] = (q / KCA) * 8;
    a_off[rep] = 0;
    if constexpr (RAGGED) {
      const int32_t R = tc.row0 + a_row[rep];
      const int32_t gi = p.fused ? fdiv(R, p.div_m) : 0, r = R - gi * p.vm;
      a_ok[rep] = q < A_SUB && R < p.vrows;
      if (a_ok[rep]) {
        const int32_t d = r + 8 > p.m ? r + 8 - p.m : 0;   // the window ends with the block
        a_off[rep] = (p.fused ? (int64_t)gi * p.a_step_m : 0) + r - d;
        a_row[rep] -= d;
      }
    } else {
      a_ok[rep] = (q < A_SUB) && row_in_a(p, tc.row0 + a_row[rep], a_off[rep]);
      if (!a_ok[rep]) a_off[rep] = 0;
    }
  }
  int64_t b_off[B_REP];
  bool b_ok[B_REP];
  int b_kc[B_REP], b_col[B_REP];
#pragma unroll
  for (int rep = 0; rep < B_REP; ++rep) {
    const int q = t + NTH * rep;
    b_kc[rep] = q % KCH;
    b_col[rep] = q / KCH;
    b_off[rep] = 0;
    b_ok[rep] = (q < B_CH) && col_in_b(p, tc.col0 + b_col[rep], b_off[rep]);
    if (!b_ok[rep]) b_off[rep] = 0;
  }

  // Two register sets for staged operands: while the MFMAs consume LDS buffer s&1, set s&1
  // receives the global loads of stage s+2 and set (s+1)&1 (loaded one stage earlier) is written
  // to LDS buffer (s+1)&1 in between the MFMAs.
  struct Staged {
    u32x4 a[A_REP][SK];
    u32x4 b[B_REP];
    int32_t kk;   // the stage's first k in its block
  };
  Staged st0;
  Staged st1;

  // Stages are loaded in order; pointer lists keep the pair and k offset of the next one.
  int64_t next_i = 0;
  int32_t next_kk = 0;
  auto load_stage = [&](StageCount s, Staged& r) {
    int64_t i;
    int32_t kk;
    if constexpr (KIND == TPP_BR_ADDRESS) {
      i = next_i;
      kk = next_kk;
      next_kk += BK;
      if (next_kk >= p.k) {
        next_kk = 0;
        ++next_i;
      }
    } else {
      i = s / ksteps;
      kk = (s - (int32_t)i * ksteps) * BK;
    }
    const uint16_t* pa;
    const uint16_t* pb;
    pair_bases_k<KIND, uint16_t>(p, in, i, pa, pb);
    const bool ktail = !FULL && kk + BK > p.k;   // uniform: the block's last, partial stage
    r.kk = kk;
#pragma unroll
    for (int rep = 0; rep < A_REP; ++rep) {
      const int32_t k0 = kk + a_kc[rep] * SK;
      const uint16_t* base = pa + a_off[rep];
      if (!ktail) {
#pragma unroll
        for (int j = 0; j < SK; ++j)
          r.a[rep][j] = ld16_unaligned(base + (int64_t)(k0 + j) * p.lda);
      } else if constexpr (!RAGGED) {   // k a multiple of 8: the SK columns exist or not together
        const uint16_t* col = base + (int64_t)(k0 < p.k ? k0 : 0) * p.lda;
#pragma unroll
        for (int j = 0; j < SK; ++j) r.a[rep][j] = ld16_unaligned(col + (int64_t)j * p.lda);
      } else {
#pragma unroll
        for (int j = 0; j < SK; ++j)
          r.a[rep][j] = ld16_unaligned(base + (int64_t)(k0 + j < p.k ? k0 + j : 0) * p.lda);
      }
    }
#pragma unroll
    for (int rep = 0; rep < B_REP; ++rep) {
      const int32_t k0 = kk + b_kc[rep] * 8;
      const uint16_t* base = pb + b_off[rep];
      if (!ktail)
        r.b[rep] = ld16_unaligned(base + k0);
      else if constexpr (RAGGED)
        r.b[rep] = ld16_unaligned(base + (k0 + 8 > p.k ? p.k - 8 : k0));   // the window's first k
      else
        r.b[rep] = ld16_unaligned(base + (k0 < p.k ? k0 : 0));
    }
  };

  // k past the end becomes zero here, on the way to LDS, and not behind the loads: a use of their
  // values there would wait for them, a memory latency per partial stage (8 pairs of 64 x 64 x 16
  // blocks on 16 x 16 instances: 12.5 us so, 10.7 here).  Before the MFMAs of the stage in front: between
  // them, next to the stores, 4 pairs of 63 x 32 x 9 blocks on 32 x 32 instances took 13.8 us and not 12.6.
  auto mask = [&](Staged& r) {
    if (FULL || r.kk + BK <= p.k) return;   // uniform
#pragma unroll
    for (int rep = 0; rep < A_REP; ++rep) {
      const int32_t k0 = r.kk + a_kc[rep] * SK;
#pragma unroll
      for (int j = 0; j < SK; ++j)
        r.a[rep][j] = keep_if(r.a[rep][j], (RAGGED ? k0 + j : k0) < p.k);
    }
#pragma unroll
    for (int rep = 0; rep < B_REP; ++rep) {
      const int32_t k0 = r.kk + b_kc[rep] * 8;
      if constexpr (RAGGED)
        r.b[rep] = shift_down(r.b[rep], k0 + 8 > p.k ? k0 + 8 - p.k : 0);
      else
        r.b[rep] = keep_if(r.b[rep], k0 < p.k);
    }
  };
  auto store_a = [&](int buf, const Staged& r) {
    uint16_t* As = lds + buf * STAGE + GUARD;
#pragma unroll
    for (int rep = 0; rep < A_REP; ++rep) {
      if (A_SUB % NTH == 0 || t + NTH * rep < A_SUB)
        store_a_transposed_v<SK>(As + a_row[rep] * LDS_ROW + a_kc[rep] * SK, r.a[rep]);
    }
  };
  auto store_b = [&](int buf, const Staged& r) {
    uint16_t* Bs = lds + buf * STAGE + GUARD + BM * LDS_ROW;
#pragma unroll
    for (int rep = 0; rep < B_REP; ++rep) {
      if (B_CH % NTH == 0 || t + NTH * rep < B_CH)
        *reinterpret_cast<u32x4*>(Bs + b_col[rep] * LDS_ROW + b_kc[rep] * 8) = r.b[rep];
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[tm][tn][v] = 0.0f;

  const int frag_row = lane & 31;
  const int frag_k = (lane >> 5) * 8;

  // MFMAs of one LDS buffer: the fragments of k-step kq+1 are read while the MFMAs of kq run;
  // hook(kq) runs after the MFMAs of k-step kq are issued.
  auto compute = [&](int buf, auto&& hook) {
    const uint16_t* As = lds + buf * STAGE + GUARD;
    const uint16_t* Bs = As + BM * LDS_ROW;
    bf16x8 fa[2][TM], fb[2][TN];
    auto frags = [&](int kq, bf16x8* a, bf16x8* b) {
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
        a[tm] = *reinterpret_cast<const bf16x8*>(
            As + (wm * WTM + tm * 32 + frag_row) * LDS_ROW + kq * 16 + frag_k);
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
        b[tn] = *reinterpret_cast<const bf16x8*>(
            Bs + (wn * WTN + tn * 32 + frag_row) * LDS_ROW + kq * 16 + frag_k);
    };
    frags(0, fa[0], fb[0]);
#pragma unroll
    for (int kq = 0; kq < BK / 16; ++kq) {
      if (kq + 1 < BK / 16) frags(kq + 1, fa[(kq + 1) & 1], fb[(kq + 1) & 1]);
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
          acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kq & 1][tm], fb[kq & 1][tn],
                                                                acc[tm][tn], 0, 0, 0);
      hook(kq);
    }
  };

  if (stages > 0) {
    load_stage(0, st0);
    if (DEPTH == 2 && stages > 1) load_stage(1, st1);
    mask(st0);
    store_a(0, st0);
    store_b(0, st0);
    __syncthreads();
    StageCount s = 0;
    // One stage; PAR = s & 1 is a compile-time constant so the register sets are never indexed
    // at run time.
    auto step = [&](auto par) {
      constexpr int PAR = decltype(par)::value;
      const bool more = s + 1 < stages;
      if constexpr (DEPTH == 2) {
        Staged& cur = PAR ? st1 : st0;   // stage s (already in LDS buffer PAR): free for s+2
        Staged& nxt = PAR ? st0 : st1;   // stage s+1, loaded one stage ago
        if (s + 2 < stages) load_stage(s + 2, cur);
        if (more) mask(nxt);
        compute(PAR, [&](int kq) {
          if (more && kq == 1) store_a(PAR ^ 1, nxt);
          if (more && kq == 2) store_b(PAR ^ 1, nxt);
        });
      } else {
        // one register set: stage s+1 is loaded now and written to LDS after the MFMAs
        if (more) load_stage(s + 1, st0);
        compute(PAR, [&](int) {});
        if (more) {
          mask(st0);
          store_a(PAR ^ 1, st0);
          store_b(PAR ^ 1, st0);
        }
      }
      __syncthreads();
      ++s;
    };
    while (s + 1 < stages) {
      step(IntC<0>());
      step(IntC<1>());
    }
    if (s < stages) step(IntC<0>());
  }

  epilogue_via_lds<WTM, WTN, TM, TN, FULL, RAGGED>(p, in, tc, wm, wn, lane, wave,
                                                  reinterpret_cast<float*>(lds), acc);
}

// ---------------------------------------------------------------------------------------------
// fp32 kernel: 64x64 tile, v_mfma_f32_32x32x2f32 (64 cycles each), stages of 64 k, two groups of four
// waves (32x32 each): a group takes half of every stage's k and the groups' sums meet in LDS at the
// end.  MFMA-bound on a full grid: a stage is 32 KB of loads per 2048 MFMA cycles of each SIMD, and
// with two workgroups per CU four waves per SIMD cover each other's reads, stores and barriers.
//   - Each thread moves two 16-byte vectors of A (4 rows of one k-column) and two of B (4 k of one
//     column) per stage, at any alignment and for every batch kind (m and k of at least 4; fewer
//     take brgemm_f32_kernel<false>, element loads).  The virtual rows of an instance are padded to
//     whole 4-row chunks (p.vm); the last chunk of a block's rows or k-run loads the window of 4
//     that ends with the block and is shifted into place in registers, k past the end as zeros.
//   - Two register sets keep the loads of two stages in flight.  No branch surrounds a load (past
//     the last stage the last one is read again, from the cache) and no step of the loop has a way
//     out of its own, so that the compiler counts the loads in flight: otherwise it waits for the
//     newest ones at every stage.
//   - The sum over k runs in the order that LDS reads like: of each 8 k, lanes 0-31 take k 0-3 and
//     lanes 32-63 k 4-7, one after the other, so a lane's four B values are one 16-byte read of its
//     column and B is stored as it comes.  The fragments of 8 k are read during the MFMAs of the
//     8 before them.
// A 2048 x 1024 x 1024 layer (512 tiles): 50.2 us with one group, 32-k stages and a ring that the
// waits emptied, 46.3 here (36 us per 1024 k, of which the MFMAs and their LDS reads are 29, and
// 10 at its ends); 192 x 1600 x 510 with a padded row: 81.0 through element loads, 15.0 here.
//   - Two LDS buffers, one barrier per stage.
//   - Split launches (few tiles, long stage lists): workgroup b reduces chunk b % split of tile
//     b / split's stages into a partial tile of the work space, and brgemm_f32_split_finish
//     adds the chunks and applies the epilogue.  (Finishing in the same launch, by the last
//     workgroup of a tile to arrive at a per-tile counter, measured 3.4 us slower per call on
//     the single 64 x 64 instance: the returning device-scope atomic and one workgroup loading
//     every chunk cost more than a second launch queued behind the first.)
// ---------------------------------------------------------------------------------------------
constexpr int F_BM = 64, F_BN = 64, F_BK = F32_STAGE_K;
constexpr int F_NT = 512;            // threads: two groups of four waves
constexpr int F_RING = 2;            // stages of global loads in flight (register sets)
constexpr int F_BROW = F_BK + 4;     // padded column of the B panel (floats): conflict-free reads

// v moved down by d elements (d >= 0), zeros past the end.
__device__ __forceinline__ f32x4 shift_down(f32x4 v, int32_t d) {
  if (d & 1) v = (f32x4){v.y, v.z, v.w, 0.0f};
  if (d & 2) v = (f32x4){v.z, v.w, 0.0f, 0.0f};
  if (d >= 4) v = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
  return v;
}

// Chunk of a split launch's stages, the tile and the instance of workgroup blockIdx.x.
struct F32Work {
  int64_t tile_bid;
  int32_t split, chunk;
  TileCoord tc;
  Instance in;
  int64_t s_lo, steps;    // first step and how many (step = pair * ksteps + k-step)
  int64_t i0;             // pair of the first step
  int32_t ksteps;
};
// PER steps of the list make a stage, of 64 k in all.
template <int PER>
__device__ __forceinline__ F32Work f32_work(const BrgemmParams& p) {
  F32Work w;
  w.split = p.split > 1 ? p.split : 1;
  w.tile_bid = p.split > 1 ? fdiv(blockIdx.x, p.div_split) : blockIdx.x;
  w.chunk = (int32_t)((int64_t)blockIdx.x - w.tile_bid * w.split);
  w.tc = decode_tile_at(p, F_BM, F_BN, w.tile_bid);
  w.in = instance_of(p, w.tc.g);
  w.ksteps = (p.k + F_BK / PER - 1) / (F_BK / PER);
  w.s_lo = 0;
  w.i0 = 0;
  w.steps = w.in.npairs * w.ksteps;
  if (p.split > 1) {   // whole stages per chunk, of which the very last may lack a step
    w.s_lo = PER * ((int64_t)w.chunk * p.split_base + min(w.chunk, p.split_rem));
    const int64_t n = PER * ((int64_t)p.split_base + (w.chunk < p.split_rem ? 1 : 0));
    w.steps = PER == 1 || w.steps - w.s_lo > n ? n : w.steps - w.s_lo;
    w.i0 = fdiv((uint32_t)w.s_lo, p.div_ks);
  }
  return w;
}

__device__ __forceinline__ void f32_finish_tile(const BrgemmParams& p, const F32Work& w, int wave,
                                                int lane, const f32x16& acc) {
  const int wm = wave & 1, wn = wave >> 1;
  if (w.split > 1) {
    // This chunk's partial tile, the accumulators in register order: thread t's group q at float
    // ((wave * 4 + q) * 64 + lane) * 4 of the chunk's 64 x 64 block, so each wave-wide 16-byte
    // store covers 1 KB of consecutive bytes.
    float* const o = p.ws + ((size_t)w.tile_bid * w.split + w.chunk) * (F_BM * F_BN) +
                     ((wave * 4) * 64 + lane) * 4;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      gst<f32x4>(o + q * 256,
                 (f32x4){acc[q * 4 + 0], acc[q * 4 + 1], acc[q * 4 + 2], acc[q * 4 + 3]});
    return;
  }
  const int32_t C = w.tc.col0 + wn * 32 + (lane & 31);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int32_t R0 = w.tc.row0 + wm * 32 + q * 8 + (lane >> 5) * 4;
    const float v[4] = {acc[q * 4 + 0], acc[q * 4 + 1], acc[q * 4 + 2], acc[q * 4 + 3]};
    if (p.vm % 4 == 0)
      store_group<false>(p, w.in, R0, C, v);
    else
      store_group<true>(p, w.in, R0, C, v);
  }
}

// A thread's part of the fp32 kernel's output rows: one 4-row chunk (chunk t % 16 of the tile), its
// bias loaded ahead of the main loop.
struct F32Rows {
  int64_t off;       // of the chunk's first row in C, from the instance base
  int32_t nr;        // rows of the chunk that exist (0: none)
  float bias[4];
};
__device__ __forceinline__ F32Rows f32_rows(const BrgemmParams& p, const F32Work& w, int chunk) {
  F32Rows o;
  const int32_t R = w.tc.row0 + chunk * 4;
  const int32_t gi = p.fused ? fdiv(R, p.div_m) : 0, r = R - gi * p.vm;
  o.off = (p.fused ? (int64_t)gi * p.c_step_m : 0) + r;
  o.nr = R >= p.vrows ? 0 : (p.m - r < 4 ? p.m - r : 4);
  const int64_t bi = p.fused ? (int64_t)gi * p.bias_step_m + r : w.in.bias + r;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    o.bias[e] = (p.flags & TPP_EPI_BIAS) && e < o.nr && w.split <= 1 ? gld<float>(p.bias + bi + e)
                                                                      : 0.0f;
  return o;
}
// The epilogue on four rows of virtual column C.
__device__ __forceinline__ void f32_store4(const BrgemmParams& p, const F32Work& w,
                                           const F32Rows& rows, int32_t C, f32x4 x) {
  if (rows.nr == 0 || C >= (p.fused ? p.vcols : p.n)) return;
  const int32_t gi = p.fused ? fdiv(C, p.div_n) : 0, c = C - gi * p.n;
  const int64_t e0 = w.in.c + rows.off + (p.fused ? (int64_t)gi * p.c_step_n : 0) + c * p.ldc;
  float v[4] = {x[0], x[1], x[2], x[3]};
  if (rows.nr < 4) {
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      if (e >= rows.nr) break;
      float u[1] = {v[e]};
      if (p.beta != 0.0f)
        u[0] = p.beta * (p.c_bf16 ? bf16_bits_to_f32(gld<uint16_t>(static_cast<uint16_t*>(p.c) + e0 + e))
                                  : gld<float>(static_cast<float*>(p.c) + e0 + e)) + u[0];
      u[0] += rows.bias[e];
      if (p.flags & EPI_AUX_MASK) epi_aux<1>(p, e0 + e, u);
      const float o = activate(u[0], p.flags);
      if (p.c_bf16) gst<uint16_t>(static_cast<uint16_t*>(p.c) + e0 + e, f32_to_bf16_bits(o));
      else gst<float>(static_cast<float*>(p.c) + e0 + e, o);
    }
    return;
  }
  if (p.c_bf16) {
    uint16_t* const cp = static_cast<uint16_t*>(p.c) + e0;
    if (p.beta != 0.0f) {
      const u32x2 h = gld<u32x2_a2>(cp);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        v[e] = p.beta * bf16_bits_to_f32(h[e >> 1] >> (16 * (e & 1)) & 0xffffu) + v[e];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += rows.bias[e];
    if (p.flags & EPI_AUX_MASK) epi_aux<4>(p, e0, v);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = activate(v[e], p.flags);
    gst<u32x2_a2>(cp, (u32x2){pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])});
  } else {
    float* const cp = static_cast<float*>(p.c) + e0;
    if (p.beta != 0.0f) {
      const f32x4 h = gld<f32x4_a4>(cp);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = p.beta * h[e] + v[e];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += rows.bias[e];
    if (p.flags & EPI_AUX_MASK) epi_aux<4>(p, e0, v);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = activate(v[e], p.flags);
    gst<f32x4_a4>(cp, (f32x4){v[0], v[1], v[2], v[3]});
  }
}

// PAIRED: a stage is two steps of 32 k, one for each group of waves, from one pair's blocks or from
// two pairs'; else one step of 64 k, half of it for each.
// LISTS: offset and pointer lists too, else stride kind alone (without the lists' code, of which every
// load of the unrolled loop has a copy).
template <bool PAIRED, bool LISTS>
__device__ __forceinline__ void f32_vec_body(const BrgemmParams& p) {
  constexpr int PER = PAIRED ? 2 : 1, STEP = F_BK / PER;
  constexpr int BQ = STEP / 4;   // 4-k vectors of a column of B in a step
  __shared__ __attribute__((aligned(16))) float As[2][F_BK * F_BM];     // [k][row]
  __shared__ __attribute__((aligned(16))) float Bs[2][F_BN * F_BROW];   // [column][k]
  const int t = threadIdx.x, lane = t & 63;
  const int wave = (t >> 6) & 3, kgrp = t >> 8;   // wave of its group; the group's half of a stage
  const int wm = wave & 1, wn = wave >> 1;
  const F32Work w = f32_work<PER>(p);
  const int64_t stages = (w.steps + PER - 1) / PER;
  const F32Rows rows = f32_rows(p, w, t & 15);

  // Thread t moves two vectors of A and two of B per stage: those of a 64-k step with q = t + 512 j
  // (j < 2), or that of step j with q = t.  A: k-column q / 16 of the step, rows 4 (q % 16) .. +3;
  // B: column q / BQ, k 4 (q % BQ) .. +3.  Byte offsets from a step's bases, in whole steps and in a
  // block's last, partial one (_t).  Rows and columns outside C read the first ones: only outputs
  // that are not stored see them.
  const bool ragged_rows = p.vm != p.m, ragged_k = p.k % 4 != 0;
  const bool ragged = p.k % STEP != 0 || ragged_rows;
  const int32_t ktail = p.k - (w.ksteps - 1) * STEP;     // k of the last k-step
  int64_t oa[2], ob[2], oa_t[2], ob_t[2];
  int32_t sr[2], sk[2];       // shifts: rows of A, k of B in the partial step
  bool ka_ok[2];              // A's k-column exists in the partial step
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int q = PAIRED ? t : t + F_NT * j;
    const int ka = q >> 4, kb = (q % BQ) * 4;
    const int32_t R = w.tc.row0 + (q & 15) * 4;
    const int32_t gi = p.fused ? fdiv(R, p.div_m) : 0;
    int32_t r = R - gi * p.vm;
    int64_t base = p.fused ? gi * p.a_step_m : 0;
    if (R >= p.vrows) {
      r = 0;
      base = 0;
    }
    sr[j] = r + 4 > p.m ? r + 4 - p.m : 0;
    base += r - sr[j];
    ka_ok[j] = ka < ktail;
    oa[j] = (base + (int64_t)ka * p.lda) * 4;
    oa_t[j] = (base + (int64_t)(ka_ok[j] ? ka : 0) * p.lda) * 4;
    int64_t col = 0;
    if (!col_in_b(p, w.tc.col0 + q / BQ, col)) col = 0;
    // the window of 4 k ends with the block (k >= 4, so it may begin in the k-step before)
    const int32_t kw = kb + 4 > ktail ? ktail - 4 : kb;
    sk[j] = kb - kw;
    ob[j] = (col + kb) * 4;
    ob_t[j] = (col + kw) * 4;
  }

  // Steps are loaded strictly in order by a cursor: pair i (bases pa, pb), k offset kk.  Offset
  // and pointer lists: lane l holds the entries of pair 64 (i / 64) + l, taken with readlane.
  int64_t ld_s = 0, ld_i = w.i0;
  int32_t ld_kk = (int32_t)(w.s_lo - ld_i * w.ksteps) * STEP;
  const char* pa = nullptr;
  const char* pb = nullptr;
  // read here: a first read between two steps' loads would hold the second step's back by its latency
  int64_t step_a = p.stride_a * 4, step_b = p.stride_b * 4;
  if (PAIRED) asm volatile("" : "+s"(step_a), "+s"(step_b));
  uint64_t list_a = 0, list_b = 0;
  const auto uni = [](uint64_t v, int src) {
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), src) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, src);
  };
  const auto fill_list = [&]() {
    const int64_t i = (ld_i & ~(int64_t)63) + lane;
    if (i >= w.in.npairs) return;
    const float *a, *b;
    pair_bases<float>(p, w.in, i, a, b);
    list_a = reinterpret_cast<uint64_t>(a);
    list_b = reinterpret_cast<uint64_t>(b);
    // the entries are waited for here, on this path alone, and not at every readlane
    asm volatile("" : "+v"(list_a), "+v"(list_b));
  };
  const auto from_list = [&]() {
    pa = reinterpret_cast<const char*>(uni(list_a, (int)(ld_i & 63)));
    pb = reinterpret_cast<const char*>(uni(list_b, (int)(ld_i & 63)));
  };
  if (!LISTS) {
    pa = static_cast<const char*>(p.a) + w.in.a * 4 + ld_i * step_a;
    pb = static_cast<const char*>(p.b) + w.in.b * 4 + ld_i * step_b;
  } else if (stages > 0) {
    fill_list();
    from_list();
  }
  f32x4 ra[F_RING][2], rb[F_RING][2];
  bool part[F_RING][PER];     // the step is a block's partial one
  bool lone[F_RING];          // PAIRED: the second step is past the list
  auto load_step = [&](auto slot, auto which) {
    constexpr int R = decltype(slot)::value, J = decltype(which)::value;
    const bool tail = ragged && ld_kk + STEP > p.k;
    part[R][J] = tail;
    const char* const a = pa + (int64_t)ld_kk * p.lda * 4;
    const char* const b = pb + (int64_t)ld_kk * 4;
#pragma unroll
    for (int j = PAIRED ? J : 0; j < (PAIRED ? J + 1 : 2); ++j) {
      ra[R][j] = gld<f32x4_a4>(a + (tail ? oa_t[j] : oa[j]));
      rb[R][j] = gld<f32x4_a4>(b + (tail ? ob_t[j] : ob[j]));
    }
    if (++ld_s >= w.steps) return;   // stay on the last step
    ld_kk += STEP;
    if (ld_kk >= p.k) {
      ld_kk = 0;
      ++ld_i;
      if (!LISTS || p.kind == TPP_BR_STRIDE) {
        pa += step_a;
        pb += step_b;
      } else {
        if ((ld_i & 63) == 0) fill_list();
        from_list();
      }
    }
  };
  auto load = [&](auto slot) {
    lone[decltype(slot)::value] = ld_s + 1 >= w.steps;
    load_step(slot, IntC<0>());
    if constexpr (PAIRED) load_step(slot, IntC<1>());
  };
  auto store = [&](int buf, auto slot) {
    constexpr int R = decltype(slot)::value;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int q = PAIRED ? t : t + F_NT * j;
      const int k0 = PAIRED ? STEP * j : 0;   // the step's place in the stage
      f32x4 a = ra[R][j], b = rb[R][j];
      const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
      if (ragged) {   // uniform, as the next three conditions but ka_ok and sk
        if (ragged_rows) a = shift_down(a, sr[j]);
        if (part[R][PAIRED ? j : 0]) {
          if (!ka_ok[j]) a = zero;
          if (ragged_k) b = shift_down(b, sk[j]);
          else if (sk[j] != 0) b = zero;   // whole windows: 4 k and more past the end
        }
      }
      if (PAIRED && j == 1 && lone[R]) a = b = zero;
      *reinterpret_cast<f32x4*>(&As[buf][(k0 + (q >> 4)) * F_BM + (q & 15) * 4]) = a;
      *reinterpret_cast<f32x4*>(&Bs[buf][q / BQ * F_BROW + k0 + (q % BQ) * 4]) = b;
    }
  };

  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
  struct Frag {
    float a[4];
    f32x4 b;
  };
  const int half = lane >> 5;
  const int k_at = kgrp * (F_BK / 2) + half * 4;
  const int a_at = k_at * F_BM + wm * 32 + (lane & 31);
  const int b_at = (wn * 32 + (lane & 31)) * F_BROW + k_at;
  auto frag = [&](int buf, int g) {   // the 8 k of step g of the wave's half stage
    Frag f;
#pragma unroll
    for (int e = 0; e < 4; ++e) f.a[e] = As[buf][a_at + (8 * g + e) * F_BM];
    f.b = *reinterpret_cast<const f32x4*>(&Bs[buf][b_at + 8 * g]);
    return f;
  };
  auto mfmas = [&](const Frag& f) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(f.a[e], f.b[e], acc, 0, 0, 0);
  };

  // groups of 8 k that a step has: fewer than four in blocks of at most 24 k
  const int32_t eights = p.k < STEP ? (p.k + 7) / 8 : 4;
  if (stages > 0) {
    load(IntC<0>());
    load(IntC<1>());
    store(0, IntC<0>());
    load(IntC<0>());
    lds_barrier();
    // Stage s: MFMAs on LDS buffer s & 1; stage s + 1 goes from its register set into the other
    // buffer (free: every wave passed the barrier after stage s - 1's MFMAs) and that set takes
    // stage s + 1 + F_RING.
    auto step = [&](auto nslot) {
      constexpr int NS = decltype(nslot)::value;   // (s + 1) % F_RING
      constexpr int BUF = NS ^ 1;                  // s & 1
      Frag f0 = frag(BUF, 0);
      Frag f1 = frag(BUF, 1);
      __builtin_amdgcn_sched_barrier(0);
      mfmas(f0);
      f0 = frag(BUF, 2);
      store(BUF ^ 1, IntC<NS>());
      load(IntC<NS>());
      __builtin_amdgcn_sched_barrier(0);
      mfmas(f1);
      if (!PAIRED || eights > 2) {   // uniform
        f1 = frag(BUF, 3);
        __builtin_amdgcn_sched_barrier(0);
        mfmas(f0);
        __builtin_amdgcn_sched_barrier(0);
        if (!PAIRED || eights > 3) mfmas(f1);
      }
      lds_barrier();   // LDS traffic only: the ring's global loads stay in flight
    };
    // whole turns of the ring without a branch between the steps (a way out of the loop after each
    // step would again make the compiler wait for the newest loads), then the rest
    for (int64_t turns = stages / F_RING; turns > 0; --turns) {
      step(IntC<1>());
      step(IntC<0>());
    }
    if (stages % F_RING != 0) step(IntC<1>());
  }
  // The second group's sums join the first's (every wave has passed the last stage's barrier), as
  // a 64 x 64 tile in LDS, column by column.
  constexpr int TROW = F_BM + 4;
  static_assert(sizeof(As) >= F_BN * TROW * sizeof(float), "the tile fits the A panels");
  float* const tile = &As[0][0];
  float* const mine = tile + (wn * 32 + (lane & 31)) * TROW + wm * 32 + half * 4;
  if (kgrp == 1) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<f32x4*>(mine + 8 * q) =
          (f32x4){acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
  }
  __syncthreads();
  if (kgrp == 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 o = *reinterpret_cast<const f32x4*>(mine + 8 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[4 * q + e] += o[e];
        o[e] = acc[4 * q + e];
      }
      if (w.split <= 1) *reinterpret_cast<f32x4*>(mine + 8 * q) = o;
    }
  }
  if (w.split > 1) {
    if (kgrp == 0) f32_finish_tile(p, w, wave, lane, acc);
    return;
  }
  __syncthreads();
  // 16 threads store a column's 64 rows: whole lines.  (Stored from the accumulators, 16 bytes per
  // column and thread with the bias loaded group by group behind the stores, the epilogue took
  // about 5 us.)
#pragma unroll
  for (int j = 0; j < F_BN * 16 / F_NT; ++j) {
    const int col = (t >> 4) + j * (F_NT / 16);
    f32_store4(p, w, rows, w.tc.col0 + col,
               *reinterpret_cast<const f32x4*>(tile + col * TROW + (t & 15) * 4));
  }
}

template <bool VEC>
__global__ __launch_bounds__(NT) void brgemm_f32_kernel(BrgemmParams p);

template <>
__global__ __launch_bounds__(F_NT, 4) void brgemm_f32_kernel<true>(BrgemmParams p) {
  f32_vec_body<false, true>(p);
}

// Blocks of an odd number of 32-k steps (k of at most 32 above all, the inner blocks of blocked
// layouts), where stages of 64 k of one pair would spend half of a pair's last stage on zeros.  64 x
// 64 blocks on 512 tiles: 32 pairs of k = 32 91.3 us in 64-k stages, 46.2 here; 128 pairs of k = 8
// 340 and 124; pointer lists of 16 pairs of k = 32 51.0 and 30.8.  Blocks of 64 k lose 1.4 % by it (a
// second cursor step per stage; 45.3 and 45.9 us for a 2048 x 1024 x 1024 layer), so an even number
// of steps keeps 64-k stages.  Stride kind has an instance without the code of the lists: one stage on
// each of 8 workgroups takes 5.9 us with it and 7.7 without.  VEC as for brgemm_f32_kernel (true).
template <bool VEC>
__global__ __launch_bounds__(F_NT, 4) void brgemm_f32_paired_kernel(BrgemmParams p) {
  f32_vec_body<true, true>(p);
}
template <bool VEC>
__global__ __launch_bounds__(F_NT, 4) void brgemm_f32_paired_stride_kernel(BrgemmParams p) {
  f32_vec_body<true, false>(p);
}

// m or k below 4: half a stage of element loads at a time, every row, column and k checked.
template <>
__global__ __launch_bounds__(NT) void brgemm_f32_kernel<false>(BrgemmParams p) {
  constexpr int ROW = F_BM + 4, HK = F_BK / 2;
  __shared__ __attribute__((aligned(16))) float As[HK * ROW];
  __shared__ __attribute__((aligned(16))) float Bs[HK * ROW];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  const F32Work w = f32_work<1>(p);
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
  // thread t: A row t % 64 and B column t % 64, k t / 64 + 4 e of each stage
  const int rc = t & 63, k0 = t >> 6;
  int64_t a_off = 0, b_off = 0;
  const bool a_ok = row_in_a(p, w.tc.row0 + rc, a_off), b_ok = col_in_b(p, w.tc.col0 + rc, b_off);
  for (int64_t h = 2 * w.s_lo; h < 2 * (w.s_lo + w.steps); ++h) {
    const int64_t i = (h / 2) / w.ksteps;
    const int32_t kk = (int32_t)(h / 2 - i * w.ksteps) * F_BK + (int32_t)(h & 1) * HK;
    if (kk >= p.k) continue;   // uniform
    const float *pa, *pb;
    pair_bases<float>(p, w.in, i, pa, pb);
    float a[8], b[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int32_t k = kk + k0 + 4 * e;
      a[e] = a_ok && k < p.k ? gld<float>(pa + a_off + (int64_t)k * p.lda) : 0.0f;
      b[e] = b_ok && k < p.k ? gld<float>(pb + b_off + k) : 0.0f;
    }
    __syncthreads();   // the stage before has been read
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      As[(k0 + 4 * e) * ROW + rc] = a[e];
      Bs[(k0 + 4 * e) * ROW + rc] = b[e];
    }
    __syncthreads();
#pragma unroll
    for (int kq = 0; kq < HK / 2; ++kq) {
      const int kr = kq * 2 + (lane >> 5);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(As[kr * ROW + wm * 32 + (lane & 31)],
                                                 Bs[kr * ROW + wn * 32 + (lane & 31)], acc, 0, 0, 0);
    }
  }
  f32_finish_tile(p, w, wave, lane, acc);
}

// Finishing step of a split fp32 launch: four workgroups per tile, thread f of a tile's 1024
// taking the partial tiles' 16-byte group f (wave f / 256, register group (f / 64) % 4, lane
// f % 64 of the main kernel: four consecutive rows of one column).  It sums the chunks in chunk
// order (the result does not depend on timing), eight loads in flight at a time, and applies
// beta * C, bias, activation and the store exactly as the unsplit kernel's epilogue.
__global__ __launch_bounds__(NT) void brgemm_f32_split_finish(BrgemmParams p) {
  const int64_t tile_bid = blockIdx.x / 4;
  const int f = (int)(blockIdx.x - tile_bid * 4) * NT + threadIdx.x;
  const int wave = f >> 8, q = (f >> 6) & 3, lane = f & 63;
  const int wm = wave & 1, wn = wave >> 1;
  const TileCoord tc = decode_tile_at(p, F_BM, F_BN, tile_bid);
  const Instance in = instance_of(p, tc.g);
  const float* w = p.ws + (size_t)tile_bid * p.split * (F_BM * F_BN) + f * 4;
  f32x4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
  int32_t ch = 0;
  for (; ch + 8 <= p.split; ch += 8) {
    f32x4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = gld<f32x4>(w + (size_t)(ch + u) * (F_BM * F_BN));
#pragma unroll
    for (int u = 0; u < 8; ++u) sum += v[u];
  }
  for (; ch < p.split; ++ch) sum += gld<f32x4>(w + (size_t)ch * (F_BM * F_BN));
  const int32_t C = tc.col0 + wn * 32 + (lane & 31);
  const int32_t R0 = tc.row0 + wm * 32 + q * 8 + (lane >> 5) * 4;
  const float v[4] = {sum[0], sum[1], sum[2], sum[3]};
  if (p.vm % 4 == 0)
    store_group<false>(p, in, R0, C, v);
  else
    store_group<true>(p, in, R0, C, v);
}

// Finishing step of a split direct-LDS launch.  A partial tile holds, for each wave (waves_m x
// waves_n of them, a WTM x WTN tile each) and 32x32 block (tm, tn), every lane's 16 accumulators
// (f32x16, lane-contiguous).  Thread item i = ((wave * TM + tm) * TN + tn) * 256 + lane * 4 + q
// takes the four consecutive rows of MFMA register group q (rows 32 tm + 8 q + 4 (lane / 32) ..
// + 3 and column 32 tn + lane % 32 of the wave tile), so consecutive threads read consecutive 16
// bytes.  It sums them over the chunks in chunk order (the result does not depend on timing) and
// applies beta * C, bias, activation, the aux steps and the store as an unsplit epilogue does.
__global__ __launch_bounds__(NT) void brgemm_dl_split_finish(BrgemmParams p, int32_t bm,
                                                             int32_t bn, int32_t waves_m,
                                                             int32_t waves_n, int32_t per_tile) {
  const int64_t tile_bid = blockIdx.x / per_tile;
  const int32_t item = (int32_t)(blockIdx.x - tile_bid * per_tile) * NT + threadIdx.x;
  const TileCoord tc = decode_tile_at(p, bm, bn, tile_bid);
  const Instance in = instance_of(p, tc.g);
  const int32_t wtm = bm / waves_m, wtn = bn / waves_n;
  const int32_t tms = wtm / 32, tns = wtn / 32;
  const int32_t lane = (item & 255) >> 2, q = item & 3;
  const int32_t rest = item >> 8;
  const int32_t tn = rest % tns, tm = (rest / tns) % tms, wave = rest / (tns * tms);
  const int32_t wm = wave % waves_m, wn = wave / waves_m;
  const float* w = p.ws + (size_t)tile_bid * (bm * bn) + (size_t)item * 4;
  const size_t step = (size_t)p.total_tiles * bm * bn;
  f32x4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
  int32_t ch = 0;
  for (; ch + 4 <= p.split; ch += 4) {
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = gld<f32x4>(w + (size_t)(ch + u) * step);
#pragma unroll
    for (int u = 0; u < 4; ++u) sum += v[u];
  }
  for (; ch < p.split; ++ch) sum += gld<f32x4>(w + (size_t)ch * step);
  const float v4[4] = {sum[0], sum[1], sum[2], sum[3]};
  store_group<false>(p, in, tc.row0 + wm * wtm + tm * 32 + 8 * q + 4 * (lane >> 5),
                     tc.col0 + wn * wtn + tn * 32 + (lane & 31), v4);
}

struct KernelInfo {
  const char* name;
  int bm, bn;
  int kstep;   // k must be a multiple of this (direct buffer->LDS stages); 1 = any k
};

constexpr KernelInfo kInfo[K_COUNT] = {
    {"bf16_256x256_w8_vec", 256, 256, 1},
    {"bf16_128x128_w4_vec", 128, 128, 1},
    {"bf16_64x64_w4_vec", 64, 64, 1},
    {"bf16_64x64_generic", 64, 64, 1},
    {"f32_64x64_generic", 64, 64, 1},
    {"bf16_256x256_w8_direct_lds", 256, 256, 32},
    {"bf16_128x128_w4_direct_lds", 128, 128, 32},
    {"bf16_64x64_w4_direct_lds", 64, 64, 32},
    {"bf16_256x256_w8_direct_lds_pingpong", 256, 256, 32},
    {"bf16_256x256_w8_direct_lds_bk64", 256, 256, 64},
    {"bf16_128x128_w4_direct_lds_bk64", 128, 128, 64},
    {"bf16_64x64_w4_direct_lds_bk64", 64, 64, 64},
};

}  // namespace

const char* kernel_name(int32_t id) { return (id >= 0 && id < K_COUNT) ? kInfo[id].name : "?"; }
int kernel_tile_m(int32_t id) { return (id >= 0 && id < K_COUNT) ? kInfo[id].bm : 64; }
int kernel_tile_n(int32_t id) { return (id >= 0 && id < K_COUNT) ? kInfo[id].bn : 64; }
int kernel_k_step(int32_t id) { return (id >= 0 && id < K_COUNT) ? kInfo[id].kstep : 1; }

bool kernel_full(int32_t id, const BrgemmParams& p) {
  const int bm = kernel_tile_m(id), bn = kernel_tile_n(id);
  return (p.k % BK == 0) && (p.vrows % bm == 0) && (p.vcols % bn == 0);
}

namespace {

const char* tf(bool v) { return v ? "true" : "false"; }

template <int BM, int BN, int WM, int WN, bool FULL, int KIND, bool RAGGED>
void launch_vec_kk(const BrgemmParams& p, dim3 grid, hipStream_t stream, std::string* name_out) {
  if (name_out) {
    char buf[128];
    std::snprintf(buf, sizeof buf, "brgemm_bf16_vec_kernel<%d, %d, %d, %d, %s, %d, %s>", BM, BN,
                  WM, WN, tf(FULL), KIND, tf(RAGGED));
    *name_out = buf;
    return;
  }
  hipLaunchKernelGGL((brgemm_bf16_vec_kernel<BM, BN, WM, WN, FULL, KIND, RAGGED>), grid,
                     dim3(64 * WM * WN), 0, stream, p);
}

template <int BM, int BN, int WM, int WN, int KIND>
void launch_vec_k(const BrgemmParams& p, bool full, dim3 grid, hipStream_t stream,
                  std::string* name_out) {
  if (p.ragged)
    launch_vec_kk<BM, BN, WM, WN, false, KIND, true>(p, grid, stream, name_out);
  else if (full)
    launch_vec_kk<BM, BN, WM, WN, true, KIND, false>(p, grid, stream, name_out);
  else
    launch_vec_kk<BM, BN, WM, WN, false, KIND, false>(p, grid, stream, name_out);
}

template <int BM, int BN, int WM, int WN>
void launch_vec(const BrgemmParams& p, bool full, dim3 grid, hipStream_t stream,
                std::string* name_out) {
  switch (p.kind) {
    case TPP_BR_STRIDE:
      launch_vec_k<BM, BN, WM, WN, TPP_BR_STRIDE>(p, full, grid, stream, name_out);
      break;
    case TPP_BR_OFFSET:
      launch_vec_k<BM, BN, WM, WN, TPP_BR_OFFSET>(p, full, grid, stream, name_out);
      break;
    default:
      launch_vec_k<BM, BN, WM, WN, TPP_BR_ADDRESS>(p, full, grid, stream, name_out);
      break;
  }
}

}  // namespace

hipError_t launch_brgemm(BrgemmParams& p, int32_t id, hipStream_t stream, std::string* name_out) {
  if (id < 0 || id >= K_COUNT) return hipErrorInvalidValue;
  // transposed operands only on the 64-k direct-to-LDS instances
  if ((p.a_trans || p.b_trans) && id != K_BF16_DL64K_256x256 && id != K_BF16_DL64K_128x128 &&
      id != K_BF16_DL64K_64x64)
    return hipErrorInvalidValue;
  const int bm = kInfo[id].bm, bn = kInfo[id].bn;
  p.tiles_m = (p.vrows + bm - 1) / bm;
  p.tiles_n = (p.vcols + bn - 1) / bn;
  p.total_tiles = p.groups * p.tiles_m * p.tiles_n;
  {
    const int32_t band = p.tiles_m < 8 ? p.tiles_m : 8;
    const int32_t last = p.tiles_m % 8 ? p.tiles_m % 8 : 8;
    const int32_t kstep = id == K_F32_GENERIC ? (f32_paired(p) ? F_BK / 2 : F_BK)
                          : kInfo[id].kstep > 1 ? kInfo[id].kstep : BK;
    p.div_m = FastDiv(p.vm);
    p.div_n = FastDiv(p.n);
    p.div_gm = FastDiv(p.gm > 0 && p.gm < (1LL << 31) ? p.gm : 1);
    p.div_group = FastDiv((int64_t)p.tiles_m * p.tiles_n);
    p.div_band = FastDiv((int64_t)band * p.tiles_n);
    p.div_tiles = FastDiv(p.total_tiles > 0 ? p.total_tiles : 1);
    p.div_rows = FastDiv(band);
    p.div_last = FastDiv(last);
    p.div_split = FastDiv(p.split > 1 ? p.split : 1);
    p.div_ks = FastDiv((p.k + kstep - 1) / kstep);
    if (p.split > 1) {   // stride and offset kinds, and single lists: `count` pairs everywhere
      const int64_t stages = id == K_F32_GENERIC ? f32_stages(p, p.count)
                                                 : p.count * ((p.k + kstep - 1) / kstep);
      p.split_base = (int32_t)(stages / p.split);
      p.split_rem = (int32_t)(stages % p.split);
    }
  }
  if (p.total_tiles <= 0) {
    if (name_out) *name_out = "";
    return hipSuccess;
  }
  const dim3 grid((unsigned)p.total_tiles), block(NT);
  const bool full = kernel_full(id, p);
  switch (id) {
    case K_BF16_256x256: launch_vec<256, 256, 2, 4>(p, full, grid, stream, name_out); break;
    case K_BF16_128x128: launch_vec<128, 128, 2, 2>(p, full, grid, stream, name_out); break;
    case K_BF16_64x64: launch_vec<64, 64, 2, 2>(p, full, grid, stream, name_out); break;
    case K_BF16_DL_256x256:
    case K_BF16_DL_128x128:
    case K_BF16_DL_64x64:
    case K_BF16_PP_256x256:
    case K_BF16_DL64K_256x256:
    case K_BF16_DL64K_128x128:
    case K_BF16_DL64K_64x64: {
      if (p.split <= 1) return launch_brgemm_dl(p, id, full, grid, stream, name_out);
      // split over the stage list: chunk partials, then the finishing sum and epilogue
      const hipError_t e = launch_brgemm_dl(p, id, full, dim3((unsigned)(p.total_tiles * p.split)),
                                            stream, name_out);
      if (e != hipSuccess) return e;
      int wm = 0, wn = 0;
      if (!dl_wave_grid(id, wm, wn)) return hipErrorInvalidValue;
      if (name_out) {
        *name_out += " + brgemm_dl_split_finish";
        return hipSuccess;
      }
      const int32_t per_tile = bm * bn / 4 / NT;
      hipLaunchKernelGGL(brgemm_dl_split_finish, dim3((unsigned)(p.total_tiles * per_tile)),
                         block, 0, stream, p, bm, bn, wm, wn, per_tile);
      break;
    }
    case K_BF16_GENERIC:
      if (name_out) {
        *name_out = "brgemm_bf16_kernel<64, 64, 2, 2>";
        return hipSuccess;
      }
      hipLaunchKernelGGL((brgemm_bf16_kernel<64, 64, 2, 2>), grid, block, 0, stream, p);
      break;
    default: {
      // windows of four rows and four k inside every block (plan_launch pads p.vm to match)
      const bool vec = f32_vec(p), paired = f32_paired(p);
      if (name_out) {
        *name_out = paired ? (p.kind == TPP_BR_STRIDE ? "brgemm_f32_paired_stride_kernel<true>"
                                                      : "brgemm_f32_paired_kernel<true>")
                    : vec  ? "brgemm_f32_kernel<true>"
                           : "brgemm_f32_kernel<false>";
        if (p.split > 1) *name_out += " + brgemm_f32_split_finish";
        return hipSuccess;
      }
      const dim3 g = p.split > 1 ? dim3((unsigned)(p.total_tiles * p.split)) : grid;
      if (paired && p.kind == TPP_BR_STRIDE)
        hipLaunchKernelGGL(brgemm_f32_paired_stride_kernel<true>, g, dim3(F_NT), 0, stream, p);
      else if (paired)
        hipLaunchKernelGGL(brgemm_f32_paired_kernel<true>, g, dim3(F_NT), 0, stream, p);
      else if (vec)
        hipLaunchKernelGGL(brgemm_f32_kernel<true>, g, dim3(F_NT), 0, stream, p);
      else
        hipLaunchKernelGGL(brgemm_f32_kernel<false>, g, block, 0, stream, p);
      if (p.split > 1)
        hipLaunchKernelGGL(brgemm_f32_split_finish, dim3((unsigned)(p.total_tiles * 4)), block, 0,
                           stream, p);
      break;
    }
  }
  return name_out ? hipSuccess : hipGetLastError();
}

bool f32_vec(const BrgemmParams& p) {
  // padded rows that still count in 32 bits, and 512 threads per tile that HIP accepts as a grid
  const int64_t rows = ((int64_t)p.m + 3) / 4 * 4 * (p.fused ? p.gm : 1);
  const int64_t tiles = p.groups * ((rows + F_BM - 1) / F_BM) * (((int64_t)p.vcols + F_BN - 1) / F_BN);
  return p.m >= 4 && p.k >= 4 && rows < (1LL << 31) - 512 && tiles * F_NT < (1LL << 32);
}

bool f32_paired(const BrgemmParams& p) { return f32_vec(p) && (p.k + 31) / 32 % 2 != 0; }

int64_t f32_stages(const BrgemmParams& p, int64_t pairs) {
  return f32_paired(p) ? (pairs * ((p.k + 31) / 32) + 1) / 2
                       : pairs * (((int64_t)p.k + F_BK - 1) / F_BK);
}

int64_t f32_split_ws_floats(int32_t split, int64_t total_tiles) {
  return (int64_t)split * total_tiles * F_BM * F_BN;
}

}  // namespace tpp
