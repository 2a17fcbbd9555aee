// equation.hip -- TPP matrix equations (Sec. 4) for gfx950: the planner of Alg. 3 / Alg. 4 on the
// host, and an executor that evaluates the planned instruction list per output element.
//
// Executor: eight output elements per thread.  Chains of steps onto one running value (the common
// forms) have a kernel of their own (equation_chain_kernel).  In general each instruction of the plan
// dispatches once and then runs over the eight elements (equation_vec_kernel); the temporaries of
// the plan are named registers, so the plan's reuse of temporaries is register reuse: the paper's
// Strategy 2.  The instruction list lives in the kernel arguments, one word per instruction.
#include <hip/hip_runtime.h>

#include <math.h>

#include <vector>

#include "brgemm_device.h"
#include "internal.h"

namespace tpp {

// ---- planner (host) --------------------------------------------------------------------------
namespace {

bool op_fits(int32_t arity, int32_t op) {
  switch (arity) {
    case TPP_EQ_LEAF: return true;
    case TPP_EQ_UNARY: return op >= TPP_EQ_IDENTITY && op <= TPP_EQ_SIGMOID;
    case TPP_EQ_BINARY: return op >= TPP_EQ_ADD && op <= TPP_EQ_MIN;
    case TPP_EQ_TERNARY: return op == TPP_EQ_MULADD;
    default: return false;
  }
}

bool is_leaf(const tpp_eq_node* nodes, int32_t i) { return nodes[i].arity == TPP_EQ_LEAF; }

// Nodes reachable from the root in post-order (children before parents), checking that every
// reachable node is reached once and well formed.  Iterative, with an explicit stack.
const char* post_order(const tpp_eq_node* nodes, int32_t n_nodes, int32_t root,
                       std::vector<int32_t>& order) {
  if (root < 0 || root >= n_nodes) return "root index out of range";
  std::vector<char> seen(n_nodes, 0);
  std::vector<std::pair<int32_t, int32_t>> stack;   // (node, next child to visit)
  stack.push_back({root, 0});
  seen[root] = 1;
  while (!stack.empty()) {
    auto& top = stack.back();
    const tpp_eq_node& x = nodes[top.first];
    if (x.arity < TPP_EQ_LEAF || x.arity > TPP_EQ_TERNARY) return "arity outside [0, 3]";
    if (!op_fits(x.arity, x.op)) return "operation of the wrong arity";
    if (top.second < x.arity) {
      const int32_t c = x.child[top.second++];
      if (c < 0 || c >= n_nodes) return "child index out of range";
      if (seen[c]) return "a node is reached twice (not a tree)";
      seen[c] = 1;
      stack.push_back({c, 0});
    } else {
      order.push_back(top.first);
      stack.pop_back();
    }
  }
  return nullptr;
}

struct TmpPool {
  uint64_t used = 0;
  int32_t high = 0;
  int32_t reserve() {   // the lowest free id
    int32_t i = 0;
    while (used >> i & 1) ++i;
    used |= uint64_t(1) << i;
    if (i + 1 > high) high = i + 1;
    return i;
  }
  void recycle(int32_t t) {
    if (t >= 0) used &= ~(uint64_t(1) << t);
  }
};

void plan_node(const tpp_eq_node* nodes, int32_t r, tpp_eq_plan_node* plan, int32_t& clock,
               TmpPool& pool) {
  const tpp_eq_node& x = nodes[r];
  if (x.arity == TPP_EQ_LEAF) return;
  // children by decreasing score; among equal scores the earlier child first (stable)
  int32_t idx[3] = {0, 1, 2};
  for (int a = 1; a < x.arity; ++a)
    for (int b = a; b > 0 && plan[x.child[idx[b]]].score > plan[x.child[idx[b - 1]]].score; --b) {
      const int32_t t = idx[b];
      idx[b] = idx[b - 1];
      idx[b - 1] = t;
    }
  for (int a = 0; a < x.arity; ++a) plan_node(nodes, x.child[idx[a]], plan, clock, pool);
  plan[r].timestamp = clock++;
  bool all_leaves = true;
  for (int a = 0; a < x.arity; ++a) all_leaves = all_leaves && is_leaf(nodes, x.child[a]);
  if (all_leaves) {
    plan[r].tmp = pool.reserve();
    return;
  }
  // the temporary the node takes over: Left's, else Right's (ternary), else the other child's
  int keep = 1;
  if (!is_leaf(nodes, x.child[0])) keep = 0;
  else if (x.arity == TPP_EQ_TERNARY && !is_leaf(nodes, x.child[2])) keep = 2;
  plan[r].tmp = plan[x.child[keep]].tmp;
  for (int a = 0; a < x.arity; ++a)
    if (a != keep) pool.recycle(plan[x.child[a]].tmp);
}

}  // namespace

const char* equation_plan(const tpp_eq_node* nodes, int32_t n_nodes, int32_t root,
                          tpp_eq_plan_node* plan, int32_t* n_tmps) {
  if (!nodes || !plan || !n_tmps) return "NULL nodes, plan or n_tmps";
  if (n_nodes < 1 || n_nodes > EQ_MAX_NODES) return "n_nodes must be in [1, 64]";
  std::vector<int32_t> order;
  if (const char* err = post_order(nodes, n_nodes, root, order)) return err;
  for (int32_t i = 0; i < n_nodes; ++i) plan[i] = {0, -1, -1};
  // Alg. 3 over the post-order (children are scored before their parent)
  for (int32_t r : order) {
    const tpp_eq_node& x = nodes[r];
    int32_t s = 0;
    if (x.arity == TPP_EQ_UNARY) {
      s = is_leaf(nodes, x.child[0]) ? 1 : plan[x.child[0]].score;
    } else if (x.arity == TPP_EQ_BINARY) {
      const int32_t a = plan[x.child[0]].score, b = plan[x.child[1]].score;
      s = a == b ? a + 1 : (a > b ? a : b);
    } else if (x.arity == TPP_EQ_TERNARY) {
      if (is_leaf(nodes, x.child[0]) && is_leaf(nodes, x.child[1]) && is_leaf(nodes, x.child[2])) {
        s = 1;
      } else {
        s = 3;
        for (int a = 0; a < 3; ++a)
          if (plan[x.child[a]].score > s) s = plan[x.child[a]].score;
      }
    }
    plan[r].score = s;
  }
  // Alg. 4
  int32_t clock = 0;
  TmpPool pool;
  plan_node(nodes, root, plan, clock, pool);
  *n_tmps = pool.high;
  return nullptr;
}

const char* equation_compile(const tpp_eq_node* nodes, int32_t n_nodes, int32_t root,
                             EqProgram& prog, bool* too_many_tmps) {
  *too_many_tmps = false;
  tpp_eq_plan_node plan[EQ_MAX_NODES];
  int32_t n_tmps = 0;
  if (const char* err = equation_plan(nodes, n_nodes, root, plan, &n_tmps)) return err;
  if (nodes[root].arity == TPP_EQ_LEAF) {   // the output is a copy of one leaf
    prog.n_instr = 1;
    prog.instr[0] = {TPP_EQ_IDENTITY, 1, 0, {EQ_LEAF_BASE + nodes[root].leaf, 0, 0}};
    return nullptr;
  }
  if (n_tmps > EQ_MAX_TMPS) {
    *too_many_tmps = true;
    return "the plan needs more than 8 temporaries";
  }
  int32_t n_instr = 0;
  for (int32_t i = 0; i < n_nodes; ++i)
    if (plan[i].timestamp >= 0) ++n_instr;
  for (int32_t i = 0; i < n_nodes; ++i) {
    const int32_t t = plan[i].timestamp;
    if (t < 0) continue;
    const tpp_eq_node& x = nodes[i];
    EqInstr& in = prog.instr[t];
    in.op = x.op;
    in.arity = x.arity;
    in.dst = plan[i].tmp;
    for (int a = 0; a < 3; ++a) {
      if (a >= x.arity) {
        in.src[a] = 0;
        continue;
      }
      const int32_t c = x.child[a];
      in.src[a] = is_leaf(nodes, c) ? EQ_LEAF_BASE + nodes[c].leaf : plan[c].tmp;
    }
  }
  prog.n_instr = n_instr;
  return nullptr;
}

// ---- executor (device) -----------------------------------------------------------------------
namespace {

using namespace dev;

constexpr int EQ_T = 256;   // threads per workgroup

constexpr int EPT = 8;   // output elements per thread
constexpr int64_t EQ_SMALL = 1 << 16;   // elements up to which few-row outputs run one per thread

// v[k] = op(a[k], b[k], cc[k]) for the EPT elements, one dispatch on op.
#define TPP_EQ_OP_CASE(op, expr) \
  case op: { _Pragma("unroll") for (int k = 0; k < EPT; ++k) v[k] = (expr); } break;
#define TPP_EQ_APPLY(opcode)                                                                    \
  switch (opcode) {                                                                             \
    TPP_EQ_OP_CASE(TPP_EQ_IDENTITY, a[k])                                                       \
    TPP_EQ_OP_CASE(TPP_EQ_NEG, -a[k])                                                           \
    TPP_EQ_OP_CASE(TPP_EQ_EXP, expf(a[k]))                                                      \
    TPP_EQ_OP_CASE(TPP_EQ_TANH, tanhf(a[k]))                                                    \
    TPP_EQ_OP_CASE(TPP_EQ_RELU, a[k] > 0.0f ? a[k] : 0.0f)                                      \
    TPP_EQ_OP_CASE(TPP_EQ_GELU_TANH, gelu_tanh(a[k]))                                           \
    TPP_EQ_OP_CASE(TPP_EQ_SQRT, sqrtf(a[k]))                                                    \
    TPP_EQ_OP_CASE(TPP_EQ_RCP, 1.0f / a[k])                                                     \
    TPP_EQ_OP_CASE(TPP_EQ_SQUARE, a[k] * a[k])                                                  \
    TPP_EQ_OP_CASE(TPP_EQ_SIGMOID, 1.0f / (1.0f + expf(-a[k])))                                 \
    TPP_EQ_OP_CASE(TPP_EQ_ADD, a[k] + b[k])                                                     \
    TPP_EQ_OP_CASE(TPP_EQ_SUB, a[k] - b[k])                                                     \
    TPP_EQ_OP_CASE(TPP_EQ_MUL, a[k] * b[k])                                                     \
    TPP_EQ_OP_CASE(TPP_EQ_DIV, a[k] / b[k])                                                     \
    TPP_EQ_OP_CASE(TPP_EQ_MAX, a[k] > b[k] ? a[k] : b[k])                                       \
    TPP_EQ_OP_CASE(TPP_EQ_MIN, a[k] < b[k] ? a[k] : b[k])                                       \
    TPP_EQ_OP_CASE(TPP_EQ_MULADD, __builtin_fmaf(a[k], b[k], cc[k]))                            \
    default: { _Pragma("unroll") for (int k = 0; k < EPT; ++k) v[k] = 0.0f; } break;            \
  }

// Packed instruction word: op, arity, destination and three operand codes.
__device__ __forceinline__ int32_t eq_op(uint32_t w) { return (int32_t)(w & 63u); }
__device__ __forceinline__ int32_t eq_arity(uint32_t w) { return (int32_t)(w >> 6 & 3u); }
__device__ __forceinline__ int32_t eq_dst(uint32_t w) { return (int32_t)(w >> 8 & 63u); }
__device__ __forceinline__ int32_t eq_src(uint32_t w, int a) {
  return (int32_t)(w >> (14 + 6 * a) & 63u);
}
// Entry j (wave-uniform) of a leaf table of which each lane holds entry lane % EQ_MAX_ARGS.
__device__ __forceinline__ EqArg eq_arg_of(const EqArg& mine, int32_t j) {
  const auto pick = [&](uint64_t v) {
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), j) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, j);
  };
  EqArg g;
  g.ptr = reinterpret_cast<const void*>(pick(reinterpret_cast<uint64_t>(mine.ptr)));
  g.ld = (int64_t)pick((uint64_t)mine.ld);
  g.bf16 = __builtin_amdgcn_readlane(mine.bf16, j);
  g.bcast = __builtin_amdgcn_readlane(mine.bcast, j);
  return g;
}

// Outputs of fewer than 8 rows (and more than EQ_SMALL elements, not contiguous):
// EPT output elements per thread, in column-major element order: element k of thread t in
// workgroup b is e = (b * EPT + k) * EQ_T + t, so for every k a wavefront covers 64 consecutive
// elements (contiguous runs of every full-tensor leaf and of the output, whatever the shape: a
// 1 x n row of statistics as well as a tall tensor).  Each instruction of the plan dispatches
// once on its operands' kind and once on its operation, then runs over the EPT elements without
// further branches: the interpretation cost is shared by EPT elements.  The temporaries are
// named register arrays (the plan's reuse of temporaries is register reuse).  WIDE: m * n does
// not fit 32 bits.
template <bool OUT_BF16, bool WIDE>
__global__ __launch_bounds__(EQ_T) void equation_kernel(EqArgs p) {
  const uint32_t words = p.instr[threadIdx.x & 63];
  const int64_t total = (int64_t)p.m * p.n;
  const int64_t step = (int64_t)gridDim.x * EPT * EQ_T;
  for (int64_t e0 = (int64_t)blockIdx.x * EPT * EQ_T + threadIdx.x; e0 < total; e0 += step) {
    int32_t r[EPT], c[EPT];
    bool ok[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const int64_t e = e0 + (int64_t)k * EQ_T;
      ok[k] = e < total;
      const int64_t ee = ok[k] ? e : 0;   // element 0 stands in past the end
      c[k] = WIDE ? (int32_t)(ee / p.m) : (int32_t)((uint32_t)ee / (uint32_t)p.m);
      r[k] = (int32_t)(ee - (int64_t)c[k] * p.m);
    }
    float t0[EPT], t1[EPT], t2[EPT], t3[EPT], t4[EPT], t5[EPT], t6[EPT], t7[EPT];
    // FETCH: operand `code` of all EPT elements into o (a temporary, or a leaf loaded for each
    // element); PUT: v into temporary `code`.  Expanded in place (statement macros), so that
    // every array index is a compile-time constant and the arrays stay in registers.
#define TPP_EQ_TMP_CASE(j, o) \
    case j: { _Pragma("unroll") for (int k = 0; k < EPT; ++k) o[k] = t##j[k]; } break;
#define FETCH(code, o)                                                                          \
    switch (code) {                                                                             \
      TPP_EQ_TMP_CASE(0, o) TPP_EQ_TMP_CASE(1, o) TPP_EQ_TMP_CASE(2, o) TPP_EQ_TMP_CASE(3, o)     \
      TPP_EQ_TMP_CASE(4, o) TPP_EQ_TMP_CASE(5, o) TPP_EQ_TMP_CASE(6, o) TPP_EQ_TMP_CASE(7, o)     \
      default: {                                                                                \
        const EqArg& g = p.varg[(code) - EQ_V_LEAF];                                          \
        _Pragma("unroll") for (int k = 0; k < EPT; ++k) {                                       \
          const int64_t at = g.bcast == TPP_BC_NONE ? (int64_t)r[k] + (int64_t)c[k] * g.ld      \
                             : g.bcast == TPP_BC_COL ? r[k] : g.bcast == TPP_BC_ROW ? c[k] : 0; \
          o[k] = g.bf16 ? bf16_bits_to_f32(gld<uint16_t>(static_cast<const uint16_t*>(g.ptr) + at)) \
                        : gld<float>(static_cast<const float*>(g.ptr) + at);                    \
        }                                                                                       \
      } break;                                                                                  \
    }
#define TPP_EQ_PUT_CASE(j) \
    case j: { _Pragma("unroll") for (int k = 0; k < EPT; ++k) t##j[k] = v[k]; } break;
#define PUT(code)                                                                               \
    switch (code) {                                                                             \
      TPP_EQ_PUT_CASE(0) TPP_EQ_PUT_CASE(1) TPP_EQ_PUT_CASE(2) TPP_EQ_PUT_CASE(3)                \
      TPP_EQ_PUT_CASE(4) TPP_EQ_PUT_CASE(5) TPP_EQ_PUT_CASE(6) TPP_EQ_PUT_CASE(7)                \
      default: break;                                                                           \
    }
    for (int32_t i = 0; i < p.n_v; ++i) {
      const uint32_t in = (uint32_t)__builtin_amdgcn_readlane((int)words, i);
      float a[EPT], b[EPT], cc[EPT], v[EPT];
      FETCH(eq_src(in, 0), a)
      if (eq_arity(in) > 1) { FETCH(eq_src(in, 1), b) }
      if (eq_arity(in) > 2) { FETCH(eq_src(in, 2), cc) }
      TPP_EQ_APPLY(eq_op(in))
      PUT(eq_dst(in))
    }
    float res[EPT];
    FETCH(eq_dst((uint32_t)__builtin_amdgcn_readlane((int)words, p.n_v - 1)), res)
#undef FETCH
#undef PUT
#undef TPP_EQ_TMP_CASE
#undef TPP_EQ_PUT_CASE
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      if (!ok[k]) continue;
      const int64_t at = (int64_t)r[k] + (int64_t)c[k] * p.ldo;
      if (OUT_BF16)
        gst<uint16_t>(static_cast<uint16_t*>(p.out) + at, f32_to_bf16_bits(res[k]));
      else
        gst<float>(static_cast<float*>(p.out) + at, res[k]);
    }
  }
}

__device__ __forceinline__ float eq_apply1(int32_t op, float a, float b, float c) {
  switch (op) {
    case TPP_EQ_IDENTITY: return a;
    case TPP_EQ_NEG: return -a;
    case TPP_EQ_EXP: return expf(a);
    case TPP_EQ_TANH: return tanhf(a);
    case TPP_EQ_RELU: return a > 0.0f ? a : 0.0f;
    case TPP_EQ_GELU_TANH: return gelu_tanh(a);
    case TPP_EQ_SQRT: return sqrtf(a);
    case TPP_EQ_RCP: return 1.0f / a;
    case TPP_EQ_SQUARE: return a * a;
    case TPP_EQ_SIGMOID: return 1.0f / (1.0f + expf(-a));
    case TPP_EQ_ADD: return a + b;
    case TPP_EQ_SUB: return a - b;
    case TPP_EQ_MUL: return a * b;
    case TPP_EQ_DIV: return a / b;
    case TPP_EQ_MAX: return a > b ? a : b;
    case TPP_EQ_MIN: return a < b ? a : b;
    case TPP_EQ_MULADD: return __builtin_fmaf(a, b, c);
    default: return 0.0f;
  }
}

// Small outputs of fewer than 8 rows (at most EQ_SMALL elements, e.g. a 1 x n row of statistics):
// one element per thread, so that the grid has as many workgroups as the elements allow, and every
// leaf of the element loaded before the first instruction runs.  Bound by latency: the kernel
// arguments (the program and the leaf table are each read by one load per wavefront, a word per
// lane), one round of leaf loads, then the instructions.  Each thread's temporaries and leaves
// live in its own column of LDS, so an operand is one LDS read at a computed address, no branches.
template <bool OUT_BF16>
__global__ __launch_bounds__(EQ_T) void equation_small_kernel(EqArgs p) {
  extern __shared__ float eq_file[];   // [EQ_V_LEAF + n_args][EQ_T]
  const int lane = threadIdx.x & 63;
  const uint32_t words = p.instr[lane];
  const EqArg mine = p.varg[lane & (EQ_MAX_ARGS - 1)];
  const int32_t total = p.m * p.n;   // at most EQ_SMALL
  const int32_t e = (int32_t)blockIdx.x * EQ_T + (int32_t)threadIdx.x;
  const int32_t ee = e < total ? e : 0;
  const int32_t c = ee / p.m, r = ee - c * p.m;
  float* const file = eq_file + threadIdx.x;
  // leaves in rounds of four, every load of a round issued before the first is stored
  for (int32_t j0 = 0; j0 < p.n_varg; j0 += 4) {
    float x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      x[k] = 0.0f;
      const EqArg g = eq_arg_of(mine, j0 + k < p.n_varg ? j0 + k : j0);
      const int64_t at = g.bcast == TPP_BC_NONE ? (int64_t)r + (int64_t)c * g.ld
                         : g.bcast == TPP_BC_COL ? r : g.bcast == TPP_BC_ROW ? c : 0;
      if (g.bf16)
        x[k] = bf16_bits_to_f32(gld<uint16_t>(static_cast<const uint16_t*>(g.ptr) + at));
      else
        x[k] = gld<float>(static_cast<const float*>(g.ptr) + at);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (j0 + k < p.n_varg) file[(EQ_V_LEAF + j0 + k) * EQ_T] = x[k];
  }
  float v = 0.0f;
  for (int32_t i = 0; i < p.n_v; ++i) {
    const uint32_t in = (uint32_t)__builtin_amdgcn_readlane((int)words, i);
    const int32_t ar = eq_arity(in);
    const float a = file[eq_src(in, 0) * EQ_T];
    const float b = ar > 1 ? file[eq_src(in, 1) * EQ_T] : 0.0f;
    const float cc = ar > 2 ? file[eq_src(in, 2) * EQ_T] : 0.0f;
    v = eq_apply1(eq_op(in), a, b, cc);
    file[eq_dst(in) * EQ_T] = v;
  }
  // the last instruction is the root
  if (e >= total) return;
  const int64_t at = (int64_t)r + (int64_t)c * p.ldo;
  if (OUT_BF16)
    gst<uint16_t>(static_cast<uint16_t*>(p.out) + at, f32_to_bf16_bits(v));
  else
    gst<float>(static_cast<float*>(p.out) + at, v);
}

struct EqRaw {   // 8 entries of a leaf as loaded: 16 bytes of bf16 (lo), or 32 of fp32
  u32x4 lo, hi;
};
__device__ __forceinline__ void eq_load8(EqRaw& w, const void* ptr, bool bf16) {
  if (bf16) {
    w.lo = gld<u32x4_a2>(ptr);
  } else {
    w.lo = gld<u32x4_a4>(ptr);
    w.hi = gld<u32x4_a4>(static_cast<const char*>(ptr) + 16);
  }
}
__device__ __forceinline__ void eq_widen8(const EqRaw& w, bool bf16, float (&o)[EPT]) {
  if (bf16) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      o[2 * q] = __uint_as_float(w.lo[q] << 16);
      o[2 * q + 1] = __uint_as_float(w.lo[q] & 0xffff0000u);
    }
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      o[q] = __uint_as_float(w.lo[q]);
      o[q + 4] = __uint_as_float(w.hi[q]);
    }
  }
}

// The row-uniform part of a program (U): lane l computes it for column c0 + l (cn columns) into the
// wavefront's file, slot by slot.
__device__ __forceinline__ void eq_column_part(const EqArgs& p, uint32_t words, const EqArg& mine_u,
                                               float* file, int32_t c0, int32_t cn) {
  const int lane = threadIdx.x & 63;
  const int32_t cu = c0 + (lane < cn ? lane : 0);
  for (int32_t j0 = 0; j0 < p.n_uarg; j0 += 4) {
    float x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const EqArg g = eq_arg_of(mine_u, j0 + k < p.n_uarg ? j0 + k : j0);
      const int64_t e = g.bcast == TPP_BC_ROW ? cu : 0;
      if (g.bf16)
        x[k] = bf16_bits_to_f32(gld<uint16_t>(static_cast<const uint16_t*>(g.ptr) + e));
      else
        x[k] = gld<float>(static_cast<const float*>(g.ptr) + e);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (j0 + k < p.n_uarg) file[(j0 + k) * 64 + lane] = x[k];
  }
  for (int32_t i = 0; i < p.n_u; ++i) {
    const uint32_t in = (uint32_t)__builtin_amdgcn_readlane((int)words, i);
    const int32_t ar = eq_arity(in);
    const float a = file[eq_src(in, 0) * 64 + lane];
    const float b = ar > 1 ? file[eq_src(in, 1) * 64 + lane] : 0.0f;
    const float cc = ar > 2 ? file[eq_src(in, 2) * 64 + lane] : 0.0f;
    file[eq_dst(in) * 64 + lane] = eq_apply1(eq_op(in), a, b, cc);
  }
}

// Chains, the programs of at least 8 rows whose per-element part is  x = leaf;  x = fma(x, X, Y) step
// by step;  one unary operation at the end.  Add, sub, mul, neg and muladd onto the running value
// are such steps with the same rounding (x + o = fma(x, 1, o), x o = fma(x, o, -0), and so on), X
// and Y being values of the column (or 1 and -0) or V leaves.  These are the forms that norms,
// softmaxes, biases, scalings and residuals take.  HBM-bound once nothing else is in the way:
//   - No operand or operation dispatch per instruction (see equation_vec_kernel).  Steps on values
//     of the column run in a loop of two LDS reads and eight fma; at most NVS steps have V leaves.
//   - The part of the tree that is the same for all rows (its leaves are row or scalar leaves: a
//     norm's mean, a softmax's reciprocal) runs once per column and not per element.  A wavefront
//     owns one group of at most 64 row chunks (8 rows each) and cw consecutive columns: before its
//     walk over them lane l computes that part for column c0 + l into the wavefront's LDS file.
//   - A lane keeps its chunk for the whole walk (q columns a step when a column has fewer than 33
//     chunks), so column leaves are loaded once; full leaves are loaded one step ahead.
//   - Loads and stores are 16 bytes at any element alignment.  The last chunk of a column takes the
//     8-row window that ends with it and stores its own rows one by one.
// Layer norm's normalize step on 1024 x 8192 bf16: 20.5 us in equation_vec_kernel, 10.8 here;
// softmax's exp(x - max) on 512 x 32768, bf16 to fp32: 26.0 and 21.6; its scaling by rcp(sum),
// fp32 to bf16: 22.5 and 19.6 (100 MB each: 4.7 and 5.1 TB/s).
// Order: n_step[0] column steps, V step A, n_step[1] column steps, V step B, n_step[2] column steps.
struct EqWalk {   // the lane's part of a wavefront's region
  int32_t c0, cn, sub, r, first;
  bool mine;
};
__device__ __forceinline__ bool eq_walk(const EqArgs& p, int lane, int wave, EqWalk& k) {
  const int64_t region = (int64_t)blockIdx.x * (EQ_T / 64) + wave;
  const int64_t tile = region / p.ng;
  if (tile >= p.tiles) return false;
  const int32_t grp = (int32_t)(region - tile * p.ng);
  k.c0 = (int32_t)(tile * p.cw);
  k.cn = p.n - k.c0 < p.cw ? p.n - k.c0 : p.cw;
  k.sub = lane / p.w;
  const int32_t chunk = grp * p.w + (lane - k.sub * p.w);
  k.mine = k.sub < p.q && chunk * 8 < p.m;
  const int32_t r0 = k.mine ? chunk * 8 : 0;
  k.first = p.m - r0 < 8 ? 8 - (p.m - r0) : 0;   // r0 + 8 may pass 2^31 - 1
  k.r = r0 - k.first;
  return true;
}

template <bool OUT_BF16>
__device__ __forceinline__ void eq_store8(void* out, int64_t o, int32_t first, const float (&v)[EPT]) {
  if (first == 0) {
    if (OUT_BF16) {
      gst<u32x4_a2>(static_cast<uint16_t*>(out) + o,
                    (u32x4){pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                            pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])});
    } else {
      float* const q = static_cast<float*>(out) + o;
      gst<f32x4_a4>(q, (f32x4){v[0], v[1], v[2], v[3]});
      gst<f32x4_a4>(q + 4, (f32x4){v[4], v[5], v[6], v[7]});
    }
    return;
  }
#pragma unroll
  for (int k = 1; k < EPT; ++k) {
    if (k < first) continue;
    if (OUT_BF16)
      gst<uint16_t>(static_cast<uint16_t*>(out) + o + k, f32_to_bf16_bits(v[k]));
    else
      gst<float>(static_cast<float*>(out) + o + k, v[k]);
  }
}

// v = op(a) for a unary operation, one dispatch for the 8 elements.
__device__ __forceinline__ void eq_unary8(int32_t op, const float (&a)[EPT], float (&v)[EPT]) {
  const float(&b)[EPT] = a, (&cc)[EPT] = a;
  TPP_EQ_APPLY(op)
}

template <bool OUT_BF16, int NVS>
__global__ __launch_bounds__(EQ_T) void equation_chain_kernel(EqArgs p) {
  constexpr int NL = 1 + 2 * NVS;      // leaves: the first, then X and Y of each V step
  extern __shared__ float eq_file[];   // [4 waves][uslots][64 columns]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  EqWalk k;
  if (!eq_walk(p, lane, wave, k)) return;   // wave-uniform; no workgroup barrier below
  float* const file = eq_file + wave * p.uslots * 64;

  EqRaw raw[NL];
  const char* at[NL];
  int64_t step[NL];
  int32_t ci = k.sub;                  // the lane's column is c0 + ci
  bool ok = k.mine && ci < k.cn;
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const EqArg& g = p.varg[j];
    const int64_t es = g.bf16 ? 2 : 4;
    const bool full = g.bcast == TPP_BC_NONE;
    at[j] = static_cast<const char*>(g.ptr) + (k.r + (full ? ((int64_t)k.c0 + ci) * g.ld : 0)) * es;
    step[j] = full ? p.q * g.ld * es : 0;
    if (ok && g.ptr) eq_load8(raw[j], at[j], g.bf16 != 0);
  }
  eq_column_part(p, p.n_u > 0 ? p.instr[lane] : 0u, p.uarg[lane & (EQ_MAX_ARGS - 1)], file, k.c0,
                 k.cn);
  file[(p.uslots - 2) * 64 + lane] = 1.0f;
  file[(p.uslots - 1) * 64 + lane] = -0.0f;
  // the columns below are read by other lanes of the wavefront than wrote them
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

  for (int32_t cs = 0; cs < k.cn; cs += p.q) {   // uniform; ci = cs + sub
    const bool ok_next = k.mine && ci + p.q < k.cn;
    const float* const col = file + (ok ? ci : 0);
    float x[EPT], op[2 * NVS > 0 ? 2 * NVS : 1][EPT];
    eq_widen8(raw[0], p.varg[0].bf16 != 0, x);
#pragma unroll
    for (int j = 1; j < NL; ++j)
      if (p.varg[j].ptr) eq_widen8(raw[j], p.varg[j].bf16 != 0, op[j - 1]);
    // the next step's full leaves, in flight during this one
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      at[j] += step[j];
      if (ok_next && step[j] != 0) eq_load8(raw[j], at[j], p.varg[j].bf16 != 0);
    }
    int32_t s = 0;
#pragma unroll
    for (int a = 0; a <= NVS; ++a) {
      for (int32_t e = s + p.n_step[a]; s < e; ++s) {
        const EqStep st = p.step[s];
        const float X = __uint_as_float(__float_as_uint(col[st.x * 64]) ^ st.xsign);
        const float Y = __uint_as_float(__float_as_uint(col[st.y * 64]) ^ st.ysign);
#pragma unroll
        for (int q = 0; q < EPT; ++q) x[q] = __builtin_fmaf(x[q], X, Y);
      }
      if (a < NVS) {
        const EqStep st = p.vstep[a];
        float(&X)[EPT] = op[2 * a < 2 * NVS ? 2 * a : 0];
        float(&Y)[EPT] = op[2 * a + 1 < 2 * NVS ? 2 * a + 1 : 0];
        if (!p.varg[1 + 2 * a].ptr) {
          const float u = col[st.x * 64];
#pragma unroll
          for (int q = 0; q < EPT; ++q) X[q] = u;
        }
        if (!p.varg[2 + 2 * a].ptr) {
          const float u = col[st.y * 64];
#pragma unroll
          for (int q = 0; q < EPT; ++q) Y[q] = u;
        }
#pragma unroll
        for (int q = 0; q < EPT; ++q)
          x[q] = __builtin_fmaf(x[q], __uint_as_float(__float_as_uint(X[q]) ^ st.xsign),
                                __uint_as_float(__float_as_uint(Y[q]) ^ st.ysign));
      }
    }
    const int64_t o = (int64_t)k.r + ((int64_t)k.c0 + ci) * p.ldo;
    if (p.act == TPP_EQ_IDENTITY) {
      if (ok) eq_store8<OUT_BF16>(p.out, o, k.first, x);
    } else {
      float v[EPT];
      eq_unary8(p.act, x, v);
      if (ok) eq_store8<OUT_BF16>(p.out, o, k.first, v);
    }
    ci += p.q;
    ok = ok_next;
  }
}

// Everything else of at least 8 rows: a thread takes 8 consecutive rows of one column (one index
// split per thread), 8 entries of a full or column leaf as one 16-byte load or two, one entry of a
// row or scalar leaf, and stores its 8 outputs the same way, at any element alignment; the last
// rows of a column as in eq_walk.  Leaves are loaded when their instruction runs: preloading them
// (and evaluating the row-uniform part once per column) in this interpreter, whose switches the
// compiler structures over 8-element arrays, took 121 against 79 us on the 4096 x 4096 fp32 example
// (164 registers against 82).
// NTMP: the temporaries the plan uses are below NTMP (fewer registers, more waves in flight).
template <bool OUT_BF16, int NTMP>
__global__ __launch_bounds__(EQ_T) void equation_vec_kernel(EqArgs p) {
  const int32_t chunks = (p.m - 1) / EPT + 1;
  const int64_t groups = (int64_t)chunks * p.n;
  for (int64_t gidx = (int64_t)blockIdx.x * EQ_T + threadIdx.x; gidx < groups;
       gidx += (int64_t)gridDim.x * EQ_T) {
    const int32_t c = (int32_t)(gidx / chunks);
    const int32_t r0 = (int32_t)(gidx - (int64_t)c * chunks) * EPT;
    const int32_t first = p.m - r0 < EPT ? EPT - (p.m - r0) : 0;   // r0 + EPT may pass 2^31 - 1
    const int32_t r = r0 - first;
    float t0[EPT], t1[EPT], t2[EPT], t3[EPT], t4[EPT], t5[EPT], t6[EPT], t7[EPT];
#define TPP_EQ_TMP_CASE(j, o) \
    case j: if constexpr (j < NTMP) { _Pragma("unroll") for (int k = 0; k < EPT; ++k) o[k] = t##j[k]; } break;
#define FETCH(code, o)                                                                          \
    switch (code) {                                                                             \
      TPP_EQ_TMP_CASE(0, o) TPP_EQ_TMP_CASE(1, o) TPP_EQ_TMP_CASE(2, o) TPP_EQ_TMP_CASE(3, o)     \
      TPP_EQ_TMP_CASE(4, o) TPP_EQ_TMP_CASE(5, o) TPP_EQ_TMP_CASE(6, o) TPP_EQ_TMP_CASE(7, o)     \
      default: {                                                                                \
        const EqArg& g = p.varg[(code) - EQ_V_LEAF];                                            \
        if (g.bcast == TPP_BC_NONE || g.bcast == TPP_BC_COL) {                                  \
          const int64_t at = g.bcast == TPP_BC_NONE ? (int64_t)r + (int64_t)c * g.ld : r;       \
          if (g.bf16) {                                                                         \
            const u32x4 w = gld<u32x4_a2>(static_cast<const uint16_t*>(g.ptr) + at);           \
            _Pragma("unroll") for (int q = 0; q < 4; ++q) {                                     \
              o[2 * q] = __uint_as_float(w[q] << 16);                                           \
              o[2 * q + 1] = __uint_as_float(w[q] & 0xffff0000u);                               \
            }                                                                                   \
          } else {                                                                              \
            const f32x4 lo = gld<f32x4_a4>(static_cast<const float*>(g.ptr) + at);             \
            const f32x4 hi = gld<f32x4_a4>(static_cast<const float*>(g.ptr) + at + 4);         \
            _Pragma("unroll") for (int q = 0; q < 4; ++q) { o[q] = lo[q]; o[q + 4] = hi[q]; }   \
          }                                                                                     \
        } else {                                                                                \
          const int64_t at = g.bcast == TPP_BC_ROW ? c : 0;                                     \
          const float x = g.bf16 ? bf16_bits_to_f32(gld<uint16_t>(static_cast<const uint16_t*>(g.ptr) + at)) \
                                 : gld<float>(static_cast<const float*>(g.ptr) + at);          \
          _Pragma("unroll") for (int k = 0; k < EPT; ++k) o[k] = x;                             \
        }                                                                                       \
      } break;                                                                                  \
    }
#define TPP_EQ_PUT_CASE(j) \
    case j: if constexpr (j < NTMP) { _Pragma("unroll") for (int k = 0; k < EPT; ++k) t##j[k] = v[k]; } break;
#define PUT(code)                                                                               \
    switch (code) {                                                                             \
      TPP_EQ_PUT_CASE(0) TPP_EQ_PUT_CASE(1) TPP_EQ_PUT_CASE(2) TPP_EQ_PUT_CASE(3)                \
      TPP_EQ_PUT_CASE(4) TPP_EQ_PUT_CASE(5) TPP_EQ_PUT_CASE(6) TPP_EQ_PUT_CASE(7)                \
      default: break;                                                                           \
    }
    for (int32_t i = 0; i < p.n_v; ++i) {
      const uint32_t in = p.instr[i];
      float a[EPT], b[EPT], cc[EPT], v[EPT];
      FETCH(eq_src(in, 0), a)
      if (eq_arity(in) > 1) { FETCH(eq_src(in, 1), b) }
      if (eq_arity(in) > 2) { FETCH(eq_src(in, 2), cc) }
      TPP_EQ_APPLY(eq_op(in))
      PUT(eq_dst(in))
    }
    float res[EPT];
    FETCH(eq_dst(p.instr[p.n_v - 1]), res)
#undef FETCH
#undef PUT
#undef TPP_EQ_TMP_CASE
#undef TPP_EQ_PUT_CASE
    eq_store8<OUT_BF16>(p.out, (int64_t)r + (int64_t)c * p.ldo, first, res);
  }
}

// ---- the kernels' form of a program (host) ---------------------------------------------------
uint32_t eq_word(int32_t op, int32_t arity, int32_t dst, const int32_t (&src)[3]) {
  return (uint32_t)op | (uint32_t)arity << 6 | (uint32_t)dst << 8 | (uint32_t)src[0] << 14 |
         (uint32_t)src[1] << 20 | (uint32_t)src[2] << 26;
}

// The program as it is, every leaf in varg (the kernels for fewer than 8 rows).
void pack_plain(const EqProgram& p, EqArgs& k) {
  for (int32_t i = 0; i < p.n_instr; ++i) {
    const EqInstr& in = p.instr[i];
    int32_t src[3];
    for (int a = 0; a < 3; ++a)
      src[a] = in.src[a] >= EQ_LEAF_BASE ? EQ_V_LEAF + in.src[a] - EQ_LEAF_BASE : in.src[a];
    k.instr[i] = eq_word(in.op, in.arity, in.dst, src);
  }
  k.n_v = p.n_instr;
  k.n_varg = p.n_args;
  for (int32_t j = 0; j < p.n_args; ++j) k.varg[j] = p.arg[j];
}

// Split into the part that is the same for all rows (U: leaves and operations that depend on row
// and scalar leaves only, each in a slot of its own of the column file) and the rest (V: the plan's
// temporaries; leaves in order of first use).
void pack_split(const EqProgram& p, EqArgs& k) {
  int32_t vslot[EQ_MAX_ARGS], uslot[EQ_MAX_ARGS], tmp_u[EQ_MAX_TMPS];
  for (int32_t j = 0; j < EQ_MAX_ARGS; ++j) vslot[j] = uslot[j] = -1;
  for (int32_t j = 0; j < EQ_MAX_TMPS; ++j) tmp_u[j] = -1;   // U slot of the temporary's value
  // U leaves take the first slots, so that their loads can be counted; every leaf that is used
  for (int32_t i = 0; i < p.n_instr; ++i)
    for (int a = 0; a < p.instr[i].arity; ++a) {
      const int32_t j = p.instr[i].src[a] - EQ_LEAF_BASE;
      if (j < 0) continue;
      const EqArg& g = p.arg[j];
      if (g.bcast == TPP_BC_ROW || g.bcast == TPP_BC_SCALAR) {
        if (uslot[j] < 0) {
          uslot[j] = k.n_uarg;
          k.uarg[k.n_uarg++] = g;
        }
      } else if (vslot[j] < 0) {
        vslot[j] = k.n_varg;
        k.varg[k.n_varg++] = g;
      }
    }
  k.uslots = k.n_uarg;
  int32_t n_v = 0;
  uint32_t vword[EQ_MAX_NODES];
  for (int32_t i = 0; i < p.n_instr; ++i) {
    const EqInstr& in = p.instr[i];
    const bool root = i + 1 == p.n_instr;
    int32_t us[3] = {0, 0, 0}, vs[3] = {0, 0, 0};
    bool uniform = !root && k.uslots < EQ_MAX_USLOTS;
    for (int a = 0; a < in.arity; ++a) {
      const int32_t s = in.src[a];
      const int32_t u = s >= EQ_LEAF_BASE ? uslot[s - EQ_LEAF_BASE] : tmp_u[s];
      us[a] = u;
      vs[a] = u >= 0 ? EQ_U_SLOT + u : s >= EQ_LEAF_BASE ? EQ_V_LEAF + vslot[s - EQ_LEAF_BASE] : s;
      uniform = uniform && u >= 0;
    }
    if (uniform) {
      k.instr[k.n_u++] = eq_word(in.op, in.arity, k.uslots, us);
      tmp_u[in.dst] = k.uslots++;
    } else {
      vword[n_v++] = eq_word(in.op, in.arity, in.dst, vs);
      tmp_u[in.dst] = -1;
    }
  }
  for (int32_t i = 0; i < n_v; ++i) k.instr[k.n_u + i] = vword[i];
  k.n_v = n_v;
}

// Whether the split program k (its n_v instructions) is a chain that equation_chain_kernel runs, and
// then its steps; *n_vsteps: how many of them have V leaves.
bool pack_chain(EqArgs& k, int32_t* n_vsteps) {
  const auto is_leaf = [](int32_t c) { return c >= EQ_V_LEAF && c < EQ_U_SLOT; };
  const auto is_u = [](int32_t c) { return c >= EQ_U_SLOT; };
  if (k.uslots + 2 > EQ_MAX_USLOTS) return false;
  const int32_t one = k.uslots, nzero = k.uslots + 1;
  constexpr uint32_t NEG = 0x80000000u;
  EqStep step[EQ_MAX_STEPS], vstep[2];
  EqArg varg[5] = {};
  int32_t n = 0, nv = 0, n_step[3] = {0, 0, 0};
  int32_t act = TPP_EQ_IDENTITY, prev = -1;
  for (int32_t i = 0; i < k.n_v; ++i) {
    const uint32_t w = k.instr[k.n_u + i];
    const int32_t op = (int32_t)(w & 63u), ar = (int32_t)(w >> 6 & 3u);
    int32_t o[3], at = -1;
    for (int a = 0; a < 3; ++a) o[a] = (int32_t)(w >> (14 + 6 * a) & 63u);
    // the running value among the operands: the previous result, or (first) a V leaf, a full one
    // if there is one
    for (int a = 0; a < ar; ++a) {
      if (i > 0) {
        if (o[a] == prev) at = at < 0 ? a : 3;
        else if (!is_leaf(o[a]) && !is_u(o[a])) return false;   // an older temporary
      } else if (is_leaf(o[a])) {
        const bool full = k.varg[o[a] - EQ_V_LEAF].bcast == TPP_BC_NONE;
        if (at < 0 || (full && k.varg[o[at] - EQ_V_LEAF].bcast != TPP_BC_NONE)) at = a;
      }
    }
    if (at < 0 || at > 2) return false;   // not there, or there twice
    if (i == 0) varg[0] = k.varg[o[at] - EQ_V_LEAF];
    prev = (int32_t)(w >> 8 & 63u);
    // X and Y as operand codes; -1: the constant 1 (X) or -0 (Y)
    int32_t X = -1, Y = -1;
    uint32_t xs = 0, ys = 0;
    if (op == TPP_EQ_IDENTITY) continue;
    else if (op == TPP_EQ_NEG) xs = NEG;
    else if (op == TPP_EQ_ADD) Y = o[1 - at];
    else if (op == TPP_EQ_SUB) {
      Y = o[1 - at];
      if (at == 0) ys = NEG;
      else xs = NEG;
    } else if (op == TPP_EQ_MUL) X = o[1 - at];
    else if (op == TPP_EQ_MULADD && at < 2) {
      X = o[1 - at];
      Y = o[2];
    } else if (ar == 1 && i + 1 == k.n_v) {
      act = op;
      break;
    } else return false;
    EqStep st = {X < 0 ? one : is_u(X) ? X - EQ_U_SLOT : 0, Y < 0 ? nzero : is_u(Y) ? Y - EQ_U_SLOT : 0,
                 xs, ys};
    if (is_leaf(X) || is_leaf(Y)) {
      if (nv == 2) return false;
      if (is_leaf(X)) varg[1 + 2 * nv] = k.varg[X - EQ_V_LEAF];
      if (is_leaf(Y)) varg[2 + 2 * nv] = k.varg[Y - EQ_V_LEAF];
      vstep[nv++] = st;
    } else {
      if (n == EQ_MAX_STEPS) return false;
      step[n++] = st;
      ++n_step[nv];
    }
  }
  for (int j = 0; j < 5; ++j) k.varg[j] = varg[j];
  for (int j = 0; j < n; ++j) k.step[j] = step[j];
  for (int j = 0; j < nv; ++j) k.vstep[j] = vstep[j];
  for (int j = 0; j < 3; ++j) k.n_step[j] = n_step[j];
  k.act = act;
  k.uslots += 2;
  *n_vsteps = nv;
  return true;
}

}  // namespace

hipError_t launch_equation(const EqProgram& prog, hipStream_t stream) {
  if (prog.m == 0 || prog.n == 0) return hipSuccess;
  EqArgs k = {};
  k.m = prog.m;
  k.n = prog.n;
  k.ldo = prog.ldo;
  k.out = prog.out;
  EqProgram flat;
  const EqProgram* use = &prog;
  const int64_t total = (int64_t)prog.m * prog.n;
  if (prog.m < 8 && total > EQ_SMALL && total <= 0x7fffffff) {
    // Fewer than 8 contiguous rows (a long row of statistics): the same elements as one column.
    // A row leaf of a single row is then a full one, a column leaf of a single row a scalar.
    bool flattens = prog.ldo == prog.m;
    for (int32_t j = 0; j < prog.n_args; ++j) {
      const EqArg& g = prog.arg[j];
      if (g.bcast == TPP_BC_NONE) flattens = flattens && g.ld == prog.m;
      else if (g.bcast != TPP_BC_SCALAR) flattens = flattens && prog.m == 1;
    }
    if (flattens) {
      flat = prog;
      for (int32_t j = 0; j < prog.n_args; ++j) {
        EqArg& g = flat.arg[j];
        if (g.bcast == TPP_BC_COL) g.bcast = TPP_BC_SCALAR;
        else if (g.bcast == TPP_BC_ROW) g.bcast = TPP_BC_NONE;
        g.ld = total;
      }
      flat.m = k.m = (int32_t)total;
      flat.n = k.n = 1;
      flat.ldo = k.ldo = total;
      use = &flat;
    }
  }
  if (use->m >= 8) {
    const int32_t chunks = (use->m - 1) / EPT + 1;
    EqArgs ch = k;
    int32_t n_vsteps = 0;
    pack_split(*use, ch);
    if (pack_chain(ch, &n_vsteps)) {
      ch.ng = (chunks + 63) / 64;
      ch.w = (chunks + ch.ng - 1) / ch.ng;
      ch.q = 64 / ch.w;
      // Columns per wavefront: enough steps to reuse its column leaves and its column values, while
      // about 16 wavefronts per CU (4096) still share the work; at most the 64 columns of its file.
      const int64_t steps = ch.ng * (((int64_t)use->n + ch.q - 1) / ch.q);
      int64_t per = steps / 4096;
      if (per < 1) per = 1;
      if (per > 64 / ch.q) per = 64 / ch.q;
      ch.cw = (int32_t)per * ch.q;
      ch.tiles = ((int64_t)use->n + ch.cw - 1) / ch.cw;
      const dim3 grid((unsigned)((ch.tiles * ch.ng + EQ_T / 64 - 1) / (EQ_T / 64)));
      const unsigned lds = (unsigned)(ch.uslots * 64 * 4 * (EQ_T / 64));
#define TPP_EQ_CHAIN(B, N) \
  hipLaunchKernelGGL((equation_chain_kernel<B, N>), grid, dim3(EQ_T), lds, stream, ch)
      if (prog.out_bf16) {
        if (n_vsteps == 0) TPP_EQ_CHAIN(true, 0);
        else if (n_vsteps == 1) TPP_EQ_CHAIN(true, 1);
        else TPP_EQ_CHAIN(true, 2);
      } else {
        if (n_vsteps == 0) TPP_EQ_CHAIN(false, 0);
        else if (n_vsteps == 1) TPP_EQ_CHAIN(false, 1);
        else TPP_EQ_CHAIN(false, 2);
      }
#undef TPP_EQ_CHAIN
      return hipGetLastError();
    }
    pack_plain(*use, k);
    int64_t vblocks = ((int64_t)chunks * use->n + EQ_T - 1) / EQ_T;
    if (vblocks > 8 * 256) vblocks = 8 * 256;   // at most 8 per CU, grid stride beyond
    int32_t ntmp = 0;
    for (int32_t i = 0; i < use->n_instr; ++i)
      if (use->instr[i].dst + 1 > ntmp) ntmp = use->instr[i].dst + 1;
    const dim3 vgrid((unsigned)vblocks);
#define TPP_EQ_VEC(B, N) hipLaunchKernelGGL((equation_vec_kernel<B, N>), vgrid, dim3(EQ_T), 0, stream, k)
    if (prog.out_bf16) {
      if (ntmp <= 2) TPP_EQ_VEC(true, 2);
      else if (ntmp <= 4) TPP_EQ_VEC(true, 4);
      else TPP_EQ_VEC(true, EQ_MAX_TMPS);
    } else {
      if (ntmp <= 2) TPP_EQ_VEC(false, 2);
      else if (ntmp <= 4) TPP_EQ_VEC(false, 4);
      else TPP_EQ_VEC(false, EQ_MAX_TMPS);
    }
#undef TPP_EQ_VEC
    return hipGetLastError();
  }
  pack_plain(prog, k);
  if (total <= EQ_SMALL) {
    const dim3 sgrid((unsigned)((total + EQ_T - 1) / EQ_T));
    const unsigned lds = (unsigned)((EQ_V_LEAF + k.n_varg) * EQ_T * 4);
    if (prog.out_bf16)
      hipLaunchKernelGGL((equation_small_kernel<true>), sgrid, dim3(EQ_T), lds, stream, k);
    else
      hipLaunchKernelGGL((equation_small_kernel<false>), sgrid, dim3(EQ_T), lds, stream, k);
    return hipGetLastError();
  }
  // enough workgroups for every element once, at most 8 per CU on the 256 CUs (grid stride
  // beyond)
  int64_t blocks = (total + EPT * EQ_T - 1) / (EPT * EQ_T);
  if (blocks > 8 * 256) blocks = 8 * 256;
  const dim3 grid((unsigned)blocks);
  const bool wide = total > 0xffffffffLL;
  if (prog.out_bf16) {
    if (wide) hipLaunchKernelGGL((equation_kernel<true, true>), grid, dim3(EQ_T), 0, stream, k);
    else hipLaunchKernelGGL((equation_kernel<true, false>), grid, dim3(EQ_T), 0, stream, k);
  } else {
    if (wide) hipLaunchKernelGGL((equation_kernel<false, true>), grid, dim3(EQ_T), 0, stream, k);
    else hipLaunchKernelGGL((equation_kernel<false, false>), grid, dim3(EQ_T), 0, stream, k);
  }
  return hipGetLastError();
}

}  // namespace tpp
