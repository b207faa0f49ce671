// Launcher prototypes of the HIP kernels (gfx950).  Every launcher enqueues on
// `st` and returns immediately; none allocates.
//
// Row model: a forward pass runs over "rows"; row r belongs to sequence slot
// row_slot[r] and sits at position row_pos[r].  For a decode iteration the rows are
// the live rollouts (written by the scheduler kernel), for prefill they are all
// prompt tokens of the admitted rollouts.  The row count lives in device memory next to
// the stop flag; kernels whose block index is beyond it exit, and a raised stop flag
// turns every kernel into a no-op once the scheduler has ended the step.
#pragma once
#include "common.h"

namespace april {

struct RowCtx {
  const int* row_slot;
  const int* row_pos;
  const int2* ctl;       // device: x = number of rows, y = stop flag (one 8-byte scalar load)
  int max_rows;          // host-known upper bound (grid size)
};

// Rows to process: 0 once the scheduler has ended the step.
__device__ inline int rows_or_zero(const RowCtx& rc) {
  const int2 v = *rc.ctl;
  return v.y ? 0 : v.x;
}
// Early exit of a one-workgroup-per-row kernel: step stopped, or row beyond the batch.
#define ROW_GUARD(rc, r) \
  if ((r) >= rows_or_zero(rc)) return;

// Rotary embedding of the pair (a, b) = (x[i], x[i + d/2]) with cos c and sin s, in one
// fixed operation order (no compiler-chosen contraction), so that every kernel that rotates
// produces the same bits.
__device__ inline float rope_first(float a, float b, float c, float s) { return __fmaf_rn(a, c, -__fmul_rn(b, s)); }
__device__ inline float rope_second(float a, float b, float c, float s) { return __fmaf_rn(b, c, __fmul_rn(a, s)); }

// ---------------------------------------------------------------------------
// Reductions inside a wavefront on the DPP lanes of the vector unit: rotations by 8, 4, 2, 1 inside the rows of 16 lanes,
// then the rows by scalar reads.  (A shuffle through the LDS unit is a round trip of 100 cycles and more, with 16
// wavefronts asking at once; six of them were most of a block-wide step.)
template <int N> __device__ inline int row_ror(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xf, 0xf, false); }
template <int N> __device__ inline double row_ror_f64(double v) {
  union { double d; int i[2]; } x{v};
  x.i[0] = row_ror<N>(x.i[0]);
  x.i[1] = row_ror<N>(x.i[1]);
  return x.d;
}
__device__ inline float as_f32(int v) { return __int_as_float(v); }
// every lane: over its row of 16 lanes
__device__ inline float row_max_f32(float v) {
  v = fmaxf(v, as_f32(row_ror<8>(__float_as_int(v))));
  v = fmaxf(v, as_f32(row_ror<4>(__float_as_int(v))));
  v = fmaxf(v, as_f32(row_ror<2>(__float_as_int(v))));
  return fmaxf(v, as_f32(row_ror<1>(__float_as_int(v))));
}
__device__ inline unsigned row_max_u32(unsigned v) {
  v = max(v, (unsigned)row_ror<8>((int)v));
  v = max(v, (unsigned)row_ror<4>((int)v));
  v = max(v, (unsigned)row_ror<2>((int)v));
  return max(v, (unsigned)row_ror<1>((int)v));
}
__device__ inline int row_min_i32(int v) {
  v = min(v, row_ror<8>(v));
  v = min(v, row_ror<4>(v));
  v = min(v, row_ror<2>(v));
  return min(v, row_ror<1>(v));
}
__device__ inline double row_sum_f64(double v) {
  v += row_ror_f64<8>(v);
  v += row_ror_f64<4>(v);
  v += row_ror_f64<2>(v);
  return v + row_ror_f64<1>(v);
}
__device__ inline double lane_f64(double v, int l) {
  union { double d; int i[2]; } x{v};
  x.i[0] = __builtin_amdgcn_readlane(x.i[0], l);
  x.i[1] = __builtin_amdgcn_readlane(x.i[1], l);
  return x.d;
}
// every lane: over the wavefront
__device__ inline float wave_max_f32(float v) {
  const int r = __float_as_int(row_max_f32(v));
  return fmaxf(fmaxf(as_f32(__builtin_amdgcn_readlane(r, 0)), as_f32(__builtin_amdgcn_readlane(r, 16))),
               fmaxf(as_f32(__builtin_amdgcn_readlane(r, 32)), as_f32(__builtin_amdgcn_readlane(r, 48))));
}
__device__ inline unsigned wave_max_u32(unsigned v) {
  const int r = (int)row_max_u32(v);
  return max(max((unsigned)__builtin_amdgcn_readlane(r, 0), (unsigned)__builtin_amdgcn_readlane(r, 16)),
             max((unsigned)__builtin_amdgcn_readlane(r, 32), (unsigned)__builtin_amdgcn_readlane(r, 48)));
}
__device__ inline int wave_min_i32(int v) {
  const int r = row_min_i32(v);
  return min(min(__builtin_amdgcn_readlane(r, 0), __builtin_amdgcn_readlane(r, 16)),
             min(__builtin_amdgcn_readlane(r, 32), __builtin_amdgcn_readlane(r, 48)));
}
__device__ inline double wave_sum_f64(double v) {
  v = row_sum_f64(v);
  return (lane_f64(v, 0) + lane_f64(v, 16)) + (lane_f64(v, 32) + lane_f64(v, 48));
}
__device__ inline float wave_sum_f32(float v) {
  v += as_f32(row_ror<8>(__float_as_int(v)));
  v += as_f32(row_ror<4>(__float_as_int(v)));
  v += as_f32(row_ror<2>(__float_as_int(v)));
  const int r = __float_as_int(v + as_f32(row_ror<1>(__float_as_int(v))));
  return (as_f32(__builtin_amdgcn_readlane(r, 0)) + as_f32(__builtin_amdgcn_readlane(r, 16))) +
         (as_f32(__builtin_amdgcn_readlane(r, 32)) + as_f32(__builtin_amdgcn_readlane(r, 48)));
}

// silu(g) * u with the hardware reciprocal (1 ulp) instead of a full-precision division: the
// result is rounded to bf16 right after, and the division was most of the SwiGLU epilogue.
__device__ inline float silu_mul(float g, float u) { return g * u * __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }

// Record of one row's 64-column group of logits, from the two 32-column accumulator tiles of an LM
// head wavefront (a, b; `two` = false: the vocabulary ends after the first): the maximum, the lowest
// column that holds it, and - when `want_sum` - the sum of exp((l - maximum) * inv_t) over the group,
// exponentials in fp32, added in fp64 in one fixed order.  nhalf: 4 * (lane / 32).  Both halves of a
// lane pair return the group's values.  Shared by every LM head kernel, so all leave the same bits.
__device__ __forceinline__ void group64_record(const f32x16& a, const f32x16& b, bool two, int nhalf, bool want_sum,
                                               float inv_t, float& max_out, int& col_out, double& sum_out) {
  float bv = -INFINITY;
  int bn = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e)                   // increasing column: a strict comparison keeps the first maximum
      if (a[4 * q + e] > bv) { bv = a[4 * q + e]; bn = 8 * q + nhalf + e; }
  if (two) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (b[4 * q + e] > bv) { bv = b[4 * q + e]; bn = 32 + 8 * q + nhalf + e; }
  }
  const float ov = __shfl_xor(bv, 32, 64);
  const int on = __shfl_xor(bn, 32, 64);
  if (ov > bv || (ov == bv && on < bn)) { bv = ov; bn = on; }
  max_out = bv;
  col_out = bn;
  if (want_sum) {
    const float ref = bv == -INFINITY ? 0.f : bv;          // a group of -inf sums to zero, not to NaN
    double s = 0.0;
#pragma unroll
    for (int e = 0; e < 16; ++e) s += (double)__expf((a[e] - ref) * inv_t);
    if (two) {
#pragma unroll
      for (int e = 0; e < 16; ++e) s += (double)__expf((b[e] - ref) * inv_t);
    }
    sum_out = s + __shfl_xor(s, 32, 64);
  }
}

// --- sampling: what its kernels and the one-launch fp32 pass share --------------
// Order-preserving map float -> unsigned (larger float <=> larger key); -0 == +0.
__device__ inline unsigned f2key(float f) {
  unsigned u = __float_as_uint(f);
  if (u == 0x80000000u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// What a sampling row works on, requested at the kernel's start: nothing behind the choice waits for memory again.
struct RowState {
  int slot, pos, g, limit, state, forced, group, eos, iter;
  long long req;
};
__device__ inline RowState load_row(const RowCtx& rc, const Slots& s, const Ctrl* ctrl, int r, int update,
                                    const long long* req_ids, const int* gen_idx) {
  RowState q{-1, 0, 0, 0, 0, -1, -1, -1, 0, 0};
  if (update) {
    q.slot = rc.row_slot[r];
    q.pos = rc.row_pos[r];
    q.eos = ctrl->eos_token;
    q.iter = ctrl->iter;
    q.g = s.gen[q.slot];
    q.req = s.req_id[q.slot];
    q.limit = s.limit[q.slot];
    q.state = s.state[q.slot];
    if (s.group != nullptr) q.group = s.group[q.slot];
    if (s.forced != nullptr) q.forced = s.forced[(size_t)q.slot * s.max_ctx + q.g];
  } else {
    // (these may lie in host memory: 2.5 us away, and a scalar load would have every wait for a scalar load wait for it)
    int at = r;
    asm volatile("" : "+v"(at));
    q.req = req_ids[at];
    q.g = gen_idx[at];
  }
  return q;
}
// Token to the caller, or appended to its rollout (one thread).
__device__ inline void finish_row(const Slots& s, Ctrl* ctrl, const RowState& q, int r, int update, int sampled, int tok, int* out_tokens) {
  if (!update) { out_tokens[r] = sampled; return; }
  s.tokens[(size_t)q.slot * s.max_ctx + q.pos + 1] = tok;
  s.gen[q.slot] = q.g + 1;
  s.kv_len[q.slot] = q.pos + 1;
  int stt = q.state;
  if (stt == SLOT_PREFILL) stt = SLOT_LIVE;
  if (q.g + 1 >= q.limit || tok == q.eos) {
    stt = SLOT_DONE;
    s.finish_iter[q.slot] = q.iter;
    // what the scheduler counts toward N: the rollout, or (instance-level completion,
    // Section 3.2.3) its group once the last member is complete
    if (q.group < 0) atomicAdd(&ctrl->finished, 1);
    else if (atomicSub(&s.grp_left[q.group], 1) == 1) atomicAdd(&ctrl->finished, 1);
  }
  s.state[q.slot] = stt;
}

// --- scheduler / allocator -------------------------------------------------
// check_only = 1: only the "N complete => stop" test (end of a chunk of iterations).
// row_cap / ctx_cap: the bounds the host sized this iteration's launches for (live rows, longest
// context); exceeding one sets error bit 2 in the control block and stops the step.
// att_items (or null): work list for the decode attention, written when rows are rebuilt: entry 0
// = {count, 0, 0, 0}, entry 1 + i = {row, KV split, slot, position}, one per (row, split of
// att_split tokens the row's context reaches), full splits first, then the rows' last splits by
// descending length (classes of att_split / 32 tokens; the order inside a class is arbitrary).
// att_cap = entries the list holds beyond the first; more items than that raise error bit 2.
void launch_sched(hipStream_t st, Ctrl* ctrl, Slots s, int* row_slot, int* row_pos,
                  int* free_stack, int blk, int check_only, int row_cap, int ctx_cap,
                  int4* att_items = nullptr, int att_split = 0, int att_cap = 0);
void launch_alloc_prefill(hipStream_t st, Ctrl* ctrl, Slots s, const int* slot_list,
                          const int* n_blocks_needed, int n, int* free_stack);
void launch_free_slots(hipStream_t st, Ctrl* ctrl, Slots s, const int* slot_list, int n,
                       int* free_stack);
void launch_init_free_stack(hipStream_t st, int* free_stack, int n_blocks);
void launch_fill_i32(hipStream_t st, int* p, int v, size_t n);

// Copies between device arrays and one pinned host buffer, many pieces in one launch (the kernel reads /
// writes the host memory itself): item = `n` ints at `dev` <-> buf + off.  `items` and `buf` are pinned.
struct XferItem { int* dev; int off, n; };
void launch_xfer(hipStream_t st, const XferItem* items, int n_items, int* buf, bool to_device);

// Group records an LM head leaves: arrays [rows][ceil(V / lmhead_group_cols())].
struct GroupOut {
  float* max;        // maximum of the group
  int* col;          // column inside the group that holds it, the lowest on ties (nullable)
  double* sum;       // sum of exp((l - maximum) * inv_t) (nullable: not wanted)
  float inv_t;
};

// --- model ------------------------------------------------------------------
// x_res = embedding of each row's token; h = rmsnorm(x_res) * gain (the first layer's norm).
template <typename T, bool XF>
void launch_embed_norm(hipStream_t st, RowCtx rc, Slots s, const T* emb, float* x_res, const float* gain, T* h, int d, float eps);

// x_res += sum of partials (if any); h = rmsnorm(x_res) * gain.  gather (nullable):
// input row index of output row r.
// pos_of / wts (nullable, mixture-of-experts combine): partial p of row r is then the row
// pos_of[r * n_partials + p] of `partials` ([packed rows][d]) weighted by wts[r * n_partials + p].
template <typename T, bool XF>
void launch_add_rmsnorm(hipStream_t st, RowCtx rc, float* x_res, const float* partials,
                        int n_partials, size_t partial_stride, const float* gain, T* h,
                        int d, float eps, const int* gather, const int* pos_of = nullptr,
                        const float* wts = nullptr, T* h_rows = nullptr, float* x_copy = nullptr);

// --- routed experts (bf16) ---------------------------------------------------------
void launch_moe_route(hipStream_t st, RowCtx rc, const float* logits, int n_partials, size_t partial_stride,
                      int E, int top_k, int* ids, float* wts);
void launch_moe_dispatch(hipStream_t st, RowCtx rc, const int* ids, int E, int top_k, int* cnt, int* base,
                         int* pos_of, int* src_row, int p_cap, Ctrl* ctrl, int tall_rows, int* group_expert);
// upper bound on the row groups (of `align` rows) of a launch over at most max_rows rows
int moe_group_count(int max_rows, int top_k, int E, int align);
// tall_rows: row bound from which a GEMM workgroup takes 4 m-tiles of an expert instead of 2
// (the dispatch aligns the expert segments accordingly: pass the same value to all three)
// LDS-tiled expert GEMMs for prefill passes (kernels_gemm_tile.hip): row groups of moe_tile_rows()
// packed rows (the dispatch must have aligned the expert segments to that), one accumulator chain
// per output element.  Return false (nothing launched) for shapes they do not take.
int moe_tile_rows();
// (gate/up, here and below: h_rows is the plain [row][d] copy of the normalised activations that
// launch_add_rmsnorm writes on request; its rows are gathered through src_row)
bool launch_moe_tile_gateup(hipStream_t st, RowCtx rc, const int* cnt, const int* base, const int* group_expert,
                            const int* src_row, const bf16_t* h_rows, const bf16_t* Wg, const bf16_t* Wu, bf16_t* act,
                            int Fe, int d, int n_groups);
bool launch_moe_tile_down(hipStream_t st, RowCtx rc, const int* cnt, const int* base, const int* group_expert,
                          const bf16_t* act, const bf16_t* Wd, float* out, int Fe, int d, int n_groups);
void launch_moe_gateup(hipStream_t st, RowCtx rc, const int* cnt, const int* base, const int* group_expert,
                       const int* src_row, const bf16_t* h_rows, const bf16_t* Wg, const bf16_t* Wu, bf16_t* act, int E,
                       int top_k, int Fe, int d, int tall_rows);
void launch_moe_down(hipStream_t st, RowCtx rc, const int* cnt, const int* base, const int* group_expert,
                     const bf16_t* act, const bf16_t* Wd, float* out, int E, int top_k, int Fe, int d, int tall_rows);

// q_bf16 (nullable): the rotated queries go there, rounded to bf16, instead of q_rot.
template <typename T>
void launch_rope_append(hipStream_t st, RowCtx rc, Slots s, const float* qkv, int n_partials,
                        size_t partial_stride, const float* rope_cos, const float* rope_sin,
                        float* q_rot, T* kv_pool, KVLayout kvl, int layer, int n_q_heads, bf16_t* q_bf16 = nullptr);

template <typename T, bool XF>
void launch_attn_ref(hipStream_t st, RowCtx rc, Slots s, const float* q_rot, const T* kv_pool,
                     KVLayout kvl, int layer, int n_q_heads, T* out);

// bf16 MFMA paged attention (KV layout mode 1).  Rows [row_base, row_base + rc.max_rows)
// of the row arrays.  A context longer than attn_split_tokens() is cut in KV splits of
// that fixed size, so a row's reduction order depends on its own length only; ws /
// counters: split workspace for rc.max_rows rows (counters zero on entry and on exit);
// max_splits <= 32.
int attn_split_tokens(int head_dim);
// fused_qkv != nullptr (decode iterations): the kernel also rotates q / the new key and
// appends the new key / value itself from the QKV GEMM's split-K partials (q_rot unused).
// items != nullptr (row_base 0, rows listed by launch_sched in this iteration): a 1-D launch of
// rc.max_rows * grid_splits * KV heads workgroups that takes its (row, split) from the work list.
void launch_attn_decode(hipStream_t st, RowCtx rc, int row_base, Slots s, const float* q_rot,
                        bf16_t* kv_pool, KVLayout kvl, int layer, int n_q_heads, bf16_t* out,
                        float* ws, int max_splits, int grid_splits,
                        const float* fused_qkv, int n_partials, size_t partial_stride,
                        const float* rope_cos, const float* rope_sin, const int4* items = nullptr);
// Causal attention over prefill rows, one workgroup per (item, KV head); an item = {slot, first
// row of the sequence in the row arrays, tokens of the sequence, first position of the tile},
// tiles of attn_prefill_tile(query heads per KV head) positions.  q (bf16 rows) and the pages must hold
// the rotated queries / keys and the values of every row (launch_gemm_tile_qkv or launch_rope_append first).
int attn_prefill_tile(int group);
void launch_attn_prefill(hipStream_t st, const int4* items, int n_items, Slots s, const bf16_t* q,
                         const bf16_t* kv_pool, KVLayout kvl, int layer, int n_q_heads, bf16_t* out);
// Merge of the KV-split partials (needed after launch_attn_decode whenever grid_splits > 1).
void launch_attn_merge(hipStream_t st, RowCtx rc, int row_base, KVLayout kvl, int n_q_heads, bf16_t* out,
                       const float* ws, int max_splits);

template <typename T, bool XF>
void launch_silu_mul(hipStream_t st, RowCtx rc, const float* gu, int F, T* act);

// fp32 path: attention over the plain KV layout (mode 0), GEMM over row-major operands.
void launch_attn_f32(hipStream_t st, RowCtx rc, Slots s, const float* q_rot, const float* kv_pool, KVLayout kvl,
                     int layer, int n_q_heads, float* out);
void launch_gemm_f32(hipStream_t st, RowCtx rc, const float* x, const float* W, float* out, int N, int K);
// fp32 models of few weights: a decode pass from the tokens to the logits in one launch, a workgroup per row (K and V of
// the new position appended), and the product that their other passes use (its sums are that pass's; K % 4 == 0).
// Which models: by their dimensions alone, so that neither a context's capacity nor the rows of a pass change a bit of a
// rollout.  Which decode passes take the one launch: by bounds on their rows and contexts (the same bits either way).
struct F32Layer { const float *attn_norm, *mlp_norm, *wqkv, *wo, *wgu, *wd; };
struct F32Model {
  const F32Layer* layers;              // device array
  const float *tok_emb, *final_norm, *lm_head, *rope_cos, *rope_sin;
  float* kv_pool;
  KVLayout kvl;
  int n_layers, d, F, n_q_heads, vocab;
  float eps;
  int lds_floats;                      // (the launcher's)
};
bool forward_f32_takes(int d, int F, int nq, int nqkv, int vocab);
bool forward_f32_pays(int rows, int ctx, int nq);
int forward_f32_ctx(int nq, bool many_rows);      // the longest contexts that it takes
// greedy: the token of every row too, as launch_sample appends it (no logits watched); ctrl is read and counted in then
void launch_forward_f32(hipStream_t st, RowCtx rc, Slots s, F32Model m, float* logits, Ctrl* ctrl, bool greedy, float temperature);
void launch_gemm_f32_dot(hipStream_t st, RowCtx rc, const float* x, const float* W, float* out, int N, int K);

// out[m][n] = sum_k x[m][k] W[n][k]; plain row-major W; reference path.
template <typename T, bool XF>
void launch_gemm_ref(hipStream_t st, RowCtx rc, const T* x, const T* W, float* out, int N, int K);

// bf16 MFMA GEMM over fragment-tiled operands.  Wp: weights re-laid by
// launch_shuffle_weights.  out: fp32 [ksplit][m_cap][N] partial sums.
void launch_gemm_mfma(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, float* out,
                      int N, int K, int ksplit, size_t partial_stride,
                      const float* ssq = nullptr, int ssq_stride = 0, float eps = 0.f);
// act[m][f] = silu(x.Wg[f]) * (x.Wu[f]) as fragment-tiled bf16.
// ssq != nullptr: the activations are residual * gain (not yet normalised); the kernel divides
// its accumulators by the row's RMS, from the sums of squares the producer left (see
// launch_gemm_mfma_resid).
void launch_gemm_mfma_swiglu(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wg,
                             const bf16_t* Wu, bf16_t* act, int F, int K, const float* ssq = nullptr,
                             int ssq_stride = 0, float eps = 0.f);
void launch_gemm_mfma_resid(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, float* x_res,
                            const float* gain, bf16_t* act, float* ssq, int ssq_stride, int N, int K);
// LDS-tiled GEMMs for tall activations (prefill); single pass over k, no partials.  _resid: added into
// the fp32 residual stream x_res [rows][N].  _qkv: rotary embedding and KV append in the epilogue,
// rotated queries as bf16 rows (false, nothing launched: shapes it does not take).
struct QkvOut {
  const int* block_table;
  int max_blocks;
  const float *rope_cos, *rope_sin;    // [pos][head_dim / 2]
  bf16_t* q;                           // [rows][n_q_heads * head_dim]
  bf16_t* kv_pool;
  KVLayout kvl;
  int layer, n_q_heads;
};
void launch_gemm_tile_resid(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, float* x_res, int N, int K);
bool launch_gemm_tile_qkv(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, int N, int K, const QkvOut& qo);
void launch_gemm_tile(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, float* out, int N, int K);
void launch_gemm_tile_swiglu(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wg, const bf16_t* Wu,
                             bf16_t* act, int F, int K);
bool launch_gemm_tile_swiglu_chain(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wg, const bf16_t* Wu,
                                   bf16_t* act, int F, int K, const float* ssq, int ssq_stride, float eps);
bool launch_gemm_tile_logits(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, float* logits,
                             const GroupOut& go, int V, int K);
// LM head: logits fp32 [rows][V] plus, per row, records of every group of lmhead_group_cols()
// consecutive logits (the last group of a vocabulary that is not a multiple of it is short).
// logits may be null: nothing but the group records is written then (all the greedy sampler
// needs, with or without log-probabilities).
int lmhead_group_cols();
void launch_gemm_mfma_logits(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, float* logits,
                             const GroupOut& go, int V, int K);
void launch_shuffle_weights(hipStream_t st, const bf16_t* src, bf16_t* dst, int N, int K);

void launch_rope_table(hipStream_t st, float* cos_t, float* sin_t, int max_pos, int head_dim,
                       float theta);

// --- sampler + per-rollout state update ---------------------------------------
// Top-k search of a vocabulary with a short last group: in the groups whose maximum reaches the k-th largest one, or over the
// whole row.  Up to 4096 logits the whole row is read once and kept in registers, and with few more than k groups most
// of them are hot and their candidates many.  us per call for 5, 1000 rows, whole row | groups: 20 of 2001 25, 48 | 27, 50, of 4095 26, 54 |
// 28, 50, of 6001 28, 63 | 28, 52; 50 of 4095 26, 55 | 28, 53, of 6001 (94 groups) 28, 64 | 29, 55, of 8001 32, 77 | 29, 56; 64 of 4095
// 26, 55 | 31, 70, of 6001 28, 65 | 29, 57, of 8001 (126) 32, 78 | 29, 58: from about 1.5 k groups on they win, 2 k is the line of earlier kernels.
inline bool topk_in_groups(int V, int k) { return V % 64 == 0 || (V > 4096 && (V + 63) / 64 >= 2 * k); }
struct SamplerCfg {
  int kind, top_k;            // kind: 0 greedy, 1 top-k (+ nucleus), 2 categorical over the whole vocabulary
  float temperature;
  unsigned long long seed;
  float top_p;                // nucleus cut of the top-k candidates; >= 1: none
};
// Whether a row's token comes from group records (else from the whole row): always, but for a top k with fewer than k groups or a
// short row.  Who makes the records asks first: nothing reads them otherwise, not even for the log-probability (whole-row
// searches have the row at hand, at most 8191 logits.  Calls with log-probabilities, records made and left unread / not made: top 50 of
// 4095, 192 and 1000 rows 33.8, 69.7 / 30.2, 64.1 us; top 64 of 8001 41.0, 101 / 37.0, 92).
inline bool sampler_takes_records(const SamplerCfg& sc, int V) {
  return sc.kind != 1 || sc.top_k <= 1 || ((V + 63) / 64 >= sc.top_k && topk_in_groups(V, sc.top_k));
}
// Rows here are sampling rows: sample_row_slot / sample_row_pos give the slot and the
// position of the LAST fed token of each row.  update = 0: only write out_tokens
// (standalone sampler; req_ids/gen_idx arrays given explicitly).
// group_max (nullable): per row the maxima of groups of 64 consecutive logits, as written by
// launch_gemm_mfma_logits and launch_group_records; lets the sampler look at a few groups only.
// group_sum (nullable, with group_max): the groups' sums of exp((l - maximum) / T), which the
// categorical sampler (fp64 exponentials: launch_group_records) and the log-probabilities need;
// without it they read the whole row.
// out_logprobs (nullable, update = 0): log softmax(logits / temperature)[token]; with update = 1
// the log-probability goes to s.logprob when that array exists.
void launch_sample(hipStream_t st, RowCtx rc, Slots s, Ctrl* ctrl, const float* logits, int vocab,
                   SamplerCfg sc, Watch w, int update, const long long* req_ids,
                   const int* gen_idx, int* out_tokens, const float* group_max,
                   float* out_logprobs = nullptr, const int* group_idx = nullptr,
                   const double* group_sum = nullptr);

// Group records (groups of 64, the last one short if 64 does not divide V) of logits that are in
// memory: maxima, and with `sums` 1 / 2 the sums of exp((l - maximum) / T) with fp32 / fp64
// exponentials.  ctl (nullable): device {rows, stop}; n_rows bounds the launch.
void launch_group_records(hipStream_t st, const float* logits, const int2* ctl, int n_rows, int V, int sums,
                          float temperature, float* group_max, double* group_sum);

}  // namespace april
