// Scheduler, allocator, embedding, RMSNorm, rotary + KV append, reference attention,
// reference GEMM, SiLU*mul.  gfx950, wave64.
#include <type_traits>

#include "kernels.h"

namespace april {

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------
__device__ inline float wave_sum(float v) { return wave_sum_f32(v); }
__device__ inline int wave_incl_scan(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    int t = __shfl_up(v, off, 64);
    if (lane >= off) v += t;
  }
  return v;
}
template <typename T> __device__ inline float to_f32(T v) { return (float)v; }
template <typename T> __device__ inline T from_f32(float v) { return (T)v; }

// ---------------------------------------------------------------------------
// Scheduler: early termination, live-batch compaction, KV page allocation.
// One workgroup.  Runs at the start of every decode iteration:
//   - if the step already stopped: nothing;
//   - if finished >= N: raise stop, remember the iteration count (early termination,
//     Section 2.2, second item of the method);
//   - else rebuild the dense list of live rollouts (slot order) and give a fresh
//     KV page to every live rollout whose next position opens a new page.  If the
//     free pages do not cover that demand, the youngest live rollout (largest request
//     id) is preempted first, repeatedly: its pages return to the stack, it keeps its
//     tokens, stops for this step and is re-prefilled when resumed;
//   - if nothing is live and nothing waits for prefill, the step ends (fewer than N).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void sched_kernel(Ctrl* c, Slots s, int* row_slot, int* row_pos,
                                                     int* free_stack, int blk, int check_only, int row_cap,
                                                     int ctx_cap, int4* att_items, int att_split, int att_cap) {
  __shared__ int sh_a[16], sh_b[16], sh_err[16];
  __shared__ long long sh_ctx[16];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int stop = c->stop, finished = c->finished, n_target = c->n_target;
  const int n_slots = c->n_slots, iter = c->iter, inflight = c->inflight;
  int free_top = c->free_top;
  __shared__ int sh_need, sh_free, sh_pending;
  if (tid == 0) { sh_need = 0; sh_pending = 0; }
  __syncthreads();
  if (stop) return;
  if (finished >= n_target) {
    if (tid == 0) { c->stop = 1; c->stop_iter = iter; c->n_rows = 0; }
    return;
  }
  if (check_only) return;
  if (free_top < inflight) {
    // the pool may be short: count this iteration's page demand, preempt if it is
    int cnt = 0;
    for (int slot = tid; slot < n_slots; slot += 1024)
      if (s.state[slot] == SLOT_LIVE) {
        const int pos = s.kv_len[slot];
        cnt += (pos % blk == 0) && (pos / blk >= s.n_blocks[slot]);
      }
    if (cnt) atomicAdd(&sh_need, cnt);
    __syncthreads();
    if (tid == 0) {
      int need = sh_need, ft = free_top;
      while (need > ft) {
        int victim = -1;
        long long best = -1;
        for (int slot = 0; slot < n_slots; ++slot)
          if (s.state[slot] == SLOT_LIVE && s.req_id[slot] > best) { best = s.req_id[slot]; victim = slot; }
        if (victim < 0) break;
        const int pos = s.kv_len[victim], nb = s.n_blocks[victim];
        if ((pos % blk == 0) && (pos / blk >= nb)) --need;
        for (int j = 0; j < nb; ++j) free_stack[ft++] = s.block_table[(size_t)victim * s.max_blocks + j];
        s.n_blocks[victim] = 0;
        s.kv_len[victim] = 0;
        s.state[victim] = SLOT_PREEMPTED;
        s.finish_iter[victim] = c->n_preempted;      // order of preemption within the step
        c->n_preempted += 1;
      }
      sh_free = ft;
    }
    __syncthreads();
    free_top = sh_free;
  }
  int base_live = 0, base_need = 0, err = 0;
  long long ctx_sum = 0;
  for (int s0 = 0; s0 < n_slots; s0 += 1024) {
    const int slot = s0 + tid;
    int live = 0, need = 0, pos = 0;
    if (slot < n_slots) {
      const int stt = s.state[slot];
      if (stt == SLOT_LIVE) {
        live = 1;
        pos = s.kv_len[slot];
        need = (pos % blk == 0) && (pos / blk >= s.n_blocks[slot]);
      } else if (stt == SLOT_PREFILL) {
        sh_pending = 1;
      }
    }
    const int ia = wave_incl_scan(live), ib = wave_incl_scan(need);
    if (lane == 63) { sh_a[wid] = ia; sh_b[wid] = ib; }
    __syncthreads();
    int wa = 0, wb = 0, ta = 0, tb = 0;
    for (int w = 0; w < 16; ++w) {
      const int va = sh_a[w], vb = sh_b[w];
      if (w < wid) { wa += va; wb += vb; }
      ta += va; tb += vb;
    }
    __syncthreads();
    if (live) {
      const int r = base_live + wa + ia - 1;
      row_slot[r] = slot;
      row_pos[r] = pos;
      ctx_sum += pos + 1;
      if (pos + 1 > ctx_cap) err |= 2;       // the host sized this iteration's launches for shorter contexts
    }
    if (need) {
      const int idx = free_top - 1 - (base_need + wb + ib - 1);
      const int bi = pos / blk;
      if (idx < 0 || bi >= s.max_blocks) {
        err |= 1;
      } else {
        s.block_table[(size_t)slot * s.max_blocks + bi] = free_stack[idx];
        s.n_blocks[slot] = bi + 1;
      }
    }
    base_live += ta;
    base_need += tb;
  }
  // Work list of the decode attention: one item per (row, KV split), longest first.  Class 0 =
  // full splits, class 1 + j = last splits that are j 32nds of a split short of full; a
  // counting sort over the classes (shared-memory counters; the order inside a class does not
  // matter, every item's result is independent of where it runs).
  if (att_items != nullptr) {
    __shared__ int sh_hist[33], sh_cur[33];
    if (tid < 33) sh_hist[tid] = 0;
    __syncthreads();                                   // also: this workgroup's row_slot / row_pos stores are visible
    for (int r = tid; r < base_live; r += 1024) {
      const int ctx = row_pos[r] + 1;
      const int ns = (ctx + att_split - 1) / att_split, last = ctx - (ns - 1) * att_split;
      const int cl = 1 + (int)(((long long)(att_split - last) * 32) / att_split);
      if (ns > 1) atomicAdd(&sh_hist[0], ns - 1);
      atomicAdd(&sh_hist[cl], 1);
    }
    __syncthreads();
    if (tid == 0) {
      int acc = 0;
      for (int i = 0; i < 33; ++i) { sh_cur[i] = acc; acc += sh_hist[i]; }
      if (acc > att_cap) { acc = 0; err |= 2; }
      sh_hist[0] = acc;
      att_items[0] = make_int4(acc, 0, 0, 0);
    }
    __syncthreads();
    if (sh_hist[0] > 0) {
      for (int r = tid; r < base_live; r += 1024) {
        const int pos = row_pos[r], slot = row_slot[r], ctx = pos + 1;
        const int ns = (ctx + att_split - 1) / att_split, last = ctx - (ns - 1) * att_split;
        const int cl = 1 + (int)(((long long)(att_split - last) * 32) / att_split);
        if (ns > 1) {
          const int p0 = atomicAdd(&sh_cur[0], ns - 1);
          for (int j = 0; j < ns - 1; ++j) att_items[1 + p0 + j] = make_int4(r, j, slot, pos);
        }
        att_items[1 + atomicAdd(&sh_cur[cl], 1)] = make_int4(r, ns - 1, slot, pos);
      }
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    ctx_sum += __shfl_xor(ctx_sum, off, 64);
    err |= __shfl_xor(err, off, 64);
  }
  if (lane == 0) { sh_ctx[wid] = ctx_sum; sh_err[wid] = err; }
  __syncthreads();
  if (tid == 0) {
    long long tot = 0; int e = 0;
    for (int w = 0; w < 16; ++w) { tot += sh_ctx[w]; e |= sh_err[w]; }
    c->n_rows = base_live;
    c->free_top = free_top - base_need < 0 ? 0 : free_top - base_need;
    if (base_live == 0 && !sh_pending) {
      c->stop = 1;                 // nothing left in flight: the step ends short of N
      c->stop_iter = iter;
    } else {
      c->iter = iter + 1;
      c->sum_live += base_live;
      c->sum_ctx += tot;
      c->iter_ctx = tot;
    }
    if (base_live > row_cap) e |= 2;         // ... or for fewer rows
    if (e) { c->error = e; c->stop = 1; c->stop_iter = iter; c->n_rows = 0; }
  }
}

void launch_sched(hipStream_t st, Ctrl* ctrl, Slots s, int* row_slot, int* row_pos, int* free_stack, int blk,
                  int check_only, int row_cap, int ctx_cap, int4* att_items, int att_split, int att_cap) {
  hipLaunchKernelGGL(sched_kernel, dim3(1), dim3(1024), 0, st, ctrl, s, row_slot, row_pos, free_stack, blk,
                     check_only, row_cap, ctx_cap, att_items, att_split, att_cap);
}

// Pages for freshly admitted rollouts (prefill): slot_list[i] gets need[i] pages.
__global__ __launch_bounds__(256) void alloc_prefill_kernel(Ctrl* c, Slots s, const int* slot_list,
                                                            const int* need, int n, int* free_stack) {
  __shared__ int s_off[2049];
  const int free_top = c->free_top;
  if (threadIdx.x == 0) {
    int acc = 0;
    for (int i = 0; i < n; ++i) { s_off[i] = acc; acc += need[i]; }
    s_off[n] = acc;
  }
  __syncthreads();
  const int total = s_off[n];
  if (total > free_top) { if (threadIdx.x == 0) c->error = 1; return; }
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const int slot = slot_list[i], nb = need[i];
    if (nb > s.max_blocks) { c->error = 1; continue; }
    for (int j = 0; j < nb; ++j)
      s.block_table[(size_t)slot * s.max_blocks + j] = free_stack[free_top - 1 - (s_off[i] + j)];
    s.n_blocks[slot] = nb;
  }
  __syncthreads();
  if (threadIdx.x == 0) c->free_top = free_top - total;
}
void launch_alloc_prefill(hipStream_t st, Ctrl* ctrl, Slots s, const int* slot_list, const int* need, int n,
                          int* free_stack) {
  if (n <= 0) return;
  hipLaunchKernelGGL(alloc_prefill_kernel, dim3(1), dim3(256), 0, st, ctrl, s, slot_list, need, n, free_stack);
}

// Return every page of the listed slots to the stack.
__global__ __launch_bounds__(256) void free_slots_kernel(Ctrl* c, Slots s, const int* slot_list, int n,
                                                         int* free_stack) {
  __shared__ int s_off[2049];
  const int free_top = c->free_top;
  if (threadIdx.x == 0) {
    int acc = 0;
    for (int i = 0; i < n; ++i) { s_off[i] = acc; acc += s.n_blocks[slot_list[i]]; }
    s_off[n] = acc;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const int slot = slot_list[i], nb = s.n_blocks[slot];
    for (int j = 0; j < nb; ++j)
      free_stack[free_top + s_off[i] + j] = s.block_table[(size_t)slot * s.max_blocks + j];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += blockDim.x) { s.n_blocks[slot_list[i]] = 0; s.kv_len[slot_list[i]] = 0; }
  if (threadIdx.x == 0) c->free_top = free_top + s_off[n];
}
void launch_free_slots(hipStream_t st, Ctrl* ctrl, Slots s, const int* slot_list, int n, int* free_stack) {
  if (n <= 0) return;
  hipLaunchKernelGGL(free_slots_kernel, dim3(1), dim3(256), 0, st, ctrl, s, slot_list, n, free_stack);
}

// The free stack starts as a permutation that puts successive pops far apart: pop j hands out
// page (j * stride) mod n with stride ~ 0.618 n, coprime to n.  A prompt takes its pages in
// one go, and a row whose pages are consecutive in memory streams slower (the attention's
// load pattern alone: 5.4 TB/s against 6.0-6.1 TB/s for scattered or interleaved pages).
__global__ void free_stack_init_kernel(int* p, int n, int stride) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = (int)(((long long)(n - 1 - i) * stride) % n);     // the top of the stack is popped first
}
void launch_init_free_stack(hipStream_t st, int* free_stack, int n_blocks) {
  int stride = (int)((double)n_blocks * 0.6180339887) | 1;
  auto gcd = [](int a, int b) { while (b) { const int t = a % b; a = b; b = t; } return a; };
  while (stride < n_blocks && gcd(stride, n_blocks) != 1) stride += 2;
  if (stride >= n_blocks) stride = 1;
  hipLaunchKernelGGL(free_stack_init_kernel, dim3(ceil_div(n_blocks, 256)), dim3(256), 0, st, free_stack, n_blocks, stride);
}
__global__ void fill_i32_kernel(int* p, int v, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}
void launch_fill_i32(hipStream_t st, int* p, int v, size_t n) {
  if (n == 0) return;
  size_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, v, n);
}

// ---------------------------------------------------------------------------
// Token and log-probability arrays of many slots <-> one pinned host buffer.  A step moved them with one
// pageable copy per rollout and array, 8 us of host time and 3 us on the stream each: 950 copies in
// a step of 384 rollouts (7 ms of 170), 0.7 of 3.7 ms in the smallest configuration.  The host side
// of a transfer is bound by the link, so one wavefront per 64 consecutive ints with several in flight is enough.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void xfer_kernel(const XferItem* items, int* buf, int to_device) {
  const XferItem it = items[blockIdx.x];
  int* host = buf + it.off;
  const int stride = gridDim.y * 256;
  for (int i = blockIdx.y * 256 + threadIdx.x; i < it.n; i += stride) {
    if (to_device) it.dev[i] = host[i];
    else host[i] = it.dev[i];
  }
}
void launch_xfer(hipStream_t st, const XferItem* items, int n_items, int* buf, bool to_device) {
  if (n_items <= 0) return;
  hipLaunchKernelGGL(xfer_kernel, dim3(n_items, 8), dim3(256), 0, st, items, buf, to_device ? 1 : 0);
}

// ---------------------------------------------------------------------------
// Residual add (deterministic sum of split-K partials) + RMSNorm.
// One workgroup per output row; each thread owns up to 4 chunks of 8 columns.
//
// In the fragment order of the result 8 rows share every 128-byte line, 16 bytes each, and workgroups go to the XCDs in turn:
// row = workgroup id gave every L2 one piece of each line.  From 64 rows on (8 rows for each of 8 XCDs), 8 consecutive rows go to
// one XCD, whose L2 puts the lines together.  us under a kernel trace, before / now: 7000 rows of 2560 on average 48.7 / 34.3,
// 15 000 rows of 896 21.7 / 14.4, 13 900 rows of 2048 80 / 56, with 8 expert partials 327 / 303; 160-240 rows with 8 partials 6.4 / 5.9.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int norm_row(const RowCtx& rc) {
  const int b = (int)blockIdx.x;
  return rc.max_rows >= 64 ? ((b >> 6) * 8 + (b & 7)) * 8 + ((b >> 3) & 7) : b;
}
static unsigned norm_grid(const RowCtx& rc) { return (unsigned)(rc.max_rows >= 64 ? ceil_div(rc.max_rows, 64) * 64 : rc.max_rows); }

template <typename T, bool XF, int NP>
__global__ __launch_bounds__(256) void add_rmsnorm_kernel(RowCtx rc, float* x_res, const float* partials,
                                                          int n_partials_rt, size_t partial_stride,
                                                          const float* gain, T* h, int d, float eps,
                                                          const int* gather, const int* pos_of,
                                                          const float* wts, T* h_rows, float* x_copy) {
  const int r = norm_row(rc);
  ROW_GUARD(rc, r);
  const int rin = gather ? gather[r] : r;
  __shared__ float sh[4];
  float v[4][8];
  float ss = 0.f;
  const int nchunk = d >> 3;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int ch = threadIdx.x + c * 256;
    if (ch < nchunk) {
      float* xp = x_res + (size_t)rin * d + ch * 8;
      // NP >= 0: compile-time partial count, every load issued before the first add
      const int n_partials = NP >= 0 ? NP : n_partials_rt;
      f32x4 xv[2] = {*reinterpret_cast<const f32x4*>(xp), *reinterpret_cast<const f32x4*>(xp + 4)};
      if (NP >= 0) {
        f32x4 pv[NP > 0 ? NP : 1][2];
        float pw[NP > 0 ? NP : 1];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          const float* pp = pos_of ? partials + (size_t)pos_of[(size_t)rin * NP + p] * d + ch * 8
                                   : partials + p * partial_stride + (size_t)rin * d + ch * 8;
          pw[p] = wts ? wts[(size_t)rin * NP + p] : 1.0f;
          pv[p][0] = *reinterpret_cast<const f32x4*>(pp);
          pv[p][1] = *reinterpret_cast<const f32x4*>(pp + 4);
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) { xv[0] += pv[p][0] * pw[p]; xv[1] += pv[p][1] * pw[p]; }
      } else {
        for (int p = 0; p < n_partials; ++p) {
          const float* pp = partials + p * partial_stride + (size_t)rin * d + ch * 8;
          xv[0] += *reinterpret_cast<const f32x4*>(pp);
          xv[1] += *reinterpret_cast<const f32x4*>(pp + 4);
        }
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) v[c][j] = xv[j >> 2][j & 3];
      if (n_partials > 0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) xp[j] = v[c][j];
      }
      if (x_copy != nullptr) {           // the residual rows packed (gathered ones go on by themselves)
        float* cp = x_copy + (size_t)r * d + ch * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j) cp[j] = v[c][j];
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) ss = __fmaf_rn(v[c][j], v[c][j], ss);
    }
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = ss;
  __syncthreads();
  ss = sh[0] + sh[1] + sh[2] + sh[3];
  const float rinv = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int ch = threadIdx.x + c * 256;
    if (ch < nchunk) {
      T* hp = h + act_index<XF>(r, ch * 8, d);
      T hv[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) hv[j] = from_f32<T>(v[c][j] * rinv * gain[ch * 8 + j]);
#pragma unroll
      for (int j = 0; j < 8; ++j) hp[j] = hv[j];
      if (h_rows != nullptr) {           // second copy, plain [row][d]: rows that a later kernel gathers one by one
        T* rp = h_rows + (size_t)r * d + ch * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j) rp[j] = hv[j];
      }
    }
  }
}
template <typename T, bool XF>
void launch_add_rmsnorm(hipStream_t st, RowCtx rc, float* x_res, const float* partials, int n_partials,
                        size_t partial_stride, const float* gain, T* h, int d, float eps, const int* gather,
                        const int* pos_of, const float* wts, T* h_rows, float* x_copy) {
#define ARN_CASE(NP)                                                                                          \
  hipLaunchKernelGGL((add_rmsnorm_kernel<T, XF, NP>), dim3(norm_grid(rc)), dim3(256), 0, st, rc, x_res, partials, \
                     n_partials, partial_stride, gain, h, d, eps, gather, pos_of, wts, h_rows, x_copy)
  switch (n_partials) {
    case 0: ARN_CASE(0); break;
    case 1: ARN_CASE(1); break;
    case 2: ARN_CASE(2); break;
    case 3: ARN_CASE(3); break;
    case 4: ARN_CASE(4); break;
    case 5: ARN_CASE(5); break;
    case 6: ARN_CASE(6); break;
    case 7: ARN_CASE(7); break;
    case 8: ARN_CASE(8); break;
    default: ARN_CASE(-1); break;
  }
#undef ARN_CASE
}
template void launch_add_rmsnorm<float, false>(hipStream_t, RowCtx, float*, const float*, int, size_t, const float*, float*, int, float, const int*, const int*, const float*, float*, float*);
template void launch_add_rmsnorm<bf16_t, true>(hipStream_t, RowCtx, float*, const float*, int, size_t, const float*, bf16_t*, int, float, const int*, const int*, const float*, bf16_t*, float*);

// ---------------------------------------------------------------------------
// Embedding gather + the first layer's RMSNorm: x_res[r] = E[token at (slot, pos)], h = rmsnorm(x_res) * gain.
// Two launches before (an embedding launch is 5 us of an iteration, all latency: slot -> token -> row); the
// sums are add_rmsnorm_kernel's, in its order.
// ---------------------------------------------------------------------------
template <typename T, bool XF>
__global__ __launch_bounds__(256) void embed_norm_kernel(RowCtx rc, Slots s, const T* emb, float* x_res, const float* gain,
                                                         T* h, int d, float eps) {
  const int r = norm_row(rc);
  ROW_GUARD(rc, r);
  const int slot = rc.row_slot[r], pos = rc.row_pos[r];
  const T* e = emb + (size_t)s.tokens[(size_t)slot * s.max_ctx + pos] * d;
  __shared__ float sh[4];
  typedef T T8 __attribute__((ext_vector_type(8)));
  float v[4][8], ss = 0.f;
  const int nchunk = d >> 3;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int ch = threadIdx.x + c * 256;
    if (ch < nchunk) {
      const T8 ev = *reinterpret_cast<const T8*>(e + ch * 8);
#pragma unroll
      for (int j = 0; j < 8; ++j) v[c][j] = to_f32(ev[j]);
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int ch = threadIdx.x + c * 256;
    if (ch < nchunk) {
      float* xp = x_res + (size_t)r * d + ch * 8;
#pragma unroll
      for (int j = 0; j < 8; ++j) { xp[j] = v[c][j]; ss = __fmaf_rn(v[c][j], v[c][j], ss); }
    }
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = ss;
  __syncthreads();
  ss = sh[0] + sh[1] + sh[2] + sh[3];
  const float rinv = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int ch = threadIdx.x + c * 256;
    if (ch < nchunk) {
      T* hp = h + act_index<XF>(r, ch * 8, d);
      T8 hv;
#pragma unroll
      for (int j = 0; j < 8; ++j) hv[j] = from_f32<T>(v[c][j] * rinv * gain[ch * 8 + j]);
      *reinterpret_cast<T8*>(hp) = hv;
    }
  }
}
template <typename T, bool XF>
void launch_embed_norm(hipStream_t st, RowCtx rc, Slots s, const T* emb, float* x_res, const float* gain, T* h, int d, float eps) {
  hipLaunchKernelGGL((embed_norm_kernel<T, XF>), dim3(norm_grid(rc)), dim3(256), 0, st, rc, s, emb, x_res, gain, h, d, eps);
}
template void launch_embed_norm<float, false>(hipStream_t, RowCtx, Slots, const float*, float*, const float*, float*, int, float);
template void launch_embed_norm<bf16_t, true>(hipStream_t, RowCtx, Slots, const bf16_t*, float*, const float*, bf16_t*, int, float);

// ---------------------------------------------------------------------------
// Rotary tables, computed once in double precision: cos/sin[pos][i], i < head_dim/2,
// angle = pos * theta^(-2i/head_dim).
// ---------------------------------------------------------------------------
__global__ void rope_table_kernel(float* cos_t, float* sin_t, int max_pos, int head_dim, float theta) {
  const int half = head_dim / 2;
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)max_pos * half) return;
  const int pos = (int)(idx / half), i = (int)(idx % half);
  const double ang = (double)pos * pow((double)theta, -2.0 * (double)i / (double)head_dim);
  cos_t[idx] = (float)cos(ang);
  sin_t[idx] = (float)sin(ang);
}
void launch_rope_table(hipStream_t st, float* cos_t, float* sin_t, int max_pos, int head_dim, float theta) {
  const size_t n = (size_t)max_pos * (head_dim / 2);
  hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, cos_t, sin_t,
                     max_pos, head_dim, theta);
}

// ---------------------------------------------------------------------------
// Rotary embedding of q and k, append of k and v to the paged cache.
// qkv: fp32 [n_partials][rows][(Hq + 2 Hkv) * dh]
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void rope_append_kernel(RowCtx rc, Slots s, const float* qkv, int n_partials,
                                                          size_t partial_stride, const float* rope_cos,
                                                          const float* rope_sin, float* q_rot, T* kv_pool,
                                                          KVLayout L, int layer, int Hq, bf16_t* q_bf16) {
  const int r = blockIdx.x;
  ROW_GUARD(rc, r);
  const int slot = rc.row_slot[r], pos = rc.row_pos[r];
  const int dh = L.head_dim, half = dh >> 1, Hkv = L.n_kv_heads;
  const int nq = Hq * dh, nkv = Hkv * dh, ncol = nq + 2 * nkv;
  const int page = s.block_table[(size_t)slot * s.max_blocks + pos / L.blk], t = pos % L.blk;
  const float* src = qkv + (size_t)r * ncol;
  const float* cs = rope_cos + (size_t)pos * half;
  const float* sn = rope_sin + (size_t)pos * half;
  auto val = [&](int col) {
    float a = src[col];
    for (int p = 1; p < n_partials; ++p) a += src[p * partial_stride + col];
    return a;
  };
  // rotations: Hq + Hkv heads, `half` pairs each
  for (int e = threadIdx.x; e < (Hq + Hkv) * half; e += blockDim.x) {
    const int hd = e / half, i = e % half;
    const float a = val(hd * dh + i), b = val(hd * dh + i + half);
    const float c = cs[i], sI = sn[i];
    const float ra = rope_first(a, b, c, sI), rb = rope_second(a, b, c, sI);
    if (hd < Hq) {
      const size_t at = (size_t)r * nq + hd * dh + i;
      if (q_bf16 != nullptr) { q_bf16[at] = (bf16_t)ra; q_bf16[at + half] = (bf16_t)rb; }
      else { q_rot[at] = ra; q_rot[at + half] = rb; }
    } else {
      const int kh = hd - Hq;
      kv_pool[L.at(layer, 0, page, kh, t, i)] = from_f32<T>(ra);
      kv_pool[L.at(layer, 0, page, kh, t, i + half)] = from_f32<T>(rb);
    }
  }
  for (int e = threadIdx.x; e < nkv; e += blockDim.x) {
    const int kh = e / dh, i = e % dh;
    kv_pool[L.at(layer, 1, page, kh, t, i)] = from_f32<T>(val(nq + nkv + e));
  }
}
template <typename T>
void launch_rope_append(hipStream_t st, RowCtx rc, Slots s, const float* qkv, int n_partials, size_t partial_stride,
                        const float* rope_cos, const float* rope_sin, float* q_rot, T* kv_pool, KVLayout kvl,
                        int layer, int n_q_heads, bf16_t* q_bf16) {
  hipLaunchKernelGGL(rope_append_kernel<T>, dim3(rc.max_rows), dim3(256), 0, st, rc, s, qkv, n_partials,
                     partial_stride, rope_cos, rope_sin, q_rot, kv_pool, kvl, layer, n_q_heads, q_bf16);
}
template void launch_rope_append<float>(hipStream_t, RowCtx, Slots, const float*, int, size_t, const float*, const float*, float*, float*, KVLayout, int, int, bf16_t*);
template void launch_rope_append<bf16_t>(hipStream_t, RowCtx, Slots, const float*, int, size_t, const float*, const float*, float*, bf16_t*, KVLayout, int, int, bf16_t*);

// ---------------------------------------------------------------------------
// Reference paged attention: one wavefront per (row, query head), one cached token
// per loop trip, online softmax.  Correctness path of the bf16 KV cache (debug switch).
// ---------------------------------------------------------------------------
template <typename T, bool XF>
__global__ __launch_bounds__(64) void attn_ref_kernel(RowCtx rc, Slots s, const float* q_rot, const T* kv_pool,
                                                      KVLayout L, int layer, int Hq, T* out) {
  const int r = blockIdx.x, a = blockIdx.y;
  ROW_GUARD(rc, r);
  const int slot = rc.row_slot[r], pos = rc.row_pos[r];
  const int ctx = pos + 1, dh = L.head_dim, lane = threadIdx.x;
  const int kvh = a / (Hq / L.n_kv_heads);
  const float* q = q_rot + (size_t)r * Hq * dh + a * dh;
  const bool has0 = lane < dh, has1 = lane + 64 < dh;
  const float q0 = has0 ? q[lane] : 0.f, q1 = has1 ? q[lane + 64] : 0.f;
  const float scale = 1.0f / sqrtf((float)dh);
  const int* bt = s.block_table + (size_t)slot * s.max_blocks;
  float m = -INFINITY, l = 0.f, o0 = 0.f, o1 = 0.f;
  for (int j = 0; j < ctx; ++j) {
    const int page = bt[j / L.blk], t = j % L.blk;
    float part = 0.f;
    if (has0) part += q0 * to_f32(kv_pool[L.at(layer, 0, page, kvh, t, lane)]);
    if (has1) part += q1 * to_f32(kv_pool[L.at(layer, 0, page, kvh, t, lane + 64)]);
    const float sc = wave_sum(part) * scale;
    const float m_new = fmaxf(m, sc);
    const float corr = expf(m - m_new), p = expf(sc - m_new);
    l = l * corr + p;
    if (has0) o0 = o0 * corr + p * to_f32(kv_pool[L.at(layer, 1, page, kvh, t, lane)]);
    if (has1) o1 = o1 * corr + p * to_f32(kv_pool[L.at(layer, 1, page, kvh, t, lane + 64)]);
    m = m_new;
  }
  const int K = Hq * dh;
  if (has0) out[act_index<XF>(r, a * dh + lane, K)] = from_f32<T>(o0 / l);
  if (has1) out[act_index<XF>(r, a * dh + lane + 64, K)] = from_f32<T>(o1 / l);
}
template <typename T, bool XF>
void launch_attn_ref(hipStream_t st, RowCtx rc, Slots s, const float* q_rot, const T* kv_pool, KVLayout kvl,
                     int layer, int n_q_heads, T* out) {
  hipLaunchKernelGGL((attn_ref_kernel<T, XF>), dim3(rc.max_rows, n_q_heads), dim3(64), 0, st, rc, s, q_rot,
                     kv_pool, kvl, layer, n_q_heads, out);
}
template void launch_attn_ref<bf16_t, true>(hipStream_t, RowCtx, Slots, const float*, const bf16_t*, KVLayout, int, int, bf16_t*);

// ---------------------------------------------------------------------------
// fp32 paged attention: one wavefront per (row, query head), 64 cached tokens per step.  The scores
// of a step are one token per lane (each lane walks its token's key), the weighted sum of the values
// one dimension per lane with 64 / DH tokens at a time, the probabilities broadcast from their
// lanes.  A step's maximum and sum are shuffle trees, steps are joined by the online softmax in
// token order: the sum's order depends on the row's own length only, in prefill and decode alike.
// One token per trip (6 dependent shuffles, 2 exponentials and 2 loads each) took 38 us per launch
// at 32 rows of 33-128 tokens; this takes 6.5 us (both with the 2 us that a profiler adds).
// Registers decide how many rows a compute unit works on: 112 to 128 here.  With a step's keys and 64 values requested together (171 for
// heads of 32, 255 of 64) two wavefronts fit a SIMD, and a whole step's address arithmetic with bounds was a third of the time.
// us per launch, that / this: prefill of 16 384 rows, 4 heads of 32 in prompts of 32, 256, 4096 tokens 167, 350, 4045 / 82, 197, 2340,
// 12 + 3 of 64 777, 1862, 22 900 / 348, 1053, 13 570; decode of 1 and 256 rows of 1024 tokens 56, 67 / 32, 50 and 97, 242 / 53, 149.
// ---------------------------------------------------------------------------
// ALONE: few wavefronts on the unit, registers to spare.  Heads of 32 then request a partial step's values together where they are more
// than 16 loads (200 rows of 32-55 tokens: 60 -> 58 us per iteration of two layers; heads of 64, 64 loads: 62 -> 63).
template <int DH, bool ALONE, class Out>
__device__ __forceinline__ void attn_f32_row(const f32x4* sq, const float* kv_pool, const int* bt, const KVLayout& L, int layer, int kvh,
                                             int ctx, Out out) {
  constexpr int TG = DH < 64 ? 64 / DH : 1;        // tokens side by side in the value product
  constexpr int DL = DH > 64 ? DH / 64 : 1;        // dimensions per lane there
  const int lane = threadIdx.x & 63;
  const float scale = 1.0f / sqrtf((float)DH);
  const int vd = (lane % (DH / DL)) * DL, vt = lane / (DH / DL);      // this lane's dimensions and token residue
  float m = -INFINITY, l = 0.f, o[DL] = {};
  for (int j0 = 0; j0 < ctx; j0 += 64) {
    const int j = j0 + lane, n = min(64, ctx - j0);
    const bool live = lane < n;
    const int page = bt[(live ? j : ctx - 1) >> 4];
    const f32x4* k = reinterpret_cast<const f32x4*>(kv_pool + L.at(layer, 0, page, kvh, (live ? j : ctx - 1) & 15, 0));
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c0 = 0; c0 < DH / 4; c0 += 8) {         // 32 dimensions of the keys in registers at a time
      f32x4 kv[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) kv[c] = k[c0 + c];
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const f32x4 qv = sq[c0 + c];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = __fmaf_rn(kv[c][e], qv[e], acc[e]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    const float sc = live ? ((acc[0] + acc[1]) + (acc[2] + acc[3])) * scale : -INFINITY;
    const float m_new = fmaxf(m, wave_max_f32(sc)), corr = expf(m - m_new), p = live ? expf(sc - m_new) : 0.f;
    l = __fmaf_rn(l, corr, wave_sum(p));
    m = m_new;
    float add[DL] = {};
    // 16 loads of values in flight.  whole: 64 tokens, as in every step but a row's last - no bounds, constant offsets in a page
    auto values = [&](int t0, auto loads, auto whole) {
      constexpr int U = decltype(loads)::value;
      float v[U][DL], pt[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int t = t0 + u * TG, tv = whole ? t + vt : min(t + vt, n - 1);       // (t + TG - 1 lies in the page of t)
        pt[u] = TG == 1 ? as_f32(__builtin_amdgcn_readlane(__float_as_int(p), tv)) : __shfl(p, tv, 64);
        const float* src = kv_pool + L.at(layer, 1, __builtin_amdgcn_readlane(page, whole ? t : min(t, n - 1)), kvh, tv & 15, vd);
#pragma unroll
        for (int e = 0; e < DL; ++e) v[u][e] = src[e];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < DL; ++e) add[e] = whole || t0 + u * TG + vt < n ? __fmaf_rn(pt[u], v[u][e], add[e]) : add[e];
    };
    using Few = std::integral_constant<int, 16>;
    using All = std::integral_constant<int, 64 / TG>;
    if (n == 64) {
#pragma unroll
      for (int t0 = 0; t0 < 64; t0 += 16 * TG) values(t0, Few{}, std::true_type{});
    } else if (ALONE && TG > 1 && n > 16 * TG) {
      values(0, All{}, std::false_type{});
    } else {
#pragma unroll 1
      for (int t0 = 0; t0 < n; t0 += 16 * TG) values(t0, Few{}, std::false_type{});
    }
#pragma unroll
    for (int e = 0; e < DL; ++e) {
#pragma unroll
      for (int off = 32; off >= DH && off > 0; off >>= 1) add[e] += __shfl_xor(add[e], off, 64);
      o[e] = __fmaf_rn(o[e], corr, add[e]);
    }
  }
  if (vt == 0) {
#pragma unroll
    for (int e = 0; e < DL; ++e) out(vd + e, o[e] / l);
  }
}
template <int DH>
__global__ __launch_bounds__(64) void attn_f32_kernel(RowCtx rc, Slots s, const float* q_rot, const float* kv_pool,
                                                      KVLayout L, int layer, int Hq, float* out) {
  const int r = blockIdx.x, a = blockIdx.y;
  ROW_GUARD(rc, r);
  const int slot = rc.row_slot[r], ctx = rc.row_pos[r] + 1, lane = threadIdx.x;
  __shared__ f32x4 sq[DH / 4];
  const f32x4* q = reinterpret_cast<const f32x4*>(q_rot + (size_t)r * Hq * DH + a * DH);
  if (lane < DH / 4) sq[lane] = q[lane];
  __syncthreads();
  float* dst = out + (size_t)r * Hq * DH + a * DH;
  attn_f32_row<DH, false>(sq, kv_pool, s.block_table + (size_t)slot * s.max_blocks, L, layer, a / (Hq / L.n_kv_heads), ctx,
                   [&](int d, float v) { dst[d] = v; });
}
void launch_attn_f32(hipStream_t st, RowCtx rc, Slots s, const float* q_rot, const float* kv_pool, KVLayout kvl, int layer,
                     int n_q_heads, float* out) {
  dim3 grid(rc.max_rows, n_q_heads);
#define ATT_F32(DH) hipLaunchKernelGGL((attn_f32_kernel<DH>), grid, dim3(64), 0, st, rc, s, q_rot, kv_pool, kvl, layer, n_q_heads, out)
  switch (kvl.head_dim) {
    case 32: ATT_F32(32); break;
    case 64: ATT_F32(64); break;
    default: ATT_F32(128); break;
  }
#undef ATT_F32
}

// ---------------------------------------------------------------------------
// act = silu(gate) * up from gu fp32 [rows][2F] (gate columns first, then up).
// ---------------------------------------------------------------------------
template <typename T, bool XF>
__global__ __launch_bounds__(256) void silu_mul_kernel(RowCtx rc, const float* gu, int F, T* act) {
  const int r = blockIdx.x;
  ROW_GUARD(rc, r);
  const float* g = gu + (size_t)r * 2 * F;
  for (int f = threadIdx.x; f < F; f += blockDim.x) {
    const float x = g[f];
    act[act_index<XF>(r, f, F)] = from_f32<T>(x / (1.0f + expf(-x)) * g[F + f]);
  }
}
template <typename T, bool XF>
void launch_silu_mul(hipStream_t st, RowCtx rc, const float* gu, int F, T* act) {
  hipLaunchKernelGGL((silu_mul_kernel<T, XF>), dim3(rc.max_rows), dim3(256), 0, st, rc, gu, F, act);
}
template void launch_silu_mul<float, false>(hipStream_t, RowCtx, const float*, int, float*);
template void launch_silu_mul<bf16_t, true>(hipStream_t, RowCtx, const float*, int, bf16_t*);

// ---------------------------------------------------------------------------
// Reference GEMM: out[m][n] = sum_k x[m][k] W[n][k], fp32 accumulate.
// One wavefront per output column n and 8 rows; lanes stride over k.
// ---------------------------------------------------------------------------
template <typename T, bool XF>
__global__ __launch_bounds__(256) void gemm_ref_kernel(RowCtx rc, const T* x, const T* W, float* out, int N, int K) {
  const int rows = rows_or_zero(rc);
  const int r0 = blockIdx.y * 8;
  if (r0 >= rows) return;
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (n >= N) return;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const T* w = W + (size_t)n * K;
  for (int k = lane; k < K; k += 64) {
    const float wv = to_f32(w[k]);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (r0 + j < rows) acc[j] += wv * to_f32(x[act_index<XF>(r0 + j, k, K)]);
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float v = wave_sum(acc[j]);
    if (lane == 0 && r0 + j < rows) out[(size_t)(r0 + j) * N + n] = v;
  }
}
template <typename T, bool XF>
void launch_gemm_ref(hipStream_t st, RowCtx rc, const T* x, const T* W, float* out, int N, int K) {
  hipLaunchKernelGGL((gemm_ref_kernel<T, XF>), dim3(ceil_div(N, 4), ceil_div(rc.max_rows, 8)), dim3(256), 0, st,
                     rc, x, W, out, N, K);
}
template void launch_gemm_ref<bf16_t, true>(hipStream_t, RowCtx, const bf16_t*, const bf16_t*, float*, int, int);

// ---------------------------------------------------------------------------
// fp32 GEMM: out[m][n] = sum_k x[m][k] W[n][k] on v_mfma_f32_16x16x4_f32 (full fp32 products and sums).
// A workgroup owns 16 columns x 16 rows, its 4 wavefronts a quarter of k each; a lane fetches 4
// consecutive k of its row of either operand (whole 64-byte pieces of the matrices, several steps in
// flight) and the products take element j of both, each j in its own accumulator: short chains, added
// pairwise, then the wavefronts through LDS.  An element's chain depends on K only.  One wavefront per
// column with a 6-step shuffle sum per row took 11 us per launch on the 128-wide fp32
// configuration (24 rows in decode, 768 in prefill); this takes 5.4 us.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void gemm_f32_kernel(RowCtx rc, const float* __restrict__ x, const float* __restrict__ W,
                                                       float* __restrict__ out, int N, int K) {
  typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
  __shared__ f32x4 red[3][64];
  const int rows = rows_or_zero(rc);
  const int m0 = blockIdx.y * 16, n0 = blockIdx.x * 16;
  if (m0 >= rows) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = lane & 15, kq = (lane >> 4) * 4;
  const float* wp = W + (size_t)min(n0 + c, N - 1) * K;
  const float* xp = x + (size_t)min(m0 + c, rows - 1) * K;
  const int steps = (K + 15) >> 4, s0 = steps * wave / 4, s1 = steps * (wave + 1) / 4;
  auto fetch = [&](const float* p, int k) -> f32x4 {
    if (k + 4 <= K) return *reinterpret_cast<const f32x4u*>(p + k);
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 4; ++e) if (k + e < K) v[e] = p[k + e];
    return v;
  };
  f32x4 acc[4] = {f32x4{}, f32x4{}, f32x4{}, f32x4{}};
  constexpr int U = 8;
  for (int st = s0; st < s1; st += U) {
    f32x4 a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = min(st + u, s1 - 1) * 16 + kq;
      a[u] = fetch(wp, k);
      b[u] = fetch(xp, k);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (st + u < s1) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][e], b[u][e], acc[e], 0, 0, 0);
      }
  }
  f32x4 v = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  if (wave > 0) red[wave - 1][lane] = v;
  __syncthreads();
  if (wave > 0) return;
  v = (v + red[0][lane]) + (red[1][lane] + red[2][lane]);
  const int m = m0 + c, n = n0 + kq;                 // accumulator: column = row m of x, rows = 4 consecutive n
  if (m < rows) {
    float* o = out + (size_t)m * N + n;
    if (n + 4 <= N) *reinterpret_cast<f32x4u*>(o) = v;
    else
      for (int e = 0; e < 4; ++e) if (n + e < N) o[e] = v[e];
  }
}
void launch_gemm_f32(hipStream_t st, RowCtx rc, const float* x, const float* W, float* out, int N, int K) {
  hipLaunchKernelGGL(gemm_f32_kernel, dim3(ceil_div(N, 16), ceil_div(rc.max_rows, 16)), dim3(256), 0, st, rc, x, W, out, N, K);
}

// ---------------------------------------------------------------------------
// Small fp32 models.  A decode iteration of one is nothing but launches: the fp32 configuration (two layers of 128,
// 24 rows) ran 22 kernels of 3-6 us for 1 MB of weights a layer.  Rows do not need each other, so here a workgroup takes a
// row through the whole model - embedding to logits, 8 wavefronts, activations in LDS - and streams the weights from its L2 at
// what one compute unit takes (30-50 bytes per clock).  That pays while a layer's weights take less than its launches did.
// us per decode iteration of two layers, contexts of 32-97 tokens, at 1, 24, 96, 256, 310 rows, separate launches / this: 1.05 MB a layer (width
// 128, 4 heads of 32) 70, 80, 84, 100, 114 / 49, 51, 56, 61, 106; 1.21 MB (8 heads) 73, 80, 92, 110, 123 / 54, 59, 64, 69, 121; 0.88 MB (2 heads
// of 128) 76, 86, 88, 104, 115 / 53, 56, 60, 65, 115.  Beyond a layer of about 1.3 MB or a head of 0.5 MB (1.48 MB: 80, 91, 105 /
// 84, 91, 91; 1.47 MB with a head of 1.3: 82, 92, 106 / 100, 103, 102) the weights take longer than the launches did.
//
// Dot products: 8 lanes, four consecutive k each per 32, an accumulator for each of the four, added pairwise, then over the
// lanes by a fixed tree (32 lanes to a column spend three times the instructions: the pass was bound by them, 27 bytes per
// clock).  The prefill product of such a model (gemm_f32_dot_kernel) and the decode row share it, and the
// norms, the rotation and the attention are the prefill's code too: a re-prefilled rollout keeps its bits.
// ---------------------------------------------------------------------------
template <int CTRL> __device__ inline float dpp_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
// sum over 8 consecutive lanes, in all of them
__device__ inline float sum8(const f32x4& acc) {
  float v = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  v = dpp_add<0xb1>(v);                       // the lanes of a pair, of a quad, the mirrored lane of the eight
  v = dpp_add<0x4e>(v);
  return dpp_add<0x141>(v);
}
__device__ inline void fma4(const f32x4& a, const f32x4& b, f32x4& acc) {
#pragma unroll
  for (int e = 0; e < 4; ++e) acc[e] = __fmaf_rn(a[e], b[e], acc[e]);
}
// f(n, W[n] . x) for the N rows of W, x in LDS; all wavefronts.  KC: pieces of 32 k per step, U columns per lane in flight.
constexpr int ROW_THREADS = 512;
template <int KC, int U, class F>
__device__ __forceinline__ void row_gemv(const float* __restrict__ W, const float* xs, int N, int K, F f) {
  constexpr int STEP = ROW_THREADS / 8;
  const int l = threadIdx.x & 7, first = (int)(threadIdx.x >> 3);
  const f32x4* x4 = reinterpret_cast<const f32x4*>(xs);
  for (int n0 = first; n0 < N + first % 8; n0 += U * STEP) {       // (the same trips for the 8 columns of a wavefront)
    f32x4 acc[U];
    const float* wp[U];
#pragma unroll
    for (int u = 0; u < U; ++u) { acc[u] = f32x4{}; wp[u] = W + (size_t)min(n0 + u * STEP, N - 1) * K; }
    for (int k0 = 4 * l; k0 < K + 4 * l; k0 += 32 * KC) {
      f32x4 w[U][KC];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < KC; ++c) {
          w[u][c] = f32x4{};
          if (k0 + c * 32 < K) w[u][c] = *reinterpret_cast<const f32x4*>(wp[u] + k0 + c * 32);
        }
#pragma unroll
      for (int c = 0; c < KC; ++c) {
        const int k = k0 + c * 32;
        const f32x4 x = k < K ? x4[k >> 2] : f32x4{};
#pragma unroll
        for (int u = 0; u < U; ++u) fma4(w[u][c], x, acc[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int n = n0 + u * STEP;
      const float v = sum8(acc[u]);
      if (l == 0 && n < N) f(n, v);
    }
  }
}
// out[m][n] = x[m] . W[n] with the same sums: 32 NC columns x 4 rows per workgroup, a lane's columns 32 apart.
template <int NC>
__global__ __launch_bounds__(256) void gemm_f32_dot_kernel(RowCtx rc, const float* __restrict__ x, const float* __restrict__ W,
                                                           float* __restrict__ out, int N, int K) {
  constexpr int MT = 4, UNROLL = NC < 4 ? 4 : 1;
  const int rows = rows_or_zero(rc), m0 = blockIdx.y * MT;
  if (m0 >= rows) return;
  const int l = threadIdx.x & 7, n = blockIdx.x * 32 * NC + (int)(threadIdx.x >> 3);
  const float *wp[NC], *xp[MT];
#pragma unroll
  for (int c = 0; c < NC; ++c) wp[c] = W + (size_t)min(n + 32 * c, N - 1) * K;
#pragma unroll
  for (int m = 0; m < MT; ++m) xp[m] = x + (size_t)min(m0 + m, rows - 1) * K;
  f32x4 acc[MT][NC];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[m][c] = f32x4{};
#pragma unroll UNROLL
  for (int k = 4 * l; k < K; k += 32) {
    f32x4 w[NC], xv[MT];
#pragma unroll
    for (int c = 0; c < NC; ++c) w[c] = *reinterpret_cast<const f32x4*>(wp[c] + k);
#pragma unroll
    for (int m = 0; m < MT; ++m) xv[m] = *reinterpret_cast<const f32x4*>(xp[m] + k);
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int c = 0; c < NC; ++c) fma4(w[c], xv[m], acc[m][c]);
  }
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const float v = sum8(acc[m][c]);
      if (l == 0 && n + 32 * c < N && m0 + m < rows) out[(size_t)(m0 + m) * N + n + 32 * c] = v;
    }
}
// A weight is read again for every 4 rows, from L1: the more columns to a lane, the more products per byte of both operands, as long
// as the workgroups still fill the chip.  us per launch, matrix instructions (gemm_f32_kernel) | 32, 64, 128 columns: 1024 x 128 at 24,
// 96, 300, 16 384 rows 4.0, 5.7, 10.9, 443 | 2.7, 3.8, 8.0, 308 | 3.0, 3.6, 6.1, 193 | 3.7, 3.8, 5.9, 146; 256 x 256 at 300, 16 384 rows
// 5.9, 113 | 5.5, 149 | 4.9, 94 | 4.8, 69; 128 x 512 at 300, 768, 16 384 rows 4.8, 6.5, 59 | 6.6, 9.1, 145 | 5.2, 7.7, 94 | 6.9, 7.1, 67.
void launch_gemm_f32_dot(hipStream_t st, RowCtx rc, const float* x, const float* W, float* out, int N, int K) {
  const int m_groups = ceil_div(rc.max_rows, 4);
  const long long units = (long long)ceil_div(N, 32) * m_groups;
#define DOT_F32(NC) hipLaunchKernelGGL((gemm_f32_dot_kernel<NC>), dim3(ceil_div(N, 32 * NC), m_groups), dim3(256), 0, st, rc, x, W, out, N, K)
  if (units <= 256) DOT_F32(1);
  else if (units < 1024 || N <= 64) DOT_F32(2);
  else DOT_F32(4);
#undef DOT_F32
}

template <int DH>
__global__ __launch_bounds__(ROW_THREADS) void forward_f32_kernel(RowCtx rc, Slots s, F32Model m, float* logits, Ctrl* ctrl, int greedy,
                                                                  float temperature) {
  extern __shared__ __align__(16) float lds[];
  const int r = blockIdx.x;
  const int slot = rc.row_slot[r], pos = rc.row_pos[r];
  ROW_GUARD(rc, r);
  const int tid = threadIdx.x, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int d = m.d, F = m.F, Hq = m.n_q_heads, Hkv = m.kvl.n_kv_heads, nq = Hq * DH, nqkv = nq + 2 * Hkv * DH;
  constexpr int HALF = DH / 2;
  float *x = lds, *h = x + d, *qkv = h + d, *att = qkv + nqkv, *gu = qkv;       // (gate / up where the queries were)
  __shared__ float part[4];
  const int* row_bt = s.block_table + (size_t)slot * s.max_blocks;
  const int page = row_bt[pos >> 4], tin = pos & 15;
  int* bt = reinterpret_cast<int*>(lds) + m.lds_floats;       // the row's pages, for every layer's attention
  for (int i = tid; i <= pos >> 4; i += ROW_THREADS) bt[i] = row_bt[i];
  {
    const float* e = m.tok_emb + (size_t)s.tokens[(size_t)slot * s.max_ctx + pos] * d;
    for (int i = tid; i < d; i += ROW_THREADS) x[i] = e[i];
  }
  // h = rmsnorm(x) * gain, the sums of add_rmsnorm_kernel (8 columns per thread, 256 threads)
  auto norm = [&](const float* gain) {
    const bool own = tid < 256 && tid < (d >> 3);
    float v[8], gn[8], ss = 0.f;
    if (own) {
#pragma unroll
      for (int j = 0; j < 8; ++j) gn[j] = gain[tid * 8 + j];
    }
    __syncthreads();
    if (tid < 256) {
      if (own) {
#pragma unroll
        for (int j = 0; j < 8; ++j) { v[j] = x[tid * 8 + j]; ss = __fmaf_rn(v[j], v[j], ss); }
      }
      ss = wave_sum(ss);
      if ((tid & 63) == 0) part[wid] = ss;
    }
    __syncthreads();
    if (own) {
      ss = part[0] + part[1] + part[2] + part[3];
      const float rinv = 1.0f / sqrtf(ss / (float)d + m.eps);
#pragma unroll
      for (int j = 0; j < 8; ++j) h[tid * 8 + j] = v[j] * rinv * gn[j];
    }
    __syncthreads();
  };
  for (int layer = 0; layer < m.n_layers; ++layer) {
    const F32Layer L = m.layers[layer];
    norm(L.attn_norm);
    row_gemv<4, 4>(L.wqkv, h, nqkv, d, [&](int n, float v) { qkv[n] = v; });
    __syncthreads();
    // rotary embedding of q and the new key, append of key and value
    for (int e = tid; e < (Hq + Hkv) * HALF; e += ROW_THREADS) {
      const int hd = e / HALF, i = e % HALF;
      const float a = qkv[hd * DH + i], b = qkv[hd * DH + i + HALF];
      const float c = m.rope_cos[(size_t)pos * HALF + i], sn = m.rope_sin[(size_t)pos * HALF + i];
      const float ra = rope_first(a, b, c, sn), rb = rope_second(a, b, c, sn);
      if (hd < Hq) {
        qkv[hd * DH + i] = ra;
        qkv[hd * DH + i + HALF] = rb;
      } else {
        m.kv_pool[m.kvl.at(layer, 0, page, hd - Hq, tin, i)] = ra;
        m.kv_pool[m.kvl.at(layer, 0, page, hd - Hq, tin, i + HALF)] = rb;
      }
    }
    for (int e = tid; e < Hkv * DH; e += ROW_THREADS)
      m.kv_pool[m.kvl.at(layer, 1, page, e / DH, tin, e % DH)] = qkv[nq + Hkv * DH + e];
    __syncthreads();                              // (the workgroup's stores are visible to its own loads behind this)
    for (int a = wid; a < Hq; a += ROW_THREADS / 64)
      attn_f32_row<DH, true>(reinterpret_cast<const f32x4*>(qkv + a * DH), m.kv_pool, bt, m.kvl, layer, a / (Hq / Hkv), pos + 1,
                       [&](int i, float v) { att[a * DH + i] = v; });
    __syncthreads();
    row_gemv<4, 2>(L.wo, att, d, nq, [&](int n, float v) { x[n] += v; });
    norm(L.mlp_norm);
    row_gemv<4, 4>(L.wgu, h, 2 * F, d, [&](int n, float v) { gu[n] = v; });
    __syncthreads();
    for (int f = tid; f < F; f += ROW_THREADS) gu[f] = gu[f] / (1.0f + expf(-gu[f])) * gu[F + f];
    __syncthreads();
    row_gemv<8, 2>(L.wd, gu, d, F, [&](int n, float v) { x[n] += v; });
  }
  norm(m.final_norm);
  row_gemv<4, 4>(m.lm_head, h, m.vocab, d, [&](int n, float v) { logits[(size_t)r * m.vocab + n] = v; });
  if (!greedy) return;
  // The greedy token and its log-probability, here where the logits are (a launch of its own was 3 of 62 us of an iteration of 24 rows): the choice,
  // the maximum and the sum of sample_rows_kernel, whose 1024 threads' partial sums a thread takes two of, in the same order.  (Forced
  // tokens come with watched logits, which the sampler's own kernel takes.)
  __shared__ unsigned red_key[8];
  __shared__ int red_idx[8], token;
  __shared__ float red_max[8];
  __shared__ double red_sum[16];
  const int V = m.vocab, lane = tid & 63;
  const float* lg = logits + (size_t)r * V;
  const RowState q = load_row(rc, s, ctrl, r, 1, nullptr, nullptr);
  __syncthreads();                                // (the workgroup's own logits, as its keys and values above)
  unsigned bk = 0u;
  int bi = 0x7fffffff;
  float M = -INFINITY;
  for (int i = tid; i < V; i += ROW_THREADS) {
    const float v = lg[i];
    const unsigned k = f2key(v);
    if (bi == 0x7fffffff || k > bk) { bk = k; bi = i; }        // ascending i: the first maximum stays
    M = fmaxf(M, v);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned ok = __shfl_xor(bk, off, 64);
    const int oi = __shfl_xor(bi, off, 64);
    if (ok > bk || (ok == bk && oi < bi)) { bk = ok; bi = oi; }
  }
  M = wave_max_f32(M);
  if (lane == 0) { red_key[wid] = bk; red_idx[wid] = bi; red_max[wid] = M; }
  __syncthreads();
  for (int x = 0; x < 8; ++x) M = fmaxf(M, red_max[x]);
  if (tid == 0) {
    for (int x = 1; x < 8; ++x)
      if (red_key[x] > bk || (red_key[x] == bk && red_idx[x] < bi)) { bk = red_key[x]; bi = red_idx[x]; }
    token = bi;
  }
  if (s.logprob != nullptr) {
    const float invT = 1.0f / temperature;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      double part = 0.0;
      for (int i = half * ROW_THREADS + tid; i < V; i += 2 * ROW_THREADS) part += (double)__expf((lg[i] - M) * invT);
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off, 64);
      if (lane == 0) red_sum[half * 8 + wid] = part;
    }
    __syncthreads();
    if (tid == 0) {
      double Z = red_sum[0];
      for (int x = 1; x < 16; ++x) Z += red_sum[x];
      s.logprob[(size_t)q.slot * s.max_ctx + q.g] = (float)((double)((lg[token] - M) * invT) - log(Z));
    }
  }
  if (tid == 0) finish_row(s, ctrl, q, r, 1, token, token, nullptr);
}
static size_t forward_f32_lds(int d, int F, int nq, int nqkv) { return (size_t)(2 * d + (nqkv + nq > 2 * F ? nqkv + nq : 2 * F)); }     // floats
bool forward_f32_takes(int d, int F, int nq, int nqkv, int vocab) {
  const size_t layer_bytes = ((size_t)nqkv * d + (size_t)nq * d + (size_t)3 * F * d) * sizeof(float);
  const size_t head_bytes = (size_t)vocab * d * sizeof(float);
  // Widths for which prefill's products lose nothing to the matrix instructions either, all of a layer's together: sums of up to
  // about 400 terms are faster here, and a longer one (the down projection, the output projection) must not outweigh the others.
  // At 16 384 rows 320 x 512 takes 185 us, 144 there; 16 x 6000 630, 107.  Activations then take at most 16 KiB of LDS.
  const bool fits = F % 4 == 0 && d <= 384 && F <= 8 * d && nq <= 8 * d;
  return fits && head_bytes <= (512u << 10) && layer_bytes <= (1280u << 10);
}
// A row's heads share one compute unit here, eight at a time, and have one wavefront each across the chip as launches of their own: past some
// length that is worth the launches, past a greater one where many rows share the chip anyway.  us per iteration of two layers at 1, 24,
// 96, 200 rows, separate launches / this: 4 heads of 32 of 500 tokens 98, 113, 124, 137 / 81, 95, 95, 96, of 1200 136, 161, 171, 231 / 144,
// 146, 148, 189, of 3000 239, 274, 357, - / 276, 281, 354, -; 8 of 32 of 160 tokens 80, 89, 106, 120 / 66, 77, 77, 79, of 500 100, 118, 131, 181
// / 106, 109, 107, 144, of 1200 141, 162, 219, 282 / 169, 173, 217, 240; 16 of 32 of 160 79, 88, 103, 120 / 79, 82, 90, 90, of 500 99, 113,
// 133, 167 / 132, 148, 149, 150; 12 of 64 of 32 tokens 80, 89, 104, 121 / 72, 76, 83, 85, of 160 93, 106, 127, 147 / 107, 121, 124, 124, of
// 500 126, 150, 173, 243 / 206, 229, 228, 269.  Beyond 256 rows a compute unit has two: 310 rows of 32, 160, 500 tokens, 4 heads of 32, 114,
// 125, 173 / 106, 129, 204.
int forward_f32_ctx(int nq, bool many_rows) { return (81920 / nq < 1024 ? 81920 / nq : 1024) * (many_rows ? 3 : 1); }
bool forward_f32_pays(int rows, int ctx, int nq) { return rows <= 256 && ctx <= forward_f32_ctx(nq, rows >= 128); }
void launch_forward_f32(hipStream_t st, RowCtx rc, Slots s, F32Model m, float* logits, Ctrl* ctrl, bool greedy, float temperature) {
  const int nq = m.n_q_heads * m.kvl.head_dim, nqkv = nq + 2 * m.kvl.n_kv_heads * m.kvl.head_dim;
  m.lds_floats = (int)forward_f32_lds(m.d, m.F, nq, nqkv);
  const size_t lds = ((size_t)m.lds_floats + s.max_blocks) * sizeof(float);
#define FWD_F32(DH) hipLaunchKernelGGL((forward_f32_kernel<DH>), dim3(rc.max_rows), dim3(ROW_THREADS), lds, st, rc, s, m, logits, ctrl, greedy ? 1 : 0, temperature)
  switch (m.kvl.head_dim) {
    case 32: FWD_F32(32); break;
    case 64: FWD_F32(64); break;
    default: FWD_F32(128); break;
  }
#undef FWD_F32
}

}  // namespace april
