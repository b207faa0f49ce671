// Routed mixture of SwiGLU experts (bf16, gfx950): router soft-max + top-k, token ->
// expert dispatch lists, grouped expert GEMMs on v_mfma_f32_32x32x16_bf16.
//
// Per token: r = softmax over all E router logits; the top_k largest r (ties: lower
// expert index) are kept and renormalised to sum 1; y = sum_k w_k * expert_k(h), added to
// the residual stream in the fixed order k = 0..top_k-1 (descending r) by the following
// add/RMSNorm kernel, so the result does not depend on where a token lands in an expert's
// batch.
#include "kernels.h"

namespace april {

// ---------------------------------------------------------------------------
// Router: one wavefront per row.  logits = sum of split-K partials [n_partials][rows][E].  A chain of top_k arg-max steps: they run
// on the DPP lanes (twelve shuffles through the LDS unit per step were most of the kernel).  128 experts, 8 per token, under a kernel
// trace: at 160-240 rows 9.0 -> 5.9 us, at 13 900 rows 31 -> 22.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void moe_route_kernel(RowCtx rc, const float* logits, int n_partials,
                                                       size_t partial_stride, int E, int top_k, int* ids,
                                                       float* wts) {
  const int r = blockIdx.x;
  ROW_GUARD(rc, r);
  const int lane = threadIdx.x;
  // up to 256 experts: 4 per lane
  float v[4];
  float mx = -INFINITY;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int e = lane + 64 * j;
    // up to 8 partials (the split-k bound) requested together, added in order
    float part[8], a = -INFINITY;
#pragma unroll
    for (int p = 0; p < 8; ++p) part[p] = logits[min(p, n_partials - 1) * partial_stride + (size_t)r * E + min(e, E - 1)];
    if (e < E) {
      a = 0.f;
#pragma unroll
      for (int p = 0; p < 8; ++p) if (p < n_partials) a += part[p];
    }
    v[j] = a;
    mx = fmaxf(mx, a);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  float sum = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j) { v[j] = lane + 64 * j < E ? expf(v[j] - mx) : 0.f; sum += v[j]; }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] /= sum;
  // top_k by repeated arg-max (value desc, index asc)
  float kept = 0.f;
  float myw = 0.f;
  int myid = -1;
  for (int k = 0; k < top_k; ++k) {
    float lv = -1.f;
    int li = 0x7fffffff;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int e = lane + 64 * j;
      if (e < E && v[j] > lv) { lv = v[j]; li = e; }      // ascending e within the lane
    }
    const float bv = wave_max_f32(lv);
    const int bi = wave_min_i32(lv == bv ? li : 0x7fffffff);
    kept += bv;
    if (lane == k) { myw = bv; myid = bi; }
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = bi == lane + 64 * j ? -2.f : v[j];   // remove the winner
  }
  if (lane < top_k) {
    ids[(size_t)r * top_k + lane] = myid;
    wts[(size_t)r * top_k + lane] = myw / kept;
  }
}

void launch_moe_route(hipStream_t st, RowCtx rc, const float* logits, int n_partials, size_t partial_stride,
                      int E, int top_k, int* ids, float* wts) {
  hipLaunchKernelGGL(moe_route_kernel, dim3(rc.max_rows), dim3(64), 0, st, rc, logits, n_partials, partial_stride,
                     E, top_k, ids, wts);
}

// ---------------------------------------------------------------------------
// Dispatch: one workgroup.  cnt[e] = tokens routed to expert e; base[e] = first packed row
// of expert e, aligned to `align` rows (the rows one GEMM workgroup covers: whole MFMA tiles, and
// no workgroup straddles two experts); pos_of[row*top_k + k] = packed row of that assignment;
// src_row[packed row] = token row (-1 in the padding); group_expert[g] = expert that owns packed
// rows [g*align, (g+1)*align), -1 past the end.  The GEMMs launch one workgroup per (n-tile
// group, row group) of that flat list: with a (expert, row group of the expert) grid sized for
// the worst case, five of six workgroups of a decode launch - and nearly all of a prefill
// launch - found nothing to do after a dependent load.
// Placement inside an expert's batch is arbitrary (LDS atomics); values never depend on it.
// (One thread adding up the 128 segments was 5 of 15 us.)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void moe_dispatch_kernel(RowCtx rc, const int* ids, int E, int top_k, int* cnt,
                                                            int* base, int* pos_of, int* src_row, int p_cap,
                                                            Ctrl* ctrl, int align, int* group_expert, int n_groups) {
  __shared__ int s_cnt[256], s_base[257];
  const int rows = rows_or_zero(rc), tid = threadIdx.x;
  if (rows == 0) return;
  if (tid < 256) s_cnt[tid] = 0;
  __syncthreads();
  const int n = rows * top_k;
  for (int a = tid; a < n; a += 1024) atomicAdd(&s_cnt[ids[a]], 1);
  __syncthreads();
  if (tid < 64) {
    // exclusive prefix sum of the aligned segments: lane l owns experts 4 l .. 4 l + 3 (E <= 256)
    int own[4], sum = 0, hit = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n_e = 4 * tid + j < E ? s_cnt[4 * tid + j] : 0;
      own[j] = (n_e + align - 1) / align * align;
      sum += own[j];
      hit += n_e > 0;
    }
    int incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int o = __shfl_up(incl, off, 64);
      if (tid >= off) incl += o;
      hit += __shfl_xor(hit, off, 64);
    }
    int acc = incl - sum;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (4 * tid + j <= E) s_base[4 * tid + j] = acc;
      acc += own[j];
    }
    if (tid == 63 && E == 256) s_base[256] = acc;
    if (tid == 0 && ctrl != nullptr) ctrl->sum_experts += hit;
  }
  __syncthreads();
  const int total = s_base[E];
  for (int p = tid; p < total && p < p_cap; p += 1024) src_row[p] = -1;
  if (tid < E)
    for (int g = s_base[tid] / align; g < s_base[tid + 1] / align && g < n_groups; ++g) group_expert[g] = tid;
  for (int g = total / align + tid; g < n_groups; g += 1024) group_expert[g] = -1;
  if (tid < E) { cnt[tid] = s_cnt[tid]; base[tid] = s_base[tid]; s_cnt[tid] = 0; }
  if (tid == 0) base[E] = total;
  __syncthreads();
  for (int a = tid; a < n; a += 1024) {
    const int e = ids[a];
    const int p = s_base[e] + atomicAdd(&s_cnt[e], 1);
    pos_of[a] = p;
    if (p < p_cap) src_row[p] = a / top_k;
  }
}

// rows per GEMM workgroup (and alignment of the expert segments) for a launch over at most max_rows rows
int moe_group_rows(int max_rows, int tall_rows) { return max_rows >= tall_rows ? 128 : 64; }
// upper bound on the row groups of such a launch
int moe_group_count(int max_rows, int top_k, int E, int align) {
  return (int)(((long long)max_rows * top_k + (long long)E * (align - 1) + align - 1) / align);
}

void launch_moe_dispatch(hipStream_t st, RowCtx rc, const int* ids, int E, int top_k, int* cnt, int* base,
                         int* pos_of, int* src_row, int p_cap, Ctrl* ctrl, int tall_rows, int* group_expert) {
  const int align = moe_group_rows(rc.max_rows, tall_rows);
  hipLaunchKernelGGL(moe_dispatch_kernel, dim3(1), dim3(1024), 0, st, rc, ids, E, top_k, cnt, base, pos_of, src_row,
                     p_cap, ctrl, align, group_expert, moe_group_count(rc.max_rows, top_k, E, align));
}

// ---------------------------------------------------------------------------
// Grouped expert GEMMs.  grid: x = n-tile group inside the expert, y = row group of the flat
// packed list (MT m-tiles of one expert, see the dispatch kernel).  The 4 wavefronts of a
// workgroup split the k range (LDS reduction in wavefront order).
//   GATHER = true : the B operand rows are token rows looked up through src_row (gate/up);
//   GATHER = false: the B operand is the packed fragment-tiled activation (down).
// ---------------------------------------------------------------------------
// The weights are the traffic (1.2 GB of a layer of 128 experts of 3 x 768 x 2048, about ten rows each), so
// the kernel is cut for many workgroups per compute unit: a group that has rows for one m-tile only
// runs the one-tile body (half the registers of the two-tile one), k-tiles are fetched in two
// alternating groups, and token rows are gathered from a plain [row][K] copy - out of the
// fragment-tiled layout a gathered row uses 16 bytes of every 128-byte line it touches, which at ten rows
// was more traffic than the weights.  At 160-240 rows, 8 of those 128 experts per row: gate/up 169 -> 144 us
// (5.6 TB/s), down 107 -> 80 us (5.0 TB/s).
constexpr int MOE_KW = 4;

struct MoeArgs {
  const int* src_row;
  const bf16x8* x;
  const bf16x8 *w0, *w1;
  size_t w_expert_stride;
  float* out;
  bf16_t* act;
  int N, K;
};

template <int NT, int MTC, bool SWIGLU, int KH>
__device__ __forceinline__ void moe_group(const MoeArgs& ma, int e, int rows_e, int p0, int mt0, float* red) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int N = ma.N, KT = ma.K >> 4;
  const int nt0 = SWIGLU ? blockIdx.x : blockIdx.x * NT;
  f32x16 acc[NT][MTC];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < MTC; ++j) acc[i][j] = f32x16{};
  const bf16x8* wp[NT];
  const bf16x8* we0 = ma.w0 + (size_t)e * ma.w_expert_stride;
  if (SWIGLU) {
    wp[0] = we0 + (size_t)nt0 * KT * 64 + lane;
    wp[NT - 1] = ma.w1 + (size_t)e * ma.w_expert_stride + (size_t)nt0 * KT * 64 + lane;
  } else {
#pragma unroll
    for (int i = 0; i < NT; ++i) wp[i] = we0 + (size_t)(nt0 + i) * KT * 64 + lane;
  }
  // B operand: a token row of the plain activation copy (gathered per lane; a k-tile of a row is two
  // 16-byte pieces; rows past the expert's repeat its last one, never written), or the packed tile
  const bf16x8* xp[MTC];
  constexpr int XS = SWIGLU ? 2 : 64;
#pragma unroll
  for (int j = 0; j < MTC; ++j) {
    if (SWIGLU) {
      const int row = ma.src_row[p0 + min((mt0 + j) * 32 + (lane & 31), rows_e - 1)];
      xp[j] = ma.x + ((size_t)(row < 0 ? 0 : row) * KT * 2 + (lane >> 5));
    } else {
      xp[j] = ma.x + ((size_t)((p0 >> 5) + mt0 + j) * KT * 64 + lane);
    }
  }
  const int kb = (int)((long long)KT * wave / MOE_KW), ke = (int)((long long)KT * (wave + 1) / MOE_KW);
  bf16x8 a[2][KH][NT], b[2][KH][MTC];
  auto fetch = [&](int g, int kt) {
#pragma unroll
    for (int u = 0; u < KH; ++u) {
      const size_t k = (size_t)(kt + u < ke ? kt + u : ke - 1);
#pragma unroll
      for (int i = 0; i < NT; ++i) a[g][u][i] = wp[i][k * 64];
#pragma unroll
      for (int j = 0; j < MTC; ++j) b[g][u][j] = xp[j][k * XS];
    }
  };
  auto multiply = [&](int g, int kt) {
#pragma unroll
    for (int u = 0; u < KH; ++u)
      if (kt + u < ke) {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
          for (int j = 0; j < MTC; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[g][u][i], b[g][u][j], acc[i][j], 0, 0, 0);
      }
  };
  if (kb < ke) {
    fetch(0, kb);
    for (int kt = kb; kt < ke; kt += 2 * KH) {
      fetch(1, kt + KH);
      __builtin_amdgcn_sched_barrier(0);
      multiply(0, kt);
      if (kt + 2 * KH < ke) fetch(0, kt + 2 * KH);
      __builtin_amdgcn_sched_barrier(0);
      multiply(1, kt + KH);
    }
  }
  constexpr int NREG = NT * MTC * 16;
  if (wave != 0) {
    float* dst = red + (size_t)(wave - 1) * NREG * 64 + lane;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < MTC; ++j)
#pragma unroll
        for (int q = 0; q < 16; ++q) dst[((i * MTC + j) * 16 + q) * 64] = acc[i][j][q];
  }
  __syncthreads();
  if (wave != 0) return;
#pragma unroll
  for (int w = 0; w < MOE_KW - 1; ++w) {
    const float* src = red + (size_t)w * NREG * 64 + lane;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < MTC; ++j)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[i][j][q] += src[((i * MTC + j) * 16 + q) * 64];
  }
  const int mloc = lane & 31, nhalf = (lane >> 5) << 2;
#pragma unroll
  for (int j = 0; j < MTC; ++j) {
    const int ml = (mt0 + j) * 32 + mloc;            // row inside the expert's batch
    if (ml >= rows_e) continue;
    const int p = p0 + ml;                           // packed row
    if (SWIGLU) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int f = nt0 * 32 + 8 * q + nhalf;
        bf16x4 v;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float g = acc[0][j][4 * q + t], u = acc[NT - 1][j][4 * q + t];
          v[t] = (bf16_t)silu_mul(g, u);
        }
        *reinterpret_cast<bf16x4*>(ma.act + act_index<true>(p, f, N)) = v;
      }
    } else {
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int n = (nt0 + i) * 32 + 8 * q + nhalf;
          f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          *reinterpret_cast<f32x4*>(ma.out + (size_t)p * N + n) = v;
        }
    }
  }
}

// (fetch groups of 6 / 4 k-tiles at two workgroups per compute unit; 4 / 2 at three, 8 / 5 at two and 2 / 1 at
// four: within 3 %)
template <int NT, int MT, bool SWIGLU>
__global__ __launch_bounds__(64 * MOE_KW, MT > 2 ? 1 : 2) void moe_gemm_kernel(const int* stop, const int* cnt, const int* base,
                                                                     const int* __restrict__ group_expert, MoeArgs ma) {
  __shared__ float red[(MOE_KW - 1) * NT * MT * 16 * 64];
  if (stop != nullptr && *stop != 0) return;
  const int e = group_expert[blockIdx.y];
  if (e < 0) return;
  const int rows_e = cnt[e];
  const int p0 = base[e];                       // first packed row of this expert (multiple of MT * 32)
  const int mt0 = (int)blockIdx.y * MT - (p0 >> 5);   // first m-tile of this group inside the expert's batch
  if (mt0 * 32 >= rows_e) return;
  const int mtc = ((rows_e + 31) >> 5) - mt0;
  if (mtc == 1) moe_group<NT, 1, SWIGLU, 6>(ma, e, rows_e, p0, mt0, red);
  else if (MT == 2 || mtc == 2) moe_group<NT, 2, SWIGLU, MT == 2 ? 4 : 2>(ma, e, rows_e, p0, mt0, red);
  else if (mtc == 3) moe_group<NT, (MT > 2 ? 3 : 1), SWIGLU, 2>(ma, e, rows_e, p0, mt0, red);
  else moe_group<NT, MT, SWIGLU, 2>(ma, e, rows_e, p0, mt0, red);
}

template <bool SWIGLU>
static void launch_moe_gemm(hipStream_t st, RowCtx rc, int n_groups_x, int align, int top_k, int E, const int* cnt, const int* base,
                            const int* group_expert, const MoeArgs& ma) {
  dim3 grid(n_groups_x, moe_group_count(rc.max_rows, top_k, E, align));
  const int* stop = reinterpret_cast<const int*>(rc.ctl) + 1;
  if (align == 128) hipLaunchKernelGGL((moe_gemm_kernel<2, 4, SWIGLU>), grid, dim3(64 * MOE_KW), 0, st, stop, cnt, base, group_expert, ma);
  else hipLaunchKernelGGL((moe_gemm_kernel<2, 2, SWIGLU>), grid, dim3(64 * MOE_KW), 0, st, stop, cnt, base, group_expert, ma);
}

void launch_moe_gateup(hipStream_t st, RowCtx rc, const int* cnt, const int* base, const int* group_expert,
                       const int* src_row, const bf16_t* h_rows, const bf16_t* Wg, const bf16_t* Wu, bf16_t* act, int E,
                       int top_k, int Fe, int d, int tall_rows) {
  // tall batches (prefill): 4 m-tiles per workgroup, so an expert's weight tile is fetched half as
  // often; the summation chain of an output element does not depend on the grouping
  launch_moe_gemm<true>(st, rc, Fe >> 5, moe_group_rows(rc.max_rows, tall_rows), top_k, E, cnt, base, group_expert,
                        MoeArgs{src_row, reinterpret_cast<const bf16x8*>(h_rows), reinterpret_cast<const bf16x8*>(Wg),
                                reinterpret_cast<const bf16x8*>(Wu), (size_t)Fe * d / 8, nullptr, act, Fe, d});
}

void launch_moe_down(hipStream_t st, RowCtx rc, const int* cnt, const int* base, const int* group_expert,
                     const bf16_t* act, const bf16_t* Wd, float* out, int E, int top_k, int Fe, int d, int tall_rows) {
  launch_moe_gemm<false>(st, rc, (d >> 5) / 2, moe_group_rows(rc.max_rows, tall_rows), top_k, E, cnt, base, group_expert,
                         MoeArgs{nullptr, reinterpret_cast<const bf16x8*>(act), reinterpret_cast<const bf16x8*>(Wd), nullptr,
                                 (size_t)d * Fe / 8, out, nullptr, d, Fe});
}

}  // namespace april
