// bf16 MFMA GEMM for skinny (decode) and tall (prefill) activations, gfx950.
//
// out[m][n] = sum_k x[m][k] * W[n][k].  Both operands are kept in the register
// layout of v_mfma_f32_32x32x16_bf16's 32x16 operand ("fragment-tiled"), so a
// wavefront fetches one fragment as 64 consecutive 16-byte pieces (1 KiB, fully
// coalesced) straight into VGPRs: the weight stream - the only HBM-sized traffic
// of a decode GEMM - is read exactly once, with no LDS staging.  The weight tile is
// the MFMA's A operand (rows = output features), the activation tile its B operand
// (columns = batch rows), so the accumulator holds out^T tiles:
//   lane l, register i  ->  n = 8*(i/4) + 4*(l/32) + i%4,  m = l%32.
#include "kernels.h"

namespace april {

__global__ __launch_bounds__(256) void shuffle_weights_kernel(const bf16_t* src, bf16x8* dst, int N, int K) {
  const size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x;      // 16-byte piece index
  const size_t total = (size_t)N * K / 8;
  if (c >= total) return;
  const int KT = K >> 4;
  const size_t tile = c >> 6;
  const int lane = (int)(c & 63);
  const int nt = (int)(tile / KT), kt = (int)(tile % KT);
  const int row = nt * 32 + (lane & 31), k = kt * 16 + ((lane >> 5) << 3);
  dst[c] = *reinterpret_cast<const bf16x8*>(src + (size_t)row * K + k);
}
void launch_shuffle_weights(hipStream_t st, const bf16_t* src, bf16_t* dst, int N, int K) {
  const size_t total = (size_t)N * K / 8;
  hipLaunchKernelGGL(shuffle_weights_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, src,
                     reinterpret_cast<bf16x8*>(dst), N, K);
}

enum { EPI_F32 = 0, EPI_SWIGLU = 1, EPI_RESID = 2 };

// RMSNorm folded into the GEMMs around it (decode).  The producer (EPI_RESID, the attention
// output projection) adds its result to the residual stream in place, writes the residual times
// the next norm's gain as the bf16 activations of the next GEMM, and leaves per row the sum of
// squares of its 32 columns (ssq[n_tile][row]).  The consumer (EPI_SWIGLU with ssq set) sums
// those partials in a fixed order and scales its accumulators by 1/sqrt(mean square + eps):
// W . (x g / rms) = (W . (x g)) / rms.  No separate normalisation launch in between.
struct NormFuse {
  const float* gain;     // producer: gain of the following norm [N]
  float* ssq;            // producer: out; consumer: in.  nullptr = not fused
  int ssq_stride;        // rows per n-tile slab
  int n_ssq;             // consumer: number of slabs (= d_model / 32)
  float inv_d, eps;      // consumer
};

constexpr int KW4 = 4;       // wavefronts of a workgroup (template parameter KW); they split the k range among themselves

// The products of one wavefront: NT weight tiles x MTC activation tiles over k-tiles [kb, ke), one accumulator
// chain per element in ascending k.  D k-tiles are in flight in registers (4 VGPRs per fragment): a slot is
// requested again as soon as its products are issued, every load unconditional (past the end the last k-tile once more),
// so the wait counts are static.  `early` requests what the epilogue wants, behind the first D k-tiles.
template <int NT, int MTC, int D, class Early>
__device__ __forceinline__ void accumulate(const bf16x8* const (&wp)[NT], const bf16x8* const (&xp)[MTC], int kb, int ke,
                                           f32x16 (&acc)[NT][MTC], Early early) {
  bf16x8 a[D][NT], b[D][MTC];
  auto fetch = [&](int u, int kt) {
    const size_t k = (size_t)(kt < ke ? kt : ke - 1) * 64;
#pragma unroll
    for (int i = 0; i < NT; ++i) a[u][i] = wp[i][k];
#pragma unroll
    for (int j = 0; j < MTC; ++j) b[u][j] = xp[j][k];
  };
  auto multiply = [&](int u) {
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < MTC; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[u][i], b[u][j], acc[i][j], 0, 0, 0);
  };
  if (kb >= ke) { early(); return; }
#pragma unroll
  for (int u = 0; u < D; ++u) fetch(u, kb + u);
  early();
  __builtin_amdgcn_sched_barrier(0);            // all of it requested before the first product waits
  int kt = kb;
  for (; kt + D < ke; kt += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      multiply(u);
      fetch(u, kt + D + u);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int u = 0; u < D; ++u)
    if (kt + u < ke) multiply(u);
}

// One workgroup of the k-splitting kernels: NT weight tiles x MTC activation tiles over k-tiles [k0, k1).  Each of
// the KW wavefronts accumulates a quarter of the k range; the partial accumulators meet in LDS, in wavefront order
// ((0 + 1) + 2) + 3, and wavefront w finishes the registers 4 w .. 4 w + 3 of every tile: four 16-byte LDS reads
// per tile and lane, and a quarter of the epilogue each.  HALF (gate/up): the tile's rows are 16 gate and 16 up features.
template <int NT, int MTC, int EPI, int KW, int D, bool HALF>
__device__ inline void gemm_group(const bf16x8* __restrict__ w0, const bf16x8* __restrict__ w1,
                                  const bf16x8* __restrict__ x, int KT, int k0, int k1, int nt0, int mt0,
                                  int rows, int N, float* __restrict__ out, bf16_t* __restrict__ act,
                                  f32x4* red, float* ssp, const NormFuse& nf) {
  static_assert(KW == 4 && MTC <= 4, "one register quarter per wavefront");
  // the wavefront index is uniform: keep it (and the k range derived from it) in scalar registers
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int mloc = lane & 31, nhalf = (lane >> 5) << 2;
  f32x16 acc[NT][MTC];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < MTC; ++j) acc[i][j] = f32x16{};

  const bf16x8* wp[NT];
  if (HALF) {
    wp[0] = (mloc < 16 ? w0 : w1) + (size_t)(nt0 >> 1) * KT * 64 + ((nt0 & 1) * 16 + (mloc & 15) + (lane & 32));
  } else if (EPI == EPI_SWIGLU) {
    wp[0] = w0 + (size_t)nt0 * KT * 64 + lane;
    if (NT > 1) wp[NT - 1] = w1 + (size_t)nt0 * KT * 64 + lane;
  } else {
#pragma unroll
    for (int i = 0; i < NT; ++i) wp[i] = w0 + (size_t)(nt0 + i) * KT * 64 + lane;
  }
  // (columns past the last row repeat it: never written, and a few rows then cost a few cache lines)
  const bf16x8* xp[MTC];
  int mrow[MTC];                                // this lane's row of every tile
#pragma unroll
  for (int j = 0; j < MTC; ++j) {
    mrow[j] = min((mt0 + j) * 32 + mloc, rows - 1);
    xp[j] = x + (size_t)(mt0 + j) * KT * 64 + ((mrow[j] & 31) | (lane & 32));
  }
  const int len = k1 - k0;
  const int kb = k0 + (int)((long long)len * wave / KW), ke = k0 + (int)((long long)len * (wave + 1) / KW);

  // Fused norm (consumer side): wavefront w adds the slabs w, w + KW, ... of its rows; the four sums are
  // added later.  The first 8 slabs per wavefront are requested behind the first operands.
  constexpr bool NORM_IN = EPI == EPI_SWIGLU || EPI == EPI_F32;
  float sq[NORM_IN ? MTC : 1][8];
  // residual epilogue: this lane's residual values and gains
  f32x4 xr[EPI == EPI_RESID ? NT : 1][EPI == EPI_RESID ? MTC : 1], gn[EPI == EPI_RESID ? NT : 1];
  auto early = [&]() {
    if (NORM_IN && nf.ssq != nullptr) {
#pragma unroll
      for (int j = 0; j < MTC; ++j)
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int t = wave + u * KW;
          sq[j][u] = nf.ssq[(size_t)(t < nf.n_ssq ? t : nf.n_ssq - 1) * nf.ssq_stride + mrow[j]];
        }
    }
    if (EPI == EPI_RESID) {
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        const int n = (nt0 + i) * 32 + 8 * wave + nhalf;
        gn[i] = *reinterpret_cast<const f32x4*>(nf.gain + n);
#pragma unroll
        for (int j = 0; j < MTC; ++j) xr[i][j] = *reinterpret_cast<const f32x4*>(out + (size_t)mrow[j] * N + n);
      }
    }
  };
  accumulate<NT, MTC, D>(wp, xp, kb, ke, acc, early);

  if (NORM_IN && nf.ssq != nullptr) {
#pragma unroll
    for (int j = 0; j < MTC; ++j) {
      float sacc = 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (wave + u * KW < nf.n_ssq) sacc += sq[j][u];
      const float* col = nf.ssq + mrow[j];
      // wide models have more than 8 slabs per wavefront: the rest in groups of 8 independent loads
      for (int t0 = wave + 8 * KW; t0 < nf.n_ssq; t0 += 8 * KW) {
        float more[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int t = t0 + u * KW;
          more[u] = col[(size_t)(t < nf.n_ssq ? t : nf.n_ssq - 1) * nf.ssq_stride];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (t0 + u * KW < nf.n_ssq) sacc += more[u];
      }
      if (lane < 32) ssp[(wave * MTC + j) * 32 + lane] = sacc;
    }
  }
  // res[i][j]: registers 4 wave .. 4 wave + 3 of tile (i, j); HALF: wavefronts 0 and 1 also take the up
  // features, registers 4 (wave + 2) .., in up[j]
  f32x4 res[NT][MTC], up[HALF ? MTC : 1];
  constexpr bool ONE = NT * MTC <= 2;           // every tile in one round, else one weight tile per round
  constexpr int TILES = (ONE ? NT : 1) * MTC;   // tiles of a round
  auto sum4 = [&](int t, int q) {
    const f32x4* src = red + (size_t)(t * 4 + q) * 64 + lane;
    f32x4 v = src[0];
#pragma unroll
    for (int w = 1; w < KW; ++w) v += src[(size_t)w * TILES * 4 * 64];
    return v;
  };
#pragma unroll
  for (int i0 = 0; i0 < NT; i0 += ONE ? NT : 1) {
    if (i0 > 0) __syncthreads();                // everyone has read the previous round
#pragma unroll
    for (int i = i0; i < (ONE ? NT : i0 + 1); ++i)
#pragma unroll
      for (int j = 0; j < MTC; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          red[((size_t)wave * TILES + (i - i0) * MTC + j) * 256 + q * 64 + lane] =
              f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
    __syncthreads();
#pragma unroll
    for (int i = i0; i < (ONE ? NT : i0 + 1); ++i)
#pragma unroll
      for (int j = 0; j < MTC; ++j) {
        if (HALF && wave >= 2) continue;
        res[i][j] = sum4((i - i0) * MTC + j, wave);
        if (HALF) up[j] = sum4(j, wave + 2);
      }
  }
  if (HALF && wave >= 2) return;

  float inv[MTC];
  if (NORM_IN) {
#pragma unroll
    for (int j = 0; j < MTC; ++j) {
      inv[j] = 1.0f;
      if (nf.ssq != nullptr) {                  // fused norm: a k-split partial scales like the sum
        float ssum = ssp[j * 32 + mloc];
#pragma unroll
        for (int w = 1; w < KW; ++w) ssum += ssp[(w * MTC + j) * 32 + mloc];
        inv[j] = 1.0f / sqrtf(__fmaf_rn(ssum, nf.inv_d, nf.eps));
      }
    }
  }
  if (EPI == EPI_F32) {
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < MTC; ++j) {
        const int m = (mt0 + j) * 32 + mloc;
        if (m < rows) *reinterpret_cast<f32x4*>(out + (size_t)m * N + (nt0 + i) * 32 + 8 * wave + nhalf) = res[i][j] * inv[j];
      }
  } else if (EPI == EPI_RESID) {
    // out = residual stream (updated in place), act = gain-scaled bf16 copy for the next GEMM
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      float ss[MTC];
#pragma unroll
      for (int j = 0; j < MTC; ++j) {
        const int m = (mt0 + j) * 32 + mloc, n = (nt0 + i) * 32 + 8 * wave + nhalf;
        const f32x4 v = xr[i][j] + res[i][j];
        bf16x4 h;
        ss[j] = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          ss[j] = __fmaf_rn(v[e], v[e], ss[j]);      // (explicit: no instance may choose another contraction)
          h[e] = (bf16_t)(v[e] * gn[i][e]);
        }
        if (m < rows) {
          *reinterpret_cast<f32x4*>(out + (size_t)m * N + n) = v;
          *reinterpret_cast<bf16x4*>(act + act_index<true>(m, n, N)) = h;
        }
        ss[j] += __shfl_xor(ss[j], 32, 64);
        if (lane < 32) ssp[((i * KW + wave) * MTC + j) * 32 + lane] = ss[j];
      }
    }
    // sum of squares of a row's 32 columns: the wavefronts' 8 columns each, in order
    __syncthreads();
    for (int t = threadIdx.x; t < NT * MTC * 32; t += 64 * KW) {
      const int i = t / (MTC * 32), jm = t % (MTC * 32), m = mt0 * 32 + jm;
      float s = ssp[i * KW * MTC * 32 + jm];
#pragma unroll
      for (int w = 1; w < KW; ++w) s += ssp[(i * KW + w) * MTC * 32 + jm];
      if (m < rows) nf.ssq[(size_t)(nt0 + i) * nf.ssq_stride + m] = s;
    }
  } else {
    // gate features in res[0] (HALF: of this tile's 16), up features in res[NT - 1] (up); N is F here
#pragma unroll
    for (int j = 0; j < MTC; ++j) {
      const int m = (mt0 + j) * 32 + mloc, f = nt0 * (HALF ? 16 : 32) + 8 * wave + nhalf;
      bf16x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float g = res[0][j][e] * inv[j], u = (HALF ? up[HALF ? j : 0][e] : res[NT - 1][j][e]) * inv[j];
        v[e] = (bf16_t)silu_mul(g, u);
      }
      if (m < rows) *reinterpret_cast<bf16x4*>(act + act_index<true>(m, f, N)) = v;
    }
  }
}

// The 4 wavefronts of a workgroup split the k range of one n-tile group.  D: k-tiles in flight with MT m-tiles, OCC:
// workgroups per compute unit the registers are cut for.  No template argument but EPI changes a bit.
// Grids.  NEAR (1-D): the m-groups of one weight tile re-read that tile, so they are placed 8
// workgroup ids apart: same XCD (ids are dealt to the 8 XCDs in turn), same moment, one HBM read:
// id = ((tile / 8) * m_groups + m_group) * 8 + tile % 8.  Else x = k slice (F32) or n-tile group, y = the
// other, z = m-group: consecutive workgroups go to consecutive XCDs, so with 8 (4) slices every XCD
// works on one (two) k slices and pulls only that slice of the activations into its L2.
// The leading arguments are what the first loads need: the compiler has them preloaded in scalar registers
// (a chain of launches that read 8 MB each: 3.24 -> 2.88 us per launch).
constexpr int ring_depth(int d, int full, int part) { return d * full / part < 16 ? d * full / part : 16; }
template <int NT, int MT, int EPI, int D, int OCC, bool NEAR, bool HALF>
__global__ __launch_bounds__(64 * KW4, OCC) void gemm_mfma_kernel(const int2* __restrict__ ctl, const bf16x8* __restrict__ x,
                                                                  const bf16x8* __restrict__ w0,
                                                                  const bf16x8* __restrict__ w1, float* __restrict__ out,
                                                                  int max_rows, int N, int K, int ksplit,
                                                                  bf16_t* __restrict__ act, size_t partial_stride, NormFuse nf) {
  constexpr int KW = KW4;
  constexpr int ROUND = NT * MT <= 2 ? NT * MT : (MT > 2 ? MT : 2);       // accumulator tiles that meet in LDS at once
  __shared__ f32x4 red[KW * ROUND * 4 * 64];
  __shared__ float ssp[(EPI == EPI_RESID ? NT : 1) * KW * MT * 32];
  const int2 cv = *ctl;
  const int rows = cv.y ? 0 : cv.x;             // none once the scheduler has ended the step
  constexpr bool SLICES = EPI == EPI_F32;
  int bgrp = SLICES ? blockIdx.y : blockIdx.x, bz = blockIdx.z;
  const int sidx = SLICES ? blockIdx.x : 0;
  if (NEAR) {
    const int m_groups = ceil_div(ceil_div(max_rows, 32), MT);
    const int rem = (int)blockIdx.x % (8 * m_groups);
    bgrp = ((int)blockIdx.x / (8 * m_groups)) * 8 + (rem & 7);
    bz = rem >> 3;
  }
  const int mt0 = bz * MT;
  if (mt0 * 32 >= rows) return;
  const int KT = K >> 4;
  const int nt0 = (EPI == EPI_SWIGLU) ? bgrp : bgrp * NT;
  if (nt0 >= (HALF ? N >> 4 : N >> 5)) return;
  const int k0 = (int)((long long)KT * sidx / ksplit), k1 = (int)((long long)KT * (sidx + 1) / ksplit);
  float* o = out ? out + sidx * partial_stride : nullptr;
  int mtc = ceil_div(rows, 32) - mt0;
  if (mtc > MT) mtc = MT;
#define GROUP(MTC, DEPTH) gemm_group<NT, (MT >= MTC ? MTC : 1), EPI, KW, DEPTH, HALF>(w0, w1, x, KT, k0, k1, nt0, mt0, rows, N, o, act, red, ssp, nf)
  constexpr int D1 = ring_depth(D, NT + MT, NT + 1), D2 = ring_depth(D, NT + MT, NT + 2), D3 = ring_depth(D, NT + MT, NT + 3);
  const int per = (k1 - k0 + KW - 1) / KW;
  // A last group of fewer m-tiles has more k-tiles in flight in the same registers; a short range, or one that D
  // does not divide, fewer (what is requested past its end costs L1 bandwidth: 20 k-tiles 4.3 us with 16, 3.7 with 10).
  auto asked = [&](int d) { return (per + d - 1) / d * d; };
  switch (mtc) {
    case 1:
      if (per <= 4) GROUP(1, (D1 < 4 ? D1 : 4));
      else if (per <= 7) GROUP(1, (D1 < 7 ? D1 : 7));
      else if (per <= 10 || asked(10) < asked(D1)) GROUP(1, (D1 < 10 ? D1 : 10));
      else GROUP(1, D1);
      break;
    case 2:
      if (per <= 4) GROUP(2, (D2 < 4 ? D2 : 4));
      else if (per <= 7) GROUP(2, (D2 < 7 ? D2 : 7));
      else GROUP(2, D2);
      break;
    case 3:
      if (MT == 3 && D == 5 && asked(4) < asked(5)) GROUP(3, 4);
      else GROUP(3, D3);
      break;
    default: GROUP(MT, D); break;
  }
#undef GROUP
}

// LM head: each wavefront owns two weight tiles (64 columns, one record group) and all of k.
constexpr int LM_MT = 4, LM_D = 10;
template <int MTC, int D>
__device__ inline void logits_group(const bf16x8* __restrict__ w0, const bf16x8* __restrict__ x, int KT, int nt0, int mt0,
                                    int rows, int N, float* __restrict__ out, const GroupOut& go) {
  const int lane = threadIdx.x & 63, mloc = lane & 31, nhalf = (lane >> 5) << 2;
  f32x16 acc[2][MTC];
  const bf16x8 *wp[2], *xp[MTC];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int nt = nt0 + i < (N >> 5) ? nt0 + i : (N >> 5) - 1;       // vocabulary of an odd number of tiles: read, never written
    wp[i] = w0 + (size_t)nt * KT * 64 + lane;
  }
#pragma unroll
  for (int j = 0; j < MTC; ++j) {
    acc[0][j] = acc[1][j] = f32x16{};
    xp[j] = x + (size_t)(mt0 + j) * KT * 64 + ((min((mt0 + j) * 32 + mloc, rows - 1) & 31) | (lane & 32));
  }
  accumulate<2, MTC, D>(wp, xp, 0, KT, acc, [] {});
  // per row: the record of this wavefront's 64 output columns - maximum, its column, sum of
  // exponentials.  With those the greedy sampler and its log-probabilities need no logits at all.
  const bool two = nt0 + 1 < (N >> 5);
#pragma unroll
  for (int j = 0; j < MTC; ++j) {
    float bv;
    int bn;
    double s = 0.0;
    group64_record(acc[0][j], acc[1][j], two, nhalf, go.sum != nullptr, go.inv_t, bv, bn, s);
    const int m = (mt0 + j) * 32 + mloc;
    if (m >= rows) continue;
    if (lane < 32) {
      const size_t gi = (size_t)m * ((N + 63) >> 6) + (nt0 >> 1);
      go.max[gi] = bv;
      if (go.col) go.col[gi] = bn;
      if (go.sum) go.sum[gi] = s;
    }
    if (out == nullptr) continue;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if (nt0 + i >= (N >> 5)) continue;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<f32x4*>(out + (size_t)m * N + (nt0 + i) * 32 + 8 * q + nhalf) =
            f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
    }
  }
}
__global__ __launch_bounds__(64 * KW4, 1) void gemm_logits_kernel(const int2* __restrict__ ctl, const bf16x8* __restrict__ x,
                                                                  const bf16x8* __restrict__ w, float* __restrict__ out,
                                                                  int N, int K, GroupOut go) {
  const int2 cv = *ctl;
  const int rows = cv.y ? 0 : cv.x, mt0 = blockIdx.z * LM_MT;
  if (mt0 * 32 >= rows) return;
  const int nt0 = ((int)blockIdx.x * KW4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * 2, KT = K >> 4;
  if (nt0 >= (N >> 5)) return;
  const int mtc = ceil_div(rows, 32) - mt0;
  if (mtc == 1) logits_group<1, ring_depth(LM_D, 2 + LM_MT, 3)>(w, x, KT, nt0, mt0, rows, N, out, go);
  else if (mtc == 2) logits_group<2, ring_depth(LM_D, 2 + LM_MT, 4)>(w, x, KT, nt0, mt0, rows, N, out, go);
  else if (mtc == 3) logits_group<3, ring_depth(LM_D, 2 + LM_MT, 5)>(w, x, KT, nt0, mt0, rows, N, out, go);
  else logits_group<LM_MT, LM_D>(w, x, KT, nt0, mt0, rows, N, out, go);
}

// Split-k projections (qkv, down).  What bounds them: at few rows the latency of one pass (first loads, LDS, epilogue);
// then a compute unit alone pulls about 50 GB/s from HBM, so the launch wants every unit busy with the same amount;
// beyond that the re-reads, the activations once per n-tile group and the weights once per m-group, at L2 speed.  So the
// tile of a workgroup grows with the rows.  us per launch, N x K in ksplit slices (rows: one side / the other):
//   * matrices below 8 M elements: single tiles at three workgroups per unit up to 64 rows and, where
//     they are at most 300 per m-tile, 128; then 1 x 2.  1152 x 896 in 4 at 96 rows 3.3 / 1 x 4 4.1, 896 x 4864 in 8 at 96, 128
//     rows 6.1, 6.8 / 1 x 2 6.4, 7.6, 1792 x 1184 in 6 (336) at 96 rows 5.0 / 1 x 2 4.7, 2 x 4 7.0.  Beyond 128 rows pairs:
//     2 x 2 for slices below 512, else 2 x 3: 1792 x 1184 at 192 rows 6.1 / 7.0, 896 x 4864 8.7 / 7.9.
//   * odd n-tile counts from about 6 M elements on: one n-tile, and the more m-tiles the fewer workgroups re-read the weights and
//     the activations; per m-tile of 256 workgroups and more the narrow tile still fills the units at 96 and 128 rows.  At 128, 192,
//     384 rows, 1 x 1 or 1 x 2 of small matrices / as here: 6176 x 4096 in 1 37.1, 34.6, 56.2 / 23.8, 31.9, 48.4; 4128 x 14336 in 2 78.0,
//     74.7, 127 / 59.2, 71.3, 107; 2592 x 9728 in 4 26.1, 31.8, 52.9 / 25.1, 31.2, 48.0; 3104 x 2048 in 3 11.1, 12.3, 19.6 / 10.4, 12.4,
//     16.7; 64 rows of 6176 x 4096 20.5 / 17.1.  1 x 4 for all: 23.8, 32.1, 48.4; 72.3, 71.6, 107; 29.6, 33.1, 48.0; 11.5, 12.1, 16.7.
//   * larger ones, up to 64 rows 2 x 2 at two workgroups per unit: 6144 x 2560 in 2 at 32, 64 rows 9.1, 11.1 / 2 x 4 9.8, 11.9.
//     96 and 128 rows 2 x 3: 12.4, 14.3 / 2 x 4 13.7, 15.0; but 2 x 4 for 128 rows of long slices that fill the units by
//     themselves: 4096 x 14336 in 4 33.3 / 2 x 3 40.1.
//   * slices below 1536 (few k-tiles per wavefront do not pay for the wider reduction): 2 x 3 at two workgroups
//     per unit.  Slices of 1280 at 160 rows 17.8 / 4 x 3 18.5, of 1621 22.4 / 21.7; of 1024 at 288, 512 rows 24.9,
//     38.4 / 30.8, 45.0.  For 7 and 8 m-tiles 4 x 4 down to slices of 1024: 19.5 / 22.5 (682: 16.5 / 16.5).
//   * longer slices, weights once: 4 x 3 to 192 rows, 4 x 4 to 256 (4096 x 14336: 38.7 / 2 x 3 45.5, 43.3 / 60.5).
//     Except 5 m-tiles over at most 96 workgroups of 4 n-tiles, where the units left over take the fifth m-tile beside
//     2 x 4: 6144 x 4096 in 2 21.8 / 23.6 (4096 x 14336 in 4, 128 workgroups: 50.7 / 36.4).
//   * 257-384 rows: 4 x 3 from 112 workgroups per m-group, else 2 x 3: 7168 x 5120 in 2 (112) at 320 rows 46.2 / 49.5,
//     6144 x 4096 in 2 (96) 34.5 / 41.6.
//   * beyond: 4 x 4 or 4 x 3, whichever has fewer m-tiles in its rounds of one workgroup per unit: 4096 x 14336 in 4
//     at 512, 1024 rows 77, 144 / 94, 171; 10240 x 8192 in 1 at 512 rows 4 x 3 116 / 4 x 4 133.
// Fetch groups of k-tiles in alternation, a reduction that one wavefront per m-tile finished, epilogue operands requested after
// it and no preloaded arguments / as here, at 1, 32, 96 rows: 1152 x 896 3.5, 3.7, 4.1 / 2.7, 2.9, 3.3; 1792 x 1184 5.8, 5.9, 8.0 /
// 3.6, 4.0, 5.0; 6144 x 2560 10.6, 10.8, 14.3 / 8.3, 9.1, 12.4; 2560 x 9728 12.7, 12.9, 16.9 / 11.2, 11.7, 15.2.
void launch_gemm_mfma(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, float* out, int N, int K,
                      int ksplit, size_t partial_stride, const float* ssq, int ssq_stride, float eps) {
  const NormFuse nf{nullptr, const_cast<float*>(ssq), ssq_stride, K >> 5, 1.0f / (float)K, eps};
  const int n_tiles = N >> 5, m_tiles = ceil_div(rc.max_rows, 32), slice = K / ksplit, per_group = n_tiles / 4 * ksplit;
  const bool quads = n_tiles % 4 == 0, long_slices = quads && slice >= 1536;
  auto round_tiles = [&](int mt) { return ceil_div(ceil_div(m_tiles, mt) * per_group, 256) * mt; };
#define GEMM_F32(NT, MT, D, OCC)                                                                                        \
  hipLaunchKernelGGL((gemm_mfma_kernel<NT, MT, EPI_F32, D, OCC, false, false>),                                         \
                     dim3(ksplit, n_tiles / NT, ceil_div(m_tiles, MT)), dim3(64 * KW4), 0, st, rc.ctl,                  \
                     reinterpret_cast<const bf16x8*>(x), reinterpret_cast<const bf16x8*>(Wp), nullptr, out,             \
                     rc.max_rows, N, K, ksplit, nullptr, partial_stride, nf)
  const bool pairs = n_tiles % 2 == 0, small = (long long)N * K < (8ll << 20);
  if (!pairs && m_tiles > 1 && (long long)N * K >= (m_tiles <= 4 ? 6ll << 20 : 5ll << 20) && (m_tiles > 2 || n_tiles > 128)) {
    if (m_tiles == 2) GEMM_F32(1, 2, 8, 3);
    else if (m_tiles <= 4 && n_tiles * ksplit >= 256) GEMM_F32(1, 2, 10, 2);
    else if (m_tiles == 5 || m_tiles == 6) GEMM_F32(1, 3, 8, 2);
    else GEMM_F32(1, 4, 6, 2);
  } else if (!pairs || (small && m_tiles <= 4)) {
    if (m_tiles <= 2 || (m_tiles <= 4 && n_tiles * ksplit <= 300)) GEMM_F32(1, 1, 12, 3);
    else GEMM_F32(1, 2, 8, 3);
  } else if (m_tiles <= 2 || (small && slice < 512)) GEMM_F32(2, 2, 6, 2);
  else if ((m_tiles == 4 && slice >= 1536 && (n_tiles / 2) * ksplit >= 224) || (m_tiles == 5 && long_slices && per_group <= 96)) GEMM_F32(2, 4, 10, 1);
  else if (m_tiles <= 4 || small) GEMM_F32(2, 3, 5, 2);
  else if (m_tiles <= 6 && long_slices) GEMM_F32(4, 3, 6, 1);
  else if ((m_tiles == 7 || m_tiles == 8) && quads && slice >= 1024) GEMM_F32(4, 4, 4, 1);
  else if (!long_slices || (m_tiles <= 12 && per_group < 112)) GEMM_F32(2, 3, 5, 2);
  else if (m_tiles <= 12 || round_tiles(3) < round_tiles(4)) GEMM_F32(4, 3, 6, 1);
  else GEMM_F32(4, 4, 4, 1);
#undef GEMM_F32
}

int lmhead_group_cols() { return 64; }

void launch_gemm_mfma_logits(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, float* logits,
                             const GroupOut& go, int V, int K) {
  dim3 grid(ceil_div(ceil_div(V >> 5, 2), KW4), 1, ceil_div(ceil_div(rc.max_rows, 32), LM_MT));
  hipLaunchKernelGGL(gemm_logits_kernel, grid, dim3(64 * KW4), 0, st, rc.ctl, reinterpret_cast<const bf16x8*>(x),
                     reinterpret_cast<const bf16x8*>(Wp), logits, V, K, go);
}

// Fused gate/up, rows below what the LDS-tiled kernel takes (see forward()).  Row tiles and workgroups per unit so that the
// launch comes close to one even round over the 256 units.  us per launch, F x K (rows: one side / the other):
//   * one m-tile: tiles of 16 gate and 16 up features where whole ones fill at most half of a round, the first or the last:
//     3104 x 1184 (97 tiles) at 1, 32 rows 5.5, 6.1 / 6.9, 7.6; 9728 x 2560 (304) at 1, 16, 32 rows 21.3, 22.1, 25.0 / 23.5, 24.0,
//     25.6; where whole ones fill more, the activations read twice as often cost more: 5120 x 4096 (160) 21.5, 25.9 / 18.7, 21.2.
//   * several m-tiles that together are no more than a round: one each.  3072 x 2048 (96) at 64 rows 9.8 / 2 x 2 12.4.
//   * 96 rows of more than 192 tiles, 128 of more than 152 (to 256): 2 x 3, whose first group alone is the round and takes all or most of
//     the rows.  2 x 2 / 2 x 3 at 96 rows: 8192 x 3072 31.5 / 25.3, 6432 x 2048 (201 tiles) 18.5 / 17.3, 5120 x 4096 (160) 25.1 / 29.9; at 128:
//     5120 x 4096 32.3 / 28.5, 5152 x 2560 (161, NEAR) 25.6 / 24.2, 7712 x 4096 (241, NEAR) 41.2 / 38.7, 4864 x 896 (152) 9.1 / 9.1.
//   * else 2 x 2: 4864 x 896 at 64 rows two workgroups per unit 8.1 / three 8.7.  Four m-tiles at one per unit against
//     three: 9728 x 2560 at 64, 96 rows 37.3, 42.5 / 30.7, 33.4.
// NEAR where the weight tiles alone are more than a round of one workgroup per unit, and where their number is no multiple
// of 8, which in grid order puts the row groups of one tile on different XCDs: 3104 x 1184 (97 tiles) at 160, 256, 512 rows
// 12.6, 14.7, 24.9 / 10.6, 11.3, 17.5; 4864 x 896 (152 tiles) at 160, 256, 512 rows 10.6, 13.2, 18.8, NEAR 10.9, 14.6, 20.5.
// Before the kernel's ring, quarter epilogues and preloaded arguments / now, at 1, 32, 64 rows: 4864 x 896 7.5, 7.5, 8.9 / 5.8, 6.3,
// 7.8; 3104 x 1184 8.8, 8.8, 10.5 / 5.4, 6.1, 7.7; 9728 x 2560 26.6, 26.6, 31.8 / 21.2, 24.9, 30.7 (a plain read of its 100 MB: 18).
void launch_gemm_mfma_swiglu(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wg, const bf16_t* Wu,
                             bf16_t* act, int F, int K, const float* ssq, int ssq_stride, float eps) {
  const int n_tiles = F >> 5, m_tiles = ceil_div(rc.max_rows, 32);
  NormFuse nf{nullptr, const_cast<float*>(ssq), ssq_stride, K >> 5, 1.0f / (float)K, eps};
#define GEMM_SW(NT, MT, D, OCC, NEAR, grid)                                                                            \
  hipLaunchKernelGGL((gemm_mfma_kernel<NT, MT, EPI_SWIGLU, D, OCC, NEAR, NT == 1>), grid, dim3(64 * KW4), 0, st,       \
                     rc.ctl, reinterpret_cast<const bf16x8*>(x), reinterpret_cast<const bf16x8*>(Wg),                  \
                     reinterpret_cast<const bf16x8*>(Wu), nullptr, rc.max_rows, F, K, 1, act, (size_t)0, nf)
  const int tiles8 = ceil_div(n_tiles, 8) * 8, wgs = n_tiles * m_tiles;
  if (wgs <= 128 || (m_tiles == 1 && (n_tiles - 1) % 256 < 128)) GEMM_SW(1, 1, 10, 3, false, dim3(2 * n_tiles, 1, m_tiles));
  else if (m_tiles == 1 || (m_tiles <= 8 && wgs <= 256)) GEMM_SW(2, 1, 8, 3, false, dim3(n_tiles, 1, m_tiles));
  else if (n_tiles <= 256 && ((m_tiles == 3 && n_tiles > 192) || (m_tiles == 4 && n_tiles > 152 && n_tiles % 8 == 0)))
    GEMM_SW(2, 3, 5, 2, false, dim3(n_tiles, 1, ceil_div(m_tiles, 3)));
  else if (n_tiles <= 256 && m_tiles == 4 && n_tiles > 152) GEMM_SW(2, 3, 5, 2, true, dim3(2 * tiles8));
  else if (m_tiles <= 2 && n_tiles <= 256) GEMM_SW(2, 2, 8, 2, false, dim3(n_tiles));
  else if (n_tiles <= 256 && n_tiles % 8 == 0) GEMM_SW(2, 2, 4, 3, false, dim3(n_tiles, 1, ceil_div(m_tiles, 2)));
  else if (n_tiles <= 256 || m_tiles <= 3) GEMM_SW(2, 2, 4, 3, true, dim3(tiles8 * ceil_div(m_tiles, 2)));
  else GEMM_SW(2, 3, 5, 2, true, dim3(tiles8 * ceil_div(m_tiles, 3)));
#undef GEMM_SW
}

// (before the epilogue's operands were requested with the first k-tiles / now, at 1, 32, 96 rows: 896 x 896 4.0, 4.0, 4.0 /
// 3.3, 3.5, 3.6; 1184 x 1280 6.4, 6.4, 6.3 / 3.7, 4.1, 4.1; 2560 x 4096 12.2, 12.2, 11.4 / 8.8, 11.4, 10.9)
// x_res += x . W^T (whole k range per workgroup, no partials); act = bf16(x_res * gain) in the
// fragment order of the next GEMM; ssq[n_tile][row] = sum of squares of the tile's 32 columns.
// As many workgroups as fit one per compute unit (256): few rows per workgroup where there are few
// n-tiles; of the row tiles that give that number of groups the largest (two groups of 3 + 1
// m-tiles are faster than 2 + 2: 14.8 against 17.0 us).  us per launch before (one m-tile up to 512 workgroups,
// else four) / as here: 2560 x 4096 at 128, 160, 256 rows 17.9, 17.2, 23.5 / 14.8, 14.5, 18.3;
// 4096 x 4096 at 96, 128, 256, 320, 384 rows 18.6, 18.8, 24.5, 35.2, 43.0 / 15.4, 16.0, 24.5, 21.2, 24.2.
// Where even one group leaves more than a third of the units idle, three m-tiles go one to a workgroup if that is at
// most two per unit: 5120 x 5120 (160 n-tiles) at 96 rows 23.4 (one group of 3: 26.2), 5632 x 5632 (176) 31.0 (28.9).
// Rows that need more than 4 m-tiles per group: 2 x 3 at one workgroup per unit, unless that takes a second round on some
// XCD where 1 x 4 at two per unit fills most of one: 5120 x 5120 at 288, 320, 384, 448 rows 2 x 3 31.1, 47.4, 55.2, 51.9,
// 1 x 4 36.9, 40.8, 49.2, 55.9; 896 x 896 at 1536, 2048 rows 10.3, 17.1 and 12.4, 13.9.
void launch_gemm_mfma_resid(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, float* x_res,
                            const float* gain, bf16_t* act, float* ssq, int ssq_stride, int N, int K) {
  const int n_tiles = N >> 5, m_tiles = ceil_div(rc.max_rows, 32);
  const NormFuse nf{gain, ssq, ssq_stride, 0, 0.f, 0.f};
#define GEMM_RESID(NT, MT, D, OCC)                                                                                      \
  hipLaunchKernelGGL((gemm_mfma_kernel<NT, MT, EPI_RESID, D, OCC, true, false>),                                        \
                     dim3(ceil_div(n_tiles / NT, 8) * 8 * ceil_div(m_tiles, MT)), dim3(64 * KW4), 0, st, rc.ctl,        \
                     reinterpret_cast<const bf16x8*>(x), reinterpret_cast<const bf16x8*>(Wp), nullptr, x_res,           \
                     rc.max_rows, N, K, 1, act, (size_t)0, nf)
  const int most = 256 / n_tiles > 0 ? 256 / n_tiles : 1;                // groups of rows
  const int groups = ceil_div(m_tiles, ceil_div(m_tiles, most));
  int mt = ceil_div(m_tiles, most);
  while (mt < 4 && (groups > 1 || mt != 3) && ceil_div(m_tiles, mt + 1) == groups) ++mt;
  if (groups == m_tiles || (groups == 1 && m_tiles == 3 && n_tiles * 3 <= 512)) mt = 1;
  const int pairs = ceil_div(n_tiles / 2, 8) * ceil_div(m_tiles, 3), singles = ceil_div(n_tiles, 8) * ceil_div(m_tiles, 4);   // workgroups per XCD
  if (mt > 4 && (n_tiles % 2 != 0 || (m_tiles > 8 && pairs > 32 && singles >= 48 && singles <= 64))) mt = 4;
  if (mt == 1) GEMM_RESID(1, 1, 16, 1);
  else if (mt == 2) GEMM_RESID(1, 2, 8, 2);
  else if (mt == 3) GEMM_RESID(1, 3, 8, 2);
  else if (mt == 4) GEMM_RESID(1, 4, 6, 2);
  else GEMM_RESID(2, 3, 8, 1);
#undef GEMM_RESID
}

}  // namespace april
