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

enum { EPI_F32 = 0, EPI_SWIGLU = 1, EPI_LOGITS = 2, EPI_RESID = 3 };

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
  GroupOut go;           // EPI_LOGITS: group records
};

constexpr int KW4 = 4;       // wavefronts of a workgroup (template parameter KW); they split the k range among themselves

// One workgroup: NT weight tiles x MTC activation tiles over k-tiles [k0, k1).  Each of
// the KW wavefronts accumulates a quarter of the k range, the partial accumulators are
// summed through LDS in a fixed tree order, wavefront 0 runs the epilogue.
template <int NT, int MTC, int EPI, bool INTRA, int KW, int KH>
__device__ inline void gemm_group(const bf16x8* __restrict__ w0, const bf16x8* __restrict__ w1,
                                  const bf16x8* __restrict__ x, int KT, int k0, int k1, int nt0, int mt0,
                                  int rows, int N, float* __restrict__ out, bf16_t* __restrict__ act,
                                  float* red, float* ssp, const NormFuse& nf) {
  // KH k-tiles per fetch group, two groups in registers (4 VGPRs per fragment).  The next group is
  // requested before the MFMAs of the current one, so a wavefront whose k range fits in two
  // groups has all of it in flight at once, and a longer range streams with one group always in
  // flight behind the arithmetic.
  // the wavefront index is uniform: keep it (and the k range derived from it) in scalar registers
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  f32x16 acc[NT][MTC];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < MTC; ++j) acc[i][j] = f32x16{};

  const bf16x8* wp[NT];
  if (EPI == EPI_SWIGLU) {
    wp[0] = w0 + (size_t)nt0 * KT * 64 + lane;
    if (NT > 1) wp[NT - 1] = w1 + (size_t)nt0 * KT * 64 + lane;
  } else {
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      int nt = nt0 + i;
      if (EPI == EPI_LOGITS && nt >= (N >> 5)) nt = (N >> 5) - 1;   // vocabulary of an odd number of tiles: read, never written
      wp[i] = w0 + (size_t)nt * KT * 64 + lane;
    }
  }
  const bf16x8* xp[MTC];
#pragma unroll
  for (int j = 0; j < MTC; ++j) xp[j] = x + (size_t)(mt0 + j) * KT * 64 + lane;

  const int len = k1 - k0;
  const int kb = INTRA ? k0 + (int)((long long)len * wave / KW) : k0;
  const int ke = INTRA ? k0 + (int)((long long)len * (wave + 1) / KW) : k1;
  // A group past the end re-reads the final k-tile (loads stay unconditional and in flight
  // together) and skips its MFMAs.
  bf16x8 a[2][KH][NT], b[2][KH][MTC];
  auto fetch = [&](int g, int kt) {
#pragma unroll
    for (int u = 0; u < KH; ++u) {
      const size_t k = (size_t)(kt + u < ke ? kt + u : ke - 1) * 64;
#pragma unroll
      for (int i = 0; i < NT; ++i) a[g][u][i] = wp[i][k];
#pragma unroll
      for (int j = 0; j < MTC; ++j) b[g][u][j] = xp[j][k];
    }
  };
  auto multiply = [&](int g, int kt) {
#pragma unroll
    for (int u = 0; u < KH; ++u) {
      if (kt + u < ke) {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
          for (int j = 0; j < MTC; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[g][u][i], b[g][u][j], acc[i][j], 0, 0, 0);
      }
    }
  };
  // Fused norm (consumer side): wavefront w adds the slabs w, w + KW, ... of its rows, wavefront
  // 0 later adds the four sums.  The first 8 slabs per wavefront are requested here and summed
  // after the k loop, so their latency hides behind the operand stream.
  constexpr bool NORM_IN = (EPI == EPI_SWIGLU || EPI == EPI_F32) && INTRA;
  float sq[NORM_IN ? MTC : 1][8];
  if (NORM_IN && nf.ssq != nullptr) {
#pragma unroll
    for (int j = 0; j < MTC; ++j) {
      const float* col = nf.ssq + (mt0 + j) * 32 + (lane & 31);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int t = wave + u * KW;
        sq[j][u] = col[(size_t)(t < nf.n_ssq ? t : nf.n_ssq - 1) * nf.ssq_stride];
      }
    }
  }
  if (kb < ke) {
    fetch(0, kb);
    for (int kt = kb; kt < ke; kt += 2 * KH) {
      fetch(1, kt + KH);
      __builtin_amdgcn_sched_barrier(0);        // both groups requested before the first MFMA waits
      multiply(0, kt);
      if (kt + 2 * KH < ke) fetch(0, kt + 2 * KH);
      __builtin_amdgcn_sched_barrier(0);
      multiply(1, kt + KH);
    }
  }

  if (NORM_IN && nf.ssq != nullptr) {
#pragma unroll
    for (int j = 0; j < MTC; ++j) {
      float sacc = 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (wave + u * KW < nf.n_ssq) sacc += sq[j][u];
      const float* col = nf.ssq + (mt0 + j) * 32 + (lane & 31);
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
  // Reduction over the KW wavefronts through LDS, and the split of the epilogue: every wavefront
  // publishes its partial tiles, then wavefront w adds the KW partials of activation tile j = w
  // in wavefront order (0 + 1 + 2 + 3) and runs the epilogue of that tile, so up to KW tiles are
  // finished in parallel.  One weight tile per round: the buffer holds KW x MTC accumulator tiles.
  constexpr int NREG = MTC * 16;
  constexpr int JT = INTRA ? 1 : MTC;           // activation tiles this wavefront finishes
  f32x16 res[NT][JT];
  if (INTRA) {
    static_assert(!INTRA || MTC <= KW, "one activation tile per wavefront");
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      if (i > 0) __syncthreads();               // everyone has read the previous round
      float* dst = red + (size_t)wave * NREG * 64 + lane;
#pragma unroll
      for (int jq = 0; jq < MTC; ++jq)
#pragma unroll
        for (int e = 0; e < 16; ++e) dst[(jq * 16 + e) * 64] = acc[i][jq][e];
      __syncthreads();
      if (wave < MTC) {
        const float* src = red + (size_t)wave * 16 * 64 + lane;      // tile j = wave of wavefront 0's slab
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          float v = src[e * 64];
#pragma unroll
          for (int w = 1; w < KW; ++w) v += src[(size_t)w * NREG * 64 + e * 64];
          res[i][0][e] = v;
        }
      }
    }
    if (wave >= MTC) return;
  } else {
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int jq = 0; jq < JT; ++jq) res[i][jq] = acc[i][jq];
  }
  const int j0 = INTRA ? wave : 0;              // first (INTRA: only) activation tile of this wavefront

  const int mloc = lane & 31, nhalf = (lane >> 5) << 2;
  if (EPI == EPI_LOGITS) {
    // per row: the record of this wavefront's 64 output columns - maximum, its column, sum of
    // exponentials.  With those the greedy sampler and its log-probabilities need no logits at all.
    const bool two = nt0 + 1 < (N >> 5);
#pragma unroll
    for (int jq = 0; jq < JT; ++jq) {
      float bv;
      int bn;
      double s = 0.0;
      group64_record(res[0][jq], res[NT - 1][jq], two, nhalf, nf.go.sum != nullptr, nf.go.inv_t, bv, bn, s);
      const int m = (mt0 + j0 + jq) * 32 + mloc;
      if (m < rows && lane < 32) {
        const size_t gi = (size_t)m * ((N + 63) >> 6) + (nt0 >> 1);
        nf.go.max[gi] = bv;
        if (nf.go.col) nf.go.col[gi] = bn;
        if (nf.go.sum) nf.go.sum[gi] = s;
      }
    }
  }
  if (EPI == EPI_F32 || (EPI == EPI_LOGITS && out != nullptr)) {
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      if (EPI == EPI_LOGITS && nt0 + i >= (N >> 5)) continue;
#pragma unroll
      for (int jq = 0; jq < JT; ++jq) {
        const int j = j0 + jq;
        const int m = (mt0 + j) * 32 + mloc;
        float inv = 1.0f;
        if (NORM_IN && nf.ssq != nullptr) {          // fused norm: a k-split partial scales like the sum
          float ssum = ssp[j * 32 + mloc];
#pragma unroll
          for (int w = 1; w < KW; ++w) ssum += ssp[(w * MTC + j) * 32 + mloc];
          inv = 1.0f / sqrtf(ssum * nf.inv_d + nf.eps);
        }
        if (m < rows) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int n = (nt0 + i) * 32 + 8 * q + nhalf;
            f32x4 v = {res[i][jq][4 * q] * inv, res[i][jq][4 * q + 1] * inv, res[i][jq][4 * q + 2] * inv, res[i][jq][4 * q + 3] * inv};
            *reinterpret_cast<f32x4*>(out + (size_t)m * N + n) = v;
          }
        }
      }
    }
  } else if (EPI == EPI_RESID) {
    // out = residual stream (updated in place), act = gain-scaled bf16 copy for the next GEMM
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int jq = 0; jq < JT; ++jq) {
        const int m = (mt0 + j0 + jq) * 32 + mloc;
        float ss = 0.f;
        if (m < rows) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int n = (nt0 + i) * 32 + 8 * q + nhalf;
            float* xr = out + (size_t)m * N + n;
            f32x4 v = *reinterpret_cast<const f32x4*>(xr);
            const f32x4 gn = *reinterpret_cast<const f32x4*>(nf.gain + n);
            bf16x4 h;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              v[e] += res[i][jq][4 * q + e];
              ss += v[e] * v[e];
              h[e] = (bf16_t)(v[e] * gn[e]);
            }
            *reinterpret_cast<f32x4*>(xr) = v;
            *reinterpret_cast<bf16x4*>(act + act_index<true>(m, n, N)) = h;
          }
        }
        ss += __shfl_xor(ss, 32, 64);
        if (m < rows && lane < 32) nf.ssq[(size_t)(nt0 + i) * nf.ssq_stride + m] = ss;
      }
  } else if (EPI == EPI_SWIGLU) {
    // acc[0] = gate tile, acc[1] = up tile of features [nt0*32, nt0*32+32); N is F here.
#pragma unroll
    for (int jq = 0; jq < JT; ++jq) {
      const int j = j0 + jq;
      const int m = (mt0 + j) * 32 + mloc;
      float inv = 1.0f;
      if (INTRA && nf.ssq != nullptr) {
        float ssum = ssp[j * 32 + mloc];
#pragma unroll
        for (int w = 1; w < KW; ++w) ssum += ssp[(w * MTC + j) * 32 + mloc];
        inv = 1.0f / sqrtf(ssum * nf.inv_d + nf.eps);
      }
      if (m < rows) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int f = nt0 * 32 + 8 * q + nhalf;
          bf16x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float g = res[0][jq][4 * q + e] * inv, u = res[NT - 1][jq][4 * q + e] * inv;
            v[e] = (bf16_t)silu_mul(g, u);
          }
          *reinterpret_cast<bf16x4*>(act + act_index<true>(m, f, N)) = v;
        }
      }
    }
  }
}

// INTRA: the 4 wavefronts of a workgroup split the k range of one n-tile group (few n-tiles, or
// fused SwiGLU); otherwise each wavefront owns its own n-tile group.  KH: k-tiles per fetch group, OCC:
// workgroups per compute unit the registers are cut for.  No template argument but EPI changes a bit.
// Grids.  NEAR (1-D): the m-groups of one weight tile re-read that tile, so they are placed 8
// workgroup ids apart: same XCD (ids are dealt to the 8 XCDs in turn), same moment, one HBM read:
// id = ((tile / 8) * m_groups + m_group) * 8 + tile % 8.  Else x = k slice (F32) or n-tile group, y = the
// other, z = m-group: consecutive workgroups go to consecutive XCDs, so with 8 (4) slices every XCD
// works on one (two) k slices and pulls only that slice of the activations into its L2.
constexpr int fetch_depth(int kh, int full, int part) { return part >= full ? kh : (kh * full / part < 8 ? kh * full / part : 8); }
// k-tiles that a wavefront with `len` of them requests in fetch groups of kh: groups go in pairs, the last one past the end too.
__device__ inline int fetched(int len, int kh) { return (len + 2 * kh - 1) / (2 * kh) * (2 * kh); }
template <int NT, int MT, int EPI, bool INTRA, int KH, int OCC, bool NEAR>
__global__ __launch_bounds__(64 * KW4, OCC) void gemm_mfma_kernel(RowCtx rc, const bf16x8* __restrict__ x,
                                                                  const bf16x8* __restrict__ w0,
                                                                  const bf16x8* __restrict__ w1, float* __restrict__ out,
                                                                  bf16_t* __restrict__ act, int N, int K, int ksplit,
                                                                  size_t partial_stride, NormFuse nf) {
  constexpr int KW = KW4;
  __shared__ float red[INTRA ? KW * MT * 16 * 64 : 1];
  __shared__ float ssp[(INTRA && (EPI == EPI_SWIGLU || EPI == EPI_F32)) ? KW * MT * 32 : 1];
  const int rows = rows_or_zero(rc);
  constexpr bool SLICES = INTRA && EPI == EPI_F32;
  int bgrp = SLICES ? blockIdx.y : blockIdx.x, bz = blockIdx.z;
  const int sidx = SLICES ? blockIdx.x : 0;
  if (NEAR) {
    const int m_groups = ceil_div(ceil_div(rc.max_rows, 32), MT);
    const int rem = (int)blockIdx.x % (8 * m_groups);
    bgrp = ((int)blockIdx.x / (8 * m_groups)) * 8 + (rem & 7);
    bz = rem >> 3;
  }
  const int mt0 = bz * MT;
  if (mt0 * 32 >= rows) return;
  const int KT = K >> 4;
  const int grp = INTRA ? bgrp : bgrp * KW + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nt0 = (EPI == EPI_SWIGLU) ? grp : grp * NT;
  if (nt0 >= (N >> 5)) return;
  const int k0 = (int)((long long)KT * sidx / ksplit), k1 = (int)((long long)KT * (sidx + 1) / ksplit);
  float* o = out ? out + sidx * partial_stride : nullptr;
  int mtc = ceil_div(rows, 32) - mt0;
  if (mtc > MT) mtc = MT;
  // A last group of fewer m-tiles fetches more k-tiles at once in the same registers.  The 2 x 4 tile of the split-k
  // projections has room for one more: used where less is then requested past the slice's end (16 k-tiles per wavefront
  // and 64 rows: groups of 8 fetch 16, groups of 7 fetch 28; 2048 x 8192 in 8 slices 11.5 against 12.4 us per launch).
  constexpr bool ONE_MORE = EPI == EPI_F32 && NT == 2 && OCC == 1;
  const int per = (k1 - k0 + KW - 1) / KW;
#define GROUP(MTC, DEPTH) gemm_group<NT, (MT >= MTC ? MTC : 1), EPI, INTRA, KW, DEPTH>(w0, w1, x, KT, k0, k1, nt0, mt0, rows, N, o, act, red, ssp, nf)
  constexpr int D1 = fetch_depth(KH, NT + MT, NT + 1), D2 = fetch_depth(KH, NT + MT, NT + 2), D3 = fetch_depth(KH, NT + MT, NT + 3);
  switch (mtc) {
    case 1: GROUP(1, D1); break;
    case 2:
      if (ONE_MORE && fetched(per, D2 + 1) < fetched(per, D2)) GROUP(2, D2 + (ONE_MORE ? 1 : 0));
      else GROUP(2, D2);
      break;
    case 3:
      if (ONE_MORE && fetched(per, D3 + 1) < fetched(per, D3)) GROUP(3, D3 + (ONE_MORE ? 1 : 0));
      else GROUP(3, D3);
      break;
    default: GROUP(MT, KH); break;
  }
#undef GROUP
}

// Split-k projections (qkv, down).  What bounds them: a compute unit alone pulls about 50 GB/s from
// HBM, so the launch wants every unit busy with the same amount; beyond that the re-reads, the
// activations once per n-tile group and the weights once per m-group, at L2 speed.  So the tile of a
// workgroup grows with the rows.  us per launch, N x K in ksplit slices (rows: one side / the other):
//   * one n-tile (two workgroups per unit) where two give less than half a workgroup per unit: 1152 x 896 in 4
//     at 64 rows 4.3 / 2 x 4 tiles 6.1.
//   * up to 128 rows 2 x 4, the weights once: 4096 x 14336 in 4 at 128 rows 33.5 / 2 x 3 in two m-groups 37.9.
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
// Against two n-tiles x four m-tiles for all: 4096 x 14336 in 4 slices at 160, 192, 256, 384 rows 50.7, 51.5, 55.2, 79.3 /
// 36.4, 38.7, 43.3, 66.3; 2560 x 9728 in 6: 26.9, 28.3, 32.3, 46.0 / 21.7, 22.9, 26.0, 39.1.
void launch_gemm_mfma(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, float* out, int N, int K,
                      int ksplit, size_t partial_stride, const float* ssq, int ssq_stride, float eps) {
  const NormFuse nf{nullptr, const_cast<float*>(ssq), ssq_stride, K >> 5, 1.0f / (float)K, eps, {}};
  const int n_tiles = N >> 5, m_tiles = ceil_div(rc.max_rows, 32), slice = K / ksplit, per_group = n_tiles / 4 * ksplit;
  const bool quads = n_tiles % 4 == 0, long_slices = quads && slice >= 1536;
  auto round_tiles = [&](int mt) { return ceil_div(ceil_div(m_tiles, mt) * per_group, 256) * mt; };
#define GEMM_F32(NT, MT, KH, OCC)                                                                                       \
  hipLaunchKernelGGL((gemm_mfma_kernel<NT, MT, EPI_F32, true, KH, OCC, false>),                                         \
                     dim3(ksplit, n_tiles / NT, ceil_div(m_tiles, MT)), dim3(64 * KW4), 0, st, rc,                      \
                     reinterpret_cast<const bf16x8*>(x), reinterpret_cast<const bf16x8*>(Wp), nullptr, out, nullptr, N, \
                     K, ksplit, partial_stride, nf)
  if (n_tiles % 2 != 0 || (n_tiles / 2) * ksplit < 128) GEMM_F32(1, 4, 3, 2);
  else if (m_tiles <= 4 || (m_tiles == 5 && long_slices && per_group <= 96)) GEMM_F32(2, 4, 5, 1);
  else if (m_tiles <= 6 && long_slices) GEMM_F32(4, 3, 3, 1);
  else if ((m_tiles == 7 || m_tiles == 8) && quads && slice >= 1024) GEMM_F32(4, 4, 2, 1);
  else if (!long_slices || (m_tiles <= 12 && per_group < 112)) GEMM_F32(2, 3, 3, 2);
  else if (m_tiles <= 12 || round_tiles(3) < round_tiles(4)) GEMM_F32(4, 3, 3, 1);
  else GEMM_F32(4, 4, 2, 1);
#undef GEMM_F32
}

int lmhead_group_cols() { return 64; }

void launch_gemm_mfma_logits(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, float* logits,
                             const GroupOut& go, int V, int K) {
  constexpr int MT = 4;
  const int n_tiles = V >> 5;
  dim3 grid(ceil_div(ceil_div(n_tiles, 2), KW4), 1, ceil_div(ceil_div(rc.max_rows, 32), MT));
  hipLaunchKernelGGL((gemm_mfma_kernel<2, MT, EPI_LOGITS, false, 5, 1, false>), grid, dim3(64 * KW4), 0, st, rc,
                     reinterpret_cast<const bf16x8*>(x), reinterpret_cast<const bf16x8*>(Wp), nullptr, logits, nullptr,
                     V, K, 1, (size_t)0, NormFuse{nullptr, nullptr, 0, 0, 0.f, 0.f, go});
}

// Fused gate/up, rows below what the LDS-tiled kernel takes (see forward()).  Workgroups of few row tiles
// at three (two) per compute unit: an MLP of 9728 features is 304 workgroups, which at one per unit ran in two
// rounds.  us per launch, four m-tiles at one per unit / as here: 2560 x 9728 at 32, 64, 96 rows 30.7,
// 37.3, 42.5 / 27.3, 32.8, 35.1, at 320, 384 rows 74.2, 81.1 / 59.4, 69.0; 4096 x 14336 at 32, 64 rows
// 48.4, 57.1 / 45.5, 53.5; 896 x 4864 at 64, 96, 192, 256 rows 9.9, 11.1, 15.2, 20.1 / 9.9, 10.2, 12.6, 14.8.
// NEAR where the weight tiles alone are more than a round of one workgroup per unit, and where their number is no multiple
// of 8, which in grid order puts the row groups of one tile on different XCDs: 3104 x 1184 (97 tiles) at 160, 256, 512 rows
// 12.6, 14.7, 24.9 / 10.6, 11.3, 17.5; 4864 x 896 (152 tiles) at 160, 256, 512 rows 10.6, 13.2, 18.8, NEAR 10.9, 14.6, 20.5.
void launch_gemm_mfma_swiglu(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wg, const bf16_t* Wu,
                             bf16_t* act, int F, int K, const float* ssq, int ssq_stride, float eps) {
  const int n_tiles = F >> 5, m_tiles = ceil_div(rc.max_rows, 32);
  NormFuse nf{nullptr, const_cast<float*>(ssq), ssq_stride, K >> 5, 1.0f / (float)K, eps, {}};
#define GEMM_SW(MT, KH, OCC, NEAR, grid)                                                                               \
  hipLaunchKernelGGL((gemm_mfma_kernel<2, MT, EPI_SWIGLU, true, KH, OCC, NEAR>), grid, dim3(64 * KW4), 0, st, rc,      \
                     reinterpret_cast<const bf16x8*>(x), reinterpret_cast<const bf16x8*>(Wg),                          \
                     reinterpret_cast<const bf16x8*>(Wu), nullptr, act, F, K, 1, (size_t)0, nf)
  const int tiles8 = ceil_div(n_tiles, 8) * 8;
  if (m_tiles <= 1) GEMM_SW(1, 4, 3, false, dim3(n_tiles));
  else if (n_tiles <= 256 && (m_tiles <= 2 || n_tiles % 8 == 0)) GEMM_SW(2, 2, 3, false, dim3(n_tiles, 1, ceil_div(m_tiles, 2)));
  else if (n_tiles <= 256 || m_tiles <= 3) GEMM_SW(2, 2, 3, true, dim3(tiles8 * ceil_div(m_tiles, 2)));
  else GEMM_SW(3, 3, 2, true, dim3(tiles8 * ceil_div(m_tiles, 3)));
#undef GEMM_SW
}

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
  const NormFuse nf{gain, ssq, ssq_stride, 0, 0.f, 0.f, {}};
#define GEMM_RESID(NT, MT, KH, OCC)                                                                                     \
  hipLaunchKernelGGL((gemm_mfma_kernel<NT, MT, EPI_RESID, true, KH, OCC, true>),                                        \
                     dim3(ceil_div(n_tiles / NT, 8) * 8 * ceil_div(m_tiles, MT)), dim3(64 * KW4), 0, st, rc,            \
                     reinterpret_cast<const bf16x8*>(x), reinterpret_cast<const bf16x8*>(Wp), nullptr, x_res, act, N, K, \
                     1, (size_t)0, nf)
  const int most = 256 / n_tiles > 0 ? 256 / n_tiles : 1;                // groups of rows
  const int groups = ceil_div(m_tiles, ceil_div(m_tiles, most));
  int mt = ceil_div(m_tiles, most);
  while (mt < 4 && (groups > 1 || mt != 3) && ceil_div(m_tiles, mt + 1) == groups) ++mt;
  if (groups == m_tiles || (groups == 1 && m_tiles == 3 && n_tiles * 3 <= 512)) mt = 1;
  const int pairs = ceil_div(n_tiles / 2, 8) * ceil_div(m_tiles, 3), singles = ceil_div(n_tiles, 8) * ceil_div(m_tiles, 4);   // workgroups per XCD
  if (mt > 4 && (n_tiles % 2 != 0 || (m_tiles > 8 && pairs > 32 && singles >= 48 && singles <= 64))) mt = 4;
  if (mt == 1) GEMM_RESID(1, 1, 8, 1);
  else if (mt == 2) GEMM_RESID(1, 2, 4, 2);
  else if (mt == 3) GEMM_RESID(1, 3, 4, 2);
  else if (mt == 4) GEMM_RESID(1, 4, 3, 2);
  else GEMM_RESID(2, 3, 4, 1);
#undef GEMM_RESID
}

}  // namespace april
