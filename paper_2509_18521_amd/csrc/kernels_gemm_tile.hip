// bf16 MFMA GEMM for tall activations (prefill: hundreds to thousands of rows), gfx950.
//
// out[m][n] = sum_k x[m][k] * W[n][k], same operand layouts as the skinny decode GEMM
// (both operands fragment-tiled for v_mfma_f32_32x32x16_bf16: one 32x16 fragment is 1 KiB of
// consecutive bytes), but compute-bound, so it is organised around operand reuse:
//   * a workgroup of WGM x WGN wavefronts owns a (WGM*MTW*32) x (WGN*NTW*32) output tile;
//     each wavefront keeps MTW x NTW accumulator tiles;
//   * the k loop advances in stages of BK k-tiles; the fragments of a stage go global -> LDS once
//     per workgroup (every fragment is one contiguous 1 KiB piece; LDS reads are lane-consecutive
//     16-byte pieces, conflict-free) while the MFMAs of earlier stages run from the ring's other
//     slots; one barrier per stage;
//   * every output element is one accumulator chain over k-tiles 0..K/16-1 in order, whatever
//     the tile shape or the number of rows: results do not depend on the batch.
// Every kernel here asks for K % 32 == 0, as april_init does of every inner dimension.
#include <algorithm>
#include <type_traits>

#include "kernels.h"

namespace april {

enum { TEPI_F32 = 0, TEPI_SWIGLU = 1, TEPI_LOGITS = 2, TEPI_RESID = 3, TEPI_QKV = 4 };   // RESID: out += result; LOGITS: F32 (optional) + records of 64-column groups

// Epilogue of one wavefront: accumulator tile = out^T (lane l, register e:
// n = 8*(e/4) + 4*(l/32) + e%4, m = l%32).  nt0: first weight tile (SwiGLU: first feature
// tile; acc[i] = gate, acc[i + NTW/2] = up), mt0: first activation tile.
template <int MTW, int NTW, int EPI>
__device__ inline void tile_epilogue(f32x16 (&acc)[NTW][MTW], int nt0, int mt0, int rows, int n_tiles, int N, int lane,
                                     float* __restrict__ out, bf16_t* __restrict__ act,
                                     const float* row_scale = nullptr, const GroupOut* go = nullptr) {
  const int mloc = lane & 31, nhalf = (lane >> 5) << 2;
  if (EPI == TEPI_LOGITS) {
    // a group is an aligned pair of weight tiles (nt0 even): this wavefront holds NTW / 2 of them
    static_assert(EPI != TEPI_LOGITS || NTW % 2 == 0, "64-column groups");
#pragma unroll
    for (int i = 0; i < NTW; i += 2) {
      if (nt0 + i >= n_tiles) continue;
      const bool two = nt0 + i + 1 < n_tiles;
#pragma unroll
      for (int j = 0; j < MTW; ++j) {
        float bv;
        int bn;
        double s = 0.0;
        group64_record(acc[i][j], acc[NTW > 1 ? i + 1 : 0][j], two, nhalf, go->sum != nullptr, go->inv_t, bv, bn, s);
        const int m = (mt0 + j) * 32 + mloc;
        if (m < rows && lane < 32) {
          const size_t gi = (size_t)m * ((N + 63) >> 6) + ((nt0 + i) >> 1);
          go->max[gi] = bv;
          if (go->col) go->col[gi] = bn;
          if (go->sum) go->sum[gi] = s;
        }
      }
    }
  }
  if (EPI == TEPI_F32 || EPI == TEPI_RESID || (EPI == TEPI_LOGITS && out != nullptr)) {
#pragma unroll
    for (int i = 0; i < NTW; ++i) {
      const int nt = nt0 + i;
      if (nt >= n_tiles) continue;
#pragma unroll
      for (int j = 0; j < MTW; ++j) {
        const int m = (mt0 + j) * 32 + mloc;
        if (m < rows) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int n = nt * 32 + 8 * q + nhalf;
            f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
            f32x4* o = reinterpret_cast<f32x4*>(out + (size_t)m * N + n);
            if (EPI == TEPI_RESID) v = *o + v;
            *o = v;
          }
        }
      }
    }
  } else if (EPI == TEPI_SWIGLU) {
    constexpr int H = NTW / 2;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const int ft = nt0 + i;
      if (ft >= n_tiles) continue;
#pragma unroll
      for (int j = 0; j < MTW; ++j) {
        const int m = (mt0 + j) * 32 + mloc;
        // folded RMSNorm (decode): the accumulators are scaled by the row's 1/rms first (this lane's row of every m-tile)
        const float inv = row_scale ? row_scale[j] : 1.0f;
        if (m < rows) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int f = ft * 32 + 8 * q + nhalf;
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float g = acc[i][j][4 * q + e] * inv, u = acc[i + H][j][4 * q + e] * inv;
              v[e] = (bf16_t)silu_mul(g, u);
            }
            *reinterpret_cast<bf16x4*>(act + act_index<true>(m, f, N)) = v;
          }
        }
      }
    }
  }
}

// Epilogue of the prefill QKV projection: rotary embedding of q and k, q to a bf16 row array, k and v to
// their pages - what a separate pass over the fp32 projection (rope_append_kernel) did, with the same
// operations.  Both members of a rotation pair sit in the same lane: a wavefront of 4 weight tiles holds whole heads (tiles
// i and i + DH / 64, or for DH = 32 registers e and e + 8), one of 2 tiles a head of 64, two of 32, or every other
// tile of a head of 128 (0 and 2, or 1 and 3).  qkv_tile: the weight tile i of the wavefront column wc.
// The separate pass took 232 us per 16384 rows of 32 + 2 x 8 heads of 128 (400 MB in, 335 MB out,
// bandwidth); with it and the residual additions of the two other projections (TEPI_RESID: the norm after
// them reads one array instead of two and writes none but its result, 130 -> 80 us) in the epilogues, prefill
// of 21 k tokens through three such layers went from 19.0 to 18.0 ms.
template <int NTW, int DH>
__device__ __forceinline__ int qkv_tile(int wc, int i) {
  static_assert(NTW == 4 || NTW == 2, "whole rotation pairs");
  return NTW * 32 < DH ? (wc >> 1) * 4 + (wc & 1) + 2 * i : wc * NTW + i;
}
template <int NTW, int MTW, int DH>
__device__ inline void qkv_epilogue(f32x16 (&acc)[NTW][MTW], int wc, int mt0, int rows, int n_tiles, int lane, const RowCtx& rc,
                                    const QkvOut& qo) {
  constexpr bool SPLIT = NTW * 32 < DH;
  constexpr int TH = SPLIT ? NTW : DH / 32, HALF = DH / 2;            // tiles per head, of this wavefront
  const int ht0 = SPLIT ? wc & 1 : 0;                   // its tile i of a head is the head's ht0 + HT i
  constexpr int HT = SPLIT ? 2 : 1;
  const int mloc = lane & 31, hf = lane >> 5;
  const int nq = qo.n_q_heads * DH, nkv = qo.kvl.n_kv_heads * DH;
#pragma unroll
  for (int j = 0; j < MTW; ++j) {
    const int m = (mt0 + j) * 32 + mloc;
    const bool ok = m < rows;
    const int mr = ok ? m : rows - 1;
    const int slot = rc.row_slot[mr], pos = rc.row_pos[mr];
    const int page = qo.block_table[(size_t)slot * qo.max_blocks + (pos >> 4)], tok = pos & 15;
#pragma unroll
    for (int h = 0; h < NTW / TH; ++h) {
      const int col0 = (qkv_tile<NTW, DH>(wc, h * TH) - ht0) * 32;   // first column of the head (wavefront-uniform)
      if (col0 >= n_tiles * 32) continue;
      if (col0 < nq + nkv) {
        const float* cs = qo.rope_cos + (size_t)pos * HALF + 32 * ht0 + 4 * hf;
        const float* sn = qo.rope_sin + (size_t)pos * HALF + 32 * ht0 + 4 * hf;
        constexpr int PAIRS = TH > 1 ? TH / 2 : 1, QN = TH > 1 ? 4 : 2;
#pragma unroll
        for (int p = 0; p < PAIRS; ++p)
#pragma unroll
          for (int q = 0; q < QN; ++q) {
            const f32x4 c = *reinterpret_cast<const f32x4*>(cs + 32 * p + 8 * q), s = *reinterpret_cast<const f32x4*>(sn + 32 * p + 8 * q);
            f32x16& ta = acc[h * TH + p][j];
            f32x16& tb = acc[h * TH + p + (TH > 1 ? TH / 2 : 0)][j];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int ra = 4 * q + e, rb = 4 * q + e + (TH > 1 ? 0 : 8);
              const float a = ta[ra], b = tb[rb];
              ta[ra] = rope_first(a, b, c[e], s[e]);
              tb[rb] = rope_second(a, b, c[e], s[e]);
            }
          }
        const bool is_q = col0 < nq;
        bf16_t* dst = is_q ? qo.q + (size_t)mr * nq + col0
                           : qo.kv_pool + qo.kvl.at(qo.layer, 0, page, (col0 - nq) / DH, tok, 0);
#pragma unroll
        for (int i = 0; i < TH; ++i)
#pragma unroll
          for (int q = 0; q < 4; q += 2) {
            // the lane halves hold alternating groups of 4 columns: they trade one, so that each stores 8
            union { bf16x4 v[2]; unsigned u[4]; bf16x8 w; } own, st8;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              own.v[0][e] = (bf16_t)acc[h * TH + i][j][4 * q + e];
              own.v[1][e] = (bf16_t)acc[h * TH + i][j][4 * q + 4 + e];
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const unsigned give = hf ? own.u[e] : own.u[2 + e], got = __shfl_xor((int)give, 32, 64);
              st8.u[e] = hf ? got : own.u[e];
              st8.u[2 + e] = hf ? own.u[2 + e] : got;
            }
            // page layout of K: [d / 32][token + 16 ((d % 32) / 8)][d % 8]
            if (ok) *reinterpret_cast<bf16x8*>(dst + (is_q ? (ht0 + HT * i) * 32 + 8 * (q + hf) : (ht0 + HT * i) * 512 + 128 * (q + hf))) = st8.w;
          }
      } else {
        bf16_t* dst = qo.kv_pool + qo.kvl.at(qo.layer, 1, page, (col0 - nq - nkv) / DH, tok, 0);   // [d][token]
        if (ok) {
#pragma unroll
          for (int i = 0; i < TH; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) dst[((ht0 + HT * i) * 32 + 8 * (e >> 2) + 4 * hf + (e & 3)) * 16] = (bf16_t)acc[h * TH + i][j][e];
        }
      }
    }
  }
}

// One wavefront-wide copy of 64 x 16 bytes from global memory (a per-lane address) to LDS
// (a wavefront-uniform base; lane l lands at base + 16*l).  Device pass only: the host pass
// has no such instruction to type-check.
__device__ inline void copy_fragment_to_lds(const bf16x8* src_lane, bf16x8* lds_base) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_global_load_lds(src_lane, lds_base, 16, 0, 0);
#else
  (void)src_lane; (void)lds_base;
#endif
}
template <int LEFT>
__device__ inline void wait_vector_memory() {   // until at most LEFT vector-memory operations are outstanding
#if defined(__HIP_DEVICE_COMPILE__)
  // s_waitcnt with the expcnt and lgkmcnt fields all-ones: only vmcnt is waited for
  __builtin_amdgcn_s_waitcnt(0x0f70 | (LEFT & 15) | ((LEFT >> 4) << 14));
#endif
}

__device__ inline void wait_lds() {             // until no LDS operation is outstanding
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_s_waitcnt(0xc07f);
#endif
  asm volatile("" ::: "memory");
}

// Between the halves of an exchange through LDS inside one wavefront: the hardware keeps a wavefront's LDS operations in order, and this
// keeps the compiler from moving one lane's loads over another lane's stores, which it takes for unrelated.
__device__ inline void wave_lds_order() { asm volatile("" ::: "memory"); }

// The stage fragments are copied global -> LDS by the memory pipeline itself
// (global_load_lds_dwordx4: each lane's 16 bytes land at consecutive LDS addresses, which is
// exactly the fragment layout), through a ring of R stage buffers.  Nothing is staged in
// registers, so R - 1 stages of loads stay in flight behind the MFMAs.  Hand-placed waits:
// the copies of stage s are this wavefront's oldest outstanding vector-memory operations, so
// "at most (R - 2) stages still outstanding" means stage s has landed; the barrier that
// follows makes that true for every wavefront's share and also says everyone has finished
// reading the buffer that the next copies overwrite.  Requires K % (16 * BK) == 0.

// What the epilogues of gemm_rows_kernel need beside the results.
struct TileNorm {
  const float* ssq;            // gate/up (CHAIN): RMSNorm folded in, [n_ssq][ssq_stride] per-row sums of squares of 32-column slabs; nullptr = none
  int ssq_stride, n_ssq;
  float inv_d, eps;
  GroupOut go;                 // LM head: group records
};

// Routed experts (MOE): blockIdx.y is a row group of the dispatch kernel's packed list (MT m-tiles
// of one expert; the expert segments are aligned to MT * 32 rows), rows are packed-row indices,
// the weights are the expert's, and the activation rows are either the packed tiles (down
// projection) or token rows gathered through src_row from a plain [row][K] copy of the
// activations (gate/up: each lane copies its own 16 bytes, so a gathered fragment lands in LDS
// exactly like a dense one; gathering from the fragment-tiled layout would use 16 bytes of
// every 128-byte line it touches).
struct TileMoe {
  const int* cnt;              // [E] rows of every expert
  const int* base;             // [E] first packed row of every expert
  const int* group_expert;     // [row groups] expert of the group, -1 = none
  const int* src_row;          // [packed rows] token row, or nullptr (activations already packed)
  size_t w_expert_stride;      // bf16x8 units between the experts' matrices
  int n_groups, near;          // length of group_expert; row groups an XCD takes in a row (0 = grid order)
};

// Row groups of an expert share its weights, the weight tiles of a row group its activations, but in grid
// order consecutive workgroups go to different XCDs and nearly every operand byte is read past the L2.  Here a 1-D grid: XCD
// (id mod 8) takes `near` row groups with all their weight tiles, then the ones 8 * near further on.
// The caller rounds the grid up; a group of n_groups or beyond does not exist.
__device__ __forceinline__ int2 moe_tile_of_block(const TileMoe& mo, int tiles) {
  if (mo.near == 0) return make_int2(blockIdx.x, blockIdx.y);
  const int xcd = (int)blockIdx.x & 7, j = (int)blockIdx.x >> 3, per = mo.near * tiles, in = j % per;
  return make_int2(in % tiles, ((j / per) * 8 + xcd) * mo.near + in / tiles);
}

// (weight tile group, row group) of a workgroup.  NEAR (LM head): a 1-D grid with the row groups
// of one weight tile group 8 ids apart - same XCD, same moment, one HBM read instead of one per row group.
// Else x = weight tile group, y = row group.
template <bool NEAR>
__device__ __forceinline__ int2 tile_of_block(const RowCtx& rc, int MT) {
  if (!NEAR) return make_int2(blockIdx.x, blockIdx.y);
  const int mg = ceil_div(ceil_div(rc.max_rows, 32), MT), rem = (int)blockIdx.x % (8 * mg);
  return make_int2(((int)blockIdx.x / (8 * mg)) * 8 + (rem & 7), rem >> 3);
}

template <int WGM, int WGN, int MTW, int NTW, int BK, int R, int EPI, bool MOE = false, int DH = 0>
__device__ __forceinline__ void tile_dma_body(RowCtx rc, const bf16x8* __restrict__ x, const bf16x8* __restrict__ w0,
                                              const bf16x8* __restrict__ w1, float* __restrict__ out,
                                              bf16_t* __restrict__ act, int N, int K, const GroupOut& go,
                                              const TileMoe& mo = TileMoe{}, const QkvOut& qo = QkvOut{}) {
  constexpr int NW = WGM * WGN, MT = WGM * MTW, NT = WGN * NTW, FR = MT + NT;
  constexpr int PER = FR * BK / NW;
  static_assert(FR * BK % NW == 0 && NW % BK == 0, "staging split");
  static_assert(EPI != TEPI_SWIGLU || NTW % 2 == 0, "gate/up pairs");
  static_assert(R >= 3 && (R - 2) * PER < 64, "ring depth");
  __shared__ bf16x8 lds[R][BK][FR][64];
  int2 at;
  if constexpr (MOE) at = moe_tile_of_block(mo, ceil_div(N >> 5, EPI == TEPI_SWIGLU ? NT / 2 : NT));
  else at = tile_of_block<EPI == TEPI_LOGITS>(rc, MT);
  const int bx = at.x, by = at.y;
  int rows = rows_or_zero(rc);
  const int m0 = by * MT;
  if constexpr (MOE) {
    if (rows == 0 || by >= mo.n_groups) return;  // step stopped, or nothing to do
    const int e = mo.group_expert[by];
    if (e < 0) return;
    const int rows_e = mo.cnt[e], p0 = mo.base[e];
    if (m0 * 32 < p0 || m0 * 32 - p0 >= rows_e) return;
    rows = p0 + rows_e;                          // one past the expert's last packed row
    w0 += (size_t)e * mo.w_expert_stride;
    if (w1 != nullptr) w1 += (size_t)e * mo.w_expert_stride;
  } else {
    if (m0 * 32 >= rows || (EPI == TEPI_LOGITS && bx * NT * 32 >= N)) return;
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int KT = K >> 4;
  const int m_last = (rows - 1) >> 5;
  const int n_tiles = N >> 5;
  auto slot_base = [&](int t) -> const bf16x8* {        // this lane's piece of the slot's fragment at k-tile 0
    if (t < MT) {
      if constexpr (MOE) {
        if (mo.src_row != nullptr) {
          int p = (m0 + t) * 32 + (lane & 31);
          if (p > rows - 1) p = rows - 1;                 // rows beyond the expert's repeat its last one (never written)
          int row = mo.src_row[p];
          if (row < 0) row = 0;
          return x + ((size_t)row * KT * 2 + (lane >> 5));   // plain [row][K]: a k-tile of a row is two 16-byte pieces
        }
      }
      int mt = m0 + t;
      if (mt > m_last) mt = m_last;
      return x + (size_t)mt * KT * 64 + lane;
    }
    const int i = t - MT;
    if (EPI == TEPI_SWIGLU) {
      constexpr int H = NTW / 2;
      const int col = i / NTW, ii = i % NTW;
      int f = bx * (NT / 2) + col * H + (ii < H ? ii : ii - H);
      if (f >= n_tiles) f = n_tiles - 1;
      return (ii < H ? w0 : w1) + (size_t)f * KT * 64 + lane;
    }
    int nt = bx * NT + i;
    if constexpr (EPI == TEPI_QKV) nt = qkv_tile<NTW, DH>(bx * WGN + i / NTW, i % NTW);
    if (nt >= n_tiles) nt = n_tiles - 1;
    return w0 + (size_t)nt * KT * 64 + lane;
  };
  const int skk = wave % BK, st0 = wave / BK;
  const bf16x8* src[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) src[u] = slot_base(st0 + (NW / BK) * u);
  const int n_stages = KT / BK;
  const bool gathered = MOE && mo.src_row != nullptr;
  auto issue = [&](int s) {
    const size_t off = (size_t)(s * BK + skk) * 64;
    const size_t off_rows = (size_t)(s * BK + skk) * 2;      // gathered activation rows advance 32 bytes per k-tile
    const int slot = s % R;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int t = st0 + (NW / BK) * u;
      copy_fragment_to_lds(src[u] + (gathered && t < MT ? off_rows : off), &lds[slot][skk][t][0]);
    }
  };

  f32x16 acc[NTW][MTW];
#pragma unroll
  for (int i = 0; i < NTW; ++i)
#pragma unroll
    for (int j = 0; j < MTW; ++j) acc[i][j] = f32x16{};

#pragma unroll
  for (int r = 0; r < R - 1; ++r)
    if (r < n_stages) issue(r);

  for (int s = 0; s < n_stages; ++s) {
    // wait for this wavefront's copies of stage s (s_waitcnt vmcnt only: expcnt/lgkmcnt fields all-ones)
    constexpr int LEFT = (R - 2) * PER;
    if (s + R - 2 < n_stages) wait_vector_memory<LEFT>();
    else wait_vector_memory<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (s + R - 1 < n_stages) issue(s + R - 1);
    const int slot = s % R;
    bf16x8 a[2][NTW], b[2][MTW];
#pragma unroll
    for (int i = 0; i < NTW; ++i) a[0][i] = lds[slot][0][MT + wn * NTW + i][lane];
#pragma unroll
    for (int j = 0; j < MTW; ++j) b[0][j] = lds[slot][0][wm * MTW + j][lane];
#pragma unroll
    for (int kk = 0; kk < BK; ++kk) {
      const int cur = kk & 1, nxt = cur ^ 1;
      if (kk + 1 < BK) {
#pragma unroll
        for (int i = 0; i < NTW; ++i) a[nxt][i] = lds[slot][kk + 1][MT + wn * NTW + i][lane];
#pragma unroll
        for (int j = 0; j < MTW; ++j) b[nxt][j] = lds[slot][kk + 1][wm * MTW + j][lane];
      }
#pragma unroll
      for (int i = 0; i < NTW; ++i)
#pragma unroll
        for (int j = 0; j < MTW; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cur][i], b[cur][j], acc[i][j], 0, 0, 0);
      if (kk + 1 < BK) {          // issue order: the LDS reads of k-tile kk+1, then the MFMAs of kk
        __builtin_amdgcn_sched_group_barrier(0x100, NTW + MTW, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, NTW * MTW, 0);
      }
    }
    asm volatile("" ::: "memory");
  }
  if constexpr (EPI == TEPI_QKV) {
    qkv_epilogue<NTW, MTW, DH>(acc, bx * WGN + wn, m0 + wm * MTW, rows, n_tiles, lane, rc, qo);
    return;
  }
  tile_epilogue<MTW, NTW, EPI>(acc, bx * (EPI == TEPI_SWIGLU ? NT / 2 : NT) + wn * (EPI == TEPI_SWIGLU ? NTW / 2 : NTW),
                               m0 + wm * MTW, rows, n_tiles, N, lane, out, act, nullptr, &go);
}

// The large tile: 256 x 256 outputs on 4 wavefronts of 128 x 128, one per SIMD.  8 wavefronts of
// 128 x 64 read 6 fragments from LDS for 8 products, which with the copies into LDS is all of the
// LDS bandwidth the products leave time for; 128 x 128 reads 8 for 16.  With nothing else
// on the SIMD the wavefront hides its own latencies: the fragments of the next k-tile are read while the
// products of this one run, across the stage boundary too, and the copies of the stage R - 1 ahead are
// spread over the second k-tile's products.  One barrier per stage, in its middle: it makes stage s + 1
// readable (every wavefront has waited for its own copies of it) and the slot of stage s - 1 free.
// With the reads or copies inside branches, or a burst of copies after the barrier, it was 5 % slower than 8 wavefronts.
// Same accumulator chain per element as every kernel here (k-tiles in order).  K % 32 == 0.
// What bounds it: power.  2 x 9728 x 2560 with SiLU at 32768 and 65536 rows: the matrix cores are busy 70 % of the cycles, at 1.80 and 1.56 GHz
// of 2.4 (1.31 and 1.14 PFLOP/s; a library product of 16384^3 reaches 1.56); output and down projections 58-71 % at 1.65-1.9 GHz.  The rest is in the rounds: a tile of K = 2560 takes 60 us on its
// compute unit, the ring's filling and a SwiGLU epilogue 6 more, and a launch lasts as long as the unit with the most tiles.
// Hence the tiles' order and the halves below.  us at 16384 rows, a grid of 256 x 256 tiles in grid order / this: gate/up of 9728 x 2560
// 1295 / 1250, of 4864 x 896 (14500 rows) 246 / 233; output projections 2560 x 4096 437 / 363, x 9728 776 / 698 (2.5 rounds of tiles),
// 4096 x 14336 (12800 rows) 1375 / 1250, 896 x 4864 (14500) 140 / 122.
constexpr int BIG_R = 4, BIG_BK = 2;
// The workgroups of a launch: `full` tiles of 256 x 256, then tiles of 256 x 128: the two halves of the last `split` tiles, 8 ids apart, and
// the `my` pieces of a last column of 128 where the columns are an odd number of those.  Halves come in sixteens; the ids that a last, partial
// sixteen leaves over go to pieces first, so that 256 halves and pieces are 32 on every XCD.  (With those ids empty and all pieces
// behind, up to 256 of them were 33 on some XCDs, a second round.  us in a padded grid of whole tiles | so | as here: 896 x 4864 at 8900 rows
// 118 | 124 | 78, 640 x 2048 at 12500 rows 53 | 61 | 39, SwiGLU of 960 x 1664 at 4300 rows 40 | 46 | 32.)
struct BigGrid {
  int nx, my;                  // tiles of 256 columns, of 256 rows
  int full, split, odd;
  __host__ __device__ int pairs() const { return ((split + 7) & ~7) * 2; }       // ids of the halves
  __host__ __device__ int spare() const { return pairs() - 2 * split; }          // those among them that are left over
  __host__ __device__ int halves() const { return pairs() + (odd && my > spare() ? my - spare() : 0); }
};
// The order of the tiles: groups of 6 row tiles, inside a group column after column; where the columns are a multiple of 8, row after row.
__device__ __forceinline__ int2 big_tile(const BigGrid& g, int t) {
  const int high = (g.nx & 7) ? 6 : 1, grp = t / (high * g.nx), in = t - grp * high * g.nx, h = min(high, g.my - grp * high), col = in / h;
  return make_int2(col, grp * high + in - col * h);
}

// One tile of WGM * MTW * 32 rows x NTW * 64 columns.  u0: its first column in units of 128 (SwiGLU: of 64 features).
//
// CHAIN (decode with many rows): the skinny decode kernel sums k in four quarters (its four
// wavefronts), each quarter its own accumulator chain, and adds them as ((q0 + q1) + q2) + q3.
// Here one wavefront walks all of k, so it closes a chain at every quarter boundary and adds
// it to a second accumulator set in that order: every output element gets the same bits from
// either kernel, and the choice between them can follow the row count.  The quarter
// boundaries must fall on stage boundaries (K % 128 == 0).
template <int EPI, int DH, int MTW, int NTW, bool CHAIN = false, int R = BIG_R, int WGM = 2>
__device__ __forceinline__ void big_body(const RowCtx& rc, const bf16x8* __restrict__ x, const bf16x8* __restrict__ w0,
                                         const bf16x8* __restrict__ w1, float* __restrict__ out, bf16_t* __restrict__ act,
                                         int N, int K, const TileNorm& tn, const QkvOut& qo, bf16x8* lds_raw, int rows, int u0, int m0) {
  constexpr int MT = WGM * MTW, NT = 2 * NTW, BK = BIG_BK, FR = MT + NT, PER = FR / WGM, READS = NTW + MTW, PRODUCTS = NTW * MTW;
  static_assert(R >= 4 && (R - 2) * PER < 64 && BK == 2 && FR % WGM == 0, "ring depth, staging split");
  auto lds = reinterpret_cast<bf16x8 (*)[BK][FR][64]>(lds_raw);
  auto slot_of = [](int s) { return (R & (R - 1)) == 0 ? s & (R - 1) : (int)((unsigned)s % (unsigned)R); };
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int KT = K >> 4, n_stages = KT / BK;
  const int m_last = (rows - 1) >> 5, n_tiles = N >> 5;
  const int nt0 = u0 * (EPI == TEPI_SWIGLU ? 2 : 4);    // first weight (feature) tile of the workgroup
  // Fragment slot t of a k-tile: activation tile m0 + t, then weight slots; weight slot i belongs to
  // wavefront column i / NTW (SwiGLU: its first half gate tiles, its second half the up tiles of the
  // same features).  Tiles past the end are clamped for the loads and never stored.
  auto slot_base = [&](int t) -> const bf16x8* {
    if (t < MT) return x + (size_t)min(m0 + t, m_last) * KT * 64;
    const int i = t - MT;
    if (EPI == TEPI_SWIGLU) {
      constexpr int H = NTW / 2;
      const int col = i / NTW, ii = i % NTW;
      return (ii < H ? w0 : w1) + (size_t)min(nt0 + col * H + (ii < H ? ii : ii - H), n_tiles - 1) * KT * 64;
    }
    int nt = nt0 + i;
    if constexpr (EPI == TEPI_QKV) nt = qkv_tile<NTW, DH>(nt0 / NTW + i / NTW, i % NTW);
    return w0 + (size_t)min(nt, n_tiles - 1) * KT * 64;
  };
  const int skk = wave & 1, st0 = wave >> 1;             // this wavefront copies k-tile skk of slots st0, st0 + WGM, ...
  const bf16x8* src[PER];                               // wavefront-uniform: scalar registers
#pragma unroll
  for (int u = 0; u < PER; ++u) src[u] = slot_base(st0 + WGM * u) + skk * 64;
  auto copy = [&](int s, int u) {
    // scalar base + 32-bit lane offset
    copy_fragment_to_lds(reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(src[u]) + (unsigned)(s * (BK * 1024) + lane * 16)),
                         &lds[slot_of(s)][skk][st0 + WGM * u][0]);
  };

  f32x16 acc[NTW][MTW];
#pragma unroll
  for (int i = 0; i < NTW; ++i)
#pragma unroll
    for (int j = 0; j < MTW; ++j) acc[i][j] = f32x16{};
  // Folded norm: 1/rms of the workgroup's rows, summed in the skinny kernel's order (wavefront w of that kernel adds the slabs w, w + 4, ...;
  // then ((s0 + s1) + s2) + s3).  The first 64 slabs (K up to 2048) are requested ahead of the ring's copies, so that their sum does not wait for
  // those; the others (16 more at 2560, 64 at 4096) come behind the copies and wait for all of them.  Threads beyond the rows repeat the last row.
  constexpr int SLABS = 64;
  float* const scale_lds = reinterpret_cast<float*>(&lds[R - 1][0][0][0]);      // (no copies go there before stage 0 is under way)
  const bool scaled = CHAIN && EPI == TEPI_SWIGLU && tn.ssq != nullptr;
  const float* const ssq_row = scaled ? tn.ssq + min(m0 * 32 + (int)threadIdx.x, rows - 1) : nullptr;
  float sl[CHAIN ? SLABS : 1];
  auto request = [&](int t0) {
#pragma unroll
    for (int u = 0; u < SLABS; ++u) sl[u] = ssq_row[(size_t)min(t0 + u, tn.n_ssq - 1) * tn.ssq_stride];
  };
  if (CHAIN && scaled) request(0);
#pragma unroll
  for (int r = 0; r < R - 1; ++r)
    if (r < n_stages) {
#pragma unroll
      for (int u = 0; u < PER; ++u) copy(r, u);
    }
  if (CHAIN && scaled) {
    float sw[4] = {0.f, 0.f, 0.f, 0.f};
    for (int t0 = 0; t0 < tn.n_ssq; t0 += SLABS) {
      if (t0 > 0) request(t0);
#pragma unroll
      for (int u = 0; u < SLABS; ++u)
        if (t0 + u < tn.n_ssq) sw[u & 3] += sl[u];
    }
    if ((int)threadIdx.x < MT * 32) scale_lds[threadIdx.x] = 1.0f / sqrtf(__fmaf_rn(((sw[0] + sw[1]) + sw[2]) + sw[3], tn.inv_d, tn.eps));
    wait_lds();
  }
  bf16x8 a[2][NTW], b[2][MTW];
  auto read = [&](int s, int kk) {
    a[kk][0] = lds[slot_of(s)][kk][MT + wn * NTW][lane];      // in the order the products want them
#pragma unroll
    for (int j = 0; j < MTW; ++j) b[kk][j] = lds[slot_of(s)][kk][wm * MTW + j][lane];
#pragma unroll
    for (int i = 1; i < NTW; ++i) a[kk][i] = lds[slot_of(s)][kk][MT + wn * NTW + i][lane];
  };
  auto products = [&](int kk) {
#pragma unroll
    for (int i = 0; i < NTW; ++i)
#pragma unroll
      for (int j = 0; j < MTW; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk][i], b[kk][j], acc[i][j], 0, 0, 0);
  };
  if (n_stages > R - 2) wait_vector_memory<(R - 2) * PER>(); else wait_vector_memory<0>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  float row_scale[MTW];                                  // of this lane's rows
#pragma unroll
  for (int j = 0; j < MTW; ++j) row_scale[j] = 1.0f;
  if (scaled) {
#pragma unroll
    for (int j = 0; j < MTW; ++j) row_scale[j] = scale_lds[(wm * MTW + j) * 32 + (lane & 31)];
    wait_lds();
  }
  read(0, 0);
  // One stage.  COPY: stage s + R - 1 exists.  (Reading k-tile 0 of stage s + 1 past the end fetches a slot's old contents, which nothing uses: the code
  // stays free of branches between the products.)
  auto stage = [&](int s, auto copying) {
    constexpr bool COPY = decltype(copying)::value;
    read(s, 1);
    products(0);
#pragma unroll
    for (int q = 0; q < READS; ++q) {                    // LDS reads between the first products: back before the last ones end
      if (q < PRODUCTS) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    if (PRODUCTS > READS) __builtin_amdgcn_sched_group_barrier(0x008, PRODUCTS - READS, 0);
    // stage s + 1 has landed when at most the copies of the stages s + 2 .. s + R - 2 are outstanding
    wait_vector_memory<COPY ? (R - 3) * PER : 0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (COPY) {
#pragma unroll
      for (int u = 0; u < PER; ++u) copy(s + R - 1, u);
    }
    read(s + 1, 0);
    products(1);
#pragma unroll
    for (int q = 0; q < READS; ++q) {
      if (q < PRODUCTS) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      if (COPY && q < PER) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
    if (PRODUCTS > READS) __builtin_amdgcn_sched_group_barrier(0x008, PRODUCTS - READS, 0);
    asm volatile("" ::: "memory");
  };
  int s = 0;
  if constexpr (CHAIN) {
    f32x16 tot[NTW][MTW];
#pragma unroll 1
    for (int quarter = 0; quarter < 4; ++quarter) {
      const int end = n_stages / 4 * (quarter + 1);
      for (; s < min(end, n_stages - R + 1); ++s) stage(s, std::true_type{});
      for (; s < end; ++s) stage(s, std::false_type{});
#pragma unroll
      for (int i = 0; i < NTW; ++i)
#pragma unroll
        for (int j = 0; j < MTW; ++j) {
          tot[i][j] = quarter == 0 ? acc[i][j] : tot[i][j] + acc[i][j];
          acc[i][j] = f32x16{};
        }
    }
#pragma unroll
    for (int i = 0; i < NTW; ++i)
#pragma unroll
      for (int j = 0; j < MTW; ++j) acc[i][j] = tot[i][j];
  } else {
    for (; s + R - 1 < n_stages; ++s) stage(s, std::true_type{});
    for (; s < n_stages; ++s) stage(s, std::false_type{});
  }
  if constexpr (EPI == TEPI_QKV) {
    qkv_epilogue<NTW, MTW, DH>(acc, nt0 / NTW + wn, m0 + wm * MTW, rows, n_tiles, lane, rc, qo);
  } else if constexpr (EPI == TEPI_RESID) {
    // out += result, a wavefront's 32 rows at a time: through LDS (its own part of the ring, which everyone has finished
    // reading) into whole rows, so that an instruction reads and writes 512 (256) consecutive bytes of a row.  From the
    // accumulators' own layout, 32 pieces of 32 bytes an instruction, this took 50 us of a round (512 KB a workgroup): 2560 x 4096
    // at 16384 rows 397 -> 363 us, 896 x 896 at 14500 44 -> 38.  (Residual values requested during the last stages, into registers
    // the products leave free, cost the k loop more than they gave: spills, or another schedule.)
    constexpr int LPR = NTW * 8, RPI = 64 / LPR, PIECES = 32 / RPI, STRIDE = NTW * 32 + 4;
    static_assert(4 * 32 * STRIDE * 4 <= (int)sizeof(bf16x8) * R * BK * FR * 64, "LDS");
    __syncthreads();
    float* buf = reinterpret_cast<float*>(lds_raw) + wave * 32 * STRIDE;
    const int wnt0 = nt0 + wn * NTW, row0 = lane / LPR, c4 = (lane % LPR) * 4, mw = (m0 + wm * MTW) * 32 + row0;
    if (wnt0 >= n_tiles) return;
    const bool col_ok = wnt0 + (c4 >> 5) < n_tiles;
    float* const col = out + (size_t)wnt0 * 32 + (col_ok ? c4 : 0);
    f32x4 v[2][PIECES];
    auto load = [&](int j) {
#pragma unroll
      for (int p = 0; p < PIECES; ++p) v[j & 1][p] = *reinterpret_cast<const f32x4*>(col + (size_t)min(mw + j * 32 + p * RPI, rows - 1) * N);
    };
    load(0);
    load(1);
#pragma unroll
    for (int j = 0; j < MTW; ++j) {
#pragma unroll
      for (int i = 0; i < NTW; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<f32x4*>(buf + (lane & 31) * STRIDE + i * 32 + 8 * q + ((lane >> 5) << 2)) =
              f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
      wave_lds_order();
#pragma unroll
      for (int p = 0; p < PIECES; ++p) {
        const int m = mw + j * 32 + p * RPI;
        const f32x4 r = v[j & 1][p] + *reinterpret_cast<const f32x4*>(buf + (row0 + p * RPI) * STRIDE + c4);
        if (m < rows && col_ok) *reinterpret_cast<f32x4*>(col + (size_t)m * N) = r;
      }
      wave_lds_order();
      if (j + 2 < MTW) load(j + 2);
    }
  } else {
    tile_epilogue<MTW, NTW, EPI>(acc, nt0 + wn * (EPI == TEPI_SWIGLU ? NTW / 2 : NTW), m0 + wm * MTW, rows, n_tiles, N, lane, out, act,
                                 CHAIN && EPI == TEPI_SWIGLU ? row_scale : nullptr, &tn.go);
  }
}

template <int EPI, int DH = 0>
__global__ __launch_bounds__(256, 1) void gemm_big_kernel(RowCtx rc, const bf16x8* __restrict__ x,
                                                          const bf16x8* __restrict__ w0, const bf16x8* __restrict__ w1,
                                                          float* __restrict__ out, bf16_t* __restrict__ act, int N, int K,
                                                          QkvOut qo, BigGrid g) {
  __shared__ bf16x8 lds[BIG_R * BIG_BK * 16 * 64];
  const int rows = rows_or_zero(rc);
  const TileNorm tn{};
  const int id = blockIdx.x;
  if (id < g.full) {
    // Workgroup ids go to the XCDs in turn.  Each XCD gets a run of the tiles, so that what its compute units hold at once
    // shares operands; row after row with a multiple of 8 columns it keeps the same few columns by itself.
    const int xcd = id & 7, per = g.full >> 3, more = g.full & 7;
    const int2 at = big_tile(g, (g.nx & 7) ? xcd * per + min(xcd, more) + (id >> 3) : id);
    if (at.y * 256 >= rows) return;
    big_body<EPI, DH, 4, 4>(rc, x, w0, w1, out, act, N, K, tn, qo, lds, rows, at.x * 2, at.y * 8);
  } else {
    const int h = id - g.full, t = (h >> 4) * 8 + (h & 7), half = (h >> 3) & 1;
    int u0, m0;
    if (t < g.split) {           // the halves of a tile 8 ids apart: same XCD
      const int2 at = big_tile(g, g.full + t);
      u0 = at.x * 2 + half;
      m0 = at.y * 8;
    } else {
      const int piece = h < g.pairs() ? t - g.split + half * (g.spare() >> 1) : h - g.pairs() + g.spare();
      if (!g.odd || piece >= g.my) return;
      u0 = 2 * g.nx;
      m0 = piece * 8;
    }
    if (m0 * 32 >= rows) return;
    big_body<EPI, DH, 4, 2>(rc, x, w0, w1, out, act, N, K, tn, qo, lds, rows, u0, m0);
  }
}

// The same for decode passes of many rows: MTW * 64 rows x NTW * 64 columns, the row groups of a column of tiles 8 workgroup ids apart
// (same XCD, same moment: one read of the weights).  The first `full` columns of tiles are whole, those behind them go as halves.
template <int EPI, int WGM, int MTW, int NTW, bool CHAIN, int OCC, int R>
__global__ __launch_bounds__(128 * WGM, OCC) void gemm_rows_kernel(RowCtx rc, const bf16x8* __restrict__ x, const bf16x8* __restrict__ w0,
                                                             const bf16x8* __restrict__ w1, float* __restrict__ out,
                                                             bf16_t* __restrict__ act, int N, int K, TileNorm tn, int full) {
  // (one array: with a second one the compiler waits for every copy in flight before it reads from this one)
  __shared__ bf16x8 lds[R * BIG_BK * (WGM * MTW + 2 * NTW) * 64];
  const int rows = rows_or_zero(rc), groups = ceil_div(ceil_div(rc.max_rows, 32), WGM * MTW);
  const int whole = (full + 7) / 8 * 8 * groups, half = (int)blockIdx.x >= whole, id = (int)blockIdx.x - (half ? whole : 0);
  const int col = id / (8 * groups) * 8 + (id & 7), m0 = (id % (8 * groups) >> 3) * WGM * MTW;
  if (m0 * 32 >= rows) return;
  if constexpr (NTW == 4) {
    if (half) {
      if ((2 * full + col) * (EPI == TEPI_SWIGLU ? 64 : 128) >= N) return;
      big_body<EPI, 0, MTW, 2, CHAIN, R, WGM>(rc, x, w0, w1, out, act, N, K, tn, QkvOut{}, lds, rows, 2 * full + col, m0);
      return;
    }
  }
  if (col >= full) return;
  big_body<EPI, 0, MTW, NTW, CHAIN, R, WGM>(rc, x, w0, w1, out, act, N, K, tn, QkvOut{}, lds, rows, NTW == 4 ? col * 2 : col, m0);
}
// The columns of tiles that stay whole, of `units` half columns: as in big_grid.
static int rows_full(int units, int groups) {
  const int tiles = units / 2 * groups, whole = tiles / 256 * 256 / groups;
  return (units - 2 * whole) * groups <= 256 ? whole : (units + 1) / 2;
}
static int rows_grid(int units, int full, int groups) { return ((full + 7) / 8 + (units > 2 * full ? (units - 2 * full + 7) / 8 : 0)) * 8 * groups; }

// units: columns in 128 (SwiGLU: features in 64).  The tiles past the last whole round of 256 workgroups go as halves where those are
// one round: it then lasts 0.57 of one (a wavefront of 128 x 64 reads 6 fragments for 8 products).
static BigGrid big_grid(int units, int m_tiles) {
  BigGrid g{units / 2, ceil_div(m_tiles, 8), 0, 0, units & 1};
  const int tiles = g.nx * g.my, last = tiles % 256;
  g.split = 2 * last + (g.odd ? g.my : 0) <= 256 ? last : 0;
  g.full = tiles - g.split;
  return g;
}

template <int WGM, int WGN, int MTW, int NTW, int BK, int R, int EPI>
__global__ __launch_bounds__(64 * WGM * WGN) __attribute__((amdgpu_waves_per_eu(2)))
void gemm_tile_dma_kernel(RowCtx rc, const bf16x8* __restrict__ x, const bf16x8* __restrict__ w0,
                          const bf16x8* __restrict__ w1, float* __restrict__ out, bf16_t* __restrict__ act, int N,
                          int K, GroupOut go) {
  tile_dma_body<WGM, WGN, MTW, NTW, BK, R, EPI>(rc, x, w0, w1, out, act, N, K, go);
}

template <int WGM, int WGN, int MTW, int NTW, int BK, int R, int DH>
__global__ __launch_bounds__(64 * WGM * WGN) __attribute__((amdgpu_waves_per_eu(2)))
void gemm_tile_qkv_kernel(RowCtx rc, const bf16x8* __restrict__ x, const bf16x8* __restrict__ w0, int N, int K, QkvOut qo) {
  tile_dma_body<WGM, WGN, MTW, NTW, BK, R, TEPI_QKV, false, DH>(rc, x, w0, nullptr, nullptr, nullptr, N, K, GroupOut{}, TileMoe{}, qo);
}

// Routed experts in prefill: 128 packed rows (one row group of the dispatch list) x 256 weight
// rows per workgroup, 4 wavefronts side by side (each 128 x 64), ring of 3 stages (72 KiB, two
// workgroups per CU).  One accumulator chain per output element, like every prefill GEMM.
template <int EPI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void moe_tile_kernel(RowCtx rc, const bf16x8* __restrict__ x, const bf16x8* __restrict__ w0,
                     const bf16x8* __restrict__ w1, float* __restrict__ out, bf16_t* __restrict__ act, int N, int K,
                     TileMoe mo) {
  tile_dma_body<1, 4, 4, 2, 2, 3, EPI, true>(rc, x, w0, w1, out, act, N, K, GroupOut{}, mo);
}

int moe_tile_rows() { return 128; }

// TileMoe::near and the grid that covers every (weight tile, row group) under it.  8 groups in a row are about what an XCD's
// 32 compute units hold at once; fewer while 64 runs of them would not exist (the XCDs stay evenly loaded), and
// grid order below 64 groups, where spreading the weights' first read counts for more.  128 experts of 768 x 2048,
// 8 per token, passes of 13 900 token rows: gate/up 1005 -> 849 us (0.70 -> 0.82 PFLOP/s); down
// unchanged at 525 us (8 weight tiles: grid order gave each XCD one of them already).
static int moe_near(int n_groups) { return n_groups >= 64 ? std::min(8, n_groups / 64) : 0; }
static dim3 moe_grid(int tiles, int n_groups) {
  const int near = moe_near(n_groups);
  return near == 0 ? dim3(tiles, n_groups) : dim3(ceil_div(n_groups, 8 * near) * 8 * near * tiles);
}

bool launch_moe_tile_gateup(hipStream_t st, RowCtx rc, const int* cnt, const int* base, const int* group_expert,
                            const int* src_row, const bf16_t* h_rows, const bf16_t* Wg, const bf16_t* Wu, bf16_t* act,
                            int Fe, int d, int n_groups) {
  if (d % 32 != 0 || Fe % 32 != 0 || n_groups <= 0 || h_rows == nullptr) return false;
  const TileMoe mo{cnt, base, group_expert, src_row, (size_t)Fe * d / 8, n_groups, moe_near(n_groups)};
  const dim3 grid = moe_grid(ceil_div(Fe >> 5, 4), n_groups);   // 4 feature tiles (gate + up: 8 weight tiles) per workgroup
  hipLaunchKernelGGL((moe_tile_kernel<TEPI_SWIGLU>), grid, dim3(256), 0, st, rc, reinterpret_cast<const bf16x8*>(h_rows),
                     reinterpret_cast<const bf16x8*>(Wg), reinterpret_cast<const bf16x8*>(Wu), nullptr, act, Fe, d, mo);
  return true;
}

bool launch_moe_tile_down(hipStream_t st, RowCtx rc, const int* cnt, const int* base, const int* group_expert,
                          const bf16_t* act, const bf16_t* Wd, float* out, int Fe, int d, int n_groups) {
  if (d % 32 != 0 || Fe % 32 != 0 || n_groups <= 0) return false;
  const TileMoe mo{cnt, base, group_expert, nullptr, (size_t)d * Fe / 8, n_groups, moe_near(n_groups)};
  const dim3 grid = moe_grid(ceil_div(d >> 5, 8), n_groups);
  hipLaunchKernelGGL((moe_tile_kernel<TEPI_F32>), grid, dim3(256), 0, st, rc, reinterpret_cast<const bf16x8*>(act),
                     reinterpret_cast<const bf16x8*>(Wd), nullptr, out, nullptr, d, Fe, mo);
  return true;
}

// Tile shapes (the choice changes no result, see the header comment).  WIDE: gemm_big_kernel, 256 x 256 outputs or 256 x 128.
// SMALL: 64 rows x 32 columns (SwiGLU: 32 features) on 2 wavefronts, ring of 16 stages, and MID: 128 x 64 on 4,
// ring of 12 (8), for passes of few rows: there a workgroup of the larger tiles walks k alone at two
// stages per memory latency, whatever the rows.  SMALL while its workgroups are at most one per compute unit, then MID
// while its are.  us, WIDE / as here: 2560 x 9728 at 37, 256, 512 rows 146, 150, 150 / 45, 64, 65; 896 x 4864
// at 37, 512 rows 73, 77 / 24, 24; 4096 x 4096 at 128, 512 rows 65, 68 / 21, 33; gate/up of
// 2560 x 9728 at 64, 128 rows 45, 46 / 28, 28, of 896 x 4864 at 37, 256 rows 17, 18 / 8, 12.  MID at two workgroups per unit | WIDE:
// 2560 x 9728 at 900, 1500 rows 131, 140 | 102, 108; 896 x 4864 at 2500, 4000 rows 71, 73 | 54, 57; 4096 x 14336 at 700 rows 185 | 147;
// 1184 x 3104 at 2000 rows 47 | 37.
#define TILE_WIDE(EPI) gemm_big_kernel<EPI>
#define TILE_SMALL(EPI) gemm_tile_dma_kernel<2, 1, 1, 1, 2, 16, EPI>
#define TILE_SMALL_SWIGLU gemm_tile_dma_kernel<2, 1, 1, 2, 2, 16, TEPI_SWIGLU>
#define TILE_MID(EPI) gemm_tile_dma_kernel<2, 2, 2, 1, 2, 12, EPI>
#define TILE_MID_SWIGLU gemm_tile_dma_kernel<2, 2, 2, 2, 2, 8, TEPI_SWIGLU>
static bool small_tile(int units, int m_tiles) { return (long long)units * ceil_div(m_tiles, 2) <= 256; }
static bool mid_tile(int units, int m_tiles) { return (long long)ceil_div(units, 2) * ceil_div(m_tiles, 4) <= 256; }

template <int EPI>
static void launch_tile(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, float* out, int N, int K) {
  const int n_tiles = N >> 5, m_tiles = ceil_div(rc.max_rows, 32);
  const bf16x8* xv = reinterpret_cast<const bf16x8*>(x);
  const bf16x8* wv = reinterpret_cast<const bf16x8*>(Wp);
  if (small_tile(n_tiles, m_tiles)) {
    hipLaunchKernelGGL((TILE_SMALL(EPI)), dim3(n_tiles, ceil_div(m_tiles, 2)), dim3(128), 0, st, rc, xv, wv, nullptr, out, nullptr, N, K, GroupOut{});
  } else if (mid_tile(n_tiles, m_tiles)) {
    hipLaunchKernelGGL((TILE_MID(EPI)), dim3(ceil_div(n_tiles, 2), ceil_div(m_tiles, 4)), dim3(256), 0, st, rc, xv, wv, nullptr, out, nullptr, N, K, GroupOut{});
  } else {
    const BigGrid g = big_grid(ceil_div(n_tiles, 4), m_tiles);
    hipLaunchKernelGGL((TILE_WIDE(EPI)), dim3(g.full + g.halves()), dim3(256), 0, st, rc, xv, wv, nullptr, out, nullptr, N, K, QkvOut{}, g);
  }
}
void launch_gemm_tile(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, float* out, int N, int K) {
  launch_tile<TEPI_F32>(st, rc, x, Wp, out, N, K);
}
void launch_gemm_tile_resid(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, float* x_res, int N, int K) {
  launch_tile<TEPI_RESID>(st, rc, x, Wp, x_res, N, K);
}
// QKV with the rotary epilogue: the same rules, 64 columns per wavefront.  us, WIDE (| as tiles of 256 x 256 alone) | SMALL | MID:
//   1152 x 896 (14 + 2 x 2 heads of 64) at 37, 768, 2048, 4096 rows  19, 22, 19, 21 (24, 31, 34, 35) | 9, 9, 26, 42 | 12, 14, 15, 29
//   1792 x 1184 (20 + 2 x 4 of 64) at 1300, 2000, 4096 rows  23, 24, 26 (.., .., 42) | .. | 17, 18, 36
//   6144 x 2560 (32 + 2 x 8 of 128) at 37, 256, 512, 1024, 1536 rows  (53, 59, .., 64, 66) | 20, 39, .., 115, 171 | 26, 29, 29, 59, 88
//   6144 x 4096 at 512, 640, 1024, 2048 rows  52, 53, 57, 102 (.., 90, 93, 119) | .., 117, 174, 339 | 42, 43, 89, 146
enum QkvShape { QKV_SMALL, QKV_MID, QKV_WIDE };
static QkvShape qkv_shape(int units, int m_tiles) {         // units of 64 columns
  if (small_tile(units, m_tiles)) return QKV_SMALL;
  return mid_tile(units, m_tiles) ? QKV_MID : QKV_WIDE;
}
bool launch_gemm_tile_qkv(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, int N, int K, const QkvOut& qo) {
  if (qo.kvl.mode != 1) return false;
  const int units = ceil_div(N >> 5, 2), m_tiles = ceil_div(rc.max_rows, 32);       // 64 columns
  const QkvShape shape = qkv_shape(units, m_tiles);
  const BigGrid big = big_grid(ceil_div(units, 2), m_tiles);
#define QKV_TILE(DH, WGN, MTW, NW, R)                                                                                  \
  hipLaunchKernelGGL((gemm_tile_qkv_kernel<2, WGN, MTW, 2, 2, R, DH>), dim3(ceil_div(units, WGN), ceil_div(m_tiles, 2 * MTW)), \
                     dim3(64 * NW), 0, st, rc, reinterpret_cast<const bf16x8*>(x), reinterpret_cast<const bf16x8*>(Wp), N, K, qo)
#define QKV_LAUNCH(DH)                                                                                                 \
  if (shape == QKV_SMALL) QKV_TILE(DH, 1, 1, 2, 16);                                                                           \
  else if (shape == QKV_MID) QKV_TILE(DH, 2, 2, 4, 8);                                                                       \
  else hipLaunchKernelGGL((gemm_big_kernel<TEPI_QKV, DH>), dim3(big.full + big.halves()), dim3(256), 0, st, rc, \
                          reinterpret_cast<const bf16x8*>(x), reinterpret_cast<const bf16x8*>(Wp), nullptr, nullptr, nullptr, N, K, qo, big)
  switch (qo.kvl.head_dim) {
    case 32: QKV_LAUNCH(32); break;
    case 64: QKV_LAUNCH(64); break;
    case 128: QKV_LAUNCH(128); break;
    default: return false;
  }
#undef QKV_LAUNCH
#undef QKV_TILE
  return true;
}

void launch_gemm_tile_swiglu(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wg, const bf16_t* Wu,
                             bf16_t* act, int F, int K) {
  const int f_tiles = F >> 5, m_tiles = ceil_div(rc.max_rows, 32);
  const bf16x8* xv = reinterpret_cast<const bf16x8*>(x);
  const bf16x8* gv = reinterpret_cast<const bf16x8*>(Wg);
  const bf16x8* uv = reinterpret_cast<const bf16x8*>(Wu);
  if (small_tile(f_tiles, m_tiles)) {
    hipLaunchKernelGGL((TILE_SMALL_SWIGLU), dim3(f_tiles, ceil_div(m_tiles, 2)), dim3(128), 0, st, rc, xv, gv, uv, nullptr, act, F, K, GroupOut{});
  } else if (mid_tile(f_tiles, m_tiles)) {
    hipLaunchKernelGGL((TILE_MID_SWIGLU), dim3(ceil_div(f_tiles, 2), ceil_div(m_tiles, 4)), dim3(256), 0, st, rc, xv, gv, uv, nullptr, act, F, K, GroupOut{});
  } else {
    const BigGrid g = big_grid(ceil_div(f_tiles, 2), m_tiles);
    hipLaunchKernelGGL((TILE_WIDE(TEPI_SWIGLU)), dim3(g.full + g.halves()), dim3(256), 0, st, rc, xv, gv, uv, nullptr, act, F, K, QkvOut{}, g);
  }
}

// Decode with many rows in flight: fused gate/up + SiLU*mul with the skinny kernel's summation
// chains (see CHAIN above) and, when ssq is set, the folded RMSNorm of that kernel.  Returns
// false (nothing launched) when the shape does not allow it.
// Workgroups of 64 features and 64, 128, 256 or 384 rows, on 4 or 8 wavefronts of 32 or 64 (384: 96) rows x 64 gate / up columns.  Eight
// wavefronts hide the barriers better than four of twice the size (256 rows 45 | 49 us), and the products of a wavefront are too few for
// the LDS reads of the next k-tile at less than 64 rows of them; what is left is LDS traffic, 5 to 7.5 KB for 8 products.  Which rows: the least
// cost in rounds of one workgroup per compute unit (two of 4 wavefronts of 64 rows: cost128x2), times below for one round of each.
// us per launch, skinny kernel | 3-stage ring of one launch form before | 64 | 128 | 128, two per unit | 256 | 384 rows:
//   9728 x 2560 (152 workgroups a row group) at 64, 96, 128 rows 31, 33, 35 | 38, 38, 38 | 28, 38, 41 | 29, 32, 33 | 31, 32, 34
//      at 192, 256, 384 rows 48, 58, 70 | 46, 45, 53 | - | 56, 59, 60 | 47, 52, 51 | 42, 45, 75 | 52, 51, 57
//   14336 x 4096 (224) at 64, 96, 128 rows 52, 67, 78 | 62, 60, 61 | 47, 62, - | 49, 52, 54 | 50, 56, 58
//      at 192, 256, 320, 384 rows 94, 119, 130, 147 | 70, 78, 129, 133 | - | 86, 92, 124, 133 | 79, 86, 109, 117 | 67, 72, 122, 126 | 85, 87, 90, 93
//   8192 x 3072 (128) at 128, 192, 256, 384 rows - | 43, 49, 51, 59 | - | 37, 35, 38, 67 | 38, 37, 40, 58 | 43, 46, 50, 50 | 54, 54, 57, 62
bool launch_gemm_tile_swiglu_chain(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wg, const bf16_t* Wu,
                                   bf16_t* act, int F, int K, const float* ssq, int ssq_stride, float eps) {
  if (K % 128 != 0 || F % 32 != 0) return false;     // quarter boundaries on stage boundaries (BK = 2)
  const int units = ceil_div(F >> 5, 2), m_tiles = ceil_div(rc.max_rows, 32);
  const TileNorm tn{ssq, ssq_stride, K >> 5, 1.0f / (float)K, eps, {}};
#define CHAIN_LAUNCH(WGM, MTW, OCC, R)                                                                                 \
  hipLaunchKernelGGL((gemm_rows_kernel<TEPI_SWIGLU, WGM, MTW, 2, true, OCC, R>), dim3(rows_grid(2 * units, units, ceil_div(m_tiles, WGM * MTW))), \
                     dim3(128 * WGM), 0, st, rc, reinterpret_cast<const bf16x8*>(x), reinterpret_cast<const bf16x8*>(Wg), \
                     reinterpret_cast<const bf16x8*>(Wu), nullptr, act, F, K, tn, units)
  const int rows = rc.max_rows;
  auto rounds = [&](int group_rows, int slots) { return ceil_div(units * ceil_div(rows, group_rows), slots); };
  const int cost128 = 100 * rounds(128, 256), cost128x2 = 153 * rounds(128, 512), cost256 = 130 * rounds(256, 256), cost384 = 172 * rounds(384, 256);
  const int least = std::min({cost128, cost128x2, cost256, cost384});
  if (rows <= 64) CHAIN_LAUNCH(2, 1, 2, 6);
  else if (least == cost128) CHAIN_LAUNCH(4, 1, 1, 6);
  else if (least == cost256) CHAIN_LAUNCH(4, 2, 1, 6);
  else if (least == cost384) CHAIN_LAUNCH(4, 3, 1, 4);
  else CHAIN_LAUNCH(2, 2, 2, 5);
#undef CHAIN_LAUNCH
  return true;
}

// LM head: logits (optional) plus the group records.  One accumulation chain per element whatever the
// tile (k-tiles in order): the choice changes no bit.  False (nothing launched): the skinny kernel is
// the one to use.
// The head is read once (from HBM: its bound up to about 200 rows) and every row group's workgroups run
// beside each other.  Tiles of 256 columns are 2.3 rounds of 151936, 3.9 of two row groups of 128256: past whole rounds they go as halves
// (gemm_rows_kernel).  us per launch, skinny | 64 x 256 | 128 x 256, ring of 3 | 256 x 256 on 8 wavefronts | gemm_rows_kernel of 128 | 192 | 256 rows, all
// measured together with the weights read from HBM; * what the rule takes:
//   151936 x 2560   7 rows 142 | 143* | 154 | 223 | 145 | 161 | 200      64   159 | 153* | 162 | 225 | 150 | 167 | 204     128  195 | 185 | 167 | 223 | 158* | 172 | 207
//                 192      321 | 233 | 222 | 228 | 228 | 183* | 211     256   355 | 288 | 228 | 229 | 236 | 298 | 216*    384  518 | 392 | 311 | 395 | 334 | 306* | 380
//   128256 x 4096   7      189* | 191 | 199 | 265 | 193 | 203 | 251      64   201 | 195* | 200 | 270 | 196 | 209 | 259     128  239 | 239 | 204* | 269 | 198 | 214 | 260
//                 192      424 | 303 | 282 | 275 | 286 | 221* | 266     256   464 | 370 | 283 | 276 | 294 | 381 | 271*    384  693 | 510 | 396 | 506 | 410 | 388* | 479
//   151936 x 2048   7      127 | 126* | 137 | 183 | 130 | 144 | 163      64   140 | 131* | 139 | 183 | 131 | 143 | 169     128  160 | 145 | 142 | 181 | 136* | 146 | 171
//                 192      262 | 179 | 182 | 186 | 185 | 152* | 175     256   289 | 228 | 185 | 188 | 193 | 247 | 178*    384  423 | 313 | 256 | 322 | 270 | 247* | 317
//   151936 x 896    7       58 | 56* | 62 | 94 | 65 | 76 | 93            64    64 | 60* | 63 | 93 | 67 | 74 | 90           128   79 | 71 | 67* | 92 | 69 | 76 | 91
//                 192      111 | 87 | 86 | 96 | 100 | 78* | 93          256   129 | 111 | 91* | 96 | 105 | 130 | 95       384  174 | 151 | 123* | 156 | 145 | 135 | 170
//   50304 x 2048    7       41* | 43 | 45 | 62 | 46 | 50 | 62            64    45 | 43* | 46 | 59 | 47 | 50 | 61           128   59 | 58 | 48 | 59 | 47* | 52 | 62
//                 192       78 | 73 | 66 | 63 | 71 | 55* | 63           256    91 | 88 | 70 | 63 | 75 | 89 | 59*          384  124 | 107 | 100 | 114 | 98 | 92* | 113
//   32032 x 1184    7       21* | 22 | 28 | 35 | 18 | 25 | 28            64    25 | 24* | 28 | 35 | 19 | 24 | 27           128   33 | 24 | 30 | 35 | 20* | 25 | 28
//                 192       30 | 34 | 29 | 34 | 29 | 26* | 28           256    33 | 33 | 30* | 35 | 30 | 34 | 30          384   50 | 44 | 41* | 40 | 48 | 36 | 44
//   50304 x 768     7       17* | 18 | 21 | 28 | 22 | 27 | 31            64    20 | 18* | 22 | 28 | 22 | 26 | 32           128   26 | 26 | 23 | 28 | 24* | 27 | 33
//                 192       34 | 32 | 31 | 29 | 36 | 28* | 34           256    39 | 39 | 33 | 30* | 38 | 46 | 35          384   56 | 48 | 48* | 52 | 49 | 48 | 60
// The skinny kernel reads the weights again for every 4 m-tiles, a grid apart: beyond 128 rows it is slower everywhere.  From 193 to 256 rows of a
// product shorter than 2048: 256 rows on 8 wavefronts where its 256-column groups fill one round (129 .. 256) or their last one, else 128 (128256 x 1024, 501
// groups, at 256 rows 81 | 82; 40960 x 768, 160 groups, 31 | 28; 50304 x 1600, 197 groups, 62 | 53); from 385 to 512 rows for more than 64 groups
// (32000 x 1024, 125 groups, at 512 rows 41 | 39; 4096 x 192, 16 groups, 9.7 | 11.9).  Where another tile is faster than the rule's, it is by 13 % at
// the most (50304 x 768 at 257 rows: 64 x 256), but for heads of few groups: 32032 x 1184 (128 rows at 7 and 64), 4096 x 192 (64 or 128 rows at 512).
bool launch_gemm_tile_logits(hipStream_t st, RowCtx rc, const bf16_t* x, const bf16_t* Wp, float* logits,
                             const GroupOut& go, int V, int K) {
  const int groups = ceil_div(V >> 5, 8), rows = rc.max_rows;            // 256-column groups
  TileNorm lm{};
  lm.go = go;
  if (rows <= 32 && (K >= 3072 || groups < 256)) return false;
#define LM_LAUNCH(KERNEL, MT, THREADS, ...)                                                                              \
  hipLaunchKernelGGL((KERNEL), dim3(ceil_div(groups, 8) * 8 * ceil_div(ceil_div(rows, 32), MT)), dim3(THREADS), 0, st, rc, \
                     reinterpret_cast<const bf16x8*>(x), reinterpret_cast<const bf16x8*>(Wp), nullptr, logits, nullptr, V, K, __VA_ARGS__)
#define LM_ROWS(MTW, R)                                                                                                \
  do {                                                                                                                 \
    const int units = ceil_div(V >> 5, 4), rg = ceil_div(ceil_div(rows, 32), 2 * MTW), full = rows_full(units, rg);                    \
    hipLaunchKernelGGL((gemm_rows_kernel<TEPI_LOGITS, 2, MTW, 4, false, 1, R>), dim3(rows_grid(units, full, rg)), dim3(256), 0, st, rc, \
                       reinterpret_cast<const bf16x8*>(x), reinterpret_cast<const bf16x8*>(Wp), nullptr, logits, nullptr, V, K, lm, full); \
  } while (0)
#define LM_64 gemm_tile_dma_kernel<1, 4, 2, 2, 2, 4, TEPI_LOGITS>
#define LM_128 gemm_tile_dma_kernel<1, 4, 4, 2, 2, 3, TEPI_LOGITS>
#define LM_256 gemm_tile_dma_kernel<2, 4, 4, 2, 2, 4, TEPI_LOGITS>
  auto split = [&](int group_rows) { const int units = ceil_div(V >> 5, 4); return 2 * rows_full(units, ceil_div(rows, group_rows)) < units; };
  const bool full = (groups > 128 && groups <= 256) || groups % 256 == 0 || groups % 256 >= 230;
  const bool tall = (rows <= 256 && full) || (rows > 384 && rows <= 512 && groups > 64);
  if (rows <= 64) LM_LAUNCH(LM_64, 2, 256, go);
  else if (rows <= 128 && (groups < 256 || (K >= 2048 && split(128)))) LM_ROWS(2, 5);
  else if (rows > 128 && (rows <= 192 || (rows > 256 && rows <= 384 && K >= 2048))) LM_ROWS(3, 4);
  else if (rows > 128 && K >= 2048 && (rows <= 256 || (tall && K > 2048))) LM_ROWS(4, 4);
  else if (rows > 128 && tall) LM_LAUNCH(LM_256, 8, 512, go);
  else LM_LAUNCH(LM_128, 4, 256, go);
#undef LM_64
#undef LM_128
#undef LM_256
#undef LM_LAUNCH
  return true;
}

}  // namespace april
