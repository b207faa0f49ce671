// Paged-attention decode for bf16 KV, gfx950.
//
// One workgroup (4 wavefronts) per (row, KV head, KV split of ATT_SPLIT tokens).  The
// wavefronts take the split's 32-token tiles round-robin, each keeps an online softmax
// in registers, the four partial results are merged through LDS in wavefront order;
// when a context spans several splits the merged partials go to a workspace and a small
// second kernel merges them in split order (deterministic: the order of every
// floating-point sum depends on the row's own length only).  The kernel boundary is the
// cheapest device-wide ordering on this chip: publishing the partials behind agent-scope
// fences and letting the last workgroup merge cost more than the extra launch.
//
// Both products run on v_mfma_f32_16x16x32_bf16, computed transposed so that no
// operand has to be re-laid between them:
//   S^T[token, head] = K[token, :] . Q[head, :]      A = K fragment, B = Q^T fragment
//   O^T[dim,  head]  = V^T[dim, token] . P^T[token, head]
// The accumulator of the first product (lane l: head l%16, tokens 4*(l/16)+i of a
// 16-token page) is, after exp(), directly the B operand of the second product: its
// k index runs over (page A tokens 4g..4g+3, page B tokens 4g..4g+3), and the V^T
// fragment is loaded with the same token order.
//
// FUSED (decode iterations): the kernel also does the rotary embedding and the KV append of
// the row's new token, so no separate kernel runs between the QKV GEMM and attention.  Every
// workgroup sums the split-K partials of its query heads and rotates them; the workgroup of
// the last KV split computes the new token's rotated key and its value, stores them in the
// page as bf16, and substitutes exactly those bf16 values into the fragments of the tile
// that holds the position, so the products are bit-identical to reading them back.
// (Prefill rows attend to each other's new keys: there the QKV projection's epilogue rotates and appends.)
//
// KV page layout (written by rope_append_kernel or here, mode 1), per (page, KV head):
//   K: MFMA A-fragment order  [d/32][lane = t + 16*((d%32)/8)][d%8]   -> 1 KiB coalesced loads
//   V: transposed             [d][t]                                 -> 8-byte loads, 512 B/wave coalesced
#include <type_traits>

#include "kernels.h"

namespace april {

#ifndef ATT_SPLIT_64
#define ATT_SPLIT_64 1024
#endif
#ifndef ATT_SPLIT_128
#define ATT_SPLIT_128 4096
#endif
// tokens per KV split, a multiple of 1024 (a lane holds one page id per 1024 tokens of the split).
// head_dim 64 (small model, 2 KV heads): 2048 was 1.6 % slower end to end than 1024; 512: 7 % slower
// on long rows.  head_dim 128, launched over the length-sorted work list: the kernel itself is
// 1 % slower with 4096-token splits than with 1024 (160.8 against 158.7 us on the 4.4 B
// configuration), but few rows then need the merge kernel at all, and the run is 1 % faster end to
// end on each of the three wide configurations (before the work list, on a grid launch, 2048-token
// splits cost 4.5 % on a ragged batch).
constexpr int att_split(int dh) { return dh == 64 ? ATT_SPLIT_64 : (dh == 128 ? ATT_SPLIT_128 : 1024); }
// wavefronts per workgroup (8 for head_dim 64: one row of 1000 tokens 7.2 against 7.5 us, but 192 rows of 40 tokens 11.0 against 6.7)
#ifndef ATT_WAVES_128
#define ATT_WAVES_128 4
#endif
constexpr int att_waves(int dh, bool fused) { return dh == 128 ? ATT_WAVES_128 : 4; }

// q_src of the kernel: FUSED: the QKV GEMM's split-K partials, fp32 [n_partials][rows][(Hq + 2 Hkv) * dh]; else
// the rotated queries, fp32 [rows][Hq * dh].
struct AttnFuse {              // the rest of the fused rotary + append (FUSED only)
  int n_partials;
  size_t partial_stride;
  const float* rope_cos;       // [pos][dh/2]
  const float* rope_sin;
};

template <int DH, bool FUSED>
__global__ __launch_bounds__(64 * att_waves(DH, FUSED)) __attribute__((amdgpu_waves_per_eu(2))) void attn_decode_kernel(
    const int4* __restrict__ items, const int2* __restrict__ ctl_p, const int* __restrict__ block_table,
    const float* __restrict__ q_src, bf16_t* kv_pool, int max_blocks, int Hkv, int Hq, int layer, RowCtx rc, int row_base,
    KVLayout L, bf16_t* __restrict__ out, float* __restrict__ ws, int max_splits, AttnFuse fz) {
  constexpr int KC = DH / 32;      // k-chunks of the QK product
  constexpr int DT = DH / 16;      // dim tiles of the PV product
  constexpr int REC = 32 + 16 * DH;   // floats of one partial result: m[16], l[16], o[16][DH]
  constexpr int ATT_WAVES = att_waves(DH, FUSED);
  constexpr int RS = DH + 4;          // padded row stride of O in LDS
  constexpr int LREC = 32 + 16 * RS;
  __shared__ float lds[ATT_WAVES * LREC];
  constexpr int QS = DH + 8;          // padded row stride of the rotated queries
  __shared__ __align__(16) bf16_t s_q[FUSED ? 16 * QS : 8], s_knew[DH], s_vnew[DH];
  // Workgroup ids are dealt to the 8 XCDs in turn, so with a row count that is a multiple of 8 the
  // plain mapping would put every (KV head, split) of a row on one XCD and a long row would
  // overload it.  Rotating the row index by the other two coordinates spreads a row's
  // workgroups over the XCDs (a bijection of blockIdx.x for fixed y and z).
  //
  // With a work list (items != nullptr; 1-D launch) the scheduler kernel has listed this
  // iteration's (row, split) pairs longest first: entry 0 holds their number, entry 1 + i =
  // {row, split, slot, position}.  Workgroup id = item * n_kv_heads + KV head, so the long items
  // start first, the launch ends on the short ones, no workgroup is launched for a split its row
  // does not have, and the KV heads of one item go to different XCDs.
  int kvh, split, wr, slot, pos;
  if (items != nullptr) {
    const int item = (int)blockIdx.x / Hkv;
    kvh = (int)blockIdx.x - item * Hkv;
    const int4 head = items[0], it = items[1 + item];
    const int2 ctl = *ctl_p;
    if (ctl.y || item >= head.x) return;
    wr = __builtin_amdgcn_readfirstlane(it.x);
    split = __builtin_amdgcn_readfirstlane(it.y);
    slot = __builtin_amdgcn_readfirstlane(it.z);
    pos = __builtin_amdgcn_readfirstlane(it.w);
  } else {
    kvh = blockIdx.y; split = blockIdx.z;
    wr = (int)((blockIdx.x + blockIdx.y + 3u * blockIdx.z) % gridDim.x);     // wr: workspace row
    // the row arrays hold max_rows entries: fetch them together with the control word
    const int slot_raw = rc.row_slot[row_base + wr], pos_raw = rc.row_pos[row_base + wr];
    ROW_GUARD(rc, row_base + wr);
    slot = slot_raw; pos = pos_raw;
  }
  const int r = row_base + wr;
  const int ctx = pos + 1;
  constexpr int ATT_SPLIT = att_split(DH), PR = ATT_SPLIT / 1024;
  static_assert(ATT_SPLIT % 1024 == 0 && PR >= 1, "split length");
  const int n_splits = (ctx + ATT_SPLIT - 1) / ATT_SPLIT;
  if (split >= n_splits) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), hh = lane & 15, g = lane >> 4;
  const int G = Hq / Hkv;
  const int t_begin = split * ATT_SPLIT, t_end = min(ctx, t_begin + ATT_SPLIT);
  const int n_tiles = (t_end - t_begin + 31) >> 5;
  const int n_pages = (t_end - t_begin + 15) >> 4;
  const size_t blk_elems = (size_t)16 * DH;
  const bf16_t* kbase = kv_pool + (size_t)layer * L.layer_stride;
  const bf16_t* vbase = kbase + L.kv_stride;

  // page ids of this split: lane i holds page i (one vector load instead of a scalar
  // load per tile inside the loop)
  const int* bt = block_table + (size_t)slot * max_blocks + (t_begin >> 4);
  int my_page[PR];
#pragma unroll
  for (int q = 0; q < PR; ++q) { const int i = q * 64 + lane; my_page[q] = bt[i < n_pages ? i : n_pages - 1]; }

  // A wavefront takes tiles wave, wave + ATT_WAVES, ... of the split.  Every load inside load_tile
  // is unconditional (a missing second page is clamped), so the wait counts around it are static.
  auto load_tile = [&](int tile, bf16x8 (&kk)[2][KC], bf16x4 (&vv)[2][DT]) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      int pl = 2 * tile + p;                                   // page within the split
      pl = pl < n_pages ? pl : n_pages - 1;                    // a missing second page re-reads the last one
      const int pls = __builtin_amdgcn_readfirstlane(pl);
      int page = __builtin_amdgcn_readlane(my_page[0], pls & 63);
#pragma unroll
      for (int q = 1; q < PR; ++q)
        if ((pls >> 6) == q) page = __builtin_amdgcn_readlane(my_page[q], pls & 63);
      const size_t off = ((size_t)page * Hkv + kvh) * blk_elems;
      const bf16x8* kp = reinterpret_cast<const bf16x8*>(kbase + off);
      const bf16x4* vp = reinterpret_cast<const bf16x4*>(vbase + off);
#pragma unroll
      for (int c = 0; c < KC; ++c) kk[p][c] = kp[c * 64 + lane];
#pragma unroll
      for (int d = 0; d < DT; ++d) vv[p][d] = vp[(d * 16 + hh) * 4 + g];
    }
  };

  // This wavefront's tiles wave, wave + ATT_WAVES, ...: R of them in flight, tile i in register slot i % R.
  constexpr int R = 2;         // (head_dim 64, one row of 400 tokens: 5.45 us with 2, 5.85 with 3; 128 has no registers for 3)
  bf16x8 kf[R][2][KC];
  bf16x4 vf[R][2][DT];
  const int cnt = (n_tiles - wave + ATT_WAVES - 1) / ATT_WAVES;      // (none: a clamped tile is requested, never used)
  auto request = [&](int u, int i) { load_tile(min(wave + i * ATT_WAVES, n_tiles - 1), kf[u], vf[u]); };
  auto first_tiles = [&]() {
    request(0, 0);
#pragma unroll
    for (int u = 1; u < R; ++u)
      if (u < cnt) request(u, u);
  };

  // Q^T fragments: lane holds q[head hh][32c + 8g .. +7]; heads beyond the group are zero.
  constexpr int HALF = DH / 2;
  const bool last_split = split == n_splits - 1;
  bf16x8 qf[KC];
  if (FUSED) {
    // The workgroup sums the partials of its query heads and rotates them, one pair (i, i + DH / 2) of a head per
    // thread, and with the last split the new token's key (rotated) and value too: "heads" G and G + 1.  Everyone
    // then reads the bf16 queries from LDS.  Loads complete in order, and the partials are requested before the
    // first tiles, which need the page ids: the rotation runs while the tiles arrive.  (With every wavefront summing
    // all of its lanes' queries itself, in 16-byte pieces of 14 rows, the L1 traffic and the round trips of more than
    // four partials were most of a short row's time.  Rows of 40 tokens, 14 + 2 heads of 64 in 4 partials, 20 + 4 in 6,
    // 32 + 8 of 128 in 2, us per launch before / now: 1 row 5.2, 6.8, 6.0 / 4.3, 4.4, 5.2; 96 rows 5.6, 10.7, 13.6 /
    // 4.7, 5.8, 11.9.)
    constexpr int THREADS = 64 * ATT_WAVES, U = 2;
    const int ncol = (Hq + 2 * Hkv) * DH, n_pairs = (last_split ? G + 2 : G) * HALF;
    const float* src = q_src + (size_t)r * ncol;
    const float* cs = fz.rope_cos + (size_t)pos * HALF;
    const float* sn = fz.rope_sin + (size_t)pos * HALF;
    const int tin = pos & 15, np = fz.n_partials, new_page = bt[(pos - t_begin) >> 4];     // (the last split's only)
    constexpr int QB = 8;                     // partials requested together
    auto trip = [&](int p0, auto first) {
      const float* col[U];
      float cv[U], sv[U], a[U], b[U], va[U][QB], vb[U][QB];
      int hd[U], ii[U];
      auto load = [&](int q0) {
#pragma unroll
        for (int q = 0; q < QB; ++q)
          if (q0 + q < np) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const float* c = col[u] + (size_t)(q0 + q) * fz.partial_stride;
              va[u][q] = c[0]; vb[u][q] = c[HALF];
            }
          }
      };
      auto add = [&](int q0) {                // in the order p = 0, 1, ...
#pragma unroll
        for (int q = 0; q < QB; ++q)
          if (q0 + q < np) {
#pragma unroll
            for (int u = 0; u < U; ++u) { a[u] += va[u][q]; b[u] += vb[u][q]; }
          }
      };
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = min(p0 + u * THREADS + (int)threadIdx.x, n_pairs - 1);
        hd[u] = e / HALF; ii[u] = e % HALF;
        col[u] = src + (size_t)(hd[u] < G ? kvh * G + hd[u] : Hq + (hd[u] - G) * Hkv + kvh) * DH + ii[u];
        cv[u] = cs[ii[u]]; sv[u] = sn[ii[u]];
        a[u] = b[u] = 0.f;
      }
      load(0);
      __builtin_amdgcn_sched_barrier(0);
      if (first) first_tiles();
      __builtin_amdgcn_sched_barrier(0);
      add(0);
      for (int q0 = QB; q0 < np; q0 += QB) { load(q0); add(q0); }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (p0 + u * THREADS + (int)threadIdx.x >= n_pairs) continue;
        const int i = ii[u];
        const bf16_t ra = (bf16_t)rope_first(a[u], b[u], cv[u], sv[u]), rb = (bf16_t)rope_second(a[u], b[u], cv[u], sv[u]);
        if (hd[u] < G) {
          s_q[hd[u] * QS + i] = ra;
          s_q[hd[u] * QS + i + HALF] = rb;
        } else {
          // the new token, to LDS and to its page
          const bool key = hd[u] == G;
          const bf16_t x = key ? ra : (bf16_t)a[u], y = key ? rb : (bf16_t)b[u];
          bf16_t* dst = key ? s_knew : s_vnew;
          dst[i] = x;
          dst[i + HALF] = y;
          kv_pool[L.at(layer, key ? 0 : 1, new_page, kvh, tin, i)] = x;
          kv_pool[L.at(layer, key ? 0 : 1, new_page, kvh, tin, i + HALF)] = y;
        }
      }
    };
    trip(0, std::true_type{});
    for (int p0 = U * THREADS; p0 < n_pairs; p0 += U * THREADS) trip(p0, std::false_type{});
    __syncthreads();
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      qf[c] = bf16x8{};
      if (hh < G) qf[c] = *reinterpret_cast<const bf16x8*>(s_q + hh * QS + 32 * c + 8 * g);
    }
  } else {
    first_tiles();
    __builtin_amdgcn_sched_barrier(0);
    const int hq = hh < G ? hh : G - 1;
    const float* q = q_src + (size_t)r * Hq * DH + (size_t)(kvh * G + hq) * DH + 8 * g;
    f32x4 qa[KC][2];
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      qa[c][0] = *reinterpret_cast<const f32x4*>(q + 32 * c);
      qa[c][1] = *reinterpret_cast<const f32x4*>(q + 32 * c + 4);
    }
#pragma unroll
    for (int c = 0; c < KC; ++c)
#pragma unroll
      for (int j = 0; j < 8; ++j) qf[c][j] = hh < G ? (bf16_t)qa[c][j >> 2][j & 3] : (bf16_t)0.f;
  }
  // Softmax in base 2, the scale folded into one multiply-add per score.  The running maximum of a head may lag the
  // true one by up to 2^8 (the conditional rescaling known from published flash-attention kernels; probabilities are
  // then at most 256, which costs no precision in bf16 or fp32), so that a tile needs no shuffle unless a
  // score passes it; each lane sums its own tokens' probabilities until the end.
  const float c2 = 1.4426950408889634f / sqrtf((float)DH);
  constexpr float RESCALE = 8.0f;
  float m_run = -INFINITY, l_run = 0.f;
  f32x4 oacc[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) oacc[d] = f32x4{};

  // Tile i of this wavefront, in slot u: scores, online softmax, PV.  last (a compile-time truth): it may be the
  // split's last tile, the one with masked tokens and the new token.
  auto compute_tile = [&](int u, int i, auto last) {
    const int tile = wave + i * ATT_WAVES, t0 = t_begin + tile * 32;
    if (FUSED && last && last_split && tile == n_tiles - 1) {
      // the tile that holds the new token: take its key / value from LDS (the page copy may
      // not be visible yet); same bf16 values as the page now holds
      const int pp = ((pos - t_begin) >> 4) & 1, tin = pos & 15;
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        if (p != pp) continue;
        if (hh == tin) {
#pragma unroll
          for (int c = 0; c < KC; ++c) kf[u][p][c] = *reinterpret_cast<const bf16x8*>(s_knew + 32 * c + 8 * g);
        }
        if ((tin >> 2) == g) {
#pragma unroll
          for (int d = 0; d < DT; ++d) {
            const bf16_t nv = s_vnew[d * 16 + hh];
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (j == (tin & 3)) vf[u][p][d][j] = nv;
          }
        }
      }
    }
    f32x4 sacc[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      sacc[p] = f32x4{};
#pragma unroll
      for (int c = 0; c < KC; ++c)
        sacc[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[u][p][c], qf[c], sacc[p], 0, 0, 0);
    }
    float sv[8];
    float mx = -INFINITY;
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int tok = t0 + p * 16 + 4 * g + i;
        const float v = !last || tok < t_end ? sacc[p][i] : -INFINITY;
        sv[p * 4 + i] = v;
        mx = fmaxf(mx, v);
      }
    mx *= c2;
    if (__any(mx > m_run + RESCALE)) {           // always in a wavefront's first tile
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const bool grow = mx > m_run + RESCALE;    // the same for the four lanes of a head
      const float corr = grow ? __builtin_amdgcn_exp2f(m_run - mx) : 1.0f;
      m_run = grow ? mx : m_run;
      l_run *= corr;
#pragma unroll
      for (int d = 0; d < DT; ++d) oacc[d] *= corr;
    }
    float rs[2] = {0.f, 0.f};
    bf16x8 pf;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float pe = __builtin_amdgcn_exp2f(__fmaf_rn(sv[e], c2, -m_run));
      rs[e & 1] += pe;
      pf[e] = (bf16_t)pe;
    }
    l_run += rs[0] + rs[1];
#pragma unroll
    for (int d = 0; d < DT; ++d) {
      bf16x8 af;
#pragma unroll
      for (int j = 0; j < 4; ++j) { af[j] = vf[u][0][d][j]; af[4 + j] = vf[u][1][d][j]; }
      oacc[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, pf, oacc[d], 0, 0, 0);
    }
  };
  // Steady state: a slot is requested again as soon as its tile is done, R - 1 tiles in flight behind the one in
  // use and no branch between them, so that every wait is for one tile only (with tiles moved from slot to slot
  // a wavefront waited in each step for what it had requested in the step before: one row of 400 tokens, 14 + 2 heads of
  // 64, 20 + 4 of 64, 32 + 4 of 128: 6.7, 8.3, 10.3 us per launch, with this loop and the start above 5.4, 5.4, 7.7; 192 rows of
  // 1000 tokens 25.1, 45.5, 84.4 / 24.5, 42.3, 78.9).  The rest has no
  // successor to request, and no wavefront ends waiting for a tile that it does not use.
  int i = 0;
  for (; i + 2 * R <= cnt; i += R) {
#pragma unroll
    for (int u = 0; u < R; ++u) {
      compute_tile(u, i + u, std::false_type{});
      __builtin_amdgcn_sched_barrier(0);
      request(u, i + R + u);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int q = 0; q < 2 * R - 1; ++q)
    if (i + q < cnt) {
      compute_tile(q % R, i + q, std::true_type{});
      if (q < R - 1 && i + q + R < cnt) request(q % R, i + q + R);
    }

  // ---- merge the wavefronts of this workgroup through LDS, in wavefront order -----------
  // Every wavefront publishes (m, l, O); then each merges its share of the dim tiles (tile d
  // goes to wavefront d % ATT_WAVES) and writes it out, so the tail of a workgroup's life is
  // shared by all of them.  Rows of O are padded by 4 floats in LDS: with a stride of DH floats
  // the 16 heads of a lane group would all hit the same banks.
  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);
  {
    float* my = lds + wave * LREC;
    if (g == 0) { my[hh] = m_run; my[16 + hh] = l_run; }
#pragma unroll
    for (int d = 0; d < DT; ++d) *reinterpret_cast<f32x4*>(my + 32 + hh * RS + d * 16 + 4 * g) = oacc[d];
  }
  __syncthreads();
  float M = lds[hh];
#pragma unroll
  for (int w = 1; w < ATT_WAVES; ++w) M = fmaxf(M, lds[w * LREC + hh]);
  float wgt[ATT_WAVES], lsum = 0.f;
#pragma unroll
  for (int w = 0; w < ATT_WAVES; ++w) {
    wgt[w] = __builtin_amdgcn_exp2f(lds[w * LREC + hh] - M);
    lsum += wgt[w] * lds[w * LREC + 16 + hh];
  }
  const int K = Hq * DH;
  const float inv = 1.0f / lsum;
  float* rec = ws + (((size_t)wr * Hkv + kvh) * max_splits + split) * REC;     // several splits: (m, l, O) for the merge kernel
  for (int d = wave; d < DT; d += ATT_WAVES) {
    f32x4 o = f32x4{};
#pragma unroll
    for (int w = 0; w < ATT_WAVES; ++w)
      o += *reinterpret_cast<const f32x4*>(lds + w * LREC + 32 + hh * RS + d * 16 + 4 * g) * wgt[w];
    if (n_splits == 1) {
      if (hh < G) {
        bf16x4 ob;
#pragma unroll
        for (int i = 0; i < 4; ++i) ob[i] = (bf16_t)(o[i] * inv);
        *reinterpret_cast<bf16x4*>(out + act_index<true>(r, (kvh * G + hh) * DH + d * 16 + 4 * g, K)) = ob;
      }
    } else if (hh < G) {
      // record layout [dim tile][head][16 dims]: the lanes of one store cover consecutive
      // addresses, and only the G heads of the group are written (and read back)
      *reinterpret_cast<f32x4*>(rec + 32 + (d * 16 + hh) * 16 + 4 * g) = o;
    }
  }
  if (n_splits > 1 && wave == 0 && g == 0) { rec[hh] = M; rec[16 + hh] = lsum; }
}

// Merge of the per-split partial results of the rows whose context spans several splits
// (one wavefront per (row, KV head); rows with a single split were finished by the main
// kernel).  Split order, so a row's result depends on its own length only.
template <int DH>
__global__ __launch_bounds__(64) void attn_merge_kernel(RowCtx rc, int row_base, int Hkv, int Hq,
                                                        bf16_t* __restrict__ out, const float* __restrict__ ws,
                                                        int max_splits) {
  constexpr int DT = DH / 16;
  constexpr int REC = 32 + 16 * DH;
  const int wr = blockIdx.x, r = row_base + wr, kvh = blockIdx.y;
  const int pos = rc.row_pos[r];
  ROW_GUARD(rc, r);
  constexpr int ATT_SPLIT = att_split(DH);
  const int n_splits = (pos + ATT_SPLIT) / ATT_SPLIT;          // ceil((pos + 1) / ATT_SPLIT)
  if (n_splits == 1) return;
  const int lane = threadIdx.x, hh = lane & 15, g = lane >> 4;
  const int G = Hq / Hkv, K = Hq * DH;
  const float* base = ws + ((size_t)wr * Hkv + kvh) * max_splits * REC;
  // every load of the merge is independent of the others: issue them in batches
  float M = -INFINITY;
#pragma unroll
  for (int k = 0; k < 8; ++k) {                      // max_splits <= 32: lane group g takes splits g, g+4, ...
    const int si = g + 4 * k;
    M = fmaxf(M, base[(size_t)(si < n_splits ? si : n_splits - 1) * REC + hh]);
  }
  M = fmaxf(M, __shfl_xor(M, 16, 64));
  M = fmaxf(M, __shfl_xor(M, 32, 64));
  float lsum = 0.f;
  f32x4 acc[DT];
#pragma unroll
  for (int d = 0; d < DT; ++d) acc[d] = f32x4{};
  for (int i0 = 0; i0 < n_splits; i0 += 2) {
    float mi[2], li[2];
    f32x4 o[2][DT];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const float* p = base + (size_t)(i0 + u < n_splits ? i0 + u : n_splits - 1) * REC;
      mi[u] = p[hh];
      li[u] = p[16 + hh];
#pragma unroll
      for (int d = 0; d < DT; ++d)
        o[u][d] = hh < G ? *reinterpret_cast<const f32x4*>(p + 32 + (d * 16 + hh) * 16 + 4 * g) : f32x4{};
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const float wgt = i0 + u < n_splits ? __builtin_amdgcn_exp2f(mi[u] - M) : 0.f;
      lsum += wgt * li[u];
#pragma unroll
      for (int d = 0; d < DT; ++d) acc[d] += o[u][d] * wgt;
    }
  }
  if (hh < G) {
    const float inv = 1.0f / lsum;
#pragma unroll
    for (int d = 0; d < DT; ++d) {
      bf16x4 o;
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = (bf16_t)(acc[d][i] * inv);
      *reinterpret_cast<bf16x4*>(out + act_index<true>(r, (kvh * G + hh) * DH + d * 16 + 4 * g, K)) = o;
    }
  }
}

// ---------------------------------------------------------------------------
// Causal attention of prefill rows, tiled over queries.
//
// The decode kernel serves one query position per workgroup; run over the rows of a prompt it
// reads the prompt's keys and values once per position.  Here a workgroup owns a tile of query
// positions of one (sequence, KV head) and streams the keys / values 0 .. last position of the
// tile once, for all of them and for all query heads of the KV head.
//
// Transposed products as in the decode kernel, on v_mfma_f32_32x32x16_bf16:
//   S^T[token, column] = K . Q^T,  O^T[dim, column] = V^T . P^T,
// column = position_in_tile * GP + head, GP = heads per KV head rounded up to a power of two.  A
// wavefront owns PF_CT = 2 tiles of 32 columns (64 / GP positions), the four wavefronts of a
// workgroup consecutive positions.  The pages of a stage of 64 tokens are copied to LDS as they lie
// (global_load_lds, two stage buffers, two workgroups per compute unit), and a fragment read from
// there feeds both column tiles: with one, the LDS reads alone would take the matrix cores' time.
//
// Row r of the first product is given the token 16 (r / 16) + 8 ((r / 4) % 2) + 4 ((r / 8) % 2) + r % 4
// (an address permutation of the K fragment), so that the accumulator registers 8 s .. 8 s + 7 of a
// lane are the tokens 16 s + 8 (lane / 32) .. + 7: converted to bf16 in place they are the B operand
// of the second product, whose V fragment is then one 16-byte read.
//
// Every column runs its own online softmax, in base 2 with the scale folded into one multiply-add
// per score.  The running maximum may lag the true one by up to 2^8 (the conditional rescaling known from
// published flash-attention kernels): the accumulators are rescaled only when a column's maximum passes its running one by more (probabilities are then at most 256,
// which costs no precision in bf16 or fp32), by exactly 1 for the columns that did not.  Each
// lane sums its own tokens' probabilities; the halves of a column meet once at the end.  Positions beyond
// the column's own are masked, in the stages that hold any.  A column's result depends on its own
// prefix only.  (Its summation order differs from the decode kernel's; so does the prefill GEMM's.)
//
// Measured per launch of 16 k rows, against a kernel on 16x16x32 products whose wavefronts each
// loaded every K / V fragment from the caches and rescaled in every 32-token step: prompts of
// 4500-8000 tokens, 32 + 8 heads of 128, 2123 -> 879 us (640 TFLOP/s: the exponentials and
// conversions of two wavefronts per SIMD beside the products); 900-4400 tokens, 14 + 2 heads of 64,
// 468 -> 162 us; 1-1999 tokens, 32 + 8 heads of 128, 574 -> 258 us.
// ---------------------------------------------------------------------------
__device__ inline void copy_piece_to_lds(const bf16x8* src_lane, bf16x8* lds_base) {   // 64 lanes x 16 bytes
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_global_load_lds(src_lane, lds_base, 16, 0, 0);
#else
  (void)src_lane; (void)lds_base;
#endif
}
constexpr int PF_CT = 2;                  // column tiles of 32 per wavefront
constexpr int PF_STAGE = 64;              // tokens per stage

template <int DH, int GP>
__global__ __launch_bounds__(256, 2) void attn_prefill_kernel(const int4* __restrict__ items, Slots s,
                                                              const bf16_t* __restrict__ qb,
                                                              const bf16_t* __restrict__ kv_pool, KVLayout L, int layer,
                                                              int Hq, bf16_t* __restrict__ out) {
  constexpr int KC = DH / 16, DT = DH / 32, CT = PF_CT, NP = PF_STAGE / 16;
  constexpr int PPT = 32 / GP;            // positions per column tile
  constexpr int PPW = CT * PPT;           // positions per wavefront
  constexpr int PIECES = DH / 32;         // KiB of K (or V) per page
  constexpr float RESCALE = 8.0f;
  __shared__ bf16x8 lds[2][2][NP][PIECES * 64];      // [buffer][K | V][page][16-byte piece]
  const int4 it = items[blockIdx.x];      // {slot, first row of the sequence, tokens of the sequence, first position of the tile}
  const int slot = it.x, row0 = it.y, nt = it.z, q0 = it.w;
  const int kvh = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), cl = lane & 31, hf = lane >> 5;
  const int Hkv = L.n_kv_heads, G = Hq / Hkv;
  const int wq0 = q0 + wave * PPW;        // this wavefront's first position (it may lie beyond the sequence: it then only copies)
  const int wlast = wq0 < nt ? min(nt, wq0 + PPW) - 1 : -1;
  const int glast = min(nt, q0 + 4 * PPW) - 1;       // last position of the workgroup
  const size_t blk_elems = (size_t)16 * DH;
  const bf16_t* kbase = kv_pool + (size_t)layer * L.layer_stride;
  const bf16_t* vbase = kbase + L.kv_stride;
  const int* bt = s.block_table + (size_t)slot * s.max_blocks;
  const int last_page = glast >> 4;
  const int n_stages = glast / PF_STAGE + 1;

  int my_page = bt[lane < last_page ? lane : last_page];     // page ids of 16 stages, one per lane
  auto issue = [&](int st) {
    const int buf = st & 1;
    bf16x8* base = &lds[buf][0][0][0];
#pragma unroll
    for (int u = 0; u < 2 * NP * PIECES / 4; ++u) {
      const int idx = wave + 4 * u;                           // piece of the stage: [K | V][page][KiB]
      const int kv = idx / (NP * PIECES), pg = (idx / PIECES) % NP, sub = idx % PIECES;
      int pl = st * NP + pg;
      pl = pl < last_page ? pl : last_page;                   // pages past the end re-read the last one (masked)
      const int page = __builtin_amdgcn_readlane(my_page, __builtin_amdgcn_readfirstlane(pl) & 63);
      const bf16_t* src = (kv ? vbase : kbase) + ((size_t)page * Hkv + kvh) * blk_elems + sub * 512;
      copy_piece_to_lds(reinterpret_cast<const bf16x8*>(src) + lane, base + idx * 64);
    }
  };
  issue(0);

  // query fragments: column cl of tile ct = (position, head); lane half hf holds dims 16 c + 8 hf .. + 7
  int qpos[CT];
  bool qok[CT];
  bf16x8 qf[CT][KC];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const int p = wq0 + ct * PPT + cl / GP, h = cl % GP;
    qok[ct] = p < nt && h < G;
    qpos[ct] = p < nt ? p : nt - 1;
    const int hc = h < G ? h : G - 1;
    const bf16_t* q = qb + (size_t)(row0 + qpos[ct]) * Hq * DH + (size_t)(kvh * G + hc) * DH + 8 * hf;
#pragma unroll
    for (int c = 0; c < KC; ++c) {
      const bf16x8 v = *reinterpret_cast<const bf16x8*>(q + 16 * c);
      qf[ct][c] = qok[ct] ? v : bf16x8{};
    }
  }
  const float c2 = 1.4426950408889634f / sqrtf((float)DH);   // scores to base-2 exponents
  float m_run[CT], l_run[CT];
  f32x16 oacc[CT][DT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    m_run[ct] = -INFINITY; l_run[ct] = 0.f;
#pragma unroll
    for (int d = 0; d < DT; ++d) oacc[ct][d] = f32x16{};
  }
  // K fragment: this lane's row of the product is token kt of page cl / 16 (see above)
  const int kt = (((cl >> 2) & 1) << 3) + (((cl >> 3) & 1) << 2) + (cl & 3);
  const int k_piece = kt + 16 * hf, v_piece = cl * 2 + hf;

  for (int st = 0; st < n_stages; ++st) {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_s_waitcnt(0x0f70);          // vmcnt(0): this wavefront's copies of the stage have landed
#endif
    __builtin_amdgcn_s_barrier();                // everyone's have, and everyone is done with the other buffer
    asm volatile("" ::: "memory");
    if (st + 1 < n_stages) {
      if (((st + 1) & 15) == 0) {                // the next stage opens a new group of 64 pages
        const int i = (st + 1) * NP + lane;
        my_page = bt[i < last_page ? i : last_page];
      }
      issue(st + 1);
    }
    const int buf = st & 1;
#pragma unroll
    for (int half = 0; half < PF_STAGE / 32; ++half) {
      const int t0 = st * PF_STAGE + half * 32;
      if (t0 > wlast) continue;                  // beyond every position of this wavefront
      const bf16x8* kl = &lds[buf][0][half * 2 + (cl >> 4)][k_piece];
      f32x16 sacc[CT];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) sacc[ct] = f32x16{};
#pragma unroll
      for (int c = 0; c < KC; ++c) {
        const bf16x8 kf = kl[(c >> 1) * 64 + 32 * (c & 1)];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) sacc[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ct][c], sacc[ct], 0, 0, 0);
      }
      bf16x8 pf[CT][2];
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        if (t0 + 31 > wq0 + ct * PPT) {          // some column of the tile does not see all 32 tokens
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (t0 + 16 * (i >> 3) + 8 * hf + (i & 7) > qpos[ct]) sacc[ct][i] = -INFINITY;
        }
        float mx = sacc[ct][0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, sacc[ct][i]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * c2;
        const bool grow = mx > m_run[ct] + RESCALE;           // always in the first tile: token 0 is visible to every position
        if (__any(grow)) {
          const float corr = grow ? __builtin_amdgcn_exp2f(m_run[ct] - mx) : 1.0f;
          m_run[ct] = grow ? mx : m_run[ct];
          l_run[ct] *= corr;
#pragma unroll
          for (int d = 0; d < DT; ++d) oacc[ct][d] *= corr;
        }
        float rs[2] = {0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float pe = __builtin_amdgcn_exp2f(__fmaf_rn(sacc[ct][i], c2, -m_run[ct]));
          rs[i & 1] += pe;
          pf[ct][i >> 3][i & 7] = (bf16_t)pe;
        }
        l_run[ct] += rs[0] + rs[1];
      }
#pragma unroll
      for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const bf16x8 vf = lds[buf][1][half * 2 + k][d * 64 + v_piece];
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) oacc[ct][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[ct][k], oacc[ct][d], 0, 0, 0);
        }
    }
    asm volatile("" ::: "memory");
  }
  const int K = Hq * DH;
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const float inv = 1.0f / (l_run[ct] + __shfl_xor(l_run[ct], 32, 64));
    const int r = row0 + qpos[ct], h = cl % GP;
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
      for (int q = 0; q < 4; q += 2) {
        // the lane halves hold alternating groups of 4 dims: they trade one, so that each stores 8
        // consecutive dims (16 bytes of the fragment-tiled layout)
        union { bf16x4 v[2]; unsigned u[4]; bf16x8 w; } own, st8;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          own.v[0][e] = (bf16_t)(oacc[ct][d][4 * q + e] * inv);
          own.v[1][e] = (bf16_t)(oacc[ct][d][4 * q + 4 + e] * inv);
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const unsigned give = hf ? own.u[e] : own.u[2 + e], got = __shfl_xor((int)give, 32, 64);
          st8.u[e] = hf ? got : own.u[e];
          st8.u[2 + e] = hf ? own.u[2 + e] : got;
        }
        if (qok[ct]) *reinterpret_cast<bf16x8*>(out + act_index<true>(r, (kvh * G + h) * DH + d * 32 + 8 * (q + hf), K)) = st8.w;
      }
  }
}

// positions per workgroup of the prefill attention for a model with `group` query heads per KV head
int attn_prefill_tile(int group) {
  int gp = 1;
  while (gp < group) gp <<= 1;
  return 4 * PF_CT * (32 / gp);
}

void launch_attn_prefill(hipStream_t st, const int4* items, int n_items, Slots s, const bf16_t* q,
                         const bf16_t* kv_pool, KVLayout kvl, int layer, int n_q_heads, bf16_t* out) {
  if (n_items <= 0) return;
  dim3 grid(n_items, kvl.n_kv_heads);
  const int G = n_q_heads / kvl.n_kv_heads;
  int gp = 1;
  while (gp < G) gp <<= 1;
#define ATT_PF(DH, GP) hipLaunchKernelGGL((attn_prefill_kernel<DH, GP>), grid, dim3(256), 0, st, items, s, q, kv_pool, kvl, layer, n_q_heads, out)
#define ATT_PF_G(DH) switch (gp) { case 1: ATT_PF(DH, 1); break; case 2: ATT_PF(DH, 2); break; case 4: ATT_PF(DH, 4); break; \
                                   case 8: ATT_PF(DH, 8); break; default: ATT_PF(DH, 16); break; }
  switch (kvl.head_dim) {
    case 32: ATT_PF_G(32); break;
    case 64: ATT_PF_G(64); break;
    default: ATT_PF_G(128); break;
  }
#undef ATT_PF_G
#undef ATT_PF
}

int attn_split_tokens(int head_dim) { return att_split(head_dim); }

void launch_attn_decode(hipStream_t st, RowCtx rc, int row_base, Slots s, const float* q_rot, bf16_t* kv_pool,
                        KVLayout kvl, int layer, int n_q_heads, bf16_t* out, float* ws,
                        int max_splits, int grid_splits, const float* fused_qkv, int n_partials,
                        size_t partial_stride, const float* rope_cos, const float* rope_sin, const int4* items) {
  // items: the scheduler's work list of this iteration (decode, row_base 0), or null
  dim3 grid(rc.max_rows, kvl.n_kv_heads, grid_splits);
  if (items != nullptr) grid = dim3((unsigned)rc.max_rows * grid_splits * kvl.n_kv_heads);
  AttnFuse fz{n_partials, partial_stride, rope_cos, rope_sin};
#define ATT_LAUNCH(DH, F)                                                                                    \
  hipLaunchKernelGGL((attn_decode_kernel<DH, F>), grid, dim3(64 * att_waves(DH, F)), 0, st, items, rc.ctl, s.block_table,      \
                     F ? fused_qkv : q_rot, kv_pool, s.max_blocks, kvl.n_kv_heads, n_q_heads, layer, rc, row_base, kvl, out, \
                     ws, max_splits, fz)
  const bool fused = fused_qkv != nullptr;
  switch (kvl.head_dim) {
    case 32: if (fused) ATT_LAUNCH(32, true); else ATT_LAUNCH(32, false); break;
    case 64: if (fused) ATT_LAUNCH(64, true); else ATT_LAUNCH(64, false); break;
    default: if (fused) ATT_LAUNCH(128, true); else ATT_LAUNCH(128, false); break;
  }
#undef ATT_LAUNCH
}

// Second pass for iterations in which some row may span several KV splits.
void launch_attn_merge(hipStream_t st, RowCtx rc, int row_base, KVLayout kvl, int n_q_heads, bf16_t* out,
                       const float* ws, int max_splits) {
  dim3 mgrid(rc.max_rows, kvl.n_kv_heads);
#define ATT_MERGE(DH)                                                                                       \
  hipLaunchKernelGGL((attn_merge_kernel<DH>), mgrid, dim3(64), 0, st, rc, row_base, kvl.n_kv_heads, n_q_heads, out, \
                     ws, max_splits)
  switch (kvl.head_dim) {
    case 32: ATT_MERGE(32); break;
    case 64: ATT_MERGE(64); break;
    default: ATT_MERGE(128); break;
  }
#undef ATT_MERGE
}

}  // namespace april
