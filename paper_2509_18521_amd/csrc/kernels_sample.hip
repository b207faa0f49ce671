// Sampler (greedy arg-max / top-k with Philox4x32-10) fused with the per-rollout
// state update: append the token, advance the generated length, detect completion
// and count it for the early-termination scheduler (Section 2.2).  One workgroup
// per sampling row.  gfx950.
//
// Top-k is exact: the k largest logits, ties broken by lower index, in descending
// order.  When the LM-head GEMM has left the maximum of every group of 64 logits, the
// k-th largest group maximum is a lower bound of the k-th largest logit (each group
// maximum is a logit), so only the groups whose maximum reaches it are read again.
// Without group maxima (or if a candidate list overflows) a 4-pass radix select over
// the whole row is used.
//
// Categorical sampling and the log-probabilities need sums over the whole row.  With one workgroup
// per row reading the row again they took 55-94 us of every decode iteration (1-380 rows of
// 152 k logits: latency at one row, 2 TB/s at many).  They now add per-group sums of exponentials
// that whoever has the logits in registers leaves (LM head epilogue: fp32 exponentials, fp64 sums)
// or that launch_group_records takes in one coalesced pass over all rows at once.
#include "kernels.h"

namespace april {

constexpr int SAMPLE_THREADS = 1024;   // of a workgroup, in both kernels (256 from group records: 17.8 against 11.3 us for a top 50)
#define MAX_TOPK 64
#define MAX_HOT 1024
#define MAX_CAND 2048

__device__ inline float key2f(unsigned k) { return __uint_as_float((k & 0x80000000u) ? k & 0x7fffffffu : ~k); }

// Philox4x32-10 (Salmon et al., SC'11): first output word.
__device__ inline unsigned philox4x32_10_word0(unsigned c0, unsigned c1, unsigned c2, unsigned c3,
                                               unsigned k0, unsigned k1) {
  const unsigned M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const unsigned hi0 = __umulhi(M0, c0), lo0 = M0 * c0;
    const unsigned hi1 = __umulhi(M1, c2), lo1 = M1 * c2;
    const unsigned n0 = hi1 ^ c1 ^ k0, n1 = lo1, n2 = hi0 ^ c3 ^ k1, n3 = lo0;
    c0 = n0; c1 = n1; c2 = n2; c3 = n3;
    k0 += W0; k1 += W1;
  }
  return c0;
}

// inclusive prefix sum over the lanes
__device__ inline double wave_scan_f64(double v) {
  const int lane = threadIdx.x & 63, l16 = lane & 15;
  double o;
  o = row_ror_f64<1>(v); if (l16 >= 1) v += o;
  o = row_ror_f64<2>(v); if (l16 >= 2) v += o;
  o = row_ror_f64<4>(v); if (l16 >= 4) v += o;
  o = row_ror_f64<8>(v); if (l16 >= 8) v += o;
  const double a = lane_f64(v, 15), b = lane_f64(v, 31), c = lane_f64(v, 47);
  return v + (lane < 16 ? 0.0 : (lane < 32 ? a : (lane < 48 ? a + b : (a + b) + c)));
}

struct SampleShared {
  unsigned hist[256];
  unsigned prefix, krem, ntie;
  int cnt, choice, watch_row, n_hot, overflow;
  // (descending order: larger key, then lower index, so the index is kept inverted and a pair compares as one number)
  __align__(16) unsigned long long cand[MAX_CAND];
  int hot[MAX_HOT];
  unsigned count[MAX_CAND];
  float sort_logit[MAX_TOPK];
  int sort_idx[MAX_TOPK];
  unsigned red_key[16];
  int red_idx[16];
  double red_d[16];
  float red_f[16];
  double total_d;
  float max_f;
};

// Block-wide maximum of vals[0..n) (all threads call; result in every thread).
__device__ inline float block_max_f32(const float* vals, int n, SampleShared& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  float m = -INFINITY;
  for (int i = tid; i < n; i += SAMPLE_THREADS) m = fmaxf(m, vals[i]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  __syncthreads();
  if (lane == 0) sh.red_f[wid] = m;
  __syncthreads();
  if (tid == 0) {
    for (int x = 1; x < SAMPLE_THREADS / 64; ++x) m = fmaxf(m, sh.red_f[x]);
    sh.max_f = m;
  }
  __syncthreads();
  return sh.max_f;
}
// Block-wide sum of one double per thread (all threads call; result in every thread), added
// in a fixed order: lanes by the shuffle tree, wavefronts in index order.
__device__ inline double block_sum_f64(double v, SampleShared& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  __syncthreads();
  if (lane == 0) sh.red_d[wid] = v;
  __syncthreads();
  if (tid == 0) {
    double t = sh.red_d[0];
    for (int x = 1; x < SAMPLE_THREADS / 64; ++x) t += sh.red_d[x];
    sh.total_d = t;
  }
  __syncthreads();
  return sh.total_d;
}

__device__ inline unsigned long long cand_pair(unsigned key, int idx) { return ((unsigned long long)key << 32) | (unsigned)~idx; }

// Key of the k-th largest of vals[0..n) (k <= n): 4 radix passes of 8 bits.  On return
// sh.prefix = that key, sh.krem = how many entries equal to it belong to the top k,
// sh.ntie = how many entries equal it.  All threads must call.  Up to 4 keys per thread are
// kept in registers across the passes (n <= 4 * SAMPLE_THREADS reads memory once).
__device__ inline void block_kth_largest(const float* vals, int n, int k, SampleShared& sh) {
  const int tid = threadIdx.x;
  const bool cached = n <= 4 * SAMPLE_THREADS;
  unsigned ck[4] = {0u, 0u, 0u, 0u};
  if (cached) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = tid + q * SAMPLE_THREADS;
      if (i < n) ck[q] = f2key(vals[i]);
    }
  }
  if (tid == 0) { sh.prefix = 0u; sh.krem = (unsigned)k; }
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    const unsigned mask_hi = pass == 0 ? 0u : (0xFFFFFFFFu << (shift + 8));
    if (tid < 256) sh.hist[tid] = 0u;
    __syncthreads();
    const unsigned prefix = sh.prefix;
    if (cached) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (tid + q * SAMPLE_THREADS < n && (ck[q] & mask_hi) == prefix) atomicAdd(&sh.hist[(ck[q] >> shift) & 255u], 1u);
    } else {
      for (int i = tid; i < n; i += SAMPLE_THREADS) {
        const unsigned key = f2key(vals[i]);
        if ((key & mask_hi) == prefix) atomicAdd(&sh.hist[(key >> shift) & 255u], 1u);
      }
    }
    __syncthreads();
    if (tid < 64) {
      // Wavefront 0 walks the histogram from the top: lane l owns bins 4l..4l+3; `above` =
      // entries in higher bins.  The one lane with above < krem <= above + own holds the digit.
      const unsigned krem = sh.krem;
      const unsigned h0 = sh.hist[4 * tid], h1 = sh.hist[4 * tid + 1], h2 = sh.hist[4 * tid + 2], h3 = sh.hist[4 * tid + 3];
      const unsigned own = h0 + h1 + h2 + h3;
      unsigned suf = own;                                   // inclusive suffix sum over lanes >= tid
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const unsigned o = __shfl_down(suf, off, 64);
        if (tid + off < 64) suf += o;
      }
      const unsigned above = suf - own;
      if (above < krem && krem <= above + own) {
        unsigned cum = above;
        const unsigned hs[4] = {h3, h2, h1, h0};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (cum + hs[q] >= krem) {
            sh.prefix = prefix | ((unsigned)(4 * tid + 3 - q) << shift);
            sh.krem = krem - cum;
            sh.ntie = hs[q];
            break;
          }
          cum += hs[q];
        }
      }
    }
    __syncthreads();
  }
}

// Block arg-max with lowest index on ties over vals[idx0 + i*stride...]: generic helper.
__device__ inline int block_argmax(const float* vals, int n, SampleShared& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  unsigned bk = 0u;
  int bi = 0x7fffffff;
  for (int i = tid; i < n; i += SAMPLE_THREADS) {
    const unsigned k = f2key(vals[i]);
    if (bi == 0x7fffffff || k > bk) { bk = k; bi = i; }     // ascending i: first maximum stays
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned ok = __shfl_xor(bk, off, 64);
    const int oi = __shfl_xor(bi, off, 64);
    if (ok > bk || (ok == bk && oi < bi)) { bk = ok; bi = oi; }
  }
  __syncthreads();
  if (lane == 0) { sh.red_key[wid] = bk; sh.red_idx[wid] = bi; }
  __syncthreads();
  if (tid == 0) {
    for (int x = 1; x < SAMPLE_THREADS / 64; ++x)
      if (sh.red_key[x] > bk || (sh.red_key[x] == bk && sh.red_idx[x] < bi)) { bk = sh.red_key[x]; bi = sh.red_idx[x]; }
    sh.choice = bi;
  }
  __syncthreads();
  return sh.choice;
}

// rc.ctl may be null (the caller states the rows)
__device__ inline int sampling_rows(const RowCtx& rc) { return rc.ctl != nullptr ? rows_or_zero(rc) : rc.max_rows; }

__device__ inline double uniform_draw(const SamplerCfg& sc, long long req, int g) {
  const unsigned long long rid = (unsigned long long)req;
  const unsigned w0 = philox4x32_10_word0((unsigned)(rid & 0xFFFFFFFFull), (unsigned)(rid >> 32), (unsigned)g, 0u,
                                          (unsigned)(sc.seed & 0xFFFFFFFFull), (unsigned)(sc.seed >> 32));
  return (double)(w0 >> 8) * (1.0 / 16777216.0);
}

// Parity-mode capture (all threads call).
__device__ inline void capture_row(const Watch& w, const Ctrl* ctrl, const RowState& q, const float* lg, int V, int sampled, SampleShared& sh) {
  if (w.req == nullptr || ctrl == nullptr) return;
  const int tid = threadIdx.x;
  if (tid == 0) {
    int row = -1;
    const int nw = ctrl->n_watch;
    for (int i = 0; i < nw; ++i)
      if (w.req[i] == q.req && q.g >= w.first[i] && q.g < w.first[i] + w.count[i]) row = w.row0[i] + (q.g - w.first[i]);
    sh.watch_row = row;
  }
  __syncthreads();
  const int row = sh.watch_row;
  if (row >= 0) {
    for (int i = tid; i < V; i += SAMPLE_THREADS) w.logits[(size_t)row * V + i] = lg[i];
    if (tid == 0) { w.sampled[row] = sampled; w.filled[row] = 1; }
  }
}
// Radix select of the row's top k into the candidate list (all threads call).
__device__ inline void topk_whole_row(const float* lg, int V, int k, SampleShared& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  block_kth_largest(lg, V, k, sh);
  const unsigned thr = sh.prefix;
  const int krem = (int)sh.krem, ntie = (int)sh.ntie;
  if (tid == 0) sh.cnt = 0;
  __syncthreads();
  // everything above the threshold, plus the threshold ties with the lowest indices
  for (int i = tid; i < V; i += SAMPLE_THREADS) {
    const unsigned key = f2key(lg[i]);
    if (key > thr || (key == thr && ntie == krem)) {
      const int p = atomicAdd(&sh.cnt, 1);
      if (p < MAX_CAND) sh.cand[p] = cand_pair(key, i);
    }
  }
  __syncthreads();
  if (ntie == krem) return;
  int last = -1;
  for (int t = 0; t < krem; ++t) {
    int best = 0x7fffffff;
    for (int i = tid; i < V; i += SAMPLE_THREADS)
      if (i > last && f2key(lg[i]) == thr) { best = i; break; }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { const int o = __shfl_xor(best, off, 64); best = o < best ? o : best; }
    if (lane == 0) sh.red_idx[wid] = best;
    __syncthreads();
    if (tid == 0) {
      for (int x = 1; x < SAMPLE_THREADS / 64; ++x) best = sh.red_idx[x] < best ? sh.red_idx[x] : best;
      const int p = sh.cnt++;
      if (p < MAX_CAND) sh.cand[p] = cand_pair(thr, best);
      sh.red_idx[0] = best;
    }
    __syncthreads();
    last = sh.red_idx[0];
    __syncthreads();
  }
}

// sh.count[e] += the sum of f(entry e, entry j) over the n entries j of the candidate list, for every entry e.  128
// entries at a time, an eighth of the list per group of 128 threads, four entries of it per round trip to LDS.  All
// threads call; the counts (zero before) are complete behind the next barrier.
template <class F>
__device__ inline void count_pairs(SampleShared& sh, int n, F f) {
  static_assert(SAMPLE_THREADS == 1024, "eight groups of 128 threads");
  const int per = (n + 31) / 32 * 4, j0 = (threadIdx.x >> 7) * per, j1 = min(n, j0 + per);
  for (int e0 = 0; e0 < n; e0 += 128) {
    const int e = e0 + (threadIdx.x & 127);
    const unsigned long long own = sh.cand[e < n ? e : 0];
    unsigned c = 0;
    for (int j = j0; j < j1; j += 4) {          // (entries past the end of the list: zero, see fill)
      const ulonglong2 x = *reinterpret_cast<const ulonglong2*>(sh.cand + j), y = *reinterpret_cast<const ulonglong2*>(sh.cand + j + 2);
      c += (f(own, x.x) + f(own, x.y)) + (f(own, y.x) + f(own, y.y));
    }
    if (e < n && c != 0) atomicAdd(&sh.count[e], c);
  }
}
// Up to three entries that come after every other, behind the list's end (one thread; no entry is zero).
__device__ inline void fill_list(SampleShared& sh, int n) {
  for (int j = n; j < (n + 3) / 4 * 4; ++j) sh.cand[j] = 0ull;
}

// The draw among the exact top k of the candidates: the rank of a candidate is its place in the descending order.
// Result in sh.choice; all threads call, with the counts zero, and meet in it but not behind it.
__device__ inline void draw_topk(int k, const SamplerCfg& sc, long long req, int g, SampleShared& sh) {
  const int tid = threadIdx.x;
  __syncthreads();
  const int n_cand = sh.cnt < MAX_CAND ? sh.cnt : MAX_CAND;
  if (tid == 0) fill_list(sh, n_cand);
  __syncthreads();
  count_pairs(sh, n_cand, [](unsigned long long own, unsigned long long x) { return x > own ? 1u : 0u; });
  __syncthreads();
  for (int c = tid; c < n_cand; c += SAMPLE_THREADS) {
    const unsigned long long own = sh.cand[c];
    const int rank = (int)sh.count[c];
    if (rank < k) { sh.sort_logit[rank] = key2f((unsigned)(own >> 32)); sh.sort_idx[rank] = ~(int)(unsigned)own; }
  }
  __syncthreads();
  if (tid >= 64) return;
  // Lane j holds candidate j (k <= 64).  fp64 softmax over the candidates and its running sum; the token is the first
  // candidate whose cumulative probability exceeds the uniform draw, the last candidate if none does.
  const int n = n_cand < k ? n_cand : k;
  const double T = (double)sc.temperature;
  const double z = (double)sh.sort_logit[tid < n ? tid : 0] / T;
  const double e = tid < n ? exp(z - lane_f64(z, 0)) : 0.0;
  const double c = wave_scan_f64(e / wave_sum_f64(e));    // inclusive prefix sum over lanes <= tid
  int keep = n;
  double tot = 1.0;
  if (sc.top_p > 0.f && sc.top_p < 1.f) {
    // nucleus: the shortest prefix whose cumulative probability reaches top_p
    const unsigned long long reach = __ballot(tid < n && c >= (double)sc.top_p);
    keep = reach ? __ffsll((long long)reach) : n;
    tot = lane_f64(c, __builtin_amdgcn_readfirstlane(keep - 1));      // mass of the nucleus: renormalise by it
  }
  const unsigned long long hit = __ballot(tid < keep && c > uniform_draw(sc, req, g) * tot);
  // (no candidate: the maxima were signalling NaN, which come back quiet, and no logit has their key; the choice stays the last token)
  if (tid == 0 && n > 0) sh.choice = sh.sort_idx[hit ? __ffsll((long long)hit) - 1 : keep - 1];
}

// ---------------------------------------------------------------------------
// Sampling from the whole row: logits without group records (small and ragged vocabularies, the fp32 path).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(SAMPLE_THREADS) void sample_rows_kernel(RowCtx rc, Slots s, Ctrl* ctrl, const float* logits, int V,
                                                                     SamplerCfg sc, Watch w, int update,
                                                                     const long long* req_ids, const int* gen_idx,
                                                                     int* out_tokens, float* out_logprobs) {
  const int r = blockIdx.x;
  if (r >= sampling_rows(rc)) return;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const float* lg = logits + (size_t)r * V;
  __shared__ SampleShared sh;
  const RowState q = load_row(rc, s, ctrl, r, update, req_ids, gen_idx);

  if (sc.kind == 0 || (sc.kind == 1 && sc.top_k <= 1)) {
    block_argmax(lg, V, sh);                               // maximum, lowest index on ties
  } else if (sc.kind == 2) {
    // Temperature sampling over the whole vocabulary: inverse CDF in index order.  Thread t owns the
    // indices [t * chunk, (t + 1) * chunk): its partial sum of exp((l - max) / T), an exclusive scan over the
    // threads (wavefront scans, then wavefront totals in order), and the thread whose range holds the
    // crossing of u * total finds the index.
    const float M = block_max_f32(lg, V, sh);
    const double invT = 1.0 / (double)sc.temperature;
    const int chunk = (V + SAMPLE_THREADS - 1) / SAMPLE_THREADS;
    const int i0 = tid * chunk, i1 = (i0 + chunk < V) ? i0 + chunk : V;
    auto mass = [&](int i) { return exp(((double)lg[i] - (double)M) * invT); };
    double part = 0.0;
    for (int i = i0; i < i1; ++i) part += mass(i);
    double incl = part;                                     // inclusive scan inside the wavefront
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const double o = __shfl_up(incl, off, 64);
      if (lane >= off) incl += o;
    }
    __syncthreads();
    if (lane == 63) sh.red_d[wid] = incl;
    __syncthreads();
    double before = 0.0, total = 0.0;
    for (int x = 0; x < SAMPLE_THREADS / 64; ++x) {
      if (x < wid) before += sh.red_d[x];
      total += sh.red_d[x];
    }
    const double target = uniform_draw(sc, q.req, q.g) * total;      // cumulative / total > u  <=>  cumulative > u * total
    const double lo = before + incl - part, hi = before + incl;
    if (tid == 0) sh.choice = V - 1;                        // rounding leaves no crossing: the last index
    __syncthreads();
    if (i0 < i1 && lo <= target && hi > target) {
      double c = lo;
      int pick = i1 - 1;
      for (int i = i0; i < i1; ++i) {
        c += mass(i);
        if (c > target) { pick = i; break; }
      }
      sh.choice = pick;
    }
    __syncthreads();
  } else {
    const int k = sc.top_k < V ? (sc.top_k < MAX_TOPK ? sc.top_k : MAX_TOPK) : (V < MAX_TOPK ? V : MAX_TOPK);
    for (int i = tid; i < MAX_CAND; i += SAMPLE_THREADS) sh.count[i] = 0u;
    topk_whole_row(lg, V, k, sh);
    draw_topk(k, sc, q.req, q.g, sh);
    __syncthreads();
  }

  const int sampled = sh.choice;
  capture_row(w, ctrl, q, lg, V, sampled, sh);
  // the token that is appended: the sampler's choice, or the teacher-forced one (parity mode)
  const int tok = q.forced >= 0 ? q.forced : sampled;
  // ---- log-probability of that token under softmax(logits / T) over the whole vocabulary ----
  float* lp_dst = update ? (s.logprob ? s.logprob + (size_t)q.slot * s.max_ctx + q.g : nullptr) : (out_logprobs ? out_logprobs + r : nullptr);
  if (lp_dst != nullptr) {
    const float M = block_max_f32(lg, V, sh);
    const float invT = 1.0f / sc.temperature;
    double part = 0.0;
    for (int i = tid; i < V; i += SAMPLE_THREADS) part += (double)__expf((lg[i] - M) * invT);
    const double Z = block_sum_f64(part, sh);
    if (tid == 0) *lp_dst = (float)((double)((lg[tok] - M) * invT) - log(Z));
  }
  if (tid == 0) finish_row(s, ctrl, q, r, update, sampled, tok, out_tokens);
}

// ---------------------------------------------------------------------------
// Sampling from group records (maximum, its column, sum of exponentials per 64 logits).  A row is 2374 records of
// a vocabulary of 152 k, so the kernel is a chain of block-wide steps, not a stream: everything is requested at the
// start (GQ records per thread in registers; a longer row reads them again), maximum, arg-max and minimum work share
// one exchange through LDS, every thread finishes an exchange for itself, and the top-k threshold comes from
// the 64 lane maxima instead of four radix passes.  Measured per launch with 152 k logits against separate passes with a
// serial sum each: one row, greedy with log-probabilities 11.7 -> 7.3 us; 5 rows, top 50 18.2 -> 10.8 us, with
// log-probabilities of 47 rows of 32 k logits 20.1 -> 10.4; 192 rows, categorical with log-probabilities 13.2 -> 8.3.
// ---------------------------------------------------------------------------
constexpr int GQ = 4;                      // records of a thread that stay in registers
template <bool CACHED>                     // n_groups <= GQ * SAMPLE_THREADS
__global__ __launch_bounds__(SAMPLE_THREADS) void sample_records_kernel(RowCtx rc, Slots s, Ctrl* ctrl, const float* logits, int V,
                                                                        SamplerCfg sc, Watch w, int update,
                                                                        const long long* req_ids, const int* gen_idx,
                                                                        int* out_tokens, const float* group_max,
                                                                        float* out_logprobs, const int* group_idx,
                                                                        const double* group_sum) {
  constexpr int W = SAMPLE_THREADS / 64;
  const int r = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int n_groups = (V + 63) >> 6;
  const float* lg = logits + (size_t)r * V;
  const float* gm = group_max + (size_t)r * n_groups;
  const double* gs = group_sum ? group_sum + (size_t)r * n_groups : nullptr;
  if (r >= sampling_rows(rc)) return;
  __shared__ SampleShared sh;
  __shared__ unsigned lane_key[W][64];
  const bool greedy = sc.kind == 0 || (sc.kind == 1 && sc.top_k <= 1), topk = !greedy && sc.kind == 1;
  // categorical: thread t owns consecutive groups (the CDF runs in index order), else every SAMPLE_THREADS-th
  const int chunk = (n_groups + SAMPLE_THREADS - 1) / SAMPLE_THREADS;
  auto group_at = [&](int e) { return sc.kind == 2 ? tid * chunk + e : tid + e * SAMPLE_THREADS; };
  float m_c[GQ];
  double s_c[GQ];
  if (CACHED) {
#pragma unroll
    for (int e = 0; e < GQ; ++e) {
      const int i = group_at(e);
      const bool in = e < chunk && i < n_groups;
      m_c[e] = in ? gm[i] : -INFINITY;
      s_c[e] = in && gs ? gs[i] : 0.0;
    }
  }
  const RowState q = load_row(rc, s, ctrl, r, update, req_ids, gen_idx);
  // f(register slot, group, maximum, sum) over this thread's groups, in registers also past the last one (-inf, 0)
  auto each = [&](auto f) {
    if constexpr (CACHED) {
#pragma unroll
      for (int e = 0; e < GQ; ++e)
        f(e, group_at(e), m_c[e], s_c[e]);
    } else {
      for (int e = 0; e < chunk; ++e)
        if (group_at(e) < n_groups) f(0, group_at(e), gm[group_at(e)], gs ? gs[group_at(e)] : 0.0);
    }
  };
  float* lp_dst = update ? (s.logprob ? s.logprob + (size_t)q.slot * s.max_ctx + q.g : nullptr) : (out_logprobs ? out_logprobs + r : nullptr);

  // ---- first exchange: the row's maximum; greedy: its group (lowest on ties); top-k: maxima by lane ----
  // (keys of real groups only: a group of NaN with the sign set comes below the -inf of the slots past the last group)
  float mx = -INFINITY;
  unsigned bk = 0u;
  int bi = 0x7fffffff;
  each([&](int, int i, float m, double) {
    mx = fmaxf(mx, m);
    const unsigned k = i < n_groups ? f2key(m) : 0u;          // (0 where a row's largest key is 0: the lowest index is a real one's)
    const bool first = bi == 0x7fffffff || k > bk;            // ascending i: the first maximum stays
    bk = first ? k : bk;
    bi = first ? i : bi;
  });
  if (topk) lane_key[wid][lane] = bk;                         // (0: no group)
  mx = wave_max_f32(mx);
  if (greedy) {
    const unsigned top = wave_max_u32(bk);
    bi = wave_min_i32(bk == top ? bi : 0x7fffffff);
    bk = top;
  }
  if (lane == 0) { sh.red_f[wid] = mx; sh.red_key[wid] = bk; sh.red_idx[wid] = bi; }
  if (tid == 0) { sh.n_hot = 0; sh.cnt = 0; sh.overflow = 0; sh.choice = V - 1; }
  if (topk)
    for (int i = tid; i < MAX_CAND; i += SAMPLE_THREADS) sh.count[i] = 0u;
  __syncthreads();
  static_assert(W == 16, "a wavefront's partial result per lane of a row");
  const float M = row_max_f32(sh.red_f[lane & (W - 1)]);
  const float invT = 1.0f / sc.temperature;
  double Z = 0.0, total = 0.0;                                // the row's sum of exponentials: this thread's part, the whole (categorical)

  if (greedy) {
    bk = sh.red_key[lane & (W - 1)];
    bi = row_min_i32(bk == row_max_u32(bk) ? sh.red_idx[lane & (W - 1)] : 0x7fffffff);
    // the column inside the group: left by the LM head, else looked up in the logits
    if (wid == 0) {
      int li;
      if (group_idx) li = group_idx[(size_t)r * n_groups + bi];
      else {
        const int i = bi * 64 + lane;
        const unsigned k = i < V ? f2key(lg[i]) : 0u;
        const unsigned top = wave_max_u32(k);
        li = wave_min_i32(i < V && k == top ? lane : 64);
      }
      if (lane == 0) sh.choice = bi * 64 + li;
    }
  } else if (topk) {
    const int k = sc.top_k < V ? (sc.top_k < MAX_TOPK ? sc.top_k : MAX_TOPK) : (V < MAX_TOPK ? V : MAX_TOPK);
    // The 64 lanes' maxima are group maxima of 64 disjoint sets, so at least k groups reach the k-th largest of them:
    // the groups that do hold the k-th largest group maximum (of 152 k logits about twice k for 50, four times k for 64, where
    // the bound is the smallest lane's).
    unsigned lk = lane_key[0][lane];
#pragma unroll
    for (int x = 1; x < W; ++x) { const unsigned o = lane_key[x][lane]; lk = o > lk ? o : lk; }
    unsigned tau0 = 0u;
#pragma unroll 1
    for (int bit = 31; bit >= 12; --bit) {                    // (the lowest bits stay zero: a slightly lower bound)
      const unsigned t = tau0 | (1u << bit);
      if (__popcll(__ballot(lk >= t)) >= k) tau0 = t;
    }
    each([&](int, int i, float m, double) {
      const unsigned key = f2key(m);
      if (key >= tau0 && i < n_groups) {
        const int p = atomicAdd(&sh.n_hot, 1);
        if (p < MAX_HOT) sh.cand[p] = cand_pair(key, i); else sh.overflow = 1;
      }
    });
    __syncthreads();
    bool have = !sh.overflow;
    if (have) {
      // those with fewer than k larger ones are the groups whose maximum reaches the k-th largest maximum, tau, a lower
      // bound of the k-th largest logit: only they are read
      const int n0 = sh.n_hot;
      if (tid == 0) { fill_list(sh, n0); sh.cnt = 0; }
      __syncthreads();
      if (tid == 0) sh.n_hot = 0;
      count_pairs(sh, n0, [](unsigned long long own, unsigned long long x) {       // larger ones, and 2^16 per equal one
        const unsigned kx = (unsigned)(x >> 32), ko = (unsigned)(own >> 32);
        return (kx > ko ? 1u : 0u) + (kx == ko ? 0x10000u : 0u);
      });
      __syncthreads();
      for (int c = tid; c < n0; c += SAMPLE_THREADS) {
        const unsigned n = sh.count[c];
        const int above = (int)(n & 0xffffu);
        sh.count[c] = 0u;
        if (above < k) {
          sh.hot[atomicAdd(&sh.n_hot, 1)] = ~(int)(unsigned)sh.cand[c];
          if (above + (int)(n >> 16) >= k) sh.prefix = (unsigned)(sh.cand[c] >> 32);
        }
      }
      __syncthreads();
      const unsigned tau = sh.prefix;
      const int n_hot = sh.n_hot;
      constexpr int HU = 4;                                   // groups of a wavefront requested together
      for (int h0 = 0; h0 < n_hot; h0 += HU * W) {
        float v[HU];
        int at[HU];
#pragma unroll
        for (int x = 0; x < HU; ++x) {
          const int h = h0 + x * W + wid;
          const int grp = h < n_hot ? sh.hot[h] : -1;
          at[x] = grp >= 0 && grp * 64 + lane < V ? grp * 64 + lane : -1;
          v[x] = lg[at[x] >= 0 ? at[x] : 0];
        }
#pragma unroll
        for (int x = 0; x < HU; ++x) {
          const unsigned key = f2key(v[x]);
          if (at[x] >= 0 && key >= tau) {
            const int p = atomicAdd(&sh.cnt, 1);
            if (p < MAX_CAND) sh.cand[p] = cand_pair(key, at[x]); else sh.overflow = 1;
          }
        }
      }
      __syncthreads();
      have = !sh.overflow;
    }
    if (!have) topk_whole_row(lg, V, k, sh);
    draw_topk(k, sc, q.req, q.g, sh);
  } else {
    // ---- temperature sampling over the whole vocabulary: inverse CDF in index order ----------
    // Masses of the groups (their sums rescaled to the row's maximum), an exclusive scan over the threads, and the
    // thread whose range holds the crossing of u * total finds the group; a wavefront then walks its logits.
    const double iT = 1.0 / (double)sc.temperature;
    double mass_c[CACHED ? GQ : 1];
    each([&](int e, int, float m, double sum) {
      const double x = sum * exp(((double)m - (double)M) * iT);
      if (CACHED) mass_c[e] = x;
      Z += x;
    });
    const double incl = wave_scan_f64(Z);                     // inclusive scan inside the wavefront
    if (lane == 63) sh.red_d[wid] = incl;
    if (tid == 0) sh.hot[0] = -1;
    __syncthreads();
    double before = 0.0;
#pragma unroll
    for (int x = 0; x < W; ++x) {
      if (x < wid) before += sh.red_d[x];
      total += sh.red_d[x];
    }
    const double target = uniform_draw(sc, q.req, q.g) * total;      // cumulative / total > u  <=>  cumulative > u * total
    const double lo = before + incl - Z, hi = before + incl;
    if (tid * chunk < n_groups && lo <= target && hi > target) {
      double c = lo, below = lo;
      int pick = -1;
      each([&](int e, int i, float m, double sum) {
        const bool go = i < n_groups && !(pick >= 0 && c > target);
        below = go ? c : below;
        c += go ? (CACHED ? mass_c[e] : sum * exp(((double)m - (double)M) * iT)) : 0.0;
        pick = go ? i : pick;
      });
      sh.hot[0] = pick;
      sh.total_d = below;
    }
    __syncthreads();
    if (wid == 0 && sh.hot[0] >= 0) {
      // the group's logits, one per lane; its last index if rounding leaves no crossing inside it
      const int first = sh.hot[0] * 64, n = min(64, V - first);
      const double c = wave_scan_f64(lane < n ? exp(((double)lg[first + lane] - (double)M) * iT) : 0.0);
      const unsigned long long hit = __ballot(lane < n && sh.total_d + c > target);
      if (lane == 0) sh.choice = first + (hit ? __ffsll((long long)hit) - 1 : n - 1);
    }
  }

  // ---- log-probability of the appended token under softmax(logits / T) over the whole vocabulary ----
  const bool sums = lp_dst != nullptr;
  if (sums && sc.kind != 2) {
    each([&](int, int, float m, double sum) { Z += sum * exp((double)((m - M) * invT)); });
    Z = wave_sum_f64(Z);
    if (lane == 0) sh.red_d[wid] = Z;
  }
  __syncthreads();
  const int sampled = sh.choice;
  capture_row(w, ctrl, q, lg, V, sampled, sh);
  if (wid != 0) return;
  // the token that is appended: the sampler's choice, or the teacher-forced one (parity mode)
  const int tok = q.forced >= 0 ? q.forced : sampled;
  if (sums) {
    // the greedy choice is the row's maximum: its logit need not have been written
    const float l = logits != nullptr ? lg[tok] : M;
    if (sc.kind != 2) {
      total = row_sum_f64(sh.red_d[lane & (W - 1)]);
    }
    if (lane == 0) *lp_dst = (float)((double)((l - M) * invT) - log(total));
  }
  if (lane == 0) finish_row(s, ctrl, q, r, update, sampled, tok, out_tokens);
}

// Group records of logits in memory.  16 lanes own a group of 64 logits (4 consecutive ones each), a
// wavefront takes 4 groups per load and GR_STEPS loads in flight, so the pass streams.  (Before, one
// thread per group walked 64 consecutive floats, and each thread of the row's workgroup 149 of them,
// twice: a call for 192 rows of 152 k logits took 724 us with the categorical sampler and
// log-probabilities and 62 us for 5 rows with top-k, 94 and 42 with this pass; 61 and 29 with the sampler above and without copies.)
// Rows start at any multiple of 4 bytes.  KEYS: maxima in the order of f2key (a NaN above everything, one with its sign set below),
// as the whole-row searches compare, a short last group as if filled up with -inf; else fmaxf.
//
// The exponentials of the fp64 sums bound that pass (192 rows of 152 k: 23 us without sums, 25 with fp32 ones), so they are
// cut to what the sums need.  2^y for y <= 0: y = n + f with |f| <= 1/2 by adding and taking away 1.5 * 2^52, the Taylor
// series of 2^f to the twelfth power (remainder 1.7e-16), n added to the exponent; zero below 2^-1022, NaN for NaN.
// Against the library's exp: 39.5 -> 37.5 us per pass.  (Four blocks of 16 groups per wavefront, the next one's loads in
// flight: 43.2 us; 2 or 8 loads in flight instead of 4: 39.9 and 44.0 against 41.3.)
__device__ inline double exp2_neg(double y) {
  const double big = 6755399441055744.0;                     // 1.5 * 2^52
  const double t = y + big, f = y - (t - big);
  // (ln 2)^k / k!
  double p = 2.56784359934882051e-11;
  p = __fma_rn(p, f, 4.44553827187081150e-10);
  p = __fma_rn(p, f, 7.05491162080112333e-09);
  p = __fma_rn(p, f, 1.01780860092396997e-07);
  p = __fma_rn(p, f, 1.32154867901443095e-06);
  p = __fma_rn(p, f, 1.52527338040598403e-05);
  p = __fma_rn(p, f, 1.54035303933816099e-04);
  p = __fma_rn(p, f, 1.33335581464284434e-03);
  p = __fma_rn(p, f, 9.61812910762847716e-03);
  p = __fma_rn(p, f, 5.55041086648215800e-02);
  p = __fma_rn(p, f, 2.40226506959100712e-01);
  p = __fma_rn(p, f, 6.93147180559945309e-01);
  p = __fma_rn(p, f, 1.0);
  const double r = __hiloint2double(__double2hiint(p) + (__double2loint(t) << 20), __double2loint(p));
  return y >= -1022.0 ? r : (y < -1022.0 ? 0.0 : y);
}
constexpr int GR_STEPS = 4;
template <int SUMS, bool KEYS>
__global__ __launch_bounds__(256) void group_records_kernel(const float* logits, const int2* ctl, int n_rows, int V,
                                                            double inv_t, float* group_max, double* group_sum) {
  const int r = blockIdx.y;
  if (ctl != nullptr) {
    const int2 v = *ctl;
    n_rows = v.y ? 0 : v.x;
  }
  if (r >= n_rows) return;
  typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
  const int n_groups = (V + 63) >> 6, lane = threadIdx.x & 63, sub = lane & 15;
  const int first = ((int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * (4 * GR_STEPS);   // first group of the wavefront
  const float* row = logits + (size_t)r * V;
  const double inv_t2 = inv_t * 1.4426950408889634074;
  auto load_whole = [&](int g0, float (&v)[GR_STEPS][4]) {
#pragma unroll
    for (int s = 0; s < GR_STEPS; ++s) {
      const f32x4u q = *reinterpret_cast<const f32x4u*>(row + (size_t)(g0 + 4 * s) * 64 + lane * 4);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[s][j] = q[j];
    }
  };
  auto load_part = [&](int g0, float (&v)[GR_STEPS][4]) {
#pragma unroll
    for (int s = 0; s < GR_STEPS; ++s)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = (g0 + 4 * s) * 64 + lane * 4 + j;
        v[s][j] = i < V ? row[i] : -INFINITY;
      }
  };
  auto records = [&](int g0, const float (&v)[GR_STEPS][4]) {
#pragma unroll
    for (int s = 0; s < GR_STEPS; ++s) {
      const int g = g0 + 4 * s + (lane >> 4);
      float m;
      if (KEYS) {
        unsigned k = f2key(v[s][0]);
        m = v[s][0];
        auto take = [&](float x) { const unsigned kx = f2key(x); if (kx > k) { k = kx; m = x; } };
#pragma unroll
        for (int j = 1; j < 4; ++j) take(v[s][j]);
        take(as_f32(row_ror<8>(__float_as_int(m))));
        take(as_f32(row_ror<4>(__float_as_int(m))));
        take(as_f32(row_ror<2>(__float_as_int(m))));
        take(as_f32(row_ror<1>(__float_as_int(m))));
      } else {
        m = row_max_f32(fmaxf(fmaxf(v[s][0], v[s][1]), fmaxf(v[s][2], v[s][3])));
      }
      double sum = 0.0;
      if (SUMS) {
        const float ref = m == -INFINITY ? 0.f : m;            // a group of -inf sums to zero, not to NaN
#pragma unroll
        for (int j = 0; j < 4; ++j)
          sum += SUMS == 2 ? exp2_neg(((double)v[s][j] - (double)ref) * inv_t2) : (double)__expf((v[s][j] - ref) * (float)inv_t);
        sum = row_sum_f64(sum);
      }
      if (sub == 0 && g < n_groups) {
        group_max[(size_t)r * n_groups + g] = m;
        if (SUMS) group_sum[(size_t)r * n_groups + g] = sum;
      }
    }
  };
  float v[GR_STEPS][4];
  if ((first + 4 * GR_STEPS) * 64 <= V) load_whole(first, v);
  else load_part(first, v);
  records(first, v);
}
void launch_group_records(hipStream_t st, const float* logits, const int2* ctl, int n_rows, int V, int sums,
                          float temperature, float* group_max, double* group_sum) {
  // grid.y holds the rows: at most 65535 of them per launch
  const double inv_t = sums == 2 ? 1.0 / (double)temperature : (double)(1.0f / temperature);
  dim3 grid(ceil_div((V + 63) / 64, 16 * GR_STEPS), n_rows);
#define GR_LAUNCH(S, K) hipLaunchKernelGGL((group_records_kernel<S, K>), grid, dim3(256), 0, st, logits, ctl, n_rows, V, inv_t, group_max, group_sum)
  const bool keys = V % 64 != 0;
  switch (sums) {
    case 0: if (keys) GR_LAUNCH(0, true); else GR_LAUNCH(0, false); break;
    case 1: if (keys) GR_LAUNCH(1, true); else GR_LAUNCH(1, false); break;
    default: if (keys) GR_LAUNCH(2, true); else GR_LAUNCH(2, false); break;
  }
#undef GR_LAUNCH
}

void launch_sample(hipStream_t st, RowCtx rc, Slots s, Ctrl* ctrl, const float* logits, int vocab, SamplerCfg sc,
                   Watch w, int update, const long long* req_ids, const int* gen_idx, int* out_tokens,
                   const float* group_max, float* out_logprobs, const int* group_idx, const double* group_sum) {
  const int n_groups = ceil_div(vocab, 64);
  const bool lp = update ? s.logprob != nullptr : out_logprobs != nullptr;
  // records serve what the call needs: sums for log-probabilities and the categorical sampler, groups enough for a top k
  const bool records = group_max != nullptr && (group_sum != nullptr || (!lp && sc.kind != 2)) && sampler_takes_records(sc, vocab);
#define SAMPLE_RECORDS(CACHED)                                                                                         \
  hipLaunchKernelGGL(sample_records_kernel<CACHED>, dim3(rc.max_rows), dim3(SAMPLE_THREADS), 0, st, rc, s, ctrl, logits, vocab, \
                     sc, w, update, req_ids, gen_idx, out_tokens, group_max, out_logprobs, group_idx, group_sum)
  if (!records)
    hipLaunchKernelGGL(sample_rows_kernel, dim3(rc.max_rows), dim3(SAMPLE_THREADS), 0, st, rc, s, ctrl, logits, vocab, sc, w,
                       update, req_ids, gen_idx, out_tokens, out_logprobs);
  else if (n_groups <= GQ * SAMPLE_THREADS) SAMPLE_RECORDS(true);
  else SAMPLE_RECORDS(false);
#undef SAMPLE_RECORDS
}

}  // namespace april
