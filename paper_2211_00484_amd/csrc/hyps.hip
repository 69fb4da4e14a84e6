// Full-sequence beam search with max-symbols 1: the comparison search of Table 5
// ("beam search"), whose state space is the whole label sequence (footnote to
// Sec. 2.2) rather than the (context, graph state) tuples of the FSA-based search.
//
// A hypothesis is a distinct blank-free label sequence y with a score.  On frame t each
// hypothesis expands to blank (y kept) and to every label c (y + c), weighted by
// log P(label | last two labels of y, t) with no blank factor; equal sequences merge by
// max or by log-add (the two merge operations of Table 3); the N best candidates by
// (score desc, first candidate index asc) are kept, in that order, where candidate
// (i, c) has index i * V + c (blank c = 0).  Two candidates can only be equal as the
// blank of a hypothesis y_i and label last(y_i) of the hypothesis y_j = y_i minus its
// last label, so sequences are carried as 64-bit hashes (of y and of y without its last
// label) plus their length; equal hashes are taken as equal sequences.
//
// Frame schedule, two launches per frame: the joiner GEMM over one row per hypothesis,
// then k_hyp_step (one workgroup per stream: merge, top-N selection, and the next frame's
// joiner rows).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.h"

namespace tbs {
namespace {

constexpr int kHypThreads = 256;
constexpr int kHypWideThreads = 1024;
constexpr size_t kHypCache = 120 * 1024;  // LDS for the candidates' scores
constexpr unsigned long long kHashInit = 0x9e3779b97f4a7c15ull;  // hash of the empty sequence
constexpr unsigned long long kHashMul = 0x100000001b3ull;       // odd multiplier

__device__ __forceinline__ unsigned long long hash_push(unsigned long long h, int c) {
  return h * kHashMul + (unsigned long long)(unsigned)c;
}

// Order-preserving code of a score (larger score, larger code); 0 for -inf: no candidate.
__device__ __forceinline__ unsigned long long score_code(double x) {
  if (x == -__builtin_inf()) return 0;
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  return (u >> 63) ? ~u : u | (1ull << 63);
}
__device__ __forceinline__ double code_score(unsigned long long c) {
  return __longlong_as_double((long long)((c >> 63) ? c & ~(1ull << 63) : ~c));
}

// Wave reductions on DPP: rotations within each row of 16 lanes, then broadcasts of lane 15
// into rows 1 and 3 and of lane 31 into rows 2 and 3; lane 63 ends with the whole wave's.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_move(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ unsigned long long max_step(unsigned long long v) {
  const int lo = dpp_move<CTRL, ROWS>((int)(unsigned)v, (int)(unsigned)v);
  const int hi = dpp_move<CTRL, ROWS>((int)(unsigned)(v >> 32), (int)(unsigned)(v >> 32));
  const unsigned long long o = (unsigned long long)(unsigned)hi << 32 | (unsigned)lo;
  return o > v ? o : v;
}
__device__ __forceinline__ unsigned long long wave_max(unsigned long long v) {
  v = max_step<0x128>(v);
  v = max_step<0x124>(v);
  v = max_step<0x122>(v);
  v = max_step<0x121>(v);
  v = max_step<0x142, 0xa>(v);
  v = max_step<0x143, 0xc>(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, 63);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), 63);
  return (unsigned long long)hi << 32 | lo;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// A candidate: score code, its first index (ties: smallest first), and its own index
// i * V + c.
struct Cand {
  unsigned long long code;
  int first;
  int idx;
};

// The best of the wave's lanes' candidates (uniform); code 0 if none has one.
__device__ __forceinline__ Cand wave_best(const Cand& x) {
  const unsigned long long top = wave_max(x.code);
  unsigned long long m = __ballot(x.code == top);
  if (m & (m - 1)) {  // equal scores: the smallest first index
    int f = x.code == top ? x.first : 0x7fffffff;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) f = min(f, __shfl_xor(f, o, 64));
    m = __ballot(x.code == top && x.first == f);
  }
  const int l = __ffsll(m) - 1;
  return Cand{top, __builtin_amdgcn_readlane(x.first, l), __builtin_amdgcn_readlane(x.idx, l)};
}

__device__ __forceinline__ bool cand_before(const Cand& x, const Cand& y) {
  return x.code > y.code || (x.code == y.code && x.first < y.first);
}

// Joiner rows of stream b's nh hypotheses, row b * N + r: h = tanh(enc + ReLU(P0[a] + P1[c]))
// for context (a, c) of ctx[r], as fp16 pairs, fp32 or bf16 (RNE).  (Hypotheses with equal contexts
// get equal rows.)  Column quads when C is a multiple of 4, kBatch of them per thread with
// all their table loads in flight together.  enc, ctx: LDS.
template <int NT>
__device__ void hyp_rows(const ModelDev& m, const HypDev& d, int b, int nh, const float* enc,
                         const int* ctx) {
  constexpr int kBatch = NT == 256 ? 4 : 2;
  const int tid = threadIdx.x, C = m.C, Kpad = m.Kpad, V = m.V;
  const size_t row0 = (size_t)b * d.N * Kpad;
  const int W = (C & 3) == 0 ? 4 : 1, per = Kpad / W, total = nh * per;
  for (int i0 = tid; i0 < total; i0 += NT * kBatch) {
    float4 p0[kBatch], p1[kBatch];
    int r[kBatch], k[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = min(i0 + u * NT, total - 1);
      r[u] = i / per;
      k[u] = W * (i - r[u] * per);
      const int c = ctx[r[u]], a = c / V;
      const float* q0 = m.P0 + (size_t)a * Kpad + k[u];
      const float* q1 = m.P1 + (size_t)(c - a * V) * Kpad + k[u];
      if (W == 4) {
        p0[u] = *reinterpret_cast<const float4*>(q0);
        p1[u] = *reinterpret_cast<const float4*>(q1);
      } else {
        p0[u].x = *q0;
        p1[u].x = *q1;
      }
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (i0 + u * NT >= total) continue;
      const size_t o = row0 + (size_t)r[u] * Kpad + k[u];
      auto at = [&](int j, float x0, float x1) {
        return k[u] + j < C ? tanh_fast(enc[k[u] + j] + fmaxf(x0 + x1, 0.f)) : 0.f;
      };
      const float h0 = at(0, p0[u].x, p1[u].x);
      if (W == 4) {
        const float h1 = at(1, p0[u].y, p1[u].y), h2 = at(2, p0[u].z, p1[u].z), h3 = at(3, p0[u].w, p1[u].w);
        if (m.bf16) {
          *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(d.h) + o) =
              make_uint2((unsigned)f32_to_bf16_rne(h0) | (unsigned)f32_to_bf16_rne(h1) << 16,
                         (unsigned)f32_to_bf16_rne(h2) | (unsigned)f32_to_bf16_rne(h3) << 16);
        } else {
          *reinterpret_cast<uint4*>(reinterpret_cast<unsigned*>(d.h) + o) = h_quad(m.direct, h0, h1, h2, h3);
        }
      } else if (m.bf16) {
        reinterpret_cast<uint16_t*>(d.h)[o] = f32_to_bf16_rne(h0);
      } else if (m.direct) {
        reinterpret_cast<float*>(d.h)[o] = h0;
      } else {
        store_split(d.h, o - k[u], k[u], h0);
      }
    }
  }
}

// The empty hypothesis of every stream and its joiner row for frame 0.
__global__ __launch_bounds__(kHypThreads) void k_hyp_init(ModelDev m, HypDev d) {
  __shared__ float s_enc[kMaxDim];
  __shared__ int s_ctx;
  const int b = blockIdx.x, tid = threadIdx.x;
  const size_t o = (size_t)b * d.N;
  if (tid == 0) {
    d.nh[0][b] = 1;
    d.hash[0][o] = kHashInit;
    d.phash[0][o] = 0;
    d.n[0][o] = 0;
    d.ctx[0][o] = 0;
    d.score[0][o] = 0.0;
    s_ctx = 0;
  }
  if (d.len[b] == 0) return;  // uniform
  for (int k = tid; k < m.C; k += kHypThreads) s_enc[k] = d.enc[(size_t)b * d.T * m.C + k];
  __syncthreads();
  hyp_rows<kHypThreads>(m, d, b, 1, s_enc, &s_ctx);
}

// One frame of stream b.  Bound: latency; a chain of the state, normalisers, N + N wave
// maxima and the next rows' gathers, so every step's loads are issued together and as early
// as their addresses allow (the logits before anything else: their rows are the
// hypotheses' own), each wave picks its own N best without a barrier, and one wave merges
// the waves' lists.  Each thread scores its candidates once, into its own column
// of LDS (CACHED; larger sets are rescored from the logits in every round), and keeps its
// best, which only the thread whose candidate a round takes has to look for again.  (The
// scores in registers took all 512 of them and twice the time.)  B = 32, V = 500, 4 hypotheses, MI355X: 26.4
// us per frame before (workgroup argmax rounds, one gather round trip per element), now
// 15.6 us.
template <int NT, bool CACHED>
__global__ __launch_bounds__(NT) void k_hyp_step(ModelDev m, HypDev d, int t,
                                                 const float* __restrict__ logits,
                                                 const float2* __restrict__ stats, int* trace) {
  constexpr int NW = NT / 64;
  __shared__ double s_lse[kMaxHyps], s_sc[kMaxHyps], s_gs[kMaxHyps];
  __shared__ int s_gfirst[kMaxHyps], s_rpar[kMaxHyps], s_rlab[kMaxHyps], s_mj[kMaxHyps];
  __shared__ int s_last[kMaxHyps], s_n[kMaxHyps], s_ctx[kMaxHyps], s_nctx[kMaxHyps];
  __shared__ unsigned long long s_h[kMaxHyps], s_ph[kMaxHyps];
  __shared__ Cand s_list[NW * kMaxHyps], s_win[kMaxHyps];
  __shared__ int s_kept;
  __shared__ float s_enc[kMaxDim];
  extern __shared__ __align__(16) unsigned long long s_code[];  // [slot][NT] (CACHED)
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int N = d.N, V = m.V, Vpad = m.Vpad, nvt = m.Vpad / kJoinerBN;
  const int cur = t & 1, nx = cur ^ 1;
  const size_t o = (size_t)b * N;
  // Every load that needs no other one's result, requested together (the kernel is a chain
  // of memory round trips otherwise): lengths, the state (rows past nh hold old values that
  // are dropped), the normalisers' partials, the next encoder frame, the logits.
  const int len = d.len[b], nh_now = d.nh[cur][b];
  const int me = min(tid, N - 1);
  const double g_sc = d.score[cur][o + me];
  const int g_ctx = d.ctx[cur][o + me], g_n = d.n[cur][o + me];
  const unsigned long long g_h = d.hash[cur][o + me], g_ph = d.phash[cur][o + me];
  const float2 g_st = stats[(o + min(wave, N - 1)) * nvt + min(lane, nvt - 1)];
  const float* enc_next = d.enc + ((size_t)b * d.T + min(t + 1, d.T - 1)) * m.C;
  float g_enc[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) g_enc[u] = enc_next[min(tid + u * NT, m.C - 1)];
  // This thread's candidates: labels c = tid, tid + NT, ... of every hypothesis i, slot
  // i * per + (c - tid) / NT of its own column of s_code: the logit first (requested now,
  // eight at a time in flight), then the score's code.
  const int per = (V + NT - 1) / NT;
  unsigned long long* code = s_code + tid;
  if (t >= len) return;  // uniform
  const int nh = nh_now;
  const bool more = t + 1 < len;
  if (CACHED) {
    int i = 0, c = 0;  // hypothesis and first label of the slot, walked (no division)
    for (int s0 = 0; s0 < N * per; s0 += 8) {
      float z[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        z[u] = logits[(o + min(i, N - 1)) * Vpad + min(c + tid, V - 1)];
        c += NT;
        if (c >= V) {
          c = 0;
          ++i;
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (s0 + u < N * per) code[(s0 + u) * NT] = __float_as_uint(z[u]);
    }
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (tid + u * NT < m.C) s_enc[tid + u * NT] = g_enc[u];
  for (int k = tid + 2 * NT; k < m.C; k += NT) s_enc[k] = enc_next[k];
  if (tid < nh) {
    s_sc[tid] = g_sc;
    s_ctx[tid] = g_ctx;
    s_n[tid] = g_n;
    s_last[tid] = g_n > 0 ? g_ctx % V : -1;
    s_h[tid] = g_h;
    s_ph[tid] = g_ph;
  }
  // normaliser of each hypothesis's joiner row, one wave each
  for (int i = wave; i < nh; i += NW) {
    const float2* st = stats + (o + i) * nvt;
    float2 x = i == wave ? g_st : st[min(lane, nvt - 1)];
    if (lane >= nvt) x = make_float2(-INFINITY, 0.f);
    float M = x.x;
    for (int k = lane + 64; k < nvt; k += 64) M = fmaxf(M, st[k].x);
    M = wave_max(M);
    float S = x.y == 0.f ? 0.f : x.y * expf(x.x - M);
    for (int k = lane + 64; k < nvt; k += 64) S += st[k].y == 0.f ? 0.f : st[k].y * expf(st[k].x - M);
    S = wave_sum(S);
    if (lane == 0) s_lse[i] = (double)M + log((double)S);
  }
  __syncthreads();
  auto logp_of = [&](int i, float zz) { return (double)(float)((double)zz - s_lse[i]); };
  auto logp = [&](int i, int c) {
    return logp_of(i, CACHED ? __uint_as_float((unsigned)s_code[(i * per + c / NT) * NT + c % NT])
                             : logits[(o + i) * Vpad + c]);
  };
  // blank of y_i merges with label last(y_i) of y_j when y_j is y_i minus that label
  if (tid < nh) {
    const int i = tid;
    const double a = s_sc[i] + logp(i, 0);
    double gs = a;
    int gfirst = i * V, rpar = i, rlab = 0, mj = -1;
    const int ni = s_n[i];
    if (ni > 0) {
      const unsigned long long ph = s_ph[i];
      for (int j = 0; j < nh; ++j)
        if (s_h[j] == ph && s_n[j] == ni - 1) mj = j;
    }
    if (mj >= 0) {
      const int c = s_last[i];
      const double bs = s_sc[mj] + logp(mj, c);
      const double hi = fmax(a, bs), lo = fmin(a, bs);
      gs = d.merge_logadd ? hi + log1p(exp(lo - hi)) : hi;
      const int jidx = mj * V + c;
      if (jidx < gfirst) gfirst = jidx;
      if (bs > a || (bs == a && jidx < i * V)) {
        rpar = mj;
        rlab = c;
      }
    }
    s_gs[i] = gs;
    s_gfirst[i] = gfirst;
    s_rpar[i] = rpar;
    s_rlab[i] = rlab;
    s_mj[i] = mj;
  }
  __syncthreads();
  // The labels' scores, and this thread's best.  Blanks (c = 0) are kept apart; a label's
  // first index is its own.  Label c of y_i is not a candidate of its own when it is the
  // blank group of some y_k.
  Cand mine{0, 0x7fffffff, -1};
  if (CACHED)
    for (int i = 0; i < nh; ++i) {
      const double sc = s_sc[i], lse = s_lse[i];
#pragma unroll 2
      for (int k = 0; k < per; ++k) {
        const int c = tid + k * NT;
        unsigned long long* e = code + (i * per + k) * NT;
        const float z = __uint_as_float((unsigned)*e);
        *e = c > 0 && c < V ? score_code(sc + (double)(float)((double)z - lse)) : 0;
      }
    }
  if (CACHED)
    for (int k = 0; k < nh; ++k)
      if (s_mj[k] >= 0 && s_last[k] % NT == tid) code[(s_mj[k] * per + s_last[k] / NT) * NT] = 0;
  auto scan = [&]() {  // (slots in ascending index order: of equal scores the first stays)
    mine.code = 0;
    for (int i = 0; i < nh; ++i)
#pragma unroll 2
      for (int k = 0; k < per; ++k) {
        const unsigned long long x = code[(i * per + k) * NT];
        if (x > mine.code) mine = Cand{x, i * V + tid + k * NT, i * V + tid + k * NT};
      }
  };
  if (CACHED) scan();
  auto merged = [&](int i, int c) {
    bool x = false;
    for (int k = 0; k < nh; ++k) x = x || (s_mj[k] == i && s_last[k] == c);
    return x;
  };
  // the blank groups: one per lane of wave 0
  Cand blank{0, 0x7fffffff, -1};
  if (tid < nh) blank = Cand{score_code(s_gs[tid]), s_gfirst[tid], tid * V};
  // each wave's N best of its own candidates
  for (int r = 0; r < N; ++r) {
    Cand best = mine;
    if (!CACHED) {
      best.code = 0;
      for (int i = 0; i < nh; ++i)
        for (int c = tid; c < V; c += NT) {
          const int idx = i * V + c;
          bool skip = c == 0 || merged(i, c);
          for (int q = 0; q < r; ++q) skip = skip || s_list[wave * N + q].idx == idx;
          if (skip) continue;
          const unsigned long long x = score_code(s_sc[i] + logp(i, c));
          if (x > best.code) best = Cand{x, idx, idx};
        }
    }
    if (blank.code != 0 && cand_before(blank, best)) best = blank;
    const Cand w = wave_best(best);
    if (lane == 0) s_list[wave * N + r] = w;
    if (w.code != 0) {  // taken: its owner looks for its next best
      if (blank.idx == w.idx) blank.code = 0;
      if (CACHED && mine.code != 0 && mine.idx == w.idx) {
        const int i = w.idx / V;
        code[(i * per + (w.idx - i * V) / NT) * NT] = 0;
        scan();
      }
    }
    if (!CACHED) {  // the wave reads its list in the next round
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
  __syncthreads();
  // the N best of the waves' lists
  if (wave == 0) {
    constexpr int Q = (NW * kMaxHyps + 63) / 64;
    Cand x[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q)
      x[q] = lane + 64 * q < NW * N ? s_list[lane + 64 * q] : Cand{0, 0x7fffffff, -1};
    int kept = 0;
    for (int r = 0; r < N; ++r) {
      Cand best = x[0];
#pragma unroll
      for (int q = 1; q < Q; ++q)
        if (cand_before(x[q], best)) best = x[q];
      const Cand w = wave_best(best);
      if (w.code == 0) break;  // uniform: no candidate left
      if (lane == 0) s_win[r] = w;
      kept = r + 1;
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (x[q].idx == w.idx) x[q].code = 0;
    }
    if (lane == 0) s_kept = kept;
  }
  __syncthreads();
  const int kept = s_kept;
  // the kept hypotheses, in rank order, and their back-pointers
  if (tid < kept) {
    const int k = tid, idx = s_win[k].idx;
    const int i = idx / V, c = idx - i * V;
    const size_t q = o + k;
    const int ctx = c == 0 ? s_ctx[i] : (s_ctx[i] % V) * V + c;
    const int par = c == 0 ? s_rpar[i] : i, lab = c == 0 ? s_rlab[i] : c;
    s_nctx[k] = ctx;
    d.ctx[nx][q] = ctx;
    d.hash[nx][q] = c == 0 ? s_h[i] : hash_push(s_h[i], c);
    d.phash[nx][q] = c == 0 ? s_ph[i] : s_h[i];
    d.n[nx][q] = s_n[i] + (c != 0);
    d.score[nx][q] = code_score(s_win[k].code);
    d.hist[((size_t)t * d.B + b) * N + k] = par << 16 | lab;
    if (trace) {
      int* tr = trace + (((size_t)(t + 1) * d.B + b) * N + k) * 2;
      tr[0] = par;
      tr[1] = lab;
    }
  }
  if (tid == 0) d.nh[nx][b] = kept;
  if (more) {  // uniform: the next frame's joiner rows
    __syncthreads();
    hyp_rows<NT>(m, d, b, kept, s_enc, s_nctx);
  }
}

// Result: the first hypothesis after the stream's last frame, traced back.  The chain of
// back-pointers is followed in LDS, over stages of the history copied there by the whole
// workgroup; the labels land at the end of out_tokens' row, last first, and are then moved
// to its front.
constexpr int kHypStage = 8192;

__global__ __launch_bounds__(256) void k_hyp_final(HypDev d, int* out_tokens, int* out_ntok,
                                                   double* out_scores) {
  __shared__ int s_hist[kHypStage];
  __shared__ int s_n;
  const int b = blockIdx.x, tid = threadIdx.x, T = d.T, N = d.N;
  const int len = d.len[b], frames = kHypStage / N;
  int* out = out_tokens + (size_t)b * T;
  int k = 0, n = 0;
  for (int f1 = len; f1 > 0; f1 -= frames) {
    const int f0 = max(0, f1 - frames);
    __syncthreads();
    for (int i = tid; i < (f1 - f0) * N; i += 256) {
      const int f = i / N;
      s_hist[i] = d.hist[((size_t)(f0 + f) * d.B + b) * N + (i - f * N)];
    }
    __syncthreads();
    if (tid == 0)
      for (int f = f1 - 1; f >= f0; --f) {
        const int v = s_hist[(f - f0) * N + k];
        if ((v & 0xffff) > 0) out[T - 1 - n++] = v & 0xffff;
        k = v >> 16;
      }
  }
  if (tid == 0) {
    out_scores[b] = d.score[len & 1][(size_t)b * N];
    out_ntok[b] = n;
    s_n = n;
  }
  __syncthreads();
  n = s_n;
  // (ascending blocks of 256: a block's targets are never later than its sources)
  for (int i0 = 0; i0 < T; i0 += 256) {
    const int i = i0 + tid;
    const int v = i < n ? out[T - n + i] : -1;
    __syncthreads();
    if (i < T) out[i] = v;
    __syncthreads();
  }
}

}  // namespace

hipError_t launch_hyp_init(const ModelDev& m, const HypDev& d, hipStream_t st) {
  hipLaunchKernelGGL(k_hyp_init, dim3(d.B), dim3(kHypThreads), 0, st, m, d);
  return hipGetLastError();
}

namespace {

template <int NT, bool CACHED>
hipError_t launch_hyp_step_t(const ModelDev& m, const HypDev& d, int t, size_t lds,
                             const float* logits, const float2* stats, int* trace, hipStream_t st) {
  static LdsGrant grant;
  if (lds > 32768) {
    const hipError_t e = grant((const void*)k_hyp_step<NT, CACHED>, lds);
    if (e != hipSuccess) return e;
  }
  hipEvent_t ea, eb;
  if (take_launch_events(&ea, &eb))  // per-kernel profiling: events in the dispatch packet
    hipExtLaunchKernelGGL((k_hyp_step<NT, CACHED>), dim3(d.B), dim3(NT), (unsigned)lds, st, ea, eb, 0u,
                          m, d, t, logits, stats, trace);
  else
    hipLaunchKernelGGL((k_hyp_step<NT, CACHED>), dim3(d.B), dim3(NT), lds, st, m, d, t, logits,
                       stats, trace);
  return hipGetLastError();
}

}  // namespace

// Four waves (the shorter merge) for up to 16 candidates per thread, sixteen while the
// scores fit the LDS.
hipError_t launch_hyp_step(const ModelDev& m, const HypDev& d, int t, const float* logits,
                           const float2* stats, int* trace, hipStream_t st) {
  auto slots = [&](int nt) { return (size_t)d.N * ((m.V + nt - 1) / nt); };
  if (slots(kHypThreads) <= 16)
    return launch_hyp_step_t<kHypThreads, true>(m, d, t, slots(kHypThreads) * kHypThreads * 8, logits,
                                                stats, trace, st);
  const size_t lds = slots(kHypWideThreads) * kHypWideThreads * 8;
  if (lds <= kHypCache) return launch_hyp_step_t<kHypWideThreads, true>(m, d, t, lds, logits, stats, trace, st);
  return launch_hyp_step_t<kHypWideThreads, false>(m, d, t, 0, logits, stats, trace, st);
}

hipError_t launch_hyp_final(const HypDev& d, int* out_tokens, int* out_ntok, double* out_scores,
                            hipStream_t st) {
  hipLaunchKernelGGL(k_hyp_final, dim3(d.B), dim3(256), 0, st, d, out_tokens, out_ntok,
                     out_scores);
  return hipGetLastError();
}

}  // namespace tbs
