// Forward recursions of the transducer losses over the (frame t, labels emitted u) grid
// (Sec. 3): the standard recursion, eq. (1); the modified transducer, eq. (2), where
// emitting a label also moves to the next frame; and the constrained transducer, eq. (3),
// where a label is followed by the blank of the new context on the same frame.  Inputs
// are the log-probabilities the joiner gives at each cell: blank [B][T][U+1] and label
// [B][T][U] (the label u+1 of the utterance, after u labels).  Scores are fp64.
//
// Two kernels, one workgroup per utterance:
//  - k_transducer_ring, the usual one: the recursion in the linear domain (described
//    with it);
//  - k_transducer_logs, in the log domain: for grids whose ring does not fit the LDS, and
//    (as a device function) for utterances with an input that is not a number within
//    [kRingMinLog, kRingMaxLog].
#include <hip/hip_runtime.h>

#include <cmath>

#include "internal.h"

namespace tbs {
namespace {

constexpr int kRingThreads = 512;  // both kernels

__device__ __forceinline__ double ninf() { return -__builtin_inf(); }

// A double's exponent field, as its high word's integer units.
__device__ __forceinline__ unsigned hi_word(double x) {
  return (unsigned)((unsigned long long)__double_as_longlong(x) >> 32);
}
__device__ __forceinline__ double with_hi(double x, unsigned hi) {
  const unsigned lo = (unsigned)(unsigned long long)__double_as_longlong(x);
  return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}
// x 2^n, for results that are normal numbers
__device__ __forceinline__ double scaled(double x, int n) {
  return with_hi(x, hi_word(x) + ((unsigned)n << 20));
}

// log(e^a + e^b); a term below e^-300 of the other adds nothing.  The series: e^f = 1 + f +
// ... + f^12 / 12! with |f| <= ln 2 / 2, and log z = 2 (s + s^3 / 3 + ... + s^21 / 21) with
// s = (z - 1) / (z + 1), z = 1 + e^(lo - hi) or half of it above sqrt 2 (|s| < 0.172).  The
// steps of the log-domain recursion are a chain of these: no branches, the constants in scalar
// registers.
struct LogAdd {
  double e[11], l[10];
  double log2e = 1.4426950408889634, shift = 6755399441055744.0;
  double ln2 = 0.69314718055994529, ln2_lo = 2.3190468138462996e-17;  // ln 2 and its rounding
  __device__ __forceinline__ LogAdd() {
    double f = 2.0;
#pragma unroll
    for (int n = 0; n < 11; ++n) {
      e[n] = 1.0 / f;  // 1 / (n + 2)!
      f *= n + 3;
      asm("" : "+s"(e[n]));
    }
#pragma unroll
    for (int n = 0; n < 10; ++n) {
      l[n] = 1.0 / (2 * n + 3);
      asm("" : "+s"(l[n]));
    }
    asm("" : "+s"(log2e), "+s"(shift), "+s"(ln2), "+s"(ln2_lo));
  }
  __device__ __forceinline__ double operator()(double a, double b) const {
    const bool ge = a >= b;  // (fmax and fmin would drop a NaN)
    const double hi = ge ? a : b, lo = ge ? b : a, d = lo - hi;
    const bool near = d >= -300.0;
    const double x = near ? d : -300.0;
    const double t = __builtin_fma(x, log2e, shift), k = t - shift;
    const double f = __builtin_fma(-k, ln2_lo, __builtin_fma(-k, ln2, x));
    double p = e[10];
#pragma unroll
    for (int n = 9; n >= 0; --n) p = __builtin_fma(p, f, e[n]);
    p = __builtin_fma(p, f, 1.0);
    p = __builtin_fma(p, f, 1.0);
    const double y = scaled(p, (int)(unsigned)(unsigned long long)__double_as_longlong(t));
    const bool half = y > 0.41421356237309503;
    const double den = y + (half ? 3.0 : 2.0), num = half ? y - 1.0 : y;
    double r = __builtin_amdgcn_rcp(den);
    r = r * __builtin_fma(-den, r, 2.0);  // two Newton steps
    r = r * __builtin_fma(-den, r, 2.0);
    const double s = num * r, s2 = s * s;
    double q = l[9];
#pragma unroll
    for (int n = 8; n >= 0; --n) q = __builtin_fma(q, s2, l[n]);
    q = __builtin_fma(q, s2, 1.0);
    const double sum = hi + __builtin_fma(2.0 * s, q, half ? ln2 : 0.0);
    return near ? sum : lo == ninf() || d == d ? hi : d;
  }
};

// Pointers of the log-domain recursion, a called function: accesses by generic ones would
// count as both kinds, and each wait for LDS data would be one for the loads in flight.
typedef __attribute__((address_space(3))) double lds_double;
typedef __attribute__((address_space(1))) float global_float;

// Workgroup barrier that orders LDS accesses only: global loads requested ahead of it stay
// in flight across it (a full barrier waits for them, a memory round trip per chunk).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Log-domain recursion of utterance b by the whole workgroup, thread tid owning cells tid
// and tid + kRingThreads of a row; step s computes row s (eq. 2, 3) or, since row t of
// eq. (1) also depends on its own left neighbour, the cells with t + u = s (eq. 1), from
// the state after step s - 1.  buf: [2][U + 1] doubles of LDS.  One log-add and one
// barrier per step, the next step's inputs in flight meanwhile.
// Bound: the log-add's instructions.  MI355X, with the ring's pass before it: modified,
// T = 250, U = 80, an infinity in every utterance: B = 32 127 us, B = 1,024 302 us (the
// library's exp and log1p and waits for every load: 225 and 560; one wave per utterance and
// no ring: 247 and 297).  By itself: standard, T = 500, U = 400, B = 4 680 us (1,070; 4,610).
template <int KIND>
__device__ __attribute__((noinline)) void log_recursion(const float* __restrict__ blank,
                                                        const float* __restrict__ label, int Tb,
                                                        int Ub, int b, int T, int U,
                                                        double* __restrict__ total,
                                                        float* __restrict__ alpha,
                                                        int* __restrict__ status, lds_double* buf) {
  constexpr int Q = 64 * kTransducerMaxK / kRingThreads;  // cells per thread
  const LogAdd log_add;
  // Short rows leave most waves idle; which ones work turns with the utterance, so that the
  // workgroups of a compute unit (every 256th, as they are handed out) load all its SIMDs.
  const int tid = (threadIdx.x + 128 * ((b + (b >> 8)) & 3)) % kRingThreads, U1 = U + 1;
  const global_float* bl = (const global_float*)blank + (size_t)b * T * U1;
  const global_float* lb = U > 0 ? (const global_float*)label + (size_t)b * T * U : bl;
  global_float* al = alpha ? (global_float*)alpha + (size_t)b * (T + 1) * U1 : nullptr;
  constexpr int kOut = KIND == 0 ? 0 : 1;  // alpha row of row i: i + kOut
  for (int u = tid; u < U1; u += kRingThreads) {
    const double v = u == 0 ? 0.0 : ninf();
    buf[u] = v;
    if (al && KIND != 0) al[u] = (float)v;
  }
  if (al)  // cells past the utterance's labels
    for (int i = 0; i < Tb; ++i)
      for (int u = Ub + 1 + tid; u < U1; u += kRingThreads) al[(size_t)(i + kOut) * U1 + u] = -INFINITY;
  const int steps = Tb + (KIND == 0 ? Ub : 0);
  auto active = [&](int s, int u, int& i) {
    i = KIND == 0 ? s - u : s;
    return i >= 0 && i < Tb && u <= Ub;
  };
  // inputs of the next step (of a cell that is inactive, another's: no branches around the
  // loads, which would make the step wait for all of them)
  float xb[Q], xl[Q];
  auto request = [&](int s) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int u = min(tid + q * kRingThreads, Ub);
      const int i = min(max(KIND == 0 ? s - u : s, 0), Tb - 1);
      xb[q] = bl[(size_t)max(i - 1 + kOut, 0) * U1 + u];
      xl[q] = lb[(size_t)i * U + max(u - 1, 0)];
    }
  };
  request(0);
  lds_barrier();
  for (int s = 0; s < steps; ++s) {
    const lds_double* prev = buf + (s & 1) * U1;
    lds_double* next = buf + (~s & 1) * U1;
    float cb[Q], cl[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      cb[q] = xb[q];
      cl[q] = xl[q];
    }
    request(s + 1);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int u = tid + q * kRingThreads;
      if (u >= U1) continue;
      int i;
      const bool act = active(s, u, i);
      const double old = prev[u];
      double v = old + (double)cb[q];
      if (KIND == 0 && i == 0) v = u == 0 ? 0.0 : ninf();
      double w = prev[max(u - 1, 0)] + (double)cl[q];
      if (KIND == 2) w += (double)cb[q];
      v = log_add(v, u > 0 ? w : ninf());
      if (al && act) al[(size_t)(i + kOut) * U1 + u] = (float)v;
      next[u] = act ? v : old;
    }
    lds_barrier();
  }
  if (tid == 0) {
    double res = buf[(steps & 1) * U1 + Ub];
    if (KIND == 0) res += (double)bl[(size_t)(Tb - 1) * U1 + Ub];
    total[b] = res;
    if (status) status[b] = 0;
  }
}

// Lengths of utterance b; false if out of range (the result is then NaN, status 1).
__device__ __forceinline__ bool utterance(const int* lengths, int b, int T, int U, double* total,
                                          int* status, bool writer, int& Tb, int& Ub) {
  Tb = lengths[2 * b];
  Ub = lengths[2 * b + 1];
  if (Tb >= 1 && Tb <= T && Ub >= 0 && Ub <= U) return true;
  if (writer) {
    total[b] = __builtin_nan("");
    if (status) status[b] = 1;
  }
  return false;
}

template <int KIND>
__global__ __launch_bounds__(kRingThreads) void k_transducer_logs(
    const float* __restrict__ blank, const float* __restrict__ label,
    const int* __restrict__ lengths, int T, int U, double* __restrict__ total,
    float* __restrict__ alpha, int* __restrict__ status) {
  __shared__ double buf[2 * 64 * kTransducerMaxK];
  const int b = blockIdx.x;
  int Tb, Ub;
  if (!utterance(lengths, b, T, U, total, status, threadIdx.x == 0, Tb, Ub)) return;
  log_recursion<KIND>(blank, label, Tb, Ub, b, T, U, total, alpha, status, (lds_double*)buf);
}

// ---------------------------------------------------------------------------
// Linear-domain recursion.  A cell is m * 2^e with m a double in [0.5, 1) and e an int, so
// nothing underflows (an unreachable cell has e near kZeroExp), and one cell is two
// products, a scaled sum and a renormalisation (thirteen instructions, the scaling and
// renormalising ones on the exponent fields as integers) where a log-add of the log domain
// is an exp and a log1p (over a hundred).  The exponentials of the inputs do not depend
// on the recursion and are taken ahead of it by the workgroup's other waves.
//
// One workgroup (eight waves) per utterance.  Step row i of cell u takes
//   eq. (2), (3): row i + 1 from row i:  pb = e^blank(i, u),     pl = e^label(i, u - 1);
//   eq. (1):      row i:                 pb = e^blank(i - 1, u), pl = e^label(i, u - 1)
// from a ring of rows in LDS, 16 bytes (pb, pl) per cell.  Work goes in chunks of R rows
// with one barrier each.  While wave 0 runs chunk c, waves 1..7
//   - turn chunk c + 1's inputs, already in registers, into ring rows, and request chunk
//     c + 2's;
//   - if alpha is asked for, take the logarithms of the rows wave 0 has finished, which
//     it left in the ring in place of their inputs, and store them, coalesced.
// Wave 0: lane l owns cells l*K .. l*K+K-1.  For eq. (1), whose row also depends on its
// left neighbour, lane l runs row s - l on step s, so the neighbour's last cell of the
// same row is the state one lane to the left after the previous step; for eq. (2) and
// (3) every lane runs row s and that state is the previous row's.  Either way it is one
// wave shift per step.
//
// Bound: wave 0 issues about 50 instructions per step with two cells per lane (some 300
// cycles, T + U / K steps); with several utterances per compute unit, that and the
// exponentials (about 30 instructions for each of T (2 U + 1) inputs) share its four
// SIMDs.  T = 250, U = 80, MI355X: B = 32 modified with alpha 310 -> 46 us, B = 1,024
// standard, ragged, without alpha 1,075 -> 115 us (before: log domain, one wave per
// utterance).  Sixteen waves instead of eight for batches of up to one utterance per
// compute unit measured the same (47 us): the workers have slack.

constexpr int kRingWorkers = kRingThreads - 64;
constexpr int kRingLoads = 5;         // blank (and label) elements per worker and chunk
// Inputs the linear domain takes: e^x is then within [2^-433, 2^73] and a term (an input
// times a mantissa) within [2^-434, 2^73].  A term may be scaled down by up to kMaxShift: it
// stays a normal number (2^-1004), and whatever is scaled down that far (an unreachable
// cell, a term that many powers of two below) is at most 2^-497, nothing beside a live term.
// (Log-probabilities are at most 0; the room above it is for unnormalised scores.)
constexpr float kRingMinLog = -300.f, kRingMaxLog = 50.f;
constexpr int kMaxShift = 570;
constexpr int kZeroExp = -(1 << 29);  // exponent of an unreachable cell; any below half of
                                      // it counts as one
constexpr int kRingMaxSteps = 200000; // (steps * 2 * 300 / ln 2 stays above kZeroExp / 2)
constexpr size_t kRingLds = kMaxLds - 1024;

// e^x for |x| <= 300, to about 2e-16: x = k ln 2 + f, Taylor series in f up to f^12 / 12!
// (|f| <= ln 2 / 2, so the rest is below 2e-16).  k comes out of the low bits of
// x / ln 2 + 1.5 * 2^52, whose unit is 1.  The constants are held in scalar registers
// (as literals each would be two moves into vector registers before its use).
struct ExpLogProb {
  double c[11];
  double log2e = 1.4426950408889634, shift = 6755399441055744.0;
  double ln2 = 0.69314718055994529, ln2_lo = 2.3190468138462996e-17;  // ln 2 and its rounding
  __device__ __forceinline__ ExpLogProb() {
    double f = 2.0;
#pragma unroll
    for (int n = 0; n < 11; ++n) {
      c[n] = 1.0 / f;  // 1 / (n + 2)!
      f *= n + 3;
      asm("" : "+s"(c[n]));
    }
    asm("" : "+s"(log2e), "+s"(shift), "+s"(ln2), "+s"(ln2_lo));
  }
  __device__ __forceinline__ double operator()(float xf) const {
    const double x = (double)xf;
    const double t = __builtin_fma(x, log2e, shift), k = t - shift;
    const double f = __builtin_fma(-k, ln2_lo, __builtin_fma(-k, ln2, x));
    double p = c[10];
#pragma unroll
    for (int n = 9; n >= 0; --n) p = __builtin_fma(p, f, c[n]);
    p = __builtin_fma(p, f, 1.0);
    p = __builtin_fma(p, f, 1.0);
    return scaled(p, (int)(unsigned)(unsigned long long)__double_as_longlong(t));
  }
};

// log(m 2^e) for m in [0.5, 1), to about 1e-12: with m moved to [sqrt 1/2, sqrt 2) and
// s = (m - 1) / (m + 1), log m = 2 (s + s^3 / 3 + s^5 / 5 + ...), |s| < 0.172.
__device__ __forceinline__ double log_cell(double m, int e) {
  if (m < 0.70710678118654752) {
    m += m;
    --e;
  }
  const double d = m + 1.0;
  double r = __builtin_amdgcn_rcp(d);
  r = r * __builtin_fma(-d, r, 2.0);  // two Newton steps
  r = r * __builtin_fma(-d, r, 2.0);
  const double s = (m - 1.0) * r, q = s * s;
  double p = 1.0 / 15.0;
  p = __builtin_fma(p, q, 1.0 / 13.0);
  p = __builtin_fma(p, q, 1.0 / 11.0);
  p = __builtin_fma(p, q, 1.0 / 9.0);
  p = __builtin_fma(p, q, 1.0 / 7.0);
  p = __builtin_fma(p, q, 1.0 / 5.0);
  p = __builtin_fma(p, q, 1.0 / 3.0);
  p = __builtin_fma(p, q, 1.0);
  return __builtin_fma((double)e, 0.69314718055994529, 2.0 * s * p);
}

// The value one lane to the left; lane 0 receives fill.
__device__ __forceinline__ int from_left(int v, int fill) {
  return __builtin_amdgcn_update_dpp(fill, v, 0x138, 0xf, 0xf, false);  // wave_shr:1
}
__device__ __forceinline__ double from_left(double v, double fill) {
  const unsigned lo = (unsigned)from_left((int)(unsigned)(unsigned long long)__double_as_longlong(v),
                                          (int)(unsigned)(unsigned long long)__double_as_longlong(fill));
  const unsigned hi = (unsigned)from_left((int)hi_word(v), (int)hi_word(fill));
  return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}

// steps whose ring cells wave 0 requests together, one group ahead of their use (an LDS
// read takes longer than a step)
template <int K>
constexpr int kRingGroup = K <= 2 ? 4 : K == 4 ? 2 : 1;

// R: rows per chunk (a multiple of 2 kRingGroup<K>; R (U + 1) <= kRingLoads kRingWorkers);
// ring: rows in LDS, a multiple of R, at least 2 R (with alpha 3 R) plus eq. (1)'s lag of
// U / K;
// rs: cells per ring row, at least U + 1 rounded up to K.
template <int K, int KIND, bool ALPHA>
__global__ __launch_bounds__(kRingThreads, K <= 4 || (K == 8 && KIND != 0) ? 4 : 2) void k_transducer_ring(
    const float* __restrict__ blank, const float* __restrict__ label,
    const int* __restrict__ lengths, int T, int U, double* __restrict__ total,
    float* __restrict__ alpha, int* __restrict__ status, int R, int ring, int rs) {
  constexpr int G = kRingGroup<K>;
  extern __shared__ __align__(16) double2 cells[];  // [ring][rs]
  __shared__ int s_bad[2];  // set in even and in odd groups of four chunks
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  int Tb, Ub;
  if (!utterance(lengths, b, T, U, total, status, tid == 0, Tb, Ub)) return;  // uniform
  const int U1 = U + 1;
  const float* bl = blank + (size_t)b * T * U1;
  const float* lb = label + (size_t)b * T * U;
  constexpr int kOut = KIND == 0 ? 0 : 1;   // alpha row of step row i: i + kOut
  const int lag = KIND == 0 ? Ub / K : 0;   // rows the last lane in use is behind lane 0
  const int nchunks = (Tb + lag + R - 1) / R;
  float* al = ALPHA ? alpha + ((size_t)b * (T + 1) + kOut) * U1 : nullptr;
  const float inv_U1 = 1.f / (float)U1;

  // alpha of step rows [i0, i1), left in the ring as (m, e)
  auto store_rows = [&](int i0, int i1, int first, int stride) {
    i0 = max(i0, 0);
    i1 = min(i1, Tb);
    const int s0 = i0 % ring;
    for (int j = first; j < (i1 - i0) * U1; j += stride) {
      const int r = (int)(((float)j + 0.5f) * inv_U1), u = j - r * U1;  // (j stays below 2^20)
      int slot = s0 + r;
      if (slot >= ring) slot -= ring;
      const double2 c = cells[slot * rs + u];
      const int e = (int)(unsigned)(unsigned long long)__double_as_longlong(c.y);
      al[(size_t)i0 * U1 + j] = u <= Ub && e > kZeroExp / 2 ? (float)log_cell(c.x, e) : -INFINITY;
    }
  };

  if (tid < 2) s_bad[tid] = 0;
  // An input the linear domain does not take ends both loops within the next group of chunks:
  // while a group reads the flag of the one before, only its own can be set, so all waves
  // see the same.  (Not for eq. (1): the check alone costs its loop 3%, and its fallback is
  // shorter than what it replaces by more than the ring's pass.)
  int end_chunk = nchunks;
  auto seen = [&](int c) {
    return KIND != 0 && c > 0 && c % 4 == 0 && __builtin_amdgcn_readfirstlane(s_bad[~(c / 4) & 1]) != 0;
  };
  if (tid >= 64) {
    // Worker w handles elements j = w, w + kRingWorkers, ... of a chunk's R x U1 blank and
    // R x U label values.  A chunk's rows are consecutive in memory and (ring being a
    // multiple of R) in the ring, so element q keeps its offset within the chunk: its
    // index in memory, its cell in the ring and its row never change.
    // An element outside the utterance is not read and counts as probability 1: what it
    // leads to is either not used (cells past the utterance's labels) or multiplies a cell
    // that is unreachable (label into cell 0, blank into row 0 of eq. 1), which keeps
    // every term a positive normal number.  The exception is eq. (1)'s first cell, whose
    // blank from a virtual row above it does have probability 1.
    const int w = tid - 64;
    int bcell[kRingLoads], lcell[kRingLoads];  // ring cell of element q within the chunk
    int brow[kRingLoads], lrow[kRingLoads];    // its row (past every Tb: never read)
    float xb[kRingLoads], xl[kRingLoads];
#pragma unroll
    for (int q = 0; q < kRingLoads; ++q) {
      const int j = w + q * kRingWorkers;
      const int rb = j / U1, ub = j - rb * U1;
      const int rl = U > 0 ? j / U : R, ul = j - rl * U + 1;  // the label leads to cell ul
      bcell[q] = rb < R ? rb * rs + ub : -1;
      lcell[q] = rl < R ? rl * rs + ul : -1;
      brow[q] = ub <= Ub ? rb : kRingMaxSteps;
      lrow[q] = ul <= Ub ? rl : kRingMaxSteps;
    }
    auto request = [&](int i0) {
      const float* gb = bl + (ptrdiff_t)(i0 - 1 + kOut) * U1;
      const float* gl = lb + (ptrdiff_t)i0 * U;
      const int left = Tb - i0;
#pragma unroll
      for (int q = 0; q < kRingLoads; ++q) {
        xb[q] = 0.f;
        xl[q] = 0.f;
        if (bcell[q] >= 0 && brow[q] < left && (KIND != 0 || i0 + brow[q] > 0))
          xb[q] = gb[w + q * kRingWorkers];
        if (lcell[q] >= 0 && lrow[q] < left) xl[q] = gl[w + q * kRingWorkers];
      }
    };
    const ExpLogProb exp_log_prob;
    // the largest and the most negative input seen, as bits (as integers of either kind a
    // NaN's are beyond any number's of its sign)
    int highest = 0;
    unsigned lowest = 0;
    auto note = [&](float x) {
      highest = max(highest, __float_as_int(x));
      lowest = max(lowest, __float_as_uint(x));
    };
    int c0 = 0;          // ring cell of the next chunk's first row
    auto produce = [&]() {
#pragma unroll
      for (int q = 0; q < kRingLoads; ++q) {
        if (bcell[q] >= 0) {
          note(xb[q]);
          reinterpret_cast<double*>(cells + c0 + bcell[q])[0] = exp_log_prob(xb[q]);
        }
        if (lcell[q] >= 0) {
          note(xl[q]);
          reinterpret_cast<double*>(cells + c0 + lcell[q])[1] = exp_log_prob(xl[q]);
        }
      }
      for (int r = w; r < R; r += kRingWorkers)  // no label leads to cell 0
        reinterpret_cast<double*>(cells + c0 + r * rs)[1] = 1.0;
      c0 += R * rs;
      if (c0 == ring * rs) c0 = 0;
    };
    request(0);
    if (ALPHA && KIND != 0)  // alpha row 0
      for (int u = w; u < U1; u += kRingWorkers) (al - U1)[u] = u == 0 ? 0.f : -INFINITY;
    produce();
    request(R);
    lds_barrier();
    for (int c = 0; c < end_chunk; ++c) {
      if (seen(c)) end_chunk = c;  // (this chunk's work is harmless)
      if (c + 1 < nchunks) produce();
      if (c + 2 < nchunks) request((c + 2) * R);
      if (ALPHA) store_rows((c - 1) * R - lag, c * R - lag, w, kRingWorkers);
      if (highest > __float_as_int(kRingMaxLog) || lowest > __float_as_uint(kRingMinLog)) s_bad[c / 4 & 1] = 1;
      lds_barrier();
    }
  } else {
    __builtin_amdgcn_s_setprio(3);  // the other waves have slack
    const int c0 = lane * K, cells_row = (U1 + K - 1) / K * K;
    const int coff = min(c0, cells_row - K);  // lanes past the row read its last cells
    const bool keep = ALPHA && c0 <= Ub;
    double m[K];
    int e[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      m[k] = 0.5;
      e[k] = c0 + k == 0 ? 1 : kZeroExp;
    }
    int row = KIND == 0 ? -lane : 0;  // this lane's next row
    // its ring cells: the row's slot is the row modulo ring
    int at = (KIND == 0 ? (ring - lane % ring) % ring : 0) * rs + coff;
    const int end = ring * rs + coff;
    double2 pa[G][K], pb[G][K];
    int sa[G], sb[G];
    auto fetch = [&](double2(&x)[G][K], int(&xs)[G]) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        xs[g] = at;
        at += rs;
        if (at >= end) at -= ring * rs;
#pragma unroll
        for (int k = 0; k < K; ++k) x[g][k] = cells[xs[g] + k];
      }
    };
    auto steps = [&](const double2(&x)[G][K], const int(&xs)[G]) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const bool act = row >= 0 && row < Tb;  // uniform for eq. (2), (3)
        ++row;
        if (KIND != 0 && !act) continue;
        double lm = from_left(m[K - 1], 0.5);
        int le = from_left(e[K - 1], kZeroExp);
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const double om = m[k];
          const int oe = e[k];
          const int top = max(oe, le);
          double v = scaled(KIND == 2 ? om : om * x[g][k].x, max(oe - top, -kMaxShift)) +
                     scaled(lm * x[g][k].y, max(le - top, -kMaxShift));
          if (KIND == 2) v *= x[g][k].x;
          const unsigned hi = hi_word(v);
          const double vm = with_hi(v, (hi & 0x000fffffu) | (1022u << 20));
          const int ve = top + (int)(hi >> 20) - 1022;
          m[k] = KIND != 0 || act ? vm : om;
          e[k] = KIND != 0 || act ? ve : oe;
          lm = KIND == 0 ? m[k] : om;
          le = KIND == 0 ? e[k] : oe;
        }
        if (keep && act) {
#pragma unroll
          for (int k = 0; k < K; ++k)
            cells[xs[g] + k] = make_double2(m[k], __longlong_as_double((long long)(unsigned)e[k]));
        }
      }
    };
    lds_barrier();
    for (int c = 0; c < end_chunk; ++c) {
      if (seen(c)) end_chunk = c;  // (this chunk's work is harmless)
      fetch(pa, sa);
      for (int g0 = 0; g0 < R; g0 += 2 * G) {
        fetch(pb, sb);
        steps(pa, sa);
        if (g0 + 2 * G < R) fetch(pa, sa);
        steps(pb, sb);
      }
      lds_barrier();
    }
    if (lane == Ub / K && !(s_bad[0] | s_bad[1])) {
      double mine = 0.5;
      int exp2 = kZeroExp;
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (c0 + k == Ub) {
          mine = m[k];
          exp2 = e[k];
        }
      double res = exp2 > kZeroExp / 2 ? __builtin_fma((double)exp2, 0.69314718055994529, log(mine)) : ninf();
      if (KIND == 0) res += (double)bl[(size_t)(Tb - 1) * U1 + Ub];
      total[b] = res;
      if (status) status[b] = 0;
    }
  }
  if (s_bad[0] | s_bad[1]) {  // uniform
    __syncthreads();  // the alpha rows stored so far are complete before others store theirs
    log_recursion<KIND>(blank, label, Tb, Ub, b, T, U, total, alpha, status,
                        (lds_double*)cells);
    return;
  }
  if (ALPHA) store_rows((nchunks - 1) * R - lag, Tb, tid, kRingThreads);
}

struct RingPlan {
  int K, R, ring, rs;  // K = 0: the ring does not fit
  size_t lds;
};

// Cells per lane and rows per chunk of k_transducer_ring.  A lane takes as few cells as
// it can (the step's chain grows with them), unless eq. (1)'s lag of U / K rows makes the
// ring too large; chunks are as long as the workers' registers and the LDS allow (fewer
// barriers).  More utterances than compute units: half the LDS, so that two workgroups
// share one.
RingPlan plan_ring(int kind, int B, int T, int U, bool alpha, int ncu) {
  const RingPlan none{0, 0, 0, 0, 0};
  const int U1 = U + 1;
  if (T + U > kRingMaxSteps) return none;
  int K0 = 1;
  while (64 * K0 < U1) K0 *= 2;
  for (int half = B > ncu; half >= 0; --half)
    for (int K = K0; K <= kTransducerMaxK; K *= 2) {
      const int cells = round_up(U1, K);
      // eq. (1): lane l reads row s - l, so the lanes' addresses step by K - rs cells: odd,
      // for distinct banks
      const int rs = kind == 0 && (cells - K) % 2 == 0 ? cells + 1 : cells;
      const int lag = kind == 0 ? U / K : 0;
      const int pair = 2 * (K <= 2 ? 4 : K == 4 ? 2 : 1);
      for (int R = 16; R >= pair; R /= 2) {
        const int ring = round_up(lag + (alpha ? 3 : 2) * R, R);
        const size_t lds = (size_t)ring * rs * sizeof(double2);
        if (R * U1 <= kRingLoads * kRingWorkers && lds <= (half ? kRingLds / 2 : kRingLds)) {
          return RingPlan{K, R, ring, rs, lds};
        }
      }
      if (kind != 0) break;  // no lag: more cells per lane save nothing
    }
  return none;
}

template <int K, int KIND, bool ALPHA>
hipError_t launch_ring_t(const RingPlan& p, const float* blank, const float* label,
                         const int* lengths, int B, int T, int U, double* total, float* alpha,
                         int* status, hipStream_t st) {
  static LdsGrant grant;
  if (p.lds > 65536) {
    const hipError_t e = grant((const void*)k_transducer_ring<K, KIND, ALPHA>, p.lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_transducer_ring<K, KIND, ALPHA>), dim3(B), dim3(kRingThreads), p.lds, st, blank,
                     label, lengths, T, U, total, alpha, status, p.R, p.ring, p.rs);
  return hipGetLastError();
}

template <int K, int KIND>
hipError_t launch_ring(const RingPlan& p, const float* blank, const float* label,
                       const int* lengths, int B, int T, int U, double* total, float* alpha,
                       int* status, hipStream_t st) {
  return alpha ? launch_ring_t<K, KIND, true>(p, blank, label, lengths, B, T, U, total, alpha, status, st)
               : launch_ring_t<K, KIND, false>(p, blank, label, lengths, B, T, U, total, alpha, status, st);
}

template <int KIND>
hipError_t launch_kind(const RingPlan& p, const float* blank, const float* label,
                       const int* lengths, int B, int T, int U, double* total, float* alpha,
                       int* status, hipStream_t st) {
  switch (p.K) {
    case 0:
      hipLaunchKernelGGL(k_transducer_logs<KIND>, dim3(B), dim3(kRingThreads), 0, st, blank, label,
                         lengths, T, U, total, alpha, status);
      return hipGetLastError();
    case 1: return launch_ring<1, KIND>(p, blank, label, lengths, B, T, U, total, alpha, status, st);
    case 2: return launch_ring<2, KIND>(p, blank, label, lengths, B, T, U, total, alpha, status, st);
    case 4: return launch_ring<4, KIND>(p, blank, label, lengths, B, T, U, total, alpha, status, st);
    case 8: return launch_ring<8, KIND>(p, blank, label, lengths, B, T, U, total, alpha, status, st);
    default: return launch_ring<16, KIND>(p, blank, label, lengths, B, T, U, total, alpha, status, st);
  }
}

}  // namespace

hipError_t launch_transducer_forward(int kind, const float* blank, const float* label,
                                     const int* lengths, int B, int T, int U, double* total,
                                     float* alpha, int* status, hipStream_t st) {
  if (B == 0) return hipSuccess;
  if (U + 1 > 64 * kTransducerMaxK) return hipErrorInvalidValue;
  const RingPlan p = plan_ring(kind, B, T, U, alpha != nullptr, device_cus());
  if (kind == 0) return launch_kind<0>(p, blank, label, lengths, B, T, U, total, alpha, status, st);
  if (kind == 1) return launch_kind<1>(p, blank, label, lengths, B, T, U, total, alpha, status, st);
  return launch_kind<2>(p, blank, label, lengths, B, T, U, total, alpha, status, st);
}

}  // namespace tbs
