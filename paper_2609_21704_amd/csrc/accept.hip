// LM-head softmax and speculative acceptance or correction (SpecQuant
// SS III-D.4 and the guess-set rule of SS III-A), stochastic (T > 0) and
// greedy (T = 0).
//
// Every vocabulary row is cut into chunks of kChunk logits so that a round's
// b * (2kd + 1) rows spread over the whole chip:
//   1. stats:    per (row, chunk) the max of z = l / T and sum exp(z - max),
//                fp64 (online-softmax partials, merged later in chunk order);
//   2. accept:   per (sequence, chunk) merge the row partials, take the kd
//                accept decisions u * q(x) < p(x) (one thread each), find the
//                first rejection n, and sum the chunk's share of the draw
//                weights R = rint(r * 2^60) in int64 (exact, so the total
//                does not depend on the summation order); the workgroup that
//                finishes a sequence's last chunk draws: it locates the chunk
//                holding t = floor(u Z / 2^24) with a block scan of the chunk
//                totals, then block-scans that chunk.
// A call is a chain of latencies (launch, load, reduce), not of bytes: the
// draw as a kernel of its own cost a third launch per call, and reductions
// through LDS permutes instead of DPP moves most of the time inside a kernel
// (one sequence, 151936 logits, T = 1: a call 15.3 -> 12.1 us).
// Probabilities are computed in fp64 and held in fp32 (prob32), the values
// q_out / p_out hand back; the decisions and the draw weights are formed in
// fp64 from those fp32 values, so that they can be reproduced exactly from
// q_out / p_out.  A -inf logit is a masked token (probability 0).  A row
// holding a NaN or +inf logit, or no finite logit, has no distribution: its
// sequence gets n_accepted = next_token = -1 (and NaN rows in q_out / p_out).
// Greedy reduces every row to the argmax of its chunks, and a second kernel
// merges them and takes the decisions.
//
// Last workgroups are found by counting arrivals.  A workgroup publishes its
// part with an agent-scope store, waits for that store and then adds to the
// counter, so the one that completes the count sees every part; nobody waits
// for another workgroup.  The counters lie in the call's scratch and the
// statistics kernel clears them, so that a call depends on nothing that an
// earlier one left behind.
#include <math.h>

#include <mutex>
#include <type_traits>

#include "sq_device.hpp"
#include "sq_internal.hpp"

#pragma clang fp contract(off)

namespace sq {
namespace {

constexpr int kThreads = 256;
constexpr int kChunk = kAcceptChunk;  // 1024: a 152k-token row spreads over 149 workgroups
constexpr int kPer = kChunk / kThreads;  // logits per thread and chunk

__device__ __forceinline__ double quotient(double a, double b, double rb) {
  const double q = a * rb;
  return __builtin_fma(__builtin_fma(-q, b, a), rb, q);
}

// What the softmax arithmetic of a thread holds in registers.  These kernels
// are bound by fp64 instructions (one per four cycles) where there are many
// rows, so the two expensive operations have forms of their own:
//   z = l / T and p = exp / S: an estimate by the reciprocal plus one
//     exact-remainder correction (Markstein 1990, on the IBM RISC System/6000),
//     the correctly rounded quotient for three operations instead of a dozen; kOne: T == 1, z = l;
//   exp of x <= 0: n = rint(x / ln 2) (Cody and Waite's two-part reduction),
//     then the minimax polynomial of degree 11 on |r| <= ln(2) / 2 (Remez
//     exchange, relative error 3.1e-18, below the rounding of its evaluation)
//     and the scaling by 2^n: 17 operations, without the library's range
//     selections.  Below -1100 (a masked logit's -inf too) it gives 0.
// The coefficients sit in vector registers, so that every step is one
// three-operand fma (72 rows of 151936 logits, statistics: 21.6 -> 13.3 us).
template <bool kOne>
struct Soft {
  static constexpr bool one = kOne;
  double t, rt;
  double c[10], l2e, magic, hi, lo;

  __device__ __forceinline__ explicit Soft(float temp)
      : t((double)temp), rt(kOne ? 1.0 : 1.0 / (double)temp),
        c{0x1.ad66168f6ec16p-26, 0x1.28b31c3ff65e9p-22, 0x1.71df45378dcabp-19, 0x1.a01992c5bfed9p-16,
          0x1.a01a0110431a9p-13, 0x1.6c16c187853cdp-10, 0x1.1111111130e38p-7, 0x1.555555554f35cp-5,
          0x1.55555555554a2p-3, 0x1.0000000000010p-1},
        l2e(0x1.71547652b82fep+0), magic(0x1.8p52), hi(-0x1.62e42fefa2000p-1), lo(-0x1.9ef35793c7673p-41) {
#pragma unroll
    for (int i = 0; i < 10; ++i) asm("" : "+v"(c[i]));
    asm("" : "+v"(l2e), "+v"(magic), "+v"(hi), "+v"(lo));
  }

  __device__ __forceinline__ double exp(double x) const {
    x = fmax(x, -1100.0);
    const double k = __builtin_fma(x, l2e, magic);  // rint(x / ln 2) in the low mantissa bits
    const double n = k - magic;
    const double r = __builtin_fma(n, lo, __builtin_fma(n, hi, x));
    double p = __builtin_fma(c[0], r, c[1]);
#pragma unroll
    for (int i = 2; i < 10; ++i) p = __builtin_fma(p, r, c[i]);
    p = __builtin_fma(p, r, 1.0);
    p = __builtin_fma(p, r, 1.0);
    return ldexp(p, (int)(uint32_t)__builtin_bit_cast(uint64_t, k));
  }

  // A masked logit (-inf) becomes a finite value far below every logit's
  // quotient (a remainder of infinities would be NaN).
  __device__ __forceinline__ double z(float l) const {
    if constexpr (kOne) return (double)l;
    return quotient(fmax((double)l, -1e250), t, rt);
  }
};

__device__ __forceinline__ int64_t grid_weight(double r) { return llrint(r * 0x1p60); }

// A probability exp(z - L) / S in fp64, held in fp32 (rS = 1 / S): the one
// expression behind q_out / p_out, the decisions and the draw weights.  Of a
// row without a distribution (S NaN) it is NaN.
template <class T>
__device__ __forceinline__ float prob32(float l, const T& sf, double L, double S, double rS) {
  return (float)quotient(sf.exp(sf.z(l) - L), S, rS);
}

// ---- wavefront reductions and scans on DPP moves (a permute through LDS costs several times the latency)
template <int Ctrl, int RowMask = 0xF>
__device__ __forceinline__ uint32_t dpp32(uint32_t v) {  // lanes without a source, or outside RowMask: 0
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, Ctrl, RowMask, 0xF, false);
}

template <int Ctrl, int RowMask = 0xF, class T>
__device__ __forceinline__ T dpp_move(T v) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, dpp32<Ctrl, RowMask>(__builtin_bit_cast(uint32_t, v)));
  } else {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = dpp32<Ctrl, RowMask>((uint32_t)u), hi = dpp32<Ctrl, RowMask>((uint32_t)(u >> 32));
    return __builtin_bit_cast(T, (uint64_t)hi << 32 | lo);
  }
}

// op over the 64 lanes, a fixed tree; every lane receives the result.
template <class T, class Op>
__device__ __forceinline__ T wave_all(T v, Op op) {
  v = op(v, dpp_move<0xB1>(v));   // quad_perm [1,0,3,2]
  v = op(v, dpp_move<0x4E>(v));   // quad_perm [2,3,0,1]
  v = op(v, dpp_move<0x141>(v));  // row_half_mirror
  v = op(v, dpp_move<0x140>(v));  // row_mirror: every lane holds its row of 16's result
  constexpr int N = sizeof(T) / 4;
  struct W {
    uint32_t w[N];
  };
  W x = __builtin_bit_cast(W, v), y;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const auto p = __builtin_amdgcn_permlane16_swap(x.w[i], x.w[i], false, false);
    const uint32_t p0 = p[0], p1 = p[1];  // scalar copies: vector element lvalues are misread
    x.w[i] = p0;
    y.w[i] = p1;
  }
  v = op(__builtin_bit_cast(T, x), __builtin_bit_cast(T, y));
  x = __builtin_bit_cast(W, v);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const auto p = __builtin_amdgcn_permlane32_swap(x.w[i], x.w[i], false, false);
    const uint32_t p0 = p[0], p1 = p[1];
    x.w[i] = p0;
    y.w[i] = p1;
  }
  return op(__builtin_bit_cast(T, x), __builtin_bit_cast(T, y));
}

__device__ __forceinline__ float wave_max_f32(float v) {
  return wave_all(v, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ double wave_max_f64(double v) {
  return wave_all(v, [](double a, double b) { return fmax(a, b); });
}
__device__ __forceinline__ double wave_sum_f64(double v) {
  return wave_all(v, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ int64_t wave_sum_i64(int64_t v) {
  return wave_all(v, [](int64_t a, int64_t b) { return a + b; });
}

// Inclusive prefix sum over the 64 lanes.
__device__ __forceinline__ int64_t wave_scan_i64(int64_t v) {
  v += dpp_move<0x111>(v);       // row_shr:1
  v += dpp_move<0x112>(v);       // row_shr:2
  v += dpp_move<0x114>(v);       // row_shr:4
  v += dpp_move<0x118>(v);       // row_shr:8
  v += dpp_move<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
  v += dpp_move<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
  return v;
}

// Exclusive prefix sum of v over the workgroup in thread order; `total`
// receives the workgroup's sum.  Integer, so exact.  sh: one cell per wavefront.
template <int kWaves>
__device__ int64_t block_exclusive_scan_i64(int64_t v, int64_t* sh, int64_t& total) {
  const int w = threadIdx.x >> 6;
  const int64_t x = wave_scan_i64(v);
  if ((threadIdx.x & 63) == 63) sh[w] = x;
  __syncthreads();
  int64_t base = 0, t = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) {
    base += i < w ? sh[i] : 0;
    t += sh[i];
  }
  total = t;
  __syncthreads();
  return base + x - v;
}

template <int kWaves>
__device__ int64_t block_sum_i64(int64_t v, int64_t* sh) {
  v = wave_sum_i64(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  int64_t t = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) t += sh[i];
  __syncthreads();
  return t;
}

// ---- parts published to a last workgroup
__device__ __forceinline__ void publish(int64_t* p, int64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int64_t published(const int64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One thread's arrival, after its parts are published: true for the last of n
// (every part is visible to it).  The parts are written through to the level
// all XCDs share, so the wait for their stores is all the release needs (a
// release fence would also write back the whole L2, measured at about 2 us),
// and they are read from there.
__device__ __forceinline__ bool arrive(int32_t* counter, int n) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  return n == 1 || __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
}

// Row r of the combined row space: target rows first ([b][kd+1] order), then
// draft rows ([kd][b] order); both arrays are contiguous in that order.
__device__ __forceinline__ const float* row_ptr(const float* draft, const float* target, int64_t rows_t, int64_t r,
                                                int v) {
  return r < rows_t ? target + r * v : draft + (r - rows_t) * v;
}

// One wavefront merges a row's chunk partials: L = max over chunks, S = the
// sum of S_c exp(L_c - L), each lane taking every 64th chunk in increasing
// order and the lanes combined in a fixed tree.  A fully masked chunk
// (S_c = 0) adds nothing; a chunk marked invalid (S_c NaN), or a row without
// any mass, gives L = S = NaN.  Every lane returns the values.
//
// The first kCells chunks of each lane are loaded ahead (load_cells: lane l
// chunks l, l + 64, ..., a chunk past the row's end replaced by the row's
// last one and ignored), so that a kernel can issue them beside its other
// independent loads.  Rows of more than 64 kCells chunks take the rest from
// memory (kWide); without kWide the code holds no loop over memory, so that
// the compiler's load counters wait for exactly the loads a value needs.
constexpr int kCells = 4;

__device__ __forceinline__ void load_cells(const double2* st, int nchunk, double2 (&e)[kCells]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < kCells; ++i) e[i] = st[min(lane + 64 * i, nchunk - 1)];
}

template <bool kWide, class T>
__device__ void merge_cells(const T& sf, const double2* st, int nchunk, const double2 (&e)[kCells], double& L,
                            double& S) {
  const int lane = threadIdx.x & 63;
  double mx = -INFINITY;
  int bad = 0;
#pragma unroll
  for (int i = 0; i < kCells; ++i) {
    const bool in = lane + 64 * i < nchunk;
    bad |= in && isnan(e[i].y) ? 1 : 0;
    if (in && e[i].y > 0.0) mx = fmax(mx, e[i].x);
  }
  if constexpr (kWide) {
    for (int c = lane + 64 * kCells; c < nchunk; c += 64) {
      const double2 f = st[c];
      bad |= isnan(f.y) ? 1 : 0;
      if (f.y > 0.0) mx = fmax(mx, f.x);
    }
  }
  mx = wave_max_f64(mx);
  const bool any_bad = __any(bad);
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < kCells; ++i)
    if (lane + 64 * i < nchunk && e[i].y > 0.0) s += e[i].y * sf.exp(e[i].x - mx);
  if constexpr (kWide) {
    for (int c = lane + 64 * kCells; c < nchunk; c += 64) {
      const double2 f = st[c];
      if (f.y > 0.0) s += f.y * sf.exp(f.x - mx);
    }
  }
  s = wave_sum_f64(s);
  if (any_bad || !(s > 0.0)) {
    mx = NAN;
    s = NAN;
  }
  L = mx;
  S = s;
}

template <class T>
__device__ void wave_merge(const T& sf, const double2* st, int nchunk, double& L, double& S) {
  double2 e[kCells];
  load_cells(st, nchunk, e);
  merge_cells<true>(sf, st, nchunk, e, L, S);
}

// 1. per (row, chunk): (max z, sum exp(z - max z)).  blockIdx.x = row * nchunk + chunk.
// One wavefront holds a whole chunk: with four, each with four logits a lane,
// the reductions and barriers were most of the instructions issued.
constexpr int kCPer = kChunk / 64;  // logits per lane where a wavefront holds a chunk

template <int N>
__device__ __forceinline__ void load_row_chunk(const float* __restrict__ l, int c, int v, float (&x)[N]) {
#pragma unroll
  for (int e = 0; e < N; ++e) x[e] = l[min(c * kChunk + e * (kChunk / N) + (int)threadIdx.x, v - 1)];
}

template <bool kOne>
__global__ __launch_bounds__(64) void stats_kernel(const float* __restrict__ draft, const float* __restrict__ target,
                                                   int64_t rows_t, int v, float temp, int nchunk, int nseq,
                                                   double2* __restrict__ stats, int32_t* __restrict__ counters) {
  const int64_t row = blockIdx.x / nchunk;
  const int c = blockIdx.x % nchunk;
  // the arrival counters of nseq sequences, for the accept kernel (there are at least as many rows)
  if (c == 0 && row < nseq && threadIdx.x == 0) counters[row] = 0;
  float x[kCPer];
  load_row_chunk(row_ptr(draft, target, rows_t, row, v), c, v, x);
  const Soft<kOne> sf(temp);
  float m32 = -INFINITY;
  int bad = 0;
#pragma unroll
  for (int e = 0; e < kCPer; ++e) {
    if (c * kChunk + e * 64 + (int)threadIdx.x >= v) x[e] = -INFINITY;
    bad |= (isnan(x[e]) || x[e] == INFINITY) ? 1 : 0;
    m32 = fmaxf(m32, x[e]);
  }
  m32 = wave_max_f32(m32);
  const bool mass = m32 > -INFINITY;  // uniform
  const double mx = mass ? sf.z(m32) : -INFINITY;  // l / T grows with l
  bad = __any(bad);
  double s = 0.0;
  if (mass && !bad) {
#pragma unroll
    for (int e = 0; e < kCPer; ++e) s += sf.exp(sf.z(x[e]) - mx);  // masked and padded cells add exp(-inf) = 0
  }
  s = wave_sum_f64(s);
  // (max, sum); a fully masked chunk is (-inf, 0); an invalid one (NaN, NaN)
  if (threadIdx.x == 0) stats[row * nchunk + c] = bad ? make_double2(NAN, NAN) : make_double2(mx, s);
}

// Optional copies of the distributions: p or q = exp(z - L) / S as fp32.
template <bool kOne>
__global__ __launch_bounds__(64) void probs_kernel(const float* __restrict__ draft, const float* __restrict__ target,
                                                   int64_t rows_t, int v, float temp, int nchunk,
                                                   const double2* __restrict__ stats, float* __restrict__ q_out,
                                                   float* __restrict__ p_out) {
  const int64_t row = blockIdx.x / nchunk;
  const int c = blockIdx.x % nchunk;
  float* out = row < rows_t ? (p_out ? p_out + row * v : nullptr) : (q_out ? q_out + (row - rows_t) * v : nullptr);
  if (!out) return;  // uniform
  float x[kCPer];
  load_row_chunk(row_ptr(draft, target, rows_t, row, v), c, v, x);
  double L, S;  // NaN for a row without a distribution: NaN out
  const Soft<kOne> sf(temp);
  wave_merge(sf, stats + row * nchunk, nchunk, L, S);
  const double rS = 1.0 / S;
#pragma unroll
  for (int e = 0; e < kCPer; ++e) {
    const int j = c * kChunk + e * 64 + (int)threadIdx.x;
    if (j < v) out[j] = prob32(x[e], sf, L, S, rS);
  }
}

// 2. per (sequence, G consecutive chunks): decisions, first rejection, the chunks' shares of the draw weights.
// zs[(s * nchunk + c) * 2 + 0] = sum of R over the chunk for the draw row
// (residual max(0, p_n - q_n) when n < kd, else p_kd); [.. + 1] = sum of R for
// p_n (the fallback when the residual mass is zero).  The last workgroup of a
// sequence draws.  A sequence with a row without a distribution gets -1.
// blockIdx.x = s * groups + group, groups = ceil(nchunk / G).
// Loads that wait for nothing computed here go out together, so that their
// round trips overlap: the draft tokens and their uniforms, the first rows of
// chunk partials, the logits at the tokens, and the first chunk of p_0 and q_0
// (the draw rows when the first draft token is rejected, or when kd = 0).
// Indices are clamped and a value that does not apply is ignored, so that no
// load waits for a condition computed from another.
// kMany: G chunks per workgroup instead of one (groups workgroups per sequence); a form of its own, as the single
// chunk's takes its sequence from an argument that arrives in a register.
template <bool kWide, bool kOne, bool kMany>
__global__ __launch_bounds__(kThreads) void accept_kernel(const float* __restrict__ draft,
                                                          const float* __restrict__ target,
                                                          const int32_t* __restrict__ tokens,
                                                          const uint32_t* __restrict__ u24, int b, int kd, int v,
                                                          float temp, int nchunk, const double2* __restrict__ stats,
                                                          int64_t* __restrict__ zs, int32_t* __restrict__ counters,
                                                          int G, int ngroups,
                                                          int32_t* __restrict__ n_accepted,
                                                          int32_t* __restrict__ next_token) {
  constexpr int kBatch = 3;  // rows of partials a wavefront holds at once
  __shared__ double sL[129], sS[129];
  __shared__ int sAcc[64];
  __shared__ int64_t sh0[4], sz[2][2][4];
  __shared__ int sLast, sChunk;
  __shared__ int64_t sOff;
  const int groups = kMany ? ngroups : nchunk;
  const int s = blockIdx.x / groups;
  const int c0 = (int)(blockIdx.x % groups) * (kMany ? G : 1);  // this workgroup's chunks
  const int c1 = kMany ? min(c0 + G, nchunk) : c0 + 1;
  const int w = threadIdx.x >> 6;
  const int nrows = 2 * kd + 1;
  const int64_t rows_t = (int64_t)b * (kd + 1);
  const float* trow = target + (int64_t)s * (kd + 1) * v;  // p_0 of the sequence
  // row rr of the sequence: target rows 0..kd, then draft rows 0..kd-1
  auto row_of = [&](int rr) -> int64_t {
    return rr <= kd ? (int64_t)s * (kd + 1) + rr : rows_t + (int64_t)(rr - kd - 1) * b + s;
  };
  // thread i < kd: draft position i; the other threads read position 0 (or,
  // with kd = 0, the sequence's uniform) and ignore it
  const bool dlane = (int)threadIdx.x < kd;
  const int di = dlane ? (int)threadIdx.x : 0;
  const int32_t* tp = kd > 0 ? tokens + (int64_t)di * b + s : (const int32_t*)(u24 + (int64_t)s * (kd + 1));
  const int32_t xraw = *tp;
  const uint32_t ut = u24[(int64_t)s * (kd + 1) + di];
  const uint32_t us = u24[(int64_t)s * (kd + 1) + kd];  // the draw's
  // the 2kd + 1 rows' statistics, one wavefront per row, kBatch rows in flight
  double2 e[kBatch][kCells];
  auto load_batch = [&](int r0) {
#pragma unroll
    for (int j = 0; j < kBatch; ++j)
      if (!kMany || r0 + 4 * j < nrows) load_cells(stats + row_of(min(r0 + 4 * j, nrows - 1)) * nchunk, nchunk, e[j]);
  };
  load_batch(w);
  // a chunk of p_0 and q_0 (of p_0 twice when kd = 0), thread t holding
  // logits t, t + 256, ...
  float pv[kPer], qv[kPer];
  const float* q0 = kd > 0 ? draft + (int64_t)s * v : trow;
  auto load_chunk = [&](const float* row, int c, float (&dst)[kPer]) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) dst[k] = row[min(c * kChunk + k * kThreads + (int)threadIdx.x, v - 1)];
  };
  load_chunk(trow, c0, pv);
  load_chunk(q0, c0, qv);
  const bool tok_ok = dlane && xraw >= 0 && xraw < v;
  const int xi = tok_ok ? xraw : 0;
  const float lpt = trow[(int64_t)di * v + xi];
  const float lqt = kd > 0 ? draft[((int64_t)di * b + s) * v + xi] : trow[xi];
  const Soft<kOne> sf(temp);
  auto merge_batch = [&](int r0) {
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int rr = r0 + 4 * j;
      if (rr < nrows) {
        double L, S;
        merge_cells<kWide>(sf, stats + row_of(rr) * nchunk, nchunk, e[j], L, S);
        if ((threadIdx.x & 63) == 0) {
          sL[rr] = L;
          sS[rr] = S;
        }
      }
    }
  };
  merge_batch(w);
  for (int r0 = w + 4 * kBatch; r0 < nrows; r0 += 4 * kBatch) {  // kd >= 6
    load_batch(r0);
    merge_batch(r0);
  }
  __syncthreads();
  // every wavefront reads all rows' sums and agrees on their validity
  int invalid = 0;
  for (int rr = threadIdx.x & 63; rr < nrows; rr += 64) invalid |= isnan(sS[rr]) ? 1 : 0;
  invalid = __any(invalid);
  if (invalid) {  // uniform across the sequence's workgroups
    if (threadIdx.x == 0 && c0 == 0) {
      n_accepted[s] = -1;
      next_token[s] = -1;
    }
    return;
  }
  int n = 0;
  if (kd > 0) {
    if (dlane) {
      const int i = threadIdx.x;
      int acc = 0;
      if (tok_ok) {
        // fp32 probabilities; u (24 bits) times q (24 bits) is exact in fp64
        const float p = prob32(lpt, sf, sL[i], sS[i], 1.0 / sS[i]);
        const float q = prob32(lqt, sf, sL[kd + 1 + i], sS[kd + 1 + i], 1.0 / sS[kd + 1 + i]);
        const double u = ldexp((double)(ut & 0xFFFFFFu), -24);
        acc = (u * (double)q < (double)p) ? 1 : 0;
      }
      sAcc[i] = acc;
    }
    __syncthreads();
    const int i = threadIdx.x & 63;  // kd <= 64: the first rejection, found by every wavefront
    const uint64_t rej = __ballot(i < kd && !sAcc[i]);
    n = rej ? __ffsll((unsigned long long)rej) - 1 : kd;
  }
  const double Lp = sL[n], Sp = sS[n], rSp = 1.0 / Sp;
  const bool resid = n < kd;
  const double Lq = resid ? sL[kd + 1 + n] : 0.0, Sq = resid ? sS[kd + 1 + n] : 1.0, rSq = 1.0 / Sq;
  const float* lp = trow + (int64_t)n * v;  // the draw rows
  const float* lq = resid ? draft + ((int64_t)n * b + s) * v : lp;
  if (n > 0) {  // uniform across the block; n = 0 uses the rows loaded ahead
    load_chunk(lp, c0, pv);
    if (resid) load_chunk(lq, c0, qv);
  }
  for (int c = c0; c < c1; ++c) {
    float pn[kPer] = {}, qn[kPer] = {};  // the next chunk's logits, on their way meanwhile
    if (kMany && c + 1 < c1) {
      load_chunk(lp, c + 1, pn);
      if (resid) load_chunk(lq, c + 1, qn);
    }
    int64_t z0 = 0, z1 = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int j = c * kChunk + k * kThreads + threadIdx.x;
      if (j >= v) break;
      const float p = prob32(pv[k], sf, Lp, Sp, rSp);
      if (resid) {
        const float q = prob32(qv[k], sf, Lq, Sq, rSq);
        const double r = (double)p - (double)q;
        z0 += grid_weight(r > 0.0 ? r : 0.0);
        z1 += grid_weight((double)p);
      } else {
        z0 += grid_weight((double)p);
      }
    }
    z0 = wave_sum_i64(z0);
    if (resid) z1 = wave_sum_i64(z1);
    int64_t(&sw)[2][4] = sz[c & 1];  // (its last reader is two barriers back)
    if ((threadIdx.x & 63) == 0) {
      sw[0][w] = z0;
      sw[1][w] = z1;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      int64_t* zc = zs + ((int64_t)s * nchunk + c) * 2;
      publish(zc, (sw[0][0] + sw[0][1]) + (sw[0][2] + sw[0][3]));
      publish(zc + 1, (sw[1][0] + sw[1][1]) + (sw[1][2] + sw[1][3]));
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      pv[k] = pn[k];
      qv[k] = qn[k];
    }
  }
  if (threadIdx.x == 0) {
    sLast = arrive(counters + s, groups);
    sChunk = -1;
  }
  __syncthreads();
  if (!sLast) return;  // uniform across the block

  // 3. the draw, by the sequence's last workgroup: the chunk holding t is
  // found with a block scan over the chunk totals (256 chunks at a time), then
  // the chunk is scanned with kPer consecutive logits per thread, so that the
  // block's exclusive scan of the thread sums orders them.  All sums are
  // int64, so exact.
  const int64_t* z = zs + (int64_t)s * nchunk * 2;
  int which = 0;
  int64_t Z = 0, pre0 = 0, zc0 = 0;  // thread t: chunk t's prefix and total
  auto totals = [&]() {
    const bool in = (int)threadIdx.x < nchunk;
    const int64_t r = published(z + 2 * min((int)threadIdx.x, nchunk - 1) + which);
    zc0 = in ? r : 0;
    pre0 = block_exclusive_scan_i64<4>(zc0, sh0, Z);
    if (nchunk > kThreads) {
      int64_t part = 0;
      for (int i = threadIdx.x + kThreads; i < nchunk; i += kThreads) part += published(z + 2 * i + which);
      Z += block_sum_i64<4>(part, sh0);
    }
  };
  totals();
  if (Z == 0 && resid) {  // uniform across the block: no residual mass on the grid, back to p_n
    which = 1;
    totals();
  }
  if (Z == 0) {  // no mass on the fixed-point grid
    if (threadIdx.x == 0) {
      n_accepted[s] = n;
      next_token[s] = -1;
    }
    return;
  }
  const uint64_t uu = us & 0xFFFFFFu;
  const uint64_t lo = uu * (uint64_t)Z;
  const uint64_t hi = __umul64hi(uu, (uint64_t)Z);
  const int64_t t = (int64_t)((hi << 40) | (lo >> 24));  // floor(u * Z / 2^24) < Z

  // the chunk i with run(i) <= t < run(i) + z_i
  if (zc0 > 0 && pre0 <= t && t < pre0 + zc0) {
    sChunk = (int)threadIdx.x;
    sOff = t - pre0;
  }
  __syncthreads();
  if (sChunk < 0 && nchunk > kThreads) {  // uniform: in a later batch of 256 chunks
    int64_t run = 0;
    for (int i0 = 0; i0 < nchunk; i0 += kThreads) {
      const int i = i0 + (int)threadIdx.x;
      const int64_t zc = i < nchunk ? published(z + 2 * i + which) : 0;
      int64_t tile;
      const int64_t pre = run + block_exclusive_scan_i64<4>(zc, sh0, tile);
      if (zc > 0 && pre <= t && t < pre + zc) {
        sChunk = i;
        sOff = t - pre;
      }
      __syncthreads();
      if (sChunk >= 0) break;  // uniform across the block
      run += tile;
    }
  }
  const int chunk = sChunk;
  if (chunk < 0) {  // cannot happen (t < Z); kept so that no index can leave the row
    if (threadIdx.x == 0) {
      n_accepted[s] = n;
      next_token[s] = -1;
    }
    return;
  }
  const int64_t off = sOff;
  const bool both = resid && which == 0;
  if (!both) lq = lp;
  int64_t R[kPer];
  int64_t local = 0;
  const int beg = chunk * kChunk + threadIdx.x * kPer;
#pragma unroll
  for (int e2 = 0; e2 < kPer; ++e2) {  // every load of the chunk in flight at once
    const int j = min(beg + e2, v - 1);
    pv[e2] = lp[j];
    qv[e2] = lq[j];
  }
#pragma unroll
  for (int e2 = 0; e2 < kPer; ++e2) {
    int64_t wt = 0;
    if (beg + e2 < v) {
      const float p = prob32(pv[e2], sf, Lp, Sp, rSp);
      if (both) {
        const float q = prob32(qv[e2], sf, Lq, Sq, rSq);
        const double r = (double)p - (double)q;
        wt = grid_weight(r > 0.0 ? r : 0.0);
      } else {
        wt = grid_weight((double)p);
      }
    }
    R[e2] = wt;
    local += wt;
  }
  int64_t tot;
  const int64_t pre = block_exclusive_scan_i64<4>(local, sh0, tot);
  if (local > 0 && pre <= off && off < pre + local) {
    int64_t acc = pre;
    int tok = beg;
#pragma unroll
    for (int e2 = 0; e2 < kPer; ++e2) {
      acc += R[e2];
      if (acc > off) {
        tok = beg + e2;
        break;
      }
    }
    next_token[s] = tok;
    n_accepted[s] = n;
  }
}

// Greedy.  A row's argmax is the largest 64-bit key (ordered logit, inverted
// index): the largest finite logit, its smallest index; 0 when it has no
// finite logit, all ones when it holds a NaN or +inf.  A workgroup takes
// kGreedyChunk logits of a row and stores their key; greedy_kernel merges a
// sequence's rows, a wavefront each, and takes the decisions (four sequences,
// 151936 logits: draws 6.2 us, accept calls of four drafts 6.7; with last
// workgroups found by counting arrivals instead, twice per call, 7.5 and 14.0).
constexpr int kGreedyPer = 16;
constexpr int kGreedyChunk = kThreads * kGreedyPer;
constexpr uint64_t kBadKey = ~0ull;

__device__ __forceinline__ uint64_t logit_key(float x, int j) {
  if (isnan(x) || x == INFINITY) return kBadKey;
  if (x == -INFINITY) return 0;
  const uint32_t u = __float_as_uint(x + 0.0f);  // -0 compares as +0
  const uint32_t o = (u & 0x80000000u) ? ~u : u | 0x80000000u;
  return (uint64_t)o << 32 | (uint32_t)~j;
}

// the index of a row's key, -1: the row has no greedy target
__device__ __forceinline__ int key_index(uint64_t k) { return k == 0 || k == kBadKey ? -1 : (int)~(uint32_t)k; }

__device__ uint64_t block_key_max(uint64_t k, uint64_t* sh) {
  k = wave_all(k, [](uint64_t a, uint64_t b) { return a > b ? a : b; });
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = k;
  __syncthreads();
  const uint64_t a = sh[0] > sh[1] ? sh[0] : sh[1], b = sh[2] > sh[3] ? sh[2] : sh[3];
  __syncthreads();
  return a > b ? a : b;
}

// keys[row][chunk]; blockIdx.x = (row - row0) * nchunk + chunk.  kDraw: one
// chunk and one row per sequence (a draw), whose key is the decision.
template <bool kDraw>
__global__ __launch_bounds__(kThreads) void argmax_kernel(const float* __restrict__ target, int v, int nchunk,
                                                          int64_t row0, int64_t* __restrict__ keys,
                                                          int32_t* __restrict__ n_accepted,
                                                          int32_t* __restrict__ next_token) {
  __shared__ uint64_t sh[4];
  const int64_t row = row0 + blockIdx.x / nchunk;
  const int c = blockIdx.x % nchunk;
  const float* l = target + row * v;
  float x[kGreedyPer];
#pragma unroll
  for (int e = 0; e < kGreedyPer; ++e) {
    const int j = c * kGreedyChunk + e * kThreads + (int)threadIdx.x;
    x[e] = l[min(j, v - 1)];
  }
  uint64_t key = 0;
#pragma unroll
  for (int e = 0; e < kGreedyPer; ++e) {  // a clamped index repeats the last logit: the same key
    const uint64_t k = logit_key(x[e], min(c * kGreedyChunk + e * kThreads + (int)threadIdx.x, v - 1));
    key = k > key ? k : key;
  }
  key = block_key_max(key, sh);
  if (threadIdx.x != 0) return;
  if constexpr (kDraw) {
    const int arg = key_index(key);
    n_accepted[row] = arg < 0 ? -1 : 0;
    next_token[row] = arg;
  } else {
    keys[row * nchunk + c] = (int64_t)key;
  }
}

// A row's key from those of its chunks, by one wavefront (every lane receives it).
__device__ __forceinline__ uint64_t row_key(const int64_t* k, int nchunk) {
  uint64_t key = 0;
  for (int i = threadIdx.x & 63; i < nchunk; i += 64) {
    const uint64_t o = (uint64_t)k[i];
    key = o > key ? o : key;
  }
  return wave_all(key, [](uint64_t a, uint64_t b) { return a > b ? a : b; });
}

// The key of logits j0 .. j1 of a row, by one wavefront.
__device__ __forceinline__ uint64_t part_key(const float* l, int j0, int j1) {
  uint64_t key = 0;
  for (int j = j0 + (threadIdx.x & 63); j < j1; j += 64 * kGreedyPer) {
    float x[kGreedyPer];
#pragma unroll
    for (int e = 0; e < kGreedyPer; ++e) x[e] = l[min(j + 64 * e, j1 - 1)];
#pragma unroll
    for (int e = 0; e < kGreedyPer; ++e) {
      const uint64_t k = logit_key(x[e], min(j + 64 * e, j1 - 1));
      key = k > key ? k : key;
    }
  }
  return wave_all(key, [](uint64_t a, uint64_t b) { return a > b ? a : b; });
}

constexpr int kMergeThreads = 1024;  // 16 wavefronts
constexpr int kGreedyStep = 64 * kGreedyPer;  // logits of a wavefront's loads at once
constexpr int kGreedySteps = 18;              // such loads of all wavefronts, at most

// A sequence's decisions from its rows' keys.  kLogits: from the rows themselves, `split` wavefronts a row (more than
// one where all rows go at once), and no launch before this one; else from the keys of their chunks.  One workgroup's
// steps against a launch (one sequence, both launches / this one): 5 steps 5.9 / 4.2 us, 10 5.9 / 4.7, 18 6.4 / 6.0, 30
// 5.9 / 7.0.
template <bool kLogits>
__global__ __launch_bounds__(kMergeThreads) void greedy_kernel(const int32_t* __restrict__ tokens, int b, int kd,
                                                               const float* __restrict__ target, int v, int split,
                                                               int nchunk, const int64_t* __restrict__ keys,
                                                               int32_t* __restrict__ n_accepted,
                                                               int32_t* __restrict__ next_token) {
  __shared__ uint64_t sKey[65];  // [row][part]: several parts of up to 16 wavefronts, or one of up to 65 rows
  __shared__ int sArg[65];
  const int s = blockIdx.x, i = threadIdx.x;
  const int32_t xt = i < kd ? tokens[(int64_t)i * b + s] : 0;  // (kd <= 64)
  const int parts = kLogits ? split : 1, len = (v + parts - 1) / parts;
  if (!kLogits && nchunk == 1) {
    if (i <= kd) sKey[i] = (uint64_t)keys[(int64_t)s * (kd + 1) + i];
  } else {
    for (int w = i >> 6; w < (kd + 1) * parts; w += blockDim.x >> 6) {
      const int64_t row = (int64_t)s * (kd + 1) + w / parts;
      const int j0 = w % parts * len;
      const uint64_t key =
          kLogits ? part_key(target + row * v, j0, min(j0 + len, v)) : row_key(keys + row * nchunk, nchunk);
      if ((i & 63) == 0) sKey[w] = key;
    }
  }
  __syncthreads();
  if (i <= kd) {
    uint64_t key = sKey[i * parts];
    for (int q = 1; q < parts; ++q) key = max(key, sKey[i * parts + q]);
    sArg[i] = key_index(key);
  }
  __syncthreads();
  if (i >= 64) return;
  // position i's greedy token on lane i (lane 0 also takes position kd)
  const int arg = i < kd ? sArg[i] : 0, last = sArg[kd];
  const bool invalid = __any(arg < 0 || last < 0);
  const uint64_t rej = __ballot(i < kd && xt != arg);  // (arg is in [0, v): so is an accepted token)
  const int n = rej ? __ffsll((unsigned long long)rej) - 1 : kd;
  if (i == 0) {
    n_accepted[s] = invalid ? -1 : n;
    next_token[s] = invalid ? -1 : sArg[n];
  }
}

// ----------------------------------------------------- several draft chains
// Multi-candidate acceptance: each sequence has c draft chains of kd tokens;
// target rows [b][c][kd+1], draft rows [kd][b][c], tokens [kd][b][c],
// uniforms [b][c kd + 1] (u[d c + j] tests chain j at depth d, u[c kd] drives
// the final draw).  The chains' prefix tree is walked with recursive rejection
// sampling on the int64 grid over the fp32 distributions:
//   first candidate at a node:   u q(x) < p(x) in fp64 (exact);
//   its rejection:               R = rint(max(0, p - q) 2^60), Z = sum R;
//   later candidates:            u q(x) Z < R(x), exact in 128-bit integers;
//   their rejection:             R <- max(0, R - floor(q Z)), Z = sum R;
//   Z == 0 after an update:      R = rint(p 2^60) (the node's p);
//   all alive candidates fail:   draw from R; after kd accepted: from p_kd.
// Integer sums do not depend on their order, so the results are those of the
// same rule applied to the fp32 distributions in any order.
//
// The candidates of a node (the chains sharing its prefix, in order) do not
// depend on what is accepted elsewhere, so all nodes and vocabulary chunks are
// worked on at once: multi_rows_kernel gives every row's merged statistics,
// p's masses, the masses after a first rejection and the first candidates'
// tests; launch i = 1 .. c - 1 of multi_step_kernel the test of every node's
// candidate i and, if that fails, the residual mass Z after it, which needs
// only the masses before it.  A node that has accepted a candidate needs no
// more: its workgroups leave at once.  R itself, and p and q unless they are
// asked for, are recomputed from the logits where they are needed, not stored.
// One workgroup per sequence (multi_walk_kernel) then walks the tree and draws.
// A launch costs 2.5 us also where nothing is left to do, so that small
// vocabularies take fewer of them, and the walk itself the candidates after
// (walk_steps()).  Up to c + 2 launches over the whole chip replace a walk of
// up to c kd passes over the vocabulary by one workgroup per sequence (two
// sequences, four chains of four, 151936 logits, the whole call: 306 -> 66 us).
constexpr int kMThreads = 1024;
constexpr int kMWaves = kMThreads / 64;
constexpr int kStepBlocks = 8192;  // workgroups of one step launch, about
constexpr int kWalkLogits = 32768;  // rows whose later candidates the walk may take

// q = m 2^e exactly (m < 2^24), from the bits of a finite q >= 0.
__device__ __forceinline__ void split_f32(float q, uint64_t& m, int& e) {
  const uint32_t bits = __float_as_uint(q);
  const uint32_t ex = (bits >> 23) & 0xFFu, man = bits & 0x7FFFFFu;
  if (ex == 0) {
    m = man;
    e = -149;
  } else {
    m = man | 0x800000u;
    e = (int)ex - 150;
  }
}

// floor(q Z), q in [0, 1], 0 <= Z < 2^62, exactly.
__device__ __forceinline__ int64_t floor_qz(float q, int64_t z) {
  uint64_t m;
  int e;
  split_f32(q, m, e);
  if (m == 0 || z == 0) return 0;
  const uint64_t lo = m * (uint64_t)z, hi = __umul64hi(m, (uint64_t)z);
  const int sh = -e;  // >= 23 for q <= 1
  if (sh >= 128) return 0;
  if (sh >= 64) return (int64_t)(hi >> (sh - 64));
  return (int64_t)((hi << (64 - sh)) | (lo >> sh));
}

// u24 / 2^24 q Z < R, exactly.
__device__ __forceinline__ bool test_grid(uint32_t u24, float q, int64_t z, int64_t r) {
  if (r <= 0) return false;
  uint64_t m;
  int e;
  split_f32(q, m, e);
  const uint64_t a = (uint64_t)(u24 & 0xFFFFFFu) * m;  // < 2^48
  const uint64_t llo = a * (uint64_t)z, lhi = __umul64hi(a, (uint64_t)z);
  const int sh = 24 - e;  // >= 47 for q <= 1
  const int bits = 64 - __clzll((unsigned long long)r);
  if (bits + sh >= 127) return true;  // r 2^sh >= 2^126 > lhs
  uint64_t rhi, rlo;
  if (sh >= 64) {
    rhi = (uint64_t)r << (sh - 64);
    rlo = 0;
  } else {
    rhi = (uint64_t)r >> (64 - sh);
    rlo = (uint64_t)r << sh;
  }
  return lhi < rhi || (lhi == rhi && llo < rlo);
}

// A row's logits and its merged statistics: prob() is prob32 of one of them.
struct Row {
  const float* l;
  double L, S, rS;
};

__device__ __forceinline__ Row row_at(const float* l, double2 ls) { return Row{l, ls.x, ls.y, 1.0 / ls.y}; }

template <class T>
__device__ __forceinline__ float prob(const Row& r, const T& sf, int y) {
  return prob32(r.l[y], sf, r.L, r.S, r.rS);
}

// Every call's rows and tables: ls [rows] merged statistics (target rows
// first), zp [rows_t][nchunk] masses of p, zs [b][kd][c][nchunk] residual
// masses after chain j's rejection, acc [b][kd][c] chain j's test.  An entry of
// zs or acc means something only where the node's candidates before it (and
// for zs chain j itself) have failed; of the others nothing is read into a result.
struct MultiArgs {
  const float* draft;
  const float* target;
  const int32_t* tokens;
  const uint32_t* u24;
  int b, c, kd, v, nchunk;
  float temp;
  double2* ls;
  int64_t* zp;
  int64_t* zs;
  int32_t* acc;
  int64_t* r;  // [b][v] R and q, where the walk takes candidates itself
  float* q;
};

// A node: the chains of sequence s that share chain j's first d tokens, and
// its target and draft rows: those of the lowest of them (their common context
// gives all of them the same).
struct Node {
  uint64_t alive;
  int64_t trow;  // the target row
  Row p, q;
};

__device__ __forceinline__ Node node_at(const MultiArgs& a, uint64_t alive, int s, int d) {
  const int j0 = __ffsll((unsigned long long)alive) - 1;
  Node n;
  n.alive = alive;
  n.trow = ((int64_t)s * a.c + j0) * (a.kd + 1) + d;
  n.p = row_at(a.target + n.trow * a.v, a.ls[n.trow]);
  if (d < a.kd) {
    const int64_t r = ((int64_t)d * a.b + s) * a.c + j0;
    n.q = row_at(a.draft + r * a.v, a.ls[(int64_t)a.b * a.c * (a.kd + 1) + r]);
  } else {
    n.q = n.p;
  }
  return n;
}

// The residual weight of p, q after the rejections of the node's candidates
// before chain `stop` (64: of all of them).  zt(j): the mass after chain j's
// rejection as summed (0: the node falls back to p, whose mass zp() gives).
// zcur receives the mass of the returned weights.
template <class ZT, class ZP>
__device__ __forceinline__ int64_t residual_at(uint64_t alive, float p, float q, int stop, ZT zt, ZP zp,
                                               int64_t& zcur) {
  int64_t w = 0, z = 0;
  bool first = true;
  for (uint64_t rest = alive; rest; rest &= rest - 1) {
    const int j = __ffsll((unsigned long long)rest) - 1;
    if (j >= stop) break;
    if (first) {
      const double r = (double)p - (double)q;
      w = grid_weight(r > 0.0 ? r : 0.0);
    } else {
      const int64_t w0 = w - floor_qz(q, z);
      w = w0 > 0 ? w0 : 0;
    }
    first = false;
    z = zt(j);
    if (z == 0) {
      w = grid_weight((double)p);
      z = zp();
    }
  }
  zcur = z;
  return w;
}

// Sum of a row of n chunk values by one wavefront (every lane receives it).
__device__ __forceinline__ int64_t wave_row_sum(const int64_t* r, int n) {
  int64_t t = 0;
  for (int i = threadIdx.x & 63; i < n; i += 64) t += r[i];
  return wave_sum_i64(t);
}

// Per (target row, chunk), by W wavefronts: the row's and its draft row's merged
// statistics (by chunk 0), the chunk's mass of p and, for the rows with a
// draft, of max(0, p - q): the mass after chain j's rejection if it is its
// node's first candidate, whose test the lane that holds its token takes.
// Copies of the distributions where asked for.
template <bool kOne, int W>
__global__ __launch_bounds__(64 * W) void multi_rows_kernel(MultiArgs a, const double2* __restrict__ stats,
                                                        float* __restrict__ q_out, float* __restrict__ p_out) {
  constexpr int N = kChunk / (64 * W);  // logits per thread
  __shared__ int64_t sh[W];
  const int64_t row = blockIdx.x / a.nchunk;  // (s c + j) (kd + 1) + d
  const int ch = blockIdx.x % a.nchunk;
  const int d = (int)(row % (a.kd + 1));
  const int64_t sj = row / (a.kd + 1), rows_t = (int64_t)a.b * a.c * (a.kd + 1);
  const bool drafted = d < a.kd;
  const int64_t drow = drafted ? (int64_t)d * a.b * a.c + sj : 0;
  float xp[N], xq[N];
  load_row_chunk(a.target + row * a.v, ch, a.v, xp);
  if (drafted) load_row_chunk(a.draft + drow * a.v, ch, a.v, xq);
  double Lp, Sp, Lq = 0.0, Sq = 1.0;
  const Soft<kOne> sf(a.temp);
  wave_merge(sf, stats + row * a.nchunk, a.nchunk, Lp, Sp);
  if (drafted) wave_merge(sf, stats + (rows_t + drow) * a.nchunk, a.nchunk, Lq, Sq);
  if (ch == 0 && threadIdx.x == 0) {
    a.ls[row] = make_double2(Lp, Sp);
    if (drafted) a.ls[rows_t + drow] = make_double2(Lq, Sq);
  }
  const double rSp = 1.0 / Sp, rSq = 1.0 / Sq;
  const int64_t s = sj / a.c, j = sj - s * a.c, cell = (s * a.kd + d) * a.c + j;
  int x = -1;
  double u = 0.0;
  if (drafted) {
    x = a.tokens[drow];
    u = ldexp((double)(a.u24[s * (a.c * a.kd + 1) + d * a.c + j] & 0xFFFFFFu), -24);
    if (ch == 0 && threadIdx.x == 0 && (x < 0 || x >= a.v)) a.acc[cell] = 0;  // no row's token: fails
  }
  int64_t zp = 0, zr = 0;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    const int y = ch * kChunk + e * (64 * W) + (int)threadIdx.x;
    if (y < a.v) {
      const float p = prob32(xp[e], sf, Lp, Sp, rSp);
      zp += grid_weight((double)p);
      if (p_out) p_out[row * a.v + y] = p;
      if (drafted) {
        const float q = prob32(xq[e], sf, Lq, Sq, rSq);
        const double r = (double)p - (double)q;
        zr += grid_weight(r > 0.0 ? r : 0.0);
        if (y == x) a.acc[cell] = u * (double)q < (double)p;
        if (q_out) q_out[drow * a.v + y] = q;
      }
    }
  }
  zp = W > 1 ? block_sum_i64<W>(zp, sh) : wave_sum_i64(zp);
  zr = W > 1 ? block_sum_i64<W>(zr, sh) : wave_sum_i64(zr);
  if (threadIdx.x == 0) {
    a.zp[row * a.nchunk + ch] = zp;
    if (drafted) a.zs[cell * a.nchunk + ch] = zr;
  }
}

// The chains that share chain j's first d tokens (c <= 64), on every lane.
__device__ __forceinline__ uint64_t sharing(const MultiArgs& a, int s, int d, int j) {
  const int lane = threadIdx.x & 63;
  bool same = lane < a.c;
#pragma unroll 4
  for (int i = 0; i < d; ++i) {
    const int32_t* tk = a.tokens + ((int64_t)i * a.b + s) * a.c;
    same &= tk[lane < a.c ? lane : 0] == tk[j];
  }
  return __ballot(same);
}

// Step `step` = 1, 2, ..: for every (sequence, depth, chain) whose chain is its
// node's candidate number `step` (from 0), and no candidate before it was
// accepted, its test and, if that fails, zs[..][chunk] = the chunk's residual
// mass after its rejection.  blockIdx.x = ((s kd + d) (c - step) + j - step)
// slices + slice (at most j candidates come before chain j); a workgroup takes
// the chunks slice, slice + slices, ...; every one of them takes the test.
template <bool kOne>
__global__ __launch_bounds__(kThreads) void multi_step_kernel(MultiArgs a, int slices, int step) {
  __shared__ int64_t sh[4];
  __shared__ int64_t sz[64];
  __shared__ int64_t szp;
  const int slice = blockIdx.x % slices, nj = a.c - step;
  const int sdj = blockIdx.x / slices, sd = sdj / nj;
  const int j = step + sdj - sd * nj, s = sd / a.kd, d = sd - s * a.kd;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t row = (int64_t)sd * a.c;
  const int done = a.acc[row + min(lane, a.c - 1)];
  const uint64_t alive = sharing(a, s, d, j), before = alive & ((1ull << j) - 1ull);
  if (__popcll(before) != step || (__ballot(done) & before)) return;  // uniform across the block
  const Node nd = node_at(a, alive, s, d);
  int64_t* zrow = a.zs + (row + j) * a.nchunk;
  // this workgroup's first logits and the token's, and the masses of the candidates before it, a wavefront each
  float xp[kPer], xq[kPer];
  auto load = [&](int ch) {
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const int y = min(ch * kChunk + e * kThreads + (int)threadIdx.x, a.v - 1);
      xp[e] = nd.p.l[y];
      xq[e] = nd.q.l[y];
    }
  };
  load(slice);
  const int32_t x = a.tokens[((int64_t)d * a.b + s) * a.c + j];
  const uint32_t u = a.u24[(int64_t)s * (a.c * a.kd + 1) + d * a.c + j];
  const bool in = x >= 0 && x < a.v;
  const float lpx = nd.p.l[in ? x : 0], lqx = nd.q.l[in ? x : 0];
  int r = 0;
  for (uint64_t rest = before; rest; rest &= rest - 1) {
    const int i = __ffsll((unsigned long long)rest) - 1;
    if ((r++ & 3) != w) continue;
    const int64_t t = wave_row_sum(zrow + (int64_t)(i - j) * a.nchunk, a.nchunk);
    if (lane == 0) sz[i] = t;
  }
  if (w == 3) {
    const int64_t t = wave_row_sum(a.zp + nd.trow * a.nchunk, a.nchunk);
    if (lane == 0) szp = t;
  }
  const Soft<kOne> sf(a.temp);
  __syncthreads();
  auto residual = [&](float p, float q, int64_t& zc) {
    return residual_at(before, p, q, 64, [&](int i) { return sz[i]; }, [&]() { return szp; }, zc);
  };
  {
    const float p = prob32(lpx, sf, nd.p.L, nd.p.S, nd.p.rS), q = prob32(lqx, sf, nd.q.L, nd.q.S, nd.q.rS);
    int64_t zc;
    const int64_t w1 = residual(p, q, zc);
    const bool acc = in && test_grid(u, q, zc, w1);  // the same on every thread of every workgroup
    if (slice == 0 && threadIdx.x == 0) a.acc[row + j] = acc;
    if (acc) return;
  }
  for (int ch = slice; ch < a.nchunk; ch += slices) {
    if (ch != slice) load(ch);
    int64_t z = 0;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      if (ch * kChunk + e * kThreads + (int)threadIdx.x >= a.v) break;
      const float p = prob32(xp[e], sf, nd.p.L, nd.p.S, nd.p.rS), q = prob32(xq[e], sf, nd.q.L, nd.q.S, nd.q.rS);
      int64_t zc;
      const int64_t w1 = residual(p, q, zc);
      const int64_t w0 = w1 - floor_qz(q, zc);
      z += w0 > 0 ? w0 : 0;
    }
    z = block_sum_i64<4>(z, sh);
    if (threadIdx.x == 0) zrow[ch] = z;
  }
}

// One workgroup per sequence: the walk and the draw.  At a node it reaches, the
// candidates up to number `steps` have their tests from the launches before;
// the others, when all of those fail, it takes here, one pass over the row each
// (R and q [v] of the sequence, logit y always on thread y % kMThreads), as
// multi_step_kernel would.  LDS: tokens [kd c], test results [kd c].
template <bool kOne>
__global__ __launch_bounds__(kMThreads) void multi_walk_kernel(MultiArgs a, int steps, int32_t* __restrict__ n_accepted,
                                                               int32_t* __restrict__ next_token,
                                                               int32_t* __restrict__ chain) {
  extern __shared__ __align__(16) char msmem[];
  __shared__ int64_t sh[kMWaves];
  __shared__ int64_t sz[64];  // a node's masses
  __shared__ int64_t sc[kWalkLogits / kChunk][kMWaves];
  __shared__ int sChunk, sTok;
  __shared__ int64_t sOff, szp, sR;
  __shared__ float sQ;
  const int c = a.c, kd = a.kd, v = a.v, nchunk = a.nchunk, np = kd * c;
  int32_t* stok = reinterpret_cast<int32_t*>(msmem);
  int32_t* sacc = stok + np;
  const int s = blockIdx.x, t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t rows_t = (int64_t)a.b * c * (kd + 1);
  // every row of the sequence must have a distribution
  int bad = 0;
  for (int rr = t; rr < c * (2 * kd + 1); rr += kMThreads) {
    const int k2 = rr - c * (kd + 1);  // draft row d * c + j
    bad |= isnan(a.ls[k2 < 0 ? (int64_t)s * c * (kd + 1) + rr : rows_t + ((int64_t)(k2 / c) * a.b + s) * c + k2 % c].y);
  }
  for (int i = t; i < np; i += kMThreads) {
    stok[i] = a.tokens[((int64_t)(i / c) * a.b + s) * c + i % c];
    sacc[i] = a.acc[(int64_t)s * np + i];
  }
  const uint32_t* u = a.u24 + (int64_t)s * (np + 1);
  const uint32_t ud = u[np];  // the draw's
  if (t == 0) sChunk = sTok = -1;
  if (__syncthreads_or(bad)) {
    if (t == 0) n_accepted[s] = next_token[s] = chain[s] = -1;
    return;
  }
  const Soft<kOne> sf(a.temp);
  int64_t* R = a.r + (int64_t)s * v;
  float* Q = a.q + (int64_t)s * v;
  // the masses after the rejections of a node's candidates (`which` of them), and of p, a wavefront each
  auto masses = [&](const Node& nd, int d, uint64_t which) {
    for (int j = w; j < c; j += kMWaves) {
      if (!((which >> j) & 1ull)) continue;
      const int64_t z = wave_row_sum(a.zs + ((int64_t)s * np + d * c + j) * nchunk, nchunk);
      if (lane == 0) sz[j] = z;
    }
    if (w == kMWaves - 1) {
      const int64_t z = wave_row_sum(a.zp + nd.trow * nchunk, nchunk);
      if (lane == 0) szp = z;
    }
    __syncthreads();
  };
  auto residual = [&](uint64_t which, float p, float q, int64_t& zc) {
    return residual_at(which, p, q, 64, [&](int o) { return sz[o]; }, [&]() { return szp; }, zc);
  };
  // every wavefront walks, chain `lane` on its lane: all values are uniform across the block
  uint64_t alive = c == 64 ? ~0ull : ((1ull << c) - 1ull);
  int n = kd;
  int64_t z = 0;  // of R, once a node's candidates past `steps` have been taken here
  bool late = false;
  for (int d = 0; d < kd; ++d) {
    const bool on = lane < c && ((alive >> lane) & 1ull);
    const bool known = __popcll(alive & ((1ull << lane) - 1ull)) <= steps;
    const int cell = d * c + min(lane, c - 1);
    const uint64_t acc = __ballot(on && known && sacc[cell]);
    int32_t x = -1;
    bool accepted = acc != 0;
    if (accepted) {
      x = stok[d * c + __ffsll((unsigned long long)acc) - 1];  // the lowest accepted one
    } else if (uint64_t rest = __ballot(on && !known)) {
      const Node nd = node_at(a, alive, s, d);
      const uint64_t before = alive & ~rest;
      masses(nd, d, before);
      for (int y = t; y < v; y += kMThreads) {
        const float q = prob(nd.q, sf, y);
        Q[y] = q;
        R[y] = residual(before, prob(nd.p, sf, y), q, z);
      }
      (void)residual(before, 0.f, 0.f, z);  // (the mass, on threads without a logit too)
      for (; rest; rest &= rest - 1) {
        const int j = __ffsll((unsigned long long)rest) - 1;
        x = stok[d * c + j];
        if (x >= 0 && x < v) {
          if (t == x % kMThreads) {
            sR = R[x];
            sQ = Q[x];
          }
          __syncthreads();
          accepted = test_grid(u[d * c + j], sQ, z, sR);
          if (accepted) break;
        }
        const int64_t z0 = z;
        z = 0;
#pragma unroll 4
        for (int y = t; y < v; y += kMThreads) {
          const int64_t w0 = R[y] - floor_qz(Q[y], z0), w1 = w0 > 0 ? w0 : 0;
          R[y] = w1;
          z += w1;
        }
        z = block_sum_i64<kMWaves>(z, sh);  // (its barriers also keep the next sR from this one's readers)
        if (z == 0) {  // no residual mass on the grid: back to p
          for (int y = t; y < v; y += kMThreads) R[y] = grid_weight((double)prob(nd.p, sf, y));
          z = szp;
        }
      }
      late = !accepted;
    }
    if (!accepted) {
      n = d;
      break;
    }
    alive &= __ballot(lane < c && stok[cell] == x);
    __syncthreads();  // (sz, sR)
  }
  const int jf = __ffsll((unsigned long long)alive) - 1;
  const Node nd = node_at(a, alive, s, n);
  const int jl = 63 - __clzll((unsigned long long)alive);  // the node's last candidate
  bool plain = false;
  const int64_t* zc = nullptr;
  if (late) {  // the draw's chunk masses, from R
    for (int ch = 0; ch < nchunk; ++ch) {
      const int y = ch * kChunk + t;  // kChunk == kMThreads
      const int64_t m = wave_sum_i64(y < v ? R[y] : 0);
      if (lane == 0) sc[ch][w] = m;
    }
    __syncthreads();
  } else {
    // the residual's after all rejections, else p's (all accepted, or no residual mass left)
    masses(nd, n, n < kd ? alive : 0);
    plain = n == kd || sz[jl] == 0;
    zc = plain ? a.zp + nd.trow * nchunk : a.zs + ((int64_t)s * np + n * c + jl) * nchunk;
    z = plain ? szp : sz[jl];
  }
  if (z > 0) {  // uniform across the block
    const uint64_t uu = ud & 0xFFFFFFu;
    const int64_t tt = (int64_t)((__umul64hi(uu, (uint64_t)z) << 40) | ((uu * (uint64_t)z) >> 24));
    int64_t run = 0;
    for (int i0 = 0; i0 < nchunk; i0 += kMThreads) {
      const int i = i0 + t;
      int64_t m = 0;
      if (late) {
        for (int k = 0; i < nchunk && k < kMWaves; ++k) m += sc[i][k];
      } else if (i < nchunk) {
        m = zc[i];
      }
      int64_t tile;
      const int64_t pre = run + block_exclusive_scan_i64<kMWaves>(m, sh, tile);
      if (m > 0 && pre <= tt && tt < pre + m) {
        sChunk = i;
        sOff = tt - pre;
      }
      __syncthreads();
      if (sChunk >= 0) break;  // uniform across the block
      run += tile;
    }
    const int ch = sChunk;
    if (ch >= 0) {  // always (tt < z)
      const int y = ch * kChunk + t;
      int64_t r = 0, zi;
      if (y < v) {
        if (late) {
          r = R[y];
        } else {
          const float p = prob(nd.p, sf, y);
          r = plain ? grid_weight((double)p) : residual(alive, p, prob(nd.q, sf, y), zi);
        }
      }
      int64_t tile;
      const int64_t pre = block_exclusive_scan_i64<kMWaves>(r, sh, tile);
      if (r > 0 && pre <= sOff && sOff < pre + r) sTok = y;
    }
  }
  __syncthreads();
  if (t == 0) {
    n_accepted[s] = n;
    next_token[s] = sTok;
    chain[s] = jf;
  }
}
static_assert(kChunk == kMThreads && kChunk % kThreads == 0, "the walk draws from a chunk, one logit per thread");

// Greedy (T = 0) over several chains: per sequence, the argmax of the lowest
// alive chain's row at each depth is accepted when an alive chain drafted it.
__global__ __launch_bounds__(kMergeThreads) void multi_greedy_kernel(const int32_t* __restrict__ tokens, int b, int c,
                                                                     int kd, int nchunk,
                                                                     const int64_t* __restrict__ keys,
                                                                     int32_t* __restrict__ n_accepted,
                                                                     int32_t* __restrict__ next_token,
                                                                     int32_t* __restrict__ chain) {
  __shared__ int sArg[64 * 65];
  const int s = blockIdx.x;
  const int rows = c * (kd + 1);
  int bad = 0;
  for (int r = threadIdx.x >> 6; r < rows; r += kMergeThreads / 64) {
    const int a = key_index(row_key(keys + ((int64_t)s * rows + r) * nchunk, nchunk));
    if ((threadIdx.x & 63) == 0) sArg[r] = a;
    bad |= a < 0 ? 1 : 0;
  }
  if (__syncthreads_or(bad)) {
    if (threadIdx.x == 0) n_accepted[s] = next_token[s] = chain[s] = -1;
    return;
  }
  if (threadIdx.x >= 64) return;
  const int lane = threadIdx.x;
  uint64_t alive = c == 64 ? ~0ull : ((1ull << c) - 1ull);
  int n = kd, tok = -1;
  for (int d = 0; d <= kd; ++d) {
    const int j0 = __ffsll((unsigned long long)alive) - 1;
    const int g = sArg[j0 * (kd + 1) + d];
    if (d == kd) {
      tok = g;
      break;
    }
    const uint64_t keep = alive & __ballot(lane < c && tokens[((int64_t)d * b + s) * c + min(lane, c - 1)] == g);
    if (!keep) {
      n = d;
      tok = g;
      break;
    }
    alive = keep;
  }
  if (lane == 0) {
    n_accepted[s] = n;
    next_token[s] = tok;
    chain[s] = __ffsll((unsigned long long)alive) - 1;
  }
}

}  // namespace

namespace {

// Scratch of one call: the greedy keys (one per chunk), or the row statistics,
// the chunk weights (each part 256-byte aligned) and the arrival counters.  The
// counters have kSeqBytes per sequence, of which they use four: what a call
// needs, and so which calls the allocation-free form takes, stays as it was.
constexpr size_t kSeqBytes = 40;

// Workgroups of the accept kernel, about; more than one chunk each beyond that:
// every workgroup merges its sequence's row statistics again, and its arrival
// holds it for about 3 us (draws at 151936 logits, one chunk each / 512 / 1024
// workgroups: 4 sequences 16.9 / 14.4 / 16.9 us, 16 38.6 / 20.9 / 23.0, 64 113 / 45.3 / 38.4).
constexpr int64_t kAcceptBlocks = 512;
struct AcceptScratch {
  size_t st_bytes, zs_bytes, cnt_bytes;
  size_t total() const { return st_bytes + zs_bytes + cnt_bytes; }
};

size_t pad256(size_t n) { return (n + 255) / 256 * 256; }

AcceptScratch accept_scratch(int b, int kd, int v, float temperature) {
  const int64_t nchunk = (v + kChunk - 1) / kChunk;
  const int64_t rows_t = (int64_t)b * (kd + 1);
  AcceptScratch a;
  if (temperature == 0.0f) {
    a.st_bytes = pad256((size_t)rows_t * nchunk * sizeof(int64_t));
    a.zs_bytes = a.cnt_bytes = 0;
    return a;
  }
  const int64_t rows = rows_t + (int64_t)b * kd;
  a.st_bytes = pad256((size_t)rows * nchunk * sizeof(double2));
  a.zs_bytes = pad256((size_t)b * nchunk * 2 * sizeof(int64_t));
  a.cnt_bytes = (size_t)b * kSeqBytes;
  return a;
}

// The keys of every row's chunks of kGreedyChunk logits into keys [rows][chunks].
hipError_t enqueue_argmax(const float* target, int v, int64_t rows, int64_t* keys, hipStream_t stream) {
  const int nchunk = (v + kGreedyChunk - 1) / kGreedyChunk;
  const int64_t per = (int64_t(1) << 23) / nchunk;  // rows per launch (a grid holds fewer than 2^32 threads)
  for (int64_t r0 = 0; r0 < rows; r0 += per) {
    const int64_t nr = rows - r0 < per ? rows - r0 : per;
    hipLaunchKernelGGL(argmax_kernel<false>, dim3((unsigned)(nr * nchunk)), dim3(kThreads), 0, stream, target, v, nchunk,
                       r0, keys, nullptr, nullptr);
  }
  return hipGetLastError();
}

// The accept kernels on the scratch `ws` (at least accept_scratch().total() bytes).
hipError_t enqueue_accept(const float* draft, const float* target, const int32_t* tokens, const uint32_t* u24, int b,
                          int kd, int v, float temperature, int32_t* n_accepted, int32_t* next_token, float* q_out,
                          float* p_out, char* ws, hipStream_t stream) {
  const int nchunk = (v + kChunk - 1) / kChunk;
  const int64_t rows_t = (int64_t)b * (kd + 1);
  const AcceptScratch a = accept_scratch(b, kd, v, temperature);
  if (temperature == 0.0f) {
    if (kd == 0 && v <= kGreedyChunk) {
      hipLaunchKernelGGL(argmax_kernel<true>, dim3((unsigned)b), dim3(kThreads), 0, stream, target, v, 1, 0, nullptr,
                         n_accepted, next_token);
      return hipGetLastError();
    }
    int64_t* keys = reinterpret_cast<int64_t*>(ws);
    // wavefronts a row and steps of a wavefront, where the rows are read by the deciding kernel
    int split = kd < 15 ? 16 / (kd + 1) : 1;
    const int all = (v + kGreedyStep - 1) / kGreedyStep;
    split = split < all ? split : all;
    const int steps = ((v + split - 1) / split + kGreedyStep - 1) / kGreedyStep;
    const bool direct = v <= kGreedyChunk && (kd + 1) * split * steps <= kGreedySteps;
    const int waves = direct ? (kd + 1) * split : kd + 1;
    auto decide = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)b), dim3(64 * (waves < 16 ? waves : 16)), 0, stream, tokens, b, kd,
                         target, v, split, (v + kGreedyChunk - 1) / kGreedyChunk, keys, n_accepted, next_token);
      return hipGetLastError();
    };
    if (direct) return decide(greedy_kernel<true>);
    const hipError_t e = enqueue_argmax(target, v, rows_t, keys, stream);
    return e != hipSuccess ? e : decide(greedy_kernel<false>);
  }
  const int64_t rows = rows_t + (int64_t)b * kd;
  double2* stats = reinterpret_cast<double2*>(ws);
  int64_t* zs = reinterpret_cast<int64_t*>(ws + a.st_bytes);
  int32_t* counters = reinterpret_cast<int32_t*>(ws + a.st_bytes + a.zs_bytes);
  // chunks per workgroup of the accept kernel
  const int64_t G = ((int64_t)b * nchunk + kAcceptBlocks - 1) / kAcceptBlocks;
  const int64_t groups = (nchunk + G - 1) / G;
  auto go = [&](auto one_tag) {
    constexpr bool One = decltype(one_tag)::value;
    hipLaunchKernelGGL(stats_kernel<One>, dim3((unsigned)(rows * nchunk)), dim3(64), 0, stream, draft, target, rows_t,
                       v, temperature, nchunk, b, stats, counters);
    if (p_out || q_out)
      hipLaunchKernelGGL(probs_kernel<One>, dim3((unsigned)(rows * nchunk)), dim3(64), 0, stream, draft, target,
                         rows_t, v, temperature, nchunk, stats, q_out, p_out);
    auto accept = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)(b * groups)), dim3(kThreads), 0, stream, draft, target, tokens, u24, b,
                         kd, v, temperature, nchunk, stats, zs, counters, (int)G, (int)groups, n_accepted, next_token);
    };
    if (nchunk > 64 * kCells)
      G > 1 ? accept(accept_kernel<true, One, true>) : accept(accept_kernel<true, One, false>);
    else
      G > 1 ? accept(accept_kernel<false, One, true>) : accept(accept_kernel<false, One, false>);
  };
  if (temperature == 1.0f)
    go(std::true_type{});
  else
    go(std::false_type{});
  return hipGetLastError();
}

// The scratch of the allocation-free entry point: one static array per GPU,
// held until the process ends.  Host code never passes `scratch` itself to a
// kernel (on the host it names a stand-in, not device memory): it uses the
// device address taken once per device with hipGetSymbolAddress.
static __device__ __align__(256) char scratch[kNoAllocScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_addr[kMaxDevices];

hipError_t noalloc_scratch(char** out) {
  *out = nullptr;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_addr[dev]) {  // first call on this device, which is current
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      (void)hipGetLastError();
      return e != hipSuccess ? e : hipErrorInvalidSymbol;
    }
    g_scratch_addr[dev] = p;
  }
  *out = static_cast<char*>(g_scratch_addr[dev]);
  return hipSuccess;
}

}  // namespace

size_t spec_accept_scratch_bytes(int b, int kd, int v, float temperature) {
  return accept_scratch(b, kd, v, temperature).total();
}

hipError_t launch_spec_accept(const float* draft, const float* target, const int32_t* tokens, const uint32_t* u24,
                              int b, int kd, int v, float temperature, int32_t* n_accepted, int32_t* next_token,
                              float* q_out, float* p_out, hipStream_t stream) {
  void* ws = nullptr;
  const hipError_t e = workspace(accept_scratch(b, kd, v, temperature).total(), stream, &ws);
  if (e != hipSuccess) return e;
  return enqueue_accept(draft, target, tokens, u24, b, kd, v, temperature, n_accepted, next_token, q_out, p_out,
                        static_cast<char*>(ws), stream);
}

hipError_t launch_spec_accept_noalloc(const float* draft, const float* target, const int32_t* tokens,
                                      const uint32_t* u24, int b, int kd, int v, float temperature,
                                      int32_t* n_accepted, int32_t* next_token, float* q_out, float* p_out,
                                      hipStream_t stream) {
  if (accept_scratch(b, kd, v, temperature).total() > kNoAllocScratchBytes) return hipErrorInvalidValue;
  char* ws = nullptr;
  const hipError_t e = noalloc_scratch(&ws);
  if (e != hipSuccess) return e;
  return enqueue_accept(draft, target, tokens, u24, b, kd, v, temperature, n_accepted, next_token, q_out, p_out, ws,
                        stream);
}


namespace {
// Step launches of a call: of a node's candidates after the first, those that
// the whole chip takes before the walk.  All of them for large rows, of which
// one workgroup would take some 40 us for each candidate.  A launch of up to
// 2.5 us with nothing left to do against a pass of one workgroup over a small
// row, where candidates are accepted early / late (us, one sequence): 16
// chains of 16000 logits, 15 / 7 / 3 launches 51 / 39 / 32 and 164 / 160 / 136; eight,
// 7 / 3 launches 39 / 31 and 77 / 95; 32 of 1000, 31 / 0 launches 73 / 24 and 86 / 29.
int walk_steps(int c, int v) {
  if (v > kWalkLogits || c - 1 <= v / 2048) return c - 1;
  return v / 4096;
}
}  // namespace

size_t spec_accept_multi_scratch_bytes(int b, int c, int kd, int v, float temperature) {
  const int64_t nchunk = (v + kChunk - 1) / kChunk;
  const int64_t rows_t = (int64_t)b * c * (kd + 1);
  if (temperature == 0.0f) return pad256((size_t)rows_t * nchunk * sizeof(int64_t));
  const int64_t rows = rows_t + (int64_t)kd * b * c;
  // chunk statistics, merged statistics, chunk masses of p and of the residuals, test results, the walk's R
  return pad256((size_t)rows * nchunk * sizeof(double2)) + pad256((size_t)rows * sizeof(double2)) +
         pad256((size_t)rows * nchunk * sizeof(int64_t)) + pad256((size_t)kd * b * c * sizeof(int32_t)) +
         (walk_steps(c, v) < c - 1 ? (size_t)b * v * (sizeof(int64_t) + sizeof(float)) : 0);
}

hipError_t launch_spec_accept_multi(const float* draft, const float* target, const int32_t* tokens,
                                    const uint32_t* u24, int b, int c, int kd, int v, float temperature,
                                    int32_t* n_accepted, int32_t* next_token, int32_t* chain, float* q_out,
                                    float* p_out, hipStream_t stream) {
  void* wsv = nullptr;
  hipError_t e = workspace(spec_accept_multi_scratch_bytes(b, c, kd, v, temperature), stream, &wsv);
  if (e != hipSuccess) return e;
  char* ws = static_cast<char*>(wsv);
  const int nchunk = (v + kChunk - 1) / kChunk;
  const int64_t rows_t = (int64_t)b * c * (kd + 1);
  if (temperature == 0.0f) {
    e = enqueue_argmax(target, v, rows_t, reinterpret_cast<int64_t*>(ws), stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(multi_greedy_kernel, dim3((unsigned)b), dim3(kMergeThreads), 0, stream, tokens, b, c, kd,
                       (v + kGreedyChunk - 1) / kGreedyChunk, reinterpret_cast<const int64_t*>(ws), n_accepted,
                       next_token, chain);
    return hipGetLastError();
  }
  const int64_t rows_d = (int64_t)kd * b * c, rows = rows_t + rows_d;
  double2* stats = reinterpret_cast<double2*>(ws);
  ws += pad256((size_t)rows * nchunk * sizeof(double2));
  MultiArgs a{draft, target, tokens, u24, b, c, kd, v, nchunk, temperature, reinterpret_cast<double2*>(ws),
              nullptr, nullptr, nullptr, nullptr, nullptr};
  ws += pad256((size_t)rows * sizeof(double2));
  a.zp = reinterpret_cast<int64_t*>(ws);
  a.zs = a.zp + rows_t * nchunk;
  ws += pad256((size_t)rows * nchunk * sizeof(int64_t));
  a.acc = reinterpret_cast<int32_t*>(ws);
  a.r = reinterpret_cast<int64_t*>(ws + pad256((size_t)kd * b * c * sizeof(int32_t)));
  a.q = reinterpret_cast<float*>(a.r + (size_t)b * v);
  // step i: at most c candidates meet at a node; most (sequence, depth, chain)
  // leave a launch at once, so their number is bounded and the chunks looped
  // over when there are many
  int64_t slices = rows_d > 0 ? kStepBlocks / rows_d : 1;
  slices = slices < 1 ? 1 : (slices > nchunk ? nchunk : slices);
  const size_t lds = (size_t)kd * c * 2 * sizeof(int32_t);  // at most 32 KB
  const int steps = walk_steps(c, v);
  auto go = [&](auto one_tag) {
    constexpr bool One = decltype(one_tag)::value;
    hipLaunchKernelGGL(stats_kernel<One>, dim3((unsigned)(rows * nchunk)), dim3(64), 0, stream, draft, target, rows_t,
                       v, temperature, nchunk, 0, stats, nullptr);
    // one wavefront per chunk issues the fewest instructions, four take less time while they do not fill the chip
    // (two chains of four, 1000 logits, the whole call: 27 / 24 us)
    auto rows_go = [&](auto kernel, int threads) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)(rows_t * nchunk)), dim3(threads), 0, stream, a, stats, q_out, p_out);
    };
    rows_t * nchunk <= 1024 ? rows_go(multi_rows_kernel<One, 4>, 256) : rows_go(multi_rows_kernel<One, 1>, 64);
    for (int i = 1; rows_d > 0 && i <= steps; ++i)
      hipLaunchKernelGGL(multi_step_kernel<One>, dim3((unsigned)(rows_d / c * (c - i) * slices)), dim3(kThreads), 0,
                         stream, a, (int)slices, i);
    hipLaunchKernelGGL(multi_walk_kernel<One>, dim3((unsigned)b), dim3(kMThreads), lds, stream, a, steps, n_accepted,
                       next_token, chain);
  };
  if (temperature == 1.0f)
    go(std::true_type{});
  else
    go(std::false_type{});
  return hipGetLastError();
}

}  // namespace sq
