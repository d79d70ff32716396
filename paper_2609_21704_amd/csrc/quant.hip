// Offline derivation of the quantized draft parents from the FP16 parent
// (SpecQuant SS III-A.1: Q4 = f(W16, 4); SS III-A.2: Q8 = f(W16, 8)).
//
// The produced bytes are those of the fp64 formulas (IEEE division, ties to
// even), a deterministic function of the FP16 input.  Both are streaming
// kernels: 2 B read per weight, 17/32 B (INT4 g128) or 1 B (FP8) written.
// In fp64 the divisions bound them, not HBM (37888 x 3584: 214 and 190 us);
// here each element takes the exact fp64 decision from fp32 arithmetic, whose
// sufficiency is shown at each step (the same matrix: 80 and 89 us, 4.3 and 4.6 TB/s).
#include "sq_device.hpp"
#include "sq_internal.hpp"

#pragma clang fp contract(off)

namespace sq {
namespace {

typedef uint16_t ushort2_t __attribute__((ext_vector_type(2)));

// Division by a reciprocal estimate, one Newton step on it and one correction
// of the quotient by its exact fused remainder: Markstein, Computation of
// elementary functions on the IBM RISC System/6000 processor, 1990.
//
// 1 / s correctly rounded or within one ulp of it, for s > 0 whose reciprocal
// is a normal float.
__device__ __forceinline__ float recip(float s) {
  const float r = __builtin_amdgcn_rcpf(s);
  return __builtin_fmaf(__builtin_fmaf(-s, r, 1.0f), r, r);
}

// v / s to within half an ulp (+ 2^-20 of one): the exact remainder of the
// first estimate corrects it.  A quotient with few bits comes out exactly.
__device__ __forceinline__ float quotient(float v, float s, float rs) {
  const float q0 = v * rs;
  return __builtin_fmaf(__builtin_fmaf(-q0, s, v), rs, q0);
}

// Smallest binary16 value >= s for a finite s > 0 that is a normal double.
// The binary16 grid near s has spacing 2^(e-10) (e = floor(log2 s) >= -14) or
// 2^-24 (subnormal range); scaling by that spacing is exact, so ceil() picks
// the next grid point exactly.
__device__ __forceinline__ double f16_ceil(double s) {
  const uint64_t bits = (uint64_t)__double_as_longlong(s);
  const int e = (int)((bits >> 52) & 0x7FF) - 1023;
  const int sp = (e < -14) ? -24 : e - 10;
  return ldexp(ceil(ldexp(s, -sp)), sp);
}

// One step of the minimum over a row of 16 lanes of two packed halves.
template <int Ctrl>
__device__ __forceinline__ half2_t dpp_min(half2_t v) {
  const int o = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), Ctrl, 0xF, 0xF, false);
  return __builtin_elementwise_min(v, __builtin_bit_cast(half2_t, o));
}

template <int R>
__device__ __forceinline__ int row_lane(int v) {  // lane R of the own row of 16 lanes
  return __builtin_amdgcn_update_dpp(0, v, 0x150 + R, 0xF, 0xF, false);
}

// INT4 g128.  A wavefront takes 16 consecutive groups at a time: lane l holds
// the 16 bytes l % 16 of groups l / 16 + 4 r, r = 0 .. 3 (1 KB contiguous per
// r).  Minimum and maximum stay packed halves (exact).  The scale and zero of
// a group, the only fp64 arithmetic, are formed once by every fourth lane of
// its row (lane l those of r = l % 4) instead of by all 16, and broadcast.
// Codes: rint(v / s) in fp64 equals rint of the fp32 quotient: v and s have
// 11-bit mantissas and |v / s| <= 15, so a quotient that is not a half-integer
// is at least 2^-12 from one, and a half-integer comes out of quotient()
// exactly.  Adding 1.5 2^23 rounds it to an integer, ties to even, in the low
// mantissa bits; the clamp to [-z, 15 - z] is one median there, and the
// nibbles are gathered by shifted adds whose common base is subtracted once.
// Groups are contiguous in memory because k % 128 == 0.
__global__ __launch_bounds__(256) void quantize_int4_kernel(const uint16_t* __restrict__ w, int64_t ngroups,
                                                            uint8_t* __restrict__ codes,
                                                            uint16_t* __restrict__ scales,
                                                            uint16_t* __restrict__ zeros, int32_t* flag) {
  const int lane = threadIdx.x & 63, sub = lane & 15, row = lane >> 4;
  const int64_t g0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16;
  if (g0 >= ngroups) return;  // uniform across the wavefront
  u32x4 raw[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t gi = g0 + 4 * r + row;
    raw[r] = *reinterpret_cast<const u32x4*>(w + (gi < ngroups ? gi : ngroups - 1) * 128 + sub * 8);
  }
  half2_t ext[4];  // (min, -max) of the group, the range widened to hold zero
  uint32_t bad = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    half2_t mn = {(half_t)0, (half_t)0}, mx = {(half_t)0, (half_t)0};
    ushort2_t mag = {0, 0};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t e = raw[r][i];  // scalar copies: vector element lvalues are misread by bit_cast
      mn = __builtin_elementwise_min(mn, __builtin_bit_cast(half2_t, e));
      mx = __builtin_elementwise_max(mx, __builtin_bit_cast(half2_t, e));
      mag = __builtin_elementwise_max(mag, __builtin_bit_cast(ushort2_t, e & 0x7FFF7FFFu));
    }
    const uint64_t nonfinite = __ballot(mag[0] >= 0x7C00 || mag[1] >= 0x7C00);
    bad |= ((nonfinite >> (16 * row)) & 0xFFFFull) != 0 ? 1u << r : 0u;
    half2_t x = {mn[0] < mn[1] ? mn[0] : mn[1], mx[0] > mx[1] ? -mx[0] : -mx[1]};
    x = dpp_min<0xB1>(x);   // quad_perm [1,0,3,2]
    x = dpp_min<0x4E>(x);   // quad_perm [2,3,0,1]
    x = dpp_min<0x141>(x);  // row_half_mirror
    x = dpp_min<0x140>(x);  // row_mirror
    ext[r] = x;
  }
  // the group r = sub % 4 of this row: scale, zero
  const int rs4 = sub & 3;
  const half2_t mine = rs4 == 0 ? ext[0] : (rs4 == 1 ? ext[1] : (rs4 == 2 ? ext[2] : ext[3]));
  const bool mybad = (bad >> rs4) & 1u;
  const float lo = (float)mine[0], hi = -(float)mine[1];
  const bool flat = hi == lo;
  // of a non-finite group only the markers are used
  const double range = mybad || flat ? 15.0 : (double)hi - (double)lo;
  const float s = (float)f16_ceil(range / 15.0);  // exactly a binary16
  const float rs = recip(s);
  float z = mybad ? 0.0f : __builtin_rintf(quotient(-lo, s, rs));
  z = z > 0.0f ? (z > 15.0f ? 15.0f : z) : 0.0f;  // also maps -0 (lo == 0) to +0
  const int64_t mygi = g0 + 4 * rs4 + row;
  if (sub < 4 && mygi < ngroups) {
    scales[mygi] = mybad ? (uint16_t)0x7E00 : f32_to_f16_bits(s);  // a NaN scale marks the group
    zeros[mygi] = f32_to_f16_bits(z);
    if (mybad && flag) atomicOr(flag, 1);
  }
  const int si = __float_as_int(s), ri = __float_as_int(rs), zi = __float_as_int(z);
  const float sg[4] = {__int_as_float(row_lane<0>(si)), __int_as_float(row_lane<1>(si)),
                       __int_as_float(row_lane<2>(si)), __int_as_float(row_lane<3>(si))};
  const float rg[4] = {__int_as_float(row_lane<0>(ri)), __int_as_float(row_lane<1>(ri)),
                       __int_as_float(row_lane<2>(ri)), __int_as_float(row_lane<3>(ri))};
  const float zg[4] = {__int_as_float(row_lane<0>(zi)), __int_as_float(row_lane<1>(zi)),
                       __int_as_float(row_lane<2>(zi)), __int_as_float(row_lane<3>(zi))};
  constexpr float kMagic = 12582912.0f;  // 1.5 2^23
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float base = kMagic - zg[r], top = base + 15.0f;  // code 0 and code 15
    uint32_t packed = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const half_t h = __builtin_bit_cast(half_t, (uint16_t)(raw[r][i >> 1] >> (16 * (i & 1))));
      const float c = __builtin_amdgcn_fmed3f(quotient((float)h, sg[r], rg[r]) + kMagic, base, top);
      packed += __float_as_uint(c) << (4 * i);  // element i -> byte i/2, nibble i%2
    }
    packed -= __float_as_uint(base) * 0x11111111u;
    if ((bad >> r) & 1u) packed = 0u;
    const int64_t gi = g0 + 4 * r + row;
    if (gi < ngroups) reinterpret_cast<uint32_t*>(codes + gi * 64)[sub] = packed;
  }
}

// Eight OCP E4M3 codes of eight halves over the row scale s: the encode of the
// fp64 quotient (nearest, ties to even, saturating, sign of zero kept).  The
// midpoint of two E4M3 values has five bits, so v / s (11 over 24 bits) that
// is not a midpoint differs from one by at least 2^-30 of its size: the fp64
// quotient decides as the exact one does, the fp32 quotient alone may not
// (it can round onto the midpoint).  So the fp32 quotient is rounded to odd:
// where its exact remainder is not zero and its last bit is even, it moves
// one ulp towards the exact quotient, which keeps it off every midpoint; the
// conversion instruction then rounds as from the exact quotient.
__device__ __forceinline__ float to_odd(float v, float s, float rs) {
  const float q = quotient(v, s, rs);
  const float r = __builtin_fmaf(-q, s, v);  // the sign of the exact remainder, zero only when that is
  const int b = __float_as_int(q);
  const int toward = ((__float_as_int(r) ^ b) >> 31) | 1;  // away from zero when the remainder has q's sign
  const int odd = b + (r != 0.0f && (b & 1) == 0 ? toward : 0);
  return __builtin_amdgcn_fmed3f(__builtin_copysignf(__int_as_float(odd), v), -448.0f, 448.0f);  // (-0 keeps its sign)
}

__device__ __forceinline__ uint2 encode8(u32x4 raw, float s, float rs) {
  uint32_t out[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    float t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      t[i] = to_odd((float)__builtin_bit_cast(half_t, (uint16_t)(raw[2 * j + (i >> 1)] >> (16 * (i & 1)))), s, rs);
    int o = __builtin_amdgcn_cvt_pk_fp8_f32(t[0], t[1], 0, false);
    o = __builtin_amdgcn_cvt_pk_fp8_f32(t[2], t[3], o, true);
    out[j] = (uint32_t)o;
  }
  return make_uint2(out[0], out[1]);
}

__device__ __forceinline__ ushort2_t mag_max(ushort2_t m, u32x4 raw) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t e = raw[i];
    m = __builtin_elementwise_max(m, __builtin_bit_cast(ushort2_t, e & 0x7FFF7FFFu));
  }
  return m;
}

// The largest fp16 magnitude over the wavefront (bit patterns of finite fp16
// magnitudes are ordered; non-finite ones, >= 0x7C00, dominate).
__device__ __forceinline__ uint32_t wave_mag(ushort2_t m) {
  uint32_t a = m[0] > m[1] ? m[0] : m[1];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const uint32_t o = __shfl_xor(a, off, 64);
    a = o > a ? o : a;
  }
  return a;
}

// The row's scale from its largest magnitude: fl32(amax / 448), 1 for an
// all-zero row, NaN for a row with a non-finite value.
__device__ __forceinline__ float row_scale(uint32_t amax) {
  if (amax >= 0x7C00u) return __builtin_nanf("");
  const double am = (double)__builtin_bit_cast(half_t, (uint16_t)amax);
  return amax == 0 ? 1.0f : (float)(am / 448.0);
}

// FP8, a row in the registers of W wavefronts (1: four rows per workgroup, no
// barrier; 4: one), NV cells of 8 values per lane: read once.  k % 16 == 0,
// so a row is whole cells and every 16-B load and 8-B store is aligned.
template <int NV, int W>
__global__ __launch_bounds__(256) void quantize_fp8_kernel(const uint16_t* __restrict__ w, int64_t n, int64_t k,
                                                           uint8_t* __restrict__ codes, float* __restrict__ scales,
                                                           int32_t* flag) {
  __shared__ uint32_t red[4];
  const int wave = threadIdx.x >> 6;
  const int t = W == 1 ? (int)(threadIdx.x & 63) : (int)threadIdx.x;
  const int64_t row = W == 1 ? (int64_t)blockIdx.x * 4 + wave : (int64_t)blockIdx.x;
  if (row >= n) return;  // uniform across the wavefront (W == 1) or never (W == 4)
  const int cells = (int)(k >> 3);
  const u32x4* src = reinterpret_cast<const u32x4*>(w + row * k);
  u32x4 raw[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = t + 64 * W * i;
    raw[i] = src[c < cells ? c : cells - 1];
  }
  ushort2_t m = {0, 0};
#pragma unroll
  for (int i = 0; i < NV; ++i) m = mag_max(m, raw[i]);
  uint32_t amax = wave_mag(m);
  if constexpr (W > 1) {
    if ((threadIdx.x & 63) == 0) red[wave] = amax;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) amax = red[i] > amax ? red[i] : amax;
  }
  const bool bad = amax >= 0x7C00u;
  const float s = row_scale(amax);
  if (t == 0) {
    scales[row] = s;
    if (bad && flag) atomicOr(flag, 1);
  }
  const float rs = recip(s);
  uint2* dst = reinterpret_cast<uint2*>(codes + row * k);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = t + 64 * W * i;
    if (c < cells) dst[c] = bad ? make_uint2(0u, 0u) : encode8(raw[i], s, rs);
  }
}

// Rows longer than the registers of a workgroup hold (k > 32768): two passes
// over the row, one workgroup per row.
__global__ __launch_bounds__(1024) void quantize_fp8_long_kernel(const uint16_t* __restrict__ w, int64_t k,
                                                                 uint8_t* __restrict__ codes,
                                                                 float* __restrict__ scales, int32_t* flag) {
  __shared__ uint32_t red[16];
  const int64_t row = blockIdx.x;
  const int cells = (int)(k >> 3);
  const u32x4* src = reinterpret_cast<const u32x4*>(w + row * k);
  ushort2_t m = {0, 0};
  for (int c = threadIdx.x; c < cells; c += 1024) m = mag_max(m, src[c]);
  uint32_t amax = wave_mag(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = amax;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; ++i) amax = red[i] > amax ? red[i] : amax;
  const bool bad = amax >= 0x7C00u;
  const float s = row_scale(amax);
  if (threadIdx.x == 0) {
    scales[row] = s;
    if (bad && flag) atomicOr(flag, 1);
  }
  const float rs = recip(s);
  uint2* dst = reinterpret_cast<uint2*>(codes + row * k);
  for (int c = threadIdx.x; c < cells; c += 1024) dst[c] = bad ? make_uint2(0u, 0u) : encode8(src[c], s, rs);
}

}  // namespace

hipError_t launch_quantize_int4(const uint16_t* w, int64_t n, int64_t k, uint8_t* codes, uint16_t* scales,
                                uint16_t* zeros, int32_t* flag, hipStream_t stream) {
  // 64 groups per workgroup; a matrix of more than 2^29 groups goes in several launches (a grid holds
  // fewer than 2^32 threads)
  const int64_t ngroups = n * (k / 128);
  constexpr int64_t kMaxBlocks = int64_t(1) << 23;
  for (int64_t g0 = 0; g0 < ngroups; g0 += kMaxBlocks * 64) {
    const int64_t ng = ngroups - g0 < kMaxBlocks * 64 ? ngroups - g0 : kMaxBlocks * 64;
    hipLaunchKernelGGL(quantize_int4_kernel, dim3((unsigned)((ng + 63) / 64)), dim3(256), 0, stream, w + g0 * 128, ng,
                       codes + g0 * 64, scales + g0, zeros + g0, flag);
  }
  return hipGetLastError();
}

hipError_t launch_quantize_fp8(const uint16_t* w, int64_t n, int64_t k, uint8_t* codes, float* scales,
                               int32_t* flag, hipStream_t stream) {
  constexpr int64_t kMaxRows = int64_t(1) << 22;  // rows per launch (a grid holds fewer than 2^32 threads)
  for (int64_t r0 = 0; r0 < n; r0 += kMaxRows) {
    const int64_t rows = n - r0 < kMaxRows ? n - r0 : kMaxRows;
    const uint16_t* wr = w + r0 * k;
    uint8_t* cr = codes + r0 * k;
    float* sr = scales + r0;
    const dim3 by_wave((unsigned)((rows + 3) / 4)), by_row((unsigned)rows);
    // a wavefront per row while a lane's share stays within 8 cells (4096 values: two rows' loads in
    // flight per SIMD and no barrier), then a workgroup per row
    auto go = [&](auto kernel, dim3 grid) {
      hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, wr, rows, k, cr, sr, flag);
    };
    if (k <= 512 * 2)
      go(quantize_fp8_kernel<2, 1>, by_wave);
    else if (k <= 512 * 4)
      go(quantize_fp8_kernel<4, 1>, by_wave);
    else if (k <= 512 * 8)
      go(quantize_fp8_kernel<8, 1>, by_wave);
    else if (k <= 2048 * 4)
      go(quantize_fp8_kernel<4, 4>, by_row);
    else if (k <= 2048 * 8)
      go(quantize_fp8_kernel<8, 4>, by_row);
    else if (k <= 2048 * 16)
      go(quantize_fp8_kernel<16, 4>, by_row);
    else
      hipLaunchKernelGGL(quantize_fp8_long_kernel, by_row, dim3(1024), 0, stream, wr, k, cr, sr, flag);
  }
  return hipGetLastError();
}

}  // namespace sq
