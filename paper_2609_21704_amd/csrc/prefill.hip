// Projections of a prompt's rows (prefill, the passes that fill the caches of
// both models before SS III-D.2 starts): y = x . W'^T for hundreds to
// thousands of activation rows, with the FP16 parent or the INT4 / FP8 draft
// copy.  The streaming kernels take at most 64 rows, so a prompt of a thousand
// tokens read every weight 32 times through them; here a weight tile meets
// 128 to 256 rows.
//
// A workgroup of 8 wavefronts (two per SIMD) forms a tile of BM = 128, 192 or
// 256 rows x 256 outputs, each wavefront BM / 2 x 64 of it, in steps of 64 k
// staged in two LDS buffers: a step's loads are issued before the previous
// step's products and awaited after them.  Activations, and FP16 weights, go from memory to
// LDS directly (16 bytes a lane); quantized weights pass through registers,
// where they become halves exactly: INT4 q - z by the mantissa trick of the
// streaming kernels, a byte permute setting a pair in k order; FP8 by
// v_cvt_scalef32_pk_f16_fp8.  LDS rows are 128 bytes with their eight 16-byte
// cells exchanged by the row number (cell ^ row % 8), so that the 16 rows of a
// fragment read fall in different banks; a direct load applies the exchange
// to its source address, as its LDS address cannot.
//
// Products: v_mfma_f32_16x16x32_f16 with the weights as the A operand, so that
// a lane ends with four consecutive outputs of one row (one 16-byte store).
// INT4: the products of a 128-k group (two steps) accumulate by themselves and
// are added once, times the group's fp32 scale: exact products of q - z and x
// and one rounding of each scaled group sum, as in the streaming kernels.
// FP8: the row scale multiplies the total.
//
// Sums: one running fp32 sum over thousands of k rounds at its full size with
// every product; the matrix core's own additions cost the more, as they do not
// round to nearest.  So the sums have levels, and their errors against 64 bits
// stay at those of the streaming kernels (3584 k, these / streaming / one
// running sum: FP16 1.4e-7 / 1.5e-7 / 3.8e-7, FP8 1.1e-7 / 1.4e-7 / 3.4e-7, INT4
// 0.69e-7 / 0.69e-7 / 0.98e-7; 18944 k: 1.8e-7 / 2.3e-7 / 6.2e-7, 1.6e-7 / 1.8e-7 /
// 5.9e-7, 0.98e-7 / 1.0e-7 / 2.2e-7):
//   BM = 128, 192: a block of fold_steps steps in registers of its own (FP16
//     and FP8: the accumulators; INT4: the scaled group sums), added to the
//     total at its end.  INT4 has registers for 128 rows only;
//   BM = 256, where the total leaves no room for that: the two products of a
//     step accumulate by themselves and are added to the total by vector
//     operations, beside the next products, up to kShortSteps steps.
//
// Where the tiles do not fill the CUs, K is cut into S parts (blockIdx
// beyond the tiles) whose fp32 partial tiles a second kernel adds in order.
// BM and S are the pair with the least estimated time (choose()).
// 2000 rows by the 37888 x 3584 gate|up matrix: FP16 0.95, FP8 0.90, INT4 0.68
// PFLOP/s (with one running sum 1.02, 1.04 and 0.71).  By the counters the matrix
// cores are busy in 51, 44 and 31 % of the busy cycles and no LDS access meets a
// bank conflict; a step waits for its fragments, as the registers hold one
// step's, and quantized weights add their conversions.  Placing INT4's between
// the products instead of after them delays the fragment reads behind their LDS
// writes (877 -> 944 us).
// Prompts in 64-row blocks through the streaming kernels ran at 0.13.
// Tiles go to the XCDs in contiguous runs, all row tiles of an output tile
// next to each other, so that the workgroups of an XCD share weight and
// activation panels in its L2.
#include <type_traits>

#include "sq_device.hpp"
#include "sq_internal.hpp"

namespace sq {
namespace {

enum : int { kW4 = 0, kW8 = 1, kF16 = 2 };
constexpr int kThreads = 512;
constexpr int kBN = 256;  // outputs per tile
constexpr int kBK = 64;   // k per step
constexpr int kRowBytes = kBK * 2;
// Steps of a K part at BM = 256, at most: the error grows with their root.  FP16, whose streaming sums round the
// most, may take up to 148 where the row is at least twice as long (18944 k: 2.3e-7 each, 4000 rows 735 -> 604 us).
constexpr int kShortSteps = 88, kShortStepsF16 = 148;
// K parts' partial outputs in the workspace, which is never given back, at most.
constexpr double kPartBytes = 128e6;

typedef __attribute__((address_space(1))) const uint32_t gword;
typedef __attribute__((address_space(3))) uint32_t lword;

// 16 bytes per lane from memory to LDS: lane l's go to dst + 16 l.
__device__ __forceinline__ void load_to_lds(const void* src, void* dst) {
  __builtin_amdgcn_global_load_lds((gword*)src, (lword*)dst, 16, 0, 0);
}

template <int KIND>
constexpr int code_bytes_per_row_step() {
  return KIND == kW4 ? kBK / 2 : (KIND == kW8 ? kBK : kBK * 2);
}

// Weight row of tile row r: consecutive outputs, or (SiLU) per wavefront 32
// gate rows, then the 32 up rows of the same outputs.
template <bool SILU>
__device__ __forceinline__ int64_t weight_row(int64_t n0, int r, int64_t n) {
  if constexpr (!SILU) {
    const int64_t row = n0 + r;
    return row < n ? row : n - 1;
  } else {
    const int64_t half = n >> 1;
    const int64_t col = n0 + (r >> 6) * 32 + (r & 31);
    return (col < half ? col : half - 1) + ((r >> 5) & 1 ? half : 0);
  }
}

template <int KIND, int BM, bool SILU>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void prefill_gemm_kernel(
    const uint16_t* __restrict__ x, int64_t m, int64_t k, const uint8_t* __restrict__ w,
    const uint16_t* __restrict__ scales16, const uint16_t* __restrict__ zeros16, const float* __restrict__ scales32,
    int64_t n, void* __restrict__ y, int out, float* __restrict__ partial, int mtiles, int ntiles, int part_steps,
    int fold_steps) {
  extern __shared__ __align__(16) char smem[];
  constexpr int MT = BM / 32, NT = 4;         // 16-row tiles per wavefront
  constexpr int kABytes = BM * kRowBytes, kBBytes = kBN * kRowBytes;
  constexpr int kAIter = kABytes / 16 / kThreads, kBIter = kBBytes / 16 / kThreads;
  char* abuf = smem;                          // [2][BM][128 bytes]
  char* bbuf = smem + 2 * kABytes;            // [2][256][128 bytes]
  float* sbuf = reinterpret_cast<float*>(smem + 2 * kABytes + 2 * kBBytes);  // INT4: [2][256] group scales
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;

  // contiguous runs of tiles per XCD (workgroups go to the XCDs in turn)
  const int total = gridDim.x, per = total >> 3, rem = total & 7;
  const int xcd = blockIdx.x & 7;
  const int tile = xcd * per + (xcd < rem ? xcd : rem) + (int)(blockIdx.x >> 3);
  const int mi = tile % mtiles, nz = tile / mtiles, ni = nz % ntiles, part = nz / ntiles;
  const int64_t m0 = (int64_t)mi * BM;
  const int64_t n0 = (int64_t)ni * (SILU ? kBN / 2 : kBN);
  const int steps_all = (int)(k / kBK);
  const int s0 = part * part_steps;
  const int s1 = s0 + part_steps < steps_all ? s0 + part_steps : steps_all;

  // source offsets of this thread's direct cells: cell c = (8 i + wave) 64 + lane of the tile is row
  // c / 8, LDS cell c % 8, memory cell (c % 8) ^ (row % 8)
  uint32_t aoff[kAIter], boff[KIND == kF16 ? kBIter : 1];
#pragma unroll
  for (int i = 0; i < kAIter; ++i) {
    const int c = (8 * i + wave) * 64 + lane, r = c >> 3;
    const int64_t row = m0 + r < m ? m0 + r : m - 1;
    aoff[i] = (uint32_t)((row - m0) * k * 2) + 16 * ((c & 7) ^ (r & 7));
  }
  if constexpr (KIND == kF16) {
#pragma unroll
    for (int i = 0; i < kBIter; ++i) {
      const int c = (8 * i + wave) * 64 + lane, r = c >> 3;
      boff[i] = (uint32_t)(weight_row<SILU>(n0, r, n) * k * 2) + 16 * ((c & 7) ^ (r & 7));
    }
  }
  const char* xb = reinterpret_cast<const char*>(x + m0 * k);
  // quantized: thread t holds 32 consecutive codes of tile row t / 2
  const int qrow = tid >> 1, qhalf = tid & 1;
  const int64_t wrow = weight_row<SILU>(n0, qrow, n);
  const uint8_t* qsrc = w + wrow * (KIND == kW4 ? k >> 1 : k) + qhalf * (KIND == kW4 ? 16 : 32);
  const int64_t grow = wrow * (k >> 7);
  u32x4 qc[KIND == kW8 ? 2 : 1];
  uint32_t qz = 0, qs = 0;

  auto issue = [&](int s, int buf) {
    const int64_t kb = (int64_t)s * kRowBytes;
#pragma unroll
    for (int i = 0; i < kAIter; ++i)
      load_to_lds(xb + kb + aoff[i], abuf + buf * kABytes + (8 * i + wave) * 1024);
    if constexpr (KIND == kF16) {
#pragma unroll
      for (int i = 0; i < kBIter; ++i)
        load_to_lds(w + kb + boff[i], bbuf + buf * kBBytes + (8 * i + wave) * 1024);
    } else if constexpr (KIND == kW8) {
      const u32x4* p = reinterpret_cast<const u32x4*>(qsrc + (int64_t)s * kBK);
      qc[0] = p[0];
      qc[1] = p[1];
    } else {
      qc[0] = *reinterpret_cast<const u32x4*>(qsrc + (int64_t)s * (kBK / 2));
      if ((s & 1) == 0) {  // a group's first step
        qz = zeros16[grow + (s >> 1)];
        qs = scales16[grow + (s >> 1)];
      }
    }
  };
  uint32_t mask = 0x00F0000Fu, magic = 0x54006400u;
  if constexpr (KIND == kW4) asm("" : "+v"(mask), "+v"(magic));
  // the registers' codes as halves into buffer buf
  auto convert = [&](int s, int buf) {
    if constexpr (KIND != kF16) {
      char* row = bbuf + buf * kBBytes + qrow * kRowBytes;
      half2_t cz;
      auto code_pair = [&](uint32_t b) {
        return __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, (b & mask) | magic) - cz);
      };
      if constexpr (KIND == kW4) {
        cz = __builtin_bit_cast(half2_t, qz | (qz << 16)) + half2_t{(half_t)1024.0f, (half_t)64.0f};
        if ((s & 1) == 0 && qhalf == 0) sbuf[((s >> 1) & 1) * kBN + qrow] = f16_bits_to_f32((uint16_t)qs);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {  // 8 codes each
        u32x4 o;
        if constexpr (KIND == kW4) {
          // byte i of the word in both halves: code 2 i in bits 0-3 (1024 + q), code 2 i + 1 in bits 4-7 (64 + q)
          const uint32_t qw = qc[0][j];
          o[0] = code_pair(__builtin_amdgcn_perm(qw, qw, 0x00000000u));
          o[1] = code_pair(__builtin_amdgcn_perm(qw, qw, 0x01010101u));
          o[2] = code_pair(__builtin_amdgcn_perm(qw, qw, 0x02020202u));
          o[3] = code_pair(__builtin_amdgcn_perm(qw, qw, 0x03030303u));
        } else {
          const uint32_t w0 = qc[j >> 1][2 * (j & 1)], w1 = qc[j >> 1][2 * (j & 1) + 1];
          o[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w0, 1.0f, false));
          o[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w0, 1.0f, true));
          o[2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w1, 1.0f, false));
          o[3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w1, 1.0f, true));
        }
        *reinterpret_cast<u32x4*>(row + 16 * ((qhalf * 4 + j) ^ (qrow & 7))) = o;
      }
    }
  };

  // the total, the block's sums (kShort: none) and (INT4) the group's products
  constexpr bool kShort = BM == 256;
  float4_t tot[MT][NT], acc[kShort ? 1 : MT][kShort ? 1 : NT], grp[KIND == kW4 ? MT : 1][KIND == kW4 ? NT : 1];
#pragma unroll
  for (int a = 0; a < MT; ++a)
#pragma unroll
    for (int b = 0; b < NT; ++b) {
      tot[a][b] = float4_t{0.f, 0.f, 0.f, 0.f};
      if constexpr (!kShort) acc[a][b] = float4_t{0.f, 0.f, 0.f, 0.f};
    }
  auto fold = [&]() {
    if constexpr (!kShort) {
#pragma unroll
      for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b) {
          tot[a][b] += acc[a][b];
          acc[a][b] = float4_t{0.f, 0.f, 0.f, 0.f};
        }
    }
  };

  // fragment of 16 rows from row r0: lane l holds row r0 + l % 16, memory cells 4 kk + l / 16
  const int fr = (lane & 15) * kRowBytes, fc0 = 16 * ((lane >> 4) ^ (lane & 7)), fc1 = 16 * ((4 + (lane >> 4)) ^ (lane & 7));
  auto compute = [&](int s, int buf) {
    const char* ab = abuf + buf * kABytes + wm * (BM / 2) * kRowBytes + fr;
    const char* bb = bbuf + buf * kBBytes + wn * 64 * kRowBytes + fr;
    auto frag = [&](const char* base, int t, int kk) {
      return *reinterpret_cast<const half8_t*>(base + t * 16 * kRowBytes + (kk ? fc1 : fc0));
    };
    const float4_t zero4 = {0.f, 0.f, 0.f, 0.f};
    if constexpr (!kShort) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        // INT4: activations one row tile ahead (all at once they would not fit its registers)
        constexpr int XF = KIND == kW4 ? 2 : MT;
        half8_t wf[NT], xf[XF];
#pragma unroll
        for (int b = 0; b < NT; ++b) wf[b] = frag(bb, b, kk);
#pragma unroll
        for (int a = 0; a < XF - (KIND == kW4); ++a) xf[a] = frag(ab, a, kk);
#pragma unroll
        for (int a = 0; a < MT; ++a) {
          if (KIND == kW4 && a + 1 < MT) xf[(a + 1) % XF] = frag(ab, a + 1, kk);
#pragma unroll
          for (int b = 0; b < NT; ++b) {
            if constexpr (KIND == kW4)
              grp[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                  wf[b], xf[a % XF], (s & 1) == 0 && kk == 0 ? zero4 : grp[a][b], 0, 0, 0);
            else
              acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[b], xf[a % XF], acc[a][b], 0, 0, 0);
          }
        }
      }
      if constexpr (KIND == kW4) {
        if (s & 1) {  // the group's last step (K slices start at whole groups)
#pragma unroll
          for (int b = 0; b < NT; ++b) {
            const float4_t sc =
                *reinterpret_cast<const float4_t*>(sbuf + ((s >> 1) & 1) * kBN + wn * 64 + b * 16 + 4 * (lane >> 4));
#pragma unroll
            for (int a = 0; a < MT; ++a) acc[a][b] += sc * grp[a][b];
          }
        }
      }
    } else {
      half8_t wf[2][NT];
#pragma unroll
      for (int b = 0; b < NT; ++b) {
        wf[0][b] = frag(bb, b, 0);
        wf[1][b] = frag(bb, b, 1);
      }
      auto products = [&](half8_t x0, half8_t x1, float4_t (&d)[NT]) {
#pragma unroll
        for (int b = 0; b < NT; ++b) d[b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[0][b], x0, zero4, 0, 0, 0);
#pragma unroll
        for (int b = 0; b < NT; ++b) d[b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[1][b], x1, d[b], 0, 0, 0);
      };
      if constexpr (KIND == kF16) {
#pragma unroll
        for (int a = 0; a < MT; ++a) {
          float4_t d[NT];
          products(frag(ab, a, 0), frag(ab, a, 1), d);
#pragma unroll
          for (int b = 0; b < NT; ++b) tot[a][b] += d[b];
        }
      } else {
        // a row tile's vector adds beside the next one's products, no more of them at once (the registers)
        float4_t d[2][NT];
        half8_t xf[2][2];
        xf[0][0] = frag(ab, 0, 0);
        xf[0][1] = frag(ab, 0, 1);
#pragma unroll
        for (int a = 0; a <= MT; ++a) {
          if (a + 1 < MT) {
            xf[(a + 1) & 1][0] = frag(ab, a + 1, 0);
            xf[(a + 1) & 1][1] = frag(ab, a + 1, 1);
          }
          if (a < MT) products(xf[a & 1][0], xf[a & 1][1], d[a & 1]);
          if (a > 0) {
#pragma unroll
            for (int b = 0; b < NT; ++b) tot[a - 1][b] += d[(a - 1) & 1][b];
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };
  auto sync = [&]() {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
  };

  issue(s0, 0);
  convert(s0, 0);
  sync();
  auto step = [&](int s, int buf) {
    if (s + 1 < s1) issue(s + 1, buf ^ 1);
    compute(s, buf);
    // (FP8 at 256 rows: after the last step the old codes go into the buffer that nobody reads any more; a branch
    // there makes the compiler keep totals in memory)
    if ((KIND == kW8 && BM == 256) || s + 1 < s1) convert(s + 1, buf ^ 1);
    sync();
  };
  // (two steps a turn: the buffers and the halves of an INT4 group alternate; s0 is even for INT4)
  int left = fold_steps;  // an even number
  for (int s = s0; s < s1; s += 2) {
    step(s, 0);
    if (s + 1 < s1) step(s + 1, 1);
    left -= 2;
    if (left == 0) {
      fold();
      left = fold_steps;
    }
  }
  fold();

  // outputs: lane l holds outputs 4 (l / 16) .. +4 of a 16-output tile for row l % 16 of a row tile
  const int q4 = 4 * (lane >> 4);
  if constexpr (KIND == kW8) {
#pragma unroll
    for (int b = 0; b < NT; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float sc = scales32[weight_row<SILU>(n0, wn * 64 + b * 16 + q4 + r, n)];
#pragma unroll
        for (int a = 0; a < MT; ++a) tot[a][b][r] *= sc;
      }
  }
  const bool vec = (n & 3) == 0;
#pragma unroll
  for (int a = 0; a < MT; ++a) {
    const int64_t row = m0 + wm * (BM / 2) + a * 16 + (lane & 15);
    if (row >= m) continue;
    if (SILU && !partial) {
      const int64_t half = n >> 1;
      uint16_t* t = reinterpret_cast<uint16_t*>(y) + row * half;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int64_t col = n0 + wn * 32 + b * 16 + q4;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (col + r < half) t[col + r] = silu_gate_bits(tot[a][b][r], tot[a][b + 2][r]);
      }
      continue;
    }
#pragma unroll
    for (int b = 0; b < NT; ++b) {
      // (SiLU partials: rows [m][n] as without it, gates then ups)
      const int64_t col = SILU ? n0 + wn * 32 + (b & 1) * 16 + q4 : n0 + wn * 64 + b * 16 + q4;
      const int64_t end = SILU ? n >> 1 : n;
      float* o = (partial ? partial + (int64_t)part * m * n : reinterpret_cast<float*>(y)) + row * n + col +
                 (SILU && b >= 2 ? n >> 1 : 0);
      const bool add = !partial && out == 1;
      if (vec && (!SILU || (n & 7) == 0) && col + 3 < end) {
        float4_t v = tot[a][b];
        if (add) v = *reinterpret_cast<const float4_t*>(o) + v;
        *reinterpret_cast<float4_t*>(o) = v;
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (col + r < end) o[r] = (add ? o[r] : 0.f) + tot[a][b][r];
      }
    }
  }
}

// The K parts' partial outputs in part order, then the output form: 0 y =, 1
// y +=, 2 t = silu(gate) * up.
__global__ __launch_bounds__(256) void prefill_reduce_kernel(const float* __restrict__ partial, int parts, int64_t m,
                                                             int64_t n, void* __restrict__ y, int out) {
  const int64_t mn = m * n, half = n >> 1, total = out == 2 ? m * half : mn;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    if (out == 2) {
      const int64_t row = i / half, g = row * n + (i - row * half);
      float a = 0.f, b = 0.f;
      for (int s = 0; s < parts; ++s) {
        a += partial[s * mn + g];
        b += partial[s * mn + g + half];
      }
      reinterpret_cast<uint16_t*>(y)[i] = silu_gate_bits(a, b);
    } else {
      float v = 0.f;
      for (int s = 0; s < parts; ++s) v += partial[s * mn + i];
      float* o = reinterpret_cast<float*>(y) + i;
      *o = out == 1 ? *o + v : v;
    }
  }
}

struct Plan {
  int bm, parts, part_steps;
};

// The pair (rows per tile, K parts) of least estimated time: rounds of tiles
// over the CUs, each of its steps and a start, and the partial outputs' way to
// memory and back.  A step takes longer the more CUs stream (the share of them
// that a last round uses), as its operands come from memory.  Constants in us,
// fitted to 210 shapes a kind (14 matrices from 1152 x 896 to 37888 x 3584 at 100 ..
// 4000 rows, in several copies, so that no operand lies in a cache) with every
// tile and up to 12 K parts: the plans it takes are within 1.2 % (FP16) and 0.4 %
// (FP8, INT4) of the fastest on average, at worst 21 % (9728 x 896, 100 rows).
Plan choose(int64_t m, int64_t n, int64_t k, int kind) {
  struct Cost {
    double step, full, start;  // a step alone, what a full chip adds to it, a round
  };
  constexpr Cost kCost[3][3] = {{{1.19, 0.24, 6.5}, {}, {}},  // [kind][BM / 64 - 2]
                                {{0.97, 0.22, 6.5}, {1.24, 0.25, 9.5}, {1.73, 0.50, 10}},
                                {{0.87, 0.51, 6}, {1.10, 0.48, 8.5}, {1.38, 0.58, 10}}};
  const int64_t cus = cu_count(), nt = (n + kBN - 1) / kBN, steps = k / kBK;
  Plan best{128, 1, (int)steps};
  double tbest = 1e30;
  for (int bm = 128; bm <= (kind == kW4 ? 128 : 256); bm += 64) {
    const Cost c = kCost[kind][bm / 64 - 2];
    const int64_t tiles = (m + bm - 1) / bm * nt;
    for (int parts = 1; parts <= 16; ++parts) {
      int64_t ps = (steps + parts - 1) / parts;
      ps += ps & 1;  // whole INT4 groups
      if (parts > 1 && (ps < 4 || (int64_t)(parts - 1) * ps >= steps)) break;
      if (parts > 1 && (double)parts * m * n * 4 > kPartBytes) break;
      if (bm == 256 && ps > kShortSteps && !(kind == kF16 && parts > 1 && ps <= kShortStepsF16)) continue;
      const int64_t whole = tiles * parts / cus, rest = tiles * parts % cus;
      double t = (double)whole * ((double)ps * (c.step + c.full) + c.start);
      if (rest > 0) t += (double)ps * (c.step + c.full * (double)rest / (double)cus) + c.start;
      if (parts > 1) t += 6.0 + (double)parts * m * n * 8 * 0.09e-6;
      if (t < tbest) {
        tbest = t;
        best = Plan{bm, parts, (int)ps};
      }
    }
  }
  return best;
}

// Steps per block of the sums: about where the roundings inside blocks and
// between them are as many (those inside count more in the accumulators).
int block_steps(int part_steps, int kind) {
  if (kind == kW4) return part_steps <= 128 ? 8 : 24;
  return part_steps <= 24 ? 4 : (part_steps <= 128 ? 6 : 8);
}

template <int KIND>
hipError_t prefill_launch(const uint16_t* x, int64_t m, int64_t k, const uint8_t* w, const uint16_t* scales16,
                          const uint16_t* zeros16, const float* scales32, int64_t n, void* y, int out,
                          hipStream_t stream) {
  if (k % (KIND == kW4 ? 128 : kBK) != 0 || m < 1 || m > (int64_t(1) << 20)) return hipErrorNotSupported;
  // 32-bit offsets inside a weight matrix and a row tile
  if ((double)n * (double)k * 2 >= 4294967296.0 || (double)k * 2 * 256 >= 4294967296.0) return hipErrorNotSupported;
  const Plan p = choose(m, n, k, KIND);
  const int64_t mt = (m + p.bm - 1) / p.bm;
  const int64_t nt = out == 2 ? (n / 2 + kBN / 2 - 1) / (kBN / 2) : (n + kBN - 1) / kBN;
  const int64_t tiles = mt * nt * p.parts;
  if (tiles > (int64_t(1) << 22)) return hipErrorNotSupported;  // a grid holds fewer than 2^32 threads
  float* partial = nullptr;
  if (p.parts > 1) {
    void* ws = nullptr;
    const hipError_t e = workspace((size_t)p.parts * m * n * sizeof(float), stream, &ws);
    if (e != hipSuccess) return e;
    partial = static_cast<float*>(ws);
  }
  auto go = [&](auto kernel, int bm) {
    const size_t lds = (size_t)2 * (bm + kBN) * kRowBytes + (KIND == kW4 ? 2 * kBN * sizeof(float) : 0);
    hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(kThreads), lds, stream, x, m, k, w, scales16, zeros16,
                       scales32, n, y, out, partial, (int)mt, (int)nt, p.part_steps, block_steps(p.part_steps, KIND));
  };
  auto form = [&](auto bm) {
    constexpr int BM = decltype(bm)::value;
    out == 2 ? go(prefill_gemm_kernel<KIND, BM, true>, BM) : go(prefill_gemm_kernel<KIND, BM, false>, BM);
  };
  if (KIND == kW4 || p.bm == 128)
    form(std::integral_constant<int, 128>{});
  else if constexpr (KIND != kW4)
    p.bm == 192 ? form(std::integral_constant<int, 192>{}) : form(std::integral_constant<int, 256>{});
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess || p.parts == 1) return err;
  const int64_t total = out == 2 ? m * (n / 2) : m * n;
  int64_t blocks = (total + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(prefill_reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, partial, p.parts, m, n, y,
                     out);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_prefill_w4(const uint16_t* x, int64_t m, int64_t k, const uint8_t* codes, const uint16_t* scales,
                             const uint16_t* zeros, int64_t n, void* y, int out, hipStream_t stream) {
  return prefill_launch<kW4>(x, m, k, codes, scales, zeros, nullptr, n, y, out, stream);
}

hipError_t launch_prefill_w8(const uint16_t* x, int64_t m, int64_t k, const uint8_t* codes, const float* scales,
                             int64_t n, void* y, int out, hipStream_t stream) {
  return prefill_launch<kW8>(x, m, k, codes, nullptr, nullptr, scales, n, y, out, stream);
}

hipError_t launch_prefill_f16(const uint16_t* x, int64_t m, int64_t k, const uint16_t* w, int64_t n, void* y, int out,
                              hipStream_t stream) {
  return prefill_launch<kF16>(x, m, k, reinterpret_cast<const uint8_t*>(w), nullptr, nullptr, nullptr, n, y, out,
                              stream);
}

}  // namespace sq
