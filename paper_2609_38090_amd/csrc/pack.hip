// Device packer: fp32/bf16 expert weights -> packed experts (paper section
// IV-B).  Per expert-hidden row r:
//   alpha_r = max(|gate[r,:]|_inf, |up[r,:]|_inf, |down[:,r]|_inf)
//   sigma_r = bf16_rne(fl32(max(alpha_r, eps) / 127))
//   q       = clamp(rint_even(fl32(w / sigma_r)), -127, 127)
// The division is the IEEE correctly rounded fp32 one (this file is built
// without fast-math), so the bytes equal the host packer's.
#include "device_util.h"
#include "int4_format.h"
#include "mira_internal.h"

namespace mira {

template <typename WT>
__device__ __forceinline__ float ldw(const WT* p, size_t i);
template <>
__device__ __forceinline__ float ldw<float>(const float* p, size_t i) { return p[i]; }
template <>
__device__ __forceinline__ float ldw<uint16_t>(const uint16_t* p, size_t i) {
  return bf16_to_f32(p[i]);
}

// amax[e][r] = max over gate row r and up row r (one wave per row)
template <typename WT>
__global__ __launch_bounds__(256) void pack_rowmax_kernel(const WT* __restrict__ wg,
                                                          const WT* __restrict__ wu, int C, int R,
                                                          uint32_t* __restrict__ amax) {
  const int e = blockIdx.y;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (r >= R) return;
  const size_t base = ((size_t)e * R + r) * C;
  float m = 0.f;
  for (int c = lane; c < C; c += 64) m = fmaxf(m, fmaxf(fabsf(ldw(wg, base + c)), fabsf(ldw(wu, base + c))));
  m = wave_max(m);
  if (lane == 0) amax[(size_t)e * R + r] = __float_as_uint(m);
}

// amax[e][r] = max(amax[e][r], max over a chunk of c of |down[c][r]|)
template <typename WT>
__global__ __launch_bounds__(256) void pack_colmax_kernel(const WT* __restrict__ wd, int C, int R,
                                                          int c_chunk, uint32_t* __restrict__ amax) {
  const int e = blockIdx.z;
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= R) return;
  const int c0 = blockIdx.y * c_chunk, c1 = min(C, c0 + c_chunk);
  const WT* p = wd + (size_t)e * C * R + r;
  float m = 0.f;
  for (int c = c0; c < c1; ++c) m = fmaxf(m, fabsf(ldw(p, (size_t)c * R)));
  // non-negative floats order like their bit patterns
  atomicMax(&amax[(size_t)e * R + r], __float_as_uint(m));
}

__device__ __forceinline__ float scale_of(uint32_t amax_bits, float eps) {
  const float s32 = fmaxf(__uint_as_float(amax_bits), eps) / 127.0f;
  return bf16_to_f32(f32_to_bf16_rne(s32));
}

__device__ __forceinline__ int8_t quant(float w, float sigma) {
  float q = rintf(w / sigma);
  q = fminf(fmaxf(q, -127.f), 127.f);
  return (int8_t)(int)q;
}

// gate/up rows: blob[e] bytes [0, 2RC) in the tiled layout; one workgroup per (row, matrix)
template <typename WT>
__global__ __launch_bounds__(256) void pack_quant_rows_kernel(const WT* __restrict__ wg,
                                                              const WT* __restrict__ wu, int C,
                                                              int R, float eps,
                                                              const uint32_t* __restrict__ amax,
                                                              int8_t* __restrict__ packed,
                                                              uint64_t stride) {
  const int e = blockIdx.z, mat = blockIdx.y, r = blockIdx.x;
  const float sigma = scale_of(amax[(size_t)e * R + r], eps);
  const WT* src = (mat == 0 ? wg : wu) + ((size_t)e * R + r) * C;
  int8_t* dst = packed + (size_t)e * stride + (size_t)mat * R * C;
  for (int c = threadIdx.x; c < C; c += 256) dst[tiled_offset(r, c, C)] = quant(ldw(src, c), sigma);
}

// down [C][R]: column r uses sigma_r; also writes sigma and zero padding
template <typename WT>
__global__ __launch_bounds__(256) void pack_quant_down_kernel(const WT* __restrict__ wd, int C,
                                                              int R, float eps,
                                                              const uint32_t* __restrict__ amax,
                                                              int8_t* __restrict__ packed,
                                                              uint64_t stride) {
  const int e = blockIdx.z, c = blockIdx.y;
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= R) return;
  const float sigma = scale_of(amax[(size_t)e * R + r], eps);
  int8_t* blob = packed + (size_t)e * stride;
  blob[(size_t)2 * R * C + tiled_offset(c, r, R)] = quant(ldw(wd, ((size_t)e * C + c) * R + r), sigma);
  if (c == 0) {
    uint16_t* sig = (uint16_t*)(blob + (size_t)3 * R * C);
    sig[r] = f32_to_bf16_rne(fmaxf(__uint_as_float(amax[(size_t)e * R + r]), eps) / 127.0f);
  }
}

__global__ __launch_bounds__(256) void pack_pad_kernel(int8_t* __restrict__ packed, uint64_t stride,
                                                       uint64_t used) {
  const int e = blockIdx.y;
  for (uint64_t i = used + (uint64_t)blockIdx.x * 256 + threadIdx.x; i < stride;
       i += (uint64_t)gridDim.x * 256)
    packed[(size_t)e * stride + i] = 0;
}

// INT4 variant: one thread per (row, group of 64 columns) of one matrix of one
// expert; it owns the group's 32 nibble bytes (four 8-byte half-runs) and its
// scale.
template <typename WT>
__global__ __launch_bounds__(256) void pack_i4_kernel(const WT* __restrict__ wg,
                                                      const WT* __restrict__ wu,
                                                      const WT* __restrict__ wd, int C, int R,
                                                      float eps, uint8_t* __restrict__ packed,
                                                      uint64_t stride) {
  const int mat = blockIdx.y, e = blockIdx.z;
  const int rows = mat == 2 ? C : R, K = mat == 2 ? R : C;
  const int groups = K / 64;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (int64_t)rows * groups) return;
  const int r = (int)(idx / groups), blk = (int)(idx - (int64_t)r * groups);
  const WT* src = (mat == 0 ? wg : mat == 1 ? wu : wd) + (size_t)e * R * C + (size_t)r * K + blk * 64;
  float w[64];
  float alpha = 0.f;
#pragma unroll
  for (int c = 0; c < 64; ++c) {
    w[c] = ldw(src, c);
    alpha = fmaxf(alpha, fabsf(w[c]));
  }
  const uint16_t sb = i4_scale_bits(fmaxf(alpha, eps) / (float)kI4QMax);
  const float s = i4_scale_value(sb);
  uint8_t* blob = packed + (size_t)e * stride + (size_t)mat * i4_matrix_bytes(R, C);  // gate, up, down
#pragma unroll
  for (int gq = 0; gq < 4; ++gq) {
    uint64_t run = 0;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const int c = 16 * gq + 8 * (b >> 2) + (b & 3);
      const int qh = (int)fminf(fmaxf(rintf(w[c] / s), -(float)kI4QMax), (float)kI4QMax);
      const int ql = (int)fminf(fmaxf(rintf(w[c + 4] / s), -(float)kI4QMax), (float)kI4QMax);
      run |= (uint64_t)(((qh & 0xF) << 4) | (ql & 0xF)) << (8 * b);
    }
    *(uint64_t*)(blob + i4_half_run_offset(r, blk, gq, K)) = run;
  }
  *(uint16_t*)(blob + i4_scale_offset(r, blk, rows, K)) = sb;
}

// ---------------------------------------------------------------------------
// Wide packers: sizes in whole 64-column blocks and 16-byte aligned weights.
// A wave works on 16-row x 64-column tiles in the packed operand order (lane l:
// row l%16, columns 16*(l/16) .. +15), so it reads 64 consecutive columns of 16
// rows with 16-byte loads and writes a packed tile as one contiguous kilobyte.
// Two Mixtral experts from bf16, INT8: row maxima 137 us (705 MB) and
// quantization 205 us (1057 MB), both at the rate of a large copy, where one
// element per thread with byte stores took 830 us.  Cutting the work into
// rounds of 48 to 192 MB, whose second read would come from the Infinity Cache,
// was slower (421 to 579 us).  The narrow kernels above take what is left:
// odd sizes and unaligned weights, and most INT4 calls (i4_wide).
// ---------------------------------------------------------------------------
// 16 consecutive weights of one lane as fp32 values.
template <typename WT>
struct W16;
template <>
struct W16<float> {
  v4f q[4];
  __device__ __forceinline__ void load(const float* p) {
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = *(const v4f*)(p + 4 * i);
  }
  __device__ __forceinline__ float get(int i) const { return q[i / 4][i % 4]; }
};
template <>
struct W16<uint16_t> {
  v4i q[2];
  __device__ __forceinline__ void load(const uint16_t* p) {
    q[0] = ld16(p);
    q[1] = ld16(p + 8);
  }
  __device__ __forceinline__ float get(int i) const {
    const uint32_t u = (uint32_t)q[i / 8][(i % 8) / 2];
    return __uint_as_float(i % 2 ? u & 0xFFFF0000u : u << 16);
  }
};

// q = clamp(rint_even(fl32(w / s)), -LIM, LIM) of 16 weights as 16 bytes, bit for
// bit, mostly without the division: t = w * fl32(1/s) is within 3 * 2^-24 |t| of
// w / s and of its rounding, so both round to the same integer unless t lies
// within kTieGap of a half (|t| < LIM + 1/2 <= 127.5: off by at most 2.3e-5).
// Lanes that hold such a t, or one past the limit, or a non-finite one, take
// the division.  t + 1.5 * 2^23 has rint_even(t) in its low mantissa bits.
constexpr float kTieGap = 1.f / 32768.f;
constexpr float kRoundMagic = 12582912.f;

template <int LIM, typename GetW, typename GetS, typename GetR>
__device__ __forceinline__ v4i quant16(GetW w, GetS sc, GetR rcp) {
  uint32_t b[16];
  float far = 0.f, big = 0.f;
  bool fine = true;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const float t = w(i) * rcp(i);
    const float u = t + kRoundMagic;
    b[i] = __float_as_uint(u);
    far = fmaxf(far, fabsf(t - (u - kRoundMagic)));
    big = fmaxf(big, fabsf(t));
    fine = fine && t == t;
  }
  if (!(fine && far < 0.5f - kTieGap && big < (float)LIM + 0.4375f)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      float q = rintf(w(i) / sc(i));
      q = fminf(fmaxf(q, -(float)LIM), (float)LIM);
      b[i] = (uint32_t)(int)q;
    }
  }
  v4i o;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t lo = __builtin_amdgcn_perm(b[4 * j + 1], b[4 * j], 0x0c0c0400u);
    const uint32_t hi = __builtin_amdgcn_perm(b[4 * j + 3], b[4 * j + 2], 0x0c0c0400u);
    o[j] = (int)(lo | (hi << 16));
  }
  return o;
}

__global__ __launch_bounds__(256) void pack_zero_kernel(uint32_t* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0;
}

// amax (pre-zeroed) of expert blockIdx.y.  Blocks x < R/4: a wave of
// gate and up.  The others: 128 rows c of down by a strip of columns, 16 bytes
// of each row per lane.
constexpr int kPackColRows = 128;

template <typename WT>
__global__ __launch_bounds__(256) void pack_max_wide_kernel(const WT* __restrict__ wg,
                                                            const WT* __restrict__ wu,
                                                            const WT* __restrict__ wd, int C, int R,
                                                            uint32_t* __restrict__ amax) {
  wg += (size_t)blockIdx.y * R * C;
  wu += (size_t)blockIdx.y * R * C;
  wd += (size_t)blockIdx.y * R * C;
  amax += (size_t)blockIdx.y * R;
  constexpr int VW = 16 / sizeof(WT);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const auto fold = [](float m, v4i v) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if constexpr (sizeof(WT) == 2) {
        m = fmaxf(m, fabsf(__uint_as_float((uint32_t)v[j] << 16)));
        m = fmaxf(m, fabsf(__uint_as_float((uint32_t)v[j] & 0xFFFF0000u)));
      } else {
        m = fmaxf(m, fabsf(__int_as_float(v[j])));
      }
    }
    return m;
  };
  const int nrow = R / 4;
  if ((int)blockIdx.x < nrow) {
    const int r = blockIdx.x * 4 + wave;
    const WT *g = wg + (size_t)r * C, *u = wu + (size_t)r * C;
    float m = 0.f;
    constexpr int B = 4;
    for (int c0 = lane * VW; c0 < C; c0 += 64 * VW * B) {
      v4i vg[B], vu[B];
#pragma unroll
      for (int b = 0; b < B; ++b) {
        const int c = c0 + 64 * VW * b;
        vg[b] = c < C ? ld16(g + c) : zero16();
        vu[b] = c < C ? ld16(u + c) : zero16();
      }
#pragma unroll
      for (int b = 0; b < B; ++b) m = fold(fold(m, vg[b]), vu[b]);
    }
    m = wave_max(m);
    // non-negative floats order like their bit patterns
    if (lane == 0) atomicMax(&amax[r], __float_as_uint(m));
    return;
  }
  constexpr int COLS = 64 * VW;
  __shared__ float red[4][COLS];
  const int strips = (R + COLS - 1) / COLS;
  const int bi = blockIdx.x - nrow;
  const int strip = bi % strips, c0 = (bi / strips) * kPackColRows + wave * (kPackColRows / 4);
  const int r = strip * COLS + lane * VW;
  const bool in = r < R;
  const int c1 = min(C, c0 + kPackColRows / 4);
  float m[VW];
#pragma unroll
  for (int j = 0; j < VW; ++j) m[j] = 0.f;
  const WT* p = wd + (in ? r : 0);
  for (int c = c0; c < c1; c += 8) {
    v4i v[8];
#pragma unroll
    for (int b = 0; b < 8; ++b) v[b] = c + b < c1 ? ld16(p + (size_t)(c + b) * R) : zero16();
#pragma unroll
    for (int b = 0; b < 8; ++b)
#pragma unroll
      for (int j = 0; j < VW; ++j) {
        float f;
        if constexpr (sizeof(WT) == 2) {
          const uint32_t u = (uint32_t)v[b][j / 2];
          f = __uint_as_float(j % 2 ? u & 0xFFFF0000u : u << 16);
        } else {
          f = __int_as_float(v[b][j]);
        }
        m[j] = fmaxf(m[j], fabsf(f));
      }
  }
#pragma unroll
  for (int j = 0; j < VW; ++j) red[wave][lane * VW + j] = m[j];
  __syncthreads();
  for (int i = threadIdx.x; i < COLS && strip * COLS + i < R; i += 256) {
    const float v = fmaxf(fmaxf(red[0][i], red[1][i]), fmaxf(red[2][i], red[3][i]));
    atomicMax(&amax[strip * COLS + i], __float_as_uint(v));
  }
}

// Quantizes expert blockIdx.y, one wave per unit: 16 column blocks of one tile row
// of gate or up (which also writes the rows' sigma), or 16 tile rows of one column
// block of down.
constexpr int kPackUnitTiles = 16;

template <typename WT>
__global__ __launch_bounds__(256) void pack_quant_wide_kernel(
    const WT* __restrict__ wg, const WT* __restrict__ wu, const WT* __restrict__ wd, int C, int R,
    float eps, const uint32_t* __restrict__ amax, int8_t* __restrict__ packed, uint64_t stride) {
  wg += (size_t)blockIdx.y * R * C;
  wu += (size_t)blockIdx.y * R * C;
  wd += (size_t)blockIdx.y * R * C;
  amax += (size_t)blockIdx.y * R;
  int8_t* blob = packed + (size_t)blockIdx.y * stride;
  const int lane = threadIdx.x & 63, r16 = lane & 15, kg = lane >> 4;
  const int unit = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int nkb = C / 64, kb_units = (nkb + kPackUnitTiles - 1) / kPackUnitTiles;
  const int row_units = 2 * (R / 16) * kb_units;
  constexpr int B = sizeof(WT) == 2 ? 4 : 2;  // tiles in flight
  if (unit < row_units) {
    const int kbu = unit % kb_units, rest = unit / kb_units;
    const int mat = rest & 1, rt = rest >> 1, r = rt * 16 + r16;
    const uint32_t am = amax[r];
    const float sigma = scale_of(am, eps), rc = 1.0f / sigma;
    if (mat == 0 && kbu == 0 && kg == 0)
      ((uint16_t*)(blob + (size_t)3 * R * C))[r] = f32_to_bf16_rne(fmaxf(__uint_as_float(am), eps) / 127.0f);
    const WT* src = (mat == 0 ? wg : wu) + (size_t)r * C + kg * 16;
    int8_t* dst = blob + (size_t)mat * R * C + (size_t)rt * nkb * 1024 + lane * 16;
    const int kb1 = min(nkb, (kbu + 1) * kPackUnitTiles);
    for (int kb = kbu * kPackUnitTiles; kb < kb1; kb += B) {
      W16<WT> w[B];
#pragma unroll
      for (int b = 0; b < B; ++b) w[b].load(src + min(kb + b, kb1 - 1) * 64);
#pragma unroll
      for (int b = 0; b < B; ++b) {
        const v4i q = quant16<127>([&](int i) { return w[b].get(i); }, [&](int) { return sigma; },
                                   [&](int) { return rc; });
        if (kb + b < kb1) *(v4i*)(dst + (size_t)(kb + b) * 1024) = q;
      }
    }
    return;
  }
  // down: the strip's column blocks side by side in a workgroup
  const int du = unit - row_units, nb = R / 64;
  const int nct = C / 16, ct0 = (du / nb) * kPackUnitTiles;
  if (ct0 >= nct) return;
  const int kb = du % nb;
  float sg[16], rc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    sg[i] = scale_of(amax[kb * 64 + kg * 16 + i], eps);
    rc[i] = 1.0f / sg[i];
  }
  const WT* src = wd + (size_t)r16 * R + kb * 64 + kg * 16;
  int8_t* dst = blob + (size_t)2 * R * C + (size_t)kb * 1024 + lane * 16;
  const int ct1 = min(nct, ct0 + kPackUnitTiles);
  for (int ct = ct0; ct < ct1; ct += B) {
    W16<WT> w[B];
#pragma unroll
    for (int b = 0; b < B; ++b) w[b].load(src + (size_t)min(ct + b, ct1 - 1) * 16 * R);
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const v4i q = quant16<127>([&](int i) { return w[b].get(i); }, [&](int i) { return sg[i]; },
                                 [&](int i) { return rc[i]; });
      if (ct + b < ct1) *(v4i*)(dst + (size_t)(ct + b) * (R / 64) * 1024) = q;
    }
  }
}

// INT4 from bf16: a wave per (matrix, tile row, run of column pairs), two
// groups of 64 columns at a time, the group maxima over the four lanes of a
// row.  For large experts (i4_wide).  A wave has one pair's loads in flight, so
// it takes many waves, in short runs of even length: with runs of up to 1 / 2 / 4 /
// 8 pairs, two Mixtral experts take 215 / 204 / 200 / 202 us, three of 4096 x 4096
// 95.4 / 92.4 / 92.8 / 95.5, four of 4096 x 4096 - / 120 / 120 / 122.
constexpr int kPackI4Run = 2;

__global__ __launch_bounds__(256) void pack_i4_wide_kernel(const uint16_t* __restrict__ wg,
                                                           const uint16_t* __restrict__ wu,
                                                           const uint16_t* __restrict__ wd, int C,
                                                           int R, float eps,
                                                           uint8_t* __restrict__ packed,
                                                           uint64_t stride) {
  const int mat = blockIdx.y, e = blockIdx.z;
  const int rows = mat == 2 ? C : R, K = mat == 2 ? R : C;
  const int lane = threadIdx.x & 63, r16 = lane & 15, kg = lane >> 4;
  const int npair = K / 128, runs = (npair + kPackI4Run - 1) / kPackI4Run;
  const int unit = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int rt = unit / runs, part = unit % runs;
  if (rt >= rows / 16) return;
  const uint16_t* src = (mat == 0 ? wg : mat == 1 ? wu : wd) + (size_t)e * R * C +
                        (size_t)(rt * 16 + r16) * K + kg * 16;
  uint8_t* m = packed + (size_t)e * stride + (size_t)mat * i4_matrix_bytes(R, C);
  const int p0 = part * npair / runs, p1 = (part + 1) * npair / runs;
  for (int p = p0; p < p1; ++p) {
    W16<uint16_t> w[2];
    w[0].load(src + p * 128);
    w[1].load(src + p * 128 + 64);
    v4i run;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float alpha = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) alpha = fmaxf(alpha, fabsf(w[h].get(i)));
      alpha = fmaxf(alpha, __shfl_xor(alpha, 16, 64));
      alpha = fmaxf(alpha, __shfl_xor(alpha, 32, 64));
      const uint16_t sb = i4_scale_bits(fmaxf(alpha, eps) / (float)kI4QMax);
      const float s = i4_scale_value(sb), rc = 1.0f / s;
      const v4i q = quant16<kI4QMax>([&](int i) { return w[h].get(i); }, [&](int) { return s; },
                                     [&](int) { return rc; });
      // bytes of columns 0-3 and 4-7 (8-11 and 12-15) to high and low nibbles
      run[2 * h] = (int)((((uint32_t)q[0] << 4) & 0xF0F0F0F0u) | ((uint32_t)q[1] & 0x0F0F0F0Fu));
      run[2 * h + 1] = (int)((((uint32_t)q[2] << 4) & 0xF0F0F0F0u) | ((uint32_t)q[3] & 0x0F0F0F0Fu));
      if (kg == 0) *(uint16_t*)(m + i4_scale_offset(rt * 16 + r16, 2 * p + h, rows, K)) = sb;
    }
    *(v4i*)(m + ((size_t)rt * npair + p) * kI4PairTile + lane * 16) = run;
  }
}

static bool wide_ok(int C, int R, const void* wg, const void* wu, const void* wd) {
  return C % 64 == 0 && R % 64 == 0 && ((uintptr_t)wg | (uintptr_t)wu | (uintptr_t)wd) % 16 == 0;
}

// Whether n INT4 experts from bf16 take whole tiles (pack_i4_wide_kernel) and not
// a thread per group (pack_i4_kernel).  The latter writes a packed tile from 16
// rows that are C/64 (gate, up) threads apart, so it loses with long rows; whole
// tiles need enough of them to fill the chip.  us, a thread per group / whole
// tiles, of n experts C x R:
//   4096 x 4096: n 1 35.5 / 36.8, 2 66.5 / 64.5, 3 98.2 / 92.3
//   2560 x 6144: n 1 32.8 / 35.1, 2 62.2 / 61.2, 3 91 / 87    2688 x 1152, 13: 75.9 / 78.3
//   2048 x 8320, 6: 188 / 181    2048 x 2048, 17: 118 / 127    8192 x 2048, 2: 70.1 / 64.4
//   2944 x 1280, 14: 98.9 / 98.5    2048 x 1408, 60: 286 / 315    512 x 15232, 18: 248 / 245
// Over 90 random shapes (C 512 to 8192, R 256 to 16384, 4 * 10^7 to 4.5 * 10^8
// weights) no call that the rule sends to whole tiles was slower for it, the
// largest 1.35 times as fast; of the others some would gain (4736 x 896, 27
// experts: 223 / 208).  From fp32 a thread per group already reads at the copy
// rate and is 5% ahead.
static bool i4_wide(int C, int R, int n) {
  const double per = (double)C * R, all = 3 * per * n;
  return per >= 5e6 && all >= 7e7 && all * C >= 4.1e11;
}

template <typename WT>
static void launch_pack_wide(int C, int R, int n, const WT* wg, const WT* wu, const WT* wd, float eps,
                             int8_t* packed, uint64_t stride, uint32_t* amax, hipStream_t st) {
  const int64_t na = (int64_t)n * R;
  hipLaunchKernelGGL(pack_zero_kernel, dim3((unsigned)((na + 255) / 256)), dim3(256), 0, st, amax, na);
  constexpr int cols = 64 * (16 / (int)sizeof(WT));
  const int mblocks = R / 4 + (R + cols - 1) / cols * ((C + kPackColRows - 1) / kPackColRows);
  hipLaunchKernelGGL(pack_max_wide_kernel<WT>, dim3(mblocks, n), dim3(256), 0, st, wg, wu, wd, C, R, amax);
  const int nkb = C / 64, nct = C / 16;
  const int units = 2 * (R / 16) * ((nkb + kPackUnitTiles - 1) / kPackUnitTiles) +
                    R / 64 * ((nct + kPackUnitTiles - 1) / kPackUnitTiles);
  hipLaunchKernelGGL(pack_quant_wide_kernel<WT>, dim3((units + 3) / 4, n), dim3(256), 0, st, wg, wu, wd, C,
                     R, eps, (const uint32_t*)amax, packed, stride);
}

hipError_t launch_pack_i4(int C, int R, int n, int w_dtype, const void* wg, const void* wu,
                          const void* wd, float eps, void* packed, uint64_t stride,
                          hipStream_t st) {
  if (n == 0) return hipSuccess;
  prof_begin("pack", st);
  const int64_t items = (int64_t)R * (C / 64);  // rows x groups, the same for all three matrices
  const dim3 grid((unsigned)((items + 255) / 256), 3, n);
  if (w_dtype == MIRA_BF16 && i4_wide(C, R, n) && wide_ok(C, R, wg, wu, wd)) {
    // tile rows x runs of column pairs, the larger of gate's and down's
    const auto waves = [](int rows, int K) {
      return (int64_t)(rows / 16) * ((K / 128 + kPackI4Run - 1) / kPackI4Run);
    };
    const int64_t units = waves(R, C) > waves(C, R) ? waves(R, C) : waves(C, R);
    hipLaunchKernelGGL(pack_i4_wide_kernel, dim3((unsigned)((units + 3) / 4), 3, n), dim3(256), 0, st,
                       (const uint16_t*)wg, (const uint16_t*)wu, (const uint16_t*)wd, C, R, eps,
                       (uint8_t*)packed, stride);
  } else if (w_dtype == MIRA_BF16)
    hipLaunchKernelGGL(pack_i4_kernel<uint16_t>, grid, dim3(256), 0, st, (const uint16_t*)wg,
                       (const uint16_t*)wu, (const uint16_t*)wd, C, R, eps, (uint8_t*)packed, stride);
  else
    hipLaunchKernelGGL(pack_i4_kernel<float>, grid, dim3(256), 0, st, (const float*)wg,
                       (const float*)wu, (const float*)wd, C, R, eps, (uint8_t*)packed, stride);
  const uint64_t used = 2 * i4_matrix_bytes(R, C) + i4_matrix_bytes(C, R);
  if (stride > used)
    hipLaunchKernelGGL(pack_pad_kernel, dim3(64, n), dim3(256), 0, st, (int8_t*)packed, stride, used);
  prof_end("pack", st);
  return hipGetLastError();
}

hipError_t launch_pack(int C, int R, int n, int w_dtype, const void* wg, const void* wu,
                       const void* wd, float eps, void* packed, uint64_t stride, hipStream_t st) {
  if (n == 0) return hipSuccess;
  // fp32 row maxima alpha_r live in a stream-ordered temporary allocation
  // (packing is offline; the forward path never allocates).
  uint32_t* amax = nullptr;
  hipError_t err = hipMallocAsync((void**)&amax, (size_t)n * R * 4, st);
  if (err != hipSuccess) return err;
  prof_begin("pack", st);
  const int c_chunk = 256;
  if (wide_ok(C, R, wg, wu, wd)) {
    if (w_dtype == MIRA_BF16)
      launch_pack_wide(C, R, n, (const uint16_t*)wg, (const uint16_t*)wu, (const uint16_t*)wd, eps,
                       (int8_t*)packed, stride, amax, st);
    else
      launch_pack_wide(C, R, n, (const float*)wg, (const float*)wu, (const float*)wd, eps,
                       (int8_t*)packed, stride, amax, st);
  } else if (w_dtype == MIRA_BF16) {
    const uint16_t *g = (const uint16_t*)wg, *u = (const uint16_t*)wu, *d = (const uint16_t*)wd;
    hipLaunchKernelGGL(pack_rowmax_kernel<uint16_t>, dim3((R + 3) / 4, n), dim3(256), 0, st, g, u,
                       C, R, amax);
    hipLaunchKernelGGL(pack_colmax_kernel<uint16_t>, dim3((R + 255) / 256, (C + c_chunk - 1) / c_chunk, n),
                       dim3(256), 0, st, d, C, R, c_chunk, amax);
    hipLaunchKernelGGL(pack_quant_rows_kernel<uint16_t>, dim3(R, 2, n), dim3(256), 0, st, g, u, C,
                       R, eps, amax, (int8_t*)packed, stride);
    hipLaunchKernelGGL(pack_quant_down_kernel<uint16_t>, dim3((R + 255) / 256, C, n), dim3(256), 0,
                       st, d, C, R, eps, amax, (int8_t*)packed, stride);
  } else {
    const float *g = (const float*)wg, *u = (const float*)wu, *d = (const float*)wd;
    hipLaunchKernelGGL(pack_rowmax_kernel<float>, dim3((R + 3) / 4, n), dim3(256), 0, st, g, u, C,
                       R, amax);
    hipLaunchKernelGGL(pack_colmax_kernel<float>, dim3((R + 255) / 256, (C + c_chunk - 1) / c_chunk, n),
                       dim3(256), 0, st, d, C, R, c_chunk, amax);
    hipLaunchKernelGGL(pack_quant_rows_kernel<float>, dim3(R, 2, n), dim3(256), 0, st, g, u, C, R,
                       eps, amax, (int8_t*)packed, stride);
    hipLaunchKernelGGL(pack_quant_down_kernel<float>, dim3((R + 255) / 256, C, n), dim3(256), 0,
                       st, d, C, R, eps, amax, (int8_t*)packed, stride);
  }
  const uint64_t used = (uint64_t)3 * R * C + (uint64_t)2 * R;
  if (stride > used)
    hipLaunchKernelGGL(pack_pad_kernel, dim3(64, n), dim3(256), 0, st, (int8_t*)packed, stride, used);
  prof_end("pack", st);
  err = hipGetLastError();
  hipError_t e2 = hipFreeAsync(amax, st);
  return err != hipSuccess ? err : e2;
}

}  // namespace mira
