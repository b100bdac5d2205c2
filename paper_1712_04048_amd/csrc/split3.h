// fp32 products on the bf16 matrix cores.
//
// An fp32 value is the exact sum of three bf16 values (24 bits of mantissa =
// 3 x 8; each part is the bf16 rounding of what the ones before leave), so a
// product of two fp32 values is the sum of nine bf16 products, each exact in
// fp32.  Six of them are formed, smallest first,
//   a3 b1 + a1 b3 + a2 b2 + a2 b1 + a1 b2 + a1 b1,
// and the other three (a2 b3, a3 b2, a3 b3) are together at most 2^-24 of the
// product, 2^-27.4 in the mean square: as large at worst as fp32's own rounding
// of it, a tenth of that as a rule.  The sums are fp32 either way, with a
// rounding per 32-deep step and term instead of one per 4-deep step, and it is
// those roundings that make the error: with eight or all nine products the
// gradients of every measured batch are as far from 64 bits as with six (1 %),
// and both are as close as the fp32 instruction's or closer (see the kernels
// that use it; db, whose errors are those of dA added up, is 1.1e-7 against
// 1.0e-7 on the SST batch).  Six 16x16x32 bf16 instructions take 96 cycles
// where eight 16x16x4 fp32 ones take 256, so the ceiling is 2.5 PFLOP/s / 6 =
// 416 TFLOP/s instead of 157.
//
// The parts hold values from about 2^-110 (smaller ones lose their last parts
// below bf16's range: what is lost is under 2^-133) up to bf16's largest,
// 3.39e38.  Of a larger value or an infinity the first part is infinite and
// the last NaN, so every output that it enters is NaN: a workgroup that finds
// a NaN in its tile forms the tile again on the fp32 instruction, as if nothing
// had been split (looking for such operands as they are split took 6 % of the
// products' time, looking at the outputs 1 to 3 %).
//
// The operands are split once per workgroup, on their way from registers to
// LDS (5.5 VALU instructions a value).
#pragma once

#include "kernels.h"

namespace cavs {

// The largest magnitude that bf16 rounds to a finite value, and that value.
constexpr float kSplitTop = 0x1.fefffep127f, kBf16Max = 0x1.fep127f;

// What has no parts (see above) at bf16's largest value: for operands whose
// infinities only have to saturate a gate.
__device__ __forceinline__ float split_clamp(float v) {
  return fabsf(v) > kSplitTop ? copysignf(kBf16Max, v) : v;
}

// eight fp32 values as three bf16 fragments
struct Split8 {
  uint4 p[3];
};
__device__ __forceinline__ Split8 split8(const float (&v)[8]) {
  Split8 s;
  uint32_t q[3][4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const f32x2 x{v[2 * e], v[2 * e + 1]};
    const bf16x2 h = __builtin_convertvector(x, bf16x2);
    const f32x2 r = x - __builtin_convertvector(h, f32x2);
    const bf16x2 m = __builtin_convertvector(r, bf16x2);
    const f32x2 l = r - __builtin_convertvector(m, f32x2);
    q[0][e] = __builtin_bit_cast(uint32_t, h);
    q[1][e] = __builtin_bit_cast(uint32_t, m);
    q[2][e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(l, bf16x2));
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) s.p[k] = make_uint4(q[k][0], q[k][1], q[k][2], q[k][3]);
  return s;
}

// The terms of the product, smallest first: operand parts (a, b).
constexpr int kSplitTerms = 6;
__device__ constexpr int kTermA[kSplitTerms] = {2, 0, 1, 1, 0, 0};
__device__ constexpr int kTermB[kSplitTerms] = {0, 2, 1, 0, 1, 0};

// One operand's LDS tile: three planes of 128 rows of 32 bf16 (64 bytes),
// the four 16-byte quads of row x at quad ^ ((x >> 2) & 3): sixteen lanes on
// sixteen rows of one quad then fall in different banks, reading and writing.
// LDS row 32 j + i holds tile row 4 i + j, so that the thread that loaded
// four adjacent columns of a k-major operand writes rows 32 apart (its
// neighbours the rows between) and a lane of the product holds four adjacent
// outputs.
constexpr int kX3Tile = 128;
constexpr int kX3Plane = kX3Tile * 64;     // bytes
constexpr int kX3Bytes = 3 * kX3Plane;     // one operand

__device__ __forceinline__ int x3_addr(int row, int quad) {
  return row * 64 + ((quad ^ ((row >> 2) & 3)) << 4);
}
// PARTS = 1: bf16 products, the operand rounded (one plane).  PARTS = 0: fp32,
// rows of 128 bytes, no swizzle (x3_mma_f32; 16 KB of the operand's 24).
template <int PARTS = 3>
__device__ __forceinline__ void x3_store(char* lds, int row, int quad, const float (&v)[8]) {
  const int a = x3_addr(row, quad);
  if constexpr (PARTS == 0) {
    float4* d = reinterpret_cast<float4*>(lds + row * 128 + quad * 32);
    d[0] = make_float4(v[0], v[1], v[2], v[3]);
    d[1] = make_float4(v[4], v[5], v[6], v[7]);
  } else if constexpr (PARTS == 1) {
    *reinterpret_cast<uint4*>(lds + a) = make_uint4(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]),
                                                    f2bf2(v[4], v[5]), f2bf2(v[6], v[7]));
  } else {
    const Split8 s = split8(v);
#pragma unroll
    for (int p = 0; p < 3; ++p) *reinterpret_cast<uint4*>(lds + p * kX3Plane + a) = s.p[p];
  }
}

// acc[j][c] += the 32-deep products of the wavefront's blocks: A blocks j are
// LDS rows 32 j + 16 wm + r, B blocks c rows 32 c + 16 wn + r.  Lane (r, g),
// element i of acc[j][c] is tile row 64 wm + 16 g + 4 i + j, column
// 64 wn + 4 r + c.
// BLOCKS: the row blocks j that are wanted (bit j).  APART: the six terms of a
// chunk are summed on their own first, so that a long chain rounds at the size
// of its total once per chunk instead of six times (a third less error; the
// six dependent instructions cost 2 to 4 % of the lazy products).
template <int PARTS = 3, int BLOCKS = 15, bool APART = false>
__device__ __forceinline__ void x3_mma(const char* As, const char* Bs, int wm, int wn,
                                       v4f (&acc)[4][4]) {
  constexpr int TERMS = PARTS == 1 ? 1 : kSplitTerms;
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  bf16x8 b[PARTS][4];
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int p = 0; p < PARTS; ++p)
      b[p][c] = *reinterpret_cast<const bf16x8*>(Bs + p * kX3Plane + x3_addr(32 * c + 16 * wn + r, g));
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (!(BLOCKS >> j & 1)) continue;
    bf16x8 a[PARTS];
#pragma unroll
    for (int p = 0; p < PARTS; ++p)
      a[p] = *reinterpret_cast<const bf16x8*>(As + p * kX3Plane + x3_addr(32 * j + 16 * wm + r, g));
    if constexpr (APART) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        v4f s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < TERMS; ++t) s = mfma_bf16_16x16x32(a[kTermA[t]], b[kTermB[t]][c], s);
        acc[j][c] += s;
        __builtin_amdgcn_sched_barrier(0);   // or four sums' registers spill
      }
      continue;
    }
#pragma unroll
    for (int t = 0; t < TERMS; ++t)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        acc[j][c] = mfma_bf16_16x16x32(a[PARTS == 1 ? 0 : kTermA[t]],
                                       b[PARTS == 1 ? 0 : kTermB[t]][c], acc[j][c]);
  }
}

// The same outputs from fp32 tiles (PARTS = 0) on the fp32 instruction.
// x3_nan: the tile of this workgroup holds a NaN (a barrier).
__device__ __forceinline__ bool x3_nan(const v4f (&acc)[4][4]) {
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) s += acc[j][c][e];
  return __builtin_expect(__syncthreads_or(s != s), 0);
}
// x3_again hides a thread index from the compiler, so that what the second
// pass derives from it is formed again instead of kept in registers meanwhile.
__device__ __forceinline__ int x3_again(int t) {
  asm volatile("" : "+v"(t));
  return t;
}
__device__ __forceinline__ void x3_mma_f32(const char* As, const char* Bs, int wm, int wn,
                                           v4f (&acc)[4][4]) {
  const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  auto frag = [&](const char* L, int row, float (&f)[8]) {
    const float4* q = reinterpret_cast<const float4*>(L + row * 128 + g * 32);
    const float4 x = q[0], y = q[1];
    f[0] = x.x; f[1] = x.y; f[2] = x.z; f[3] = x.w;
    f[4] = y.x; f[5] = y.y; f[6] = y.z; f[7] = y.w;
  };
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float a[8];
    frag(As, 32 * j + 16 * wm + r, a);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      float b[8];
      frag(Bs, 32 * c + 16 * wn + r, b);
#pragma unroll
      for (int s = 0; s < 8; ++s) acc[j][c] = mfma_f32_16x16x4(a[s], b[s], acc[j][c]);
    }
  }
}

}  // namespace cavs
