// Pieces of the GEMM kernels: the order of the tiles, direct loads into LDS; and of the small-tile ones: operand order,
// the multiply-and-fold pipeline of one 32 x 32 sub-tile, stores of a sub-tile.
#pragma once
#include "fq_device.h"
#include "fq_kernels.h"

namespace fq {
namespace {

constexpr int kXcds = 8;          // accelerator complex dies, each with a private L2
constexpr int kFragRows = 4096;   // bytes of one 32-row group of a block (128 contraction positions)

// Row (of the 32 in a group) that lane i of operand half ch = 0, 1 supplies.  The result registers
// of lane group g = i / 4 are 4 consecutive operand rows; with this order the two halves give a lane
// 8 consecutive columns of C, columns 8 g + 4 ch' ..., and both the first 8 and the 16 lanes of an
// LDS read fall into distinct banks (ch' = ch or 1 - ch by g, which store_unit undoes).
__device__ __forceinline__ int perm_col(int i, int ch) {
  const int g = i >> 2;
  const int sigma = (g ^ (g >> 1)) & 1;        // 0, 1, 1, 0
  return 8 * g + 4 * (ch ^ sigma) + (i & 3);
}

// 16 columns x 16 rows x 64: lane l supplies operand row l % 16 and contraction bytes of group l / 16.
__device__ __forceinline__ v4i mfma16(const v4i& b, const v4i& a, const v4i& c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(b, a, c, 0, 0, 0);
}

// Writes a lane's 16 values of a 32 x 32 sub-tile: element 4 q + r, quadrant q = 2 ch + rh (column half
// ch, row half rh).  bad: a flagged block of these rows found no residual slot, the rows become NaN.
__device__ __forceinline__ void store_unit(const GemmParams& p, const float (&acc)[16], int row0, int col0,
                                           int lane, bool bad) {
  const int g = lane >> 4;
  const bool swap = ((g ^ (g >> 1)) & 1) != 0;
  const int col = col0 + 8 * g;
#pragma unroll
  for (int rh = 0; rh < 2; ++rh) {
    const int row = row0 + 16 * rh + (lane & 15);
    float v[8];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float x = acc[4 * rh + r], y = acc[8 + 4 * rh + r];   // quadrants (ch 0, rh), (ch 1, rh)
      v[r] = bad ? __int_as_float(0x7FC00000) : (swap ? y : x);
      v[4 + r] = bad ? __int_as_float(0x7FC00000) : (swap ? x : y);
    }
    if (row >= p.M || col >= p.N) continue;
    if (p.out_bf16) {
      uint16_t* dst = reinterpret_cast<uint16_t*>(p.c) + (int64_t)row * p.ldc + col;
      if (p.vec_ok && col + 8 <= p.N) {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        v4i o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          f32x2 t = {v[2 * i], v[2 * i + 1]};
          o[i] = __builtin_bit_cast(int, __builtin_convertvector(t, bf16x2));
        }
        *reinterpret_cast<v4i*>(dst) = o;
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (col + e < p.N) dst[e] = (uint16_t)float_to_bf16_bits(v[e]);
      }
    } else {
      float* dst = reinterpret_cast<float*>(p.c) + (int64_t)row * p.ldc + col;
      if (p.vec_ok && col + 8 <= p.N) {
        reinterpret_cast<float4*>(dst)[0] = make_float4(v[0], v[1], v[2], v[3]);
        reinterpret_cast<float4*>(dst)[1] = make_float4(v[4], v[5], v[6], v[7]);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (col + e < p.N) dst[e] = v[e];
      }
    }
  }
}

// Workgroup b of `total` -> its place in the tile order: workgroups are dealt to the XCDs round-robin,
// so each XCD gets a contiguous run of tiles, whose B blocks then come through one L2.
__device__ __forceinline__ int xcd_run(int b, int total) {
  const int xcd = b % kXcds, l = b / kXcds;
  const int q = total / kXcds, rem = total % kXcds;
  return xcd * q + min(xcd, rem) + l;
}

// Place L of the tile order -> tile: groups of kGroupN tile columns, walked row by row.
template <int kGroupN>
__device__ __forceinline__ void tile_at(int L, int tiles_i, int tiles_j, int& ti, int& tj) {
  const int group = kGroupN * tiles_i;
  const int g0 = (L / group) * kGroupN;
  const int gn = min(kGroupN, tiles_j - g0);
  const int within = L - (L / group) * group;
  tj = g0 + within % gn;
  ti = within / gn;
}

// Empty volatile asm statements that take values as read-write register operands.  The
// compiler may not reorder volatile asm, so the instructions producing the operands stay
// before the statement and their consumers after it: this pins the source order of otherwise
// freely movable pure instructions (MFMA, convert, FMA) without emitting any code.
__device__ __forceinline__ void pin(v4i& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void pin(float& a, float& b) { asm volatile("" : "+v"(a), "+v"(b)); }

// One unit: a 32 x 32 sub-tile of one k-block.  kPar: parity of the unit in the wavefront's sequence of
// units.  Multiplies a with b into P[kPar] and folds the finished tile P[kPar ^ 1] of the unit before
// it into `acc` with the scale f of that unit: per slot one MFMA, the two FMAs of the elements
// converted in the slot before, two converts.  extra(n) adds slot n's loads.
template <int kPar, class Extra>
__device__ __forceinline__ void unit(v4i (&P)[2][4], const v4i (&b)[2][2], float (&acc)[16], const v4i (&a)[2][2],
                                     float f, const Extra& extra) {
  float T[2] = {0.0f, 0.0f};
#pragma unroll
  for (int n = 0; n < 8; ++n) {
    const int ks = n >> 2, q = n & 3, ch = q >> 1, rh = q & 1;
    const v4i z = {0, 0, 0, 0};
    P[kPar][q] = mfma16(b[ch][ks], a[rh][ks], ks ? P[kPar][q] : z);
    extra(n);
    pin(P[kPar][q]);
    __builtin_amdgcn_sched_barrier(0);
    if (n > 0) {
      acc[2 * n - 2] = __builtin_fmaf(T[0], f, acc[2 * n - 2]);
      acc[2 * n - 1] = __builtin_fmaf(T[1], f, acc[2 * n - 1]);
      pin(acc[2 * n - 2], acc[2 * n - 1]);
      __builtin_amdgcn_sched_barrier(0);
    }
    T[0] = (float)P[kPar ^ 1][n >> 1][2 * (n & 1)];
    T[1] = (float)P[kPar ^ 1][n >> 1][2 * (n & 1) + 1];
    pin(T[0], T[1]);
    __builtin_amdgcn_sched_barrier(0);
  }
  acc[14] = __builtin_fmaf(T[0], f, acc[14]);
  acc[15] = __builtin_fmaf(T[1], f, acc[15]);
  pin(acc[14], acc[15]);
}

typedef __attribute__((address_space(3))) void lds_void;

// Address of a __shared__ object as the LDS instructions take it.
__device__ __forceinline__ uint32_t lds_address(const void* q) { return (uint32_t)(uintptr_t)(lds_void*)q; }

// Direct global -> LDS loads as assembly, without register results (the compiler would turn every wait for
// an LDS read into a wait for all of them).  kN KiB from src, wave-uniform, to dst.  The block keeps the
// wait states its loads need by itself: the second move is the one between a write to m0 and its use, and
// leaves the base written by the scalar unit, whatever wrote it before.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"     // that m0 is a register nobody keeps values in is known
template <int kN>
__device__ __forceinline__ void load_lds(const int8_t* src, uint32_t dst, int lane) {
  static_assert(kN >= 1 && kN <= 4);
  const unsigned voff = (unsigned)lane * 16u;
  const uint64_t addr = reinterpret_cast<uint64_t>(src);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)addr);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(addr >> 32));
  uint64_t base = ((uint64_t)hi << 32) | lo;
  const uint32_t to = __builtin_amdgcn_readfirstlane(dst);
#define FQ_LOAD "global_load_lds_dwordx4 %2, %0"
  if constexpr (kN == 1)
    asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %0\n\t" FQ_LOAD : "+s"(base) : "s"(to), "v"(voff) : "memory", "m0");
  else if constexpr (kN == 2)
    asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %0\n\t" FQ_LOAD "\n\t" FQ_LOAD " offset:1024"
                 : "+s"(base) : "s"(to), "v"(voff) : "memory", "m0");
  else if constexpr (kN == 3)
    asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %0\n\t" FQ_LOAD "\n\t" FQ_LOAD " offset:1024\n\t" FQ_LOAD
                 " offset:2048" : "+s"(base) : "s"(to), "v"(voff) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %0\n\t" FQ_LOAD "\n\t" FQ_LOAD " offset:1024\n\t" FQ_LOAD
                 " offset:2048\n\t" FQ_LOAD " offset:3072" : "+s"(base) : "s"(to), "v"(voff) : "memory", "m0");
#undef FQ_LOAD
}
// A dword per lane from base + off to dst + 4 lane.
__device__ __forceinline__ void load_lds_dword(const void* from, unsigned off, uint32_t dst) {
  const uint64_t addr = reinterpret_cast<uint64_t>(from);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)addr);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(addr >> 32));
  uint64_t base = ((uint64_t)hi << 32) | lo;
  const uint32_t to = __builtin_amdgcn_readfirstlane(dst);
  asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %0\n\tglobal_load_lds_dword %2, %0"
               : "+s"(base) : "s"(to), "v"(off) : "memory", "m0");
}
#pragma clang diagnostic pop

}  // namespace
}  // namespace fq
