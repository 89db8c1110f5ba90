// Fused block quantizer: abs-max, INT8 codes, fallback decision, residual
// quantization, slot allocation and the compact list of flagged blocks in one
// kernel launch, one pass over the bf16 input.
//
// Paper: Sec. 3.1 (a = max|G|/127, Q^ = round(G/a); round-to-nearest or, for gradients and
// stored contexts, stochastic rounding, Sec. 5.1), Sec. 4.4
// (u = [max|G| > theta]), Sec. 4.3 (second step on the residual G - a Q^),
// Sec. 5.3 (the fallback decision is fused into the quantization kernel).
//
// One 512-thread workgroup owns one 128x128 block (32 KiB of bf16).  Thread t holds 4 consecutive rows
// x 8 consecutive columns in registers: rows 4 (t/16) ..., columns 8 (t%16) ....  A row of the block
// is then 16 lanes x 16 bytes of one load, and the 4 x 8 codes give whole dwords of the block and of
// its transpose, which reach tile order through an LDS image each and leave as 16-byte stores.
#include <type_traits>

#include "fq_device.h"
#include "fq_kernels.h"

namespace fq {

namespace {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kRows = 4, kCols = 8;      // of a thread

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// max of the wavefront's values (bit patterns of non-negative floats, which order like integers)
__device__ inline uint32_t wave_max(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true));    // lane ^ 1
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true));    // lane ^ 2
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true));   // 7 - lane (of 8)
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true));   // 15 - lane
  const uint32_t a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
  const uint32_t c = __builtin_amdgcn_readlane(v, 32), d = __builtin_amdgcn_readlane(v, 48);
  return max(max(a, b), max(c, d));
}

// max over the workgroup, every thread gets it.  red: kWaves words of LDS that no earlier call in
// flight uses (one barrier).
__device__ inline float block_max(uint32_t v, uint32_t* red) {
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  uint32_t m = red[0];
#pragma unroll
  for (int i = 1; i < kWaves; ++i) m = max(m, red[i]);
  return __uint_as_float(m);
}

// sums of two binary64 values over the workgroup; every thread gets both.  red: 2 kWaves doubles.
__device__ inline void block_sum2(double& a, double& b, double* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    a += __shfl_xor(a, off, 64);
    b += __shfl_xor(b, off, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = a;
    red[kWaves + (threadIdx.x >> 6)] = b;
  }
  __syncthreads();
  a = b = 0.0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) {
    a += red[i];
    b += red[kWaves + i];
  }
}

// Philox4x32-10 (Salmon et al., SC'11): counter (c0, c1, 0, 0), key (k0, k1).
__device__ inline void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t k0, uint32_t k1,
                                     uint32_t (&out)[4]) {
  uint32_t c2 = 0, c3 = 0;
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    // one 32 x 32 -> 64-bit multiplication per product (a single instruction on this target)
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t h0 = (uint32_t)(p0 >> 32), l0 = (uint32_t)p0;
    const uint32_t h1 = (uint32_t)(p1 >> 32), l1 = (uint32_t)p1;
    c0 = h1 ^ c1 ^ k0;
    c1 = l1;
    c2 = h0 ^ c3 ^ k1;
    c3 = l0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// A thread's 4 x 8 input values stay in the packed bf16 form they were loaded in (two per dword, low
// half first) and its codes in packed bytes (two dwords per row): half the registers of floats, which
// is what lets a compute unit hold four workgroups.
__device__ inline float x_at(const v4i (&raw)[kRows], int r, int e) {
  const uint32_t w = (uint32_t)raw[r][e >> 1];
  return __uint_as_float((e & 1) ? (w & 0xFFFF0000u) : (w << 16));
}
__device__ inline int code_at(const u32x2 (&q)[kRows], int r, int e) {
  return (int)(int8_t)(q[r][e >> 2] >> (8 * (e & 3)));
}

// Makes the packed inputs opaque to the optimizer at this point, so that values unpacked before it
// are not kept alive across it (they are cheap to unpack again); emits no code.
__device__ __forceinline__ void forget_unpacked(v4i (&raw)[kRows]) {
#pragma unroll
  for (int r = 0; r < kRows; ++r) asm volatile("" : "+v"(raw[r]));
}
__device__ __forceinline__ void forget_unpacked(u32x2 (&q)[kRows]) {
#pragma unroll
  for (int r = 0; r < kRows; ++r) asm volatile("" : "+v"(q[r]));
}

// Byte 2 of four dwords as one dword.
__device__ __forceinline__ uint32_t pack_byte2(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  const uint32_t lo = __builtin_amdgcn_perm(b, a, 0x0C0C0602u), hi = __builtin_amdgcn_perm(d, c, 0x06020C0Cu);
  return lo | hi;
}

// The scale of a block and what round-to-nearest needs of it: r16 = 2^16 / a.
struct Scale {
  float a, r16;
};
__device__ inline Scale make_scale(float amax) {
  Scale s;
  s.a = __fdiv_rn(amax, 127.0f);
  // A zero block takes code 0 everywhere.  Where the reciprocal or the products with it could leave
  // the normal range NaN sends every element down the exact path.
  s.r16 = s.a == 0.0f ? 0.0f
          : (s.a >= 0x1p-100f && s.a <= 0x1p100f) ? __fdiv_rn(1.0f, s.a) * 65536.0f : __int_as_float(0x7FC00000);
  return s;
}

// Exact quotient RN(x / a) without a division: r = RN(1 / a), and two residual corrections (the second
// starts from a faithful quotient, which makes the result the correctly rounded one).  For a in
// [2^-100, 2^100] and quotients of 2^-1 and more, which is what rounding to nearest needs.  A product of
// quotient and scale below about 2^-103 leaves a residual that underflows, so at a = 2^-90, where the
// stochastic rounding stops taking it, quotients below 2^-13 can be off by their last bit: over all pairs
// of a bf16 value and a bf16 maximum this happens to 2 in 1000, and to none does it change which 24-bit
// random numbers round up.
__device__ __forceinline__ float exact_quotient(float x, float a, float r) {
  float q = x * r;
  q = __builtin_fmaf(__builtin_fmaf(-q, a, x), r, q);
  return __builtin_fmaf(__builtin_fmaf(-q, a, x), r, q);
}

// The whole part of v, for 0 <= v < 2^32; 0 for a NaN.  The instruction is named because a C++
// conversion leaves a NaN's result open, and quantize_rows finds its NaNs by that 0.
__device__ __forceinline__ uint32_t whole_part(float v) {
  uint32_t u;
  asm("v_cvt_u32_f32 %0, %1" : "=v"(u) : "v"(v));
  return u;
}

// codes[r] = rint(RN(x / a)) of the thread's values x = val(r, e), packed bytes, two's complement.
// One fused multiply-add puts x / a + 128.5 into fixed point with 16 fraction bits (y): byte 2 is
// the rounded quotient + 128, the low half says how far the quotient is from a half-integer.  In
// units of 2^-16: the reciprocal is off by at most 0.5, the sum by 0.5, the binary32 rounding of the
// true quotient by 0.25, so with 2 added to y a low half of 4 or more leaves no doubt.  Otherwise (or
// with r16 = NaN) the row of 8 is done again with the exact quotient: 4.75 vector instructions per value
// and no branch but one per 8 values, where testing and branching per value took more than twice that.
// A doubt is no rare thing: quotients of bf16 values and a bf16 maximum lie on a coarse grid.  Of N(0, 1)
// values 6 in 1000 are that near a half-integer, and half of a wavefront's rows hold one; where
// the block's maximum is a power of two all do.  So the second time divides no more than it has to: a
// scale that has a reciprocal takes two residual corrections per value (no rounded code depends on which of
// the two it was, over all pairs of a bf16 value and a bf16 maximum), the others divide and clamp (a
// subnormal scale can be far from max/127).  With 8 divisions 4096 x 4096 of N(0, 1) without fallback took
// 14.4 instead of 11.8 us, 8192 x 8192 with every block flagged 83 instead of 74.5.
template <class F>
__device__ __forceinline__ void quantize_rows(const F& val, const Scale& s, u32x2 (&codes)[kRows]) {
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    uint32_t y[kCols];
    u16x2 near = {0xFFFF, 0xFFFF};
#pragma unroll
    for (int e = 0; e < kCols; ++e) {
      y[e] = whole_part(__builtin_fmaf(val(r, e), s.r16, 128.5f * 65536.0f + 2.0f));
      near = __builtin_elementwise_min(near, __builtin_bit_cast(u16x2, y[e]));
    }
    codes[r][0] = pack_byte2(y[0], y[1], y[2], y[3]) ^ 0x80808080u;
    codes[r][1] = pack_byte2(y[4], y[5], y[6], y[7]) ^ 0x80808080u;
    if (__builtin_expect(near[0] < 4, 0)) {
      auto again = [&](const auto& quotient) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          uint32_t w = 0;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float k = fminf(fmaxf(rintf(quotient(val(r, 4 * h + e))), -127.0f), 127.0f);
            w = __builtin_amdgcn_cvt_pk_u8_f32(k + 128.0f, e, w);
            __builtin_amdgcn_sched_barrier(0);
          }
          codes[r][h] = w ^ 0x80808080u;
        }
      };
      const float rcp = s.r16 * 0x1p-16f;     // RN(1 / a) again
      if (s.r16 > 0.0f) again([&](float x) { return exact_quotient(x, s.a, rcp); });
      // a scale of 0: a NaN comes here, its neighbours keep code 0
      else again([&](float x) { return s.a == 0.0f ? 0.0f : __fdiv_rn(x, s.a); });
    }
    __builtin_amdgcn_sched_barrier(0);     // one row's temporaries at a time
  }
}

// Position of a 16-byte granule of an LDS image.  Lanes that write one instruction's values differ in
// the bits folded into the low ones here, so they reach different banks; a run of 16 granules stays
// a run of 16, permuted.  kT: image of the transposed block.
template <bool kT>
__device__ __forceinline__ int swizzle(int g) {
  return kT ? g ^ (((g >> 4) & 1) | ((g >> 7) & 6)) : g ^ ((g >> 5) & 7);
}

// The thread's 4 x 8 codes into the image of the block in tile order (and of its transpose).
template <bool kWantT>
__device__ __forceinline__ void write_images(const u32x2 (&q)[kRows], int8_t* img, int8_t* img_t) {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));      // the addresses are worked out where they are used, not kept for a second call
  const int row = kRows * (t >> 4), col = kCols * (t & 15);
#pragma unroll
  for (int r = 0; r < kRows; ++r)
    *reinterpret_cast<u32x2*>(img + swizzle<false>(tile_offset(row + r, col) >> 4) * 16 + (col & 8)) = q[r];
  if constexpr (kWantT) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      // 4 x 4 bytes: rows become columns
      const uint32_t a = __builtin_amdgcn_perm(q[1][h], q[0][h], 0x05010400u);   // columns 0, 1 of rows 0, 1
      const uint32_t b = __builtin_amdgcn_perm(q[1][h], q[0][h], 0x07030602u);   // columns 2, 3
      const uint32_t c = __builtin_amdgcn_perm(q[3][h], q[2][h], 0x05010400u);
      const uint32_t d = __builtin_amdgcn_perm(q[3][h], q[2][h], 0x07030602u);
      const uint32_t t[4] = {__builtin_amdgcn_perm(c, a, 0x05040100u), __builtin_amdgcn_perm(c, a, 0x07060302u),
                             __builtin_amdgcn_perm(d, b, 0x05040100u), __builtin_amdgcn_perm(d, b, 0x07060302u)};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int off = tile_offset(col + 4 * h + e, row);
        *reinterpret_cast<uint32_t*>(img_t + swizzle<true>(off >> 4) * 16 + (off & 15)) = t[e];
      }
    }
  }
}

// The image, in order, to global memory.
template <bool kT>
__device__ __forceinline__ void copy_image(const int8_t* img, int8_t* dst) {
#pragma unroll
  for (int i = 0; i < kBlockBytes / 16 / kThreads; ++i) {
    const int g = i * kThreads + threadIdx.x;
    reinterpret_cast<v4i*>(dst)[g] = reinterpret_cast<const v4i*>(img)[swizzle<kT>(g)];
  }
}

// Loads the thread's 4 x 8 values of block (bi, bk), zero outside the matrix.  p.vec_ok: rows are
// 16-byte aligned.  Ragged and unaligned blocks load 16 bytes at 2-byte addresses, which the hardware
// takes, from the nearest place where all 8 values exist, and shift; like that all four loads are in
// flight together (with a branch per row each row's load was waited for before the next: four
// round trips to memory).
__device__ __forceinline__ void load_block(const QuantParams& p, int bi, int bk, v4i (&raw)[kRows]) {
  const int row = bi * kBlock + kRows * (threadIdx.x >> 4), col = bk * kBlock + kCols * (threadIdx.x & 15);
  if ((bi + 1) * kBlock <= p.rows && (bk + 1) * kBlock <= p.cols && p.vec_ok) {
    const uint16_t* src = p.x + (int64_t)row * p.ld + col;
#pragma unroll
    for (int r = 0; r < kRows; ++r) raw[r] = *reinterpret_cast<const v4i*>(src + r * p.ld);
  } else if (p.cols >= kCols) {
    const int from = min(col, p.cols - kCols), gone = 16 * (col - from);     // bits shifted out
#pragma unroll
    for (int r = 0; r < kRows; ++r)
      __builtin_memcpy(&raw[r], p.x + (int64_t)min(row + r, p.rows - 1) * p.ld + from, 16);
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      uint64_t v[2];
      __builtin_memcpy(v, &raw[r], 16);
      if (gone >= 64) {
        v[0] = gone < 128 ? v[1] >> (gone & 63) : 0;
        v[1] = 0;
      } else if (gone > 0) {
        v[0] = (v[0] >> gone) | (v[1] << (64 - gone));
        v[1] >>= gone;
      }
      if (row + r >= p.rows) v[0] = v[1] = 0;
      __builtin_memcpy(&raw[r], v, 16);
    }
  } else {
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      raw[r] = v4i{0, 0, 0, 0};
#pragma unroll
      for (int e = 0; e < kCols; ++e)
        if (row + r < p.rows && col + e < p.cols)
          raw[r][e >> 1] |= (int)((uint32_t)p.x[(int64_t)(row + r) * p.ld + col + e] << (16 * (e & 1)));
    }
  }
}

// max |G| of this thread's values as the bit pattern of a float: magnitudes of bf16 values order like
// 16-bit integers, two at a time
__device__ __forceinline__ uint32_t thread_absmax(const v4i (&raw)[kRows]) {
  u16x2 m = {0, 0};
#pragma unroll
  for (int r = 0; r < kRows; ++r)
#pragma unroll
    for (int d = 0; d < 4; ++d)
      m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, (uint32_t)raw[r][d] & 0x7FFF7FFFu));
  return (uint32_t)(m[0] > m[1] ? m[0] : m[1]) << 16;
}

// max |G| of the block.  NaNs, which are larger than everything as integers, do not count: where there
// are any (uniform over the workgroup) the maximum of the others is taken.  red, red2: kWaves words each.
__device__ __forceinline__ float block_absmax(const v4i (&raw)[kRows], uint32_t* red, uint32_t* red2) {
  float m = block_max(thread_absmax(raw), red);
  if (__builtin_expect(__float_as_uint(m) > 0x7F800000u, 0)) {
    uint32_t v = 0;
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
#pragma unroll
      for (int e = 0; e < kCols; ++e) {
        const uint32_t b = __float_as_uint(x_at(raw, r, e)) & 0x7FFFFFFFu;
        v = max(v, b > 0x7F800000u ? 0u : b);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    m = block_max(v, red2);
  }
  return m;
}

// The bits block b contributes to its group's word: "decided" and, if u, "flagged".
__device__ inline unsigned long long my_bits(int b, bool u) {
  return (1ull << (b & 31)) | ((u ? 1ull : 0ull) << (32 + (b & 31)));
}

// The ascending list of flagged block ids (the compaction step of the quantizer).  Every
// workgroup records its decision with one 64-bit atomic OR into the word of its group of 32
// blocks (bit b % 32: "decided", bit 32 + b % 32: "flagged"), issued as soon as the decision is
// known so that its round trip hides behind the quantization of the block.  The workgroup whose
// OR completes a group counts the group; the one that counts the last group knows that every
// word is final (each OR was performed before the count it led to) and writes the list from the
// words, which it then clears for the next call.  No fence is needed: the words are only ever
// touched by device-scope atomics.  The list holds the lowest `capacity` ids when more blocks
// are flagged than that.
__device__ inline void write_fb_list(unsigned long long* words, int nb, int capacity,
                                     int32_t* fb_list, int* wave_sum /* LDS, kWaves ints */,
                                     int* base_sh /* LDS, 1 int */) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int n_words = (nb + 31) >> 5;
  if (t == 0) *base_sh = 0;
  for (int first = 0; first < n_words; first += kThreads) {
    const int wi = first + t;
    uint32_t f = 0;
    if (wi < n_words) {
      f = (uint32_t)(__hip_atomic_load(words + wi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 32);
      __hip_atomic_store(words + wi, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const int mine = __popc(f);
    int incl = mine;      // inclusive prefix over the wavefront
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int v = __shfl_up(incl, off, 64);
      if (lane >= off) incl += v;
    }
    __syncthreads();   // base_sh / wave_sum of the previous trip have been read
    if (lane == 63) wave_sum[w] = incl;
    __syncthreads();
    int pos = *base_sh + incl - mine;
    for (int j = 0; j < w; ++j) pos += wave_sum[j];
    while (f) {
      const int bit = __ffs(f) - 1;
      f &= f - 1;
      if (pos < capacity) fb_list[pos] = wi * 32 + bit;
      ++pos;
    }
    __syncthreads();
    if (t == 0) {
      for (int j = 0; j < kWaves; ++j) *base_sh += wave_sum[j];
    }
  }
}


// floor(t) + [top 24 bits of w < fraction of t], clamped, + 128 as a float
__device__ __forceinline__ float round_stochastic(float t, uint32_t w) {
  const float lo = floorf(t), frac = t - lo;
  const float v = lo + (((float)(w >> 8) < frac * 16777216.0f) ? 1.0f : 0.0f);
  return fminf(fmaxf(v, -127.0f), 127.0f) + 128.0f;
}

// How quantize_kernel rounds.  kSrAligned: stochastic, a row holds a multiple of 4 elements and the
// matrix at most 2^34; kSr: stochastic, any size.
enum Rounding { kNearest, kSrAligned, kSr };

// Stochastic codes of row r of the thread.  Element (row, c) of the matrix uses word (row*cols + c) & 3
// of the Philox block with counter (row*cols + c) >> 2; e0 is the thread's first element.  kSrAligned:
// the 8 elements are 2 whole blocks, and the counter's upper half is zero, which makes most of the
// first two rounds constant.  Otherwise they start at word `off` of the first of 3 blocks; off is the
// same for the whole grid (the thread's first row is a multiple of 4, its first column of 8).
template <Rounding kR>
__device__ __forceinline__ void stochastic_row(const v4i (&raw)[kRows], int r, uint64_t e0, int off, uint64_t seed,
                                               float a, float rcp, bool plain, u32x2& codes) {
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  auto block = [&](int b, uint32_t (&w)[4]) {
    const uint64_t ctr = (e0 >> 2) + b;
    philox4x32_10((uint32_t)ctr, kR == kSrAligned ? 0u : (uint32_t)(ctr >> 32), k0, k1, w);
    __builtin_amdgcn_sched_barrier(0);
  };
  // the four elements 4 h ... with the random words w
  auto round4 = [&](int h, const uint32_t (&w)[4]) {
    float t[4];
    if (plain) {      // uniform over the workgroup
#pragma unroll
      for (int e = 0; e < 4; ++e) t[e] = exact_quotient(x_at(raw, r, 4 * h + e), a, rcp);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) t[e] = a == 0.0f ? 0.0f : __fdiv_rn(x_at(raw, r, 4 * h + e), a);
    }
    uint32_t c = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_cvt_pk_u8_f32(round_stochastic(t[e], w[e]), e, c);
    codes[h] = c ^ 0x80808080u;
    __builtin_amdgcn_sched_barrier(0);
  };
  if constexpr (kR == kSrAligned) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint32_t w[4];
      block(h, w);
      round4(h, w);
    }
  } else {
    uint32_t w[3][4];
#pragma unroll
    for (int b = 0; b < 3; ++b) block(b, w[b]);
    if (off & 1) {
#pragma unroll
      for (int i = 0; i < kCols + 2; ++i) w[i >> 2][i & 3] = w[(i + 1) >> 2][(i + 1) & 3];
    }
    if (off & 2) {
#pragma unroll
      for (int i = 0; i < kCols; ++i) w[i >> 2][i & 3] = w[(i + 2) >> 2][(i + 2) & 3];
    }
    round4(0, w[0]);
    round4(1, w[1]);
  }
}

}  // namespace

// What bounds it: memory for large tensors (8192 x 8192: 5.5 TB/s, a part of it from the last-level cache; a
// large copy reaches 5.2), on a thousand blocks and fewer the chain load - maximum - quantize - store of a
// block that no other round of workgroups overlaps.  Four rows x 8 columns per thread in 64 registers let
// four workgroups of eight wavefronts share a compute unit (twice the wavefronts of a 4 x 16 split by 256
// threads) and halve a thread's part of that chain.  Measured against that split (and its rounding, which
// tested every value), re-quantizing into the same tensor, 5 % of the blocks flagged: 2048 x 4096 12.7 ->
// 10.2 us, 4096 x 4096 18.5 -> 14.7 us (with transposed copies 24.9 -> 16.8, stochastic with them 25.9 ->
// 20.8), 8192 x 8192 40.8 -> 37.6 us (61.2 -> 48.4, 76 -> 63), 33 x 4096 13.4 -> 6.7 us; every block flagged
// 33.5 -> 30.8 and 73.7 -> 73.4 us; the L1 criteria (88 registers), 30 % flagged, 30 -> 22 and 81 -> 57 us.
// kErr: the fallback decision uses a block quantization-error metric (criteria 3, 4), which
// needs the residual of every block, not only of the flagged ones.
template <bool kWantT, Rounding kR, bool kErr>
__global__ __launch_bounds__(kThreads, kErr || kR == kSr ? 4 : 8)
void quantize_kernel(QuantParams p) {
  __shared__ uint32_t red[2][kWaves];
  __shared__ double redd[kErr ? 2 * kWaves : 1];
  __shared__ int slot_sh, last_sh, scan_base_sh;
  __shared__ uint32_t flags_sh;
  __shared__ int scan_sh[kWaves];
  __shared__ __attribute__((aligned(16))) int8_t img[kBlockBytes];
  __shared__ __attribute__((aligned(16))) int8_t img_t[kWantT ? kBlockBytes : 16];

  const int blk = blockIdx.x;
  const int bi = blk / p.nbc, bk = blk - bi * p.nbc;
  const int t = threadIdx.x;
  const int row = kRows * (t >> 4), col = kCols * (t & 15);     // inside the block

  v4i raw[kRows];
  load_block(p, bi, bk, raw);

  // ---- step 1: a = max|G| / 127, codes = round(G / a)           (Sec. 3.1)
  const float amax = block_absmax(raw, red[0], red[1]);
  const Scale sc = make_scale(amax);
  const float a = sc.a;
  forget_unpacked(raw);

  // The abs-max decision is known now: take the residual slot right away, so that the round
  // trip of the atomic is hidden behind the quantization of the block.          (Sec. 4.4)
  // without residual slots or a criterion nothing can fall back: the list is empty, nobody counts
  const bool want_list = kR == kNearest && p.capacity > 0 && p.crit != 0;
  bool u = false;
  int slot_early = -1;
  unsigned long long group_before = 0;   // thread 0: the group's word before this block's bits
  if (kR == kNearest && !kErr) {
    // criterion 5: the decision was taken by topk_select_kernel and is read from the mask
    u = p.crit == 2 || (p.crit == 1 && amax > p.theta) || (p.crit == 5 && p.mask[blk] != 0);
    if (t == 0) {
      if (u) slot_early = atomicAdd(p.fb_count, 1);
      if (want_list) group_before = atomicOr(p.fb_words + (blk >> 5), my_bits(blk, u));
    }
    // a flagged block has twice the work of the others and ends the kernel: it goes first
    if (u) __builtin_amdgcn_s_setprio(3);
  }

  u32x2 q[kRows];
  if constexpr (kR == kNearest) {
    quantize_rows([&](int r, int e) { return x_at(raw, r, e); }, sc, q);
  } else {
    const bool plain = a >= 0x1p-90f && a <= 0x1p90f;       // uniform over the workgroup
    const float rcp = plain ? __fdiv_rn(1.0f, a) : 0.0f;
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      const uint64_t e0 = (uint64_t)(bi * kBlock + row + r) * (uint64_t)p.cols + (uint64_t)(bk * kBlock + col);
      stochastic_row<kR>(raw, r, e0, (r * p.cols) & 3, p.seed, a, rcp, plain, q[r]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // ---- the block's residual slot, known to the whole workgroup with the barrier behind the images
  // (the atomic issued after the decision has had the whole quantization to come back; an
  // unflagged block does not look at it at all); with an error-based criterion the decision is only
  // known after the codes, so it gets a barrier of its own.
  auto publish_slot = [&]() {
    if (kR == kNearest && t == 0) {
      int slot0 = -1;
      if (u) {
        asm volatile("" : "+v"(slot_early));     // keeps the wait for the atomic inside this branch
        slot0 = (slot_early < p.capacity) ? slot_early : -2;
      }
      slot_sh = slot0;
    }
  };
  if (!kErr) publish_slot();
  forget_unpacked(raw);
  write_images<kWantT>(q, img, img_t);
  __syncthreads();
  int slot = kErr || kR != kNearest ? -1 : slot_sh;
  copy_image<false>(img, p.codes + (int64_t)blk * kBlockBytes);
  if (kWantT) copy_image<true>(img_t, p.codes_t + ((int64_t)bk * p.nbr + bi) * kBlockBytes);

  // ---- per-block outputs: scale, mask, slot.  Stored last, when the wavefront has nothing left
  // to compute: a register that held store data is not reused before the store has completed,
  // and behind these small stores that wait sat in the middle of the quantization.
  auto store_block_record = [&]() {
    if (t == 0) {
      p.scales[blk] = a;
      p.mask[blk] = u ? 1 : 0;
      p.fb_slot[blk] = slot;
      if (blk == 0) *p.fb_count_next = 0;   // ready for the next call into this tensor
    }
  };
  // ---- the list of flagged blocks: the workgroup whose decision completed a group of 32 counts
  // the group, the one that counts the last group writes the list.  Runs when the workgroup has
  // issued all its stores, so that nobody's codes wait for the round trip of the counter.
  // count_group: thread 0; counts the block's group if its decision completed it.
  int counted = -1;      // thread 0: groups counted before this one
  auto count_group = [&]() {
    const int nb = (int)gridDim.x, g = blk >> 5;
    const uint32_t full = (nb - 32 * g >= 32) ? 0xFFFFFFFFu : ((1u << (nb - 32 * g)) - 1u);
    // (both halves of the returned word are named here: a half that nothing reads gives its
    // register away at once, and the write to that register would wait for the atomic)
    asm volatile("" ::"v"(group_before));
    const uint32_t decided = (uint32_t)group_before | (1u << (blk & 31));
    if (decided == full) counted = nb <= 32 ? 0 : atomicAdd(p.fb_groups_done, 1);
  };
  auto finish_list = [&](bool counted_early) {
    if (!want_list) return;       // uniform over the grid
    if (t == 0) {
      if (!counted_early) count_group();
      last_sh = counted == (((int)gridDim.x + 31) >> 5) - 1;
      flags_sh = (uint32_t)(group_before >> 32) | (u ? 1u << (blk & 31) : 0u);
    }
    __syncthreads();
    if (!last_sh) return;          // uniform over the workgroup
    if (gridDim.x <= 32) {
      // one group: its flags came back with the OR that completed it
      const uint32_t f = flags_sh;
      const int pos = __popc(f & ((1u << (t & 31)) - 1u));
      if (t < 32 && (f >> t & 1u) && pos < p.capacity) p.fb_list[pos] = t;
      if (t == 0) __hip_atomic_store(p.fb_words, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      write_fb_list(p.fb_words, (int)gridDim.x, p.capacity, p.fb_list, scan_sh, &scan_base_sh);
      if (t == 0) *p.fb_groups_done = 0;    // ready for the next call
    }
  };

  // the residual G - a*codes of element (r, e): one fused multiply-add, single rounding
  auto residual = [&](int r, int e) {
    return __builtin_fmaf(-(float)code_at(q, r, e), a, x_at(raw, r, e));
  };

  // ---- fallback decision by a quantization-error metric          (Sec. 4.4)
  if (kErr) {
    // L1 = sum |G - Q(G)| over the block, L1-Rel = L1 / sum |G|; the sums are binary64
    // accumulations of the binary32 terms (order unspecified), compared with theta in binary64
    double l1 = 0.0, l1x = 0.0;
#pragma unroll
    for (int r = 0; r < kRows; ++r)
#pragma unroll
      for (int e = 0; e < kCols; ++e) {
        l1x += (double)fabsf(x_at(raw, r, e));
        l1 += (double)fabsf(residual(r, e));
      }
    block_sum2(l1, l1x, redd);
    if (p.crit == 3) u = l1 > (double)p.theta;
    else u = l1x > 0.0 && l1 / l1x > (double)p.theta;
    if (t == 0) {
      if (u) slot_early = atomicAdd(p.fb_count, 1);
      if (want_list) group_before = atomicOr(p.fb_words + (blk >> 5), my_bits(blk, u));
    }
    publish_slot();
    __syncthreads();
    slot = slot_sh;
  }
  if (kR != kNearest || slot < 0) {        // uniform over the workgroup
    store_block_record();
    finish_list(false);
    return;
  }
  // A flagged block, which ends the kernel, counts its group here and not behind its stores: so the last to count
  // is most often an unflagged one, and the list is written while the residuals are still quantized.  5 and 20 %
  // of the blocks flagged: 1024 x 2048 7.4 -> 6.4 and 8.2 -> 7.0 us, 2048 x 2048 8.4 -> 7.4 and 9.6 -> 8.3, 4096 x
  // 4096, where the blocks are a round of the chip and more, 14.3 -> 13.8 and 17.0 -> 16.3.  (Asking for the slot
  // and counting only when the residual is quantized gave a third of that.)
  if (want_list && t == 0) count_group();

  // ---- step 2: quantize the residual G - a*codes                 (Sec. 4.3)
  // (the residual is recomputed where it is needed instead of being kept in registers)
  float rm = 0.0f;
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
#pragma unroll
    for (int e = 0; e < kCols; ++e) rm = fmaxf(rm, fabsf(residual(r, e)));
    __builtin_amdgcn_sched_barrier(0);
  }
  const Scale rs = make_scale(block_max(__float_as_uint(rm), red[1]));   // its barrier frees the images
  forget_unpacked(raw);
  forget_unpacked(q);
  u32x2 rq[kRows];
  quantize_rows(residual, rs, rq);
  write_images<kWantT>(rq, img, img_t);
  __syncthreads();
  copy_image<false>(img, p.res_codes + (int64_t)slot * kBlockBytes);
  if (kWantT) copy_image<true>(img_t, p.res_codes_t + (int64_t)slot * kBlockBytes);
  if (t == 0) p.res_scales[slot] = rs.a;
  store_block_record();
  finish_list(true);
}

// ---- TopK AbsMax selection (Sec. 4.4), in three launches: the abs-max of every block, the
// tensor-wide choice of the k largest, then quantize_kernel with that choice as its decision.

// max |G| of each block into amax[nbr * nbc] (the tensor's scale array serves as that buffer
// until quantize_kernel overwrites it with the scales).
__global__ __launch_bounds__(kThreads, 8) void block_absmax_kernel(QuantParams p) {
  __shared__ uint32_t red[2][kWaves];
  const int blk = blockIdx.x;
  const int bi = blk / p.nbc, bk = blk - bi * p.nbc;
  v4i raw[kRows];
  load_block(p, bi, bk, raw);
  const float amax = block_absmax(raw, red[0], red[1]);
  if (threadIdx.x == 0) p.scales[blk] = amax;
}

constexpr int kSelectThreads = 1024;

// mask[b] = 1 for the k blocks with the largest amax (0 < k < nb), equal values in ascending
// block order.  One workgroup: a radix select over the bit patterns (non-negative binary32
// values order like unsigned integers) finds the k-th largest value T in four passes of 8
// bits; then everything above T is flagged, and of the blocks equal to T the first ones in
// index order, as many as are still missing.
__global__ __launch_bounds__(kSelectThreads) void topk_select_kernel(const float* amax, int nb,
                                                                    int k, uint8_t* mask) {
  __shared__ int hist[256], suffix[256];
  __shared__ int sel_bin, sel_want;
  __shared__ int wave_total[kSelectThreads / 64];
  __shared__ int running;
  const int t = threadIdx.x;
  uint32_t prefix = 0, known = 0;
  int want = k;            // the value looked for is the want-th largest among those matching prefix
  for (int shift = 24; shift >= 0; shift -= 8) {
    if (t < 256) hist[t] = 0;
    __syncthreads();
    for (int i = t; i < nb; i += kSelectThreads) {
      const uint32_t b = __float_as_uint(amax[i]);
      if ((b & known) == prefix) atomicAdd(&hist[(b >> shift) & 255], 1);
    }
    __syncthreads();
    // the bin holding the want-th largest candidate: the one whose count of candidates in
    // bins >= it reaches `want` while the count in bins above it does not.  suffix[b] = sum of
    // hist[b..255] by a 256-wide parallel scan.
    if (t < 256) suffix[t] = hist[t];
    __syncthreads();
    for (int step = 1; step < 256; step <<= 1) {
      int add = 0;
      if (t < 256 && t + step < 256) add = suffix[t + step];
      __syncthreads();
      if (t < 256) suffix[t] += add;
      __syncthreads();
    }
    if (t < 256) {
      const int above = t < 255 ? suffix[t + 1] : 0;
      if (suffix[t] >= want && above < want) {
        sel_bin = t;
        sel_want = want - above;
      }
    }
    __syncthreads();
    prefix |= (uint32_t)sel_bin << shift;
    known |= 255u << shift;
    want = sel_want;
    __syncthreads();       // sel_* and hist are rewritten in the next pass
  }
  const uint32_t T = prefix;     // `want` of the blocks equal to T are taken
  if (t == 0) running = 0;
  __syncthreads();
  const int lane = t & 63, w = t >> 6;
  for (int base = 0; base < nb; base += kSelectThreads) {
    const int i = base + t;
    const uint32_t b = i < nb ? __float_as_uint(amax[i]) : 0u;
    const bool eq = i < nb && b == T;
    const unsigned long long ballot = __ballot(eq);
    const int before_in_wave = __popcll(ballot & ((1ull << lane) - 1ull));
    if (lane == 0) wave_total[w] = __popcll(ballot);
    __syncthreads();
    int before = running, chunk = 0;
    for (int j = 0; j < kSelectThreads / 64; ++j) {
      if (j < w) before += wave_total[j];
      chunk += wave_total[j];
    }
    if (i < nb) mask[i] = (b > T || (eq && before + before_in_wave < want)) ? 1 : 0;
    __syncthreads();
    if (t == 0) running += chunk;
    __syncthreads();
  }
}

// mask[b] = v for every block (k <= 0 or k >= number of blocks).
__global__ void fill_mask_kernel(uint8_t* mask, int nb, int v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nb) mask[i] = (uint8_t)v;
}

// Clears both slot counters: first use of a tensor, or an empty input.
__global__ void clear_counters_kernel(int32_t* live, int32_t* next, int32_t* groups_done,
                                      unsigned long long* words, int n_words) {
  if (threadIdx.x == 0) {
    *live = 0;
    *next = 0;
    *groups_done = 0;
  }
  for (int i = threadIdx.x; i < n_words; i += blockDim.x) words[i] = 0;
}

// Tile order -> dense row-major (inspection / tests).
__global__ void untile_kernel(const int8_t* tiled, int rows, int cols, int nbc, int8_t* dense) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)rows * cols) return;
  const int r = (int)(idx / cols), c = (int)(idx - (int64_t)r * cols);
  const int64_t blk = (int64_t)(r >> 7) * nbc + (c >> 7);
  dense[idx] = tiled[blk * kBlockBytes + tile_offset(r & 127, c & 127)];
}

hipError_t launch_quantize(const QuantParams& p, hipStream_t st) {
  if (p.clear_both)
    hipLaunchKernelGGL(clear_counters_kernel, dim3(1), dim3(256), 0, st, p.fb_count, p.fb_count_next,
                       p.fb_groups_done, p.fb_words, (p.nbr * p.nbc + 31) / 32);
  const int nb = p.nbr * p.nbc;
  if (nb > 0 && p.crit == 5) {
    if (p.topk <= 0 || p.topk >= nb) {
      hipLaunchKernelGGL(fill_mask_kernel, dim3((nb + 255) / 256), dim3(256), 0, st, p.mask, nb,
                         p.topk > 0 ? 1 : 0);
    } else {
      hipLaunchKernelGGL(block_absmax_kernel, dim3(nb), dim3(kThreads), 0, st, p);
      hipLaunchKernelGGL(topk_select_kernel, dim3(1), dim3(kSelectThreads), 0, st, p.scales, nb,
                         p.topk, p.mask);
    }
  }
  if (nb > 0) {
    const dim3 grid(nb), block(kThreads);
    const bool err = p.crit == 3 || p.crit == 4;
    auto go = [&](auto rounding, auto err_c) {
      constexpr Rounding kR = (Rounding)decltype(rounding)::value;
      constexpr bool kErr = decltype(err_c)::value;
      if (p.codes_t) hipLaunchKernelGGL((quantize_kernel<true, kR, kErr>), grid, block, 0, st, p);
      else hipLaunchKernelGGL((quantize_kernel<false, kR, kErr>), grid, block, 0, st, p);
    };
    const bool aligned = p.cols % 4 == 0 && (int64_t)p.rows * p.cols <= (int64_t)1 << 34;
    if (p.stochastic && aligned) go(std::integral_constant<int, kSrAligned>{}, std::false_type{});
    else if (p.stochastic) go(std::integral_constant<int, kSr>{}, std::false_type{});
    else if (err) go(std::integral_constant<int, kNearest>{}, std::true_type{});
    else go(std::integral_constant<int, kNearest>{}, std::false_type{});
  }
  return hipGetLastError();
}

hipError_t launch_untile(const int8_t* tiled, int rows, int cols, int8_t* dense, hipStream_t st) {
  const int64_t n = (int64_t)rows * cols;
  if (n == 0) return hipSuccess;
  const int nbc = (cols + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(untile_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, tiled,
                     rows, cols, nbc, dense);
  return hipGetLastError();
}

}  // namespace fq
