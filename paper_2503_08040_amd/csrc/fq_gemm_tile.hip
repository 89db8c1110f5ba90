// Fallback block GEMM for outputs that 256 x 256 tiles do not fill the chip with (few tokens, small
// layers, ragged batches): Alg. 1 of the paper on smaller tiles.
//
// Same operands, same accumulation order per output element (k ascending, main term then residual
// term, binary32 FMAs) and therefore the same bits as gemm_kernel of fq_gemm.hip, which stays the
// kernel for outputs of about a chip's worth of 256 x 256 tiles and more.  That kernel gives a
// compute unit one 256 x 256 tile; an output of 64 such tiles leaves three quarters of the chip
// idle, and one of 33 rows multiplies mostly padding.  Here the contraction is never split (the
// order of the FP32 terms is part of the interface), so parallelism comes from the tile size alone:
//   gemm_wave_kernel            one wavefront per 32 x 32 tile, both operands straight from global
//                               memory into registers, no LDS, no barrier
//   gemm_tile_kernel<2>   128 x 64 tiles, 4 wavefronts of 32 x 64
//   gemm_tile_kernel<4>   128 x 128 tiles, 4 wavefronts of 32 x 128
// A wavefront owns 32 whole rows, so its A operands go from global memory into registers and only
// the B operands, which the wavefronts of a column share, pass through LDS.  A 32 x 32 x 128 step
// asks the compute unit's vector cache for 8, 3 and 2 KiB of operands in the three forms (1 KiB in
// gemm_kernel), and on a full chip that is what they lose to the larger tiles by: with the loads taken out
// of the loop 4096^3 runs at 1773 and 2008 TOP/s on the first two instead of 486 and 1525.  With few tiles it is
// latency: a third of a wavefront's time is waiting for loads (or the barrier) and a third the issue of its own
// matrix and vector instructions, one after the other; 33 x 4096 x 11008 keeps the matrix cores busy 12 % of
// the cycles.  So the 128 x 64 and 128 x 128 forms are for outputs of more than a round of the tiles of
// fq_gemm_ring.hip and less than about a round of gemm_kernel's (and for short contractions), where two or three workgroups on a compute unit
// hide each other's latency and start and end at different times; plan_small in fq_gemm.hip has the rule.
// Measured (GEMM alone, bf16 output, gemm_kernel -> the form chosen): 33 x 4096 x 11008 70.6 -> 12.2 us,
// 256 x 11008 x 4096 182 -> 28.1 us (5 % of the blocks flagged), 1536 x 4096 x 4096 76 -> 34.1 us, 3072^3
// 61 -> 42 us.
//
// The MFMA operands are swapped (D = B A^T): a lane then holds consecutive columns of one row of C
// and stores them without a transposition through LDS.
#include <type_traits>

#include "fq_device.h"
#include "fq_gemm_unit.h"
#include "fq_kernels.h"

namespace fq {

namespace {


constexpr int kGroupN = 4;        // tile columns per rasterization group
constexpr int kTileThreads = 256;

// Keeps a wave-uniform address in scalar registers: loads then take the scalar-base form, and no
// vector register is written as an address while loads into its neighbours are in flight.
typedef const __attribute__((address_space(1))) int8_t gbl_i8;
typedef const __attribute__((address_space(1))) v4i gbl_v4i;
__device__ __forceinline__ gbl_i8* scalar_ptr(const int8_t* q) {
  gbl_i8* g = (gbl_i8*)q;
  asm("" : "+s"(g));
  return g;
}
// The per-lane part of such an address, opaque so that it stays a 32-bit offset at its use.
__device__ __forceinline__ unsigned lane_offset(unsigned v) {
  asm("" : "+v"(v));
  return v;
}
__device__ __forceinline__ v4i load16(gbl_i8* base, unsigned off, int imm) {
  return *(gbl_v4i*)(base + off + imm);
}

}  // namespace

// Scales and residual slots of 64 consecutive k-blocks, one per lane: main scale product, scale of B,
// residual scale and slot of block (ib, k0 + lane).  Read back with v_readlane, they cost the k-loop no
// scalar loads, whose unordered counter would wait for the youngest of them at every use.  Loaded in
// two steps because the residual scales depend on the slots.
struct KFirst {
  float sa, sb;
  int slot;
};
struct KLane {
  float s, sb, rs;
  int slot;
};

__device__ __forceinline__ KFirst load_first(const GemmParams& p, int ib, int jb, int k0, int lane) {
  const int k = min(k0 + lane, p.nkb - 1);
  KFirst r;
  r.slot = p.a_slot ? p.a_slot[ib * p.a_si + k * p.a_sk] : -1;
  r.sb = p.b_scales[jb * p.b_sj + k * p.b_sk];
  r.sa = p.a_scales[ib * p.a_si + k * p.a_sk];
  return r;
}
__device__ __forceinline__ KLane finish(const GemmParams& p, const KFirst& f) {
  KLane r;
  r.rs = p.a_slot ? p.a_res_scales[max(f.slot, 0)] : 0.0f;
  r.s = f.sa * f.sb;
  r.sb = f.sb;
  r.slot = f.slot;
  return r;
}
__device__ __forceinline__ int lane_int(int v, int k) { return __builtin_amdgcn_readlane(v, k & 63); }
__device__ __forceinline__ float lane_float(float v, int k) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k & 63));
}

// step(k + d, d, reload) for d in [kFrom, kTo) as long as k + d < end
template <int kFrom, int kTo, class F>
__device__ __forceinline__ void steps(int k, int end, F& step, bool reload) {
  if constexpr (kFrom < kTo) {
    if (k + kFrom < end) {
      step(k + kFrom, std::integral_constant<int, kFrom>{}, reload);
      steps<kFrom + 1, kTo>(k, end, step, reload);
    }
  }
}

// ---- one wavefront per 32 x 32 output tile, operands straight from global memory.  kD k-blocks are in
// flight (32 registers each); the steps of a trip are straight-line code, so that the compiler's wait
// for a k-block leaves the younger ones in flight.  A k-block's tile is folded under the next one's
// MFMAs, which matters where a wavefront has its SIMD to itself: 33 x 11008 x 4096 23.3 -> 21.4 us, 64 x
// 2048 x 2048 6.5 -> 6.1, 128 x 4096 x 4096 11.3 -> 10.7.  33 x 4096 x 11008 (12.2 us) reads its 45 MB of
// weights at 3.7 TB/s: its 688 wavefronts have 5.6 MB of them in flight, since the two row groups of a column
// ask for the same ones.
template <int kD>
__global__ __launch_bounds__(64, 2) void gemm_wave_kernel(GemmParams p) {
  const int lane = threadIdx.x;
  const int nrg = (p.M + 31) >> 5;
  const int L = xcd_run(blockIdx.x, gridDim.x);
  const int cg = L / nrg, rg = L - cg * nrg;
  const int ib = rg >> 2, jb = cg >> 2;
  const int nkb = p.nkb;
  const int kg = lane >> 4, l15 = lane & 15;
  const int koff = (kg >> 1) * 1024 + (kg & 1) * 512;
  const unsigned aoff = koff + l15 * 16;
  const unsigned boff[2] = {(unsigned)(koff + perm_col(l15, 0) * 16), (unsigned)(koff + perm_col(l15, 1) * 16)};
  const int8_t* const abase = p.a_codes + (int64_t)ib * nkb * kBlockBytes + (rg & 3) * kFragRows;
  const int8_t* const rbase = p.a_res + (rg & 3) * kFragRows;
  const int8_t* const bbase = p.b_codes + (int64_t)jb * nkb * kBlockBytes + (cg & 3) * kFragRows;

  v4i A[kD][2][2], B[kD][2][2], R[2][2];
  float acc[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
  bool bad = false;

  auto load_main = [&](int k, v4i (&a)[2][2], v4i (&b)[2][2]) {
    k = min(k, nkb - 1);
    gbl_i8* as = scalar_ptr(abase + (int64_t)k * kBlockBytes);
    gbl_i8* bs = scalar_ptr(bbase + (int64_t)k * kBlockBytes);
    const unsigned ao = lane_offset(aoff), bo0 = lane_offset(boff[0]), bo1 = lane_offset(boff[1]);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        b[i][ks] = load16(bs, i ? bo1 : bo0, ks * 2048);
        a[i][ks] = load16(as, ao, i * 256 + ks * 2048);
      }
  };
  auto load_res = [&](int slot) {
    gbl_i8* as = scalar_ptr(rbase + (int64_t)slot * kBlockBytes);
    const unsigned ao = lane_offset(aoff);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        R[i][ks] = load16(as, ao, i * 256 + ks * 2048);
  };
  v4i P[2][4];
  auto fold = [&](const v4i (&t)[4], float f) {
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = __builtin_fmaf((float)t[e >> 2][e & 3], f, acc[e]);
  };

  if (nkb > 0) {
    // the first k-blocks' scales are requested in front of the operands: loads return in order, and
    // the residual scales take a second trip
    const KFirst first = load_first(p, ib, jb, 0, lane);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < kD; ++d) load_main(d, A[d], B[d]);
#pragma unroll
    for (int q = 0; q < 4; ++q) P[1][q] = v4i{0, 0, 0, 0};
    float sp = 0.0f;      // scale of the unit whose tile is still to be folded
    auto chunk = [&](const KLane& kl, int k0) {
      bad |= __ballot(kl.slot == -2) != 0;
      const int n = min(64, nkb - k0);
      int slot = lane_int(kl.slot, 0);
      if (slot >= 0) load_res(slot);
      auto step = [&](int k, auto d_c, bool reload) {
        constexpr int d = decltype(d_c)::value, par = d & 1;
        unit<par>(P, B[d], acc, A[d], sp, [](int) {});
        sp = lane_float(kl.s, k);
        if (slot >= 0) {
          // the residual's tile takes the main one's place: fold that now
          fold(P[par], sp);
#pragma unroll
          for (int q = 0; q < 4; ++q) P[par][q] = mfma16(B[d][q >> 1][0], R[q & 1][0], v4i{0, 0, 0, 0});
#pragma unroll
          for (int q = 0; q < 4; ++q) P[par][q] = mfma16(B[d][q >> 1][1], R[q & 1][1], P[par][q]);
          sp = lane_float(kl.rs, k) * lane_float(kl.sb, k);
        }
        if (reload) load_main(k0 + k + kD, A[d], B[d]);
        slot = k + 1 < n ? lane_int(kl.slot, k + 1) : -1;
        if (slot >= 0) load_res(slot);
      };
      int k = 0;
      for (; k + kD <= n; k += kD) steps<0, kD>(k, k + kD, step, true);
      // what is left is the end of the contraction (64 is a multiple of kD)
      steps<0, kD - 1>(k, n, step, false);
    };
    chunk(finish(p, first), 0);
    for (int k0 = 64; k0 < nkb; k0 += 64) chunk(finish(p, load_first(p, ib, jb, k0, lane)), k0);
    if (nkb & 1) fold(P[0], sp);
    else fold(P[1], sp);
  }
  store_unit(p, acc, rg * 32, cg * 32, lane, bad);
}

// ---- one workgroup of four wavefronts per output tile of 128 rows x 32 kWU columns, every wavefront 32
// rows x kWU column groups ("units"), kWU = 2 or 4

// A unit whose successor's B operands are fetched from LDS (b_next) into bq[kPar ^ 1].
template <int kPar>
__device__ __forceinline__ void tile_unit(v4i (&P)[2][4], v4i (&bq)[2][2][2], float (&acc)[16], const v4i (&a)[2][2],
                                          const int8_t* b_next, const int (&boff)[2], float f) {
  unit<kPar>(P, bq[kPar], acc, a, f, [&](int n) {
    if (n < 4) bq[kPar ^ 1][n >> 1][n & 1] = *reinterpret_cast<const v4i*>(b_next + boff[n >> 1] + (n & 1) * 2048);
  });
}

// Units [kFrom, kTo) of a wavefront with kWU units per k-block, every one with its
// successor in the same B stage bs.  sp: scale of the unit folded by unit 0, s: by the others.
template <int kWU, int kFrom, int kTo>
__device__ __forceinline__ void tile_units(v4i (&P)[2][4], v4i (&bq)[2][2][2], float (&acc)[kWU][16],
                                           const v4i (&a)[2][2], const int8_t* bs, const int (&boff)[2], float s,
                                           float sp) {
  if constexpr (kFrom < kTo) {
    tile_unit<kFrom & 1>(P, bq, acc[(kFrom + kWU - 1) % kWU], a, bs + (kFrom + 1) % kWU * kFragRows, boff,
                         kFrom ? s : sp);
    tile_units<kWU, kFrom + 1, kTo>(P, bq, acc, a, bs, boff, s, sp);
  }
}

// The B blocks of k-block k + 1 go from registers into the other LDS stage in front of the last unit of
// k-block k, behind it the barrier, then the loads for k + 2; A operands are requested one k-block
// ahead.  (Direct global-to-LDS loads were tried: with them in the loop the compiler waits for every
// load at the first use of an A operand; deeper register rings measured the same.)
template <int kWU>
__global__ __launch_bounds__(kTileThreads, 2) void gemm_tile_kernel(GemmParams p, int tiles_i, int tiles_j) {
  constexpr int kStageBytes = kWU * kFragRows;
  constexpr int kBL = kWU;                        // 1 KiB loads of a wavefront per B stage
  __shared__ __attribute__((aligned(1024))) int8_t lds[2 * kStageBytes];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nkb = p.nkb;
  int ti, tj;
  tile_at<kGroupN>(xcd_run(blockIdx.x, gridDim.x), tiles_i, tiles_j, ti, tj);
  const int cg0 = tj * kWU, ib = ti, jb = cg0 >> 2, rg = 4 * ti + w;
  const int kg = lane >> 4, l15 = lane & 15;
  const int koff = (kg >> 1) * 1024 + (kg & 1) * 512;
  const unsigned aoff = koff + l15 * 16;
  const int boff[2] = {koff + perm_col(l15, 0) * 16, koff + perm_col(l15, 1) * 16};
  const int8_t* const abase = p.a_codes + (int64_t)ib * nkb * kBlockBytes + w * kFragRows;
  const int8_t* const rbase = p.a_res + w * kFragRows;
  const int8_t* const bbase = p.b_codes + (int64_t)jb * nkb * kBlockBytes + (cg0 & 3) * kFragRows + w * (kBL * 1024);

  float acc[kWU][16];
  v4i bq[2][2][2], P[2][4];
#pragma unroll
  for (int u = 0; u < kWU; ++u)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[u][e] = 0.0f;
  bool bad = false;

  auto load_a = [&](const int8_t* ptr, v4i (&a)[2][2]) {
    gbl_i8* src = scalar_ptr(ptr);
    const unsigned ao = lane_offset(aoff);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i][ks] = load16(src, ao, i * 256 + ks * 2048);
  };
  // this wavefront's share of a B stage: registers, then LDS
  auto load_b = [&](int k, v4i (&b)[kBL]) {
    gbl_i8* src = scalar_ptr(bbase + (int64_t)min(k, nkb - 1) * kBlockBytes);
    const unsigned bo = lane_offset((unsigned)lane * 16u);
#pragma unroll
    for (int i = 0; i < kBL; ++i) b[i] = load16(src, bo, i * 1024);
  };
  auto write_b = [&](int stage, const v4i (&b)[kBL]) {
    int8_t* dst = lds + stage * kStageBytes + w * (kBL * 1024) + lane * 16;
#pragma unroll
    for (int i = 0; i < kBL; ++i) *reinterpret_cast<v4i*>(dst + i * 1024) = b[i];
  };

  if (nkb > 0) {
    v4i A[2][2][2], R[2][2], bn[kBL];
    load_b(0, bn);
    load_a(abase, A[0]);
    write_b(0, bn);
    load_b(1, bn);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int i = 0; i < 4; ++i)
      bq[0][i >> 1][i & 1] = *reinterpret_cast<const v4i*>(lds + boff[i >> 1] + (i & 1) * 2048);
#pragma unroll
    for (int q = 0; q < 4; ++q) P[1][q] = v4i{0, 0, 0, 0};
    float sp = 0.0f;      // scale of the unit whose tile is still to be folded
    for (int k0 = 0; k0 < nkb; k0 += 64) {
      const KLane kl = finish(p, load_first(p, ib, jb, k0, lane));
      const float residual_scales = kl.rs * kl.sb;
      bad |= __ballot(kl.slot == -2) != 0;
      const int kend = min(k0 + 64, nkb);
      // k-block k of parity j: its A operands are in A[j], its B blocks in LDS stage j
      auto step = [&](int k, auto j_c) {
        constexpr int j = decltype(j_c)::value;
        v4i (&a)[2][2] = A[j];
        const int slot = lane_int(kl.slot, k);
        load_a(abase + (int64_t)min(k + 1, nkb - 1) * kBlockBytes, A[j ^ 1]);
        if (slot >= 0) load_a(rbase + (int64_t)slot * kBlockBytes, R);
        float s = lane_float(kl.s, k);
        const float t = lane_float(residual_scales, k);
        const int8_t* const bs = lds + j * kStageBytes;
        tile_units<kWU, 0, kWU - 1>(P, bq, acc, a, bs, boff, s, sp);
        if (slot >= 0) {
          // the residual product re-uses the B blocks on chip; its last unit is the common one below
          tile_unit<1>(P, bq, acc[kWU - 2], a, bs, boff, s);
          tile_units<kWU, 0, kWU - 1>(P, bq, acc, R, bs, boff, t, s);
#pragma unroll
          for (int i = 0; i < 4; ++i) a[i >> 1][i & 1] = R[i >> 1][i & 1];
          s = t;
        }
        write_b(j ^ 1, bn);
        load_b(k + 2, bn);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        tile_unit<1>(P, bq, acc[kWU - 2], a, lds + (j ^ 1) * kStageBytes, boff, s);
        sp = s;
      };
      int k = k0;
      for (; k + 2 <= kend; k += 2) {
        step(k, std::integral_constant<int, 0>{});
        step(k + 1, std::integral_constant<int, 1>{});
      }
      if (k < kend) step(k, std::integral_constant<int, 0>{});
    }
#pragma unroll
    for (int e = 0; e < 16; ++e)     // the last unit
      acc[kWU - 1][e] = __builtin_fmaf((float)P[1][e >> 2][e & 3], sp, acc[kWU - 1][e]);
  }
#pragma unroll
  for (int u = 0; u < kWU; ++u)
    store_unit(p, acc[u], rg * 32, (cg0 + u) * 32, lane, bad);
}

hipError_t launch_gemm_small(const GemmParams& p, SmallTile tile, hipStream_t st) {
  auto tiles = [&](int r, int c) { return dim3(((p.M + r - 1) / r) * ((p.N + c - 1) / c)); };
  switch (tile) {
    case SmallTile::k32x32: hipLaunchKernelGGL(gemm_wave_kernel<4>, tiles(32, 32), dim3(64), 0, st, p); break;
    case SmallTile::k128x64:
      hipLaunchKernelGGL(gemm_tile_kernel<2>, tiles(128, 64), dim3(kTileThreads), 0, st, p, p.nib, (p.N + 63) / 64);
      break;
    case SmallTile::k128x128:
      hipLaunchKernelGGL(gemm_tile_kernel<4>, tiles(128, 128), dim3(kTileThreads), 0, st, p, p.nib, p.njb);
      break;
    case SmallTile::kNone: break;
    default: return launch_gemm_ring(p, tile, st);
  }
  return hipGetLastError();
}

}  // namespace fq
