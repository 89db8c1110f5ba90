// Fallback block GEMM for outputs that fit the chip in one round of 128 x 64, 128 x 128 or 128 x 256 tiles:
// wavefronts that only load, wavefronts that only multiply, and a ring of operand stages in LDS between them.
//
// Alg. 1 of the paper with the same accumulation order per output element as the other kernels (k ascending,
// main term then residual term, binary32 FMAs) and so the same bits.  The contraction is a list of items, the
// main product of k-block k and, where the tile's A block is flagged at k, its residual product.  An item is a
// stage of the ring: the A block (codes or residual codes) and the B blocks.  Four loaders, one per SIMD, bring
// the items by direct global -> LDS loads kS - 1 ahead of the multiplication, and keep the scales and slots of
// 128 k-blocks in LDS tables.  The others own 64 x 32 or 64 x 64 of the output each, take their operands from
// LDS half an item to an item ahead, and meet the loaders at one barrier per item, in its middle.
//
// Why so.  The multiplication alone (no loads, no LDS reads, no barrier) runs these tiles at the rate of the bare
// instruction stream, 2.4 POP/s.  What a k-loop adds is what wavefronts cannot issue meanwhile: a direct load
// holds its wavefront for some 30 cycles (1024 x 11008 x 4096, one 128 x 128 tile per compute unit, without
// flagged blocks: 60.0 us with the loads among the multiplication, 51.6 without them; 54.8 us with loaders, 46.5 without
// their loads), scalar bookkeeping at the barrier holds all of them at once (so the loaders do the bookkeeping), and two bodies of the
// loop made the compiler keep the accumulators twice (so there is one body: an operand is fetched right behind
// its last use, the accumulators are updated by an instruction that writes where it reads).  LDS reads are what
// is left: 6 KiB per 32 x 32 x 128 step for 64 x 32, 4 KiB for 64 x 64 (with loaders and without LDS reads 47.2 us).
// Measured, bf16 output, against the tiles of fq_gemm_tile.hip (us):
//   777 x 1544 x 2200, 5 % of the blocks flagged      10.5 ->  9.5   128 x 64, one per compute unit
//   512 x 4096 x 4096, 5 %                            18.9 -> 16.3   128 x 64, one per compute unit
//   2048 x 2048 x 2048, none / 20 %            15.4 -> 13.1, 18.8 -> 16.0   128 x 128
//   1024 x 11008 x 4096, 10 %                         69.8 -> 62.1   128 x 128
//   2048 x 4096 x 4096, 5 %                           46.8 -> 42.4   128 x 256
// A second round of tiles has nothing to hide its start and end behind, and two or three small workgroups on a
// compute unit do: from there on the kernels of fq_gemm_tile.hip are the faster ones; on contractions of a few k-blocks
// too, as nothing is multiplied here before the loaders have brought the first items (plan_small, fq_gemm.hip).
#include <atomic>
#include <type_traits>

#include "fq_device.h"
#include "fq_gemm_unit.h"
#include "fq_kernels.h"

namespace fq {

namespace {

constexpr int kMaxDevices = 64;   // per-device host-side caches
constexpr int kTab = 128;         // k-blocks whose scales and slots are in LDS

constexpr int kLoaders = 4;       // wavefronts that only load, one per SIMD

// kWR x kWC multiplying wavefronts of 64 rows x 32 kCG columns, kS stages; kOcc: wavefronts of a SIMD.  One tile is
// 128 rows: a residual item is work for all of its wavefronts or there is none.
template <int kWR_, int kWC_, int kCG_, int kS_, int kOcc_>
struct RingGeo {
  static constexpr int kWR = kWR_, kWC = kWC_;      // wavefronts along rows / columns
  static constexpr int kRG = 2, kCG = kCG_;         // 32-row / 32-column groups of a wavefront
  static constexpr int kS = kS_;                    // stages
  static constexpr int kOcc = kOcc_;
  static constexpr int kWaves = kWR * kWC, kThreads = 64 * (kWaves + kLoaders);
  static constexpr int kRows = kWR * kRG, kCols = kWC * kCG;      // groups of the tile
  static constexpr int kStageA = kRows * kFragRows, kStage = (kRows + kCols) * kFragRows;
  static constexpr int kLA = kRows * 4 / kLoaders, kLB = kCols * 4 / kLoaders, kL = kLA + kLB;   // 1 KiB loads of a loader
  static constexpr int kJB = (kCols + 3) / 4;       // quantization blocks across
  static_assert(kRows == 4, "one i-block");
  static constexpr int kUnits = kRG * kCG;
  static constexpr int kGroupN = 16 / kCols;    // tile columns per rasterization group: 512 columns, as
                                                   // wide as the rows that an XCD's 32 tiles then span are high
  static constexpr int kSA = 0, kRS = kTab, kSlot = 2 * kTab, kSB = 3 * kTab;     // dword offsets of the tables
  static constexpr int kLds = kS * kStage + (3 + kJB) * kTab * 4;
};

// s_waitcnt vmcnt(kVm) lgkmcnt(0)
template <int kVm>
__device__ __forceinline__ void wait_vm() {
  static_assert(kVm < 64);
  __builtin_amdgcn_s_waitcnt((kVm & 15) | (kVm >> 4) << 14 | 0x0070);
}

// Scalars worked out in front of this statement.
__device__ __forceinline__ void pin(int& a, int& b) {
  a = __builtin_amdgcn_readfirstlane(a);
  b = __builtin_amdgcn_readfirstlane(b);
  asm volatile("" : "+s"(a), "+s"(b));
}

// acc += t * f in place: the compiler's own choice has a destination of its own, and copies.
__device__ __forceinline__ void fma_in_place(float& acc, float t, float f) {
  asm volatile("v_fmac_f32_e32 %0, %1, %2" : "+v"(acc) : "v"(t), "v"(f));
}

// s_waitcnt lgkmcnt(0)
__device__ __forceinline__ void wait_lgkm0() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// One unit, a 32 x 32 sub-tile of one item, as `unit` of fq_gemm_unit.h with the scale in a vector register.
template <int kPar, class Extra>
__device__ __forceinline__ void ring_unit(v4i (&P)[2][4], const v4i (&b)[2][2], float (&acc)[16], const v4i (&a)[2][2],
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
      fma_in_place(acc[2 * n - 2], T[0], f);
      fma_in_place(acc[2 * n - 1], T[1], f);
      __builtin_amdgcn_sched_barrier(0);
    }
    T[0] = (float)P[kPar ^ 1][n >> 1][2 * (n & 1)];
    T[1] = (float)P[kPar ^ 1][n >> 1][2 * (n & 1) + 1];
    pin(T[0], T[1]);
    __builtin_amdgcn_sched_barrier(0);
  }
  fma_in_place(acc[14], T[0], f);
  fma_in_place(acc[15], T[1], f);
}

template <class G>
__global__ __launch_bounds__(G::kThreads, G::kOcc) void gemm_ring_kernel(GemmParams p, int tiles_i, int tiles_j) {
  extern __shared__ __attribute__((aligned(1024))) int8_t lds[];
  constexpr int kRG = G::kRG, kCG = G::kCG, kS = G::kS, kU = G::kUnits;
  float* const tab = reinterpret_cast<float*>(lds + kS * G::kStage);
  int* const tab_slot = reinterpret_cast<int*>(tab + G::kSlot);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nkb = p.nkb;
  int ti, tj;
  tile_at<G::kGroupN>(xcd_run(blockIdx.x, gridDim.x), tiles_i, tiles_j, ti, tj);
  const int rg0 = ti * G::kRows, cg0 = tj * G::kCols;       // first groups of the tile
  const int ib = rg0 >> 2;
  auto jb_of = [&](int group) { return min((cg0 + group) >> 2, p.njb - 1); };
  const bool has_fb = p.a_slot != nullptr;
  // which of the k-blocks of chunk c have a residual block, from the slots in LDS
  auto flags_of = [&](int c) -> unsigned long long {
    return has_fb ? __ballot(64 * c + lane < nkb && tab_slot[(c & 1) * 64 + lane] >= 0) : 0ull;
  };
  const int chunks = (nkb + 63) >> 6;

  if (w >= G::kWaves) {
    // ---- a loader: a quarter of every item's operands
    if (nkb == 0) return;
    __builtin_amdgcn_s_setprio(3);
    const int apart = (w - G::kWaves) * (G::kLA * 1024), bpart = (w - G::kWaves) * (G::kLB * 1024);
    const int8_t* const amain = p.a_codes + (int64_t)ib * nkb * kBlockBytes + (rg0 & 3) * kFragRows + apart;
    const int8_t* const ares = p.a_res + (rg0 & 3) * kFragRows + apart;
    const int8_t* const bmain = p.b_codes + (int64_t)jb_of(bpart / kFragRows) * nkb * kBlockBytes +
                                ((cg0 & 3) * kFragRows + bpart) % kBlockBytes;
    const uint32_t lds0 = lds_address(lds), tab0 = lds0 + kS * G::kStage;
    // tables: chunk c of 64 k-blocks in half c & 1 of each
    auto k_of = [&](int c) { return min(64 * c + lane, nkb - 1); };
    auto load_slots = [&](int c) {
      load_lds_dword(p.a_slot, (unsigned)(ib * p.a_si + k_of(c) * p.a_sk) * 4u, tab0 + (G::kSlot + (c & 1) * 64) * 4);
    };
    auto load_scales = [&](int c) {
      load_lds_dword(p.a_scales, (unsigned)(ib * p.a_si + k_of(c) * p.a_sk) * 4u, tab0 + (G::kSA + (c & 1) * 64) * 4);
#pragma unroll
      for (int j = 0; j < G::kJB; ++j)
        load_lds_dword(p.b_scales, (unsigned)(jb_of(4 * j) * p.b_sj + k_of(c) * p.b_sk) * 4u,
                       tab0 + (G::kSB + j * kTab + (c & 1) * 64) * 4);
    };
    auto load_residual_scales = [&](int c) {
      load_lds_dword(p.a_res_scales, (unsigned)max(tab_slot[(c & 1) * 64 + lane], 0) * 4u,
                     tab0 + (G::kRS + (c & 1) * 64) * 4);
    };
    // the next item to request: k-block k, residual or main
    int k = 0, res = 0, slots = -1;
    unsigned long long mask = 0;
    uint32_t wr = lds0;          // its stage
    auto enter_chunk = [&](int c) {
      if (!has_fb) return;
      slots = tab_slot[(c & 1) * 64 + lane];
      mask = flags_of(c);
      if (c > 1) load_residual_scales(c);
    };
    auto issue = [&]() {
      const int slot = __builtin_amdgcn_readlane(slots, k & 63);
      const int8_t* const src = (res ? ares : amain) + (int64_t)(res ? slot : k) * kBlockBytes;
      load_lds<G::kLA>(src, wr + apart, lane);
      const int8_t* const srcb = bmain + (int64_t)k * kBlockBytes;
      load_lds<(G::kLB > 4 ? 4 : G::kLB)>(srcb, wr + G::kStageA + bpart, lane);
      if constexpr (G::kLB > 4) load_lds<G::kLB - 4>(srcb + 4096, wr + G::kStageA + bpart + 4096, lane);
      wr = wr == lds0 + (kS - 1) * G::kStage ? lds0 : wr + G::kStage;
    };
    auto advance = [&]() {
      res = (int)(mask >> (k & 63)) & 1 & (res ^ 1);
      k += res ^ 1;
      if (!res && (k & 63) == 0 && k < nkb) enter_chunk(k >> 6);
    };
    if (has_fb) {
      load_slots(0);
      if (nkb > 64) load_slots(1);
    }
    issue();
    load_scales(0);
    if (nkb > 64) load_scales(1);
    if (has_fb) {
      wait_vm<G::kL + 1 + G::kJB>();
      asm volatile("" ::: "memory");
      enter_chunk(0);
      load_residual_scales(0);
      if (nkb > 64) load_residual_scales(1);
    }
    advance();
    int ahead = 0;               // items requested behind the current one
#pragma unroll
    for (int d = 1; d < kS; ++d)
      if (k < nkb) {
        issue();
        advance();
        ++ahead;
      }
    if (ahead == kS - 1) wait_vm<(kS - 1) * G::kL>();
    else wait_vm<0>();
    asm volatile("s_barrier" ::: "memory");
    for (int c = 0; c < chunks; ++c) {
      const int n = min(64, nkb - 64 * c) + (int)__popcll(flags_of(c));
      if (c > 0 && c + 1 < chunks) {        // the half of the tables that chunk c - 1 had
        if (has_fb) load_slots(c + 1);
        load_scales(c + 1);
      }
      for (int i = 0; i < n; ++i) {
        // item t + 1 has to be there, those behind it may be under way
        if (ahead == kS - 1) wait_vm<(kS - 2) * G::kL>();
        else wait_vm<0>();
        asm volatile("s_barrier" ::: "memory");
        if (k < nkb) {
          issue();
          advance();
        } else {
          --ahead;
        }
      }
    }
    wait_vm<0>();      // nothing may be under way into LDS when the workgroup ends
    return;
  }

  const int wr = w / G::kWC, wc = w % G::kWC;
  const int kg = lane >> 4, l15 = lane & 15;
  const int koff = (kg >> 1) * 1024 + (kg & 1) * 512;
  const int aoff = koff + l15 * 16 + wr * kRG * kFragRows;
  const int boff[2] = {koff + perm_col(l15, 0) * 16 + G::kStageA + wc * kCG * kFragRows,
                       koff + perm_col(l15, 1) * 16 + G::kStageA + wc * kCG * kFragRows};
  float acc[kRG][kCG][16];
  v4i a[kRG][2][2], b[kCG][2][2], P[2][4];
#pragma unroll
  for (int i = 0; i < kRG; ++i)
#pragma unroll
    for (int j = 0; j < kCG; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
  bool bad = false;

  if (nkb > 0) {
    asm volatile("s_barrier" ::: "memory");
    const int8_t* rd = lds;      // stage of the operands to fetch
    auto fetch_a = [&](int i, int h, int ks) {
      a[i][h][ks] = *reinterpret_cast<const v4i*>(rd + aoff + i * kFragRows + h * 256 + ks * 2048);
    };
    auto fetch_b = [&](int j, int h, int ks) {
      b[j][h][ks] = *reinterpret_cast<const v4i*>(rd + boff[h] + j * kFragRows + ks * 2048);
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) fetch_a(0, i >> 1, i & 1);
    if constexpr (kCG == 2) {
#pragma unroll
      for (int i = 0; i < 4; ++i) fetch_b(0, i >> 1, i & 1);
    } else {
      fetch_b(0, 0, 0);
      fetch_b(0, 1, 0);
    }
    const float* const tab_b = tab + G::kSB + (wc * kCG >> 2) * kTab;
    int k = 0, res = 0;
    unsigned long long mask = 0;
    float s = tab[G::kSA] * tab_b[0], sp = 0.0f, sa_n = 0.0f, sb_n = 0.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q) P[1][q] = v4i{0, 0, 0, 0};

    // Item t.  Its barrier lies in the middle: item t + 1 is in LDS, and everybody has the operands of item t
    // in registers, so that its stage can be written.
    auto step = [&]() {
      constexpr int kMid = kU / 2;
      auto run = [&](auto u_c) {
        constexpr int u = decltype(u_c)::value;
        constexpr int pu = (u + kU - 1) % kU;
        if constexpr (u == kMid) {
          wait_lgkm0();
          asm volatile("s_barrier" ::: "memory");
          rd = rd == lds + (kS - 1) * G::kStage ? lds : rd + G::kStage;
        }
        ring_unit<u & 1>(P, b[u % kCG], acc[pu / kCG][pu % kCG], a[u / kCG], u ? s : sp, [&](int n) {
          if constexpr (kCG == 2) {
            if (u == 0) {
              if (n < 4) fetch_b(1, n >> 1, n & 1);
              else fetch_a(1, (n >> 1) & 1, n & 1);
            }
            if (u == 2 && n < 4) fetch_a(0, n >> 1, n & 1);
            if (u == 3 && n < 4) fetch_b(0, n >> 1, n & 1);
          } else {
            if (u == 0) {
              if (n == 0) { fetch_b(0, 0, 1); fetch_b(0, 1, 1); }
              if (n == 1) { fetch_a(1, 0, 0); fetch_a(1, 1, 0); }
              if (n == 2) { fetch_a(1, 0, 1); fetch_a(1, 1, 1); }
            } else {
              if (n < 2) { fetch_a(0, 0, n); fetch_a(0, 1, n); }
              if (n == 4) fetch_b(0, 0, 0);
              if (n == 5) fetch_b(0, 1, 0);
            }
          }
          if (u == 0 && n == 3) {
            res = (int)(mask >> (k & 63)) & 1 & (res ^ 1);
            k += res ^ 1;
            pin(res, k);
          }
          if (u == kMid && n == 2) {
            sa_n = tab[(res ? G::kRS : G::kSA) + (k & (kTab - 1))];
            sb_n = tab_b[k & (kTab - 1)];
          }
        });
      };
      run(std::integral_constant<int, 0>{});
      run(std::integral_constant<int, 1>{});
      if constexpr (kU > 2) {
        run(std::integral_constant<int, 2>{});
        run(std::integral_constant<int, 3>{});
      }
      sp = s;
      s = sa_n * sb_n;
    };
    for (int c = 0; c < chunks; ++c) {
      mask = flags_of(c);
      if (has_fb) bad |= __ballot(64 * c + lane < nkb && tab_slot[(c & 1) * 64 + lane] == -2) != 0;
      const int n = min(64, nkb - 64 * c) + (int)__popcll(mask);
      for (int i = 0; i < n; ++i) step();
    }
#pragma unroll
    for (int e = 0; e < 16; ++e)
      acc[kRG - 1][kCG - 1][e] = __builtin_fmaf((float)P[1][e >> 2][e & 3], sp, acc[kRG - 1][kCG - 1][e]);
  }
#pragma unroll
  for (int i = 0; i < kRG; ++i)
#pragma unroll
    for (int j = 0; j < kCG; ++j)
      store_unit(p, acc[i][j], (rg0 + wr * kRG + i) * 32, (cg0 + wc * kCG + j) * 32, lane, bad);
}

template <class G>
hipError_t go(const GemmParams& p, hipStream_t st) {
  // the kernel needs more dynamic LDS than the default limit: raise it once per device
  static std::atomic<bool> attr_set[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) dev = 0;
  if (!attr_set[dev].load(std::memory_order_acquire)) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_ring_kernel<G>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, G::kLds);
    if (e != hipSuccess) return e;
    attr_set[dev].store(true, std::memory_order_release);
  }
  const int ti = (p.M + 32 * G::kRows - 1) / (32 * G::kRows), tj = (p.N + 32 * G::kCols - 1) / (32 * G::kCols);
  hipLaunchKernelGGL(gemm_ring_kernel<G>, dim3(ti * tj), dim3(G::kThreads), G::kLds, st, p, ti, tj);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_ring(const GemmParams& p, SmallTile tile, hipStream_t st) {
  switch (tile) {
    case SmallTile::kRing128x64: return go<RingGeo<2, 2, 1, 3, 4>>(p, st);      // two on a compute unit
    case SmallTile::kRing128x128: return go<RingGeo<2, 4, 1, 3, 3>>(p, st);
    case SmallTile::kRing128x256: return go<RingGeo<2, 4, 2, 3, 3>>(p, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fq
