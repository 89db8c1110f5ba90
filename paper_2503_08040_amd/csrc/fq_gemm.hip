// Fallback block GEMM on the gfx950 INT8 matrix cores.
//
// Paper: Sec. 4.2 Eq. (1) (INT8 x INT8 -> INT32 block product, dequantized by
// a^A a^B, FP32 accumulator), Sec. 4.3 Alg. 1 (k-loop on chip; for a flagged
// A block a second INT8 product with the residual codes against the same B
// block), Sec. 4.5 / App. C (the GEMM tile need not equal the quantization
// block).
//
// Shape of the kernel (differs from the paper's 128^3 CUDA tile on purpose):
//   - workgroup = 8 wavefronts (2 per SIMD), output tile 256 x 256 = 2 x 2
//     quantization blocks.  Wavefront (h, c) owns all 128 rows of i-block h and
//     the 64-column quarter c of the tile: 4 x 2 sub-tiles of 32 x 32, 128 FP32
//     accumulators per lane in architectural VGPRs (the vector ALU cannot read
//     accumulation registers, so the accumulators it updates must not live
//     there).  A second geometry, 1 x 3 blocks (128 x 384, 2 x 3 sub-tiles per
//     wavefront), covers the last block columns or rows when the 2 x 2 tiles
//     would leave the final round of the chip mostly idle;
//   - the k-loop runs over "items": the main product of k-block k and, when
//     one of the tile's A blocks is flagged at k, a residual item right
//     after it.  A and B operands sit in two double-buffered LDS rings (64 KiB
//     each for 2 x 2) that advance with k; the residual
//     product re-uses the B blocks already on chip exactly as Alg. 1 says.
//     The residual A blocks have 32 KiB of their own.
//     A residual item is work only for the wavefronts whose i-block is flagged
//     at that k: the others wait at the barrier behind it, so with one of
//     the two blocks flagged the item runs on one wavefront per SIMD and costs
//     half of a full item;
//   - operands reach LDS by direct global->LDS 16-byte loads (blocks are stored
//     in operand order, see fq.h), one barrier per k-block and one more where
//     there are residual blocks;
//   - per 32 x 32 sub-tile: 8 v_mfma_i32_16x16x64_i8 (four 16 x 16 quadrants x
//     two halves of K = 128) into an INT32 tile, then one convert + one FMA per
//     element folds it into the FP32 accumulators with the scalar scale of that
//     block pair.  (The 16x16x64 form sustains a third more than 32x32x32 on this
//     part and leaves the dequantizing pipeline about 10 % faster.)
// The accumulation order per output element is exactly Alg. 1's (k ascending,
// main term then residual term) in both geometries, so results match a
// sequential evaluation bit for bit and do not depend on the tile plan.  Outputs too small for a chip's
// worth of these tiles are computed by the kernels of fq_gemm_tile.hip and fq_gemm_ring.hip, also bit for bit.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <type_traits>

#include "fq_device.h"
#include "fq_gemm_unit.h"
#include "fq_kernels.h"

// Ablation switches (measurement support; the library itself is built with none of them, and a
// build with one computes wrong products on purpose).  Each removes or adds one component of the
// k-loop so that its cost can be read off a timing of the whole kernel:
//   FQ_ABLATE_NO_DMA        no global -> LDS loads (the rings keep whatever they hold)
//   FQ_ABLATE_NO_MULTIPLY   no wavefront multiplies: loads, waits, barriers and epilogue only
//   FQ_ABLATE_NO_DEQUANT    the MFMAs and their LDS reads, without the converts and FMAs
//   FQ_ABLATE_EXTRA_SALU=n  n dependent scalar additions behind every barrier of the k-loop
//   FQ_ABLATE_DMA_HOT       every global -> LDS load reads from the first MiB of the A codes (which
//                           must be that large), so that all of them hit the L2
//   FQ_ABLATE_ONE_STAGER    wavefronts 0-3 (one per SIMD) issue all loads, 16 each, 4-7 none
//   FQ_ABLATE_TEAM_SKEW     (computes the right products) the two wavefronts of a SIMD half an item
//                           apart in the 2 x 2 geometry: the wavefronts of i-block 0 and of i-block
//                           1 form two teams with two barriers per item, each the item boundary of
//                           one team and the middle of the item of the other; a team loads its own
//                           A block, team 0 the B blocks as well.  The B operands of an item sit in
//                           registers after its first two units, which is why two ring slots still
//                           suffice.
namespace fq {

namespace {

constexpr int kThreads = 512;
constexpr int kMaxDevices = 64;   // per-device host-side caches
constexpr int kGroupN = 4;    // tile columns per rasterization group
constexpr int kRingBytes = 2 * kBlockBytes;     // one A pair or one B pair
constexpr int kLdsBytes = 5 * kRingBytes;       // all 160 KiB: two A sets, two B sets, the residual blocks of an
                                                // A set; the epilogue staging patches re-use the same memory

// One wavefront copies 4 KiB (4 fragments) global -> LDS with direct loads.  `src` and `lds_dst` are
// wave-uniform; the per-lane part of the address is the 32-bit offset lane*16 (scalar-base form), and
// the 4 loads share one base and differ only in the instruction offset.  Written as assembly (the
// loads have no register results) because the compiler counts the builtin as an access to both memories
// of unknown order: with one in flight every wait for an LDS read became a wait for all of them, the
// ones issued just before included.  Whoever reads the LDS waits with s_waitcnt vmcnt(0) and a barrier.
// 8192^3 with a fifth of the blocks flagged 678 -> 665 us, 4096 x 4096 x 11008 220.6 -> 217.5.
__device__ __forceinline__ void stage_quarter_block(const int8_t* src, uint32_t lds_dst, int lane) {
#ifdef FQ_ABLATE_NO_DMA
  if (lane >= 0) return;
#endif
  static_assert(kFragBytes == 1024);
  load_lds<4>(src, lds_dst, lane);
}
// 8 KiB
__device__ __forceinline__ void stage_half_block(const int8_t* src, uint32_t lds_dst, int lane) {
  stage_quarter_block(src, lds_dst, lane);
  stage_quarter_block(src + 4 * kFragBytes, lds_dst + 4 * kFragBytes, lane);
}

// two floats -> two bf16 (round-to-nearest-even) in one dword, low half first
__device__ inline int pack_bf16x2(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  f32x2 v = {a, b};
  return __builtin_bit_cast(int, __builtin_convertvector(v, bf16x2));
}

// One operand of v_mfma_i32_16x16x64_i8 out of a block stored in tile order: rows (or
// columns) [32 rg + 16 rh, +16), contraction [64 ks, +64).  Lane l supplies row l % 16 and the
// 16 contraction-contiguous bytes of group l / 16, i.e. the bytes at tile_offset(row, 64 ks +
// 16 (l / 16)): whole 256-byte runs per 16 lanes, conflict-free.  The order of the contraction
// inside the instruction does not matter as long as both operands use the same one.
__device__ inline v4i lds_frag(const int8_t* blk, int rg, int rh, int ks, int lane) {
  return *reinterpret_cast<const v4i*>(blk + ((rg * 4 + ks * 2) * 64 + rh * 16) * 16 +
                                       (lane + 16 * (lane >> 4)) * 16);
}


// acc += s * t, s uniform.
__device__ __forceinline__ void fma_in_place(float& acc, float s, float t) {
  asm volatile("v_fmac_f32_e32 %0, %1, %2" : "+v"(acc) : "s"(s), "v"(t));
}

// Geometry of a workgroup tile: kBI x kBJ quantization blocks, computed by 8 wavefronts laid
// out 2 (row halves h) x 4 (column groups c).  Wavefront (h, c) owns rows [64h, 64h+64) of every
// i-block of the tile and the 32*kBJ columns starting at 32*kBJ*c: kSI x kSJ sub-tiles of
// 32 x 32.  Two geometries are used: 2 x 2 blocks (256 x 256, 8 sub-tiles per wavefront) for
// the bulk of the output and 1 x 3 blocks (128 x 384, 6 sub-tiles) for the columns left over
// when the 2 x 2 tiles do not fill a whole number of rounds of the chip (see launch_gemm).
template <int kBI_, int kBJ_>
struct Geo {
  static constexpr int kBI = kBI_, kBJ = kBJ_;
  static constexpr int kSI = 2 * kBI;        // 32-row groups per wavefront
  static constexpr int kSJ = kBJ;            // 32-column groups per wavefront
  static constexpr int kUnits = kSI * kSJ;   // sub-tiles per wavefront and item
  static constexpr int kASet = kBI * kBlockBytes;   // the A blocks of one item in LDS
  static constexpr int kBSet = kBJ * kBlockBytes;   // the B blocks of one k-block in LDS
  // A wavefront's columns lie in one j-block when kBJ = 2 and in up to two when kBJ = 3, so the
  // scale of a sub-tile depends on sj only in the second case.
  static constexpr int kSC = (kBJ == 2) ? 1 : kSJ;  // distinct scale columns per i-block
  static constexpr int kSP = (kBJ == 2) ? 1 : 2;    // distinct scales of an item's last two units
  static constexpr int kStageCols = 32 * kSJ;
  static constexpr int kStagePitch = kStageCols + 4;   // floats per staged row: 4 rows apart = 16 banks apart
  static constexpr int kStageBytesPerWave = 32 * kStagePitch * 4;
  // Rows of a wavefront.  With two i-blocks per tile, wavefront half h owns all 128 rows of
  // i-block h (so that a residual item of one flagged block is work for that half of the
  // wavefronts only); with one i-block it owns rows [64h, 64h+64) of it.  si counts the
  // wavefront's 32-row groups: its i-block and its row group inside that block.
  __device__ static constexpr int a_block(int h, int /*si*/) { return kBI == 2 ? h : 0; }
  __device__ static constexpr int a_group(int h, int si) { return kBI == 2 ? si : 2 * h + si; }
  static_assert(3 * kASet + 2 * kBSet <= kLdsBytes, "operand rings and residual blocks must fit");
  static_assert(8 * kStageBytesPerWave <= kLdsBytes, "epilogue staging must fit");
  static_assert(kBI + kBJ == 4, "8 wavefronts stage 8 half-blocks per item");
};

// Per-wavefront register state of the k-loop.
template <class G>
struct WaveState {
  // FP32 accumulators: sub-tile (si, sj), 16 elements per lane; element 4 q + r belongs to
  // quadrant q = 2 rh + ch of the sub-tile: row 16 rh + 4 (lane / 16) + r, column 16 ch + lane % 16
  float acc[G::kSI][G::kSJ][16];
  v4i aq[2][2][2];                 // A operands [rh][ks] of two consecutive si: si uses aq[si & 1]
  v4i bq[G::kSJ][2][2];            // B operands [ch][ks] of this wave's column groups
  v4i P[2][4];                     // INT32 quadrants: sub-tile u accumulates into P[u & 1]
  float T[2];                      // elements converted in the previous slot, waiting for their FMA
};

// Scales of one item as this wavefront's units see them: s[sc] = a^A (or a~^A) of the
// wavefront's i-block times a^B of the j-block that scale column sc lies in.
template <class G>
struct ItemScales {
  float s[G::kSC];
};

// The k-loop is one continuous software pipeline over sub-tiles ("units": u = kSJ*si + sj).
// A unit is 8 slots.  Slot n issues one v_mfma_i32_16x16x64_i8 of unit u: contraction half
// ks = n / 4 of quadrant q = n % 4 (q = 2 rh + ch: row half rh, column half ch of the 32 x 32
// sub-tile), so the two MFMAs that accumulate into the same quadrant are four slots apart.  In
// the 16 cycles the matrix core needs for it the slot also issues 4 vector-ALU instructions that
// fold the finished INT32 tile of unit u-1 into the FP32 accumulators: the 2 FMAs of the
// elements converted one slot earlier, then the 2 converts of elements 2n, 2n+1.  An FMA never
// waits for its convert, and a convert reads a quadrant whose last MFMA is at least four slots
// old.  Operand registers are refilled from LDS well before their next use: the A operands of
// si+1 are fetched into a second register buffer while si is being multiplied (LDS latency
// under load is several hundred cycles), and the last two units fetch the B operands and the
// first A operands of the NEXT item (a B operand right after its last use), so that no item
// starts with a burst of LDS reads.  Scheduling fences pin this order.
//   a_cur: A set of the current item in LDS; a_nxt / b_nxt: A set / B set of the next item.
//   sc: scales of the current item; sp: scales of the previous item's last two units.
//   h, c: this wavefront's row half and column group.
//   kBiased: the tolerance variant (see gemm_biased_kernel): the first MFMA of a quadrant starts
//   from `magic` (the bit pattern of 1.25 * 2^23 in every element) instead of zero, so that the
//   finished INT32 value, read as binary32, IS 1.25 * 2^23 + P, exactly; the slot then issues only
//   the 2 FMAs of elements 2n, 2n+1 of unit u-1 straight from that tile and no converts.
template <class G, int u, bool kBiased>
__device__ __forceinline__ void run_unit(WaveState<G>& st, const int8_t* a_cur, const int8_t* a_nxt,
                                         const int8_t* b_nxt, int h, int c, int lane,
                                         const ItemScales<G>& sc, const float (&sp)[G::kSP],
                                         const v4i& magic) {
  constexpr int kSJ = G::kSJ, kUnits = G::kUnits;
  constexpr int si = u / kSJ, sj = u % kSJ;
  // B operand (ch, ks) of column group cg = kSJ*c + j of the tile: block cg / 4, group cg % 4
  auto b_frag = [&](int j, int ch, int ks) {
    const int cg = kSJ * c + j;
    return lds_frag(b_nxt + (cg >> 2) * kBlockBytes, cg & 3, ch, ks, lane);
  };
#pragma unroll
  for (int n = 0; n < 8; ++n) {
    const int ks = n >> 2, rh = (n >> 1) & 1, ch = n & 1, q = 2 * rh + ch;
    {
      const v4i z = {0, 0, 0, 0};
      st.P[u & 1][q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
          st.aq[si & 1][rh][ks], st.bq[sj][ch][ks], ks ? st.P[u & 1][q] : (kBiased ? magic : z), 0, 0, 0);
      // B operand (ch, ks) was used for the last time in the slot with rh = 1
      const bool b_done = rh == 1;
      // the other four slots (rh = 0) carry a load each into a free buffer: operand i = 0..3
      const int i = 2 * ks + ch, irh = i >> 1, iks = i & 1;
      // A operands of the next si go into the other aq buffer a whole unit before their use.  Unit 0
      // starts its reads two slots later: at its first MFMA the compiler waits for every read in flight
      // (two paths lead here), and one issued just before would be waited for in full
      // (4096 x 16384 x 4096 271 -> 266 us)
      if (si + 1 < G::kSI && sj == 0 && (u == 0 ? b_done : !b_done))
        st.aq[(si + 1) & 1][irh][iks] = lds_frag(a_cur + G::a_block(h, si + 1) * kBlockBytes,
                                                 G::a_group(h, si + 1), irh, iks, lane);
      // the last two units (same si, odd: they use aq[1]) fetch the next item's first operands
      if (u == kUnits - 2) {
        if (b_done) st.bq[sj][ch][ks] = b_frag(sj, ch, ks);
        else st.aq[0][irh][iks] = lds_frag(a_nxt + G::a_block(h, 0) * kBlockBytes,
                                           G::a_group(h, 0), irh, iks, lane);
      }
      if (u == kUnits - 1) {
        if (b_done) st.bq[sj][ch][ks] = b_frag(sj, ch, ks);
        else if (kSJ == 3) st.bq[0][irh][iks] = b_frag(0, irh, iks);
      }
      pin(st.P[u & 1][q]);
    }
    __builtin_amdgcn_sched_barrier(0);   // MFMA first: its destination must not alias live tiles
#ifndef FQ_ABLATE_NO_DEQUANT
    if constexpr (kBiased) {
      constexpr int kLastSi = G::kSI - 1;
      constexpr int fu = u - 1;
      constexpr bool prev = fu < 0;                     // the last unit of the previous item
      constexpr int pu = fu + kUnits;
      constexpr int fsi = prev ? kLastSi : fu / kSJ, fsj = prev ? pu % kSJ : fu % kSJ;
      const float s = prev ? sp[G::kSP - 1] : sc.s[G::kSC == 1 ? 0 : fsj];
      const int fe = 2 * n;
      st.acc[fsi][fsj][fe] = __builtin_fmaf(
          __int_as_float(st.P[(u - 1) & 1][n >> 1][2 * (n & 1)]), s, st.acc[fsi][fsj][fe]);
      st.acc[fsi][fsj][fe + 1] = __builtin_fmaf(
          __int_as_float(st.P[(u - 1) & 1][n >> 1][2 * (n & 1) + 1]), s, st.acc[fsi][fsj][fe + 1]);
      pin(st.acc[fsi][fsj][fe], st.acc[fsi][fsj][fe + 1]);
      __builtin_amdgcn_sched_barrier(0);
    } else {
      // FMAs of the 2 elements converted in the previous slot (unit u-1, or u-2 for n = 0);
      // negative units are the last two units of the previous item
      constexpr int kLastSi = G::kSI - 1;
      const int fu = n ? u - 1 : u - 2, fe = n ? 2 * (n - 1) : 14;
      const bool prev = fu < 0;
      const int pu = fu + kUnits;                       // unit index in the previous item
      const int fsi = prev ? kLastSi : fu / kSJ, fsj = prev ? pu % kSJ : fu % kSJ;
      const float s = prev ? sp[G::kSP == 1 ? 0 : pu - (kUnits - 2)]
                           : sc.s[G::kSC == 1 ? 0 : fsj];
      fma_in_place(st.acc[fsi][fsj][fe], s, st.T[0]);
      fma_in_place(st.acc[fsi][fsj][fe + 1], s, st.T[1]);
    }
    if constexpr (!kBiased) {
      __builtin_amdgcn_sched_barrier(0);   // FMAs before converts
      st.T[0] = (float)st.P[(u - 1) & 1][n >> 1][2 * (n & 1)];
      st.T[1] = (float)st.P[(u - 1) & 1][n >> 1][2 * (n & 1) + 1];
      pin(st.T[0], st.T[1]);
      __builtin_amdgcn_sched_barrier(0);
    }
#endif
  }
}

// Units [kFrom, kTo) of one item, in order.
template <class G, int kFrom, int kTo, bool kBiased>
__device__ __forceinline__ void run_units_range(WaveState<G>& st, const int8_t* a_cur,
                                                const int8_t* a_nxt, const int8_t* b_nxt, int h,
                                                int c, int lane, const ItemScales<G>& sc,
                                                const float (&sp)[G::kSP], const v4i& magic) {
  if constexpr (kFrom < kTo) {
    run_unit<G, kFrom, kBiased>(st, a_cur, a_nxt, b_nxt, h, c, lane, sc, sp, magic);
    run_units_range<G, kFrom + 1, kTo, kBiased>(st, a_cur, a_nxt, b_nxt, h, c, lane, sc, sp, magic);
  }
}

// Folds the last two units of the last item (scales sp) into the accumulators.
template <class G, bool kBiased>
__device__ __forceinline__ void drain(WaveState<G>& st, const float (&sp)[G::kSP]) {
  constexpr int kLastSi = G::kSI - 1, kSJ = G::kSJ, kP = (G::kUnits - 1) & 1;
  if constexpr (kBiased) {      // only the last unit is pending: all 16 elements of its biased tile
    const float s = sp[G::kSP - 1];
#pragma unroll
    for (int e = 0; e < 16; ++e)
      st.acc[kLastSi][kSJ - 1][e] =
          __builtin_fmaf(__int_as_float(st.P[kP][e >> 2][e & 3]), s, st.acc[kLastSi][kSJ - 1][e]);
    return;
  }
#pragma unroll
  for (int n = 0; n < 8; ++n) {
    const int fsj = n ? kSJ - 1 : kSJ - 2, fe = n ? 2 * (n - 1) : 14;
    const float s = sp[G::kSP == 1 ? 0 : (n ? 1 : 0)];
    st.acc[kLastSi][fsj][fe] = __builtin_fmaf(st.T[0], s, st.acc[kLastSi][fsj][fe]);
    st.acc[kLastSi][fsj][fe + 1] = __builtin_fmaf(st.T[1], s, st.acc[kLastSi][fsj][fe + 1]);
    st.T[0] = (float)st.P[kP][n >> 1][2 * (n & 1)];
    st.T[1] = (float)st.P[kP][n >> 1][2 * (n & 1) + 1];
  }
  const float s = sp[G::kSP - 1];
  st.acc[kLastSi][kSJ - 1][14] = __builtin_fmaf(st.T[0], s, st.acc[kLastSi][kSJ - 1][14]);
  st.acc[kLastSi][kSJ - 1][15] = __builtin_fmaf(st.T[1], s, st.acc[kLastSi][kSJ - 1][15]);
}

// Scalars of one k-block as a wavefront needs them: whether its own A block is flagged (bit 0) and whether any
// of the tile's is (bit 1), the residual slot of the A block it stages (-1: none, or it stages B), and per scale
// column of its own i-block a^A a^B and a~^A a^B, as bit patterns (a choice between floats would be made by the
// vector unit).
template <class G>
struct KRec {
  int flags, slot;
  int s[G::kSC], t[G::kSC];
};

// The same of 64 consecutive k-blocks, one per lane (flags: one per bit).  Read back with v_readlane
// they cost the k-loop no scalar loads.  Those shared the LDS reads' counter and come back in any
// order, so every item waited for the youngest of them at its first LDS read, and where a transposed
// operand's scales are a row of the grid apart each was a miss.  4096 x 11008 x 4096 as NN 203.6 ->
// 196.5 us, 4096 x 16384 x 4096 as TN 301 -> 291, 8192^3 (NT, a fifth of the blocks flagged) 712 -> 704.
template <class G>
struct KChunk {
  int flags, slot;
  float s[G::kSC], t[G::kSC];
};

}  // namespace

namespace {

// One output tile of geometry G whose first blocks are (ib_first, jb_first).  Blocks beyond
// the matrix repeat the last valid one (their products are never stored).
// kBiased: the tolerance variant.  Every item adds (1.25 * 2^23 + P) * s instead of P * s to the
// accumulators; the wavefront keeps the sum of the scales it has used per scale column and,
// after every kBiasWindow items it took part in (and at the end), folds the pending unit and
// subtracts 1.25 * 2^23 times that sum with one FMA per accumulator.  The window bounds the
// magnitude the accumulators carry, and with it the rounding error of the additions, whatever K.
constexpr int kBiasWindow = 4;
constexpr int kMagicBits = 0x4B200000;          // 1.25 * 2^23 as binary32: with |P| <= 128 * 127^2 < 2^21 the sum
                                                // stays inside [2^23, 2^24), where one ulp is 1
constexpr float kMagic = 10485760.0f;

#ifdef FQ_ABLATE_EXTRA_SALU
__device__ __forceinline__ void extra_salu(int chain) {
#pragma unroll
  for (int i = 0; i < FQ_ABLATE_EXTRA_SALU; ++i) asm volatile("s_add_i32 %0, %0, 1" : "+s"(chain));
  asm volatile("" ::"s"(chain));
}
#endif

// Where the residual blocks of the tile's A blocks lie in LDS.
template <class G>
constexpr int kResOffset = 2 * (G::kASet + G::kBSet);

template <class G, bool kBiased, bool kFb = true>
__device__ __forceinline__ void tile_body(const GemmParams& p, int ib_first, int jb_first,
                                          int8_t* lds) {
  constexpr int kBI = G::kBI, kBJ = G::kBJ, kSI = G::kSI, kSJ = G::kSJ, kUnits = G::kUnits;
#ifdef FQ_ABLATE_TEAM_SKEW
  constexpr bool kSkew = kBI == 2 && kBJ == 2;
#else
  constexpr bool kSkew = false;
#endif
  int8_t* const a_ring = lds;                    // [2][kBI blocks]
  int8_t* const b_ring = lds + 2 * G::kASet;     // [2][kBJ blocks]

  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = w >> 2, c = w & 3;

  int ib[kBI], jbt[kBJ];
#pragma unroll
  for (int i = 0; i < kBI; ++i) ib[i] = min(ib_first + i, p.nib - 1);
#pragma unroll
  for (int j = 0; j < kBJ; ++j) jbt[j] = min(jb_first + j, p.njb - 1);
  // the (up to two) j-blocks this wave's columns lie in, as indices into the tile's blocks
  const int jlo = (kSJ * c) >> 2, jhi = (kSJ * c + kSJ - 1) >> 2;

  // ---- what this wave stages: 8 KiB (half a block) per item; the first 2*kBI waves the A
  // blocks, the others the B blocks
#ifdef FQ_ABLATE_ONE_STAGER
  const bool stager = w < 4;                      // whole blocks: A blocks first, then B blocks
  const bool stage_a = w < kBI;
  const int sidx = stage_a ? w : (w - kBI) & 3;
  const int spart = 0;
#else
  const bool stage_a = w < 2 * kBI;
  const int sidx = stage_a ? (w >> 1) : ((w - 2 * kBI) >> 1);   // which block of the set
  const int spart = (w & 1) * (kBlockBytes / 2);
#endif
  int sblk = 0;
#pragma unroll
  for (int i = 0; i < kBI; ++i) if (stage_a && sidx == i) sblk = ib[i];
#pragma unroll
  for (int j = 0; j < kBJ; ++j) if (!stage_a && sidx == j) sblk = jbt[j];
  const int soff = sidx * kBlockBytes + spart;
  const int8_t* const smain = (stage_a ? p.a_codes : p.b_codes) +
                              (int64_t)sblk * p.nkb * kBlockBytes + spart;

  const bool has_fb = kFb && p.a_slot != nullptr;
  int ia[kBI];
#pragma unroll
  for (int i = 0; i < kBI; ++i) ia[i] = ib[i] * p.a_si;
  int jlo_blk = jbt[0], jhi_blk = jbt[0];
#pragma unroll
  for (int j = 0; j < kBJ; ++j) {
    if (jlo == j) jlo_blk = jbt[j];
    if (jhi == j) jhi_blk = jbt[j];
  }
  const int ibj_lo = jlo_blk * p.b_sj, ibj_hi = jhi_blk * p.b_sj;
  const int nkb = p.nkb;

  bool poison = false;           // this wavefront's i-block has a flagged block without a slot
  KChunk<G> kc;
  auto load_chunk = [&](int k0) {
    const int k = min(k0 + lane, nkb - 1);
    const bool in = k0 + lane < nkb;
    int slot[kBI], ia_own = ia[0];
#pragma unroll
    for (int i = 0; i < kBI; ++i) {
      slot[i] = -1;
      if (has_fb) slot[i] = p.a_slot[ia[i] + k * p.a_sk];
      if (G::a_block(h, 0) == i) ia_own = ia[i];
    }
    const float sa = p.a_scales[ia_own + k * p.a_sk];
    float sb[G::kSC];
#pragma unroll
    for (int q = 0; q < G::kSC; ++q)
      sb[q] = p.b_scales[((G::kSC > 1 && ((kSJ * c + q) >> 2) != jlo) ? ibj_hi : ibj_lo) + k * p.b_sk];
    int own = slot[0];
#pragma unroll
    for (int i = 1; i < kBI; ++i) if (G::a_block(h, 0) == i) own = slot[i];
    const float rs = has_fb ? p.a_res_scales[max(own, 0)] : 0.0f;
    kc.slot = -1;
    int any = -1;
#pragma unroll
    for (int i = 0; i < kBI; ++i) {
      any = max(any, slot[i]);
      if (kSkew ? h == i : stage_a && sidx == i) kc.slot = slot[i];
    }
    kc.flags = kFb && in ? (own >= 0 ? 1 : 0) | (any >= 0 ? 2 : 0) : 0;
    if (kFb) poison |= __ballot(in && own == -2) != 0;
#pragma unroll
    for (int q = 0; q < G::kSC; ++q) {
      kc.s[q] = sa * sb[q];
      kc.t[q] = rs * sb[q];
    }
  };
  auto lane_bits = [](float v, int l) { return __builtin_amdgcn_readlane(__float_as_int(v), l); };
  // k in the chunk that is loaded; behind the last k-block flags and slot mean nothing
  auto rec_of = [&](int k) -> KRec<G> {
    KRec<G> r;
    r.flags = kFb ? __builtin_amdgcn_readlane(kc.flags, k & 63) : 0;
    r.slot = kFb ? __builtin_amdgcn_readlane(kc.slot, k & 63) : -1;
#pragma unroll
    for (int q = 0; q < G::kSC; ++q) {
      r.s[q] = lane_bits(kc.s[q], k & 63);
      r.t[q] = kFb ? lane_bits(kc.t[q], k & 63) : 0;
    }
    return r;
  };
  // This wave's 8 KiB share of k-block k into its ring, or of residual slot `slot` behind the rings.
  auto stage_share = [&](const int8_t* src, uint32_t dst) {
#ifdef FQ_ABLATE_ONE_STAGER
    if (!stager) return;
#endif
#ifdef FQ_ABLATE_DMA_HOT
    src = p.a_codes + (reinterpret_cast<uintptr_t>(src) & 0xFE000u);
#endif
    stage_half_block(src, dst, lane);
#ifdef FQ_ABLATE_ONE_STAGER
    stage_half_block(src + kBlockBytes / 2, dst + kBlockBytes / 2, lane);
#endif
  };
  const uint32_t lds0 = lds_address(lds);
  const uint32_t my_ring = lds0 + (stage_a ? 0 : 2 * G::kASet) + soff;
  const int my_set = stage_a ? G::kASet : G::kBSet;
  auto stage_main = [&](int k) { stage_share(smain + (int64_t)k * kBlockBytes, my_ring + (k & 1 ? my_set : 0)); };
  auto stage_res = [&](int slot) {
    stage_share(p.a_res + (int64_t)slot * kBlockBytes + spart, lds0 + kResOffset<G> + soff);
  };
  // kSkew: this wavefront's share of item (k, res) when the two teams (h = 0, 1: the wavefronts
  // of i-block h, one per SIMD each) run half an item apart: a quarter of its own team's A block,
  // and for team 0 half a B block as well.
  auto stage_team = [&](int k, int res, const KRec<G>& r, int asel, bool new_b) {
    int blk = ib[0];
#pragma unroll
    for (int i = 1; i < kBI; ++i) if (h == i) blk = ib[i];
    const int quarter = c * (kBlockBytes / 4);
    const uint32_t dst = lds_address(a_ring) + asel * G::kASet + h * kBlockBytes + quarter;
    if (!res) stage_quarter_block(p.a_codes + ((int64_t)blk * p.nkb + k) * kBlockBytes + quarter, dst, lane);
    else if (r.slot >= 0) stage_quarter_block(p.a_res + (int64_t)r.slot * kBlockBytes + quarter, dst, lane);
    if (h == 0 && new_b) {
      int jb = jbt[0];
#pragma unroll
      for (int j = 1; j < kBJ; ++j) if ((c >> 1) == j) jb = jbt[j];
      const int part = (c >> 1) * kBlockBytes + (c & 1) * (kBlockBytes / 2);
      stage_half_block(p.b_codes + ((int64_t)jb * p.nkb + k) * kBlockBytes + (c & 1) * (kBlockBytes / 2),
                       lds_address(b_ring) + (k & 1) * G::kBSet + part, lane);
    }
  };
  WaveState<G> st;
#pragma unroll
  for (int si = 0; si < kSI; ++si)
#pragma unroll
    for (int sj = 0; sj < kSJ; ++sj)
#pragma unroll
      for (int r = 0; r < 16; ++r) st.acc[si][sj][r] = 0.0f;
  v4i magic = {kMagicBits, kMagicBits, kMagicBits, kMagicBits};
  if (kBiased) asm volatile("" : "+v"(magic));   // stays in registers: an MFMA operand cannot be a literal
  float bias_s[G::kSC];          // kBiased: sum of the scales used since the bias was last removed
#pragma unroll
  for (int q = 0; q < G::kSC; ++q) bias_s[q] = 0.0f;
  int bias_items = 0;
  // removes the bias accumulated so far; the pipeline must have been drained
  auto remove_bias = [&]() {
#pragma unroll
    for (int si = 0; si < kSI; ++si)
#pragma unroll
      for (int sj = 0; sj < kSJ; ++sj)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          st.acc[si][sj][e] = __builtin_fmaf(bias_s[G::kSC == 1 ? 0 : sj], -kMagic, st.acc[si][sj][e]);
#pragma unroll
    for (int q = 0; q < G::kSC; ++q) bias_s[q] = 0.0f;
    bias_items = 0;
  };

  if (nkb > 0) {
    // ---- prologue: k-blocks 0 and 1 into the two ring slots, and the residual blocks of k-block 0
    int k = 0, res = 0;
    [[maybe_unused]] int t = 0;
    KRec<G> r0{}, r1;      // k-blocks k and k + 1
    if constexpr (kSkew) stage_team(0, 0, r0, 0, true);
    else stage_main(0);
    load_chunk(0);
    r0 = rec_of(0);
    r1 = rec_of(1);
    if constexpr (kSkew) {
      if (r0.flags) stage_team(0, 1, r0, 1, false);
      else if (1 < nkb) stage_team(1, 0, r1, 1, true);
    } else {
      if (r0.slot >= 0) stage_res(r0.slot);
      if (1 < nkb) stage_main(1);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);    // vmcnt(0): this wave's direct-to-LDS loads landed
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      st.aq[0][i >> 1][i & 1] = lds_frag(a_ring + G::a_block(h, 0) * kBlockBytes, G::a_group(h, 0),
                                         i >> 1, i & 1, lane);
#pragma unroll
      for (int j = 0; j < kSJ; ++j) {
        const int cg = kSJ * c + j;
        st.bq[j][i >> 1][i & 1] =
            lds_frag(b_ring + (cg >> 2) * kBlockBytes, cg & 3, i >> 1, i & 1, lane);
      }
    }
#pragma unroll
    for (int qd = 0; qd < 4; ++qd) st.P[1][qd] = v4i{0, 0, 0, 0};
    st.T[0] = st.T[1] = 0.0f;
    float sp[G::kSP];                      // scales of the previous item's last two units
#pragma unroll
    for (int i = 0; i < G::kSP; ++i) sp[i] = 0.0f;

    auto after_units = [&](const ItemScales<G>& sc) {
#pragma unroll
      for (int i = 0; i < G::kSP; ++i) sp[i] = sc.s[G::kSC == 1 ? 0 : kSJ - 2 + i];
      if constexpr (kBiased) {
#pragma unroll
        for (int q = 0; q < G::kSC; ++q) bias_s[q] += sc.s[q];
        if (++bias_items == kBiasWindow) {
          // fold the pending unit, take the bias out, and restart the pipeline: the next unit 0
          // folds the same tile again with scale 0, which adds nothing
          drain<G, true>(st, sp);
          remove_bias();
#pragma unroll
          for (int i = 0; i < G::kSP; ++i) sp[i] = 0.0f;
        }
      }
    };
    auto next_k = [&]() {
      ++k;
      r0 = r1;
      if (__builtin_expect(((k + 1) & 63) == 0, 0)) {
        if (k + 1 < nkb) load_chunk(k + 1);
      }
      r1 = rec_of(k + 1);
    };
#ifdef FQ_ABLATE_NO_MULTIPLY
    const bool multiply = p.M < 0;
#else
    constexpr bool multiply = true;
#endif
    if constexpr (!kSkew) {
      // One turn is the main product of k-block k or, for the wavefronts whose i-block is flagged at k, its
      // residual product behind it: the same code, with the A operands from the residual blocks instead of the
      // ring and without the ring's barrier.  The end of a k-block with residual blocks is one more barrier, which the
      // wavefronts without one go to at once, and behind which its B blocks and the residual blocks may be
      // overwritten.  A turn fetches the first operands of the wavefront's own next turn.
      // What a wavefront does between its units it does while the others do the same and the matrix cores
      // idle, some 9 cycles per dependent scalar instruction: addresses and parities are carried along instead of
      // worked out, one v_readlane brings a k-block's flags, choices are made between integers.  And one body for both
      // kinds of turn leaves no paths to join that hold operands (a branch around the units and a fetch
      // beside them took all 256 registers, this 230).  Against that form, us: 4096 x 4096 x 11008 215 -> 205, 4096 x
      // 11008 x 4096 197 -> 188 (5 % of the blocks flagged), 8192^3 665 -> 639 (a fifth), 545 -> 508 without residual
      // items; gemm_biased_kernel 4096 x 4096 x 11008 190 -> 180.
      const int a_sum = G::kASet, b0 = 2 * G::kASet, b_sum = 2 * b0 + G::kBSet;     // offset in LDS of the other slot = sum - it
      int a_at = 0, a_ring_at = 0, b_at = b0;       // A operands of this turn; ring slots of k-block k
      // what this wavefront requests next: A k-block k + 2, behind the barrier of k; B k-block k + 1, at the top of
      // the turn behind, if it has not been requested
      const int8_t* src = smain + (stage_a ? 2 : 1) * kBlockBytes;
      const uint32_t dst_sum = 2 * my_ring + my_set;
      uint32_t dst = stage_a ? my_ring : my_ring + my_set;
      int late = 0, left = nkb - 2;                // k-blocks behind k + 1
      int cur[G::kSC];
#pragma unroll
      for (int q = 0; q < G::kSC; ++q) cur[q] = r0.s[q];
      for (;;) {
        // The B stagers request their blocks here, two units after the barrier that freed the
        // ring slot, not right behind it: right after the barrier the four A stagers (one per
        // SIMD) are blocked on their eight load instructions each, and while they wait for the
        // address unit to take them, the B stagers, which share their SIMDs, run the last two
        // units of the item.  With all 64 loads issued at once, both wavefronts of every SIMD sat
        // blocked and the matrix cores idled for about a fifth of every item.
        if (late) stage_share(src, dst);
        late = 0;
        ItemScales<G> sc;
#pragma unroll
        for (int q = 0; q < G::kSC; ++q) sc.s[q] = __int_as_float(cur[q]);
        const int8_t* const a_cur = lds + a_at;
        if (multiply) run_units_range<G, 0, kUnits - 2, kBiased>(st, a_cur, a_cur, b_ring, h, c, lane, sc, sp, magic);
        if (!kFb || !res) {
          // All LDS reads of this k-block are issued (the last two units run from registers).  Wait
          // for them and for the next one's direct-to-LDS loads, then the barrier publishes the next
          // k-block and frees this one's ring slots.
          __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
          __syncthreads();
#ifdef FQ_ABLATE_EXTRA_SALU
          extra_salu(k);
#endif
          if (stage_a) {
            if (left > 0) stage_share(src, dst);
            if (kFb && !r0.flags && r1.slot >= 0 && left >= 0) stage_res(r1.slot);
          } else {
            late = kFb && r0.flags ? 0 : max(left, 0);
          }
        }
        const int again = kFb ? r0.flags & (res ^ 1) & 1 : 0;
        const int a_next = kFb && again ? kResOffset<G> : a_sum - a_ring_at;
        const int b_next = kFb && again ? b_at : b_sum - b_at;
        if (multiply)
          run_units_range<G, kUnits - 2, kUnits, kBiased>(st, a_cur, lds + a_next, lds + b_next, h, c, lane, sc, sp, magic);
        a_at = a_next;
        after_units(sc);
        if (kFb && again) {
          res = 1;
#pragma unroll
          for (int q = 0; q < G::kSC; ++q) cur[q] = r0.t[q];
          continue;
        }
        if (left < 0) break;
        if (kFb && r0.flags) {
          res = 0;
          __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
          asm volatile("s_barrier" ::: "memory");
          if (!stage_a && left > 0) stage_share(src + kBlockBytes, dst_sum - dst);
          if (r1.slot >= 0) stage_res(r1.slot);
        }
        // ---- k-block k + 1
        --left;
        a_ring_at = a_sum - a_ring_at;
        b_at = b_sum - b_at;
        dst = dst_sum - dst;
        src += kBlockBytes;
        next_k();
#pragma unroll
        for (int q = 0; q < G::kSC; ++q) cur[q] = r0.s[q];
      }
    } else {
    if (h == 1) asm volatile("s_barrier" ::: "memory");   // team 1 starts one barrier later
    for (;;) {
      // ---- the items after this one
      const int n1res = (r0.flags >> 1) & (res ^ 1), n1k = k + 1 - n1res;
      const int n2res = (r1.flags >> 1) & (n1res ^ 1), n2k = k + 2 - (n1res | n2res);
      // a residual item is work only for the wavefronts whose i-block is flagged at this k
      const bool active = !res || (r0.flags & 1);
      ItemScales<G> sc;
#pragma unroll
      for (int q = 0; q < G::kSC; ++q) sc.s[q] = __int_as_float(res ? r0.t[q] : r0.s[q]);
      const int8_t* const a_cur = a_ring + (t & 1) * G::kASet;
      const int8_t* const a_nxt = a_ring + ((t + 1) & 1) * G::kASet;
      const int8_t* const b_nxt = b_ring + (n1k & 1) * G::kBSet;
      // two barriers per item: this one is the other team's item boundary, in the middle of ours
      if (active) run_units_range<G, 0, 2, kBiased>(st, a_cur, a_nxt, b_nxt, h, c, lane, sc, sp, magic);
      // Behind this barrier team 0 may overwrite the B set this wavefront took its operands
      // from.  An active wavefront has multiplied with all of them by now; one that skips the
      // item has not used them yet and waits for the reads here.
      else __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
      asm volatile("s_barrier" ::: "memory");
      if (active) run_units_range<G, 2, kUnits - 2, kBiased>(st, a_cur, a_nxt, b_nxt, h, c, lane, sc, sp, magic);
      __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
      __syncthreads();
      if (n2k < nkb) stage_team(n2k, n2res, r1, t & 1, !n2res);
      if (active) {
        run_units_range<G, kUnits - 2, kUnits, kBiased>(st, a_cur, a_nxt, b_nxt, h, c, lane, sc, sp, magic);
        after_units(sc);
      } else {
        // nothing to multiply in this item: the pipeline state (the pending tile of the last active item and
        // its scale) stays as it is; only fetch the next item's first operands
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          st.aq[0][i >> 1][i & 1] = lds_frag(a_nxt + G::a_block(h, 0) * kBlockBytes, G::a_group(h, 0),
                                             i >> 1, i & 1, lane);
#pragma unroll
          for (int j = 0; j < kSJ; ++j) {
            const int cg = kSJ * c + j;
            st.bq[j][i >> 1][i & 1] =
                lds_frag(b_nxt + (cg >> 2) * kBlockBytes, cg & 3, i >> 1, i & 1, lane);
          }
        }
      }
      if (n1k >= nkb) break;
      ++t;
      res = n1res;
      if (!n1res) next_k();
    }
    }
    if (kSkew && h == 0) asm volatile("s_barrier" ::: "memory");   // team 1's last item boundary
    drain<G, kBiased>(st, sp);
    if constexpr (kBiased) remove_bias();
  }

  // ---- epilogue.  The MFMA result layout (lane = column, registers = rows) would give 32-byte
  // global stores; instead each wavefront transposes its tile through a private LDS patch
  // (32 rows x 32*kSJ columns at a time) and writes whole row segments with 16-byte stores.
  // A wavefront whose tile lies inside the output stores it without a condition: in the general form behind it every
  // 16 bytes have a branch, 30 integer instructions and an LDS read of their own to wait for.  Such a wavefront also
  // converts to bf16 in front of the patch, two rows to a dword (row pitch + 8 dwords: 2 pitch = 16 banks), which halves
  // the LDS traffic: 16 KiB x 8 wavefronts written and read at 128 bytes a cycle is what is left, 0.9 us.  One workgroup
  // is all a compute unit holds, so nothing passes behind its end.  us, without fallback: 11008 x 4096 x 4096 as TN,
  // binary32 output, 223 -> 214; 11008 x 2048 x 4096 129 -> 121; 4096 x 11008 x 4096, bf16, 206 -> 204 (on a box where
  // the clock is low).  Non-temporal stores: up to 4 % slower.
  __syncthreads();   // every wavefront is done reading the operand rings
  float* const stg = reinterpret_cast<float*>(lds + w * G::kStageBytesPerWave);
  const int col0 = jb_first * kBlock + c * G::kStageCols;   // first column of this wave's tile
  const int last_row = (ib_first + G::a_block(h, kSI - 1)) * kBlock + G::a_group(h, kSI - 1) * 32 + 31;
  if (p.vec_ok && last_row < p.M && col0 + G::kStageCols <= p.N && p.ldc < (1 << 24) && !poison) {      // offsets in 32 bits
    const uint32_t ldc = (uint32_t)p.ldc;
    if (p.out_bf16) {
      uint32_t* const pair = reinterpret_cast<uint32_t*>(stg);
      constexpr int kPitch = G::kStageCols + 8, kChunks = G::kStageCols / 8;
      static_assert(16 * kPitch * 4 <= G::kStageBytesPerWave);
#pragma unroll
      for (int si = 0; si < kSI; ++si) {
#pragma unroll
        for (int sj = 0; sj < kSJ; ++sj)
#pragma unroll
          for (int e = 0; e < 16; e += 2)
            pair[(8 * (e >> 3) + 2 * (lane >> 4) + ((e >> 1) & 1)) * kPitch + sj * 32 + 16 * ((e >> 2) & 1) + (lane & 15)] =
                pack_bf16x2(st.acc[si][sj][e], st.acc[si][sj][e + 1]);
        const int row0 = (ib_first + G::a_block(h, si)) * kBlock + G::a_group(h, si) * 32;
        char* const dst = reinterpret_cast<char*>(p.c) + ((int64_t)row0 * p.ldc + col0) * 2;
#pragma unroll
        for (int it = 0; it < 16 * kChunks / 64; ++it) {
          const int idx = it * 64 + lane;
          const int rp = idx / kChunks, c8 = (idx % kChunks) * 8;
          const v4i a = *reinterpret_cast<const v4i*>(pair + rp * kPitch + c8);
          const v4i b = *reinterpret_cast<const v4i*>(pair + rp * kPitch + c8 + 4);
          v4i lo, hi;
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            lo[i] = __builtin_amdgcn_perm(a[2 * i + 1], a[2 * i], 0x05040100);
            lo[2 + i] = __builtin_amdgcn_perm(b[2 * i + 1], b[2 * i], 0x05040100);
            hi[i] = __builtin_amdgcn_perm(a[2 * i + 1], a[2 * i], 0x07060302);
            hi[2 + i] = __builtin_amdgcn_perm(b[2 * i + 1], b[2 * i], 0x07060302);
          }
          const uint32_t off = (2 * rp * ldc + c8) * 2;
          *reinterpret_cast<v4i*>(dst + off) = lo;
          *reinterpret_cast<v4i*>(dst + p.ldc * 2 + off) = hi;
        }
      }
    } else {
      constexpr int kChunks = G::kStageCols / 4;
#pragma unroll
      for (int si = 0; si < kSI; ++si) {
#pragma unroll
        for (int sj = 0; sj < kSJ; ++sj)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            stg[(16 * (e >> 3) + 4 * (lane >> 4) + (e & 3)) * G::kStagePitch + sj * 32 + 16 * ((e >> 2) & 1) + (lane & 15)] =
                st.acc[si][sj][e];
        const int row0 = (ib_first + G::a_block(h, si)) * kBlock + G::a_group(h, si) * 32;
        char* const dst = reinterpret_cast<char*>(p.c) + ((int64_t)row0 * p.ldc + col0) * 4;
#pragma unroll
        for (int it = 0; it < 32 * kChunks / 64; ++it) {
          const int idx = it * 64 + lane;
          const int rl = idx / kChunks, c4 = (idx % kChunks) * 4;
          *reinterpret_cast<float4*>(dst + (rl * ldc + c4) * 4) =
              *reinterpret_cast<const float4*>(stg + rl * G::kStagePitch + c4);
        }
      }
    }
    return;
  }
  // 32 rows x 32*kSJ columns of FP32 at a time, row pitch + 4 floats
#pragma unroll
  for (int si = 0; si < kSI; ++si) {
    // a flagged block whose residual found no slot cannot be computed: poison its rows
    const bool bad = poison;
#pragma unroll
    for (int sj = 0; sj < kSJ; ++sj)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int rl = 16 * (e >> 3) + 4 * (lane >> 4) + (e & 3);
        const int cl = sj * 32 + 16 * ((e >> 2) & 1) + (lane & 15);
        stg[rl * G::kStagePitch + cl] = bad ? __int_as_float(0x7FC00000) : st.acc[si][sj][e];
      }
    const int row0 = (ib_first + G::a_block(h, si)) * kBlock + G::a_group(h, si) * 32;
    if (p.out_bf16) {
      uint16_t* const C = reinterpret_cast<uint16_t*>(p.c);
      constexpr int kChunks = G::kStageCols / 8;         // 16-byte chunks per row
#pragma unroll
      for (int it = 0; it < 32 * kChunks / 64; ++it) {
        const int idx = it * 64 + lane;
        const int rl = idx / kChunks, c8 = (idx % kChunks) * 8;
        const int row = row0 + rl, col = col0 + c8;
        const float4 lo = *reinterpret_cast<const float4*>(stg + rl * G::kStagePitch + c8);
        const float4 hi = *reinterpret_cast<const float4*>(stg + rl * G::kStagePitch + c8 + 4);
        if (row >= p.M || col >= p.N) continue;
        uint16_t* dst = C + (int64_t)row * p.ldc + col;
        if (p.vec_ok && col + 8 <= p.N) {
          v4i o;
          o[0] = pack_bf16x2(lo.x, lo.y); o[1] = pack_bf16x2(lo.z, lo.w);
          o[2] = pack_bf16x2(hi.x, hi.y); o[3] = pack_bf16x2(hi.z, hi.w);
          *reinterpret_cast<v4i*>(dst) = o;
        } else {
          const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (col + e < p.N) dst[e] = (uint16_t)float_to_bf16_bits(v[e]);
        }
      }
    } else {
      float* const C = reinterpret_cast<float*>(p.c);
      constexpr int kChunks = G::kStageCols / 4;
#pragma unroll
      for (int it = 0; it < 32 * kChunks / 64; ++it) {
        const int idx = it * 64 + lane;
        const int rl = idx / kChunks, c4 = (idx % kChunks) * 4;
        const int row = row0 + rl, col = col0 + c4;
        const float4 v = *reinterpret_cast<const float4*>(stg + rl * G::kStagePitch + c4);
        if (row >= p.M || col >= p.N) continue;
        float* dst = C + (int64_t)row * p.ldc + col;
        if (p.vec_ok && col + 4 <= p.N) {
          *reinterpret_cast<float4*>(dst) = v;
        } else {
          const float e4[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (col + e < p.N) dst[e] = e4[e];
        }
      }
    }
  }
}

// Workgroups are dealt to the 8 XCDs round-robin by id, and each XCD has its own L2.  Remap ids
// so that one XCD works through a contiguous run of tiles, and order the tiles in groups of
// kGroupN tile-columns walked row by row: the ~32 tiles resident on an XCD then form a patch
// that shares its A and B blocks through that L2.  Grouping by columns (not rows) gives every
// XCD tiles from all tile-rows, so fallback blocks clustered in a few block-rows (the worst
// case of Sec. 6.3) load the XCDs evenly.  b in [0, tiles_i * tiles_j) -> (ti, tj), a bijection.
__device__ __forceinline__ void tile_of(int b, int tiles_i, int tiles_j, int& ti, int& tj) {
  tile_at<kGroupN>(xcd_run(b, tiles_i * tiles_j), tiles_i, tiles_j, ti, tj);
}

}  // namespace

// Grid: p.n_main workgroups compute 2 x 2-block tiles covering block rows [0, 2*main_ti) and columns
// [0, 2*main_tj), the rest 1 x 3-block tiles covering the columns or the rows that are left.
__global__ __launch_bounds__(kThreads, 2) void gemm_kernel(GemmParams p) {
  extern __shared__ __attribute__((aligned(1024))) int8_t lds[];
  int ti, tj;
  if ((int)blockIdx.x < p.n_main) {
    tile_of(blockIdx.x, p.main_ti, p.main_tj, ti, tj);
    tile_body<Geo<2, 2>, false>(p, 2 * ti, 2 * tj, lds);
  } else {
    tile_of(blockIdx.x - p.n_main, p.tail_ni, p.tail_tj, ti, tj);
    tile_body<Geo<1, 3>, false>(p, p.tail_i0 + ti, p.tail_j0 + 3 * tj, lds);
  }
}

// gemm_kernel for an A operand that cannot fall back (gradients of the paper's recipe, activations quantized
// without a criterion): every turn is a k-block, and what tells the two kinds apart is gone from the scalar work around
// the barrier, where no wavefront has anything else to issue.  Same bits; with residual slots that nobody uses ->
// here, us: 8192^3 519 -> 508, 4096 x 4096 x 11008 196 -> 190; as TN 11008 x 4096 x 4096 with binary32 output 215 -> 202
// against the kernel before both had one body.  The first p.n_lead of the 1 x 3-block tiles come before the others.
__global__ __launch_bounds__(kThreads, 2) void gemm_main_kernel(GemmParams p) {
  extern __shared__ __attribute__((aligned(1024))) int8_t lds[];
  int ti, tj;
  const int b = (int)blockIdx.x - p.n_lead;
  if (b >= 0 && b < p.n_main) {
    tile_of(b, p.main_ti, p.main_tj, ti, tj);
    tile_body<Geo<2, 2>, false, false>(p, 2 * ti, 2 * tj, lds);
  } else {
    tile_of(b < 0 ? (int)blockIdx.x : (int)blockIdx.x - p.n_main, p.tail_ni, p.tail_tj, ti, tj);
    tile_body<Geo<1, 3>, false, false>(p, p.tail_i0 + ti, p.tail_j0 + 3 * tj, lds);
  }
}

// The tolerance variant of gemm_kernel: same tiles, same k-loop, same order of the terms, but the
// INT32 block products are folded into the FP32 accumulators without being converted: the first
// MFMA of every 16 x 16 quadrant accumulates onto the bit pattern of 1.25 * 2^23, so that the
// finished INT32 value read as binary32 is exactly 1.25 * 2^23 + P (|P| <= 128 * 127^2 < 2^21), one
// FMA per element adds (1.25 * 2^23 + P) * s, and the bias 1.25 * 2^23 * (sum of the scales used) is
// taken out every kBiasWindow items.  Half the vector-ALU instructions of Eq. (1) (the two left per
// MFMA are the ones its issue leaves free); the additions round at the magnitude of the biased
// sums, so results differ from gemm_kernel's by up to about 2e-4 of max |C|, whatever K.
__global__ __launch_bounds__(kThreads, 2) void gemm_biased_kernel(GemmParams p) {
  extern __shared__ __attribute__((aligned(1024))) int8_t lds[];
  int ti, tj;
  if ((int)blockIdx.x < p.n_main) {
    tile_of(blockIdx.x, p.main_ti, p.main_tj, ti, tj);
    tile_body<Geo<2, 2>, true>(p, 2 * ti, 2 * tj, lds);
  } else {
    tile_of(blockIdx.x - p.n_main, p.tail_ni, p.tail_tj, ti, tj);
    tile_body<Geo<1, 3>, true>(p, p.tail_i0 + ti, p.tail_j0 + 3 * tj, lds);
  }
}

// The INT32 block product of one k-block, main or residual term (inspection / tests): one
// workgroup per 128 x 128 output block, wavefront w computes rows [32w, 32w+32) straight from
// global memory.
__global__ __launch_bounds__(256) void partials_kernel(GemmParams p) {
  const int ib = blockIdx.x / p.njb, jb = blockIdx.x - ib * p.njb;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int k = p.debug_k;
  const int8_t* ablk = p.a_codes + ((int64_t)ib * p.nkb + k) * kBlockBytes;
  bool zero = false;
  if (p.debug_residual) {
    const int slot = p.a_slot ? p.a_slot[ib * p.a_si + k * p.a_sk] : -1;
    zero = slot < 0;
    ablk = p.a_res + (int64_t)(zero ? 0 : slot) * kBlockBytes;
  }
  const int8_t* bblk = p.b_codes + ((int64_t)jb * p.nkb + k) * kBlockBytes;
  int32_t* const out = reinterpret_cast<int32_t*>(p.c);
#pragma unroll
  for (int sj = 0; sj < 4; ++sj) {
    v16i P = {0};
    if (!zero) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const v4i a = *reinterpret_cast<const v4i*>(ablk + ((w * 4 + ks) * 64 + lane) * 16);
        const v4i b = *reinterpret_cast<const v4i*>(bblk + ((sj * 4 + ks) * 64 + lane) * 16);
        P = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, P, 0, 0, 0);
      }
    }
    const int col = jb * kBlock + sj * 32 + (lane & 31);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = ib * kBlock + w * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
      if (row < p.M && col < p.N) out[(int64_t)row * p.ldc + col] = P[r];
    }
  }
}

namespace {

struct TilePlan {
  int n_main;    // workgroups computing 2 x 2-block tiles: main_ti x main_tj of them, over the block
  int main_ti, main_tj;      // rows [0, 2*main_ti) and columns [0, 2*main_tj)
  int tail_i0, tail_ni, tail_j0, tail_tj;    // 1 x 3-block tiles: tail_ni rows from block row tail_i0,
                                             // tail_tj tile columns from block column tail_j0
  double cost;   // rounds of the chip, in units of one 2 x 2 tile per compute unit
};

// All of the output in 2 x 2-block tiles, unless their number leaves the last round of the
// chip mostly idle: then the last block columns are cut into 1 x 3-block tiles (3/4 of the work
// of a 2 x 2 tile each) so that the final round is shorter.  Costs are in units of one 2 x 2
// tile per compute unit.
TilePlan plan_columns(int nib, int njb, int cus) {
  const int tiles_i = (nib + 1) / 2, tiles_j = (njb + 1) / 2;
  const int total = tiles_i * tiles_j;
  const double cost_all = cus > 0 ? (total + cus - 1) / cus : 1;
  const TilePlan all{total, tiles_i, tiles_j, 0, nib, njb, 0, cost_all};
  if (cus <= 0 || total <= cus || total % cus == 0) return all;
  const int rounds = total / cus;
  const int cm = std::min(tiles_j, rounds * cus / tiles_i);
  const int tail_cols = njb - 2 * cm;
  if (cm <= 0 || tail_cols <= 0) return all;
  const int tail_tj = (tail_cols + 2) / 3;
  const int n_tail = nib * tail_tj;
  const double cost_split = (cm * tiles_i + cus - 1) / cus + 0.75 * ((n_tail + cus - 1) / cus);
  if (cost_split + 0.05 < cost_all) return TilePlan{cm * tiles_i, tiles_i, cm, 0, nib, 2 * cm, tail_tj, cost_split};
  return all;
}

// The same with the last block rows instead of the last block columns where that ends earlier: what
// columns leave over is a multiple of the (many) tile rows of a tall output, such as the weight
// gradient of an up projection.  11008 x 4096: 688 tiles are three rounds, and ten of 32 block
// columns of 86 rows are 344 1 x 3 tiles, two more rounds; 22 block rows of 32 columns are 242, one.
// 11008 x 4096 x 4096, binary32 output: 235 -> 227 us.
TilePlan plan_tiles(int nib, int njb, int cus) {
  const TilePlan cols = plan_columns(nib, njb, cus);
  const int tiles_i = (nib + 1) / 2, tiles_j = (njb + 1) / 2, total = tiles_i * tiles_j;
  if (cus <= 0 || total <= cus || total % cus == 0) return cols;
  const int rm = std::min(tiles_i, total / cus * cus / tiles_j);
  const int tail_rows = nib - 2 * rm;
  if (rm <= 0 || tail_rows <= 0) return cols;
  const int tail_tj = (njb + 2) / 3;
  const double cost = (rm * tiles_j + cus - 1) / cus + 0.75 * ((tail_rows * tail_tj + cus - 1) / cus);
  if (cost + 0.05 < cols.cost) return TilePlan{rm * tiles_j, rm, tiles_j, 2 * rm, tail_rows, 0, tail_tj, cost};
  return cols;
}

// Smaller tile for this output, or kNone: the tiles above.  Estimated nanoseconds per k-block (K = 128) of the
// busiest compute unit, from measurements over 256 <= M, N <= 4096 and 512 <= K <= 11008 (33 rows too); the
// launch and the ends of the kernel cost all forms about the same 3 us.  A form has a latency below which a
// k-block does not get however few tiles there are, and a throughput:
//   32 x 32     240, or 80 per tile and compute unit            (33 x 11008 x 4096; 512 x 4096 x 4096)
//   128 x 64    1000 for up to three of them (three are resident), or 390 each         (1536 x 4096 x 4096; 3072^3)
//   128 x 128   850 alone on its compute unit, 1360 a pair (two are resident)
//   256 x 256   2340 for an A with residual slots, 2050 without, one is resident; gemm_biased_kernel 2050
//                                                               (4096^3; 2048 x 4096 x 11008)
// and the forms of fq_gemm_ring.hip, for one round of the chip and no more:
//   128 x 64    380 alone on its compute unit, 675 a pair       (512 x 8192 x 4096; 1024 x 8192 x 4096)
//   128 x 128   600                                             (1024 x 8192 x 4096)
//   128 x 256   1090                                            (2048 x 8192 x 4096)
// Those start later: nothing is multiplied before a loader has brought the first items, and with residual slots the slots
// before them.  So they are for contractions that make up for it.  M x K x N, bf16, us, without loaders -> with them:
//   without slots     2048 x 256 x 2048   5.9 -> 6.4    512 x 256 x 4096   4.6 -> 4.8    2048 x 896 x 4096   14.9 -> 14.1
//                     2048 x 1024 x 2048  9.7 -> 9.4    512 x 1024 x 4096  7.4 -> 7.0
//   10 % flagged      2048 x 256 x 2048   6.2 -> 6.9    512 x 256 x 4096   5.0 -> 5.4    2048 x 896 x 4096   16.3 -> 17.3
//   20 % flagged      2048 x 1280 x 2048 13.0 -> 12.7   512 x 1280 x 4096  9.2 -> 8.9    2048 x 1536 x 4096  24.6 -> 26.3
//                     2048 x 1536 x 2048 15.0 -> 13.8   512 x 1536 x 4096 10.4 -> 10.1   2048 x 2048 x 4096  33.4 -> 32.2
// Hence 8 k-blocks without slots, 12 with, 16 for 128 x 256.  On fewer, 128 x 64 tiles without loaders are priced by their
// latency, 520 for one, and 390 for each of more.  32 x 32 tiles start soonest: with up to five of them per compute unit
// they are as fast without slots and faster with, as long as A stays in an XCD's L2, 4 MiB (20 % flagged, 32 x 32 and
// loaders: 1024 x 2048 x 1280 10.4 and 11.5, x 4096 20.1 and 18.5; 2048 x 1536 x 640 9.3 and 9.7, x 2048 13.0 and 11.8;
// 4096 x 1024 x 320 9.5 and 8.0).  With six per compute unit the loaders take 5 to 15 % less without slots from 8 k-blocks
// on, as much with 20 % flagged from 16 on (1024 x 1536 x 1536 8.6 and 8.0, 9.6 and 9.8), up to 7 % more with half of them.
// So 2048 x 4096 x 4096 takes 128 x 256 (39 us without flagged blocks, 43.5 with 128 x 128 pairs, 76 with
// 256 x 256), 1536 x 4096 x 4096 three 128 x 64 per compute unit (34.1; 35.1 with 128 x 256, 36.0 with 128 x 64 of
// the ring in two rounds), 3072^3 128 x 64 too (42; 44 and 48 in two and three rounds of the ring's 128 x 64 and
// 128 x 128, 61 with 256 x 256) and 4096^3 256 x 256 (79 us; 82 in two rounds of 128 x 256).  Flagged blocks cost
// 256 x 256 tiles more than the others, and how many there are is not known here, so the line for an A with slots lies where
// up to 30 % are no loss: 3584 x 4096 x 3584 takes 256 x 256 (70 us at 10 %, 85 at 30 %; 81 and 92 with 128 x 64) and so
// does 1280 x 1024 x 9856 (23.6 and 28.4; 25.3 and 27.9), but not 1280 x 2048 x 9000 (42.5 us with 128 x 64 at 20 %; 44.9).
// Without slots that one (34.6; 35.7) and 4096 x 4096 x 5760 (112; 123 with 128 x 128) take them too.  512 x 4096 x 4096
// takes the ring's 128 x 64 (16.3 us; 18.9 with the other, 23.5 with 32 x 32), 256 x 4096 x 4096 32 x 32 (10.8 us,
// 15.4 with the ring) and 256 x 11008 x 4096 too (28.6 us, 33.2).  64 x 64 tiles were never better than the nearer
// of their neighbours by more than 3 %.  The smaller tiles have no biased form, so fq_gemm_biased takes them where
// they beat its own kernel: 2048 x 4096 x 4096 (42 us against 68), but not 2048 x 4096 x 11008 (129 against 117)
// or 3072 x 11008 x 4096 (170 against 151), which fq_gemm computes on 128 x 128.
SmallTile plan_small(int M, int N, int nkb, const TilePlan& big, int cus, bool biased, bool slots) {
  const double c = cus > 0 ? cus : 256;
  auto tiles = [&](int r, int s) { return (double)((M + r - 1) / r) * ((N + s - 1) / s) / c; };
  const double n64 = tiles(128, 64), n128 = tiles(128, 128);
  const double pairs = std::floor(n128 / 2.0), rest = n128 - 2.0 * pairs;
  constexpr double kNever = 1e300;
  constexpr int64_t kXcdL2 = 4 << 20;
  const bool loaders = nkb >= (slots ? 12 : 8);
  const double ring64 = (int64_t)M * nkb * kBlock >= kXcdL2 ? 380.0 : slots && nkb < 16 ? 520.0 : 400.0;
  const struct { SmallTile kind; double est; } form[] = {
      {SmallTile::k32x32, std::max(240.0, 80.0 * tiles(32, 32))},
      {SmallTile::k128x64, n64 > 3.0 ? 390.0 * n64 : loaders ? 1000.0 : std::max(520.0, 390.0 * (n64 <= 2.0 ? std::ceil(n64) : n64))},
      {SmallTile::k128x128, 1360.0 * pairs + (rest > 1.0 ? 1360.0 : rest > 0.0 ? 850.0 : 0.0)},
      {SmallTile::kRing128x64, !loaders ? kNever : n64 <= 1.0 ? ring64 : n64 <= 2.0 ? 675.0 : kNever},
      {SmallTile::kRing128x128, loaders && n128 <= 1.0 ? 600.0 : kNever},
      {SmallTile::kRing128x256, loaders && (!slots || nkb >= 16) && tiles(128, 256) <= 1.0 ? 1090.0 : kNever}};
  double best = (slots && !biased ? 2340.0 : 2050.0) * big.cost;
  SmallTile tile = SmallTile::kNone;
  for (const auto& f : form)
    if (f.est < best) {
      best = f.est;
      tile = f.kind;
    }
  return tile;
}

// Compute units the planner assumes: the device's, or the value of the environment variable
// FQ_GEMM_CUS when it is set to a positive number (tuning and tests: a small value makes small
// problems take the mixed-geometry path).
int planning_cus() {
  if (const char* e = std::getenv("FQ_GEMM_CUS")) {
    const int v = std::atoi(e);
    if (v > 0) return v;
  }
  // per device, filled on first use (a race between threads only repeats the query)
  static std::atomic<int> cached[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return -1;
  if (dev < 0 || dev >= kMaxDevices) dev = 0;
  int v = cached[dev].load(std::memory_order_relaxed);
  if (v == 0) {
    hipDeviceProp_t prop;
    v = hipGetDeviceProperties(&prop, dev) == hipSuccess ? prop.multiProcessorCount : -1;
    cached[dev].store(v, std::memory_order_relaxed);
  }
  return v;
}

}  // namespace

void gemm_tile_plan(int nib, int njb, int cus, int out[3]) {
  const TilePlan plan = plan_columns(nib, njb, cus > 0 ? cus : planning_cus());
  out[0] = plan.n_main;
  out[1] = plan.main_tj;
  out[2] = plan.tail_tj;
}

namespace {

int ceil_tiles(int n, int edge) { return (int)(((int64_t)n + edge - 1) / edge); }

struct Choice {
  TilePlan plan;
  SmallTile tile;       // kNone: the plan's
};

// What a product of nkb k-blocks is computed with; M and N are not zero.
Choice choose(int M, int N, int nkb, int cus, bool biased, bool slots) {
  const TilePlan plan = plan_tiles(ceil_tiles(M, kBlock), ceil_tiles(N, kBlock), cus);
  return {plan, plan_small(M, N, nkb, plan, cus, biased, slots)};
}

}  // namespace

void gemm_form(int M, int N, int K, int cus, bool biased, bool slots, int out[2]) {
  out[0] = out[1] = 0;
  if (M == 0 || N == 0) return;
  const Choice c = choose(M, N, ceil_tiles(K, kBlock), cus > 0 ? cus : planning_cus(), biased, slots);
  constexpr int kEdges[][2] = {{0, 0}, {32, 32}, {128, 64}, {128, 128}, {128, 64}, {128, 128}, {128, 256}};
  const int* const e = kEdges[(int)c.tile];
  out[0] = (int)c.tile;
  out[1] = c.tile == SmallTile::kNone ? c.plan.n_main + c.plan.tail_ni * c.plan.tail_tj
                                      : ceil_tiles(M, e[0]) * ceil_tiles(N, e[1]);
}

void gemm_path(int M, int N, int cus, bool biased, int out[4]) {
  out[0] = out[1] = out[2] = out[3] = 0;
  if (M == 0 || N == 0) return;
  constexpr int kLong = 1 << 20;      // k-blocks
  const Choice c = choose(M, N, kLong, cus > 0 ? cus : planning_cus(), biased, true);
  switch (c.tile) {
    case SmallTile::kNone:
      out[1] = c.plan.n_main;
      out[c.plan.tail_i0 > 0 ? 3 : 2] = c.plan.tail_ni * c.plan.tail_tj;
      return;
    case SmallTile::k32x32:
      out[0] = 1;
      out[1] = ceil_tiles(M, 32) * ceil_tiles(N, 32);
      return;
    case SmallTile::k128x64:
    case SmallTile::kRing128x64:
      out[0] = 2;
      out[1] = ceil_tiles(M, 128) * ceil_tiles(N, 64);
      return;
    case SmallTile::k128x128:
    case SmallTile::kRing128x128:
    case SmallTile::kRing128x256:
      out[0] = 3;
      out[1] = ceil_tiles(M, 128) * ceil_tiles(N, 128);
      return;
  }
}

hipError_t launch_gemm(const GemmParams& p_in, bool debug, hipStream_t st) {
  if (debug) {
    if (p_in.nib * p_in.njb == 0) return hipSuccess;
    hipLaunchKernelGGL(partials_kernel, dim3(p_in.nib * p_in.njb), dim3(256), 0, st, p_in);
    return hipGetLastError();
  }
  if (p_in.nib == 0 || p_in.njb == 0) return hipSuccess;
  GemmParams p = p_in;
  const auto [plan, tile] = choose(p.M, p.N, p.nkb, planning_cus(), p.biased != 0, p.a_slot != nullptr);
  if (tile != SmallTile::kNone) return launch_gemm_small(p, tile, st);
  p.n_main = plan.n_main;
  p.main_ti = plan.main_ti;
  p.main_tj = plan.main_tj;
  p.tail_i0 = plan.tail_i0;
  p.tail_ni = plan.tail_ni;
  p.tail_j0 = plan.tail_j0;
  p.tail_tj = plan.tail_tj;
  // A round of binary32 tiles is 67 MB that all compute units store at once, while nothing multiplies.  Half of the
  // 3/4 tiles go first there, so that half of the chip ends its rounds a quarter of one before or behind the other; the
  // sum of the rounds stays what it is.  Neighbours that no longer work in step share less through L2, which costs more
  // the longer the contraction is, and tiles of uneven length (fallback) end better with the short ones last.  us,
  // binary32: 5120 x 5120 x 2048 73.8 -> 70.3, 11008 x 4096 x 1000 74.5 -> 69.3, x 2048 121.8 -> 117.7; with K = 4096
  // -1.5 (11008 x 4096) to +2 % (5120 x 5120); with 20 % flagged 4096 x 11008 x 2048 137.1 -> 139.2; with bf16 output,
  // half as much to store, -4 to +2 %.
  constexpr int kMaxLeadK = 16;    // k-blocks
  const int n_tail = plan.tail_ni * plan.tail_tj;
  p.n_lead = !p.a_slot && !p.biased && !p.out_bf16 && p.nkb <= kMaxLeadK ? n_tail / 2 / kXcds * kXcds : 0;
  const int grid = plan.n_main + n_tail;
  // the kernel needs more dynamic LDS than the default limit: raise it once per device
  static std::atomic<bool> attr_set[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) dev = 0;
  if (!attr_set[dev].load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_biased_kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_main_kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    if (e != hipSuccess) return e;
    attr_set[dev].store(true, std::memory_order_release);
  }
  if (p.biased) hipLaunchKernelGGL(gemm_biased_kernel, dim3(grid), dim3(kThreads), kLdsBytes, st, p);
  else if (!p.a_slot) hipLaunchKernelGGL(gemm_main_kernel, dim3(grid), dim3(kThreads), kLdsBytes, st, p);
  else hipLaunchKernelGGL(gemm_kernel, dim3(grid), dim3(kThreads), kLdsBytes, st, p);
  return hipGetLastError();
}

}  // namespace fq
