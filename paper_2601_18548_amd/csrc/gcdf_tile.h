// Tile engine of the fused batched neural-GCDF query for gfx950 (MI355X):
// device code shared by the query, sphere-query and serving kernels.
//
// One workgroup owns a tile of 64 queries: 64 points of one knot (dense all-pairs
// mode) or 64 entries of a pair list.  It has 8 waves, two per SIMD, at width 512 in
// the 16-bit modes, and 4 waves elsewhere, at width 256 two such workgroups per
// compute unit, each running its own tile (pure BF16 at width 256: one of 8 waves).
// For the tile it runs the whole query without touching HBM in between:
//   base-frame transform -> input layer (FP32, VALU) -> hidden layers on
//   matrix cores -> output dot -> reverse sweep on matrix cores (transposed
//   weights) -> input-layer gradient (FP32) -> chain rule to (x, y, yaw, arm)
//   -> stores of d / J -> per-knot minimum (64-bit atomic maximum of inverted
//   ordered keys).
// What bounds it (BF16X2_F16; profiles/fused_query_bf16x2_f16_counters.md): width 512,
// 128 x 16,384 pairs, matrix cores busy 59 % of the cycles and the vector ALU 37 %, with
// 8 % of them together, at 1.9 GHz (the power limit); width 256, 77 x 5,003 pairs, 44 %,
// 47 % and 12 %.  Two 4-wave workgroups per compute unit at width 256, the input layer
// and its gradient on the matrix cores, weight fragments requested a layer ahead,
// addresses formed per phase and a J-free variant took, on one box: 77 x 5,003 W=256
// 574 -> 499 us; FP32 64 x 4,096 1.662 -> 1.529 ms; distances only, 128 x 2,048 W=512
// BF16X2 704 -> 679 us; 128 x 16,384 W=512 9.17 -> 8.84 ms (1 to 4 % by box).
// (Steps of the query: Sec. III-B base-frame transform and chain rule,
// Sec. III-C network on [p', a], Sec. IV-A constraint over all knot/point
// pairs, Sec. IV-A knot-major stacking.)
//
// Work split inside the tile: every hidden layer is C[W x 64] = M[W x W] B[W x 64]
// with M = W_l (forward) or W_l^T (reverse) and B = the previous layer's
// activations (forward) or back-propagated gradients (reverse).  With n waves,
// wave w owns output rows [w*W/n, (w+1)*W/n) for all 64 queries; B lives in LDS
// (written by the epilogue of the previous layer, read by every wave); the A fragments
// stream from global memory (L2-resident, pre-packed so each 32x16 fragment is
// one contiguous 1 KiB block: one dwordx4 per lane).  Each weight byte fetched
// is used for 64 queries.
//
// Precision modes:
//   FP32   : v_mfma_f32_32x32x2_f32, activations FP32 in LDS.
//   BF16   : v_mfma_f32_32x32x16_bf16, activations rounded to BF16, FP32 accumulate.
//   BF16X2 : as BF16 but each activation is split x = hi + lo (both BF16) and both
//            halves are multiplied (2 MFMAs per fragment pair); hidden weights must
//            lie on the BF16 grid to be exact.
//   BF16X2F16 : forward layers as BF16X2; the reverse sweep multiplies FP16
//            back-propagated values by the FP16 copy of the transposed BF16 weights
//            (v_mfma_f32_32x32x16_f16, one MFMA per fragment pair), the values
//            scaled by 2^6 to keep them in FP16's normal range.
// The SiLU derivative needed by the reverse sweep is kept in FP32 registers for
// layers 2 and 3 and recomputed for layer 1 from the input layer.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "gcdf_internal.h"

// Waves per workgroup of the split modes at width 256: 4, with two workgroups on a
// compute unit, but 8 in the source for launches of one round (see one_round), which
// keeps its instantiations apart in an inline namespace.
#ifdef GCDF_ONE_ROUND
namespace gcdf {
inline namespace one_round_tiles {
constexpr int kSplitWaves256 = 8;
#else
namespace gcdf {
constexpr int kSplitWaves256 = 4;
#endif

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
typedef __attribute__((__vector_size__(8 * sizeof(_Float16)))) _Float16 f16x8;
typedef __attribute__((__vector_size__(4 * sizeof(_Float16)))) _Float16 f16x4;

constexpr float kLog2e = 1.4426950408889634f;

// SiLU and its derivative from one exp and one reciprocal.
__device__ __forceinline__ float sigmoid(float z) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-z * kLog2e));
}
__device__ __forceinline__ void silu_fwd(float z, float& h, float& dh) {
  const float sg = sigmoid(z);
  h = z * sg;
  dh = sg + h * (1.0f - sg);  // s (1 + z (1 - s))
}
__device__ __forceinline__ float silu_only(float z) { return z * sigmoid(z); }
__device__ __forceinline__ float silu_prime_only(float z) {
  float t = __builtin_amdgcn_exp2f(-z * kLog2e);
  float sg = __builtin_amdgcn_rcpf(1.0f + t);
  return sg + z * sg * (1.0f - sg);
}

// The reverse sweep's SiLU' values are parked in accumulation registers
// (AGPRs), which the matrix cores do not need because accumulators are kept in
// ordinary VGPRs; vector ALU instructions cannot read AGPRs, so values move with
// v_accvgpr_write / v_accvgpr_read.
__device__ __forceinline__ float park(float x) {
  float a;
  asm("v_accvgpr_write_b32 %0, %1" : "=a"(a) : "v"(x));
  return a;
}
// `after` is an extra input that orders the read after the value it is used
// with (the layer's finished accumulator); otherwise the compiler hoists the
// read above the K loop and keeps every unparked value live through it.
__device__ __forceinline__ float unpark(float a, float after) {
  float x;
  asm("v_accvgpr_read_b32 %0, %1 ; %2" : "=v"(x) : "a"(a), "v"(after));
  return x;
}

// Input-layer pre-activation, in one fixed order shared by every path (each step
// one fused multiply-add): c = b1 + sum_a W1[r][3+a] arm[a] (the knot's arm term),
// then z1 = c + W1[r][0] p'x + W1[r][1] p'y + W1[r][2] p'z (see input_preact_tile).
__device__ __forceinline__ float arm_term(float b1, float w3, float w4, float w5, float w6, float w7, float w8,
                                          const float* arm) {
  float c = b1;
  c += w3 * arm[0];
  c += w4 * arm[1];
  c += w5 * arm[2];
  c += w6 * arm[3];
  c += w7 * arm[4];
  c += w8 * arm[5];
  return c;
}
__device__ __forceinline__ float input_preact(float c, float w0, float w1, float w2, const float* x) {
  return c + w0 * x[0] + w1 * x[1] + w2 * x[2];
}
// Sphere obstacles (network input [p', r, a]): the radius term comes last,
// z1 = c + W1[r][0] p'x + W1[r][1] p'y + W1[r][2] p'z + W1[r][radius] r, with r
// at position kXinRadius of the per-query record (0 for point obstacles, whose
// packed radius weight is 0 too).
constexpr int kXinRadius = 12;
constexpr int kXinTarget = 13;  // training with the fused loss: the sample's target distance

// Waves per workgroup: 8 (two per SIMD) for width 512 on BF16 matrix cores, where
// the per-wave registers of four waves (accumulators, parked SiLU' values, the
// weight prefetch) would fill the register file and leave nothing to hide the
// weight stream's L2 latency, and for pure BF16 (the training tiles' LDS leaves no
// room for a second workgroup); 4 otherwise.
template <int W, int MODE>
constexpr int waves_for() {
  return MODE == kFP32 ? 4 : W == 512 || MODE == kBF16 ? 8 : kSplitWaves256;
}

// Arithmetic of one K loop and of the LDS stores that feed it.  Every mode
// uses its own throughout, except kBF16X2F16: BF16X2 forward, and kF16 (single
// FP16 products; an arithmetic kind, never a context mode) in the reverse sweep.
constexpr int kF16 = 4;
template <int MODE>
constexpr int fwd_arith() {
  return MODE == kBF16X2F16 ? kBF16X2 : MODE;
}
template <int MODE>
constexpr int rev_arith() {
  return MODE == kBF16X2F16 ? kF16 : MODE;
}
// Scale of the reverse sweep's seed (kBF16X2F16): back-propagated values between
// ~1e-6 and ~1e3 stay normal FP16 numbers; the input-layer gradient is
// multiplied back by its inverse.  Powers of two, so both steps are exact.
template <int MODE>
constexpr float rev_scale() {
  return MODE == kBF16X2F16 ? 64.0f : 1.0f;
}

// The split modes order each K step's elements as the accumulators hold them (see
// the activation tile below), so no lanes are exchanged before the LDS stores.
template <int MODE>
constexpr bool lane_k_order() {
  return MODE == kBF16X2 || MODE == kBF16X2F16;
}

// CB: 32-wide column blocks of a tile.  Tiles of one block (32 queries) serve launches
// too small to give every compute unit a 64-query tile (see narrow_tiles): half the
// work per tile, and with it little more than half the time of a call.  Their waves
// have room for longer rings of weight and activation fragments (AR, BR), which their
// shorter K steps need against the same latencies.  A query's arithmetic and the order
// of its sums do not depend on CB.
template <int W, int MODE, int CB = 2>
struct Geo {
  static constexpr int TQ = 32 * CB;                 // queries per tile
  static constexpr int NW = CB == 1 && MODE != kFP32 ? 8 : waves_for<W, MODE>();  // waves per workgroup
  static constexpr bool SHORT_STEPS = CB == 1 && MODE != kFP32;
  // (8 waves at W=256 are in the same place: in pure BF16, one product per fragment, two
  // K steps are 64 cycles of a SIMD.  BF16 training, batch 65,536: 180 us a step
  // with AR = 2, 167 with 4, the same with longer rings of B.)
  static constexpr int AR = SHORT_STEPS ? (W == 256 ? 8 : 4) : W == 256 && NW == 8 ? 4 : 2;  // K steps of A in flight
  static constexpr int BR = SHORT_STEPS && W == 256 ? 4 : 2;  // K steps of B, the current one included
  static constexpr int THREADS = 64 * NW;
  static constexpr int MT = W / (32 * NW);           // 32-row M tiles per wave
  // The packed matrices and row vectors are laid out for 4 row groups of PMT M
  // tiles each (pack_matrix, lane_major_pos); with 8 waves, waves 2p and 2p+1
  // split row group p, SUB waves per group.
  static constexpr int PMT = W / (32 * kWaves);
  static constexpr int SUB = NW / kWaves;
  // Row groups of the final sums over the rows: each group's rows are summed in one
  // chain, the groups then in order, however many waves share them (GPW groups per
  // wave), so a result's bits do not depend on the wave count.
  static constexpr int RG = MODE != kFP32 ? 8 : 4;
  static constexpr int GPW = RG / NW;
  // the per-query reduction buffer shares the activation tile when it would not
  // leave room for 8 waves, or for a second workgroup (the tile is idle by then)
  static constexpr bool RED_IN_ACT = NW > kWaves || W == 256;
  static constexpr int NKB = W / 16;                 // 16-deep K blocks (bf16)
  // bytes of the activation tile per K step (16 rows in the BF16 modes, 8 in FP32);
  // BF16X2 keeps a step's hi and lo halves next to each other, lo at LO_OFF
  static constexpr int STEP_BYTES = (fwd_arith<MODE>() == kBF16X2 ? 64 : 32) * TQ;
  static constexpr int LO_OFF = 32 * TQ;
  static constexpr int NK8 = W / 8;                  // 8-deep K groups (fp32: 4 MFMAs of K=2)
  static constexpr int ACT_BYTES = W * TQ * 4;   // fp32, or bf16 hi + bf16 lo
  static constexpr int XIN_FLOATS = 17;              // per query: p'(3), cos, sin, arm(6), seed, radius, target, pad; odd stride: lanes reading one field of 32 queries hit 32 different banks
  static constexpr int RED_VALS = 9;                 // d, dd/dp'x, dd/dp'y, dd/da1..dd/da6
  static constexpr int RED_BYTES = RG * RED_VALS * TQ * 4;
  static constexpr int LDS_BYTES = ACT_BYTES + TQ * XIN_FLOATS * 4 + W * 4 + (RED_IN_ACT ? 0 : RED_BYTES) + 4 * W * 4;
  // Workgroups per compute unit.  One 4-wave workgroup alone leaves the matrix cores
  // idle in its epilogues and the vector ALU in its K loops; where two fit in LDS and
  // registers they run their layers independently.
  static constexpr int WGS = NW == kWaves && W == 256 ? 2 : 1;
  static constexpr int WPE = WGS * NW / 4;  // waves per SIMD that the registers have to leave room for
  static_assert(WGS * (LDS_BYTES + 2304 + 16) <= 160 * 1024, "the workgroups exceed the compute unit's LDS");
  static_assert(!RED_IN_ACT || RED_BYTES <= ACT_BYTES, "reduction buffer must fit the activation tile");
  static_assert(GPW == 1 || GPW == MT, "a wave's row groups are its M tiles");
  static_assert(MT >= 1 && PMT == SUB * MT, "row groups must split evenly");
};

// ----------------------------------------------------------------------------
// Activation tile in LDS (64 query columns; byte counts for 32 are half).
//  bf16 modes: K step s (rows 16s .. 16s+15) occupies STEP_BYTES at s*STEP_BYTES:
//    its hi half, then (BF16X2) its lo half at +LO_OFF, so one base register with
//    small immediate offsets reaches both.  A half holds 16-byte groups (kh, n) at
//    byte kh*1024 + n*16.  Pure BF16: group (kh, n) holds rows 16s + 8kh + j at
//    position j.  The split modes (lane_k_order) hold rows 16s + 8(j/4) + 4kh + j%4
//    at position j instead, which is the set of rows lane (n, kh) has in its
//    accumulators, so their epilogues store without exchanging lanes; the packed
//    weights order their K elements the same way (the sum over K is unchanged).
//    The B fragment of step s, column block nt is the 2 KiB half, lane (n0, kh)
//    reading the 16 bytes at kh*1024 + nt*512 + n0*16: every lane reads its own
//    consecutive 16 bytes (no bank conflicts).
//  fp32 mode : element (k, n) at (((k/8)*64 + n)*2 + k%2)*4 + (k%8)/2 floats; the
//    B fragment of step s, block nt starts at s*2048 + nt*1024, lane (n0, kh) at
//    +n0*32 + kh*16.
//
// Every address below is a per-lane base (computed once) plus a compile-time
// constant, so the constants fold into the instructions' offset fields instead
// of occupying registers.
// ----------------------------------------------------------------------------
template <int W, int MODE, int CB = 2>
struct Lane {
  static constexpr int MT = Geo<W, MODE, CB>::MT;
  int lane, wave, h, n0, kh, rbase;
  char* act_w;        // write base, hi plane (or the fp32 tile)
  char* act_w_lo;     // write base, lo plane
  const char* act_r;  // read base
  // tid: the thread; wv: its wave, uniform (a scalar register)
  __device__ __forceinline__ Lane(char* act, int tid, int wv) {
    lane = tid & 63;
    wave = wv;
    h = lane >> 5;
    kh = h;
    n0 = lane & 31;
    rbase = 32 * MT * wave;
    if constexpr (MODE == kFP32) {
      act_w = act + 4 * (((rbase >> 3) * Geo<W, MODE, CB>::TQ + n0) * 8 + 2 * h);
      act_r = act + n0 * 32 + kh * 16;
    } else {
      act_w = act + (rbase >> 4) * Geo<W, MODE, CB>::STEP_BYTES + h * 16 * Geo<W, MODE, CB>::TQ + n0 * 16;
      act_r = act + kh * 16 * Geo<W, MODE, CB>::TQ + n0 * 16;
    }
    act_w_lo = act_w + Geo<W, MODE, CB>::LO_OFF;
  }
};

// Write rows R0..R0+3 (R0 = rbase + 32 i + 8 g + 4 h) of column n = 32 nt + n0 (fp32).
template <int W, int MODE, int CB, int I, int G, int NT>
__device__ __forceinline__ void act_store4_fp32(const Lane<W, MODE, CB>& L, const float v[4]) {
  constexpr int off = (4 * I + G) * Geo<W, MODE, CB>::STEP_BYTES + NT * 1024;
  *reinterpret_cast<f32x2*>(L.act_w + off) = f32x2{v[0], v[2]};       // rows R0, R0+2 (k%2 = 0)
  *reinterpret_cast<f32x2*>(L.act_w + off + 16) = f32x2{v[1], v[3]};  // rows R0+1, R0+3 (k%2 = 1)
}

// Pack four floats into two dwords of bf16 (FP16 for kF16), round to nearest even.
template <int AM>
__device__ __forceinline__ void pack4(const float v[4], uint32_t& d0, uint32_t& d1) {
  f32x2 d;
  if constexpr (AM == kF16) {
    f16x4 h4;
#pragma unroll
    for (int r = 0; r < 4; ++r) h4[r] = (_Float16)v[r];
    d = __builtin_bit_cast(f32x2, h4);
  } else {
    bf16x4 h4;
#pragma unroll
    for (int r = 0; r < 4; ++r) h4[r] = (__bf16)v[r];
    d = __builtin_bit_cast(f32x2, h4);
  }
  d0 = __float_as_uint(d[0]);
  d1 = __float_as_uint(d[1]);
}

// bf16 modes: write rows of the group pair g = 2 GP, 2 GP + 1 (v[0..3] for g = 2 GP,
// v[4..7] for g = 2 GP + 1) of column n = 32 nt + n0.  Lane (n0, h) holds k%8 in
// [4h, 4h+4) of both 8-groups kh = 0 (g even) and kh = 1 (g odd).  SWAP (pure
// BF16): one swap across the lane halves gives lane (n0, kh) the whole 8-group kh,
// written as 16 bytes; otherwise (lane_k_order) the lane writes its own 8 values.
// act_pack8 forms the 16-byte words (w[0..3] for the hi plane, w[4..7] for the lo
// plane) and act_write8 stores them, so a caller can do the arithmetic before a
// barrier and the stores after it.  AM: the arithmetic (fwd_arith / rev_arith).
// The values come as products x[k] y[k], whose unrounded difference from hi is lo.
template <int AM, bool SWAP>
__device__ __forceinline__ void act_pack8(const float x[8], const float y[8], uint32_t (&w)[8]) {
  float v[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = x[k] * y[k];
  auto put = [&](const uint32_t e0, const uint32_t e1, const uint32_t o0, const uint32_t o1, uint32_t* out) {
    if constexpr (!SWAP) {
      out[0] = e0;
      out[1] = e1;
      out[2] = o0;
      out[3] = o1;
      return;
    }
    // e: g even (kh 0), o: g odd (kh 1).  Lanes 32..63 of the first operand trade
    // with lanes 0..31 of the second: afterwards lane (n0, kh) has k%8 in [0, 4)
    // in the first and [4, 8) in the second
    const auto s0 = __builtin_amdgcn_permlane32_swap(e0, o0, false, false);
    const auto s1 = __builtin_amdgcn_permlane32_swap(e1, o1, false, false);
    out[0] = s0[0];
    out[1] = s1[0];
    out[2] = s0[1];
    out[3] = s1[1];
  };
  uint32_t d[4];  // bf16 pairs (v0 v1), (v2 v3), (v4 v5), (v6 v7)
  pack4<AM>(v, d[0], d[1]);
  pack4<AM>(v + 4, d[2], d[3]);
  if constexpr (AM == kBF16X2) {
    // lo = x y - hi, with hi read back from the packed pairs (the same rounding);
    // formed before the swaps, which overwrite their operands
    float lo[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      lo[2 * k] = __builtin_fmaf(x[2 * k], y[2 * k], -__uint_as_float(d[k] << 16));
      lo[2 * k + 1] = __builtin_fmaf(x[2 * k + 1], y[2 * k + 1], -__uint_as_float(d[k] & 0xffff0000u));
    }
    uint32_t l[4];
    pack4<AM>(lo, l[0], l[1]);
    pack4<AM>(lo + 4, l[2], l[3]);
    put(l[0], l[1], l[2], l[3], w + 4);
  }
  put(d[0], d[1], d[2], d[3], w);
}

template <int W, int MODE, int CB, int I, int GP, int NT, int AM = fwd_arith<MODE>()>
__device__ __forceinline__ void act_write8(const Lane<W, MODE, CB>& L, const uint32_t (&w)[8]) {
  constexpr int off = (2 * I + GP) * Geo<W, MODE, CB>::STEP_BYTES + NT * 512;
  typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
  *reinterpret_cast<u32x4*>(L.act_w + off) = u32x4{w[0], w[1], w[2], w[3]};
  if constexpr (AM == kBF16X2) *reinterpret_cast<u32x4*>(L.act_w_lo + off) = u32x4{w[4], w[5], w[6], w[7]};
}

template <int W, int MODE, int CB, int I, int GP, int NT, int AM = fwd_arith<MODE>()>
__device__ __forceinline__ void act_store8(const Lane<W, MODE, CB>& L, const float x[8], const float y[8]) {
  uint32_t w[8];
  act_pack8<AM, !lane_k_order<MODE>()>(x, y, w);
  act_write8<W, MODE, CB, I, GP, NT, AM>(L, w);
}

// Either layout: rows of groups g = 2 GP, 2 GP + 1 (see act_store8), the products
// x[k] y[k].
template <int W, int MODE, int CB, int I, int GP, int NT, int AM = fwd_arith<MODE>()>
__device__ __forceinline__ void act_store_pair(const Lane<W, MODE, CB>& L, const float x[8], const float y[8]) {
  if constexpr (MODE == kFP32) {
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = x[k] * y[k];
    act_store4_fp32<W, MODE, CB, I, 2 * GP, NT>(L, v);
    act_store4_fp32<W, MODE, CB, I, 2 * GP + 1, NT>(L, v + 4);
  } else {
    act_store8<W, MODE, CB, I, GP, NT, AM>(L, x, y);
  }
}
// The same for plain values (FP32 and pure BF16: no lo part).
template <int W, int MODE, int CB, int I, int GP, int NT, int AM = fwd_arith<MODE>()>
__device__ __forceinline__ void act_store_pair(const Lane<W, MODE, CB>& L, const float v[8]) {
  static_assert(AM != kBF16X2, "the split forms take the values as products");
  const float one[8] = {1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f};
  act_store_pair<W, MODE, CB, I, GP, NT, AM>(L, v, one);
}

// Compile-time loop helper: f(integral_constant<0>), ..., f(integral_constant<N-1>).
template <int N, int B = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < N) {
    f(std::integral_constant<int, B>{});
    static_for<N, B + 1>(f);
  }
}

// ----------------------------------------------------------------------------
// acc[i][nt] += M[rows of wave, :] x act[:, 32nt .. 32nt+31]
// A fragments come through a buffer descriptor (uniform, SGPRs) of the matrix's
// packed stream, laid out for 4 row groups of PMT M tiles: fragment (kstep, j) of
// row group p at byte p*stream_bytes + ((kstep*PMT + j)*64 + lane)*16.  A wave
// that is share s of group p reads j = s*MT + i, so one 32-bit VGPR offset
// (voff = p*stream_bytes + s*MT*1024 + lane*16) serves every matrix and step; the
// step goes in the scalar offset and i*1024 in the instruction's immediate.
// Software pipeline: A is loaded AR K steps ahead, B (LDS) BR - 1 (see Geo).
// AM is the K loop's arithmetic (fwd_arith / rev_arith of the tile's mode).
// ----------------------------------------------------------------------------
template <int AM, int CB>
struct BFrag {
  bf16x8 h[CB], l[CB];
  f32x4 f[CB];
};

template <int W, int MODE, int CB, int AM>
__device__ __forceinline__ void load_b(BFrag<AM, CB>& b, const char* br) {
  if constexpr (AM == kFP32) {
#pragma unroll
    for (int nt = 0; nt < CB; ++nt) b.f[nt] = *reinterpret_cast<const f32x4*>(br + nt * 1024);
  } else {
#pragma unroll
    for (int nt = 0; nt < CB; ++nt) {
      b.h[nt] = *reinterpret_cast<const bf16x8*>(br + nt * 512);
      if constexpr (AM == kBF16X2) b.l[nt] = *reinterpret_cast<const bf16x8*>(br + Geo<W, MODE, CB>::LO_OFF + nt * 512);
    }
  }
}

template <int W, int MODE, int CB>
__device__ __forceinline__ void load_a(f32x4 (&af)[(Geo<W, MODE, CB>::MT)], __amdgpu_buffer_rsrc_t rs, int voff, int step) {
  const int soff = step * Geo<W, MODE, CB>::PMT * 1024;
#pragma unroll
  for (int i = 0; i < Geo<W, MODE, CB>::MT; ++i)
    af[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, voff + i * 1024, soff, 0));
}

// One K step: for each M tile i, its MFMAs (hi then lo halves alternating over
// the two column blocks, so accumulations into one tile are two MFMAs apart),
// then at once the reload of a[i] for step `next` -- the fragment's registers
// are free as soon as its last MFMA has issued.  The scheduling barriers keep
// the compiler from sinking the loads to the end of the loop body.  ZC: the
// accumulators start at zero, so the first product of each tile reads a zero C
// operand instead of registers cleared beforehand.
template <int W, int MODE, int CB, int AM, bool ZC = false>
__device__ __forceinline__ void mma_step_reload(f32x16 (&acc)[(Geo<W, MODE, CB>::MT)][CB], f32x4 (&af)[(Geo<W, MODE, CB>::MT)],
                                                const BFrag<AM, CB>& b, __amdgpu_buffer_rsrc_t rs, int voff,
                                                int next) {
  constexpr int MT = Geo<W, MODE, CB>::MT;
  const int soff = next * Geo<W, MODE, CB>::PMT * 1024;
  const f32x16 zero = {};
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    if constexpr (AM == kFP32) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int nt = 0; nt < CB; ++nt)
          acc[i][nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[i][q], b.f[nt][q], (ZC && q == 0) ? zero : acc[i][nt],
                                                            0, 0, 0);
    } else if constexpr (AM == kF16) {
      const f16x8 a8 = __builtin_bit_cast(f16x8, af[i]);
#pragma unroll
      for (int nt = 0; nt < CB; ++nt)
        acc[i][nt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a8, __builtin_bit_cast(f16x8, b.h[nt]),
                                                            ZC ? zero : acc[i][nt], 0, 0, 0);
    } else {
      const bf16x8 a8 = __builtin_bit_cast(bf16x8, af[i]);
#pragma unroll
      for (int nt = 0; nt < CB; ++nt)
        acc[i][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a8, b.h[nt], ZC ? zero : acc[i][nt], 0, 0, 0);
      if constexpr (AM == kBF16X2) {
#pragma unroll
        for (int nt = 0; nt < CB; ++nt)
          acc[i][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a8, b.l[nt], acc[i][nt], 0, 0, 0);
      }
    }
    af[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, voff + i * 1024, soff, 0));
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <int W, int MODE, int CB>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t stream_rsrc(const void* base) {
  constexpr int bytes = W * W * (MODE == kFP32 ? 4 : 2);
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, bytes, 0x00020000);
}

// The A fragments of a layer's first AR K steps, loaded ahead of the layer.  (In
// training that is before the previous layer's dump too: the vector-memory counter
// completes in order, so a wait for fragments issued after the dump's stores would
// also wait for those stores.)
template <int W, int MODE, int CB = 2>
struct APre {
  f32x4 a[Geo<W, MODE, CB>::AR][Geo<W, MODE, CB>::MT];
};
template <int W, int MODE, int CB>
__device__ __forceinline__ void preload_a(APre<W, MODE, CB>& p, const void* mat, int voff) {
  const __amdgpu_buffer_rsrc_t rs = stream_rsrc<W, MODE, CB>(mat);
#pragma unroll
  for (int u = 0; u < Geo<W, MODE, CB>::AR; ++u) load_a<W, MODE, CB>(p.a[u], rs, voff, u);
}

// With two workgroups per compute unit, a wave in an epilogue goes before the other
// workgroup's wave in its K loop: the vector instructions issue in the gaps that each
// matrix instruction leaves (32 cycles for 4 of issue), so both advance.  FP32
// 64 x 4,096 pairs 1.548 -> 1.520 ms, BF16X2_F16 128 x 8,192 (W=256) 1.318 -> 1.304 ms;
// a fixed order of the two workgroups, or the K loop first, measured as no priority.
template <int W, int MODE, int CB>
__device__ __forceinline__ void epilogue_priority(bool epilogue) {
  if constexpr (Geo<W, MODE, CB>::WGS > 1) {
    if (epilogue) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
  }
}

// ZERO: acc starts at zero (its contents on entry are not read).  p: the A
// fragments of the first AR steps, already requested; on return those of the layer
// streamed from `next` (its loads take the place of the last steps' reloads, so they
// are in flight during the epilogue, and the next K loop does not start with the
// weight stream's L2 latency).
template <int W, int MODE, int CB, int AM, bool ZERO = false>
__device__ __forceinline__ void layer_gemm(f32x16 (&acc)[(Geo<W, MODE, CB>::MT)][CB], const void* mat, const void* next,
                                           int voff, const char* br, APre<W, MODE, CB>& p) {
  using G = Geo<W, MODE, CB>;
  constexpr int NS = (MODE == kFP32) ? G::NK8 : G::NKB;
  constexpr int SB = G::STEP_BYTES, U = G::AR, R = G::BR;  // U steps per round of the loop
  static_assert(NS % U == 0 && NS > U && U % R == 0, "whole rounds, and whole turns of both rings");
  epilogue_priority<W, MODE, CB>(false);
  BFrag<AM, CB> b[R];
#pragma unroll
  for (int u = 0; u < R - 1; ++u) load_b<W, MODE, CB, AM>(b[u], br + u * SB);
  // one round: steps s .. s + U - 1; the B fragments of R - 1 steps further, and the A
  // fragments of U steps further, which in the last round are the next layer's first
  auto round = [&](int s, auto zc) {
    const bool more = s + U < NS;
    const __amdgpu_buffer_rsrc_t rn = stream_rsrc<W, MODE, CB>(more ? mat : next);
    const int sn = more ? s + U : 0;
    const char* bw = more ? br : br - U * SB;  // (nothing reads past the tile's last step)
    static_for<U>([&](auto u) {
      load_b<W, MODE, CB, AM>(b[(u + R - 1) % R], (u + R - 1 < U ? br : bw) + (u + R - 1) * SB);
      __builtin_amdgcn_sched_barrier(0);
      mma_step_reload<W, MODE, CB, AM, (decltype(zc)::value && u == 0)>(acc, p.a[u], b[u % R], rn, voff, sn + u);
    });
    br += U * SB;
  };
  int s = 0;
  if constexpr (ZERO) {  // the first round, its first step writing acc from a zero C operand
    round(0, std::true_type{});
    s = U;
  }
#pragma unroll 1
  for (; s < NS; s += U) round(s, std::false_type{});
  epilogue_priority<W, MODE, CB>(true);
}

// The reverse layers' accumulators start at zero: in single FP16 the first
// products read a zero C operand (no clearing moves); the split forms clear the
// registers first (the peeled first steps cost them spilled registers at W=512).
template <int MODE>
constexpr bool rev_zero_c() {
  return rev_arith<MODE>() == kF16;
}
template <int W, int MODE, int CB>
__device__ __forceinline__ void zero_acc(f32x16 (&acc)[(Geo<W, MODE, CB>::MT)][CB]) {
#pragma unroll
  for (int i = 0; i < Geo<W, MODE, CB>::MT; ++i)
#pragma unroll
    for (int nt = 0; nt < CB; ++nt)
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[i][nt][j] = 0.f;
}

__device__ __forceinline__ uint32_t ordered_bits(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Per-knot minimum keys: (ordered distance bits << 32 | point index), stored inverted,
// so that the minimum is an atomic maximum over words that start at zero, and a word
// no tile has touched is zero.  Whoever decodes a word sets it back to zero for the
// next call, which needs no launch to prepare its keys.
__device__ __forceinline__ void minkey_decode(unsigned long long stored, float& d, int32_t& index) {
  const unsigned long long k = ~stored;
  const uint32_t o = (uint32_t)(k >> 32);
  d = __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
  // every knot of a launch receives at least one key; an untouched word would
  // decode to index 0 rather than an out-of-range point
  index = stored == 0 ? 0 : (int32_t)(uint32_t)(k & 0xffffffffu);
}

// ----------------------------------------------------------------------------
// Training: copy the LDS activation tile (hi plane for the BF16 modes) to HBM in
// the blocked feature-major layout: element (f, i) of a [W x batch] array sits at
// ((i / S) * W + f) * S + i % S with S = 16 bytes of samples (8 BF16 or 4 FP32),
// so the 16-byte fragments of consecutive features are adjacent.  Zeros for the
// ragged tail of the tile.  All threads take part.  (The stores go through the
// caches on purpose: the weight-gradient kernels that follow read the dumps back,
// largely from the last-level cache; non-temporal stores made the backward pass
// half again as slow.)
// BF16: wave w copies features 32w .. 32w + 31 of the 64 samples.  It transposes them
// on the matrix cores: 32 samples x 16 features as A fragments (16 bytes a lane, as
// they lie in the tile) times the identity give 32 x 32 blocks with a feature per lane
// and samples in its registers; half a dozen moves and one exchange of lane halves
// pack 8 samples of a feature into 16 bytes, and a wave's store writes 1 KiB of
// consecutive pieces.  The product of a finite BF16 value with 1 plus zeros is exact; an
// infinity or NaN makes its sample's whole block NaN or infinite, so a wave whose sums
// come out not finite copies and sums again, element by element, and only the values
// that are not finite themselves reach HBM and the sums.  (The dumps without sums, h1 to
// h3, need no second copy: such a value in h_l makes all of the sample's z_{l+1}, and so
// its SiLU' and every g of it, not finite.)  Transposing 8 x 8 blocks with vector instructions through a 32 KiB LDS
// stage, and the sums below on the vector ALU, a dump took 3.1-3.6 K cycles and the
// sums-only copies of h4 and g1 4.4 and 5.0 K, in all 30 K of a tile's 79 K; here 1.1-1.3,
// 1.6 and 2.1 K of 52 K (batch 65,536: the kernel 155 -> 121 us; with the check for
// values that are not finite the step takes 1 % more, 181.3 -> 183.0 us).
// BF16, with sums: the copy also adds, over the tile's samples i, to LDS rows
// (per feature f) sum_i x[f][i] w_i (w_i = seed_i, or 1), and optionally
// sum_i x[f][i] v_c(i) for the nine network inputs v_c: products over samples on the
// matrix cores, with the pieces as B fragments (the seeds in three BF16 parts, which
// hold all 24 bits; v in BF16 hi + lo).  store false: the sums only, nothing written
// to HBM.
// FP32, with sums: the same sums, thread f those of feature f: row sums sample by
// sample on the vector ALU, those with the inputs four at a time by v_mfma_f32_4x4x1_16b_f32, whose
// 16 blocks take a wave's 64 features as columns (the vector ALU read every input of
// every sample by a load of its own: 20 us of a step of 734 at batch 65,536).  They go to
// the workgroup's rows in global memory (each entry has one thread, so program order is
// the order of the sum).  They replaced passes over the dumps that read 64 to 320 MB
// back (batch 65,536) or ran on ten workgroups (batch 5,001: 42 us).  The copy is short
// of instruction cache, not of LDS: four blocks of samples per trip cost 20 us a step
// more than two, all sixteen 190; lanes starting at different samples, which removes its
// 8-way bank conflicts, 20.  With both changes 734 -> 723 us (batch 5,001: 153.6 -> 150.5).
// ----------------------------------------------------------------------------
constexpr int kVtSeed = 18, kVtRows = 21;  // rows of the transposed inputs (DumpSums::vt)
struct DumpSums {
  float* row;          // [W]: sum_i x[f][i] w_i (NULL: not wanted)
  const float* seed;   // w_i = seed[i * XIN_FLOATS] (the records' seed slot), or NULL: w_i = 1
  float* in_rows;      // [9][W]: sum_i x[f][i] v_c(i), or NULL
  const __bf16* vt;    // BF16: the tile's inputs v_c(i) as BF16 hi [9][64], lo [9][64], then the seeds' parts [3][64]
  // FP32: v_c(i) at in[i * in_stride + c], from c = 3 on at + in_gap further
  const float* in;
  int in_stride, in_gap;
};

template <int W, int MODE>
__device__ __forceinline__ void dump_tile(const char* act, void* dst, int64_t ldb, int64_t q0,
                                          int nvalid, const DumpSums* sums = nullptr, bool store = true) {
  (void)ldb;
  if constexpr (MODE == kFP32) {
    static_assert(Geo<W, MODE>::THREADS == W, "a thread per feature");
    constexpr int XF = Geo<W, MODE>::XIN_FLOATS;
    const int f = threadIdx.x;
    const float* a = reinterpret_cast<const float*>(act) + (((f >> 3) * kTileQ) * 2 + (f & 1)) * 4 + ((f & 7) >> 1);
    const bool row = sums && sums->row, in = sums && sums->in_rows;
    float s = 0.f;
    f32x4 sv[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) sv[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the field of a sample's record that this lane's row 4 j + lane % 4 of the input
    // sums takes (rows 9..11: any)
    int xo[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int c = 4 * j + (int)(threadIdx.x & 3);
      xo[j] = c < 3 ? c : c < 9 ? c + (sums ? sums->in_gap : 0) : 0;
    }
    auto copy = [&](auto FULL) {
#pragma unroll 2
      for (int n = 0; n < kTileQ; n += 4) {
        f32x4 v;
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = FULL || n + u < nvalid ? a[(n + u) * 8] : 0.f;
        if (store) *reinterpret_cast<f32x4*>(static_cast<float*>(dst) + (((q0 + n) >> 2) * W + f) * 4) = v;
        if (row) {
#pragma unroll
          for (int u = 0; u < 4; ++u) s += sums->seed ? v[u] * sums->seed[(n + u) * XF] : v[u];
        }
        if (in) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float* x = sums->in + (n + u) * sums->in_stride;
#pragma unroll
            for (int j = 0; j < 3; ++j) sv[j] = __builtin_amdgcn_mfma_f32_4x4x1f32(x[xo[j]], v[u], sv[j], 0, 0, 0);
          }
        }
      }
    };
    if (nvalid == kTileQ) copy(std::integral_constant<bool, true>{});
    else copy(std::integral_constant<bool, false>{});
    if (row) sums->row[f] += s;
    if (in) {
#pragma unroll
      for (int c = 0; c < 9; ++c) sums->in_rows[c * W + f] += sv[c >> 2][c & 3];
    }
  }
  if constexpr (MODE != kFP32) {
    // The hi plane holds, for each group of 8 features and each query n, the 8
    // features' values as one 16-byte word.
    static_assert(MODE == kBF16, "the dumps of the training precisions");
    typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
    // the tile's pieces are consecutive in the dump: piece P at element ((q0 / 8) W + P) 8
    constexpr int T = Geo<W, MODE>::THREADS;
    static_assert(T % W == 0, "a thread's pieces share one feature");
    static_assert(T / 64 == W / 32, "the copy: one 32-feature block per wave");
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int f = 32 * (threadIdx.x >> 6) + (lane & 31);
    __bf16* o = static_cast<__bf16*>(dst) + (q0 >> 3) * W * 8;
    f32x16 dacc;
#pragma unroll
    for (int j = 0; j < 16; ++j) dacc[j] = 0.f;
    const int c = lane & 31;
    // identity fragments of the wave's two K steps: lane (c, half) of step k holds rows
    // 16 k + 8 half + e, e = 0..7, of column c
    bf16x8 eye[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      u32x4 d;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        d[e] = (c >> 1) == 8 * k + 4 * half + e ? ((c & 1) ? 0x3f800000u : 0x00003f80u) : 0u;
      eye[k] = __builtin_bit_cast(bf16x8, d);
    }
    const int s0 = 2 * (threadIdx.x >> 6);  // this wave's first K step of the tile
    // one 16-sample round: store lane (c, half)'s piece v, samples 8 nb .. 8 nb + 7 of
    // feature f, and add it to the sums: the pieces are the B fragments of a product over
    // samples, row c of A holds what column sums are wanted of
    auto round = [&](int nb, const u32x4& v) {
      const int P = nb * W + f;
      if (store) *reinterpret_cast<u32x4*>(o + P * 8) = v;
      if (sums) {
        const int n0 = nb * 8;
        bf16x8 ah, al;
#pragma unroll
        for (int e = 0; e < 8; ++e) ah[e] = al[e] = (__bf16)0.f;
        if (sums->in_rows) {
          if (c < 9) {
            ah = *reinterpret_cast<const bf16x8*>(sums->vt + c * kTileQ + n0);
            al = *reinterpret_cast<const bf16x8*>(sums->vt + (9 + c) * kTileQ + n0);
          }
        } else if (sums->seed) {
          if (c < 3) ah = *reinterpret_cast<const bf16x8*>(sums->vt + (kVtSeed + c) * kTileQ + n0);
        }
        if (!sums->seed && c == (sums->in_rows ? 9 : 0)) {
#pragma unroll
          for (int e = 0; e < 8; ++e) ah[e] = (__bf16)1.f;
        }
        dacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, __builtin_bit_cast(bf16x8, v), dacc, 0, 0, 0);
        if (sums->in_rows)
          dacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, __builtin_bit_cast(bf16x8, v), dacc, 0, 0, 0);
      }
    };
#pragma unroll
    for (int h = 0; h < kTileQ / 32; ++h) {  // 32 samples: lane (m, half) reads sample m's features 8 half + e of each step
      const int n = 32 * h + c;
      f32x16 z;
#pragma unroll
      for (int j = 0; j < 16; ++j) z[j] = 0.f;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const u32x4 x = n < nvalid ? *reinterpret_cast<const u32x4*>(act + (s0 + k) * Geo<W, MODE>::STEP_BYTES +
                                                                     half * 16 * kTileQ + n * 16)
                                   : u32x4{0u, 0u, 0u, 0u};
        z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x), eye[k], z, 0, 0, 0);
      }
      // lane (c, half): feature c, samples 8 g + 4 half + r of the 32 in z[4 g + r]
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        uint32_t p[4];  // samples (0 1), (2 3) of g = 2 t, then of g = 2 t + 1
#pragma unroll
        for (int q = 0; q < 4; ++q)
          p[q] = __builtin_amdgcn_perm(__float_as_uint(z[8 * t + 2 * q + 1]), __float_as_uint(z[8 * t + 2 * q]), 0x07060302u);
        const auto x0 = __builtin_amdgcn_permlane32_swap(p[0], p[2], false, false);
        const auto x1 = __builtin_amdgcn_permlane32_swap(p[1], p[3], false, false);
        round(4 * h + 2 * t + half, u32x4{x0[0], x1[0], x0[1], x1[1]});
      }
    }
    if (sums) {
      // rows 0 (ones), 9 (ones beside the inputs) or 0..2 (seeds' parts) meet every value
      // of the wave's features; in the upper lanes these are rows of zeros
      float t = sums->in_rows ? dacc[5] : sums->seed ? dacc[2] + dacc[1] + dacc[0] : dacc[0];
      if (__builtin_amdgcn_ballot_w64(!__builtin_isfinite(t))) {
        float part = 0.f;  // the seeds as they are: an infinite one has no BF16 parts
#pragma unroll
        for (int j = 0; j < 16; ++j) dacc[j] = 0.f;
        int g = f;
        asm volatile("" : "+v"(g));  // (addresses formed here, not kept through the tile for this rare case)
        const char* a = act + (g >> 4) * Geo<W, MODE>::STEP_BYTES + ((g >> 3) & 1) * 16 * kTileQ + (g & 7) * 2;
#pragma unroll 1
        for (int nb = half; nb < kTileQ / 8; nb += 2) {
          u32x4 v;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int n = 8 * nb + e;
            const uint32_t x = n < nvalid ? *reinterpret_cast<const uint16_t*>(a + n * 16) : 0u;
            v[e >> 1] = (e & 1) ? v[e >> 1] | (x << 16) : x;
            if (sums->seed) part += __uint_as_float(x << 16) * sums->seed[n * Geo<W, MODE>::XIN_FLOATS];
          }
          round(nb, v);
        }
        if (sums->seed) {
          part += __shfl_xor(part, 32);
          dacc[0] = part;
          dacc[1] = dacc[2] = 0.f;
        }
      }
    }
    if (sums) {
      // lane (feature f % 32, half) holds rows 8 (j/4) + 4 half + j%4
      int r = f;
      asm volatile("" : "+v"(r));  // (the rows' addresses too are formed here)
      if (sums->in_rows) {
#pragma unroll
        for (int j = 0; j < 4; ++j) sums->in_rows[(4 * half + j) * W + r] += dacc[j];
        if (half == 0) {
          sums->in_rows[8 * W + r] += dacc[4];
          sums->row[r] += dacc[5];
        }
      } else if (half == 0) {
        sums->row[r] += sums->seed ? dacc[2] + dacc[1] + dacc[0] : dacc[0];
      }
    }
  }
}

// ----------------------------------------------------------------------------
// Layer bodies (compile-time layer index so every register array is static).
// Element j of acc[i][nt] is row R = rbase + 32 i + 8 (j/4) + 4 (lane/32) + j%4
// of the layer output and query column n = 32 nt + lane%32.
// ----------------------------------------------------------------------------
// Row-indexed vectors (b1..b4, w_out, the input-layer rows and the per-knot
// arm term) are stored in lane-major order: the 16*MT rows one lane touches,
// R = rbase + 32 i + 8 g + 4 h + r, sit at position
// ((p*2 + h)*PMT + s*MT + i)*16 + 4 g + r for a wave that is share s of row
// group p (with 4 waves, p = wave, s = 0, PMT = MT), so each lane addresses them
// from one base with small constant offsets.
template <int W, int MODE, int CB = 2>
struct Bases {
  const float* bh;    // LDS copy of b2, b3, b4 (lane-major), at this lane's block
  const float* w5;    // LDS copy of w_out (lane-major), at this lane's block
  const float* w1;    // input layer rows (lane-major, 12 floats per row), at this lane's block
  const float* w1a;   // input layer row rbase + lane%32 (its A fragment row in M tile 0; tile i at +16 i rows)
  const float* crow;  // per-knot input-layer constant (LDS, lane-major), at this lane's block
  const float* xin;   // xin + n0 * XIN_FLOATS
  int voff;           // lane offset inside a matrix's fragment stream (see load_a)
};

// ----------------------------------------------------------------------------
// Per-workgroup state.
// ----------------------------------------------------------------------------
template <int W, int MODE, int CB = 2>
struct TileCtx {
  char* act;
  float* xin;   // [TQ][XIN_FLOATS]
  float* crow;  // [W]
  float* red;   // [RG][RED_VALS][TQ]
  uint32_t* ovf;  // LDS word: a tile of this workgroup overflowed FP16 (see report_overflow)
  float b5;       // the output bias, read once (every tile's final sum adds it)
  // BF16 training, wave 0: the next tile's inputs (knot, point, target) of this
  // lane's query, fetched during the tile before (see process_tile)
  float nx[13];
  bool nx_ok;
  float* vec;  // LDS [4][W]: b2, b3, b4, w_out (lane-major)
  const float* w1p;
  int wave;    // uniform
  __device__ __forceinline__ TileCtx(char* lds, uint32_t* ovf_word, const DevNet& net, int tid)
      : act(lds), ovf(ovf_word), b5(*net.b5p), nx_ok(false), w1p(net.w1p), wave(__builtin_amdgcn_readfirstlane(tid >> 6)) {
    if (tid == 0) *ovf = 0u;  // ordered before any tile's use by the tile's first barrier
    using G = Geo<W, MODE, CB>;
    xin = reinterpret_cast<float*>(lds + G::ACT_BYTES);
    crow = xin + G::TQ * G::XIN_FLOATS;
    float* after = crow + W;
    if constexpr (G::RED_IN_ACT) {
      red = reinterpret_cast<float*>(lds);
    } else {
      red = after;
      after += G::RED_BYTES / 4;
    }
    vec = after;
    // w_out carries the reverse sweep's scale (a power of two, taken out of d and J
    // at the end of the tile)
    for (int i = tid; i < 4 * W; i += G::THREADS) vec[i] = i < 3 * W ? net.bh[i] : net.w5[i - 3 * W] * rev_scale<MODE>();
    // Two waves per SIMD: the first four waves take the matrix cores first, so
    // they reach each layer's epilogue (vector ALU) early and run it while the
    // other four are still in their K loops.
    if constexpr (G::SUB > 1) {
      if (wave < kWaves) __builtin_amdgcn_s_setprio(1);
    }
  }
};

// A thread's place in the tile and the addresses that follow from it, formed anew
// from the thread index by each phase of the tile (a few instructions): kept through
// the tile they took a dozen registers per lane of the 128 that a width-512 wave has
// beside its parked SiLU' values, and pushed some of those into scratch memory.
template <int W, int MODE, int CB = 2>
struct View {
  Lane<W, MODE, CB> ln;
  Bases<W, MODE, CB> b;
  __device__ __forceinline__ explicit View(const TileCtx<W, MODE, CB>& tc) : ln(tc.act, fresh_tid(), tc.wave) {
    using G = Geo<W, MODE, CB>;
    constexpr int MT = G::MT;
    // bytes of one row group's fragment stream (1 KiB per fragment, PMT per K step)
    constexpr int stream_bytes = (MODE == kFP32 ? G::NK8 : G::NKB) * G::PMT * 1024;
    const int pw = ln.wave / G::SUB, sub = ln.wave % G::SUB;  // row group, and this wave's share of it
    // this lane's block of lane-major rows (see lane_major_pos: 16 PMT per (group, h))
    const int lblk = ((pw * 2 + ln.h) * G::PMT + sub * MT) * 16;
    b.bh = tc.vec + lblk;
    b.w5 = tc.vec + 3 * W + lblk;
    b.w1 = tc.w1p + lblk * 12;
    {  // row m = lane%32 of M tile 0 is lane-major row ((pw 2 + h_m) PMT + sub MT) 16 + 4 g_m + r_m
      const int m = ln.n0;
      b.w1a = tc.w1p + ((((pw * 2 + ((m >> 2) & 1)) * G::PMT + sub * MT) * 16) + 4 * (m >> 3) + (m & 3)) * 12;
    }
    b.crow = tc.crow + lblk;
    b.xin = tc.xin + ln.n0 * G::XIN_FLOATS;
    b.voff = pw * stream_bytes + sub * MT * 1024 + ln.lane * 16;
  }
  __device__ __forceinline__ static int fresh_tid() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
  }
};

// Dump of the current LDS tile for training (no-op when not training).
struct TileDump {
  const char* act;  // the LDS activation tile
  void* H;
  void* G;
  int64_t ldb, q0;
  int nvalid;
  size_t layer_elems;  // W * ldb
  size_t elem_bytes;
  // fused MSE loss (Job::target): per-wave output partial sums and the per-query
  // records (slot 11 takes the seed)
  float* dred;
  float* xin;
  const float* target;
  float* d_out;  // the distances, when asked for
  float mse_scale, inv_b;
  float b5;  // the output bias
  // per-workgroup sums over its samples ([kTrainSumRows][width]; BF16 in LDS, FP32 in
  // the workgroup's part of Job::bias_part): rows 0..3 the bias
  // gradients sum_i g_l (l = 1..4), row 4 dL/dw_out = sum_i seed_i h4_i, rows
  // 5..13 dW1[:, c] = sum_i g1_i v_c(i), row 14 (first entry) db_out = sum_i seed_i,
  // row 15 (first entry) the fused loss sum_i (d_i - target_i)^2 / B
  float* bsum;
  __bf16* vt;  // with bsum: the tile's network inputs, transposed (DumpSums::vt)
  float* sp1;  // BF16: SiLU'(z1) of the input layer kept in LDS for the reverse sweep (see train_sp1)
  int width;
  __device__ __forceinline__ float* row(int r) const { return bsum + r * width; }
  // h_{l+1}, l = 0..2, and g_{l+1}, l = 1..3 (h_4 and g_1 are only summed)
  __device__ __forceinline__ void* h(int l) const { return static_cast<char*>(H) + l * layer_elems * elem_bytes; }
  __device__ __forceinline__ void* g(int l) const { return static_cast<char*>(G) + (l - 1) * layer_elems * elem_bytes; }
};

// Whether a hidden-layer epilogue keeps its packed results in registers across
// the barrier (two waves of one workgroup per SIMD), except training's last forward
// layer, which stores h4 first.
template <int W, int MODE, int CB, bool TRAIN>
constexpr bool defer_stores(bool last_forward) {
  return Geo<W, MODE, CB>::SUB > 1 && (!last_forward || !TRAIN);
}

// The packed words of elements 8 GP .. 8 GP + 7 of an accumulator go back into
// those elements (consumed in order, so no extra registers), and are written out
// after the barrier.
template <int MODE, int AM, int GP>
__device__ __forceinline__ void park_packed(const float x[8], const float y[8], f32x16& a) {
  uint32_t w[8];
  act_pack8<AM, !lane_k_order<MODE>()>(x, y, w);
  constexpr int NWORDS = AM == kBF16X2 ? 8 : 4;  // hi and lo words, or hi only
#pragma unroll
  for (int k = 0; k < NWORDS; ++k) a[8 * GP + k] = __uint_as_float(w[k]);
}

template <int W, int MODE, int CB, int AM>
__device__ __forceinline__ void write_packed(const Lane<W, MODE, CB>& ln, const f32x16 (&acc)[(Geo<W, MODE, CB>::MT)][CB]) {
  static_for<Geo<W, MODE, CB>::MT>([&](auto I) {
    static_for<2>([&](auto GP) {
      static_for<CB>([&](auto NT) {
        uint32_t w[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) w[k] = __float_as_uint(acc[I][NT][8 * GP + k]);
        act_write8<W, MODE, CB, I, GP, NT, AM>(ln, w);
      });
    });
  });
}

template <int W, int MODE, int CB, int L, bool TRAIN, bool GRAD>
__device__ __forceinline__ void fwd_hidden(const DevNet& net, const TileCtx<W, MODE, CB>& tc,
                                           float (&sp)[2][(Geo<W, MODE, CB>::MT)][CB][16], float (&dpart)[Geo<W, MODE, CB>::GPW][CB],
                                           const TileDump& td, APre<W, MODE, CB>& ap) {
  constexpr int MT = Geo<W, MODE, CB>::MT;
  const View<W, MODE, CB> v0(tc);
  f32x16 acc[MT][CB];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4 b4 = *reinterpret_cast<const f32x4*>(v0.b.bh + L * W + 16 * i + 4 * g);
#pragma unroll
      for (int nt = 0; nt < CB; ++nt)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][nt][4 * g + r] = b4[r];
    }
  const void* next = L < 2 ? net.fwd[L + 1] : net.bwd[2];
  layer_gemm<W, MODE, CB, fwd_arith<MODE>()>(acc, net.fwd[L], next, v0.b.voff,
                                             v0.ln.act_r, ap);
  const View<W, MODE, CB> vw(tc);
  const Lane<W, MODE, CB>& ln = vw.ln;
  const Bases<W, MODE, CB>& b = vw.b;
  // arithmetic of what this layer stores: the next layer's activations, or g4
  // for the reverse sweep
  constexpr int SA = L == 2 ? rev_arith<MODE>() : fwd_arith<MODE>();
  // With two waves per SIMD the epilogue arithmetic runs before the barrier (the
  // results wait in registers), overlapping the K loops of waves still running;
  // only the stores into the tile they read wait for it.
  constexpr bool DEFER = defer_stores<W, MODE, CB, TRAIN>(L == 2);
  if constexpr (!DEFER) __syncthreads();
  if constexpr (TRAIN && L == 2) {
    // training: the layer-4 activations h4 go through LDS first (for dL/dw_out),
    // and the output-layer partial sums are taken here, so that a fused loss can
    // finish d before the reverse sweep
    static_for<MT>([&](auto I) {
      static_for<2>([&](auto GP) {
        const f32x4 w5r[2] = {*reinterpret_cast<const f32x4*>(b.w5 + 16 * I + 8 * GP),
                              *reinterpret_cast<const f32x4*>(b.w5 + 16 * I + 8 * GP + 4)};
        static_for<CB>([&](auto NT) {
          float v[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            // SiLU' replaces z4 in the accumulator, for g4 below
            float dv;
            silu_fwd(acc[I][NT][8 * GP + q], v[q], dv);
            acc[I][NT][8 * GP + q] = dv;
            dpart[0][NT] += w5r[q >> 2][q & 3] * v[q];
          }
          act_store_pair<W, MODE, CB, I, GP, NT>(ln, v);
        });
      });
    });
    if (td.target) {
      // d over the rows: lane halves, then waves in order, as at the end of the tile
#pragma unroll
      for (int nt = 0; nt < CB; ++nt) {
        const float dp = dpart[0][nt] + __shfl_xor(dpart[0][nt], 32);
        if (ln.h == 0) td.dred[ln.wave * kTileQ + 32 * nt + ln.n0] = dp;
      }
    }
    __syncthreads();
    if (threadIdx.x < kTileQ) {  // wave 0, one lane per query
      const int n = threadIdx.x;
      float* seedp = td.xin + n * Geo<W, MODE, CB>::XIN_FLOATS + 11;
      float sq = 0.f;
      if (td.target) {
        float sum = td.dred[n];
#pragma unroll
        for (int w = 1; w < Geo<W, MODE, CB>::NW; ++w) sum += td.dred[w * kTileQ + n];
        const float dv = sum + td.b5;
        const bool valid = n < td.nvalid;
        const int64_t q = td.q0 + n;
        const float r = valid ? dv - td.xin[n * Geo<W, MODE, CB>::XIN_FLOATS + kXinTarget] : 0.f;
        const float seed = td.mse_scale * r;  // dL/dd for L = mean (d - target)^2
        sq = td.inv_b * (r * r);
        *seedp = seed;
        if (valid && td.d_out) td.d_out[q] = dv;
      }
      if constexpr (MODE == kBF16) {  // the seeds' parts for the sums over h4
        const float sd = *seedp;
        const __bf16 hi = (__bf16)sd;
        const float r1 = sd - (float)hi;
        const __bf16 mid = (__bf16)r1;
        td.vt[kVtSeed * kTileQ + n] = hi;
        td.vt[(kVtSeed + 1) * kTileQ + n] = mid;
        td.vt[(kVtSeed + 2) * kTileQ + n] = (__bf16)(r1 - (float)mid);
      }
      {
        // db_out = sum_i seed_i and the loss, over the tile (fixed butterfly), then
        // over this workgroup's tiles in order
        float sd = *seedp;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
          sd += __shfl_xor(sd, off);
          sq += __shfl_xor(sq, off);
        }
        if (n == 0) {
          td.row(14)[0] += sd;
          td.row(15)[0] += sq;
        }
      }
    }
    // h4 is needed only for dL/dw_out = sum_i seed_i h4_i, summed here (after a
    // barrier: wave 0 wrote the seeds the copy reads)
    __syncthreads();
    const DumpSums sm{td.row(4), td.xin + 11, nullptr, td.vt, nullptr, 0, 0};
    dump_tile<W, MODE>(td.act, nullptr, td.ldb, td.q0, td.nvalid, &sm, false);
    __syncthreads();  // h4 fully read before g4 overwrites the tile; seeds written
  }
  static_for<MT>([&](auto I) {
    static_for<2>([&](auto GP) {
      f32x4 w5r[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
      if constexpr (L == 2) {
        w5r[0] = *reinterpret_cast<const f32x4*>(b.w5 + 16 * I + 8 * GP);
        w5r[1] = *reinterpret_cast<const f32x4*>(b.w5 + 16 * I + 8 * GP + 4);
      }
      static_for<CB>([&](auto NT) {
        const float seed = TRAIN ? b.xin[NT * 32 * Geo<W, MODE, CB>::XIN_FLOATS + 11] : 1.f;
        float x[8], y[8];  // what is stored, as products
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int j = 8 * GP + q;  // accumulator element: g = 2 GP + q/4, r = q%4
          const float z = acc[I][NT][j];
          float sg = 0.f, hv = 0.f, dv = 0.f;
          if constexpr (TRAIN && L == 2) {
            dv = z;  // SiLU'(z4), kept above
          } else {
            sg = sigmoid(z);
            hv = z * sg;
            dv = sg + hv * (1.0f - sg);
          }
          if constexpr (L < 2) {
            if constexpr (GRAD) sp[L][I][NT][j] = park(dv);
            x[q] = z;
            y[q] = sg;
          } else {
            if constexpr (!TRAIN) dpart[Geo<W, MODE, CB>::GPW > 1 ? (int)I : 0][NT] += w5r[q >> 2][q & 3] * hv;  // (training: above)
            // g4 = seed * w5 * SiLU'(z4); the query's seed 1 (times rev_scale) is in w5
            x[q] = w5r[q >> 2][q & 3] * dv;
            asm("" : "+v"(x[q]));  // rounded before the seed (1 in the query) multiplies it
            y[q] = seed;
          }
        }
        if constexpr (L < 2 || GRAD) {
          if constexpr (DEFER) park_packed<MODE, SA, GP>(x, y, acc[I][NT]);
          else act_store_pair<W, MODE, CB, I, GP, NT, SA>(ln, x, y);
        }
      });
      __builtin_amdgcn_sched_barrier(0);
    });
  });
  if constexpr (L == 2) {
    // Materialise the output-layer partial sums here; left alone, the compiler
    // sinks them to their use after the reverse sweep and keeps every h4 and
    // w_out value live through it.
#pragma unroll
    for (int k = 0; k < Geo<W, MODE, CB>::GPW; ++k)
#pragma unroll
      for (int nt = 0; nt < CB; ++nt) asm volatile("" : "+v"(dpart[k][nt]));
  }
  if constexpr (DEFER) {
    __syncthreads();  // every wave has finished reading the tile
    if constexpr (L < 2 || GRAD) write_packed<W, MODE, CB, SA>(ln, acc);
  }
  __syncthreads();
  // training: h2, h3 (layers 2, 3) or g4 (layer 4) to HBM; the tile is next
  // overwritten only after the following K loop and its barrier
  if constexpr (TRAIN) {  // h2, h3, or g4 (with db4 = sum_i g4_i)
    const DumpSums sm{td.row(3), nullptr, nullptr, td.vt, nullptr, 0, 0};
    dump_tile<W, MODE>(td.act, L < 2 ? td.h(L + 1) : td.g(3), td.ldb, td.q0, td.nvalid, L == 2 ? &sm : nullptr);
  }
}

template <int W, int MODE, int CB, int L, bool TRAIN>
__device__ __forceinline__ void bwd_hidden(const DevNet& net, const TileCtx<W, MODE, CB>& tc,
                                           const float (&sp)[2][(Geo<W, MODE, CB>::MT)][CB][16], const TileDump& td,
                                           APre<W, MODE, CB>& ap) {
  constexpr int MT = Geo<W, MODE, CB>::MT;
  f32x16 acc[MT][CB];
  constexpr int RA = rev_arith<MODE>();
  // Single FP16 products use only the hi halves of the tile, so the two reverse
  // layers alternate halves: g4 (hi) -> g3 (lo) -> g2 (hi).  Nobody reads the half
  // a layer writes, so its stores need no barrier before them.
  constexpr bool PP = RA == kF16 && !TRAIN;
  const View<W, MODE, CB> v0(tc);
  const char* br = (PP && L == 1) ? v0.ln.act_r + Geo<W, MODE, CB>::LO_OFF : v0.ln.act_r;
  if constexpr (!rev_zero_c<MODE>()) zero_acc<W, MODE, CB>(acc);
  layer_gemm<W, MODE, CB, RA, rev_zero_c<MODE>()>(acc, net.bwd[L], net.bwd[L - 1], v0.b.voff,
                                                  br, ap);
  const View<W, MODE, CB> vw(tc);
  const Lane<W, MODE, CB>& ln = vw.ln;
  constexpr bool DEFER = !PP && defer_stores<W, MODE, CB, TRAIN>(false);  // as in fwd_hidden
  if constexpr (!DEFER && !PP) __syncthreads();
  static_for<MT>([&](auto I) {
    static_for<2>([&](auto GP) {
      static_for<CB>([&](auto NT) {
        float x[8], y[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int j = 8 * GP + q;
          x[q] = acc[I][NT][j];
          y[q] = unpark(sp[L - 1][I][NT][j], x[q]);
        }
        if constexpr (PP) {
          uint32_t w[8];
          act_pack8<RA, !lane_k_order<MODE>()>(x, y, w);
          typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
          constexpr int off = (2 * I + GP) * Geo<W, MODE, CB>::STEP_BYTES + NT * 512;
          *reinterpret_cast<u32x4*>((L == 2 ? ln.act_w_lo : ln.act_w) + off) = u32x4{w[0], w[1], w[2], w[3]};
        } else if constexpr (DEFER) {
          park_packed<MODE, RA, GP>(x, y, acc[I][NT]);
        } else {
          act_store_pair<W, MODE, CB, I, GP, NT, RA>(ln, x, y);
        }
      });
      __builtin_amdgcn_sched_barrier(0);
    });
  });
  if constexpr (DEFER) {
    __syncthreads();  // every wave has finished reading the tile
    write_packed<W, MODE, CB, RA>(ln, acc);
  }
  __syncthreads();
  if constexpr (TRAIN) {  // g3 or g2, with their bias sums
    const DumpSums sm{td.row(L), nullptr, nullptr, td.vt, nullptr, 0, 0};
    dump_tile<W, MODE>(td.act, td.g(L), td.ldb, td.q0, td.nvalid, &sm);
  }
}

// Pure-BF16 pair-list tiles of width 256 (point obstacles; the training
// configuration) take the input layer's pre-activations from the matrix cores:
// z1 = b1 + W1 v over the 9 inputs, K
// padded to 16 (p' at k = 0..2, the arm joints at 3..8), as the split products
// W1h vh + W1h vl + W1l vh accumulated in FP32 (h: the BF16 rounding, l: the BF16
// rounding of the rest; the terms left out are below 2^-16 |W1| |v|).  The
// prologue stages the tile's inputs as B fragments at `vb` (query n at byte 64 n:
// 16 BF16 hi, then 16 lo).  The forward and the reverse sweep's recomputation
// both call this for M tile I, so they see the same z1.
template <int W, int MODE>
constexpr bool mma_input(bool pairs, bool sph) {
  return W == 256 && MODE == kBF16 && pairs && !sph;  // (at width 512 the recomputation would spill)
}
constexpr int kVbBytes = 64;  // per query: B fragments of the inputs, hi then lo

template <int W, int MODE, int CB, int I>
__device__ __forceinline__ void input_gemm(const Lane<W, MODE, CB>& ln, const Bases<W, MODE, CB>& b, const char* vb,
                                           f32x16 (&z)[CB]) {
  bf16x8 bh[CB], bl[CB];
#pragma unroll
  for (int nt = 0; nt < CB; ++nt) {
    const char* p = vb + (32 * nt + ln.n0) * kVbBytes + ln.kh * 16;
    bh[nt] = *reinterpret_cast<const bf16x8*>(p);
    bl[nt] = *reinterpret_cast<const bf16x8*>(p + 32);
  }
  // A: row m = lane%32 of the tile, inputs 8 kh .. 8 kh + 7
  const float* w = b.w1a + I * 16 * 12;
  const f32x4 wa = *reinterpret_cast<const f32x4*>(w);
  const f32x4 wb = *reinterpret_cast<const f32x4*>(w + 4);
  const f32x2 wc = *reinterpret_cast<const f32x2*>(w + 8);
  const float lo8[8] = {wa[0], wa[1], wa[2], wb[0], wb[1], wb[2], wb[3], wc[0]};  // k = 0..7 (slot 3 is b1)
  bf16x8 ah, al;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float a = ln.kh ? (e == 0 ? wc[1] : 0.f) : lo8[e];  // k = 8: the last arm joint
    const __bf16 hi = (__bf16)a;
    ah[e] = hi;
    al[e] = (__bf16)(a - (float)hi);
  }
  // b1 of the accumulator layout's rows (lane-major block of this lane)
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float bias = b.w1[(16 * I + 4 * g + r) * 12 + 3];
#pragma unroll
      for (int nt = 0; nt < CB; ++nt) z[nt][4 * g + r] = bias;
    }
#pragma unroll
  for (int nt = 0; nt < CB; ++nt) {
    z[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh[nt], z[nt], 0, 0, 0);
    z[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl[nt], z[nt], 0, 0, 0);
    z[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh[nt], z[nt], 0, 0, 0);
  }
}

// Pre-activations z1 of M tile I (32 rows) and column block NT, in FP32 on the
// matrix cores: z = c + W1 x with two steps (p'x, p'y), (p'z, radius) of
// v_mfma_f32_32x32x2_f32 on top of the knot's arm term (dense tiles; pair lists:
// b1, then three steps for the arm joints first).  That instruction adds its two
// products one after the other as fused multiply-adds, so z1 has the bits of the
// chain c + w0 x0 + w1 x1 + w2 x2 of arm_term's order, at 2 issue slots for 16
// elements instead of 48, and a row's weights are loaded once per tile of rows
// rather than by every lane.
template <int W, int MODE, int CB, bool PAIRS>
__device__ __forceinline__ void input_preact_tile(const Lane<W, MODE, CB>& ln, const Bases<W, MODE, CB>& b, int i, int nt,
                                                  f32x16& z) {
  constexpr int XF = Geo<W, MODE, CB>::XIN_FLOATS;
  const float* w = b.w1a + i * 16 * 12;    // A: row lane%32 of the tile, step element kh
  const float* x = b.xin + nt * 32 * XF;   // B: query lane%32 of the block, step element kh
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    f32x4 c4;
    if constexpr (PAIRS) {
#pragma unroll
      for (int r = 0; r < 4; ++r) c4[r] = b.w1[(16 * i + 4 * g + r) * 12 + 3];  // b1
    } else {
      c4 = *reinterpret_cast<const f32x4*>(b.crow + 16 * i + 4 * g);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) z[4 * g + r] = c4[r];
  }
  if constexpr (PAIRS) {
#pragma unroll
    for (int a = 0; a < 6; a += 2) z = __builtin_amdgcn_mfma_f32_32x32x2f32(w[4 + a + ln.kh], x[5 + a + ln.kh], z, 0, 0, 0);
  }
  z = __builtin_amdgcn_mfma_f32_32x32x2f32(w[ln.kh], x[ln.kh], z, 0, 0, 0);
  z = __builtin_amdgcn_mfma_f32_32x32x2f32(w[2 + 8 * ln.kh], x[2 + (kXinRadius - 2) * ln.kh], z, 0, 0, 0);
}

// Last reverse layer: g1 = (W2^T g2) * SiLU'(z1) with z1 recomputed, then the eight
// input-gradient components that J needs (p'x, p'y, a1..a6; dd/dp'z is not a
// configuration coordinate), summed per lane in FP32: lane (n, h) adds w_r[c] g1[r]
// over its rows r in order, four components per v_mfma_f32_4x4x1_16b_f32.  In that
// instruction's 4-lane blocks lane l supplies component l%4 of the row (A) and its
// own g1 (B) and holds the four sums of its own column (D), each the fused
// multiply-add chain that the vector ALU would run, at 2 issue slots for an element's
// 8 sums; a lane loads 2 floats of a row instead of 12, one group of four rows ahead.
template <int CB>
struct GradSums {
  f32x4 v[CB][2];  // [column block][p'x p'y a1 a2 | a3..a6]
};

template <int W, int MODE, int CB, bool PAIRS, bool TRAIN, bool SPH, class F>
__device__ __forceinline__ void bwd_input(const DevNet& net, const TileCtx<W, MODE, CB>& tc,
                                          GradSums<CB> (&epart)[Geo<W, MODE, CB>::GPW], const TileDump& td, const char* vb,
                                          APre<W, MODE, CB>& ap, F&& before_copy) {
  constexpr int MT = Geo<W, MODE, CB>::MT;
  const View<W, MODE, CB> v0(tc);
  f32x16 acc[MT][CB];
  if constexpr (!rev_zero_c<MODE>()) zero_acc<W, MODE, CB>(acc);
  layer_gemm<W, MODE, CB, rev_arith<MODE>(), rev_zero_c<MODE>()>(acc, net.bwd[0], net.bwd[0], v0.b.voff, v0.ln.act_r, ap);
  const View<W, MODE, CB> vw(tc);
  const Lane<W, MODE, CB>& ln = vw.ln;
  const Bases<W, MODE, CB>& b = vw.b;
  float g1keep[TRAIN ? MT : 1][CB][16];
  constexpr bool KEPT = TRAIN && MODE == kBF16;  // SiLU'(z1) kept by the input layer
  if constexpr (KEPT) {
    constexpr int T = Geo<W, MODE, CB>::THREADS;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int nt = 0; nt < CB; ++nt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 sv = *reinterpret_cast<const f32x4*>(td.sp1 + (((i * 2 + nt) * 4 + g) * T + threadIdx.x) * 4);
#pragma unroll
          for (int r = 0; r < 4; ++r) g1keep[i][nt][4 * g + r] = acc[i][nt][4 * g + r] * sv[r];
        }
  }
  // this lane's component pair of packed row k (slots p'x p'y . . a1 a2 a3 a4 a5 a6 . .)
  const float* we = b.w1 + (ln.lane & 3);
  const int c0 = (ln.lane & 2);  // a1, a2 sit two slots past p'x, p'y
  float a[2][4][2];
  auto load_rows = [&](float (&x)[4][2], int grp) {  // rows 4 grp .. 4 grp + 3 of this lane
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float* w = we + (4 * grp + r) * 12;
      x[r][0] = w[c0];
      x[r][1] = w[6];
    }
  };
  if constexpr (!KEPT) {
    if constexpr (!TRAIN) load_rows(a[0], 0);
    static_for<MT>([&](auto I) {
      if constexpr (mma_input<W, MODE>(PAIRS, SPH)) {
        f32x16 z[CB];
        input_gemm<W, MODE, CB, I>(ln, b, vb, z);
#pragma unroll
        for (int nt = 0; nt < CB; ++nt)
#pragma unroll
          for (int j = 0; j < 16; ++j) acc[I][nt][j] *= silu_prime_only(z[nt][j]);
      } else {
#pragma unroll
        for (int nt = 0; nt < CB; ++nt) {
          f32x16 z;
          input_preact_tile<W, MODE, CB, PAIRS>(ln, b, I, nt, z);
#pragma unroll
          for (int j = 0; j < 16; ++j) acc[I][nt][j] *= silu_prime_only(z[j]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if constexpr (TRAIN) {  // training needs g1, not J
#pragma unroll
        for (int nt = 0; nt < CB; ++nt)
#pragma unroll
          for (int j = 0; j < 16; ++j) g1keep[I][nt][j] = acc[I][nt][j];
      } else {
        GradSums<CB>& ep = epart[Geo<W, MODE, CB>::GPW > 1 ? (int)I : 0];
        static_for<4>([&](auto GG) {
          constexpr int grp = 4 * I + GG;
          if constexpr (grp + 1 < 4 * MT) load_rows(a[(grp + 1) & 1], grp + 1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
              for (int nt = 0; nt < CB; ++nt)
                ep.v[nt][k] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[grp & 1][r][k], acc[I][nt][4 * GG + r], ep.v[nt][k], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        });
      }
    });
  }
  if constexpr (TRAIN) {
    // training: g1 through LDS to HBM (every wave has finished reading g2)
    __syncthreads();
    static_for<MT>([&](auto I) {
      static_for<2>([&](auto GP) {
        static_for<CB>([&](auto NT) {
          float v[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) v[q] = g1keep[I][NT][8 * GP + q];
          act_store_pair<W, MODE, CB, I, GP, NT>(ln, v);
        });
      });
    });
    __syncthreads();
    before_copy();
    // g1 is needed only for db1 and dW1 = sum_i g1_i v_i^T, summed here
    const DumpSums sm{td.row(0), nullptr, td.row(5), td.vt, td.xin, Geo<W, MODE>::XIN_FLOATS, 2};
    dump_tile<W, MODE>(td.act, nullptr, td.ldb, td.q0, td.nvalid, &sm, false);
  }
}

// Input layer (FP32): z1 = W1 [p'; a] + b1, h1 = SiLU(z1) -> LDS.  KEEP: SiLU'(z1)
// also goes to sp1 (train_sp1's layout) for the reverse sweep.
template <int W, int MODE, int CB, bool PAIRS, bool SPH, bool KEEP = false>
__device__ __forceinline__ void fwd_input(const TileCtx<W, MODE, CB>& tc, const char* vb,
                                          float* sp1 = nullptr) {
  constexpr int MT = Geo<W, MODE, CB>::MT;
  const View<W, MODE, CB> vw(tc);
  const Lane<W, MODE, CB>& ln = vw.ln;
  const Bases<W, MODE, CB>& b = vw.b;
  static_assert(!KEEP || mma_input<W, MODE>(PAIRS, SPH), "SiLU'(z1) is kept by the BF16 training tiles");
  if constexpr (mma_input<W, MODE>(PAIRS, SPH)) {
    static_for<MT>([&](auto I) {
      f32x16 z[CB];
      input_gemm<W, MODE, CB, I>(ln, b, vb, z);
      static_for<2>([&](auto GP) {
        static_for<CB>([&](auto NT) {
          float v[8], dv[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            if constexpr (KEEP) silu_fwd(z[NT][8 * GP + q], v[q], dv[q]);
            else v[q] = silu_only(z[NT][8 * GP + q]);
          }
          act_store_pair<W, MODE, CB, I, GP, NT>(ln, v);
          if constexpr (KEEP) {
            constexpr int T = Geo<W, MODE, CB>::THREADS;
            constexpr int k = ((I * 2 + NT) * 16 + 8 * GP) / 4;  // first of the two 16-byte groups
#pragma unroll
            for (int h = 0; h < 2; ++h)
              *reinterpret_cast<f32x4*>(sp1 + ((k + h) * T + threadIdx.x) * 4) =
                  f32x4{dv[4 * h], dv[4 * h + 1], dv[4 * h + 2], dv[4 * h + 3]};
          }
        });
        __builtin_amdgcn_sched_barrier(0);
      });
    });
    return;
  }
  static_for<MT>([&](auto I) {
    static_for<CB>([&](auto NT) {
      f32x16 z;
      input_preact_tile<W, MODE, CB, PAIRS>(ln, b, I, NT, z);
      static_for<2>([&](auto GP) {
        float x[8], y[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          x[q] = z[8 * GP + q];
          y[q] = sigmoid(x[q]);
        }
        act_store_pair<W, MODE, CB, I, GP, NT>(ln, x, y);
      });
      __builtin_amdgcn_sched_barrier(0);
    });
  });
}

// LDS that training adds after the query's own: the fused loss's per-wave
// partial sums ([waves][64]) and, for pure BF16, the per-workgroup sums of
// TileDump::bsum ([kTrainSumRows][W]) and the tile's transposed inputs
// (TileDump::vt).
template <int W, int MODE>
constexpr int train_extra_lds() {
  return Geo<W, MODE>::NW * kTileQ * 4 +
         (MODE == kBF16 ? kTrainSumRows * W * 4 + kVtRows * kTileQ * 2 + W * kTileQ * 4 : 0);
}
template <int W, int MODE>
__device__ __forceinline__ float* train_bsum(char* lds) {
  if constexpr (MODE == kBF16) return reinterpret_cast<float*>(lds + Geo<W, MODE>::LDS_BYTES + Geo<W, MODE>::NW * kTileQ * 4);
  return nullptr;
}
template <int W, int MODE>
__device__ __forceinline__ __bf16* train_vt(char* lds) {
  if constexpr (MODE == kBF16) return reinterpret_cast<__bf16*>(train_bsum<W, MODE>(lds) + kTrainSumRows * W);
  return nullptr;
}
// BF16 training: SiLU'(z1) of the tile (W x 64 floats), written by the input layer
// and read back by the last reverse layer, each thread its own values (16-byte
// group k of thread t at float (k THREADS + t) 4), so no barrier orders them.
template <int W, int MODE>
__device__ __forceinline__ float* train_sp1(char* lds) {
  if constexpr (MODE == kBF16) return reinterpret_cast<float*>(train_vt<W, MODE>(lds) + kVtRows * kTileQ);
  return nullptr;
}

// A load that stays a vector load, also where its address is the same for a whole wave.
__device__ __forceinline__ float live_load(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// One tile: 64 points of knot kk starting at point q0 (dense), or pair-list
// entries q0 .. q0+63 (pairs).  Every thread of the workgroup calls it; consecutive
// calls can reuse the shared memory, but the last stores of J are issued after the
// last barrier.  GRAD: the reverse sweep and J too; without it the tile ends with d
// (and keeps no SiLU').  SPH: the
// obstacles are spheres (x, y, z, r) and the network input is [p', r, a].  LIVE: the
// knots may have been rewritten since the kernel started (serving), so they are read
// through the vector caches, which the workgroup has invalidated when it saw the request
// published; no fence of the running kernel reaches the scalar cache.
template <int W, int MODE, int CB, bool GRAD, bool PAIRS, bool TRAIN = false, bool GATHER = false, bool SPH = false,
          bool LIVE = false>
__device__ __forceinline__ void process_tile(const DevNet& net, const Job& job, int64_t kk, int64_t q0,
                                             TileCtx<W, MODE, CB>& tc) {
  using G = Geo<W, MODE, CB>;
  constexpr int MT = G::MT;
  constexpr int XF = G::XIN_FLOATS;
  constexpr int TQ = G::TQ;
  static_assert(!TRAIN || CB == 2, "training runs 64-sample tiles");
  const int tid = threadIdx.x;
  float* xin = tc.xin;
  float* crow = tc.crow;
  float* red = tc.red;
  const int64_t qlimit = PAIRS ? job.npairs : (GATHER ? job.row_off[kk + 1] : job.Np);

  // BF16 training: sample i = knot i, point i; the inputs of a workgroup's next tile
  // are fetched before this tile's last copy (no vector-memory wait comes between
  // them and the barrier that ends the tile) and read from registers by its prologue
  constexpr bool PREFETCH = TRAIN && PAIRS && MODE == kBF16 && !SPH;
  const bool fetched = PREFETCH && tc.nx_ok;
  auto fetch_next = [&]() {
    if constexpr (PREFETCH) {
      const int64_t qn = q0 + (int64_t)gridDim.x * TQ;
      tc.nx_ok = qn < qlimit && !job.pidx32;
      if (tid < TQ && tc.nx_ok) {
        const int64_t q = qn + tid;
        const int64_t qc = q < qlimit ? q : qlimit - 1;
        const float* kn = job.knots + qc * kInDim;
#pragma unroll
        for (int c = 0; c < kInDim; ++c) tc.nx[c] = kn[c];
        const float* pt = job.points + qc * 3;
#pragma unroll
        for (int c = 0; c < 3; ++c) tc.nx[kInDim + c] = pt[c];
        tc.nx[12] = (!job.seed && job.target && q < qlimit) ? job.target[qc] : 0.f;
      }
    }
  };

  // ---- prologue: base-frame points (+ per-knot arm term of the input layer) ----
  if (tid < TQ) {
    const int64_t q = q0 + tid;
    const int64_t qc = q < qlimit ? q : qlimit - 1;   // clamp the ragged tail (never stored)
    int64_t ki = 0, pi = 0;
    if constexpr (PAIRS) {
      ki = qc;
      if (!TRAIN && job.dec_keys) {
        // J at the minimum: pair q is knot q and the point its key names; the minimum
        // and its index are written here too
        float dm;
        int32_t am;
        minkey_decode(job.dec_keys[qc], dm, am);
        if (q < qlimit) {
          job.dec_dmin[q] = dm;
          job.dec_argmin[q] = am;
          job.dec_keys[q] = 0ull;
        }
        pi = am;
      } else {
        pi = job.pidx32 ? (int64_t)job.pidx32[qc] : qc;
      }
    } else {
      ki = kk;
      pi = GATHER ? (int64_t)job.pgather[qc] : qc;
    }
    float kn[kInDim], pxyz[4];
    if (fetched) {
#pragma unroll
      for (int c = 0; c < kInDim; ++c) kn[c] = tc.nx[c];
#pragma unroll
      for (int c = 0; c < 3; ++c) pxyz[c] = tc.nx[kInDim + c];
      pxyz[3] = 0.f;
    } else {
      if constexpr (PAIRS) {
        const float* knp = job.knots + ki * kInDim;
#pragma unroll
        for (int c = 0; c < kInDim; ++c) kn[c] = knp[c];
      } else if constexpr (LIVE) {
#pragma unroll
        for (int c = 0; c < kInDim; ++c) kn[c] = live_load(job.knots + ki * kInDim + c);
      } else {
        // one knot per tile: scalar loads (the knots are read-only during the launch)
        const __attribute__((address_space(4))) float* knp =
            (const __attribute__((address_space(4))) float*)(job.knots + ki * kInDim);
#pragma unroll
        for (int c = 0; c < kInDim; ++c) kn[c] = knp[c];
      }
      if ((PAIRS || GATHER) && (uint64_t)pi >= (uint64_t)job.Np) {
        pxyz[0] = pxyz[1] = pxyz[2] = pxyz[3] = __builtin_nanf("");  // bad point index: NaN results
      } else {
        const float* pt = job.points + pi * (SPH ? 4 : 3);
        pxyz[0] = pt[0];
        pxyz[1] = pt[1];
        pxyz[2] = pt[2];
        pxyz[3] = SPH ? pt[3] : 0.f;
      }
    }
    float sn, cs;
    sincosf(kn[2], &sn, &cs);
    const float ux = pxyz[0] - kn[0], uy = pxyz[1] - kn[1];
    // the record's address is formed here, once per tile: hoisted out of the tile
    // loop, its pieces were kept in spill slots and reloaded one by one
    int tq = tid;
    asm volatile("" : "+v"(tq));
    float* x = xin + tq * XF;
    x[0] = cs * ux + sn * uy;
    x[1] = -sn * ux + cs * uy;
    x[2] = pxyz[2];
    x[3] = cs;
    x[4] = sn;
#pragma unroll
    for (int c = 0; c < 6; ++c) x[5 + c] = kn[3 + c];
    // reverse-sweep seed: dL/dd for training, else 1 (multiplying by 1 is exact;
    // the constant is formed here, a copy kept from before the tile loop was spilled)
    float one = 1.f;
    asm volatile("" : "+v"(one));
    x[11] = job.seed ? (q < qlimit ? job.seed[qc] : 0.f) : one;
    // the fused loss's target, fetched with the inputs rather than after the forward
    if constexpr (TRAIN)
      x[kXinTarget] = fetched ? tc.nx[12] : (!job.seed && job.target && q < qlimit) ? job.target[qc] : 0.f;
    if constexpr (TRAIN && MODE == kBF16) {
      // the network inputs transposed and split into BF16 hi + lo, for dW1 on the
      // matrix cores (the ragged tail's inputs meet zero gradients)
      __bf16* vt = train_vt<W, MODE>(tc.act);
#pragma unroll
      for (int c = 0; c < 9; ++c) {
        const float v = x[c < 3 ? c : c + 2];
        const __bf16 hi = (__bf16)v;
        vt[c * TQ + tid] = hi;
        vt[(9 + c) * TQ + tid] = (__bf16)(v - (float)hi);
      }
    }
    x[kXinRadius] = SPH ? pxyz[3] : 0.f;  // the radius passes through the rigid transform
    if constexpr (mma_input<W, MODE>(PAIRS, SPH)) {
      // the inputs as B fragments of the matrix-core input layer (input_gemm), in
      // the idle half of the activation tile
      const float v[16] = {x[0], x[1], x[2], x[5], x[6], x[7], x[8], x[9], x[10], 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      bf16x8 vh[2], vl[2];
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const __bf16 hi = (__bf16)v[k];
        vh[k >> 3][k & 7] = hi;
        vl[k >> 3][k & 7] = (__bf16)(v[k] - (float)hi);
      }
      char* o = tc.act + G::ACT_BYTES / 2 + tid * kVbBytes;
      *reinterpret_cast<bf16x8*>(o) = vh[0];
      *reinterpret_cast<bf16x8*>(o + 16) = vh[1];
      *reinterpret_cast<bf16x8*>(o + 32) = vl[0];
      *reinterpret_cast<bf16x8*>(o + 48) = vl[1];
    }
  }
  if constexpr (!PAIRS) {
    // the knot's arm joints, by scalar loads as above
    float arm[6];
    if constexpr (LIVE) {
#pragma unroll
      for (int c = 0; c < 6; ++c)
        arm[c] = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(live_load(job.knots + kk * kInDim + 3 + c))));
    } else {
      const __attribute__((address_space(4))) float* ka =
          (const __attribute__((address_space(4))) float*)(job.knots + kk * kInDim + 3);
#pragma unroll
      for (int c = 0; c < 6; ++c) arm[c] = ka[c];
    }
    int r0 = tid;  // (opaque, so the addresses below are formed here, per tile, not kept spilled)
    asm volatile("" : "+v"(r0));
    for (int r = r0; r < W; r += G::THREADS) {  // r: lane-major position
      const float* w = net.w1p + r * 12;
      crow[r] = arm_term(w[3], w[4], w[5], w[6], w[7], w[8], w[9], arm);
    }
  }
  __syncthreads();

  TileDump td{};
  if constexpr (TRAIN) {
    td.act = tc.act;
    td.H = job.dumpH;
    td.G = job.dumpG;
    td.ldb = job.ldb;
    td.q0 = q0;
    td.nvalid = (int)(qlimit - q0 < TQ ? qlimit - q0 : TQ);
    td.layer_elems = (size_t)W * job.ldb;
    td.elem_bytes = MODE == kFP32 ? 4 : 2;
    // LDS beyond the query's own: the fused loss's partial sums ([waves][64])
    td.dred = reinterpret_cast<float*>(tc.act + G::LDS_BYTES);
    td.bsum = MODE == kBF16 ? train_bsum<W, MODE>(tc.act) : job.bias_part + (int64_t)blockIdx.x * kTrainSumRows * W;
    td.vt = train_vt<W, MODE>(tc.act);
    td.sp1 = train_sp1<W, MODE>(tc.act);
    td.width = W;
    td.xin = xin;
    td.target = job.seed ? nullptr : job.target;
    td.d_out = job.seed ? nullptr : job.d;
    td.mse_scale = job.mse_scale;
    td.b5 = tc.b5;
    td.inv_b = job.inv_b;
  }
  APre<W, MODE, CB> ap;  // each layer's first weight fragments, requested ahead of it
  preload_a<W, MODE, CB>(ap, net.fwd[0], View<W, MODE, CB>(tc).b.voff);
  fwd_input<W, MODE, CB, PAIRS, SPH, TRAIN && MODE == kBF16>(tc, tc.act + G::ACT_BYTES / 2, td.sp1);
  __syncthreads();
  if constexpr (TRAIN) {
    dump_tile<W, MODE>(td.act, td.h(0), td.ldb, td.q0, td.nvalid);  // h1
  }

  // ---- hidden layers 2..4 (forward), keeping SiLU' of layers 2 and 3 ----
  float sp[2][MT][CB][16];
  float dpart[G::GPW][CB];
#pragma unroll
  for (int k = 0; k < G::GPW; ++k)
#pragma unroll
    for (int nt = 0; nt < CB; ++nt) dpart[k][nt] = 0.f;
  fwd_hidden<W, MODE, CB, 0, TRAIN, GRAD>(net, tc, sp, dpart, td, ap);
  fwd_hidden<W, MODE, CB, 1, TRAIN, GRAD>(net, tc, sp, dpart, td, ap);
  fwd_hidden<W, MODE, CB, 2, TRAIN, GRAD>(net, tc, sp, dpart, td, ap);

  // ---- reverse sweep: W4^T, W3^T (into LDS), W2^T (into the input-layer gradient) ----
  GradSums<CB> epart[G::GPW];
#pragma unroll
  for (int k = 0; k < G::GPW; ++k)
#pragma unroll
    for (int nt = 0; nt < CB; ++nt)
#pragma unroll
      for (int t = 0; t < 2; ++t) epart[k].v[nt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  if constexpr (GRAD) {
    bwd_hidden<W, MODE, CB, 2, TRAIN>(net, tc, sp, td, ap);
    bwd_hidden<W, MODE, CB, 1, TRAIN>(net, tc, sp, td, ap);
    bwd_input<W, MODE, CB, PAIRS, TRAIN, SPH>(net, tc, epart, td, tc.act + G::ACT_BYTES / 2, ap, fetch_next);
    if constexpr (rev_arith<MODE>() == kF16) {
      // a lane whose output partial sum is finite but whose input-gradient partial
      // sums are not: the FP16 reverse sweep overflowed (the forward accumulates in
      // FP32; a non-finite input point makes every partial non-finite).  Noted in
      // LDS, reported to the host once per workgroup when the kernel ends
      // (report_overflow).
      uint32_t bad = 0;
#pragma unroll
      for (int k = 0; k < G::GPW; ++k)
#pragma unroll
        for (int nt = 0; nt < CB; ++nt) {
          float t = 0.f;
#pragma unroll
          for (int c = 0; c < 8; ++c) t += epart[k].v[nt][c >> 2][c & 3];
          bad |= (uint32_t)(!__builtin_isfinite(t)) & (uint32_t)__builtin_isfinite(dpart[k][nt]);
        }
      if (bad) *tc.ovf = 1u;
    }
  }

  // ---- reduce d and e over the rows: lane halves, then row groups (fixed order) ----
  // (training needs neither: the fused loss finished d inside the tile)
  if constexpr (!TRAIN) {
#pragma unroll
    for (int k = 0; k < G::GPW; ++k)
#pragma unroll
      for (int nt = 0; nt < CB; ++nt) {
        dpart[k][nt] += __shfl_xor(dpart[k][nt], 32);
#pragma unroll
        for (int c = 0; c < (GRAD ? 8 : 0); ++c)
          epart[k].v[nt][c >> 2][c & 3] += __shfl_xor(epart[k].v[nt][c >> 2][c & 3], 32);
      }
    // the reduction buffer may share the activation tile: every wave must have
    // finished reading it
    if constexpr (G::RED_IN_ACT) __syncthreads();
    const Lane<W, MODE, CB> ln(tc.act, View<W, MODE, CB>::fresh_tid(), tc.wave);
#pragma unroll
    for (int k = 0; k < G::GPW; ++k)
#pragma unroll
      for (int nt = 0; nt < CB; ++nt) {
        // lane half 0 stores d and the first four components, half 1 the other four
        float* r = red + (ln.wave * G::GPW + k) * G::RED_VALS * TQ + 32 * nt + ln.n0;
        if (ln.h == 0) r[0] = dpart[k][nt];
#pragma unroll
        for (int c = 0; c < (GRAD ? 4 : 0); ++c)
          r[(1 + 4 * ln.h + c) * TQ] = ln.h ? epart[k].v[nt][1][c] : epart[k].v[nt][0][c];
      }
    __syncthreads();

    // ---- per query: final sums, chain rule, stores, per-knot minimum ----
    // Wave 0 finishes d, wave 1 dd/dp' and J's base columns, the others the arm
    // columns (a single wave doing all of it kept the rest waiting for 72 LDS reads).
    // J's rows of the tile are staged in the idle activation tile and copied out as
    // contiguous dwords.
    {
      // n: recomputed here rather than kept from the prologue (the compiler would
      // otherwise hold q0 + tid through the whole tile, in a spill slot)
      int n = tid & 63;
      asm volatile("" : "+v"(n));
      auto total = [&](int c) {
        float sum = red[c * TQ + n % TQ];
#pragma unroll
        for (int w = 1; w < G::RG; ++w) sum += red[(w * G::RED_VALS + c) * TQ + n % TQ];
        return sum * (1.0f / rev_scale<MODE>());
      };
      float* jt = G::RED_IN_ACT ? red + G::RED_BYTES / 4 : reinterpret_cast<float*>(tc.act);  // [TQ][9]
      static_assert((G::RED_IN_ACT ? G::RED_BYTES : 0) + TQ * kInDim * 4 <= G::ACT_BYTES / (mma_input<W, MODE>(PAIRS, SPH) ? 2 : 1),
                    "J's staged rows stay clear of what the next prologue writes into the tile");
      const bool want_J = GRAD && job.J;
      const int64_t out0 = (PAIRS || GATHER) ? q0 : kk * job.Np + q0;
      if (ln.wave == 0) {
        const float dv = total(0) + tc.b5;
        const int64_t q = q0 + n;
        const bool valid = n < TQ && q < qlimit;
        // outputs are streamed with non-temporal stores: written once and never read
        // here, they would otherwise evict the packed weights from L2
        if (valid && job.d) __builtin_nontemporal_store(dv, job.d + out0 + n);
        if constexpr (!PAIRS) {
          if (job.minkey) {
            unsigned long long key = valid ? (((unsigned long long)ordered_bits(dv) << 32) | (uint32_t)q) : ~0ull;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
              unsigned long long o = __shfl_xor(key, off);
              key = o < key ? o : key;
            }
            if (n == 0 && key != ~0ull) atomicMax(job.minkey + kk, ~key);  // (stored inverted, see minkey_decode)
          }
        }
      } else if (ln.wave == 1) {
        if (want_J && n < TQ) {
          const float* x = xin + n * XF;
          const float cs = x[3], sn = x[4], e0 = total(1), e1 = total(2);
          // (which product is fused is spelled out, so that every instantiation rounds alike)
          jt[n * kInDim + 0] = -__builtin_fmaf(cs, e0, -(sn * e1));
          jt[n * kInDim + 1] = -__builtin_fmaf(cs, e1, sn * e0);
          jt[n * kInDim + 2] = __builtin_fmaf(e0, x[1], -(e1 * x[0]));
        }
      } else if (want_J && n < TQ) {
#pragma unroll
        for (int c = 0; c < 6; c += G::NW - 2) {
          const int a = c + ln.wave - 2;
          jt[n * kInDim + 3 + a] = total(3 + a);
        }
      }
      __syncthreads();
      if (want_J) {
        const int64_t left = (qlimit - q0) * kInDim;
        float* Jo = job.J + out0 * kInDim;
        for (int t = tid; t < TQ * kInDim; t += G::THREADS)
          if (t < left) __builtin_nontemporal_store(jt[t], Jo + t);
      }
    }
  }  // !TRAIN
  // The next tile's prologue rewrites xin and crow, which nobody reads after the last
  // barrier above; the staged rows of J are read before its first barrier, and the
  // tile is written after it, but for mma_input's fragments, which the prologue writes
  // past the staged rows (checked above).
  if constexpr (TRAIN) __syncthreads();
}

// End of a kernel that ran tiles: if any tile of this workgroup flagged an FP16
// overflow, write the context's host-visible flag (all threads call it).
template <int W, int MODE, int CB>
__device__ __forceinline__ void report_overflow(const DevNet& net, const TileCtx<W, MODE, CB>& tc) {
  if constexpr (rev_arith<MODE>() == kF16) {
    __syncthreads();
    if (threadIdx.x == 0 && *tc.ovf && net.overflow)
      __hip_atomic_store(net.overflow, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// ----------------------------------------------------------------------------
// One-shot kernel: a persistent grid strides over all tiles of one job.
// ----------------------------------------------------------------------------
// WPE: waves per SIMD that the registers leave room for.
template <int W, int MODE, int CB, bool GRAD, bool PAIRS, bool TRAIN = false, bool GATHER = false, bool SPH = false,
          int WPE = Geo<W, MODE, CB>::WPE>
__global__ __launch_bounds__((Geo<W, MODE, CB>::THREADS), WPE) void fused_query(const DevNet net, const Job job,
                                                                                int64_t ntiles) {
  static_assert(Geo<W, MODE, CB>::LDS_BYTES + (TRAIN ? train_extra_lds<W, MODE>() : 0) + 16 <= 160 * 1024,
                "the workgroup's LDS exceeds the compute unit's 160 KiB");
  __shared__ __attribute__((aligned(16))) char lds[Geo<W, MODE, CB>::LDS_BYTES + (TRAIN ? train_extra_lds<W, MODE>() : 0)];
  __shared__ uint32_t ovf;
  TileCtx<W, MODE, CB> tc(lds, &ovf, net, threadIdx.x);
  float* bsum = TRAIN ? train_bsum<W, MODE>(lds) : nullptr;
  if constexpr (TRAIN) {  // ordered before the first tile's sums by its barriers (FP32: the same thread adds to them)
    float* rows = bsum ? bsum : job.bias_part + (int64_t)blockIdx.x * kTrainSumRows * W;
    for (int j = threadIdx.x; j < kTrainSumRows * W; j += Geo<W, MODE, CB>::THREADS) rows[j] = 0.f;
  }
  const int64_t nblk = PAIRS ? 0 : (job.Np + (Geo<W, MODE, CB>::TQ) - 1) / (Geo<W, MODE, CB>::TQ);
  int64_t kk = PAIRS ? 0 : blockIdx.x / nblk;  // dense: the knot of the current tile
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    if constexpr (PAIRS) {
      process_tile<W, MODE, CB, GRAD, true, TRAIN, false, SPH>(net, job, 0, tile * (Geo<W, MODE, CB>::TQ), tc);
    } else if constexpr (GATHER) {
      if (tile >= job.tile_off[job.K]) break;  // the grid is sized by an upper bound
      int64_t lo = 0, hi = job.K - 1;            // knot: the last i with tile_off[i] <= tile
      while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (job.tile_off[mid] <= tile) lo = mid; else hi = mid - 1;
      }
      process_tile<W, MODE, CB, GRAD, false, false, true, SPH>(net, job, lo,
                                                           job.row_off[lo] + (tile - job.tile_off[lo]) * (Geo<W, MODE, CB>::TQ), tc);
    } else {
      process_tile<W, MODE, CB, GRAD, false, false, false, SPH>(net, job, kk, (tile - kk * nblk) * (Geo<W, MODE, CB>::TQ), tc);
      // the next tile's knot: at most one knot further when a knot has at least as
      // many tiles as the grid has workgroups, with no 64-bit division then
      const int64_t next = tile + gridDim.x;
      if (next < (kk + 2) * nblk) kk += next >= (kk + 1) * nblk ? 1 : 0;
      else kk = next / nblk;
    }
  }
  if (bsum) {  // this workgroup's sums; summed over workgroups in order afterwards
    __syncthreads();
    for (int j = threadIdx.x; j < kTrainSumRows * W; j += Geo<W, MODE, CB>::THREADS)
      job.bias_part[(int64_t)j * gridDim.x + blockIdx.x] = bsum[j];
  }
  report_overflow<W, MODE, CB>(net, tc);
}

// ----------------------------------------------------------------------------
// Host-side launchers of fused_query (grid = min(tiles, workgroups that fit)); each source file
// instantiates the obstacle kind (SPH) it serves.
// ----------------------------------------------------------------------------
template <int W, int MODE, int CB, bool GRAD, bool PAIRS, bool SPH>
static hipError_t launch_t(const DevNet& net, const Job& job, int num_cu, hipStream_t s) {
  using G = Geo<W, MODE, CB>;
  const int64_t ntiles = query_tiles(job, PAIRS, G::TQ);
  if (ntiles <= 0) return hipSuccess;
  const dim3 grid((unsigned)fused_grid(ntiles, num_cu * G::WGS)), block(G::THREADS);
  if constexpr (CB == 2 && GRAD && PAIRS && W == 256 && (MODE == kFP32 || MODE == kBF16) && !SPH) {  // training: width 256, FP32 or BF16
    if (job.dumpH) {
      // the kernel writes its sums to bias_part, no J, and d only with the fused loss
      static_assert(train_wgs(MODE) == G::WGS, "the per-workgroup sums follow the grid");
      if (!job.bias_part || (int)grid.x > job.bias_parts || job.J || (job.d && !job.target)) return hipErrorInvalidValue;
      // FP32 batches of at most one tile per compute unit: with the whole register file
      // the tile's h4 copy spills no SiLU' values (batch 5,001: step 176 -> 154 us); past
      // that, two workgroups per compute unit are worth more than the spill (20,000:
      // 321 -> 312 us)
      if constexpr (MODE == kFP32) {
        if (ntiles <= num_cu) {
          hipLaunchKernelGGL((fused_query<W, MODE, CB, true, true, true, false, false, 1>), grid, block, 0, s, net, job,
                             ntiles);
          return hipGetLastError();
        }
      }
      hipLaunchKernelGGL((fused_query<W, MODE, CB, true, true, true>), grid, block, 0, s, net, job, ntiles);
      return hipGetLastError();
    }
  }
  if (job.dumpH || job.seed) return hipErrorInvalidValue;  // a seed is honoured by the training instantiation only
  if constexpr (!PAIRS) {
    if (job.tile_off) {
      hipLaunchKernelGGL((fused_query<W, MODE, CB, GRAD, false, false, true, SPH>), grid, block, 0, s, net, job, ntiles);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((fused_query<W, MODE, CB, GRAD, PAIRS, false, false, SPH>), grid, block, 0, s, net, job, ntiles);
  return hipGetLastError();
}

template <int W, int MODE, int CB, bool SPH>
static hipError_t launch_m(const DevNet& net, const Job& job, bool pairs, bool want_grad, int num_cu, hipStream_t s) {
  if (want_grad)
    return pairs ? launch_t<W, MODE, CB, true, true, SPH>(net, job, num_cu, s) : launch_t<W, MODE, CB, true, false, SPH>(net, job, num_cu, s);
  return pairs ? launch_t<W, MODE, CB, false, true, SPH>(net, job, num_cu, s) : launch_t<W, MODE, CB, false, false, SPH>(net, job, num_cu, s);
}

template <int W, int CB, bool SPH>
static hipError_t launch_w(const DevNet& net, const Job& job, bool pairs, bool want_grad, int num_cu, hipStream_t s) {
  switch (net.mode) {
    case kFP32: return launch_m<W, kFP32, CB, SPH>(net, job, pairs, want_grad, num_cu, s);
    case kBF16: return launch_m<W, kBF16, CB, SPH>(net, job, pairs, want_grad, num_cu, s);
    case kBF16X2F16: return launch_m<W, kBF16X2F16, CB, SPH>(net, job, pairs, want_grad, num_cu, s);
    default: return launch_m<W, kBF16X2, CB, SPH>(net, job, pairs, want_grad, num_cu, s);
  }
}

#ifdef GCDF_ONE_ROUND
}  // inline namespace one_round_tiles
#endif
}  // namespace gcdf
