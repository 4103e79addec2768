// Prefill-size products (M > 32) with 4-bit operands and per-group weight
// scales: Q(X) Q(W^d) and Q(C) Q(W^u) for W4A8 / W4A4 / W8A4 layers (Eq. 11-12,
// Section 4's per-group int4 weights).
//
// Same pipeline as the int8 kernel (operands global -> LDS with
// global_load_lds_dwordx4, NS stages of 128 contraction elements, one barrier
// per stage) on 128 x 128 tiles of four 64 x 64 waves, two workgroups per CU.
// A stage row holds 128 codes: 128 bytes (int8) or 64 bytes (int4, element 2i
// in the low nibble of byte i).  A lane takes 32 codes of a row at once (one
// 16-byte read of an int4 row, two of an int8 row), the A and the B lanes the
// same ones; int4 codes are widened in registers to int8 bytes holding
// 16 * code before v_mfma_i32_32x32x32_i8, so every product is exact and the
// int32 sums are exact multiples of 16 or 256.
//
// What bounds it: the vector operations of a group of 128 per 32 x 32 tile,
// 48 for the fold below and 24 for the widening, take 288 cycles where its
// products take 128.  So the fold is kept to its three operations (the
// products of a group start from a literal zero, the accumulators stay in
// vector registers) and runs tile by tile between the next group's first
// products.  W4A4, 5632 x 15360 x 2048: 382 -> 288 us.
//
// Per-group scales (groups of G contraction elements, G a multiple of 64):
// after each group the int32 tile is folded into an fp32 tile as
// S = S + f32(acc_g) * s[g][n] (each product and sum rounded to fp32, groups
// in order) and the int32 tile restarts from zero; the output is S * s_row.
// Per-channel scales: (f32(acc) * s_row) * s_col.  Both are the definition's
// rounding sequence.
#include "common.h"
#include "launch.h"

namespace qsvd {

typedef __attribute__((address_space(3))) void q4_lds_void_t;
typedef __attribute__((address_space(1))) void q4_glb_void_t;

constexpr int QBK = 128;

template <int N>
__device__ __forceinline__ void q4_wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

template <int LPW, int R>
__device__ __forceinline__ void q4_wait_stage(int rem) {
  if constexpr (R == 0) {
    q4_wait_barrier<0>();
  } else {
    if (rem >= R) q4_wait_barrier<R * LPW>();
    else q4_wait_stage<LPW, R - 1>(rem);
  }
}

// LDS position of 16-byte chunk `chunk` of a row in an operand tile whose rows
// are RB bytes (128: eight chunks, 64: four).  The XOR keeps the rows of one
// fragment read (16 consecutive rows, same chunk) on distinct banks.
template <int RB>
__device__ __forceinline__ int q4_swz(int row, int chunk) {
  return RB == 128 ? chunk ^ ((row >> 1) & 7) : chunk ^ ((row >> 2) & 3);
}

// 16 int4 codes (8 bytes, element 2i in the low nibble of byte i) -> 16 int8
// holding 16 * code, in the element order 0,2,4,6, 1,3,5,7, 8,10,12,14,
// 9,11,13,15: (w << 4) & 0xF0F0F0F0 moves every even element into the high
// half of its byte and w & 0xF0F0F0F0 keeps every odd one there, so each
// code's sign bit lands on bit 7 (three operations per eight codes).
__device__ __forceinline__ i32x4 q4_widen(uint2 p) {
  return i32x4{(int32_t)((p.x << 4) & 0xF0F0F0F0u), (int32_t)(p.x & 0xF0F0F0F0u),
               (int32_t)((p.y << 4) & 0xF0F0F0F0u), (int32_t)(p.y & 0xF0F0F0F0u)};
}

// 16 int8 codes in element order -> the element order of q4_widen (one byte
// permute per four codes), for an int8 operand multiplied with an int4 one.
__device__ __forceinline__ i32x4 q4_interleave(i32x4 v) {
  return i32x4{(int32_t)__builtin_amdgcn_perm((uint32_t)v[1], (uint32_t)v[0], 0x06040200u),
               (int32_t)__builtin_amdgcn_perm((uint32_t)v[1], (uint32_t)v[0], 0x07050301u),
               (int32_t)__builtin_amdgcn_perm((uint32_t)v[3], (uint32_t)v[2], 0x06040200u),
               (int32_t)__builtin_amdgcn_perm((uint32_t)v[3], (uint32_t)v[2], 0x07050301u)};
}

// The 32 codes of lane (row, hl) in half h of a stage (elements 64 h + 32 hl
// .. +31): as read from LDS, and as the fragments of its two 16-code steps, in
// natural order when both operands are int8, else in q4_widen's order (the
// same order in both operands, so the sum runs over the same products).
template <int BITS>
struct Q4Raw {
  i32x4 r[BITS / 4];
};
template <int BITS>
__device__ __forceinline__ Q4Raw<BITS> q4_read(const uint8_t* base, int row, int h, int hl) {
  constexpr int RB = QBK * BITS / 8;
  Q4Raw<BITS> o;
#pragma unroll
  for (int i = 0; i < BITS / 4; ++i)
    o.r[i] = *reinterpret_cast<const i32x4*>(base + row * RB + 16 * q4_swz<RB>(row, (BITS / 4) * (2 * h + hl) + i));
  return o;
}
template <int BITS, int OTHER>
__device__ __forceinline__ i32x4 q4_step(const Q4Raw<BITS>& w, int kk) {
  if constexpr (BITS == 8) {
    if constexpr (OTHER == 8) return w.r[kk];
    else return q4_interleave(w.r[kk]);
  } else {
    return q4_widen(make_uint2((uint32_t)w.r[0][2 * kk], (uint32_t)w.r[0][2 * kk + 1]));
  }
}

struct Q4Segs {
  _Float16* p0; _Float16* p1; _Float16* p2;
  int64_t ld0, ld1, ld2;
  int32_t a0, a1, a2, e0, e1, e2;
};

__device__ __forceinline__ _Float16* q4_col(const Q4Segs& sg, int32_t n, int64_t* ld) {
  const bool in0 = n >= sg.a0 && n < sg.e0, in1 = n >= sg.a1 && n < sg.e1, in2 = n >= sg.a2 && n < sg.e2;
  _Float16* base = in0 ? sg.p0 : in1 ? sg.p1 : in2 ? sg.p2 : nullptr;
  *ld = in0 ? sg.ld0 : in1 ? sg.ld1 : sg.ld2;
  return base ? base + (n - (in0 ? sg.a0 : in1 ? sg.a1 : sg.a2)) : nullptr;
}

// Scale groups: none (one scale per channel), 128 elements (a stage each), or
// any other multiple of 64.
enum { Q4_CHANNEL = 0, Q4_G128 = 1, Q4_GROUP = 2 };

template <int ABITS, int BBITS, int GM, int QT>
struct Q4Cfg {
  static constexpr int QBM = QT, QBN = QT, QWM = QT / 2, QWN = QT / 2;   // tile, and its four waves'
  static constexpr int RBA = QBK * ABITS / 8, RBB = QBK * BBITS / 8;   // stage row bytes
  static constexpr int SA = QBM * RBA, SB = QBN * RBB;
  static constexpr int kScaleRows = GM;                                // scale rows per stage: 0, 1 or 2
  static constexpr int kStage = SA + SB + kScaleRows * 1024;           // each of the four waves has 64 columns' scales
  static constexpr int LPW = (SA + SB) / 4096;                         // 16-byte direct loads per wave per stage
  static constexpr int NS = SA + SB <= 16384 ? 4 : SA + SB <= 24576 ? 3 : 2;
  static constexpr int kOut = 4 * QWM * (QWN + 8) * 2;
  static constexpr size_t kLds = NS * kStage > kOut ? NS * kStage : kOut;
  static_assert(2 * (kLds + 1024) <= 160 * 1024, "two workgroups per CU");
  static_assert((SA + SB) % 4096 == 0 && SA % 1024 == 0, "whole 1 KB loads per wave");
};

template <int ABITS, int BBITS, int GM, int QT>
__global__ void __launch_bounds__(256, 2)
gemm_q4_pipe_kernel(const uint8_t* __restrict__ A, const uint8_t* __restrict__ B,
                    const float* __restrict__ rs, const float* __restrict__ cs, int32_t sstride,
                    int64_t M, int32_t N, int32_t K, int32_t group, int32_t n_tiles_n, int32_t gm, Q4Segs sg) {
  using C = Q4Cfg<ABITS, BBITS, GM, QT>;
  constexpr int QBM = C::QBM, QBN = C::QBN, QWM = C::QWM, QWN = C::QWN;
  constexpr bool GROUPED = GM != Q4_CHANNEL;
  constexpr int RBA = C::RBA, RBB = C::RBB, SA = C::SA, LPW = C::LPW, NS = C::NS;
  constexpr int LPS = LPW + C::kScaleRows;                            // direct loads per wave per stage
  constexpr int TI = QWM / 32, TJ = QWN / 32;
  extern __shared__ __attribute__((aligned(1024))) uint8_t q4_smem[];
  __shared__ __attribute__((aligned(16))) float s_rs[QBM];
  // int4 operands enter the products as 16 * code: the int32 sums are exact
  // multiples of 16 (or 256) and are shifted back exactly before use
  constexpr int SH = (ABITS == 4 ? 4 : 0) + (BBITS == 4 ? 4 : 0);
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w >> 1, wn = w & 1;
  const int l32 = lane & 31, hl = lane >> 5;
  int tm, tn;
  xcd_tile(blockIdx.x, gridDim.x, n_tiles_n, gm, &tm, &tn);
  const int64_t m0 = (int64_t)tm * QBM;
  const int32_t n0 = tn * QBN;
  const int nkf = K / QBK, nk = (K + QBK - 1) / QBK;                  // whole stages, stages (the last may be half a one)
  const int64_t KA = (int64_t)K * ABITS / 8, KB = (int64_t)K * BBITS / 8;   // row bytes in memory

  // Per-lane source offsets of this wave's direct loads from the tile's first
  // row (fixed over the contraction; a stage advances the base by a row's
  // stage bytes): byte o of a stage holds A tile rows first, then B tile
  // rows; lane p of load j of wave w covers bytes 1024*(w*LPW + j) + 16p.
  // In a half stage (K a multiple of 64 only) the lanes of a row's upper half
  // re-read the lower one.
  const uint8_t* a_tile = A + m0 * KA;
  const uint8_t* b_tile = B + (int64_t)n0 * KB;
  uint32_t voff[LPW];
#pragma unroll
  for (int j = 0; j < LPW; ++j) {
    const int blk = w * LPW + j;                                     // wave-uniform
    const bool is_a = blk * 1024 < SA;
    const int o = blk * 1024 + 16 * lane - (is_a ? 0 : SA);
    if (is_a) {
      const int row = o / RBA, chunk = q4_swz<RBA>(row, (o % RBA) / 16);
      voff[j] = (uint32_t)(min((int64_t)row, M - 1 - m0) * KA + 16 * chunk);
    } else {
      const int row = o / RBB, chunk = q4_swz<RBB>(row, (o % RBB) / 16);
      voff[j] = (uint32_t)(min((int64_t)row, (int64_t)N - 1 - n0) * KB + 16 * chunk);
    }
  }
  const int gsteps = GROUPED ? group / 64 : 1;                       // half stages per group
  const int ncl = min(n0 + wn * QWN + lane, N - 1);                  // the column whose scales this lane loads
  auto issue = [&](int st) {
    uint8_t* base = q4_smem + (st % NS) * C::kStage;
#pragma unroll
    for (int j = 0; j < LPW; ++j) {
      const int blk = w * LPW + j;
      const bool is_a = blk * 1024 < SA;
      const int rb = is_a ? RBA : RBB;
      uint32_t off = voff[j];
      if (st >= nkf) {
        const int o = blk * 1024 + 16 * lane - (is_a ? 0 : SA);
        const int chunk = is_a ? q4_swz<RBA>(o / RBA, (o % RBA) / 16) : q4_swz<RBB>(o / RBB, (o % RBB) / 16);
        if (16 * chunk >= rb / 2) off -= rb / 2;
      }
      const uint8_t* src = (is_a ? a_tile : b_tile) + (int64_t)st * rb + off;
      __builtin_amdgcn_global_load_lds((q4_glb_void_t*)src, (q4_lds_void_t*)(base + blk * 1024), 16, 0, 0);
    }
#pragma unroll
    for (int h = 0; h < C::kScaleRows; ++h) {
      const int g = min(GM == Q4_G128 ? st : (2 * st + h) / gsteps, K / group - 1);
      __builtin_amdgcn_global_load_lds((q4_glb_void_t*)(cs + (int64_t)g * sstride + ncl),
                                       (q4_lds_void_t*)(base + SA + C::SB + (4 * h + w) * 256), 4, 0, 0);
    }
  };

  // row scales and per-channel column scales first, into registers (their
  // waits leave the stage loads in flight)
  const float rsv = tid < QBM ? rs[min(m0 + tid, M - 1)] : 0.f;
  float csn[TJ];
#pragma unroll
  for (int j = 0; j < TJ; ++j) csn[j] = GROUPED ? 0.f : cs[min(n0 + wn * QWN + 32 * j + l32, N - 1)];
#pragma unroll
  for (int st = 0; st < NS - 1; ++st)
    if (st < nk) issue(st);
  if (tid < QBM) s_rs[tid] = rsv;

  i32x16 acc[TI][TJ];
  f32x16 S[GROUPED ? TI : 1][GROUPED ? TJ : 1];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j) acc[i][j] = i32x16{};
  if constexpr (GROUPED) {
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j) S[i][j] = f32x16{};
  }

  Q4Raw<ABITS> ra[TI];
  Q4Raw<BBITS> rb[TJ];
  auto read_half = [&](int kt, int h) {
    const uint8_t* sa = q4_smem + (kt % NS) * C::kStage;
#pragma unroll
    for (int i = 0; i < TI; ++i) ra[i] = q4_read<ABITS>(sa, wm * QWM + 32 * i + l32, h, hl);
#pragma unroll
    for (int j = 0; j < TJ; ++j) rb[j] = q4_read<BBITS>(sa + SA, wn * QWN + 32 * j + l32, h, hl);
  };
  // the scales of half h's group for this lane's columns, times 2^-SH:
  // (float)acc * (s_g 2^-SH) is the same real number as (float)(acc >> SH) * s_g
  // (acc is an exact multiple of 2^SH and acc >> SH, at most 4.2e6 for the
  // longest groups, 4096, has 24 bits or fewer; scaling s_g by a power of two
  // is exact), so it rounds the same; the shift is saved on every element
  float gss[TJ];
  auto read_scales = [&](int kt, int h) {
    const float* src = reinterpret_cast<const float*>(q4_smem + (kt % NS) * C::kStage + SA + C::SB + (4 * h + w) * 256);
#pragma unroll
    for (int j = 0; j < TJ; ++j) gss[j] = mul_rn(src[32 * j + l32], 1.f / (float)(1 << SH));
  };
  auto fold = [&](int i, int j) {
#pragma unroll
    for (int v = 0; v < 16; ++v) S[i][j][v] = add_rn(S[i][j][v], mul_rn((float)acc[i][j][v], gss[j]));
  };
  i32x4 af[2][TI], bf[2][TJ];
  auto widen = [&](int kk) {
#pragma unroll
    for (int i = 0; i < TI; ++i) af[kk][i] = q4_step<ABITS, BBITS>(ra[i], kk);
#pragma unroll
    for (int j = 0; j < TJ; ++j) bf[kk][j] = q4_step<BBITS, ABITS>(rb[j], kk);
  };
  auto products = [&](int kk) {
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[kk][i], bf[kk][j], acc[i][j], 0, 0, 0);
  };
  // First products of a group: each tile's sums of the group before are folded
  // (zeros before the first group), then its accumulators start anew.
  auto restart = [&]() {
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        fold(i, j);
        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[0][i], bf[0][j], i32x16{}, 0, 0, 0);
      }
  };

  // Waiting for stage s (its loads landed; every wave has finished reading
  // stage s - 1) frees slot (s - 1) % NS for stage s + NS - 1.  The next half
  // is read while this one's products run, both steps of it where kEarly: the
  // registers hold that but for two int8 operands, and beside the fold at any
  // half (after the last half: an unused read of a stage slot).
  constexpr bool kEarly = GM != Q4_GROUP && !(ABITS == 8 && BBITS == 8);
  q4_wait_stage<LPS, NS - 2>(nk - 1);
  if (NS - 1 < nk) issue(NS - 1);
  read_half(0, 0);
  if constexpr (GROUPED) {
#pragma unroll
    for (int j = 0; j < TJ; ++j) gss[j] = 0.f;
  }
  // next(): whatever comes before the next half's reads, and those
  auto half = [&](int kt, int h, bool start, auto&& next) {
    widen(0);
    if constexpr (kEarly) {
      widen(1);
      next();
    }
    if (GROUPED && start) restart();
    else products(0);
    if (GROUPED && (GM == Q4_GROUP || h == 0)) read_scales(kt, GM == Q4_GROUP ? h : 0);
    if constexpr (!kEarly) {
      widen(1);
      products(1);
      next();
    } else {
      products(1);
    }
  };
  for (int kt = 0; kt < nkf; ++kt) {
    half(kt, 0, GM == Q4_G128 || (GM == Q4_GROUP && (2 * kt) % gsteps == 0), [&]() { read_half(kt, 1); });
    half(kt, 1, GM == Q4_GROUP && (2 * kt + 1) % gsteps == 0, [&]() {
      __builtin_amdgcn_sched_barrier(0);
      // (on the last stage: a full wait and barrier, nothing left to issue)
      q4_wait_stage<LPS, NS - 2>(nk - 2 - kt);
      if (kt + NS < nk) issue(kt + NS);
      __builtin_amdgcn_sched_barrier(0);
      read_half(kt + 1, 0);
    });
  }
  if (nkf < nk) half(nkf, 0, GM == Q4_G128 || (GM == Q4_GROUP && (2 * nkf) % gsteps == 0), []() {});
  if constexpr (GROUPED) {
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j) fold(i, j);
  }

  // Epilogue: the dequantized fp16 tile of each wave is staged in LDS and
  // written back as 16-byte runs of one row.  Lane holds column
  // wn*64 + 32j + l32 and rows wm*64 + 32i + 8(v/4) + 4hl + v%4.
  q4_wait_barrier<0>();
  constexpr int OST = QWN + 8;
  _Float16* ost = reinterpret_cast<_Float16*>(q4_smem) + w * QWM * OST;
#pragma unroll
  for (int j = 0; j < TJ; ++j)
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int vq = 0; vq < 4; ++vq) {
        const int rl = 32 * i + 8 * vq + 4 * hl;
        const f32x4 r4 = *reinterpret_cast<const f32x4*>(&s_rs[wm * QWM + rl]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int v = 4 * vq + e;
          const float y = GROUPED ? mul_rn(S[i][j][v], r4[e]) : mul_rn(mul_rn((float)(acc[i][j][v] >> SH), r4[e]), csn[j]);
          ost[(rl + e) * OST + 32 * j + l32] = to_f16(y);
        }
      }
  constexpr int CPR = QWN / 8;
  for (int e = lane; e < QWM * CPR; e += 64) {
    const int row = e / CPR, c8 = e % CPR;
    const int64_t m = m0 + wm * QWM + row;
    const int32_t n = n0 + wn * QWN + 8 * c8;
    if (m >= M || n >= N) continue;
    int64_t ld;
    _Float16* p = q4_col(sg, n, &ld);
    if (p) __builtin_nontemporal_store(*reinterpret_cast<const f16x8*>(ost + row * OST + 8 * c8), reinterpret_cast<f16x8*>(p + m * ld));
  }
}

// 128 x 128 tiles from so many on, else 64 x 64 (four waves of one 32 x 32
// product each): these widen twice the operand elements per output, but four
// times as many workgroups take part.  W4A8, tiles of 128, us with 128 and 64:
// 32 tiles 34.8, 17.4; 88 tiles 36.7, 23.5; 112 tiles 17.9, 11.1; 396 tiles
// 23.9, 29.1; 504 tiles 24.3, 36.3.
constexpr int64_t kQ4BigTiles = 256;

template <int ABITS, int BBITS, int GM, int QT>
static hipError_t launch_q4_tiles(const GemmArgs& g, const Q4Segs& sg, int32_t group, int32_t sstride, hipStream_t s) {
  using C = Q4Cfg<ABITS, BBITS, GM, QT>;
  auto kern = gemm_q4_pipe_kernel<ABITS, BBITS, GM, QT>;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::kLds);
  if (e != hipSuccess) return e;
  const int tn = (g.N + QT - 1) / QT;
  const int64_t tm = (g.M + QT - 1) / QT;
  KernelScope ks("gemm_q4_pipe", s);
  QSVD_LAUNCH(ks, kern, dim3((unsigned)(tm * tn)), dim3(256), C::kLds, s, (const uint8_t*)g.a, (const uint8_t*)g.b,
              g.row_scale, g.col_scale, sstride, g.M, g.N, g.K, group, tn, xcd_group_rows(tm, tn), sg);
  return hipGetLastError();
}

template <int ABITS, int BBITS, int GM>
static hipError_t launch_q4(const GemmArgs& g, const Q4Segs& sg, int32_t group, int32_t sstride, hipStream_t s) {
  const int64_t tiles = ((g.M + 127) / 128) * ((g.N + 127) / 128);
  return tiles >= kQ4BigTiles ? launch_q4_tiles<ABITS, BBITS, GM, 128>(g, sg, group, sstride, s)
                              : launch_q4_tiles<ABITS, BBITS, GM, 64>(g, sg, group, sstride, s);
}

template <int ABITS, int BBITS>
static hipError_t launch_q4_grouped(const GemmArgs& g, const Q4Segs& sg, int32_t group, int32_t sstride, hipStream_t s) {
  return group == QBK ? launch_q4<ABITS, BBITS, Q4_G128>(g, sg, group, sstride, s)
                      : launch_q4<ABITS, BBITS, Q4_GROUP>(g, sg, group, sstride, s);
}

hipError_t launch_gemm_q4(const GemmArgs& g, int32_t abits, int32_t wbits, int32_t group, int32_t sstride,
                          hipStream_t s) {
  if (g.M == 0 || g.N == 0) return hipSuccess;
  if (g.K % 64 || (group && (group % 64 || g.K % group))) return hipErrorInvalidValue;
  if ((abits != 8 && abits != 4) || (wbits != 8 && wbits != 4) || (wbits == 4 && !group)) return hipErrorInvalidValue;
  for (int i = 0; i < g.n_seg; ++i)
    if (g.seg[i].n0 % 8 || g.seg[i].n % 8 || g.seg[i].ld % 8 || ((uintptr_t)g.seg[i].ptr & 15))
      return hipErrorInvalidValue;
  Q4Segs sg{};
  _Float16** ps[3] = {&sg.p0, &sg.p1, &sg.p2};
  int64_t* lds[3] = {&sg.ld0, &sg.ld1, &sg.ld2};
  int32_t* as[3] = {&sg.a0, &sg.a1, &sg.a2};
  int32_t* es[3] = {&sg.e0, &sg.e1, &sg.e2};
  for (int i = 0; i < 3; ++i) {
    if (i < g.n_seg) {
      *ps[i] = g.seg[i].ptr; *lds[i] = g.seg[i].ld; *as[i] = g.seg[i].n0; *es[i] = g.seg[i].n0 + g.seg[i].n;
    } else {
      *ps[i] = nullptr; *lds[i] = 0; *as[i] = *es[i] = i > 0 ? *es[i - 1] : 0;
    }
  }
  hipError_t e;
  if (abits == 8 && wbits == 4) e = launch_q4_grouped<8, 4>(g, sg, group, sstride, s);
  else if (abits == 4 && wbits == 4) e = launch_q4_grouped<4, 4>(g, sg, group, sstride, s);
  else if (abits == 4 && group) e = launch_q4_grouped<4, 8>(g, sg, group, sstride, s);
  else if (abits == 4) e = launch_q4<4, 8, Q4_CHANNEL>(g, sg, 0, sstride, s);
  else e = launch_q4_grouped<8, 8>(g, sg, group, sstride, s);     // 8-bit codes, per-group scales
  if (e != hipSuccess || !g.cq) return e;
  return launch_quantize_rows(g.seg[0].ptr, g.M, g.N, g.seg[0].ld, g.abits, 1.f, g.cq, g.sc, s, "latent_quant");
}

}  // namespace qsvd
