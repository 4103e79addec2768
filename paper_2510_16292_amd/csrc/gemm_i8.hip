// int8 x int8 -> int32 products on the gfx950 matrix cores (v_mfma_i32_32x32x32_i8)
// with the per-row / per-column dequantization epilogue of the quantized
// projections Q(X) Q(W^d) and Q(C) Q(W^u) (Eq. 11-12).
//
// Operand layout of one 32x32x32 MFMA: lane l supplies row (l % 32) of A and
// column (l % 32) of B, 16 bytes each along the contraction.  Which 16 bytes a
// lane supplies only has to agree between A and B: integer sums are exact in
// any order, so each kernel assigns contraction bytes to lanes in whatever
// order its loads are cheapest.  Output: lane l holds column (l % 32) and rows
// 8*(v/4) + 4*(l/32) + (v%4) for accumulator registers v = 0..15.
#include "common.h"
#include "launch.h"
#include <type_traits>

namespace qsvd {

// Output segments (columns [n0, n0 + n) of the product go to ptr with row
// stride ld); fields are spelled out per segment so that a store only ever
// reads kernel arguments at constant offsets.
struct DevSegs {
  _Float16* p0; _Float16* p1; _Float16* p2;
  int64_t ld0, ld1, ld2;
  int32_t a0, a1, a2;      // first column of each segment
  int32_t e0, e1, e2;      // one past the last column
};

// Where column n of the product goes: its first element's address and the row
// stride (NULL if the column is not stored).  Selects rather than branches, so
// the three segment pointers stay in registers.
struct ColOut {
  _Float16* p;
  int64_t ld;
};

__device__ __forceinline__ ColOut col_out(const DevSegs& sg, int32_t n) {
  const bool in0 = n >= sg.a0 && n < sg.e0;
  const bool in1 = n >= sg.a1 && n < sg.e1;
  const bool in2 = n >= sg.a2 && n < sg.e2;
  _Float16* p = in0 ? sg.p0 + (n - sg.a0) : in1 ? sg.p1 + (n - sg.a1) : in2 ? sg.p2 + (n - sg.a2) : nullptr;
  if (!(in0 ? sg.p0 : in1 ? sg.p1 : in2 ? sg.p2 : nullptr)) p = nullptr;
  const int64_t ld = in0 ? sg.ld0 : in1 ? sg.ld1 : sg.ld2;
  return ColOut{p, ld};
}

// Dequantize one integer accumulator: (f32(acc) * row_scale) * col_scale, each
// product rounded to fp32 on its own.
__device__ __forceinline__ float dequant(int32_t acc, float rs, float cs) {
  return mul_rn(mul_rn((float)acc, rs), cs);
}
__device__ __forceinline__ float dequant(float acc, float rs, float cs) { return mul_rn(mul_rn(acc, rs), cs); }

// ---------------------------------------------------------------------------
// Pipelined kernel: BM x BN output tile per workgroup of 4 or 8 waves (each
// WM x WN), the contraction in stages of 128 bytes.  With F16 the operands are
// fp16 (a stage is 64 contraction elements, v_mfma_f32_32x32x16_f16, fp32
// accumulators; a 16-byte slot is 8 elements, so the slot layout, the loads
// and the fragment reads are the same) and K counts bytes per row.  Operands go from global
// memory straight into LDS (global_load_lds_dwordx4: lane i of a wave writes
// 16 bytes at base + 16 i), NS stages deep, so NS - 1 stages are in flight
// while one is multiplied; one barrier per stage.
//
// A stage is one 128-byte cache line of every row: a direct load covers 8
// rows x 128 bytes.  (Stages of 64 bytes fetch each line from L2 twice, half
// of it unused each time.)
//
// LDS layout of a stage: rows of 128 bytes; 16-byte slot chunk ^ (row / 2 % 8)
// of a row holds its contraction chunk `chunk`.  A fragment read (16
// consecutive rows, one chunk) then touches every bank once.
// ---------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) void glb_void_t;

constexpr int PBK = 128;        // contraction bytes per stage
constexpr int PKK = PBK / 32;   // products' steps per stage

// Wait until at most N direct loads of this wave are outstanding (and its LDS
// reads are done), then meet the other waves.  Written as one asm statement
// so that the compiler neither adds a full wait nor moves LDS accesses across.
template <int N>
__device__ __forceinline__ void vm_wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// The stage being consumed was issued `rem` stages before the newest one.
template <int LPW, int R>
__device__ __forceinline__ void vm_wait_stage(int rem) {
  if constexpr (R == 0) {
    vm_wait_barrier<0>();
  } else {
    if (rem >= R) vm_wait_barrier<R * LPW>();
    else vm_wait_stage<LPW, R - 1>(rem);
  }
}

__device__ __forceinline__ int pipe_slot(int row, int chunk) {
  return row * PBK + (chunk ^ ((row >> 1) & 7)) * 16;
}

// Sum over LP = 4, 8 or 16 neighbouring lanes, every lane receiving it: lane
// exchanges within quads, then between mirrored quads and mirrored halves of
// a row of 16 (whose lanes already agree).
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
template <int LP>
__device__ __forceinline__ float lanes_sum(float x) {
  x = dpp_add<0xB1>(x);                       // quad_perm 1 0 3 2
  x = dpp_add<0x4E>(x);                       // quad_perm 2 3 0 1
  if constexpr (LP >= 8) x = dpp_add<0x141>(x);   // row_half_mirror
  if constexpr (LP >= 16) x = dpp_add<0x140>(x);  // row_mirror
  return x;
}

template <int BM, int BN, int WM, int WN, int NS>
struct PipeCfg {
  static constexpr int kWaves = (BM / WM) * (BN / WN);
  static_assert(kWaves == 4 || kWaves == 8, "four or eight waves");
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kABlocks = BM / 8, kBBlocks = BN / 8;
  static_assert((kABlocks + kBBlocks) % kWaves == 0, "whole 1 KB loads per wave");
  static constexpr int kLPW = (kABlocks + kBBlocks) / kWaves;   // direct loads per wave per stage
  static constexpr int kStage = (kABlocks + kBBlocks) * 1024;
  static constexpr size_t kStages = (size_t)NS * kStage;
  static constexpr size_t kOut = (size_t)kWaves * WM * (WN + 8) * 2;   // fp16 output staging
  static constexpr size_t kLds = kStages > kOut ? kStages : kOut;
};

template <int BM, int BN, int WM, int WN, int NS, bool DBG, bool F16, int RS = 0>
__global__ void __launch_bounds__((PipeCfg<BM, BN, WM, WN, NS>::kThreads))
gemm_i8_pipe_kernel(const int8_t* __restrict__ A, const int8_t* __restrict__ B,
                    const float* __restrict__ rs, const float* __restrict__ cs,
                    int64_t M, int32_t N, int32_t K, int32_t n_tiles_n, int32_t gm, DevSegs sg,
                    int32_t* __restrict__ dbg, RopeEpi re) {
  using C = PipeCfg<BM, BN, WM, WN, NS>;
  using Acc = std::conditional_t<F16, f32x16, i32x16>;
  static_assert(!(DBG && F16), "accumulator dumps are for the integer products");
  constexpr int TI = WM / 32, TJ = WN / 32;
  extern __shared__ __attribute__((aligned(1024))) uint8_t pipe_smem[];
  __shared__ __attribute__((aligned(16))) float s_rs[BM];
  __shared__ __attribute__((aligned(16))) float s_cs[BN];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w / (BN / WN), wn = w % (BN / WN);
  const int l32 = lane & 31, hl = lane >> 5;
  int tm, tn;
  xcd_tile(blockIdx.x, gridDim.x, n_tiles_n, gm, &tm, &tn);
  const int64_t m0 = (int64_t)tm * BM;
  const int32_t n0 = tn * BN;
  const int nkf = K / PBK, nk = (K + PBK - 1) / PBK;   // whole stages, stages (the last may be half a one)

  // Each direct load of this wave covers one 8-row block of A or B; its
  // per-lane source offset from the tile's first row is fixed, so a stage
  // only advances the (scalar) tile base by 128 bytes.  In a half stage (K a
  // multiple of 64 only) the upper half's lanes re-read the lower half.
  const int8_t* a_tile = A + m0 * K;
  const int8_t* b_tile = B + (int64_t)n0 * K;
  uint32_t voff[C::kLPW];
  // (row / 2 % 8 of lane p's row in block blk is 4 (blk % 2) + p / 16)
  const int chunk0 = (lane & 7) ^ (lane >> 4);
  static_assert(C::kLPW % 2 == 0 && C::kABlocks % 2 == 0, "block parity of load j is j's");
#pragma unroll
  for (int j = 0; j < C::kLPW; ++j) {
    const int blk = w * C::kLPW + j;                         // wave-uniform
    const bool is_a = blk < C::kABlocks;
    const int row = 8 * (is_a ? blk : blk - C::kABlocks) + (lane >> 3);
    const int64_t last = is_a ? M - 1 - m0 : (int64_t)N - 1 - n0;   // clamp ragged tiles to the last row
    voff[j] = (uint32_t)(min((int64_t)row, last) * K + 16 * (chunk0 ^ (4 * (j & 1))));
  }
  auto issue = [&](int st) {
    uint8_t* base = pipe_smem + (st % NS) * C::kStage;
    const int64_t k0 = (int64_t)st * PBK;
#pragma unroll
    for (int j = 0; j < C::kLPW; ++j) {
      const int blk = w * C::kLPW + j;
      const uint32_t back = st < nkf ? 0 : 16 * ((chunk0 ^ (4 * (j & 1))) & 4);
      const int8_t* src = (blk < C::kABlocks ? a_tile : b_tile) + k0 + (voff[j] - back);
      __builtin_amdgcn_global_load_lds((glb_void_t*)src, (lds_void_t*)(base + blk * 1024), 16, 0, 0);
    }
  };

  // RS: the rows of this wave's part of the score epilogue (below), LPR lanes
  // per row: their sequences and positions, and, like the scales, the lengths
  // before the stage loads, so that the epilogue does not wait for them.  One
  // 64-bit division per lane; the steps' rows follow one another.
  constexpr int RH = RS > 0 ? RS : 128;
  constexpr int half = RH / 2, LPR = RH / 8, RPS = 64 / LPR;     // lanes per row, rows per step
  constexpr int RW = BM / C::kWaves, STEPS = RW / RPS;           // rows of the wave
  static_assert(RW % RPS == 0 && (RS == 0 || BN % RH == 0) && half % 4 == 0, "whole steps, whole heads");
  const int row0 = w * RW + lane / LPR;
  int row_b[RS > 0 ? STEPS : 1], row_t[RS > 0 ? STEPS : 1], row_l[RS > 0 ? STEPS : 1];
  if constexpr (RS > 0) {
    const int64_t bt0 = re.row0 + min(m0 + row0, M - 1);
    int b = (int)(bt0 / re.capacity), t = (int)(bt0 - (int64_t)b * re.capacity);
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      const bool in = m0 + row0 + s * RPS < M;
      if (s > 0 && in)
        for (t += RPS; t >= re.capacity; t -= re.capacity) ++b;
      row_b[s] = b;
      row_t[s] = t;
      row_l[s] = in ? re.seq_len[b] : 0;
    }
  }

  // Scales first, into a register: their wait then leaves the stage loads in
  // flight (fp16 operands: a NULL scale vector means no scale).
  static_assert(BM + BN <= C::kThreads, "at most one scale per thread");
  const float* sp = tid < BM ? rs : cs;
  const int64_t si = tid < BM ? min(m0 + tid, M - 1) : (int64_t)min(n0 + tid - BM, N - 1);
  const float sv = (!F16 || sp) ? sp[si] : 1.f;
#pragma unroll
  for (int st = 0; st < NS - 1; ++st)
    if (st < nk) issue(st);
  if (tid < BM + BN) (tid < BM ? s_rs[tid] : s_cs[tid - BM]) = sv;
  if constexpr (RS > 0) {
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
      if (row_t[s] >= min(row_l[s], re.capacity)) row_b[s] = -1;   // no score wanted
  }

  Acc acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j) acc[i][j] = Acc{};

  // Fragments of one stage, by 32-byte step kk: af[kk % 2][i], bf[kk % 2][j].
  // Each step is read while the products of the step before run.
  i32x4 af[2][TI], bf[2][TJ];
  auto read_step = [&](int kt, int kk) {
    const uint8_t* sa = pipe_smem + (kt % NS) * C::kStage;
    const uint8_t* sb = sa + C::kABlocks * 1024;
#pragma unroll
    for (int i = 0; i < TI; ++i)
      af[kk & 1][i] = *reinterpret_cast<const i32x4*>(sa + pipe_slot(wm * WM + 32 * i + l32, 2 * kk + hl));
#pragma unroll
    for (int j = 0; j < TJ; ++j)
      bf[kk & 1][j] = *reinterpret_cast<const i32x4*>(sb + pipe_slot(wn * WN + 32 * j + l32, 2 * kk + hl));
  };
  auto products = [&](int kk) {
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j)
        if constexpr (F16)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, bf[kk & 1][j]),
                                                             __builtin_bit_cast(f16x8, af[kk & 1][i]), acc[i][j], 0, 0, 0);
        else
          acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(bf[kk & 1][j], af[kk & 1][i], acc[i][j], 0, 0, 0);
  };

  // One MFMA goes out before each LDS read of the next step, so the reads
  // run under the products and every wait the compiler places before a
  // product only covers reads issued before it.
  auto interleave = [&]() {
    if constexpr (C::kWaves == 8 || TI * TJ < TI + TJ) return;   // (the reads go out before all of the products)
#pragma unroll
    for (int r = 0; r < TI + TJ; ++r) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
    }
    __builtin_amdgcn_sched_group_barrier(0x008, TI * TJ - (TI + TJ), 0);
  };

  // Waiting for stage s (its loads landed; every wave has finished reading
  // stage s - 1) frees slot (s - 1) % NS for stage s + NS - 1.
  vm_wait_stage<C::kLPW, NS - 2>(nk - 1);
  if (NS - 1 < nk) issue(NS - 1);
  read_step(0, 0);
  for (int kt = 0; kt < nkf; ++kt) {
#pragma unroll
    for (int kk = 0; kk < PKK; ++kk) {
      __builtin_amdgcn_sched_barrier(0);
      if (kk == PKK - 1) {
        // (on the last stage: a full wait and barrier, nothing left to issue)
        vm_wait_stage<C::kLPW, NS - 2>(nk - 2 - kt);
        if (kt + NS < nk) issue(kt + NS);
        __builtin_amdgcn_sched_barrier(0);
      }
      // after the last stage's last step: an unused read of a stage slot,
      // which keeps this loop free of branches around products
      read_step(kk == PKK - 1 ? kt + 1 : kt, (kk + 1) % PKK);
      if (C::kWaves == 8 || TI * TJ < TI + TJ) __builtin_amdgcn_sched_barrier(0);
      products(kk);
      interleave();
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  if (nkf < nk) {                                // the half stage
    products(0);
    read_step(nkf, 1);
    products(1);
  }

  // Epilogue.  The integer accumulators are dumped as they are (debug only);
  // the dequantized fp16 tile of each wave is staged in LDS (the stages are
  // free once every wave is past its last product) and written back as
  // 16-byte runs of one row.  The products take B's fragment as their first
  // operand, so lane holds row wm*WM + 32i + l32 and the four consecutive
  // columns wn*WN + 32j + 8(v/4) + 4hl + 0..3: one 8-byte LDS write per
  // four outputs.
  if constexpr (DBG) {
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int64_t m = m0 + wm * WM + 32 * i + l32;
          const int32_t n = n0 + wn * WN + 32 * j + 8 * (v >> 2) + 4 * hl + (v & 3);
          if (m < M && n < N) dbg[m * N + n] = acc[i][j][v];
        }
    }
  }
  vm_wait_barrier<0>();
  constexpr int OST = WN + 8;                   // staged row stride in halves
  _Float16* ost = reinterpret_cast<_Float16*>(pipe_smem) + w * WM * OST;
#pragma unroll
  for (int i = 0; i < TI; ++i) {
    const int rl = 32 * i + l32;                 // this lane's row
    const float rsm = s_rs[wm * WM + rl];
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int vq = 0; vq < 4; ++vq) {
        const int cl = 32 * j + 8 * vq + 4 * hl;  // its 4 consecutive columns
        const f32x4 c4 = *reinterpret_cast<const f32x4*>(&s_cs[wn * WN + cl]);
        f16x4 o4;
#pragma unroll
        for (int e = 0; e < 4; ++e) o4[e] = to_f16(dequant(acc[i][j][4 * vq + e], rsm, c4[e]));
        *reinterpret_cast<f16x4*>(ost + rl * OST + cl) = o4;
        // one accumulator block at a time: keeps the live registers few
        __builtin_amdgcn_sched_barrier(0);
      }
  }
  if constexpr (RS > 0) {
    // Rotary scores of the tile's rows, RS = head_dim.  A wave takes rows of
    // the tile, LPR lanes per row with four pairs each: a row's (cos, sin) are
    // then one contiguous load per lane group (a lane per row read a line of
    // its own for every 16 bytes: a 65792 x 4096 x 1536 rebuild took 929 us,
    // against 831), kept for every head of the tile.  The
    // staged element (row, col) sits in the LDS rows of wave (row / WM, col / WN).
    __syncthreads();
    const int li = lane % LPR, j4 = 4 * li;
    f32x4 tb[STEPS][2];
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      const f32x4* src = reinterpret_cast<const f32x4*>(re.rope + (int64_t)(row_b[s] < 0 ? 0 : row_t[s]) * half + j4);
      tb[s][0] = src[0];
      tb[s][1] = src[1];
    }
    auto staged = [&](int row, int col) {
      const int wv = (row / WM) * (BN / WN) + col / WN;
      return *reinterpret_cast<const f16x4*>(reinterpret_cast<const _Float16*>(pipe_smem) +
                                             (size_t)wv * WM * OST + (row % WM) * OST + col % WN);
    };
    for (int col0 = 0; col0 < BN && n0 + col0 < N; col0 += RS) {
      const int gkv = (n0 + col0) / RS;
      for (int g = 0; g < re.G; ++g) {
        const int h = gkv * re.G + g;
        int qb_of = -2;                                          // sequence whose query is in qa, qb
        f32x4 qa = f32x4{}, qb = f32x4{};
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
          if (__any(row_b[s] != qb_of && row_b[s] >= 0)) {
            qb_of = row_b[s] >= 0 ? row_b[s] : qb_of;
            const float* qh = re.qrot + ((int64_t)max(qb_of, 0) * re.Hq + h) * RS;
            qa = *reinterpret_cast<const f32x4*>(qh + j4);
            qb = *reinterpret_cast<const f32x4*>(qh + half + j4);
          }
          // rot(k) . q over the lane's pairs (j, j + half):
          //   cos * (k_j q_j + k'_j q'_j) + sin * (k_j q'_j - k'_j q_j)
          const int row = row0 + s * RPS;
          const f16x4 ka = staged(row, col0 + j4), kb = staged(row, col0 + half + j4);
          float acc = 0.f;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float a = (float)ka[i], bb = (float)kb[i];
            const float uu = fmaf(bb, qb[i], a * qa[i]), vv = fmaf(-bb, qa[i], a * qb[i]);
            acc = fmaf(tb[s][i >> 1][2 * (i & 1)], uu, acc);
            acc = fmaf(tb[s][i >> 1][2 * (i & 1) + 1], vv, acc);
          }
          acc = lanes_sum<LPR>(acc);
          if (li == 0 && row_b[s] >= 0) re.pre[(re.row0 + m0 + row) * 32 + h] = acc;
        }
      }
      if (gkv == 0)
#pragma unroll
        for (int s = 0; s < STEPS; ++s)
          for (int h = re.Hq + li; h < 32; h += LPR)
            if (row_b[s] >= 0) re.pre[(re.row0 + m0 + row0 + s * RPS) * 32 + h] = 0.f;
    }
    return;
  }
  // Output rows leave non-temporally: the tile is written once and read by
  // a later kernel, so it need not displace the operands in L2.
  constexpr int CPR = WN / 8;                   // 16-byte chunks per staged row
  for (int e = lane; e < WM * CPR; e += 64) {
    const int row = e / CPR, c8 = e % CPR;
    const int64_t m = m0 + wm * WM + row;
    const int32_t n = n0 + wn * WN + 8 * c8;
    if (m >= M || n >= N) continue;
    const ColOut co = col_out(sg, n);
    if (co.p) __builtin_nontemporal_store(*reinterpret_cast<const f16x8*>(ost + row * OST + 8 * c8), reinterpret_cast<f16x8*>(co.p + m * co.ld));
  }
}

// Segments are consecutive and ascending in the column range; missing ones
// become empty ranges past the last column.
static DevSegs to_dev(const GemmArgs& g) {
  DevSegs d{};
  _Float16** ps[3] = {&d.p0, &d.p1, &d.p2};
  int64_t* lds[3] = {&d.ld0, &d.ld1, &d.ld2};
  int32_t* as[3] = {&d.a0, &d.a1, &d.a2};
  int32_t* es[3] = {&d.e0, &d.e1, &d.e2};
  for (int s = 0; s < 3; ++s) {
    if (s < g.n_seg) {
      *ps[s] = g.seg[s].ptr;
      *lds[s] = g.seg[s].ld;
      *as[s] = g.seg[s].n0;
      *es[s] = g.seg[s].n0 + g.seg[s].n;
    } else {
      *ps[s] = nullptr;
      *lds[s] = 0;
      *as[s] = *es[s] = s > 0 ? *es[s - 1] : 0;
    }
  }
  return d;
}

// Tiles one XCD runs at once: its 32 CUs, one workgroup each.
constexpr int kGemmTilesPerXcd = 32;

// Fewer 128 x 128 tiles than this: 64 x 64 instead (whole W8A8 projections of
// d = 4096, r = 1536, N = 12288, whose down-projection has 12 tiles per 128
// tokens: 33 tokens 45.8 -> 34.2 us, 260 tokens 58.2 -> 49.9, 900 tokens 74.4
// -> 67.3).
constexpr int64_t kSmallTiles = 128;

template <int BM, int BN, int WM, int WN, int NS, bool DBG, bool F16 = false, int RS = 0>
static hipError_t launch_pipe(const GemmArgs& g, const DevSegs& sg, hipStream_t s, const RopeEpi& re = RopeEpi{}) {
  using C = PipeCfg<BM, BN, WM, WN, NS>;
  auto kern = gemm_i8_pipe_kernel<BM, BN, WM, WN, NS, DBG, F16, RS>;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)C::kLds);
  if (e != hipSuccess) return e;
  const int tn = (g.N + BN - 1) / BN;
  const int64_t tm = (g.M + BM - 1) / BM;
  const int32_t kbytes = F16 ? 2 * g.K : g.K;
  KernelScope ks(RS ? "rope_rebuild_scores" : F16 ? "gemm_f16_pipe" : "gemm_i8_pipe", s);
  QSVD_LAUNCH(ks, kern, dim3((unsigned)(tm * tn)), dim3(C::kThreads), C::kLds, s, g.a, g.b, g.row_scale, g.col_scale,
                     g.M, g.N, kbytes, tn, xcd_group_rows(tm, tn, kGemmTilesPerXcd), sg, g.dbg, re);
  return hipGetLastError();
}

hipError_t launch_gemm_i8(const GemmArgs& g, hipStream_t s) {
  if (g.M == 0 || g.N == 0) return hipSuccess;
  if (g.K % 64) return hipErrorInvalidValue;
  // outputs are written in 16-byte runs of 8 columns
  for (int i = 0; i < g.n_seg; ++i)
    if (g.seg[i].n0 % 8 || g.seg[i].n % 8 || g.seg[i].ld % 8 || ((uintptr_t)g.seg[i].ptr & 15))
      return hipErrorInvalidValue;
  const DevSegs sg = to_dev(g);
  // 256 x 256 tiles once they fill the chip, 64 x 64 where even 128 x 128 ones
  // leave most of it idle, 128 x 128 otherwise (and for the accumulator dumps)
  const int64_t big_tiles = ((g.M + 255) / 256) * ((g.N + 255) / 256);
  const int64_t tiles = ((g.M + 127) / 128) * ((g.N + 127) / 128);
  hipError_t e = g.dbg ? launch_pipe<128, 128, 64, 64, 4, true>(g, sg, s)
                 : big_tiles >= 256 ? launch_pipe<256, 256, 128, 64, 2, false>(g, sg, s)
                 : tiles < kSmallTiles ? launch_pipe<64, 64, 32, 32, 4, false>(g, sg, s)
                                       : launch_pipe<128, 128, 64, 64, 4, false>(g, sg, s);
  if (e != hipSuccess || !g.cq) return e;
  return launch_quantize_rows(g.seg[0].ptr, g.M, g.N, g.seg[0].ld, g.abits, 1.f, g.cq, g.sc, s, "latent_quant");
}

hipError_t launch_gemm_f16(const GemmArgs& g, hipStream_t s) {
  if (g.M == 0 || g.N == 0) return hipSuccess;
  if (g.K % 32 || g.dbg || g.cq) return hipErrorInvalidValue;
  for (int i = 0; i < g.n_seg; ++i)
    if (g.seg[i].n0 % 8 || g.seg[i].n % 8 || g.seg[i].ld % 8 || ((uintptr_t)g.seg[i].ptr & 15))
      return hipErrorInvalidValue;
  const DevSegs sg = to_dev(g);
  const int64_t big_tiles = ((g.M + 255) / 256) * ((g.N + 255) / 256);
  return big_tiles >= 256 ? launch_pipe<256, 256, 128, 64, 2, false, true>(g, sg, s)
                          : launch_pipe<128, 128, 64, 64, 4, false, true>(g, sg, s);
}

template <int DH>
static hipError_t launch_rope_scores(const GemmArgs& g, const DevSegs& sg, hipStream_t s, const RopeEpi& re, bool f16,
                                     bool big) {
  if (f16)
    return big ? launch_pipe<256, 256, 128, 64, 2, false, true, DH>(g, sg, s, re)
               : launch_pipe<128, 128, 64, 64, 4, false, true, DH>(g, sg, s, re);
  return big ? launch_pipe<256, 256, 128, 64, 2, false, false, DH>(g, sg, s, re)
             : launch_pipe<128, 128, 64, 64, 4, false, false, DH>(g, sg, s, re);
}

hipError_t launch_gemm_rope_scores(const GemmArgs& g, const RopeEpi& re, bool f16, hipStream_t s) {
  if (g.M == 0 || g.N == 0) return hipSuccess;
  if ((f16 ? g.K % 32 : g.K % 64) || g.dbg || g.cq) return hipErrorInvalidValue;
  if (re.dh < 32 || 128 % re.dh || g.N % re.dh || re.Hq > 32 || re.G < 1) return hipErrorInvalidValue;
  const DevSegs sg{};
  const int64_t big_tiles = ((g.M + 255) / 256) * ((g.N + 255) / 256);
  const bool big = big_tiles >= 256;
  return re.dh == 32   ? launch_rope_scores<32>(g, sg, s, re, f16, big)
         : re.dh == 64 ? launch_rope_scores<64>(g, sg, s, re, f16, big)
                       : launch_rope_scores<128>(g, sg, s, re, f16, big);
}

}  // namespace qsvd
