// Causal self-attention of a prefill block over its own projections.
//
// In prefill every prompt token's keys and values are at hand: the
// up-projection Y' = Q(C) Q(W^u) (Eq. 11) produces Q, K and V of all tokens at
// once (K = C W^u_k, V = C W^u_v, Eq. 5), so the prompt attends over those
// rows directly: 4 Hq dh flop per (query, key) pair, against 4 Hq r for the
// latent form, which the decode path uses because there only one query row
// per sequence meets the whole cache.
//
// The unit of work is a wave: 32 consecutive queries of one query head.  The
// units of one (sequence, key/value head) are numbered query block by query
// block, the G = Hq / Hkv heads of a block next to each other, and a workgroup
// takes four or eight consecutive ones: they read the same key/value tiles, and with
// grouped heads they sit at (nearly) the same positions, so little is computed
// past the diagonal.  Key/value tiles of 64 tokens are staged in LDS for the
// workgroup, double-buffered (one barrier per tile): the values, and the keys
// of layers without rotary embedding, by direct loads that stay in flight
// while the tile before is used.  Per tile and wave, on the 32x32x16 fp16
// matrix cores:
//   S^T (64 keys x 32 queries) = K_tile Q^T          (contraction over dh)
//   online softmax per query in fp32 (a query is one lane column; its 64
//   scores sit in that lane and in lane l ^ 32)
//   O^T (dh x 32 queries) += V_tile^T P^T            (contraction over keys)
// The query rows stay in registers for the whole kernel.  Keys past a query's
// position, or past the sequence end, are masked.
//
// What bounds it: every key and value fragment is read from LDS once per
// wave and tile, 256 dh bytes, while the tile's products take 8 dh cycles of
// the wave's SIMD: with 32 queries per wave the LDS reads of a CU's eight
// waves (128 bytes per cycle) take as long as their products, with 16 queries
// twice as long.  The softmax's vector operations come next (32 exponentials
// and about ten operations per pair of scores and lane: 1.6 times the
// products' cycles), so the rest is kept few.  Measured against units of 16
// queries on the 16x16x32 products with one tile buffer: 4 x 640 tokens, 32
// heads: 37.8 -> 28.3 us; six rotary prompts of 1477 to 2531 tokens, 28 heads
// over 4: 541 -> 301 us (593 TFLOP/s).
//
// Rotary layers (ROPE): a query row is turned once, in registers, at its
// position within the sequence; a key row is turned while its tile moves from
// registers into LDS, at its own position (flash.h says how).
#include <math.h>

#include <algorithm>

#include "common.h"
#include "flash.h"
#include "flash_map.h"
#include "launch.h"

namespace qsvd {

constexpr int kFaQW = 32;       // queries per wave

template <int DH, int NW, int KSP>
struct FaCfg {
  static constexpr int UW = NW / KSP;                         // units (query blocks) per workgroup
  static constexpr int RUNS = DH / 8;                         // 16-byte runs per row
  static constexpr int OST = DH + 8;                          // output staging row stride (halves)
  static constexpr int kTile = kFaK * DH * 2;                 // bytes of a K (or V) tile
  static constexpr int kBuf = 2 * kTile;                      // K then V
  static constexpr int kOut = UW * kFaQW * OST * 2;
  static constexpr int kJoin = KSP > 1 ? UW * (64 * 4 * (DH / 2) + 64 * 8) : 0;   // a share's fp32 rows and (m, l)
  static constexpr size_t kLds = std::max({2 * KSP * kBuf, kOut, kJoin});
  static constexpr size_t kLdsRope = kLds + (size_t)(DH / 2) * sizeof(double);   // + revolutions per position of each pair
  static constexpr int kLPW = kTile / 1024 / UW;              // direct loads per wave and tile of one operand
  static_assert(kTile % (1024 * UW) == 0 && (KSP == 1 || KSP == 2), "whole 1 KB loads per wave");
};

// Rotary embedding: none, queries and keys turned in the kernel, or queries
// only (the keys were turned before).
enum { FA_PLAIN = 0, FA_ROPE = 1, FA_ROPE_Q = 2 };

// LDS position of 16-byte run c of row `row` in a tile (rows of DH / 8 runs,
// unpadded, since direct loads write lane after lane): the runs of a row are
// permuted so that 16 consecutive rows' reads of one run (K), or the 4 rows x
// 64 bytes of a transposing read (V), fall on distinct banks.
template <int DH>
__device__ __forceinline__ int fa_kslot(int row, int c) {
  return row * (DH / 8) + (c ^ (DH == 128 ? row & 15 : (row >> 1) & 7));
}
template <int DH>
__device__ __forceinline__ int fa_vslot(int row, int c) {
  return row * (DH / 8) + (c ^ (DH == 128 ? (row & 3) << 2 : ((row >> 1) & 1) << 2));
}

// Direct load, 16 bytes per lane: lane p's run at base + off goes to LDS bytes
// lds + 16 p (`lds` wave-uniform).  Written as asm, so that the compiler does
// not wait for every load in flight before each transposing LDS read (it
// cannot tell that they read the other buffer); it has no register outputs,
// and the s_waitcnt + s_barrier at the head of the tile loop is what completes
// it.  The s_nop separates the write of M0 from its use.
__device__ __forceinline__ void fa_direct_load(const _Float16* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base)
               : "memory", "m0");
}

// Cache mode: the queries are the last q_len positions of each sequence of a
// cache and the keys and values its rebuilt rows (row b * capacity + t,
// position t < seq_len[b], row stride ldkv).
struct FaCacheArgs {
  const int32_t* seq_len;
  int32_t capacity, q_len, ldkv;
};

template <int DH, int MODE, bool CACHE, int NW, int KSP>
__global__ void __launch_bounds__(NW * 64, 2)
prefill_flash_kernel(const _Float16* __restrict__ q, const _Float16* __restrict__ k, const _Float16* __restrict__ v,
                     const int32_t* __restrict__ cu, int32_t n_seq, int32_t Hq, int32_t Hkv, int32_t n_wg, int32_t parts,
                     float scale_log2, double log2_theta, FaCacheArgs ca, _Float16* __restrict__ out) {
  using C = FaCfg<DH, NW, KSP>;
  constexpr bool ROPE = MODE == FA_ROPE;
  constexpr int UW = C::UW;
  constexpr int KS = DH / 16;      // contraction steps of the score product
  constexpr int OB = DH / 32;      // 32-channel blocks of the output
  constexpr int RUNS = C::RUNS;
  extern __shared__ __attribute__((aligned(1024))) uint8_t fa_smem[];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hl = lane >> 5;

  const FaWork work = fa_work(blockIdx.x, n_seq * Hkv, n_wg, parts);
  if (!work.any) return;
  const int grp = work.group, wg = work.wg;
  const int b = grp / Hkv, g_kv = grp - b * Hkv, G = Hq / Hkv;
  // this sequence's rows: query i (i < nq) is row q_row0 + i at position
  // q_off + i, key t (t < nk) is row k_row0 + t at position t; query i sees
  // the keys at positions <= q_off + i
  int q_row0, nq, k_row0, nk, q_off;
  if (CACHE) {
    nk = min(ca.seq_len[b], ca.capacity);
    nq = ca.q_len;
    q_row0 = b * nq;
    k_row0 = b * ca.capacity;
    q_off = nk - nq;
  } else {
    q_row0 = k_row0 = cu[b];
    nq = nk = min(cu[b + 1] - q_row0, ca.q_len);     // (q_len: the launch's longest sequence)
    q_off = 0;
  }
  const int first = wg * UW / G * kFaQW;                        // first query of the workgroup
  if (first >= nq) return;
  // Waves w, w + UW (KSP 2) have the same unit and take every other key tile.
  const int wu = w % UW, share = w / UW;
  const int u = wg * UW + wu;                                   // this wave's unit
  const int qw0 = u / G * kFaQW;                                // its first query
  const int h = g_kv * G + u % G;                               // its query head
  const int last_q = min(nq, ((wg + 1) * UW - 1) / G * kFaQW + kFaQW);   // one past the workgroup's last query
  const int kend = min(nk, q_off + last_q);                     // keys the workgroup can see
  const int n_tiles = kend > 0 ? (kend + kFaK - 1) / kFaK : 0;
  const int ldq = Hq * DH, ldkv = CACHE ? ca.ldkv : Hkv * DH;
  const bool live = qw0 < nq;                                   // the unit has queries
  const int my_pos = q_off + qw0 + l32;                         // this lane's query position
  const int wave_last = live ? min(q_off + qw0 + kFaQW - 1, q_off + nq - 1) : -1;

  double* freq = reinterpret_cast<double*>(fa_smem + C::kLds);
  if (MODE != FA_PLAIN) {
    if (tid < DH / 2) freq[tid] = fa_freq(tid, DH, log2_theta);
    __syncthreads();
  }

  // query slots of the score product: step s, lane half hl -> channels 16 s + 8 hl .. +7
  f16x8 qf[KS];
  {
    const int qi = min(qw0 + l32, nq - 1);
    const _Float16* qrow = q + (int64_t)(q_row0 + qi) * ldq + h * DH + 8 * hl;
#pragma unroll
    for (int s = 0; s < KS; ++s) qf[s] = *reinterpret_cast<const f16x8*>(qrow + 16 * s);
    if (MODE != FA_PLAIN) {                         // slot s pairs with slot s + KS/2 (channels dh/2 further)
#pragma unroll
      for (int s = 0; s < KS / 2; ++s) fa_rope8(qf[s], qf[s + KS / 2], q_off + qi, freq + 16 * s + 8 * hl);
    }
  }

  // (their wait is here, not in the tile loop, where it would hold up the direct loads)
#pragma unroll
  for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(qf[s]));

  // Direct loads of a tile into LDS: load j of this wave fills 1 KB, lane p its
  // 16 bytes at position 64 * (kLPW wu + j) + p of its share's tile, from the row and
  // run that belong there.  Rows past the sequence end (only in its last tile)
  // re-read its last row; they are masked.
  uint32_t koff[ROPE ? 1 : C::kLPW], voff[C::kLPW];
  const int p0 = wu * C::kLPW * 64 + lane;
#pragma unroll
  for (int j = 0; j < C::kLPW; ++j) {
    const int row = (p0 + 64 * j) / RUNS, c = (p0 + 64 * j) % RUNS;
    if (!ROPE) koff[j] = 2u * (uint32_t)(row * ldkv + 8 * (fa_kslot<DH>(row, c) - row * RUNS));
    voff[j] = 2u * (uint32_t)(row * ldkv + 8 * (fa_vslot<DH>(row, c) - row * RUNS));
  }
  auto stage = [&](const _Float16* src, const uint32_t* off, int t, uint32_t base) {
    const _Float16* tile = src + (int64_t)(k_row0 + t * kFaK) * ldkv + g_kv * DH;
    const uint32_t lds = base + wu * C::kLPW * 1024;
    if ((t + 1) * kFaK <= nk) {
#pragma unroll
      for (int j = 0; j < C::kLPW; ++j) fa_direct_load(tile, off[j], lds + j * 1024);
    } else {
#pragma unroll
      for (int j = 0; j < C::kLPW; ++j) {
        const int over = max(t * kFaK + (p0 + 64 * j) / RUNS - (nk - 1), 0);
        fa_direct_load(tile, off[j] - 2u * (uint32_t)(over * ldkv), lds + j * 1024);
      }
    }
  };
  // Rotary keys: thread st of a share turns, in key rows st / PR + kRows i, the
  // 8 pairs of run pc (channels 8 pc .. +7 with their partners dh/2 further).
  constexpr int PR = DH / 16, kRows = 64 * UW / PR, kTurns = (kFaK + kRows - 1) / kRows;
  constexpr bool kAllTurn = !ROPE || kRows * kTurns == kFaK;
  const int krow = (wu * 64 + lane) / PR, kpc = lane % PR;
  i32x4 kr[kTurns][2];
  auto load_keys = [&](int t) {
#pragma unroll
    for (int i = 0; i < kTurns; ++i)
      if (kAllTurn || krow + kRows * i < kFaK) {
        const int key = min(t * kFaK + krow + kRows * i, nk - 1);
        const _Float16* src = k + (int64_t)(k_row0 + key) * ldkv + g_kv * DH + 8 * kpc;
        kr[i][0] = *reinterpret_cast<const i32x4*>(src);
        kr[i][1] = *reinterpret_cast<const i32x4*>(src + DH / 2);
      }
  };
  auto store_keys = [&](int t, uint8_t* base) {
    _Float16* ks = reinterpret_cast<_Float16*>(base);
#pragma unroll
    for (int i = 0; i < kTurns; ++i)
      if (kAllTurn || krow + kRows * i < kFaK) {
        const int row = krow + kRows * i;
        f16x8 a = __builtin_bit_cast(f16x8, kr[i][0]), bb = __builtin_bit_cast(f16x8, kr[i][1]);
        fa_rope8(a, bb, t * kFaK + row, freq + 8 * kpc);
        *reinterpret_cast<f16x8*>(ks + 8 * fa_kslot<DH>(row, kpc)) = a;
        *reinterpret_cast<f16x8*>(ks + 8 * fa_kslot<DH>(row, kpc + PR)) = bb;
      }
  };

  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)fa_smem);
  f32x16 o[OB];
#pragma unroll
  for (int ob = 0; ob < OB; ++ob) o[ob] = f32x16{};
  float m_run = -INFINITY, l_run = 0.f;
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

  // Tile t of the sequence belongs to share t % KSP; round i works on tiles
  // KSP i .. KSP i + KSP - 1 in buffer i % 2 of each share.
  const int n_rounds = (n_tiles + KSP - 1) / KSP;
  auto buffer = [&](int i) { return (KSP * (i & 1) + share) * C::kBuf; };
  if (share < n_tiles) {
    if (ROPE) {
      load_keys(share);
      store_keys(share, fa_smem + buffer(0));
    } else {
      stage(k, koff, share, lds0 + buffer(0));
    }
    stage(v, voff, share, lds0 + buffer(0) + C::kTile);
  }
  for (int i = 0; i < n_rounds; ++i) {
    const int t = KSP * i + share;
    uint8_t* buf = fa_smem + buffer(i);
    // these tiles have landed and every wave is done with the ones
    // before, whose buffers take the next
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const bool more = t + KSP < n_tiles;
    if (more) {
      if (ROPE) load_keys(t + KSP);
      else stage(k, koff, t + KSP, lds0 + buffer(i + 1));
      stage(v, voff, t + KSP, lds0 + buffer(i + 1) + C::kTile);
    }
    const int kt0 = t * kFaK;
    if (t < n_tiles && kt0 <= wave_last) {           // else every key of the tile is after this wave's queries
      const _Float16* ks = reinterpret_cast<const _Float16*>(buf);
      const _Float16* vs = reinterpret_cast<const _Float16*>(buf + C::kTile);
      // S^T: key block kb, lane (query l32, half hl) holds keys kt0 + 32 kb + 8 (v / 4) + 4 hl + v % 4.
      // The key fragments of two contraction steps are read while the two before multiply.
      f32x16 sacc[2];
      sacc[0] = sacc[1] = f32x16{};
      f16x8 kf[2][4];
      auto read_k = [&](int g) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          kf[g & 1][i] = *reinterpret_cast<const f16x8*>(ks + 8 * fa_kslot<DH>(32 * (i & 1) + l32, 2 * (2 * g + (i >> 1)) + hl));
      };
      read_k(0);
#pragma unroll
      for (int g = 0; g < KS / 2; ++g) {
        if (g + 1 < KS / 2) read_k(g + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          sacc[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[g & 1][i], qf[2 * g + (i >> 1)], sacc[i & 1], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      // Value fragments of the 16-key step st: the A operand comes from
      // transposing reads: lane a of a 16-lane group addresses key base + a/4,
      // channels 4 (a % 4) .. +3 of the group's 16 channels, and receives
      // channel a at keys base .. base + 3.
      f16x8 vf[2][OB];
      auto read_v = [&](int st) {
        const int key = 16 * st + 4 * hl + ((lane & 15) >> 2);
#pragma unroll
        for (int ob = 0; ob < OB; ++ob) {
          const int ch = 32 * ob + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (lds_s16x4*)(vs + 8 * fa_vslot<DH>(key, ch >> 3) + (ch & 7)));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (lds_s16x4*)(vs + 8 * fa_vslot<DH>(key + 8, ch >> 3) + (ch & 7)));
          const f16x4 flo = __builtin_bit_cast(f16x4, lo), fhi = __builtin_bit_cast(f16x4, hi);
          vf[st & 1][ob] = f16x8{flo[0], flo[1], flo[2], flo[3], fhi[0], fhi[1], fhi[2], fhi[3]};
        }
      };
      read_v(0);                                     // arrives under the softmax
      // The wait of the scores' first read after the last product, spelled out
      // before the branch below: the compiler pads one side of it only.
      asm volatile("s_nop 7\n\ts_nop 7");
      __builtin_amdgcn_sched_barrier(0);
      // tiles wholly before this wave's first query and inside the sequence need no mask
      if (!(kt0 + kFaK - 1 <= q_off + qw0 && kt0 + kFaK <= nk)) {
        const int lim = min(my_pos, nk - 1) - kt0 - 4 * hl;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int vv = 0; vv < 16; ++vv)
            sacc[kb][vv] = 32 * kb + 8 * (vv >> 2) + (vv & 3) <= lim ? sacc[kb][vv] : -INFINITY;
      }
      // (v_maximum3: fmaxf would first quiet every product; a NaN score makes
      // its row NaN either way)
      float mx = __builtin_elementwise_maximum(sacc[0][0], sacc[1][0]);
#pragma unroll
      for (int vv = 1; vv < 16; ++vv)
        mx = __builtin_elementwise_maximum(mx, __builtin_elementwise_maximum(sacc[0][vv], sacc[1][vv]));
      const float m_new = fmaxf(m_run, fa_pair_max(mx) * scale_log2);
      if (__any(m_new != m_run)) {
        const float alpha = m_new == m_run ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int ob = 0; ob < OB; ++ob) o[ob] *= alpha;
      }
      // (a query with no visible key yet: every exponential below is exp2(-inf) = 0)
      const float m_use = m_run == -INFINITY ? 0.f : m_run;
      float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int vv = 0; vv < 16; ++vv) {
          sacc[kb][vv] = __builtin_amdgcn_exp2f(fmaf(sacc[kb][vv], scale_log2, -m_use));
          ps[vv & 3] += sacc[kb][vv];
        }
      l_run += fa_pair_sum((ps[0] + ps[1]) + (ps[2] + ps[3]));
      // O^T += V^T P^T in four 16-key steps: k-slot e of lane half hl is key
      // 16 st + 8 (e / 4) + 4 hl + e % 4, i.e. score element 8 (st % 2) + e of
      // key block st / 2.
#pragma unroll
      for (int st = 0; st < 4; ++st) {
        f16x8 pf;
#pragma unroll
        for (int e = 0; e < 8; ++e) pf[e] = (_Float16)sacc[st >> 1][8 * (st & 1) + e];
        if (st < 3) read_v(st + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ob = 0; ob < OB; ++ob) o[ob] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[st & 1][ob], pf, o[ob], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (ROPE && more) store_keys(t + KSP, fa_smem + buffer(i + 1));
  }

  if constexpr (KSP > 1) {
    // Share 1 leaves its rows, lane by lane, for share 0 of the same unit.
    __syncthreads();
    f32x4* jo = reinterpret_cast<f32x4*>(fa_smem) + wu * 64 * (DH / 8);
    float2* jm = reinterpret_cast<float2*>(fa_smem + UW * 64 * 4 * (DH / 2)) + wu * 64;
    if (share == 1) {
#pragma unroll
      for (int ob = 0; ob < OB; ++ob)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq)
          jo[(4 * ob + vq) * 64 + lane] = f32x4{o[ob][4 * vq], o[ob][4 * vq + 1], o[ob][4 * vq + 2], o[ob][4 * vq + 3]};
      jm[lane] = make_float2(m_run, l_run);
    }
    __syncthreads();
    if (share == 0) {
      const float2 ml = jm[lane];
      const float m = fmaxf(m_run, ml.x), mu = m == -INFINITY ? 0.f : m;
      const float a0 = __builtin_amdgcn_exp2f(m_run - mu), a1 = __builtin_amdgcn_exp2f(ml.x - mu);
      l_run = l_run * a0 + ml.y * a1;
#pragma unroll
      for (int ob = 0; ob < OB; ++ob)
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
          const f32x4 x = jo[(4 * ob + vq) * 64 + lane];
#pragma unroll
          for (int e = 0; e < 4; ++e) o[ob][4 * vq + e] = o[ob][4 * vq + e] * a0 + x[e] * a1;
        }
    }
  }
  const float inv_l = l_run > 0.f ? 1.f / l_run : 0.f;
  // O / l through LDS, so that each query row leaves as 16-byte runs: lane
  // (l32, hl) holds query qw0 + l32 at channels 32 ob + 8 (v / 4) + 4 hl + v % 4.
  __syncthreads();
  if (!live || share) return;
  _Float16* ost = reinterpret_cast<_Float16*>(fa_smem) + wu * kFaQW * C::OST;
#pragma unroll
  for (int ob = 0; ob < OB; ++ob)
#pragma unroll
    for (int vq = 0; vq < 4; ++vq) {
      const f16x4 v4 = {(_Float16)(o[ob][4 * vq] * inv_l), (_Float16)(o[ob][4 * vq + 1] * inv_l),
                        (_Float16)(o[ob][4 * vq + 2] * inv_l), (_Float16)(o[ob][4 * vq + 3] * inv_l)};
      *reinterpret_cast<f16x4*>(ost + l32 * C::OST + 32 * ob + 8 * vq + 4 * hl) = v4;
    }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the rows below are this wave's own
#pragma unroll
  for (int i = 0; i < kFaQW * RUNS / 64; ++i) {
    const int e = lane + 64 * i, row = e / RUNS, c8 = e - row * RUNS;
    if (qw0 + row < nq)
      *reinterpret_cast<f16x8*>(out + (int64_t)(q_row0 + qw0 + row) * ldq + h * DH + 8 * c8) =
          *reinterpret_cast<const f16x8*>(ost + row * C::OST + 8 * c8);
  }
}

// Workgroups of one (sequence, key/value head): NW units of 32 queries of one
// of the G heads each.
static int fa_workgroups(int queries, int G, int nw) {
  return (int)(((int64_t)((queries + kFaQW - 1) / kFaQW) * G + nw - 1) / nw);
}

template <int DH, int MODE, bool CACHE, int NW, int KSP>
static hipError_t launch_flash(const PrefillAttnArgs& a, const FaCacheArgs& ca, hipStream_t s) {
  using C = FaCfg<DH, NW, KSP>;
  auto kern = prefill_flash_kernel<DH, MODE, CACHE, NW, KSP>;
  const size_t lds = MODE != FA_PLAIN ? C::kLdsRope : C::kLds;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  const int n_wg = fa_workgroups(CACHE ? ca.q_len : a.max_seqlen, a.n_q_heads / a.n_kv_heads, C::UW);
  const int64_t groups = (int64_t)a.batch * a.n_kv_heads;
  const int parts = fa_parts(groups, n_wg);
  const int64_t blocks = fa_blocks(groups, n_wg, parts);
  KernelScope ks(CACHE ? "cache_flash" : MODE != FA_PLAIN ? "prefill_flash_rope" : "prefill_flash", s);
  QSVD_LAUNCH(ks, kern, dim3((unsigned)blocks), dim3(NW * 64), lds, s, a.q, a.k, a.v, a.cu_seqlens, a.batch,
              a.n_q_heads, a.n_kv_heads, n_wg, parts, a.sm_scale * kFaLog2e,
              MODE != FA_PLAIN ? log2((double)a.rope_theta) : 0.0, ca, a.out);
  return hipGetLastError();
}

bool prefill_attention_supported(int32_t head_dim) { return head_dim == 64 || head_dim == 128; }

// The forms a prompt's attention is launched in: the short-prompt kernel
// (flash_short.hip), and this one with four units in four waves (two
// workgroups per CU cover each other's barriers), four units in two key shares
// (eight waves: half the chain per workgroup, one workgroup per CU) or eight
// units (eight waves: the keys of a rotary layer are turned once for all).
enum FaForm { FA_SHORT, FA_4, FA_4x2, FA_8 };

// Chosen by how many workgroups of four units the call makes (w), the longest
// prompt (n), and whether query heads share keys (G > 1, where this kernel's
// units of several heads fill a workgroup that one head of a short prompt
// leaves half empty).  us, per form, rotary (r) or not (p), heads Hq/Hkv of 128:
//   up to 128 tokens the short kernel, but for few tokens or grouped heads
//   over many prompts.  SHORT, 4: 40 heads 8 x 64 r 9.6, 10.2; 40 heads 64 x
//   128 r 68.9, 74.9; 28/4 32 x 64 r 16.8, 12.5; 28/4 64 x 100 p 29.6, 31.0;
//   32 heads 64 x 16 p 20.1, 18.5.
//   w <= 256, no more than one workgroup per CU: a wave's own chain counts.
//   SHORT, 4x2: 28/4 1 x 300 r 15.2, 16.1; 3 x 384 r 17.9, 19.2; 32 heads
//   1 x 448 r 19.5, 18.7; 28/4 1 x 1000 r 38.3, 33.1.
//   w <= 512, up to two: for long prompts still 4x2.  4, 4x2: 28/4 1 x 2000 r
//   72.7, 62.4; 2 x 640 p 21.3, 18.0; 32 heads 3 x 640 r 31.8, 35.1.
//   More: 4, which without rotary embedding always is within 20% of the best;
//   SHORT only where its tiles of 128 queries have no idle ones.  SHORT, 4:
//   32 heads 12 x 256 p 24.5, 28.9; 32 x 256 p 59.2, 54.8; 16 x 384 p 48.9,
//   55.1; 12 x 200 p 23.6, 23.4.
//   Rotary, 8 where that leaves few units without queries: 4, 8: 32 heads
//   2 x 1500 77.6, 67.8; 4 x 800 53.1, 55.4; 4 x 640 37.4, 42.1; 28/4 8 x 640
//   62.3, 55.9; 40 heads 4 x 800 81.1, 69.9.
static FaForm fa_form(const PrefillAttnArgs& a) {
  const bool rope = a.rope_theta > 0.f;
  const int n = a.max_seqlen, G = a.n_q_heads / a.n_kv_heads;
  const int64_t groups = (int64_t)a.batch * a.n_kv_heads;
  const int64_t w = groups * fa_workgroups(n, G, 4), w8 = groups * fa_workgroups(n, G, 8);
  const int64_t tiles = (int64_t)a.batch * a.n_q_heads * (((int64_t)n + 127) / 128);   // of the short kernel
  if (n <= 128) {
    if (tiles <= 256) return FA_SHORT;
    return (!rope && n <= 32) || (G > 1 && (n <= 64 || w <= 512)) ? FA_4 : FA_SHORT;
  }
  if (w <= 256) {
    if (n <= 256 || (n <= 384 && (rope || tiles <= 128))) return FA_SHORT;
    return n <= 384 ? FA_4 : FA_4x2;
  }
  if ((w <= 384 && n > 576) || (w <= 512 && n > 1024)) return FA_4x2;
  const bool full_tiles = (n - 1) % 128 > 120;
  if (G == 1 && full_tiles && (n > 256 ? w > 1024 && n <= 384 : !rope && w > 576 && w < 1024)) return FA_SHORT;
  const bool few_idle = 20 * w8 <= 11 * w;      // at most a tenth more units than with four
  if (rope && ((w > 1024 && n > 512) || (w > 576 && few_idle && n > (G > 1 ? 256 : 512)))) return FA_8;
  return FA_4;
}

template <int DH, int MODE>
static hipError_t launch_prefill(const PrefillAttnArgs& a, FaForm f, hipStream_t s) {
  FaCacheArgs none{};
  none.q_len = a.max_seqlen;                // rows past it are left alone
  if constexpr (MODE == FA_ROPE)
    if (f == FA_8) return launch_flash<DH, MODE, false, 8, 1>(a, none, s);
  return f == FA_4x2 ? launch_flash<DH, MODE, false, 8, 2>(a, none, s) : launch_flash<DH, MODE, false, 4, 1>(a, none, s);
}

hipError_t launch_prefill_attention(const PrefillAttnArgs& a, hipStream_t s) {
  if (a.batch == 0 || a.max_seqlen == 0) return hipSuccess;
  const FaForm f = fa_form(a);
  if (f == FA_SHORT) return launch_prefill_attention_short(a, s);
  if (a.rope_theta > 0.f) return a.head_dim == 128 ? launch_prefill<128, FA_ROPE>(a, f, s) : launch_prefill<64, FA_ROPE>(a, f, s);
  return a.head_dim == 128 ? launch_prefill<128, FA_PLAIN>(a, f, s) : launch_prefill<64, FA_PLAIN>(a, f, s);
}

// Rebuilt keys turned in place at their positions, for layers with rotary
// embedding: thread (position t, pair run) of a sequence turns that run in
// kRkHeads key/value heads (blockIdx.z: which).  Once per call, where the
// attention's workgroups (28 per sequence and key/value head for 100 queries
// of 7 heads each) would each turn every key they read.
constexpr int kRkHeads = 4;

template <int DH>
__global__ void __launch_bounds__(256)
rope_keys_kernel(_Float16* __restrict__ kv, const int32_t* __restrict__ seq_len, int32_t capacity, int32_t ldkv,
                 int32_t Hkv, double log2_theta) {
  constexpr int PR = DH / 16;
  __shared__ double freq[DH / 2];
  const int b = blockIdx.y, t = (blockIdx.x * 256 + threadIdx.x) / PR, pc = threadIdx.x % PR;
  const int g0 = blockIdx.z * kRkHeads;
  const bool in = t < min(seq_len[b], capacity);
  _Float16* row = kv + ((int64_t)b * capacity + t) * ldkv + g0 * DH + 8 * pc;
  f16x8 x[kRkHeads], y[kRkHeads];
#pragma unroll
  for (int i = 0; i < kRkHeads; ++i)
    if (in && g0 + i < Hkv) {
      x[i] = *reinterpret_cast<const f16x8*>(row + i * DH);
      y[i] = *reinterpret_cast<const f16x8*>(row + i * DH + DH / 2);
    }
  if (threadIdx.x < DH / 2) freq[threadIdx.x] = fa_freq(threadIdx.x, DH, log2_theta);
  __syncthreads();
  float c[8], sn[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) fa_angle(t, freq[8 * pc + e], &c[e], &sn[e]);
#pragma unroll
  for (int i = 0; i < kRkHeads; ++i)
    if (in && g0 + i < Hkv) {
      fa_turn8(x[i], y[i], c, sn);
      *reinterpret_cast<f16x8*>(row + i * DH) = x[i];
      *reinterpret_cast<f16x8*>(row + i * DH + DH / 2) = y[i];
    }
}

// Few queries over many keys leave few workgroups: their waves share the keys
// in two halves (4x2) until there is more than one workgroup of four units per
// CU, or one where the keys are few.  100 queries of 28 heads over 4, four
// sequences of 1899 tokens: 87 -> 44 us; whole calls, 4 and 4x2: 160 queries,
// 1899 tokens, 32 heads, eight sequences 523, 544 (512 workgroups), four 294,
// 288 (256); 28/4, eight sequences 117, 128 (288); 100 queries, 300 tokens, 32
// heads, eight sequences 116, 119 (256).
// The keys of rotary layers are turned in the attention where each is read
// once (no grouped heads) by enough workgroups, or where they are few.  Whole
// calls, in it (4x2) and before it: 32 heads, 16 queries, 1899 tokens, one
// sequence 112, 102, four 256, 265, eight 445, 501; 300 tokens, one sequence
// 49.4, 50.8; 28/4, 300 tokens 23.6, 26.1, 600 tokens 55.8, 54.2, 1899 tokens
// 65.3, 53.5.  With a workgroup of eight units for every CU those share them:
// 32 heads, eight sequences, 4x2 and 8: 160 queries, 1899 tokens 567, 523, 100
// queries, 300 tokens 124, 121; four sequences (128 workgroups), 160 queries,
// 1899 tokens 303, 327.
template <int DH>
static hipError_t launch_cache(const CacheAttnArgs& c, const PrefillAttnArgs& a, const FaCacheArgs& ca, hipStream_t s) {
  const int G = c.n_q_heads / c.n_kv_heads;
  const int64_t w = (int64_t)c.batch * c.n_kv_heads * fa_workgroups(c.q_len, G, 4);
  const int64_t w8 = (int64_t)c.batch * c.n_kv_heads * fa_workgroups(c.q_len, G, 8);
  const bool filled = w > 256, few_keys = c.max_len <= 512;
  if (c.rope_theta <= 0.f)
    return filled || (w == 256 && few_keys) ? launch_flash<DH, FA_PLAIN, true, 4, 1>(a, ca, s) : launch_flash<DH, FA_PLAIN, true, 8, 2>(a, ca, s);
  if (G == 1 && w8 >= 256) return launch_flash<DH, FA_ROPE, true, 8, 1>(a, ca, s);
  if (G == 1 ? few_keys || w >= 96 : few_keys && !filled) return launch_flash<DH, FA_ROPE, true, 8, 2>(a, ca, s);
  {
    KernelScope ks("rope_keys", s);
    const dim3 grid((unsigned)(((int64_t)c.max_len * (DH / 16) + 255) / 256), c.batch,
                    (c.n_kv_heads + kRkHeads - 1) / kRkHeads);
    QSVD_LAUNCH(ks, rope_keys_kernel<DH>, grid, dim3(256), 0, s, c.kv, c.seq_len, c.capacity, ca.ldkv, c.n_kv_heads,
                log2((double)c.rope_theta));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return filled ? launch_flash<DH, FA_ROPE_Q, true, 4, 1>(a, ca, s) : launch_flash<DH, FA_ROPE_Q, true, 8, 2>(a, ca, s);
}

// Queries of several positions per sequence over a cache's rebuilt K^ | V^
// rows (the reconstruct form with q_len > 1).
hipError_t launch_cache_attention(const CacheAttnArgs& c, hipStream_t s) {
  if (c.batch == 0 || c.q_len == 0) return hipSuccess;
  const int nkv = c.n_kv_heads * c.head_dim;
  const PrefillAttnArgs a{c.q, c.kv, c.kv + nkv, nullptr, c.batch, c.q_len, c.n_q_heads, c.n_kv_heads, c.head_dim,
                          c.sm_scale, c.out, c.rope_theta};
  const FaCacheArgs ca{c.seq_len, c.capacity, c.q_len, 2 * nkv};
  return c.head_dim == 128 ? launch_cache<128>(c, a, ca, s) : launch_cache<64>(c, a, ca, s);
}

}  // namespace qsvd
