// Causal self-attention of short prompts: the same product as flash.hip, for
// the calls sent here by fa_form there (few workgroups, or up to 128 tokens;
// its comment has the figures of both).
//
// One workgroup of eight waves takes 128 consecutive queries of one
// (sequence, query head); wave w owns the 16-query block q0 + 16w .. +15.
// With half the queries per wave of flash.hip's units every LDS read serves
// half the products, but a wave's chain through a tile (scores, softmax,
// output) is half as long and twice as many waves fit a CU, which is what
// counts while the chip is not full or the chains are short.
//
// Key/value tiles of 64 tokens are staged in LDS (shared by the waves; the
// next tile's rows are already in registers while the current one is used).
// Per tile and wave, on the 16x16x32 fp16 matrix cores:
//   S^T (64 keys x 16 queries) = K_tile Q^T          (contraction over dh)
//   online softmax per query in fp32 (a query is one lane column; its 64
//   scores sit in that lane and the three lanes l ^ 16, l ^ 32, l ^ 48)
//   O^T (dh x 16 queries) += V_tile^T P^T            (contraction over keys)
// The query rows stay in registers for the whole kernel.  Keys past a query's
// position, or past the sequence end, are masked.
//
// Rotary layers (ROPE): a query row is turned once, in registers, at its
// position within the sequence; a key row is turned while its tile moves from
// registers into LDS, at its own position (flash.h says how).
#include <math.h>

#include "common.h"
#include "flash.h"
#include "launch.h"

namespace qsvd {

constexpr int kFsQ = 128;       // queries per workgroup
constexpr int kFsWaves = 8;
constexpr int kFsQW = kFsQ / kFsWaves;   // queries per wave: one block of 16
static_assert(kFsQW == 16);

template <int DH>
struct FsCfg {
  static constexpr int KST = DH + 8;       // K tile row stride (halves): 16-byte row reads hit every bank once
  static constexpr int VST = DH + 16;      // V tile row stride: the transposing reads hit distinct banks
  static constexpr int OST = DH + 8;       // output staging row stride
  static constexpr size_t kK = (size_t)kFaK * KST * 2, kV = (size_t)kFaK * VST * 2;
  static constexpr size_t kOut = (size_t)kFsWaves * kFsQW * OST * 2;
  static constexpr size_t kLds = kK + kV > kOut ? kK + kV : kOut;
  static constexpr size_t kLdsRope = kLds + (size_t)(DH / 2) * sizeof(double);   // + revolutions per position of each pair
  static constexpr int kChunks = kFaK * DH / 8;               // 16-byte runs per K (or V) tile
  static constexpr int kPerThread = kChunks / (kFsWaves * 64);
  static_assert(kChunks % (kFsWaves * 64) == 0, "whole runs per thread");
};

// Rotary staging of a key tile: thread tid turns the 8 pairs of run pc
// (channels 8 pc .. +7 with their partners dh/2 further) of row tid / PR.
template <int DH>
struct FsRope {
  static constexpr int PR = DH / 16;                     // pair runs per row
  static constexpr int kActive = kFaK * PR;              // threads with a key row to turn
  static_assert(kActive <= kFsWaves * 64, "one pair run per thread");
  static constexpr int KR = FsCfg<DH>::kPerThread > 2 ? FsCfg<DH>::kPerThread : 2;   // key registers per thread
};

// Key/value tile t of the rows this thread stages (rows past the sequence end
// re-read its last row; they are masked).  With ROPE the key registers hold
// the two halves of one pair run instead.
template <int DH, bool ROPE>
__device__ __forceinline__ void fs_load_tile(const _Float16* __restrict__ k, const _Float16* __restrict__ v, int tok0,
                                             int n, int ldkv, int g, int t, int tid,
                                             i32x4 (&kr)[FsRope<DH>::KR], i32x4 (&vr)[FsCfg<DH>::kPerThread]) {
  constexpr int RUNS = DH / 8;
#pragma unroll
  for (int i = 0; i < FsCfg<DH>::kPerThread; ++i) {
    const int e = tid + kFsWaves * 64 * i, row = e / RUNS, c8 = e - row * RUNS;
    const int key = min(t * kFaK + row, n - 1);
    const int64_t off = (int64_t)(tok0 + key) * ldkv + g * DH + 8 * c8;
    if (!ROPE) kr[i] = *reinterpret_cast<const i32x4*>(k + off);
    vr[i] = *reinterpret_cast<const i32x4*>(v + off);
  }
  if (ROPE && tid < FsRope<DH>::kActive) {
    constexpr int PR = FsRope<DH>::PR;
    const int row = tid / PR, pc = tid - row * PR;
    const int key = min(t * kFaK + row, n - 1);
    const _Float16* src = k + (int64_t)(tok0 + key) * ldkv + g * DH + 8 * pc;
    kr[0] = *reinterpret_cast<const i32x4*>(src);
    kr[1] = *reinterpret_cast<const i32x4*>(src + DH / 2);
  }
}

// ... and its copy into the LDS tiles (turning the keys of a rotary layer at
// positions t * 64 + row).
template <int DH, bool ROPE>
__device__ __forceinline__ void fs_store_tile(_Float16* ks, _Float16* vs, int tid, int t, const double* freq,
                                              const i32x4 (&kr)[FsRope<DH>::KR],
                                              const i32x4 (&vr)[FsCfg<DH>::kPerThread]) {
  constexpr int RUNS = DH / 8;
#pragma unroll
  for (int i = 0; i < FsCfg<DH>::kPerThread; ++i) {
    const int e = tid + kFsWaves * 64 * i, row = e / RUNS, c8 = e - row * RUNS;
    if (!ROPE) *reinterpret_cast<i32x4*>(ks + row * FsCfg<DH>::KST + 8 * c8) = kr[i];
    *reinterpret_cast<i32x4*>(vs + row * FsCfg<DH>::VST + 8 * c8) = vr[i];
  }
  if (ROPE && tid < FsRope<DH>::kActive) {
    constexpr int PR = FsRope<DH>::PR;
    const int row = tid / PR, pc = tid - row * PR;
    f16x8 a = __builtin_bit_cast(f16x8, kr[0]), b = __builtin_bit_cast(f16x8, kr[1]);
    fa_rope8(a, b, t * kFaK + row, freq + 8 * pc);
    *reinterpret_cast<f16x8*>(ks + row * FsCfg<DH>::KST + 8 * pc) = a;
    *reinterpret_cast<f16x8*>(ks + row * FsCfg<DH>::KST + 8 * pc + DH / 2) = b;
  }
}

template <int DH, bool ROPE>
__global__ void __launch_bounds__(kFsWaves * 64, 2)
prefill_flash_short_kernel(const _Float16* __restrict__ q, const _Float16* __restrict__ k, const _Float16* __restrict__ v,
                           const int32_t* __restrict__ cu, int32_t n_seq, int32_t Hq, int32_t Hkv, int32_t n_qt,
                           float scale_log2, double log2_theta, int32_t max_seqlen, _Float16* __restrict__ out) {
  using C = FsCfg<DH>;
  constexpr int KS = DH / 32;      // contraction steps of the score product
  constexpr int OB = DH / 16;      // 16-channel blocks of the output
  constexpr int RUNS = DH / 8;     // 16-byte runs per row
  extern __shared__ __attribute__((aligned(16))) uint8_t fs_smem[];
  _Float16* ks = reinterpret_cast<_Float16*>(fs_smem);
  _Float16* vs = reinterpret_cast<_Float16*>(fs_smem + C::kK);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;

  // Workgroup -> (sequence, head, query tile).  The query tiles of one
  // (sequence, head) read the same key/value rows, so they get ids that one
  // XCD receives (the chip hands workgroup i to XCD i % 8) and share its L2;
  // within a group the longest tiles (most keys) go first.
  const int groups = n_seq * Hq, total = groups * n_qt;
  int lin = blockIdx.x;
  if (total % 8 == 0) lin = (lin % 8) * (total / 8) + lin / 8;
  const int grp = lin / n_qt, qt = n_qt - 1 - (lin - grp * n_qt);
  const int b = grp / Hq, h = grp - b * Hq;
  // this sequence's rows: query i sees the keys at positions <= i
  const int row0 = cu[b], n = min(cu[b + 1] - row0, max_seqlen);
  const int q0 = qt * kFsQ;
  if (q0 >= n) return;
  double* freq = reinterpret_cast<double*>(fs_smem + C::kLds);
  if (ROPE) {
    if (tid < DH / 2) freq[tid] = fa_freq(tid, DH, log2_theta);
    __syncthreads();
  }
  const int g_kv = (h * Hkv) / Hq;
  const int ldq = Hq * DH, ldkv = Hkv * DH;
  const int kend = min(n, q0 + kFsQ);               // keys this tile of queries can see
  const int n_tiles = (kend + kFaK - 1) / kFaK;
  const int qw0 = q0 + kFsQW * w;                   // this wave's first query
  const int my_q = qw0 + l16;                       // this lane's query

  // query slots of the score product: step s, lane group g -> channels 32 s + 8 g .. +7
  f16x8 qf[KS];
  const _Float16* qrow = q + (int64_t)(row0 + min(my_q, n - 1)) * ldq + h * DH + 8 * g;
#pragma unroll
  for (int s = 0; s < KS; ++s) qf[s] = *reinterpret_cast<const f16x8*>(qrow + 32 * s);
  if (ROPE) {                                       // slot s pairs with slot s + KS/2 (channels dh/2 further)
#pragma unroll
    for (int s = 0; s < KS / 2; ++s) fa_rope8(qf[s], qf[s + KS / 2], min(my_q, n - 1), freq + 32 * s + 8 * g);
  }

  i32x4 kr[FsRope<DH>::KR], vr[C::kPerThread];
  f32x4 o[OB];
#pragma unroll
  for (int ob = 0; ob < OB; ++ob) o[ob] = f32x4{};
  float m_run = -INFINITY, l_run = 0.f;
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

  fs_load_tile<DH, ROPE>(k, v, row0, n, ldkv, g_kv, 0, tid, kr, vr);
  for (int t = 0; t < n_tiles; ++t) {
    __syncthreads();                                // every wave is done with the previous tile
    fs_store_tile<DH, ROPE>(ks, vs, tid, t, freq, kr, vr);
    __syncthreads();
    if (t + 1 < n_tiles) fs_load_tile<DH, ROPE>(k, v, row0, n, ldkv, g_kv, t + 1, tid, kr, vr);
    const int kt0 = t * kFaK;
    if (kt0 > qw0 + kFsQW - 1) continue;            // every key of the tile is after this wave's queries
    // S^T: key block kb, lane (query l16, group g) holds keys kt0 + 16 kb + 4 g + v
    f32x4 sacc[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      sacc[kb] = f32x4{};
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const f16x8 kf = *reinterpret_cast<const f16x8*>(ks + (16 * kb + l16) * C::KST + 32 * s + 8 * g);
        sacc[kb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, qf[s], sacc[kb], 0, 0, 0);
      }
    }
    // softmax (tiles wholly before this wave's first query and inside the
    // sequence need no mask)
    const bool full = kt0 + kFaK - 1 <= qw0 && kt0 + kFaK <= n;
    float p[4][4];
    float mx = -INFINITY;
    if (full) {
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int vv = 0; vv < 4; ++vv) {
          p[kb][vv] = sacc[kb][vv] * scale_log2;
          mx = fmaxf(mx, p[kb][vv]);
        }
    } else {
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int vv = 0; vv < 4; ++vv) {
          const int key = kt0 + 16 * kb + 4 * g + vv;
          p[kb][vv] = (key <= my_q && key < n) ? sacc[kb][vv] * scale_log2 : -INFINITY;
          mx = fmaxf(mx, p[kb][vv]);
        }
    }
    const float m_new = fmaxf(m_run, fa_rows4_max(mx));
    float alpha = 1.f, ps = 0.f;
    if (m_new == -INFINITY) {
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int vv = 0; vv < 4; ++vv) p[kb][vv] = 0.f;
    } else {
      alpha = __builtin_amdgcn_exp2f(m_run - m_new);
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int vv = 0; vv < 4; ++vv) {
          p[kb][vv] = __builtin_amdgcn_exp2f(p[kb][vv] - m_new);
          ps += p[kb][vv];
        }
    }
    l_run = l_run * alpha + fa_rows4_sum(ps);
    m_run = m_new;
    if (__any(alpha != 1.f)) {
#pragma unroll
      for (int ob = 0; ob < OB; ++ob) o[ob] *= alpha;
    }
    // O^T += V^T P^T in two 32-key steps st: k-slot e of lane group g is key
    // 32 st + 16 (e / 4) + 4 g + e % 4, i.e. score p[2 st + e / 4][e % 4].
    // The A operand comes from transposing reads: lane a of group g addresses
    // key 4g + a/4 of the 16-key block, channels 16 ob + 4 (a % 4) .. +3, and
    // lane i receives element i % 4 of the chunks of lanes i/4, 4 + i/4,
    // 8 + i/4, 12 + i/4: channel 16 ob + i at keys 4g .. 4g+3 of the block.
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      f16x8 pf;
#pragma unroll
      for (int e = 0; e < 8; ++e) pf[e] = (_Float16)p[2 * st + (e >> 2)][e & 3];
      const int key = 32 * st + 4 * g + (l16 >> 2);
#pragma unroll
      for (int ob = 0; ob < OB; ++ob) {
        const _Float16* a0 = vs + key * C::VST + 16 * ob + 4 * (l16 & 3);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)a0);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(a0 + 16 * C::VST));
        const f16x4 flo = __builtin_bit_cast(f16x4, lo), fhi = __builtin_bit_cast(f16x4, hi);
        const f16x8 a = {flo[0], flo[1], flo[2], flo[3], fhi[0], fhi[1], fhi[2], fhi[3]};
        o[ob] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, pf, o[ob], 0, 0, 0);
      }
    }
  }

  // O / l through LDS, so that each query row leaves as 16-byte runs: lane
  // (l16, g) holds query qw0 + l16 at channels 16 ob + 4 g .. +3.
  __syncthreads();
  _Float16* ost = reinterpret_cast<_Float16*>(fs_smem) + w * kFsQW * C::OST;
  const float inv_l = l_run > 0.f ? 1.f / l_run : 0.f;
#pragma unroll
  for (int ob = 0; ob < OB; ++ob) {
    const f16x4 v4 = {(_Float16)(o[ob][0] * inv_l), (_Float16)(o[ob][1] * inv_l), (_Float16)(o[ob][2] * inv_l),
                      (_Float16)(o[ob][3] * inv_l)};
    *reinterpret_cast<f16x4*>(ost + l16 * C::OST + 16 * ob + 4 * g) = v4;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kFsQW * RUNS / 64; ++i) {
    const int e = lane + 64 * i, row = e / RUNS, c8 = e - row * RUNS;
    const int qq = qw0 + row;
    if (qq < n)
      *reinterpret_cast<f16x8*>(out + (int64_t)(row0 + qq) * ldq + h * DH + 8 * c8) =
          *reinterpret_cast<const f16x8*>(ost + row * C::OST + 8 * c8);
  }
}

template <int DH, bool ROPE>
static hipError_t launch_short(const PrefillAttnArgs& a, hipStream_t s) {
  using C = FsCfg<DH>;
  auto kern = prefill_flash_short_kernel<DH, ROPE>;
  const size_t lds = ROPE ? C::kLdsRope : C::kLds;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  const int n_qt = (a.max_seqlen + kFsQ - 1) / kFsQ;
  KernelScope ks(ROPE ? "prefill_flash_rope" : "prefill_flash", s);
  QSVD_LAUNCH(ks, kern, dim3((unsigned)(a.batch * a.n_q_heads * n_qt)), dim3(kFsWaves * 64), lds, s, a.q, a.k, a.v,
              a.cu_seqlens, a.batch, a.n_q_heads, a.n_kv_heads, n_qt, a.sm_scale * kFaLog2e,
              ROPE ? log2((double)a.rope_theta) : 0.0, a.max_seqlen, a.out);
  return hipGetLastError();
}

hipError_t launch_prefill_attention_short(const PrefillAttnArgs& a, hipStream_t s) {
  if (a.rope_theta > 0.f) return a.head_dim == 128 ? launch_short<128, true>(a, s) : launch_short<64, true>(a, s);
  return a.head_dim == 128 ? launch_short<128, false>(a, s) : launch_short<64, false>(a, s);
}

}  // namespace qsvd
