// Contribution score of every row at a pruning layer: the column sums of
// the normalised soft-score matrices, summed over heads,
//     s[j] = sum_h sum_i exp(q_i . k_j * scale - lse_h[i]),
// over the rows i the mask lets see row j. The normalised probability needs
// each query row's final log-sum-exp, which the attention pass has already
// written, so this is a second sweep over Q K^T that never stores P.
//
// bf16, head_dim 64/128 (MFMA): S = Q K^T with v_mfma_f32_32x32x16_bf16 in
// the *non*-transposed layout, where a lane owns one key column and 16 query
// rows, so the column sum is in-lane adds. One partial vector per head
// ([H][T]); the top-k kernel adds the H partials in a fixed order. No
// atomics: the result is bitwise reproducible. score_wide_kernel: a wave
// owns 64 keys and goes over all queries; score_mfma_kernel (grids of few
// workgroups): a workgroup's eight waves share 128 keys and stride over the
// queries. Under the causal mask both start at the first query that can see
// their keys.
//
// fp32 / other head dims: the same on the fp32 matrix instruction.
#include <math.h>

#include "zsa_internal.h"

namespace zsa {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kScoreWaves = 8;

template <int HD, int KB>
__global__ __launch_bounds__(64 * kScoreWaves) __attribute__((amdgpu_waves_per_eu(HD == 64 ? 4 : 2))) void score_mfma_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, int64_t rs,
    const float* __restrict__ lse, int H, int kv_group, int causal, float scale_log2,
    const int32_t* __restrict__ cu, int T, float* __restrict__ partials, int pairs) {
  constexpr int NW = kScoreWaves, NT = 64 * NW;
  constexpr int KLD = HD + 8;  // K tile row stride (bf16): conflict-free fragment reads
  constexpr int KK = HD / 16;
  constexpr int KS = KB / 32;  // 32-key columns
  constexpr int LPR = HD / 8;   // lanes per 16-byte-chunked Q row
  constexpr int RPI = 64 / LPR;  // Q rows per load
  constexpr int NQI = 32 / RPI;  // loads per 32-row tile
  static_assert(KB * KLD * 2 >= NW * KB * 4, "the reduction fits the K tile");
  __shared__ __align__(16) unsigned char smem[KB * KLD * 2];
  __shared__ __align__(16) unsigned char qbuf[NW][32 * HD * 2];  // each wave's Q tile
  bf16_t* Ks = reinterpret_cast<bf16_t*>(smem);

  Place at;
  if (!place(H, kv_group, pairs, true, &at)) return;
  const int b = at.b, h = at.h;
  const int lo = cu[b];
  const int n = cu[b + 1] - lo;
  const int j0 = at.i * KB;
  if (j0 >= n) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int hf = lane >> 5, l32 = lane & 31;

  for (int c = tid; c < KB * HD / 8; c += NT) {
    const int r = c / (HD / 8), ch = (c % (HD / 8)) * 8;
    // keys past the sequence repeat the last row; their columns are not written
    *reinterpret_cast<uint4*>(Ks + r * KLD + ch) =
        *reinterpret_cast<const uint4*>(K + static_cast<int64_t>(lo + min(j0 + r, n - 1)) * rs +
                                        (h / kv_group) * HD + ch);
  }
  __syncthreads();

  float colsum[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) colsum[ks] = 0.f;
  // this head's log-sum-exp of the sequence's rows, in exp2 units; rows past
  // the sequence read as zeros (their scores are masked)
  const __amdgpu_buffer_rsrc_t lres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(lse + static_cast<int64_t>(h) * T + lo), 0, static_cast<uint32_t>(n) * 4u,
      0x00020000);
  // Query tiles of 32 rows, strided over the waves; the next tile's Q is
  // loaded while this tile's products and exps run. Rows past the sequence
  // are clamped and masked. The loads cover whole cache lines (HD / 8 lanes
  // per row); the wave passes each tile through its LDS buffer (chunk c of
  // row r at r * 2 HD + (c ^ (r % 8)) * 16) into the MFMA fragments (lane
  // l: row l % 32, chunk 2 kk + l / 32). Fragments loaded straight from
  // memory would touch 32 lines per load, a quarter of each.
  const bf16_t* qh = Q + static_cast<int64_t>(lo) * rs + h * HD + (lane % LPR) * 8;
  unsigned char* const qw = qbuf[wave];
  int i0 = (causal ? (j0 & ~31) : 0) + wave * 32;
  u32x4 qn[NQI];
  if (i0 < n) {
#pragma unroll
    for (int i = 0; i < NQI; ++i)
      qn[i] = *reinterpret_cast<const u32x4*>(qh + static_cast<int64_t>(min(i0 + RPI * i + lane / LPR, n - 1)) * rs);
  }
  for (; i0 < n; i0 += 32 * NW) {
    // LDS operations of a wave run in order: these stores follow the last
    // tile's fragment reads
#pragma unroll
    for (int i = 0; i < NQI; ++i) {
      const int r = RPI * i + lane / LPR;
      *reinterpret_cast<u32x4*>(qw + r * (HD * 2) + (((lane % LPR) ^ (r & 7)) << 4)) = qn[i];
    }
    bf16x8_t qa[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
      qa[kk] = __builtin_bit_cast(
          bf16x8_t, *reinterpret_cast<const u32x4*>(qw + l32 * (HD * 2) + (((2 * kk + hf) ^ (l32 & 7)) << 4)));
    const int inext = i0 + 32 * NW;
    if (inext < n) {
#pragma unroll
      for (int i = 0; i < NQI; ++i)
        qn[i] = *reinterpret_cast<const u32x4*>(qh + static_cast<int64_t>(min(inext + RPI * i + lane / LPR, n - 1)) * rs);
    }
    // this lane's 16 query rows: i0 + 8 (r/4) + 4 hf + r%4
    float L[16];
#pragma unroll
    for (int r = 0; r < 16; ++r)
      L[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                           lres, static_cast<uint32_t>(i0 + 8 * (r >> 2) + 4 * hf + (r & 3)) * 4u, 0, 0)) *
             kLog2e;
    // S for the tile and key column ks: acc[r] = query i0 + 8 (r/4) + 4 hf + r%4,
    // key j0 + 32 ks + l32
    auto block = [&](int ks) {
      f32x16_t acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const bf16x8_t kf = __builtin_bit_cast(
            bf16x8_t, *reinterpret_cast<const u32x4*>(Ks + (ks * 32 + l32) * KLD + kk * 16 + hf * 8));
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qa[kk], kf, acc, 0, 0, 0);
      }
      return acc;
    };
    if (i0 + 32 <= n && (!causal || i0 >= j0 + KB)) {
      // every query of the tile sees every key of the block: no masks, and
      // column ks + 1's products are issued before column ks's exps
      f32x16_t a0 = block(0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        f32x16_t a1;
        if (ks + 1 < KS) a1 = block(ks + 1);
        float tsum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) tsum += __builtin_amdgcn_exp2f(fmaf(a0[r], scale_log2, -L[r]));
        colsum[ks] += tsum;
        if (ks + 1 < KS) a0 = a1;
      }
    } else {
      // the tile crosses the sequence end or the diagonal
      const bool tail = i0 + 32 > n;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        // under the causal mask no query of the tile sees this or any later
        // column once its first key is past the tile's last query
        if (causal && j0 + 32 * ks > i0 + 31) break;
        const f32x16_t acc = block(ks);
        float tsum = 0.f;
        if (!tail && (!causal || j0 + 32 * ks + 31 <= i0)) {
#pragma unroll
          for (int r = 0; r < 16; ++r) tsum += __builtin_amdgcn_exp2f(fmaf(acc[r], scale_log2, -L[r]));
        } else {
          const int j = j0 + ks * 32 + l32;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int i = i0 + 8 * (r >> 2) + 4 * hf + (r & 3);
            const bool ok = i < n && (!causal || j <= i);
            tsum += ok ? __builtin_amdgcn_exp2f(fmaf(acc[r], scale_log2, -L[r])) : 0.f;
          }
        }
        colsum[ks] += tsum;
      }
    }
  }
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) colsum[ks] = half_swap_sum(colsum[ks]);
  __syncthreads();  // every wave is done with the K tile
  float* red = reinterpret_cast<float*>(smem);  // [NW][KB]
  if (hf == 0) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) red[wave * KB + 32 * ks + l32] = colsum[ks];
  }
  __syncthreads();
  for (int c = tid; c < KB; c += NT) {
    const int j = j0 + c;
    float v = red[c];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += red[w * KB + c];
    if (j < n) partials[static_cast<int64_t>(h) * T + lo + j] = v;
  }
}

// Grids of enough workgroups (launch_score). A wave owns 64 keys, their operand in registers, and goes
// over the queries in steps of 32: in step u it issues the products
// S(u + 1) = Q K^T one at a time with the exponentials and sums of step u
// between them (scheduling barriers fix the order), three waves per SIMD (two
// at head dim 128, where a third spills) so that each fills the others' gaps. Query tiles of 64 rows and their
// log-sum-exp go straight to LDS two tiles ahead, shared by the four waves
// (256 keys), as K and V do in the attention kernel. A key's sum is one
// wave's, in query order: no reduction over waves. The earlier kernel above
// split a block's queries over eight waves that each staged its own tiles
// through registers.
// Same box, us with the sum over heads, earlier kernel / this one: 8 x 2048
// causal rows, 32 heads of 64, 176 / 130; 32 x 512, 12 heads of 64, 31.8 /
// 29.1; 4 x 4096 causal, 32 heads of 128, 520 / 301; 12 ragged sequences of up
// to 4095 rows 1054 / 423; and with few workgroups, where the earlier one
// keeps more waves busy: 32 x 256, 12 heads of 64, 15.6 / 17.5.
template <int HD, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(HD == 64 ? 3 : 2, HD == 64 ? 3 : 2))) void score_wide_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, int64_t rs,
    const float* __restrict__ lse, int H, int kv_group, int causal, float scale_log2,
    const int32_t* __restrict__ cu, int T, float* __restrict__ partials, int pairs) {
  constexpr int KW = 64, KB = KW * NW, QT = 64;
  constexpr int KK = HD / 16, CPR = HD / 8, RB = HD * 2;
  constexpr int QBYTES = QT * RB, BUF = QBYTES + 1024, NB = 3;
  constexpr int RPL = 1024 / RB, LPW = QBYTES / 1024 / NW;  // rows per load, loads per wave
  static_assert(LPW * NW * 1024 == QBYTES, "tile split");
  __shared__ __align__(1024) unsigned char smem[NB * BUF];

  Place at;
  if (!place(H, kv_group, pairs, true, &at)) return;
  const int b = at.b, h = at.h;
  const int lo = cu[b];
  const int n = cu[b + 1] - lo;
  const int j0 = at.i * KB;
  if (j0 >= n) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, l32 = lane & 31;
  const int wk0 = j0 + wave * KW;  // the wave's first key

  const uint32_t row_bytes = static_cast<uint32_t>(rs * 2);
  // rows past the sequence read as zeros (masked)
  const u32x4 qres = buffer_resource(Q + static_cast<int64_t>(lo) * rs + h * HD, static_cast<uint32_t>(n) * row_bytes);
  const u32x4 lres = buffer_resource(lse + static_cast<int64_t>(h) * T + lo, static_cast<uint32_t>(n) * 4u);
  // row r keeps its 16-byte chunk c at c ^ qsw(r): the 16 rows of a read
  // phase fall on all banks
  auto qsw = [](int r) { return HD == 64 ? (r >> 1) & 7 : r & 15; };
  uint32_t qoff[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int r = (wave + NW * i) * RPL + lane / CPR;
    qoff[i] = r * row_bytes + (((lane % CPR) ^ qsw(r)) << 4);
  }
  const uint32_t lds0 = lds_address(smem);
  auto load_tile = [&](int t, int buf) {
    const uint32_t t0 = static_cast<uint32_t>(t) * (QT * row_bytes);
#pragma unroll
    for (int i = 0; i < LPW; ++i) lds_load16(lds0 + buf * BUF + (wave + NW * i) * 1024, qoff[i] + t0, qres);
    if (wave == 0) lds_load4(lds0 + buf * BUF + QBYTES, static_cast<uint32_t>(t * QT + lane) * 4u, lres);
  };

  const int t0 = causal ? j0 / QT : 0, nt = (n + QT - 1) / QT;
  // the wave's own tiles: under the causal mask none before its first key
  const int tw = causal ? min(wk0 / QT, nt) : 0;
  load_tile(t0, 0);
  if (t0 + 1 < nt) load_tile(t0 + 1, 1);

  bf16x8_t kf[2][KK];
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
      // keys past the sequence repeat the last row; their sums are not written
      kf[kb][kk] = __builtin_bit_cast(
          bf16x8_t, *reinterpret_cast<const u32x4*>(K + static_cast<int64_t>(lo + min(wk0 + 32 * kb + l32, n - 1)) * rs +
                                                    (h / kv_group) * HD + kk * 16 + half * 8));
  float colsum[2] = {0.f, 0.f};
  f32x16_t sa[2], sb[2];
  uint32_t qaddr[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) qaddr[kk] = l32 * RB + (((2 * kk + half) ^ qsw(l32)) << 4);
  auto read_q = [&](const unsigned char* base, int kk) {
    return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(base + qaddr[kk]));
  };
  const f32x16_t zero = {};
  // step u: the sums of its scores s (tile in buffer bufc) beside the
  // products S(u + 1) = sn (tile in buffer bufn)
  auto step = [&](int u, int bufc, int bufn, int qn, f32x16_t (&s)[2], f32x16_t (&sn)[2]) {
    constexpr int FA = 2, NS = 2 * KK, NU = 32;
    const unsigned char* qp = smem + bufn * BUF + qn * (32 * RB);
    const float* lp = reinterpret_cast<const float*>(smem + bufc * BUF + QBYTES) + 32 * (u & 1) + 4 * half;
    bf16x8_t fr[FA + 1];
    auto product = [&](int i) {
      const int kk = i >> 1, kb = i & 1;
      sn[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[kk % (FA + 1)], kf[kb][kk], kk == 0 ? zero : sn[kb], 0, 0, 0);
    };
    float4 L[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) L[a] = *reinterpret_cast<const float4*>(lp + 8 * a);
#pragma unroll
    for (int f = 0; f < FA; ++f) fr[f] = read_q(qp, f);
    auto lse2 = [&](int r) {
      const float4 l = L[r >> 2];
      return ((r & 3) == 0 ? l.x : (r & 3) == 1 ? l.y : (r & 3) == 2 ? l.z : l.w) * kLog2e;
    };
    const int i0 = 32 * u;
    if (i0 + 32 <= n && !(causal && i0 < wk0 + KW - 1)) {
      float nl[16], p0 = 0.f, p1 = 0.f, a0 = 0.f, a1 = 0.f;
      auto work = [&](int w) {
        const int r = (w >> 1) & 14, kb = (w >> 1) & 1;  // pairs of rows, both key blocks of a pair in turn
        if ((w & 1) == 0) {
          if (kb == 0) {
            nl[r] = lse2(r);
            nl[r + 1] = lse2(r + 1);
          }
          p0 = __builtin_amdgcn_exp2f(fmaf(s[kb][r], scale_log2, -nl[r]));
          p1 = __builtin_amdgcn_exp2f(fmaf(s[kb][r + 1], scale_log2, -nl[r + 1]));
          asm volatile("" : "+v"(p0), "+v"(p1));  // computed here, beside this step's products
        } else if (kb == 0) {
          a0 = r == 0 ? p0 + p1 : a0 + (p0 + p1);
          asm volatile("" : "+v"(a0));
        } else {
          a1 = r == 0 ? p0 + p1 : a1 + (p0 + p1);
          asm volatile("" : "+v"(a1));
        }
      };
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        if ((i & 1) == 0 && i / 2 + FA < KK) fr[(i / 2 + FA) % (FA + 1)] = read_q(qp, i / 2 + FA);
        product(i);
#pragma unroll
        for (int k = NU * i / NS; k < NU * (i + 1) / NS; ++k) work(k);
        __builtin_amdgcn_sched_barrier(0);
      }
      colsum[0] += a0;
      colsum[1] += a1;
    } else {
      // the step crosses the sequence end or the diagonal
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        if ((i & 1) == 0 && i / 2 + FA < KK) fr[(i / 2 + FA) % (FA + 1)] = read_q(qp, i / 2 + FA);
        product(i);
      }
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        // rows below this lane's first visible one, and past the sequence, count nothing
        const int from = causal ? wk0 + 32 * kb + l32 - i0 - 4 * half : -64, to = n - i0 - 4 * half;
        float a = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int i = 8 * (r >> 2) + (r & 3);
          const float p = __builtin_amdgcn_exp2f(fmaf(s[kb][r], scale_log2, -lse2(r)));
          a += i >= from && i < to ? p : 0.f;
        }
        colsum[kb] += a;
      }
    }
  };
  int bc = 0, bn = 1, bf = 2;  // buffers of tiles t, t + 1, t + 2
  auto turn = [&]() {
    const int f = bc;
    bc = bn;
    bn = bf;
    bf = f;
  };
  int t = t0;
  turn_over();
  if (t0 + 2 < nt) load_tile(t0 + 2, bf);
  for (; t < tw && t + 1 < nt; ++t) {  // the tiles of the block's earlier keys
    turn();
    turn_over();
    if (t + 3 < nt) load_tile(t + 3, bf);
  }
  if (tw < nt) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const bf16x8_t a = read_q(smem + bc * BUF, kk);
      sa[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, kf[0][kk], kk == 0 ? zero : sa[0], 0, 0, 0);
      sa[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, kf[1][kk], kk == 0 ? zero : sa[1], 0, 0, 0);
    }
    while (true) {
      step(2 * t, bc, bc, 1, sa, sb);
      step(2 * t + 1, bc, bn, 0, sb, sa);
      if (++t >= nt) break;
      turn();
      turn_over();
      if (t + 2 < nt) load_tile(t + 2, bf);
    }
  }
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    const float v = half_swap_sum(colsum[kb]);
    const int j = wk0 + 32 * kb + l32;
    if (half == kb && j < n) partials[static_cast<int64_t>(h) * T + lo + j] = v;
  }
}

// fp32 storage (and bf16 at head dims 16 and 32), on
// v_mfma_f32_32x32x2_f32 with fp32 operands: one workgroup of four waves per
// (32 keys, query head, sequence). A wave keeps its keys' operand in
// registers and strides over the 32-query tiles; operands come straight
// from memory (the matrix instruction, at 64 cycles, is the slower side).
// One partial vector per head, as in the bf16 kernel. The exponentials are
// expf, as in the fp32 attention and for its reason. A vector-ALU kernel
// that summed all heads of a key in one thread held this place: 94 us on
// 4 x 64 rows, 4 heads of 32, and 1657 us on 8 ragged sequences of up
// to 200 rows, 12 heads of 64 (now 6.5 and 17.7 with the sum over heads).
template <typename T, int HD>
__global__ __launch_bounds__(256) void score_f32_kernel(const T* __restrict__ Q,
                                                        const T* __restrict__ K, int64_t rs,
                                                        const float* __restrict__ lse,
                                                        int kv_group, int causal, float scale,
                                                        const int32_t* __restrict__ cu, int Tn,
                                                        float* __restrict__ partials) {
  constexpr int NW = 4, KK = HD / 8;
  __shared__ float red[NW][32];
  const int b = blockIdx.z, h = blockIdx.y;
  const int lo = cu[b];
  const int n = cu[b + 1] - lo;
  const int j0 = blockIdx.x * 32;
  if (j0 >= n) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, l32 = lane & 31;
  const int j = j0 + l32;
  float4 kf[KK];
#pragma unroll
  for (int t = 0; t < KK; ++t)
    kf[t] = load4<T>(K + static_cast<int64_t>(lo + min(j, n - 1)) * rs + (h / kv_group) * HD + 8 * t + 4 * half);
  const float* lh = lse + static_cast<int64_t>(h) * Tn + lo;
  float colsum = 0.f;
  for (int i0 = (causal ? j0 : 0) + wave * 32; i0 < n; i0 += 32 * NW) {
    float L[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) L[r] = lh[min(i0 + 8 * (r >> 2) + 4 * half + (r & 3), n - 1)];
    const T* qp = Q + static_cast<int64_t>(lo + min(i0 + l32, n - 1)) * rs + h * HD + 4 * half;
    f32x16_t s = {};
#pragma unroll
    for (int t = 0; t < KK; ++t) {
      const float4 q4 = load4<T>(qp + 8 * t);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(q4.x, kf[t].x, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(q4.y, kf[t].y, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(q4.z, kf[t].z, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(q4.w, kf[t].w, s, 0, 0, 0);
    }
    // s[r]: query i0 + 8 (r/4) + 4 half + r%4, key j
    const bool edge = i0 + 32 > n || (causal && j0 + 31 > i0);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = i0 + 8 * (r >> 2) + 4 * half + (r & 3);
      const float p = expf(fmaf(s[r], scale, -L[r]));
      colsum += edge && (i >= n || (causal && j > i)) ? 0.f : p;
    }
  }
  colsum = half_swap_sum(colsum);
  if (half == 0) red[wave][l32] = colsum;
  __syncthreads();
  if (tid < 32 && j < n)
    partials[static_cast<int64_t>(h) * Tn + lo + j] = red[0][l32] + red[1][l32] + red[2][l32] + red[3][l32];
}

template <typename T>
hipError_t f32_dispatch(hipStream_t s, const void* q, const void* k, int64_t rs,
                        const float* lse, int H, int kvg, int hd, int causal, float scale, int B,
                        int max_len, int Trows, const int32_t* cu, float* partials) {
  const dim3 grid((max_len + 31) / 32, H, B), block(256);
  const T* qp = static_cast<const T*>(q);
  const T* kp = static_cast<const T*>(k);
  switch (hd) {
    case 16: return launch(K_SCORE, score_f32_kernel<T, 16>, grid, block, 0, s, qp, kp, rs, lse, kvg, causal, scale, cu, Trows, partials);
    case 32: return launch(K_SCORE, score_f32_kernel<T, 32>, grid, block, 0, s, qp, kp, rs, lse, kvg, causal, scale, cu, Trows, partials);
    case 64: return launch(K_SCORE, score_f32_kernel<T, 64>, grid, block, 0, s, qp, kp, rs, lse, kvg, causal, scale, cu, Trows, partials);
    case 128: return launch(K_SCORE, score_f32_kernel<T, 128>, grid, block, 0, s, qp, kp, rs, lse, kvg, causal, scale, cu, Trows, partials);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// Partial vectors per row: one per query head.
int score_groups(int dtype, int H, int hd, int T) {
  (void)dtype;
  (void)hd;
  (void)T;
  return H;
}

// The wide kernel from two of its workgroups per CU on (its comment), one at
// head dim 128 (4 x 500 causal rows, 32 heads: 32.1 -> 26.0 us). Past 1024 rows,
// where a workgroup takes long, those that hold keys count, of which a ragged
// batch's grid has fewer: about half a block a sequence more than its rows
// fill (3 sequences of up to 2344 causal rows, 20 heads of 64, 600
// workgroups in the grid, about 380 live: the other kernel 44.3, this one 48.7
// us; 8 of up to 2553, 4 heads of 128, 320 and 212: 42.7 and 58.0; but 8 of up to
// 500, 16 heads of 128, 256 and 208: 17.6 and 15.7). Long sequences under the
// mask need 1.6 per CU at head dim 128: the first keys' workgroups see every
// query and run about twice the mean, and below that the call waits for them
// alone (162 calls of 1100..4096 rows with one to two live per CU, 1.05 of the
// faster kernel's time with the line at 1.2, 1.01 at 1.6, 1.02 at 2; 2 of 4096, 12
// heads, ragged, 67.1 / 88.8; 6 of up to 3300, 6 heads, 52.8 / 74.7; above
// it 7 of up to 4096, 6 heads, 108 / 91). At any length: short sequences leave some of
// its waves without keys and are still faster on it (us with the sum over
// heads, the other kernel / this one: 32 heads of 64, no mask, 128 x 20 rows
// 34.5 / 25.1, 64 x 64 17.8 / 14.6, 64 x 128 21.7 / 20.9, 64 x 256 46.6 / 35.6;
// causal 64 x 64 19.2 / 13.2, 64 x 256 47.1 / 45.7, at worst 64 x 128 23.6 /
// 25.2; 32 heads of 128 on 8, 64 x 64 34.0 / 22.1, 64 x 128 causal 46.7 / 37.9).
bool score_wide(int hd, int H, int B, int max_len, int T, int causal, int cus) {
  int64_t blocks = (static_cast<int64_t>(max_len) + 255) / 256 * B;
  if (max_len > 1024 && static_cast<int64_t>(B) * max_len != T)
    blocks = std::min<int64_t>(blocks, std::max(B, T / 256 + B / 2));
  const int64_t five = hd == 64 ? 10 : causal && max_len > 1024 ? 8 : 5;  // fifths of a workgroup per CU
  return 5 * blocks * H >= five * cus;
}

hipError_t launch_score(hipStream_t s, int dtype, const void* q, const void* k,
                        int64_t row_stride, const float* lse, int H, int kv_group, int hd, int causal,
                        float scale, int B, int max_len, int T, const int32_t* cu_dev,
                        float* partials, int groups) {
  if (B == 0 || max_len == 0) return hipSuccess;
  if (groups != H) return hipErrorInvalidValue;
  if (dtype == 1 && (hd == 64 || hd == 128)) {
    const bf16_t* qp = static_cast<const bf16_t*>(q);
    const bf16_t* kp = static_cast<const bf16_t*>(k);
    const float sl = scale * kLog2e;
    const bool take = score_wide(hd, H, B, max_len, T, causal, device_cu_count());
    const PlaceGrid at = place_grid(H, kv_group, B, max_len, T, causal, take ? 256 : 128);
    auto go = [&](auto kernel, int threads) {
      return launch(K_SCORE, kernel, at.grid, dim3(threads), 0, s, qp, kp, row_stride, lse, H, kv_group, causal,
                    sl, cu_dev, T, partials, at.pairs);
    };
    if (take) return hd == 64 ? go(score_wide_kernel<64, 4>, 256) : go(score_wide_kernel<128, 4>, 256);
    return hd == 64 ? go(score_mfma_kernel<64, 128>, 64 * kScoreWaves)
                    : go(score_mfma_kernel<128, 128>, 64 * kScoreWaves);
  }
  if (dtype == 1)
    return f32_dispatch<bf16_t>(s, q, k, row_stride, lse, H, kv_group, hd, causal, scale, B,
                                max_len, T, cu_dev, partials);
  return f32_dispatch<float>(s, q, k, row_stride, lse, H, kv_group, hd, causal, scale, B, max_len,
                             T, cu_dev, partials);
}

}  // namespace zsa
