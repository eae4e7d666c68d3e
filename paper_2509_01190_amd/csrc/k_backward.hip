// Backward pass through the pruned block (the fine-tuning step of Eq. 3
// trains through the pruned forward; the kept rows are constants).
//
// Row-wise pieces: transposes of the weights (so a projection's input
// gradient runs on the forward's NT GEMM; its weight gradient is k_wgrad.hip),
// LayerNorm / RMSNorm backward with the gain and shift gradients, GELU /
// SwiGLU backward with the recomputed activation, the scatter that undoes
// compaction (dropped rows get zero gradient), the per-row dot
// D_i = dO_i . O_i, and the inverse rotary rotation.
//
// Attention backward (bf16, head_dim 64 / 128, MFMA), with P recomputed
// from the forward's log-sum-exp:
//     dV = P^T dO,  dP = dO V^T,  dS = P o (dP - D),  dK = scale dS^T Q,
//     dQ = scale dS K.
// attn_bwd_dkdv: one workgroup per (128-key block, key/value head,
// sequence), 32 keys per wave; the waves walk the query tiles together,
// compute S = Q K^T and dP = dO V^T in the layout where a lane owns one key,
// and multiply P and dS, packed as MFMA A operands, with the transposed
// tiles. Each key's dK / dV is summed by one wave in query order (no
// atomics). For grouped-query attention the workgroup also loops over the
// query heads that read its key/value head.
// attn_bwd_dq: one workgroup per (128-query block, head, sequence), laid out
// like the forward attention: S^T and dP^T with a lane owning one query, dS
// packed as the B operand of dQ^T += K^T dS^T.
// Both take tiles straight to LDS in rows, one tile ahead, and read them
// both ways: rows with 16-byte reads, and transposed with the transposing
// reads (bwd_swizzle serves the two without bank conflicts). Staged through
// registers into a row and a transposed copy, the transposition was most of
// the vector work. us, dK dV / dQ, before and now: 16 x 512 rows, 12 heads of
// 64, 78 / 43 and 42 / 27; 2 x 2048 causal, 32 heads of 64, 248 / 90 and 194 / 57;
// 2 x 2048 causal, 32 heads of 128 on 8 key/value heads, 695 / 535 (256
// workgroups, one per CU, whose waves wait for one another) and 395 / 135.
#include <math.h>

#include "zsa_internal.h"

namespace zsa {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ void load8(const bf16_t* p, float* v) {
  unpack16(*reinterpret_cast<const uint4*>(p), v, bf16_t());
}
__device__ __forceinline__ void store8(bf16_t* p, const float* v) {
  *reinterpret_cast<uint4*>(p) = pack16(v, bf16_t());
}

// ---------------------------------------------------------------------------
// out = in^T of the layer's weights, one launch for all of them: four
// launches of 4 to 5 us of which the launch itself is most (2.4 M weights of
// a 768-wide block)
// ---------------------------------------------------------------------------
struct TransposeArgs {
  TransposeArg m[4];
  int first[5];  // first tile of each matrix
};

// bf16, 64 x 64 tiles with 16-byte loads and stores (r and c multiples of 8)
__global__ __launch_bounds__(256) void transpose64_kernel(const TransposeArgs p) {
  __shared__ bf16_t tile[64][64 + 2];
  int i = 0;
  while (static_cast<int>(blockIdx.x) >= p.first[i + 1]) ++i;
  const bf16_t* __restrict__ in = static_cast<const bf16_t*>(p.m[i].in);
  bf16_t* __restrict__ out = static_cast<bf16_t*>(p.m[i].out);
  const int R = p.m[i].r, C = p.m[i].c, tc = (C + 63) / 64;
  const int id = static_cast<int>(blockIdx.x) - p.first[i];
  const int r0 = id / tc * 64, c0 = id % tc * 64;
  const int t = threadIdx.x;
  for (int k = t; k < 64 * 8; k += 256) {
    const int r = k / 8, ch = (k % 8) * 8;
    const int gr = r0 + r, gc = c0 + ch;
    if (gr < R && gc < C) {
      const uint4 v = *reinterpret_cast<const uint4*>(in + static_cast<int64_t>(gr) * C + gc);
      const bf16_t* e = reinterpret_cast<const bf16_t*>(&v);
#pragma unroll
      for (int j = 0; j < 8; ++j) tile[r][ch + j] = e[j];
    }
  }
  __syncthreads();
  for (int k = t; k < 64 * 8; k += 256) {
    const int c = k / 8, rh = (k % 8) * 8;   // output row c0 + c, columns r0 + rh ..
    const int gc = c0 + c, gr = r0 + rh;
    if (gc >= C || gr >= R) continue;
    uint4 v;
    bf16_t* e = reinterpret_cast<bf16_t*>(&v);
#pragma unroll
    for (int j = 0; j < 8; ++j) e[j] = tile[rh + j][c];
    *reinterpret_cast<uint4*>(out + static_cast<int64_t>(gc) * R + gr) = v;
  }
}

// ---------------------------------------------------------------------------
// norm backward: one wave per row, four past 2048 columns (WPR).
//   LN:  dx = rstd (g dh - mean(g dh) - xhat mean(g dh xhat))
//   RMS: dx = rstd (g dh - xhat mean(g dh xhat))
// out = res + dx (res may alias out, or be NULL). The gain and shift
// gradients, the column sums of dh xhat and dh, are summed on the way: each
// wave over its rows, a workgroup's waves in order into a row of `part`
// [blocks][(1 or 2) d], and col_total_kernel over the blocks. (As passes of
// their own they read dh twice and x once more: 40 us of five launches for
// 8192 rows of 768 where this takes two.)
// ---------------------------------------------------------------------------
constexpr int kNormBwdBlocks = 512;

template <int RMS, int NC, int WPR>
__global__ __launch_bounds__(256) void norm_bwd_kernel(const bf16_t* __restrict__ x,
                                                       const bf16_t* __restrict__ g,
                                                       const bf16_t* __restrict__ dh, const bf16_t* res,
                                                       bf16_t* out, int R, int d, float eps,
                                                       float* __restrict__ part) {
  // a wave of a row's WPR owns 8-column chunks lane, lane + 64 WPR, ... (NC of
  // them, d <= NC * WPR * 512); rows stay packed in registers across the
  // passes, chunks past d zero
  constexpr int NS = RMS ? 1 : 2, RPB = 4 / WPR;  // rows per workgroup and pass
  __shared__ float red[4][NS][512];
  __shared__ float wsum[4][4];  // a row's sums by wave: x, (x - mean)^2, g dh, g dh xhat
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int sub = WPR == 1 ? 0 : wave;
  auto col = [&](int k) { return ((k * WPR + sub) * 64 + lane) * 8; };
  // sums a wave's value over the row (all waves of a row get here together)
  auto row_sum = [&](float v, int slot, bool wait) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (WPR == 1) return v;
    if (lane == 0) wsum[slot][wave] = v;
    if (!wait) return 0.f;
    __syncthreads();
    return wsum[slot][0] + wsum[slot][1] + wsum[slot][2] + wsum[slot][3];
  };
  const u32x4 none = {0u, 0u, 0u, 0u};
  auto unpack = [](const u32x4& v, int e) {
    const uint32_t w = v[e >> 1];
    return __uint_as_float((e & 1) ? (w & 0xffff0000u) : (w << 16));
  };
  u32x4 gv[NC];
  float gs[NC][8], bs[NC][8];
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const int c = col(k);
    gv[k] = c < d ? *reinterpret_cast<const u32x4*>(g + c) : none;
#pragma unroll
    for (int e = 0; e < 8; ++e) gs[k][e] = bs[k][e] = 0.f;
  }
  // the next row's loads are in flight while this one is worked on
  u32x4 xn[NC], dn[NC];
  const int step = RPB * static_cast<int>(gridDim.x);
  auto fetch = [&](int row, u32x4* xr, u32x4* dr) {
    const int64_t base = static_cast<int64_t>(row) * d;
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const int c = col(k);
      xr[k] = c < d && row < R ? *reinterpret_cast<const u32x4*>(x + base + c) : none;
      dr[k] = c < d && row < R ? *reinterpret_cast<const u32x4*>(dh + base + c) : none;
    }
  };
  int row = static_cast<int>(blockIdx.x) * RPB + (WPR == 1 ? wave : 0);
  fetch(row, xn, dn);
  for (; row < R; row += step) {
    const int64_t base = static_cast<int64_t>(row) * d;
    u32x4 xv[NC], dv[NC];
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      xv[k] = xn[k];
      dv[k] = dn[k];
    }
    fetch(row < R - step ? row + step : R, xn, dn);
    float mean = 0.f;
    if (!RMS) {
#pragma unroll
      for (int k = 0; k < NC; ++k)
#pragma unroll
        for (int e = 0; e < 8; ++e) s += unpack(xv[k], e);
      mean = row_sum(s, 0, true) / d;
    }
    float ss = 0.f;
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      if (col(k) < d) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float v = unpack(xv[k], e) - mean;
          ss += v * v;
        }
      }
    }
    ss = row_sum(ss, 1, true);
    const float rstd = 1.0f / sqrtf(ss / d + eps);
    float s1 = 0.f, s2 = 0.f;  // sum(g dh), sum(g dh xhat)
#pragma unroll
    for (int k = 0; k < NC; ++k)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float h = unpack(dv[k], e), gd = h * unpack(gv[k], e), xh = (unpack(xv[k], e) - mean) * rstd;
        s1 += gd;
        s2 += gd * xh;  // zero on chunks past d
        gs[k][e] += h * xh;
        if (!RMS) bs[k][e] += h;
      }
    s1 = row_sum(s1, 2, false);
    s2 = row_sum(s2, 3, true);
    if (WPR > 1) s1 = wsum[2][0] + wsum[2][1] + wsum[2][2] + wsum[2][3];
    const float m1 = RMS ? 0.f : s1 / d, m2 = s2 / d;
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const int c = col(k);
      if (c < d) {
        float o[8], rv[8];
        if (res != nullptr) load8(res + base + c, rv);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float xh = (unpack(xv[k], e) - mean) * rstd;
          o[e] = rstd * (unpack(dv[k], e) * unpack(gv[k], e) - m1 - xh * m2) + (res != nullptr ? rv[e] : 0.f);
        }
        store8(out + base + c, o);
      }
    }
  }
  float* prow = part + static_cast<int64_t>(blockIdx.x) * NS * d;
  if constexpr (WPR > 1) {
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const int c = col(k);
      if (c >= d) continue;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        prow[c + e] = gs[k][e];
        if (!RMS) prow[d + c + e] = bs[k][e];
      }
    }
    return;
  }
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    if (k > 0) __syncthreads();
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      red[wave][0][lane * 8 + e] = gs[k][e];
      if (!RMS) red[wave][NS - 1][lane * 8 + e] = bs[k][e];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < NS * 512; i += 256) {
      const int which = i >> 9, j = i & 511, c = k * 512 + j;
      if (c < d) prow[which * d + c] = red[0][which][j] + red[1][which][j] + red[2][which][j] + red[3][which][j];
    }
  }
}

// out0[c] (c < d) and out1[c - d] = the sum of column c of part [rows][cols]:
// 32 columns and 32 row lanes a workgroup, added in a fixed order, the lanes in
// pairs (8192 positive rows: 3.4e-8 off; one lane after another 8.8e-8)
__global__ __launch_bounds__(256) void col_total_kernel(const float* __restrict__ part, int rows, int cols,
                                                        int d, float* __restrict__ out0,
                                                        float* __restrict__ out1) {
  __shared__ float red[32][33];
  const int q = threadIdx.x & 7, rl = threadIdx.x >> 3;
  const int c0 = blockIdx.x * 32, c = c0 + 4 * q;
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (c < cols) {  // a multiple of 8
#pragma unroll 8
    for (int r = rl; r < rows; r += 32) {
      const float4 t = *reinterpret_cast<const float4*>(part + static_cast<int64_t>(r) * cols + c);
      v.x += t.x;
      v.y += t.y;
      v.z += t.z;
      v.w += t.w;
    }
  }
  red[rl][4 * q] = v.x;
  red[rl][4 * q + 1] = v.y;
  red[rl][4 * q + 2] = v.z;
  red[rl][4 * q + 3] = v.w;
  __syncthreads();
  const int oc = c0 + static_cast<int>(threadIdx.x);
  if (threadIdx.x < 32 && oc < cols) {
    const float s = lane_rows_total(red, threadIdx.x);
    if (oc < d) out0[oc] = s;
    else if (out1 != nullptr) out1[oc - d] = s;
  }
}

// ---------------------------------------------------------------------------
// activation backward. GELU: du = dF (Phi(u) + u phi(u)). SwiGLU on
// interleaved columns (2f gate, 2f+1 up): dgate = dF up silu'(gate),
// dup = dF silu(gate), silu'(z) = s (1 + z (1 - s)), s = sigmoid(z).
// ---------------------------------------------------------------------------
// The activation f itself (recomputed for the down projection's weight
// gradient) comes from the same read of u: a pass of its own took 11.4 us for
// 4096 rows of 3072 beside this one's 15.2.
__global__ __launch_bounds__(256) void act_bwd_kernel(const bf16_t* __restrict__ dF,
                                                      const bf16_t* __restrict__ u, bf16_t* __restrict__ du,
                                                      bf16_t* __restrict__ fo, int64_t rows, int F,
                                                      int swiglu) {
  // 8 consecutive outputs f..f+7 of one row per thread
  const int64_t i = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) * 8;
  if (i >= rows * F) return;
  const int64_t r = i / F;
  const int f = static_cast<int>(i - r * F);
  float g[8], a[8];
  load8(dF + i, g);
  if (swiglu) {
    float u0[8], u1[8], o0[8], o1[8];
    load8(u + r * 2 * F + 2 * f, u0);       // gate, up of outputs f .. f+3
    load8(u + r * 2 * F + 2 * f + 8, u1);   // ... of f+4 .. f+7
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float z0 = u0[2 * e], up0 = u0[2 * e + 1], e0 = 1.0f + expf(-z0), s0 = 1.0f / e0;
      const float z1 = u1[2 * e], up1 = u1[2 * e + 1], e1 = 1.0f + expf(-z1), s1 = 1.0f / e1;
      o0[2 * e] = g[e] * up0 * s0 * (1.0f + z0 * (1.0f - s0));
      o0[2 * e + 1] = g[e] * z0 * s0;
      o1[2 * e] = g[4 + e] * up1 * s1 * (1.0f + z1 * (1.0f - s1));
      o1[2 * e + 1] = g[4 + e] * z1 * s1;
      a[e] = z0 / e0 * up0;
      a[4 + e] = z1 / e1 * up1;
    }
    store8(du + r * 2 * F + 2 * f, o0);
    store8(du + r * 2 * F + 2 * f + 8, o1);
  } else {
    float z[8], o[8];
    load8(u + i, z);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float cdf = 0.5f * (1.0f + erff(z[e] * 0.70710678118654752f));
      const float pdf = 0.39894228040143268f * __expf(-0.5f * z[e] * z[e]);
      o[e] = g[e] * (cdf + z[e] * pdf);
      a[e] = z[e] * cdf;
    }
    store8(du + i, o);
  }
  store8(fo + i, a);
}

// ---------------------------------------------------------------------------
// undo compaction of two arrays: dst[kept[i]] = src[i], zeros elsewhere. A wave
// takes a row of dst and looks it up in kept, which ascends, 64 entries at a
// time (two steps up to 4096 kept rows). An inverse index (filled, then
// written, then read by one scatter per array) took six launches, 21 us for
// 8192 rows of 768; this one 8. (A wave per kept row that also clears the
// dropped rows before it was as fast there, but 97 us a layer where long runs
// of rows are dropped.)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void scatter_rows_kernel(const u32x4* __restrict__ src0, u32x4* __restrict__ dst0,
                                                           const u32x4* __restrict__ src1, u32x4* __restrict__ dst1,
                                                           const int32_t* __restrict__ kept, int t_out, int t_in,
                                                           int cpr) {
  const int lane = threadIdx.x & 63;
  const int r = __builtin_amdgcn_readfirstlane(static_cast<int>(blockIdx.x) * 4 + static_cast<int>(threadIdx.x >> 6));
  if (r >= t_in) return;
  int lo = 0, len = t_out;
  while (len > 64) {
    const int stride = (len + 63) / 64;
    const int64_t i = static_cast<int64_t>(lane + 1) * stride - 1;
    const bool below = i < len && kept[lo + i] < r;
    const int c = __popcll(__builtin_amdgcn_ballot_w64(below));
    lo += c * stride;
    len = min(stride, len - c * stride);
  }
  const uint64_t hit = __builtin_amdgcn_ballot_w64(lane < len && kept[lo + min(lane, max(len - 1, 0))] == r);
  const int64_t at = hit != 0 ? static_cast<int64_t>(lo + __builtin_ctzll(hit)) * cpr : -1;
  const int64_t to = static_cast<int64_t>(r) * cpr;
  const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll 2
  for (int c = lane; c < cpr; c += 64) {
    dst0[to + c] = at >= 0 ? src0[at + c] : zero;
    dst1[to + c] = at >= 0 ? src1[at + c] : zero;
  }
}

// LD[h][r] = (lse[h][r] log2 e, D) with D = sum_c dO[r][h hd + c] O[r][h hd +
// c]: each thread takes 8 consecutive columns, the L = hd / 8 threads of one
// head (L a power of two up to 64, adjacent lanes of one wave) add theirs in a
// fixed butterfly
__global__ __launch_bounds__(256) void rowdot_kernel(const bf16_t* __restrict__ dO,
                                                     const bf16_t* __restrict__ O, int64_t ld, int T_,
                                                     int H, int hd, const float* __restrict__ lse,
                                                     float2* __restrict__ LD) {
  const int L = hd / 8, per_row = H * L;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const bool live = i < static_cast<int64_t>(T_) * per_row;
  const int r = live ? static_cast<int>(i / per_row) : 0;
  const int c8 = live ? static_cast<int>(i - static_cast<int64_t>(r) * per_row) : 0;
  float s = 0.f;
  if (live) {
    float va[8], vb[8];
    load8(dO + static_cast<int64_t>(r) * ld + c8 * 8, va);
    load8(O + static_cast<int64_t>(r) * ld + c8 * 8, vb);
#pragma unroll
    for (int e = 0; e < 8; ++e) s = fmaf(va[e], vb[e], s);
  }
  // groups of L lanes start at multiples of L within the wave (64 % L == 0
  // and each block is 256 threads), so the butterfly stays inside one head
  for (int o = 1; o < L; o <<= 1) s += __shfl_xor(s, o, 64);
  if (live && (c8 & (L - 1)) == 0) {
    const int64_t at = static_cast<int64_t>(c8 / L) * T_ + r;
    LD[at] = make_float2(lse[at] * kLog2e, s);
  }
}

// inverse rotary rotation of the gradient, in place, on the first `cols`
// columns (whole heads) of rows of a [rows, ld] array
__global__ __launch_bounds__(256) void rope_bwd_kernel(bf16_t* __restrict__ g, int64_t ld, int rows,
                                                       int cols, int hd,
                                                       const int32_t* __restrict__ pos,
                                                       EpiParams ep) {
  const int half = hd / 2;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int pairs = cols / 2;
  if (i >= static_cast<int64_t>(rows) * pairs) return;
  const int r = static_cast<int>(i / pairs);
  const int pr = static_cast<int>(i % pairs);
  const int head = pr / half, k = pr % half;
  const int64_t a = static_cast<int64_t>(r) * ld + head * hd + k;
  float sn, cs;
  rope_angle(pos[r], ep.inv_freq[k], &sn, &cs);
  const float x = to_f32(g[a]), y = to_f32(g[a + half]);
  g[a] = f32_to_bf16(x * cs + y * sn);
  g[a + half] = f32_to_bf16(y * cs - x * sn);
}

// ---------------------------------------------------------------------------
// attention backward
// ---------------------------------------------------------------------------
// Tile row r keeps its 16-byte chunk c at c ^ swizzle(r). The 16 rows of a
// row read's phase fall on all 64 banks, and so do the four rows r .. r + 3
// (r a multiple of four) by four chunks of a transposing read's.
template <int HD>
__device__ __forceinline__ constexpr int bwd_swizzle(int r) {
  return HD == 64 ? ((r >> 1) & 1) << 2 | ((r >> 2) & 1) << 1 | ((r >> 3) & 1) : (r & 3) << 2 | ((r >> 2) & 3);
}

// The reading side of a tile of HD-wide rows: a lane's offsets of the row
// fragment of channels 16 kk .. (row l32, channels 16 kk + 8 half + 0 .. 7)
// and of the transposed fragment of channels 32 ct .. (channel 32 ct + l32,
// rows 4 half + 0 .. 3 and these + 8)
template <int HD>
struct TileReads {
  static constexpr int RB = HD * 2, KK = HD / 16, CT = HD / 32;
  uint32_t row[KK], lo[CT], hi[CT];
  __device__ __forceinline__ explicit TileReads(int lane) {
    const int half = lane >> 5, l32 = lane & 31;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) row[kk] = l32 * RB + (((2 * kk + half) ^ bwd_swizzle<HD>(l32)) << 4);
    const int r = 4 * half + ((lane & 15) >> 2), ch = 2 * ((lane >> 4) & 1) + ((lane >> 1) & 1);
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      lo[ct] = r * RB + (((4 * ct + ch) ^ bwd_swizzle<HD>(r)) << 4) + (lane & 1) * 8;
      hi[ct] = (r + 8) * RB + (((4 * ct + ch) ^ bwd_swizzle<HD>(r + 8)) << 4) + (lane & 1) * 8;
    }
  }
  __device__ __forceinline__ bf16x8_t rows(const unsigned char* tile, int kk) const {
    return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(tile + row[kk]));
  }
  // tile rows 16 g + ...
  __device__ __forceinline__ bf16x8_t cols(const unsigned char* tile, int g, int ct) const {
    return __builtin_bit_cast(bf16x8_t, lds_read_columns(tile + lo[ct] + g * (16 * RB), tile + hi[ct] + g * (16 * RB)));
  }
};

__device__ __forceinline__ bf16x8_t pack_slots(const f32x16_t& v, int g) {
  const int r = 8 * g;
  const u32x4 w = {pack_bf16x2(v[r], v[r + 1]), pack_bf16x2(v[r + 2], v[r + 3]), pack_bf16x2(v[r + 4], v[r + 5]),
                   pack_bf16x2(v[r + 6], v[r + 7])};
  return __builtin_bit_cast(bf16x8_t, w);
}

// Rows per tile: 64 at head dim 64, 32 at 128 (8 KB an operand either way),
// two tiles in LDS.
template <int HD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 4))) void attn_bwd_dkdv_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    int64_t rs, const bf16_t* __restrict__ dO, int64_t ors, const float2* __restrict__ LD, int T,
    int Hkv, int kv_group, int causal, float scale, float scale_log2, const int32_t* __restrict__ cu,
    bf16_t* __restrict__ dK, bf16_t* __restrict__ dV, int64_t grs, int pairs) {
  constexpr int KW = 128, QT = HD == 64 ? 64 : 32;
  constexpr int KK = HD / 16, CT = HD / 32, CPR = HD / 8, RB = HD * 2, OLD = HD + 8;
  constexpr int TB = QT * RB, BUF = 2 * TB + 1024;  // Q, dO, (lse, D) pairs
  constexpr int RPL = 1024 / RB, LPW = TB / 4096;   // rows per load, loads per wave and operand
  constexpr int SBYTES = 2 * BUF > 8 * 32 * OLD * 2 ? 2 * BUF : 8 * 32 * OLD * 2;
  static_assert(LPW * 4096 == TB, "tile split");
  __shared__ __align__(1024) unsigned char smem[SBYTES];

  Place at;
  if (!place(Hkv, 1, pairs, true, &at)) return;
  const int b = at.b, g = at.h;
  const int lo = cu[b];
  const int n = cu[b + 1] - lo;
  const int j0 = at.i * KW;
  if (j0 >= n) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, l32 = lane & 31;
  const int jw = j0 + wave * 32;  // the wave's first key

  const uint32_t q_row = static_cast<uint32_t>(rs * 2), o_row = static_cast<uint32_t>(ors * 2);
  const int lrow = wave * RPL + lane / CPR;  // tile row of the wave's first load
  const uint32_t lchunk = ((lane % CPR) ^ bwd_swizzle<HD>(lrow)) << 4;
  const uint32_t qoff = lrow * q_row + lchunk, ooff = lrow * o_row + lchunk;
  const uint32_t lds0 = lds_address(smem);
  // queries before the first key see none of the keys (causal)
  const int qs = causal ? j0 : 0;
  const int ntile = (n - qs + QT - 1) / QT;
  const int rounds = ntile * kv_group;
  // rows past the sequence read as zeros (masked)
  auto load_tile = [&](int t, int buf) {
    const int e = t / ntile, i0 = qs + (t - e * ntile) * QT, h = g * kv_group + e;
    const u32x4 qres = buffer_resource(Q + static_cast<int64_t>(lo) * rs + h * HD, static_cast<uint32_t>(n) * q_row);
    const u32x4 ores = buffer_resource(dO + static_cast<int64_t>(lo) * ors + h * HD, static_cast<uint32_t>(n) * o_row);
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      const uint32_t d = lds0 + buf * BUF + wave * 1024 + i * 4096;
      lds_load16(d, qoff + static_cast<uint32_t>(i0 + i * 4 * RPL) * q_row, qres);
      lds_load16(d + TB, ooff + static_cast<uint32_t>(i0 + i * 4 * RPL) * o_row, ores);
    }
    if (wave < QT / 32) {
      const u32x4 lres = buffer_resource(LD + static_cast<int64_t>(h) * T + lo, static_cast<uint32_t>(n) * 8u);
      lds_load4(lds0 + buf * BUF + 2 * TB + wave * 256, static_cast<uint32_t>(i0) * 8u + (wave * 64 + lane) * 4u, lres);
    }
  };
  load_tile(0, 0);

  bf16x8_t kf[KK], vf[KK];
  {
    // keys past the sequence repeat its last row; they are not written
    const int64_t at_row = static_cast<int64_t>(lo + min(jw + l32, n - 1)) * rs + g * HD + half * 8;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      kf[kk] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(K + at_row + kk * 16));
      vf[kk] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(V + at_row + kk * 16));
    }
  }
  f32x16_t dk[CT] = {}, dv[CT] = {};
  const TileReads<HD> rd(lane);
  const f32x16_t zero = {};
  for (int t = 0; t < rounds; ++t) {
    turn_over();
    if (t + 1 < rounds) load_tile(t + 1, (t + 1) & 1);
    const int i_tile = qs + (t % ntile) * QT;
    const unsigned char* tq = smem + (t & 1) * BUF;
#pragma unroll 1
    for (int u = 0; u < QT / 32; ++u) {
      const int i0 = i_tile + 32 * u;
      // steps past the sequence, and a wave whose keys all lie past the sequence or the step's last query
      if (i0 >= n || jw >= n || (causal && jw > i0 + 31)) continue;
      const unsigned char *uq = tq + u * (32 * RB), *ud = uq + TB;
      const float4* lp = reinterpret_cast<const float4*>(tq + 2 * TB) + 16 * u + 2 * half;
      f32x16_t s, dp;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rd.rows(uq, kk), kf[kk], kk == 0 ? zero : s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rd.rows(ud, kk), vf[kk], kk == 0 ? zero : dp, 0, 0, 0);
      }
      // s[r], dp[r]: query i0 + 8 (r/4) + 4 half + r%4, key jw + l32
#pragma unroll
      for (int a = 0; a < 8; ++a) {
        const float4 w = lp[4 * (a >> 1) + (a & 1)];  // (lse, D) of queries 8 (a/2) + 4 half + 2 (a%2) and the next
        const int r = 2 * a;
        s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], scale_log2, -w.x));
        s[r + 1] = __builtin_amdgcn_exp2f(fmaf(s[r + 1], scale_log2, -w.z));
        dp[r] -= w.y;
        dp[r + 1] -= w.w;
      }
      if (i0 + 32 > n || (causal && jw + 31 > i0)) {
        // queries from first on (and before n) see the key
        const int first = (causal ? jw + l32 : 0) - i0 - 4 * half, last = n - i0 - 4 * half;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int q = 8 * (r >> 2) + (r & 3);
          if (q < first || q >= last) s[r] = 0.f;
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) dp[r] *= s[r];
#pragma unroll
      for (int gg = 0; gg < 2; ++gg) {
        const bf16x8_t pa = pack_slots(s, gg), sa = pack_slots(dp, gg);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          dv[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pa, rd.cols(ud, gg, ct), dv[ct], 0, 0, 0);
          dk[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sa, rd.cols(uq, gg, ct), dk[ct], 0, 0, 0);
        }
      }
    }
  }
  __syncthreads();
  // acc[ct][r]: key jw + 8 (r/4) + 4 half + r%4, channel ct*32 + l32; staged
  // as bf16 rows in LDS (the wave's own region), then written 16 bytes a lane
  bf16_t* ov = reinterpret_cast<bf16_t*>(smem) + wave * 2 * 32 * OLD;
  bf16_t* ok = ov + 32 * OLD;
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = 8 * (r >> 2) + 4 * half + (r & 3);
      ov[key * OLD + ct * 32 + l32] = f32_to_bf16(dv[ct][r]);
      ok[key * OLD + ct * 32 + l32] = f32_to_bf16(dk[ct][r] * scale);
    }
  __syncthreads();
  for (int c = lane; c < 32 * CPR; c += 64) {
    const int key = c / CPR, ch = (c % CPR) * 8;
    if (jw + key >= n) continue;
    const int64_t o = static_cast<int64_t>(lo + jw + key) * grs + g * HD + ch;
    *reinterpret_cast<u32x4*>(dV + o) = *reinterpret_cast<const u32x4*>(ov + key * OLD + ch);
    *reinterpret_cast<u32x4*>(dK + o) = *reinterpret_cast<const u32x4*>(ok + key * OLD + ch);
  }
}

template <int HD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 4))) void attn_bwd_dq_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    int64_t rs, const bf16_t* __restrict__ dO, int64_t ors, const float2* __restrict__ LD, int T, int H,
    int kv_group, int causal, float scale, float scale_log2, const int32_t* __restrict__ cu,
    bf16_t* __restrict__ dQ, int64_t grs, int pairs) {
  constexpr int BQ = 128, KT = HD == 64 ? 64 : 32;
  constexpr int KK = HD / 16, CT = HD / 32, CPR = HD / 8, RB = HD * 2, OLD = HD + 8;
  constexpr int TB = KT * RB, BUF = 2 * TB;        // K, V
  constexpr int RPL = 1024 / RB, LPW = TB / 4096;  // rows per load, loads per wave and operand
  constexpr int SBYTES = 2 * BUF > 4 * 32 * OLD * 2 ? 2 * BUF : 4 * 32 * OLD * 2;
  static_assert(LPW * 4096 == TB, "tile split");
  __shared__ __align__(1024) unsigned char smem[SBYTES];

  Place at;
  if (!place(H, kv_group, pairs, false, &at)) return;
  const int b = at.b, h = at.h;
  const int lo = cu[b];
  const int n = cu[b + 1] - lo;
  const int q0 = at.i * BQ;
  if (q0 >= n) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, l32 = lane & 31;
  const int wq0 = q0 + wave * 32, hk = h / kv_group;

  const uint32_t row_bytes = static_cast<uint32_t>(rs * 2);
  const int lrow = wave * RPL + lane / CPR;  // tile row of the wave's first load
  const uint32_t off = lrow * row_bytes + (((lane % CPR) ^ bwd_swizzle<HD>(lrow)) << 4);
  const uint32_t lds0 = lds_address(smem) + wave * 1024;
  // keys past the sequence read as zeros (masked)
  const u32x4 kres = buffer_resource(K + static_cast<int64_t>(lo) * rs + hk * HD, static_cast<uint32_t>(n) * row_bytes);
  const u32x4 vres = buffer_resource(V + static_cast<int64_t>(lo) * rs + hk * HD, static_cast<uint32_t>(n) * row_bytes);
  auto load_tile = [&](int t, int buf) {
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      const uint32_t d = lds0 + buf * BUF + i * 4096, o = off + static_cast<uint32_t>(t * KT + i * 4 * RPL) * row_bytes;
      lds_load16(d, o, kres);
      lds_load16(d + TB, o, vres);
    }
  };
  load_tile(0, 0);

  // queries past the sequence repeat its last row; they are not written
  const int64_t qr = lo + min(wq0 + l32, n - 1);
  bf16x8_t qf[KK], df[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    qf[kk] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(Q + qr * rs + h * HD + kk * 16 + half * 8));
    df[kk] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(dO + qr * ors + h * HD + kk * 16 + half * 8));
  }
  const float2 ld = LD[static_cast<int64_t>(h) * T + qr];
  f32x16_t acc[CT] = {};
  const TileReads<HD> rd(lane);
  const f32x16_t zero = {};
  const int kend = causal ? min(n, q0 + BQ) : n;
  const int nt = (kend + KT - 1) / KT;
  for (int t = 0; t < nt; ++t) {
    turn_over();
    if (t + 1 < nt) load_tile(t + 1, (t + 1) & 1);
    const unsigned char* tk = smem + (t & 1) * BUF;
#pragma unroll 1
    for (int u = 0; u < KT / 32; ++u) {
      const int j0 = t * KT + 32 * u;
      // steps past the sequence, and under the causal mask past the wave's last query
      if (j0 >= n || (causal && j0 > wq0 + 31)) continue;
      const unsigned char *uk = tk + u * (32 * RB), *uv = uk + TB;
      f32x16_t s, dp;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rd.rows(uk, kk), qf[kk], kk == 0 ? zero : s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rd.rows(uv, kk), df[kk], kk == 0 ? zero : dp, 0, 0, 0);
      }
      // s[r], dp[r]: key j0 + 8 (r/4) + 4 half + r%4, query wq0 + l32
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], scale_log2, -ld.x));
      if (j0 + 32 > n || (causal && j0 + 31 > wq0)) {
        // keys from this lane's limit on are masked
        const int lim = (causal ? min(n, wq0 + l32 + 1) : n) - j0 - 4 * half;
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (8 * (r >> 2) + (r & 3) >= lim) s[r] = 0.f;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] *= dp[r] - ld.y;  // dS
#pragma unroll
      for (int gg = 0; gg < 2; ++gg) {
        const bf16x8_t sb = pack_slots(s, gg);
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
          acc[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rd.cols(uk, gg, ct), sb, acc[ct], 0, 0, 0);
      }
    }
  }
  // acc[ct][r] = dQ^T[channel ct*32 + 8 (r/4) + 4 half + r%4][query wq0 + l32] / scale
  __syncthreads();
  bf16_t* Os = reinterpret_cast<bf16_t*>(smem) + wave * 32 * OLD;
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int r = 0; r < 16; r += 4) {
      const uint2 w = {pack_bf16x2(acc[ct][r] * scale, acc[ct][r + 1] * scale),
                       pack_bf16x2(acc[ct][r + 2] * scale, acc[ct][r + 3] * scale)};
      *reinterpret_cast<uint2*>(Os + l32 * OLD + ct * 32 + 2 * r + 4 * half) = w;
    }
  __syncthreads();
  for (int c = lane; c < 32 * CPR; c += 64) {
    const int r = c / CPR, ch = (c % CPR) * 8;
    const int q = wq0 + r;
    if (q < n)
      *reinterpret_cast<u32x4*>(dQ + static_cast<int64_t>(lo + q) * grs + h * HD + ch) =
          *reinterpret_cast<const u32x4*>(Os + r * OLD + ch);
  }
}

}  // namespace

bool backward_supported(int dtype, int hd) { return dtype == 1 && (hd == 64 || hd == 128); }

hipError_t launch_transposes(hipStream_t s, const TransposeArg* m, int count) {
  if (count < 1 || count > 4) return hipErrorInvalidValue;
  TransposeArgs p;
  int total = 0;
  for (int i = 0; i < 4; ++i) {
    p.m[i] = m[std::min(i, count - 1)];
    p.first[i] = total;
    if (i >= count) continue;
    if (m[i].r % 8 != 0 || m[i].c % 8 != 0) return hipErrorInvalidValue;
    total += ((m[i].r + 63) / 64) * ((m[i].c + 63) / 64);
  }
  p.first[4] = total;
  if (total == 0) return hipSuccess;
  return launch(K_MISC, transpose64_kernel, dim3(total), dim3(256), 0, s, p);
}

static int norm_bwd_blocks(int R) { return std::max(1, std::min((R + 7) / 8, kNormBwdBlocks)); }

size_t norm_bwd_scratch_floats(int R, int d) { return static_cast<size_t>(norm_bwd_blocks(R)) * 2 * d; }

hipError_t launch_norm_bwd(hipStream_t s, int kind, const void* x, const void* g, const void* dh,
                           const void* res, void* out, int R, int d, float eps, float* scratch,
                           float* dg, float* db) {
  if (d % 8 != 0 || d > 16 * 512) return hipErrorInvalidValue;
  const int blocks = norm_bwd_blocks(R), cols = kind == 1 ? d : 2 * d, nc = (d + 511) / 512;
  auto go = [&](auto rms, auto layer) {
    return launch(K_NORM, kind == 1 ? rms : layer, dim3(blocks), dim3(256), 0, s,
                  static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(g),
                  static_cast<const bf16_t*>(dh), static_cast<const bf16_t*>(res),
                  static_cast<bf16_t*>(out), R, d, eps, scratch);
  };
  const hipError_t e = nc <= 1   ? go(norm_bwd_kernel<1, 1, 1>, norm_bwd_kernel<0, 1, 1>)
                       : nc <= 2 ? go(norm_bwd_kernel<1, 2, 1>, norm_bwd_kernel<0, 2, 1>)
                       : nc <= 4 ? go(norm_bwd_kernel<1, 4, 1>, norm_bwd_kernel<0, 4, 1>)
                       : nc <= 8 ? go(norm_bwd_kernel<1, 2, 4>, norm_bwd_kernel<0, 2, 4>)
                                 : go(norm_bwd_kernel<1, 4, 4>, norm_bwd_kernel<0, 4, 4>);
  if (e != hipSuccess) return e;
  return launch(K_NORM, col_total_kernel, dim3((cols + 31) / 32), dim3(256), 0, s,
                static_cast<const float*>(scratch), blocks, cols, d, dg, db);
}

hipError_t launch_act_bwd(hipStream_t s, const void* dF, const void* u, void* du, void* f, int rows,
                          int F, int swiglu) {
  const int64_t total = static_cast<int64_t>(rows) * F;
  if (total == 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>((total / 8 + 255) / 256));  // F % 8 == 0
  return launch(K_MISC, act_bwd_kernel, grid, dim3(256), 0, s, static_cast<const bf16_t*>(dF),
                static_cast<const bf16_t*>(u), static_cast<bf16_t*>(du), static_cast<bf16_t*>(f),
                static_cast<int64_t>(rows), F, swiglu);
}

hipError_t launch_scatter_rows(hipStream_t s, int d, const void* src0, void* dst0, const void* src1,
                               void* dst1, const int32_t* kept, int t_out, int t_in) {
  if (t_in == 0) return hipSuccess;
  return launch(K_MISC, scatter_rows_kernel, dim3((t_in + 3) / 4), dim3(256), 0, s,
                static_cast<const u32x4*>(src0), static_cast<u32x4*>(dst0),
                static_cast<const u32x4*>(src1), static_cast<u32x4*>(dst1), kept, t_out, t_in,
                d * 2 / 16);
}

hipError_t launch_rowdot(hipStream_t s, const void* dO, const void* O, int64_t ld, int T, int H,
                         int hd, const float* lse, float* LD) {
  const int L = hd / 8;
  if (hd % 8 != 0 || L > 64 || (L & (L - 1)) != 0) return hipErrorInvalidValue;
  const int64_t total = static_cast<int64_t>(T) * H * L;
  if (total == 0) return hipSuccess;
  return launch(K_MISC, rowdot_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, s,
                static_cast<const bf16_t*>(dO), static_cast<const bf16_t*>(O), ld, T, H, hd, lse,
                reinterpret_cast<float2*>(LD));
}

hipError_t launch_rope_bwd(hipStream_t s, int dtype, void* g, int64_t ld, int rows, int cols,
                           int hd, const int32_t* pos, const EpiParams& ep) {
  const int64_t total = static_cast<int64_t>(rows) * (cols / 2);
  if (total == 0) return hipSuccess;
  if (dtype != 1) return hipErrorInvalidValue;
  return launch(K_MISC, rope_bwd_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0, s,
                static_cast<bf16_t*>(g), ld, rows, cols, hd, pos, ep);
}

hipError_t launch_attention_bwd(hipStream_t s, const void* q, const void* k, const void* v,
                                int64_t rs, const void* dO, int64_t ors, const float* LD, int H,
                                int kv_group, int hd, int causal, float scale, int B, int max_len,
                                int T, const int32_t* cu_dev, void* dq, void* dk, void* dv,
                                int64_t grs) {
  if (B == 0 || max_len == 0) return hipSuccess;
  const int Hkv = H / kv_group;
  auto go = [&](auto dkdv, auto dq_kernel) {
    const float sl = scale * kLog2e;
    auto* qp = static_cast<const bf16_t*>(q);
    auto* kp = static_cast<const bf16_t*>(k);
    auto* vp = static_cast<const bf16_t*>(v);
    auto* op = static_cast<const bf16_t*>(dO);
    auto* lp = reinterpret_cast<const float2*>(LD);
    // (a key/value head's queries are one workgroup's in dkdv: nothing is shared between its pairs)
    const PlaceGrid ak = place_grid(Hkv, 1, B, max_len, T, causal, 128), aq = place_grid(H, kv_group, B, max_len, T, causal, 128);
    const hipError_t e = launch(K_ATTENTION, dkdv, ak.grid, dim3(256), 0, s, qp,
                                kp, vp, rs, op, ors, lp, T, Hkv, kv_group, causal, scale, sl, cu_dev,
                                static_cast<bf16_t*>(dk), static_cast<bf16_t*>(dv), grs, ak.pairs);
    if (e != hipSuccess) return e;
    return launch(K_ATTENTION, dq_kernel, aq.grid, dim3(256), 0, s, qp, kp, vp, rs,
                  op, ors, lp, T, H, kv_group, causal, scale, sl, cu_dev, static_cast<bf16_t*>(dq), grs, aq.pairs);
  };
  return hd == 64 ? go(attn_bwd_dkdv_kernel<64>, attn_bwd_dq_kernel<64>)
                  : go(attn_bwd_dkdv_kernel<128>, attn_bwd_dq_kernel<128>);
}

}  // namespace zsa
