// Weight and bias gradients of a projection y = x W^T + b (bf16 rows, fp32
// gradients): dW = dY^T X, the contraction running over the rows, and db the
// column sums of dY.
//
// Both operands are read as they lie, [rows, columns]: slices of rows go
// straight to LDS (buffer loads with the LDS destination) and the matrix
// fragments, which want eight consecutive rows of a column per lane, come
// from the transposing LDS reads. The two operands are read with the same
// row order within a fragment, which leaves the contraction unchanged. The
// kernel this replaces wanted the rows consecutive in memory, so each
// product first transposed both operands.
//
// db is summed from the same fragments, each (column tile of X, wave column)
// taking the slices that are its turn, so that the additions are spread over
// the workgroups of a row of tiles. They are added in levels (pairs of a
// fragment, a slice, a wave's slices, waves and splits in pairs): in one chain
// per wave and then over the waves, 4096 positive rows of 768 columns were off
// by 7.9e-8 of the sums (2-norm, against 64 bits), so by 3.4e-8.
//
// The rows are split over S workgroups per tile where the tiles alone would
// not fill the chip; wgrad_sum_kernel adds the S partial results in order.
// us with all their launches, before (two transposes, product, sum, two
// column-sum passes) / now: 4096 rows, 3072 x 768 63.4 / 35, 768 x 768 45.5 /
// 17.4, 2304 x 768 54.3 / 29.1; 8192 rows, 2304 x 768 85.6 / 43.7. What bounds the
// product: the partial results it writes (28 MB at 3072 x 768) and the LDS, whose
// reads and writes take 1.5 times the matrix instructions' time and more (the
// transposing reads measure about half the rate of plain ones).
#include "zsa_internal.h"

namespace zsa {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kBiasTiles = 4;  // column tiles that share the bias sums

struct WgradArgs {
  const bf16_t *a, *b;   // dY [rows, m], X [rows, n]
  int rows, m, n;
  int tm, tn, splits;    // tiles of m and n, row splits
  int chunk;             // rows per split, a multiple of 64 (the last slice may be part-filled)
  float* out;            // splits == 1: [m, n]; else [splits][m, n]
  float* bias;           // [splits * wave columns * min(tn, kBiasTiles)][m], or null
};

// TILE x TILE outputs on WM x WN waves, BK rows per slice, NB slices in LDS,
// NB - 1 of them in flight; one barrier per slice. 64 KB of LDS a workgroup at
// the narrower tiles: two slices of 64 (128) rows beat four of half as many,
// whose barriers are twice as many (us with the sums: 4096 rows, 3072 x 768
// 37.7 / 34.6, 768 x 768 18.2 / 17.4; 8192 rows, 2304 x 768 45.4 / 43.7); at 256
// the two are alike.
template <int TILE, int WM, int WN, int BK, int NB>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(2, 2))) void wgrad_kernel(const WgradArgs p) {
  constexpr int NW = WM * WN, RB = TILE * 2, CPR = TILE / 8;  // bytes and 16-byte chunks of a slice row
  constexpr int HALF = BK * RB, BUF = 2 * HALF;
  constexpr int RPL = 1024 / RB, LPW = HALF / 1024 / NW;  // rows per load, loads per wave and operand
  constexpr int FM = TILE / 32 / WM, FN = TILE / 32 / WN;  // 32-wide fragments per wave
  static_assert(LPW * NW * 1024 == HALF, "slice split");
  __shared__ __align__(1024) unsigned char smem[NB * BUF];

  // an XCD (workgroup number mod 8) takes neighbouring tiles of one split,
  // whose rows its L2 then holds
  const int total = p.tm * p.tn * p.splits, per = (total + 7) / 8;
  const int id = static_cast<int>(blockIdx.x & 7) * per + static_cast<int>(blockIdx.x >> 3);
  if (static_cast<int>(blockIdx.x >> 3) >= per || id >= total) return;
  const int split = id / (p.tm * p.tn), tile = id - split * (p.tm * p.tn);
  const int im = tile / p.tn, in = tile - im * p.tn;
  const int m0 = im * TILE, n0 = in * TILE;
  const int r_begin = split * p.chunk, r_end = min(p.rows, r_begin + p.chunk);
  const int slices = r_end > r_begin ? (r_end - r_begin + BK - 1) / BK : 0;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, l32 = lane & 31;
  const int wm = wave / WN, wn = wave % WN;
  // slice row r keeps its 16-byte chunk c at c ^ sw(r): the four rows a
  // transposing read takes fall on all banks
  auto sw = [](int r) { return TILE == 64 ? ((r >> 1) & 1) << 2 : (r & 3) << 2; };
  const int lrow = wave * RPL + lane / CPR;  // slice row of the wave's first load
  const uint32_t a_row = static_cast<uint32_t>(p.m) * 2, b_row = static_cast<uint32_t>(p.n) * 2;
  const uint32_t lchunk = ((lane % CPR) ^ sw(lrow)) << 4;
  const uint32_t aoff = lrow * a_row + lchunk, boff = lrow * b_row + lchunk;
  const uint32_t lds0 = lds_address(smem) + wave * 1024;
  // the resource covers this slice's rows from the tile's first column on:
  // rows past the split (or the whole slice, past the last) read as zeros;
  // columns past the matrix read its next row and feed outputs that are not
  // stored
  auto resource = [&](const bf16_t* base, int width, int col, int r0) {
    const int live = max(0, min(BK, r_end - r0));
    const uint32_t bytes = live > 0 ? static_cast<uint32_t>(live) * width * 2 - col * 2 : 0;
    return buffer_resource(base + static_cast<int64_t>(r0) * width + col, bytes);
  };
  auto load_slice = [&](int t, int buf) {
    const int r0 = t < slices ? r_begin + t * BK : r_end;
    const u32x4 ar = resource(p.a, p.m, m0, r0), br = resource(p.b, p.n, n0, r0);
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      const uint32_t d = lds0 + buf * BUF + i * (NW * 1024);
      lds_load16(d, aoff + i * (NW * RPL) * a_row, ar);
      lds_load16(d + HALF, boff + i * (NW * RPL) * b_row, br);
    }
  };

  // a fragment: columns 32 c + l32 of slice rows 16 g + 4 half + 0 .. 3 and
  // + 8 of these
  const int vrow = 4 * half + ((lane & 15) >> 2);
  const int vch = 2 * ((lane >> 4) & 1) + ((lane >> 1) & 1);
  const uint32_t f0 = vrow * RB + (lane & 1) * 8;
  uint32_t fa[FM], fb[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i) fa[i] = f0 + (((4 * (wm * FM + i) + vch) ^ sw(vrow)) << 4);
#pragma unroll
  for (int j = 0; j < FN; ++j) fb[j] = HALF + f0 + (((4 * (wn * FN + j) + vch) ^ sw(vrow)) << 4);
  auto frag = [&](const unsigned char* at) {
    return __builtin_bit_cast(bf16x8_t, lds_read_columns(at, at + 8 * RB));
  };

  f32x16_t acc[FM][FN] = {};
  float sum[FM] = {};  // of column l32 of each fragment, over this half's rows
  const int nsum = WN * min(p.tn, kBiasTiles);
  int turn = p.bias != nullptr && in < kBiasTiles ? WN * in + wn : -1;  // next slice this wave sums

#pragma unroll
  for (int t = 0; t < NB - 1; ++t) load_slice(t, t);
  for (int t = 0; t < slices; ++t) {
    __builtin_amdgcn_sched_barrier(0);
    // slice t has landed (NB - 2 later ones may be in flight), and every wave
    // is done with slice t - 1, whose buffer the next load takes
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NB - 2) * 2 * LPW) : "memory");
    __builtin_amdgcn_sched_barrier(0);
    load_slice(t + NB - 1, (t + NB - 1) % NB);
    const unsigned char* base = smem + (t % NB) * BUF;
    const bool mine = t == turn;
    if (mine) turn += nsum;
    float part[FM] = {};
#pragma unroll
    for (int g = 0; g < BK / 16; ++g) {
      bf16x8_t av[FM], bv[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) av[i] = frag(base + fa[i] + g * (16 * RB));
#pragma unroll
      for (int j = 0; j < FN; ++j) bv[j] = frag(base + fb[j] + g * (16 * RB));
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i], bv[j], acc[i][j], 0, 0, 0);
      if (mine) {
#pragma unroll
        for (int i = 0; i < FM; ++i) {
          const u32x4 w = __builtin_bit_cast(u32x4, av[i]);
          float two[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) two[e] = __uint_as_float(w[e] << 16) + __uint_as_float(w[e] & 0xffff0000u);
          part[i] += (two[0] + two[1]) + (two[2] + two[3]);
        }
      }
    }
    if (mine) {
#pragma unroll
      for (int i = 0; i < FM; ++i) sum[i] += part[i];
    }
  }
  // no load may still be writing LDS when the workgroup ends
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  // acc[i][j][r]: row m0 + 32 (wm FM + i) + 8 (r/4) + 4 half + r%4, column n0 + 32 (wn FN + j) + l32
  float* out = p.out + static_cast<int64_t>(split) * p.m * p.n;
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = m0 + 32 * (wm * FM + i) + 8 * (r >> 2) + 4 * half + (r & 3);
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int n = n0 + 32 * (wn * FN + j) + l32;
        if (m < p.m && n < p.n) out[static_cast<int64_t>(m) * p.n + n] = acc[i][j][r];
      }
    }
  if (p.bias != nullptr && in < kBiasTiles) {
    float* row = p.bias + (static_cast<int64_t>(split) * nsum + WN * in + wn) * p.m;
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const float v = half_swap_sum(sum[i]);
      const int m = m0 + 32 * (wm * FM + i) + l32;
      if (half == 0 && m < p.m) row[m] = v;
    }
  }
}

// The sums of the split rows' partial products (total4 float4, `splits` of
// them; none when total4 is 0) and, in the workgroups past those, of the
// bias rows [brows][m] -- 32 columns a workgroup, 32 row lanes -- in order.
__global__ __launch_bounds__(256) void wgrad_sum_kernel(const float4* __restrict__ part, int splits,
                                                        int64_t total4, int blocks4,
                                                        float4* __restrict__ out,
                                                        const float* __restrict__ bias, int brows, int m,
                                                        float* __restrict__ db) {
  if (static_cast<int>(blockIdx.x) < blocks4) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= total4) return;
    float4 v = part[i];
#pragma unroll 4
    for (int y = 1; y < splits; ++y) {
      const float4 t = part[y * total4 + i];
      v.x += t.x;
      v.y += t.y;
      v.z += t.z;
      v.w += t.w;
    }
    out[i] = v;
    return;
  }
  __shared__ float red[32][33];
  const int q = threadIdx.x & 7, rl = threadIdx.x >> 3;
  const int c0 = (blockIdx.x - blocks4) * 32, c = c0 + 4 * q;
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (c < m) {  // m is a multiple of 8
#pragma unroll 4
    for (int r = rl; r < brows; r += 32) {
      const float4 t = *reinterpret_cast<const float4*>(bias + static_cast<int64_t>(r) * m + c);
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
  if (threadIdx.x < 32 && c0 + static_cast<int>(threadIdx.x) < m) {
    db[c0 + threadIdx.x] = lane_rows_total(red, threadIdx.x);
  }
}

// The tile width, and the splits that fill the workgroups the chip holds at
// once (one of 256 per CU, two of the others); a split keeps at least 128
// rows, 512 where a partial result is 2 MB or more (1000 rows, 3072 x 768: one
// split 18.8 us, three 23.1). 128-wide tiles read each operand half as often as 64-wide ones, which
// need fewer splits and so write fewer partial results: 768 x 768 over 4096
// rows, 19.7 us in 36 tiles of 128 and 13 splits (30 MB) with the kernel of
// before, 14.6 in 144 tiles of 64 and 3. 256-wide ones, where they number at
// least one per CU, halve both operands' reads again: the four products of a
// 4096-wide block with 14336 hidden and of a 2048-wide one with 8192 (2048 to
// 4096 rows) 1739 us in 128-wide tiles, 1550 with the 256-wide ones.
struct WgradPlan { int tile, waves_n, tm, tn, splits, chunk; };

WgradPlan wgrad_tiles(int m, int n) {
  auto tiles = [&](int64_t w) { return ((m + w - 1) / w) * ((n + w - 1) / w); };
  WgradPlan p{};
  p.tile = tiles(256) >= 256 ? 256 : tiles(128) >= 64 ? 128 : 64;
  p.waves_n = p.tile == 256 ? 4 : 2;
  p.tm = (m + p.tile - 1) / p.tile;
  p.tn = (n + p.tile - 1) / p.tile;
  return p;
}

int wgrad_splits(const WgradPlan& p, int rows) {
  const int64_t want = (p.tile == 256 ? 256 : 512) / (static_cast<int64_t>(p.tm) * p.tn);
  const int least = static_cast<int64_t>(p.tm) * p.tn * p.tile * p.tile >= (1 << 19) ? 512 : 128;
  return static_cast<int>(std::min<int64_t>(std::max<int64_t>(1, want), std::max(1, rows / least)));
}

WgradPlan wgrad_plan(int rows, int m, int n) {
  WgradPlan p = wgrad_tiles(m, n);
  const int s = wgrad_splits(p, rows);
  p.chunk = std::max(64, ((rows + s - 1) / s + 63) / 64 * 64);
  p.splits = std::max(1, (rows + p.chunk - 1) / p.chunk);
  return p;
}

size_t bias_rows(const WgradPlan& p, int splits) {
  return static_cast<size_t>(splits) * p.waves_n * std::min(p.tn, kBiasTiles);
}

}  // namespace

size_t wgrad_workspace_bytes(int max_rows, int m, int n) {
  // the tiles do not depend on the rows, and fewer rows never take more splits
  const WgradPlan p = wgrad_tiles(m, n);
  const int s = wgrad_splits(p, max_rows);
  return ((s > 1 ? static_cast<size_t>(s) * m * n : 0) + bias_rows(p, s) * m) * sizeof(float);
}

hipError_t launch_wgrad(hipStream_t s, const void* dy, int m, const void* x, int n, int rows,
                        float* dw, float* db, void* ws, size_t ws_bytes) {
  if (m == 0 || n == 0) return hipSuccess;
  const WgradPlan p = wgrad_plan(rows, m, n);
  const size_t part = p.splits > 1 ? static_cast<size_t>(p.splits) * m * n : 0;
  const size_t brows = db != nullptr ? bias_rows(p, p.splits) : 0;
  if (m % 8 != 0 || n % 8 != 0 || ws_bytes < (part + brows * m) * sizeof(float)) return hipErrorInvalidValue;
  float* w = static_cast<float*>(ws);
  WgradArgs a;
  a.a = static_cast<const bf16_t*>(dy);
  a.b = static_cast<const bf16_t*>(x);
  a.rows = rows;
  a.m = m;
  a.n = n;
  a.tm = p.tm;
  a.tn = p.tn;
  a.splits = p.splits;
  a.chunk = p.chunk;
  a.out = p.splits > 1 ? w : dw;
  a.bias = db != nullptr ? w + part : nullptr;
  const unsigned grid = static_cast<unsigned>((static_cast<int64_t>(p.tm) * p.tn * p.splits + 7) / 8 * 8);
  const hipError_t e = p.tile == 256   ? launch(K_GEMM, wgrad_kernel<256, 2, 4, 32, 4>, dim3(grid), dim3(512), 0, s, a)
                       : p.tile == 128 ? launch(K_GEMM, wgrad_kernel<128, 2, 2, 64, 2>, dim3(grid), dim3(256), 0, s, a)
                                       : launch(K_GEMM, wgrad_kernel<64, 2, 2, 128, 2>, dim3(grid), dim3(256), 0, s, a);
  if (e != hipSuccess || (part == 0 && db == nullptr)) return e;
  const int64_t total4 = part ? static_cast<int64_t>(m) * n / 4 : 0;
  const int blocks4 = static_cast<int>((total4 + 255) / 256);
  return launch(K_GEMM, wgrad_sum_kernel, dim3(blocks4 + (db != nullptr ? (m + 31) / 32 : 0)), dim3(256), 0, s,
                reinterpret_cast<const float4*>(w), p.splits, total4, blocks4, reinterpret_cast<float4*>(dw),
                static_cast<const float*>(a.bias), static_cast<int>(brows), m, db);
}

}  // namespace zsa
