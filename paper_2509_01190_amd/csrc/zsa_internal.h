// Internal declarations shared by the HIP kernels and the C-ABI layer.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <utility>

namespace zsa {

typedef uint16_t bf16_t;

// ---------------------------------------------------------------------------
// storage conversions (fp32 compute, f32 or bf16 storage)
// ---------------------------------------------------------------------------
__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t h) {
  return __uint_as_float(static_cast<uint32_t>(h) << 16);
}

// fp32 -> bf16 by v_cvt_pk_bf16_f32: round to nearest even, bit-identical
// to the integer rounding (u + 0x7fff + lsb) >> 16 for every normal and
// infinite input (checked exhaustively on gfx950; only subnormal inputs,
// |x| < 2^-126, differ); NaN stays NaN.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
// the pair {x[l], x[l ^ 32]} of lane l in one VALU op (v_permlane32_swap:
// the first result is x[l & 31], the second x[(l & 31) + 32] on every
// lane), so combining the two gives the same value, in the same operand
// order, on both halves of the wave -- without an LDS round trip
__device__ __forceinline__ float half_swap_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_swap_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  return static_cast<bf16_t>(pack_bf16x2(f, 0.f) & 0xffffu);
}

template <typename T>
__device__ __forceinline__ T from_f32(float x);
template <>
__device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <>
__device__ __forceinline__ bf16_t from_f32<bf16_t>(float x) { return f32_to_bf16(x); }

// 16-byte vector of storage elements
template <typename T>
struct Vec16 {
  static constexpr int N = 16 / sizeof(T);
};

__device__ __forceinline__ void unpack16(const uint4& v, float* out, float) {
  out[0] = __uint_as_float(v.x); out[1] = __uint_as_float(v.y);
  out[2] = __uint_as_float(v.z); out[3] = __uint_as_float(v.w);
}
__device__ __forceinline__ void unpack16(const uint4& v, float* out, bf16_t) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    out[2 * i] = __uint_as_float(w[i] << 16);
    out[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}
__device__ __forceinline__ uint4 pack16(const float* in, float) {
  return make_uint4(__float_as_uint(in[0]), __float_as_uint(in[1]), __float_as_uint(in[2]),
                    __float_as_uint(in[3]));
}
__device__ __forceinline__ uint4 pack16(const float* in, bf16_t) {
  return make_uint4(pack_bf16x2(in[0], in[1]), pack_bf16x2(in[2], in[3]),
                    pack_bf16x2(in[4], in[5]), pack_bf16x2(in[6], in[7]));
}

// native 16-byte vector (first-class in LLVM, so arrays of it stay in
// registers; HIP's uint4 is a struct whose copies can end up on the stack)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// keep a 16-byte value or zero it, without a select between two uint4 objects
// (which the compiler lowers through a stack slot)
__device__ __forceinline__ uint4 keep16(const uint4& v, bool keep) {
  const uint32_t m = keep ? 0xffffffffu : 0u;
  return make_uint4(v.x & m, v.y & m, v.z & m, v.w & m);
}

// ---------------------------------------------------------------------------
// tiles straight from memory to LDS, and fragments out of them
// ---------------------------------------------------------------------------
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) const char lds_char;

// a buffer of `bytes` bytes (wave-uniform): loads past it read as zeros
__device__ __forceinline__ u32x4 buffer_resource(const void* p, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  const u32x4 r = {static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(a))),
                   static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(a >> 32))) & 0xffffu,
                   static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(bytes))), 0x00020000u};
  return r;
}

// The lanes' 16 (4) bytes at res + off, to 16 (4) bytes a lane from LDS
// address lds on (wave-uniform). In asm, without outputs: the compiler would
// wait for a load it knows to write LDS before any later LDS read; the caller
// waits (turn_over). The LDS address is an operand in m0, so that the compiler
// sets that register itself and knows what it holds.
__device__ __forceinline__ void lds_load16(uint32_t lds, uint32_t off, const u32x4& res) {
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"{m0}"(lds), "v"(off), "s"(res) : "memory");
}
__device__ __forceinline__ void lds_load4(uint32_t lds, uint32_t off, const u32x4& res) {
  asm volatile("s_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"{m0}"(lds), "v"(off), "s"(res) : "memory");
}
// address of a __shared__ array for the loads
__device__ __forceinline__ uint32_t lds_address(const void* smem) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_char*)smem));
}

// every wave's tile loads have landed, and all waves are past their LDS reads
__device__ __forceinline__ void turn_over() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Eight rows of a column per lane out of a tile kept in rows: two transposing
// reads. Each gives a lane of a 16-lane group element (its number in the
// group) of four 16-element rows, row r pieced together from the 8-byte runs
// at the addresses of the group's lanes 4r .. 4r + 3.
__device__ __forceinline__ u32x4 lds_read_columns(const void* first, const void* second) {
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)((lds_char*)first));
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)((lds_char*)second));
  const uint2 a2 = __builtin_bit_cast(uint2, a), b2 = __builtin_bit_cast(uint2, b);
  const u32x4 v = {a2.x, a2.y, b2.x, b2.y};
  return v;
}

// four consecutive elements in fp32
template <typename T>
__device__ __forceinline__ float4 load4(const T* p);
template <>
__device__ __forceinline__ float4 load4<float>(const float* p) {
  return *reinterpret_cast<const float4*>(p);
}
template <>
__device__ __forceinline__ float4 load4<bf16_t>(const bf16_t* p) {
  const uint2 v = *reinterpret_cast<const uint2*>(p);
  return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
                     __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u));
}

// The sum of column c over the 32 row lanes of a workgroup's partial sums, in
// pairs: added one after another the 32 roundings add up (k_wgrad.hip has
// the errors)
__device__ __forceinline__ float lane_rows_total(const float (&red)[32][33], int c) {
  float v[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) v[k] = red[k][c] + red[k + 16][c];
#pragma unroll
  for (int w = 8; w > 0; w >>= 1)
#pragma unroll
    for (int k = 0; k < w; ++k) v[k] += v[k + w];
  return v[0];
}

// ---------------------------------------------------------------------------
// placement of attention workgroups
// ---------------------------------------------------------------------------
// Which (sequence, head, block of queries or keys) an attention or score
// workgroup takes. Workgroup L runs on XCD L % 8, in order of L within it. The (sequence,
// head) pairs are dealt to the XCDs in turn, and an XCD walks `chunk` of its
// pairs at a time, last query block first. Where `group` heads share a
// key/value head and the heads are a multiple of 8, an XCD takes neighbouring
// ones, and their K and V stay in its L2 (32 heads on 8, 32 ragged sequences
// of up to 300 rows 50 us, in plain order 57); heads that share nothing are in
// plain order (64 x 128 rows, 32 heads of 64: 26.6, neighbours 27.4). With
// the query block in the grid's fastest dimension, as these kernels had it,
// equal sequences put the same query block on the same XCD throughout: under
// the causal mask one XCD got every longest block and another every shortest
// (the same kernel: 4 x 4096 causal rows, 32 heads of 128, 918 -> 596 us; 8 x
// 2048, 32 heads of 64, 286 -> 182; 12 ragged sequences of up to 4095 rows,
// 1697 -> 852). Measured with attn_wide_kernel, us, one pair at a time / a
// sequence's / all: causal, 8 x 2048 of 64 211 / 174 / 162, 16 x 1024, 12
// heads of 64, 55.9 / 55.1 / 43.1; without a mask, where every block of a
// sequence is as long and the neighbours' K and V are still in L2, 8 x 2048
// of 64 267 / 263 / 282, 32 x 512, 12 heads, 36.0 / 35.8 / 37.4. So all of
// them (the longest blocks first, the shortest at the end) under the mask or
// with sequences of several lengths, and a sequence's otherwise. A caller may
// cap the former (`most`) where an XCD has many pairs and each much K and V:
// walked all at once, a pair's are gone from the caches by its next block.
// Two kinds of calls keep the query block in the fastest dimension (`pairs`
// negative): sequences of one block and heads that share nothing, where there
// is no order to choose and the division below costs 4 % (107 x 37 rows, 20
// heads of 128, 26.8 / 27.8), and without a mask pairs that do not spread evenly
// over the XCDs, which dealing by blocks does (scores of 1 x 2049 rows, 12 heads
// of 64 on 3, 22.3 / 28.9; attention of 5 ragged sequences of up to 1711 rows,
// 12 heads of 128, 76 / 85). So do long sequences of several lengths whose heads
// do not divide by eight: an XCD then meets some of the sequences more often
// than others (with 4 heads every second one), and the call ends with the one
// that has the longest. By blocks / by pairs: 16 ragged sequences of up to 2494
// rows, 12 heads of 64, 154 / 205 and their scores 111 / 155; 8 of up to 3114,
// 4 heads of 128, 101 / 138 and 68 / 117. From 24 heads on the difference is
// under a fourth and the keys that stay in an XCD's L2 count for more (20 of up
// to 1962, 36 heads of 64, 449 / 352), as they do in shorter sequences (scores
// of 48 of up to 600, 4 heads of 64, 24.6 / 20.7).
struct Place { int b, h, i; };
// grid (place_grid): x = 8 * chunk (XCD fastest), y = blocks, z = chunks of
// pairs, or, with all pairs in x, runs of blocks; i counts the blocks from the
// last (attention: the queries that see most keys) or, with `first`, from the
// first (scores: the keys that most queries see)
__host__ __device__ __forceinline__ bool place_at(dim3 grid, dim3 at_block, int H, int group, int pairs,
                                                  bool first, Place* at) {
  if (pairs < 0) {
    at->b = static_cast<int>(at_block.z);
    at->h = static_cast<int>(at_block.y);
    at->i = static_cast<int>(first ? at_block.x : grid.x - 1 - at_block.x);
    return true;
  }
  const uint32_t chunk = grid.x >> 3;
  const bool whole = 8 * static_cast<uint64_t>(chunk) >= static_cast<uint64_t>(pairs);
  const uint32_t pz = whole ? 0 : at_block.z, iz = whole ? at_block.z : 0;
  const uint32_t e = (pz * chunk + (at_block.x >> 3)) * 8 + (at_block.x & 7);
  if (e >= static_cast<uint32_t>(pairs)) return false;
  at->b = static_cast<int>(e) / H;
  const int x = static_cast<int>(e) - at->b * H;
  at->h = group > 1 && H % 8 == 0 ? (x & 7) * (H >> 3) + (x >> 3) : x;
  const uint32_t i = iz * grid.y + at_block.y, blocks = grid.y * (whole ? grid.z : 1);
  at->i = static_cast<int>(first ? i : blocks - 1 - i);
  return true;
}
__device__ __forceinline__ bool place(int H, int group, int pairs, bool first, Place* at) {
  return place_at(gridDim, blockIdx, H, group, pairs, first, at);
}

constexpr uint32_t kGridYZ = 65535;  // HIP's limit on a grid's y and z

struct PlaceGrid {
  dim3 grid;
  int pairs;  // H * B, or -1: blocks in x, heads in y, sequences in z
};
// (most: pairs an XCD walks at a time where it has 80 or more; 0: no cap. Not for short sequences of several lengths,
// whose missing blocks leave gaps in every chunk: 300 of up to 130 rows, 32 heads of 128, 165 us all at once, 176 in eights)
inline PlaceGrid place_grid(int H, int group, int B, int max_len, int T, int causal, int block, int most = 0) {
  const int64_t p8 = (static_cast<int64_t>(H) * B + 7) / 8;  // pairs per XCD
  const bool alike = !causal && static_cast<int64_t>(B) * max_len == T;
  const int64_t blocks = (static_cast<int64_t>(max_len) + block - 1) / block, spare = 8 * p8 - static_cast<int64_t>(H) * B;
  const bool uneven = 20 * spare > static_cast<int64_t>(H) * B || (!alike && max_len > 1024 && H % 8 != 0 && H < 24);
  if ((blocks == 1 && group == 1) || (!causal && uneven))
    if (H <= static_cast<int>(kGridYZ) && B <= static_cast<int>(kGridYZ))
      return {dim3(static_cast<uint32_t>(blocks), static_cast<uint32_t>(H), static_cast<uint32_t>(B)), -1};
  // (a sequence's pairs only where they divide evenly: slots left over in the last chunk go out between others, which
  // an XCD's shader engines take in turn, and one of them gets more of the work: 2 x 2959 rows, 20 heads of 64, one pair
  // at a time 117 us, two 140)
  int64_t chunk = alike ? (H % 8 == 0 ? std::min<int64_t>(p8, H / 8) : 1) : p8;
  if (most > 0 && !alike && p8 >= 80 && (max_len > 256 || static_cast<int64_t>(B) * max_len == T)) chunk = most;
  // the chunks number at most 65535, and at 512 threads a workgroup x stays below 2^32 threads
  chunk = std::min<int64_t>(std::max(chunk, (p8 + kGridYZ - 1) / kGridYZ), (1 << 20) - 1);
  // sequences of more blocks than y holds (8.4 M rows in 128-row blocks): all pairs in x, the blocks in y and z
  if (blocks > kGridYZ)
    return {dim3(static_cast<uint32_t>(8 * p8), kGridYZ, static_cast<uint32_t>((blocks + kGridYZ - 1) / kGridYZ)), H * B};
  return {dim3(static_cast<uint32_t>(8 * chunk), static_cast<uint32_t>(blocks), static_cast<uint32_t>((p8 + chunk - 1) / chunk)), H * B};
}

// ---------------------------------------------------------------------------
// launch helper with the optional per-class timing hook
// ---------------------------------------------------------------------------
enum KClass { K_GEMM = 0, K_ATTENTION = 1, K_SCORE = 2, K_SELECT = 3, K_GATHER = 4,
              K_NORM = 5, K_MISC = 6, K_NCLASS = 7 };

// returns true and a (start, stop) pair if the next launch of this class is timed
bool timing_take(int kclass, hipEvent_t* start, hipEvent_t* stop);
// records the thread's last error text (zsa_last_error) and returns code
int set_error(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));

template <typename... KArgs, typename... Args>
inline hipError_t launch(int kclass, void (*kernel)(KArgs...), dim3 grid, dim3 block,
                         size_t shmem, hipStream_t stream, Args... args) {
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (timing_take(kclass, &e0, &e1)) {
    hipExtLaunchKernelGGL(kernel, grid, block, static_cast<uint32_t>(shmem), stream, e0, e1, 0,
                          static_cast<KArgs>(args)...);
  } else {
    hipLaunchKernelGGL(kernel, grid, block, static_cast<uint32_t>(shmem), stream,
                       static_cast<KArgs>(args)...);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// GEMM epilogue parameters (shared by the MFMA and the vector-ALU GEMMs)
// ---------------------------------------------------------------------------
enum Epi { EPI_NONE = 0, EPI_GELU = 1, EPI_SWIGLU = 2, EPI_RESIDUAL = 3, EPI_ROPE = 4 };

constexpr int kMaxHalfHead = 64;  // head_dim <= 128 for the rotary epilogue

// sine and cosine of the rotary angle pos * inv_freq: the angle is formed in
// double and reduced to [-pi, pi] with a two-constant (Cody-Waite)
// subtraction of multiples of 2*pi before the fp32 sincos
__device__ __forceinline__ void rope_angle(int p, double inv_freq, float* s, float* c) {
  const double two_pi_hi = 6.283185307179586;       // nearest double to 2*pi
  const double two_pi_lo = 2.4492935982947064e-16;  // 2*pi - two_pi_hi
  const double a = static_cast<double>(p) * inv_freq;
  const double q = rint(a * 0.15915494309189535);   // a / (2*pi)
  double r = fma(-q, two_pi_hi, a);
  r = fma(-q, two_pi_lo, r);
  sincosf(static_cast<float>(r), s, c);
}

struct EpiParams {
  int epi;
  const void* bias;      // [N] or null
  const void* residual;  // [M, ldy] or null
  void* y;               // output
  int ldy;               // output row stride (elements)
  const int32_t* pos;    // [M] rotary positions
  int head_dim;
  int rope_cols;
  // per-row rotary table [M][head_dim / 2] of (cos, sin) pairs (fp32), the
  // values rope_angle gives for that row's position; null: each kernel forms
  // the angles itself
  const float* rope_cs;
  double inv_freq[kMaxHalfHead];  // theta^(-2i/hd), computed on the host in double
};

// bytes of a rotary table for M rows (launch_rope_table)
inline size_t rope_table_bytes(int M, int head_dim) {
  return static_cast<size_t>(M) * (head_dim / 2) * 2 * sizeof(float);
}
// out[m][i] = (cos, sin) of pos[m] * inv_freq[i] for i < head_dim / 2
hipError_t launch_rope_table(hipStream_t s, const int32_t* pos, int M, const EpiParams& ep,
                             float* out);

// ---------------------------------------------------------------------------
// kernel launchers (one translation unit each)
// ---------------------------------------------------------------------------
hipError_t launch_norm(hipStream_t s, int dtype, int kind, const void* x, const void* g,
                       const void* b, int rows, int d, float eps, void* y);

// y = epi(x W^T + bias); x [M, K], W [N, K]. ws (may be NULL) holds split-K
// partials; the bf16 path splits K for small grids when ws_bytes covers it.
hipError_t launch_gemm(hipStream_t s, int dtype, const void* x, int M, int K, const void* w,
                       int N, const EpiParams& ep, void* ws, size_t ws_bytes);
// split-K plan of the bf16 path and its workspace (0 when K is not split)
void splitk_plan(int M, int N, int K, int* S, int* kchunk);
size_t splitk_bytes(int S, int M, int N);
size_t gemm_workspace_bytes(int dtype, int M, int N, int K);
// the most any M <= max_rows needs
size_t gemm_workspace_bound(int dtype, int max_rows, int N, int K);

int device_cu_count();  // compute units of the current device

// Few-row product (bf16, up to 4096 rows of x in blocks of 16): W streamed
// into MFMA operands, one workgroup per 16 output columns and 16 rows over
// the whole of K (no workspace).
// With pn (gain non-null; skinny_norm_ok: M <= 8, K <= 4096, few output
// tiles) x is first normalised as launch_norm would (LayerNorm with shift,
// or RMSNorm).
struct PreNorm {
  const bf16_t* g;  // gain [K], or null: x is used as it is
  const bf16_t* b;  // LayerNorm shift [K] or null
  int rms;          // 1: RMSNorm, 0: LayerNorm
  float eps;
};
bool skinny_ok(int dtype, int M, int N, int K, const EpiParams& ep);
bool skinny_pays(int M, int N, int K, const EpiParams& ep);  // launch_gemm takes it for such shapes
bool skinny_norm_ok(int M, int N, int K);
// tiles launch_gemm takes for a bf16 product of few output tiles
enum ShortGrid { kNoShort, kShort64, kShort128x64, kShort128 };
ShortGrid short_grid(int M, int N, int K, const EpiParams& ep, bool split);
// launch_gemm runs this product on the few-row kernel
bool gemm_takes_skinny(int dtype, int M, int N, int K, const EpiParams& ep);
hipError_t launch_gemm_skinny(hipStream_t s, const void* x, int M, int K, const void* w, int N,
                              const EpiParams& ep, const PreNorm* pn = nullptr);

// query head h reads key/value head h / kv_group (kv_group = H / H_kv)
hipError_t launch_attention(hipStream_t s, int dtype, const void* q, const void* k,
                            const void* v, int64_t row_stride, int H, int kv_group, int hd,
                            int causal, float scale, int B, int max_len, int T,
                            const int32_t* cu_dev, void* out, int64_t out_stride, float* lse);

// the long-sequence kernel takes this bf16 call (head_dim 64 or 128)
bool attention_wide(int hd, int H, int B, int max_len, int causal, int cus);

// writes G partial score vectors [G][T] (G = head groups); returns G via *groups
hipError_t launch_score(hipStream_t s, int dtype, const void* q, const void* k,
                        int64_t row_stride, const float* lse, int H, int kv_group, int hd,
                        int causal, float scale, int B, int max_len, int T,
                        const int32_t* cu_dev, float* partials, int groups);
int score_groups(int dtype, int H, int hd, int T);
// the kernel of 256-key workgroups takes this bf16 call (head_dim 64 or 128)
bool score_wide(int hd, int H, int B, int max_len, int T, int causal, int cus);

hipError_t launch_score_finalize(hipStream_t s, const float* partials, int groups, int T,
                                 float* scores);

// per-sequence top-k over sum_g partials[g*T + row]; cu_out gives output
// offsets; keep_last always keeps each sequence's last row
hipError_t launch_select(hipStream_t s, const float* partials, int groups, int T, int B,
                         int max_len, const int32_t* cu_in_dev, const int32_t* cu_out_dev,
                         int32_t* kept_rows, float* scores_out, int keep_last);

// generation: key/value cache rows and the attention of one new row per
// sequence (cache layout [batch][cap][k | v] per layer, kvd = H_kv * hd)
hipError_t launch_kv_store(hipStream_t s, int dtype, const void* src, int64_t src_stride,
                           int src_col, int kvd, int B, int max_rows, const int32_t* cu_dev,
                           const int32_t* start_dev, void* cache_layer, int cap);
// qkv [B, q_stride]: query heads at column 0, the new row's k | v at kv_col;
// appends them at cache row len - 1, then attends over len rows. Partials:
// m, l [B][H][decode_splits_bound(cap)], o [...][hd]
hipError_t launch_decode_attention(hipStream_t s, const void* qkv, int64_t q_stride, int kv_col,
                                   void* cache_layer, int cap, int hd, int H, int Hkv,
                                   const int32_t* len_dev, int B, int max_len, float scale,
                                   float* m_part, float* l_part, float* o_part, void* out,
                                   int64_t out_stride);
int decode_splits_bound(int cap);
bool decode_supported(int dtype, int hd, int group);

// backward pass (bf16, head_dim 64 / 128 for the attention part)
bool backward_supported(int dtype, int hd);
// dW [m, n] = dY^T X over `rows` rows and db [m] = the column sums of dY (db
// may be NULL), both fp32
hipError_t launch_wgrad(hipStream_t s, const void* dy, int m, const void* x, int n, int rows,
                        float* dw, float* db, void* ws, size_t ws_bytes);
// the most any number of rows up to max_rows needs
size_t wgrad_workspace_bytes(int max_rows, int m, int n);
// out = in^T for up to four bf16 matrices [r, c] in one launch
struct TransposeArg { const void* in; void* out; int r, c; };
hipError_t launch_transposes(hipStream_t s, const TransposeArg* t, int count);
// out = res + dL/dx of a norm whose output has gradient dh, dg and db [d] the
// gradients of its gain and shift (db may be NULL; unused by RMSNorm).
// scratch: norm_bwd_scratch_floats of the largest R
size_t norm_bwd_scratch_floats(int R, int d);
hipError_t launch_norm_bwd(hipStream_t s, int kind, const void* x, const void* g, const void* dh,
                           const void* res, void* out, int R, int d, float eps, float* scratch,
                           float* dg, float* db);
// f = act(u) and du = dF act'(u)
hipError_t launch_act_bwd(hipStream_t s, const void* dF, const void* u, void* du, void* f, int rows,
                          int F, int swiglu);
// undoes compaction of two arrays of d-wide rows: dst[kept[i]] = src[i],
// zeros elsewhere (kept ascending)
hipError_t launch_scatter_rows(hipStream_t s, int d, const void* src0, void* dst0, const void* src1,
                               void* dst1, const int32_t* kept, int t_out, int t_in);
// LD[h][r] = (lse[h][r] log2 e, dO_r . O_r over head h's columns)
hipError_t launch_rowdot(hipStream_t s, const void* dO, const void* O, int64_t ld, int T, int H,
                         int hd, const float* lse, float* LD);
hipError_t launch_rope_bwd(hipStream_t s, int dtype, void* g, int64_t ld, int rows, int cols,
                           int hd, const int32_t* pos, const EpiParams& ep);
hipError_t launch_attention_bwd(hipStream_t s, const void* q, const void* k, const void* v,
                                int64_t rs, const void* dO, int64_t ors, const float* LD, int H,
                                int kv_group, int hd, int causal, float scale, int B, int max_len,
                                int T, const int32_t* cu_dev, void* dq, void* dk, void* dv,
                                int64_t grs);

// row gather of up to two [*, d] arrays plus pos
hipError_t launch_gather(hipStream_t s, int dtype, int d, int t_in, const int32_t* kept,
                         int t_out, const void* src0, void* dst0, const void* src1, void* dst1,
                         const int32_t* pos, int32_t* pos_out);

hipError_t launch_upload_i32(hipStream_t s, int32_t* dst, const int32_t* host_vals, int n);
hipError_t launch_copy_i32(hipStream_t s, int32_t* dst, const int32_t* src, int n);

}  // namespace zsa
