// Attention of Eq. 1, softmax(Q K^T * scale + M) V, per sequence and head
// (query head h reads key/value head h / kv_group: grouped-query attention),
// over packed variable-length rows; also writes the natural-log
// log-sum-exp of every score row (used by the contribution scores).
//
// bf16, head_dim 64/128 (MFMA): every kernel computes the *transposed* score
// tile S^T = K Q^T with v_mfma_f32_32x32x16_bf16, so a lane holds the scores
// of one query: the softmax sums are in-lane plus one swap with lane l^32,
// and the probabilities already sit in the B-operand layout of
// O^T += V^T P^T (P rounded to bf16), with no trip through LDS. The k-slot
// order of P^T is whatever the accumulator gives; V^T is read from LDS in
// that same order, which leaves the contraction unchanged.
//  * attn_wide_kernel (longer sequences): 32-key steps, each step's
//    exponentials interleaved with the products of its neighbours, K/V tiles
//    loaded straight into LDS;
//  * attn_mfma_kernel (shorter ones, and grids of few workgroups:
//    attention_wide): one workgroup of NW waves per 32 NW-query block, 64-key
//    tiles staged through registers.
//
// fp32 (and bf16 at any other head_dim): the same transposed scores on the
// fp32 matrix instruction, four waves sharing 32 queries' keys.
#include <math.h>

#include <type_traits>

#include "zsa_internal.h"

namespace zsa {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Shorter sequences (up to 256 rows at head dim 64, 384 at 128) and, up to
// 512 rows at 128 and under the mask of any length at 64, grids of few
// workgroups. Four waves per SIMD at head dim 64 (128 registers), two
// at 128, walking 64-key tiles staged in LDS (K row-major; V transposed at
// head dim 64, row-major at 128 and read through transposing LDS reads). A
// workgroup reads every K and V row of its sequence and head once, so the bytes moved
// per query fall as the query block grows: the loads, not the MFMAs or the
// exponentials, bound the kernel where the chip is full (32 sequences x 12
// heads x 512 rows, which the long-sequence kernel has now: a copy without
// any of the compute took 35 of 48.5 us with 4 waves). 8 waves (256 queries,
// two workgroups per CU; head dim 64 past 128 rows) halve them: 45.9.
template <int HD, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(HD == 64 ? 4 : 2))) void attn_mfma_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    int64_t rs, int kv_group, int causal, float scale_log2, const int32_t* __restrict__ cu,
    bf16_t* __restrict__ O, int64_t os, float* __restrict__ lse, int T, int H, int pairs) {
  constexpr int NT = 64 * NW, BQ = 32 * NW, BKEY = 64;
  constexpr int KLD = HD + 8;    // K tile row stride (bf16)
  // V^T tile row stride (bf16): 34 dwords. The fragment reads (32
  // consecutive rows, 8 bytes each) hit distinct bank pairs and stay 8-byte
  // aligned, so they are ds_read_b64 with immediate offsets. In row r the
  // 8-byte chunk of keys 4c .. 4c + 3 sits at chunk c ^ (VSW * (r / 32)):
  // the transposing writes of a wave (rows 8j + e of 8 channel blocks j, 8
  // key pairs) then cover all 64 banks once, where rows j and j + 4
  // otherwise met in one bank (2-way), while the 32 rows of a fragment read
  // share one XOR and stay conflict-free (1 % at head dim 64 over 2048 rows).
  constexpr int VLD = BKEY + 4;
  constexpr int VSW = HD == 64 ? 4 : 0;
  // Head dim 128 stores V as it comes (key rows, the K tile's row stride)
  // and reads the V^T fragments with gfx950's transposing LDS reads
  // (ds_read_b64_tr_b16): 6 % over 4096 rows. At head dim 64 the same reads
  // gained nothing over 2048 rows and lost 4 % over 512 (40.6 -> 42.2 us on
  // 32 x 512, 12 heads), so it keeps the transposed tile.
  constexpr bool VTR = HD == 128;
  constexpr int OLD = HD + 8;    // output staging row stride
  constexpr int KBYTES = BKEY * KLD * 2, VBYTES = VTR ? KBYTES : HD * VLD * 2;
  constexpr int BUF = KBYTES + VBYTES;
  // K/V tile buffers: eight-wave blocks (head dim 64) keep four (tiles stored
  // two ahead, a barrier after every second tile: 11.2 -> 10.2 us on 8 x 256
  // causal rows, 32 heads); four-wave blocks two (one ahead, a barrier per
  // tile), which keeps four of them on a CU
  constexpr int NB = NW == 8 ? 4 : 2, LA = NB / 2;
  constexpr int SBYTES = NB * BUF > NW * 32 * OLD * 2 ? NB * BUF : NW * 32 * OLD * 2;
  constexpr int KITEMS = BKEY * HD / 8;        // 16-byte K chunks per tile
  constexpr int VITEMS = (BKEY / 2) * (HD / 8);  // V row-pair chunks per tile
  static_assert(KITEMS % NT == 0 && (VITEMS % NT == 0 || VITEMS < NT), "tile split");
  constexpr int KCH = KITEMS / NT;                   // per thread
  constexpr int VPR = VITEMS < NT ? 1 : VITEMS / NT;  // per thread (some idle if fewer)
  __shared__ __align__(16) unsigned char smem[SBYTES];

  Place at;
  if (!place(H, kv_group, pairs, false, &at)) return;
  const int b = at.b, h = at.h;
  const int lo = cu[b];
  const int n = cu[b + 1] - lo;
  const int q0 = at.i * BQ;
  if (q0 >= n) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, l32 = lane & 31;
  const int qrow = q0 + wave * 32 + l32;
  bf16x8_t qf[HD / 16];
#pragma unroll
  for (int kk = 0; kk < HD / 16; ++kk) {
    // rows past the sequence are clamped, not zeroed: their outputs are not stored
    const int qr = min(qrow, n - 1);
    qf[kk] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(
                                              Q + static_cast<int64_t>(lo + qr) * rs + h * HD + kk * 16 + half * 8));
  }

  // K/V tiles of a later key block are prefetched into registers while the
  // current block is computed, and stored LA blocks ahead into NB LDS
  // buffers; a barrier follows every LA blocks.
  // The loads go through a buffer resource spanning this sequence's rows,
  // so keys past the sequence read as zeros (they are masked to probability
  // 0); a thread's offsets within a tile are fixed, plus the tile's start.
  // grouped-query attention: query head h reads key/value head h / kv_group
  const int hk = h / kv_group;
  const uint32_t seq_bytes = static_cast<uint32_t>(static_cast<int64_t>(n) * rs * 2);
  const __amdgpu_buffer_rsrc_t kres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(K + static_cast<int64_t>(lo) * rs + hk * HD), 0, seq_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t vres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(V + static_cast<int64_t>(lo) * rs + hk * HD), 0, seq_bytes, 0x00020000);
  uint32_t koff[KCH], voff[VPR];
#pragma unroll
  for (int i = 0; i < KCH; ++i) {
    const int c = tid + i * NT;
    koff[i] = static_cast<uint32_t>((c / (HD / 8)) * rs + (c % (HD / 8)) * 8) * 2u;
  }
  // threads past the tile's V chunks (when there are fewer than threads)
  // load from past the buffer range (zeros) and store nothing
  const bool vth = VITEMS >= NT || tid < VITEMS;
#pragma unroll
  for (int i = 0; i < VPR; ++i) {
    const int c = tid + i * NT;
    voff[i] = vth ? static_cast<uint32_t>((2 * (c / (HD / 8))) * rs + (c % (HD / 8)) * 8) * 2u
                  : 0x80000000u;
  }
  const uint32_t row_bytes = static_cast<uint32_t>(rs * 2);
  u32x4 kreg[KCH], vreg[VPR][2], vrow[KCH];
  auto load_tile = [&](int j0) {
    const uint32_t t0 = static_cast<uint32_t>(j0) * row_bytes;
    // the whole offset goes in the vector operand, which the range check covers
#pragma unroll
    for (int i = 0; i < KCH; ++i)
      kreg[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(kres, koff[i] + t0, 0, 0));
    if constexpr (VTR) {
      // V rows at the K offsets (one row stride)
#pragma unroll
      for (int i = 0; i < KCH; ++i)
        vrow[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(vres, koff[i] + t0, 0, 0));
      return;
    }
#pragma unroll
    for (int i = 0; i < VPR; ++i) {
      vreg[i][0] = __builtin_bit_cast(
          u32x4, __builtin_amdgcn_raw_buffer_load_b128(vres, voff[i] + t0, 0, 0));
      vreg[i][1] = __builtin_bit_cast(
          u32x4, __builtin_amdgcn_raw_buffer_load_b128(vres, voff[i] + t0 + row_bytes, 0, 0));
    }
  };
  auto store_tile = [&](int buf) {
    bf16_t* Ks = reinterpret_cast<bf16_t*>(smem + buf * BUF);
    bf16_t* Vt = reinterpret_cast<bf16_t*>(smem + buf * BUF + KBYTES);
#pragma unroll
    for (int i = 0; i < KCH; ++i) {
      const int c = tid + i * NT;
      const int r = c / (HD / 8), ch = (c % (HD / 8)) * 8;
      *reinterpret_cast<u32x4*>(Ks + r * KLD + ch) = kreg[i];
      if constexpr (VTR) *reinterpret_cast<u32x4*>(Vt + r * KLD + ch) = vrow[i];
    }
    if (VTR || !vth) return;
#pragma unroll
    for (int i = 0; i < VPR; ++i) {
      const int c = tid + i * NT;
      const int rp = c / (HD / 8), ch = (c % (HD / 8)) * 8;
      // rows ch .. ch + 7 share one 32-row group, hence one swizzle
      bf16_t* vt = Vt + ch * VLD + 4 * ((rp >> 1) ^ (VSW * (ch >> 5))) + 2 * (rp & 1);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t w0 = vreg[i][0][e >> 1], w1 = vreg[i][1][e >> 1];
        const uint32_t x0 = (e & 1) ? (w0 >> 16) : (w0 & 0xffffu);
        const uint32_t x1 = (e & 1) ? (w1 & 0xffff0000u) : (w1 << 16);
        *reinterpret_cast<uint32_t*>(vt + e * VLD) = x0 | x1;
      }
    }
  };

  float m_run = -INFINITY, l_run = 0.f;  // running max in raw score units
  f32x16_t o[HD / 32];
#pragma unroll
  for (int ct = 0; ct < HD / 32; ++ct)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[ct][r] = 0.f;

  const int kend = causal ? min(n, q0 + BQ) : n;
  const int wave_q0 = q0 + wave * 32;
  load_tile(0);
  store_tile(0);
  if (LA == 2 && BKEY < kend) {
    load_tile(BKEY);
    store_tile(1);
  }
  if (LA * BKEY < kend) load_tile(LA * BKEY);
  __syncthreads();
  int t = 0;
  for (int j0 = 0; j0 < kend; j0 += BKEY, ++t) {
    const int buf = t % NB;
    if (j0 + LA * BKEY < kend) {
      // the buffer of block t + LA was last read by block t + LA - NB, before
      // the last barrier; the barrier after block t + LA - 1 publishes it
      store_tile((t + LA) % NB);
      if (j0 + (LA + 1) * BKEY < kend) load_tile(j0 + (LA + 1) * BKEY);
    }
    const bf16_t* Ks = reinterpret_cast<const bf16_t*>(smem + buf * BUF);
    const bf16_t* Vt = reinterpret_cast<const bf16_t*>(smem + buf * BUF + KBYTES);
    if (!causal || j0 <= wave_q0 + 31) {
      f32x16_t s[2];
      const f32x16_t zero = {};
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
        for (int kk = 0; kk < HD / 16; ++kk) {
          const bf16x8_t a = __builtin_bit_cast(
              bf16x8_t, *reinterpret_cast<const u32x4*>(Ks + (ks * 32 + l32) * KLD + kk * 16 + half * 8));
          s[ks] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[kk], kk == 0 ? zero : s[ks], 0, 0, 0);
        }
      }
      // s[ks][r]: query qrow, key j0 + 32 ks + 8 (r/4) + 4 half + r%4 (raw q.k)
      // masks only on the tiles that cross the sequence end or the diagonal
      if (j0 + BKEY > n || (causal && j0 + BKEY - 1 > wave_q0)) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int j = j0 + ks * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
            if (j >= n || (causal && j > qrow)) s[ks][r] = -INFINITY;
          }
      }
      float mloc = -INFINITY;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int r = 0; r < 16; ++r) mloc = fmaxf(mloc, s[ks][r]);
      mloc = half_swap_max(mloc);
      const float m_new = fmaxf(m_run, mloc);
      // The reference max moves (and the sums and accumulators are rescaled)
      // only when some query's max has grown by more than 2^8 in exp2 units
      // since the reference was set: probabilities stay below 256 (exact in
      // fp32, full relative precision in bf16), and since the output and the
      // log-sum-exp are both taken relative to the reference, the result is
      // the same for any reference. A row's first valid scores always move
      // it (from -inf). scale > 0, so the max of the scaled scores is the
      // scaled max.
      if (__builtin_amdgcn_ballot_w64(m_new == -INFINITY ? false
                                                         : !((m_new - m_run) * scale_log2 <= 8.0f)) != 0) {
        const float alpha = m_new == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f((m_run - m_new) * scale_log2);
        l_run *= alpha;
#pragma unroll
        for (int ct = 0; ct < HD / 32; ++ct)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[ct][r] *= alpha;
        m_run = m_new;
      }
      const float m_use = m_run == -INFINITY ? 0.f : m_run * scale_log2;
      float rsum = 0.f;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = __builtin_amdgcn_exp2f(fmaf(s[ks][r], scale_log2, -m_use));
          s[ks][r] = p;
          rsum += p;
        }
      rsum = half_swap_sum(rsum);
      l_run += rsum;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int ks = g >> 1, rb = (g & 1) * 8;
        const u32x4 pw = {pack_bf16x2(s[ks][rb], s[ks][rb + 1]), pack_bf16x2(s[ks][rb + 2], s[ks][rb + 3]),
                          pack_bf16x2(s[ks][rb + 4], s[ks][rb + 5]), pack_bf16x2(s[ks][rb + 6], s[ks][rb + 7])};
        const bf16x8_t pb = __builtin_bit_cast(bf16x8_t, pw);
        if constexpr (VTR) {
          // pb's slots 0..3 hold keys kb + 4 half + 0..3 and slots 4..7 keys
          // kb + 8 + 4 half + 0..3 (kb = 32 ks + 16 (g & 1)); the V^T
          // fragment gives channel ct * 32 + l32 the same keys in the same
          // slots: a 16-lane group's lanes point at key rows kb + 4 half + r
          // and channel runs 16 ((lane / 16) & 1) + 4 (lane & 3).
          const bf16_t* tr0 = Vt + (ks * 32 + (g & 1) * 16 + 4 * half + ((lane & 15) >> 2)) * KLD +
                              16 * ((lane >> 4) & 1) + 4 * (lane & 3);
#pragma unroll
          for (int ct = 0; ct < HD / 32; ++ct) {
            const bf16_t* vr = tr0 + ct * 32;
            const u32x4 av = lds_read_columns(vr, vr + 8 * KLD);
            o[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, av), pb, o[ct], 0, 0, 0);
          }
          continue;
        }
        // key chunks 8 ks + 4 (g & 1) + half and that + 2; the swizzle is even,
        // so it leaves half (the only lane-dependent part) alone and the
        // offsets stay immediates on one base address
        const bf16_t* vr0 = Vt + l32 * VLD + 4 * half;
#pragma unroll
        for (int ct = 0; ct < HD / 32; ++ct) {
          const bf16_t* vr = vr0 + ct * 32 * VLD;
          const int c0 = ks * 8 + (g & 1) * 4;
          const uint2 lo4 = *reinterpret_cast<const uint2*>(vr + 4 * (c0 ^ (VSW * ct)));
          const uint2 hi4 = *reinterpret_cast<const uint2*>(vr + 4 * ((c0 + 2) ^ (VSW * ct)));
          const u32x4 av = {lo4.x, lo4.y, hi4.x, hi4.y};
          o[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, av), pb, o[ct], 0, 0, 0);
        }
      }
    }
    if (t % LA == LA - 1) __syncthreads();
  }
  if (LA > 1) __syncthreads();  // every wave is past the tiles before the output staging reuses them

  // o[ct][r] = O^T[channel ct*32 + 8 (r/4) + 4 half + r%4][query qrow]
  const float inv_l = l_run > 0.f ? 1.0f / l_run : 0.f;
  bf16_t* Os = reinterpret_cast<bf16_t*>(smem) + wave * 32 * OLD;
#pragma unroll
  for (int ct = 0; ct < HD / 32; ++ct)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int c = ct * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
      Os[l32 * OLD + c] = f32_to_bf16(o[ct][r] * inv_l);
    }
  __syncthreads();
  for (int c = lane; c < 32 * HD / 8; c += 64) {
    const int r = c / (HD / 8), ch = (c % (HD / 8)) * 8;
    const int qr = q0 + wave * 32 + r;
    if (qr < n)
      *reinterpret_cast<u32x4*>(O + static_cast<int64_t>(lo + qr) * os + h * HD + ch) =
          *reinterpret_cast<const u32x4*>(Os + r * OLD + ch);
  }
  if (lse != nullptr && half == 0 && qrow < n)
    lse[static_cast<int64_t>(h) * T + lo + qrow] = (m_run * scale_log2 + log2f(l_run)) * kLn2;
}

// Longer sequences. A wave owns 32 QB queries (QB = 2 at head dim 64: each K
// and V fragment read from LDS serves two products; 1 at 128, whose output
// and query fragments fill the registers) and goes over the keys in steps of
// 32. In step u it issues the products S(u + 1) = K Q^T and O += V P(u - 1) one
// at a time with the exponentials, sums and packing of step u between them,
// in an order fixed by scheduling barriers: the matrix instruction takes 8
// passes after its issue, which the vector instructions of the same wave fill
// (probe: one product and 8 fma 18.5 ns interleaved at four waves per SIMD
// against 14.0 + 10.3 apart; with 8 exponentials 32 against 14 + 30). Two
// waves per SIMD: alone a wave issues a vector instruction every 5.6 cycles
// where several reach 2.7, and a form with 64 queries of head dim 128 on one
// wave per SIMD was slower (310 against 256 us on 8 x 2048 rows, 16 heads).
//  * No row max per step. P is taken relative to a reference, the max
//    over the first 64 keys; it moves (and O, the sum and this step's P are
//    redone) only when a lane's 16 probabilities sum to over 2^12, which any
//    one of them above that does. P up to 2^12 is exact enough: bf16 keeps
//    its relative precision, the sums are fp32, and output and log-sum-exp
//    are both taken relative to the reference.
//  * K and V tiles of 64 keys go straight to LDS, two tiles ahead, one
//    barrier per tile: staged through registers they cost 50 of 310 us (8 x
//    2048 rows, 16 heads of 128). Rows are unpadded; 16-byte chunk c of
//    row r lies at c ^ ksw(r) (K: the 16 rows of a read phase fall on all 64
//    banks) or c ^ vsw(r) (V: the four rows a transposing read takes do).
// Same box, us, this kernel against the register-staged one above in the same
// workgroup order: 4 x 4096 causal, 32 heads of 128, 543 / 603; 8 x 2048, 32
// heads of 64, 186 / 205 causal, 291 / 331 without; 32 x 512, 12 heads of 64,
// 37.2 / 40.7; 4 x 500 causal, 32 heads of 128, 20.7 / 22.7; and where it
// loses: 8 x 300 of 128 27.6 / 23.8, 32 x 256, 12 of 64, 17.9 / 17.4, 128 x
// 64 of 64 21.4 / 15.5 (graph replays, fresh outputs each call).
template <int HD, int QB, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_wide_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    int64_t rs, int kv_group, int causal, float scale_log2, const int32_t* __restrict__ cu,
    bf16_t* __restrict__ O, int64_t os, float* __restrict__ lse, int T, int H, int pairs) {
  constexpr int WQ = 32 * QB, BQ = WQ * NW, BK = 64;
  constexpr int KK = HD / 16, CT = HD / 32, CPR = HD / 8;
  constexpr int RB = HD * 2, HALF = BK * RB, BUF = 2 * HALF, NB = 3, OLD = HD + 8;
  constexpr int SBYTES = NB * BUF > NW * WQ * OLD * 2 ? NB * BUF : NW * WQ * OLD * 2;
  constexpr int RPL = 1024 / RB, LPW = HALF / 1024 / NW;  // rows per load, loads per wave and operand
  static_assert(LPW * NW * 1024 == HALF && NW % 4 == 0, "tile split");
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
  const int wq0 = q0 + wave * WQ;  // the wave's first query

  const int hk = h / kv_group;
  const uint32_t row_bytes = static_cast<uint32_t>(rs * 2);
  const uint32_t seq_bytes = static_cast<uint32_t>(n) * row_bytes;
  const u32x4 kres = buffer_resource(K + static_cast<int64_t>(lo) * rs + hk * HD, seq_bytes);
  const u32x4 vres = buffer_resource(V + static_cast<int64_t>(lo) * rs + hk * HD, seq_bytes);
  // K row r keeps its 16-byte chunk c at c ^ ksw(r), V row r at c ^ vsw(r)
  auto ksw = [](int r) { return HD == 64 ? (r >> 1) & 7 : r & 15; };
  auto vsw = [](int r) { return HD == 64 ? ((r >> 1) & 1) << 2 : (r & 3) << 2; };
  const int lrow = wave * RPL + lane / CPR;  // tile row of the wave's first load
  const uint32_t koff = lrow * row_bytes + (((lane % CPR) ^ ksw(lrow)) << 4);
  const uint32_t voff = lrow * row_bytes + (((lane % CPR) ^ vsw(lrow)) << 4);
  const uint32_t lds0 = lds_address(smem) + wave * 1024;
  auto load_tile = [&](int t, int buf) {
    const uint32_t t0 = static_cast<uint32_t>(t) * (BK * row_bytes);
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      const uint32_t d = lds0 + buf * BUF + i * (NW * 1024), so = t0 + i * (NW * RPL) * row_bytes;
      lds_load16(d, koff + so, kres);
      lds_load16(d + HALF, voff + so, vres);
    }
  };

  const int kend = causal ? min(n, q0 + BQ) : n;
  const int nt = (kend + BK - 1) / BK;
  // the wave's own tiles: under the causal mask none past its last query
  const int ntw = causal ? min(nt, (wq0 + WQ + BK - 1) / BK) : nt;
  load_tile(0, 0);
  if (nt > 1) load_tile(1, 1);

  bf16x8_t qf[QB][KK];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      // rows past the sequence are clamped, not zeroed: their outputs are not stored
      const int qr = min(wq0 + 32 * qb + l32, n - 1);
      qf[qb][kk] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(
                                                    Q + static_cast<int64_t>(lo + qr) * rs + h * HD + kk * 16 + half * 8));
    }

  float mu[QB], l_run[QB];  // reference max (scaled, exp2 units); sum over this lane's keys
  f32x16_t o[QB][CT], sa[QB], sb[QB];
  bf16x8_t pf[QB][2];  // P of the last step: [query block][16 keys]
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    l_run[qb] = 0.f;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[qb][ct][r] = 0.f;
  }

  // fragment addresses within a tile: K rows l32 (+ 32), chunk 2 kk + half;
  // V key rows 4 half + r (+ 8, 16 ..), the channel runs of a transposing read
  const uint32_t kf0 = l32 * RB, vrow = 4 * half + ((lane & 15) >> 2);
  const int ks0 = ksw(l32), vs0 = vsw(vrow);
  const uint32_t vf0 = HALF + vrow * RB + (lane & 1) * 8;
  const int vch = 2 * ((lane >> 4) & 1) + ((lane >> 1) & 1);
  uint32_t kaddr[KK], vaddr[CT];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) kaddr[kk] = kf0 + (((2 * kk + half) ^ ks0) << 4);
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) vaddr[ct] = vf0 + (((4 * ct + vch) ^ vs0) << 4);
  auto read_k = [&](const unsigned char* base, int kk) {
    return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4*>(base + kaddr[kk]));
  };
  auto read_v = [&](const unsigned char* base, int g, int ct) {
    const unsigned char* vr = base + vaddr[ct] + g * (16 * RB);
    return __builtin_bit_cast(bf16x8_t, lds_read_columns(vr, vr + 8 * RB));
  };
  const f32x16_t zero = {};
  auto row_max = [&](const f32x16_t& s) {
    float mx = fmaxf(fmaxf(s[0], s[1]), s[2]);
#pragma unroll
    for (int r = 3; r < 15; r += 2) mx = fmaxf(fmaxf(mx, s[r]), s[r + 1]);
    return half_swap_max(fmaxf(mx, s[15]));
  };
  auto mask = [&](int u, f32x16_t (&s)[QB]) {
    const int j0 = 32 * u;
    if (j0 + 32 <= n && !(causal && j0 + 31 > wq0)) return;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      // keys from this lane's limit on are masked
      int lim = (causal ? min(n, wq0 + 32 * qb + l32 + 1) : n) - j0 - 4 * half;
      asm("" : "+v"(lim));  // the comparisons stay here (hoisted, their masks fill the scalar registers)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (8 * (r >> 2) + (r & 3) >= lim) s[qb][r] = -INFINITY;
    }
  };
  // one step: the exponentials of step u (scores s) beside the products of
  // O += V P(u - 1) and S(u + 1) = sn (the first step: alone)
  auto step = [&](int u, int bufn, int ksn, int bufp, int ksp, f32x16_t (&s)[QB], f32x16_t (&sn)[QB], auto first_c) {
    constexpr bool first = decltype(first_c)::value;
    if (!first) mask(u, s);
    constexpr int FA = 2;                                   // fragments in flight ahead of their use
    constexpr int NF = KK + 2 * CT, NS = QB * NF;           // operand fragments, matrix instructions
    constexpr int NU = 16 * QB;                             // pieces of vector work
    const unsigned char* kp = smem + bufn * BUF + ksn * (32 * RB);
    const unsigned char* vp = smem + bufp * BUF + ksp * (32 * RB);
    bf16x8_t fr[FA + 1];
    auto read = [&](int f) { fr[f % (FA + 1)] = f < KK ? read_k(kp, f) : read_v(vp, (f - KK) / CT, (f - KK) % CT); };
    auto product = [&](int i) {
      const int f = i / QB, qb = i % QB;
      if (f < KK)
        sn[qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[f % (FA + 1)], qf[qb][f], f == 0 ? zero : sn[qb], 0, 0, 0);
      else
        o[qb][(f - KK) % CT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            fr[f % (FA + 1)], pf[qb][(f - KK) / CT], o[qb][(f - KK) % CT], 0, 0, 0);
    };
    float rsum[QB], a0 = 0.f, a1 = 0.f, p0 = 0.f, p1 = 0.f;
    u32x4 pn[QB][2];
    auto work = [&](int w) {
      const int qb = w >> 4, r = w & 14;
      if ((w & 1) == 0) {
        p0 = __builtin_amdgcn_exp2f(fmaf(s[qb][r], scale_log2, -mu[qb]));
        p1 = __builtin_amdgcn_exp2f(fmaf(s[qb][r + 1], scale_log2, -mu[qb]));
        asm volatile("" : "+v"(p0), "+v"(p1));  // computed here, beside this step's products
      } else {
        uint32_t pw = pack_bf16x2(p0, p1);
        a0 = r == 0 ? p0 : a0 + p0;
        a1 = r == 0 ? p1 : a1 + p1;
        asm volatile("" : "+v"(pw), "+v"(a0), "+v"(a1));
        pn[qb][r >> 3][(r >> 1) & 3] = pw;
        if (r == 14) rsum[qb] = a0 + a1;
      }
    };
    if constexpr (first) {
#pragma unroll
      for (int k = 0; k < NU; ++k) work(k);
    } else {
#pragma unroll
      for (int f = 0; f < FA; ++f) read(f);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        if (i % QB == 0 && i / QB + FA < NF) read(i / QB + FA);
        product(i);
#pragma unroll
        for (int k = NU * i / NS; k < NU * (i + 1) / NS; ++k) work(k);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    bool high = false;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) high |= !(rsum[qb] <= 4096.f);
    if (!first && __builtin_amdgcn_ballot_w64(high) != 0) {
      // a score far above the reference: move it, and redo this step's P
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        const float m_new = fmaxf(mu[qb], row_max(s[qb]) * scale_log2);
        const float alpha = __builtin_amdgcn_exp2f(mu[qb] - m_new);
        mu[qb] = m_new;
        l_run[qb] *= alpha;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[qb][ct][r] *= alpha;
        rsum[qb] = 0.f;
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          const float e0 = __builtin_amdgcn_exp2f(fmaf(s[qb][r], scale_log2, -m_new));
          const float e1 = __builtin_amdgcn_exp2f(fmaf(s[qb][r + 1], scale_log2, -m_new));
          rsum[qb] += e0 + e1;
          pn[qb][r >> 3][(r >> 1) & 3] = pack_bf16x2(e0, e1);
        }
      }
    }
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      l_run[qb] += rsum[qb];
      pf[qb][0] = __builtin_bit_cast(bf16x8_t, pn[qb][0]);
      pf[qb][1] = __builtin_bit_cast(bf16x8_t, pn[qb][1]);
    }
  };

  int bp = 2, bc = 0, bn = 1;  // buffers of tiles t - 1, t, t + 1
  auto turn = [&]() {
    const int f = bp;
    bp = bc;
    bc = bn;
    bn = f;
  };
  turn_over();
  // the first tile's scores, and the reference: the max over its 64 keys
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const bf16x8_t a0 = read_k(smem, kk), a1 = read_k(smem + 32 * RB, kk);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      sa[qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, qf[qb][kk], kk == 0 ? zero : sa[qb], 0, 0, 0);
      sb[qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, qf[qb][kk], kk == 0 ? zero : sb[qb], 0, 0, 0);
    }
  }
  mask(0, sa);
  mask(1, sb);
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
    mu[qb] = fmaxf(fmaxf(row_max(sa[qb]), row_max(sb[qb])) * scale_log2, -1e30f);
  step(0, bc, 1, bp, 1, sa, sb, std::true_type());
  if (nt > 2) load_tile(2, bp);
  step(1, bn, 0, bc, 0, sb, sa, std::false_type());
  int t = 1;
  for (; t < ntw; ++t) {
    turn();
    step(2 * t, bc, 1, bp, 1, sa, sb, std::false_type());
    turn_over();
    if (t + 2 < nt) load_tile(t + 2, bp);
    step(2 * t + 1, bn, 0, bc, 0, sb, sa, std::false_type());
  }
#pragma unroll
  for (int g = 0; g < 2; ++g)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const bf16x8_t a = read_v(smem + bc * BUF + 32 * RB, g, ct);
#pragma unroll
      for (int qb = 0; qb < QB; ++qb)
        o[qb][ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pf[qb][g], o[qb][ct], 0, 0, 0);
    }
  for (; t < nt; ++t) {  // the tiles of the block's later queries
    turn();
    turn_over();
    if (t + 2 < nt) load_tile(t + 2, bp);
  }
  turn_over();  // every wave is past the tiles before the output staging reuses them

  // o[qb][ct][r] = O^T[channel ct*32 + 8 (r/4) + 4 half + r%4][query wq0 + 32 qb + l32]
  bf16_t* Os = reinterpret_cast<bf16_t*>(smem) + wave * WQ * OLD;
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const float l = half_swap_sum(l_run[qb]);
    const float inv_l = l > 0.f ? 1.0f / l : 0.f;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int r = 0; r < 16; r += 4) {
        const uint2 w = {pack_bf16x2(o[qb][ct][r] * inv_l, o[qb][ct][r + 1] * inv_l),
                         pack_bf16x2(o[qb][ct][r + 2] * inv_l, o[qb][ct][r + 3] * inv_l)};
        *reinterpret_cast<uint2*>(Os + (32 * qb + l32) * OLD + ct * 32 + 2 * r + 4 * half) = w;
      }
    const int qrow = wq0 + 32 * qb + l32;
    if (lse != nullptr && half == 0 && qrow < n)
      lse[static_cast<int64_t>(h) * T + lo + qrow] = (mu[qb] + log2f(l)) * kLn2;
  }
  // each wave stores its own rows: its LDS writes are in order before its reads
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  for (int c = lane; c < WQ * CPR; c += 64) {
    const int r = c / CPR, ch = (c % CPR) * 8;
    const int qr = wq0 + r;
    if (qr < n)
      *reinterpret_cast<u32x4*>(O + static_cast<int64_t>(lo + qr) * os + h * HD + ch) =
          *reinterpret_cast<const u32x4*>(Os + r * OLD + ch);
  }
}

// fp32 storage (and bf16 at head dims 16 and 32): every product on
// v_mfma_f32_32x32x2_f32, fp32 operands and sums. One workgroup of four
// waves per (32 queries, head, sequence); the waves take the 32-key tiles in
// turn and their (max, sum, O) are merged through LDS in wave order, so a
// short sequence still spreads over the four SIMDs. The matrix instruction
// is slow enough (64 cycles for 4096 FLOP) that operands come straight from
// memory: 16 bytes of a K row a lane, and single V elements, 32 consecutive
// channels of a row a half-wave. S^T = K Q^T leaves a lane with 16 keys of
// one query, which is the B operand of O^T += V^T P^T (the two keys of a
// step are those of the two lane halves). The exponentials are expf: the
// hardware one of an argument multiplied by log2 e in fp32 is off by 2^-24
// times that argument (2e-6 at e^-40), and saves 0.4 of 5.8 and 1.4 of 22.2 us.
// A vector-ALU kernel with one query per thread held this place: 37.1 us on 4 x
// 64 rows, 4 heads of 32, and 256 us on 8 ragged sequences of up to 200 rows,
// 12 heads of 64 (now 5.8 and 22.2).
template <typename T, int HD>
__global__ __launch_bounds__(256) void attn_f32_kernel(const T* __restrict__ Q,
                                                       const T* __restrict__ K,
                                                       const T* __restrict__ V, int64_t rs,
                                                       int kv_group, int causal, float scale,
                                                       const int32_t* __restrict__ cu,
                                                       T* __restrict__ O, int64_t os,
                                                       float* __restrict__ lse, int Tn) {
  constexpr int NW = 4, KK = HD / 8;
  constexpr int CT = HD < 32 ? 1 : HD / 32;  // 32-channel blocks of O (half empty at HD 16)
  constexpr int HP = 33;                     // merge row stride: [channel][query]
  __shared__ float so[NW][HD * HP];
  __shared__ float sm[NW][32], sl[NW][32];
  const int b = blockIdx.z, h = blockIdx.y;
  const int lo = cu[b];
  const int n = cu[b + 1] - lo;
  const int nqb = (n + 31) / 32;
  if (static_cast<int>(blockIdx.x) >= nqb) return;
  const int qb = causal ? nqb - 1 - static_cast<int>(blockIdx.x) : static_cast<int>(blockIdx.x);
  const int q0 = qb * 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, l32 = lane & 31;
  const int qrow = q0 + l32;
  const T* kb = K + static_cast<int64_t>(lo) * rs + (h / kv_group) * HD;
  const T* vb = V + static_cast<int64_t>(lo) * rs + (h / kv_group) * HD;
  const bool vch = HD >= 32 || l32 < HD;  // lanes whose channel exists
  float4 qf[KK];
#pragma unroll
  for (int s = 0; s < KK; ++s)
    qf[s] = load4<T>(Q + static_cast<int64_t>(lo + min(qrow, n - 1)) * rs + h * HD + 8 * s + 4 * half);
  float m_run = -INFINITY, l_run = 0.f;  // of the scaled scores; l_run: this lane's keys only
  f32x16_t o[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[ct][r] = 0.f;
  const int kend = causal ? min(n, q0 + 32) : n;
  for (int j0 = wave * 32; j0 < kend; j0 += 32 * NW) {
    float vr[CT][16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      // rows past the sequence count as zeros (their probability is 0)
      const int j = j0 + 8 * (r >> 2) + 4 * half + (r & 3);
      const T* vp = vb + static_cast<int64_t>(min(j, n - 1)) * rs;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
        vr[ct][r] = j < n && vch ? to_f32(vp[ct * 32 + (HD < 32 ? l32 % HD : l32)]) : 0.f;
    }
    f32x16_t s = {};
    const T* kp = kb + static_cast<int64_t>(min(j0 + l32, n - 1)) * rs + 4 * half;
#pragma unroll
    for (int t = 0; t < KK; ++t) {
      const float4 k4 = load4<T>(kp + 8 * t);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(k4.x, qf[t].x, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(k4.y, qf[t].y, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(k4.z, qf[t].z, s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f32_32x32x2f32(k4.w, qf[t].w, s, 0, 0, 0);
    }
    // s[r]: key j0 + 8 (r/4) + 4 half + r%4, query qrow
    const bool edge = j0 + 32 > n || (causal && j0 + 31 > q0);
    float mloc = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = j0 + 8 * (r >> 2) + 4 * half + (r & 3);
      s[r] = edge && (j >= n || (causal && j > qrow)) ? -INFINITY : s[r] * scale;
      mloc = fmaxf(mloc, s[r]);
    }
    mloc = half_swap_max(mloc);
    const float m_new = fmaxf(m_run, mloc);
    if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {
      const float alpha = m_new == -INFINITY ? 1.0f : expf(m_run - m_new);
      l_run *= alpha;
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[ct][r] *= alpha;
      m_run = m_new;
    }
    const float m_use = m_run == -INFINITY ? 0.f : m_run;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = expf(s[r] - m_use);
      l_run += s[r];
    }
    // A masked key's V row must not reach a query that cannot see it, also
    // where it holds an infinity or a NaN, which a product with its zero
    // probability would spread. Such rows are rare: the tile then goes
    // through the vector ALU, key by key.
    bool odd = false;
    if (edge && causal) {
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int r = 0; r < 16; ++r) odd |= !(fabsf(vr[ct][r]) <= 3.402823466e38f);
      odd = __builtin_amdgcn_ballot_w64(odd) != 0;
    }
    if (!odd) {
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          o[ct] = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[ct][r], s[r], o[ct], 0, 0, 0);
    } else {
#pragma unroll
      for (int kk = 0; kk < 32; ++kk) {
        // key j0 + kk: register (kk / 8) * 4 + kk % 4 of lane half (kk / 4) % 2
        const float p = __shfl(s[(kk >> 3) * 4 + (kk & 3)], l32 + 32 * ((kk >> 2) & 1), 64);
        if (j0 + kk <= qrow && j0 + kk < n) {
          const T* vp = vb + static_cast<int64_t>(j0 + kk) * rs;
#pragma unroll
          for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const int c = ct * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
              if (c < HD) o[ct][r] = fmaf(p, to_f32(vp[c]), o[ct][r]);
            }
        }
      }
    }
  }
  l_run = half_swap_sum(l_run);
  if (half == 0) {
    sm[wave][l32] = m_run;
    sl[wave][l32] = l_run;
  }
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int c = ct * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
      if (c < HD) so[wave][c * HP + l32] = o[ct][r];
    }
  __syncthreads();
  for (int it = tid; it < 32 * (HD / 4); it += 64 * NW) {
    const int q = it / (HD / 4), c0 = (it % (HD / 4)) * 4;
    if (q0 + q >= n) continue;
    float m = sm[0][q];
#pragma unroll
    for (int w = 1; w < NW; ++w) m = fmaxf(m, sm[w][q]);
    float l = 0.f, v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      // a wave without keys for this query holds the empty sum
      if (sm[w][q] == -INFINITY && sl[w][q] == 0.f) continue;
      const float f = expf(sm[w][q] - (m == -INFINITY ? 0.f : m));
      l = fmaf(f, sl[w][q], l);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = fmaf(f, so[w][(c0 + e) * HP + q], v[e]);
    }
    const float inv = 1.0f / l;
    T* op = O + static_cast<int64_t>(lo + q0 + q) * os + h * HD + c0;
#pragma unroll
    for (int e = 0; e < 4; ++e) op[e] = from_f32<T>(v[e] * inv);
    if (c0 == 0 && lse != nullptr) lse[static_cast<int64_t>(h) * Tn + lo + q0 + q] = m + logf(l);
  }
}

template <typename T>
hipError_t f32_dispatch(hipStream_t s, const void* q, const void* k, const void* v, int64_t rs,
                         int H, int kvg, int hd, int causal, float scale, int B, int max_len, int Trows,
                         const int32_t* cu, void* out, int64_t os, float* lse) {
  const dim3 grid((max_len + 31) / 32, H, B), block(256);
  const T* qp = static_cast<const T*>(q);
  const T* kp = static_cast<const T*>(k);
  const T* vp = static_cast<const T*>(v);
  T* op = static_cast<T*>(out);
  switch (hd) {
    case 16: return launch(K_ATTENTION, attn_f32_kernel<T, 16>, grid, block, 0, s, qp, kp, vp, rs, kvg, causal, scale, cu, op, os, lse, Trows);
    case 32: return launch(K_ATTENTION, attn_f32_kernel<T, 32>, grid, block, 0, s, qp, kp, vp, rs, kvg, causal, scale, cu, op, os, lse, Trows);
    case 64: return launch(K_ATTENTION, attn_f32_kernel<T, 64>, grid, block, 0, s, qp, kp, vp, rs, kvg, causal, scale, cu, op, os, lse, Trows);
    case 128: return launch(K_ATTENTION, attn_f32_kernel<T, 128>, grid, block, 0, s, qp, kp, vp, rs, kvg, causal, scale, cu, op, os, lse, Trows);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// Whether attn_wide_kernel takes the call: from the lengths on at which it
// pays (its comment), but not where the grid of 256-query blocks leaves CUs
// with one workgroup or none and the other kernel's waves wait less. us, the
// other kernel / this one, head dim 64 under the mask: 12 heads, 1 x 500 rows
// 13.3 / 14.7, 8 x 400 (192 workgroups) 13.3 / 14.2, 16 x 300 (384) 15.7 /
// 15.0; 32 heads, 4 x 500 (256) 15.4 / 16.5, 8 x 400 (512) 19.7 / 18.8;
// without it the two are alike there (12 heads, 1 x 500 13.7 / 13.6, 1 x 2048
// 40.2 / 39.6) and from one workgroup per CU on this one is ahead (32 heads, 1
// x 2048 48.3 / 46.6). Head dim 128 up to 512 rows, 16 heads: 1 x 500 (32
// workgroups) 15.8 / 16.9, 4 x 500 (128) 17.4 / 18.4, 8 x 400 (256) 23.7 /
// 20.4; past 512 rows it is ahead on any grid (1 x 1000 34.5 / 27.6).
bool attention_wide(int hd, int H, int B, int max_len, int causal, int cus) {
  const int64_t wgs = (static_cast<int64_t>(max_len) + 255) / 256 * H * B;
  if (hd == 64) return max_len > 256 && (!causal || wgs > cus);
  return max_len > 384 && (max_len > 512 || wgs >= cus);
}

hipError_t launch_attention(hipStream_t s, int dtype, const void* q, const void* k,
                            const void* v, int64_t row_stride, int H, int kv_group, int hd,
                            int causal, float scale, int B, int max_len, int T,
                            const int32_t* cu_dev, void* out, int64_t out_stride, float* lse) {
  if (B == 0 || max_len == 0) return hipSuccess;
  if (dtype == 1 && (hd == 64 || hd == 128)) {
    const float sl = scale * kLog2e;
    // Heads of 128 that share no keys: an XCD with 80 pairs or more walks
    // eight at a time (place_grid). us, all of them / eight, causal, 32 heads:
    // 80 x 380 rows 327 / 256, 160 x 200 307 / 254, 48 x 512 234 / 198, 20 x 1024
    // 252 / 220; with fewer pairs the tail of each eight costs more (32 heads
    // on 8, 8 x 300 23.5 / 28.0; 16 heads, 16 x 257 25.9 / 28.3). Head dim 64, half
    // the bytes a pair, 32 heads: 48 x 512 112 / 121, 20 x 1024 126 / 131.
    const int most = hd == 128 && kv_group == 1 ? 8 : 0;
    auto go = [&](auto kernel, int bq, int threads) {
      const PlaceGrid at = place_grid(H, kv_group, B, max_len, T, causal, bq, most);
      return launch(K_ATTENTION, kernel, at.grid, dim3(threads), 0, s,
                    static_cast<const bf16_t*>(q), static_cast<const bf16_t*>(k),
                    static_cast<const bf16_t*>(v), row_stride, kv_group, causal, sl, cu_dev,
                    static_cast<bf16_t*>(out), out_stride, lse, T, H, at.pairs);
    };
    const bool wide = attention_wide(hd, H, B, max_len, causal, device_cu_count());
    if (hd == 64) {
      if (wide) return go(attn_wide_kernel<64, 2, 4>, 256, 256);
      if (max_len > 128) return go(attn_mfma_kernel<64, 8>, 256, 512);
      return go(attn_mfma_kernel<64, 4>, 128, 256);
    }
    if (wide) return go(attn_wide_kernel<128, 1, 8>, 256, 512);
    return go(attn_mfma_kernel<128, 4>, 128, 256);
  }
  if (dtype == 1)
    return f32_dispatch<bf16_t>(s, q, k, v, row_stride, H, kv_group, hd, causal, scale, B,
                                 max_len, T, cu_dev, out, out_stride, lse);
  return f32_dispatch<float>(s, q, k, v, row_stride, H, kv_group, hd, causal, scale, B, max_len,
                              T, cu_dev, out, out_stride, lse);
}

}  // namespace zsa
