// Host checks of how calls are laid out on the GPU and which kernel takes
// them: launch grids within HIP's limits, every block of work reached exactly
// once. Prints "ok <checks>" and exits 0 when every check holds.
#include <stdio.h>
#include <stdlib.h>

#include <vector>

#include "../../paper_2509_01190_amd/csrc/zsa_internal.h"

namespace {

int g_checks = 0;

void check(bool ok, const char* what, int line) {
  ++g_checks;
  if (!ok) {
    fprintf(stderr, "check failed (line %d): %s\n", line, what);
    exit(1);
  }
}
#define CHECK_TRUE(cond) check((cond), #cond, __LINE__)

// every (sequence, head, block) has exactly one workgroup of a legal grid
void check_place(int H, int B, int max_len, int T, int causal, int block, int most = 0) {
  fprintf(stderr, "place: %d heads, %d sequences of up to %d rows, %d in all, causal %d, blocks of %d\n", H, B,
          max_len, T, causal, block);
  const int blocks = (max_len + block - 1) / block;
  for (int first = 0; first < 2; ++first) {
    const int group = first && H % 2 == 0 ? 2 : 1;
    const zsa::PlaceGrid pg = zsa::place_grid(H, group, B, max_len, T, causal, block, most);
    const dim3 g = pg.grid;
    CHECK_TRUE(g.y <= 65535 && g.z <= 65535 && 512ull * g.x <= 0xffffffffull);
    std::vector<unsigned char> hit(static_cast<size_t>(B) * H * blocks, 0);
    for (uint32_t z = 0; z < g.z; ++z)
      for (uint32_t y = 0; y < g.y; ++y)
        for (uint32_t x = 0; x < g.x; ++x) {
          zsa::Place at;
          if (!zsa::place_at(g, dim3(x, y, z), H, group, pg.pairs, first != 0, &at)) continue;
          if (at.i >= blocks) continue;  // past every sequence: the kernels return
          if (at.b < 0 || at.b >= B || at.h < 0 || at.h >= H || at.i < 0) CHECK_TRUE(!"out of range");
          if (hit[(static_cast<size_t>(at.b) * H + at.h) * blocks + at.i]++) CHECK_TRUE(!"reached twice");
        }
    for (unsigned char h : hit)
      if (!h) CHECK_TRUE(!"not reached");
    ++g_checks;
  }
}

void places() {
  for (int causal = 0; causal < 2; ++causal) {
    for (int H : {1, 3, 7, 8, 12, 16, 32}) {
      check_place(H, 1, 1, 1, causal, 128);
      check_place(H, 5, 300, 5 * 300, causal, 128);
      check_place(H, 5, 300, 5 * 300 - 7, causal, 256);
      check_place(H, 33, 1000, 33 * 1000, causal, 128);
      check_place(H, 33, 1000, 33 * 1000 - 5, causal, 128, 8);
      check_place(H, 700, 300, 700 * 300 - 5, causal, 128, 8);
    }
    // as many sequences as a grid's z once held, one pair of rows each
    check_place(12, 65535, 2, 2 * 65535, causal, 128);
    check_place(7, 65535, 2, 2 * 65535, causal, 256);
    check_place(2, 65535, 3, 3 * 65535, causal, 256);
    check_place(16, 43700, 1, 43700, causal, 128);
    check_place(12, 65535, 2, 2 * 65535, causal, 128, 8);
    // one sequence of more blocks than a grid's y holds
    check_place(1, 1, 9000000, 9000000, causal, 128);
    check_place(3, 2, 8388481, 8388482, causal, 128);
  }
}

// An XCD (workgroup number mod 8) takes neighbouring heads where they share
// key/value heads, and every eighth one where they share nothing
void head_order() {
  const int H = 32, B = 4;
  for (int rows : {128, 300})  // one block: heads that share nothing keep their own order
    for (int group : {1, 4}) {
      const zsa::PlaceGrid pg = zsa::place_grid(H, group, B, rows, B * rows, 0, 128);
      const dim3 g = pg.grid;
      CHECK_TRUE((pg.pairs < 0) == (rows == 128 && group == 1));
      for (uint32_t z = 0; z < g.z; ++z)
        for (uint32_t y = 0; y < g.y; ++y)
          for (uint32_t x = 0; x < g.x; ++x) {
            zsa::Place at;
            if (!zsa::place_at(g, dim3(x, y, z), H, group, pg.pairs, false, &at)) continue;
            const uint32_t xcd = (x + g.x * (y + g.y * z)) % 8;
            CHECK_TRUE(static_cast<int>(xcd) == (group == 1 ? at.h % 8 : at.h / (H / 8)));
          }
    }
}

// Long sequences of several lengths without a mask: no XCD gets more than 1.2
// times its share of the blocks that have rows, however the lengths alternate
void long_ragged() {
  const int longest = 2494, B = 16, block = 128;
  for (int H : {4, 6, 8, 12, 20})
    for (int period : {2, 4}) {
      auto len = [&](int b) { return b % period == 0 ? longest : 300; };
      int T = 0;
      for (int b = 0; b < B; ++b) T += len(b);
      const zsa::PlaceGrid pg = zsa::place_grid(H, 1, B, longest, T, 0, block);
      const dim3 g = pg.grid;
      int per_xcd[8] = {}, all = 0;
      for (uint32_t z = 0; z < g.z; ++z)
        for (uint32_t y = 0; y < g.y; ++y)
          for (uint32_t x = 0; x < g.x; ++x) {
            zsa::Place at;
            if (!zsa::place_at(g, dim3(x, y, z), H, 1, pg.pairs, false, &at) || at.i * block >= len(at.b)) continue;
            ++per_xcd[(x + g.x * (y + g.y * z)) % 8];
            ++all;
          }
      fprintf(stderr, "long ragged: %d heads, every %dth sequence long\n", H, period);
      for (int n : per_xcd) CHECK_TRUE(8 * n <= 1.2 * all);
    }
}

// Equal sequences without a mask: no workgroup without work but for the pairs
// that fill up the XCDs' last one
void no_gaps() {
  for (int H : {1, 3, 8, 12, 16, 20, 24, 32})
    for (int B : {1, 2, 5, 33}) {
      const zsa::PlaceGrid g = zsa::place_grid(H, 2, B, 300, B * 300, 0, 128);
      if (g.pairs < 0) CHECK_TRUE((H * B + 7) / 8 * 8 - H * B > H * B / 20);
      else CHECK_TRUE(g.grid.x / 8 * g.grid.z == static_cast<uint32_t>((H * B + 7) / 8));
    }
}

// Which kernel takes a bf16 product of few output tiles (256 CUs)
void products() {
  using namespace zsa;
  auto ep = [](int epi, int head_dim) {
    EpiParams e{};
    e.epi = epi;
    e.head_dim = head_dim;
    return e;
  };
  struct Case { int M, N, K, epi, head_dim; bool few_row; ShortGrid split, whole; };
  const Case cases[] = {
      {16, 768, 768, EPI_NONE, 0, true, kShort64, kShort64},
      // either side of 150 64 x 64 tiles
      {640, 768, 3072, EPI_RESIDUAL, 0, true, kShort64, kShort64},
      {800, 768, 3072, EPI_RESIDUAL, 0, false, kShort64, kShort64},
      {300, 2304, 768, EPI_ROPE, 64, false, kShort64, kShort64},
      {300, 1856, 1024, EPI_NONE, 0, true, kShort64, kShort64},
      {1000, 576, 768, EPI_GELU, 0, true, kShort64, kShort64},
      // past two 64 x 64 tiles per CU, and past one 128 x 128
      {4000, 768, 3072, EPI_RESIDUAL, 0, false, kShort128, kShort128},
      {6001, 768, 3072, EPI_NONE, 0, false, kNoShort, kNoShort},
      {1100, 384, 4608, EPI_NONE, 0, false, kNoShort, kShort64},
      {2100, 768, 4160, EPI_NONE, 0, false, kNoShort, kShort128x64},
      {2500, 2048, 8192, EPI_NONE, 0, false, kNoShort, kNoShort},
      // few columns and a long K: either side of (K / 64)^2 / 64 tiles of 64 x 64
      {1616, 64, 3520, EPI_RESIDUAL, 0, false, kNoShort, kShort64},
      {1616, 128, 3072, EPI_NONE, 0, false, kShort64, kShort64},
      {4096, 64, 4096, EPI_NONE, 0, false, kNoShort, kShort64},
      {2100, 128, 4096, EPI_NONE, 0, false, kShort64, kShort64},
      // K = 4096: either side of 0.6 of a 128 x 128 tile per CU
      {2100, 1024, 4096, EPI_NONE, 0, false, kNoShort, kShort128},
      {4096, 640, 4096, EPI_NONE, 0, false, kShort128, kShort128},
      // K no multiple of 64: no tiled bf16 kernel takes it
      {640, 768, 3104, EPI_NONE, 0, true, kNoShort, kNoShort},
      {800, 768, 3104, EPI_NONE, 0, true, kNoShort, kNoShort},
      {300, 2304, 800, EPI_NONE, 0, true, kNoShort, kNoShort},
      // rotary heads of 128 lie in no 64-wide tile
      {65, 6144, 4096, EPI_ROPE, 128, true, kNoShort, kShort128},
      {128, 6144, 4096, EPI_ROPE, 128, true, kNoShort, kShort128},
      {256, 3072, 1024, EPI_ROPE, 128, true, kNoShort, kNoShort},
      {128, 12288, 4096, EPI_ROPE, 128, false, kNoShort, kShort128},
      {512, 6144, 4096, EPI_ROPE, 128, false, kNoShort, kShort128},
      {1100, 2048, 4160, EPI_NONE, 0, false, kNoShort, kShort128},
  };
  for (const Case& c : cases) {
    fprintf(stderr, "product: %d x %d x %d, epilogue %d, heads of %d\n", c.M, c.N, c.K, c.epi, c.head_dim);
    const EpiParams e = ep(c.epi, c.head_dim);
    CHECK_TRUE(gemm_takes_skinny(1, c.M, c.N, c.K, e) == c.few_row);
    CHECK_TRUE(short_grid(c.M, c.N, c.K, e, true) == c.split);
    CHECK_TRUE(short_grid(c.M, c.N, c.K, e, false) == c.whole);
  }
}

// Which attention kernel takes a call (256 CUs)
void attentions() {
  using zsa::attention_wide;
  // head dim 64: past 256 rows, under the mask from more than one workgroup per CU on
  CHECK_TRUE(!attention_wide(64, 12, 64, 256, 0, 256) && !attention_wide(64, 12, 64, 256, 1, 256));
  CHECK_TRUE(attention_wide(64, 12, 1, 257, 0, 256) && attention_wide(64, 12, 16, 257, 1, 256));
  CHECK_TRUE(!attention_wide(64, 12, 8, 500, 1, 256) && !attention_wide(64, 32, 4, 500, 1, 256));
  CHECK_TRUE(attention_wide(64, 32, 8, 300, 1, 256) && attention_wide(64, 32, 8, 2048, 1, 256));
  // head dim 128: past 512 rows, past 384 from one workgroup per CU on
  CHECK_TRUE(!attention_wide(128, 32, 64, 384, 1, 256) && !attention_wide(128, 32, 1, 500, 0, 256));
  CHECK_TRUE(!attention_wide(128, 16, 4, 500, 1, 256) && attention_wide(128, 16, 8, 400, 1, 256));
  CHECK_TRUE(attention_wide(128, 1, 1, 513, 0, 256));
}

// Which score kernel takes a call (256 CUs)
void scores() {
  using zsa::score_wide;
  CHECK_TRUE(score_wide(64, 12, 43, 20, 43 * 20, 0, 256) && !score_wide(64, 12, 42, 20, 42 * 20, 0, 256));
  CHECK_TRUE(score_wide(128, 32, 4, 500, 4 * 500, 0, 256) && !score_wide(128, 32, 3, 500, 3 * 500, 0, 256));
  CHECK_TRUE(score_wide(64, 20, 3, 2344, 3 * 2344, 0, 256) && !score_wide(64, 20, 3, 2344, 4681, 0, 256));
  CHECK_TRUE(score_wide(128, 16, 8, 500, 2450, 0, 256));
  CHECK_TRUE(score_wide(128, 4, 8, 2553, 8 * 2553, 0, 256) && !score_wide(128, 4, 8, 2553, 12600, 0, 256));
  // long sequences under the mask, heads of 128: from 1.6 workgroups with keys per CU on
  CHECK_TRUE(score_wide(128, 12, 3, 3300, 3 * 3300, 1, 256) && !score_wide(128, 12, 2, 3300, 2 * 3300, 1, 256));
  CHECK_TRUE(score_wide(128, 12, 2, 3300, 2 * 3300, 0, 256) && !score_wide(128, 6, 6, 3300, 12000, 1, 256));
  CHECK_TRUE(score_wide(128, 32, 4, 1000, 4 * 1000, 1, 256) && score_wide(64, 12, 4, 3300, 4 * 3300, 1, 256));
}

}  // namespace

int main() {
  places();
  long_ragged();
  head_order();
  no_gaps();
  products();
  attentions();
  scores();
  printf("ok %d\n", g_checks);
  return 0;
}
