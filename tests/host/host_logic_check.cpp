// Host check of libbpd's sizing and dispatch logic (paper_1811_03115_amd/csrc/bpd_host_logic.h) on many random
// configurations inside what bpd_create accepts: workspace regions are aligned, disjoint and inside the reported size;
// the staging area holds the largest tensor bpd_load_weights may stage; key / slice / partial-result buffers hold what
// the launches write into them; the tile rule only returns tiles the library instantiates.
// Built by tests/test_host_logic.py with the system compiler under -fsanitize=address,undefined.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
#include <utility>

#include "../../paper_1811_03115_amd/csrc/bpd_host_logic.h"
#include "../../paper_1811_03115_amd/csrc/bpd_tile_map.h"

static long bad = 0;
#define EXPECT(cond, ...) do { if (!(cond)) { ++bad; if (bad < 20) { fprintf(stderr, "violated: %s  [", #cond); fprintf(stderr, __VA_ARGS__); fprintf(stderr, "]\n"); } } } while (0)

// tiles (rows / 16, columns / 64) the LDS-staged GEMM is instantiated for (the dispatch lists in bpd.hip)
static const std::set<std::pair<int, int>> TILES = {{3, 1}, {2, 1}, {1, 1}, {8, 2}, {7, 2}, {5, 2}, {4, 2}, {3, 2}, {2, 2}, {1, 2},
                                                    {8, 4}, {7, 4}, {5, 4}, {4, 4}, {3, 4}, {2, 4}, {1, 4}};

static void check_config(const bpd_config& c) {
  Layout L;
  std::vector<std::pair<size_t, size_t>> log;
  const size_t total = build_layout(c, nullptr, L, &log);
  Layout L2;
  EXPECT(build_layout(c, nullptr, L2) == total, "size is a pure function of the configuration");
  size_t end = 0;
  for (auto& r : log) {
    EXPECT(r.first % ALIGN == 0, "aligned region at %zu", r.first);
    EXPECT(r.first >= end, "regions overlap at %zu", r.first);
    end = r.first + r.second;
  }
  EXPECT(end <= total && total % ALIGN == 0, "last region ends at %zu of %zu", end, total);
  const size_t d = c.d_model, F = c.d_ff, V = c.vocab, k = c.k_max, S = c.max_src_len, slots = (size_t)c.max_out_len + c.k_max + 1;
  const size_t B = c.max_batch, M = B * k;
  // every tensor bpd_load_weights accepts (include/bpd.h), as fp32 from the host
  const size_t tensors[] = {V * d, S * d, slots * d, d * d, d * F, F * d, F, d, k * d * F, k * F, k * F * d, k * d};
  for (size_t t : tensors) EXPECT(t * 4 <= L.staging_bytes, "staging %zu < tensor %zu", L.staging_bytes, t * 4);
  // distances between neighbouring regions that launches rely on
  EXPECT((char*)L.kpart - (char*)L.attn_part >= (long)((size_t)ATTN_PART_SLOTS * 16 * (d / c.n_heads + 2) * 4), "attention partials");
  EXPECT((size_t)((char*)L.xn - (char*)L.kpart) >= L.n_kpart * 4, "K slices");
  // the encoder's slices of a long K, of as many source rows as leave any
  const size_t sliced = std::min(B * S, (size_t)LEAN_PART_M);
  if (c.d_ff > LEAN_K_WHOLE && lean_encoder_ok(c, (long)sliced)) EXPECT((size_t)((char*)L.xn - (char*)L.kpart) >= F / 1024 * sliced * d * 4, "the encoder's K slices, %zu rows, d=%zu F=%zu k=%zu B=%zu", sliced, d, F, k, B);
  EXPECT((size_t)((char*)L.keys_h1 - (char*)L.keys) >= M * k * 8, "keys");
  EXPECT((size_t)((char*)L.hn2 - (char*)L.keys_h1) >= 2 * M * 8, "head-1 and second-phase keys");
  EXPECT(L.n_zeros >= std::max({k * F, V, 3 * d}), "zero vector");
  // folded copies of the decoder's matrices: there whenever a block of the context needs them, and only then
  bool needed = false;
  for (long rows = 1; rows <= (long)M; ++rows) needed = needed || (c.dtype == BPD_BF16 && rows > LDSX_LN_M_MAX && !lean_ok(c, rows) && d % 64 == 0 && d <= 1024);
  EXPECT((L.dec[0].f_qkv.W != nullptr) == needed && (L.dec[0].f_w1.W != nullptr) == needed, "folded copies d=%zu F=%zu rows=%zu", d, F, M);
  // split factors stay inside their buffers for every block the context may see
  for (int b = 1; b <= c.max_batch; b += (c.max_batch > 8 ? 3 : 1))
    for (int kk = 1; kk <= c.k_max; kk += (c.k_max > 6 ? 2 : 1)) {
      const int Mb = b * kk;
      for (int K : {c.d_model, c.d_ff}) {
        const int ns = residual_k_slices_of(c.d_model, L.n_kpart, Mb, c.d_model, K);
        EXPECT(ns >= 1 && ns <= KSPLIT_MAX && (ns == 1 || ((size_t)ns * Mb * c.d_model <= L.n_kpart && K % (ns * 512) == 0)), "K slices %d", ns);
      }
      for (long steps : {0L, 3L, 50L, 400L})
        for (int causal : {0, 1}) {
          const int cap = causal ? (int)slots : c.max_src_len;
          const int ns = attention_nsplit_of(c, steps, 0, 0, cap, b, kk, causal);
          const int wgs = c.n_heads * b * ((kk + 15) / 16);
          EXPECT(ns >= 1 && ns <= 16 && (ns == 1 || ns * wgs <= ATTN_PART_SLOTS), "attention split %d x %d", ns, wgs);
        }
    }
  if (stack_shape_ok(c)) {
    EXPECT(L.stack_ex && L.stack_flags && L.stack_layers, "decoder stack buffers");
    EXPECT((size_t)((char*)L.stack_flags - (char*)L.stack_ex) >= (size_t)c.n_dec_layers * stack_ex(c.d_model, c.d_ff).total, "exchange buffers");
  }
}

int main() {
  std::mt19937 rng(1811);
  auto U = [&](int lo, int hi) { return (int)(lo + rng() % (unsigned)(hi - lo + 1)); };
  long configs = 0;
  for (int it = 0; it < 3000; ++it) {
    bpd_config c{};
    c.dtype = U(0, 3) == 0 ? BPD_F32 : BPD_BF16;
    const int dh = (c.dtype == BPD_F32 || U(0, 2) == 0) ? 16 : 64;
    c.n_heads = U(1, dh == 16 ? 16 : 32);
    c.d_model = dh * c.n_heads;
    c.d_ff = U(0, 1) ? 32 * U(1, 160) : 512 * U(1, 9);
    c.vocab = 16 * U(1, 2200);
    c.k_max = U(1, 16);
    c.n_enc_layers = U(1, 6); c.n_dec_layers = U(1, 8);
    c.max_batch = U(1, 40); c.max_src_len = U(1, 200); c.max_out_len = U(1, 3100);
    c.eos_id = U(-1, 15); c.pad_id = 0; c.ln_eps = 1e-6f;
    if (!config_ok(c)) continue;
    check_config(c);
    ++configs;
  }
  // the five workloads' shapes
  const int W[5][9] = {{2, 2, 64, 4, 256, 256, 4, 1, 32}, {6, 6, 512, 8, 2048, 32000, 8, 1, 64}, {6, 6, 1024, 16, 4096, 32768, 10, 32, 128},
                       {6, 6, 1024, 16, 4096, 32768, 10, 1, 128}, {6, 6, 512, 8, 2048, 256, 10, 8, 3072}};
  for (auto& w : W) {
    bpd_config c{};
    c.n_enc_layers = w[0]; c.n_dec_layers = w[1]; c.d_model = w[2]; c.n_heads = w[3]; c.d_ff = w[4]; c.vocab = w[5]; c.k_max = w[6];
    c.max_batch = w[7]; c.max_out_len = w[8]; c.max_src_len = w[8] == 3072 ? 192 : 128;
    c.dtype = w[2] == 64 ? BPD_F32 : BPD_BF16; c.eos_id = 2; c.ln_eps = 1e-6f;
    EXPECT(config_ok(c), "workload shape accepted");
    check_config(c);
    ++configs;
  }
  // one workgroup per sequence or launches: measured us of both (d, d_ff, vocab, layers, rows, keys: one, launches), and the
  // rule takes the faster one wherever they differ by more than a tenth
  const int STEPS[][8] = {{64, 256, 256, 2, 4, 1, 68, 134}, {64, 256, 256, 2, 4, 64, 71, 157}, {64, 256, 256, 2, 4, 512, 102, 163}, {64, 256, 256, 2, 4, 1000, 135, 158},
                          {64, 256, 256, 2, 4, 1900, 197, 164}, {64, 256, 256, 2, 4, 3900, 364, 175}, {64, 1024, 1024, 8, 4, 1, 279, 715}, {64, 256, 256, 8, 16, 1, 563, 498},
                          {64, 256, 256, 8, 16, 1000, 1698, 537}, {128, 512, 256, 2, 4, 1, 118, 180}, {128, 512, 256, 2, 4, 512, 195, 200}, {128, 512, 256, 2, 4, 1000, 272, 197},
                          {128, 512, 256, 4, 4, 1, 192, 369}, {256, 512, 256, 1, 4, 1, 154, 144}, {256, 256, 256, 3, 1, 1, 169, 252}, {256, 256, 256, 3, 1, 512, 252, 352},
                          {256, 256, 256, 3, 1, 1000, 337, 366}, {256, 256, 256, 3, 1, 1900, 497, 378}, {32, 64, 64, 1, 16, 1, 95, 74}, {64, 256, 256, 2, 8, 1, 105, 141},
                          {64, 256, 256, 4, 8, 1, 158, 245}, {128, 512, 256, 2, 8, 1, 209, 216}, {64, 256, 4096, 2, 4, 1, 115, 166}, {64, 256, 256, 2, 16, 1, 255, 146},
                          {64, 256, 256, 2, 12, 1, 185, 143}, {32, 128, 256, 2, 8, 1, 75, 117}, {64, 256, 256, 2, 1, 1, 50, 121}};
  const int ENCODES[][8] = {{64, 256, 256, 2, 4, 16, 134, 231}, {64, 256, 256, 2, 4, 33, 235, 234}, {64, 256, 256, 2, 4, 64, 334, 209}, {64, 256, 256, 2, 4, 128, 736, 239},
                            {64, 256, 256, 2, 4, 300, 2549, 242}, {64, 1024, 1024, 8, 4, 16, 567, 1280}, {64, 1024, 1024, 8, 4, 64, 1595, 1307}, {64, 1024, 1024, 8, 4, 128, 3545, 1451},
                            {64, 256, 256, 8, 16, 16, 433, 796}, {128, 512, 256, 2, 4, 16, 233, 283}, {128, 512, 256, 2, 4, 32, 353, 284}, {128, 512, 256, 4, 4, 16, 397, 640},
                            {256, 512, 256, 1, 4, 16, 272, 223}, {256, 256, 256, 3, 1, 16, 488, 573}, {32, 64, 64, 1, 16, 16, 75, 120}, {32, 64, 64, 1, 16, 128, 276, 130},
                            {64, 256, 256, 2, 8, 16, 141, 219}, {64, 256, 256, 4, 8, 16, 227, 419}, {128, 512, 256, 2, 8, 16, 261, 301}, {64, 256, 4096, 2, 4, 16, 166, 263},
                            {64, 256, 256, 2, 16, 16, 155, 226}, {64, 256, 256, 2, 1, 16, 128, 220}, {32, 128, 256, 2, 8, 16, 110, 191}};
  auto fp32_model = [](const int* m) {
    bpd_config c{};
    c.n_enc_layers = c.n_dec_layers = m[3]; c.d_model = m[0]; c.n_heads = m[0] / 16; c.d_ff = m[1]; c.vocab = m[2]; c.k_max = m[4];
    c.max_batch = 1; c.max_src_len = 300; c.max_out_len = 4000; c.dtype = BPD_F32; c.eos_id = 2; c.ln_eps = 1e-6f;
    return c;
  };
  for (auto& m : STEPS) {
    const bpd_config c = fp32_model(m);
    EXPECT(config_ok(c) && small_shape(c), "measured shape d %d", m[0]);
    if (10 * std::min(m[6], m[7]) < 9 * std::max(m[6], m[7]))
      EXPECT(small_step_pays(c, m[4], m[5] + m[4], 16) == (m[6] < m[7]), "step d %d F %d L %d rows %d keys %d: %.0f %.0f", m[0], m[1], m[3], m[4], m[5], small_step_us(c, m[4], m[4], m[5] + m[4], 16), launched_step_us(c));
  }
  for (auto& m : ENCODES) {
    const bpd_config c = fp32_model(m);
    if (10 * std::min(m[6], m[7]) < 9 * std::max(m[6], m[7])) EXPECT(small_encode_pays(c, m[5]) == (m[6] < m[7]), "encode d %d F %d L %d S %d", m[0], m[1], m[3], m[5]);
  }
  // the tile rule: every answer is a tile the library has, K is a multiple of the chunk depth, the cap on rows is kept
  long tiles = 0;
  for (int M : {17, 20, 33, 48, 64, 80, 100, 128, 153, 252, 320, 512, 1000, 3200, 4096})
    for (int N : {64, 256, 528, 1024, 3072, 4096, 32768, 40960})
      for (int K : {64, 128, 192, 256, 320, 512, 1024, 2048, 4096})
        for (long z : {1L, 2L, 4L, 10L, 16L})
          for (int cap : {8, 3}) {
            int mt = 0, nt = 0;
            pick_tile(M, N, K, z, mt, nt, cap);
            EXPECT(TILES.count({mt, nt}) == 1, "tile %d x %d for M=%d N=%d K=%d", mt, nt, M, N, K);
            EXPECT(mt <= cap && K % (256 / nt) == 0, "tile %d x %d cap %d K %d", mt, nt, cap, K);
            // the 256-column tiles of 64+ rows walk K two chunks of 64 at a time (no code for an odd last chunk)
            EXPECT(!(nt == 4 && mt >= 4) || K % 128 == 0, "deep tile %d x %d with K = %d", mt, nt, K);
            ++tiles;
          }
  // the workgroup -> tile map of the LDS-staged GEMM: every (group, row block, column block) of a grid exactly once,
  // for one group, K slices in z, and several groups (with and without the grouped map)
  long grids = 0;
  for (unsigned NB : {1u, 2u, 3u, 4u, 6u, 8u, 10u, 16u, 20u, 24u, 40u, 128u, 160u})
    for (unsigned MB : {1u, 2u, 3u, 5u, 7u, 20u, 25u})
      for (unsigned Z : {1u, 2u, 4u, 8u, 9u, 10u, 16u})
        for (int ksplit : {1, 4}) {
          if (ksplit > 1 && Z != 4) continue;
          const LdsxMap m = ldsx_map_of(1024, 64, ksplit, NB, MB, Z);
          EXPECT(m.nchunks == 16 / ksplit, "chunks %d", m.nchunks);
          std::vector<char> seen((size_t)NB * MB * Z, 0);
          for (unsigned z = 0; z < Z; ++z)
            for (unsigned y = 0; y < MB; ++y)
              for (unsigned x = 0; x < NB; ++x) {
                int g = (int)z, by = -1, bx = -1;
                ldsx_tile_of(m, NB, MB, x, y, z, g, by, bx);
                const bool ok = g >= 0 && g < (int)Z && by >= 0 && by < (int)MB && bx >= 0 && bx < (int)NB;
                EXPECT(ok, "map NB=%u MB=%u Z=%u (%u,%u,%u) -> g %d by %d bx %d", NB, MB, Z, x, y, z, g, by, bx);
                if (ok) { char& c = seen[((size_t)g * MB + by) * NB + bx]; EXPECT(c == 0, "tile twice NB=%u MB=%u Z=%u", NB, MB, Z); c = 1; }
              }
          ++grids;
        }
  printf("%ld configurations, %ld tile choices, %ld grids checked, %ld violations\n", configs, tiles, grids, bad);
  return bad ? 1 : 0;
}
