// Host check of libbpd's sizing and dispatch logic (paper_1811_03115_amd/csrc/bpd_host_logic.h) on many random
// configurations inside what bpd_create accepts: workspace regions are aligned, disjoint and inside the reported size;
// the staging area holds the largest tensor bpd_load_weights may stage; key / slice / partial-result buffers hold what
// the launches write into them; the tile rule only returns tiles the library instantiates.
// Built by tests/test_host_logic.py with the system compiler under -fsanitize=address,undefined.
#include <algorithm>
#include <array>
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
  // activations that kernels write and read by whole row tiles (packed_at())
  const size_t as = act_size(c), Mt = (M + 15) / 16 * 16, Met = (B * S + 15) / 16 * 16;
  auto room = [&](const void* p) { for (auto& r : log) if (r.first == (size_t)p) return r.second; return (size_t)0; };      // (the layout starts at null)
  for (const void* p : {L.xn, L.attn}) EXPECT(room(p) >= Mt * d * as, "normalised rows, attention: %zu of %zu rows", room(p), Mt);
  EXPECT(room(L.ffh) >= Mt * F * as, "hidden layer: %zu of %zu rows", room(L.ffh), Mt);
  for (const void* p : {L.xen, L.attne, L.mem}) EXPECT(room(p) >= Met * d * as, "the encoder's rows: %zu of %zu rows", room(p), Met);
  EXPECT(room(L.ffhe) >= Met * F * as, "the encoder's hidden layer: %zu of %zu rows", room(L.ffhe), Met);
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
  // one workgroup per sequence or launches: measured us of both (d, d_ff, vocab, layers, rows, keys or source tokens: one, launches), the shortest of a shape
  // and those on both sides of where the two cross, and the rule takes the faster one wherever they differ by more than a tenth
  const int STEPS[][8] = {{64, 256, 256, 2, 4, 61, 53, 123}, {64, 256, 256, 2, 4, 1120, 84, 126}, {64, 256, 256, 2, 4, 2020, 110, 131},
                          {64, 256, 256, 2, 4, 3620, 203, 132}, {64, 1024, 1024, 8, 4, 61, 221, 741}, {64, 1024, 1024, 8, 4, 1120, 391, 767},
                          {64, 1024, 1024, 8, 4, 2020, 543, 771}, {64, 1024, 1024, 8, 4, 3620, 822, 788}, {64, 256, 256, 8, 16, 241, 469, 528},
                          {64, 256, 256, 8, 16, 960, 706, 517}, {64, 256, 256, 8, 16, 2400, 1430, 549}, {128, 512, 256, 2, 4, 61, 100, 173},
                          {128, 512, 256, 2, 4, 632, 150, 176}, {128, 512, 256, 2, 4, 1120, 188, 176}, {128, 512, 256, 4, 4, 61, 162, 337},
                          {128, 512, 256, 4, 4, 632, 245, 352}, {128, 512, 256, 4, 4, 1120, 327, 368}, {128, 512, 256, 4, 4, 2020, 475, 370},
                          {256, 512, 256, 1, 4, 61, 130, 135}, {256, 512, 256, 1, 4, 240, 142, 137}, {256, 512, 256, 1, 4, 1120, 217, 140},
                          {256, 256, 256, 3, 1, 16, 155, 270}, {256, 256, 256, 3, 1, 1029, 249, 327}, {256, 256, 256, 3, 1, 1929, 336, 329},
                          {32, 64, 64, 1, 16, 241, 87, 70}, {32, 64, 64, 1, 16, 2400, 141, 71}, {64, 256, 256, 2, 8, 121, 89, 132},
                          {64, 256, 256, 2, 8, 480, 104, 142}, {64, 256, 256, 2, 8, 960, 131, 138}, {64, 256, 256, 2, 8, 1240, 147, 140},
                          {64, 256, 256, 4, 8, 121, 133, 241}, {64, 256, 256, 4, 8, 480, 163, 256}, {64, 256, 256, 4, 8, 960, 237, 249},
                          {64, 256, 256, 4, 8, 1240, 279, 254}, {128, 512, 256, 2, 8, 121, 190, 206}, {128, 512, 256, 2, 8, 480, 223, 219},
                          {128, 512, 256, 2, 8, 1240, 327, 221}, {64, 256, 4096, 2, 4, 61, 84, 161}, {64, 256, 4096, 2, 4, 1120, 117, 165},
                          {64, 256, 4096, 2, 4, 2020, 157, 165}, {64, 256, 4096, 2, 4, 3620, 241, 170}, {64, 256, 256, 2, 16, 241, 224, 148},
                          {64, 256, 256, 2, 16, 2400, 471, 148}, {64, 256, 256, 2, 12, 181, 155, 139}, {64, 256, 256, 2, 12, 1800, 287, 141},
                          {32, 128, 256, 2, 8, 121, 66, 111}, {32, 128, 256, 2, 8, 960, 88, 116}, {32, 128, 256, 2, 8, 1240, 95, 114},
                          {32, 128, 256, 2, 8, 2144, 122, 119}, {64, 256, 256, 2, 1, 16, 47, 121}, {64, 256, 256, 2, 1, 1029, 67, 127},
                          {64, 256, 256, 2, 1, 1929, 83, 122}, {64, 256, 256, 2, 1, 3529, 129, 126}, {128, 256, 1024, 6, 4, 61, 197, 454},
                          {128, 256, 1024, 6, 4, 632, 322, 469}, {128, 256, 1024, 6, 4, 1120, 442, 477}, {128, 256, 1024, 6, 4, 2020, 668, 480},
                          {32, 128, 1024, 4, 16, 241, 252, 229}, {32, 128, 1024, 4, 16, 2400, 472, 231}, {256, 256, 256, 1, 8, 121, 187, 120},
                          {256, 256, 256, 1, 8, 1240, 332, 126}, {128, 64, 4096, 1, 6, 91, 202, 147}, {32, 128, 1024, 4, 13, 196, 208, 211},
                          {32, 128, 1024, 4, 13, 780, 254, 218}, {192, 32, 2048, 4, 1, 16, 176, 348}, {192, 32, 2048, 4, 1, 1029, 300, 367},
                          {192, 32, 2048, 4, 1, 1929, 409, 373}, {64, 64, 64, 1, 7, 106, 49, 67}, {64, 64, 64, 1, 7, 420, 57, 72},
                          {64, 64, 64, 1, 7, 840, 68, 70}, {64, 64, 64, 1, 7, 1211, 78, 70}, {64, 64, 256, 5, 11, 166, 198, 260},
                          {64, 64, 256, 5, 11, 660, 271, 274}, {64, 64, 256, 5, 11, 990, 355, 272}, {64, 512, 4096, 4, 6, 91, 249, 309},
                          {64, 512, 4096, 4, 6, 360, 272, 329}, {64, 512, 4096, 4, 6, 720, 320, 326}, {64, 512, 4096, 4, 6, 1182, 385, 334},
                          {96, 256, 256, 3, 9, 136, 215, 209}, {32, 128, 512, 1, 11, 166, 83, 67}, {32, 128, 512, 5, 16, 241, 228, 287},
                          {32, 128, 512, 5, 16, 960, 297, 266}, {32, 1024, 256, 4, 4, 61, 96, 318}, {32, 1024, 256, 4, 4, 2020, 234, 327},
                          {32, 1024, 256, 4, 4, 3620, 356, 334}, {64, 256, 512, 6, 9, 136, 244, 352}, {64, 256, 512, 6, 9, 540, 316, 380},
                          {64, 256, 512, 6, 9, 810, 385, 368}, {128, 32, 2048, 6, 10, 151, 498, 432}, {32, 256, 64, 4, 11, 166, 159, 218},
                          {32, 256, 64, 4, 11, 660, 196, 230}, {32, 256, 64, 4, 11, 990, 231, 232}, {32, 256, 64, 4, 11, 1320, 264, 232},
                          {256, 128, 512, 3, 3, 46, 175, 310}, {256, 128, 512, 3, 3, 339, 227, 322}, {256, 128, 512, 3, 3, 603, 279, 331},
                          {256, 128, 512, 3, 3, 1089, 377, 336}, {32, 64, 4096, 6, 9, 136, 298, 293}, {128, 1024, 1024, 3, 2, 31, 152, 327},
                          {128, 1024, 1024, 3, 2, 1060, 228, 365}, {128, 1024, 1024, 3, 2, 1960, 300, 366}, {128, 1024, 1024, 3, 2, 3560, 428, 374},
                          {32, 64, 1024, 6, 5, 76, 123, 276}, {32, 64, 1024, 6, 5, 665, 171, 281}, {32, 64, 1024, 6, 5, 1150, 209, 286},
                          {32, 64, 1024, 6, 5, 2050, 289, 283}, {32, 256, 512, 3, 15, 226, 195, 189}, {96, 256, 1024, 3, 4, 61, 98, 203},
                          {96, 256, 1024, 3, 4, 632, 152, 210}, {96, 256, 1024, 3, 4, 1120, 235, 213}, {64, 32, 1024, 5, 12, 181, 250, 269},
                          {64, 32, 1024, 5, 12, 720, 328, 278}};
  const int ENCODES[][8] = {{64, 256, 256, 2, 4, 1, 95, 175}, {64, 256, 256, 2, 4, 32, 157, 193}, {64, 256, 256, 2, 4, 33, 204, 192},
                          {64, 1024, 1024, 8, 4, 1, 428, 1173}, {64, 1024, 1024, 8, 4, 33, 1002, 1270}, {64, 1024, 1024, 8, 4, 48, 1067, 1258},
                          {64, 1024, 1024, 8, 4, 64, 1346, 1258}, {64, 256, 256, 8, 16, 1, 324, 651}, {64, 256, 256, 8, 16, 32, 562, 694},
                          {64, 256, 256, 8, 16, 33, 749, 704}, {128, 512, 256, 2, 4, 1, 165, 244}, {128, 512, 256, 2, 4, 17, 257, 268},
                          {128, 512, 256, 2, 4, 32, 282, 264}, {128, 512, 256, 4, 4, 1, 279, 543}, {128, 512, 256, 4, 4, 17, 456, 590},
                          {128, 512, 256, 4, 4, 32, 504, 580}, {128, 512, 256, 4, 4, 33, 663, 582}, {256, 512, 256, 1, 4, 1, 186, 194},
                          {256, 256, 256, 3, 1, 1, 315, 533}, {32, 64, 64, 1, 16, 1, 57, 87}, {32, 64, 64, 1, 16, 32, 78, 91}, {32, 64, 64, 1, 16, 33, 96, 92},
                          {64, 256, 256, 2, 8, 1, 100, 179}, {64, 256, 256, 2, 8, 32, 161, 197}, {64, 256, 256, 2, 8, 33, 209, 199},
                          {64, 256, 256, 4, 8, 1, 163, 351}, {64, 256, 256, 4, 8, 32, 282, 360}, {64, 256, 256, 4, 8, 33, 376, 357},
                          {128, 512, 256, 2, 8, 1, 192, 249}, {128, 512, 256, 2, 8, 16, 215, 268}, {128, 512, 256, 2, 8, 17, 284, 268},
                          {64, 256, 4096, 2, 4, 1, 120, 206}, {64, 256, 4096, 2, 4, 32, 182, 230}, {64, 256, 4096, 2, 4, 48, 243, 228},
                          {64, 256, 256, 2, 16, 1, 111, 172}, {64, 256, 256, 2, 16, 32, 172, 196}, {64, 256, 256, 2, 16, 33, 220, 199},
                          {64, 256, 256, 2, 12, 1, 107, 174}, {64, 256, 256, 2, 12, 32, 168, 197}, {64, 256, 256, 2, 12, 33, 216, 201},
                          {32, 128, 256, 2, 8, 1, 84, 143}, {32, 128, 256, 2, 8, 32, 126, 160}, {32, 128, 256, 2, 8, 48, 168, 158},
                          {64, 256, 256, 2, 1, 1, 91, 176}, {64, 256, 256, 2, 1, 32, 154, 192}, {64, 256, 256, 2, 1, 48, 215, 190},
                          {128, 256, 1024, 6, 4, 1, 346, 690}, {128, 256, 1024, 6, 4, 17, 584, 759}, {128, 256, 1024, 6, 4, 32, 644, 758},
                          {128, 256, 1024, 6, 4, 33, 861, 758}, {32, 128, 1024, 4, 16, 1, 141, 261}, {32, 128, 1024, 4, 16, 32, 222, 295},
                          {32, 128, 1024, 4, 16, 64, 377, 284}, {256, 256, 256, 1, 8, 4, 178, 172}, {128, 64, 4096, 1, 6, 1, 112, 173},
                          {128, 64, 4096, 1, 6, 17, 149, 182}, {128, 64, 4096, 1, 6, 32, 161, 185}, {128, 64, 4096, 1, 6, 33, 194, 181},
                          {32, 128, 1024, 4, 13, 1, 141, 266}, {32, 128, 1024, 4, 13, 32, 222, 296}, {32, 128, 1024, 4, 13, 48, 303, 289},
                          {192, 32, 2048, 4, 1, 1, 329, 543}, {192, 32, 2048, 4, 1, 17, 549, 582}, {192, 32, 2048, 4, 1, 32, 614, 593},
                          {128, 64, 64, 3, 15, 1, 158, 256}, {128, 64, 64, 3, 15, 17, 268, 278}, {128, 64, 64, 3, 15, 32, 304, 287},
                          {64, 64, 64, 1, 7, 1, 58, 93}, {64, 64, 64, 1, 7, 32, 87, 101}, {64, 64, 64, 1, 7, 33, 109, 98}, {64, 64, 256, 5, 11, 1, 170, 341},
                          {64, 64, 256, 5, 11, 32, 306, 378}, {64, 64, 256, 5, 11, 33, 408, 376}, {64, 512, 4096, 4, 6, 1, 224, 424},
                          {64, 512, 4096, 4, 6, 32, 359, 458}, {64, 512, 4096, 4, 6, 48, 489, 474}, {96, 256, 256, 3, 9, 1, 189, 268},
                          {96, 256, 256, 3, 9, 16, 215, 302}, {96, 256, 256, 3, 9, 32, 322, 307}, {32, 128, 512, 1, 11, 1, 60, 86},
                          {32, 128, 512, 1, 11, 32, 83, 92}, {32, 128, 512, 1, 11, 33, 101, 95}, {32, 128, 512, 5, 16, 1, 169, 515},
                          {32, 128, 512, 5, 16, 32, 265, 349}, {32, 128, 512, 5, 16, 48, 366, 343}, {256, 128, 1024, 1, 14, 1, 181, 191},
                          {96, 256, 2048, 1, 15, 1, 130, 140}, {96, 256, 2048, 1, 15, 16, 138, 149}, {96, 256, 2048, 1, 15, 17, 168, 144},
                          {32, 1024, 256, 4, 4, 1, 185, 491}, {32, 1024, 256, 4, 4, 48, 426, 523}, {32, 1024, 256, 4, 4, 64, 534, 516},
                          {64, 256, 512, 6, 9, 1, 242, 460}, {64, 256, 512, 6, 9, 32, 425, 519}, {64, 256, 512, 6, 9, 33, 565, 527},
                          {128, 32, 2048, 6, 10, 1, 310, 580}, {128, 32, 2048, 6, 10, 17, 522, 650}, {128, 32, 2048, 6, 10, 32, 587, 649},
                          {128, 32, 2048, 6, 10, 33, 775, 647}, {32, 256, 64, 4, 11, 1, 149, 283}, {32, 256, 64, 4, 11, 32, 236, 321},
                          {32, 256, 64, 4, 11, 64, 403, 328}, {256, 128, 512, 3, 3, 1, 304, 491}, {32, 64, 4096, 6, 9, 1, 198, 374},
                          {32, 64, 4096, 6, 9, 32, 312, 419}, {32, 64, 4096, 6, 9, 64, 533, 416}, {128, 1024, 1024, 3, 2, 1, 280, 564},
                          {128, 1024, 1024, 3, 2, 17, 446, 597}, {128, 1024, 1024, 3, 2, 32, 485, 603}, {128, 1024, 1024, 3, 2, 33, 635, 603},
                          {32, 64, 1024, 6, 5, 1, 183, 365}, {32, 64, 1024, 6, 5, 33, 394, 411}, {32, 64, 1024, 6, 5, 64, 516, 411},
                          {32, 256, 512, 3, 15, 1, 124, 223}, {32, 256, 512, 3, 15, 32, 190, 258}, {32, 256, 512, 3, 15, 64, 316, 257},
                          {96, 256, 1024, 3, 4, 1, 168, 285}, {96, 256, 1024, 3, 4, 17, 273, 311}, {96, 256, 1024, 3, 4, 32, 303, 317},
                          {96, 256, 1024, 3, 4, 33, 397, 315}, {64, 32, 1024, 5, 12, 1, 172, 335}, {64, 32, 1024, 5, 12, 32, 307, 379},
                          {64, 32, 1024, 5, 12, 33, 408, 378}};
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
  // packed source rows: whole row tiles, of LDS-staged GEMMs pairs of them, that hold every token and are fewer than the places there are (buffers are sized for those), and few different
  // numbers of them, since recorded encodes are found by it; up to d = 512 five sixths at most (of up to 128 places: less than three quarters), for narrow widths and those without
  // kernels of constant K only of many places or where the padding is beyond those kernels
  // or beyond LayerNorm inside them (256 rows)
  for (int d : {64, 128, 384, 512, 640, 768, 1024}) {
    bpd_config c{};
    c.d_model = d; c.d_ff = 4 * d; c.n_heads = d / 64; c.dtype = BPD_BF16;
    for (long places : {1L, 31L, 32L, 33L, 40L, 64L, 120L, 250L, 256L, 528L, 768L, 800L, 1280L, 1365L, 1366L, 2240L, 4096L, 8192L}) {
      std::set<long> seen;
      for (long tokens = 1; tokens <= places; ++tokens) {
        const long rows = packed_source_rows(c, tokens, places);
        seen.insert(rows);
        if (rows == 16) {                        // (one row tile: kernels of its own)
          EXPECT(tokens <= 16 && d > 256 && places > (d == 384 || d == 640 ? 18 : 32), "d %d, one row tile of %ld places", d, places);
          continue;
        }
        EXPECT(rows == 0 || (rows % (rows <= 256 && d != 64 && d != 384 && d != 640 ? 16 : 32) == 0 && rows >= tokens && 8 * rows <= 7 * places), "packed rows %ld of %ld tokens, %ld places", rows, tokens, places);
        EXPECT(rows == 0 || d > 512 || (places <= 128 ? 4 * rows < 3 * places : 6 * rows <= 5 * places), "d %d, packed rows %ld of %ld places", d, rows, places);
        EXPECT(rows == 0 || (d >= 512 && d != 640) || places * d >= 1L << 19 || (d == 128 && ((rows <= 640 && places > 640) || (rows <= 256 && places > 256))), "d %d, packed rows %ld of %ld places", d, rows, places);
      }
      EXPECT(seen.size() <= 16, "%zu numbers of packed rows, %ld places", seen.size(), places);
      EXPECT(seen.size() > 1 || places <= 42 || ((d < 512 || d == 640) && places * d < 1L << 19 && (places <= 256 || d != 128)), "d %d, nothing packed of %ld places", d, places);
    }
  }
  // the tile rule: every answer is a tile the library has, K is a multiple of the chunk depth, the cap on rows is kept
  long tiles = 0;
  // (by_cost: products that store; more rows than LDSX_COST_M otherwise go by area, too)
  for (int M : {17, 20, 33, 48, 64, 80, 100, 128, 153, 252, 320, 512, 640, 641, 660, 704, 1000, 3200, 4096, 5001, 8192})
    for (int N : {64, 256, 528, 1024, 3072, 4096, 32768, 40960})
      for (int K : {64, 128, 192, 256, 320, 512, 1024, 2048, 4096})
        for (long z : {1L, 2L, 4L, 10L, 16L})
          for (int cap : {8, 3})
            for (bool by_cost : {false, true}) {
              int mt = 0, nt = 0;
              pick_tile(M, N, K, z, mt, nt, cap, by_cost);
              EXPECT(TILES.count({mt, nt}) == 1, "tile %d x %d for M=%d N=%d K=%d", mt, nt, M, N, K);
              EXPECT(mt <= cap && K % (256 / nt) == 0, "tile %d x %d cap %d K %d", mt, nt, cap, K);
              // the 256-column tiles of 64+ rows walk K two chunks of 64 at a time (no code for an odd last chunk)
              EXPECT(!(nt == 4 && mt >= 4) || K % 128 == 0, "deep tile %d x %d with K = %d", mt, nt, K);
              // the cost rule is asked where it says it is, and nowhere else
              int am = 0, an = 0, cm = 0, cn = 0;
              pick_tile(M, N, K, z, am, an, cap, false);
              const bool asked = by_cost && M > (K >= 320 ? 640 : 5000) && z == 1 && cap >= 8;
              if (asked && pick_tile_by_cost(M, N, K, cm, cn)) EXPECT(mt == cm && nt == cn, "tile %d x %d by cost %d x %d", mt, nt, cm, cn);
              else EXPECT(mt == am && nt == an, "tile %d x %d by area %d x %d", mt, nt, am, an);
              ++tiles;
            }
  // many groups of many columns: tiles of 128 columns where one round of them fills the chip and the map deals whole groups to XCDs (groups, rows, N, tile)
  for (auto& w : {std::array<int, 5>{16, 60, 2048, 2, 2}, {16, 104, 2048, 4, 2}, {16, 144, 2048, 5, 2}, {10, 96, 2048, 2, 2}, {10, 128, 2048, 3, 2}, {12, 96, 1536, 2, 2},
                  {12, 96, 2048, 3, 1}, {13, 96, 1536, 3, 1}, {14, 96, 1536, 3, 1}}) {
    int mt = 0, nt = 0;
    pick_tile(w[1], w[2], 4096, w[0], mt, nt);
    EXPECT(mt == w[3] && nt == w[4], "tile %d x %d of %d rows, %d groups of %d columns", mt, nt, w[1], w[0], w[2]);
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
