// Host-side logic of libbpd that decides sizes and launch shapes: workspace layout, tile choice of the LDS-staged
// GEMM, split factors.  No HIP dependency: bpd.hip includes it, and tests/host/host_logic_check.cpp compiles it with the
// system compiler under the address / undefined-behaviour sanitizers (both defects the first GPU runs of this library
// found were in code of this kind: a staging area one tensor did not fit, a dispatch rule that took the wrong kernel).
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

#include "../../include/bpd.h"
#include "bpd_layers_jobs.h"
#include "bpd_stack_sched.h"

namespace {

constexpr size_t ALIGN = 256;

// Scratch of bpd_step_static: the device memory of a step that is neither input nor output nor decode state (arg-max
// keys that the vocabulary projection merges with atomic max, split-KV attention partials, split-K slices), for callers
// that may not allocate and hand over no workspace for it.  One copy per GPU, held until the process ends; every call
// on a GPU shares it, so calls that overlap on one GPU race.  In host code `scratch` is only a handle: the address on
// the current device comes from hipGetSymbolAddress (bpd_create keeps it per device).
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)8 << 20;
constexpr int MAX_DEVICES = 64;
constexpr int KSPLIT_MAX = 16;          // K slices of a split-K GEMM
constexpr int ATTN_LIMF_MIN_WGS = 256;  // attention launches of at least this many workgroups clamp their K/V loads to the length
constexpr int ATTN_PART_SLOTS = 512;   // workgroups of one split attention launch (partial-result slots); 1024 (one 256-key chunk per
                                       // workgroup up to 16 chunks) measured slower: C4 step at 3000 cached rows 0.383 vs 0.362 ms


struct Arena {
  char* base;
  size_t off = 0;
  std::vector<std::pair<size_t, size_t>>* log = nullptr;     // (offset, bytes) of every region, for the host check
  explicit Arena(char* b) : base(b) {}
  void* take(size_t bytes) {
    off = (off + ALIGN - 1) / ALIGN * ALIGN;
    void* p = base + off;
    if (log) log->push_back({off, bytes});
    off += bytes;
    return p;
  }
};

struct LnW { float *g, *b; };
struct EncL { LnW ln1, ln2; void *wqkv, *wo, *w1, *w2; float *b1, *b2; };
// (FoldW: a matrix with the LayerNorm in front of it folded in, see fold_layernorm_kernel; W == nullptr: not kept)
struct FoldW { void* W = nullptr; float* c = nullptr; float* d = nullptr; };
struct DecL { LnW ln1, ln2, ln3; void *wqkv, *wo, *cq, *co, *ckv, *w1, *w2; float *b1, *b2; FoldW f_qkv, f_cq, f_w1; };

struct Layout {
  // weights
  void* emb; float *emb_t, *pos_src, *pos_tgt;            // (emb_t: the embedding transposed, small fp32 models)
  std::vector<EncL> enc; LnW enc_lnf;
  std::vector<DecL> dec; LnW dec_lnf;
  void *hw1, *hw2; float *hb1, *hb2;
  // caches
  void *selfK, *selfV, *crossK, *crossV;        // [n_dec][B][kv_rows(slots | max_src)][d]
  // decoder activations (M = max_batch * k_max rows)
  float *x, *q, *h, *stats_ln, *stats_big, *zeros, *attn_part, *kpart; size_t n_zeros, n_kpart; void *xn, *attn, *ffh, *hn, *H, *O;
  unsigned long long* keys; unsigned long long* keys_h1; float* logits_h1; int* topn_ok;
  void* hn2; float* h2; int* sel;
  // decoder stack kernel (blocks of at most 16 rows): exchange buffers, flags, error word, probe output
  unsigned char* stack_ex = nullptr; unsigned* stack_flags = nullptr; unsigned* stack_err = nullptr; unsigned* xcc_map = nullptr;
  unsigned long long* stack_trace = nullptr; void* stack_layers = nullptr;
  void* layers_xn = nullptr; float* layers_slices = nullptr;     // tall_layers_kernel: LayersP::xn, slices
  float *layers_x1 = nullptr, *layers_x3 = nullptr; void *layers_attn2 = nullptr, *layers_ffh = nullptr;      // layers_kernel: LayersP::x1, x3, attn2; wide_layers_kernel: x1, attn, ffh
  unsigned* layers_sync = nullptr;               // layers_kernel: what its workgroups count in
  // encoder activations (max_batch * max_src rows)
  float *xe, *qe; void *xen, *ke, *ve, *attne, *ffhe, *mem;
  // state
  int *src_row0, *src_seq, *src_pos, *src_packed;         // packed source rows: PackP
  int *L, *j, *finished, *max_len, *src_len, *src_ids, *P, *A, *accepted, *out_ids, *step_counter, *imposed1, *sched;
  void* dyn; int *tick, *imp_next; int *steps_done, *fin_step, *slot_seq, *slot_L, *slot_src, *slot_row, *n_live;
  long long* stats;
  void* staging; size_t staging_bytes;
  size_t total;
};

size_t act_size(const bpd_config& c) { return c.dtype == BPD_BF16 ? 2 : 4; }

// 64-wide heads in bf16: K and V are kept in operand order, in groups of 32 keys (bpd_attention.h)
bool kv_grouped(const bpd_config& c) { return c.dtype == BPD_BF16 && c.d_model == 64 * c.n_heads; }
size_t kv_rows(const bpd_config& c, size_t rows) { return kv_grouped(c) ? (rows + 31) / 32 * 32 : rows; }

bool config_ok(const bpd_config& c) {
  if (c.n_enc_layers < 1 || c.n_dec_layers < 1 || c.d_model < 32 || c.n_heads < 1) return false;
  if (c.d_model % c.n_heads) return false;
  const int dh = c.d_model / c.n_heads;
  if (dh != 16 && dh != 64) return false;
  if (c.dtype == BPD_F32 && dh != 16) return false;     // fp32 mode is for small models only
  if (c.d_model % 32 || c.d_ff % 32 || c.vocab % 16 || c.vocab < 16) return false;
  if (c.d_model > 2048) return false;                   // LayerNorm kernel keeps a row in registers
  if (c.k_max < 1 || c.k_max > 16) return false;
  if (c.max_batch < 1 || c.max_src_len < 1 || c.max_out_len < 1) return false;
  if (c.dtype != BPD_F32 && c.dtype != BPD_BF16) return false;
  if (c.eos_id >= c.vocab || c.ln_eps <= 0.f) return false;
  return true;
}

// Small fp32 models can run with a workgroup per sequence (bpd_small.h): shapes whose weights are laid out for it.  Whether a call
// does is for small_step_pays() and small_encode_pays() to say.
constexpr size_t SMALL_WEIGHTS_MAX = (size_t)8 << 20;
bool small_shape(const bpd_config& c) {
  const size_t d = c.d_model, F = c.d_ff, V = c.vocab, k = c.k_max;
  return c.dtype == BPD_F32 && d <= 256 && V <= 4096 && c.n_dec_layers <= 8 && c.n_enc_layers <= 8 && (c.n_dec_layers * (6 * d * d + 2 * d * F) + 2 * k * d * F + V * d) * 4 <= SMALL_WEIGHTS_MAX;
}

// Does one workgroup per sequence beat the launches?  It walks the phases of the layers one after the other, with weights and cache rows
// at the rate one CU gets and keys 64 at a time by eight waves; the launches cost 3.5 us each, and their products walk K (the vocabulary's: V rows
// among 256 threads) serially.  Estimates in us, their constants fitted to 273 steps and 345 encodes of 40 shapes, half of them drawn: within a third
// of all but a hundredth of them, and the faster way wherever the two differ by more than a tenth (tests/host holds a choice of them).  (one, launches):
//   steps    d = 64, 2 layers, 4 rows    61 keys: 53, 123    632: 70, 126     1120: 84, 126     2020: 110, 131    3620: 203, 132
//            d = 64, 8 layers, 16 rows   241: 469, 528       960: 706, 517            d = 64, 2 layers, 12 rows   181: 155, 139
//            d = 128, 2 layers, 4 rows   61: 100, 173        1120: 188, 176           d = 256, 1 layer, 4 rows    61: 130, 135
//   encodes  d = 64, 2 layers    16 tokens: 104, 199   33: 204, 192   64: 272, 195   128: 548, 196   300: 1611, 226
//            d = 128, 2 layers   16: 187, 270          32: 282, 264   33: 363, 264
inline double small_bytes_us(double floats) { return floats * 4 / 65e3; }
// `rows` rows per sequence with k heads, over `keys` keys of its own and `src` of its source
inline double small_step_us(const bpd_config& c, int rows, int k, long keys, long src) {
  const double d = c.d_model, F = c.d_ff, V = c.vocab, L = c.n_dec_layers;
  const auto up = [](long a, long b) { return (double)((a + b - 1) / b); };
  const double phases = L * (c.d_model <= 64 ? 8 : 11) + 2, phase = rows <= 4 ? 1.3 : (rows <= 8 ? 2 : 2.8);
  return phase * phases + small_bytes_us(L * (6 * d * d + 2 * d * F) + 2 * k * d * F + V * d + 2 * L * d * (keys + src)) +
         0.36 * L * up((long)c.n_heads * rows, 8) * (up(keys, 64) + up(src, 64)) + 4.5 * up((long)rows * k, 16) * up(c.vocab, 512);
}
inline double launched_step_us(const bpd_config& c) {
  const double d = c.d_model, F = c.d_ff, V = c.vocab, L = c.n_dec_layers;
  return 3.5 * (11 * L + 6) + 0.032 * (L * (5 * d + F) + d + F) + 0.15e-3 * V * d;
}
inline bool small_step_pays(const bpd_config& c, int k, long keys, long src) { return small_step_us(c, k, k, keys, src) < launched_step_us(c); }
// (a source tile of 16 rows walks the encoder's phases, with the weights at 55 KB/us, and attends to every other)
inline bool small_encode_pays(const bpd_config& c, int S) {
  const double d = c.d_model, F = c.d_ff, E = c.n_enc_layers, L = c.n_dec_layers, tiles = (S + 15) / 16;
  const double one = tiles * (2.7 * (E * (c.d_model <= 64 ? 6 : 7) + 1 + L) + (E * (4 * d * d + 2 * d * F) + L * 2 * d * d) * 4 / 55e3 + 0.8 * E * tiles * d / 64) + small_step_us(c, 1, c.k_max, 1, S);
  return one < 1.1 * (7 * E + L + 4) + 0.03 * (E * (3 * d + F) + L * d) + launched_step_us(c);
}

// Shapes and row counts that run on the kernels with a constant K (bpd_row_gemm.h).
// Decoder layers, us with them and without (the LDS-staged GEMMs on folded weights), by block rows:
//   d = 1024, d_ff 4096   160: 348, 375   200: 380, 389   260: 461, 483   320: 458, 430   400: 538, 531   480: 531, 497   560: 669, 701   640: 622, 597
//   d = 512, d_ff 2048    160: 206, 234   256: 230, 251   320: 276, 281   448: 291, 295   512: 304, 301   576: 341, 343   640: 344, 334
// They cross at 300 and at 500 rows.  From there to 640 the constant K costs up to 6 % of the layers and stays: folded weights round
// the residual stream to bf16 before its LayerNorm and not after, and contexts of up to 640 rows need no second copy of three
// matrices per layer (Transformer-big: 96 MB).
// Encodes (without: LayerNorm kernels and LDS-staged GEMMs, the same roundings), by source rows:
//   d = 1024   128: 471, 472   256: 553, 575   384: 644, 629   512: 703, 679   640: 791, 749        -> up to 320 rows
//   d = 512    128: 293, 292   256: 332, 357   384: 374, 394   512: 401, 408   640: 447, 450        -> up to 640
constexpr int LEAN_M_MAX = 640;
constexpr int LEAN_ENC_WIDE_M_MAX = 320;      // encoder, d > 512
bool lean_width(int d) { return d == 128 || d == 256 || d == 512 || d == 768 || d == 1024; }
bool lean_ok(const bpd_config& c, long M) {
  return c.dtype == BPD_BF16 && M <= LEAN_M_MAX && lean_width(c.d_model) &&
         (c.d_ff == 512 || c.d_ff == 1024 || c.d_ff == 2048 || c.d_ff == 3072 || c.d_ff == 4096);
}
// The residual GEMM of K = d_ff runs as one kernel up to this K, beyond in K slices of 1024 that the next LayerNorm adds up
// (4096 x 1024 at 10 rows: 5.5 us whole, 3.4 us in slices, and the LayerNorm kernel with them 2.0 us, which takes the LayerNorm
// out of the next GEMM: 4.2 -> 3.05 us.  2048 x 512: 3.3 us whole, and 2.1 + 1.9 - 0.8 us in slices).
constexpr int LEAN_K_WHOLE = 2048;
constexpr int LEAN_PART_M = 192;        // more rows: the slices of the LDS-staged kernel (192 rows 6.8 against 7.25 us, 256 rows 8.0 against 7.3)
bool lean_encoder_ok(const bpd_config& c, long M) { return lean_ok(c, M) && (c.d_model <= 512 || M <= LEAN_ENC_WIDE_M_MAX); }
// LayerNorm inside the GEMM that follows, or in a kernel of its own?  (with K = 1024 every column block of 64 KB of x costs: 24 rows
// 5.05 us against 1.9 + 3.6, 40 rows 6.6 against 2.0 + 4.3; with K = 512 80 rows 3.3 against 1.9 + 2.5, 256 rows 5.4 against 1.9 + 3.9, 320 rows 6.8
// against 1.9 + 4.3)
bool lean_fuse(int d, long M) { return d <= 512 ? M <= 256 : M <= 32; }

// Rows of the encoder for sources of `tokens` tokens together in B x S places: packed, where that pays; otherwise all of them (0).
// A packed encode looks up each row's sequence and position: a load ahead of each attention, two at the entry of the GEMMs that store keys and values, some 0.5 us
// each.  Whole calls, ms, padded and packed: 13 sequences, 319 of 780 places, d = 512 2.158, 2.066;  32, 1090 of 2240, d = 1024 17.63, 17.39;  5, 250 places
// 4.690, 4.633.  Encodes of 64 .. 8192 places, 30 .. 84 % of them tokens, us, padded and packed:
//   d = 1024  seven eighths of the places and less: 960 places, 589 tokens 843, 772;  512, 442 687, 671.  Slower where the tiles of so many rows are poor ones: 1120 of 1280 rows
//             996, 1013 (d = 768 740, 786), 3584 of 4096 1643, 1664, 96 of 120 428, 433
//   d = 512   as fast or faster up to five sixths (960, 589 448, 429), beyond the tiles decide (832 of 960 rows 458, 470;  1120 of 1280 542, 564;  1568 of 1792 588, 625;  2688 of 3072 752, 711).
//             Up to 128 places, where a row tile less saves nothing, below three quarters (96 of 128 rows 240, 242;  64 of 128 251, 246)
//   narrower  layers too short for the lookups: d = 384, 768, 440 654, 673;  256, 162 486, 501;  d = 128, 2048, 1146 324, 335;  d = 64, 1024, 587 365, 370.  It pays
//             with many places (d = 384, 2048, 1146 758, 695;  d = 256, 2048, 1146 401, 363;  d = 128, 4096, 2266 382, 345) and where the padding alone is beyond the
//             kernels of constant K (d = 128, 768, 566 307, 249;  d = 256, 768, 566 319, 302) or beyond LayerNorm inside them (by rows of 288 .. 448 places, d = 128, 256: 128 .. 256
//             6 .. 13 % faster, 288 .. 384 0 .. 2 % slower)
//   d = 640, 896   (wider, but without kernels of constant K) as the narrower ones: by rows of 384 places, 160: 6, 3 % slower, 288: 7, 3, 320: 6, 6;  of 1024, d = 640, 512: 6 % faster
//   one row tile   goes through the kernels for it: d = 384, 28 places 463, 407;  d = 640, 24 568, 481;  d = 512, 42 231, 228;  d = 1024, 42 364, 335, but 28 333, 327, with d_ff 8192
//             579, 588;  d = 64, 128, 256, 39 306, 325;  191, 193;  218, 220
// In steps of a sixteenth of the places: recorded encodes are found by their rows, and lengths that change from call to call have at most fifteen of them, mostly two to six
// (in steps of one row tile few of their encodes were recorded: 32 sequences in 4096 places 306 us of host time, 66 so; 5 in 250, d = 768, the first 40 calls 2.64 ms,
// 2.52;  13 in 780 4.25, 3.85;  in steps of an eighth more rows are computed for nothing: encodes of 13 in 780 357 us, so 349, of 32 in 4096 1283, 1265, of 24 in 1440, where the
// tiles decide, 440, 448).  Whole pairs of row tiles, which is what the LDS-staged GEMMs walk in: d = 1024, 544 rows 760 us, 560 849, 576 761, all 800 places 824;  d = 1536, 172
// tokens of 256 places in 176 rows 1047, in 192 929, padded 975.  Up to 256 rows of the kernels of constant K single ones (d = 1024, 210 of 528 in 240 rows 601, in 288 648).
constexpr long PACKED_NARROW_PLACES = 1L << 19;      // places x d_model from which on packing pays for them
inline int packed_source_rows(const bpd_config& c, long tokens, long places) {
  if (tokens <= 16 && c.d_model > 256 && (places > 32 || (places > 18 && c.d_model < 1024 && !lean_width(c.d_model)))) return 16;
  const long step = (places + 255) / 256 * 16, tiles = (tokens + step - 1) / step * step;
  const long rows = tiles > 16 && tiles <= 256 && lean_encoder_ok(c, tiles) ? tiles : (tiles + 31) / 32 * 32;
  if (c.d_model > 512 ? rows * 8 > places * 7 : (places <= 128 ? rows * 4 >= places * 3 : rows * 6 > places * 5)) return 0;
  const bool narrow = (c.d_model < 512 || (c.d_model < 1024 && !lean_width(c.d_model))) && places * c.d_model < PACKED_NARROW_PLACES;
  const bool other = lean_encoder_ok(c, rows) && (!lean_encoder_ok(c, places) || (lean_fuse(c.d_model, rows) && !lean_fuse(c.d_model, places)));
  return narrow && !other ? 0 : (int)rows;
}

// Other decoder blocks of more than 128 rows run their LayerNorm-then-GEMM pairs as one GEMM on weights with the LayerNorm
// folded in (ROWAFF in bpd_gemm.h); contexts that can see such blocks keep a folded copy of those matrices.
constexpr int LDSX_LN_M_MAX = 128;     // LayerNorm-fused consumers and statistics-writing producers: blocks of at most 128 rows
bool fold_kept(const bpd_config& c) {
  const long rows = (long)c.max_batch * c.k_max;
  return c.dtype == BPD_BF16 && rows > LDSX_LN_M_MAX && !lean_ok(c, rows) && c.d_model % 64 == 0 && c.d_model <= 1024;
}

// All decoder layers as one kernel: the shapes that those of bpd_layers.h and bpd_wide_layers.h are built for
bool layers_shape(const bpd_config& c) { return c.dtype == BPD_BF16 && c.d_model == 512 && c.n_heads == 8 && c.d_ff == 2048; }
bool wide_layers_shape(const bpd_config& c) { return c.dtype == BPD_BF16 && c.d_model == 1024 && c.n_heads == 16 && c.d_ff == 4096; }

// Shapes the decoder stack kernel is built for (what a step additionally needs is checked per launch)
bool stack_shape_ok(const bpd_config& c) {
  const int d = c.d_model;
  return c.dtype == BPD_BF16 && d == 64 * c.n_heads && (d == 128 || d == 256 || d == 512 || d == 768 || d == 1024) &&
         c.d_ff % 128 == 0 && c.n_dec_layers <= STACK_MAX_LAYERS;
}
constexpr int XCC_MAP_MAX = 1024;          // compute units the placement probe can record

size_t build_layout(const bpd_config& c, char* base, Layout& L, std::vector<std::pair<size_t, size_t>>* log = nullptr) {
  Arena a(base);
  a.log = log;
  const size_t d = c.d_model, F = c.d_ff, V = c.vocab, k = c.k_max, ws = act_size(c), as = act_size(c);
  const size_t slots = (size_t)c.max_out_len + c.k_max + 1;
  auto vec = [&](size_t n) { return (float*)a.take(n * 4); };
  auto mat = [&](size_t kk, size_t nn) { return a.take(kk * nn * ws); };
  auto ln = [&]() { LnW w; w.g = vec(d); w.b = vec(d); return w; };
  L.emb = mat(V, d);
  L.emb_t = small_shape(c) ? vec(V * d) : nullptr;
  L.pos_src = vec((size_t)c.max_src_len * d);
  L.pos_tgt = vec(slots * d);
  L.enc.resize(c.n_enc_layers);
  for (auto& e : L.enc) {
    e.ln1 = ln(); e.wqkv = mat(d, 3 * d); e.wo = mat(d, d); e.ln2 = ln();
    e.w1 = mat(d, F); e.b1 = vec(F); e.w2 = mat(F, d); e.b2 = vec(d);
  }
  L.enc_lnf = ln();
  L.dec.resize(c.n_dec_layers);
  for (auto& e : L.dec) {
    e.ln1 = ln(); e.wqkv = mat(d, 3 * d); e.wo = mat(d, d);
    e.ln2 = ln(); e.cq = mat(d, d); e.co = mat(d, d); e.ckv = mat(d, 2 * d);
    e.ln3 = ln(); e.w1 = mat(d, F); e.b1 = vec(F); e.w2 = mat(F, d); e.b2 = vec(d);
  }
  L.dec_lnf = ln();
  if (fold_kept(c)) {
    auto fold = [&](size_t nn) { FoldW f; f.W = mat(d, nn); f.c = vec(nn); f.d = vec(nn); return f; };
    for (auto& e : L.dec) { e.f_qkv = fold(3 * d); e.f_cq = fold(d); e.f_w1 = fold(F); }
  }
  L.hw1 = mat(d, k * F); L.hb1 = vec(k * F); L.hw2 = mat(k * F, d); L.hb2 = vec(k * d);
  const size_t B = c.max_batch, nd = c.n_dec_layers, S = c.max_src_len;
  const size_t self_rows = kv_rows(c, slots), src_rows = kv_rows(c, S);
  L.selfK = a.take(nd * B * self_rows * d * as); L.selfV = a.take(nd * B * self_rows * d * as);
  L.crossK = a.take(nd * B * src_rows * d * as); L.crossV = a.take(nd * B * src_rows * d * as);
  const size_t M = B * k;
  L.x = vec(M * d); L.q = vec(M * d); L.h = vec(M * d); L.stats_ln = vec(64 * 16 * 2);
  L.n_zeros = k * F; if (V > L.n_zeros) L.n_zeros = V; if (3 * d > L.n_zeros) L.n_zeros = 3 * d;
  L.zeros = vec(L.n_zeros);
  L.attn_part = vec((size_t)ATTN_PART_SLOTS * 16 * (d / c.n_heads + 2));
  L.n_kpart = (size_t)KSPLIT_MAX * M * d;      // K slices of one residual update of the decoder block
  // ... and the encoder's d_ff / 1024 slices of up to LEAN_PART_M source rows, which may be more than that
  size_t enc_part = 0;
  if (c.d_ff > LEAN_K_WHOLE && lean_encoder_ok(c, 1)) enc_part = F / 1024 * (B * S < (size_t)LEAN_PART_M ? B * S : (size_t)LEAN_PART_M) * d;
  L.kpart = vec(L.n_kpart > enc_part ? L.n_kpart : enc_part);
  const size_t Mt = (M + 15) / 16 * 16;       // (whole row tiles: packed_at())
  L.xn = a.take(Mt * d * as); L.attn = a.take(Mt * d * as); L.ffh = a.take(Mt * F * as);
  L.hn = a.take(M * d * as); L.H = a.take(M * k * F * as); L.O = a.take(M * k * d * as);
  L.keys = (unsigned long long*)a.take(M * k * 8);
  L.keys_h1 = (unsigned long long*)a.take(2 * M * 8);     // keys of head 1 at the step's B*k rows, then the second phase's B*(k-1)
  L.hn2 = a.take(B * d * as); L.h2 = vec(B * d);
  L.logits_h1 = vec(M * V);
  const size_t Me = B * S;
  L.stats_big = vec((size_t)(d / 64 + 1) * (M > Me ? M : Me) * 2);   // per 64-column block and row: sum, sum of squares
  L.xe = vec(Me * d); L.qe = vec(Me * d);
  const size_t Met = (Me + 15) / 16 * 16;
  L.xen = a.take(Met * d * as); L.ke = a.take(B * src_rows * d * as); L.ve = a.take(B * src_rows * d * as);
  L.attne = a.take(Met * d * as); L.ffhe = a.take(Met * F * as); L.mem = a.take(Met * d * as);
  auto ints = [&](size_t n) { return (int*)a.take(n * 4); };
  L.L = ints(B); L.j = ints(B); L.finished = ints(B); L.max_len = ints(B); L.src_len = ints(B);
  L.src_ids = ints(Me); L.P = ints(B * k); L.A = ints(B * k * k); L.accepted = ints(B); L.topn_ok = ints(B * k); L.sel = ints(B);
  L.out_ids = ints(B * (size_t)c.max_out_len); L.step_counter = ints(1); L.imposed1 = ints(B);
  L.sched = ints(B * (size_t)c.max_out_len);
  if (kv_grouped(c)) { L.src_row0 = ints(B); L.src_seq = ints(Me); L.src_pos = ints(Me); L.src_packed = ints(Me); }
  L.dyn = a.take(64); L.tick = ints(B); L.imp_next = ints(B); L.steps_done = ints(B); L.fin_step = ints(B); L.slot_seq = ints(B); L.slot_L = ints(B); L.slot_src = ints(B); L.slot_row = ints(B); L.n_live = ints(1);
  L.stats = (long long*)a.take(32 * 8);
  if (wide_layers_shape(c)) {                  // (what both of them use: of the larger one)
    const size_t rows = M > 16 ? TALL_LAYERS_ROWS : 16;
    L.layers_xn = a.take((size_t)LK_JOBS * 4 * rows * d * as);
    L.layers_x1 = vec((M > 16 ? 4 : 6) * rows * d); L.layers_attn2 = a.take(4 * rows * d * as); L.layers_ffh = a.take(2 * rows * F * as);
    if (M > 16) L.layers_slices = vec((size_t)2 * 4 * rows * d);
  }
  if (layers_shape(c)) { L.layers_x1 = vec((size_t)2 * LK_JOBS * 16 * d); L.layers_x3 = vec((size_t)LK_JOBS * 16 * d); L.layers_attn2 = a.take((size_t)LK_JOBS * 16 * d * as); }
  L.layers_sync = layers_shape(c) || wide_layers_shape(c) ? (unsigned*)a.take((size_t)LK_WORDS * 4) : nullptr;
  L.xcc_map = (unsigned*)a.take(XCC_MAP_MAX * 4);
  L.stack_err = (unsigned*)a.take(256);
  if (stack_shape_ok(c)) {
    L.stack_ex = (unsigned char*)a.take((size_t)c.n_dec_layers * stack_ex(c.d_model, c.d_ff).total);
    L.stack_flags = (unsigned*)a.take((size_t)c.n_dec_layers * STACK_OPS * STACK_FLAG_STRIDE * 4);
    L.stack_trace = (unsigned long long*)a.take((size_t)STACK_FLAG_STRIDE * c.n_dec_layers * STACK_OPS * 8 * 8);
    L.stack_layers = a.take(STACK_LAYER_TABLE_BYTES);
  }
  size_t biggest = V * d;                    // largest tensor a bpd_load_weights call may stage (elements)
  if (k * d * F > biggest) biggest = k * d * F;
  if (slots * d > biggest) biggest = slots * d;
  if (S * d > biggest) biggest = S * d;
  if (3 * d * d > biggest) biggest = 3 * d * d;
  L.staging_bytes = biggest * 4;
  L.staging = a.take(L.staging_bytes);
  L.total = (a.off + ALIGN - 1) / ALIGN * ALIGN;
  return L.total;
}

constexpr int LDSX_LN_MT_MAX = 3;      // LayerNorm-fused consumers and statistics-writing producers: tiles of at most 48 rows
constexpr long LDSX_MIN_WGS = 440;
constexpr long LDSX_MIN_WGS_LONGK = 400;   // K >= 2048, fewer than 1024 rows: a workgroup lives long enough that about 1.5 per CU suffice
// The largest useful area that fills the chip: several groups, K slices, arg-max, up to LDSX_COST_M rows (chosen at 80 .. 320 rows)
void pick_tile_by_area(int M, int N, int K, long zdim, int& mt, int& nt, int mt_max) {
  const int mts[7] = {8, 7, 5, 4, 3, 2, 1};
  long best_area = 0, best_pad = 0;
  mt = 1; nt = (K % 256 == 0) ? 1 : 4;
  for (int n : {1, 2, 4}) {
    if (K % (256 / n) != 0) continue;
    const long cols = (N / 16 + 4 * n - 1) / (4 * n);
    for (int m : mts) {
      if ((n == 1 && m > 3) || m > mt_max) continue;
      if (n == 4 && m >= 4 && K % 128 != 0) continue;       // these tiles walk K two chunks of 64 at a time
      const long bm = 16 * m, mblocks = (M + bm - 1) / bm, pad = mblocks * bm;
      if (mblocks * cols * zdim < (K >= 2048 && M < 1024 ? LDSX_MIN_WGS_LONGK : LDSX_MIN_WGS)) continue;
      const long area = (long)m * n;                  // compared as area * M / pad: padded rows are wasted work
      if (best_area == 0 || area * best_pad > best_area * pad || (area * best_pad == best_area * pad && pad < best_pad)) {
        best_area = area; best_pad = pad; mt = m; nt = n;
      }
    }
  }
}
// Workgroups of a tile that one CU holds, by registers and LDS (tests/test_kernel_resources.py has the built kernels' numbers)
inline int ldsx_side_by_side(int mt, int nt) {
  if (nt == 1) return mt == 2 ? 4 : 3;
  return mt <= (nt == 2 ? 3 : 2) ? 4 : (mt <= (nt == 2 ? 5 : 4) ? 3 : 2);
}
// More rows than the kernels of constant K take, one group, results that are stored (encoders; the heads' hidden layers and decoder blocks of so many rows): the tile of the least
// estimated time.  In us, per 1024 of K: a workgroup on its own `lat`, the busiest of 256 CUs with w workgroups `area` per tile of 16 x 64 (mt * nt) and `edge` per operand tile that it
// fetches (mt + 4 nt); once: `fixed`, and `out` per 8 tiles of 16 x 64 that the CU stores.  Measured on 426 products of 660 .. 8192 rows, 384 .. 4096 columns, K 384 .. 4096, each with all
// fifteen tiles (products, residual updates, queries with keys and values): 4 % slower than the best tile on average, 13 % at the ninth decile, where the largest useful area is 11 % and 30 %; on
// 42 hidden layers of 660 .. 1024 rows, 8192 .. 40960 columns, K 512 and 1024: 2 % and 6 %, by area 3 % and 8 % (1024 x 8192 x 512 17.1 us, so 14.0; 660 x 16384 x 1024 30.5, 27.1; slowest
// against it 960 x 8192 x 512 13.0, 13.9).  us, by area (beyond K = 3072: one round of 256-column tiles) and by this: 2560 x 1024 x 4096 47.1, 33.2;  4096 x 3072 x 1024 40.4, 31.6;  8192
// x 1024 x 1024 32.8, 25.5;  3072 x 1536 x 512 12.7, 9.9.  By more than 10 % slower than the best 65 of the 468 (900 x 3072 x 1024 14.9, 10.9).  Fitted again to these the constants choose as well.
// Shorter K, where a workgroup's first loads are most of its time, goes by area up to 5000 rows: of 178 products of K = 64 .. 256 slower than the best tile on average, by area and by cost: up to
// 1100 rows 7 %, 15;  up to 5000 9, 16;  8192 rows 9, 8.  (K = 320 6, 5.)  Encodes, us: d = 64, 2048 rows 175, 184;  d = 128, 2048 167, 176;  d = 256, 4096 261, 271;  1536 206, 204;  d = 128,
// 8192 258, 247.
constexpr int LDSX_COST_M = 640, LDSX_COST_K = 320, LDSX_COST_SHORT_K_M = 5000;
inline float ldsx_cost(int M, int N, int K, int mt, int nt) {
  struct C { float fixed, area, edge, lat, out; };
  constexpr C of[4] = {{3.65f, .20f, .15f, 1.46f, 1.05f}, {1.49f, .30f, .09f, 8.05f, 1.36f}, {3.31f, .34f, .12f, 3.81f, .75f}, {3.15f, .42f, .18f, 1.98f, .56f}};
  const C& c = of[nt == 4 ? (mt >= 4 ? 0 : 1) : (nt == 2 ? 2 : 3)];
  const long wgs = (long)((M + 16 * mt - 1) / (16 * mt)) * ((N + 64 * nt - 1) / (64 * nt)), w = (wgs + 255) / 256;
  const int side_by_side = ldsx_side_by_side(mt, nt);
  const float k = K / 1024.f, busy = w * (c.area * (mt * nt) + c.edge * (mt + 4 * nt)) * k, alone = (w + side_by_side - 1) / side_by_side * c.lat * k;
  return c.fixed + (busy > alone ? busy + .5f * alone : alone + .5f * busy) + c.out * w * (mt * nt) * .125f;
}
inline bool pick_tile_by_cost(int M, int N, int K, int& mt, int& nt) {
  float best = 0.f;
  for (int n : {4, 2, 1})
    for (int m : {8, 7, 5, 4, 3, 2, 1}) {
      if (K % (n == 4 && m >= 4 ? 128 : 256 / n) != 0 || (n == 1 ? m > 3 : m == 1)) continue;
      const float c = ldsx_cost(M, N, K, m, n);
      if (best == 0.f || c < best) { best = c; mt = m; nt = n; }
    }
  return best > 0.f;
}
// Several groups with a long K and few rows (the heads' output layers) stream their weights, and what counts are the rounds of one workgroup per CU: us by row tiles and rounds, of
// 8 and 10 groups of 4096 x 1024 out of memory.  us, by largest useful area and by this: 8 groups, 64 rows 26.1, 22.7;  80 33.2, 23.9;  104 35.2, 29.4;  130 46.0, 33.4;  10 groups,
// 64 rows 36.9, 30.7;  80 35.6, 28.0;  130 37.3, 33.3;  2048 x 512, 10 groups, 104 rows 12.6, 10.4.  (Two groups: not measured.)  K slices of 2048 or more go by it, too: six layers of d = 1024, d_ff = 8192, 130 rows 438, 420, in four slices of
// 48-row tiles instead of eight of 32;  d_ff = 16384 578, 548;  d = 2048, d_ff = 8192 783, 744;  other sliced blocks of 24 .. 144 rows the same.  Up to 256 column blocks of 64 in all groups
// together: of 427 of 3 .. 16 groups, K 2048 .. 4096, N 256 .. 2048, 17 .. 144 rows, that come out otherwise, 344 are faster by more than 2 % (4096 x 1024, 16 groups, 144 rows 92.7, 49.1),
// 47 slower, by up to 8 %, at 280 .. 360 workgroups of 16 rows (3 groups, 96 rows 18.8, 20.2).  More column blocks have tiles of 32 rows or more and 128 columns, two to a CU in one
// round, where the map deals whole groups to XCDs (ldsx_map_of): those are kept: 4096 x 2048, 16 groups, 64 rows 55.6, by rounds 65.6;  128 rows 69.3, 88.3;  6144 x 1536, 12
// groups, 96 rows 63.3, 74.1.  (The map does not: 13 groups, 96 rows 124.9, by rounds 79.5.  More than one round: 4096 x 2048, 12 groups, 96 rows 69.7, 54.8.)
constexpr int LDSX_ROUNDS_M = 144, LDSX_ROUNDS_COLS = 256;
inline int ldsx_rounds_cost(int mt, long wgs) {
  constexpr int us[3][4] = {{190, 235, 340, 430}, {225, 290, 365, 440}, {239, 334, 430, 530}};
  const long r = (wgs + 255) / 256;
  return r <= 4 ? us[mt - 1][r - 1] : us[mt - 1][3] + (int)(r - 4) * 100;
}
// by_cost: not for the vocabulary projection, which stores nothing
void pick_tile(int M, int N, int K, long zdim, int& mt, int& nt, int mt_max = 8, bool by_cost = true) {
  if (by_cost && M > (K >= LDSX_COST_K ? LDSX_COST_M : LDSX_COST_SHORT_K_M) && zdim == 1 && mt_max >= 8 && pick_tile_by_cost(M, N, K, mt, nt)) return;
  pick_tile_by_area(M, N, K, zdim, mt, nt, mt_max);
  if (zdim > 2 && K >= 2048 && K % 256 == 0 && M > 16 && M <= LDSX_ROUNDS_M && mt_max >= 3) {
    const long wide = (N / 16 + 7) / 8;
    if ((N / 16 + 3) / 4 * zdim > LDSX_ROUNDS_COLS && nt == 2 && mt >= 2 && (M + 16 * mt - 1) / (16 * mt) * wide * zdim <= 2 * LDSX_ROUNDS_COLS && wide % 2 == 0 && wide / 2 * zdim % 8 == 0) return;
    int best = 0;
    for (int m : {1, 2, 3}) {
      const int c = ldsx_rounds_cost(m, (long)((M + 16 * m - 1) / (16 * m)) * ((N / 16 + 3) / 4) * zdim);
      if (best == 0 || c < best) { best = c; mt = m; nt = 1; }
    }
    return;
  }
}

// In-place residual update with a long K and few output tiles on the LDS-staged kernel: the number of K slices it is
// split into (1: not split): the fewest with which a tile of at least 48 rows still fills the chip; if no slicing gets
// there, the most slices allowed (each at least 512 deep: two chunks; 80 x 2048 x 512 took 4 us more per step as eight
// slices of 256 than as four of 512).  n_kpart: capacity of the slice buffer in floats.
inline int residual_k_slices_of(int d_model, size_t n_kpart, int M, int N, int K) {
  if (N != d_model || K < 2048 || K % 64 != 0) return 1;
  int mt, nt, ns = 1;
  pick_tile(M, N, K, 1, mt, nt, 8, false);
  if (nt == 1 && mt < 3) {
    for (int t = 2; t <= KSPLIT_MAX && K % (t * 512) == 0 && (size_t)t * M * N <= n_kpart; t *= 2) {
      ns = t;
      pick_tile(M, N, K / t, t, mt, nt);
      if (nt > 1 || mt >= 3) break;
    }
  }
  return ns;
}

// Workgroups per (head, sequence, row tile) of an attention launch: few such pairs over a long cache deal the 256-key
// chunks to several workgroups whose partial softmax results a second kernel merges.
// (the committed length is on the device, but it grows by at most k_max per step: the host knows a bound on the keys)
inline int attention_nsplit_of(const bpd_config& c, long steps, int local_q, int local_m, int cap, int B, int R, int causal) {
  long keys_max = cap;
  if (causal && steps * c.k_max + R < keys_max) keys_max = steps * c.k_max + R;
  // (local attention: the chunks start at the first row's window and end at the last row)
  if (causal && local_q > 0 && (long)local_q + local_m + R < keys_max) keys_max = (long)local_q + local_m + R;
  const int tiles = (R + 15) / 16, chunks = (int)((keys_max + 255) / 256), wgs = c.n_heads * B * tiles;
  int nsplit = 1;
  if (chunks >= 3 && wgs * 2 <= ATTN_PART_SLOTS) {
    nsplit = ATTN_PART_SLOTS / wgs;
    if (nsplit > chunks) nsplit = chunks;
    if (nsplit > 16) nsplit = 16;
  }
  return nsplit;
}

}  // namespace
