// Host side of libbpd: workspace layout, weight loading, and the launch sequences behind
// the C ABI declared in include/bpd.h.  Every step of the method runs in the kernels of
// bpd_kernels.h; this file only orders them on the caller's stream.
#include "../../include/bpd.h"
#include "bpd_kernels.h"
#include "bpd_stack.h"
#include "bpd_host_logic.h"

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <array>
#include <atomic>
#include <initializer_list>
#include <map>
#include <string>
#include <vector>

namespace {

}  // namespace
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];
namespace {
void* g_scratch_ptr[MAX_DEVICES] = {};     // address of `scratch` on each device that has created a context

enum Kind { MAT, MATK_CAT, MATK_SEP, EMB, VEC };
struct WEntry {
  Kind kind;
  int nd; int64_t shape[4];
  void* dst;
  int K, N, ldw, n_off;      // matrices: source K x N, destination row length, column offset
  bool loaded;
};

// A sequence of launches that depends on nothing but `key`: one word for each setting (packed into one word, settings of any size collide)
typedef std::array<long, 9> PlanKey;
struct Plan { PlanKey key; int seen; bool failed; hipGraphExec_t exec; unsigned long long used; };

}  // namespace

struct bpd_ctx {
  bpd_config cfg;
  hipStream_t stream;
  Layout lay;
  std::map<std::string, WEntry> table;
  std::string err;
  int B = 0, S = 0;
  bool encoded = false;
  bool fold_ready = false;        // the folded copies match the loaded weights
  int64_t steps = 0;              // steps enqueued since bpd_encode: bounds the cache lengths (the count itself is on the device, StateP::steps_done)
  int distance_eps = 0, min_block = 1, top_n = 1, two_phase = 0;
  int local_q = 0, local_m = 0;   // 1D local self-attention in the decoder (0: full causal), bpd_set_local_attention
  int num_cus = 256;                   // compute units of the device the context was created on
  int device = 0;                      // that device's index
  // decoder stack kernel: placement of workgroups on XCDs as probed at creation (workers = 0: not usable), the value
  // its flags take next, and whether a launch has reported a timeout (then the per-operator kernels take over)
  int stack_xcc = 0, stack_nx = 0, stack_workers = 0;
  unsigned stack_epoch = 0;
  bool stack_off = false;
  int x_ready_k = 0, x_ready_slots = 0;  // x_ready_k > 0: the last step's accept kernel already embedded the next block: that many rows
                                         // for each of so many slots
  // rows of the invocation being run: slots of sequences (StateP::slot_seq).  seq: their sequences (null: slot = sequence);
  // live: their number on the device where the host only knows a bound, Bs (null: exactly Bs)
  int Bs = 0; const int* seq = nullptr; const int* live = nullptr;
  int live1 = -1, live2 = -1;            // sequences that had not ended after the last step and after the one before (-1: not known)
  int budget_min = 0;                    // smallest length budget of the batch as far as the host knows
  // workgroups per XCD that layers_kernel and wide_layers_kernel wait for (for tests, BPD_LAYERS_GROUP at creation: fewer; 33: they wait in vain; 64 n
  // added: the second one is left to n XCDs).  0: none of the kernels of all layers is used
  int layers_group = LK_PLACES;
  bool layers_ran = false;             // a kernel of all layers has been launched and the kernel behind it has not (that one clears layers_sync)
  bool layers_normed = false;          // ... and has left the normalised rows in hn and h
  bool weights_exceed_llc = false;     // decoder-side weights read per step > 192 MB (the Infinity Cache holds 256 MB)
  const int* cur_imposed = nullptr; int cur_imposed_stride = 0, cur_imposed_step = 0;   // of the step being run
  // pinned host memory, read and written by kernels directly: the words that say what has happened, the arguments of
  // bpd_encode / a host schedule, and results on their way to the caller
  unsigned long long* report = nullptr;       // [2][max_batch] bpd_decode: tokens still to come, tagged with the step; steps
                                              // take turns (the next one may report before the host has looked)
  unsigned long long* done = nullptr;         // [0]: last finished fetch, [1]: last encode whose staged arguments have been read
  int *stage_in = nullptr, *stage_sched = nullptr, *stage_out = nullptr;
  size_t n_stage_out = 0;
  unsigned long long fetch_tag = 0, encode_tag = 0;        // encode_tag: of the last encode whose arguments were staged
  unsigned report_tag = 0;
  bool replayable = false;                     // a call has been captured by the caller: forget_replayed()
  std::vector<int> remaining;                  // tokens still to come per sequence as far as the host knows (-1: it does not)
  std::vector<Plan> plans[2];                  // launches seen before, as graphs (run_planned): encodes, steps
  std::vector<hipGraphExec_t> retired;         // ... given up, but perhaps still running (release_retired)
  hipStream_t plan_stream = nullptr;           // where they are recorded
  int prof_phase = 0;
  std::vector<hipEvent_t> prof_ev;
  size_t prof_used = 0;
  int64_t prof_launches = 0;
  // a split-K residual update whose slices the next LayerNorm of `pend_x` still has to add
  int pend_slices = 0; const float* pend_bias = nullptr; const float* pend_x = nullptr;
};

namespace {

int fail(bpd_ctx* c, int code, const std::string& msg) {
  if (c) c->err = msg;
  return code;
}
#define HIPCHK(expr)                                                                   \
  do {                                                                                 \
    hipError_t _e = (expr);                                                            \
    if (_e != hipSuccess)                                                              \
      return fail(ctx, BPD_E_HIP, std::string(#expr) + ": " + hipGetErrorString(_e)); \
  } while (0)
#define LAUNCHCHK() HIPCHK(hipGetLastError())

void add_entry(bpd_ctx* ctx, const std::string& name, Kind kind, std::vector<int64_t> shape, void* dst,
               int K = 0, int N = 0, int ldw = 0, int n_off = 0) {
  WEntry e{};
  e.kind = kind; e.nd = (int)shape.size();
  for (int i = 0; i < e.nd; ++i) e.shape[i] = shape[i];
  e.dst = dst; e.K = K; e.N = N; e.ldw = ldw; e.n_off = n_off; e.loaded = false;
  ctx->table[name] = e;
}

void build_table(bpd_ctx* ctx) {
  const bpd_config& c = ctx->cfg;
  Layout& L = ctx->lay;
  const int d = c.d_model, F = c.d_ff, V = c.vocab, k = c.k_max;
  const int slots = c.max_out_len + c.k_max + 1;
  auto ln = [&](const std::string& p, LnW w) {
    add_entry(ctx, p + ".g", VEC, {d}, w.g);
    add_entry(ctx, p + ".b", VEC, {d}, w.b);
  };
  add_entry(ctx, "emb", EMB, {V, d}, L.emb, d, V, V, 0);
  add_entry(ctx, "pos_src", VEC, {c.max_src_len, d}, L.pos_src);
  add_entry(ctx, "pos_tgt", VEC, {slots, d}, L.pos_tgt);
  for (int l = 0; l < c.n_enc_layers; ++l) {
    const std::string p = "enc." + std::to_string(l);
    EncL& e = L.enc[l];
    ln(p + ".ln1", e.ln1); ln(p + ".ln2", e.ln2);
    add_entry(ctx, p + ".self.wq", MAT, {d, d}, e.wqkv, d, d, 3 * d, 0);
    add_entry(ctx, p + ".self.wk", MAT, {d, d}, e.wqkv, d, d, 3 * d, d);
    add_entry(ctx, p + ".self.wv", MAT, {d, d}, e.wqkv, d, d, 3 * d, 2 * d);
    add_entry(ctx, p + ".self.wo", MAT, {d, d}, e.wo, d, d, d, 0);
    add_entry(ctx, p + ".ffn.w1", MAT, {d, F}, e.w1, d, F, F, 0);
    add_entry(ctx, p + ".ffn.b1", VEC, {F}, e.b1);
    add_entry(ctx, p + ".ffn.w2", MAT, {F, d}, e.w2, F, d, d, 0);
    add_entry(ctx, p + ".ffn.b2", VEC, {d}, e.b2);
  }
  ln("enc.lnf", L.enc_lnf);
  for (int l = 0; l < c.n_dec_layers; ++l) {
    const std::string p = "dec." + std::to_string(l);
    DecL& e = L.dec[l];
    ln(p + ".ln1", e.ln1); ln(p + ".ln2", e.ln2); ln(p + ".ln3", e.ln3);
    add_entry(ctx, p + ".self.wq", MAT, {d, d}, e.wqkv, d, d, 3 * d, 0);
    add_entry(ctx, p + ".self.wk", MAT, {d, d}, e.wqkv, d, d, 3 * d, d);
    add_entry(ctx, p + ".self.wv", MAT, {d, d}, e.wqkv, d, d, 3 * d, 2 * d);
    add_entry(ctx, p + ".self.wo", MAT, {d, d}, e.wo, d, d, d, 0);
    add_entry(ctx, p + ".cross.wq", MAT, {d, d}, e.cq, d, d, d, 0);
    add_entry(ctx, p + ".cross.wk", MAT, {d, d}, e.ckv, d, d, 2 * d, 0);
    add_entry(ctx, p + ".cross.wv", MAT, {d, d}, e.ckv, d, d, 2 * d, d);
    add_entry(ctx, p + ".cross.wo", MAT, {d, d}, e.co, d, d, d, 0);
    add_entry(ctx, p + ".ffn.w1", MAT, {d, F}, e.w1, d, F, F, 0);
    add_entry(ctx, p + ".ffn.b1", VEC, {F}, e.b1);
    add_entry(ctx, p + ".ffn.w2", MAT, {F, d}, e.w2, F, d, d, 0);
    add_entry(ctx, p + ".ffn.b2", VEC, {d}, e.b2);
  }
  ln("dec.lnf", L.dec_lnf);
  add_entry(ctx, "head.w1", MATK_CAT, {k, d, F}, L.hw1, d, F, k * F, 0);
  add_entry(ctx, "head.b1", VEC, {k, F}, L.hb1);
  add_entry(ctx, "head.w2", MATK_SEP, {k, F, d}, L.hw2, F, d, d, 0);
  add_entry(ctx, "head.b2", VEC, {k, d}, L.hb2);
}

// ------------------------------------------------------------------------------- launches

template <int MT, int NT, int KS>
void launch_gemm_bf16(const GemmP& p, const Epi& e, int groups, hipStream_t s) {
  const int ntiles = p.N / 16;
  dim3 grid(KS == 4 ? (ntiles + NT - 1) / NT : (ntiles + 4 * NT - 1) / (4 * NT), (p.M + 16 * MT - 1) / (16 * MT), groups);
  hipLaunchKernelGGL((gemm_bf16_kernel<MT, NT, KS>), grid, dim3(256), 0, s, p, e);
}

// ---- skinny path: M <= 16 -------------------------------------------------------------
template <int MT, int NT, int XLN, bool ARGMAX, int WAVES, int U, int DEPTH, bool STREAM>
void launch_skinny_cfg(const bpd_ctx* ctx, const GemmP& p, const Epi& e_in, const LnP& ln, unsigned long long* keys,
                       float* logits, int groups) {
  hipStream_t s = ctx->stream;
  Epi e = e_in;                                 // the kernel loads bias and residual unconditionally
  if (!e.bias) { e.bias = ctx->lay.zeros; e.bias_g = 0; }
  if (!e.R) { e.R = ctx->lay.zeros; e.ldr = 0; e.r_g = 0; }
  const int ntiles = p.N / 16;
  const int ngroups = (ntiles + NT - 1) / NT;
  // more column-tile groups than CUs: one workgroup per CU walks several of them (a second workgroup on a CU would only
  // start once the first has finished: the kernel fills the register file)
  const int cap = ctx->num_cus;
  const int gx = ngroups > cap ? cap : ngroups;
  dim3 grid(gx, (p.M + 16 * MT - 1) / (16 * MT), groups);
  const size_t lds = (size_t)2 * WAVES * MT * NT * 1024;
  if (ngroups > gx) {
    auto k = skinny_gemm_kernel<XLN == 2 ? 0 : MT, NT, XLN != 0, ARGMAX, WAVES, U, DEPTH, STREAM>;
    static bool attr = false;
    if (!attr) { (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); attr = true; }
    hipLaunchKernelGGL(k, grid, dim3(64 * WAVES), lds, s, p, e, ln, keys, logits);
  } else {
    auto k = skinny_gemm_kernel<XLN == 2 ? 0 : MT, NT, XLN != 0, ARGMAX, WAVES, U, 0, STREAM>;
    static bool attr = false;
    if (!attr) { (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); attr = true; }
    hipLaunchKernelGGL(k, grid, dim3(64 * WAVES), lds, s, p, e, ln, keys, logits);
  }
}

// One 16-row tile (M <= 16): K split over the waves so that each wave holds all its k-steps.
template <int NT, int XLN, bool ARGMAX, bool STREAM>
void launch_skinny_s(const bpd_ctx* ctx, const GemmP& p, const Epi& e, const LnP& ln, unsigned long long* keys, float* logits,
                     int groups) {
  // waves x k-steps per wave cover K / 32 without idle slots (an idle slot still costs its clamped load)
  if (XLN && p.K <= 512) launch_skinny_cfg<1, NT, XLN, ARGMAX, 4, 4, 2, STREAM>(ctx, p, e, ln, keys, logits, groups);
  else if (XLN) launch_skinny_cfg<1, NT, XLN, ARGMAX, 8, 4, 2, STREAM>(ctx, p, e, ln, keys, logits, groups);       // K <= 1024
  else if (p.K <= 512) launch_skinny_cfg<1, NT, 0, ARGMAX, 4, 4, 2, STREAM>(ctx, p, e, ln, keys, logits, groups);
  else if (p.K <= 1024) launch_skinny_cfg<1, NT, 0, ARGMAX, 4, 8, 2, STREAM>(ctx, p, e, ln, keys, logits, groups);
  else if (p.K <= 2048) launch_skinny_cfg<1, NT, 0, ARGMAX, 8, 8, 1, STREAM>(ctx, p, e, ln, keys, logits, groups);
  else launch_skinny_cfg<1, NT, 0, ARGMAX, 8, 16, 1, STREAM>(ctx, p, e, ln, keys, logits, groups);             // K <= 4096
}
// Streams of at least 32 MB in a model whose per-step weights exceed the last-level cache bypass it.
template <int NT, int XLN, bool ARGMAX>
void launch_skinny(const bpd_ctx* ctx, const GemmP& p, const Epi& e, const LnP& ln, unsigned long long* keys, float* logits,
                   int groups) {
  const size_t wbytes = (size_t)p.K * p.N * groups * 2;
  if (ctx->weights_exceed_llc && wbytes >= ((size_t)32 << 20)) launch_skinny_s<NT, XLN, ARGMAX, true>(ctx, p, e, ln, keys, logits, groups);
  else launch_skinny_s<NT, XLN, ARGMAX, false>(ctx, p, e, ln, keys, logits, groups);
}

bool skinny_ok(const bpd_ctx* ctx, const GemmP& p) { return ctx->cfg.dtype == BPD_BF16 && p.M <= 16 && p.K <= 4096; }

// ---- streaming path: M <= 16, K = 2048 / 4096, several column tiles per CU ---------------------
// (the heads' output layers at batch 1).  One workgroup per CU walks a contiguous range of at most
// 8 column tiles of one group.
constexpr int STREAM_TILES_MAX = 8;
size_t stream_lds_bytes(const GemmP& p) { return (size_t)16384 + 8192 + 1536 + (size_t)p.M * (p.K + 8) * 2; }
bool stream_ok(const bpd_ctx* ctx, const GemmP& p, const Epi& e, int groups) {
  return skinny_ok(ctx, p) && p.M >= 1 && e.mode == 0 && !e.stats_out && (p.K == 2048 || p.K == 4096) && p.N % 16 == 0 &&
         2L * groups * (p.N / 16) >= 3L * ctx->num_cus && stream_lds_bytes(p) <= (size_t)160 * 1024;
}
template <int U, bool STREAM>
void launch_stream_cfg(const bpd_ctx* ctx, const GemmP& p, const Epi& e_in, int groups) {
  Epi e = e_in;                                 // bias and residual are loaded unconditionally
  if (!e.bias) { e.bias = ctx->lay.zeros; e.bias_g = 0; }
  if (!e.R) { e.R = ctx->lay.zeros; e.ldr = 0; e.r_g = 0; }
  const int ntiles = p.N / 16;
  int gx = ctx->num_cus / groups;
  const int gx_min = (ntiles + STREAM_TILES_MAX - 1) / STREAM_TILES_MAX;
  gx = gx < gx_min ? gx_min : gx;
  gx = gx > ntiles ? ntiles : gx;
  const size_t lds = stream_lds_bytes(p);
  auto k = stream_gemm_kernel<U, STREAM>;
  static size_t attr = 0;                       // per instantiation: allow more than 64 KiB of LDS
  if (attr < lds) { (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); attr = lds; }
  hipLaunchKernelGGL(k, dim3(gx, 1, groups), dim3(512), lds, ctx->stream, p, e);
}
void launch_stream(const bpd_ctx* ctx, const GemmP& p, const Epi& e, int groups) {
  const size_t wbytes = (size_t)p.K * p.N * groups * 2;
  const bool nt = ctx->weights_exceed_llc && wbytes >= ((size_t)32 << 20);
  if (p.K == 4096) { if (nt) launch_stream_cfg<16, true>(ctx, p, e, groups); else launch_stream_cfg<16, false>(ctx, p, e, groups); }
  else { if (nt) launch_stream_cfg<8, true>(ctx, p, e, groups); else launch_stream_cfg<8, false>(ctx, p, e, groups); }
}
// The accept kernel of a step embeds the next step's block (accept_embed_kernel: bf16, at most 64 column tiles)
bool embed_in_accept(const bpd_ctx* ctx) {
  return ctx->cfg.dtype == BPD_BF16 && ctx->cfg.d_model <= 1024;
}
// Rows of ended sequences are left out of the steps of a batch: the accept kernel that also embeds the next block deals the
// slots (with one sequence there is nothing to pack).
bool slots_used(const bpd_ctx* ctx) { return embed_in_accept(ctx) && ctx->B > 1; }
// Which slots the next invocation of the block runs on.  exact: their number, as a decode knows it (-1: not known, all of
// the batch with the number on the device, unless no sequence can have ended yet).
void use_slots(bpd_ctx* ctx, int exact) {
  ctx->Bs = ctx->B; ctx->seq = nullptr; ctx->live = nullptr;
  if (!slots_used(ctx) || exact == ctx->B) return;
  if (exact < 0 && ctx->cfg.eos_id < 0 && (ctx->steps - 1) * ctx->cfg.k_max < ctx->budget_min) return;
  ctx->seq = ctx->lay.slot_seq;
  if (exact > 0) ctx->Bs = exact; else ctx->live = ctx->lay.n_live;
}
// ... and how a kernel of M rows (of all slots launched) is told to stop short
LiveP live_rows(const bpd_ctx* ctx, int M) { return ctx->live ? LiveP{ctx->live, M / ctx->Bs} : LiveP{nullptr, 0}; }
// LayerNorm statistics ride along with the residual stream when the whole block is one MFMA row tile and every GEMM
// that updates the stream is one the skinny kernel takes (it is the one that writes them: K = d_ff must fit it)
bool stats_path(const bpd_ctx* ctx, int M) {
  return !lean_ok(ctx->cfg, M) && ctx->cfg.dtype == BPD_BF16 && M <= 16 && ctx->cfg.d_model <= 1024 && ctx->cfg.d_ff <= 4096;
}

// ---- ldsx path: many rows ---------------------------------------------------------------
template <int MT, int NT, int KC, bool ARGMAX, bool XLN = false, bool STATS = false, bool ROWAFF = false>
void launch_ldsx(const GemmP& p, const Epi& e, unsigned long long* keys, float* logits, int groups, hipStream_t s, const LiveP& live,
                 const LnP& ln = LnP{}) {
  const int ntiles = p.N / 16;
  dim3 grid((ntiles + 4 * NT - 1) / (4 * NT), (p.M + 16 * MT - 1) / (16 * MT), groups);
  const size_t lds = ldsx_lds_bytes<MT, NT, KC>();
  static bool attr_set = false;                 // per instantiation: allow more than 64 KiB of LDS
  if (!attr_set) {
    (void)hipFuncSetAttribute((const void*)gemm_ldsx_kernel<MT, NT, KC, ARGMAX, XLN, STATS, ROWAFF>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    attr_set = true;
  }
  GemmP q = p;
  q.lx = ldsx_map_of(p.K, KC, p.ksplit, grid.x, grid.y, grid.z);            // (grid.x * grid.y * grid.y * 4 < 2^32 by far: at most a few thousand blocks each way)
  hipLaunchKernelGGL((gemm_ldsx_kernel<MT, NT, KC, ARGMAX, XLN, STATS, ROWAFF>), grid, dim3(256), lds, s, q, e, keys, logits, ln, live);
}

// Tile of the LDS-staged GEMM: 16*mt rows x 64*nt columns per workgroup, K walked in chunks of
// 256 / 128 / 64 for nt = 1 / 2 / 4 (eight weight fragments per wave in flight either way).
// Chosen: the largest tile that still gives the chip about two workgroups per CU (counting K
// slices and groups); ties go to less row padding, then to the narrower tile (longer chunks).
// With nt = 1 at most 48 rows, so that the two 256-deep staging buffers leave room for three
// workgroups per CU.  If nothing qualifies the smallest tile spreads the work furthest.
// e.stats_out (mode 0, one group, no split over K): the kernel also writes the LayerNorm statistics of its output, which
// only the tiles of at most 48 rows are built for.  Returns whether it did.
// Small tiles fetch bias and residual at kernel entry (Epi::pre_epi): absent operands are replaced by a zero-filled vector.
void prefetch_epilogue(Epi& e, const GemmP& p, int mt, int nt, const float* zeros) {
  if (!zeros || mt * nt > 3 || e.mode != 0 || p.ksplit > 1) return;
  if (!e.bias) { e.bias = zeros; e.bias_g = 0; }
  if (!e.R) { e.R = zeros; e.ldr = 0; e.r_g = 0; }
  e.pre_epi = 1;
}

template <bool ARGMAX>
bool dispatch_ldsx(const GemmP& p, const Epi& e_in, unsigned long long* keys, float* logits, int groups, hipStream_t s,
                   const LiveP& live, const float* zeros = nullptr, const LnP& ln = LnP{}) {
  Epi e = e_in;
  int mt, nt;
  const int kslice = p.ksplit > 1 ? p.K / p.ksplit : p.K;
  const bool stats_req = !ARGMAX && e.mode == 0 && e.stats_out != nullptr && groups == 1 && p.ksplit <= 1;
  pick_tile(p.M, p.N, kslice, groups, mt, nt, stats_req ? LDSX_LN_MT_MAX : 8, !ARGMAX);   // groups = K slices for a split-K launch
  // (the statistics are per 64-column block: every wave of a workgroup must own whole tiles of it)
  const bool stats = stats_req && p.N % (64 * nt) == 0;
  if constexpr (!ARGMAX) prefetch_epilogue(e, p, mt, nt, zeros);
  if constexpr (!ARGMAX) {
    if (stats) {
#define BPD_CASE(MT_, NT_, KC_) if (mt == MT_ && nt == NT_) { launch_ldsx<MT_, NT_, KC_, false, false, true>(p, e, keys, logits, groups, s, live); return true; }
      BPD_CASE(3, 1, 256) BPD_CASE(2, 1, 256) BPD_CASE(1, 1, 256)
      BPD_CASE(3, 2, 128) BPD_CASE(2, 2, 128) BPD_CASE(1, 2, 128)
      BPD_CASE(3, 4, 64) BPD_CASE(2, 4, 64) BPD_CASE(1, 4, 64)
#undef BPD_CASE
    }
  }
#define BPD_CASE(MT_, NT_, KC_) if (mt == MT_ && nt == NT_) { launch_ldsx<MT_, NT_, KC_, ARGMAX>(p, e, keys, logits, groups, s, live, ln); return false; }
  BPD_CASE(3, 1, 256) BPD_CASE(2, 1, 256) BPD_CASE(1, 1, 256)
  BPD_CASE(8, 2, 128) BPD_CASE(7, 2, 128) BPD_CASE(5, 2, 128) BPD_CASE(4, 2, 128) BPD_CASE(3, 2, 128) BPD_CASE(2, 2, 128) BPD_CASE(1, 2, 128)
  BPD_CASE(8, 4, 64) BPD_CASE(7, 4, 64) BPD_CASE(5, 4, 64) BPD_CASE(4, 4, 64) BPD_CASE(3, 4, 64) BPD_CASE(2, 4, 64) BPD_CASE(1, 4, 64)
#undef BPD_CASE
  return false;
}

// Y = epilogue(LayerNorm(ln.x) W) on more than 16 rows with the LayerNorm applied while the activations are staged
// (tiles of at most 48 rows: the staging registers).
void dispatch_ldsx_ln(const GemmP& p, const Epi& e_in, const LnP& ln, hipStream_t s, const float* zeros) {
  Epi e = e_in;
  int mt, nt;
  pick_tile(p.M, p.N, p.K, 1, mt, nt, LDSX_LN_MT_MAX);
  prefetch_epilogue(e, p, mt, nt, zeros);
#define BPD_CASE(MT_, NT_, KC_) if (mt == MT_ && nt == NT_) { launch_ldsx<MT_, NT_, KC_, false, true>(p, e, nullptr, nullptr, 1, s, LiveP{}, ln); return; }
  BPD_CASE(3, 1, 256) BPD_CASE(2, 1, 256) BPD_CASE(1, 1, 256)
  BPD_CASE(3, 2, 128) BPD_CASE(2, 2, 128) BPD_CASE(1, 2, 128)
  BPD_CASE(3, 4, 64) BPD_CASE(2, 4, 64) BPD_CASE(1, 4, 64)
#undef BPD_CASE
}
// Y = epilogue(LayerNorm(x) W) with the LayerNorm folded into the weights (e.ra_*): X is the raw bf16 copy of x.
void dispatch_ldsx_fold(const GemmP& p, const Epi& e_in, hipStream_t s, const float* zeros) {
  Epi e = e_in;
  int mt, nt;
  pick_tile(p.M, p.N, p.K, 1, mt, nt, LDSX_LN_MT_MAX);
  prefetch_epilogue(e, p, mt, nt, zeros);
#define BPD_CASE(MT_, NT_, KC_) if (mt == MT_ && nt == NT_) { launch_ldsx<MT_, NT_, KC_, false, false, false, true>(p, e, nullptr, nullptr, 1, s, LiveP{}); return; }
  BPD_CASE(3, 1, 256) BPD_CASE(2, 1, 256) BPD_CASE(1, 1, 256)
  BPD_CASE(3, 2, 128) BPD_CASE(2, 2, 128) BPD_CASE(1, 2, 128)
  BPD_CASE(3, 4, 64) BPD_CASE(2, 4, 64) BPD_CASE(1, 4, 64)
#undef BPD_CASE
}
bool ldsx_ln_ok(const bpd_ctx* ctx, const GemmP& p) {
  return ctx->cfg.dtype == BPD_BF16 && p.M > 16 && p.K == ctx->cfg.d_model && p.K % 64 == 0 && p.K <= 1024 && p.N % 16 == 0;
}

int residual_k_slices(const bpd_ctx* ctx, const GemmP& p) {
  return residual_k_slices_of(ctx->cfg.d_model, ctx->lay.n_kpart, p.M, p.N, p.K);
}

// What the next kernel clears: the words that a kernel of all layers has counted in
uint4* clear_behind_layers(bpd_ctx* ctx, int& n) {
  if (!ctx->layers_ran) return nullptr;
  ctx->layers_ran = false;
  n = LK_WORDS / 4;
  return (uint4*)ctx->lay.layers_sync;
}

// Y = epilogue(X W).  bf16 mode: M <= 16 -> skinny kernel; otherwise the LDS-staged kernel
// (K % 64 == 0) or the plain MFMA kernel.  fp32 mode: one thread per output.
// Returns true if the kernel left the per-tile LayerNorm statistics of its output in e.stats_out in the layout of the
// LDS-staged kernel (more than 16 rows, no split over K).
bool gemm(bpd_ctx* ctx, const GemmP& p, const Epi& e_in, int groups = 1) {
  hipStream_t s = ctx->stream;
  Epi e = e_in;
  if (ctx->cfg.dtype != BPD_BF16) {
    dim3 grid((p.N + 127) / 128, p.M, groups);
    hipLaunchKernelGGL(gemm_f32_kernel, grid, dim3(128), 0, s, p, e);
    return false;
  }
  LnP none{};
  if (stream_ok(ctx, p, e, groups)) {
    launch_stream(ctx, p, e, groups);
  } else if (skinny_ok(ctx, p)) {
    if (p.N / 16 >= 2048) launch_skinny<2, 0, false>(ctx, p, e, none, nullptr, nullptr, groups);
    else launch_skinny<1, 0, false>(ctx, p, e, none, nullptr, nullptr, groups);
  } else if (p.K % 64 == 0) {
    // In-place residual update with a long K and few output tiles: split K over workgroups.  The
    // slices are added, in a fixed order, by the LayerNorm kernel that reads the residual next.
    if (groups == 1 && e.mode == 0 && e.R && e.R == e.Yf && !e.Ya && !e.relu && !e.lnR_stats &&
        e.ldr == p.N && e.ldyf == p.N && p.N == ctx->cfg.d_model && p.K >= 2048) {
      const int ns = residual_k_slices(ctx, p);
      if (ns > 1) {
        GemmP q = p;
        q.ksplit = ns; q.part = ctx->lay.kpart;
        e.stats_out = nullptr;                     // the slices are raw products: no statistics of the sum yet
        dispatch_ldsx<false>(q, e, nullptr, nullptr, ns, s, live_rows(ctx, p.M), ctx->lay.zeros);
        ctx->pend_slices = ns; ctx->pend_bias = e.bias ? e.bias : ctx->lay.zeros; ctx->pend_x = e.Yf;
        return false;
      }
    }
    if (!e.stats_out) none.clear = clear_behind_layers(ctx, none.nclear);
    return dispatch_ldsx<false>(p, e, nullptr, nullptr, groups, s, live_rows(ctx, p.M), ctx->lay.zeros, none);
  } else {
    e.stats_out = nullptr;
    if (p.M > 64) launch_gemm_bf16<8, 1, 4>(p, e, groups, s);
    else launch_gemm_bf16<4, 1, 4>(p, e, groups, s);
  }
  return false;
}

void layernorm(bpd_ctx* ctx, float* x, LnW w, int M, void* ya, float* yf, bool packed = false);

// Y = epilogue(LayerNorm(x) W).  Block of <= 16 rows: LayerNorm is applied inside the skinny
// kernel from the partial statistics the producer of x left in L.stats_ln.  More rows, with per-tile statistics of
// x in L.stats_big: applied while the LDS-staged kernel stages its activations (up to 128 rows) or folded into the
// weights (beyond).  Otherwise a LayerNorm kernel (into `xn`, and `yf` in fp32 if given) followed by the GEMM.
void gemm_ln(bpd_ctx* ctx, float* x, LnW w, void* xn, float* yf, GemmP p, const Epi& e, bool with_stats, bool big_stats = false,
             const FoldW* fold = nullptr) {
  // fold: the producer of x left its bf16 copy in xn and per-tile statistics in L.stats_big (more than 128 rows): one
  // GEMM on the weights with this LayerNorm folded in
  if (fold && fold->W && big_stats && !yf && ldsx_ln_ok(ctx, p)) {
    p.X = xn; p.W = fold->W;
    Epi ef = e;
    ef.ra_stats = ctx->lay.stats_big; ef.ra_c = fold->c; ef.ra_d = fold->d; ef.ra_eps = ctx->cfg.ln_eps;
    dispatch_ldsx_fold(p, ef, ctx->stream, ctx->lay.zeros);
    return;
  }
  // with_stats: the producer of x left its partial LayerNorm statistics in L.stats_ln (decoder block of one
  // row tile only; the encoder's kernels do not write them)
  if (with_stats && stats_path(ctx, p.M) && p.K == ctx->cfg.d_model) {
    LnP ln{x, w.g, w.b, ctx->lay.stats_ln, ctx->cfg.ln_eps};
    if (p.N / 16 >= 2048) launch_skinny<2, 1, false>(ctx, p, e, ln, nullptr, nullptr, 1);
    else launch_skinny<1, 1, false>(ctx, p, e, ln, nullptr, nullptr, 1);
    return;
  }
  // big_stats: more than 16 rows and the GEMM that produced x left per-tile statistics in L.stats_big
  if (big_stats && !yf && p.M <= LDSX_LN_M_MAX && ldsx_ln_ok(ctx, p)) {
    LnP ln{x, w.g, w.b, ctx->lay.stats_big, ctx->cfg.ln_eps};
    dispatch_ldsx_ln(p, e, ln, ctx->stream, ctx->lay.zeros);
    return;
  }
  layernorm(ctx, x, w, p.M, xn, yf);
  p.X = xn;
  gemm(ctx, p, e);
}

// Vocabulary projection with fused arg-max (bf16 mode).
// ---- streaming vocabulary projection: 17 .. 128 rows, K = 512 / 1024, at least one column tile per wave ----
size_t stream_vocab_lds_bytes(const GemmP& p) {
  const int rows = p.M < 64 ? p.M : 64;
  return (size_t)8 * 64 * 8 + (size_t)rows * (p.K + 8) * 2;
}
// workgroups per row block: one per CU of the row block's share, fewer when that leaves a wave less than two units of
// 16 weight loads to take turns with (K = 512: a unit is a whole column tile; 32000 columns at 64 rows: 14.5 us with
// 100 .. 167 workgroups, 15.5 us with 250, whose 250 atomics per row also cost more)
int stream_vocab_gx(const bpd_ctx* ctx, const GemmP& p) {
  const int rb = (p.M + 63) / 64, per = p.K == 512 ? 12 : 8;      // column tiles per workgroup, at least
  int gx = ctx->num_cus / rb;
  if (gx > p.N / 16 / per) gx = p.N / 16 / per;
  return gx < 1 ? 1 : gx;
}
bool stream_vocab_ok(const bpd_ctx* ctx, const GemmP& p) {
  const int rb = (p.M + 63) / 64;
  return ctx->cfg.dtype == BPD_BF16 && p.M > 16 && p.M <= 128 && (p.K == 512 || p.K == 1024) && p.N % 16 == 0 &&
         p.ldx % 8 == 0 && 2 * rb * stream_vocab_gx(ctx, p) >= ctx->num_cus &&       // at least half the chip streams
         stream_vocab_lds_bytes(p) <= (size_t)160 * 1024;
}
template <int NT, int UPT>
void launch_stream_vocab_cfg(const bpd_ctx* ctx, const GemmP& p, unsigned long long* keys, float* logits) {
  const size_t lds = stream_vocab_lds_bytes(p);
  auto k = stream_vocab_kernel<4, NT, UPT, false>;
  static size_t attr = 0;                       // per instantiation: allow more than 64 KiB of LDS
  if (attr < lds) { (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); attr = lds; }
  hipLaunchKernelGGL(k, dim3(stream_vocab_gx(ctx, p), (p.M + 63) / 64), dim3(512), lds, ctx->stream, p, keys, logits, live_rows(ctx, p.M));
}
void launch_stream_vocab(const bpd_ctx* ctx, const GemmP& p, unsigned long long* keys, float* logits) {
  // one column tile at a time.  Two at a time (NT = 2: one LDS read feeds two MFMAs) measured slower, 20.2 vs 18.5 us at
  // 100 x 1024 x 32768, and so did non-temporal loads (the second row block reads the same weights out of L2).
  if (p.K == 1024) launch_stream_vocab_cfg<1, 2>(ctx, p, keys, logits);
  else launch_stream_vocab_cfg<1, 1>(ctx, p, keys, logits);
}

void vocab_argmax(bpd_ctx* ctx, const GemmP& p, unsigned long long* keys, float* logits) {
  hipStream_t s = ctx->stream;
  Epi none{};
  LnP noln{};
  if (skinny_ok(ctx, p)) launch_skinny<2, 0, true>(ctx, p, none, noln, keys, logits, 1);
  else if (stream_vocab_ok(ctx, p)) launch_stream_vocab(ctx, p, keys, logits);
  else if (p.K % 64 == 0) dispatch_ldsx<true>(p, none, keys, logits, 1, s, live_rows(ctx, p.M));
  else {
    const int ntiles = p.N / 16;
    dim3 grid(ntiles, (p.M + 127) / 128, 1);
    hipLaunchKernelGGL((vocab_argmax_bf16_kernel<8, 1, 4>), grid, dim3(256), 0, s, p, keys, logits);
  }
}

GemmP gp(const void* X, int ldx, const void* W, int ldw, int M, int N, int K) {
  GemmP p{};
  p.X = X; p.ldx = ldx; p.W = W; p.ldw = ldw; p.M = M; p.N = N; p.K = K;
  return p;
}
Epi plain(const float* bias, int relu, const float* R, int ldr, float* Yf, int ldyf, void* Ya, int ldya) {
  Epi e{};
  e.mode = 0; e.bias = bias; e.relu = relu; e.R = R; e.ldr = ldr; e.Yf = Yf; e.ldyf = ldyf; e.Ya = Ya; e.ldya = ldya;
  return e;
}
Epi split(float* Qf, void* Ka, void* Va, int dsplit, int chunk0, int rows_per_seq, int cap, const int* base) {
  Epi e{};
  e.mode = 1; e.Qf = Qf; e.Ka = Ka; e.Va = Va; e.dsplit = dsplit; e.chunk0 = chunk0;
  e.rows_per_seq = rows_per_seq; e.cap = cap; e.base = base;
  return e;
}
// Where a block's keys and values go: `rows` cache rows per sequence, R new ones for each slot at base (null: from the first)
Epi kv_split(const bpd_ctx* ctx, float* Qf, void* Ka, void* Va, int chunk0, int R, int rows, const int* lens, const int* seq) {
  const bool grouped = kv_grouped(ctx->cfg);
  Epi e = split(Qf, Ka, Va, ctx->cfg.d_model, chunk0, R, seq && !grouped ? 0 : rows, seq && !grouped ? ctx->lay.slot_row : lens);
  if (grouped) { e.capg = (rows + 31) / 32; e.seq = seq; }
  return e;
}

template <int D>
void launch_ln_row(bpd_ctx* ctx, float* x, LnW w, int M, void* ya, float* yf, int nsl, const float* bias, bool packed) {
  const dim3 grid(packed ? (M + 127) / 128 * 128 : M);
#define BPD_LN(NSL) hipLaunchKernelGGL((ln_row_kernel<D, NSL>), grid, dim3(ln_row_threads(D)), 0, ctx->stream, x, w.g, w.b, M, ctx->cfg.ln_eps, \
                                       (bf16_t*)ya, yf, (const float*)ctx->lay.kpart, bias, clear, nclear, (int)packed)
  int nclear = 0;
  u32x4* clear = (u32x4*)clear_behind_layers(ctx, nclear);
  switch (nsl) {
    case 0: BPD_LN(0); break;
    case 2: BPD_LN(2); break;
    case 3: BPD_LN(3); break;
    case 4: BPD_LN(4); break;
    case 8: BPD_LN(8); break;
    default: BPD_LN(16); break;
  }
#undef BPD_LN
}
// packed (widths of constant K): ya as row_gemm_kernel reads it
void layernorm(bpd_ctx* ctx, float* x, LnW w, int M, void* ya, float* yf, bool packed) {
  const int d = ctx->cfg.d_model;
  dim3 grid((M + 3) / 4);
  int nsl = 0;
  const float* bias = nullptr;
  if (ctx->pend_slices && ctx->pend_x == x) { nsl = ctx->pend_slices; bias = ctx->pend_bias; ctx->pend_slices = 0; }
  if (ctx->cfg.dtype == BPD_BF16 && lean_width(d) && (nsl == 0 || nsl == 2 || nsl == 3 || nsl == 4 || nsl == 8 || nsl == 16)) {
    switch (d) {
      case 128: launch_ln_row<128>(ctx, x, w, M, ya, yf, nsl, bias, packed); break;
      case 256: launch_ln_row<256>(ctx, x, w, M, ya, yf, nsl, bias, packed); break;
      case 512: launch_ln_row<512>(ctx, x, w, M, ya, yf, nsl, bias, packed); break;
      case 768: launch_ln_row<768>(ctx, x, w, M, ya, yf, nsl, bias, packed); break;
      default: launch_ln_row<1024>(ctx, x, w, M, ya, yf, nsl, bias, packed); break;
    }
    return;
  }
#define BPD_LN(ACT_, V_) hipLaunchKernelGGL((layernorm_kernel<ACT_, V_>), grid, dim3(256), 0, ctx->stream, x, w.g, w.b, M, d, \
                                            ctx->cfg.ln_eps, (ACT_*)ya, yf, (const float*)ctx->lay.kpart, nsl, bias)
  if (ctx->cfg.dtype == BPD_BF16) {
    if (d <= 1024) BPD_LN(bf16_t, 4); else BPD_LN(bf16_t, LN_V);
  } else {
    if (d <= 1024) BPD_LN(float, 4); else BPD_LN(float, LN_V);
  }
#undef BPD_LN
}

// merge of the split attention's partial results: as few partials read per thread as the split needs
template <typename ACT, int DH>
void launch_combine(const AttnP& p, dim3 grid, hipStream_t s) {
  if (p.nsplit <= 4) hipLaunchKernelGGL((attention_combine_kernel<ACT, DH, 4>), grid, dim3(256), 0, s, p);
  else if (p.nsplit <= 8) hipLaunchKernelGGL((attention_combine_kernel<ACT, DH, 8>), grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL((attention_combine_kernel<ACT, DH, 16>), grid, dim3(256), 0, s, p);
}

int attention_nsplit(const bpd_ctx* ctx, int cap, int B, int R, int causal) {
  return attention_nsplit_of(ctx->cfg, (long)ctx->steps, ctx->local_q, ctx->local_m, cap, B, R, causal);
}

// keys of a sequence as far as the host knows a bound
long attention_keys(const bpd_ctx* ctx, int cap, int R, int causal) {
  return causal ? std::min<long>(cap, (long)ctx->steps * ctx->cfg.k_max + 1 + R) : cap;
}

// Cross-attention whose query projection runs inside the attention kernel: LayerNorm statistics of x at hand (the
// caller checks), at most 16 rows per sequence, 64-wide heads, d = 128 / 256 / 512 / 1024, one workgroup per (head,
// sequence) and few enough of them that each streaming its head's 128 d bytes of weights beats one GEMM doing it once.
constexpr int ATTN_QPROJ_MAX_WGS = 128;       // (512 workgroups, batch 32 of Transformer-big: the step took 26 us longer than with the separate GEMM)
// More of them, up to a workgroup per CU, go two sequences to a workgroup (d = 512, 1024, whose parts of 128 columns divide among eight waves; room for at most 128 source tokens, a group of
// 32 keys for each wave).  Steps of four layers, us, as separate kernels and so, by sequences x rows:  d = 1024, d_ff 4096, 32 x 10 403, 380;  d_ff 1280 (statistics, folded weights) 10 x 4 210, 196;
// 20 x 10 302, 292;  d = 512, d_ff 2048, 40 x 4 172, 159;  64 x 8 264, 248;  folded weights 60 x 12 318, 312;  64 x 16 395, 390.  More workgroups than CUs gain nothing: d = 1024, 40 x 5 304, 308;
// 48 x 10 542, 544;  48 x 1 201, 213;  64 x 5 372, 367.  The kernel alone by trace 9.9 at 32 x 10 rows, 8.9 at 32 x 1.
constexpr int ATTN_QPROJ_MAX_PAIRS = 256;
bool attention_qproj_pairs(const bpd_ctx* ctx, int B) {
  const bpd_config& c = ctx->cfg;
  return c.n_heads * B > ATTN_QPROJ_MAX_WGS && c.n_heads * ((B + 1) / 2) <= ATTN_QPROJ_MAX_PAIRS && (c.d_model == 512 || c.d_model == 1024) && c.max_src_len <= 128;
}
bool attention_qproj_ok(const bpd_ctx* ctx, int B, int R) {
  const bpd_config& c = ctx->cfg;
  const int d = c.d_model;
  return c.dtype == BPD_BF16 && R <= 16 && d == 64 * c.n_heads && (d == 128 || d == 256 || d == 512 || d == 1024) &&
         (c.n_heads * B <= ATTN_QPROJ_MAX_WGS || attention_qproj_pairs(ctx, B)) && attention_nsplit(ctx, c.max_src_len, B, R, 0) == 1;
}

template <int QU>
void launch_attention_pairs(const bpd_ctx* ctx, const AttnP& p, const QProjP& qp, int B) {
  constexpr int lds = AttnPairsLds<QU>::BYTES;
  static bool attr_set = false;                 // per width: allow more than 64 KiB of LDS
  if (!attr_set) {
    for (const void* k : {(const void*)attention_mfma_pairs_kernel<QU, true>, (const void*)attention_mfma_pairs_kernel<QU, false>}) (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    attr_set = true;
  }
  const dim3 grid(ctx->cfg.n_heads, (B + 1) / 2);
  if (p.seq) hipLaunchKernelGGL((attention_mfma_pairs_kernel<QU, true>), grid, dim3(64 * ATTN_WAVES), lds, ctx->stream, p, qp, B);
  else hipLaunchKernelGGL((attention_mfma_pairs_kernel<QU, false>), grid, dim3(64 * ATTN_WAVES), lds, ctx->stream, p, qp, B);
}
constexpr int ATTN_TILES_MIN = 1024;             // (row tile, head, sequence) triples from which on a wave takes whole ones: 4096 gain 8 us of 21, 320 lose 1 of 5.  Packed
                                                 // rows: of the padded shape, of which 0.3 .. 0.8 are there; encodes so and dealt to waves, us: 624 of 1024 858, 861;  640 of 1280 515, 513;  2288 of 5120 1391, 1400
void attention(bpd_ctx* ctx, const float* Q, const void* Kc, const void* Vc, void* out, int cap,
               int B, int R, const int* limit, int causal, const int* seq, bool packed, const QProjP* qproj = nullptr, const int* row0 = nullptr) {
  const long kv_seq_stride = (long)cap * ctx->cfg.d_model;
  const int capg = (cap + 31) / 32;
  const bpd_config& c = ctx->cfg;
  const int dh = c.d_model / c.n_heads;
  AttnP p{};
  p.Q = Q; p.Kc = Kc; p.Vc = Vc; p.out = out; p.kv_seq_stride = kv_seq_stride; p.cap = cap; p.capg = capg; p.d = c.d_model; p.R = R;
  p.packed = packed; p.limit = limit; p.causal = causal; p.seq = seq; p.scale = 1.0f / sqrtf((float)dh);
  const bool local = causal && ctx->local_q > 0;
  p.local_q = local ? ctx->local_q : 0; p.local_m = local ? ctx->local_m : 0;
  const int tiles = (R + 15) / 16, wgs = c.n_heads * B * tiles;
  const int nsplit = attention_nsplit(ctx, cap, B, R, causal);
  p.nsplit = nsplit; p.part = ctx->lay.attn_part;
  dim3 grid(c.n_heads, B, tiles * nsplit), cgrid(c.n_heads, B, tiles);
  if (c.dtype == BPD_BF16) {
    if (dh == 64) {
      // a K/V buffer beyond half the last-level cache is streamed past it
      const size_t kv_bytes = (size_t)2 * c.n_dec_layers * B * cap * c.d_model * 2;
      // many workgroups: fetch only the rows in use (the length is read first); few: one round trip, rows past the end too
      // (a split launch walks a long cache, where nearly all fetched rows are in use: measured slower with the extra round trip)
      // (local attention: where the keys start depends on the length, so it is always read first)
      const bool limf = (nsplit == 1 && wgs >= ATTN_LIMF_MIN_WGS) || local;
#define BPD_ATTN(A_, B_, QU_) { if (seq) hipLaunchKernelGGL((attention_mfma_slots_kernel<A_, B_, QU_>), grid, dim3(64 * (QU_ > 0 ? ATTN_WAVES : waves)), 0, ctx->stream, p, qp_); \
                                else hipLaunchKernelGGL((attention_mfma_kernel<A_, B_, QU_>), grid, dim3(64 * (QU_ > 0 ? ATTN_WAVES : waves)), 0, ctx->stream, p, qp_); }
      // up to 128 keys: four waves; more: eight, or four with two groups each where there are many workgroups or where the keys
      // are dealt to several of them (8 x 8 heads, 3072 keys: 97 ms per decode, 110 with one group each)
      const bool few = attention_keys(ctx, cap, R, causal) <= 128, two = !few && (limf || nsplit > 1);
      const int waves = few || two ? 4 : ATTN_WAVES;
      const QProjP qp_ = qproj ? *qproj : QProjP{};
      if (qproj && attention_qproj_pairs(ctx, B)) {
        if (c.d_model == 512) launch_attention_pairs<4>(ctx, p, qp_, B); else launch_attention_pairs<8>(ctx, p, qp_, B);
        return;
      }
      if (qproj) {                               // queries projected in the kernel (attention_qproj_ok() holds)
        switch (c.d_model / 128) {
          case 1: BPD_ATTN(false, false, 1) break;
          case 2: BPD_ATTN(false, false, 2) break;
          case 4: BPD_ATTN(false, false, 4) break;
          default: BPD_ATTN(false, false, 8) break;
        }
        return;
      }
      const bool nt = causal && kv_bytes > ((size_t)128 << 20);
      // the encoder
      p.row0 = row0;                             // (packed: packed_source_rows())
      if (few && !causal && !seq && nsplit == 1 && tiles > 1 && wgs >= ATTN_TILES_MIN) {
        const int per = std::max(1, std::min(tiles, wgs / (8 * ctx->num_cus)));           // (two waves per SIMD)
        const dim3 tgrid(c.n_heads, B, (tiles + 4 * per - 1) / (4 * per));
        if (row0) hipLaunchKernelGGL(attention_mfma_tiles_kernel<true>, tgrid, dim3(256), 0, ctx->stream, p, per);
        else hipLaunchKernelGGL(attention_mfma_tiles_kernel<false>, tgrid, dim3(256), 0, ctx->stream, p, per);
        return;
      }
      if (row0) {
        if (few) hipLaunchKernelGGL(attention_mfma_packed_kernel<0>, grid, dim3(64 * 4), 0, ctx->stream, p, qp_);
        else hipLaunchKernelGGL(attention_mfma_packed_kernel<-1>, grid, dim3(64 * 4), 0, ctx->stream, p, qp_);
        return;
      }
      if (two) {
        if (nt && limf) BPD_ATTN(true, true, -1) else if (nt) BPD_ATTN(true, false, -1) else if (limf) BPD_ATTN(false, true, -1) else BPD_ATTN(false, false, -1)
      } else {
        if (nt && limf) BPD_ATTN(true, true, 0) else if (nt) BPD_ATTN(true, false, 0) else if (limf) BPD_ATTN(false, true, 0) else BPD_ATTN(false, false, 0)
      }
#undef BPD_ATTN
      if (nsplit > 1) launch_combine<bf16_t, 64>(p, cgrid, ctx->stream);
    } else {
      hipLaunchKernelGGL((attention_kernel<bf16_t, 16>), grid, dim3(256), 0, ctx->stream, p);
      if (nsplit > 1) launch_combine<bf16_t, 16>(p, cgrid, ctx->stream);
    }
  } else {
    hipLaunchKernelGGL((attention_kernel<float, 16>), grid, dim3(256), 0, ctx->stream, p);
    if (nsplit > 1) launch_combine<float, 16>(p, cgrid, ctx->stream);
  }
}

void embed(bpd_ctx* ctx, const int* tok, int tok_ld, const int* base, int rows_per_seq, int M, const float* pos,
           float* x, int zero_input, unsigned long long* keys = nullptr, int nkeys = 0, const int* seq = nullptr) {
  const bpd_config& c = ctx->cfg;
  const long n = (long)M * c.d_model;
  dim3 grid((unsigned)((n + 255) / 256));
  const float scale = sqrtf((float)c.d_model);
  if (stats_path(ctx, M) && x == ctx->lay.x) {
    hipLaunchKernelGGL(embed_stats_kernel, dim3(c.d_model / 16), dim3(64), 0, ctx->stream, tok, tok_ld, base, rows_per_seq, M,
                       c.d_model, (const bf16_t*)ctx->lay.emb, c.vocab, pos, scale, x, zero_input, ctx->lay.stats_ln, keys, nkeys, seq);
    return;
  }
  if (c.dtype == BPD_BF16)
    hipLaunchKernelGGL(embed_kernel<true>, grid, dim3(256), 0, ctx->stream, tok, tok_ld, base, rows_per_seq, M, c.d_model,
                       ctx->lay.emb, c.vocab, pos, scale, x, zero_input, keys, nkeys, seq);
  else
    hipLaunchKernelGGL(embed_kernel<false>, grid, dim3(256), 0, ctx->stream, tok, tok_ld, base, rows_per_seq, M, c.d_model,
                       ctx->lay.emb, c.vocab, pos, scale, x, zero_input, keys, nkeys, seq);
}

void fill_i32(bpd_ctx* ctx, int* p, long n, int v) {
  hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, ctx->stream, p, n, v);
}

// ------------------------------------------------------------------------------- decoder stack kernel
// The decoder layers of a block of at most 16 rows as one kernel on one XCD (bpd_stack.h).  Usable when the workgroup
// placement probe of bpd_create found the regular round-robin, the model has a shape the kernel is built for, both
// attentions run unsplit (short caches), and the largest operator's LDS fits.
StackShape stack_shape_of(const bpd_ctx* ctx, int B, int R) {
  const bpd_config& c = ctx->cfg;
  StackShape s;
  s.n_layers = c.n_dec_layers; s.d = c.d_model; s.F = c.d_ff; s.heads = c.n_heads; s.B = B; s.M = B * R;
  s.workers = ctx->stack_workers; s.KU = c.d_model / 128;
  return s;
}
int stack_lds_bytes(const bpd_ctx* ctx, int B, int R) { return stack_lds_need(stack_shape_of(ctx, B, R), (int)AttnLds::BYTES); }
bool stack_usable(const bpd_ctx* ctx, int B, int R) {
  const bpd_config& c = ctx->cfg;
  const int M = B * R;
  return ctx->stack_workers > 0 && !ctx->stack_off && !ctx->replayable && ctx->lay.stack_ex != nullptr && M >= 1 && M <= 16 && ctx->local_q == 0 && ctx->seq == nullptr &&
         attention_nsplit(ctx, c.max_out_len + c.k_max + 1, B, R, 1) == 1 && attention_nsplit(ctx, c.max_src_len, B, R, 0) == 1 &&
         stack_lds_bytes(ctx, B, R) <= 160 * 1024 &&
         (std::max(3 * c.d_model, c.d_ff) / 16 + ctx->stack_workers - 1) / ctx->stack_workers <= 8;     // tiles a helper wave finishes: two
}
template <int KU>
void launch_stack_ku(bpd_ctx* ctx, const StackP& p) {
  auto k = decoder_stack_kernel<KU>;
  static int attr = 0;                            // per instantiation: allow more than 64 KiB of LDS
  if (attr < p.lds_bytes) { (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, p.lds_bytes); attr = p.lds_bytes; }
  hipLaunchKernelGGL(k, dim3(p.nx * p.workers), dim3(512), p.lds_bytes, ctx->stream, p);
}
void launch_stack(bpd_ctx* ctx, int R) {
  const bpd_config& c = ctx->cfg;
  Layout& L = ctx->lay;
  const int d = c.d_model, slots = c.max_out_len + c.k_max + 1;
  StackP p{};
  p.L = (const StackLayerP*)L.stack_layers;
  p.n_layers = c.n_dec_layers; p.d = d; p.F = c.d_ff; p.heads = c.n_heads; p.B = ctx->B; p.R = R; p.M = ctx->B * R;
  p.slots = slots; p.max_src = c.max_src_len;
  p.Lbase = L.L; p.src_len = L.src_len; p.x_in = L.x; p.x_out = L.x; p.stats_out = L.stats_ln;
  p.ex = L.stack_ex; p.flags = L.stack_flags; p.err = L.stack_err;
  if (++ctx->stack_epoch == 0) ctx->stack_epoch = 1;
  p.epoch = ctx->stack_epoch;
  p.spin_limit = 1 << 21;
  p.xcc = ctx->stack_xcc; p.nx = ctx->stack_nx; p.workers = ctx->stack_workers;
  p.eps = c.ln_eps; p.scale = 1.0f / sqrtf(64.f);
  p.lds_bytes = stack_lds_bytes(ctx, ctx->B, R);
  p.trace = getenv("BPD_STACK_TRACE") ? L.stack_trace : nullptr;
  switch (d / 128) {
    case 1: launch_stack_ku<1>(ctx, p); break;
    case 2: launch_stack_ku<2>(ctx, p); break;
    case 4: launch_stack_ku<4>(ctx, p); break;
    case 6: launch_stack_ku<6>(ctx, p); break;
    default: launch_stack_ku<8>(ctx, p); break;
  }
}
// After a synchronisation: has a stack launch reported a wait that ran out?  Then the per-operator kernels take over
// for the rest of the context's life and the caller learns that results since the last check cannot be trusted.
int stack_check(bpd_ctx* ctx) {
  if (ctx->stack_workers == 0 || ctx->stack_off || ctx->stack_epoch == 0) return BPD_OK;
  unsigned e = 0;
  HIPCHK(hipMemcpy(&e, ctx->lay.stack_err, 4, hipMemcpyDeviceToHost));
  if (e == 0) return BPD_OK;
  ctx->stack_off = true;
  HIPCHK(hipMemsetAsync(ctx->lay.stack_err, 0, 4, ctx->stream));
  return fail(ctx, BPD_E_HIP, "decoder stack kernel: a bounded wait ran out (code " + std::to_string(e) +
                              "); the results of this decode are invalid, later steps use the per-operator kernels");
}

// ------------------------------------------------------------------------------- all layers in one kernel (bpd_layers.h)
enum { LAYERS_CHAIN, LAYERS_JOBS, LAYERS_WIDE, LAYERS_TALL };         // kernels one by one, layers_kernel, wide_layers_kernel, tall_layers_kernel
int layers_way(const bpd_ctx* ctx, int slots, int R) {
  const bpd_config& c = ctx->cfg;
  if (!ctx->lay.layers_sync || ctx->layers_group == 0 || ctx->num_cus < LK_JOBS * LK_PLACES) return LAYERS_CHAIN;
  if (layers_shape(c)) return layers_fit(slots, R) ? LAYERS_JOBS : LAYERS_CHAIN;
  const long keys = attention_keys(ctx, c.max_out_len + c.k_max + 1, R, 1);
  if (wide_layers_fit(slots, R, keys, ctx->S)) return LAYERS_WIDE;
  return ctx->lay.layers_slices && tall_layers_fit(slots, R, keys, ctx->S) ? LAYERS_TALL : LAYERS_CHAIN;
}
int layers_split_of(const bpd_ctx* ctx, int slots, int R) {
  const bpd_config& c = ctx->cfg;
  long keys = attention_keys(ctx, c.max_out_len + c.k_max + 1, R, 1);
  if (ctx->local_q > 0) keys = std::min(keys, (long)ctx->local_q + ctx->local_m + R);
  return layers_split(slots, keys);
}
template <bool KVNT>
void launch_layers_kernel(const bpd_ctx* ctx, const LayersP& p) {
  static bool attr_set = false;                 // per instantiation: allow more than 64 KiB of LDS
  if (!attr_set) { (void)hipFuncSetAttribute((const void*)layers_kernel<2048, KVNT>, hipFuncAttributeMaxDynamicSharedMemorySize, LkLds<2048>::BYTES); attr_set = true; }
  hipLaunchKernelGGL((layers_kernel<2048, KVNT>), dim3(LK_JOBS * LK_PLACES), dim3(512), LkLds<2048>::BYTES, ctx->stream, p);
}
template <int MT>
void launch_tall_layers(const bpd_ctx* ctx, const LayersP& p) {
  static bool attr_set = false;
  if (!attr_set) { (void)hipFuncSetAttribute((const void*)tall_layers_kernel<MT>, hipFuncAttributeMaxDynamicSharedMemorySize, TkLds<MT>::BYTES); attr_set = true; }
  hipLaunchKernelGGL(tall_layers_kernel<MT>, dim3(WK_XCDS * LK_PLACES), dim3(512), TkLds<MT>::BYTES, ctx->stream, p);
}
void launch_layers(bpd_ctx* ctx, int R, int way) {
  const bpd_config& c = ctx->cfg;
  Layout& L = ctx->lay;
  const size_t d = c.d_model, slots = (size_t)c.max_out_len + c.k_max + 1;
  const DecL& w = L.dec[0];
  LayersP p{};
  p.wqkv = (const char*)w.wqkv; p.wo = (const char*)w.wo; p.cq = (const char*)w.cq; p.co = (const char*)w.co; p.w1 = (const char*)w.w1; p.w2 = (const char*)w.w2;
  p.ln1 = w.ln1.g; p.ln2 = w.ln2.g; p.ln3 = w.ln3.g; p.b1 = w.b1; p.b2 = w.b2;      // (a bias follows its gain: both are d floats, whole units of ALIGN)
  p.stride = c.n_dec_layers > 1 ? (long)((const char*)L.dec[1].wqkv - (const char*)w.wqkv) : 0;      // (every layer's arrays are laid out alike)
  p.n_layers = c.n_dec_layers; p.R = R; p.slots = ctx->Bs; p.per_job = layers_per_job(ctx->Bs); p.jobs = (ctx->Bs + p.per_job - 1) / p.per_job;
  p.split = layers_split_of(ctx, ctx->Bs, R);
  p.x = L.x; p.q = (bf16_t*)L.q; p.part = L.attn_part; p.attn = (bf16_t*)L.attn; p.ffh = (bf16_t*)L.ffh;
  p.selfK = (bf16_t*)L.selfK; p.selfV = (bf16_t*)L.selfV; p.crossK = (const bf16_t*)L.crossK; p.crossV = (const bf16_t*)L.crossV;
  p.self_layer = (long)c.max_batch * kv_rows(c, slots) * d; p.src_layer = (long)c.max_batch * kv_rows(c, c.max_src_len) * d;
  p.self_groups = (int)((slots + 31) / 32); p.src_groups = (c.max_src_len + 31) / 32;
  p.seq = ctx->seq; p.base = ctx->seq ? L.slot_L : L.L; p.src_len = ctx->seq ? L.slot_src : L.src_len;
  p.eps = c.ln_eps; p.scale = 1.0f / sqrtf(64.f); p.local_q = ctx->local_q; p.local_m = ctx->local_m;
  p.group = way == LAYERS_JOBS ? ctx->layers_group & 63 : ctx->layers_group;
  p.sync = L.layers_sync; p.error = L.stats + 31;
  if (ctx->layers_ran) fill_i32(ctx, (int*)L.layers_sync, LK_WORDS, 0);         // (nobody came between)
  ctx->layers_ran = true; ctx->layers_normed = false;
  if (way == LAYERS_WIDE) {
    p.jobs = p.per_job = p.split = 0;
    p.xn = (bf16_t*)L.layers_xn; p.x1 = L.layers_x1; p.attn = (bf16_t*)L.layers_attn2; p.ffh = (bf16_t*)L.layers_ffh;
    static bool attr_set = false;
    if (!attr_set) { (void)hipFuncSetAttribute((const void*)wide_layers_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, WkLds::BYTES); attr_set = true; }
    hipLaunchKernelGGL(wide_layers_kernel, dim3(WK_XCDS * LK_PLACES), dim3(512), WkLds::BYTES, ctx->stream, p);
    return;
  }
  if (way == LAYERS_TALL) {
    p.jobs = p.per_job = p.split = 0;
    p.xn = (bf16_t*)L.layers_xn; p.x1 = L.layers_x1; p.attn = (bf16_t*)L.layers_attn2; p.ffh = (bf16_t*)L.layers_ffh; p.slices = L.layers_slices; p.part = L.kpart;
    const int tiles = (ctx->Bs * R + 15) / 16;
    if (tiles <= 2) launch_tall_layers<2>(ctx, p);
    else if (tiles == 3) launch_tall_layers<3>(ctx, p);
    else launch_tall_layers<4>(ctx, p);
    ctx->pend_slices = 4; ctx->pend_bias = L.dec[c.n_dec_layers - 1].b2; ctx->pend_x = L.x;
    return;
  }
  p.x1 = L.layers_x1; p.x3 = L.layers_x3; p.attn2 = (bf16_t*)L.layers_attn2;
  // One row tile is normalised by the GEMM behind; more rows here: 1.0 us instead of 4.7 in a kernel of its own (24 and 80 rows)
  if (ctx->Bs * R > 16) { p.lnf = L.dec_lnf.g; p.h = L.h; p.hn = (bf16_t*)L.hn; ctx->layers_normed = true; }
  const bool nt = (size_t)2 * c.n_dec_layers * ctx->Bs * slots * d * 2 > ((size_t)128 << 20);       // (as in attention())
  if (nt) launch_layers_kernel<true>(ctx, p); else launch_layers_kernel<false>(ctx, p);
}

// ------------------------------------------------------------------------------- profiling

hipEvent_t prof_event(bpd_ctx* ctx) {
  if (ctx->prof_used == ctx->prof_ev.size()) {
    hipEvent_t e;
    (void)hipEventCreate(&e);
    ctx->prof_ev.push_back(e);
  }
  return ctx->prof_ev[ctx->prof_used++];
}
struct PhaseTimer {
  bpd_ctx* ctx; bool on;
  PhaseTimer(bpd_ctx* c, int phase) : ctx(c), on(c->prof_phase == phase) {
    if (on) (void)hipEventRecord(prof_event(ctx), ctx->stream);
  }
  ~PhaseTimer() {
    if (on) { (void)hipEventRecord(prof_event(ctx), ctx->stream); ctx->prof_launches++; }
  }
};

// ------------------------------------------------------------------------------- the model invocation

StateP state_params(bpd_ctx* ctx);

// Heads and vocabulary projection of one step in two dependent phases (same tokens as the k x k
// table, fewer rows): p_1 at the k block rows -> verify -> the heads 2..k at row k-hat only, which
// is all the accept and predict substeps read (Section 3: verification uses p_1, the next
// proposals are row k-hat of the table).  2k - 1 rows of the vocabulary projection per sequence
// instead of k^2.  Needs more than 16 block rows (the single-tile path keeps its fused LayerNorm).
int heads_two_phase(bpd_ctx* ctx, int k) {
  const bpd_config& c = ctx->cfg;
  Layout& L = ctx->lay;
  const int B = ctx->Bs, d = c.d_model, F = c.d_ff, M = B * k;
  const size_t as = act_size(c);
  const int* seq = ctx->seq;
  // phase 1: head 1 (the base model's p_1) at every block row
  if (!(ctx->layers_ran && ctx->layers_normed)) layernorm(ctx, L.x, L.dec_lnf, M, L.hn, L.h);
  gemm(ctx, gp(L.hn, d, L.hw1, c.k_max * F, M, F, d), plain(L.hb1, 1, nullptr, 0, nullptr, 0, L.H, F));
  gemm(ctx, gp(L.H, F, L.hw2, d, M, d, F), plain(L.hb2, 0, L.h, d, nullptr, 0, L.O, d));
  unsigned long long* keys2 = L.keys_h1 + M;           // this step's second-phase keys follow its M head-1 keys: one fill clears both
  fill_i32(ctx, (int*)L.keys_h1, 4L * M, 0);
  const bool topn = ctx->top_n > 1;
  vocab_argmax(ctx, gp(L.O, d, L.emb, c.vocab, M, c.vocab, d), L.keys_h1, topn ? L.logits_h1 : nullptr);
  if (topn)
    hipLaunchKernelGGL(topn_rank_kernel, dim3(k - 1, B), dim3(TOPN_T), 0, ctx->stream, (const float*)L.logits_h1, (long)c.vocab, c.vocab,
                       (const int*)L.P, c.k_max, k, ctx->top_n, L.topn_ok, seq);
  StateP st = state_params(ctx);
  st.imposed = ctx->cur_imposed; st.imposed_stride = ctx->cur_imposed_stride;
  hipLaunchKernelGGL(select_row_kernel, dim3(B), dim3(256), 0, ctx->stream, st, (const unsigned long long*)L.keys_h1, k,
                     ctx->cur_imposed_step, (const bf16_t*)L.hn, (const float*)L.h, d, L.sel, (bf16_t*)L.hn2, L.h2, seq);
  // phase 2: heads 2..k at the selected row of each sequence
  const int kh = k - 1;
  const char* w1 = (const char*)L.hw1 + (size_t)F * d * as;          // packed by 16-column tiles: head 2 starts F columns in
  const char* w2 = (const char*)L.hw2 + (size_t)F * d * as;
  gemm(ctx, gp(L.hn2, d, w1, c.k_max * F, B, kh * F, d), plain(L.hb1 + F, 1, nullptr, 0, nullptr, 0, L.H, kh * F));
  {
    GemmP p = gp(L.H, kh * F, w2, d, B, d, F);
    p.x_g = F; p.w_g = (long)F * d;
    Epi e = plain(L.hb2 + d, 0, L.h2, d, nullptr, 0, L.O, kh * d);
    e.bias_g = d; e.r_g = 0; e.ya_g = d;
    gemm(ctx, p, e, kh);
  }
  vocab_argmax(ctx, gp(L.O, d, L.emb, c.vocab, B * kh, c.vocab, d), keys2, nullptr);
  hipLaunchKernelGGL(assemble_keys_kernel, dim3(B), dim3(256), 0, ctx->stream, (const unsigned long long*)L.keys_h1,
                     (const unsigned long long*)keys2, (const int*)L.sel, k, L.keys, seq);
  LAUNCHCHK();
  if (ctx->pend_slices) return fail(ctx, BPD_E_STATE, "split-K slices were left unreduced");
  return BPD_OK;
}

// The folded copies of the decoder's LayerNorm + GEMM pairs follow the loaded weights: bpd_load_weights marks them stale, and
// once every tensor is there calls this.
void refresh_folded_weights(bpd_ctx* ctx) {
  Layout& L = ctx->lay;
  if (ctx->fold_ready || !L.dec[0].f_qkv.W) return;
  const bpd_config& c = ctx->cfg;
  const int d = c.d_model;
  auto fold = [&](const void* W, const FoldW& f, const LnW& w, int N) {
    hipLaunchKernelGGL(fold_layernorm_kernel, dim3(N / 16), dim3(64), 0, ctx->stream, (const bf16_t*)W, (bf16_t*)f.W, w.g, w.b, f.c, f.d, d / 32);
  };
  for (auto& e : L.dec) { fold(e.wqkv, e.f_qkv, e.ln1, 3 * d); fold(e.cq, e.f_cq, e.ln2, d); fold(e.w1, e.f_w1, e.ln3, c.d_ff); }
  ctx->fold_ready = true;
}

// ------------------------------------------------------------------------------- blocks of few rows (bpd_row_gemm.h)
constexpr int LEAN_WHOLE_M = 256;       // more rows: the slices of the LDS-staged kernel for K = 2048, too (256 rows 4.6 against 4.3 us, 320 rows 5.6 against 5.2)
int lean_slices(const bpd_ctx* ctx, int M) {
  const bpd_config& c = ctx->cfg;
  if (c.d_ff > LEAN_K_WHOLE && M <= LEAN_PART_M) return c.d_ff / 1024;
  return c.d_ff > LEAN_K_WHOLE || (c.d_ff == LEAN_K_WHOLE && M > LEAN_WHOLE_M) ? residual_k_slices(ctx, gp(nullptr, c.d_ff, nullptr, c.d_model, M, c.d_model, c.d_ff)) : 1;
}

template <int WAVES, int U, bool LN, int EPI>
void launch_row_gemm(const bpd_ctx* ctx, const RowGemmP& p, int slices) {
  // the smallest tile that needs no more workgroups than there are CUs: a second round of workgroups costs more than the wider tile
  // (no tile gets there: two rows of tiles, many workgroups)
  auto wgs = [&](int mt, int nt) { return (long)((p.ntiles + nt - 1) / nt) * ((p.M + 16 * mt - 1) / (16 * mt)) * slices; };
#define BPD_RG(MT_, NT_) hipLaunchKernelGGL((row_gemm_kernel<WAVES, U, MT_, NT_, LN, EPI>), dim3((p.ntiles + NT_ - 1) / NT_, (p.M + 16 * MT_ - 1) / (16 * MT_), slices), \
                                            dim3(64 * WAVES), 0, ctx->stream, p)
  if (wgs(1, 1) <= ctx->num_cus) BPD_RG(1, 1);
  else if (wgs(1, 2) <= ctx->num_cus) BPD_RG(1, 2);
  else if (LN || U > 4 || wgs(1, 4) <= ctx->num_cus) BPD_RG(1, 4);
  else if constexpr (!LN && U <= 4) {      // (U = 8: K = 2048, at most 256 rows)
    if (wgs(2, 4) <= ctx->num_cus) BPD_RG(2, 4);
    else if (wgs(3, 4) <= ctx->num_cus) BPD_RG(3, 4);
    else if (wgs(4, 4) <= ctx->num_cus) BPD_RG(4, 4);
    else BPD_RG(2, 4);
  }
#undef BPD_RG
}
template <bool LN, int EPI>
void row_gemm(const bpd_ctx* ctx, const RowGemmP& p, int K, int z = 1) {
  switch (K) {
    case 128: launch_row_gemm<4, 1, LN, EPI>(ctx, p, z); break;
    case 256: launch_row_gemm<4, 2, LN, EPI>(ctx, p, z); break;
    case 512: launch_row_gemm<4, 4, LN, EPI>(ctx, p, z); break;
    case 768: launch_row_gemm<8, 3, LN, EPI>(ctx, p, z); break;
    case 1024: launch_row_gemm<8, 4, LN, EPI>(ctx, p, z); break;
    default: if constexpr (EPI == RG_RES) launch_row_gemm<8, 8, LN, EPI>(ctx, p, z); break;      // 2048
  }
}
// Y = relu(LayerNorm(x) W + b), or queries / K / V from LayerNorm(x) W.  xn: room for the normalised rows
template <int EPI>
void lean_ln_gemm(bpd_ctx* ctx, float* x, LnW w, void* xn, RowGemmP p) {
  const int d = ctx->cfg.d_model;
  p.eps = ctx->cfg.ln_eps; p.ldx = d;
  if (ctx->pend_slices == 0 && lean_fuse(d, p.M)) {
    p.X = x; p.g = w.g; p.b = w.b;
    row_gemm<true, EPI>(ctx, p, d);
  } else {
    layernorm(ctx, x, w, p.M, xn, nullptr, true);
    p.X = xn;
    row_gemm<false, EPI>(ctx, p, d);
  }
}
RowGemmP rg(const void* X, int ldx, const void* W, int M, int N) {
  RowGemmP p{};
  p.X = X; p.ldx = ldx; p.W = W; p.M = M; p.ntiles = N / 16;
  return p;
}
RowGemmP rg_kv(const bpd_ctx* ctx, const void* X, const void* W, int M, int N, const Epi& e) {
  RowGemmP p = rg(X, ctx->cfg.d_model, W, M, N);
  p.Y = e.Qf; p.chunk0 = e.chunk0; p.R = e.rows_per_seq; p.heads = ctx->cfg.n_heads; p.capg = e.capg; p.cap = e.cap;
  p.Kc = (bf16_t*)e.Ka; p.Vc = (bf16_t*)e.Va; p.base = e.base; p.seq = e.seq;
  return p;
}
// (X as rows: the LDS-staged kernel's)
bool residual_by_rows(int K, int M) { return K >= LEAN_K_WHOLE && M > (K > LEAN_K_WHOLE ? LEAN_PART_M : LEAN_WHOLE_M); }
// x += X W + bias; K slices of a long K are left for the LayerNorm of x that follows (ctx->pend_*)
void lean_residual(bpd_ctx* ctx, const void* X, int K, const void* W, const float* bias, int M, float* x) {
  const int d = ctx->cfg.d_model;
  RowGemmP p = rg(X, K, W, M, d);
  p.ldy = d; p.bias = bias;
  if (residual_by_rows(K, M)) {
    gemm(ctx, gp(X, K, W, d, M, d, K), plain(bias, 0, x, d, x, d, nullptr, 0));
  } else if (K > LEAN_K_WHOLE) {
    p.Y = ctx->lay.kpart; p.ksteps = K / 32;
    launch_row_gemm<8, 4, false, RG_PART>(ctx, p, K / 1024);
    ctx->pend_slices = K / 1024; ctx->pend_bias = bias ? bias : ctx->lay.zeros; ctx->pend_x = x;
  } else {
    p.Y = x;
    row_gemm<false, RG_RES>(ctx, p, K);
  }
}
void lean_ffn(bpd_ctx* ctx, float* x, LnW ln, void* xn, const void* w1, const float* b1, void* hidden, const void* w2, const float* b2, int M) {
  const int F = ctx->cfg.d_ff;
  RowGemmP p = rg(nullptr, 0, w1, M, F);
  p.bias = b1; p.Y = hidden; p.ldy = F; p.packed = !residual_by_rows(F, M);
  lean_ln_gemm<RG_RELU>(ctx, x, ln, xn, p);
  lean_residual(ctx, hidden, F, w2, b2, M, x);
}

// One invocation of the combined model on R new rows per sequence (R = 1 for the first call
// on the empty prefix, R = k afterwards) with the first k heads; fills keys[B*R*k].
int forward(bpd_ctx* ctx, int R, int k, int zero_input, float* logits) {
  const bpd_config& c = ctx->cfg;
  Layout& L = ctx->lay;
  const int B = ctx->Bs, d = c.d_model, F = c.d_ff, M = B * R;
  const int slots = c.max_out_len + c.k_max + 1;
  const size_t as = act_size(c);
  const long nk = (long)M * k;
  const bool lean = lean_ok(c, M), sp = stats_path(ctx, M);
  const size_t self_layer = (size_t)c.max_batch * kv_rows(c, slots) * d * as, src_layer = (size_t)c.max_batch * kv_rows(c, c.max_src_len) * d * as;
  const int* seq = ctx->seq;
  const int *base = seq ? L.slot_L : L.L, *srcs = seq ? L.slot_src : L.src_len;
  // residual update x += ...; on the statistics path the kernel also leaves LayerNorm partial sums
  // with more rows the LDS-staged kernel leaves them per tile in L.stats_big for the LayerNorm-fused GEMM that follows
  // (up to 128 rows: with more, every column block repeating the normalisation of its rows costs more than the kernel saved)
  const bool bigs = !sp && !lean && c.dtype == BPD_BF16 && M > 16 && M <= LDSX_LN_M_MAX && d % 64 == 0 && d <= 1024;
  // more than 128 rows: the GEMMs that update x also leave its bf16 copy in L.xn, and the LayerNorm + GEMM that follows
  // runs as one GEMM on folded weights (unless that update is split over K: its slices are summed by a LayerNorm kernel)
  const bool folds = !sp && !bigs && c.dtype == BPD_BF16 && M > LDSX_LN_M_MAX && L.dec[0].f_qkv.W != nullptr;
  auto residual = [&](const float* bias, int K) {
    Epi e = plain(bias, 0, L.x, d, L.x, d, nullptr, 0);
    if (sp) e.stats_out = L.stats_ln;
    else if (bigs) e.stats_out = L.stats_big;
    else if (folds && residual_k_slices(ctx, gp(nullptr, K, nullptr, d, M, d, K)) == 1) { e.stats_out = L.stats_big; e.Ya = L.xn; e.ldya = d; }
    return e;
  };
  bool xs = false;      // L.stats_big describes the current L.x
  {
    PhaseTimer t(ctx, BPD_PHASE_LAYERS);
    // (the previous step's accept kernel may already have embedded this block, with its statistics (and, beyond 16 rows,
    // its bf16 copy in L.xn), and cleared the keys)
    const bool have_x = embed_in_accept(ctx) && !zero_input && R == k && ctx->x_ready_k == k && ctx->x_ready_slots == B && !(logits && slots_used(ctx));
    ctx->x_ready_k = 0;
    xs = have_x && !sp;
    if (!have_x) embed(ctx, L.P, c.k_max, base, R, M, L.pos_tgt, L.x, zero_input, L.keys, (int)nk, seq);
    const bool stack = M <= 16 && (lean || sp) && stack_usable(ctx, B, R);
    const int way = stack || !lean ? LAYERS_CHAIN : layers_way(ctx, B, R);
    const bool one = way != LAYERS_CHAIN;
    if (stack) launch_stack(ctx, R);
    else if (one) launch_layers(ctx, R, way);
    for (int l = 0; l < (stack || one ? 0 : c.n_dec_layers); ++l) {
      DecL& w = L.dec[l];
      char* Kl = (char*)L.selfK + self_layer * l;
      char* Vl = (char*)L.selfV + self_layer * l;
      char* cK = (char*)L.crossK + src_layer * l;
      char* cV = (char*)L.crossV + src_layer * l;
      const Epi kv = kv_split(ctx, L.q, Kl, Vl, 0, R, slots, base, seq);
      const bool qproj = attention_qproj_ok(ctx, B, R);
      if (lean) {
        if (zero_input && R == 1) {              // on the empty prefix: a row sees one key, its own, and its attention is that key's value
          RowGemmP q = rg_kv(ctx, nullptr, (const char*)w.wqkv + (size_t)d * d * as, M, 2 * d, kv);
          q.chunk0 = 1; q.vout = (bf16_t*)L.attn;
          lean_ln_gemm<RG_QKV>(ctx, L.x, w.ln1, L.xn, q);
        } else {
          lean_ln_gemm<RG_QKV>(ctx, L.x, w.ln1, L.xn, rg_kv(ctx, nullptr, w.wqkv, M, 3 * d, kv));
          attention(ctx, L.q, Kl, Vl, L.attn, slots, B, R, base, 1, seq, lean);
        }
        lean_residual(ctx, L.attn, d, w.wo, nullptr, M, L.x);
        if (qproj) {
          const QProjP qp{L.x, w.ln2.g, w.ln2.b, w.cq, c.ln_eps};
          attention(ctx, nullptr, cK, cV, L.attn, c.max_src_len, B, R, srcs, 0, seq, lean, &qp);
        } else {
          lean_ln_gemm<RG_QKV>(ctx, L.x, w.ln2, L.xn, rg_kv(ctx, nullptr, w.cq, M, d, kv));
          attention(ctx, L.q, cK, cV, L.attn, c.max_src_len, B, R, srcs, 0, seq, lean);
        }
        lean_residual(ctx, L.attn, d, w.co, nullptr, M, L.x);
        lean_ffn(ctx, L.x, w.ln3, L.xn, w.w1, w.b1, L.ffh, w.w2, w.b2, M);
        continue;
      }
      // self-attention sublayer: K/V of the block rows go straight into the cache at L_b + i'
      gemm_ln(ctx, L.x, w.ln1, L.xn, nullptr, gp(L.xn, d, w.wqkv, 3 * d, M, 3 * d, d), kv, sp, xs, folds ? &w.f_qkv : nullptr);
      attention(ctx, L.q, Kl, Vl, L.attn, slots, B, R, base, 1, seq, lean);
      xs = gemm(ctx, gp(L.attn, d, w.wo, d, M, d, d), residual(nullptr, d));
      // cross-attention sublayer over the encoder memory
      if (qproj) {
        const QProjP qp{L.x, w.ln2.g, w.ln2.b, w.cq, c.ln_eps};
        attention(ctx, nullptr, cK, cV, L.attn, c.max_src_len, B, R, srcs, 0, seq, lean, &qp);
      } else {
        gemm_ln(ctx, L.x, w.ln2, L.xn, nullptr, gp(L.xn, d, w.cq, d, M, d, d), plain(nullptr, 0, nullptr, 0, L.q, d, nullptr, 0), sp, xs, folds ? &w.f_cq : nullptr);
        attention(ctx, L.q, cK, cV, L.attn, c.max_src_len, B, R, srcs, 0, seq, lean);
      }
      xs = gemm(ctx, gp(L.attn, d, w.co, d, M, d, d), residual(nullptr, d));
      // feed-forward sublayer
      gemm_ln(ctx, L.x, w.ln3, L.xn, nullptr, gp(L.xn, d, w.w1, F, M, F, d), plain(w.b1, 1, nullptr, 0, nullptr, 0, L.ffh, F), sp, xs, folds ? &w.f_w1 : nullptr);
      xs = gemm(ctx, gp(L.ffh, F, w.w2, d, M, d, F), residual(w.b2, F));
    }
  }
  { PhaseTimer t(ctx, BPD_PHASE_EMPTY); }       // calibration of the event bracketing itself
  if (ctx->two_phase && R == k && k > 1 && M > 16 && !logits && c.dtype == BPD_BF16) return heads_two_phase(ctx, k);
  // the k residual FFN heads: final LayerNorm + hidden layers side by side (h kept in fp32
  // for the residual), then one output layer per head
  {
    PhaseTimer t(ctx, BPD_PHASE_HEAD_HIDDEN);
    // behind the layers kernels one row tile is normalised by the GEMM that reads it
    if (ctx->layers_ran && ctx->layers_normed) {
      gemm(ctx, gp(L.hn, d, L.hw1, c.k_max * F, M, k * F, d), plain(L.hb1, 1, nullptr, 0, nullptr, 0, L.H, k * F));
    } else if (ctx->layers_ran && M <= 16 && !ctx->pend_slices) {
      GemmP p = gp(nullptr, d, L.hw1, c.k_max * F, M, k * F, d);
      LnP ln{L.x, L.dec_lnf.g, L.dec_lnf.b, nullptr, c.ln_eps, L.h};
      ln.clear = clear_behind_layers(ctx, ln.nclear);
      const Epi e = plain(L.hb1, 1, nullptr, 0, nullptr, 0, L.H, k * F);
      if (p.N / 16 >= 2048) launch_skinny<2, 2, false>(ctx, p, e, ln, nullptr, nullptr, 1);
      else launch_skinny<1, 2, false>(ctx, p, e, ln, nullptr, nullptr, 1);
    } else if (lean) {
      layernorm(ctx, L.x, L.dec_lnf, M, L.hn, L.h);
      gemm(ctx, gp(L.hn, d, L.hw1, c.k_max * F, M, k * F, d), plain(L.hb1, 1, nullptr, 0, nullptr, 0, L.H, k * F));
    } else gemm_ln(ctx, L.x, L.dec_lnf, L.hn, L.h, gp(L.hn, d, L.hw1, c.k_max * F, M, k * F, d),
            plain(L.hb1, 1, nullptr, 0, nullptr, 0, L.H, k * F), sp);
  }
  {
    PhaseTimer t(ctx, BPD_PHASE_HEAD_OUT);
    GemmP p = gp(L.H, k * F, L.hw2, d, M, d, F);
    p.x_g = F; p.w_g = (long)F * d;
    Epi e = plain(L.hb2, 0, L.h, d, nullptr, 0, L.O, k * d);
    e.bias_g = d; e.r_g = 0; e.ya_g = d;
    if (sp) {          // h = LayerNorm(x) is recomputed from x and the partial statistics
      e.R = L.x; e.lnR_stats = L.stats_ln; e.lnR_g = L.dec_lnf.g; e.lnR_b = L.dec_lnf.b; e.lnR_K = d; e.lnR_eps = c.ln_eps;
    }
    gemm(ctx, p, e, k);
  }
  {
    PhaseTimer t(ctx, BPD_PHASE_VOCAB);
    // top-n acceptance: the scores of head 1 (every k-th row of O) are kept, for the rank of each proposal among them (a second pass
    // over the vocabulary for those rows alone, as before, was 13 us of a step of 13 slots, k = 6, over 32 000 tokens at d = 512)
    const bool rank = ctx->top_n > 1 && R == k && k > 1;
    float* const kept = logits ? logits : (rank ? L.logits_h1 : nullptr);
    const int lstep = logits ? 1 : k;
    if (c.dtype == BPD_BF16) {
      GemmP p = gp(L.O, d, L.emb, c.vocab, (int)nk, c.vocab, d);
      p.lstep = lstep;
      vocab_argmax(ctx, p, L.keys, kept);
    } else {
      hipLaunchKernelGGL(vocab_argmax_f32_kernel, dim3((unsigned)nk), dim3(256), 0, ctx->stream, (const float*)L.O, d,
                         (const float*)L.emb, (int)nk, c.vocab, d, L.keys, kept, lstep);
    }
    if (rank)
      hipLaunchKernelGGL(topn_rank_kernel, dim3(k - 1, B), dim3(TOPN_T), 0, ctx->stream, (const float*)kept,
                         (long)(logits ? k : 1) * c.vocab, c.vocab, (const int*)L.P, c.k_max, k, ctx->top_n, L.topn_ok, seq);
  }
  LAUNCHCHK();
  if (ctx->pend_slices) return fail(ctx, BPD_E_STATE, "split-K slices were left unreduced");
  return BPD_OK;
}

StateP state_params(bpd_ctx* ctx) {
  Layout& L = ctx->lay;
  StateP s{};
  s.L = L.L; s.j = L.j; s.finished = L.finished; s.max_len = L.max_len; s.P = L.P; s.A = L.A;
  s.accepted = L.accepted; s.out_ids = L.out_ids; s.stats = L.stats; s.imposed = nullptr; s.imposed_stride = 0;
  s.kmax = ctx->cfg.k_max; s.max_out = ctx->cfg.max_out_len;
  s.eos_id = ctx->cfg.eos_id; s.distance_eps = ctx->distance_eps; s.min_block = ctx->min_block;
  s.topn_ok = ctx->top_n > 1 ? ctx->lay.topn_ok : nullptr;
  s.dyn = nullptr; s.tick = L.tick; s.imp_next = L.imp_next; s.steps_done = L.steps_done; s.fin_step = L.fin_step; s.slot_seq = L.slot_seq; s.slot_L = L.slot_L; s.slot_src = L.slot_src; s.slot_row = L.slot_row; s.cache_rows = ctx->cfg.max_out_len + ctx->cfg.k_max + 1; s.n_live = L.n_live; s.src_len = L.src_len;
  return s;
}

// ------------------------------------------------------------------------------- small fp32 models (bpd_small.h)
constexpr size_t SMALL_LDS_MAX = 160 * 1024;
SmallLds small_decode_lds(const bpd_config& c, int rows, int k, int hgroup, bool topn) {
  return small_lds(c.d_model, c.d_ff, c.vocab, rows, k, hgroup, 0, topn, small_decoder_phases(c.d_model, c.n_dec_layers, k, hgroup));
}
// Heads whose hidden layers fit the LDS together; 0: not even one does, or steps over caches between as many rows as the host knows
// there may be and `more` others are faster launch by launch (about the mean of those lengths)
int small_hgroup(const bpd_ctx* ctx, int k, long more) {
  const bpd_config& c = ctx->cfg;
  if (!small_shape(c)) return 0;
  const long cap = c.max_out_len + c.k_max + 1, from = std::min(cap, (long)ctx->steps * c.k_max + 1 + k);
  long keys = (from + std::min(cap, from + more)) / 2;
  if (ctx->local_q > 0) keys = std::min(keys, (long)ctx->local_q + ctx->local_m + k);
  if (!small_step_pays(c, k, keys, ctx->S)) return 0;
  int h = k;
  while (h > 0 && (size_t)small_decode_lds(c, k, k, h, ctx->top_n > 1 && k > 1).total * 4 > SMALL_LDS_MAX) --h;
  return h;
}
SmallLds small_encode_lds(const bpd_config& c, int S) {
  return small_lds(c.d_model, c.d_ff, c.vocab, 16, 1, 1, (S + 15) / 16 * 16, false, small_encoder_phases(c.d_model, c.n_enc_layers, c.n_dec_layers));
}
SmallLds small_prime_lds(const bpd_config& c) { return small_lds(c.d_model, c.d_ff, c.vocab, 4, 4, c.k_max, 0, false, small_decoder_phases(c.d_model, c.n_dec_layers, c.k_max, c.k_max)); }
bool small_encode_ok(const bpd_ctx* ctx) {
  return small_shape(ctx->cfg) && ctx->prof_phase == 0 && small_encode_pays(ctx->cfg, ctx->S) && (size_t)small_encode_lds(ctx->cfg, ctx->S).total * 4 <= SMALL_LDS_MAX &&
         (size_t)small_prime_lds(ctx->cfg).total * 4 <= SMALL_LDS_MAX;
}
SmallP small_params(bpd_ctx* ctx) {
  const bpd_config& c = ctx->cfg;
  Layout& L = ctx->lay;
  SmallP p{};
  p.s = state_params(ctx);
  p.d = c.d_model; p.F = c.d_ff; p.V = c.vocab; p.heads = c.n_heads; p.n_enc = c.n_enc_layers; p.n_dec = c.n_dec_layers; p.max_src = c.max_src_len;
  p.slots = c.max_out_len + c.k_max + 1; p.S = ctx->S;
  p.eps = c.ln_eps; p.escale = sqrtf((float)c.d_model); p.qscale = 1.0f / sqrtf((float)(c.d_model / c.n_heads));
  p.local_q = ctx->local_q; p.local_m = ctx->local_m;
  const EncL& e = L.enc[0];
  const DecL& w = L.dec[0];
  p.enc.wqkv = (const float*)e.wqkv; p.enc.wo = (const float*)e.wo; p.enc.w1 = (const float*)e.w1; p.enc.w2 = (const float*)e.w2; p.enc.b1 = e.b1; p.enc.b2 = e.b2;
  p.enc.ln1g = e.ln1.g; p.enc.ln1b = e.ln1.b; p.enc.ln2g = e.ln2.g; p.enc.ln2b = e.ln2.b;
  p.enc.cq = p.enc.co = p.enc.ckv = p.enc.ln3g = p.enc.ln3b = p.enc.wqkv;                    // (not used by the encoder)
  p.dec.wqkv = (const float*)w.wqkv; p.dec.wo = (const float*)w.wo; p.dec.cq = (const float*)w.cq; p.dec.co = (const float*)w.co; p.dec.ckv = (const float*)w.ckv;
  p.dec.w1 = (const float*)w.w1; p.dec.w2 = (const float*)w.w2; p.dec.b1 = w.b1; p.dec.b2 = w.b2;
  p.dec.ln1g = w.ln1.g; p.dec.ln1b = w.ln1.b; p.dec.ln2g = w.ln2.g; p.dec.ln2b = w.ln2.b; p.dec.ln3g = w.ln3.g; p.dec.ln3b = w.ln3.b;
  // (build_layout takes every layer's arrays in the same order)
  p.enc_stride = c.n_enc_layers > 1 ? (const float*)L.enc[1].wqkv - (const float*)e.wqkv : 0;
  p.dec_stride = c.n_dec_layers > 1 ? (const float*)L.dec[1].wqkv - (const float*)w.wqkv : 0;
  p.enc_g = L.enc_lnf.g; p.enc_b = L.enc_lnf.b; p.dec_g = L.dec_lnf.g; p.dec_b = L.dec_lnf.b;
  p.hw1 = (const float*)L.hw1; p.hb1 = L.hb1; p.hw2 = (const float*)L.hw2; p.hb2 = L.hb2; p.emb = (const float*)L.emb; p.emb_t = L.emb_t; p.pos_src = L.pos_src; p.pos_tgt = L.pos_tgt;
  p.selfK = (float*)L.selfK; p.selfV = (float*)L.selfV; p.crossK = (float*)L.crossK; p.crossV = (float*)L.crossV; p.qe = L.qe; p.ke = (float*)L.ke; p.ve = (float*)L.ve;
  p.self_layer = (long)c.max_batch * p.slots * c.d_model; p.src_layer = (long)c.max_batch * c.max_src_len * c.d_model;
  p.src_ids = L.src_ids;
  return p;
}
template <void (*kernel)(SmallP)>
void small_launch(bpd_ctx* ctx, const SmallP& p, const SmallLds& n) {
  const int lds = n.total * 4;
  static bool attr = false;                       // per kernel: allow more than 64 KiB of LDS
  if (!attr) { (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)SMALL_LDS_MAX); attr = true; }
  hipLaunchKernelGGL(kernel, dim3(ctx->B), dim3(SMALL_T), lds, ctx->stream, p);
}
void small_encode(bpd_ctx* ctx) {
  SmallP p = small_params(ctx);
  p.k = p.hgroup = ctx->cfg.k_max;
  small_launch<small_encode_kernel>(ctx, p, small_encode_lds(ctx->cfg, ctx->S));
  small_launch<small_prime_kernel>(ctx, p, small_prime_lds(ctx->cfg));
}
// `steps` steps of every sequence (hgroup: of small_hgroup()), or with logits one invocation's scores
void small_decode(bpd_ctx* ctx, int k, int hgroup, int steps, const int* imposed, int imposed_stride, int* accepted, float* logits) {
  SmallP p = small_params(ctx);
  p.s.imposed = imposed; p.s.imposed_stride = imposed_stride;
  p.k = k; p.hgroup = hgroup; p.steps = steps; p.top_n = ctx->top_n; p.accepted_out = accepted; p.logits = logits;
  const SmallLds n = small_decode_lds(ctx->cfg, k, k, hgroup, p.top_n > 1 && k > 1);
  ctx->x_ready_k = 0;
  if (k <= 4) small_launch<small_decode_kernel<1>>(ctx, p, n);
  else if (k <= 8) small_launch<small_decode_kernel<2>>(ctx, p, n);
  else small_launch<small_decode_kernel<4>>(ctx, p, n);
}

// rows: of packed sources (packed_source_rows()), 0: B x S
int encoder(bpd_ctx* ctx, int rows) {
  const bpd_config& c = ctx->cfg;
  Layout& L = ctx->lay;
  const int B = ctx->B, S = ctx->S, d = c.d_model, F = c.d_ff, M = rows ? rows : B * S;
  const size_t as = act_size(c);
  // packed rows are slots of one row each, at their positions
  const int R = rows ? 1 : S;
  const int *pos = rows ? L.src_pos : nullptr, *seq = rows ? L.src_seq : nullptr, *row0 = rows ? L.src_row0 : nullptr;
  if (rows) embed(ctx, L.src_packed, 1, pos, 1, M, L.pos_src, L.xe, 0);
  else embed(ctx, L.src_ids, S, nullptr, S, M, L.pos_src, L.xe, 0);
  // 17 .. 128 source rows of a width that bpd_row_gemm.h is not built for: the residual GEMMs leave LayerNorm statistics for the LayerNorm-fused GEMM that follows
  const bool lean = lean_encoder_ok(c, M), bigs = !lean && c.dtype == BPD_BF16 && M > 16 && M <= LDSX_LN_M_MAX && d % 64 == 0 && d <= 1024;
  auto residual = [&](const float* bias) {
    Epi e = plain(bias, 0, L.xe, d, L.xe, d, nullptr, 0);
    if (bigs) e.stats_out = L.stats_big;
    return e;
  };
  bool xs = false;      // L.stats_big describes the current L.xe
  for (int l = 0; l < c.n_enc_layers; ++l) {
    EncL& w = L.enc[l];
    const Epi kv = kv_split(ctx, L.qe, L.ke, L.ve, 0, R, S, pos, seq);
    if (lean) {
      lean_ln_gemm<RG_QKV>(ctx, L.xe, w.ln1, L.xen, rg_kv(ctx, nullptr, w.wqkv, M, 3 * d, kv));
      attention(ctx, L.qe, L.ke, L.ve, L.attne, S, B, S, L.src_len, 0, nullptr, lean, nullptr, row0);
      lean_residual(ctx, L.attne, d, w.wo, nullptr, M, L.xe);
      lean_ffn(ctx, L.xe, w.ln2, L.xen, w.w1, w.b1, L.ffhe, w.w2, w.b2, M);
      continue;
    }
    gemm_ln(ctx, L.xe, w.ln1, L.xen, nullptr, gp(L.xen, d, w.wqkv, 3 * d, M, 3 * d, d), kv, false, xs);
    attention(ctx, L.qe, L.ke, L.ve, L.attne, S, B, S, L.src_len, 0, nullptr, lean, nullptr, row0);
    xs = gemm(ctx, gp(L.attne, d, w.wo, d, M, d, d), residual(nullptr));
    gemm_ln(ctx, L.xe, w.ln2, L.xen, nullptr, gp(L.xen, d, w.w1, F, M, F, d), plain(w.b1, 1, nullptr, 0, nullptr, 0, L.ffhe, F), false, xs);
    xs = gemm(ctx, gp(L.ffhe, F, w.w2, d, M, d, F), residual(w.b2));
  }
  layernorm(ctx, L.xe, L.enc_lnf, M, L.mem, nullptr, lean);
  // cross keys and values of all decoder layers in one launch (fp32 and shapes without a tiled kernel: one each)
  const size_t src_layer = (size_t)c.max_batch * kv_rows(c, c.max_src_len) * d;
  const long wz = c.n_dec_layers > 1 ? ((const char*)L.dec[1].ckv - (const char*)L.dec[0].ckv) / (long)as : 0;      // (every layer's arrays are laid out alike)
  const bool together = lean || (c.dtype == BPD_BF16 && d % 64 == 0 && M > 16);
  for (int l = 0; l < (together ? 1 : c.n_dec_layers); ++l) {
    Epi kv = kv_split(ctx, nullptr, (char*)L.crossK + src_layer * l * as, (char*)L.crossV + src_layer * l * as, 1, R, c.max_src_len, pos, seq);
    if (lean) {
      RowGemmP p = rg_kv(ctx, L.mem, L.dec[l].ckv, M, 2 * d, kv);
      p.wz = wz; p.kvz = (long)src_layer;
      row_gemm<false, RG_QKV>(ctx, p, d, c.n_dec_layers);
    } else {
      GemmP p = gp(L.mem, d, L.dec[l].ckv, 2 * d, M, 2 * d, d);
      if (together) { p.w_g = wz; kv.kv_g = (long)src_layer; }
      gemm(ctx, p, kv, together ? c.n_dec_layers : 1);
    }
  }
  LAUNCHCHK();
  return BPD_OK;
}

bool is_host_ptr(const void* p) {
  hipPointerAttribute_t a;
  if (hipPointerGetAttributes(&a, p) != hipSuccess) { (void)hipGetLastError(); return true; }
  return a.type != hipMemoryTypeDevice && a.type != hipMemoryTypeManaged;
}

// Is the caller recording the context's stream into a graph of its own?
bool capturing(const bpd_ctx* ctx) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(ctx->stream, &cap) != hipSuccess) { (void)hipGetLastError(); return false; }
  return cap != hipStreamCaptureStatusNone;
}

// Start of every call that reads or changes the decode: once a call has been captured, its replays may have encoded or stepped
// unseen since the last call, so nothing is left of what the host knew of the decode: tokens to come, sequences in use, the block
// embedded ahead of time, the bound on the cache lengths.  (The decoder stack kernel counts its launches on the host: not used.)
void forget_replayed(bpd_ctx* ctx) {
  if (!ctx->replayable) ctx->replayable = capturing(ctx);
  if (!ctx->replayable) return;
  std::fill(ctx->remaining.begin(), ctx->remaining.end(), -1);
  ctx->live1 = ctx->live2 = -1;
  ctx->budget_min = 0;
  ctx->x_ready_k = 0;
  ctx->steps = std::max<int64_t>(ctx->steps, ctx->cfg.max_out_len);
}

// Graphs given up by run_planned are destroyed once the stream has been waited for past their last launch (run_planned waits for it
// itself when PLANS_MAX of them have come together: encodes that nobody waits for).
void release_retired(bpd_ctx* ctx) {
  for (auto g : ctx->retired) (void)hipGraphExecDestroy(g);
  ctx->retired.clear();
}

// Launches of one kind (an encode, a decode's step) that come again and again with the same arguments are recorded and replayed as
// a graph, since a launch costs the host 3 us: a step of the base model has 43, an encode some 90.  `enqueue` launches on
// ctx->stream and may only depend on the key.  Of each kind the last PLANS_MAX keys are kept, and a key is recorded when it comes
// for the PLAN_SIGHTS'th time while it is among them.  Recording costs 0.2 .. 0.6 ms.
//   Steps (keys: batch sizes and cache lengths) at the second sight.  Without: base model, one sentence 4.09 instead of 3.83 ms, big
//   model, greedy 8.11 instead of 7.13, eight images 102.4 instead of 96.5.
//   Encodes (keys: batch sizes, source lengths, packed rows) at the eighth.  The GPU is no sooner done with a recorded one (base model, one
//   sentence of 64 tokens: 282 us launch by launch, 289), but the host is (50 instead of 220 us), which steps that go out launch by launch then
//   have as a lead (five sentences in steps of the big model 5.58 instead of 5.93 ms, thirteen of the base model 3.62 instead of
//   3.87).  At the second sight source lengths as they come cost more than that: 100 lengths in turn are recorded, given up and
//   recorded again (base model 318 -> 368 us per sentence, big 448 -> 521); eight sights among the last 24 keys are what lengths
//   that do recur have.
constexpr size_t PLANS_MAX = 24;
enum { PLAN_ENCODE, PLAN_STEP };
constexpr int PLAN_SIGHTS[2] = {8, 2};
template <class F>
int run_planned(bpd_ctx* ctx, int kind, const PlanKey& key, F enqueue) {
  // (not while phases are timed, nor inside a graph of the caller's, nor with the decoder stack kernel, whose flags count its launches)
  if (ctx->prof_phase != 0 || (ctx->stack_workers > 0 && !ctx->stack_off) || capturing(ctx)) return enqueue();
  static std::atomic<unsigned long long> clock{0};
  auto& plans = ctx->plans[kind];
  Plan* p = nullptr;
  for (auto& q : plans)
    if (q.key == key) { p = &q; break; }
  if (!p) {
    if (plans.size() >= PLANS_MAX) {             // the one not used for longest goes
      auto old = std::min_element(plans.begin(), plans.end(), [](const Plan& a, const Plan& b) { return a.used < b.used; });
      if (old->exec) ctx->retired.push_back(old->exec);
      plans.erase(old);
      if (ctx->retired.size() >= PLANS_MAX) { HIPCHK(hipStreamSynchronize(ctx->stream)); release_retired(ctx); }
    }
    plans.push_back(Plan{key, 0, false, nullptr, 0});
    p = &plans.back();
  }
  p->used = ++clock;
  if (p->exec) {
    HIPCHK(hipGraphLaunch(p->exec, ctx->stream));
    return BPD_OK;
  }
  if (p->failed || ++p->seen < PLAN_SIGHTS[kind]) return enqueue();
  if (!ctx->plan_stream && hipStreamCreateWithFlags(&ctx->plan_stream, hipStreamNonBlocking) != hipSuccess) ctx->plan_stream = nullptr;
  hipGraph_t graph = nullptr;
  bool ok = ctx->plan_stream && hipStreamBeginCapture(ctx->plan_stream, hipStreamCaptureModeThreadLocal) == hipSuccess;
  if (ok) {
    const hipStream_t user = ctx->stream;
    ctx->stream = ctx->plan_stream;
    const int rc = enqueue();
    ctx->stream = user;
    ok = hipStreamEndCapture(ctx->plan_stream, &graph) == hipSuccess && rc == BPD_OK && graph;
  }
  ok = ok && hipGraphInstantiate(&p->exec, graph, nullptr, nullptr, 0) == hipSuccess;
  if (graph) (void)hipGraphDestroy(graph);
  if (!ok) {                                     // (nothing has run: launch by launch, from now on)
    (void)hipGetLastError();
    p->exec = nullptr; p->failed = true;
    return enqueue();
  }
  HIPCHK(hipGraphLaunch(p->exec, ctx->stream));
  return BPD_OK;
}

unsigned long long* report_of(bpd_ctx* ctx, unsigned tag) { return ctx->report + (size_t)(tag & 1) * ctx->cfg.max_batch; }

// Waits (on the CPU, which polls) until a kernel of the context's stream has stored what `there` looks for in pinned memory.
// Ends also when the stream has nothing left to run: then it is there, or the launch failed.
template <class There>
int wait_until(bpd_ctx* ctx, There there) {
  for (unsigned spin = 1; !there(); ++spin) {
    __builtin_ia32_pause();
    if (spin % 8192) continue;
    const hipError_t e = hipStreamQuery(ctx->stream);
    if (e == hipErrorNotReady) continue;
    if (e != hipSuccess) return fail(ctx, BPD_E_HIP, std::string("waiting for the stream: ") + hipGetErrorString(e));
    if (!there()) return fail(ctx, BPD_E_HIP, "waiting for the stream: it ended without the awaited result");
  }
  return BPD_OK;
}
// ... a counter that only grows, or the report of a step (its tag in the upper half)
int wait_done(bpd_ctx* ctx, const unsigned long long* word, unsigned long long tag) {
  return wait_until(ctx, [&] { return __atomic_load_n(word, __ATOMIC_ACQUIRE) >= tag; });
}
int wait_report(bpd_ctx* ctx, const unsigned long long* word, unsigned tag) {
  return wait_until(ctx, [&] { return __atomic_load_n(word, __ATOMIC_ACQUIRE) >> 32 == tag; });
}

// Copies up to five arrays of ints to the caller (host or device memory; null: not wanted) and waits for them.
struct Fetch { const int* src; size_t n; void* dst; };
constexpr size_t FETCH_KERNEL_MAX = 32768;     // ints: one workgroup's copy, about 10 us; more goes through copies
int fetch(bpd_ctx* ctx, std::initializer_list<Fetch> list) {
  FetchP f{};
  size_t total = 0;
  int na = 0;
  bool direct = true;
  for (const Fetch& a : list) {
    if (!a.dst || !a.n) continue;
    f.src[na] = a.src; f.n[na] = (int)a.n; ++na;
    total += a.n;
    direct = direct && is_host_ptr(a.dst);
  }
  if (direct && total && total <= FETCH_KERNEL_MAX && total <= ctx->n_stage_out) {
    f.dst = ctx->stage_out; f.done = &ctx->done[0]; f.tag = ++ctx->fetch_tag;
    hipLaunchKernelGGL(fetch_kernel, dim3(1), dim3(1024), 0, ctx->stream, f);
    LAUNCHCHK();
    const int rc = wait_done(ctx, &ctx->done[0], f.tag);
    if (rc) return rc;
    release_retired(ctx);
    const int* from = ctx->stage_out;
    for (const Fetch& a : list)
      if (a.dst && a.n) { memcpy(a.dst, from, a.n * 4); from += a.n; }
    return BPD_OK;
  }
  for (const Fetch& a : list)
    if (a.dst && a.n) HIPCHK(hipMemcpyAsync(a.dst, a.src, a.n * 4, hipMemcpyDefault, ctx->stream));
  HIPCHK(hipStreamSynchronize(ctx->stream));
  release_retired(ctx);
  return BPD_OK;
}

}  // namespace

// ------------------------------------------------------------------------------- C ABI

extern "C" {

size_t bpd_workspace_bytes(const bpd_config* cfg) {
  if (!cfg || !config_ok(*cfg)) return 0;
  Layout L;
  return build_layout(*cfg, nullptr, L);
}

int bpd_create(const bpd_config* cfg, void* workspace, size_t workspace_bytes, void* hip_stream, bpd_ctx** out) {
  if (!cfg || !workspace || !out) return BPD_E_ARG;
  if (!config_ok(*cfg)) return BPD_E_ARG;
  if (((uintptr_t)workspace) % ALIGN) return BPD_E_ARG;
  Layout probe;
  if (workspace_bytes < build_layout(*cfg, nullptr, probe)) return BPD_E_CAPACITY;
  bpd_ctx* ctx = new bpd_ctx();
  ctx->cfg = *cfg;
  ctx->stream = (hipStream_t)hip_stream;
  {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) { delete ctx; return BPD_E_HIP; }
    ctx->device = dev;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0) ctx->num_cus = cus;
    if (!g_scratch_ptr[dev]) {               // once per device, with that device current
      void* sp = nullptr;
      if (hipGetSymbolAddress(&sp, HIP_SYMBOL(scratch)) != hipSuccess || !sp) { (void)hipGetLastError(); delete ctx; return BPD_E_HIP; }
      g_scratch_ptr[dev] = sp;
    }
  }
  build_layout(*cfg, (char*)workspace, ctx->lay);
  build_table(ctx);
  {
    const size_t d = cfg->d_model, F = cfg->d_ff, V = cfg->vocab, k = cfg->k_max;
    const size_t step_weights = ((size_t)cfg->n_dec_layers * (6 * d * d + 2 * d * F) + 2 * k * d * F + V * d) * act_size(*cfg);
    ctx->weights_exceed_llc = step_weights > ((size_t)192 << 20);
  }
  (void)hipMemsetAsync(ctx->lay.stack_err, 0, 256, ctx->stream);
  if (ctx->lay.stack_ex && ctx->num_cus <= XCC_MAP_MAX) {
    // placement probe: which XCD does workgroup i of a one-workgroup-per-CU grid land on?  The stack kernel needs the
    // regular round-robin (workgroup i on XCD i mod nx, every XCD equally often) and at most 64 workers per XCD.
    const char* env = getenv("BPD_DECODER_STACK");
    std::vector<StackLayerP> table(STACK_MAX_LAYERS);        // the layers' weights and caches: fixed addresses in the workspace
    {
      const bpd_config& c = *cfg;
      Layout& L = ctx->lay;
      const size_t d = c.d_model, slots = (size_t)c.max_out_len + c.k_max + 1, as = 2;
      for (int l = 0; l < c.n_dec_layers; ++l) {
        const DecL& w = L.dec[l];
        StackLayerP& q = table[l];
        q.wqkv = w.wqkv; q.wo = w.wo; q.cq = w.cq; q.co = w.co; q.w1 = w.w1; q.w2 = w.w2;
        q.ln1g = w.ln1.g; q.ln1b = w.ln1.b; q.ln2g = w.ln2.g; q.ln2b = w.ln2.b; q.ln3g = w.ln3.g; q.ln3b = w.ln3.b;
        q.b1 = w.b1; q.b2 = w.b2;
        q.selfK = (char*)L.selfK + (size_t)l * c.max_batch * kv_rows(c, slots) * d * as;
        q.selfV = (char*)L.selfV + (size_t)l * c.max_batch * kv_rows(c, slots) * d * as;
        q.crossK = (char*)L.crossK + (size_t)l * c.max_batch * kv_rows(c, c.max_src_len) * d * as;
        q.crossV = (char*)L.crossV + (size_t)l * c.max_batch * kv_rows(c, c.max_src_len) * d * as;
      }
      (void)hipMemcpyAsync(ctx->lay.stack_layers, table.data(), sizeof(StackLayerP) * STACK_MAX_LAYERS, hipMemcpyHostToDevice, ctx->stream);
    }
    (void)hipMemsetAsync(ctx->lay.stack_flags, 0, (size_t)cfg->n_dec_layers * STACK_OPS * STACK_FLAG_STRIDE * 4, ctx->stream);
    hipLaunchKernelGGL(xcc_map_kernel, dim3(ctx->num_cus), dim3(64), 0, ctx->stream, ctx->lay.xcc_map);
    std::vector<unsigned> map(ctx->num_cus);
    if (hipMemcpyAsync(map.data(), ctx->lay.xcc_map, map.size() * 4, hipMemcpyDeviceToHost, ctx->stream) == hipSuccess &&
        hipStreamSynchronize(ctx->stream) == hipSuccess && env && env[0] == '1') {      // opt-in: slower than the kernel chain so far
      int nx = 1;
      while (nx < ctx->num_cus && map[nx] != map[0]) ++nx;
      bool ok = ctx->num_cus % nx == 0 && ctx->num_cus / nx <= STACK_FLAG_STRIDE;
      for (int i = 0; ok && i < ctx->num_cus; ++i) ok = map[i] == map[i % nx];
      for (int i = 0; ok && i < nx; ++i)
        for (int j = 0; ok && j < i; ++j) ok = map[i] != map[j];
      if (ok) { ctx->stack_nx = nx; ctx->stack_xcc = (int)map[0]; ctx->stack_workers = ctx->num_cus / nx; }
    }
    (void)hipGetLastError();
  }
  if (const char* env = getenv("BPD_LAYERS_GROUP")) ctx->layers_group = std::max(0, atoi(env));
  if (ctx->lay.layers_sync) (void)hipMemsetAsync(ctx->lay.layers_sync, 0, (size_t)LK_WORDS * 4, ctx->stream);
  (void)hipMemsetAsync(ctx->lay.zeros, 0, ctx->lay.n_zeros * 4, ctx->stream);
  (void)hipMemsetAsync(ctx->lay.step_counter, 0, 4, ctx->stream);
  (void)hipMemsetAsync(ctx->lay.stats, 0, 32 * 8, ctx->stream);
  (void)hipMemsetAsync(ctx->lay.stats_ln, 0, 64 * 16 * 2 * 4, ctx->stream);
  {
    const size_t B = cfg->max_batch, k = cfg->k_max, S = cfg->max_src_len, T = cfg->max_out_len;
    const size_t n_in = B * S + 3 * B, n_sched = B * T;
    ctx->n_stage_out = std::min(FETCH_KERNEL_MAX, std::max(B * T + B, B * k * (k + 1) + 2 * B) + 64);      // (64: the statistics)
    const size_t ints = 4 * B + 16 + n_in + n_sched + ctx->n_stage_out;
    if (hipHostMalloc((void**)&ctx->report, ints * sizeof(int), hipHostMallocDefault) != hipSuccess) {
      (void)hipGetLastError();
      delete ctx;
      return BPD_E_HIP;
    }
    ctx->done = ctx->report + 2 * B;
    ctx->stage_in = (int*)(ctx->done + 8); ctx->stage_sched = ctx->stage_in + n_in; ctx->stage_out = ctx->stage_sched + n_sched;
    memset(ctx->report, 0, (2 * B + 8) * 8);
    ctx->remaining.assign(B, -1);
  }
  *out = ctx;
  return BPD_OK;
}

int bpd_destroy(bpd_ctx* ctx) {
  if (!ctx) return BPD_E_ARG;
  (void)hipStreamSynchronize(ctx->stream);
  if (const char* path = getenv("BPD_STACK_TRACE")) {      // debugging aid: the last stack launch's timestamps, raw
    if (ctx->lay.stack_trace && ctx->stack_workers > 0) {
      const size_t n = (size_t)ctx->stack_workers * ctx->cfg.n_dec_layers * STACK_OPS * 8;
      std::vector<unsigned long long> t(n);
      if (hipMemcpy(t.data(), ctx->lay.stack_trace, n * 8, hipMemcpyDeviceToHost) == hipSuccess)
        if (FILE* f = fopen(path, "wb")) { fwrite(t.data(), 8, n, f); fclose(f); }
    }
  }
  release_retired(ctx);
  for (auto& kind : ctx->plans)
    for (auto& q : kind)
      if (q.exec) (void)hipGraphExecDestroy(q.exec);
  if (ctx->plan_stream) (void)hipStreamDestroy(ctx->plan_stream);
  for (auto e : ctx->prof_ev) (void)hipEventDestroy(e);
  if (ctx->report) (void)hipHostFree(ctx->report);
  delete ctx;
  return BPD_OK;
}

const char* bpd_last_error(const bpd_ctx* ctx) { return ctx ? ctx->err.c_str() : "null context"; }

int bpd_load_weights(bpd_ctx* ctx, const bpd_tensor* tensors, int n) {
  if (!ctx || !tensors || n < 0) return fail(ctx, BPD_E_ARG, "bpd_load_weights: null argument");
  const bool bf = ctx->cfg.dtype == BPD_BF16;
  // validate everything first so that a bad tensor leaves the loaded set unchanged
  for (int t = 0; t < n; ++t) {
    const bpd_tensor& T = tensors[t];
    if (!T.name || !T.data) return fail(ctx, BPD_E_ARG, "bpd_load_weights: tensor without name or data");
    auto it = ctx->table.find(T.name);
    if (it == ctx->table.end()) return fail(ctx, BPD_E_WEIGHTS, std::string("unknown tensor ") + T.name);
    const WEntry& e = it->second;
    if (T.dtype != BPD_F32 && T.dtype != BPD_BF16) return fail(ctx, BPD_E_WEIGHTS, std::string("bad dtype for ") + T.name);
    bool ok = T.ndim == e.nd;
    for (int i = 0; ok && i < e.nd; ++i) ok = T.shape[i] == e.shape[i];
    if (!ok) return fail(ctx, BPD_E_WEIGHTS, std::string("wrong shape for ") + T.name);
    size_t count = 1;
    for (int i = 0; i < e.nd; ++i) count *= (size_t)e.shape[i];
    if (!T.on_device && count * (T.dtype == BPD_F32 ? 4 : 2) > ctx->lay.staging_bytes)
      return fail(ctx, BPD_E_CAPACITY, std::string("staging area too small for ") + T.name);
  }
  for (int t = 0; t < n; ++t) {
    const bpd_tensor& T = tensors[t];
    WEntry& e = ctx->table[T.name];
    size_t count = 1;
    for (int i = 0; i < e.nd; ++i) count *= (size_t)e.shape[i];
    const size_t esz = T.dtype == BPD_F32 ? 4 : 2;
    const void* src = T.data;
    if (!T.on_device) {                          // (fits the staging area: checked above)
      HIPCHK(hipMemcpyAsync(ctx->lay.staging, T.data, count * esz, hipMemcpyHostToDevice, ctx->stream));
      src = ctx->lay.staging;
    }
    const dim3 blk(256);
    auto conv_mat = [&](const void* s, void* dst, int K, int N, int transposed, int ldw, int n_off) {
      const long tot = (long)K * N;
      dim3 grid((unsigned)((tot + 255) / 256));
      if (T.dtype == BPD_F32) {
        if (bf) hipLaunchKernelGGL((convert_matrix_kernel<float, true>), grid, blk, 0, ctx->stream, (const float*)s, dst, K, N, transposed, ldw, n_off);
        else hipLaunchKernelGGL((convert_matrix_kernel<float, false>), grid, blk, 0, ctx->stream, (const float*)s, dst, K, N, transposed, ldw, n_off);
      } else {
        if (bf) hipLaunchKernelGGL((convert_matrix_kernel<bf16_t, true>), grid, blk, 0, ctx->stream, (const bf16_t*)s, dst, K, N, transposed, ldw, n_off);
        else hipLaunchKernelGGL((convert_matrix_kernel<bf16_t, false>), grid, blk, 0, ctx->stream, (const bf16_t*)s, dst, K, N, transposed, ldw, n_off);
      }
    };
    auto conv_vec = [&](const void* s, float* dst, size_t cnt) {
      dim3 grid((unsigned)((cnt + 255) / 256));
      if (T.dtype == BPD_F32) hipLaunchKernelGGL(convert_vector_kernel<float>, grid, blk, 0, ctx->stream, (const float*)s, dst, (long)cnt);
      else hipLaunchKernelGGL(convert_vector_kernel<bf16_t>, grid, blk, 0, ctx->stream, (const bf16_t*)s, dst, (long)cnt);
    };
    const size_t wsz = bf ? 2 : 4;
    switch (e.kind) {
      case VEC: conv_vec(src, (float*)e.dst, count); break;
      case MAT: conv_mat(src, e.dst, e.K, e.N, 0, e.ldw, e.n_off); break;
      case EMB:
        if (bf) conv_mat(src, e.dst, e.K, e.N, 1, e.ldw, 0);      // as the projection matrix W[d][V] = E^T
        else {
          conv_vec(src, (float*)e.dst, count);                      // fp32 kernels read E[V][d] directly
          if (ctx->lay.emb_t) conv_mat(src, ctx->lay.emb_t, e.K, e.N, 1, e.ldw, 0);
        }
        break;
      case MATK_CAT:
        for (int i = 0; i < (int)e.shape[0]; ++i)
          conv_mat((const char*)src + (size_t)i * e.K * e.N * esz, e.dst, e.K, e.N, 0, e.ldw, i * e.N);
        break;
      case MATK_SEP:
        for (int i = 0; i < (int)e.shape[0]; ++i)
          conv_mat((const char*)src + (size_t)i * e.K * e.N * esz, (char*)e.dst + (size_t)i * e.K * e.N * wsz, e.K, e.N, 0, e.ldw, 0);
        break;
    }
    LAUNCHCHK();
    HIPCHK(hipStreamSynchronize(ctx->stream));   // the staging area and the caller's buffer are free again
    e.loaded = true;
    ctx->fold_ready = false;
  }
  ctx->encoded = false;
  bool all = true;
  for (auto& kv : ctx->table) all = all && kv.second.loaded;
  if (all) { refresh_folded_weights(ctx); LAUNCHCHK(); }      // (here and not in bpd_encode: a captured one would fold at its replays only)
  return BPD_OK;
}

int bpd_encode(bpd_ctx* ctx, const int32_t* src_ids, const int32_t* src_len, const int32_t* max_len, int B, int S) {
  if (!ctx || !src_ids || !src_len) return fail(ctx, BPD_E_ARG, "bpd_encode: null argument");
  const bpd_config& c = ctx->cfg;
  if (B < 1 || S < 1) return fail(ctx, BPD_E_ARG, "bpd_encode: B and S must be positive");
  if (B > c.max_batch || S > c.max_src_len) return fail(ctx, BPD_E_CAPACITY, "bpd_encode: batch or source length over the configured maximum");
  for (auto& kv : ctx->table)
    if (!kv.second.loaded) return fail(ctx, BPD_E_STATE, "bpd_encode: tensor not loaded: " + kv.first);
  // Host arrays are validated here and pass through the pinned staging area (free again once the last encode that used it has
  // read its own); the kernel that takes them clamps, so device arrays are safe as well.  In a graph of the caller's the area
  // would be read at every replay, whatever lies there by then: host arrays are copied from where they are instead.
  int *h_ids = ctx->stage_in, *h_len = h_ids + (size_t)c.max_batch * c.max_src_len, *h_max = h_len + c.max_batch, *h_first = h_max + c.max_batch;
  const bool host_ids = is_host_ptr(src_ids), host_len = is_host_ptr(src_len), host_max = max_len && is_host_ptr(max_len);
  if (host_len) {
    for (int b = 0; b < B; ++b)
      if (src_len[b] < 1 || src_len[b] > S) return fail(ctx, BPD_E_ARG, "bpd_encode: src_len out of range");
  }
  if (host_ids) {
    for (long i = 0; i < (long)B * S; ++i)
      if (src_ids[i] < 0 || src_ids[i] >= c.vocab) return fail(ctx, BPD_E_ARG, "bpd_encode: source id out of range");
  }
  if (host_max) {
    for (int b = 0; b < B; ++b)
      if (max_len[b] < 1 || max_len[b] > c.max_out_len) return fail(ctx, BPD_E_ARG, "bpd_encode: max_len out of range");
  }
  Layout& L = ctx->lay;
  forget_replayed(ctx);
  ctx->B = B; ctx->S = S; ctx->encoded = false; ctx->x_ready_k = 0;
  refresh_folded_weights(ctx);                    // (every tensor is loaded: checked above; nothing to do unless bpd_load_weights failed halfway)
  const int *from_ids = src_ids, *from_len = src_len, *from_max = max_len;
  const bool host = host_ids || host_len || host_max, staged = host && !capturing(ctx);
  if (staged) {
    const int rc = wait_done(ctx, &ctx->done[1], ctx->encode_tag);
    if (rc) return rc;
    if (host_ids) { memcpy(h_ids, src_ids, (size_t)B * S * 4); from_ids = h_ids; }
    if (host_len) { memcpy(h_len, src_len, (size_t)B * 4); from_len = h_len; }
    if (host_max) { memcpy(h_max, max_len, (size_t)B * 4); from_max = h_max; }
  } else if (host) {
    if (host_ids) { HIPCHK(hipMemcpyAsync(L.src_ids, src_ids, (size_t)B * S * 4, hipMemcpyHostToDevice, ctx->stream)); from_ids = L.src_ids; }
    if (host_len) { HIPCHK(hipMemcpyAsync(L.src_len, src_len, (size_t)B * 4, hipMemcpyHostToDevice, ctx->stream)); from_len = L.src_len; }
    if (host_max) { HIPCHK(hipMemcpyAsync(L.max_len, max_len, (size_t)B * 4, hipMemcpyHostToDevice, ctx->stream)); from_max = L.max_len; }
  }
  // Lengths that the host has: without the padding.  (In a graph of the caller's they are whatever lies there at the replay.)
  PackP packed{};
  if (staged && host_len && kv_grouped(c) && attention_nsplit(ctx, S, B, S, 0) == 1) {
    long tokens = 0;
    for (int b = 0; b < B; ++b) { h_first[b] = (int)tokens; tokens += h_len[b]; }
    packed = PackP{h_first, packed_source_rows(c, tokens, (long)B * S), L.src_row0, L.src_seq, L.src_pos, L.src_packed};
  }
  for (int b = 0; b < B; ++b) ctx->remaining[b] = !max_len ? c.max_out_len : (host_max ? max_len[b] : -1);
  {
    const size_t most = std::max((size_t)B * S, (size_t)B * std::max(c.max_out_len, c.k_max * c.k_max));
    hipLaunchKernelGGL(encode_init_kernel, dim3((unsigned)std::min<size_t>(256, (most + 255) / 256)), dim3(256), 0, ctx->stream, state_params(ctx),
                       from_ids, from_len, from_max, L.src_ids, L.src_len, B, S, c.vocab, c.pad_id,
                       (unsigned*)L.step_counter, staged ? &ctx->done[1] : nullptr, ctx->encode_tag + 1, packed);
    LAUNCHCHK();
    if (staged) ++ctx->encode_tag;
  }
  use_slots(ctx, B);
  if (small_encode_ok(ctx)) {
    small_encode(ctx);
  } else {
    ctx->steps = 0;
    const int rc = run_planned(ctx, PLAN_ENCODE, {B, S, ctx->local_q, ctx->local_m, layers_way(ctx, B, 1), packed.rows}, [&]() -> int {
      int rc = encoder(ctx, packed.rows);
      if (rc) return rc;
      // first invocation: position 0 only, all heads -> first proposals
      rc = forward(ctx, 1, c.k_max, 1, nullptr);
      if (rc) return rc;
      hipLaunchKernelGGL(prime_kernel, dim3(B), dim3(64), 0, ctx->stream, state_params(ctx), L.keys, B);
      LAUNCHCHK();
      return BPD_OK;
    });
    if (rc) return rc;
  }
  LAUNCHCHK();
  ctx->steps = 0;
  ctx->live1 = ctx->live2 = B;
  ctx->budget_min = !max_len ? c.max_out_len : (host_max ? *std::min_element(max_len, max_len + B) : 0);
  ctx->encoded = true;
  return BPD_OK;
}

// A step in two parts: the model invocation on the slots of use_slots(), then verify / accept / commit, which also embeds
// the next block, for next_slots slots.
static int step_forward(bpd_ctx* ctx, int k, const int* imposed_dev, int imposed_stride, int imposed_step) {
  ctx->cur_imposed = imposed_dev; ctx->cur_imposed_stride = imposed_stride; ctx->cur_imposed_step = imposed_step;
  return forward(ctx, k, k, 0, nullptr);
}
// report_tag: bpd_decode's tag of this step (0: not a step of bpd_decode)
static int step_accept(bpd_ctx* ctx, int k, int* accepted_dev, int next_slots, unsigned report_tag) {
  Layout& L = ctx->lay;
  {
    PhaseTimer t(ctx, BPD_PHASE_ACCEPT);
    StateP s = state_params(ctx);
    s.imposed = ctx->cur_imposed; s.imposed_stride = ctx->cur_imposed_stride;
    if (report_tag) s.dyn = (const StepDyn*)L.dyn;
    const bpd_config& c = ctx->cfg;
    const int imposed_step = ctx->cur_imposed_step;
    if (embed_in_accept(ctx)) {
      // the accept kernel also embeds the next block (same k assumed; checked by forward); its LayerNorm statistics go
      // where the first layer will look for them: the single-tile layout for at most 16 rows, per-tile rows otherwise
      const int rows = next_slots * k;
      const bool sp = stats_path(ctx, rows), lean = lean_ok(c, rows);
      hipLaunchKernelGGL(accept_embed_kernel, dim3(ctx->B), dim3(1024), 0, ctx->stream, s, L.keys, k, ctx->B, imposed_step, accepted_dev,
                         c.d_model, (const bf16_t*)L.emb, c.vocab, (const float*)L.pos_tgt, sqrtf((float)c.d_model), L.x,
                         lean ? nullptr : (sp ? L.stats_ln : L.stats_big), sp ? 16 : rows, sp || lean ? (bf16_t*)nullptr : (bf16_t*)L.xn,
                         !slots_used(ctx) ? 0 : (ctx->seq ? 2 : 1), ctx->two_phase && k > 1 && ctx->B * k > 16);
      ctx->x_ready_k = k; ctx->x_ready_slots = next_slots;
    } else {
      hipLaunchKernelGGL(accept_kernel, dim3(ctx->B), dim3(64), 0, ctx->stream, s, L.keys, k, ctx->B, 1, imposed_step, accepted_dev, (float*)nullptr, 0);
      ctx->x_ready_k = 0;
    }
  }
  LAUNCHCHK();
  ctx->steps++;
  return BPD_OK;
}
// A whole step that the host does not follow (bpd_step, bpd_step_static).
static int step_impl(bpd_ctx* ctx, int k, const int* imposed_dev, int* accepted_dev) {
  PhaseTimer whole(ctx, BPD_PHASE_STEP);
  std::fill(ctx->remaining.begin(), ctx->remaining.end(), -1);
  ctx->live1 = ctx->live2 = -1;
  use_slots(ctx, -1);
  const int hgroup = ctx->prof_phase == 0 || ctx->prof_phase == BPD_PHASE_STEP ? small_hgroup(ctx, k, 0) : 0;
  if (hgroup > 0) {
    small_decode(ctx, k, hgroup, 1, imposed_dev, 0, accepted_dev, nullptr);
    LAUNCHCHK();
    ctx->steps++;
    return BPD_OK;
  }
  const int rc = step_forward(ctx, k, imposed_dev, 0, 0);
  if (rc) return rc;
  return step_accept(ctx, k, accepted_dev, ctx->B, 0);
}

int bpd_step(bpd_ctx* ctx, int k, const int32_t* imposed_accept, int32_t* accepted_len) {
  if (!ctx) return BPD_E_ARG;
  if (!ctx->encoded) return fail(ctx, BPD_E_STATE, "bpd_step: call bpd_encode first");
  if (k < 1 || k > ctx->cfg.k_max) return fail(ctx, BPD_E_ARG, "bpd_step: k outside 1..k_max");
  Layout& L = ctx->lay;
  forget_replayed(ctx);
  // device pointers are used in place by the accept kernel; host arrays go through a copy
  const int* imp = nullptr;
  if (imposed_accept) {
    if (is_host_ptr(imposed_accept)) {
      HIPCHK(hipMemcpyAsync(L.imposed1, imposed_accept, (size_t)ctx->B * 4, hipMemcpyHostToDevice, ctx->stream));
      imp = L.imposed1;
    } else {
      imp = imposed_accept;
    }
  }
  const bool out_host = accepted_len && is_host_ptr(accepted_len);
  int rc = step_impl(ctx, k, imp, out_host ? nullptr : accepted_len);
  if (rc) return rc;
  if (out_host) HIPCHK(hipMemcpyAsync(accepted_len, L.accepted, (size_t)ctx->B * 4, hipMemcpyDeviceToHost, ctx->stream));
  return BPD_OK;
}

int bpd_step_static(bpd_ctx* ctx, int k, const int32_t* imposed_accept, int32_t* accepted_len) {
  if (!ctx) return BPD_E_ARG;
  if (!ctx->encoded) return fail(ctx, BPD_E_STATE, "bpd_step_static: call bpd_encode first");
  if (k < 1 || k > ctx->cfg.k_max) return fail(ctx, BPD_E_ARG, "bpd_step_static: k outside 1..k_max");
  Layout& L = ctx->lay;
  const bpd_config& c = ctx->cfg;
  forget_replayed(ctx);
  char* sp = (char*)g_scratch_ptr[ctx->device];
  if (!sp) return fail(ctx, BPD_E_STATE, "bpd_step_static: no scratch address for this device");
  // what this step needs: its k x k keys per sequence, the head-1 / second-phase keys, the attention partials, and as
  // many K slices as bpd_step would use for the same block (so that both sum in the same order)
  const size_t M = (size_t)ctx->B * k, d = c.d_model;
  auto up = [](size_t v) { return (v + ALIGN - 1) / ALIGN * ALIGN; };
  const size_t keys_b = up(M * k * 8), keys_h1_b = up(2 * M * 8);
  size_t attn_b = 0;                       // partial results of a split attention launch: splits x (head, sequence, row tile)
  for (int causal : {1, 0}) {
    const int ns = attention_nsplit(ctx, causal ? c.max_out_len + c.k_max + 1 : c.max_src_len, ctx->B, k, causal);
    const size_t wgs = (size_t)c.n_heads * ctx->B * ((k + 15) / 16);
    if (ns > 1) attn_b = std::max(attn_b, up(ns * wgs * 16 * (d / c.n_heads + 2) * 4));
  }
  if (layers_way(ctx, ctx->B, k) == LAYERS_JOBS && layers_split_of(ctx, ctx->B, k) > 1) attn_b = std::max(attn_b, up((size_t)layers_split_of(ctx, ctx->B, k) * c.n_heads * ctx->B * 16 * 66 * 4));
  size_t slices = 1;
  if (lean_ok(c, (int)M)) slices = lean_slices(ctx, (int)M);
  else if (c.dtype == BPD_BF16 && M > 16)
    for (int K : {c.d_model, c.d_ff}) {
      const int ns = residual_k_slices(ctx, gp(nullptr, K, nullptr, c.d_model, (int)M, c.d_model, K));
      if ((size_t)ns > slices) slices = ns;
    }
  const size_t kpart_b = slices > 1 ? up(slices * M * d * 4) : 0;
  if (keys_b + keys_h1_b + attn_b + kpart_b > STATIC_SCRATCH_BYTES)
    return fail(ctx, BPD_E_CAPACITY, "bpd_step_static: this step needs " + std::to_string(keys_b + keys_h1_b + attn_b + kpart_b) +
                                     " bytes of scratch, the static array holds " + std::to_string(STATIC_SCRATCH_BYTES));
  const int* imp = nullptr;
  if (imposed_accept) {
    if (is_host_ptr(imposed_accept)) {
      HIPCHK(hipMemcpyAsync(L.imposed1, imposed_accept, (size_t)ctx->B * 4, hipMemcpyHostToDevice, ctx->stream));
      imp = L.imposed1;
    } else {
      imp = imposed_accept;
    }
  }
  const bool out_host = accepted_len && is_host_ptr(accepted_len);
  // the step's kernels take their scratch from the layout: point it at the static array for this call
  unsigned long long* const keys0 = L.keys; unsigned long long* const keys_h10 = L.keys_h1;
  float* const attn0 = L.attn_part; float* const kpart0 = L.kpart;
  L.keys = (unsigned long long*)sp;
  L.keys_h1 = (unsigned long long*)(sp + keys_b);
  L.attn_part = (float*)(sp + keys_b + keys_h1_b);
  L.kpart = (float*)(sp + keys_b + keys_h1_b + attn_b);
  // the array keeps the last call's contents and the keys are merged with atomic max: they start at zero
  // (a fill kernel, not a memset node: callers may be capturing the stream)
  fill_i32(ctx, (int*)L.keys, (long)(2 * M * k), 0);
  int rc = step_impl(ctx, k, imp, out_host ? nullptr : accepted_len);
  L.keys = keys0; L.keys_h1 = keys_h10; L.attn_part = attn0; L.kpart = kpart0;
  // (this step's accept kernel cleared the static keys, not the workspace's: the next step embeds its block and clears
  // its keys itself)
  ctx->x_ready_k = 0;
  if (rc) return rc;
  if (out_host) HIPCHK(hipMemcpyAsync(accepted_len, L.accepted, (size_t)ctx->B * 4, hipMemcpyDeviceToHost, ctx->stream));
  return BPD_OK;
}

int bpd_set_acceptance(bpd_ctx* ctx, int distance_eps, int min_block) {
  if (!ctx) return BPD_E_ARG;
  if (distance_eps < 0 || min_block < 1 || min_block > ctx->cfg.k_max) return fail(ctx, BPD_E_ARG, "bpd_set_acceptance: out of range");
  ctx->distance_eps = distance_eps; ctx->min_block = min_block;
  return BPD_OK;
}

int bpd_set_top_n(bpd_ctx* ctx, int n) {
  if (!ctx) return BPD_E_ARG;
  if (n < 1 || n > ctx->cfg.vocab) return fail(ctx, BPD_E_ARG, "bpd_set_top_n: n outside 1..vocab");
  ctx->top_n = n;
  return BPD_OK;
}

int bpd_set_two_phase(bpd_ctx* ctx, int on) {
  if (!ctx) return BPD_E_ARG;
  ctx->two_phase = on != 0;
  return BPD_OK;
}

int bpd_set_local_attention(bpd_ctx* ctx, int query_block, int memory_len) {
  if (!ctx) return BPD_E_ARG;
  if (query_block < 0 || memory_len < 0 || (query_block == 0 && memory_len != 0))
    return fail(ctx, BPD_E_ARG, "local attention: query_block >= 0, memory_len >= 0 (and 0 when query_block is 0)");
  ctx->local_q = query_block; ctx->local_m = memory_len;
  return BPD_OK;
}

static void stats_of(const bpd_ctx* ctx, const long long* raw, bpd_stats* st) {
  st->steps = raw[20]; st->invocations = ctx->encoded ? raw[20] + 1 : 0;
  st->seq_steps = raw[0]; st->accepted_total = raw[1]; st->finished = (int32_t)raw[2];
  for (int i = 0; i < 17; ++i) st->hist[i] = raw[3 + i];
}

// Has a wait of a whole-layer kernel run out since the last bpd_encode (which clears the word)?  Everything since is invalid, whoever asks for
// it, and the context's later steps and encodes go kernel by kernel.
static int layers_check(bpd_ctx* ctx, const long long* raw) {
  if (!raw[31]) return BPD_OK;
  ctx->layers_group = 0;
  return fail(ctx, BPD_E_HIP, "decoder layers: a bounded wait ran out; results since the last bpd_encode are invalid, later steps use the per-operator kernels");
}

int bpd_get_stats(bpd_ctx* ctx, bpd_stats* st) {
  if (!ctx || !st) return BPD_E_ARG;
  long long raw[32];
  int rc = fetch(ctx, {{(const int*)ctx->lay.stats, 64, raw}});
  if (rc == BPD_OK) rc = layers_check(ctx, raw);
  if (rc) return rc;
  stats_of(ctx, raw, st);
  return stack_check(ctx);
}

static int output_and_stats(bpd_ctx* ctx, int32_t* out_ids, int32_t* out_len, bpd_stats* st, bool count_steps = false) {
  Layout& L = ctx->lay;
  long long raw[32];
  int rc = fetch(ctx, {{L.out_ids, (size_t)ctx->B * ctx->cfg.max_out_len, out_ids}, {L.j, (size_t)ctx->B, out_len},
                       {(const int*)L.stats, 64, raw}});
  if (rc == BPD_OK) rc = layers_check(ctx, raw);
  if (rc) return rc;
  if (count_steps) ctx->steps = raw[20];
  if (st) stats_of(ctx, raw, st);
  return stack_check(ctx);
}

int bpd_get_output(bpd_ctx* ctx, int32_t* out_ids, int32_t* out_len) {
  if (!ctx) return BPD_E_ARG;
  if (!ctx->encoded) return fail(ctx, BPD_E_STATE, "bpd_get_output: nothing decoded");
  return output_and_stats(ctx, out_ids, out_len, nullptr);
}

// The host follows the decode through words that the accept kernel of every step stores in pinned memory (StateP::report),
// and stays one step ahead of them: step s is enqueued while step s - 1 runs, then the host waits for the report of s - 1
// (and tells the accept kernel of step s how many sequences step s + 1 will still have).
// Enqueueing takes less than a step, so the stream never runs dry, and at most one step is enqueued in vain: where an
// end-of-sequence token, not the length budget, ends the last sequence.  If the budgets say that step s - 1 may be the
// last one, its report is awaited before step s is enqueued.  (Stopping the stream every four steps to ask cost 25 us per
// step of the base model at batch 1 and up to three steps in vain at the end.)
int bpd_decode(bpd_ctx* ctx, int k, const int32_t* schedule, int max_steps, int32_t* out_ids, int32_t* out_len, bpd_stats* stats) {
  if (!ctx) return BPD_E_ARG;
  if (!ctx->encoded) return fail(ctx, BPD_E_STATE, "bpd_decode: call bpd_encode first");
  if (k < 1 || k > ctx->cfg.k_max || max_steps < 0) return fail(ctx, BPD_E_ARG, "bpd_decode: bad k or max_steps");
  forget_replayed(ctx);
  Layout& L = ctx->lay;
  const int B = ctx->B;
  const int* imp = nullptr;
  const int* host_sched = nullptr;
  if (schedule) {
    // a live sequence takes at least one token per step, so max_out_len rows always suffice
    if (max_steps > ctx->cfg.max_out_len) max_steps = ctx->cfg.max_out_len;
    imp = L.sched;
  }
  {
    const int rows = schedule ? max_steps : 0;
    const int* src = schedule;
    if (rows > 0 && is_host_ptr(schedule)) {     // (the decode before this one has ended: its copy has been made)
      memcpy(ctx->stage_sched, schedule, (size_t)rows * B * 4);
      src = host_sched = ctx->stage_sched;
    }
    if (ctx->report_tag > 0x7FFFFFFFu) ctx->report_tag = 2;        // (turns kept; far from the tags that old words hold)
    const long n = (long)rows * B;
    const StepDyn dyn{imp, B, rows, ctx->report_tag, ctx->report, ctx->cfg.max_batch};
    if (max_steps > 0)
      hipLaunchKernelGGL(decode_init_kernel, dim3((unsigned)((std::max<long>(n, B) + 255) / 256)), dim3(256), 0, ctx->stream, state_params(ctx), dyn, (StepDyn*)L.dyn,
                         src, L.sched, n, B);
    LAUNCHCHK();
  }
  auto& rem = ctx->remaining;
  long more = (long)max_steps * k;               // rows that the caches may grow by
  if (std::find(rem.begin(), rem.begin() + B, -1) == rem.begin() + B) more = std::min(more, (long)*std::max_element(rem.begin(), rem.begin() + B));
  if (const int hgroup = ctx->prof_phase == 0 ? small_hgroup(ctx, k, more) : 0) {      // the whole decode as one kernel
    if (max_steps > 0) {
      std::fill(rem.begin(), rem.end(), -1);
      small_decode(ctx, k, hgroup, max_steps, imp, B, nullptr, nullptr);
      LAUNCHCHK();
    }
    return output_and_stats(ctx, out_ids, out_len, stats, true);
  }
  // may step s end the last sequence by its budget, as far as the reports before s tell?
  auto may_be_last = [&](int s) {
    for (int b = 0; b < B; ++b) {
      if (rem[b] < 0) return false;              // not known: run ahead, the report will tell
      int most = k;
      if (host_sched) { const int a = host_sched[(size_t)s * B + b]; most = a < 1 ? 1 : (a > k ? k : a); }
      if (rem[b] > most) return false;
    }
    return true;
  };
  // the report of the step that was given this tag: the sequences that go on after it
  auto await = [&](unsigned tag, int& going) {
    const unsigned long long* words = report_of(ctx, tag);
    going = 0;
    for (int b = 0; b < B; ++b) {
      const int rc = wait_report(ctx, &words[b], tag);
      if (rc) return rc;
      rem[b] = (int)(unsigned)words[b];
      going += rem[b] > 0;
    }
    return (int)BPD_OK;
  };
  bool ended = true;                             // (known from an earlier decode: nothing is left to do)
  for (int b = 0; b < B; ++b) ended = ended && rem[b] == 0;
  for (int s = 0; s < max_steps && !ended; ++s) {
    PhaseTimer whole(ctx, BPD_PHASE_STEP);
    const unsigned before = ctx->report_tag;     // of step s - 1
    bool know = s == 0;
    if (s > 0 && may_be_last(s - 1)) {
      const int rc = await(before, ctx->live1);
      if (rc) return rc;
      if (ctx->live1 == 0) break;
      know = true;
    }
    // A step like the one before, of all sequences and for all of them (one sentence; images before the first ends): recorded once, replayed
    // from then on.  All sequences go on after step s - 1 for certain: there is one, or only budgets end them and none is that short.
    bool planned = s > 0 && !ctx->two_phase && embed_in_accept(ctx) && ctx->x_ready_k == k && ctx->x_ready_slots == B && (B == 1 || (ctx->cfg.eos_id < 0 && ctx->live2 == B));
    for (int b = 0; planned && B > 1 && b < B; ++b) planned = rem[b] > (know ? 0 : k);
    if (planned) {
      use_slots(ctx, B);
      const int cap = ctx->cfg.max_out_len + ctx->cfg.k_max + 1;
      const bool few = attention_keys(ctx, cap, k, 1) <= 128;
      const int way = layers_way(ctx, B, k), nsplit = way == LAYERS_JOBS ? layers_split_of(ctx, B, k) : attention_nsplit(ctx, cap, B, k, 1);
      const int rc = run_planned(ctx, PLAN_STEP, {B, k, nsplit * 4 + way, few, ctx->top_n, ctx->local_q, ctx->local_m, ctx->distance_eps, ctx->min_block},
                                 [&]() -> int {
                                   const int ready = ctx->x_ready_k;
                                   const int64_t steps = ctx->steps;
                                   int rc = step_forward(ctx, k, nullptr, B, 0);
                                   if (rc == BPD_OK) rc = step_accept(ctx, k, nullptr, B, 1);
                                   ctx->x_ready_k = ready; ctx->steps = steps;       // (what a replay leaves as well)
                                   return rc;
                                 });
      if (rc) return rc;
      ctx->steps++;
      ++ctx->report_tag;
      if (!know) { const int rc2 = await(before, ctx->live1); if (rc2) return rc2; }
      if (ctx->live1 == 0) { ctx->x_ready_k = 0; break; }      // step s - 1 was the last: this one finds nothing to do
      ctx->live2 = ctx->live1; ctx->live1 = -1;
      if (s + 1 == max_steps) { const int rc2 = await(ctx->report_tag, ctx->live1); if (rc2) return rc2; }
      continue;
    }
    // Slots of this step: the sequences that had not ended after step s - 2 (live2); of the next: not after s - 1 (live1),
    // which the host waits for while the GPU has this step's layers to do
    use_slots(ctx, ctx->live2);
    int rc = step_forward(ctx, k, imp, B, s);
    if (rc == BPD_OK && !know) rc = await(before, ctx->live1);
    if (rc) return rc;
    if (ctx->live1 == 0) { ctx->x_ready_k = 0; break; }      // step s - 1 was the last: this one accepts nothing
    ++ctx->report_tag;
    const bool exact = slots_used(ctx) && ctx->live1 > 0;
    rc = step_accept(ctx, k, nullptr, exact ? ctx->live1 : B, ctx->report_tag);
    if (rc) return rc;
    ctx->live2 = ctx->live1; ctx->live1 = -1;
    if (s + 1 == max_steps) { rc = await(ctx->report_tag, ctx->live1); if (rc) return rc; }
  }
  return output_and_stats(ctx, out_ids, out_len, stats);
}

int bpd_get_state(bpd_ctx* ctx, int32_t* P, int32_t* A, int32_t* j, int32_t* finished) {
  if (!ctx) return BPD_E_ARG;
  if (!ctx->encoded) return fail(ctx, BPD_E_STATE, "bpd_get_state: call bpd_encode first");
  Layout& L = ctx->lay;
  const size_t B = ctx->B, k = ctx->cfg.k_max;
  long long raw[32];
  int rc = fetch(ctx, {{L.P, B * k, P}, {L.A, B * k * k, A}, {L.j, B, j}, {L.finished, B, finished}, {(const int*)L.stats, 64, raw}});
  if (rc == BPD_OK) rc = layers_check(ctx, raw);
  if (rc) return rc;
  return stack_check(ctx);
}

int bpd_set_proposals(bpd_ctx* ctx, const int32_t* P) {
  if (!ctx || !P) return fail(ctx, BPD_E_ARG, "bpd_set_proposals: null argument");
  if (!ctx->encoded) return fail(ctx, BPD_E_STATE, "bpd_set_proposals: call bpd_encode first");
  forget_replayed(ctx);
  const size_t n = (size_t)ctx->B * ctx->cfg.k_max;
  if (is_host_ptr(P)) {
    for (size_t i = 0; i < n; ++i)
      if (P[i] < 0 || P[i] >= ctx->cfg.vocab) return fail(ctx, BPD_E_ARG, "bpd_set_proposals: token id out of range");
  }
  HIPCHK(hipMemcpyAsync(ctx->lay.P, P, n * 4, hipMemcpyDefault, ctx->stream));
  ctx->x_ready_k = 0;              // a block embedded ahead of time used the old proposals
  return BPD_OK;
}

int bpd_debug_step_logits(bpd_ctx* ctx, int k, float* logits) {
  if (!ctx || !logits) return fail(ctx, BPD_E_ARG, "bpd_debug_step_logits: null argument");
  if (!ctx->encoded) return fail(ctx, BPD_E_STATE, "bpd_debug_step_logits: call bpd_encode first");
  if (k < 1 || k > ctx->cfg.k_max) return fail(ctx, BPD_E_ARG, "bpd_debug_step_logits: k outside 1..k_max");
  forget_replayed(ctx);
  use_slots(ctx, ctx->B);                         // every sequence, ended or not
  if (const int hgroup = ctx->prof_phase == 0 ? small_hgroup(ctx, k, 0) : 0) {
    small_decode(ctx, k, hgroup, 1, nullptr, 0, nullptr, logits);
    LAUNCHCHK();
    return BPD_OK;
  }
  int rc = forward(ctx, k, k, 0, logits);
  if (rc) return rc;
  hipLaunchKernelGGL(accept_kernel, dim3(ctx->B), dim3(64), 0, ctx->stream, state_params(ctx), ctx->lay.keys, k, ctx->B, 0, 0, nullptr, logits, ctx->cfg.vocab);
  LAUNCHCHK();
  return BPD_OK;
}

int bpd_profile_enable(bpd_ctx* ctx, int phase) {
  if (!ctx || phase < 0 || phase > BPD_PHASE_EMPTY) return BPD_E_ARG;
  (void)hipStreamSynchronize(ctx->stream);
  ctx->prof_phase = phase; ctx->prof_used = 0; ctx->prof_launches = 0;
  return BPD_OK;
}

int bpd_profile_read(bpd_ctx* ctx, double* total_ms, int64_t* launches) {
  if (!ctx || !total_ms || !launches) return BPD_E_ARG;
  return bpd_profile_samples(ctx, nullptr, 0, total_ms, launches);
}

int bpd_profile_samples(bpd_ctx* ctx, float* ms_out, int64_t capacity, double* total_ms, int64_t* launches) {
  if (!ctx || !total_ms || !launches || capacity < 0 || (capacity > 0 && !ms_out)) return BPD_E_ARG;
  HIPCHK(hipStreamSynchronize(ctx->stream));
  double tot = 0;
  int64_t n = 0;
  for (size_t i = 0; i + 1 < ctx->prof_used; i += 2, ++n) {
    float ms = 0.f;
    HIPCHK(hipEventElapsedTime(&ms, ctx->prof_ev[i], ctx->prof_ev[i + 1]));
    tot += ms;
    if (n < capacity) ms_out[n] = ms;
  }
  *total_ms = tot; *launches = ctx->prof_launches;
  ctx->prof_used = 0; ctx->prof_launches = 0;
  return BPD_OK;
}

// ------------------------------------------------------------------------------- machine peaks

int bpd_measure_hbm_read(void* buf_dev, size_t bytes, void* hip_stream, int iters, double* gbps) {
  if (!buf_dev || !gbps || iters < 1 || bytes < (1u << 20) || bytes % 4096 != 0) return BPD_E_ARG;
  hipStream_t s = (hipStream_t)hip_stream;
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) return BPD_E_HIP;
  const long n16 = (long)(bytes / 16);
  double best = 0;
  for (int rep = 0; rep < 3; ++rep) {
    (void)hipEventRecord(e0, s);
    for (int i = 0; i < iters; ++i)
      hipLaunchKernelGGL(peak_read_kernel, dim3(2048), dim3(256), 0, s, (const uint4*)buf_dev, n16, (unsigned*)buf_dev);
    (void)hipEventRecord(e1, s);
    if (hipStreamSynchronize(s) != hipSuccess) return BPD_E_HIP;
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, e0, e1);
    const double r = (double)bytes * iters / (ms * 1e6);
    if (rep > 0 && r > best) best = r;
  }
  (void)hipEventDestroy(e0); (void)hipEventDestroy(e1);
  *gbps = best;
  return BPD_OK;
}

int bpd_measure_mfma_bf16(void* scratch_dev, void* hip_stream, int iters, double* tflops) {
  if (!scratch_dev || !tflops || iters < 1) return BPD_E_ARG;
  hipStream_t s = (hipStream_t)hip_stream;
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) return BPD_E_HIP;
  int dev = 0, cus = 0;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  const int wgs = 2 * cus;                     // two 4-wave workgroups per CU: two waves per SIMD
  double best = 0;
  for (int rep = 0; rep < 3; ++rep) {
    (void)hipEventRecord(e0, s);
    hipLaunchKernelGGL(peak_mfma_kernel, dim3(wgs), dim3(256), 0, s, (float*)scratch_dev, iters, 1u + rep);
    (void)hipEventRecord(e1, s);
    if (hipStreamSynchronize(s) != hipSuccess) return BPD_E_HIP;
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, e0, e1);
    const double r = (double)wgs * 4 * iters * 16 * 16384.0 / (ms * 1e9);
    if (rep > 0 && r > best) best = r;
  }
  (void)hipEventDestroy(e0); (void)hipEventDestroy(e1);
  *tflops = best;
  return BPD_OK;
}

}  // extern "C"
