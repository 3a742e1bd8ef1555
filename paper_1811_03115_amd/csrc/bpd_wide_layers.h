// All decoder layers of a block of up to 16 rows as one kernel on the whole chip (bf16, d = 1024, d_ff = 4096, 64-wide heads).  Included by
// bpd_kernels.h, after bpd_layers.h, whose division of a workgroup into compute and helper waves it shares.
//
// A layer of this shape has 29 MB of weights, more than one XCD streams in the time that the chain of operators takes (25 us at 1.2 TB/s), so all
// XCDs work on one block: 256 members, one per CU, hold a layer's weights in their registers, fetched while they have no part in
// an operator, and hand the block over between XCDs: results are written through to memory (sc1), read past the L1, and tell by themselves that they have come
// (EMPTY_WORD, as in bpd_layers.h).  (With flags, gathered by one member of each XCD and passed on to all, six layers of one row took 120 us instead of 101, of ten
// rows 151 instead of 137.)  Flags remain where the block's keys and values lie among older ones, inside an XCD, and to tell once that everybody has emptied what it
// writes.  What bounds a hand-over of more rows is traffic: whoever waits asks memory again and again, and 256 members that fetch 40 KB a round to
// normalise it are slower than ten waves per XCD that fetch a row each and hand 20 KB on inside the XCD.
//
// Places.  Place 32 x + r is that of member r on XCD x:  every place has a tile of the first FFN layer;  r < 8: one of the second;  r >= 8:
// one of the queries, keys and values, those of heads 2 x and 2 x + 1, whose self-attention is with places r >= 24 of the same XCD (so that
// this hand-over stays inside it: plain stores, local flags);  8 .. 15, 16 .. 23: output projections of the self- and the cross-attention;  24 ..:
// cross-attention, beside the self-attention where there is room.
//
// Six layers of 10 rows, 20 .. 120 keys, 27 source tokens: 132 us (as a chain of 60 kernels some 200), of one row 101.  What bounds it is the hand-over, six times a layer
// between XCDs: 0.5 .. 0.8 us until a result is seen elsewhere, a round of asking (0.7), another for all of the input; then the input's
// staging and 0.7 us from there to the stores.
//
// Members register as in bpd_layers.h.  The first on each XCD closes its list when 32 have come or LK_CLOSE_TICKS have passed, and tells all XCDs
// how many there are; an XCD where nobody has come is closed by others.  Fewer than 256 members share the places out, fetch weights as
// they go and hand everything over through memory (six layers of 10 rows by members per XCD, by events, us: 32 135, 31 155, 16 220, 8 357; seven XCDs of 32 308, which includes
// 60 until the eighth is given up (288 when flags were polled: whoever normalises all rows asks memory for them, round after round); bpd_tall_layers.h, 40 rows: 181, 360, 370, 559; 454).
#pragma once

constexpr int WK_HOLD = 40, WK_GAP = 1;           // pauses of the compute waves, as LK_HOLD and LK_GAP (hold 12 .. 64: within 1 us of each other at 1 x 1, 1 x 10, 5 x 8, 8 x 8 and 16 x 4 rows)
// Blocks of more rows than this share what is normalised: see stage_norm (128 tokens of ten rows a step: 5.1 ms, 5.5 with every member normalising all; greedy: 5.0 ms,
// 5.2 shared)
constexpr int WK_ROWS_ALONE = 4;
constexpr int WK_XCDS = 8, WK_CENSUS = 32, WK_GLOBAL = 64, WK_LOCAL = 96, WK_NORM = 224, WK_AREA = 288;      // words of an XCD's area: [0] registered; members of each XCD; its operators done; flags [wave][member]; flags of the rows that its waves normalise (tall_layers_kernel)
static_assert(WK_XCDS * WK_AREA <= LK_WORDS, "both kernels count in the same words");

__device__ __forceinline__ void wk_store4(unsigned* p, unsigned v) { asm volatile("global_store_dword %0, %1, off sc1" ::"v"(p), "v"(v) : "memory"); }
__device__ __forceinline__ void wk_store8(void* p, u32x2 v) { asm volatile("global_store_dwordx2 %0, %1, off sc1" ::"v"(p), "v"(v) : "memory"); }
// (more than 64 bits: two wait states until an instruction may write the data registers, which the compiler cannot see to here)
__device__ __forceinline__ void wk_store16(void* p, f32x4 v) { asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory"); }
__device__ __forceinline__ void wk_store2(bf16_t* p, unsigned v) { asm volatile("global_store_short %0, %1, off sc1" ::"v"(p), "v"(v) : "memory"); }

// LayerNorm of up to 16 rows of 1024 into LDS as bf16, rows 1032 apart; wave hw takes rows hw, hw + 4, ..
template <int N>
__device__ __forceinline__ void wk_norm_rows(const rsrc_t& xr, int rows, const f32x4 (&g)[4], const f32x4 (&b)[4], float eps, bf16_t* xs, int hw, int lane, LkPoll poll) {
  constexpr int D = 1024;
  f32x4 v[N][4];
  poll.first<4>(xr, hw * D * 4, lane);
  poll([&] {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int h = 0; h < 4; ++h) v[i][h] = __builtin_bit_cast(f32x4, lk_load16(xr, ((hw + 4 * i) * D + h * 256 + lane * 4) * 4));
    __builtin_amdgcn_sched_barrier(0);
    unsigned top = 0;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int h = 0; h < 4; ++h) top = lk_top(top, __builtin_bit_cast(u32x4, v[i][h]));
    return top;
  });
  float mu[N], q[N];
#pragma unroll
  for (int i = 0; i < N; ++i) { const f32x4 s = (v[i][0] + v[i][1]) + (v[i][2] + v[i][3]); mu[i] = (s[0] + s[1]) + (s[2] + s[3]); }
#pragma unroll
  for (int i = 0; i < N; ++i) mu[i] = wave_sum(mu[i]) * (1.f / D);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      v[i][h] -= mu[i];
#pragma unroll
      for (int r = 0; r < 4; ++r) s[r] = fmaf(v[i][h][r], v[i][h][r], s[r]);
    }
    q[i] = (s[0] + s[1]) + (s[2] + s[3]);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) q[i] = wave_sum(q[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float rs = inv_sqrt(fmaf(q[i], 1.f / D, eps));
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      f32x4 y;
#pragma unroll
      for (int r = 0; r < 4; ++r) y[r] = fmaf(v[i][h][r] * rs, g[h][r], b[h][r]);
      if (hw + 4 * i < rows) *(u32x2*)(xs + (hw + 4 * i) * (D + 8) + h * 256 + lane * 4) = u32x2{cvt_pk_bf16(y[0], y[1]), cvt_pk_bf16(y[2], y[3])};
    }
  }
}
// One row: the same for a wave that holds it (columns 256 h + 4 lane ..); store(h, bf16 of these)
template <class Store>
__device__ __forceinline__ void wk_norm_row(f32x4 (&v)[4], const f32x4 (&g)[4], const f32x4 (&b)[4], float eps, Store&& store) {
  constexpr int D = 1024;
  const f32x4 t = (v[0] + v[1]) + (v[2] + v[3]);
  const float mu = wave_sum((t[0] + t[1]) + (t[2] + t[3])) * (1.f / D);
  f32x4 q = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    v[h] -= mu;
#pragma unroll
    for (int r = 0; r < 4; ++r) q[r] = fmaf(v[h][r], v[h][r], q[r]);
  }
  const float rs = inv_sqrt(fmaf(wave_sum((q[0] + q[1]) + (q[2] + q[3])), 1.f / D, eps));
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    f32x4 y;
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = fmaf(v[h][r] * rs, g[h][r], b[h][r]);
    store(h, u32x2{cvt_pk_bf16(y[0], y[1]), cvt_pk_bf16(y[2], y[3])});
  }
}
__device__ __forceinline__ void wk_norm(const float* x, int rows, const f32x4 (&g)[4], const f32x4 (&b)[4], float eps, bf16_t* xs, int hw, int lane, LkPoll poll = {nullptr, nullptr, false}) {
  const rsrc_t xr = rsrc_of(x, (unsigned)rows * 1024 * 4);
  if (rows <= 4) wk_norm_rows<1>(xr, rows, g, b, eps, xs, hw, lane, poll);
  else if (rows <= 8) wk_norm_rows<2>(xr, rows, g, b, eps, xs, hw, lane, poll);
  else if (rows <= 12) wk_norm_rows<3>(xr, rows, g, b, eps, xs, hw, lane, poll);
  else { wk_norm_rows<2>(xr, rows, g, b, eps, xs, hw, lane, poll); wk_norm_rows<2>(xr, rows, g, b, eps, xs, hw + 8, lane, poll); }         // (registers)
}

enum { WK_QKV, WK_SELF, WK_O, WK_CROSS, WK_CO, WK_UP, WK_DOWN };
struct WkMember {
  int place, members, slots, rows;               // rows of the block
  bool full;                                     // 256 members
  int xcd, rank, here; unsigned xcds;            // where it runs: XCD, rank and members there; XCDs with members
  // The places' parts (-1: none)
  __device__ __forceinline__ static int tile(int op, int place) {
    const int x = place >> 5, r = place & 31;
    if (op == WK_QKV) return r < 8 ? -1 : ((r - 8) >> 3) * 64 + x * 8 + ((r - 8) & 7);
    if (op == WK_UP) return place;
    const int first = op == WK_DOWN ? 0 : (op == WK_O ? 8 : 16);
    return r < first || r >= first + 8 ? -1 : x * 8 + r - first;
  }
  __device__ __forceinline__ int cross_first() const { return slots <= 2 ? 2 * slots : 0; }
  // attention: (slot, head) as slot * 16 + head
  __device__ __forceinline__ int item(int op, int place) const {
    const int x = place >> 5, k = ((place & 31) - 24 - (op == WK_CROSS ? cross_first() : 0)) & 31;
    return k < 2 * slots ? (k >> 1) * 16 + 2 * x + (k & 1) : -1;
  }
};

struct WkHelper {
  static constexpr int D = 1024, F = 4096, H = 16;
  bf16_t* xs;
  f32x4* red;
  AttnLds sm;
  u32x2* q_s;
  int hw;
  WkMember j;
  int key, sb;                                   // of row lr: its row in the cache, its sequence
  unsigned op = 0;
  bool broken = false;
  unsigned ahead[8];                             // fetch_ahead()
  bool fetched = false;

  __device__ __forceinline__ unsigned* area() const { return lk_args().sync + j.xcd * WK_AREA; }
  // (One piece first where a wait for everything would be 20 .. 80 KB a member, out of memory, round after round: 128 tokens of ten rows a step 5.1 ms, 5.5 without,
  // and 5.3 if all ask for the same piece.)
  __device__ __forceinline__ LkPoll poll(bool on = true) { return LkPoll{&broken, lk_args().error, on, j.rows > WK_ROWS_ALONE ? j.rank : -1}; }
  // Operator `target` is done everywhere
  __device__ __forceinline__ void wait(unsigned target) {
    if (broken || target == 0) return;
    const int lane = lk_lane();
    const unsigned* g = area() + WK_GLOBAL + (lane & 7);
    const bool of = j.xcds >> (lane & 7) & 1;
#pragma unroll 1
    for (int s = 0; s < LK_SPINS; ++s) {
      const unsigned v = lk_load(g);
      if (__all(!of || v >= target)) return;
    }
    broken = true;
    if (lane == 0) *lk_args().error = 1;
  }
  // This wave's part of the operator is in memory; a member of the XCD passes it on when all members' parts are: those of waves < NF of members from ..
  // from + count - 1 (not full: of all waves of all)
  template <int NF>
  __device__ __forceinline__ void done(bool mine, int from, int count, bool pass_on) {
    const int lane = lk_lane();
    unsigned* flags = area() + WK_LOCAL;
    if (!j.full || (mine && hw < NF)) lk_raise(flags + hw * 32 + j.rank, op, lane);
    if (hw != 3 || j.rank != 0 || !(pass_on || !j.full)) return;
    if (j.full) lk_wait<NF>(flags, op, from, count, lane, broken, lk_args().error);
    else lk_wait<4>(flags, op, 0, j.here, lane, broken, lk_args().error);
    if (lane < WK_XCDS) wk_store4(lk_args().sync + lane * WK_AREA + WK_GLOBAL + j.xcd, op);
  }
  __device__ __forceinline__ f32x4 partial_sums(int tiles, int t, int lane) const {
    f32x4 part[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) part[w] = red[(w * tiles + t) * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
    return ((part[0] + part[1]) + part[2]) + part[3];
  }
  __device__ __forceinline__ static void load_norm(const float* ln, f32x4 (&g)[4], f32x4 (&b)[4], int lane) {
#pragma unroll
    for (int h = 0; h < 4; ++h) { g[h] = *(const f32x4*)(ln + h * 256 + lane * 4); b[h] = *(const f32x4*)(ln + D + h * 256 + lane * 4); }
  }

  // Columns col .. col + 3 of a row of queries (c = 0; lo: D columns on), keys (1) or values (2): within the XCD, or (not full) to memory
  __device__ __forceinline__ void store_qkv(int l, int c, int col, int row, f32x4 v) const {
    const LayersP& p = lk_args();
    if (c == 0) {
      u32x2 hi, lo;
      lk_halves(v * p.scale, hi, lo);
      bf16_t* q = p.q + (size_t)row * (2 * D) + col;
      if (j.full) { *(u32x2*)q = hi; *(u32x2*)(q + D) = lo; }
      else { wk_store8(q, hi); wk_store8(q + D, lo); }
    } else if (sb >= 0) {
      const unsigned lo = cvt_pk_bf16(v[0], v[1]), hi = cvt_pk_bf16(v[2], v[3]);
      bf16_t* cache = (c == 1 ? p.selfK : p.selfV) + l * p.self_layer;
      if (j.full) kv_frag_store(cache, c == 2, sb, H, p.self_groups, key, col, lo, hi);
      else {
        bf16_t* dst = cache + ((size_t)sb * H + (col >> 6)) * p.self_groups * KV_GROUP;
        if (c == 1) wk_store8(dst + k_frag_at(key, col & 63), u32x2{lo, hi});
        else { dst += v_frag_at(key, col & 63); wk_store2(dst, lo); wk_store2(dst + 8, lo >> 16); wk_store2(dst + 16, hi); wk_store2(dst + 24, hi >> 16); }
      }
    }
  }

  // Buffers of what is handed over, two of each, which the layers use in turn: the residual stream behind the attentions (stage 1, 2) and between layers (3),
  // the attentions' results, the hidden layer.
  __device__ __forceinline__ static float* between(int stage, int l) { return lk_args().x1 + ((stage - 1) * 2 + (l & 1)) * (16 * D); }
  __device__ __forceinline__ static float* stream(int l, int stage) {
    const LayersP& p = lk_args();
    if (stage == 0) return l == 0 ? p.x : between(3, l - 1);
    return stage == 3 && l + 1 == p.n_layers ? p.x : between(stage, l);
  }
  __device__ __forceinline__ static bf16_t* heads(int which, int l) { return lk_args().attn + ((which == WK_CROSS ? 2 : 0) + (l & 1)) * (16 * D); }
  __device__ __forceinline__ static bf16_t* hidden(int l) { return lk_args().ffh + (l & 1) * (16 * F); }
  // Normalised rows of an XCD, for QKV and UP: each row by a wave of one member (hw 3 of member 8 + row), who hands it on inside the XCD
  __device__ __forceinline__ bool shared(int op, int l) const { return j.full && j.rows > WK_ROWS_ALONE && !(op == WK_QKV && l == 0); }
  __device__ __forceinline__ bf16_t* normed(int op, int l) const { return lk_args().xn + (size_t)((j.xcd * 2 + (op == WK_UP ? 1 : 0)) * 2 + (l & 1)) * (16 * D); }
  __device__ __forceinline__ int norm_of() const { return hw == 3 && j.rank >= 8 && j.rank - 8 < j.rows ? j.rank - 8 : -1; }
  __device__ __forceinline__ void empty_normed(int op, int l, int lane) const {
    const int m = norm_of();
    if (!j.full || m < 0) return;
#pragma unroll
    for (int h = 0; h < 4; ++h) *(u32x2*)(normed(op, l) + m * D + h * 256 + lane * 4) = u32x2{EMPTY_WORD, EMPTY_WORD};
  }
  __device__ __forceinline__ void stage_norm(int op, int l, const float* in, const f32x4 (&g)[4], const f32x4 (&b)[4], int lane) {
    const LayersP& p = lk_args();
    if (!shared(op, l)) { wk_norm(in, j.rows, g, b, p.eps, xs, hw, lane, poll(op != WK_QKV || l > 0)); return; }
    const int m = norm_of();
    if (m >= 0) {
      const rsrc_t xr = rsrc_of(in, (unsigned)j.rows * D * 4);
      f32x4 v[4];
      LkPoll{&broken, p.error, true}([&] {
        unsigned top = 0;
#pragma unroll
        for (int h = 0; h < 4; ++h) v[h] = __builtin_bit_cast(f32x4, lk_load16(xr, (m * D + h * 256 + lane * 4) * 4));
#pragma unroll
        for (int h = 0; h < 4; ++h) top = lk_top(top, __builtin_bit_cast(u32x4, v[h]));
        return top;
      });
      wk_norm_row(v, g, b, p.eps, [&](int h, u32x2 w) { *(u32x2*)(normed(op, l) + m * D + h * 256 + lane * 4) = full_words(w); });
    }
    lk_copy<D>(normed(op, l), j.rows, xs, hw, lane, poll());
  }
  // They are emptied (EMPTY_WORD) by who writes them, a layer after that, when all are known to have read them, and ahead of an operator of the writer's that
  // the next readers wait for: QKV for CO's results, UP for all others.
  __device__ __forceinline__ void empty_tile(float* x, int tile, int lane) const {
    const int lr = lane & 15;
    const float e = __uint_as_float(EMPTY_WORD);
    if (hw == 0 && tile >= 0 && lr < j.rows) wk_store16(x + (size_t)lr * D + tile * 16 + (lane >> 4) * 4, f32x4{e, e, e, e});
  }
  __device__ __forceinline__ void rows_of_head(bf16_t* attn, int item, unsigned with, int lane) const {
    const LayersP& p = lk_args();
    const int lr = lane & 15;
    if (item >= 0 && lr < p.R) wk_store8(attn + (size_t)((item >> 4) * p.R + lr) * D + (item & 15) * 64 + hw * 16 + (lane >> 4) * 4, u32x2{with, with});
  }
  __device__ __forceinline__ void empty_hidden(int l, int place, int lane) const {
    const int lr = lane & 15;
    if (hw == 0 && lr < j.rows) wk_store8(hidden(l) + (size_t)lr * F + place * 16 + (lane >> 4) * 4, u32x2{EMPTY_WORD, EMPTY_WORD});
  }
  // What place writes, both buffers of everything: ahead of the first hand-over, nothing is assumed of what they hold
  __device__ __forceinline__ void empty_all(int lane) const {
    for (int l = 0; l < 2; ++l) { empty_normed(WK_QKV, l, lane); empty_normed(WK_UP, l, lane); }
#pragma unroll 1
    for (int place = j.place; place < 256; place += j.members)
#pragma unroll 1
      for (int l = 0; l < 2; ++l) {
        empty_tile(between(1, l), WkMember::tile(WK_O, place), lane); empty_tile(between(2, l), WkMember::tile(WK_CO, place), lane);
        empty_tile(between(3, l), WkMember::tile(WK_DOWN, place), lane); empty_hidden(l, place, lane);
        rows_of_head(heads(WK_SELF, l), j.item(WK_SELF, place), EMPTY_WORD, lane); rows_of_head(heads(WK_CROSS, l), j.item(WK_CROSS, place), EMPTY_WORD, lane);
      }
  }

  template <int OP, int K>
  __device__ __forceinline__ void product(int l) {
    constexpr bool LN = OP == WK_QKV || OP == WK_UP, BIAS = OP == WK_UP || OP == WK_DOWN, RES = !LN;
    const LayersP& p = lk_args();
    const int lane = lk_lane(), lr = lane & 15, lq = lane >> 4;
    if constexpr (OP == WK_QKV) ++op;
    bool staged = false;
#pragma unroll 1
    for (int place = j.place; place < 256; place += j.members) {
      const int tile = WkMember::tile(OP, place);
      if (tile < 0) continue;
      const int n = tile * 16 + lq * 4;
      f32x4 bs, res;
      if constexpr (BIAS) if (hw == 0) bs = *(const f32x4*)((const float*)((const char*)(OP == WK_UP ? p.b1 : p.b2) + l * p.stride) + n);
      float* const in = stream(l, OP == WK_QKV || OP == WK_O ? 0 : (OP == WK_CO ? 1 : 2));        // LN: the rows; otherwise what the result is added to
      const rsrc_t rr = rsrc_of(in, (unsigned)j.rows * D * 4);
      f32x4 g[4], b[4];
      if constexpr (LN) if (!staged) load_norm((const float*)((const char*)(OP == WK_QKV ? p.ln1 : p.ln3) + l * p.stride), g, b, lane);
      if (!staged && OP != WK_QKV && OP != WK_DOWN && l == 0) wait(1);         // (everybody has emptied what it writes)
      if constexpr (RES) if (hw == 0) res = __builtin_bit_cast(f32x4, lk_load16(rr, (lr * D + n) * 4));
      if (!staged) {
        if constexpr (LN) stage_norm(OP, l, in, g, b, lane);
        else if constexpr (OP == WK_DOWN) lk_copy<F>(hidden(l), j.rows, xs, hw, lane, poll());
        else lk_copy<D>(heads(OP == WK_O ? WK_SELF : WK_CROSS, l), j.rows, xs, hw, lane, poll());
      }
      lk_barrier();                              // the input is staged, the partial sums of the place before are read
      if constexpr (OP == WK_QKV) {
        if (j.full) fetch_ahead(l, j.item(WK_SELF, place));
        if (l > 0) empty_normed(WK_UP, l - 1, lane);
        if (l > 0) empty_tile(between(2, l - 1), WkMember::tile(WK_CO, place), lane);          // (x3 of the layer before is there: DOWN and UP have read x2)
        else if (j.full) { empty_all(lane); lk_stores_done(); }
      }
      if constexpr (OP == WK_UP) {               // (x2 is there: CO has read x1 and the cross-attention's results, O the self-attention's and x3)
        empty_normed(WK_QKV, l, lane);
        empty_tile(between(1, l), WkMember::tile(WK_O, place), lane);
        rows_of_head(heads(WK_SELF, l), j.item(WK_SELF, place), EMPTY_WORD, lane); rows_of_head(heads(WK_CROSS, l), j.item(WK_CROSS, place), EMPTY_WORD, lane);
        if (l > 0) { empty_tile(between(3, l - 1), WkMember::tile(WK_DOWN, place), lane); empty_hidden(l - 1, place, lane); }
      }
      // (the cross-attention has read all of x1, but this wave may have asked too early; x2 and x3 it has read itself)
      if constexpr (OP == WK_CO) if (hw == 0) poll()([&] {
        if (__any(lk_top(0, __builtin_bit_cast(u32x4, res)) == EMPTY_WORD)) res = __builtin_bit_cast(f32x4, lk_load16(rr, (lr * D + n) * 4));
        return lk_top(0, __builtin_bit_cast(u32x4, res));
      });
      lk_barrier();                              // the partial sums are there
      staged = true;
      if (hw > 0) continue;
      f32x4 v = partial_sums(1, 0, lane);
      if (lr >= j.rows) continue;
      if constexpr (OP == WK_QKV) {
        store_qkv(l, tile >> 6, n - (tile >> 6) * D, lr, v);
      } else if constexpr (OP == WK_UP) {
        v += bs;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.f);
        wk_store8(hidden(l) + (size_t)lr * F + n, full_words(u32x2{cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3])}));
      } else {
        if constexpr (BIAS) v += bs;
        v += res;
        wk_store16(stream(l, OP == WK_O ? 1 : (OP == WK_CO ? 2 : 3)) + (size_t)lr * D + n, __builtin_bit_cast(f32x4, full_words(v)));
      }
    }
    if constexpr (OP == WK_QKV) {
      if (l == 0) done<1>(true, 0, 32, true);      // (that everything is empty: to all)
      else done<1>(staged, 8, 24, false);
    }
  }

  __device__ __forceinline__ static AttnP attn_args(bool self) {
    const LayersP& p = lk_args();
    AttnP a{};
    a.capg = self ? p.self_groups : p.src_groups;
    a.d = D; a.R = p.R; a.nsplit = 1; a.causal = self;
    a.local_q = self ? p.local_q : 0; a.local_m = p.local_m;
    return a;
  }
  __device__ __forceinline__ static int sequence(int slot) { const LayersP& p = lk_args(); return p.seq ? lk_const(p.seq, slot) : slot; }

  // Up to 128 keys: a group of 32 per wave
  __device__ __forceinline__ static bool few(int slot) {
    const LayersP& p = lk_args();
    const int lim = lk_const(p.base, slot);
    return ((lim + p.R + 31) >> 5) - (attn_first_key(attn_args(true), lim) >> 5) <= 4;
  }
  // As LkHelper::fetch_ahead: by a wave that stores no queries, keys and values (only where this XCD writes the block's own among them)
  __device__ __forceinline__ void fetch(const rsrc_t& kr, const rsrc_t& vr, int first, int lane) {
    if (hw != 3) return;
#pragma unroll
    for (int i = 0; i < 8; ++i) ahead[i] = __builtin_amdgcn_raw_buffer_load_b32(i < 4 ? kr : vr, lane * 128, (first + 2 * (i & 3)) * (KV_GROUP * 2), 16);
  }
  __device__ __forceinline__ void fetch_ahead(int l, int item) {
    if (item < 0) return;
    const LayersP& p = lk_args();
    const int slot = item >> 4, s = sequence(slot), lim = lk_const(p.base, slot), held = (lim + p.R + 31) >> 5, groups = held < p.self_groups ? held : p.self_groups;
    const size_t at = l * p.self_layer + ((size_t)(s < 0 ? 0 : s) * H + (item & 15)) * p.self_groups * KV_GROUP;
    fetch(rsrc_of(p.selfK + at, (unsigned)groups * (KV_GROUP * 2)), rsrc_of(p.selfV + at, (unsigned)groups * (KV_GROUP * 2)), attn_first_key(attn_args(true), lim) >> 5, lk_lane());
    fetched = true;
  }
  template <int NF, int STORE>
  __device__ __forceinline__ void self_item(int l, int item, unsigned after, bf16_t* out, bool first_item) {
    if (few(item >> 4)) self_groups<1, NF, STORE>(l, item, after, out, first_item); else self_groups<2, NF, STORE>(l, item, after, out, first_item);
  }
  template <int G, int NF, int STORE>
  __device__ __forceinline__ void self_groups(int l, int item, unsigned after, bf16_t* out, bool first_item) {
    const LayersP& p = lk_args();
    const int lane = lk_lane(), lr = lane & 15, lq = lane >> 4;
    const int h = item & 15, slot = item >> 4, s = sequence(slot);
    const AttnP a = attn_args(true);
    const int lim = lk_const(p.base, slot), held = (lim + p.R + 31) >> 5, groups = held < p.self_groups ? held : p.self_groups;
    const int first = attn_first_key(a, lim) >> 5;
    const size_t at = l * p.self_layer + ((size_t)(s < 0 ? 0 : s) * H + h) * p.self_groups * KV_GROUP;
    const rsrc_t kr = rsrc_of(p.selfK + at, (unsigned)groups * (KV_GROUP * 2)), vr = rsrc_of(p.selfV + at, (unsigned)groups * (KV_GROUP * 2));
    const rsrc_t qr = rsrc_of(p.q + (size_t)slot * p.R * (2 * D), (unsigned)p.R * (4 * D));
    if (!first_item) {
      lk_barrier();                              // the results of the item before are out of LDS
    } else if (j.full && NF == 4) {              // (all four waves store queries, keys and values)
      unsigned t[G];
#pragma unroll
      for (int g = 0; g < G; ++g) t[g] = __builtin_amdgcn_raw_buffer_load_b32(lane < 32 ? kr : vr, (lane & 31) * 128, (first + hw + g * 4) * (KV_GROUP * 2), 16);
      lk_wait<NF>(area() + WK_LOCAL, after, 8, 24, lane, broken, p.error);
#pragma unroll
      for (int g = 0; g < G; ++g) asm volatile("" ::"v"(t[g]));
    } else if (j.full) {
      if (!fetched) fetch(kr, vr, first, lane);
      lk_wait<NF>(area() + WK_LOCAL, after, 8, 24, lane, broken, p.error);
      if (hw == 3)
#pragma unroll
        for (int i = 0; i < 8; ++i) asm volatile("" ::"v"(ahead[i]));
      fetched = false;
    } else {
      wait(after);
    }
    if (s < 0) {                                 // (rows of nobody; a barrier as the attention's own)
      if (STORE == ATTN_THROUGH_WORDS) rows_of_head(out, item, 0, lane);
      lk_barrier();
      return;
    }
    const unsigned off = lr * (4 * D) + (h * 64 + 8 * lq) * 2;
    bf16x8 qhi[2], qlo[2];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      qhi[s2] = __builtin_bit_cast(bf16x8, lk_load16(qr, off + s2 * 64));
      qlo[s2] = __builtin_bit_cast(bf16x8, lk_load16(qr, off + s2 * 64 + 2 * D));
    }
    u32x4 kf[G][4], vf[G][4];
    attn_load_kv<false, G>(kr, vr, first + hw, 4, lane, kf, vf);
    __builtin_amdgcn_sched_barrier(0);
    attention_mfma_core<false, true, G == 2 ? -1 : 0, G, STORE>(a, sm, h, slot, 0, 0, 0, p.R, H, 1, hw * 64 + lane, 4, first, 4 * G, kr, vr, kf, vf, qhi, qlo, lim, out);
  }
  __device__ __forceinline__ void self_attention(int l) {
    bool mine = false;
#pragma unroll 1
    for (int place = j.place; place < 256; place += j.members) {
      const int item = j.item(WK_SELF, place);
      if (item < 0) continue;
      self_item<1, ATTN_THROUGH_WORDS>(l, item, op, heads(WK_SELF, l), !mine);
      mine = true;
    }
  }
  template <int STORE>
  __device__ __forceinline__ void cross_item(int l, int item, const float* x, unsigned after, LkPoll poll, bf16_t* out, bool first_item) {
    const LayersP& p = lk_args();
    const int lane = lk_lane(), lr = lane & 15, lq = lane >> 4;
    const AttnP a = attn_args(false);
    const int h = item & 15, slot = item >> 4, s = sequence(slot);
    const size_t at = l * p.src_layer + ((size_t)(s < 0 ? 0 : s) * H + h) * p.src_groups * KV_GROUP;
    const rsrc_t kr = rsrc_of(p.crossK + at, (unsigned)p.src_groups * (KV_GROUP * 2)), vr = rsrc_of(p.crossV + at, (unsigned)p.src_groups * (KV_GROUP * 2));
    u32x4 kf[1][4], vf[1][4];
    f32x4 g[4], b[4];
    load_norm((const float*)((const char*)p.ln2 + l * p.stride), g, b, lane);
    attn_load_kv<false, 1>(kr, vr, hw, 4, lane, kf, vf);
    const int lim = lk_const(p.src_len, slot);
    if (first_item) wait(after);
    else lk_barrier();                         // the results of the item before are out of LDS
    wk_norm(x + (size_t)slot * p.R * D, p.R, g, b, p.eps, xs, hw, lane, poll);
    lk_barrier();
    lk_barrier();
    {
      u32x2 hi, lo;
      lk_halves(partial_sums(4, hw, lane) * p.scale, hi, lo);
      // operand lane 16 q + lr of half s holds columns 32 s + 8 q .. + 7
      const int to = ((hw >> 1) * 64 + ((hw & 1) * 2 + (lq >> 1)) * 16 + lr) * 2 + (lq & 1);
      q_s[to] = hi; q_s[256 + to] = lo;
    }
    lk_barrier();
    bf16x8 qhi[2], qlo[2];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      qhi[s2] = __builtin_bit_cast(bf16x8, *(const u32x4*)&q_s[(s2 * 64 + lane) * 2]);
      qlo[s2] = __builtin_bit_cast(bf16x8, *(const u32x4*)&q_s[256 + (s2 * 64 + lane) * 2]);
    }
    if (s < 0) { if (STORE == ATTN_THROUGH_WORDS) rows_of_head(out, item, 0, lane); lk_barrier(); return; }     // (as the attention's own)
    attention_mfma_core<false, false, 0, 1, STORE>(a, sm, h, slot, 0, 0, 0, p.R, H, 1, hw * 64 + lane, 4, 0, 4, kr, vr, kf, vf, qhi, qlo, lim, out);
  }
  __device__ __forceinline__ void cross_attention(int l) {
    bool mine = false;
#pragma unroll 1
    for (int place = j.place; place < 256; place += j.members) {
      const int item = j.item(WK_CROSS, place);
      if (item < 0) continue;
      cross_item<ATTN_THROUGH_WORDS>(l, item, stream(l, 1), l == 0, poll(), heads(WK_CROSS, l), !mine);
      mine = true;
    }
  }

  __device__ __forceinline__ void run() {
    const int layers = lk_args().n_layers;
    {
      const LayersP& p = lk_args();
      const int lr = lk_lane() & 15, m = lr < j.rows ? lr : 0, slot = m / p.R;
      sb = p.seq ? p.seq[slot] : slot;
      key = p.base[slot] + m - slot * p.R;
    }
    if (!j.full || j.rank < 8) {                 // (the others: in the first operator, which these have no part in)
      empty_all(lk_lane());
      lk_stores_done();
    }
#pragma unroll 1
    for (int l = 0; l < layers; ++l) {
      product<WK_QKV, D>(l);
      self_attention(l);
      product<WK_O, D>(l);
      cross_attention(l);
      product<WK_CO, D>(l);
      product<WK_UP, D>(l);
      product<WK_DOWN, F>(l);
    }
  }
};

struct WkCompute {
  const bf16_t* xs;
  f32x4* red;
  int cw;
  WkMember j;
  u32x4 aq[1][8], a1[1][8], ax[4][8];            // ax: an output projection (its first tile), the head's queries, or the second FFN layer (one tile)

  template <int PACE = 0, int N, int U> __device__ __forceinline__ void load(u32x4 (&a)[N][U], const char* LayersP::*w, int l, int tile) {
    const LayersP& p = lk_args();
    lk_weights<PACE>(a, p.*w + l * p.stride, tile, cw, lk_lane());
  }
  __device__ __forceinline__ u32x4 (&one())[1][8] { return *reinterpret_cast<u32x4 (*)[1][8]>(&ax); }
  __device__ __forceinline__ u32x4 (&deep())[1][32] { return *reinterpret_cast<u32x4 (*)[1][32]>(&ax); }
  template <int OP, int U> __device__ __forceinline__ void product(u32x4 (&a)[1][U], const char* LayersP::*w, int l) {
#pragma unroll 1
    for (int place = j.place; place < 256; place += j.members) {
      const int tile = WkMember::tile(OP, place);
      if (tile < 0) continue;
      if (!j.full) load(a, w, l, tile);
      lk_barrier();
      lk_multiply<1, U>(a, xs, j.rows, red, cw, lk_lane());
      lk_barrier();
    }
  }
  __device__ __forceinline__ void run() {
    const int layers = lk_args().n_layers, r = j.place & 31;
    const bool full = j.full, self = full && j.item(WK_SELF, j.place) >= 0, cross = full && j.item(WK_CROSS, j.place) >= 0;
    const bool down = full && r < 8, qkv = full && r >= 8, o = full && r >= 8 && r < 16, co = full && r >= 16 && r < 24;
    if (full) load(a1, &LayersP::w1, 0, j.place);
    if (qkv) load(aq, &LayersP::wqkv, 0, WkMember::tile(WK_QKV, j.place));
    if (o) load(one(), &LayersP::wo, 0, WkMember::tile(WK_O, j.place));
    if (down) load(deep(), &LayersP::w2, 0, WkMember::tile(WK_DOWN, j.place));
#pragma unroll 1
    for (int l = 0; l < layers; ++l) {
      const int next = l + 1 < layers ? l + 1 : l;                   // (past the last layer: once more, read by nobody)
      product<WK_QKV>(aq, &LayersP::wqkv, l);
      if (qkv && !self) {
        __builtin_amdgcn_s_sleep(WK_HOLD);       // (the operator's own results first)
        if (cross) load<WK_GAP>(ax, &LayersP::cq, l, (j.item(WK_CROSS, j.place) & 15) * 4);
        if (co) load<WK_GAP>(one(), &LayersP::co, l, WkMember::tile(WK_CO, j.place));
        if (!o) load<WK_GAP>(aq, &LayersP::wqkv, next, WkMember::tile(WK_QKV, j.place));
      }
#pragma unroll 1
      for (int place = j.place, mine = 0; place < 256; place += j.members) {
        if (j.item(WK_SELF, place) < 0) continue;
        if (mine) lk_barrier();
        mine = 1;
        lk_barrier();
      }
      product<WK_O>(one(), &LayersP::wo, l);
      if (o || self) {
        __builtin_amdgcn_s_sleep(WK_HOLD);
        if (self && cross) load(ax, &LayersP::cq, l, (j.item(WK_CROSS, j.place) & 15) * 4);
        load<WK_GAP>(aq, &LayersP::wqkv, next, WkMember::tile(WK_QKV, j.place));
        if (o) load<WK_GAP>(one(), &LayersP::wo, next, WkMember::tile(WK_O, j.place));
      }
#pragma unroll 1
      for (int place = j.place, mine = 0; place < 256; place += j.members) {
        const int item = j.item(WK_CROSS, place);
        if (item < 0) continue;
        if (!full) load(ax, &LayersP::cq, l, (item & 15) * 4);
        if (mine) lk_barrier();
        mine = 1;
        lk_barrier();
        lk_multiply(ax, xs, lk_args().R, red, cw, lk_lane());
        lk_barrier();
        lk_barrier();
        lk_barrier();
      }
      product<WK_CO>(one(), &LayersP::co, l);
      product<WK_UP>(a1, &LayersP::w1, l);
      if (qkv) { __builtin_amdgcn_s_sleep(WK_HOLD); load<WK_GAP>(a1, &LayersP::w1, next, j.place); }
      product<WK_DOWN>(deep(), &LayersP::w2, l);
      if (down) {
        __builtin_amdgcn_s_sleep(WK_HOLD);
        load<WK_GAP>(deep(), &LayersP::w2, next, WkMember::tile(WK_DOWN, j.place));
        load<WK_GAP>(a1, &LayersP::w1, next, j.place);
      }
    }
  }
};

struct WkLds {
  static constexpr int XS = 16 * (4096 + 8) * 2, RED = 4 * 4 * 64 * 16, ATTN = 16 * (1024 + 8) * 2;      // (the attention works behind the first 16 rows of 1024)
  static constexpr int BYTES = XS + RED + 64;
  static_assert(ATTN + (int)AttnLds::BYTES + 512 * 8 <= XS && BYTES <= 160 * 1024, "LDS");
};

// Registers the workgroup: its part in j, or false if it has none
__device__ __forceinline__ bool wk_register(const LayersP& p, int* word, int wave, int lane, int xcd, WkMember& j) {
  const int group = p.group & 63, most_xcds = p.group >> 6 ? p.group >> 6 : WK_XCDS;
  unsigned* area = p.sync + xcd * WK_AREA;
  if (xcd >= most_xcds) return false;
  if (wave == 0) {
    unsigned old = 0;
    if (lane == 0) old = __hip_atomic_fetch_add(area, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    old = __builtin_amdgcn_readfirstlane(old);
    int rank = (int)(old & 0xFFFFu);
    if (rank >= group || rank >= LK_PLACES || (old & LK_CLOSED)) rank = -1;
    const long long t0 = wall_clock64();
    if (rank == 0) {
      unsigned v;
      do v = __builtin_amdgcn_readfirstlane(lk_load(area));
      while ((int)(v & 0xFFFFu) < group && wall_clock64() - t0 < LK_CLOSE_TICKS);
      if ((int)(v & 0xFFFFu) < group) {
        if (lane == 0) v = __hip_atomic_fetch_or(area, LK_CLOSED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        v = __builtin_amdgcn_readfirstlane(v);
      }
      int n = (int)(v & 0xFFFFu);
      n = n < group ? n : group;
      n = n < LK_PLACES ? n : LK_PLACES;
      if (lane < WK_XCDS) wk_store4(p.sync + lane * WK_AREA + WK_CENSUS + xcd, (unsigned)n + 1);
    }
    if (rank >= 0) {
      unsigned v = 0;
#pragma unroll 1
      for (int s = 0; s < LK_SPINS; ++s) {
        v = lk_load(area + WK_CENSUS + (lane & 7));
        if (__all(v != 0)) break;
        if (rank == 0 && wall_clock64() - t0 > 3 * LK_CLOSE_TICKS && lane < WK_XCDS && v == 0 &&
            atomicCAS(p.sync + lane * WK_AREA, 0u, LK_CLOSED) == 0u) {       // nobody there: closed (whoever comes leaves)
          for (int y = 0; y < WK_XCDS; ++y) wk_store4(p.sync + y * WK_AREA + WK_CENSUS + lane, 1u);
        }
      }
      const bool missing = !__all(v != 0);
      int n = (int)v - 1, all = 0, before = 0;
      unsigned xcds = 0;
#pragma unroll
      for (int x = 0; x < WK_XCDS; ++x) {
        const int m = __builtin_amdgcn_readlane(n, x);
        if (x < xcd) before += m;
        all += m;
        xcds |= (m > 0 ? 1u : 0u) << x;
      }
      if (lane == 0) {
        word[1] = all; word[2] = before + rank; word[3] = __builtin_amdgcn_readlane(n, xcd); word[4] = (int)xcds;
        if (missing) *p.error = 1;
      }
      if (missing) rank = -1;
    }
    if (lane == 0) word[0] = rank;
  }
  lk_barrier();
  j.rank = __builtin_amdgcn_readfirstlane(word[0]);
  if (j.rank < 0) return false;
  j.members = __builtin_amdgcn_readfirstlane(word[1]); j.place = __builtin_amdgcn_readfirstlane(word[2]);
  j.here = __builtin_amdgcn_readfirstlane(word[3]); j.xcds = (unsigned)__builtin_amdgcn_readfirstlane(word[4]);
  j.xcd = xcd; j.full = j.members == WK_XCDS * LK_PLACES;
  j.slots = p.slots; j.rows = p.slots * p.R;
  return true;
}

__global__ __launch_bounds__(512, 2) void wide_layers_kernel(LayersP p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lk_smem[];
  bf16_t* xs = (bf16_t*)lk_smem;
  f32x4* red = (f32x4*)(lk_smem + WkLds::XS);
  unsigned char* attn = lk_smem + WkLds::ATTN;
  u32x2* q_s = (u32x2*)(attn + AttnLds::BYTES);
  int* word = (int*)(lk_smem + WkLds::XS + WkLds::RED);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int xcd = __builtin_amdgcn_readfirstlane((int)lk_xcd());
  WkMember j;
  if (!wk_register(p, word, wave, lane, xcd, j)) return;
  if (wave >= 4) {
    WkCompute c{xs, red, wave - 4, j};
    c.run();
  } else {
    __builtin_amdgcn_s_setprio(3);
    WkHelper h{xs, red, AttnLds::carve(attn), q_s, wave, j, 0, 0};
    h.run();
  }
}
