// As bpd_wide_layers.h, for blocks of 17 .. 64 rows of up to 16 slots: MT = 2 .. 4 MFMA row tiles.  Included by bpd_kernels.h behind it.
//
// With one row tile every member normalises all rows of an operator's input itself, which costs 0.42 us a row and wave: here a wave has
// one row, and the XCD's waves hand their rows on inside the XCD (every XCD normalises all rows: a hand-over between XCDs
// costs more than the row).  The second FFN layer (four times as long as the others) is split over K among four members per tile, all 256 of
// them: each multiplies 1024 of 4096, as everywhere else, so that one staging buffer of 16 MT x 1024 holds any input; the LayerNorm that follows adds the
// four slices, and so does ln_row_kernel behind the last layer.  Since every XCD reads the residual stream that this LayerNorm writes, two
// buffers of it take turns; the last layer's is LayersP::x.
//
// Six layers of 40 rows in five slots: 264 us as a chain of 60 kernels, 187 here; of 18 rows in two slots 160, of 32 in four 170 (with MT = 3 170 and 180),
// of 56 in seven 207, of 64 in four 222, in sixteen 240 (chain: 280 .. 300).  It is bound as the other is, by eight hand-overs a layer, the two of
// normalised rows inside the XCD (0.6 us), and by staging 2 KB a row for each operator (40 rows: 0.9 .. 1.4 us).
//
// Places.  r < 8: no queries, keys and values, but the cross-attention's first eight heads of an XCD, 24 .. 31: the self-attention's (the
// other way round for more; from nine slots on two heads or more per place); 8 .. 15, 16 .. 23: the output projections; every place has a tile of the first FFN layer and one K slice of a tile of the second.
#pragma once

constexpr int TK_ROWS = TALL_LAYERS_ROWS;        // rows of the XCD's copies of normalised rows
constexpr int WK_NORM = WK_HEADS;                // flags of the rows that the XCD's waves normalise (the heads' words are free: eight slots do not use them)
enum { TK_DOWN = WK_DOWN };

struct TkPlaces {
  // Attention: items k = order, order + 16, .. < 2 slots of the place's XCD are a place's (one head's), -1: none
  __device__ __forceinline__ static int order(int op, int place) {
    const int r = place & 31;
    return r >= 8 && r < 24 ? -1 : (op == WK_SELF ? (r + 8) & 31 : (r < 8 ? r : r - 16));
  }
  // (slot, head) as slot * 16 + head
  __device__ __forceinline__ static int item(int place, int k) { return (k >> 1) * 16 + 2 * (place >> 5) + (k & 1); }
  __device__ __forceinline__ static bool any(int op, int place, int slots) { const int k = order(op, place); return k >= 0 && k < 2 * slots; }
  // the members of an XCD that have one
  __device__ __forceinline__ static unsigned mask(int op, int slots) {
    const int n = slots < 8 ? 2 * slots : 16, a = n < 8 ? n : 8, b = n - a;
    const unsigned first = (1u << a) - 1, rest = (1u << b) - 1;
    return op == WK_SELF ? first << 24 | rest : first | rest << 24;
  }
};

template <int MT>
struct TkHelper : WkHelper {
  __device__ __forceinline__ const float* residual(int l) const { const LayersP& p = lk_args(); return (p.n_layers - 1 - l) & 1 ? p.x2 : p.x; }

  // The first NF waves of the members in the mask have done this XCD's part: its first member passes it on (not full: all waves of all)
  template <int NF>
  __device__ __forceinline__ void done(bool mine, unsigned mask, bool pass_on) {
    const int lane = lk_lane();
    unsigned* flags = area() + WK_LOCAL;
    if (!j.full || (mine && hw < NF)) lk_raise(flags + hw * 32 + j.rank, op, lane);
    if (hw != 3 || j.rank != 0 || !(pass_on || !j.full)) return;
    const int waves = j.full ? NF : 4;
    if (!j.full) mask = j.here < 32 ? (1u << j.here) - 1 : ~0u;
    const bool in = mask >> (lane & 31) & 1;
    if (!broken) {
      bool seen = false;
#pragma unroll 1
      for (int s = 0; s < LK_SPINS; ++s) {
        unsigned v0, v1;
        asm volatile("global_load_dword %0, %2, off sc1\n\tglobal_load_dword %1, %2, off offset:256 sc1\n\ts_waitcnt vmcnt(0)" : "=&v"(v0), "=&v"(v1) : "v"(flags + lane) : "memory");
        const int w = lane >> 5;
        if (__all(!in || ((w >= waves || v0 >= op) && (w + 2 >= waves || v1 >= op)))) { seen = true; break; }
      }
      if (!seen) { broken = true; if (lane == 0) *lk_args().error = 1; }
    }
    if (lane < WK_XCDS) wk_store4(lk_args().sync + lane * WK_AREA + WK_GLOBAL + j.xcd, op);
  }

  // Row m of layer l's residual stream: of its buffer or, first, what the layer before left (merge)
  __device__ __forceinline__ void load_row(int l, int m, bool merge, f32x4 (&v)[4]) {
    const LayersP& p = lk_args();
    const int lane = lk_lane();
    const float* from = merge ? (l > 0 ? residual(l - 1) : p.x) : residual(l);
    const rsrc_t xr = rsrc_of(from, (unsigned)j.rows * D * 4), pr = rsrc_of(p.part, (unsigned)j.rows * D * 16);
    f32x4 s[4][4], bias[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) v[h] = __builtin_bit_cast(f32x4, lk_load16(xr, (m * D + h * 256 + lane * 4) * 4));
    if (merge && l > 0) {
      const float* b2 = (const float*)((const char*)p.b2 + (l - 1) * p.stride);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int h = 0; h < 4; ++h) s[i][h] = __builtin_bit_cast(f32x4, lk_load16(pr, ((i * j.rows + m) * D + h * 256 + lane * 4) * 4));
#pragma unroll
      for (int h = 0; h < 4; ++h) bias[h] = *(const f32x4*)(b2 + h * 256 + lane * 4);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int h = 0; h < 4; ++h) v[h] += (((s[0][h] + s[1][h]) + s[2][h]) + s[3][h]) + bias[h];
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  __device__ __forceinline__ void keep_row(int l, int m, const f32x4 (&v)[4]) {
    float* x = (float*)residual(l) + (size_t)m * D;
#pragma unroll
    for (int h = 0; h < 4; ++h) wk_store16(x + h * 256 + lk_lane() * 4, v[h]);
  }
  __device__ __forceinline__ void norm_row(f32x4 (&v)[4], const f32x4 (&g)[4], const f32x4 (&b)[4], bf16_t* to) {
    const int lane = lk_lane();
    wk_norm_row(v, g, b, lk_args().eps, [&](int h, u32x2 w) { *(u32x2*)(to + h * 256 + lane * 4) = w; });
  }
  // Does layer l's first LayerNorm find its rows in another buffer than its own?
  __device__ __forceinline__ bool moved(int l) const { return l > 0 || residual(0) != lk_args().x; }
  // bf16 rows of 1024 (ld: bytes between them) into LDS, 1032 apart
  __device__ __forceinline__ void stage(const bf16_t* src, unsigned ld) {
    const int lane = lk_lane();
    const rsrc_t r = rsrc_of(src, (unsigned)(j.rows - 1) * ld + D * 2);
    u32x4 v[4 * MT][2];
#pragma unroll
    for (int i = 0; i < 4 * MT; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) v[i][h] = lk_load16(r, (hw + 4 * i) * ld + h * 1024 + lane * 16);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4 * MT; ++i)
      if (hw + 4 * i < j.rows) {
#pragma unroll
        for (int h = 0; h < 2; ++h) *(u32x4*)(xs + (hw + 4 * i) * (D + 8) + h * 512 + lane * 8) = v[i][h];
      }
  }
  // LayerNorm of all rows into LDS
  __device__ __forceinline__ void stage_norm(int l, const float* ln, bool merge) {
    const LayersP& p = lk_args();
    const int lane = lk_lane(), m = hw < 3 && j.rank >= 8 ? hw * 24 + j.rank - 8 : TK_ROWS;         // (full: the members with queries, keys and values)
    f32x4 g[4], b[4], v[4];
    load_norm(ln, g, b, lane);
    wait(op - 1);
    if (!j.full) {
#pragma unroll 1
      for (int r = hw; r < j.rows; r += 4) {
        load_row(l, r, merge, v);
        if (merge && moved(l) && j.place == 8 % j.members) keep_row(l, r, v);      // (place 8: the first with a tile here)
        norm_row(v, g, b, xs + r * (D + 8));
      }
      return;
    }
    bf16_t* mine = p.xn + (size_t)j.xcd * TK_ROWS * D;
    unsigned* flags = area() + WK_NORM;
    if (m < j.rows) {
      load_row(l, m, merge, v);
      norm_row(v, g, b, mine + (size_t)m * D);
      lk_raise(flags + m, op, lane);
    }
    if (!broken) {
      bool seen = false;
#pragma unroll 1
      for (int s = 0; s < LK_SPINS; ++s) {
        const unsigned v = lk_load(flags + lane);
        if (__all(lane >= j.rows || v >= op)) { seen = true; break; }
      }
      if (!seen) { broken = true; if (lane == 0) *p.error = 1; }
    }
    stage(mine, D * 2);
  }

  template <int OP>
  __device__ __forceinline__ void product(int l) {
    const LayersP& p = lk_args();
    const int lane = lk_lane(), lr = lane & 15, lq = lane >> 4, m = hw * 16 + lr;
    ++op;
    bool staged = false;
#pragma unroll 1
    for (int place = j.place; place < 256; place += j.members) {
      const int tile = OP == TK_DOWN ? place >> 2 : WkMember::tile(OP, place);
      if (tile < 0) continue;
      const int n = tile * 16 + lq * 4;
      f32x4 bs, res;
      if constexpr (OP == WK_UP) bs = *(const f32x4*)((const float*)((const char*)p.b1 + l * p.stride) + n);
      if (!staged) {
        if constexpr (OP == WK_QKV) stage_norm(l, (const float*)((const char*)p.ln1 + l * p.stride), true);
        else if constexpr (OP == WK_UP) stage_norm(l, (const float*)((const char*)p.ln3 + l * p.stride), false);
        else wait(op - 1);
      }
      if constexpr (OP == WK_O || OP == WK_CO) res = __builtin_bit_cast(f32x4, lk_load16(rsrc_of(residual(l), (unsigned)j.rows * D * 4), (m * D + n) * 4));
      if constexpr (OP == TK_DOWN) stage(p.ffh + (place & 3) * D, F * 2);          // (another place: another slice)
      else if constexpr (OP == WK_O || OP == WK_CO) { if (!staged) stage(p.attn, D * 2); }
      staged = true;
      lk_barrier();                              // the input is staged, the partial sums of the place before are read
      lk_barrier();                              // the partial sums are there
      if (hw >= MT) continue;
      f32x4 part[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) part[w] = red[(w * MT + hw) * 64 + lane];
      __builtin_amdgcn_sched_barrier(0);
      f32x4 v = ((part[0] + part[1]) + part[2]) + part[3];
      if (m >= j.rows) continue;
      if constexpr (OP == WK_QKV) {
        store_qkv(l, tile >> 6, n - (tile >> 6) * D, m, v);
      } else if constexpr (OP == WK_UP) {
        v += bs;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.f);
        wk_store8(p.ffh + (size_t)m * F + n, u32x2{cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3])});
      } else if constexpr (OP == TK_DOWN) {
        wk_store16(p.part + ((size_t)(place & 3) * j.rows + m) * D + n, v);
      } else {
        v += res;
        wk_store16((float*)residual(l) + (size_t)m * D + n, v);
      }
    }
    // Members without queries, keys and values carry the residual stream over to the layer's own buffer (one of those that normalise it took 1.2 us
    // longer for it, and all waited).  Their flags count with the self-attention's: the next operator that reads it follows that
    if (OP == WK_QKV && j.full && j.rank < 8 && hw == 0 && moved(l) && j.rank * 8 + j.xcd < j.rows) {
      f32x4 v[4];
      wait(op - 1);
      load_row(l, j.rank * 8 + j.xcd, true, v);
      keep_row(l, j.rank * 8 + j.xcd, v);
    }
    constexpr unsigned MASK = OP == WK_QKV ? 0xFFFFFF00u : (OP == WK_O ? 0xFF00u : (OP == WK_CO ? 0xFF0000u : 0xFFFFFFFFu));
    this->template done<MT>(staged, MASK, OP != WK_QKV);
  }
  template <int OP>
  __device__ __forceinline__ void attention(int l) {
    ++op;
    bool mine = false;
#pragma unroll 1
    for (int place = j.place; place < 256; place += j.members) {
      const int first = TkPlaces::order(OP, place);
      if (first < 0) continue;
#pragma unroll 1
      for (int k = first; k < 2 * j.slots; k += 16) {
        const int item = TkPlaces::item(place, k);
        if constexpr (OP == WK_CROSS) cross_item<ATTN_THROUGH>(l, item, residual(l), op - 1, poll(false), lk_args().attn, !mine);
        else self_item<MT, ATTN_THROUGH>(l, item, op - 1, lk_args().attn, !mine);
        mine = true;
      }
    }
    this->template done<4>(mine || (OP == WK_SELF && j.rank < 8), TkPlaces::mask(OP, j.slots) | (OP == WK_SELF ? 0xFFu : 0u), true);
  }
  __device__ __forceinline__ void run() {
    const int layers = lk_args().n_layers;
    {
      const LayersP& p = lk_args();
      const int at = hw * 16 + (lk_lane() & 15), m = at < j.rows ? at : 0, slot = m / p.R;
      sb = p.seq ? p.seq[slot] : slot;
      key = p.base[slot] + m - slot * p.R;
    }
#pragma unroll 1
    for (int l = 0; l < layers; ++l) {
      this->template product<WK_QKV>(l);
      this->template attention<WK_SELF>(l);
      this->template product<WK_O>(l);
      this->template attention<WK_CROSS>(l);
      this->template product<WK_CO>(l);
      this->template product<WK_UP>(l);
      this->template product<TK_DOWN>(l);
    }
  }
};

template <int MT>
struct TkCompute {
  const bf16_t* xs;
  f32x4* red;
  int cw;
  WkMember j;
  u32x4 aq[1][8], a1[1][8], ax[4][8];            // ax: the head's queries; or an output projection, and the second FFN layer (behind the queries)

  template <int PACE = 0, int N, int U> __device__ __forceinline__ void load(u32x4 (&a)[N][U], const char* LayersP::*w, int l, int tile) {
    const LayersP& p = lk_args();
    lk_weights<PACE>(a, p.*w + l * p.stride, tile, cw, lk_lane());
  }
  __device__ __forceinline__ u32x4 (&one())[1][8] { return *reinterpret_cast<u32x4 (*)[1][8]>(&ax[0]); }
  __device__ __forceinline__ u32x4 (&second())[1][8] { return *reinterpret_cast<u32x4 (*)[1][8]>(&ax[1]); }
  // (two steps of operands for the row tiles at a time: registers)
  __device__ __forceinline__ void multiply(const u32x4 (&a)[1][8]) {
    const int lane = lk_lane(), lr = lane & 15;
    const bf16_t* row[MT];
    f32x4 acc[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int m = t * 16 + lr;
      row[t] = xs + (m < j.rows ? m : 0) * (1024 + 8) + cw * 256 + (lane >> 4) * 8;
      acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
      bf16x8 b[2][MT];
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int t = 0; t < MT; ++t) b[e][t] = __builtin_bit_cast(bf16x8, *(const u32x4*)(row[t] + (i + e) * 32));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int t = 0; t < MT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[0][i + e]), b[e][t], acc[t], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < MT; ++t) red[(cw * MT + t) * 64 + lane] = acc[t];
  }
  template <int OP> __device__ __forceinline__ void product(u32x4 (&a)[1][8], const char* LayersP::*w, int l) {
#pragma unroll 1
    for (int place = j.place; place < 256; place += j.members) {
      const int tile = OP == TK_DOWN ? place : WkMember::tile(OP, place);          // (a K slice of a tile of the second FFN layer lies like a tile of K = 1024)
      if (tile < 0) continue;
      if (!j.full) load(a, w, l, tile);
      lk_barrier();
      multiply(a);
      lk_barrier();
    }
  }
  // Weights are fetched while a member idles: see the places
  __device__ __forceinline__ void run() {
    const int layers = lk_args().n_layers, r = j.place & 31, slots = j.slots;
    const int cross_tile = (2 * (j.place >> 5) + (TkPlaces::order(WK_CROSS, j.place) & 1)) * 4;      // (of the head's queries)
    const bool full = j.full, self = full && TkPlaces::any(WK_SELF, j.place, slots), cross = full && TkPlaces::any(WK_CROSS, j.place, slots);
    const bool low = full && r < 8, qkv = full && r >= 8, o = full && r >= 8 && r < 16, co = full && r >= 16 && r < 24;
    if (qkv) load(aq, &LayersP::wqkv, 0, WkMember::tile(WK_QKV, j.place));
    if (o) load(one(), &LayersP::wo, 0, WkMember::tile(WK_O, j.place));
#pragma unroll 1
    for (int l = 0; l < layers; ++l) {
      const int next = l + 1 < layers ? l + 1 : l;                   // (past the last layer: once more, read by nobody)
      if (low) {
        if (l > 0) __builtin_amdgcn_s_sleep(WK_HOLD);
        if (cross) load<WK_GAP>(ax, &LayersP::cq, l, cross_tile);
        load<WK_GAP>(a1, &LayersP::w1, l, j.place);
        if (!cross) load<WK_GAP>(second(), &LayersP::w2, l, j.place);
      }
      product<WK_QKV>(aq, &LayersP::wqkv, l);
      if (qkv && !self && !o) {
        __builtin_amdgcn_s_sleep(WK_HOLD);       // (the operator's own results first)
        if (cross) load<WK_GAP>(ax, &LayersP::cq, l, cross_tile);
        if (co) load<WK_GAP>(one(), &LayersP::co, l, WkMember::tile(WK_CO, j.place));
        load<WK_GAP>(aq, &LayersP::wqkv, next, WkMember::tile(WK_QKV, j.place));
        load<WK_GAP>(a1, &LayersP::w1, l, j.place);
        if (!cross) load<WK_GAP>(second(), &LayersP::w2, l, j.place);
      }
#pragma unroll 1
      for (int place = j.place, mine = 0; place < 256; place += j.members) {
        const int first = TkPlaces::order(WK_SELF, place);
        for (int k = first < 0 ? 2 * slots : first; k < 2 * slots; k += 16) {
          if (mine) lk_barrier();
          mine = 1;
          lk_barrier();
        }
      }
      product<WK_O>(one(), &LayersP::wo, l);
      if (qkv && (self || o)) {
        __builtin_amdgcn_s_sleep(WK_HOLD);
        if (cross) load(ax, &LayersP::cq, l, cross_tile);
        load<WK_GAP>(aq, &LayersP::wqkv, next, WkMember::tile(WK_QKV, j.place));
        if (o) load<WK_GAP>(one(), &LayersP::wo, next, WkMember::tile(WK_O, j.place));
        load<WK_GAP>(a1, &LayersP::w1, l, j.place);
        if (!cross) load<WK_GAP>(second(), &LayersP::w2, l, j.place);
      }
#pragma unroll 1
      for (int place = j.place, mine = 0; place < 256; place += j.members) {
        const int first = TkPlaces::order(WK_CROSS, place);
        if (first < 0 || first >= 2 * slots) continue;
        if (!full) load(ax, &LayersP::cq, l, (TkPlaces::item(place, first) & 15) * 4);
#pragma unroll 1
        for (int k = first; k < 2 * slots; k += 16) {
          if (mine) lk_barrier();
          mine = 1;
          lk_barrier();
          lk_multiply(ax, xs, lk_args().R, red, cw, lk_lane());
          lk_barrier();
          lk_barrier();
          lk_barrier();
        }
      }
      if (cross) load<WK_GAP>(second(), &LayersP::w2, l, j.place);
      product<WK_CO>(one(), &LayersP::co, l);
      product<WK_UP>(a1, &LayersP::w1, l);
      product<TK_DOWN>(second(), &LayersP::w2, l);
    }
  }
};

// (the attention works where the partial sums lie: they are read, and not yet written again)
template <int MT>
struct TkLds {
  static constexpr int XS = 16 * MT * (1024 + 8) * 2, RED = 4 * 4 * 64 * 16, ATTN = (int)AttnLds::BYTES > RED ? (int)AttnLds::BYTES : RED;
  static constexpr int BYTES = XS + ATTN + 512 * 8 + 64;
  static_assert(BYTES <= 160 * 1024, "LDS");
};

template <int MT>
__global__ __launch_bounds__(512, 2) void tall_layers_kernel(LayersP p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lk_smem[];
  using Lds = TkLds<MT>;
  bf16_t* xs = (bf16_t*)lk_smem;
  f32x4* red = (f32x4*)(lk_smem + Lds::XS);
  u32x2* q_s = (u32x2*)(lk_smem + Lds::XS + Lds::ATTN);
  int* word = (int*)(q_s + 512);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int xcd = __builtin_amdgcn_readfirstlane((int)lk_xcd());
  WkMember j;
  if (!wk_register(p, word, wave, lane, xcd, j)) return;
  if (wave >= 4) {
    TkCompute<MT> c{xs, red, wave - 4, j};
    c.run();
  } else {
    __builtin_amdgcn_s_setprio(3);
    TkHelper<MT> h;
    h.xs = xs; h.red = red; h.sm = AttnLds::carve((unsigned char*)red); h.q_s = q_s; h.hw = wave; h.j = j;
    h.run();
  }
}
