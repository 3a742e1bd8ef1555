// As bpd_wide_layers.h, for blocks of 17 .. 64 rows of up to 16 slots: MT = 2 .. 4 MFMA row tiles.  Included by bpd_kernels.h behind it.
//
// With one row tile of a few rows every member normalises all of an operator's input itself, which costs 0.42 us a row and wave: here a wave has
// one row, and the XCD's waves hand their rows on inside the XCD (every XCD normalises all rows: a hand-over between XCDs
// costs more than the row).  The second FFN layer (four times as long as the others) is split over K among four members per tile, all 256 of
// them: each multiplies 1024 of 4096, as everywhere else, so that one staging buffer of 16 MT x 1024 holds any input; whoever reads the residual stream next adds the
// four slices: the LayerNorm and the output projection that follow, and ln_row_kernel behind the last layer.  Results tell by themselves that they have come, as there.
//
// Six layers of 40 rows in five slots: 264 us as a chain of 60 kernels, 181 here (with flags behind the results, gathered per XCD and passed on, 192); of 32 rows in
// four slots 154 (171), of 56 .. 64 in seven 206 (225).  A layer of 40 rows, us from the results of the operator before: first LayerNorm staged 4.0, queries, keys and values out 1.2;
// self-attention out 2.4; output projection staged 2.6, out 0.9; cross-attention out 4.9; its projection staged 1.6, out 0.9; third LayerNorm staged 3.7, first FFN layer
// out 1.2; second staged 2.9, out 1.0.  Staging is what bounds it: a trip to memory, then 80 KB a member from the L2 and into the LDS (0.9 .. 1.4 us).
//
// Places.  r < 8: no queries, keys and values, but the cross-attention's first eight heads of an XCD, 24 .. 31: the self-attention's (the
// other way round for more; from nine slots on two heads or more per place); 8 .. 15, 16 .. 23: the output projections; every place has a tile of the first FFN layer and one K slice of a tile of the second.
#pragma once

constexpr int TK_ROWS = TALL_LAYERS_ROWS;        // rows of the XCD's copies of normalised rows
static_assert(WK_NORM + TK_ROWS <= WK_AREA, "a flag per row");
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
};

template <int MT>
struct TkHelper : WkHelper {
  // Buffers of what is handed over, two of each, which the layers use in turn: the residual stream behind the attentions (stage 1, 2), the attentions' results, the hidden
  // layer, the second FFN layer's four slices (the last layer's: LayersP::part, for the kernel behind), and an XCD's normalised rows.
  __device__ __forceinline__ static float* between(int stage, int l) { return lk_args().x1 + ((stage - 1) * 2 + (l & 1)) * (TK_ROWS * D); }
  __device__ __forceinline__ static bf16_t* heads(int which, int l) { return lk_args().attn + ((which == WK_CROSS ? 2 : 0) + (l & 1)) * (TK_ROWS * D); }
  __device__ __forceinline__ static bf16_t* hidden(int l) { return lk_args().ffh + (l & 1) * (TK_ROWS * F); }
  __device__ __forceinline__ static float* slices(int l) { const LayersP& p = lk_args(); return l + 1 == p.n_layers ? p.part : p.slices + (l & 1) * (4 * TK_ROWS * D); }
  __device__ __forceinline__ bf16_t* normed(int op, int l) const { return lk_args().xn + (size_t)((j.xcd * 2 + (op == WK_UP ? 1 : 0)) * 2 + (l & 1)) * (TK_ROWS * D); }
  // the row that this wave normalises for its XCD (full: the members with queries, keys and values)
  __device__ __forceinline__ int norm_of() const { const int m = hw < 3 && j.rank >= 8 ? hw * 24 + j.rank - 8 : TK_ROWS; return m < j.rows ? m : -1; }
  __device__ __forceinline__ LkPoll poll() { return LkPoll{&broken, lk_args().error, true, j.rank}; }

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

  // Row m ahead of layer l's first LayerNorm (OP = WK_QKV: what the layer before left, its slices being what is waited for: the rows behind the cross-attention were there
  // for the LayerNorm in between), or ahead of its third
  template <int OP>
  __device__ __forceinline__ void load_row(int l, int m, f32x4 (&v)[4]) {
    const LayersP& p = lk_args();
    const int lane = lk_lane();
    const rsrc_t xr = rsrc_of(OP == WK_UP ? between(2, l) : (l > 0 ? between(2, l - 1) : p.x), (unsigned)j.rows * D * 4);
    if constexpr (OP == WK_UP) {
      LkPoll w = poll();
      w.turn = -1;
      w([&] {
#pragma unroll
        for (int h = 0; h < 4; ++h) v[h] = __builtin_bit_cast(f32x4, lk_load16(xr, (m * D + h * 256 + lane * 4) * 4));
        unsigned top = 0;
#pragma unroll
        for (int h = 0; h < 4; ++h) top = lk_top(top, __builtin_bit_cast(u32x4, v[h]));
        return top;
      });
    } else if (l == 0) {
#pragma unroll
      for (int h = 0; h < 4; ++h) v[h] = __builtin_bit_cast(f32x4, lk_load16(xr, (m * D + h * 256 + lane * 4) * 4));
    } else {
      const rsrc_t pr = rsrc_of(slices(l - 1), (unsigned)j.rows * D * 16);
      const float* b2 = (const float*)((const char*)p.b2 + (l - 1) * p.stride);
      f32x4 s[4][4], bias[4];
#pragma unroll
      for (int h = 0; h < 4; ++h) bias[h] = *(const f32x4*)(b2 + h * 256 + lane * 4);
#pragma unroll
      for (int h = 0; h < 4; ++h) v[h] = __builtin_bit_cast(f32x4, lk_load16(xr, (m * D + h * 256 + lane * 4) * 4));
      LkPoll w = poll();
      w.first<4>(pr, ((j.rank >> 2 & 3) * j.rows + m) * (D * 4), lane);
      w([&] {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int h = 0; h < 4; ++h) s[i][h] = __builtin_bit_cast(f32x4, lk_load16(pr, ((i * j.rows + m) * D + h * 256 + lane * 4) * 4));
        __builtin_amdgcn_sched_barrier(0);
        unsigned top = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int h = 0; h < 4; ++h) top = lk_top(top, __builtin_bit_cast(u32x4, s[i][h]));
        return top;
      });
#pragma unroll
      for (int h = 0; h < 4; ++h) v[h] += (((s[0][h] + s[1][h]) + s[2][h]) + s[3][h]) + bias[h];
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  // bf16 rows of 1024 (ld: bytes between them) into LDS, 1032 apart; poll: until they have come.  (One piece first, as in bpd_wide_layers.h; then of all rows those that
  // are missing again: 80 KB a member each time would be too much.)
  __device__ __forceinline__ void stage(const bf16_t* src, unsigned ld, bool wait_for) {
    const int lane = lk_lane();
    const rsrc_t r = rsrc_of(src, (unsigned)(j.rows - 1) * ld + D * 2);
    u32x4 v[4 * MT][2];
    if (wait_for) poll().template first<2>(r, hw * ld, lane);
#pragma unroll
    for (int i = 0; i < 4 * MT; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) v[i][h] = lk_load16(r, (hw + 4 * i) * ld + h * 1024 + lane * 16);
    __builtin_amdgcn_sched_barrier(0);
    if (wait_for && !broken) {
      bool seen = false;
#pragma unroll 1
      for (int s = 0; s < LK_POLLS; ++s) {
        unsigned top = 0;
#pragma unroll
        for (int i = 0; i < 4 * MT; ++i) { top = lk_top(top, v[i][0]); top = lk_top(top, v[i][1]); }
        if (!__any(top == EMPTY_WORD)) { seen = true; break; }
#pragma unroll
        for (int i = 0; i < 4 * MT; ++i)
          if (__any(lk_top(lk_top(0, v[i][0]), v[i][1]) == EMPTY_WORD)) {
#pragma unroll
            for (int h = 0; h < 2; ++h) v[i][h] = lk_load16(r, (hw + 4 * i) * ld + h * 1024 + lane * 16);
          }
        asm volatile("" ::: "memory");
      }
      if (!seen) { broken = true; if (lane == 0) *lk_args().error = 1; }
    }
#pragma unroll
    for (int i = 0; i < 4 * MT; ++i)
      if (hw + 4 * i < j.rows) {
#pragma unroll
        for (int h = 0; h < 2; ++h) *(u32x4*)(xs + (hw + 4 * i) * (D + 8) + h * 512 + lane * 8) = v[i][h];
      }
  }
  // LayerNorm of all rows into LDS
  template <int OP>
  __device__ __forceinline__ void stage_norm(int l, const float* ln) {
    const LayersP& p = lk_args();
    const int lane = lk_lane();
    f32x4 g[4], b[4], v[4];
    load_norm(ln, g, b, lane);
    if (!j.full) {
#pragma unroll 1
      for (int r = hw; r < j.rows; r += 4) {
        load_row<OP>(l, r, v);
        wk_norm_row(v, g, b, p.eps, [&](int h, u32x2 w) { *(u32x2*)(xs + r * (D + 8) + h * 256 + lane * 4) = w; });
      }
      return;
    }
    const int m = norm_of();
    bf16_t* to = normed(OP, l);
    if (m >= 0) {
      load_row<OP>(l, m, v);
      wk_norm_row(v, g, b, p.eps, [&](int h, u32x2 w) { *(u32x2*)(to + (size_t)m * D + h * 256 + lane * 4) = full_words(w); });
    }
    if (OP == WK_QKV && l == 0) {                // (nothing is empty yet: a flag each)
      unsigned* flags = area() + WK_NORM;
      if (m >= 0) lk_raise(flags + m, op, lane);
      if (!broken) {
        bool seen = false;
#pragma unroll 1
        for (int s = 0; s < LK_SPINS; ++s) {
          const unsigned f = lk_load(flags + lane);
          if (__all(lane >= j.rows || f >= op)) { seen = true; break; }
        }
        if (!seen) { broken = true; if (lane == 0) *p.error = 1; }
      }
    }
    stage(to, D * 2, OP != WK_QKV || l > 0);
  }

  // Emptied (EMPTY_WORD) by the waves that write it, a layer later, when all have read it, and ahead of a result of the writer's that the next readers wait for: the
  // first FFN layer's input is there when both attentions' results, what they read, the first LayerNorm's rows and the slices, rows and hidden layer of the layer
  // before have been read; the next layer's first input when the third LayerNorm's rows have.  A wave's stores have arrived when loads behind them have, and its next
  // operator stages, meets the other waves and then stores.
  __device__ __forceinline__ void empty_normed(int op, int l, int lane) const {
    const int m = norm_of();
    if (!j.full || m < 0) return;
#pragma unroll
    for (int h = 0; h < 4; ++h) *(u32x2*)(normed(op, l) + m * D + h * 256 + lane * 4) = u32x2{EMPTY_WORD, EMPTY_WORD};
  }
  __device__ __forceinline__ void empty_tile(float* x, int tile, int lane) const {
    const int m = hw * 16 + (lane & 15);
    const float e = __uint_as_float(EMPTY_WORD);
    if (hw < MT && tile >= 0 && m < j.rows) wk_store16(x + (size_t)m * D + tile * 16 + (lane >> 4) * 4, f32x4{e, e, e, e});
  }
  __device__ __forceinline__ void empty_heads(int which, int l, int place, int lane) const {
    const int first = TkPlaces::order(which, place);
    if (first < 0) return;
#pragma unroll 1
    for (int k = first; k < 2 * j.slots; k += 16) rows_of_head(heads(which, l), TkPlaces::item(place, k), EMPTY_WORD, lane);
  }
  __device__ __forceinline__ void empty_hidden(int l, int place, int lane) const {
    const int m = hw * 16 + (lane & 15);
    if (hw < MT && m < j.rows) wk_store8(hidden(l) + (size_t)m * F + place * 16 + (lane >> 4) * 4, u32x2{EMPTY_WORD, EMPTY_WORD});
  }
  __device__ __forceinline__ void empty_slice(int l, int place, int lane) const { empty_tile(slices(l) + (size_t)(place & 3) * j.rows * D, place >> 2, lane); }
  // Everything that this member writes, but what the first LayerNorm of the first layer has written
  __device__ __forceinline__ void empty_all(int lane) const {
    const int layers = lk_args().n_layers;
    empty_normed(WK_QKV, 1, lane);
    for (int l = 0; l < 2; ++l) empty_normed(WK_UP, l, lane);
#pragma unroll 1
    for (int place = j.place; place < 256; place += j.members)
#pragma unroll 1
      for (int l = 0; l < 2; ++l) {
        empty_tile(between(1, l), WkMember::tile(WK_O, place), lane); empty_tile(between(2, l), WkMember::tile(WK_CO, place), lane);
        empty_heads(WK_SELF, l, place, lane); empty_heads(WK_CROSS, l, place, lane);
        empty_hidden(l, place, lane);
        if (l + 1 < layers) empty_slice(l, place, lane);
      }
  }

  template <int OP>
  __device__ __forceinline__ void product(int l) {
    const LayersP& p = lk_args();
    const int lane = lk_lane(), lr = lane & 15, lq = lane >> 4, m = hw * 16 + lr;
    if constexpr (OP == WK_QKV) ++op;
    bool staged = false;
#pragma unroll 1
    for (int place = j.place; place < 256; place += j.members) {
      const int tile = OP == TK_DOWN ? place >> 2 : WkMember::tile(OP, place);
      if (tile < 0) continue;
      const int n = tile * 16 + lq * 4;
      f32x4 bs, res;
      if (!staged && OP != WK_QKV && OP != TK_DOWN && l == 0) wait(1);       // (everybody has emptied what it writes)
      const rsrc_t rr = rsrc_of(OP == WK_CO ? between(1, l) : (l > 0 ? between(2, l - 1) : p.x), (unsigned)j.rows * D * 4);
      if constexpr (OP == WK_O || OP == WK_CO) res = __builtin_bit_cast(f32x4, lk_load16(rr, (m * D + n) * 4));
      if constexpr (OP == WK_O) if (l > 0) {     // (all there: the first LayerNorm has read them)
        const rsrc_t pr = rsrc_of(slices(l - 1), (unsigned)j.rows * D * 16);
        f32x4 s[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] = __builtin_bit_cast(f32x4, lk_load16(pr, ((i * j.rows + m) * D + n) * 4));      // (rows past the last: of another slice, not used)
        bs = *(const f32x4*)((const float*)((const char*)p.b2 + (l - 1) * p.stride) + n);
        __builtin_amdgcn_sched_barrier(0);
        res += (((s[0] + s[1]) + s[2]) + s[3]) + bs;
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (OP == TK_DOWN) stage(hidden(l) + (place & 3) * D, F * 2, true);          // (another place: another slice)
      else if (!staged) {
        if constexpr (OP == WK_QKV) stage_norm<OP>(l, (const float*)((const char*)p.ln1 + l * p.stride));
        else if constexpr (OP == WK_UP) stage_norm<OP>(l, (const float*)((const char*)p.ln3 + l * p.stride));
        else stage(heads(OP == WK_O ? WK_SELF : WK_CROSS, l), D * 2, true);
      }
      lk_barrier();                              // the input is staged, the partial sums of the place before are read
      if constexpr (OP == WK_QKV) {
        if (MT < 4 && j.full && TkPlaces::any(WK_SELF, place, j.slots)) fetch_ahead(l, TkPlaces::item(place, TkPlaces::order(WK_SELF, place)));
        if (l > 0) { if (!staged) empty_normed(WK_UP, l - 1, lane); }
        else if (j.full) { empty_all(lane); lk_stores_done(); }          // (ahead of the barrier: which wave stores an attention's results depends on the keys)
      }
      if constexpr (OP == WK_UP) {
        bs = *(const f32x4*)((const float*)((const char*)p.b1 + l * p.stride) + n);          // (not ahead of the staging: registers)
        if (!staged) empty_normed(WK_QKV, l, lane);
        empty_tile(between(1, l), WkMember::tile(WK_O, place), lane);
        empty_heads(WK_SELF, l, place, lane); empty_heads(WK_CROSS, l, place, lane);
        if (l > 0) { empty_tile(between(2, l - 1), WkMember::tile(WK_CO, place), lane); empty_hidden(l - 1, place, lane); empty_slice(l - 1, place, lane); }
      }
      // (the cross-attention has read all of x1, but this wave may have asked too early)
      if constexpr (OP == WK_CO) poll()([&] {
        if (__any(lk_top(0, __builtin_bit_cast(u32x4, res)) == EMPTY_WORD)) res = __builtin_bit_cast(f32x4, lk_load16(rr, (m * D + n) * 4));
        return lk_top(0, __builtin_bit_cast(u32x4, res));
      });
      staged = true;
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
        wk_store8(hidden(l) + (size_t)m * F + n, full_words(u32x2{cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3])}));
      } else if constexpr (OP == TK_DOWN) {
        wk_store16(slices(l) + ((size_t)(place & 3) * j.rows + m) * D + n, __builtin_bit_cast(f32x4, full_words(v)));
      } else {
        v += res;
        const f32x4 w = __builtin_bit_cast(f32x4, full_words(v));
        wk_store16(between(OP == WK_O ? 1 : 2, l) + (size_t)m * D + n, w);
        if (OP == WK_CO && l + 1 == p.n_layers) wk_store16(p.x + (size_t)m * D + n, v);          // (for the kernel behind)
      }
    }
    if constexpr (OP == WK_QKV) {
      if (l == 0) this->template done<4>(true, ~0u, true);       // (that everything is empty: to all)
      else this->template done<MT>(staged, 0xFFFFFF00u, false);
    }
  }
  template <int OP>
  __device__ __forceinline__ void attention(int l) {
    bool mine = false;
#pragma unroll 1
    for (int place = j.place; place < 256; place += j.members) {
      const int first = TkPlaces::order(OP, place);
      if (first < 0) continue;
#pragma unroll 1
      for (int k = first; k < 2 * j.slots; k += 16) {
        const int item = TkPlaces::item(place, k);
        if constexpr (OP == WK_CROSS) cross_item<ATTN_THROUGH_WORDS>(l, item, between(1, l), l == 0, poll(), heads(OP, l), !mine);
        else {
          if (l == 0 && !mine && j.rank < 8) wait(1);         // (its waves have met no barrier since they emptied these)
          self_item<MT, ATTN_THROUGH_WORDS>(l, item, op, heads(OP, l), !mine);
        }
        mine = true;
      }
    }
  }
  __device__ __forceinline__ void run() {
    const int layers = lk_args().n_layers;
    {
      const LayersP& p = lk_args();
      const int at = hw * 16 + (lk_lane() & 15), m = at < j.rows ? at : 0, slot = m / p.R;
      sb = p.seq ? p.seq[slot] : slot;
      key = p.base[slot] + m - slot * p.R;
    }
    if (!j.full || j.rank < 8) empty_all(lk_lane());          // (the others: in the first operator, which these have no part in)
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
