// Attention of 64-wide bf16 heads on the matrix cores, over keys and values kept in operand order.  Included by
// bpd_kernels.h (after AttnP).
#pragma once

// K and V of one sequence and head, 64-wide heads in bf16: `capg` groups of 32 keys, 4 KiB of each per group, as the
// operands of v_mfma_f32_16x16x32_bf16 that the attention feeds them to, so that every fragment is one coalesced 1 KiB
// load and nothing passes through LDS:
//   K group: [key tile t][dimensions 32 s .. + 31][lane][8]: lane 16 q' + row holds dimensions 32 s + 8 q' .. + 7 of the key
//            8 (row / 4) + 4 t + row % 4 of the group: the scores that a lane of the product holds are then those of
//            keys 8 (lane / 16) .. + 7 (tiles 0 and 1 in turn), which is what the second product takes from it.
//   V group: [dimensions 16 t .. + 15][lane][8]: lane 16 q + c holds dimension 16 t + c of keys 8 q .. + 7.
constexpr int KV_GROUP = 2048;                   // elements of a group of 32 keys x 64 dimensions
__device__ __forceinline__ unsigned k_frag_at(int key, int c) {        // c % 4 == 0: four dimensions lie side by side
  return (unsigned)(key >> 5) * KV_GROUP + ((key >> 2) & 1) * 1024 + (c >> 5) * 512 + (((c >> 3) & 3) * 16 + ((key >> 3) & 3) * 4 + (key & 3)) * 8 + (c & 7);
}
__device__ __forceinline__ unsigned v_frag_at(int key, int c) {        // dimension c + 1 lies 8 elements on
  return (unsigned)(key >> 5) * KV_GROUP + (c >> 4) * 512 + (((key >> 3) & 3) * 16 + (c & 15)) * 8 + (key & 7);
}
// Columns col .. col + 3 (col % 4 == 0) of key row `key` of sequence sb
__device__ __forceinline__ void kv_frag_store(bf16_t* cache, bool is_v, int sb, int heads, int capg, int key, int col, unsigned lo, unsigned hi) {
  bf16_t* dst = cache + ((size_t)sb * heads + (col >> 6)) * capg * KV_GROUP;
  if (!is_v) {
    *(u32x2*)(dst + k_frag_at(key, col & 63)) = u32x2{lo, hi};
  } else {
    bf16_t* v = dst + v_frag_at(key, col & 63);
    v[0] = (bf16_t)lo; v[8] = (bf16_t)(lo >> 16); v[16] = (bf16_t)hi; v[24] = (bf16_t)(hi >> 16);
  }
}

// What a word holds whose value is still to come, in buffers whose readers wait for the values themselves (bpd_layers.h): no value that is stored there is this
// one (a NaN of these bits goes as the NaN beside it).
constexpr unsigned EMPTY_WORD = 0xFFFFFFFFu;
__device__ __forceinline__ unsigned full_word(unsigned v) { return v < EMPTY_WORD - 1 ? v : EMPTY_WORD - 1; }
__device__ __forceinline__ u32x2 full_words(u32x2 v) { return u32x2{full_word(v[0]), full_word(v[1])}; }
__device__ __forceinline__ u32x4 full_words(f32x4 f) { const u32x4 v = __builtin_bit_cast(u32x4, f); return u32x4{full_word(v[0]), full_word(v[1]), full_word(v[2]), full_word(v[3])}; }

// fp32 operands (queries, probabilities) go to the matrix cores as a bf16 pair hi + lo, which keeps them to ~2^-17.
__device__ __forceinline__ void split_bf16x8(const float (&v)[8], bf16x8& hi, bf16x8& lo) {
  unsigned h[4], l[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    h[j] = cvt_pk_bf16(v[2 * j], v[2 * j + 1]);
    l[j] = cvt_pk_bf16(v[2 * j] - __uint_as_float(h[j] << 16), v[2 * j + 1] - __uint_as_float(h[j] & 0xFFFF0000u));
  }
  hi = __builtin_bit_cast(bf16x8, (u32x4{h[0], h[1], h[2], h[3]}));
  lo = __builtin_bit_cast(bf16x8, (u32x4{l[0], l[1], l[2], l[3]}));
}

// Four columns of scaled queries as the attention's operands
__device__ __forceinline__ void lk_halves(const f32x4& v, u32x2& hi, u32x2& lo) {
  hi = u32x2{cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3])};
  lo = u32x2{cvt_pk_bf16(v[0] - __uint_as_float(hi[0] << 16), v[1] - __uint_as_float(hi[0] & 0xFFFF0000u)),
             cvt_pk_bf16(v[2] - __uint_as_float(hi[1] << 16), v[3] - __uint_as_float(hi[1] & 0xFFFF0000u))};
}
// Workgroup barrier that leaves global loads under way (the waves meet over LDS only)
__device__ __forceinline__ void lk_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// QU > 0 (at most 16 rows per sequence, d = 128 * QU): the queries are projected inside the kernel,
//   Q = LayerNorm(x) Wq[:, 64 h .. 64 h + 63]   (x: fp32 residual stream),
// instead of being read from p.Q: the waves split the contraction, their partial sums meet in LDS, and the K/V loads of
// the first chunk are already in flight meanwhile.  Saves the projection's kernel and its round trip.
struct QProjP {
  const float* x;       // [M][d] residual stream
  const float* g;       // LayerNorm gain, bias
  const float* b;
  const void* W;        // packed [d/16 column tiles][d/32 k-steps][64 lanes][8]
  float eps;
};

// LDS of one attention workgroup of up to ATTN_WAVES waves: the kernel below declares it; a caller that runs the body from
// inside another kernel carves it out of its own LDS (four waves, QU == 0).
constexpr int ATTN_WAVES = 8;
struct AttnLds {
  static constexpr int RT = 16, DH = 64;
  f32x4 (*o_s)[4][64];        // [waves][4][64]  per wave and output tile: un-normalised out^T
  float (*m_s)[RT];           // [waves][RT]     per wave: running maximum per query row
  float (*l_s)[RT];           // [waves][RT]     ... and sum
  u32x2* q_s;                 // QU > 0: [hi, lo][2][64][2] projected queries as MFMA operands
  float* gb_s;                // QU > 0: per wave, gain and bias of its columns; and the row sums of x
  float2* st_s;
  static constexpr size_t OS_BYTES = (size_t)4 * 4 * 64 * 16, ML_BYTES = (size_t)4 * RT * 4;
  static constexpr size_t BYTES = OS_BYTES + 2 * ML_BYTES;        // four waves, QU == 0
  __device__ static AttnLds carve(unsigned char* base) {          // (16-byte aligned base)
    AttnLds s;
    s.o_s = (f32x4 (*)[4][64])base;
    s.m_s = (float (*)[RT])(base + OS_BYTES);
    s.l_s = (float (*)[RT])(base + OS_BYTES + ML_BYTES);
    s.q_s = nullptr; s.gb_s = nullptr; s.st_s = nullptr;
    return s;
  }
};

// Largest maximum M, sum L and values o (both relative to M) of NW waves' results for row lane % 16, output tile dt
template <int NW>
__device__ __forceinline__ void attention_merge(const AttnLds& sm, int dt, int lane, float& M, float& L, f32x4& o) {
  // (every LDS read under way before the first is waited for: left alone the compiler reads and waits wave by wave, 0.4 us for four)
  float mw[NW], lw[NW];
  f32x4 ow[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) mw[w] = sm.m_s[w][lane & 15];
#pragma unroll
  for (int w = 0; w < NW; ++w) { lw[w] = sm.l_s[w][lane & 15]; ow[w] = sm.o_s[w][dt][lane]; }
  __builtin_amdgcn_sched_barrier(0);
  M = -INFINITY; L = 0.f;
  o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < NW; ++w) M = fmaxf(M, mw[w]);
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const float wgt = (mw[w] == -INFINITY) ? 0.f : __expf(mw[w] - M);
    L = fmaf(lw[w], wgt, L);
    o += ow[w] * wgt;
  }
}

// K and V of the groups c, c + nw, .. (G of them) as operands
template <bool KVNT, int G>
__device__ __forceinline__ void attn_load_kv(rsrc_t kr, rsrc_t vr, int c, int nw, int lane, u32x4 (&kf)[G][4], u32x4 (&vf)[G][4]) {
#pragma unroll
  for (int gg = 0; gg < G; ++gg) {
    const unsigned at = (unsigned)__builtin_amdgcn_readfirstlane(c + gg * nw) * (KV_GROUP * 2);
#pragma unroll
    for (int x = 0; x < 4; ++x) kf[gg][x] = __builtin_amdgcn_raw_buffer_load_b128(kr, lane * 16 + x * 1024, at, KVNT ? 2 : 0);
#pragma unroll
    for (int x = 0; x < 4; ++x) vf[gg][x] = __builtin_amdgcn_raw_buffer_load_b128(vr, lane * 16 + x * 1024, at, KVNT ? 2 : 0);
  }
}
// ... one of the two
template <bool KVNT, int G>
__device__ __forceinline__ void attn_load_one(rsrc_t r, int c, int nw, int lane, u32x4 (&f)[G][4]) {
#pragma unroll
  for (int gg = 0; gg < G; ++gg) {
    const unsigned at = (unsigned)__builtin_amdgcn_readfirstlane(c + gg * nw) * (KV_GROUP * 2);
#pragma unroll
    for (int x = 0; x < 4; ++x) f[gg][x] = __builtin_amdgcn_raw_buffer_load_b128(r, lane * 16 + x * 1024, at, KVNT ? 2 : 0);
  }
}
// The item's work from the point where its queries (qhi + qlo) and the first groups of K and V are at hand or under way (parameters as in
// attention_mfma_body; first, hop: this split's first group and the distance to its next round; lim: limit[b]).  STORE: no word of the results is EMPTY_WORD (ATTN_WORDS),
// and they are written through the L2 (ATTN_THROUGH_WORDS).  ONCE: no wave has a second round.  AHEAD: the next round's keys and values are asked for within this one.
enum { ATTN_PLAIN, ATTN_WORDS, ATTN_THROUGH_WORDS };
template <int STORE>
__device__ __forceinline__ void attention_store(bf16_t* to, const f32x4& v) {
  u32x2 w = u32x2{cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3])};
  if constexpr (STORE != ATTN_PLAIN) w = full_words(w);
  if constexpr (STORE == ATTN_THROUGH_WORDS) asm volatile("global_store_dwordx2 %0, %1, off sc1" ::"v"(to), "v"(w) : "memory");      // (to memory, for other XCDs)
  else *(u32x2*)to = w;
}
template <bool KVNT, bool LIMF, int QU, int G, int STORE = ATTN_PLAIN, bool ONCE = false>
__device__ __forceinline__ void attention_mfma_core(const AttnP& p, const AttnLds& sm, int h, int b, int tile, int split, int r0, int nrows,
                                                    int nheads, int nz, int tid, int nw, int first, int hop, rsrc_t kr, rsrc_t vr,
                                                    u32x4 (&kf)[G][4], u32x4 (&vf)[G][4], const bf16x8 (&qhi)[2], const bf16x8 (&qlo)[2], int lim, bf16_t* out) {
  constexpr int RT = 16, DH = 64;
  constexpr bool AHEAD = STORE == ATTN_WORDS && G == 2;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lq = lane >> 4;
  lim = lim < 0 ? 0 : lim;
  int nkeys = p.causal ? lim + r0 + nrows : lim;
  nkeys = nkeys < p.capg * 32 ? nkeys : p.capg * 32;
  const int ngr = (nkeys + 31) >> 5;
  const int nvis = lr < nrows ? (p.causal ? lim + r0 + lr + 1 : lim) : 0;     // keys row lr may see: nlo .. nvis - 1
  const int nlo = LIMF ? attn_first_key(p, lim + r0 + lr) : 0;
  float m_run = -INFINITY, l_run = 0.f;          // of query row lr over this wave's keys (the 4 lanes of a row agree)
  f32x4 acc[4];                                  // out^T tile dt: head dimensions 16*dt + 4*lq + r, row lr
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int c = first; c + wave < ngr; c += hop) {
    // scores: sacc[gg][t][r] = key 32 (c + wave + gg nw) + 8 lq + 4 t + r against query row lr
    f32x4 sacc[G][2];
    float mx = -INFINITY;
#pragma unroll
    for (int gg = 0; gg < G; ++gg)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f}, al = a;       // (two chains)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          const bf16x8 ka = __builtin_bit_cast(bf16x8, kf[gg][2 * t + s2]);
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qhi[s2], a, 0, 0, 0);
          al = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qlo[s2], al, 0, 0, 0);
        }
        a += al;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int key = 32 * (c + wave + gg * nw) + 8 * lq + 4 * t + r;
          a[r] = (key < nvis && (!LIMF || key >= nlo)) ? a[r] : -INFINITY;
          mx = fmaxf(mx, a[r]);
        }
        sacc[gg][t] = a;
      }
    // The next round's keys are asked for as soon as their registers are free, also past the last round (the buffer ends there: nothing is read): behind a condition the
    // compiler would wait for them together with this round's values.  layers_kernel, eight images of up to 3000 intensities, mean over a decode 142.9 us, 140.6 (at 3000
    // keys 168, 166); three with windows of 520 keys 100.7, 99.9.  Not kept: both sets of registers twice (spills); the later rounds fetched into the L2 by the compute waves
    // while queries, keys and values are multiplied (147.7 with one round, 151.8 with two: the CU's loads return in order, and the waits for flags queue behind); two
    // groups per wave in cross-attentions of 192 keys (one round instead of two, 140.8).
    if constexpr (AHEAD) {
      __builtin_amdgcn_sched_barrier(0);
      attn_load_one<KVNT, G>(kr, c + hop + wave, nw, lane, kf);
      __builtin_amdgcn_sched_barrier(0);
    }
    mx = max_rows(mx);
    const float m_new = fmaxf(m_run, mx);
    float sum = 0.f;
#pragma unroll
    for (int gg = 0; gg < G; ++gg)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float pv = (m_new == -INFINITY) ? 0.f : __expf(sacc[gg][t][r] - m_new);
          sacc[gg][t][r] = pv;
          sum += pv;
        }
    sum = sum_rows(sum);
    // What there was before is relative to another maximum.  (The first round skips that in layers_kernel: three images of up to 3000 intensities 58.0 ms, 57.6; in the others'
    // code the branch costs more than it saves: tall_layers_kernel, five sentences 4.46 ms, 4.50.)
    if (STORE == ATTN_WORDS && c == first) l_run = sum;
    else {
      const float alpha = (m_new == -INFINITY) ? 1.f : __expf(m_run - m_new);
      l_run = l_run * alpha + sum;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) acc[dt] *= alpha;
    }
    m_run = m_new;
#pragma unroll
    for (int gg = 0; gg < G; ++gg) {
      const int g0 = 32 * (c + wave + gg * nw);
      if (G > 1 && g0 >= nkeys) continue;        // (the same for the whole wave)
      if (g0 + 32 > nkeys) {                     // values of keys past the last one: their probabilities are zero, their bits unknown
        const int left = nkeys - g0 - 8 * lq;    // of this lane's eight
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const unsigned known = left > 2 * w + 1 ? ~0u : (left > 2 * w ? 0xFFFFu : 0u);
#pragma unroll
          for (int dt = 0; dt < 4; ++dt) vf[gg][dt][w] &= known;
        }
      }
      const float pv[8] = {sacc[gg][0][0], sacc[gg][0][1], sacc[gg][0][2], sacc[gg][0][3], sacc[gg][1][0], sacc[gg][1][1], sacc[gg][1][2], sacc[gg][1][3]};
      bf16x8 phi, plo;
      split_bf16x8(pv, phi, plo);
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        const bf16x8 va = __builtin_bit_cast(bf16x8, vf[gg][dt]);
        acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, phi, acc[dt], 0, 0, 0);
        acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, plo, acc[dt], 0, 0, 0);
      }
    }
    if constexpr (ONCE) break;
    if constexpr (AHEAD) attn_load_one<KVNT, G>(vr, c + hop + wave, nw, lane, vf);
    else if (c + hop + wave < ngr) attn_load_kv<KVNT, G>(kr, vr, c + hop + wave, nw, lane, kf, vf);
  }
  // (16 dimensions on: 16 elements, or 256 of the packed form)
  const bool packed = STORE == ATTN_PLAIN && p.packed;
  bf16_t* const to = out + (packed ? packed_at((long)b * p.R + r0 + lr, h * DH + 4 * lq, p.d) : ((size_t)b * p.R + r0 + lr) * p.d + h * DH + 4 * lq);
  const int on = packed ? 256 : 16;
  // At most 32 keys: the first wave has them all, and all 64 dimensions.  (Through the LDS as below, four waves storing 16 each: 0.25 us more.)
  if (QU >= 0 && ngr - first <= 1 && p.nsplit == 1) {
    if (wave == 0 && lr < nrows) {
      float inv = __builtin_amdgcn_rcpf(l_run);
      inv = inv * fmaf(-l_run, inv, 2.f);        // (one Newton step: the quotient to fp32)
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) attention_store<STORE>(to + dt * on, acc[dt] * inv);
    }
    __syncthreads();
    return;
  }
  // the waves meet (those without keys bring zeros): wave w of the first four finishes head dimensions 16w .. 16w+15
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) sm.o_s[wave][dt][lane] = acc[dt];
  if (lq == 0) { sm.m_s[wave][lr] = m_run; sm.l_s[wave][lr] = l_run; }
  __syncthreads();
  if (wave >= 4) return;
  float M, L;
  f32x4 o;
  if (QU >= 0 && ngr - first <= 1) { M = sm.m_s[0][lr]; L = sm.l_s[0][lr]; o = sm.o_s[0][wave][lane]; }         // (the first wave has all keys)
  else if (QU <= 0 && (QU < 0 || nw == 4)) attention_merge<4>(sm, wave, lane, M, L, o);
  else attention_merge<ATTN_WAVES>(sm, wave, lane, M, L, o);
  const int dim = 16 * wave + 4 * lq;
  if (p.nsplit == 1) {
    if (lr < nrows) {
      float inv = __builtin_amdgcn_rcpf(L);
      inv = inv * fmaf(-L, inv, 2.f);            // (one Newton step: the quotient to fp32)
      attention_store<STORE>(to + wave * on, o * inv);
    }
  } else {
    const int tiles = nz / p.nsplit;
    float* part = p.part + ((((long)b * nheads + h) * tiles + tile) * p.nsplit + split) * (RT * (DH + 2));
    if constexpr (STORE == ATTN_WORDS) {
      *(u32x4*)(part + lr * DH + dim) = full_words(o);
      if (tid < RT) { part[RT * DH + tid] = __uint_as_float(full_word(__float_as_uint(M))); part[RT * DH + RT + tid] = __uint_as_float(full_word(__float_as_uint(L))); }
    } else {
      *(f32x4*)(part + lr * DH + dim) = o;
      if (tid < RT) { part[RT * DH + tid] = M; part[RT * DH + RT + tid] = L; }
    }
  }
}
// One (head h, sequence b (in the K/V buffer: sb), z = row tile * nsplit + split) item of the attention, run by nw whole
// waves (tid 0 .. 64 nw - 1) that share `sm`; nheads / nz: the extents the partial-result layout is indexed with.  Every
// __syncthreads() inside is reached by all of them; a caller whose workgroup has more waves makes those arrive at as many
// barriers (one with QU == 0, four with QU > 0).
// The waves split the keys: of every nw groups of 32 keys each takes one (QU < 0: two of every 2 nw, for long caches: fewer rounds,
// more loads in flight), and keeps its own running maximum, sum and
// weighted values in registers; the results of the waves that had keys meet once, in LDS, at the end.  Per group
//   scores^T = K Q^T     keys are the 16-wide "feature" side of the MFMA, the <= 16 query rows the other
//   softmax              maximum and sum in the lane, then across the 4 lanes of a row; the probabilities stay in
//                        registers: as they lie they are the second MFMA operand of a contraction over the 32 keys
//   out^T += V^T P^T     64 head dimensions = 4 output tiles
// What bounds it at the step's sizes is the chain of latencies (launch, one trip for K, V and Q together, two products, the
// waves' meeting).  With K and V as rows of d (V staged and transposed through LDS, 64 two-byte reads per wave and 64 keys)
// a decoder layer's self-attention took 5.6 us at 8 rows, 8 heads, 30 keys.
// KVNT: K and V are fetched with non-temporal loads (a cache too large for the last-level cache is a stream that should
// not evict the weights).
// LIMF: the sequence's length is fetched first and only groups that hold keys are fetched: one more dependent round trip
// (many sequences: the traffic is what counts; local attention: where the keys start depends on it).
// ARGS: p lies in the kernel's arguments.
// PACKED: as many query rows as keys, from AttnP::row0[b] on (nothing to do for tiles past the last); no splits, not causal.
template <bool KVNT, bool LIMF, int QU, bool ARGS, bool PACKED = false>
__device__ __forceinline__ void attention_mfma_body(const AttnP& p, const QProjP& qp, const AttnLds& sm, int h, int b, int sb, int z,
                                                    int nheads, int nz, int tid, int nw) {
  constexpr int RT = 16, DH = 64, G = QU < 0 ? 2 : 1;       // groups of keys per wave and round
  int split = 0, tile = z;
  if (p.nsplit > 1) { tile = z / p.nsplit; split = z - tile * p.nsplit; }
  static_assert(!PACKED || (LIMF && QU <= 0), "the length is read first");
  const int r0 = tile * RT;
  int nrows = min(RT, p.R - r0);
  long row = (long)b * p.R + r0;                 // of the queries and the results
  if constexpr (PACKED) {
    row = p.row0[b] + r0;
    nrows = min(RT, p.limit[b] - r0);
    if (nrows <= 0) return;                      // (the whole workgroup)
  }
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lq = lane >> 4;
  const size_t head_at = ((size_t)sb * nheads + h) * p.capg * KV_GROUP;
  int glim = p.capg;                             // groups that may be fetched
  int gbeg = 0;                                  // group of the first key (local attention: LIMF only)
  if (LIMF) {
    int l0 = p.limit[b];
    l0 = l0 < 0 ? 0 : l0;
    const int g0 = ((p.causal ? l0 + r0 + nrows : l0) + 31) >> 5;
    glim = g0 < glim ? g0 : glim;
    gbeg = attn_first_key(p, l0 + r0) >> 5;
  }
  const int first = gbeg + split * (G * nw), hop = p.nsplit * (G * nw);
  const rsrc_t kr = rsrc_of((const bf16_t*)p.Kc + head_at, (unsigned)glim * (KV_GROUP * 2));
  const rsrc_t vr = rsrc_of((const bf16_t*)p.Vc + head_at, (unsigned)glim * (KV_GROUP * 2));
  u32x4 kf[G][4], vf[G][4];                      // K: [tile][half of the dimensions], V: [16 dimensions]
  // queries: row lr (zeros beyond the last), head dimensions 32s + 8*lq .. +8, scaled, as bf16 hi + lo
  bf16x8 qhi[2], qlo[2];
  int lim;
  bf16_t* out;
  if constexpr (QU > 0) {
    constexpr int NW = ATTN_WAVES, K = 128 * QU, KSTEPS = K / 32, U = (KSTEPS + NW - 1) / NW;
    const bool mine = wave * U < KSTEPS;         // (K = 128: four waves have k-steps)
    const int ks0 = mine ? wave * U : 0;
    // every global load of the kernel is issued before the first wait, in the order in which they are used
    const f32x4 gbv = *(const f32x4*)((lane % (U * 16) < U * 8 ? qp.g : qp.b) + ks0 * 32 + (lane % (U * 8)) * 4);
    u32x4 wf[4][U], xv[U][2];
    {
      const rsrc_t xr = rsrc_of(qp.x + (size_t)b * p.R * K, mine ? (unsigned)p.R * K * 4 : 0);
      const unsigned off = (lr * K + ks0 * 32 + lq * 8) * 4;
#pragma unroll
      for (int i = 0; i < U; ++i) { xv[i][0] = buf_load16(xr, off + i * 128, 0); xv[i][1] = buf_load16(xr, off + i * 128 + 16, 0); }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < U; ++i) wf[j][i] = *(const u32x4*)((const char*)qp.W + ((size_t)(4 * h + j) * KSTEPS + ks0 + i) * 1024 + lane * 16);
    attn_load_kv<KVNT, G>(kr, vr, first + wave, nw, lane, kf, vf);
    lim = p.limit[b];
    out = (bf16_t*)p.out;
    if (ARGS) out = arg_now(out);
    __builtin_amdgcn_sched_barrier(0);
    float* gw = sm.gb_s + wave * (U * 64);
    if (lane < U * 16) *(f32x4*)(gw + lane * 4) = gbv;
    f32x4 g4[U][2], b4[U][2];
#pragma unroll
    for (int i = 0; i < U; ++i)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        g4[i][hh] = *(const f32x4*)(gw + i * 32 + lq * 8 + 4 * hh);
        b4[i][hh] = *(const f32x4*)(gw + U * 32 + i * 32 + lq * 8 + 4 * hh);
      }
    __builtin_amdgcn_sched_barrier(0);
    float mw;                                    // mean of the wave's own columns; the registers then hold the distances to it
    {
      f32x4 s4 = f32x4{0.f, 0.f, 0.f, 0.f}, q4 = s4;
#pragma unroll
      for (int i = 0; i < U; ++i)
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) s4 += __builtin_bit_cast(f32x4, xv[i][hh]);
      const float s = sum_rows((s4[0] + s4[1]) + (s4[2] + s4[3]));
      mw = s * (1.f / (32 * U));
#pragma unroll
      for (int i = 0; i < U; ++i)
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          const f32x4 c = __builtin_bit_cast(f32x4, xv[i][hh]) - mw;
          xv[i][hh] = __builtin_bit_cast(u32x4, c);
#pragma unroll
          for (int r = 0; r < 4; ++r) q4[r] = fmaf(c[r], c[r], q4[r]);
        }
      const float q = sum_rows((q4[0] + q4[1]) + (q4[2] + q4[3]));
      if (lq == 0) sm.st_s[wave * 16 + lr] = make_float2(s, q);
    }
    __syncthreads();
    f32x4 qa[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) qa[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    {
      float mu, rs;
      row_moments<KSTEPS / U, 32 * U>(sm.st_s + lr, 16, qp.eps, mu, rs);      // (of the waves that have k-steps)
      const float off = (mw - mu) * rs;
#pragma unroll
      for (int i = 0; i < U; ++i) {
        float y[8];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          const f32x4 v = __builtin_bit_cast(f32x4, xv[i][hh]);
#pragma unroll
          for (int r = 0; r < 4; ++r) y[4 * hh + r] = fmaf(fmaf(v[r], rs, off), g4[i][hh][r], b4[i][hh][r]);
        }
        u32x4 yb = u32x4{cvt_pk_bf16(y[0], y[1]), cvt_pk_bf16(y[2], y[3]), cvt_pk_bf16(y[4], y[5]), cvt_pk_bf16(y[6], y[7])};
        if (U * NW != KSTEPS && !mine) yb = u32x4{0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < 4; ++j)
          qa[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf[j][i]), __builtin_bit_cast(bf16x8, yb), qa[j], 0, 0, 0);
      }
    }
    f32x4* red = &sm.o_s[0][0][0];               // [wave][column tile][lane], before the final merge uses it
#pragma unroll
    for (int j = 0; j < 4; ++j) red[(wave * 4 + j) * 64 + lane] = qa[j];
    __syncthreads();
    if (wave < 4) {                              // wave w finishes column tile w: a lane holds row lr, columns 16w + 4lq ..
      f32x4 part[NW];                            // (all reads under way before the first is waited for)
#pragma unroll
      for (int w = 0; w < NW; ++w) part[w] = red[(w * 4 + wave) * 64 + lane];
      __builtin_amdgcn_sched_barrier(0);
      f32x4 sum = part[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) sum += part[w];
#pragma unroll
      for (int r = 0; r < 4; ++r) sum[r] *= p.scale;       // (one by one: as a vector product the compiler keeps p.scale in scratch memory)
      const u32x2 hi = u32x2{cvt_pk_bf16(sum[0], sum[1]), cvt_pk_bf16(sum[2], sum[3])};
      const u32x2 lo = u32x2{cvt_pk_bf16(sum[0] - __uint_as_float(hi[0] << 16), sum[1] - __uint_as_float(hi[0] & 0xFFFF0000u)),
                             cvt_pk_bf16(sum[2] - __uint_as_float(hi[1] << 16), sum[3] - __uint_as_float(hi[1] & 0xFFFF0000u))};
      // operand lane 16 q + lr of half s holds columns 32 s + 8 q .. + 7
      const int at = ((wave >> 1) * 64 + ((wave & 1) * 2 + (lq >> 1)) * 16 + lr) * 2 + (lq & 1);
      sm.q_s[at] = hi; sm.q_s[256 + at] = lo;
    }
    __syncthreads();
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      qhi[s2] = __builtin_bit_cast(bf16x8, *(const u32x4*)&sm.q_s[(s2 * 64 + lane) * 2]);
      qlo[s2] = __builtin_bit_cast(bf16x8, *(const u32x4*)&sm.q_s[256 + (s2 * 64 + lane) * 2]);
    }
  } else {
    const rsrc_t qr = rsrc_of(p.Q + row * p.d, (unsigned)nrows * p.d * 4);
    const unsigned off = (lr * p.d + h * DH + 8 * lq) * 4;
    u32x4 qa[2][2];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) { qa[s2][0] = __builtin_amdgcn_raw_buffer_load_b128(qr, off + s2 * 128, 0, 0); qa[s2][1] = __builtin_amdgcn_raw_buffer_load_b128(qr, off + s2 * 128 + 16, 0, 0); }
    attn_load_kv<KVNT, G>(kr, vr, first + wave, nw, lane, kf, vf);
    lim = p.limit[b];
    out = (bf16_t*)p.out;
    if (ARGS) out = arg_now(out);
    __builtin_amdgcn_sched_barrier(0);            // every global load above is in flight before the first wait
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      const f32x4 q0 = __builtin_bit_cast(f32x4, qa[s2][0]), q1 = __builtin_bit_cast(f32x4, qa[s2][1]);
      const float v[8] = {q0[0] * p.scale, q0[1] * p.scale, q0[2] * p.scale, q0[3] * p.scale, q1[0] * p.scale, q1[1] * p.scale, q1[2] * p.scale, q1[3] * p.scale};
      split_bf16x8(v, qhi[s2], qlo[s2]);
    }
  }
  // (the results' row is b * p.R + r0; what lies past the last key only r0 of a causal block tells)
  if constexpr (PACKED) attention_mfma_core<KVNT, LIMF, QU>(p, sm, h, 0, tile, split, (int)row, nrows, nheads, nz, tid, nw, first, hop, kr, vr, kf, vf, qhi, qlo, lim, out);
  else attention_mfma_core<KVNT, LIMF, QU>(p, sm, h, b, tile, split, r0, nrows, nheads, nz, tid, nw, first, hop, kr, vr, kf, vf, qhi, qlo, lim, out);
}
// SLOTS: a step of a batch some of whose sequences may have ended (AttnP::seq); a kernel of its own, since looking the
// sequence up is one more round trip ahead of the K/V loads.
template <bool KVNT, bool LIMF, int QU, bool SLOTS, bool PACKED = false>
__device__ __forceinline__ void attention_mfma_entry(const AttnP& p, const QProjP& qp) {
  constexpr int NW = ATTN_WAVES, RT = 16;
  __shared__ f32x4 o_s[NW][4][64];
  __shared__ float m_s[NW][RT], l_s[NW][RT];
  __shared__ __attribute__((aligned(16))) u32x2 q_s[QU > 0 ? 512 : 1];
  __shared__ __attribute__((aligned(16))) float gb_s[QU > 0 ? NW * ((4 * QU + NW - 1) / NW) * 64 : 4];
  __shared__ float2 st_s[QU > 0 ? NW * 16 : 1];
  AttnLds sm;
  sm.o_s = o_s; sm.m_s = m_s; sm.l_s = l_s; sm.q_s = q_s; sm.gb_s = gb_s; sm.st_s = st_s;
  const int sb = SLOTS ? p.seq[blockIdx.y] : blockIdx.y;
  if (SLOTS && sb < 0) return;
  attention_mfma_body<KVNT, LIMF, QU, true, PACKED>(p, qp, sm, blockIdx.x, blockIdx.y, sb, blockIdx.z, gridDim.x, gridDim.z, threadIdx.x, QU > 0 ? NW : blockDim.x >> 6);
}
// (QU == 0: four or eight waves; QU < 0: four; otherwise eight)
template <bool KVNT, bool LIMF, int QU>
__global__ __launch_bounds__(64 * ATTN_WAVES) void attention_mfma_kernel(AttnP p, QProjP qp) { attention_mfma_entry<KVNT, LIMF, QU, false>(p, qp); }
template <bool KVNT, bool LIMF, int QU>
__global__ __launch_bounds__(64 * ATTN_WAVES) void attention_mfma_slots_kernel(AttnP p, QProjP qp) { attention_mfma_entry<KVNT, LIMF, QU, true>(p, qp); }
// The same with queries projected inside (QU > 1) for two sequences of up to 128 keys per workgroup: one reading of the head's weights serves two row tiles, and each half of the waves
// then has one of the sequences.  (One workgroup per sequence: with more than 128 of them the weights, 128 KB each at d = 1024, cost more than the kernels saved.)
// A wave normalises whole rows, half a line of eight places at a time, and the operands are read out of the LDS: as operands straight from the rows in memory a load touches 64 lines, which the
// L1 looks up one by one (64 cycles instead of 16: of 20 rows the last wave had its sums 4 us after the launch).
// Every sum is taken in the order of row_gemm_kernel with LayerNorm inside: moments of 128 columns by four lanes each, products of 128 of K one behind the other, these parts in turn.  Up to
// where that kernel is the other way (lean_fuse()) the queries have its bits.
template <int QU>
struct AttnPairsLds {
  static constexpr int K = 128 * QU, XS = 32 * (K + 8) * 2, RED = QU * 8 * 64 * 16, QS = 2 * 512 * 8, ML = 2 * ATTN_WAVES * 16 * 4;
  static constexpr int BYTES = XS + RED + QS + ML;
  static_assert(RED >= 2 * (int)AttnLds::OS_BYTES && QS >= 32 * QU * 8, "the halves' results; a row's moments");
};
template <int QU, bool SLOTS>
__global__ __launch_bounds__(64 * ATTN_WAVES) void attention_mfma_pairs_kernel(AttnP p, QProjP qp, int B) {
  // parts of 128 columns, of U k-steps; row tiles per wave; rows that a wave normalises at once, and how often
  constexpr int NW = ATTN_WAVES, K = 128 * QU, U = 4, KSTEPS = QU * U, TW = 2 * QU / NW, RW = 16 / QU, PASSES = 32 / (NW * RW);
  static_assert(TW * NW == 2 * QU && PASSES * NW * RW == 32, "every wave has a part and row tiles, every row lanes");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  using Lds = AttnPairsLds<QU>;
  bf16_t* xs = (bf16_t*)smem_raw;                // normalised rows, K + 8 apart, k-step i of part w at i ^ (w & 3): the pieces that 16 lanes store lie in different banks
  f32x4* red = (f32x4*)(smem_raw + Lds::XS);     // partial sums [part][row tile, column tile][lane]; then the halves' results, as AttnLds
  u32x2* q_s = (u32x2*)(smem_raw + Lds::XS + Lds::RED);
  float (*m_s)[16] = (float (*)[16])(smem_raw + Lds::XS + Lds::RED + Lds::QS), (*l_s)[16] = m_s + NW;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = wave >> 2;
  const int lr = lane & 15, lq = lane >> 4, h = blockIdx.x, b0 = 2 * blockIdx.y, b = b0 + half, there = b0 + 1 < B ? 2 : 1;
  const int bc = half < there ? b : b0;
  int sb = half < there ? b : -1;
  if (SLOTS) {
    const int s0 = p.seq[b0], s1 = there > 1 ? p.seq[b0 + 1] : -1;
    if (s0 < 0 && s1 < 0) return;                // (the whole workgroup)
    sb = half ? s1 : s0;
  }
  const int kg = wave % QU, t0 = wave / QU * TW, ks0 = kg * U, rows = __builtin_amdgcn_readfirstlane(there * p.R);
  // every load of the kernel but keys and values: rows of x first (those past the last: zeros).  A lane has k-steps of eight columns of a part, as the operands are
  const int part = (lane >> 2) % QU, pq = lane & 3, row0 = wave * RW + (lane >> 2) / QU, at = part * 128 + pq * 8;
  f32x4 v[PASSES][U][2], gb[U][2];               // (gain in the lower half of the lanes, bias in the upper one)
  const rsrc_t xr = rsrc_of(qp.x + (size_t)b0 * p.R * K, (unsigned)rows * K * 4);
#pragma unroll
  for (int n = 0; n < PASSES; ++n) {
    if ((wave + NW * n) * RW >= rows) break;
#pragma unroll
    for (int i = 0; i < U; ++i)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) v[n][i][hh] = __builtin_bit_cast(f32x4, buf_load16(xr, (unsigned)((row0 + NW * RW * n) * K + at + i * 32 + hh * 4) * 4, 0));
  }
#pragma unroll
  for (int i = 0; i < U; ++i)
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) gb[i][hh] = *(const f32x4*)((lane < 32 ? qp.g : qp.b) + at + i * 32 + hh * 4);
  int lim = p.limit[bc];
  u32x4 wf[4][U];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < U; ++i) wf[j][i] = *(const u32x4*)((const char*)qp.W + ((size_t)(4 * h + j) * KSTEPS + ks0 + i) * 1024 + lane * 16);
  bf16_t* out = arg_now((bf16_t*)p.out);
  __builtin_amdgcn_sched_barrier(0);
  // K and V of this half's sequence
  lim = sb < 0 || lim < 0 ? 0 : __builtin_amdgcn_readfirstlane(lim);
  const int glim = (lim + 31) >> 5 < p.capg ? (lim + 31) >> 5 : p.capg;
  const size_t head_at = ((size_t)(sb < 0 ? 0 : sb) * gridDim.x + h) * p.capg * KV_GROUP;
  const rsrc_t kr = rsrc_of((const bf16_t*)p.Kc + head_at, (unsigned)glim * (KV_GROUP * 2));
  const rsrc_t vr = rsrc_of((const bf16_t*)p.Vc + head_at, (unsigned)glim * (KV_GROUP * 2));
  u32x4 kf[1][4], vf[1][4];
  attn_load_kv<false, 1>(kr, vr, wave & 3, 4, lane, kf, vf);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int n = 0; n < PASSES; ++n) {
    if ((wave + NW * n) * RW >= rows) break;
    float2* const st = (float2*)q_s + (row0 + NW * RW * n) * QU;       // (of this wave's rows: written and read by it alone)
    f32x4 s4 = f32x4{0.f, 0.f, 0.f, 0.f}, q4 = s4;
#pragma unroll
    for (int i = 0; i < U; ++i)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) s4 += v[n][i][hh];
    const float s = quad_sum((s4[0] + s4[1]) + (s4[2] + s4[3])), mw = s * (1.f / 128);
#pragma unroll
    for (int i = 0; i < U; ++i)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        v[n][i][hh] -= mw;
#pragma unroll
        for (int r = 0; r < 4; ++r) q4[r] = fmaf(v[n][i][hh][r], v[n][i][hh][r], q4[r]);
      }
    const float q = quad_sum((q4[0] + q4[1]) + (q4[2] + q4[3]));
    if (pq == 0) st[part] = make_float2(s, q);
    __builtin_amdgcn_wave_barrier();
    float mu, rs;
    row_moments<QU, 128>(st, 1, qp.eps, mu, rs);
    const float off = (mw - mu) * rs;
#pragma unroll
    for (int i = 0; i < U; ++i) {
      float y[8];
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(gb[i][hh][r]), __float_as_uint(gb[i][hh][r]), false, false);
          y[4 * hh + r] = fmaf(fmaf(v[n][i][hh][r], rs, off), __uint_as_float(w[0]), __uint_as_float(w[1]));
        }
      *(u32x4*)(xs + (row0 + NW * RW * n) * (K + 8) + part * 128 + (i ^ (part & 3)) * 32 + pq * 8) =
          u32x4{cvt_pk_bf16(y[0], y[1]), cvt_pk_bf16(y[2], y[3]), cvt_pk_bf16(y[4], y[5]), cvt_pk_bf16(y[6], y[7])};
    }
  }
  lk_barrier();
  f32x4 qa[TW][4];
  const bf16_t* row[TW];                         // (rows past the last: the last)
#pragma unroll
  for (int t = 0; t < TW; ++t) {
    const int m = (t0 + t) * p.R + (lr < p.R ? lr : p.R - 1);
    row[t] = xs + (m < rows ? m : rows - 1) * (K + 8) + ks0 * 32 + lq * 8;
#pragma unroll
    for (int j = 0; j < 4; ++j) qa[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int i = 0; i < U; ++i)
#pragma unroll
    for (int t = 0; t < TW; ++t) {
      const bf16x8 x8 = __builtin_bit_cast(bf16x8, *(const u32x4*)(row[t] + (i ^ (kg & 3)) * 32));
#pragma unroll
      for (int j = 0; j < 4; ++j) qa[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf[j][i]), x8, qa[t][j], 0, 0, 0);
    }
#pragma unroll
  for (int t = 0; t < TW; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j) red[(kg * 8 + (t0 + t) * 4 + j) * 64 + lane] = qa[t][j];
  lk_barrier();
  {                                              // wave 4 t + j finishes column tile j of row tile t
    f32x4 part[QU];
#pragma unroll
    for (int w = 0; w < QU; ++w) part[w] = red[(w * 8 + wave) * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
    f32x4 sum = part[0];
#pragma unroll
    for (int w = 1; w < QU; ++w) sum += part[w];
#pragma unroll
    for (int r = 0; r < 4; ++r) sum[r] *= p.scale;
    u32x2 hi, lo;
    lk_halves(sum, hi, lo);
    const int j = wave & 3, at = half * 512 + ((j >> 1) * 64 + ((j & 1) * 2 + (lq >> 1)) * 16 + lr) * 2 + (lq & 1);       // (as in attention_mfma_body)
    q_s[at] = hi; q_s[256 + at] = lo;
  }
  lk_barrier();
  bf16x8 qhi[2], qlo[2];
#pragma unroll
  for (int s2 = 0; s2 < 2; ++s2) {
    qhi[s2] = __builtin_bit_cast(bf16x8, *(const u32x4*)&q_s[half * 512 + (s2 * 64 + lane) * 2]);
    qlo[s2] = __builtin_bit_cast(bf16x8, *(const u32x4*)&q_s[half * 512 + 256 + (s2 * 64 + lane) * 2]);
  }
  AttnLds sm = AttnLds::carve((unsigned char*)(red + half * (4 * 4 * 64)));
  sm.m_s = m_s + half * 4; sm.l_s = l_s + half * 4;
  attention_mfma_core<false, false, 0, 1, ATTN_PLAIN, true>(p, sm, h, b, 0, 0, 0, sb < 0 ? 0 : p.R, gridDim.x, 1, threadIdx.x & 255, 4, 0, 4, kr, vr, kf, vf, qhi, qlo, lim, out);
}
// Source rows of up to 128 keys: a wave has all keys and values of its (sequence, head) in registers and `per` row tiles of 16 in turn, the next one's queries under way
// meanwhile.  With the keys dealt to four waves, as above, a launch of many tiles is bound by instructions, half of them the softmax's exchange between lanes and
// the waves' meeting, which here come once per 128 keys and not at all.  No LDS, no barrier.  32 sequences of 128 tokens, 16 heads, 8 row tiles: 20.6 us dealt to waves (with a
// workgroup's keys and values kept for four tiles 21.8: not what bounds it), 12.6 here; launches of few tiles wait for one wave's chain instead: 4 x 40 tokens, 8 heads 4.2, 4.8,
// 5 x 50, 16 heads 4.7, 5.7.
// PACKED: as in attention_mfma_body.
template <bool PACKED>
__global__ __launch_bounds__(256, 2) void attention_mfma_tiles_kernel(AttnP p, int per) {
  constexpr int RT = 16, DH = 64, G = 4;
  const int h = blockIdx.x, b = blockIdx.y, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lr = lane & 15, lq = lane >> 4;
  const int len = p.limit[b], rows = PACKED ? len : p.R, first = (blockIdx.z * 4 + wave) * per;
  const long row0 = PACKED ? p.row0[b] : (long)b * p.R;
  const int end = min(first + per, (rows + RT - 1) / RT);
  if (first >= end) return;
  const int cap = min(p.capg, G) * 32, lim = len < 0 ? 0 : (len < cap ? len : cap), ngr = (lim + 31) >> 5;
  const size_t head_at = ((size_t)b * gridDim.x + h) * p.capg * KV_GROUP;
  const rsrc_t kr = rsrc_of((const bf16_t*)p.Kc + head_at, (unsigned)ngr * (KV_GROUP * 2)), vr = rsrc_of((const bf16_t*)p.Vc + head_at, (unsigned)ngr * (KV_GROUP * 2));
  const rsrc_t qr = rsrc_of(p.Q + row0 * p.d, (unsigned)rows * p.d * 4);
  u32x4 qa[4], kf[G][4], vf[G][4];
  auto queries = [&](int tile) {
#pragma unroll
    for (int i = 0; i < 4; ++i) qa[i] = buf_load16(qr, ((tile * RT + lr) * p.d + h * DH + 8 * lq) * 4 + (i >> 1) * 128 + (i & 1) * 16, 0);
  };
  queries(first);
#pragma unroll
  for (int g = 0; g < G; ++g) {
    if (g >= ngr) continue;                      // (the same for the whole wave, as every test of g below)
#pragma unroll
    for (int x = 0; x < 4; ++x) { kf[g][x] = buf_load16(kr, lane * 16 + x * 1024, g * (KV_GROUP * 2)); vf[g][x] = buf_load16(vr, lane * 16 + x * 1024, g * (KV_GROUP * 2)); }
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int g = 0; g < G; ++g)
    if (g < ngr && 32 * g + 32 > lim) {          // values of keys past the last one: their probabilities are zero, their bits unknown
      const int left = lim - 32 * g - 8 * lq;    // of this lane's eight
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int w = 0; w < 4; ++w) vf[g][dt][w] = left > 2 * w + 1 ? vf[g][dt][w] : (left > 2 * w ? vf[g][dt][w] & 0xFFFFu : 0u);
    }
#pragma unroll 1
  for (int tile = first; tile < end; ++tile) {
    bf16x8 qhi[2], qlo[2];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      const f32x4 q0 = __builtin_bit_cast(f32x4, qa[2 * s2]), q1 = __builtin_bit_cast(f32x4, qa[2 * s2 + 1]);
      const float v[8] = {q0[0] * p.scale, q0[1] * p.scale, q0[2] * p.scale, q0[3] * p.scale, q1[0] * p.scale, q1[1] * p.scale, q1[2] * p.scale, q1[3] * p.scale};
      split_bf16x8(v, qhi[s2], qlo[s2]);
    }
    if (tile + 1 < end) queries(tile + 1);
    // scores: s[g][t][r] = key 32 g + 8 lq + 4 t + r against query row lr
    f32x4 s[G][2];
    float mx = -INFINITY;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (g >= ngr) continue;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f}, al = a;       // (two chains)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          const bf16x8 ka = __builtin_bit_cast(bf16x8, kf[g][2 * t + s2]);
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qhi[s2], a, 0, 0, 0);
          al = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qlo[s2], al, 0, 0, 0);
        }
        s[g][t] = a + al;
      }
      if (32 * g + 32 > lim)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) s[g][t][r] = 32 * g + 8 * lq + 4 * t + r < lim ? s[g][t][r] : -INFINITY;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx = fmaxf(mx, s[g][t][r]);
    }
    mx = max_rows(mx);
    float sum = 0.f;
    f32x4 acc[4];                                // out^T tile dt: head dimensions 16 dt + 4 lq + r, row lr
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (g >= ngr) continue;
      float pv[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) { pv[i] = __expf(s[g][i >> 2][i & 3] - mx); sum += pv[i]; }
      bf16x8 phi, plo;
      split_bf16x8(pv, phi, plo);
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        const bf16x8 va = __builtin_bit_cast(bf16x8, vf[g][dt]);
        acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, phi, acc[dt], 0, 0, 0);
        acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, plo, acc[dt], 0, 0, 0);
      }
    }
    sum = sum_rows(sum);
    float inv = __builtin_amdgcn_rcpf(sum);
    inv = inv * fmaf(-sum, inv, 2.f);            // (one Newton step: the quotient to fp32)
    if (tile * RT + lr < rows) {
      bf16_t* to = (bf16_t*)p.out + attn_out_at<bf16_t>(p, row0 + tile * RT + lr, h * DH + 4 * lq);
      const int on = p.packed ? 256 : 16;        // 16 dimensions on
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) *(u32x2*)(to + dt * on) = u32x2{cvt_pk_bf16(acc[dt][0] * inv, acc[dt][1] * inv), cvt_pk_bf16(acc[dt][2] * inv, acc[dt][3] * inv)};
    }
  }
}
// Source rows that lie one sequence behind the other (encoder of a ragged batch)
template <int QU>
__global__ __launch_bounds__(64 * ATTN_WAVES) void attention_mfma_packed_kernel(AttnP p, QProjP qp) { attention_mfma_entry<false, true, QU, false, true>(p, qp); }
