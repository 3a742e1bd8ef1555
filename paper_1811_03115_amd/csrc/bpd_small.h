// Small fp32 models: a whole encode, and a whole decode, of a sequence in one workgroup.  Included by bpd_kernels.h.
//
// A step of a two-layer, 64-wide model is some 27 dependent kernels of 2 .. 10 us, 125 us in all, for 1 MB of weights and 1.2
// million multiply-adds: launches and nothing else.  Sequences do not depend on each other, so one workgroup of eight waves
// takes a sequence through all its steps: activations in LDS, weights out of the L2 (they stay there), barriers instead
// of launches.  What bounds it is the number of dependent phases (eight per layer: the partial sums' meeting in LDS, two barriers) and, within
// them, instructions at two waves per SIMD: every phase is one copy of the same code, driven by a table in LDS.  The products run on
// v_mfma_f32_4x4x1_16b, fp32, with weights as they come from memory 16 bytes a lane, requested a phase ahead (small_load, SmallFetch).  A
// step of 4 rows at d = 64, two layers, takes 88,000 cycles: 2,200 .. 5,300 a phase, 8,400 and 7,000 the heads' two (512 KB of weights at the
// 64 bytes a cycle that a CU gets: 8,200 together), 8,300 the scores (fp32 matrix rate: 2,000).  (Loads of 4 bytes a lane behind the barrier: 125,000.  Plain
// multiply-adds, with 16 LDS reads of the rows for 64 of them, took 80 us instead of 68 before that.)
#pragma once

constexpr int SMALL_T = 512, SMALL_W = SMALL_T / 64;      // threads and waves of the workgroup
struct SmallLayerP { const float *wqkv, *wo, *cq, *co, *ckv, *w1, *w2, *b1, *b2, *ln1g, *ln1b, *ln2g, *ln2b, *ln3g, *ln3b; };
struct SmallP {
  StateP s;
  int d, F, V, heads, n_enc, n_dec, max_src, slots, S;
  float eps, escale, qscale;
  int local_q, local_m;
  SmallLayerP enc, dec;                    // of the first layer; the others lie enc_stride / dec_stride floats on
  long enc_stride, dec_stride;
  const float *enc_g, *enc_b, *dec_g, *dec_b, *hw1, *hb1, *hw2, *hb2, *emb, *emb_t, *pos_src, *pos_tgt;
  float *selfK, *selfV, *crossK, *crossV, *qe, *ke, *ve;
  long self_layer, src_layer;              // floats per layer of the caches
  const int* src_ids;
  // decode
  int k, steps, hgroup, top_n;             // hgroup: heads whose hidden layers are in LDS together
  int* accepted_out;
  float* logits;                           // not null: one invocation's scores [B * k][k][V]; nothing is accepted
};

// The table: one entry per phase
enum { SD_W = 0, SD_BIAS = 2, SD_G = 4, SD_GB = 6, SD_P0 = 8, SD_P1 = 10, SD_P2 = 12, SD_N = 14, SD_K, SD_LDW, SD_X, SD_LDX, SD_DST, SD_LDO, SD_MODE, SD_NCB, SD_INV,
       SD_SLICES, SD_KN, SD_GW, SD_WG, SD_XG, SD_XN, SD_WORDS = 32 };
// STORE, RELU: dst = X W + bias (ReLU);  ADD: dst += ...;  QKV: queries to dst or P2, keys and values to the rows at P0, P1;  KV: without queries;
// HEAD: dst[row * k + head] = ... + LayerNorm(x);  SELF, CROSS: attention;  NORM: LayerNorm of its own (d > 64: otherwise part of the phase that
// finishes the rows)
enum { SM_STORE, SM_RELU, SM_ADD, SM_QKV, SM_KV, SM_HEAD, SM_SELF, SM_CROSS, SM_NORM };

// Offsets of LDS regions in floats.  Rows are d + 4 (F + 4, ..) floats apart: four rows are read at once.
struct SmallLds { int x, xn, att, big, o, red, z, best, misc, table, total; };
__host__ __device__ inline SmallLds small_lds(int d, int F, int V, int rows, int k, int hgroup, int xrows, bool topn, int phases) {
  SmallLds n;
  const int r4 = (rows + 3) / 4 * 4, wide = 3 * d > F * hgroup ? 3 * d : F * hgroup;
  n.x = 0;
  n.xn = n.x + (xrows > r4 ? xrows : r4) * (d + 4);
  n.att = n.xn + r4 * (d + 4);
  n.big = n.att + r4 * (d + 4);
  n.o = n.big + r4 * (wide + 4);
  n.red = n.o + ((rows * k + 15) / 16 * 16) * (d + 4);
  n.z = n.red + SMALL_W * 4 * 64 * 4;      // [wave][row quad][lane] of four floats
  n.best = n.z + (topn ? rows * V : 0);
  n.best = (n.best + 3) / 4 * 4;
  n.misc = n.best + 512 + SMALL_W * 32;    // best keys [256] and, per wave and row, the candidates (value, column)
  n.table = n.misc + 64;
  n.total = n.table + phases * SD_WORDS;
  return n;
}

// The thread's index, opaque where it is asked for: otherwise what the phases derive from it is computed ahead of their loop and kept in
// registers, more of them than there are.
__device__ __forceinline__ int small_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}
// The kernel's arguments, likewise: read where they are used (a scalar load) instead of all ahead of the loops, where a hundred pointers
// found no registers and went through vector lanes at every use.
__device__ __forceinline__ const SmallP& small_args() {
  auto q = (const __attribute__((address_space(4))) SmallP*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(q));
  return *(const SmallP*)q;
}
// Reductions over the wave of four values at once.  First over the four 16-lane rows, which leaves value i in row i (three exchanges instead of eight)
template <typename T, typename Op>
__device__ __forceinline__ T small_rows4(T v0, T v1, T v2, T v3, Op op) {
  auto pair = [&](bool half, T a, T b) {
    const unsigned x = __builtin_bit_cast(unsigned, a), y = __builtin_bit_cast(unsigned, b);
    const auto r = half ? __builtin_amdgcn_permlane32_swap(x, y, false, false) : __builtin_amdgcn_permlane16_swap(x, y, false, false);
    return op(__builtin_bit_cast(T, (unsigned)r[0]), __builtin_bit_cast(T, (unsigned)r[1]));
  };
  const T a = pair(true, v0, v2), b = pair(true, v1, v3);
  return pair(false, a, b);
}
template <int CTRL, typename T> __device__ __forceinline__ T small_dpp(T v) { return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true)); }
template <typename T, typename Op>
__device__ __forceinline__ void small_wave4(T (&v)[4], Op op) {
  T r = small_rows4(v[0], v[1], v[2], v[3], op);
  r = op(r, small_dpp<0xB1>(r)); r = op(r, small_dpp<0x4E>(r)); r = op(r, small_dpp<0x141>(r)); r = op(r, small_dpp<0x140>(r));
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, r), 16 * i));
}
struct SmallAdd { template <typename T> __device__ __forceinline__ T operator()(T a, T b) const { return a + b; } };
struct SmallMax { template <typename T> __device__ __forceinline__ T operator()(T a, T b) const { return a > b ? a : b; } };

// Fills a table entry (one thread)
struct SmallEntry {
  int* e;
  __device__ __forceinline__ void ptr(int i, const void* p) { e[i] = (int)(unsigned)(unsigned long long)p; e[i + 1] = (int)(unsigned)((unsigned long long)p >> 32); }
  __device__ __forceinline__ void gemm(int mode, const float* W, int ldw, int N, int K, const float* bias, int X, int ldx, int dst, int ldo) {
    const int ncb = (N + 63) / 64, per = ncb < SMALL_W ? ncb : SMALL_W;
    int slices = SMALL_W / per;
    while (slices > 1 && K % (16 * slices)) --slices;
    ptr(SD_W, W); ptr(SD_BIAS, bias); ptr(SD_G, nullptr); ptr(SD_GB, nullptr); ptr(SD_P0, nullptr); ptr(SD_P1, nullptr); ptr(SD_P2, nullptr);
    e[SD_N] = N; e[SD_K] = K; e[SD_LDW] = ldw; e[SD_X] = X; e[SD_LDX] = ldx; e[SD_DST] = dst; e[SD_LDO] = ldo; e[SD_MODE] = mode;
    e[SD_NCB] = ncb; e[SD_INV] = 65536 / per + 1; e[SD_SLICES] = slices; e[SD_KN] = K / slices; e[SD_GW] = 0; e[SD_WG] = 0; e[SD_XG] = 0; e[SD_XN] = -1;
  }
  // the rows that a phase finishes pass through LayerNorm into xn (one wave has whole rows: d <= 64)
  __device__ __forceinline__ void norm(const float* g, const float* b, int xn) { ptr(SD_G, g); ptr(SD_GB, b); e[SD_XN] = xn; }
};
#define BPD_SD(i) __builtin_amdgcn_readlane(dv, i)
// (global pointers: put together from a table they would otherwise be flat ones, whose loads also wait for LDS)
typedef __attribute__((address_space(1))) float gfloat;
typedef __attribute__((address_space(1))) f32x4 gfloat4;
__device__ __forceinline__ gfloat* small_ptr(int lo, int hi) { return (gfloat*)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo); }
#define BPD_SDP(i) small_ptr(BPD_SD(i), BPD_SD((i) + 1))

// LayerNorm of a row that a wave holds (four columns per lane, zeros past d): into out
__device__ __forceinline__ void small_norm_row(const float (&v)[4], float* out, int d, int lane, const gfloat* g, const gfloat* b, float eps) {
  float s = 0.f, q = 0.f, gv[4], bv[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = lane + 64 * i;
    gv[i] = c < d ? g[c] : 0.f; bv[i] = c < d ? b[c] : 0.f;
    s += v[i];
  }
  const float mu = wave_sum(s) / d;
#pragma unroll
  for (int i = 0; i < 4; ++i) q += lane + 64 * i < d ? (v[i] - mu) * (v[i] - mu) : 0.f;
  const float rs = 1.0f / sqrtf(wave_sum(q) / d + eps);
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (lane + 64 * i < d) out[lane + 64 * i] = (v[i] - mu) * rs * gv[i] + bv[i];
}

// kv_at: cache row of the block's first row; x_at: where the tile being worked on lies in x (encoder)
struct SmallCtx { float* lds; int red, xn, d, k, heads, L, src, local_q, local_m, kv_at, x_at; float eps, qscale; };

// How a wave's 64 columns x 16 rows of weights lie in its registers: load t of four brings, 16 bytes a lane, row 4 (lane / 16) + t of columns
// 4 (lane % 16) ..  An instruction multiplies one column of every lane: its sixteen blocks of four lanes have different k, so the rows' operand is
// one 16-byte LDS read per lane for all sixteen k, and the row of 16 lanes g has the sums over k = 4 g ..; the exchange that adds the four up leaves
// column 4 (lane % 16) + lane / 16 in the lane.  (A load of one row of 64 columns, 4 bytes a lane, at a time: 16 loads and 4 LDS reads for the same,
// 1000 instead of 250 cycles.)
__device__ __forceinline__ int small_col(int lane) { return (lane & 15) * 4 + (lane >> 4); }

// What a wave brings along into a phase, requested while the phase before still meets in LDS: its row of the table, its first sixteen rows of
// weights, where they lie, and bias and gains of the column that it will finish
struct SmallFetch { int dv, s, cb, xo; unsigned at; f32x4 w[4]; float bias, g, b; };

__device__ __forceinline__ void small_load(const rsrc_t& wr, unsigned at, int ldw, f32x4 (&w)[4]) {
#pragma unroll
  for (int t = 0; t < 4; ++t) w[t] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(wr, at, t * ldw * 4, 0));
}
// Slice s of column block cb of an entry's matrix: the lane's first byte, and where its part of x lies behind the row's start
__device__ __forceinline__ unsigned small_column(int dv, int cb, int s, int lane, int& xo) {
  const int N = BPD_SD(SD_N), gw = BPD_SD(SD_GW), k = s * BPD_SD(SD_KN) + (lane >> 4) * 4, col = cb * 64 + (lane & 15) * 4;
  int c = col < N ? col : N - 4;
  xo = k;
  if (gw) { const int h = (int)(((float)c + 0.5f) * __builtin_amdgcn_rcpf((float)gw)); c += h * (BPD_SD(SD_WG) - gw); xo += h * BPD_SD(SD_XG); }
  return (unsigned)(c + k * BPD_SD(SD_LDW)) * 4;
}
// The pair (column block, row quad) that a wave finishes first, counted from the last wave: where the product leaves waves idle they finish
__device__ __forceinline__ int small_pair(int wave) { return SMALL_W - 1 - wave; }
template <int RQ>
__device__ __forceinline__ void small_fetch(const SmallCtx& m, int dv, SmallFetch& f) {
  const int tid = small_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  f.dv = dv;
  if (BPD_SD(SD_MODE) >= SM_SELF) return;
  const int N = BPD_SD(SD_N), slices = BPD_SD(SD_SLICES), ncb = BPD_SD(SD_NCB);
  f.s = slices == 1 ? 0 : (wave * BPD_SD(SD_INV)) >> 16;
  f.cb = wave - f.s * ncb;
  if (f.s < slices && f.cb < ncb) {
    f.at = small_column(dv, f.cb, f.s, lane, f.xo);
    small_load(rsrc_of((const void*)BPD_SDP(SD_W), 0x7FFFFFFF), f.at, BPD_SD(SD_LDW), f.w);
  }
  const int col = (slices == 1 ? f.cb : small_pair(wave) / RQ) * 64 + small_col(lane), c = col < N ? col : 0;
  const gfloat* bias = BPD_SDP(SD_BIAS);
  f.bias = 0.f;
  if (bias) f.bias = bias[c];
  if (BPD_SD(SD_XN) >= 0) { f.g = BPD_SDP(SD_G)[c]; f.b = BPD_SDP(SD_GB)[c]; }
}

// Four rows (4 q ..) of one column, finished: v = X W.  (Rows past the last: there is room for whole quads everywhere but in the caches and in o.)
__device__ __forceinline__ void small_finish(const SmallCtx& m, int dv, int mode, int rows, int q, int col, float bias, float gv, float bv, f32x4 v, int lane) {
  float* lds = m.lds;
  const int d = m.d, N = BPD_SD(SD_N), dst = BPD_SD(SD_DST), ldo = BPD_SD(SD_LDO), xn = BPD_SD(SD_XN);
  const bool in = col < N;
  if (mode == SM_QKV || mode == SM_KV) {
    const int c = mode == SM_KV ? col + d : col;
    gfloat *q2 = BPD_SDP(SD_P2), *k0 = BPD_SDP(SD_P0), *v0 = BPD_SDP(SD_P1);
    if (c < d && !q2) {
      float* at = lds + dst + 4 * q * ldo + c;
#pragma unroll
      for (int i = 0; i < 4; ++i) at[i * ldo] = v[i];
    } else if (in) {
      gfloat* at = (c < d ? q2 + c : (c < 2 * d ? k0 + (c - d) : v0 + (c - 2 * d))) + (long)(m.kv_at + 4 * q) * d;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (4 * q + i < rows) at[i * d] = v[i];
    }
    return;
  }
  f32x4 t = v + bias;
  if (mode == SM_HEAD) {
    const int h = (int)(((float)col + 0.5f) * __builtin_amdgcn_rcpf((float)d)), c = col - h * d;
    const float* x = lds + m.xn + 4 * q * (d + 4) + c;
    float xv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) xv[i] = x[i * (d + 4)];
    float* at = lds + dst + (4 * q * m.k + h) * ldo + c;
    if (in) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (4 * q + i < rows) at[i * m.k * ldo] = t[i] + xv[i];
    }
    return;
  }
  float* at = lds + dst + (mode == SM_ADD ? m.x_at : 0) + 4 * q * ldo + (in ? col : 0);
  if (mode == SM_RELU) {
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = fmaxf(t[i], 0.f);
  }
  if (mode == SM_ADD) {
    f32x4 x;
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = at[i * ldo];
    t += x;
  }
  if (in) {
#pragma unroll
    for (int i = 0; i < 4; ++i) at[i * ldo] = t[i];
  }
  if (xn >= 0) {                                 // four rows at once: their reductions overlap
    const float inv = 1.0f / d;
    float mu[4], va[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) mu[i] = in ? t[i] : 0.f;
    small_wave4(mu, SmallAdd());
#pragma unroll
    for (int i = 0; i < 4; ++i) { mu[i] = fmaf(-mu[i], inv, t[i]); va[i] = in ? mu[i] * mu[i] : 0.f; }
    small_wave4(va, SmallAdd());
    float* out = lds + xn + 4 * q * (d + 4) + (in ? col : 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x = fmaf(va[i], inv, m.eps), r0 = __builtin_amdgcn_rsqf(x), rs = r0 * fmaf(-0.5f * x * r0, r0, 1.5f);
      va[i] = mu[i] * rs * gv + bv;
    }
    if (in) {
#pragma unroll
      for (int i = 0; i < 4; ++i) out[i * (d + 4)] = va[i];
    }
  }
}

// X W of one wave: 64 columns and kn (sixteens) of the k, 4 RQ rows.  w: the first sixteen rows of weights, which `at` (small_column) starts at;
// x: the lane's row and k
template <int RQ>
__device__ __forceinline__ void small_product(const rsrc_t& wr, unsigned at, int ldw, const float* x, int ldx, int kn, f32x4 (&w)[4], f32x4 (&out)[RQ]) {
  f32x4 acc[RQ][4];
#pragma unroll
  for (int q = 0; q < RQ; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[q][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int left = kn;;) {
    f32x4 next[4], xv[RQ];                       // (the next sixteen rows on their way meanwhile)
    left -= 16;
    at += 64 * ldw;
    if (left > 0) small_load(wr, at, ldw, next);
#pragma unroll
    for (int q = 0; q < RQ; ++q) xv[q] = *(const f32x4*)(x + 4 * q * ldx);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int q = 0; q < RQ; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[q][i] = __builtin_amdgcn_mfma_f32_4x4x1f32(xv[q][t], w[t][i], acc[q][i], 0, 0, 0);
    if (left <= 0) break;
    x += 16;
#pragma unroll
    for (int t = 0; t < 4; ++t) w[t] = next[t];
  }
#pragma unroll
  for (int q = 0; q < RQ; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) out[q][r] = small_rows4(acc[q][0][r], acc[q][1][r], acc[q][2][r], acc[q][3][r], SmallAdd());
}
// The sum of the slices' partial results at red[at], `step` apart
__device__ __forceinline__ f32x4 small_partials(const f32x4* red, int slices, int step) {
  f32x4 v[4];                                    // (all reads of four under way together)
#pragma unroll
  for (int t = 0; t < 4; ++t) v[t] = red[(t < slices ? t : 0) * step];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int t = 1; t < 4; ++t)
    if (t < slices) v[0] += v[t];
#pragma unroll 1
  for (int t = 4; t < slices; ++t) v[0] += red[t * step];
  return v[0];
}

// The keys of small_attention
template <int NI>
__device__ __forceinline__ void small_keys(const SmallCtx& m, const rsrc_t& kr, const rsrc_t& vr, int span, const int (&k0)[2], const int (&k1)[2], const int (&h)[2], int lane,
                                           const f32x4 (&qv)[2], f32x4 (&acc)[2], float (&l)[2]) {
  const int d = m.d, dim = (lane & 3) * 4;
  float mx[2] = {-INFINITY, -INFINITY};
#pragma unroll 1
  for (int s0 = 0; s0 < span; s0 += 16 * NI) {
    f32x4 kv[2][NI], vv[2][NI];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int key = k0[u] + s0 + 16 * i + (lane >> 2);
        const unsigned at = (unsigned)((key < k1[u] ? key : k1[u] - 1) * d + h[u] * 16 + dim) * 4;
        kv[u][i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(kr, at, 0, 0));
        vv[u][i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(vr, at, 0, 0));
      }
    __builtin_amdgcn_sched_barrier(0);
    float sc[2][NI], top[2];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        float v = qv[u][0] * kv[u][i][0];
#pragma unroll
        for (int e = 1; e < 4; ++e) v = fmaf(qv[u][e], kv[u][i][e], v);
        v += small_dpp<0xB1>(v);
        v += small_dpp<0x4E>(v);
        sc[u][i] = k0[u] + s0 + 16 * i + (lane >> 2) < k1[u] ? v * m.qscale : -INFINITY;      // (a pair that is done: nothing but these, and its maximum stays)
      }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      top[u] = sc[u][0];
#pragma unroll
      for (int i = 1; i < NI; ++i) top[u] = fmaxf(top[u], sc[u][i]);
      top[u] = fmaxf(top[u], small_dpp<0x124>(top[u]));         // (row_ror: the other quads of the row)
      top[u] = fmaxf(top[u], small_dpp<0x128>(top[u]));
      top[u] = max_rows(top[u]);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const float mn = fmaxf(mx[u], top[u]), a = __expf(mx[u] - mn);
      mx[u] = mn;
      l[u] *= a; acc[u] *= a;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const float p = __expf(sc[u][i] - mn);
        l[u] += p;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[u][e] = fmaf(p, vv[u][i][e], acc[u][e]);
      }
    }
  }
}
// Attention of 16-wide heads, a wave per two (head, row) pairs, whose chains overlap.  16 NI keys at a time: four lanes have a key's sixteen numbers, load
// i brings keys 16 i + lane / 4, and a lane keeps the probabilities of its NI keys for its four dimensions of their values.  (A lane per key and 16
// bytes of it a load: 64 lines each, 4400 cycles for the 16 pairs of four rows and 20 keys.)
__device__ __forceinline__ void small_attention(const SmallCtx& m, int dv, int rows, int wave, int lane) {
  const int d = m.d, pairs = m.heads * rows;
  const bool self = BPD_SD(SD_MODE) == SM_SELF;
  const gfloat* qg = BPD_SDP(SD_P2);
  const int X = BPD_SD(SD_X), ldx = BPD_SD(SD_LDX), dim = (lane & 3) * 4;
  const rsrc_t kr = rsrc_of((const void*)BPD_SDP(SD_P0), 0x7FFFFFFF), vr = rsrc_of((const void*)BPD_SDP(SD_P1), 0x7FFFFFFF);
#pragma unroll 1
  for (int p0 = wave; p0 < pairs; p0 += 2 * SMALL_W) {
    int h[2], r[2], k0[2], k1[2];
    f32x4 qv[2], acc[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int pr = p0 + u * SMALL_W < pairs ? p0 + u * SMALL_W : p0;
      h[u] = (int)(((float)pr + 0.5f) * __builtin_amdgcn_rcpf((float)rows)); r[u] = pr - h[u] * rows;
      k1[u] = self ? m.L + r[u] + 1 : m.src;
      k0[u] = 0;
      if (self && m.local_q > 0) { k0[u] = (m.L + r[u]) / m.local_q * m.local_q - m.local_m; k0[u] = k0[u] > 0 ? k0[u] : 0; }
      qv[u] = qg ? *(const gfloat4*)(qg + (long)(m.kv_at + r[u]) * d + h[u] * 16 + dim) : *(const f32x4*)(m.lds + X + r[u] * ldx + h[u] * 16 + dim);
      acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int n0 = k1[0] - k0[0], n1 = k1[1] - k0[1], span = n0 > n1 ? n0 : n1;
    float l[2] = {0.f, 0.f};
    if (span <= 16) small_keys<1>(m, kr, vr, span, k0, k1, h, lane, qv, acc, l);
    else if (span <= 32) small_keys<2>(m, kr, vr, span, k0, k1, h, lane, qv, acc, l);
    else small_keys<4>(m, kr, vr, span, k0, k1, h, lane, qv, acc, l);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      // over the rows of 16 lanes (dimension e of the four in row e), then over the quads
      float o = small_rows4(acc[u][0], acc[u][1], acc[u][2], acc[u][3], SmallAdd());
      o += small_dpp<0x124>(o); o += small_dpp<0x128>(o);
      l[u] += small_dpp<0x124>(l[u]); l[u] += small_dpp<0x128>(l[u]);
      l[u] = sum_rows(l[u]);
      if ((lane & 12) == 0 && p0 + u * SMALL_W < pairs) m.lds[BPD_SD(SD_DST) + r[u] * BPD_SD(SD_LDO) + h[u] * 16 + dim + (lane >> 4)] = o / l[u];
    }
  }
}

// One phase for up to 4 RQ rows: the one f was fetched for; that of entry `next` (-1: none) is fetched on the way.  Ends with a barrier.
template <int RQ>
__device__ __forceinline__ void small_phase(const SmallCtx& m, SmallFetch& f, int next, int rows) {
  const int tid = small_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int dv = f.dv, mode = BPD_SD(SD_MODE), d = m.d;
  const int dn = next >= 0 ? ((const int*)m.lds)[next + (lane & 31)] : 0;
  const int ncb = BPD_SD(SD_NCB), N = BPD_SD(SD_N), slices = BPD_SD(SD_SLICES);
  const gfloat* bias = BPD_SDP(SD_BIAS);
  const float bs0 = f.bias, gv = f.g, bv = f.b;
  f32x4* red = (f32x4*)(m.lds + m.red);
  if (mode < SM_SELF && f.s < slices) {
    const int ldw = BPD_SD(SD_LDW), ldx = BPD_SD(SD_LDX), kn = BPD_SD(SD_KN);
    const rsrc_t wr = rsrc_of((const void*)BPD_SDP(SD_W), 0x7FFFFFFF);
    const float* x = m.lds + BPD_SD(SD_X) + (lane & 3) * ldx;
    f32x4 acc[RQ];
#pragma unroll 1
    for (int cb = f.cb; cb < ncb; cb += SMALL_W) {
      small_product<RQ>(wr, f.at, ldw, x + f.xo, ldx, kn, f.w, acc);
      if (slices > 1) {                          // (at most SMALL_W column blocks)
#pragma unroll
        for (int q = 0; q < RQ; ++q) red[(wave * RQ + q) * 64 + lane] = acc[q];
        break;
      }
      // a wave finishes what it multiplied
      if (cb + SMALL_W < ncb) { f.at = small_column(dv, cb + SMALL_W, 0, lane, f.xo); small_load(wr, f.at, ldw, f.w); }
      const int col = cb * 64 + small_col(lane);
      float bs = bs0;
      if (cb != wave && bias) bs = bias[col < N ? col : N - 1];
#pragma unroll 1
      for (int q = 0; q < RQ && 4 * q < rows; ++q) {
        f32x4 v = acc[0];
#pragma unroll
        for (int i = 1; i < RQ; ++i) v = q == i ? acc[i] : v;
        small_finish(m, dv, mode, rows, q, col, bs, gv, bv, v, lane);
      }
    }
  }
  if (next >= 0) small_fetch<RQ>(m, dn, f);
  if (mode < SM_SELF) {
    if (slices > 1) {
      const int pair = small_pair(wave), step = ncb * RQ * 64;
      __syncthreads();
#pragma unroll 1
      for (int pr = pair; pr < ncb * RQ; pr += SMALL_W) {
        const int c = pr / RQ, q = pr - c * RQ, col = c * 64 + small_col(lane);
        if (4 * q >= rows) continue;
        const float bs = pr == pair ? bs0 : (bias ? bias[col < N ? col : N - 1] : 0.f);
        small_finish(m, dv, mode, rows, q, col, bs, gv, bv, small_partials(red + (c * RQ + q) * 64 + lane, slices, step), lane);
      }
    }
  } else if (mode == SM_NORM) {
    for (int r = wave; r < rows; r += SMALL_W) {
      float v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = lane + 64 * i < d ? m.lds[BPD_SD(SD_X) + m.x_at + r * (d + 4) + lane + 64 * i] : 0.f;
      small_norm_row(v, m.lds + BPD_SD(SD_XN) + r * (d + 4), d, lane, BPD_SDP(SD_G), BPD_SDP(SD_GB), m.eps);
    }
  } else {
    small_attention(m, dv, rows, wave, lane);
  }
  __syncthreads();
}
// The phases of the entries first .. last - 1 for the same rows
template <int RQ>
__device__ __forceinline__ void small_phases(const SmallCtx& m, int table, int first, int last, int rows) {
  SmallFetch f;
  small_fetch<RQ>(m, ((const int*)m.lds)[table + first * SD_WORDS + (small_tid() & 31)], f);
#pragma unroll 1
  for (int ph = first; ph < last; ++ph) small_phase<RQ>(m, f, ph + 1 < last ? table + (ph + 1) * SD_WORDS : -1, rows);
}

// Rows of the next block: x = scale E[token] + pos (zero: without token), with the LayerNorm of the first phase (g null: without).  A wave per row, no barrier.
__device__ __forceinline__ void small_embed(const SmallCtx& m, int x, int rows, const int* tok, bool zero, const float* pos, const float* g, const float* b) {
  const SmallP& p = small_args();
  const int tid = small_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), d = p.d;
  for (int r = wave; r < rows; r += SMALL_W) {
    int t = zero ? 0 : tok[r];
    t = t < 0 ? 0 : (t >= p.V ? p.V - 1 : t);
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = lane + 64 * i;
      v[i] = 0.f;
      if (c < d) {
        v[i] = pos[(long)r * d + c];
        if (!zero) v[i] += p.escale * p.emb[(long)t * d + c];
        m.lds[x + r * (d + 4) + c] = v[i];
      }
    }
    if (g) small_norm_row(v, m.lds + m.xn + r * (d + 4), d, lane, (const gfloat*)g, (const gfloat*)b, p.eps);
  }
}

// Table of the decoder's phases: threads fill one entry each.  Returns their number.
__host__ __device__ inline int small_decoder_phases(int d, int n_dec, int k, int hgroup) { return n_dec * (d <= 64 ? 8 : 11) + 2 * ((k + hgroup - 1) / hgroup); }
__device__ __forceinline__ int small_decoder_phases(const SmallP& p) { return small_decoder_phases(p.d, p.n_dec, p.k, p.hgroup); }
__device__ __forceinline__ void small_decoder_table(const SmallP& p, const SmallLds& n, float* lds, int b) {
  const int d = p.d, F = p.F, per = d <= 64 ? 8 : 11, layers = per * p.n_dec, count = small_decoder_phases(p), ld = d + 4;
  for (int ph = threadIdx.x; ph < count; ph += SMALL_T) {
    SmallEntry e{(int*)lds + n.table + ph * SD_WORDS};
    const int l = ph / per;
    if (ph < layers) {
      int what = ph - l * per;                   // d > 64: 2, 5, 8 + 2 are LayerNorms of their own (behind WO, CO, W2)
      const long at = p.dec_stride * l;
      const bool last = l + 1 == p.n_dec;
      const float* g2 = p.dec.ln2g + at; const float* b2 = p.dec.ln2b + at; const float* g3 = p.dec.ln3g + at; const float* b3 = p.dec.ln3b + at;
      const float* g1 = last ? p.dec_g : p.dec.ln1g + at + p.dec_stride; const float* b1 = last ? p.dec_b : p.dec.ln1b + at + p.dec_stride;
      const float* gs[3] = {g2, g3, g1}; const float* bs[3] = {b2, b3, b1};
      if (d > 64) {
        // order: QKV SELF WO NORM | CQ CROSS CO NORM | W1 W2 NORM
        const int sub = what < 4 ? 0 : (what < 8 ? 1 : 2), i = what - 4 * sub, norm_at = sub < 2 ? 3 : 2;
        if (i == norm_at) {
          e.gemm(SM_NORM, nullptr, 0, d, d, nullptr, n.x, ld, n.xn, ld);
          const float* g = sub == 0 ? gs[0] : (sub == 1 ? gs[1] : gs[2]);
          const float* bb = sub == 0 ? bs[0] : (sub == 1 ? bs[1] : bs[2]);
          e.norm(g, bb, n.xn);
          continue;
        }
        what = 3 * sub + i;
      }
      const bool fuse = d <= 64;
      const long kv = p.self_layer * l + (long)b * p.slots * d, ckv = p.src_layer * l + (long)b * p.max_src * d;
      switch (what) {
        case 0: e.gemm(SM_QKV, p.dec.wqkv + at, 3 * d, 3 * d, d, nullptr, n.xn, ld, n.big, ld); e.ptr(SD_P0, p.selfK + kv); e.ptr(SD_P1, p.selfV + kv); break;
        case 1: e.gemm(SM_SELF, nullptr, 0, d, d, nullptr, n.big, ld, n.att, ld); e.ptr(SD_P0, p.selfK + kv); e.ptr(SD_P1, p.selfV + kv); break;
        case 2: e.gemm(SM_ADD, p.dec.wo + at, d, d, d, nullptr, n.att, ld, n.x, ld); if (fuse) e.norm(g2, b2, n.xn); break;
        case 3: e.gemm(SM_STORE, p.dec.cq + at, d, d, d, nullptr, n.xn, ld, n.big, ld); break;
        case 4: e.gemm(SM_CROSS, nullptr, 0, d, d, nullptr, n.big, ld, n.att, ld); e.ptr(SD_P0, p.crossK + ckv); e.ptr(SD_P1, p.crossV + ckv); break;
        case 5: e.gemm(SM_ADD, p.dec.co + at, d, d, d, nullptr, n.att, ld, n.x, ld); if (fuse) e.norm(g3, b3, n.xn); break;
        case 6: e.gemm(SM_RELU, p.dec.w1 + at, F, F, d, p.dec.b1 + at, n.xn, ld, n.big, F + 4); break;
        default: e.gemm(SM_ADD, p.dec.w2 + at, d, d, F, p.dec.b2 + at, n.big, F + 4, n.x, ld); if (fuse) e.norm(g1, b1, n.xn); break;
      }
    } else {                                     // heads: hidden and output layers, hgroup of them at a time
      const int i = ph - layers, h0 = i / 2 * p.hgroup, hn = p.k - h0 < p.hgroup ? p.k - h0 : p.hgroup;
      if ((i & 1) == 0) {
        e.gemm(SM_RELU, p.hw1 + (long)h0 * F, p.s.kmax * F, hn * F, d, p.hb1 + h0 * F, n.xn, ld, n.big, hn * F + 4);
      } else {
        e.gemm(SM_HEAD, p.hw2 + (long)h0 * F * d, d, hn * d, F, p.hb2 + h0 * d, n.big, hn * F + 4, n.o + h0 * ld, ld);
        e.e[SD_GW] = d; e.e[SD_WG] = F * d; e.e[SD_XG] = F;
      }
    }
  }
}

// First weights of column block cb from row k0 of the transposed table on; returns where they lie
__device__ __forceinline__ unsigned small_vocab_load(const rsrc_t& wr, int V, int cb, int k0, int lane, f32x4 (&w)[4]) {
  const int col = cb * 64 + (lane & 15) * 4;
  const unsigned at = (unsigned)((col < V ? col : V - 4) + (k0 + (lane >> 4) * 4) * V) * 4;
  small_load(wr, at, V, w);
  return at;
}
// As small_product, for sixteen rows: with v_mfma_f32_16x16x4 the same loads need no exchange; acc[i]: columns 4 (lane % 16) + i of rows
// 4 (lane / 16) ..
__device__ __forceinline__ void small_product16(const rsrc_t& wr, unsigned at, int ldw, const float* x, int kn, f32x4 (&w)[4], f32x4 (&acc)[4]) {
#pragma unroll 1
  for (int left = kn;;) {
    f32x4 next[4];
    left -= 16;
    at += 64 * ldw;
    if (left > 0) small_load(wr, at, ldw, next);
    const f32x4 xv = *(const f32x4*)x;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[t], w[t][i], acc[i], 0, 0, 0);
    if (left <= 0) break;
    x += 16;
#pragma unroll
    for (int t = 0; t < 4; ++t) w[t] = next[t];
  }
}

// The decoder's phases, then scores and arg-max: fills best[row * k + head] for the first k heads (and logits, z where wanted).  x and xn hold
// the block (small_embed).
template <int RQ>
__device__ __forceinline__ void small_forward(const SmallCtx& m, const SmallLds& n, int rows, float* logits, bool want_z) {
  const SmallP& p = small_args();
  const int count = small_decoder_phases(p), k = p.k, V = p.V, d = p.d;
  // scores: sixteen rows at a time; column blocks of 64, up to SMALL_W of them with K in slices, else one wave each
  const int tid = small_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = rows * k, ncb = (V + 63) / 64, per = ncb < SMALL_W ? ncb : SMALL_W;
  int slices = SMALL_W / per;
  while (slices > 1 && d % (16 * slices)) --slices;
  const int kn = d / slices, s = wave / per, cb0 = wave - s * per, ld = d + 4;
  f32x4* red = (f32x4*)(m.lds + m.red);
  unsigned long long* best = (unsigned long long*)(m.lds + n.best);
  unsigned* cand = (unsigned*)(m.lds + n.best + 512);                // [wave][16][2]
  const rsrc_t wr = rsrc_of(p.emb_t, 0x7FFFFFFF);
  f32x4 w[4];                                    // (the first ones come while the phases run)
  unsigned at = 0;
  if (s < slices && cb0 < ncb) at = small_vocab_load(wr, V, cb0, s * kn, lane, w);
  small_phases<RQ>(m, n.table, 0, count, rows);
#pragma unroll 1
  for (int m0 = 0; m0 < M; m0 += 16) {
    unsigned bu[4] = {0, 0, 0, 0}, bi[4] = {0, 0, 0, 0};           // best of rows 4 (lane / 16) .. over the columns this wave finished
#pragma unroll 1
    for (int cbase = 0; cbase < ncb; cbase += SMALL_W) {
      const int lane = small_tid() & 63, cb = cbase + cb0;
      f32x4 acc[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (s < slices && cb < ncb) {
        if (m0 > 0 || cbase > 0) at = small_vocab_load(wr, V, cb, s * kn, lane, w);
        small_product16(wr, at, V, m.lds + n.o + (m0 + (lane & 15)) * ld + s * kn + (lane >> 4) * 4, kn, w, acc);
      }
      if (slices > 1) {
        if (s < slices) {
#pragma unroll
          for (int i = 0; i < 4; ++i) red[(wave * 4 + i) * 64 + lane] = acc[i];
        }
        __syncthreads();
      }
      // two of a lane's four columns at a time: with slices (column block, half) pairs wave, wave + SMALL_W, .., without the wave's own block
#pragma unroll 1
      for (int pr = slices > 1 ? wave : 2 * cb; pr < (slices > 1 ? 2 * per : 2 * cb + 2); pr += slices > 1 ? SMALL_W : 1) {
        const int c = pr >> 1, i0 = (pr & 1) * 2, col = c * 64 + (lane & 15) * 4 + i0, g = lane >> 4;
        if (c >= ncb || (slices == 1 && s > 0)) break;         // (not a block of this wave)
        f32x4 v[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) v[e] = slices > 1 ? small_partials(red + (c * 4 + i0 + e) * 64 + lane, slices, per * 256) : (i0 ? acc[2 + e] : acc[e]);
        const bool in = col < V;
        unsigned key[4], top[4];
        bool second[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const unsigned k0 = (unsigned)(argmax_key(v[0][r], 0u) >> 32), k1 = (unsigned)(argmax_key(v[1][r], 0u) >> 32);
          second[r] = k1 > k0;
          top[r] = key[r] = in ? (second[r] ? k1 : k0) : 0u;
        }
        auto over_lanes = [&](auto step) {
#pragma unroll
          for (int r = 0; r < 4; ++r) { const unsigned o = step(top[r]); top[r] = o > top[r] ? o : top[r]; }
        };
        over_lanes([](unsigned x) { return small_dpp<0xB1>(x); });
        over_lanes([](unsigned x) { return small_dpp<0x4E>(x); });
        over_lanes([](unsigned x) { return small_dpp<0x141>(x); });
        over_lanes([](unsigned x) { return small_dpp<0x140>(x); });
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          // (of equal ones the lowest column: the lowest lane's, and of two pairs' or passes' the lower)
          const unsigned long long has = __ballot(in && key[r] == top[r]) >> (16 * g), odd = __ballot(second[r]) >> (16 * g);
          const int first = __ffs((int)((unsigned)has & 0xFFFFu)) - 1;
          const unsigned at = (unsigned)(c * 64 + first * 4 + i0) + ((unsigned)odd >> (first & 15) & 1u);
          const bool better = top[r] > bu[r] || (top[r] == bu[r] && at < bi[r]);
          bi[r] = better ? at : bi[r];
          bu[r] = better ? top[r] : bu[r];
          const int mm = m0 + 4 * g + r;
          if (logits && in && mm < M) { logits[(long)mm * V + col] = v[0][r]; logits[(long)mm * V + col + 1] = v[1][r]; }
          if (want_z && in && mm < M && mm % k == 0) { m.lds[n.z + mm / k * V + col] = v[0][r]; m.lds[n.z + mm / k * V + col + 1] = v[1][r]; }
        }
      }
      if (slices > 1) __syncthreads();
    }
    if ((lane & 15) == 0) {
      u32x4* to = (u32x4*)(cand + (wave * 16 + (lane >> 4) * 4) * 2);
      to[0] = u32x4{bu[0], bi[0], bu[1], bi[1]}; to[1] = u32x4{bu[2], bi[2], bu[3], bi[3]};
    }
    __syncthreads();
    if (tid < 16 && m0 + tid < M) {
      u32x2 c[SMALL_W];
#pragma unroll
      for (int w = 0; w < SMALL_W; ++w) c[w] = *(const u32x2*)(cand + (w * 16 + tid) * 2);
      __builtin_amdgcn_sched_barrier(0);
      unsigned long long top = 0ull;
#pragma unroll
      for (int w = 0; w < SMALL_W; ++w) {
        const unsigned long long key = c[w][0] ? ((unsigned long long)c[w][0] << 32) | (0xFFFFFFFFu - c[w][1]) : 0ull;
        top = key > top ? key : top;
      }
      best[m0 + tid] = top;
    }
    __syncthreads();
  }
}

__device__ __forceinline__ SmallCtx small_ctx(const SmallP& p, const SmallLds& n, float* lds) {
  SmallCtx m;
  m.lds = lds; m.red = n.red; m.xn = n.xn; m.d = p.d; m.k = p.k; m.heads = p.heads; m.L = 0; m.src = 0; m.local_q = p.local_q; m.local_m = p.local_m; m.kv_at = 0; m.x_at = 0;
  m.eps = p.eps; m.qscale = p.qscale;
  return m;
}

// The steps of one sequence: model, verify / accept / commit, next block, until it has ended or p.steps are done.
template <int RQ>
__global__ __launch_bounds__(SMALL_T) void small_decode_kernel(SmallP args) {
  extern __shared__ __attribute__((aligned(16))) float small_smem[];
  const int b = blockIdx.x, k = args.k, d = args.d, steps = args.steps;
  const bool topn = args.top_n > 1 && k > 1;
  const SmallLds n = small_lds(d, args.F, args.V, k, k, args.hgroup, 0, topn, small_decoder_phases(args));
  SmallCtx m = small_ctx(args, n, small_smem);
  int* tok = (int*)small_smem + n.misc;            // proposals [16], then length, ended, accepted, budget, steps; top-n flags [16]
  unsigned long long* best = (unsigned long long*)(small_smem + n.best);
  {
    const SmallP& p = small_args();
    const StateP& s = p.s;
    const int tid = threadIdx.x;
    if (tid < k) tok[tid] = s.P[b * s.kmax + tid];
    if (tid == 0) { tok[16] = s.L[b]; tok[17] = s.finished[b]; tok[18] = s.j[b]; tok[19] = s.max_len[b]; tok[20] = s.steps_done[b]; }
    m.src = s.src_len[b];
    small_decoder_table(p, n, small_smem, b);
    __syncthreads();
  }
#pragma unroll 1
  for (int step = 0; step < steps; ++step) {
    const SmallP& p = small_args();
    const StateP& s = p.s;
    const int tid = small_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tok[17] && !p.logits) {
      if (tid == 0) { s.accepted[b] = 0; if (p.accepted_out) p.accepted_out[b] = 0; }
      break;                                     // (the same for the whole workgroup)
    }
    m.L = __builtin_amdgcn_readfirstlane(tok[16]);
    m.kv_at = m.L;
    const int imposed = s.imposed && wave == 0 ? s.imposed[(long)step * s.imposed_stride + b] : 0;
    small_embed(m, n.x, k, tok, false, p.pos_tgt + (long)m.L * d, p.dec.ln1g, p.dec.ln1b);
    __syncthreads();
    small_forward<RQ>(m, n, k, p.logits ? p.logits + (long)b * k * k * p.V : nullptr, topn);
    for (int e = tid; e < k * k; e += SMALL_T) s.A[(b * s.kmax + e / k) * s.kmax + e % k] = key_index(best[e]);
    if (p.logits) break;
    if (topn) {                                  // is proposal i + 1 among the n best of p_1 at row i?
      if (wave < k - 1) {
        int t = tok[wave + 1];
        t = t < 0 ? 0 : (t >= p.V ? p.V - 1 : t);
        const float* z = small_smem + n.z + wave * p.V;
        const unsigned long long kt = argmax_key(z[t], (unsigned)t);
        int cnt = 0;
        for (int v = lane; v < p.V; v += 64) cnt += argmax_key(z[v], (unsigned)v) > kt;
        for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off, 64);
        if (lane == 0) tok[32 + wave] = cnt < p.top_n;
      }
      __syncthreads();
    }
    if (wave == 0) {
      const int myP = lane < k ? tok[lane] : -1;
      const bool test = lane >= 1 && lane < k;
      const int a1 = test ? key_index(best[(lane - 1) * k]) : 0;
      int khat = verified_length_v(s, k, lane, myP, a1, topn && test ? tok[32 + lane - 1] : 0, imposed);
      bool eos = false;
      const int j = tok[18], max_len = tok[19];
      khat = cut_length_v(s, lane, myP, khat, max_len - j, eos);
      if (lane < khat) s.out_ids[(long)b * s.max_out + j + lane] = myP;
      const int nextP = lane < k ? key_index(best[(khat > 0 ? khat - 1 : 0) * k + lane]) : 0;
      if (lane < k) { s.P[b * s.kmax + lane] = nextP; tok[lane] = nextP; }
      if (lane == 0) {
        const int fin = eos || (j + khat >= max_len), done = tok[20] + 1;
        s.j[b] = j + khat; s.L[b] = m.L + khat; s.finished[b] = fin; s.accepted[b] = khat; s.steps_done[b] = done;
        tok[16] = m.L + khat; tok[17] = fin; tok[18] = j + khat; tok[20] = done;
        if (p.accepted_out) p.accepted_out[b] = khat;
        atomicAdd((unsigned long long*)&s.stats[0], 1ull);
        atomicAdd((unsigned long long*)&s.stats[1], (unsigned long long)khat);
        if (fin) atomicAdd((unsigned long long*)&s.stats[2], 1ull);
        atomicAdd((unsigned long long*)&s.stats[3 + khat], 1ull);
        atomicMax((unsigned long long*)&s.stats[20], (unsigned long long)done);
      }
    }
    __syncthreads();
  }
}

// Encoder and cross keys and values of every decoder layer, of one sequence: 16 rows at a time through every phase (x holds all rows).
__host__ __device__ inline int small_encoder_phases(int d, int n_enc, int n_dec) { return n_enc * (d <= 64 ? 6 : 7) + 1 + n_dec; }
__global__ __launch_bounds__(SMALL_T) void small_encode_kernel(SmallP p) {
  extern __shared__ __attribute__((aligned(16))) float small_smem[];
  const int b = blockIdx.x, d = p.d, F = p.F, S = p.S, ld = d + 4, tiles = (S + 15) / 16;
  const int per = d <= 64 ? 6 : 7, layers = per * p.n_enc;
  const SmallLds n = small_lds(d, F, p.V, 16, 1, 1, tiles * 16, false, small_encoder_phases(d, p.n_enc, p.n_dec));
  SmallCtx m = small_ctx(p, n, small_smem);
  m.src = p.s.src_len[b];
  for (int ph = threadIdx.x; ph < layers + 1 + p.n_dec; ph += SMALL_T) {
    SmallEntry e{(int*)small_smem + n.table + ph * SD_WORDS};
    if (ph > layers) {
      const int l = ph - layers - 1;
      const long kv = p.src_layer * l + (long)b * p.max_src * d;
      e.gemm(SM_KV, p.dec.ckv + p.dec_stride * l, 2 * d, 2 * d, d, nullptr, n.xn, ld, 0, 0);
      e.ptr(SD_P0, p.crossK + kv); e.ptr(SD_P1, p.crossV + kv);
      continue;
    }
    float *Q = p.qe + (long)b * S * d, *K = p.ke + (long)b * S * d, *Vv = p.ve + (long)b * S * d;
    const int l = ph / per;
    int what = ph - l * per;                     // NORM QKV CROSS WO [NORM] W1 W2
    const long at = p.enc_stride * l;
    const float* g2 = p.enc.ln2g + at; const float* b2 = p.enc.ln2b + at;
    if (what == 0 || (d > 64 && what == 4)) {
      e.gemm(SM_NORM, nullptr, 0, d, d, nullptr, n.x, ld, n.xn, ld);
      e.norm(ph == layers ? p.enc_g : (what == 0 ? p.enc.ln1g + at : g2), ph == layers ? p.enc_b : (what == 0 ? p.enc.ln1b + at : b2), n.xn);
      continue;
    }
    if (d > 64 && what > 4) --what;
    switch (what) {
      case 1: e.gemm(SM_QKV, p.enc.wqkv + at, 3 * d, 3 * d, d, nullptr, n.xn, ld, 0, 0); e.ptr(SD_P0, K); e.ptr(SD_P1, Vv); e.ptr(SD_P2, Q); break;
      case 2: e.gemm(SM_CROSS, nullptr, 0, d, d, nullptr, 0, 0, n.att, ld); e.ptr(SD_P0, K); e.ptr(SD_P1, Vv); e.ptr(SD_P2, Q); break;
      case 3: e.gemm(SM_ADD, p.enc.wo + at, d, d, d, nullptr, n.att, ld, n.x, ld); if (d <= 64) e.norm(g2, b2, n.xn); break;
      case 4: e.gemm(SM_RELU, p.enc.w1 + at, F, F, d, p.enc.b1 + at, n.xn, ld, n.big, F + 4); break;
      default: e.gemm(SM_ADD, p.enc.w2 + at, d, d, F, p.enc.b2 + at, n.big, F + 4, n.x, ld); break;
    }
  }
  small_embed(m, n.x, S, p.src_ids + (long)b * S, false, p.pos_src, nullptr, nullptr);      // (ids: clamped by encode_init_kernel)
  __syncthreads();
  // layer by layer: LayerNorm and queries, keys, values of all tiles, then the rest tile by tile; at the end cross keys and values
#pragma unroll 1
  for (int part = 0; part <= 2 * p.n_enc; ++part) {
    const int first = part == 2 * p.n_enc ? layers : (part >> 1) * per + (part & 1 ? 2 : 0), last = part == 2 * p.n_enc ? layers + 1 + p.n_dec : (part >> 1) * per + (part & 1 ? per : 2);
#pragma unroll 1
    for (int t = 0; t < tiles; ++t) {
      m.kv_at = t * 16; m.x_at = t * 16 * ld;
      small_phases<4>(m, n.table, first, last, S - t * 16 < 16 ? S - t * 16 : 16);
    }
  }
}

// The first invocation of one sequence, on the empty prefix with all heads: the first proposals.
__global__ __launch_bounds__(SMALL_T) void small_prime_kernel(SmallP p) {
  extern __shared__ __attribute__((aligned(16))) float small_smem[];
  const int b = blockIdx.x, tid = threadIdx.x, kmax = p.s.kmax;
  const SmallLds n = small_lds(p.d, p.F, p.V, 4, 4, kmax, 0, false, small_decoder_phases(p));
  SmallCtx m = small_ctx(p, n, small_smem);
  m.src = p.s.src_len[b];
  small_decoder_table(p, n, small_smem, b);
  small_embed(m, n.x, 1, nullptr, true, p.pos_tgt, p.dec.ln1g, p.dec.ln1b);
  __syncthreads();
  small_forward<1>(m, n, 1, nullptr, false);
  if (tid < kmax) {
    const int a = key_index(((const unsigned long long*)(small_smem + n.best))[tid]);
    p.s.P[b * kmax + tid] = a;
    p.s.A[(long)b * kmax * kmax + tid] = a;
  }
  if (tid == 0) { p.s.L[b] = 1; p.s.j[b] = 0; p.s.finished[b] = 0; p.s.accepted[b] = 0; }
}
#undef BPD_SD
#undef BPD_SDP
