// Small fp32 models: a whole encode, and a whole decode, of a sequence in one workgroup.  Included by bpd_kernels.h.
//
// A step of a two-layer, 64-wide model is some 27 dependent kernels of 2 .. 10 us, 125 us in all, for 1 MB of weights and 1.2
// million multiply-adds: launches and nothing else.  Sequences do not depend on each other, so one workgroup of eight waves
// takes a sequence through all its steps: activations in LDS, weights out of the L2 (they stay there), barriers instead
// of launches.  What bounds it is the number of dependent phases (eight per layer: one trip to the L2, the partial sums'
// meeting in LDS) and, within them, instructions: every phase is one copy of the same code, driven by a table in LDS, and
// the products run on v_mfma_f32_4x4x1_16b: 4 rows x 64 columns per instruction and k, fp32, the lane's column of weights as it
// comes from memory (plain multiply-adds, with 16 LDS reads of the rows for 64 of them, took 80 us per step).
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
__device__ __forceinline__ float wave_max_f(float v) {
  v = fmaxf(v, dpp_move<0xB1>(v)); v = fmaxf(v, dpp_move<0x4E>(v)); v = fmaxf(v, dpp_move<0x141>(v)); v = fmaxf(v, dpp_move<0x140>(v));
  return max_rows(v);
}
__device__ __forceinline__ unsigned wave_max_u(unsigned v) {
#define BPD_STEP(C) { const unsigned o = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, C, 0xF, 0xF, true); v = o > v ? o : v; }
  BPD_STEP(0xB1) BPD_STEP(0x4E) BPD_STEP(0x141) BPD_STEP(0x140)
#undef BPD_STEP
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = a[0] > a[1] ? a[0] : a[1];
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return b[0] > b[1] ? b[0] : b[1];
}

// Fills a table entry (one thread)
struct SmallEntry {
  int* e;
  __device__ __forceinline__ void ptr(int i, const void* p) { e[i] = (int)(unsigned)(unsigned long long)p; e[i + 1] = (int)(unsigned)((unsigned long long)p >> 32); }
  __device__ __forceinline__ void gemm(int mode, const float* W, int ldw, int N, int K, const float* bias, int X, int ldx, int dst, int ldo) {
    const int ncb = (N + 63) / 64, per = ncb < SMALL_W ? ncb : SMALL_W;
    int slices = SMALL_W / per;
    while (slices > 1 && K % (4 * slices)) --slices;
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

// Four rows (4 q ..) of one column, finished: v = X W
__device__ __forceinline__ void small_finish(const SmallCtx& m, int dv, int mode, int rows, int q, int col, float bias, f32x4 v, int lane) {
  float* lds = m.lds;
  const int d = m.d, N = BPD_SD(SD_N), dst = BPD_SD(SD_DST), ldo = BPD_SD(SD_LDO), xn = BPD_SD(SD_XN);
  const bool in = col < N;
  if (mode == SM_QKV || mode == SM_KV) {
    const int c = mode == SM_KV ? col + d : col;
    gfloat *q2 = BPD_SDP(SD_P2), *k0 = BPD_SDP(SD_P0), *v0 = BPD_SDP(SD_P1);
    if (in) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 4 * q + i;
        if (r >= rows) break;
        if (c < d) { if (q2) q2[(long)(m.kv_at + r) * d + c] = v[i]; else lds[dst + r * ldo + c] = v[i]; }
        else if (c < 2 * d) k0[(long)(m.kv_at + r) * d + c - d] = v[i];
        else v0[(long)(m.kv_at + r) * d + c - 2 * d] = v[i];
      }
    }
    return;
  }
  int at = dst + (mode == SM_ADD ? m.x_at : 0) + col;
  if (mode == SM_HEAD) { const int h = (int)(((float)col + 0.5f) * __builtin_amdgcn_rcpf((float)d)), c = col - h * d; at = dst + h * ldo + c; col = c; }
  f32x4 t;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 4 * q + i;
    t[i] = v[i] + bias;
    if (mode == SM_RELU) t[i] = fmaxf(t[i], 0.f);
    if (!in || r >= rows) { t[i] = 0.f; continue; }
    if (mode == SM_HEAD) lds[at + r * m.k * ldo] = t[i] + lds[m.xn + r * (d + 4) + col];
    else {
      if (mode == SM_ADD) t[i] += lds[at + r * ldo];
      lds[at + r * ldo] = t[i];
    }
  }
  if (xn >= 0) {                                 // four rows at once: their reductions overlap
    const gfloat *g = BPD_SDP(SD_G), *b = BPD_SDP(SD_GB);
    const float gv = g[in ? col : 0], bv = b[in ? col : 0], inv = 1.0f / d;
    float mu[4], va[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) mu[i] = wave_sum(t[i]) * inv;
#pragma unroll
    for (int i = 0; i < 4; ++i) { const float c = in ? t[i] - mu[i] : 0.f; va[i] = wave_sum(c * c); }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x = fmaf(va[i], inv, m.eps), r0 = __builtin_amdgcn_rsqf(x), rs = r0 * fmaf(-0.5f * x * r0, r0, 1.5f);
      if (in && 4 * q + i < rows) lds[xn + (4 * q + i) * (d + 4) + col] = (t[i] - mu[i]) * rs * gv + bv;
    }
  }
}

// X W of one wave: 64 columns (col: this lane's) and kn of the k, 4 RQ rows
template <int RQ>
__device__ __forceinline__ void small_product(const SmallCtx& m, int dv, int col, int s, int lane, f32x4 (&acc)[RQ]) {
  const int N = BPD_SD(SD_N), ldw = BPD_SD(SD_LDW), ldx = BPD_SD(SD_LDX), kn = BPD_SD(SD_KN), gw = BPD_SD(SD_GW);
  int c = col < N ? col : N - 1, xo = 0;
  if (gw) { const int h = (int)(((float)c + 0.5f) * __builtin_amdgcn_rcpf((float)gw)); c += h * (BPD_SD(SD_WG) - gw); xo = h * BPD_SD(SD_XG); }
  // (rows of W are scalar offsets: one register of address for all loads)
  const rsrc_t wr = rsrc_of((const void*)BPD_SDP(SD_W), 0x7FFFFFFF);
  unsigned at = (unsigned)(c + s * kn * ldw) * 4;
  const float* x = m.lds + BPD_SD(SD_X) + xo + (lane & 3) * ldx + s * kn;
  f32x4 a2[RQ];
#pragma unroll
  for (int q = 0; q < RQ; ++q) { acc[q] = f32x4{0.f, 0.f, 0.f, 0.f}; a2[q] = acc[q]; }
  // sixteen k at a time, the next sixteen weights on their way meanwhile
  float wa[16], wb[16];
#define BPD_SLOAD(w, left)                                                                      \
  {                                                                                             \
    _Pragma("unroll") for (int j = 0; j < 16; ++j) w[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(wr, at, (j < (left) ? j : 0) * ldw * 4, 0)); \
    at += 64 * ldw;                                                                             \
  }
#define BPD_SMULT(w, left)                                                                      \
  {                                                                                             \
    _Pragma("unroll") for (int j = 0; j < 16; j += 4) {                                         \
      if (j >= (left)) break;                    /* (the same for the whole wave) */            \
      _Pragma("unroll") for (int q = 0; q < RQ; ++q) {                                          \
        const f32x4 xv = *(const f32x4*)(x + 4 * q * ldx + j);                                  \
        acc[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(xv[0], w[j], acc[q], 0, 0, 0);              \
        a2[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(xv[1], w[j + 1], a2[q], 0, 0, 0);            \
        acc[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(xv[2], w[j + 2], acc[q], 0, 0, 0);          \
        a2[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(xv[3], w[j + 3], a2[q], 0, 0, 0);            \
      }                                                                                         \
    }                                                                                           \
    x += 16;                                                                                    \
  }
  BPD_SLOAD(wa, kn)
  if (kn <= 16) {                                // (one batch: no loop around it, which would wait for the loads at its head)
    BPD_SMULT(wa, kn)
  } else {
    int left = kn;
#pragma unroll 1
    for (;;) {
      BPD_SLOAD(wb, left - 16)
      BPD_SMULT(wa, 16)
      left -= 16;
      if (left <= 16) { BPD_SMULT(wb, left) break; }
      BPD_SLOAD(wa, left - 16)
      BPD_SMULT(wb, 16)
      left -= 16;
      if (left <= 16) { BPD_SMULT(wa, left) break; }
    }
  }
#undef BPD_SMULT
#undef BPD_SLOAD
#pragma unroll
  for (int q = 0; q < RQ; ++q) acc[q] += a2[q];
}

// One phase for up to 4 RQ rows.  Ends with a barrier.
template <int RQ>
__device__ __forceinline__ void small_phase(const SmallCtx& m, int entry, int rows) {
  const int tid = small_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int dv = ((const int*)m.lds)[entry + (lane & 31)];
  const int mode = BPD_SD(SD_MODE), d = m.d;
  if (mode == SM_NORM) {
    for (int r = wave; r < rows; r += SMALL_W) {
      float v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = lane + 64 * i < d ? m.lds[BPD_SD(SD_X) + m.x_at + r * (d + 4) + lane + 64 * i] : 0.f;
      small_norm_row(v, m.lds + BPD_SD(SD_XN) + r * (d + 4), d, lane, BPD_SDP(SD_G), BPD_SDP(SD_GB), m.eps);
    }
  } else if (mode >= SM_SELF) {
    // Attention of 16-wide heads, a wave per (head, row): scores with a lane per key, then values with a lane per dimension and 16 of 64 keys
    const bool self = mode == SM_SELF;
    const gfloat *Kc = BPD_SDP(SD_P0), *Vc = BPD_SDP(SD_P1), *qg = BPD_SDP(SD_P2);
    float* pb = m.lds + m.red + wave * 64;
    for (int pr = wave; pr < m.heads * rows; pr += SMALL_W) {
      const int h = (int)(((float)pr + 0.5f) * __builtin_amdgcn_rcpf((float)rows)), r = pr - h * rows;
      const int k1 = self ? m.L + r + 1 : m.src;
      int k0 = 0;
      if (self && m.local_q > 0) { k0 = (m.L + r) / m.local_q * m.local_q - m.local_m; k0 = k0 > 0 ? k0 : 0; }
      f32x4 qv[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) qv[j] = qg ? *(const gfloat4*)(qg + (long)(m.kv_at + r) * d + h * 16 + 4 * j) : *(const f32x4*)(m.lds + BPD_SD(SD_X) + r * BPD_SD(SD_LDX) + h * 16 + 4 * j);
      float mx = -INFINITY, l = 0.f, acc = 0.f;
      for (int s0 = k0; s0 < k1; s0 += 64) {
        const int key = s0 + lane < k1 ? s0 + lane : k1 - 1;
        const gfloat4* kp = (const gfloat4*)(Kc + (long)key * d + h * 16);
        f32x4 kv[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) kv[j] = kp[j];
        float vv[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int kk = s0 + 16 * (lane >> 4) + i;
          vv[i] = Vc[(long)(kk < k1 ? kk : k1 - 1) * d + h * 16 + (lane & 15)];
        }
        float sc = 0.f;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i) sc = fmaf(qv[j][i], kv[j][i], sc);
        sc = s0 + lane < k1 ? sc * m.qscale : -INFINITY;
        const float mn = fmaxf(mx, wave_max_f(sc)), a = __expf(mx - mn), p = __expf(sc - mn);
        mx = mn;
        l = fmaf(l, a, p);
        pb[lane] = p;                            // (a wave's LDS accesses execute in order)
        acc *= a;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x4 pv = *(const f32x4*)(pb + 16 * (lane >> 4) + 4 * i);
          acc = fmaf(pv[0], vv[4 * i], acc); acc = fmaf(pv[1], vv[4 * i + 1], acc); acc = fmaf(pv[2], vv[4 * i + 2], acc); acc = fmaf(pv[3], vv[4 * i + 3], acc);
        }
      }
      l = wave_sum(l);
      acc = sum_rows(acc);
      if (lane < 16) m.lds[BPD_SD(SD_DST) + r * BPD_SD(SD_LDO) + h * 16 + lane] = acc / l;
    }
  } else {
    const int ncb = BPD_SD(SD_NCB), N = BPD_SD(SD_N), slices = BPD_SD(SD_SLICES);
    const gfloat* bias = BPD_SDP(SD_BIAS);
    if (slices == 1) {                           // a wave finishes what it multiplied
      for (int cb = wave; cb < ncb; cb += SMALL_W) {
        const int col = cb * 64 + lane;
        const float bs = bias ? bias[col < N ? col : N - 1] : 0.f;
        f32x4 acc[RQ];
        small_product<RQ>(m, dv, col, 0, lane, acc);
#pragma unroll
        for (int q = 0; q < RQ; ++q) small_finish(m, dv, mode, rows, q, col, bs, acc[q], lane);
      }
    } else {                                     // (at most SMALL_W column blocks)
      f32x4* red = (f32x4*)(m.lds + m.red);
      const int s = (wave * BPD_SD(SD_INV)) >> 16, cb = wave - s * ncb;
      // bias of what this wave will finish: (column block, row quad) pairs wave, wave + SMALL_W, ..
      const int col0 = (wave / RQ) * 64 + lane;
      const float bs0 = bias ? bias[col0 < N ? col0 : N - 1] : 0.f;
      if (s < slices) {
        f32x4 acc[RQ];
        small_product<RQ>(m, dv, cb * 64 + lane, s, lane, acc);
#pragma unroll
        for (int q = 0; q < RQ; ++q) red[(wave * RQ + q) * 64 + lane] = acc[q];
      }
      __syncthreads();
      for (int pr = wave; pr < ncb * RQ; pr += SMALL_W) {
        const int c = pr / RQ, q = pr - c * RQ, col = c * 64 + lane;
        const float bs = pr == wave ? bs0 : (bias ? bias[col < N ? col : N - 1] : 0.f);
        f32x4 v = red[(c * RQ + q) * 64 + lane];
#pragma unroll
        for (int t = 1; t < SMALL_W; ++t)        // (a branch each, all reads under way together)
          if (t < slices) v += red[((t * ncb + c) * RQ + q) * 64 + lane];
        small_finish(m, dv, mode, rows, q, col, bs, v, lane);
      }
    }
  }
  __syncthreads();
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

// The decoder's phases, then scores and arg-max: fills best[row * k + head] for the first k heads (and logits, z where wanted).  x and xn hold
// the block (small_embed).
template <int RQ>
__device__ __forceinline__ void small_forward(const SmallCtx& m, const SmallLds& n, int rows, float* logits, bool want_z) {
  const SmallP& p = small_args();
  const int count = small_decoder_phases(p), k = p.k, V = p.V, d = p.d;
#pragma unroll 1
  for (int ph = 0; ph < count; ++ph) small_phase<RQ>(m, n.table + ph * SD_WORDS, rows);
  // sixteen rows at a time; column blocks of 64, up to SMALL_W of them with K in slices, else one wave each
  const int tid = small_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = rows * k, ncb = (V + 63) / 64, per = ncb < SMALL_W ? ncb : SMALL_W;
  int slices = SMALL_W / per;
  while (slices > 1 && d % (4 * slices)) --slices;
  const int kn = d / slices, s = wave / per, cb0 = wave - s * per, ld = d + 4;
  f32x4* red = (f32x4*)(m.lds + m.red);
  unsigned long long* best = (unsigned long long*)(m.lds + n.best);
  unsigned* cand = (unsigned*)(m.lds + n.best + 512);                // [wave][16][2]
  const rsrc_t wr = rsrc_of(p.emb_t, 0x7FFFFFFF);
#pragma unroll 1
  for (int m0 = 0; m0 < M; m0 += 16) {
    unsigned bu = 0, bi = 0;                     // lane r < 16: best of row r over the columns this wave finished
#pragma unroll 1
    for (int cbase = 0; cbase < ncb; cbase += SMALL_W) {
      f32x4 acc[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int cb = cbase + cb0;
      if (s < slices && cb < ncb) {
        const int col = cb * 64 + lane;
        unsigned at = (unsigned)((col < V ? col : V - 1) + s * kn * V) * 4;
        const float* x = m.lds + n.o + (m0 + (lane & 3)) * ld + s * kn;
        for (int left = kn; left > 0; left -= 16) {
          float w[16];
#pragma unroll
          for (int j = 0; j < 16; ++j) w[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(wr, at, (j < left ? j : 0) * V * 4, 0));
          at += 64 * V;
#pragma unroll
          for (int j = 0; j < 16; j += 4) {
            if (j >= left) break;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const f32x4 xv = *(const f32x4*)(x + 4 * q * ld + j);
#pragma unroll
              for (int i = 0; i < 4; ++i) acc[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(xv[i], w[j + i], acc[q], 0, 0, 0);
            }
          }
          x += 16;
        }
      }
      if (slices > 1) {
        if (s < slices) {
#pragma unroll
          for (int q = 0; q < 4; ++q) red[(wave * 4 + q) * 64 + lane] = acc[q];
        }
        __syncthreads();
      }
      // (column block, row quad) pairs: with slices a wave takes the pairs wave, wave + SMALL_W, .., without it has all four quads of its block
      for (int pr = slices > 1 ? wave : 0; pr < (slices > 1 ? per * 4 : 4); pr += slices > 1 ? SMALL_W : 1) {
        const int c = slices > 1 ? pr >> 2 : cb, q = pr & 3, col = c * 64 + lane;
        f32x4 v;
        if (slices > 1) {
          v = red[(c * 4 + q) * 64 + lane];
#pragma unroll
          for (int t = 1; t < SMALL_W; ++t)
            if (t < slices) v += red[((t * per + c) * 4 + q) * 64 + lane];
        } else {
          v = q == 0 ? acc[0] : (q == 1 ? acc[1] : (q == 2 ? acc[2] : acc[3]));
          if (cb >= ncb || s > 0) break;         // (not a block of this wave)
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = 4 * q + i, mm = m0 + r;
          if (mm >= M) break;
          const unsigned key = col < V ? (unsigned)(argmax_key(v[i], 0u) >> 32) : 0u, top = wave_max_u(key);
          const int first = __ffsll((long long)__ballot(key == top && col < V)) - 1;
          // (columns ascend from pair to pair and pass to pass: an equal later one loses)
          if (lane == r && top > bu) { bu = top; bi = (unsigned)(c * 64 + first); }
          if (logits && col < V) logits[(long)mm * V + col] = v[i];
          if (want_z && col < V && mm % k == 0) m.lds[n.z + mm / k * V + col] = v[i];
        }
      }
      if (slices > 1) __syncthreads();
    }
    if (lane < 16) { cand[(wave * 16 + lane) * 2] = bu; cand[(wave * 16 + lane) * 2 + 1] = bi; }
    __syncthreads();
    if (tid < 16 && m0 + tid < M) {
      unsigned long long top = 0ull;
      for (int w = 0; w < SMALL_W; ++w) {
        const unsigned u = cand[(w * 16 + tid) * 2], i = cand[(w * 16 + tid) * 2 + 1];
        const unsigned long long key = u ? ((unsigned long long)u << 32) | (0xFFFFFFFFu - i) : 0ull;
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
#pragma unroll 1
      for (int ph = first; ph < last; ++ph) small_phase<4>(m, n.table + ph * SD_WORDS, S - t * 16 < 16 ? S - t * 16 : 16);
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
