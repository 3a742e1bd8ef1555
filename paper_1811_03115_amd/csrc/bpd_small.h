// Small fp32 models: a whole encode, and a whole decode, of a sequence in one workgroup.  Included by bpd_kernels.h.
//
// A step of a two-layer, 64-wide model is some 27 dependent kernels of 2 .. 10 us, 125 us in all, for 1 MB of weights and 1.2
// million multiply-adds: launches and nothing else.  Sequences do not depend on each other, so one workgroup of 16 waves
// takes a sequence through all its steps: activations in LDS, weights out of the L2 (they stay there), barriers instead
// of launches.  What bounds it is the number of dependent phases (about ten per layer, 0.5 .. 1 us each: one trip to
// the L2, the partial sums' meeting in LDS), beyond that one CU's 64 bytes per clock.
#pragma once

constexpr int SMALL_T = 1024;              // threads of the workgroup
struct SmallLayerP { const float *wqkv, *wo, *cq, *co, *ckv, *w1, *w2, *b1, *b2, *ln1g, *ln1b, *ln2g, *ln2b, *ln3g, *ln3b; };
struct SmallP {
  StateP s;
  int d, F, V, heads, n_enc, n_dec, max_src, slots, B, S;
  float eps, escale, qscale;
  int local_q, local_m;
  SmallLayerP enc, dec;                    // of the first layer; the others lie enc_stride / dec_stride floats on
  long enc_stride, dec_stride;
  const float *enc_g, *enc_b, *dec_g, *dec_b, *hw1, *hb1, *hw2, *hb2, *emb, *pos_src, *pos_tgt;
  float *selfK, *selfV, *crossK, *crossV, *qe, *ke, *ve;
  long self_layer, src_layer;              // floats per layer of the caches
  const int* src_ids;
  // decode
  int k, steps, hgroup, top_n;             // hgroup: heads whose hidden layers are in LDS together
  int* accepted_out;
  float* logits;                           // not null: one invocation's scores [B * k][k][V]; nothing is accepted
};

// LDS of the kernels in floats: rows of the residual stream, four row buffers, the widest hidden block, the heads' outputs, the
// partial sums, the scores of head 1 (top-n); see SmallLds
struct SmallLdsSize { int x, row, big, o, red, z; };
__host__ __device__ inline SmallLdsSize small_lds_size(int d, int F, int V, int rows, int k, int hgroup, int xrows, bool topn) {
  SmallLdsSize n;
  const int wide = 3 * d > F * hgroup ? 3 * d : F * hgroup;
  n.x = (xrows > rows ? xrows : rows) * d; n.row = rows * d; n.big = rows * (wide > F ? wide : F);
  n.o = ((rows * k + 15) / 16 * 16) * d;
  n.red = SMALL_T * 16; n.z = topn ? rows * V : 0;
  return n;
}
__host__ __device__ inline int small_lds_floats(const SmallLdsSize& n) { return n.x + 2 * n.row + n.big + n.o + n.red + n.z + 1024; }

#ifdef __HIPCC__
__device__ __forceinline__ float wave_max_f(float v) {
  v = fmaxf(v, dpp_move<0xB1>(v)); v = fmaxf(v, dpp_move<0x4E>(v)); v = fmaxf(v, dpp_move<0x141>(v)); v = fmaxf(v, dpp_move<0x140>(v));
  return max_rows(v);
}

// out(r, c, sum over k of X[r][k + xoff(c)] W(c)[k * ldw]) for r < rows <= RT, c < N; K % 4 == 0, X in LDS (rows of ldx floats, RT of
// them there).  A thread takes one column and one of `slices` equal parts of K; the parts meet in `red`.  WCONT: a column's
// weights lie one after the other (ldw == 1).  Ends with a barrier.
template <int RT, bool WCONT, class WCol, class XOff, class Out>
__device__ __forceinline__ void small_gemm(const float* X, int ldx, int rows, int N, int K, int ldw, float* red, WCol wcol, XOff xoff, Out out) {
  const int tid = threadIdx.x;
  for (int c0 = 0; c0 < N; c0 += SMALL_T) {
    const int nc = N - c0 < SMALL_T ? N - c0 : SMALL_T;
    int slices = 1;
    while (2 * slices * nc <= SMALL_T && K % (8 * slices) == 0) slices *= 2;
    const int sl = (int)(((float)tid + 0.5f) * __builtin_amdgcn_rcpf((float)nc)), c = tid - sl * nc, kn = K / slices;
    float acc[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) acc[r] = 0.f;
    if (sl < slices) {
      const float* w = wcol(c0 + c) + (WCONT ? sl * kn : (long)sl * kn * ldw);
      const float* x = X + xoff(c0 + c) + sl * kn;
      for (int k = 0; k < kn; k += 16) {         // sixteen weights in flight
        const int left = kn - k;
        float wv[16];
        if (WCONT) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float4 t = *(const float4*)(w + (4 * j < left ? k + 4 * j : k));
            wv[4 * j] = t.x; wv[4 * j + 1] = t.y; wv[4 * j + 2] = t.z; wv[4 * j + 3] = t.w;
          }
        } else {
#pragma unroll
          for (int j = 0; j < 16; ++j) wv[j] = w[(long)(j < left ? k + j : k) * ldw];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (4 * j >= left) break;              // (the same for the whole workgroup)
#pragma unroll
          for (int r = 0; r < RT; ++r) {
            const float4 xv = *(const float4*)(x + r * ldx + k + 4 * j);
            acc[r] = fmaf(xv.x, wv[4 * j], acc[r]); acc[r] = fmaf(xv.y, wv[4 * j + 1], acc[r]);
            acc[r] = fmaf(xv.z, wv[4 * j + 2], acc[r]); acc[r] = fmaf(xv.w, wv[4 * j + 3], acc[r]);
          }
        }
      }
    }
    if (slices == 1) {
      if (sl == 0) {
#pragma unroll
        for (int r = 0; r < RT; ++r)
          if (r < rows) out(r, c0 + c, acc[r]);
      }
      __syncthreads();
      continue;
    }
    if (sl < slices) {
#pragma unroll
      for (int r = 0; r < RT; ++r) red[(sl * RT + r) * nc + c] = acc[r];
    }
    __syncthreads();
    for (int o = tid; o < rows * nc; o += SMALL_T) {
      const int r = (int)(((float)o + 0.5f) * __builtin_amdgcn_rcpf((float)nc)), cc = o - r * nc;
      float v = red[o];
      for (int t = 1; t < slices; ++t) v += red[t * RT * nc + o];
      out(r, c0 + cc, v);
    }
    __syncthreads();
  }
}

// LayerNorm of rows of d columns in LDS, a wave per row.  Ends with a barrier.
__device__ __forceinline__ void small_norm(const float* x, float* y, int rows, int d, const float* g, const float* b, float eps) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int r = wave; r < rows; r += SMALL_T / 64) {
    float v[4], gv[4], bv[4], s = 0.f;           // d <= 256
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = lane + 64 * i;
      v[i] = c < d ? x[r * d + c] : 0.f; gv[i] = c < d ? g[c] : 0.f; bv[i] = c < d ? b[c] : 0.f;
      s += v[i];
    }
    const float mu = wave_sum(s) / d;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) q += lane + 64 * i < d ? (v[i] - mu) * (v[i] - mu) : 0.f;
    const float rs = 1.0f / sqrtf(wave_sum(q) / d + eps);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (lane + 64 * i < d) y[r * d + lane + 64 * i] = (v[i] - mu) * rs * gv[i] + bv[i];
  }
  __syncthreads();
}

// Attention of 16-wide heads: a wave per (head, row), a lane per key with a running maximum of its own.  q: rows of ldq floats in LDS or
// memory (not scaled); K, V: rows of d.  Row r sees the keys lo(r) .. hi(r) - 1.  Ends with a barrier.
template <class Lo, class Hi>
__device__ __forceinline__ void small_attention(const float* q, int ldq, const float* K, const float* V, float* out, int rows, int d, int heads, float scale, Lo lo, Hi hi) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int pr = wave; pr < heads * rows; pr += SMALL_T / 64) {
    const int h = pr / rows, r = pr - h * rows, k1 = hi(r);
    float4 qv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      qv[j] = *(const float4*)(q + (long)r * ldq + h * 16 + 4 * j);
      qv[j].x *= scale; qv[j].y *= scale; qv[j].z *= scale; qv[j].w *= scale;
    }
    float m = -INFINITY, l = 0.f, acc[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[j] = 0.f;
    for (int s = lo(r) + lane; s < k1; s += 64) {
      const float4* kp = (const float4*)(K + (long)s * d + h * 16);
      const float4* vp = (const float4*)(V + (long)s * d + h * 16);
      float4 kv[4], vv[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) { kv[j] = kp[j]; vv[j] = vp[j]; }
      float sc = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) { sc = fmaf(qv[j].x, kv[j].x, sc); sc = fmaf(qv[j].y, kv[j].y, sc); sc = fmaf(qv[j].z, kv[j].z, sc); sc = fmaf(qv[j].w, kv[j].w, sc); }
      const float mn = fmaxf(m, sc), a = __expf(m - mn), p = __expf(sc - mn);
      l = fmaf(l, a, p); m = mn;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        acc[4 * j] = fmaf(acc[4 * j], a, p * vv[j].x); acc[4 * j + 1] = fmaf(acc[4 * j + 1], a, p * vv[j].y);
        acc[4 * j + 2] = fmaf(acc[4 * j + 2], a, p * vv[j].z); acc[4 * j + 3] = fmaf(acc[4 * j + 3], a, p * vv[j].w);
      }
    }
    const float M = wave_max_f(m), f = m == -INFINITY ? 0.f : __expf(m - M);
    l = wave_sum(l * f);
    const float inv = 1.0f / l;
    float o = 0.f;
#pragma unroll
    for (int j = 0; j < 16; ++j) { const float t = wave_sum(acc[j] * f); o = lane == j ? t : o; }
    if (lane < 16) out[r * d + h * 16 + lane] = o * inv;
  }
  __syncthreads();
}

struct SmallLds { float *x, *xn, *att, *big, *o, *red, *z; int* tok; unsigned long long* best; };
__device__ __forceinline__ SmallLds small_lds(float* base, const SmallLdsSize& n) {
  SmallLds m;
  m.x = base; m.xn = m.x + n.x; m.att = m.xn + n.row; m.big = m.att + n.row; m.o = m.big + n.big; m.red = m.o + n.o; m.z = m.red + n.red;
  m.best = (unsigned long long*)(m.z + n.z);         // [256]
  m.tok = (int*)(m.best + 256);                      // [16] proposals, then length, ended, top-n flags [16]
  return m;
}
__device__ __forceinline__ SmallLayerP small_layer(const SmallLayerP& a, long at) {
  SmallLayerP r;
  r.wqkv = a.wqkv + at; r.wo = a.wo + at; r.cq = a.cq + at; r.co = a.co + at; r.ckv = a.ckv + at; r.w1 = a.w1 + at; r.w2 = a.w2 + at; r.b1 = a.b1 + at; r.b2 = a.b2 + at;
  r.ln1g = a.ln1g + at; r.ln1b = a.ln1b + at; r.ln2g = a.ln2g + at; r.ln2b = a.ln2b + at; r.ln3g = a.ln3g + at; r.ln3b = a.ln3b + at;
  return r;
}
// y += LayerNorm-free pieces of a layer: rows of x in LDS
template <int RT>
__device__ __forceinline__ void small_residual(const SmallLds& m, const float* X, int ldx, int rows, int d, int K, const float* W, const float* bias, float* x) {
  small_gemm<RT, false>(X, ldx, rows, d, K, d, m.red, [&](int c) { return W + c; }, [](int) { return 0; },
                        [&](int r, int c, float v) { x[r * d + c] += bias ? v + bias[c] : v; });
}
template <int RT>
__device__ __forceinline__ void small_ffn(const SmallP& p, const SmallLds& m, float* x, int rows, const float* g, const float* b, const SmallLayerP& w) {
  small_norm(x, m.xn, rows, p.d, g, b, p.eps);
  small_gemm<RT, false>(m.xn, p.d, rows, p.F, p.d, p.F, m.red, [&](int c) { return w.w1 + c; }, [](int) { return 0; },
                        [&](int r, int c, float v) { m.big[r * p.F + c] = fmaxf(v + w.b1[c], 0.f); });
  small_residual<RT>(m, m.big, p.F, rows, p.d, p.F, w.w2, w.b2, x);
}

// One invocation of the model on `rows` positions from L with the tokens in m.tok (zero: on the empty prefix): fills m.best[row * k + head]
// with the arg-max keys of the first k heads (and p.logits, m.z where wanted).
template <int RT>
__device__ __forceinline__ void small_forward(const SmallP& p, const SmallLds& m, int b, int rows, int k, int L, bool zero, float* logits, bool want_z) {
  const int tid = threadIdx.x, d = p.d, F = p.F, lane = tid & 63, wave = tid >> 6;
  for (int e = tid; e < rows * d; e += SMALL_T) {
    const int r = e / d, c = e - r * d;
    int t = zero ? 0 : m.tok[r];
    t = t < 0 ? 0 : (t >= p.V ? p.V - 1 : t);
    float v = p.pos_tgt[(long)(L + r) * d + c];
    if (!zero) v += p.escale * p.emb[(long)t * d + c];
    m.x[e] = v;
  }
  __syncthreads();
  const int src = p.s.src_len[b];
  for (int l = 0; l < p.n_dec; ++l) {
    const SmallLayerP w = small_layer(p.dec, p.dec_stride * l);
    float* Kc = p.selfK + p.self_layer * l + (long)b * p.slots * d;
    float* Vc = p.selfV + p.self_layer * l + (long)b * p.slots * d;
    const float* cK = p.crossK + p.src_layer * l + (long)b * p.max_src * d;
    const float* cV = p.crossV + p.src_layer * l + (long)b * p.max_src * d;
    small_norm(m.x, m.xn, rows, d, w.ln1g, w.ln1b, p.eps);
    small_gemm<RT, false>(m.xn, d, rows, 3 * d, d, 3 * d, m.red, [&](int c) { return w.wqkv + c; }, [](int) { return 0; },
                          [&](int r, int c, float v) {
                            if (c < d) m.big[r * d + c] = v;
                            else if (c < 2 * d) Kc[(long)(L + r) * d + c - d] = v;
                            else Vc[(long)(L + r) * d + c - 2 * d] = v;
                          });
    small_attention(m.big, d, Kc, Vc, m.att, rows, d, p.heads, p.qscale,
                    [&](int r) { const int t = L + r, lo = p.local_q > 0 ? t / p.local_q * p.local_q - p.local_m : 0; return lo > 0 ? lo : 0; },
                    [&](int r) { return L + r + 1; });
    small_residual<RT>(m, m.att, d, rows, d, d, w.wo, nullptr, m.x);
    small_norm(m.x, m.xn, rows, d, w.ln2g, w.ln2b, p.eps);
    small_gemm<RT, false>(m.xn, d, rows, d, d, d, m.red, [&](int c) { return w.cq + c; }, [](int) { return 0; }, [&](int r, int c, float v) { m.big[r * d + c] = v; });
    small_attention(m.big, d, cK, cV, m.att, rows, d, p.heads, p.qscale, [](int) { return 0; }, [&](int) { return src; });
    small_residual<RT>(m, m.att, d, rows, d, d, w.co, nullptr, m.x);
    small_ffn<RT>(p, m, m.x, rows, w.ln3g, w.ln3b, w);
  }
  // heads: O[row * k + head] = LN(x) + W2 relu(W1 LN(x) + b1) + b2, hgroup of them at a time
  small_norm(m.x, m.xn, rows, d, p.dec_g, p.dec_b, p.eps);
  for (int h0 = 0; h0 < k; h0 += p.hgroup) {
    const int hn = k - h0 < p.hgroup ? k - h0 : p.hgroup, HF = hn * F;
    small_gemm<RT, false>(m.xn, d, rows, HF, d, p.s.kmax * F, m.red, [&](int c) { return p.hw1 + (long)h0 * F + c; }, [](int) { return 0; },
                          [&](int r, int c, float v) { m.big[r * HF + c] = fmaxf(v + p.hb1[h0 * F + c], 0.f); });
    small_gemm<RT, false>(m.big, HF, rows, hn * d, F, d, m.red, [&](int c) { const int h = c / d; return p.hw2 + (long)(h0 + h) * F * d + (c - h * d); },
                          [&](int c) { return c / d * F; },
                          [&](int r, int c, float v) {
                            const int h = c / d, cc = c - h * d;
                            m.o[(r * k + h0 + h) * d + cc] = v + p.hb2[(h0 + h) * d + cc] + m.xn[r * d + cc];
                          });
  }
  // scores and arg-max: sixteen rows at a time, SMALL_T columns at most; a wave per row looks for the best
  const int M = rows * k, V = p.V;
  for (int m0 = 0; m0 < M; m0 += 16) {
    const int mr = M - m0 < 16 ? M - m0 : 16;
    unsigned long long best = 0ull;
    for (int v0 = 0; v0 < V; v0 += SMALL_T) {
      const int nc = V - v0 < SMALL_T ? V - v0 : SMALL_T;
      float* sc = m.red;                         // the sums replace the partial sums of their own column: [row][nc]
      small_gemm<16, true>(m.o + m0 * d, d, mr, nc, d, 1, m.red, [&](int c) { return p.emb + (long)(v0 + c) * d; }, [](int) { return 0; },
                           [&](int r, int c, float v) { sc[r * nc + c] = v; });
      if (wave < mr) {
        const int mm = m0 + wave;
        for (int c = lane; c < nc; c += 64) {
          const float v = sc[wave * nc + c];
          const unsigned long long key = argmax_key(v, (unsigned)(v0 + c));
          best = key > best ? key : best;
          if (logits) logits[(long)mm * V + v0 + c] = v;
          if (want_z && mm % k == 0) m.z[mm / k * V + v0 + c] = v;
        }
      }
      __syncthreads();
    }
    for (int off = 32; off > 0; off >>= 1) { const unsigned long long o = __shfl_xor(best, off, 64); best = o > best ? o : best; }
    if (wave < mr && lane == 0) m.best[m0 + wave] = best;
  }
  __syncthreads();
}

// The steps of one sequence: model, verify / accept / commit, next block, until it has ended or p.steps are done.
template <int RT>
__global__ __launch_bounds__(SMALL_T) void small_decode_kernel(SmallP p) {
  extern __shared__ __attribute__((aligned(16))) float small_smem[];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, k = p.k;
  const StateP& s = p.s;
  const bool topn = p.top_n > 1 && k > 1;
  const SmallLds m = small_lds(small_smem, small_lds_size(p.d, p.F, p.V, k, k, p.hgroup, 0, topn));
  int* L_s = m.tok + 16;
  int* fin_s = m.tok + 17;
  int* ok_s = m.tok + 18;
  if (tid < k) m.tok[tid] = s.P[b * s.kmax + tid];
  if (tid == 0) { *L_s = s.L[b]; *fin_s = s.finished[b]; }
  __syncthreads();
  for (int step = 0; step < p.steps; ++step) {
    if (*fin_s && !p.logits) {
      if (tid == 0) { s.accepted[b] = 0; if (p.accepted_out) p.accepted_out[b] = 0; }
      break;                                     // (the same for the whole workgroup)
    }
    const int L = *L_s;
    small_forward<RT>(p, m, b, k, k, L, false, p.logits ? p.logits + (long)b * k * k * p.V : nullptr, topn);
    for (int e = tid; e < k * k; e += SMALL_T) s.A[(b * s.kmax + e / k) * s.kmax + e % k] = key_index(m.best[e]);
    if (p.logits) break;
    if (topn) {                                  // is proposal i + 1 among the n best of p_1 at row i?
      if (wave < k - 1) {
        int t = m.tok[wave + 1];
        t = t < 0 ? 0 : (t >= p.V ? p.V - 1 : t);
        const float* z = m.z + wave * p.V;
        const unsigned long long kt = argmax_key(z[t], (unsigned)t);
        int cnt = 0;
        for (int v = lane; v < p.V; v += 64) cnt += argmax_key(z[v], (unsigned)v) > kt;
        for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off, 64);
        if (lane == 0) ok_s[wave] = cnt < p.top_n;
      }
      __syncthreads();
    }
    if (wave == 0) {
      const int myP = lane < k ? m.tok[lane] : -1;
      const bool test = lane >= 1 && lane < k;
      const int a1 = test ? key_index(m.best[(lane - 1) * k]) : 0;
      const int imposed = s.imposed ? s.imposed[(long)step * s.imposed_stride + b] : 0;
      int khat = verified_length_v(s, k, lane, myP, a1, topn && test ? ok_s[lane - 1] : 0, imposed);
      bool eos = false;
      const int j = s.j[b], max_len = s.max_len[b];
      khat = cut_length_v(s, lane, myP, khat, max_len - j, eos);
      if (lane < khat) s.out_ids[(long)b * s.max_out + j + lane] = myP;
      const int nextP = lane < k ? key_index(m.best[(khat > 0 ? khat - 1 : 0) * k + lane]) : 0;
      if (lane < k) { s.P[b * s.kmax + lane] = nextP; m.tok[lane] = nextP; }
      if (lane == 0) {
        const int fin = eos || (j + khat >= max_len);
        s.j[b] = j + khat; s.L[b] = L + khat; s.finished[b] = fin; s.accepted[b] = khat;
        *L_s = L + khat; *fin_s = fin;
        if (p.accepted_out) p.accepted_out[b] = khat;
        const int done = s.steps_done[b] + 1;
        s.steps_done[b] = done;
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

// Encoder, cross keys and values of every decoder layer, and the first invocation (on the empty prefix, all heads) of one sequence
__global__ __launch_bounds__(SMALL_T) void small_encode_kernel(SmallP p) {
  extern __shared__ __attribute__((aligned(16))) float small_smem[];
  const int b = blockIdx.x, tid = threadIdx.x, d = p.d, S = p.S;
  const SmallLds m = small_lds(small_smem, small_lds_size(d, p.F, p.V, 16, p.s.kmax, 1, (S + 15) / 16 * 16, false));
  const int* ids = p.src_ids + (long)b * S;
  for (int e = tid; e < S * d; e += SMALL_T) {
    const int r = e / d, c = e - r * d;
    const int t = ids[r];                        // (clamped by encode_init_kernel)
    m.x[e] = p.pos_src[(long)r * d + c] + p.escale * p.emb[(long)t * d + c];
  }
  __syncthreads();
  float *Q = p.qe + (long)b * S * d, *K = p.ke + (long)b * S * d, *Vv = p.ve + (long)b * S * d;
  const int src = p.s.src_len[b];
  for (int l = 0; l < p.n_enc; ++l) {
    const SmallLayerP w = small_layer(p.enc, p.enc_stride * l);
    for (int r0 = 0; r0 < S; r0 += 16) {
      const int rows = S - r0 < 16 ? S - r0 : 16;
      small_norm(m.x + r0 * d, m.xn, rows, d, w.ln1g, w.ln1b, p.eps);
      small_gemm<16, false>(m.xn, d, rows, 3 * d, d, 3 * d, m.red, [&](int c) { return w.wqkv + c; }, [](int) { return 0; },
                            [&](int r, int c, float v) { (c < d ? Q : (c < 2 * d ? K : Vv))[(long)(r0 + r) * d + (c < d ? c : (c < 2 * d ? c - d : c - 2 * d))] = v; });
    }
    for (int r0 = 0; r0 < S; r0 += 16) {
      const int rows = S - r0 < 16 ? S - r0 : 16;
      small_attention(Q + (long)r0 * d, d, K, Vv, m.att, rows, d, p.heads, p.qscale, [](int) { return 0; }, [&](int) { return src; });
      small_residual<16>(m, m.att, d, rows, d, d, w.wo, nullptr, m.x + r0 * d);
      small_ffn<16>(p, m, m.x + r0 * d, rows, w.ln2g, w.ln2b, w);
    }
  }
  for (int r0 = 0; r0 < S; r0 += 16) {
    const int rows = S - r0 < 16 ? S - r0 : 16;
    small_norm(m.x + r0 * d, m.xn, rows, d, p.enc_g, p.enc_b, p.eps);
    for (int l = 0; l < p.n_dec; ++l) {
      const float* W = p.dec.ckv + p.dec_stride * l;
      float* cK = p.crossK + p.src_layer * l + ((long)b * p.max_src + r0) * d;
      float* cV = p.crossV + p.src_layer * l + ((long)b * p.max_src + r0) * d;
      small_gemm<16, false>(m.xn, d, rows, 2 * d, d, 2 * d, m.red, [&](int c) { return W + c; }, [](int) { return 0; },
                            [&](int r, int c, float v) { if (c < d) cK[(long)r * d + c] = v; else cV[(long)r * d + c - d] = v; });
    }
  }
  const int kmax = p.s.kmax;
  small_forward<4>(p, m, b, 1, kmax, 0, true, nullptr, false);
  if (tid < kmax) {
    const int a = key_index(m.best[tid]);
    p.s.P[b * kmax + tid] = a;
    p.s.A[(long)b * kmax * kmax + tid] = a;
  }
  if (tid == 0) { p.s.L[b] = 1; p.s.j[b] = 0; p.s.finished[b] = 0; p.s.accepted[b] = 0; }
}
#endif
