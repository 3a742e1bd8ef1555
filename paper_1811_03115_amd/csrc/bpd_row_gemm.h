// GEMMs and LayerNorms of blocks of up to 640 rows, one memory round trip per kernel.  Included by bpd_kernels.h.
//
// A decoding step is a chain of small dependent kernels.  A kernel that does nothing costs 1.7 us in such a chain, and
// what the step's kernels took beyond that (2.2 .. 5.3 us) was mostly not data: four rounds of argument loads, 64-bit
// group arithmetic and index work for epilogues not in use stood between the launch and the first load (0.75 us), the
// LayerNorm prologue passed through two more barriers, and the LDS-staged kernel walks K in chunks, one trip each.  Here K
// is a compile-time constant, all of it is in flight at once, addresses are one register plus constants (buffer loads, whose
// bounds check also takes care of rows past the last one), and each epilogue is a kernel of its own.
#pragma once

enum { RG_RELU, RG_RES, RG_QKV, RG_PART };
struct RowGemmP {
  const void* W;                       // packed tiles
  const void* X;                       // LN: fp32 residual stream [M][K];  otherwise bf16, packed_at() with K = ldx
  const float* g; const float* b;      // LN: gain, bias
  int M, ntiles, ldx, ldy;
  bool packed;
  const float* bias;                   // RELU, RES (null: none)
  void* Y;                             // RELU: bf16 [M][ldy], packed: packed_at() with K = ldy;  RES: fp32 [M][ldy], added to;  PART: fp32 [slice][M][ldy];  QKV: fp32 queries [M][K]
  float eps;
  int ksteps;                          // PART: k-steps of all slices
  // QKV: columns of K each go to the queries (chunk 0), K cache (1), V cache (2), counted from chunk0
  int chunk0, R, heads;                // R: rows per sequence
  int capg, cap;                       // 64-wide heads: groups of 32 keys per sequence (bpd_attention.h); otherwise 0, and rows per sequence
  bf16_t* Kc; bf16_t* Vc;
  const int* base; const int* seq;     // first key row of each slot (null: 0) and its sequence (null: the slot; -1: none)
  long wz, kvz;                        // several matrices and caches side by side (grid z; cross keys and values of all layers): elements between them
  bf16_t* vout;                        // not null: values also to [M][K], packed_at() (a row that sees one key: its attention is that key's value)
};

// Y = epilogue(X W) for 16 MT rows x 16 NT columns per workgroup, K = 32 * WAVES * U (PART: of one slice, grid z).  The waves
// split K (wave w takes k-steps w U .. w U + U - 1), every load of the kernel is issued at its entry, and the waves' partial
// sums meet in LDS once.
// LN: X = LayerNorm(x): every wave takes mean and squared distances of its columns of the rows, these meet in LDS (row_moments), and
// the wave normalises in registers the fragments it already holds.  One barrier more than without, and twice the bytes for x: 0.8 us at K = 512,
// 1.2 us at K = 1024, against 1.9 us for a LayerNorm kernel of its own; but every column block repeats it, so that with
// K = 1024 and more than 32 rows (K = 512: 256) the kernel of its own is the faster one (lean_fuse() in bpd_host_logic.h).
// 8 x 512 x 1536 with LayerNorm: 3.95 -> 2.84 us per kernel of a chain;  10 x 1024 x 3072: 5.6 -> 4.2;  8 x 512 x 512: 3.2 -> 2.1;
// 10 x 1024 x 1024: 3.7 -> 2.6.  More waves (16) and fewer columns per workgroup (8, 4 of a tile) are slower; more columns (NT), then more
// rows (MT), pay once the workgroups would outnumber the CUs: 192 x 1024 x 3072 8.1 us with MT = 1, 7.05 with 3 (the LDS-staged kernel 10.2), 320 x 1024 x
// 1024 5.1 with 2 (5.85).
template <int WAVES, int U, int MT, int NT, bool LN, int EPI>
__global__ __launch_bounds__(WAVES * 64) void row_gemm_kernel(RowGemmP p) {
  constexpr int KSTEPS = WAVES * U, K = 32 * KSTEPS, TILES = MT * NT, OWN = (TILES + WAVES - 1) / WAVES, XB = LN ? 4 : 2;
  __shared__ f32x4 red[WAVES * TILES * 64];
  __shared__ float2 st[LN ? WAVES * 16 * MT : 1];
  __shared__ __attribute__((aligned(16))) float gb[LN ? WAVES * U * 64 : 4];       // per wave: gain, bias of its columns
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lq = lane >> 4;
  const int m0 = blockIdx.y * (16 * MT), tile0 = blockIdx.x * NT;
  const int ksteps = EPI == RG_PART ? p.ksteps : KSTEPS, ks0 = (EPI == RG_PART ? (int)blockIdx.z * KSTEPS : 0) + wave * U;
  f32x4 gbv;                                     // (first: it passes through LDS while x is on its way)
  if constexpr (LN) gbv = *(const f32x4*)((lane % (U * 16) < U * 8 ? p.g : p.b) + ks0 * 32 + (lane % (U * 8)) * 4);
  u32x4 a[NT][U];
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int tile = NT > 1 && tile0 + u >= p.ntiles ? p.ntiles - 1 : tile0 + u;
    const char* Wb = (const char*)p.W + ((size_t)tile * ksteps + ks0) * 1024 + (EPI == RG_QKV ? blockIdx.z * p.wz * 2 : 0);
#pragma unroll
    for (int i = 0; i < U; ++i) a[u][i] = *(const u32x4*)(Wb + i * 1024 + lane * 16);
  }
  const int ldx = LN ? K : p.ldx;
  const rsrc_t xr = rsrc_of(p.X, (unsigned)(LN ? p.M : (p.M + 15) & ~15) * ldx * XB);
  u32x4 xv[MT][U][LN ? 2 : 1];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    const unsigned off = LN ? ((m0 + t * 16 + lr) * ldx + ks0 * 32 + lq * 8) * XB : (((m0 >> 4) + t) * (ldx >> 5) + ks0) * 1024 + lane * 16;
#pragma unroll
    for (int i = 0; i < U; ++i) {
      xv[t][i][0] = buf_load16(xr, off + i * (LN ? 32 * XB : 1024), 0);
      if constexpr (LN) xv[t][i][1] = buf_load16(xr, off + i * (32 * XB) + 16, 0);
    }
  }
  // operands of the epilogue, for the tiles that this wave finishes
  f32x4 bias[OWN], res[OWN];
  int key0[OWN], sb[OWN], row0[OWN];
#pragma unroll
  for (int j = 0; j < OWN; ++j) {
    const int id = wave + WAVES * j;
    if (id >= TILES) continue;
    const int tile = tile0 + id % NT, n = (NT > 1 && tile >= p.ntiles ? p.ntiles - 1 : tile) * 16 + lq * 4, m = m0 + (id / NT) * 16 + lr;
    if constexpr (EPI == RG_RELU || EPI == RG_RES) bias[j] = p.bias ? *(const f32x4*)(p.bias + n) : f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (EPI == RG_RES) res[j] = __builtin_bit_cast(f32x4, buf_load16(rsrc_of(p.Y, (unsigned)p.M * p.ldy * 4), (m * p.ldy + n) * 4, 0));
    if constexpr (EPI == RG_QKV) {
      const int mm = m < p.M ? m : 0, q = (int)(((float)mm + 0.5f) * __builtin_amdgcn_rcpf((float)p.R));      // mm / R (mm < 2^16: exact)
      row0[j] = mm - q * p.R + (p.capg ? 0 : q * p.cap);       // (slots: cap is 0 and base counts rows over all sequences)
      sb[j] = q; key0[j] = 0;
      if (p.seq) sb[j] = p.seq[q];
      if (p.base) key0[j] = p.base[q];
    }
  }
  void* Y = arg_now(p.Y);
  bf16_t *Kc = nullptr, *Vc = nullptr;
  if constexpr (EPI == RG_QKV) { Kc = arg_now(p.Kc); Vc = arg_now(p.Vc); }
  __builtin_amdgcn_sched_barrier(0);
  f32x4 acc[MT][NT];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int u = 0; u < NT; ++u) acc[t][u] = f32x4{0.f, 0.f, 0.f, 0.f};
  if constexpr (LN) {
    float* gw = gb + wave * (U * 64);            // written and read by this wave alone: no barrier
    float mw[MT];                                // mean of the wave's own columns
    if (lane < U * 16) *(f32x4*)(gw + lane * 4) = gbv;
    f32x4 g4[U][2], b4[U][2];
#pragma unroll
    for (int i = 0; i < U; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        g4[i][h] = *(const f32x4*)(gw + i * 32 + lq * 8 + 4 * h);
        b4[i][h] = *(const f32x4*)(gw + U * 32 + i * 32 + lq * 8 + 4 * h);
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      // (sums in four chains; the registers then hold the distances to that mean)
      f32x4 s4 = f32x4{0.f, 0.f, 0.f, 0.f}, q4 = s4;
#pragma unroll
      for (int i = 0; i < U; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) s4 += __builtin_bit_cast(f32x4, xv[t][i][h]);
      const float s = sum_rows((s4[0] + s4[1]) + (s4[2] + s4[3]));
      mw[t] = s * (1.f / (32 * U));
#pragma unroll
      for (int i = 0; i < U; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f32x4 c = __builtin_bit_cast(f32x4, xv[t][i][h]) - mw[t];
          xv[t][i][h] = __builtin_bit_cast(u32x4, c);
#pragma unroll
          for (int r = 0; r < 4; ++r) q4[r] = fmaf(c[r], c[r], q4[r]);
        }
      const float q = sum_rows((q4[0] + q4[1]) + (q4[2] + q4[3]));
      if (lq == 0) st[(wave * MT + t) * 16 + lr] = make_float2(s, q);
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      float mu, rs;
      row_moments<WAVES, 32 * U>(st + t * 16 + lr, MT * 16, p.eps, mu, rs);
      const float off = (mw[t] - mu) * rs;
#pragma unroll
      for (int i = 0; i < U; ++i) {
        float y[8];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f32x4 v = __builtin_bit_cast(f32x4, xv[t][i][h]);
#pragma unroll
          for (int r = 0; r < 4; ++r) y[4 * h + r] = fmaf(fmaf(v[r], rs, off), g4[i][h][r], b4[i][h][r]);
        }
        const u32x4 yb = u32x4{cvt_pk_bf16(y[0], y[1]), cvt_pk_bf16(y[2], y[3]), cvt_pk_bf16(y[4], y[5]), cvt_pk_bf16(y[6], y[7])};
#pragma unroll
        for (int u = 0; u < NT; ++u)
          acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[u][i]), __builtin_bit_cast(bf16x8, yb), acc[t][u], 0, 0, 0);
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < U; ++i)
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int u = 0; u < NT; ++u)
          acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[u][i]), __builtin_bit_cast(bf16x8, xv[t][i][0]), acc[t][u], 0, 0, 0);
  }
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int u = 0; u < NT; ++u) red[(wave * TILES + t * NT + u) * 64 + lane] = acc[t][u];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < OWN; ++j) {
    const int id = wave + WAVES * j;
    if (id >= TILES) continue;
    // (all reads under way before the first is waited for: left alone the compiler reads and waits two by two, 130 cycles each time)
    f32x4 part[WAVES];
#pragma unroll
    for (int w = 0; w < WAVES; ++w) part[w] = red[(w * TILES + id) * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
    f32x4 v = part[0];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) v += part[w];
    const int tile = tile0 + id % NT, n = tile * 16 + lq * 4, m = m0 + (id / NT) * 16 + lr;
    if (NT > 1 && tile >= p.ntiles) continue;
    if (m >= p.M) continue;
    if constexpr (EPI == RG_RELU) {
      v += bias[j];
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.f);
      *(u32x2*)((bf16_t*)Y + (p.packed ? packed_at(m, n, p.ldy) : (size_t)m * p.ldy + n)) = u32x2{cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3])};
    } else if constexpr (EPI == RG_RES) {
      v += bias[j];
      v += res[j];
      *(f32x4*)((float*)Y + (size_t)m * p.ldy + n) = v;
    } else if constexpr (EPI == RG_PART) {
      *(f32x4*)((float*)Y + ((size_t)blockIdx.z * p.M + m) * p.ldy + n) = v;
    } else {
      const int c = tile / (K / 16), col = n - c * K;
      if (c + p.chunk0 == 0) {
        *(f32x4*)((float*)Y + (size_t)m * K + col) = v;
      } else if (sb[j] >= 0) {                   // (a slot behind the last one has no cache rows)
        bf16_t* cache = (c + p.chunk0 == 1 ? Kc : Vc) + blockIdx.z * p.kvz;
        const unsigned lo = cvt_pk_bf16(v[0], v[1]), hi = cvt_pk_bf16(v[2], v[3]);
        if (p.vout && c + p.chunk0 == 2) *(u32x2*)(p.vout + packed_at(m, col, K)) = u32x2{lo, hi};
        if (p.capg) kv_frag_store(cache, c + p.chunk0 == 2, sb[j], p.heads, p.capg, key0[j] + row0[j], col, lo, hi);
        else *(u32x2*)(cache + (size_t)(key0[j] + row0[j]) * K + col) = u32x2{lo, hi};
      }
    }
  }
}

// LayerNorm of one row of D columns per workgroup.  clear: behind layers_kernel, the words it counts in (nclear pieces of 16 bytes).  NSL > 0: x is the sum of itself, a bias and NSL raw K slices of a split
// GEMM, in this order of slices, and is stored.  One load of everything, one barrier (each wave takes the squares about the mean of its
// own columns, row_moments puts the waves together; against sums of squares about zero this costs 0.5 % of a sentence's decode): 1.9 us in a chain of kernels where one
// wave per row took 4.2 us (D = 512, 80 rows) .. 5.2 us (D = 1024, 8 slices).
// packed: ya as packed_at(), in pieces of 8 bytes.  Means of rows and packed by turns on two cards, us: 80 .. 320 rows of 1024 with four slices 4.03, 3.95 and 3.76, 4.27;  up to 256 rows without 3.11, 2.99 and
// 3.35, 2.89;  96 of 512 with four 3.70, 3.61 and 3.31, 3.18.  A tile's rows on one XCD against rows in order: big-batch32 15.72 ms, 15.77, two-phase 14.27, 14.32, base-batch13-top2 2.020, 2.031; eight
// or four rows on one XCD as sixteen.  A wave per row and four or eight rows per workgroup, which leave through LDS in pieces of 16 bytes: big-batch32 15.79 and 16.00 ms for 15.69.
constexpr int ln_row_threads(int D) { return D < 256 ? 64 : D / 4; }
template <int D, int NSL>
__global__ __launch_bounds__(ln_row_threads(D)) void ln_row_kernel(float* x, const float* g, const float* b, int M, float eps, bf16_t* ya, float* yf,
                                                                   const float* part, const float* pbias, u32x4* clear, int nclear, int packed) {
  constexpr int WAVES = ln_row_threads(D) / 64;
  __shared__ float2 st[WAVES];
  const int tid = threadIdx.x;
  const bool in = 4 * tid < D;                   // (D < 256: the last lanes hold zeros)
  int row = blockIdx.x;
  if (packed) {                                  // ya: packed_at(); a row tile's rows in workgroups of one XCD, whose L2 puts their pieces together
    row = ((row >> 7) * 8 + (row & 7)) * 16 + ((row >> 3) & 15);
    if (row >= M) return;
  }
  const size_t at = (size_t)row * D + (in ? 4 * tid : 0);
  f32x4 v = *(const f32x4*)(x + at);
  f32x4 pv[NSL > 0 ? NSL : 1], pb;
  if constexpr (NSL > 0) {
#pragma unroll
    for (int i = 0; i < NSL; ++i) pv[i] = *(const f32x4*)(part + (size_t)i * M * D + at);
    pb = *(const f32x4*)(pbias + (in ? 4 * tid : 0));
  }
  const f32x4 gv = *(const f32x4*)(g + (in ? 4 * tid : 0)), bv = *(const f32x4*)(b + (in ? 4 * tid : 0));
  __builtin_amdgcn_sched_barrier(0);
  if (clear && blockIdx.x == 0) {
    for (int i = tid; i < nclear; i += WAVES * 64) clear[i] = u32x4{0, 0, 0, 0};
  }
  if constexpr (NSL > 0) {
#pragma unroll
    for (int i = 1; i < NSL; ++i) pv[0] += pv[i];
    v += pv[0] + pb;
    if (in) *(f32x4*)(x + at) = v;
  }
  if (!in) v = f32x4{0.f, 0.f, 0.f, 0.f};
  const float s = wave_sum((v[0] + v[1]) + (v[2] + v[3])), mw = s * ((float)WAVES / D);
  f32x4 c = v - mw;                              // distances to the mean of the wave's own columns
  if (!in) c = f32x4{0.f, 0.f, 0.f, 0.f};
  const float q = wave_sum((c[0] * c[0] + c[1] * c[1]) + (c[2] * c[2] + c[3] * c[3]));
  float mu = mw, rs, off = 0.f;
  if constexpr (WAVES > 1) {
    if ((tid & 63) == 0) st[tid >> 6] = make_float2(s, q);
    __syncthreads();
    row_moments<WAVES, D / WAVES>(st, 1, eps, mu, rs);
    off = (mw - mu) * rs;
  } else rs = inv_sqrt(fmaf(q, 1.f / D, eps));
#pragma unroll
  for (int r = 0; r < 4; ++r) v[r] = fmaf(fmaf(c[r], rs, off), gv[r], bv[r]);
  if (!in) return;
  if (ya) *(u32x2*)(ya + (packed ? packed_at(row, 4 * tid, D) : at)) = u32x2{cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3])};
  if (yf) *(f32x4*)(yf + at) = v;
}
