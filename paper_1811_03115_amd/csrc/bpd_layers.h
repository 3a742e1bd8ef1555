// All decoder layers of a block as one kernel, a job of up to 16 rows per XCD (bf16, d = 512, d_ff = 2048, 64-wide heads).  Included by
// bpd_kernels.h.
//
// A layer is seven dependent operators.  As kernels of their own each costs 2.5 .. 6 us, of which a launch that does nothing is 1.7;
// the workgroups of one XCD share an L2, and there a hand-over takes 0.3 us one way even by a flag (store, acknowledgement, the flag, a poll that sees it: 690 cycles;
// between XCDs 950, with the data written through to memory), less where the result itself is polled for (Memory, below).  Six layers of 8 rows, 40 keys, 32 source tokens: 156 us
// as 42 kernels, 80 us here; eight such blocks on eight XCDs 90 us (chain of kernels over 64 rows: 200 us).  What bounds it now is the chain within
// an operator: a load of lines that another CU has just written (550 .. 900 cycles), LayerNorm or softmax at one wave
// per SIMD (4 cycles an instruction), LDS twice: 1.1 .. 2.9 us each.
//
// Work.  Sequences do not depend on each other: a job is the rows of up to four sequences, at most 16 rows, one MFMA row tile.  A group, the
// 32 workgroups that run on one XCD, takes a job through all layers, and every XCD streams all the weights (7.3 MB a layer, 0.5 TB/s) for
// its own job.  The tiles of an operator are dealt to 32 "places", each the same columns in every layer.
//
// A group forms itself: a workgroup registers with the XCD that it finds itself on and the first 32 to come are members.
// If fewer have come LK_CLOSE_TICKS after the first (CUs held by other launches), the group closes with those and they share the places out (six layers
// of 8 rows by members, by events, us: 32 84, 31 111, 16 111, 8 161).
// So whoever waits waits for a workgroup that is running: no residency of the whole grid is assumed, launches on several
// streams cannot block each other, and the mapping of workgroups to XCDs matters for speed only.  Groups fetch jobs until none is left.
// What launches on several streams do is take turns, since a workgroup fills its CU: decodes of one sentence, ms, chains of kernels and this: one context 3.8,
// 2.5, two 4.2, 3.1, four 5.8, 5.1; bpd_wide_layers.h, d = 1024: 6.3, 5.2; 8.5, 9.2; 12.3, 17.1 (BPD_LAYERS_GROUP=0 at creation: a context of chains).
//
// Inside a workgroup.  Four compute waves hold weights, K split over them; four helper waves poll for the operator's input, stage it in
// LDS (through LayerNorm where it has one), add the compute waves' partial sums, store the results and do the
// attention.  Loads return in order, per wave and, in the L1, per CU: a wave with weights under way can neither poll nor fetch
// activations without waiting for them too, and the helpers' loads queue behind the compute waves'.  Hence weights are not fetched when their
// registers fall free (110 us) but, a layer's at a time, while the member idles: in the self-attention or the cross-attention, which eight
// places each take part in (one sequence per job), others than each other where there is room (90 us; with no weights fetched at all: 88).
//
// Memory.  Results are plain stores into the XCD's L2; what this kernel has written is read past the L1 (sc1: the L1 may hold the lines as they were an
// operator or a layer ago).  A result tells by itself that it has come: its words hold EMPTY_WORD before, and who needs them loads them until none does.
// (With a flag stored behind the acknowledgement of the results, and the results loaded behind the flag, a hand-over was two trips to the L2 longer: six layers
// of 8 rows 89 us instead of 82, eight blocks of 10 rows over up to 3000 keys 150 on average instead of 144.)  The block's keys and values lie among older ones that
// any word may have: flags, raised by the waves that store queries, keys and values, announce these.  Keys and values are read
// once per launch, past nothing.
#pragma once

#include "bpd_layers_jobs.h"

constexpr unsigned LK_CLOSED = 0x10000u, LK_NO_JOB = 0xFFFFu;
constexpr long long LK_CLOSE_TICKS = 2000;                      // of the 100 MHz counter: 20 us
constexpr int LK_HOLD = 20, LK_GAP = 1, LK_PACE = 2;            // pauses of the compute waves, units of 64 cycles: LkCompute::job (hold 12: a sentence 2.52 ms, three images 59.1, 20: 2.54, 58.3, 28: 2.55, 58.3, 40: 2.56, 58.6)
constexpr int LK_SPINS = 1 << 22;                               // (a second: only a defect gets there)

struct LayersP {
  const char *wqkv, *wo, *cq, *co, *w1, *w2;     // of the first layer; packed tiles
  const float *ln1, *ln2, *ln3, *b1, *b2;        // gains, biases of a LayerNorm d floats behind
  long stride;                                   // bytes to the next layer's
  int n_layers, R, slots, per_job, jobs, group;  // R rows per slot; slots per job; members that a group waits for
  int split;                                     // workgroups per (head, slot) of the self-attention
  float *x, *part;
  bf16_t *q, *attn, *ffh, *selfK, *selfV;         // q: a row is 2 d wide (bf16 hi and lo parts)
  const float* lnf; float* h; bf16_t* hn;         // layers_kernel: the LayerNorm behind the layers (gains, then biases) and where it goes; hn null: x is stored as it is
  float *x1, *x3;                                // layers_kernel: the residual stream behind the two attentions (x1, then x2) and between layers
  bf16_t *attn2;                                  // ... and the cross-attention's results
  const bf16_t *crossK, *crossV;
  long self_layer, src_layer;                    // elements of a layer's caches
  int self_groups, src_groups;                   // groups of 32 keys per sequence
  const int *base, *src_len, *seq;               // per slot: cache rows, source length, sequence (null: the slot; -1: none)
  float eps, scale;
  int local_q, local_m;
  bf16_t* xn; float* slices;                     // normalised rows, copies per XCD; tall_layers_kernel: the second FFN layer's K slices between layers (of the last: part)
  unsigned* sync;                                // [LK_WORDS], zero at the start of a launch (cleared by the next kernel: the LayerNorm or the GEMM of the heads' hidden layers)
  long long* error;                              // set to 1 if a wait ran out
};

__device__ __forceinline__ unsigned lk_xcd() {
  unsigned v;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(v));
  return v & (LK_XCDS - 1);
}
__device__ __forceinline__ unsigned lk_load(const unsigned* p) {
  unsigned v;
  asm volatile("global_load_dword %0, %1, off sc1\n\ts_waitcnt vmcnt(0)" : "=v"(v) : "v"(p) : "memory");
  return v;
}
__device__ __forceinline__ void lk_store(unsigned* p, unsigned v) { asm volatile("global_store_dword %0, %1, off" ::"v"(p), "v"(v) : "memory"); }
__device__ __forceinline__ void lk_stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ u32x4 lk_load16(rsrc_t r, unsigned off) { return __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 16); }      // sc1
// The kernel's arguments and the lane, opaque where they are asked for: otherwise what every operator derives from them is computed ahead of the
// loop over the layers and kept in registers, more of them than there are.
__device__ __forceinline__ const LayersP& lk_args() {
  auto q = (const __attribute__((address_space(4))) LayersP*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(q));
  return *(const LayersP*)q;
}
// An int that nothing changes while this kernel runs
__device__ __forceinline__ int lk_const(const int* p, int i) { return ((const __attribute__((address_space(4))) int*)p)[i]; }
__device__ __forceinline__ int lk_lane() {
  int t = threadIdx.x & 63;
  asm volatile("" : "+v"(t));
  return t;
}
// ---- compute waves
// The N tiles from `tile` on, this wave's U k-steps of each.  PACE > 0: a pause between requests (units of 64 cycles)
template <int PACE, int N, int U>
__device__ __forceinline__ void lk_weights(u32x4 (&a)[N][U], const char* W, int tile, int cw, int lane) {
  const rsrc_t r = rsrc_of(W, 0x7FFFFFFF);
#pragma unroll
  for (int t = 0; t < N; ++t)
#pragma unroll
    for (int i = 0; i < U; ++i) {
      a[t][i] = buf_load16(r, lane * 16 + i % 4 * 1024, ((tile + t) * (4 * U) + cw * U + i / 4 * 4) * 1024);
      if (PACE) { __builtin_amdgcn_sched_barrier(0); __builtin_amdgcn_s_sleep(PACE); __builtin_amdgcn_sched_barrier(0); }
    }
}
// Partial sums of the N tiles over this wave's part of K
template <int N, int U>
__device__ __forceinline__ void lk_multiply(const u32x4 (&a)[N][U], const bf16_t* xs, int rows, f32x4* part, int cw, int lane) {
  constexpr int K = 128 * U, CH = N == 1 && U > 4 ? 4 : 1;         // (one long product: four chains)
  const int lr = lane & 15;
  const bf16_t* row = xs + (lr < rows ? lr : 0) * (K + 8) + cw * U * 32 + (lane >> 4) * 8;         // (rows past the last: one address, no bank conflicts)
  f32x4 acc[N][CH];
#pragma unroll
  for (int t = 0; t < N; ++t)
#pragma unroll
    for (int c = 0; c < CH; ++c) acc[t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < U; ++i) {
    const bf16x8 b = __builtin_bit_cast(bf16x8, *(const u32x4*)(row + i * 32));
#pragma unroll
    for (int t = 0; t < N; ++t) acc[t][i % CH] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[t][i]), b, acc[t][i % CH], 0, 0, 0);
    if (U > 16 && i % 8 == 7) __builtin_amdgcn_sched_barrier(0);       // (reads of eight steps at most ahead: no registers for more)
  }
#pragma unroll
  for (int t = 0; t < N; ++t) {
    if constexpr (CH == 4) acc[t][0] = (acc[t][0] + acc[t][1]) + (acc[t][2] + acc[t][3]);
    part[(cw * N + t) * 64 + lane] = acc[t][0];
  }
}

// ---- helper waves
// The first NF helper waves of each of `producers` members from `from` on have raised their flags to `target`
template <int NF>
__device__ __forceinline__ void lk_wait(const unsigned* flags, unsigned target, int from, int producers, int lane, bool& broken, long long* error) {
  if (broken) return;
#pragma unroll 1
  for (int s = 0; s < LK_SPINS; ++s) {
    unsigned v0, v1 = target;
    if constexpr (NF > 2) asm volatile("global_load_dword %0, %2, off sc1\n\tglobal_load_dword %1, %2, off offset:256 sc1\n\ts_waitcnt vmcnt(0)" : "=&v"(v0), "=&v"(v1) : "v"(flags + lane) : "memory");
    else v0 = lk_load(flags + lane);
    const bool in = (unsigned)((lane & 31) - from) < (unsigned)producers;
    bool ok = !in || (lane >= 32 && NF < 2) || v0 >= target;
    if (NF > 2) ok = ok && (!in || (lane >= 32 && NF < 4) || v1 >= target);
    if (__all(ok)) return;
  }
  broken = true;
  if (lane == 0) *error = 1;
}
// This wave's results are in the L2
__device__ __forceinline__ void lk_raise(unsigned* flag, unsigned v, int lane) {
  lk_stores_done();
  if (lane == 0) lk_store(flag, v);
}
// Results that carry their own news (EMPTY_WORD: bpd_attention.h): a buffer is empty in every word until its producers store into it, so that whoever loads it
// again and again until no word is empty needs no flag, and the producers wait for no acknowledgement.
constexpr int LK_POLLS = 1 << 20;                               // (as LK_SPINS; a round takes longer)
__device__ __forceinline__ unsigned lk_top(unsigned top, const u32x4& v) {
  const unsigned a = v[0] > v[1] ? v[0] : v[1], b = v[2] > v[3] ? v[2] : v[3];
  top = top > a ? top : a;
  return top > b ? top : b;
}
struct LkPoll {
  bool* broken;
  long long* error;
  bool on;                                       // (off: the data is known to be there)
  int turn = -1;                                 // first()
  // One of N pieces of 1 KB, ahead of all: a longer wait with less traffic (turn: members that wait for the same ask for different ones)
  template <int N> __device__ __forceinline__ void first(const rsrc_t& r, unsigned at, int lane) const {
    if (turn < 0 || !on || *broken) return;
    const unsigned off = at + turn % N * 1024 + lane * 16;
#pragma unroll 1
    for (int s = 0; s < LK_POLLS; ++s) {
      if (!__any(lk_top(0, lk_load16(r, off)) == EMPTY_WORD)) return;
      asm volatile("" ::: "memory");
    }
  }
  // load: fetches and returns the largest word
  template <class Load> __device__ __forceinline__ void operator()(Load&& load) const {
#pragma unroll 1
    for (int s = 0; s < LK_POLLS; ++s) {
      const unsigned top = load();
      if (!on || *broken || !__any(top == EMPTY_WORD)) return;
      asm volatile("" ::: "memory");
    }
    *broken = true;
    if (lk_lane() == 0) *error = 1;
  }
};
// LayerNorm of up to 16 rows of 512 into LDS as bf16, rows 520 apart; wave hw takes rows hw, hw + 4, ..
template <int N>
__device__ __forceinline__ void lk_norm_rows(const rsrc_t& xr, int rows, const f32x4 (&g)[2], const f32x4 (&b)[2], float eps, bf16_t* xs, int hw, int lane, LkPoll poll) {
  constexpr int D = 512;
  f32x4 v[N][2];
  poll([&] {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) v[i][h] = __builtin_bit_cast(f32x4, lk_load16(xr, ((hw + 4 * i) * D + lane * 8 + h * 4) * 4));
    __builtin_amdgcn_sched_barrier(0);
    unsigned top = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) { top = lk_top(top, __builtin_bit_cast(u32x4, v[i][0])); top = lk_top(top, __builtin_bit_cast(u32x4, v[i][1])); }
    return top;
  });
  float mu[N], q[N];
#pragma unroll
  for (int i = 0; i < N; ++i) { const f32x4 s = v[i][0] + v[i][1]; mu[i] = (s[0] + s[1]) + (s[2] + s[3]); }
#pragma unroll
  for (int i = 0; i < N; ++i) mu[i] = wave_sum(mu[i]) * (1.f / D);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    v[i][0] -= mu[i]; v[i][1] -= mu[i];
    f32x4 s = v[i][0] * v[i][0];
#pragma unroll
    for (int r = 0; r < 4; ++r) s[r] = fmaf(v[i][1][r], v[i][1][r], s[r]);
    q[i] = (s[0] + s[1]) + (s[2] + s[3]);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) q[i] = wave_sum(q[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float rs = inv_sqrt(fmaf(q[i], 1.f / D, eps));
    f32x4 y[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) y[h][r] = fmaf(v[i][h][r] * rs, g[h][r], b[h][r]);
    if (hw + 4 * i < rows)
      *(u32x4*)(xs + (hw + 4 * i) * (D + 8) + lane * 8) = u32x4{cvt_pk_bf16(y[0][0], y[0][1]), cvt_pk_bf16(y[0][2], y[0][3]), cvt_pk_bf16(y[1][0], y[1][1]), cvt_pk_bf16(y[1][2], y[1][3])};
  }
}
__device__ __forceinline__ void lk_norm(const float* x, int rows, const f32x4 (&g)[2], const f32x4 (&b)[2], float eps, bf16_t* xs, int hw, int lane, LkPoll poll) {
  const rsrc_t xr = rsrc_of(x, (unsigned)rows * 512 * 4);
  if (rows <= 8) lk_norm_rows<2>(xr, rows, g, b, eps, xs, hw, lane, poll);
  else if (rows <= 12) lk_norm_rows<3>(xr, rows, g, b, eps, xs, hw, lane, poll);
  else lk_norm_rows<4>(xr, rows, g, b, eps, xs, hw, lane, poll);
}
// bf16 rows of K into LDS, rows K + 8 apart
template <int K, int M>
__device__ __forceinline__ void lk_copy_rows(const rsrc_t& r, int rows, bf16_t* xs, int hw, int lane, LkPoll poll) {
  constexpr int N = K / 512;
  u32x4 v[M][N];
  poll.first<N>(r, hw * K * 2, lane);
  poll([&] {
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
      for (int j = 0; j < N; ++j) v[i][j] = lk_load16(r, ((hw + 4 * i) * K + j * 512 + lane * 8) * 2);
    __builtin_amdgcn_sched_barrier(0);
    unsigned top = 0;
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
      for (int j = 0; j < N; ++j) top = lk_top(top, v[i][j]);
    return top;
  });
#pragma unroll
  for (int i = 0; i < M; ++i)
    if (hw + 4 * i < rows) {
#pragma unroll
      for (int j = 0; j < N; ++j) *(u32x4*)(xs + (hw + 4 * i) * (K + 8) + j * 512 + lane * 8) = v[i][j];
    }
}
template <int K>
__device__ __forceinline__ void lk_copy(const bf16_t* src, int rows, bf16_t* xs, int hw, int lane, LkPoll poll = {nullptr, nullptr, false}) {
  const rsrc_t r = rsrc_of(src, (unsigned)rows * K * 2);
  if (rows <= 8) lk_copy_rows<K, 2>(r, rows, xs, hw, lane, poll);
  else if (rows <= 12) lk_copy_rows<K, 3>(r, rows, xs, hw, lane, poll);
  else if constexpr (K <= 2048) lk_copy_rows<K, 4>(r, rows, xs, hw, lane, poll);
  else { lk_copy_rows<K, 2>(r, rows, xs, hw, lane, poll); lk_copy_rows<K, 2>(r, rows, xs, hw + 8, lane, poll); }         // (registers)
}
// Rows of the attention left by `split` workgroups per (head, slot) (attention_mfma_core) put together, into LDS like lk_copy<512>
__device__ __forceinline__ void lk_merge(const float* part, int split, int slot0, int R, int rows, bf16_t* xs, int hw, int lane, LkPoll poll) {
  constexpr int H = 8, REC = 16 * 66;
  const int h = lane >> 3, dim = (lane & 7) * 8;
#pragma unroll 1
  for (int m = hw; m < rows; m += 4) {
    const int s = m / R, r = m - s * R;
    const rsrc_t pr = rsrc_of(part + (size_t)(slot0 + s) * H * split * REC, (unsigned)(H * split * REC) * 4);
    f32x4 o[LK_SPLITS][2];
    float M[LK_SPLITS], L[LK_SPLITS];
    poll([&] {
#pragma unroll
      for (int i = 0; i < LK_SPLITS; ++i) {
        const unsigned at = i < split ? (unsigned)((h * split + i) * REC) * 4 : 0x40000000u;         // (past the end: zeros)
        o[i][0] = __builtin_bit_cast(f32x4, lk_load16(pr, at + (r * 64 + dim) * 4));
        o[i][1] = __builtin_bit_cast(f32x4, lk_load16(pr, at + (r * 64 + dim + 4) * 4));
        M[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(pr, (int)(at + (1024 + r) * 4), 0, 16));
        L[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(pr, (int)(at + (1040 + r) * 4), 0, 16));
      }
      __builtin_amdgcn_sched_barrier(0);
      unsigned top = 0;
#pragma unroll
      for (int i = 0; i < LK_SPLITS; ++i) {
        top = lk_top(top, __builtin_bit_cast(u32x4, o[i][0])); top = lk_top(top, __builtin_bit_cast(u32x4, o[i][1]));
        const unsigned m = __float_as_uint(M[i]) > __float_as_uint(L[i]) ? __float_as_uint(M[i]) : __float_as_uint(L[i]);
        top = top > m ? top : m;
      }
      return top;
    });
    float top = M[0], l = 0.f;
#pragma unroll
    for (int i = 1; i < LK_SPLITS; ++i) top = i < split ? fmaxf(top, M[i]) : top;
    f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f}, b = a;
#pragma unroll
    for (int i = 0; i < LK_SPLITS; ++i) {
      const float w = i < split && M[i] != -INFINITY ? __expf(M[i] - top) : 0.f;
      l = fmaf(L[i], w, l);
      a += o[i][0] * w; b += o[i][1] * w;
    }
    float inv = __builtin_amdgcn_rcpf(l);
    inv = inv * fmaf(-l, inv, 2.f);
    *(u32x4*)(xs + m * 520 + lane * 8) = u32x4{cvt_pk_bf16(a[0] * inv, a[1] * inv), cvt_pk_bf16(a[2] * inv, a[3] * inv), cvt_pk_bf16(b[0] * inv, b[1] * inv), cvt_pk_bf16(b[2] * inv, b[3] * inv)};
  }
}

// What a member knows of its group and job
struct LkJob {
  int rank, members, slot0, slots, rows, row0;
  // The cross-attention's places (slot, head) start behind the self-attention's where there is room: a member that idles
  // in one of the two fetches weights then
  __device__ __forceinline__ int cross_places() const { return 8 * slots; }
  __device__ __forceinline__ int cross_first() const {
    const int first = 8 * slots * lk_args().split;
    return members == LK_PLACES && first + 8 * slots <= LK_PLACES ? first : 0;
  }
  __device__ __forceinline__ int cross() const { const int c = rank - cross_first(); return c < 0 ? c + LK_PLACES : c; }
};

template <int F, bool KVNT>
struct LkHelper {
  bf16_t* xs;
  f32x4* red;                                    // [compute wave][tile][lane]
  AttnLds sm;
  u32x2* q_s;
  unsigned* flags;
  int hw;
  LkJob j;
  int key, sb;                                   // of row lr: its row in the cache, its sequence
  unsigned op;                                   // first products done
  bool broken;
  unsigned ahead[8];                             // fetch_ahead()

  __device__ __forceinline__ void raise() { lk_raise(flags + hw * 32 + j.rank, op, lk_lane()); }

  // of this wave's tile, of N (all reads under way before the first is waited for)
  template <int N> __device__ __forceinline__ f32x4 partial_sums(int lane) const {
    f32x4 part[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) part[w] = red[(w * N + hw) * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
    return ((part[0] + part[1]) + part[2]) + part[3];
  }

  __device__ __forceinline__ LkPoll poll(bool on = true) { return LkPoll{&broken, lk_args().error, on}; }
  // The residual stream on its way through layer l (stage 0: into it, 1, 2: behind its attentions, 3: out of it)
  __device__ __forceinline__ static float* stream(int l, int stage) {
    const LayersP& p = lk_args();
    if (stage == 0) return l == 0 ? p.x : p.x3;
    if (stage == 3) return l + 1 == p.n_layers && !p.hn ? p.x : p.x3;
    return stage == 1 ? p.x1 : p.x1 + LK_JOBS * 16 * 512;
  }
  // What this member writes is emptied when everybody is known to have read it: by the lanes that wrote it, at the latest an operator ahead of its own
  // part in what its next reader has waited for.
  __device__ __forceinline__ void empty_tile(float* x, int place, int lane) const {
    const int lr = lane & 15;
    if (hw == 0 && lr < j.rows) *(u32x4*)(x + (size_t)(j.row0 + lr) * 512 + place * 16 + (lane >> 4) * 4) = u32x4{EMPTY_WORD, EMPTY_WORD, EMPTY_WORD, EMPTY_WORD};
  }
  __device__ __forceinline__ void empty_hidden(int lane) const {
    const int lr = lane & 15;
    if (lr >= j.rows || (F < 2048 && hw >= F / 512)) return;
#pragma unroll 1
    for (int place = j.rank; place < LK_PLACES; place += j.members)
      *(u32x2*)(lk_args().ffh + (size_t)(j.row0 + lr) * F + (place * (F / 512) + hw) * 16 + (lane >> 4) * 4) = u32x2{EMPTY_WORD, EMPTY_WORD};
  }
  __device__ __forceinline__ void empty_rows(bf16_t* attn, int slot, int h, u32x2 with, int lane) const {
    const LayersP& p = lk_args();
    const int lr = lane & 15;
    if (lr < p.R) *(u32x2*)(attn + (size_t)(slot * p.R + lr) * 512 + h * 64 + hw * 16 + (lane >> 4) * 4) = with;
  }
  __device__ __forceinline__ void part_rows(int slot, int h, int split, f32x4 o, float M, float L, int lane) const {
    const LayersP& p = lk_args();
    float* part = p.part + (((long)slot * 8 + h) * p.split + split) * (16 * 66);
    *(f32x4*)(part + (lane & 15) * 64 + hw * 16 + (lane >> 4) * 4) = o;
    if (hw == 0 && lane < 16) { part[1024 + lane] = M; part[1040 + lane] = L; }
  }
  __device__ __forceinline__ void empty_self(int lane) const {
    const int items = self_places(), split = lk_args().split;
    const float e = __uint_as_float(EMPTY_WORD);
#pragma unroll 1
    for (int place = j.rank; place < items; place += j.members) {
      const int ss = place >> 3, sp = split > 1 ? ss / j.slots : 0, slot = j.slot0 + ss - sp * j.slots;
      if (split > 1) part_rows(slot, place & 7, sp, f32x4{e, e, e, e}, e, e, lane);
      else empty_rows(lk_args().attn, slot, place & 7, u32x2{EMPTY_WORD, EMPTY_WORD}, lane);
    }
  }
  __device__ __forceinline__ void empty_cross(int lane) const {
#pragma unroll 1
    for (int place = j.cross(); place < j.cross_places(); place += j.members) empty_rows(lk_args().attn2, j.slot0 + (place >> 3), place & 7, u32x2{EMPTY_WORD, EMPTY_WORD}, lane);
  }
  // Ahead of a job's first hand-over: nothing is assumed of what the buffers hold
  __device__ __forceinline__ void empty_all(int lane) const {
    const LayersP& p = lk_args();
#pragma unroll 1
    for (int place = j.rank; place < LK_PLACES; place += j.members) {
      empty_tile(stream(0, 1), place, lane); empty_tile(stream(0, 2), place, lane); empty_tile(p.x3, place, lane);
    }
    empty_self(lane); empty_cross(lane);
  }

  // One operator with a product
  enum { QKV, O, CO, UP, DOWN };
  template <int OP, int N, int K>
  __device__ __forceinline__ void product(int l) {
    constexpr int D = 512;
    constexpr bool LN = OP == QKV || OP == UP, RES = !LN;
    const LayersP& p = lk_args();
    const int lane = lk_lane(), lr = lane & 15, lq = lane >> 4;
    const float *ln = nullptr, *bias = nullptr;
    if constexpr (LN) ln = (const float*)((const char*)(OP == QKV ? p.ln1 : p.ln3) + l * p.stride);
    if constexpr (OP == UP || OP == DOWN) bias = (const float*)((const char*)(OP == UP ? p.b1 : p.b2) + l * p.stride);
    f32x4 g[2], b[2], bs, res;
    float* const in = stream(l, OP == QKV || OP == O ? 0 : (OP == CO ? 1 : 2));        // LN: the rows; otherwise what the result is added to
    const rsrc_t xr = rsrc_of(in + (size_t)j.row0 * D, (unsigned)j.rows * D * 4);
    auto operands = [&](int place) {
      const int n = (place * N + hw) * 16 + lq * 4;
      if (N < 4 && hw >= N) return;
      if constexpr (OP == UP || OP == DOWN) bs = *(const f32x4*)(bias + n);
      if constexpr (RES) res = __builtin_bit_cast(f32x4, lk_load16(xr, (lr * D + n) * 4));           // (its own: the tile is its place's in all of O, CO and DOWN)
    };
    if constexpr (LN) {
#pragma unroll
      for (int h = 0; h < 2; ++h) { g[h] = *(const f32x4*)(ln + lane * 8 + h * 4); b[h] = *(const f32x4*)(ln + D + lane * 8 + h * 4); }
    }
    operands(j.rank);
    // (everybody has emptied what it writes)
    if (OP == O && l == 0) lk_wait<4>(flags, op, 0, j.members, lane, broken, p.error);
    if constexpr (LN) lk_norm(in + (size_t)j.row0 * D, j.rows, g, b, p.eps, xs, hw, lane, poll(OP != QKV || l > 0));
    else if constexpr (OP == DOWN) lk_copy<K>(p.ffh + (size_t)j.row0 * K, j.rows, xs, hw, lane, poll());
    else if (OP == O && p.split > 1) lk_merge(p.part, p.split, j.slot0, p.R, j.rows, xs, hw, lane, poll());
    else lk_copy<K>((OP == O ? p.attn : p.attn2) + (size_t)j.row0 * K, j.rows, xs, hw, lane, poll());
#pragma unroll 1
    for (int place = j.rank; place < LK_PLACES; place += j.members) {
      if (place != j.rank) operands(place);
      lk_barrier();                              // the input is staged, the partial sums of the place before are read
      if (place == j.rank) {
        if constexpr (OP == QKV) { fetch_ahead(l); empty_hidden(lane); if (l == 0) { empty_all(lane); lk_stores_done(); } }         // (read: DOWN's results are there)
        if constexpr (OP == CO) empty_self(lane);                                                // (O's results were there ahead of the cross-attention's)
        if constexpr (OP == UP) empty_cross(lane);                                               // (CO's are there)
      }
      lk_barrier();                              // the partial sums are there
      if (N < 4 && hw >= N) continue;
      f32x4 v = partial_sums<N>(lane);
      if (lr >= j.rows) continue;
      const int tile = place * N + hw, n = tile * 16 + lq * 4;
      if constexpr (OP == QKV) {
        const int c = tile / (D / 16), col = n - c * D;
        if (c == 0) {                            // (lo: D columns on)
          u32x2 hi, lo;
          lk_halves(v * p.scale, hi, lo);
          bf16_t* q = p.q + (size_t)(j.row0 + lr) * (2 * D) + col;
          *(u32x2*)q = hi; *(u32x2*)(q + D) = lo;
        }
        else if (sb >= 0) kv_frag_store((c == 1 ? p.selfK : p.selfV) + l * p.self_layer, c == 2, sb, D / 64, p.self_groups, key, col, cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]));
      } else if constexpr (OP == UP) {
        v += bs;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.f);
        *(u32x2*)(p.ffh + (size_t)(j.row0 + lr) * F + n) = full_words(u32x2{cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3])});
      } else {
        if constexpr (OP == DOWN) v += bs;
        v += res;
        float* const out = stream(l, OP == O ? 1 : (OP == CO ? 2 : 3));
        *(u32x4*)(out + (size_t)(j.row0 + lr) * D + n) = full_words(v);
        if (OP != O || l > 0) empty_tile(in, place, lane);          // (everybody has read the input: it has led to what this operator waited for)
      }
    }
    if constexpr (OP == QKV) { ++op; if (hw < 3 || l == 0) raise(); }         // (the wave without a tile: that it has emptied what it writes)
  }

  __device__ __forceinline__ static AttnP attn_args(bool self) {
    const LayersP& p = lk_args();
    AttnP a{};
    a.capg = self ? p.self_groups : p.src_groups;
    a.d = 512; a.R = p.R; a.nsplit = self ? p.split : 1; a.causal = self;
    a.local_q = self ? p.local_q : 0; a.local_m = p.local_m; a.part = p.part;
    return a;
  }
  __device__ __forceinline__ static int sequence(int slot) { const LayersP& p = lk_args(); return p.seq ? lk_const(p.seq, slot) : slot; }

  // Places (split, slot, head), the heads fastest
  __device__ __forceinline__ int self_places() const { return 8 * j.slots * lk_args().split; }
  // Keys and values of the first round of this member's part of the self-attention come out of memory into the L2 (they lie in the same lines as the block's own to come:
  // nothing may enter the L1) while it multiplies for them: asked for by the wave that has no tile of queries, keys and values, since loads return in order, and acknowledgements
  // with them.  (Asked for by each wave ahead of its wait for the flags, which then waited for them, too, a sentence of 64 tokens took 2.607 ms instead of 2.578.)
  __device__ __forceinline__ void fetch_ahead(int l) {
    const LayersP& p = lk_args();
    if (hw != 3 || j.rank >= self_places()) return;
    const int lane = lk_lane(), ss = j.rank >> 3, split = p.split > 1 ? ss / j.slots : 0, slot = j.slot0 + ss - split * j.slots, s = sequence(slot);
    const int lim = lk_const(p.base, slot), held = (lim + p.R + 31) >> 5, groups = held < p.self_groups ? held : p.self_groups;
    const int first = (attn_first_key(attn_args(true), lim) >> 5) + split * 8;
    const size_t at = l * p.self_layer + ((size_t)(s < 0 ? 0 : s) * 8 + (j.rank & 7)) * p.self_groups * KV_GROUP;
    const rsrc_t kr = rsrc_of(p.selfK + at, (unsigned)groups * (KV_GROUP * 2)), vr = rsrc_of(p.selfV + at, (unsigned)groups * (KV_GROUP * 2));
#pragma unroll
    for (int i = 0; i < 8; ++i) ahead[i] = __builtin_amdgcn_raw_buffer_load_b32(i < 4 ? kr : vr, lane * 128, (first + 2 * (i & 3)) * (KV_GROUP * 2), 16);      // (a word of each line of two groups)
  }
  // G groups of 32 keys per wave and round
  template <int G>
  __device__ __forceinline__ void self_place(int l, int place) {
    const LayersP& p = lk_args();
    const int lane = lk_lane(), lr = lane & 15, lq = lane >> 4;
    const int h = place & 7, ss = place >> 3, split = p.split > 1 ? ss / j.slots : 0, slot = j.slot0 + ss - split * j.slots, s = sequence(slot);
    const AttnP a = attn_args(true);
    const int lim = lk_const(p.base, slot), held = (lim + p.R + 31) >> 5, groups = held < p.self_groups ? held : p.self_groups;
    const int first = (attn_first_key(a, lim) >> 5) + split * (4 * G), hop = p.split * (4 * G);
    const size_t at = l * p.self_layer + ((size_t)(s < 0 ? 0 : s) * 8 + h) * p.self_groups * KV_GROUP;
    const rsrc_t kr = rsrc_of(p.selfK + at, (unsigned)groups * (KV_GROUP * 2)), vr = rsrc_of(p.selfV + at, (unsigned)groups * (KV_GROUP * 2));
    const rsrc_t qr = rsrc_of(p.q + (size_t)slot * p.R * 1024, (unsigned)p.R * 2048);
    bf16_t* out = p.attn;
    if (place != j.rank) {
      lk_barrier();                              // the results of the place before are out of LDS
    } else {
      lk_wait<3>(flags, op, 0, j.members, lane, broken, p.error);
      if (hw == 3)
#pragma unroll
        for (int i = 0; i < 8; ++i) asm volatile("" ::"v"(ahead[i]));
    }
    if (s < 0) {                                 // (rows of nobody; a barrier as the attention's own)
      if (p.split > 1) part_rows(slot, h, split, f32x4{0.f, 0.f, 0.f, 0.f}, 0.f, 1.f, lane); else empty_rows(out, slot, h, u32x2{0, 0}, lane);
      lk_barrier();
      return;
    }
    const unsigned off = lr * 2048 + (h * 64 + 8 * lq) * 2;
    bf16x8 qhi[2], qlo[2];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      qhi[s2] = __builtin_bit_cast(bf16x8, lk_load16(qr, off + s2 * 64));
      qlo[s2] = __builtin_bit_cast(bf16x8, lk_load16(qr, off + s2 * 64 + 1024));
    }
    u32x4 kf[G][4], vf[G][4];
    attn_load_kv<KVNT, G>(kr, vr, first + hw, 4, lane, kf, vf);
    __builtin_amdgcn_sched_barrier(0);
    attention_mfma_core<KVNT, true, G == 2 ? -1 : 0, G, ATTN_WORDS>(a, sm, h, slot, 0, split, 0, p.R, 8, p.split, hw * 64 + lane, 4, first, hop, kr, vr, kf, vf, qhi, qlo, lim, out);
  }
  __device__ __forceinline__ void self_attention(int l) {
    const int items = self_places();
#pragma unroll 1
    for (int place = j.rank; place < items; place += j.members) {
      const LayersP& p = lk_args();
      const int lim = lk_const(p.base, j.slot0 + (place >> 3) % j.slots);
      // (up to 128 keys: a group of 32 per wave)
      if (p.split == 1 && ((lim + p.R + 31) >> 5) - (attn_first_key(attn_args(true), lim) >> 5) <= 4) self_place<1>(l, place); else self_place<2>(l, place);
    }
  }
  // LayerNorm, queries of one head and attention over the source
  __device__ __forceinline__ void cross_attention(int l) {
    constexpr int D = 512;
    const LayersP& p = lk_args();
    const int lane = lk_lane(), lr = lane & 15, lq = lane >> 4;
    const int items = j.cross_places(), mine = j.cross();
    const float* ln = (const float*)((const char*)p.ln2 + l * p.stride);
    const AttnP a = attn_args(false);
    f32x4 g[2], b[2];
    if (mine < items) {
#pragma unroll
      for (int h = 0; h < 2; ++h) { g[h] = *(const f32x4*)(ln + lane * 8 + h * 4); b[h] = *(const f32x4*)(ln + D + lane * 8 + h * 4); }
    }
#pragma unroll 1
    for (int place = mine; place < items; place += j.members) {
      const int h = place & 7, slot = j.slot0 + (place >> 3), s = sequence(slot);
      const size_t at = l * p.src_layer + ((size_t)(s < 0 ? 0 : s) * 8 + h) * p.src_groups * KV_GROUP;
      const rsrc_t kr = rsrc_of(p.crossK + at, (unsigned)p.src_groups * (KV_GROUP * 2)), vr = rsrc_of(p.crossV + at, (unsigned)p.src_groups * (KV_GROUP * 2));
      u32x4 kf[1][4], vf[1][4];
      attn_load_kv<false, 1>(kr, vr, hw, 4, lane, kf, vf);
      const int lim = lk_const(p.src_len, slot);
      if (place != mine) lk_barrier();           // the results of the place before are out of LDS
      lk_norm(p.x1 + (size_t)slot * p.R * D, p.R, g, b, p.eps, xs, hw, lane, poll());
      lk_barrier();
      lk_barrier();
      {
        u32x2 hi, lo;
        lk_halves(partial_sums<4>(lane) * p.scale, hi, lo);
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
      if (s < 0) { empty_rows(p.attn2, slot, h, u32x2{0, 0}, lane); lk_barrier(); continue; }     // (as the attention's own)
      attention_mfma_core<false, false, 0, 1, ATTN_WORDS>(a, sm, h, slot, 0, 0, 0, p.R, 8, 1, hw * 64 + lane, 4, 0, 4, kr, vr, kf, vf, qhi, qlo, lim, p.attn2);
    }
  }

  // The LayerNorm behind the last layer, a row per member
  __device__ __forceinline__ void final_norm() {
    constexpr int D = 512;
    const LayersP& p = lk_args();
    if (hw != 3 || !p.hn) return;
    const int lane = lk_lane();
    f32x4 g[2], b[2], v[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) { g[h] = *(const f32x4*)(p.lnf + lane * 8 + h * 4); b[h] = *(const f32x4*)(p.lnf + D + lane * 8 + h * 4); }
#pragma unroll 1
    for (int m = j.rank; m < j.rows; m += j.members) {
      const size_t row = (size_t)(j.row0 + m) * D;
      const rsrc_t xr = rsrc_of(p.x3 + row, D * 4);
      poll()([&] {
        v[0] = __builtin_bit_cast(f32x4, lk_load16(xr, lane * 32)); v[1] = __builtin_bit_cast(f32x4, lk_load16(xr, lane * 32 + 16));
        return lk_top(lk_top(0, __builtin_bit_cast(u32x4, v[0])), __builtin_bit_cast(u32x4, v[1]));
      });
      const f32x4 s = v[0] + v[1];
      const float mu = wave_sum((s[0] + s[1]) + (s[2] + s[3])) * (1.f / D);
      v[0] -= mu; v[1] -= mu;
      f32x4 q = v[0] * v[0];
#pragma unroll
      for (int r = 0; r < 4; ++r) q[r] = fmaf(v[1][r], v[1][r], q[r]);
      const float rs = inv_sqrt(fmaf(wave_sum((q[0] + q[1]) + (q[2] + q[3])), 1.f / D, p.eps));
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[h][r] = fmaf(v[h][r] * rs, g[h][r], b[h][r]);
      *(f32x4*)(p.h + row + lane * 8) = v[0]; *(f32x4*)(p.h + row + lane * 8 + 4) = v[1];
      *(u32x4*)(p.hn + row + lane * 8) = u32x4{cvt_pk_bf16(v[0][0], v[0][1]), cvt_pk_bf16(v[0][2], v[0][3]), cvt_pk_bf16(v[1][0], v[1][1]), cvt_pk_bf16(v[1][2], v[1][3])};
    }
  }

  __device__ __forceinline__ void job() {
    const int layers = lk_args().n_layers;
    {
      const LayersP& p = lk_args();
      const int lr = lk_lane() & 15;
      const int m = lr < j.rows ? lr : 0, s = m / p.R, slot = j.slot0 + s;
      sb = p.seq ? p.seq[slot] : slot;
      key = p.base[slot] + m - s * p.R;
    }
#pragma unroll 1
    for (int l = 0; l < layers; ++l) {
      // (the first operator of a job follows the launch, or the last operator of the job before, whose rows are others)
      product<QKV, 3, 512>(l);
      self_attention(l);
      product<O, 1, 512>(l);
      cross_attention(l);
      product<CO, 1, 512>(l);
      product<UP, F / 512, 512>(l);
      product<DOWN, 1, F>(l);
    }
    final_norm();
  }
};

template <int F>
struct LkCompute {
  static constexpr int N1 = F / 512, U2 = F / 128;
  const bf16_t* xs;
  f32x4* red;
  int cw;
  LkJob j;
  u32x4 aq[3][4], ao[1][4], ac[1][4], ax[U2 > 16 ? U2 / 4 : 4][4], a1[N1][4];          // ax: the head's queries, the second FFN layer (one tile)

  template <int PACE = 0, int N, int U> __device__ __forceinline__ void load(u32x4 (&a)[N][U], const char* LayersP::*w, int l, int tile) {
    const LayersP& p = lk_args();
    lk_weights<PACE>(a, p.*w + l * p.stride, tile, cw, lk_lane());
  }
  __device__ __forceinline__ u32x4 (&second())[1][U2] { return *reinterpret_cast<u32x4 (*)[1][U2]>(&ax); }
  // An operator: this member's place, whose weights are in registers, then (in a group that is not full) others, fetched as they come
  template <int N, int U>
  __device__ __forceinline__ void product(u32x4 (&a)[N][U], const char* LayersP::*w, int l) {
    lk_barrier();
    lk_multiply<N, U>(a, xs, j.rows, red, cw, lk_lane());
    lk_barrier();
#pragma unroll 1
    for (int place = j.rank + j.members; place < LK_PLACES; place += j.members) {
      load(a, w, l, place * N);
      lk_barrier();
      lk_multiply<N, U>(a, xs, j.rows, red, cw, lk_lane());
      lk_barrier();
    }
  }
  __device__ __forceinline__ void job(unsigned* next_job) {
    load(aq, &LayersP::wqkv, 0, j.rank * 3);
    // A member fetches a layer's weights while it idles: in the self-attention (early) or in the cross-attention; half of those with no part in either
    // take the first
    const bool cross = j.cross() < j.cross_places(), early = cross || ((j.rank & 1) && j.rank >= 8 * j.slots * lk_args().split);
    if (!early) load(ao, &LayersP::wo, 0, j.rank);
    const int layers = lk_args().n_layers;
#pragma unroll 1
    for (int l = 0; l < layers; ++l) {
      const int next = l + 1 < layers ? l + 1 : l;                   // (past the last layer: once more, read by nobody)
      product(aq, &LayersP::wqkv, l);
      if (early) {
        __builtin_amdgcn_s_sleep(LK_HOLD);       // (the operator's own results first)
        load<LK_GAP>(ao, &LayersP::wo, l, j.rank);
        if (cross) load<LK_GAP>(ax, &LayersP::cq, l, (j.cross() & 7) * 4);
        else load<LK_GAP>(second(), &LayersP::w2, l, j.rank);
        load<LK_GAP>(ac, &LayersP::co, l, j.rank);
        load<LK_GAP>(a1, &LayersP::w1, l, j.rank * N1);
        load<LK_GAP>(aq, &LayersP::wqkv, next, j.rank * 3);
      }
      // (the group's next job is fetched in the last layer, when every group has long had its first)
      if (l + 1 == layers && j.rank == 0 && cw == 3 && lk_lane() == 0) {
        const LayersP& p = lk_args();
        const unsigned job = __hip_atomic_fetch_add(p.sync + LK_NEXT_JOB, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        lk_store(next_job, job < (unsigned)p.jobs ? job + 1 : LK_NO_JOB);
      }
      const int self_items = 8 * j.slots * lk_args().split;
#pragma unroll 1
      for (int place = j.rank; place < self_items; place += j.members) {
        if (place != j.rank) lk_barrier();
        lk_barrier();
      }
      product(ao, &LayersP::wo, l);
      if (!early) {
        __builtin_amdgcn_s_sleep(LK_HOLD);
        load<LK_GAP>(ac, &LayersP::co, l, j.rank);
        load<LK_GAP>(a1, &LayersP::w1, l, j.rank * N1);
        load<LK_GAP>(second(), &LayersP::w2, l, j.rank);
        load<LK_GAP>(aq, &LayersP::wqkv, next, j.rank * 3);
        load<LK_GAP>(ao, &LayersP::wo, next, j.rank);
      }
#pragma unroll 1
      for (int place = j.cross(); place < j.cross_places(); place += j.members) {
        if (place != j.cross()) { load(ax, &LayersP::cq, l, (place & 7) * 4); lk_barrier(); }
        lk_barrier();
        lk_multiply(ax, xs, lk_args().R, red, cw, lk_lane());
        lk_barrier();
        lk_barrier();
        lk_barrier();
      }
      product(ac, &LayersP::co, l);
      if (cross) load<LK_PACE>(second(), &LayersP::w2, l, j.rank);
      product(a1, &LayersP::w1, l);
      product(second(), &LayersP::w2, l);
    }
  }
};

template <int F>
struct LkLds {
  static constexpr int XS = 16 * (F + 8) * 2, RED = 4 * 4 * 64 * 16;
  static constexpr int BYTES = XS + RED + (int)AttnLds::BYTES + 512 * 8 + 64;
};

template <int F, bool KVNT>
__global__ __launch_bounds__(512, 2) void layers_kernel(LayersP p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lk_smem[];
  using Lds = LkLds<F>;
  bf16_t* xs = (bf16_t*)lk_smem;
  f32x4* red = (f32x4*)(lk_smem + Lds::XS);
  unsigned char* attn = lk_smem + Lds::XS + Lds::RED;
  u32x2* q_s = (u32x2*)(attn + AttnLds::BYTES);
  int* word = (int*)(q_s + 512);                 // rank, members, job
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  unsigned* area = p.sync + lk_xcd() * LK_AREA;
  unsigned* ctl = area + LK_CTL;
  if (tid == 0) {
    const unsigned old = __hip_atomic_fetch_add(area, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int rank = (int)(old & 0xFFFFu), members = 0;
    if (rank >= p.group || rank >= LK_PLACES || (old & LK_CLOSED)) rank = -1;
    if (rank == 0) {
      const unsigned job = __hip_atomic_fetch_add(p.sync + LK_NEXT_JOB, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const long long t0 = wall_clock64();
      unsigned v;
      do v = lk_load(area);
      while ((int)(v & 0xFFFFu) < p.group && wall_clock64() - t0 < LK_CLOSE_TICKS);
      if ((int)(v & 0xFFFFu) < p.group) v = __hip_atomic_fetch_or(area, LK_CLOSED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      members = (int)(v & 0xFFFFu);
      members = members < p.group ? members : p.group;
      members = members < LK_PLACES ? members : LK_PLACES;
      lk_store(ctl + 1, job < (unsigned)p.jobs ? job + 1 : LK_NO_JOB);
      lk_stores_done();
      lk_store(ctl, members);
    }
    word[0] = rank; word[1] = members;
  }
  lk_barrier();
  LkJob j;
  j.rank = __builtin_amdgcn_readfirstlane(word[0]);
  if (j.rank < 0) return;
  unsigned op = 0;
  bool broken = false;
#pragma unroll 1
  for (int turn = 0;; ++turn) {
    if (wave == 0) {
      unsigned m = word[1], job = 0;
#pragma unroll 1
      for (int s = 0; s < LK_SPINS && (m == 0 || job == 0); ++s) {
        if (m == 0) m = lk_load(ctl);
        if (m != 0) job = lk_load(ctl + 1 + turn);
      }
      if (lane == 0) { word[1] = m; word[2] = job == 0 ? LK_NO_JOB : job; if (job == 0) *p.error = 1; }
    }
    lk_barrier();
    j.members = __builtin_amdgcn_readfirstlane(word[1]);
    const int job = __builtin_amdgcn_readfirstlane(word[2]);
    lk_barrier();
    if (job == (int)LK_NO_JOB) return;
    j.slot0 = (job - 1) * p.per_job;
    j.slots = p.slots - j.slot0 < p.per_job ? p.slots - j.slot0 : p.per_job;
    j.row0 = j.slot0 * p.R; j.rows = j.slots * p.R;
    if (wave >= 4) {
      LkCompute<F> c{xs, red, wave - 4, j};
      c.job(ctl + 2 + turn);
    } else {
      __builtin_amdgcn_s_setprio(3);
      LkHelper<F, KVNT> h{xs, red, AttnLds::carve(attn), q_s, area + LK_FLAGS, wave, j, 0, 0, op, broken};
      h.job();
      op = h.op; broken = h.broken;
    }
  }
}
