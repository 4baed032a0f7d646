// Decode steps of a SMALL model as one kernel on one XCD.
//
// A model whose matrices stream in less time than a kernel boundary costs spends a step on launches: five kernels per
// layer of 3.8 us each at d_model 256, and 8 us between two graph replays.  Here 32 workgroups stay: they
// hand the activations over through memory, five times per layer (q/k/v, attention partials, residual, SwiGLU output,
// residual) and once for the argmax, for as many steps as one call asks for.  Per greedy step, this kernel against the
// kernel chain: 1 / 2 / 8 layers of d_model 256, F 688 11.1 / 19.5 / 72.1 us against 32.7 / 50.6 / 161.2;
// 2 of those layers at 100 / 800 / 1900 keys 23.0 / 29.7 / 36.5 against 51.4 / 52.0 / 53.1; 4 layers of 384 / 1024 51.4
// against 89.3, of 512 / 1408 61.7 against 92.7.  Wider models are left to the chain (4 layers of 512 / 2048 were level at 94
// us, of 768 / 2048 97 against 98): one XCD does not take their weights in fast enough.  Nor does it a long cache or a large
// vocabulary, see sm_max_keys.
//
// What is left: a phase (1.8 us, five to a layer) is one hand-off (store, L2, poll) and a chain of some hundred dependent
// instructions in one wave, whose latencies (9 cycles a product-add, 12 a lane-crossing one, 92 a sum over the wave) weigh as
// much as memory does; some 250 scalars that find no register sit in lanes of vector registers and are read back one by one.
//
// Why one XCD.  Its 32 CUs share an L2, so a value stored by one (the L1s write through) is one L2 hit away from the
// others: one word between two workgroups 0.28 us from store to arrival, polled as here, against 0.43 where they sit on
// different XCDs, and there a vector that all workgroups wait for goes through memory once for every XCD.
// Workgroups are dealt to the XCDs in turn, so every eighth workgroup of the grid takes part and the others leave at
// once.  Were the dealing ever different, a workgroup elsewhere would read SM_EMPTY from its own L2 until its wait runs
// out; it cannot read a wrong value.
//
// Hand-offs without flags, counters or fences.  Every value travels as its own 32-bit word in a buffer that holds the
// bit pattern SM_EMPTY until the value is stored; a reader polls the words it needs until none is SM_EMPTY.
// That is one store and one load of latency, where "store, drain, raise a counter, poll it, load" is a chain of four
// round trips.  SM_EMPTY is a NaN pattern; a result that happens to have it is stored as the default NaN.  Every
// word is written once per step (each layer has its own) and there are two sets of buffers: a step uses the set of
// its epoch and empties the other one once it has seen a whole residual vector behind a down projection, which every
// wave of the grid has contributed to (a row of gate/up each) after it left the previous step.  A wave's
// stores, these and the new key and value rows, are complete before its workgroup hands over its argmax, which
// everyone awaits before the next step.
//
// One wave finishes whole rows: it polls its input straight into registers, multiplies, reduces, finishes and stores,
// with no barrier and no LDS but for the argmax.  (With the input staged in LDS by two waves per workgroup, behind a
// barrier, a step of two layers took 29.6 us instead of 20.0.)  The weights of a phase are requested in front of
// its poll, whose round trip covers theirs; loads return in order.  A wave owns the same two rows of the residual stream
// throughout and keeps them in registers.
//
// Every poll is bounded: past `spin_limit` rounds the wave raises DevState::fault, polls no more and stores no hand-off and no
// cache row any more, so whoever depends on it runs out as well and the grid drains.  No index depends on a value that was
// waited for, and the position and epoch that indexes do depend on are advanced only by a wave that nobody let down: a
// workgroup that starts after the others gave up works at the position they worked at.  The steps without a token report
// -1 and the host takes the multi-kernel path from there.
#pragma once
#include "ll_device.h"

typedef unsigned SmWords __attribute__((ext_vector_type(4)));

#define SM_THREADS 512
#define SM_WAVES (SM_THREADS / 64)
#define SM_XCDS 8              // every SM_XCDS-th workgroup of the grid takes part
#define SM_MAX_WGS 32
#define SM_EMPTY 0xFFFFFFFFu
#define SM_MAX_D 512           // a row is at most one 16-byte piece per lane
#define SM_MAX_F 1536
#define SM_MAX_SPLITS 8        // waves that share the keys of a head, a power of two ...
#define SM_KEYS_PER_SPLIT 64   // ... each with at least this many

struct SmArgs {
  const MkLayer* layers;        // device table, n_layers entries
  const half_t *final_norm, *lm_head, *emb;
  float* x;                     // in: embedding row of the token to feed; out: that of the next one, or the last residual row (steps = 0)
  float* x_keep;                // hidden state of the last step
  float* logits;
  float* amax_val;              // steps = 0: [workgroups taking part]
  int* amax_idx;
  const float2* rope;
  DevState* st;
  int* host_ring;
  float* xch;                   // two sets of hand-off buffers, see SmLayout
  int* epoch;                   // steps run so far; its parity selects the set
  int steps;                    // greedy steps of this launch; 0: one step, its token left to the selection kernel
  int ring_size, n_layers, d, n_heads, F, vocab, max_seq, max_splits, spin_limit;
  int give_up;                  // token (counted from the reset) from which on no wave waits any more; past the ring: none
  float eps;
};

// Hand-off buffers of one layer, in floats: q, k, v [d] each; attention partials [head][max_splits][head_dim + 4]
// (accumulator, m, l, two unused words); residual after the O projection [d]; SwiGLU output [F]; residual after down [d].
// Behind the layers of a set: one argmax candidate (value, index) per workgroup.
struct SmLayout { int q, part, x1, m, x2, total; };
__host__ __device__ inline SmLayout sm_layout(int d, int n_heads, int head_dim, int F, int max_splits) {
  SmLayout L;
  L.q = 0;
  L.part = 3 * d;
  L.x1 = L.part + n_heads * max_splits * (head_dim + 4);
  L.m = L.x1 + d;
  L.x2 = L.m + F;
  L.total = L.x2 + d;
  return L;
}
__host__ __device__ inline size_t sm_set_floats(const SmLayout& L, int n_layers) {
  return (size_t)n_layers * L.total + 2 * SM_MAX_WGS;
}

// Workgroups that take part, 0 where the model is not for this kernel: one per CU of an XCD at most, a row of gate/up for
// every wave, and no more than one row pair of the residual stream per wave
inline int sm_grid(int d, int F, int cus) {
  if (d > SM_MAX_D || F > SM_MAX_F) return 0;
  int g = cus / SM_XCDS < SM_MAX_WGS ? cus / SM_XCDS : SM_MAX_WGS;
  if (g > F / SM_WAVES) g = F / SM_WAVES;
  return g * SM_WAVES * 2 >= d ? g : 0;
}
// Largest number of keys, the new one among them, with which a step is faster here than in the kernel chain; 0: never.
// What the chain's launches cost is won, 10 us a step and 11 a layer; what one XCD takes longer for than eight is lost: 2.45 us
// per million weights of a layer, 3 us per 1000 keys and layer, 0.27 us per row pair of the LM head and wave; and a sampled
// step (one launch of its own, the candidates in memory) wins 12 us less.  Fitted to steps of 1 .. 8 layers of 64 / 136 ..
// 512 / 1536 (d_model / ffn_hidden), both ways; us here / us in the chain, on either side of the line:
//   vocabulary, 20 keys      1 layer of 256 / 688: 32000 37.2 / 42.1, 64000 62.2 / 52.3    1 of 512 / 1408: 16384 34.3 / 38.6,
//                            32000 50.3 / 44.3    4 of 512 / 1408: 32000 93.1 / 103.6, 64000 125.3 / 114.2
//   sampled, top-k 50        1 of 256 / 688: 8192 42.3 / 45.4, 16384 51.0 / 49.3
//   keys, vocabulary 1024    1 of 256 / 688: 6000 34.1 / 38.8, 8000 41.5 / 39.4    8 of 256 / 688: 3000 161.9 / 188.8, 6000
//                            247.9 / 221.7    4 of 512 / 1408: 800 85.6 / 96.1, 3000 116.3 / 105.6
inline int sm_max_keys(int d, int F, int n_layers, int vocab, int grid, bool sampled) {
  const double weights = 4.0 * d * d + 3.0 * d * F;
  const double won = 10.0 + n_layers * (11.0 - 2.45e-6 * weights) - 0.27 * vocab / (2.0 * grid * SM_WAVES) - (sampled ? 12.0 : 0.0);
  const double keys = won / (0.003 * n_layers);
  return keys < 1.0 ? 0 : keys > (1 << 30) ? 1 << 30 : (int)keys;
}
inline int sm_max_splits(int grid, int n_heads) {
  int s = SM_MAX_SPLITS;
  while (s > 1 && n_heads * s > grid * SM_WAVES) s >>= 1;
  return s;
}

// First position of a launch: the state's, but never one from which its steps would run past the cache
__host__ __device__ inline int sm_first_pos(int pos, int steps, int max_seq) {
  const int last = max_seq - (steps > 1 ? steps : 1);
  return pos < last ? pos : last;
}

// Stores that other CUs of the XCD wait for: workgroup scope is through the L1 into the L2 they share
__device__ __forceinline__ unsigned sm_word(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  return u == SM_EMPTY ? 0x7FC00000u : u;
}
__device__ __forceinline__ void sm_put(float* base, unsigned off, float v) {
  __hip_atomic_store(as_global(reinterpret_cast<unsigned*>(reinterpret_cast<char*>(base) + off * 4u)), sm_word(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

struct SmWait {                 // a wave's state of its bounded waits
  DevState* st;
  int limit;
  bool dead;                    // wave-uniform
  __device__ __forceinline__ void give_up() {
    dead = true;
    if ((threadIdx.x & 63) == 0) st_dev_i(&st->fault, 1);
  }
};

// Polls of 16 bytes per lane and item at byte offsets `off` from a buffer of `bytes` bytes, past the L1, until no word
// is SM_EMPTY.  An offset past the buffer reads zeros.
// Who polls stands back, at the lowest priority and with a pause between rounds: without, the older waves of a SIMD kept
// the vector memory pipe to themselves and the younger ones, whose values they waited for, did not get their loads out.
template <int N>
__device__ __forceinline__ void sm_poll(SmWait& w, const float* base, int bytes, const int (&off)[N], SmWords (&v)[N]) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, bytes, 0x00027000);
  __builtin_amdgcn_s_setprio(0);
  for (int spins = 0;; ++spins) {
    asm volatile("" ::: "memory");          // every round loads again
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = __builtin_bit_cast(SmWords, __builtin_amdgcn_raw_buffer_load_b128(r, off[i], 0, 16));
    unsigned top = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) top = max(max(top, max(v[i][0], v[i][1])), max(v[i][2], v[i][3]));
    if (w.dead || !__any(top == SM_EMPTY)) break;
    if (spins >= w.limit) {
      w.give_up();
      break;
    }
    if (spins < 64) __builtin_amdgcn_s_sleep(4);
    else __builtin_amdgcn_s_sleep(64);
  }
  __builtin_amdgcn_s_setprio(3);
  __builtin_amdgcn_sched_barrier(0);        // what follows is requested behind the poll
}
__device__ __forceinline__ f4 sm_f4(SmWords v) { return __builtin_bit_cast(f4, v); }

// Value of lane ^ 16 combined with the lane's own, and of lane ^ 32: the odd rows of one copy change places with the even
// rows of the other (halves likewise), which leaves both values of a pair in every lane.  (The wait states are those the
// compiler puts between a vector instruction and its own use of these; its builtin returned the first result twice.)
template <class Op>
__device__ __forceinline__ float sm_across16(float v, Op op) {
  float w = v;
  asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(v), "+v"(w));
  return op(v, w);
}
template <class Op>
__device__ __forceinline__ float sm_across32(float v, Op op) {
  float w = v;
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(v), "+v"(w));
  return op(v, w);
}
struct SmSum { __device__ float operator()(float a, float b) const { return a + b; } };
struct SmMax { __device__ float operator()(float a, float b) const { return fmaxf(a, b); } };
// over the lane groups of a wave (HD / 8 lanes each): every lane gets the result of its column
template <int HD, class Op>
__device__ __forceinline__ float sm_across_groups(float v, Op op) {
  if (HD == 64) v = op(v, dpp_mov<0x128>(v));       // row_ror:8 = lane ^ 8
  return sm_across32(sm_across16(v, op), op);
}

// (v, i) of the largest v over a wave, the lowest i among equals
__device__ __forceinline__ void sm_argmax(float& v, int& i) {
  float top = fmaxf(v, dpp_mov<0xB1>(v));
  top = fmaxf(top, dpp_mov<0x4E>(top));
  top = fmaxf(top, dpp_mov<0x141>(top));
  top = fmaxf(top, dpp_mov<0x140>(top));
  top = sm_across32(sm_across16(top, SmMax()), SmMax());
  unsigned long long at = __ballot(v == top);
  int low = 0x7fffffff;
  for (; at; at &= at - 1) low = min(low, __builtin_amdgcn_readlane(i, __builtin_ctzll(at)));
  v = top;
  i = low;
}

// Lower half: a summed over lanes i and i ^ 32; upper half: b.  Likewise even and odd rows of 16.
__device__ __forceinline__ float sm_trade32(float a, float b) {
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  return a + b;
}
__device__ __forceinline__ float sm_trade16(float a, float b) {
  asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  return a + b;
}

// A pair of weight rows of at most NI * 512 (HALF: 256) columns.  HALF: the two halves of the wave hold a row each, one
// 16-byte piece per lane; otherwise piece lane + 64 i of both rows.  A piece past the row re-reads the last one and
// meets zeros.
template <int NI, bool HALF> struct SmPair { h8 w[HALF ? 1 : 2 * NI]; };
template <int NI, bool HALF>
__device__ __forceinline__ void sm_load(SmPair<NI, HALF>& w, const half_t* pa, const half_t* pb, int nch, int lane) {
  if (HALF) {
    w.w[0] = load_h8((lane < 32 ? pa : pb) + min(lane & 31, nch - 1) * 8);
  } else {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = min(lane + 64 * i, nch - 1) * 8;
      w.w[2 * i] = load_h8(pa + c);
      w.w[2 * i + 1] = load_h8(pb + c);
    }
  }
}
// (two chains of four: a dependent product-add is waited for twice as long as it is issued)
__device__ __forceinline__ float sm_dot8(h8 w, const f4 (&x)[2]) {
  float a = (float)w[0] * x[0][0], b = (float)w[4] * x[1][0];
#pragma unroll
  for (int e = 1; e < 4; ++e) {
    a += (float)w[e] * x[0][e];
    b += (float)w[4 + e] * x[1][e];
  }
  return a + b;
}
// sums over the two halves of a wave (wave-uniform)
__device__ __forceinline__ float2 sm_half_sums(float v) {
  const int b = __builtin_bit_cast(int, group_sum<16>(v));
  return make_float2(
      __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 0)) + __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 16)),
      __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 32)) + __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 48)));
}
template <int NI, bool HALF>
__device__ __forceinline__ float2 sm_dot(const SmPair<NI, HALF>& w, const f4 (&x)[NI][2]) {
  if (HALF) return sm_half_sums(sm_dot8(w.w[0], x[0]));
  float ra = 0.f, rb = 0.f;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    ra += sm_dot8(w.w[2 * i], x[i]);
    rb += sm_dot8(w.w[HALF ? 0 : 2 * i + 1], x[i]);
  }
  return sm_half_sums(sm_trade32(ra, rb));
}

// Row pair p of the Q/K/V projection: RoPE partners of q or k, neighbours of v
struct SmRows { int sec, a, b; };
template <int HD>
__device__ __forceinline__ SmRows sm_qkv_rows(int p, int d) {
  const int half = d >> 1, sec = p >= 2 * half ? 2 : p >= half ? 1 : 0, pp = p - sec * half;
  if (sec < 2) {
    const int r = pp / (HD / 2) * HD + pp % (HD / 2);
    return {sec, r, r + HD / 2};
  }
  return {sec, 2 * pp, 2 * pp + 1};
}

struct SmQkv { const half_t *q, *k, *v, *gain; };

// HD: head_dim; NF: 512-column pieces of an F-vector; HALF: d_model <= 256
template <int HD, int NF, bool HALF>
__global__ __launch_bounds__(SM_THREADS) void decode_small_kernel(SmArgs a) {
  constexpr int LPR = HD / 8, GPW = 64 / LPR, UK = 4, HH = HD / 2;
  constexpr int RQ = 2, RG = 3;    // row pairs per wave fetched ahead: Q/K/V and LM head, gate/up
  typedef SmPair<1, HALF> Pair;
  __shared__ float s_bv[SM_WAVES];
  __shared__ int s_bi[SM_WAVES];
  if (blockIdx.x % SM_XCDS != 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wg = blockIdx.x / SM_XCDS, nwg = gridDim.x / SM_XCDS;
  const int gw = wg * SM_WAVES + wave, GW = nwg * SM_WAVES;
  const int d = a.d, F = a.F, nch_d = d >> 3, nch_f = F >> 3;
  const int n_qkv = 3 * (d >> 1), n_lm = (a.vocab + 1) >> 1;
  const bool owner = 2 * gw < d;                   // of residual rows 2 gw and 2 gw + 1
  const int epoch0 = ld_dev_i(a.epoch), pos0 = sm_first_pos(a.st->pos, a.steps, a.max_seq), ring0 = a.st->steps;
  const SmLayout L = sm_layout(d, a.n_heads, HD, F, a.max_splits);
  const LL_GLOBAL MkLayer* table = as_global(a.layers);
  const int piece = HALF ? lane & 31 : lane;       // this lane's 8 columns of a d-vector
  const int fault0 = ld_dev_i(&a.st->fault);       // from memory, not from a scalar cache
  SmWait wait{a.st, a.spin_limit, false};

  SmRows rows[RQ];
#pragma unroll
  for (int i = 0; i < RQ; ++i) rows[i] = sm_qkv_rows<HD>(min(gw + i * GW, n_qkv - 1), d);
  Pair wq[RQ], wo, wgu[RG];
  SmPair<NF, false> wd;
  h8 gn;
  auto load_qkv = [&](Pair& w, const SmRows& r, const SmQkv& t) {
    const half_t* base = r.sec == 0 ? t.q : r.sec == 1 ? t.k : t.v;
    sm_load(w, base + (size_t)r.a * d, base + (size_t)r.b * d, nch_d, lane);
  };
  auto load_lm = [&](Pair& w, int p) {
    sm_load(w, a.lm_head + (size_t)(2 * p) * d, a.lm_head + (size_t)min(2 * p + 1, a.vocab - 1) * d, nch_d, lane);
  };
  auto load_gain = [&](const half_t* gain) { gn = load_h8(gain + min(piece, nch_d - 1) * 8); };
  auto qkv_of = [&](int l) { return SmQkv{table[l].wq, table[l].wk, table[l].wv, table[l].attn_norm}; };
  auto fetch_qkv = [&](const SmQkv& t) {
#pragma unroll
    for (int i = 0; i < RQ; ++i) load_qkv(wq[i], rows[i], t);
    load_gain(t.gain);
  };
  const SmQkv first_qkv = qkv_of(0);

  // the residual row (raw) and the wave's two elements of it
  f4 x[1][2], xg[1][2];
  float res0 = 0.f, res1 = 0.f;
  x[0][0] = x[0][1] = f4{0.f, 0.f, 0.f, 0.f};
  if (piece < nch_d) {
    x[0][0] = *as_global(reinterpret_cast<const f4*>(a.x + piece * 8));
    x[0][1] = *as_global(reinterpret_cast<const f4*>(a.x + piece * 8 + 4));
  }
  if (owner) { res0 = a.x[2 * gw]; res1 = a.x[2 * gw + 1]; }
  fetch_qkv(first_qkv);
  wait.dead = __builtin_amdgcn_readfirstlane(fault0) != 0;     // where an earlier step of the call gave up, this one does at once
  auto poll_x = [&](const float* src) {
    const int off[2] = {piece * 32, piece * 32 + 16};
    SmWords v[2];
    sm_poll(wait, src, d * 4, off, v);
    x[0][0] = sm_f4(v[0]);
    x[0][1] = sm_f4(v[1]);
  };
  // xg = x * gain; returns the norm's factor
  auto norm = [&]() {
    float ss = 0.f;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        ss += x[0][h][e] * x[0][h][e];
        xg[0][h][e] = x[0][h][e] * (float)gn[h * 4 + e];
      }
    const float s = HALF ? sm_half_sums(ss).x : wave_sum(ss);
    return 1.0f / sqrtf(s / (float)d + a.eps);
  };
  auto put2 = [&](float* base, unsigned oa, unsigned ob, float va, float vb) {     // two words, by lanes 0 and 1
    if (lane < 2 && !wait.dead) sm_put(base, lane ? ob : oa, lane ? vb : va);
  };

  int tok = 0;
  for (int step = 0; step == 0 || step < a.steps; ++step) {
    if (ring0 + step >= a.give_up) wait.give_up();
    const int epoch = epoch0 + step, pos = pos0 + step, n_keys = pos + 1;
    float* set = a.xch + (size_t)(epoch & 1) * sm_set_floats(L, a.n_layers);
    auto empty_other = [&]() {
      float* other = a.xch + (size_t)((epoch & 1) ^ 1) * sm_set_floats(L, a.n_layers);
      const size_t n4 = sm_set_floats(L, a.n_layers) / 4;
      const SmWords e = {SM_EMPTY, SM_EMPTY, SM_EMPTY, SM_EMPTY};
      if (!wait.dead)
        for (size_t i = (size_t)wg * SM_THREADS + tid; i < n4; i += (size_t)nwg * SM_THREADS)
          *as_global(reinterpret_cast<SmWords*>(other + i * 4)) = e;
    };
    // waves that share a head's keys (a power of two), and this wave's first (head, split)
    int ls = 0;
    while ((2 << ls) <= a.max_splits && (SM_KEYS_PER_SPLIT << ls) < n_keys) ++ls;
    // (dealt from the last wave on: the first ones have a row pair more to finish)
    const int S = 1 << ls, task0 = (SM_WAVES - 1 - wave) * nwg + nwg - 1 - wg;
    const int gi = lane / LPR, li = lane % LPR;
    const int last_old = pos > 0 ? pos - 1 : 0;        // the new row comes through the hand-off, not from the cache
    float2 cs[RQ];
#pragma unroll
    for (int i = 0; i < RQ; ++i) {
      cs[i] = make_float2(1.f, 0.f);
      if (rows[i].sec < 2) cs[i] = a.rope[(size_t)pos * HH + rows[i].a % HD];
    }

    for (int l = 0; l < a.n_layers; ++l) {
      float* B = set + (size_t)l * L.total;
      half_t *kc = table[l].kc, *vc = table[l].vc;
      const SmQkv next_qkv = qkv_of(min(l + 1, a.n_layers - 1));
      const half_t *w_o = table[l].wo, *w_g = table[l].w_gate, *w_u = table[l].w_up, *w_d = table[l].w_down;

      // ---- RMSNorm, Q/K/V, RoPE, cache row
      if (l > 0) poll_x(B - L.total + L.x2);
      h8 kk[UK], vv[UK];
      auto fetch_keys = [&](int head, int base) {
        const half_t* kh = kc + (size_t)head * a.max_seq * HD + li * 8;
        const half_t* vh = vc + (size_t)head * a.max_seq * HD + li * 8;
#pragma unroll
        for (int j = 0; j < UK; ++j) {
          const int u = min(base + ((j * GPW) << ls), last_old);
          kk[j] = load_h8(kh + (size_t)u * HD);
          vv[j] = load_h8(vh + (size_t)u * HD);
        }
      };
      if (l == 1) empty_other();
      float inv = norm();
      // lanes 2 i and 2 i + 1 finish the two elements of pair i
      float2 t[RQ];
#pragma unroll
      for (int i = 0; i < RQ; ++i) t[i] = sm_dot(wq[i], xg);
      auto finish_qkv = [&](float2 t, const SmRows& r, float2 c) {
        const bool second = lane & 1;
        const float own = (second ? t.y : t.x) * inv, other = (second ? t.x : t.y) * inv;
        float v = own * c.x + (second ? other : -other) * c.y;
        const int row = second ? r.b : r.a;
        if (r.sec > 0) {
          const half_t h = (half_t)v;
          if (!wait.dead) ((r.sec == 1 ? kc : vc) + ((size_t)(row / HD) * a.max_seq + pos) * HD)[row % HD] = h;
          v = (float)h;
        }
        if (!wait.dead) sm_put(B, L.q + r.sec * d + row, v);
      };
      {
        SmRows r = rows[0];
        float2 tt = t[0], c = cs[0];
#pragma unroll
        for (int i = 1; i < RQ; ++i)
          if (lane >= 2 * i) { r = rows[i]; tt = t[i]; c = cs[i]; }
        if (lane < 2 * RQ && gw + (lane >> 1) * GW < n_qkv) finish_qkv(tt, r, c);
      }
      for (int p = gw + RQ * GW; p < n_qkv; p += GW) {
        const SmRows r = sm_qkv_rows<HD>(p, d);
        Pair w;
        load_qkv(w, r, qkv_of(l));
        float2 c = make_float2(1.f, 0.f);
        if (r.sec < 2) c = a.rope[(size_t)pos * HH + r.a % HD];
        const float2 tp = sm_dot(w, xg);
        if (lane < 2) finish_qkv(tp, r, c);
      }
      if (task0 < a.n_heads << ls) fetch_keys(task0 >> ls, (task0 & (S - 1)) * GPW + gi);
      if (owner) sm_load(wo, w_o + (size_t)(2 * gw) * d, w_o + (size_t)(2 * gw + 1) * d, nch_d, lane);

      // ---- attention of the new query: wave task = (head, split), keys dealt round robin over all lane groups of a
      // head's splits
      for (int task = task0; task < a.n_heads << ls; task += GW) {
        const int head = task >> ls, first = (task & (S - 1)) * GPW + gi, stride = GPW << ls;
        if (task != task0) fetch_keys(head, first);
        // the query; the lane group that is dealt the new key also waits for its key and value
        const bool mine = (pos & (stride - 1)) == first;
        const int oq = (head * HD + li * 8) * 4, ok = mine ? oq + d * 4 : 0x40000000, ov = mine ? oq + d * 8 : 0x40000000;
        const int off[6] = {oq, oq + 16, ok, ok + 16, ov, ov + 16};
        SmWords hv[6];
        sm_poll(wait, B + L.q, 3 * d * 4, off, hv);
        const f4 q0 = sm_f4(hv[0]), q1 = sm_f4(hv[1]);
        h8 kn, vn;                                    // (zeros where the new key is another group's)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          kn[e] = (half_t)sm_f4(hv[2])[e]; kn[4 + e] = (half_t)sm_f4(hv[3])[e];
          vn[e] = (half_t)sm_f4(hv[4])[e]; vn[4 + e] = (half_t)sm_f4(hv[5])[e];
        }
        float m = -INFINITY, l_sum = 0.f, acc[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = 0.f;
        const float scale = 1.0f / sqrtf((float)HD);
        for (int base = first; base - gi < n_keys; base += UK * stride) {      // (uniform over a wave: groups differ by gi)
          if (base != first) fetch_keys(head, base);
          float dot[UK], mn = m;
#pragma unroll
          for (int j = 0; j < UK; ++j) {
            const int u = base + j * stride;
            if (u >= pos) { kk[j] = kn; vv[j] = vn; }                          // the new key; behind it: anything finite
            float t = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) t += q0[e] * (float)kk[j][e] + q1[e] * (float)kk[j][4 + e];
            t = group_sum<LPR>(t) * scale;
            dot[j] = u < n_keys ? t : -INFINITY;
            mn = fmaxf(mn, dot[j]);
          }
          const float corr = (m == mn) ? 1.0f : __expf(m - mn);       // also m = mn = -inf
          l_sum *= corr;
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] *= corr;
#pragma unroll
          for (int j = 0; j < UK; ++j) {
            const float w = (dot[j] > -INFINITY) ? __expf(dot[j] - mn) : 0.f;
            l_sum += w;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += w * (float)vv[j][e];
          }
          m = mn;
        }
        // the lane groups' states into one: maximum and denominator in every lane; of the accumulators, halves and then rows
        // trade the columns they do not finish, so a lane ends with columns li * 8 + 2 (lane / 16) and + 1
        const float M = sm_across_groups<HD>(m, SmMax());
        const float wgt = (m > -INFINITY) ? __expf(m - M) : 0.f;
        l_sum = sm_across_groups<HD>(l_sum * wgt, SmSum());
        float r4[4], r2[2];
#pragma unroll
        for (int e = 0; e < 4; ++e) r4[e] = sm_trade32(acc[e] * wgt, acc[4 + e] * wgt);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          r2[e] = sm_trade16(r4[e], r4[2 + e]);
          if (HD == 64) r2[e] += dpp_mov<0x128>(r2[e]);
        }
        const unsigned out = L.part + (head * a.max_splits + (task & (S - 1))) * (HD + 4);
        if (!wait.dead) {
          if (HD == 128 || (lane & 8) == 0) {
            sm_put(B, out + li * 8 + 2 * (lane >> 4), r2[0]);
            sm_put(B, out + li * 8 + 2 * (lane >> 4) + 1, r2[1]);
          }
          if (lane < 4) sm_put(B, out + HD + lane, lane == 0 ? M : lane == 1 ? l_sum : 0.f);
        }
      }

      // ---- merge of the partials, O projection, residual
      if (owner) {
        const int head = piece * 8 / HD, col = piece * 8 % HD;
        float mm = -INFINITY, den = 0.f;
        f4 o[1][2];
        o[0][0] = o[0][1] = f4{0.f, 0.f, 0.f, 0.f};
        if (S == 1) {
          const int p0 = piece < nch_d ? head * a.max_splits * (HD + 4) * 4 : 0x40000000;
          const int off[3] = {p0 + col * 4, p0 + col * 4 + 16, p0 + HD * 4};
          SmWords v[3];
          sm_poll(wait, B + L.part, a.n_heads * a.max_splits * (HD + 4) * 4, off, v);
          o[0][0] = sm_f4(v[0]);
          o[0][1] = sm_f4(v[1]);
          den = sm_f4(v[2])[1];
        } else {
          // first the (m, l) words alone, one per lane and head: polling whole partials from every wave would be 3 MB a round
          for (int i0 = 0; i0 < a.n_heads << ls; i0 += 64) {
            const int i = i0 + lane;
            const int off[1] = {i < a.n_heads << ls ? (((i >> ls) * a.max_splits + (i & (S - 1))) * (HD + 4) + HD) * 4 : 0x40000000};
            SmWords v[1];
            sm_poll(wait, B + L.part, a.n_heads * a.max_splits * (HD + 4) * 4, off, v);
          }
        }
        for (int s0 = 0; S > 1 && s0 < S; s0 += 4) {              // four partials per round trip
          int off[12];
          SmWords v[12];
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int p0 = piece < nch_d && s0 + s < S ? (head * a.max_splits + s0 + s) * (HD + 4) * 4 : 0x40000000;
            off[3 * s] = p0 + col * 4;
            off[3 * s + 1] = p0 + col * 4 + 16;
            off[3 * s + 2] = p0 + HD * 4;
          }
          sm_poll(wait, B + L.part, a.n_heads * a.max_splits * (HD + 4) * 4, off, v);
          float M = mm, ms[4];
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            ms[s] = s0 + s < S ? sm_f4(v[3 * s + 2])[0] : -INFINITY;
            M = fmaxf(M, ms[s]);
          }
          const float keep = mm > -INFINITY ? __expf(mm - M) : 0.f;
          den *= keep;
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) o[0][h][e] *= keep;
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const float w = ms[s] > -INFINITY ? __expf(ms[s] - M) : 0.f;
            if (s0 + s < S) {
              den += w * sm_f4(v[3 * s + 2])[1];
#pragma unroll
              for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) o[0][h][e] += w * sm_f4(v[3 * s + h])[e];
            }
          }
          mm = M;
        }
        const float r = 1.0f / den;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[0][h][e] = piece < nch_d ? o[0][h][e] * r : 0.f;
        const float2 t = sm_dot(wo, o);
        res0 += t.x;
        res1 += t.y;
        put2(B, L.x1 + 2 * gw, L.x1 + 2 * gw + 1, res0, res1);
      }
#pragma unroll
      for (int i = 0; i < RG; ++i) {
        const size_t row = (size_t)min(gw + i * GW, F - 1) * d;
        sm_load(wgu[i], w_g + row, w_u + row, nch_d, lane);
      }
      load_gain(table[l].ffn_norm);

      // ---- RMSNorm, gate/up, SwiGLU
      poll_x(B + L.x1);
      if (owner) sm_load(wd, w_d + (size_t)(2 * gw) * F, w_d + (size_t)(2 * gw + 1) * F, nch_f, lane);
      inv = norm();
      // lane i finishes pair i of up to RG at a time
      for (int p = gw; p < F; p += RG * GW) {
        float2 t[RG];
#pragma unroll
        for (int i = 0; i < RG; ++i) t[i] = sm_dot(wgu[i], xg);
        if (p + RG * GW < F)
#pragma unroll
          for (int i = 0; i < RG; ++i) {
            const size_t row = (size_t)min(p + (RG + i) * GW, F - 1) * d;
            sm_load(wgu[i], w_g + row, w_u + row, nch_d, lane);
          }
        float2 tt = t[0];
#pragma unroll
        for (int i = 1; i < RG; ++i)
          if (lane == i) tt = t[i];
        const float h = pt_swiglu(tt.x * inv, tt.y * inv);
        if (lane < RG && p + lane * GW < F && !wait.dead) sm_put(B, L.m + p + lane * GW, h);
      }

      // ---- down projection, residual
      if (l + 1 < a.n_layers) {
        fetch_qkv(next_qkv);
      } else {
#pragma unroll
        for (int i = 0; i < RQ; ++i) load_lm(wq[i], min(gw + i * GW, n_lm - 1));
        load_gain(a.final_norm);
      }
      if (owner) {
        f4 xm[NF][2];
        int off[2 * NF];
        SmWords v[2 * NF];
#pragma unroll
        for (int i = 0; i < NF; ++i) {
          off[2 * i] = (lane + 64 * i) * 32;
          off[2 * i + 1] = off[2 * i] + 16;
        }
        sm_poll(wait, B + L.m, F * 4, off, v);
#pragma unroll
        for (int i = 0; i < NF; ++i) {
          xm[i][0] = sm_f4(v[2 * i]);
          xm[i][1] = sm_f4(v[2 * i + 1]);
        }
        const float2 t = sm_dot(wd, xm);
        res0 += t.x;
        res1 += t.y;
        put2(B, L.x2 + 2 * gw, L.x2 + 2 * gw + 1, res0, res1);
      }
    }

    // ---- final RMSNorm, LM head, argmax candidates
    poll_x(set + (size_t)(a.n_layers - 1) * L.total + L.x2);
    if (a.n_layers == 1) empty_other();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this wave's stores for later steps are in the L2
    const float inv = norm();
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    auto finish_lm = [&](float2 t, int p) {
      const float ra = t.x * inv, rb = t.y * inv;
      const int r0 = 2 * p;
      const bool two = r0 + 1 < a.vocab;
      if (lane == 0) {
        a.logits[r0] = ra;
        if (two) a.logits[r0 + 1] = rb;
      }
      if (ra > bv) { bv = ra; bi = r0; }             // rows come in ascending order: ties keep the lower index
      if (two && rb > bv) { bv = rb; bi = r0 + 1; }
    };
    float2 t[RQ];
#pragma unroll
    for (int i = 0; i < RQ; ++i) t[i] = sm_dot(wq[i], xg);
#pragma unroll
    for (int i = 0; i < RQ; ++i)
      if (gw + i * GW < n_lm) finish_lm(t[i], gw + i * GW);
    if (gw + RQ * GW < n_lm) {
      load_lm(wq[0], gw + RQ * GW);
      for (int p = gw + RQ * GW; p < n_lm; p += GW) {
        const Pair w = wq[0];
        if (p + GW < n_lm) load_lm(wq[0], p + GW);
        finish_lm(sm_dot(w, xg), p);
      }
    }
    if (lane == 0) {
      s_bv[wave] = bv;
      s_bi[wave] = wait.dead ? -1 : bi;
    }
    if (wg == 0 && wave == 0 && !wait.dead && lane == piece && piece < nch_d) {
      float* keep = (a.steps > 0 ? a.x_keep : a.x) + piece * 8;
      *as_global(reinterpret_cast<f4*>(keep)) = x[0][0];
      *as_global(reinterpret_cast<f4*>(keep + 4)) = x[0][1];
    }
    __syncthreads();
    float* cand = set + (size_t)a.n_layers * L.total;
    if (wave == 0) {
      bv = lane < SM_WAVES ? s_bv[lane] : -INFINITY;
      bi = lane < SM_WAVES ? s_bi[lane] : 0x7fffffff;
      wait.dead |= __any(bi < 0) != 0;               // a wave of this workgroup has nothing to compare
      sm_argmax(bv, bi);
      if (a.steps == 0 && lane == 0) {
        a.amax_val[wg] = bv;
        a.amax_idx[wg] = wait.dead ? 0x7fffffff : bi;   // (no candidate)
      }
      if (a.steps > 0) {
        put2(cand, 2 * wg, 2 * wg + 1, bv, __builtin_bit_cast(float, bi));
        if ((nwg & 1) && wg == nwg - 1) put2(cand, 2 * nwg, 2 * nwg + 1, -INFINITY, __builtin_bit_cast(float, 0x7fffffff));
      }
    }
    if (a.steps == 0) break;
    if (step + 1 < a.steps) fetch_qkv(first_qkv);
    // the workgroups' candidates, two per lane, and the token
    const int off[1] = {2 * lane < nwg ? lane * 16 : 0x40000000};
    SmWords c[1];
    sm_poll(wait, cand, 2 * SM_MAX_WGS * 4, off, c);
    const bool second = sm_f4(c[0])[2] > sm_f4(c[0])[0] || (sm_f4(c[0])[2] == sm_f4(c[0])[0] && (int)c[0][3] < (int)c[0][1]);
    bv = 2 * lane < nwg ? sm_f4(c[0])[second ? 2 : 0] : -INFINITY;
    bi = 2 * lane < nwg ? (int)(second ? c[0][3] : c[0][1]) : 0x7fffffff;
    sm_argmax(bv, bi);
    tok = (unsigned)bi < (unsigned)a.vocab ? bi : 0;      // every logit NaN, or a wait ran out: still a valid id
    if (wg == 0 && tid == 0 && ring0 + step < a.ring_size) a.host_ring[ring0 + step] = wait.dead ? -1 : tok;
    // the next step's input: the token's embedding row
    const half_t* e = a.emb + (size_t)tok * d;
    if (piece < nch_d) {
      const h8 v = load_h8(e + piece * 8);
#pragma unroll
      for (int i = 0; i < 8; ++i) x[0][i >> 2][i & 3] = (float)v[i];
    }
    if (owner) {
      res0 = (float)*as_global(e + 2 * gw);
      res1 = (float)*as_global(e + 2 * gw + 1);
    }
  }
  // Only where no wait ran out: then every workgroup has read the state, each one having stored a part of a SwiGLU output
  // that this wave waited for.  Otherwise one may still be to come, and the host writes the state anew.
  if (wg == 0 && wave == 0 && !wait.dead) {
    if (a.steps > 0 && lane == piece && piece < nch_d) {
      *as_global(reinterpret_cast<f4*>(a.x + piece * 8)) = x[0][0];
      *as_global(reinterpret_cast<f4*>(a.x + piece * 8 + 4)) = x[0][1];
    }
    if (lane == 0) {
      const int run = a.steps > 0 ? a.steps : 1;
      *a.epoch = epoch0 + run;
      if (a.steps > 0) {
        a.st->pos = pos0 + run;
        a.st->steps = ring0 + run;
        a.st->next_token = tok;
      }
    }
  }
}
