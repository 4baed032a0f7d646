// Projections of a prompt of 33..1024 rows for gfx950 (Sec. IV-E / Table I, the upper part of the TTFT range)
// where the workspace holds the fragment-major weight copy: fp16 activations times fp16 weights on
// v_mfma_f32_32x32x16_f16, the layer's own epilogue (RoPE + KV-cache write, SwiGLU) in the same kernel.
//
// A tile spans the whole K loop wherever the output is wide (Q/K/V, gate/up), so that the epilogue runs on
// finished sums in registers: a 32-row weight block is two 16-row blocks of the copy, whose RoPE partners and
// gate / up rows land in the same lane.  Tile sizes are chosen so that one round of workgroups covers the
// projection (e.g. gate/up at 512 rows: 2 x 115 tiles of 256 x 192).  The residual projections have only
// d_model columns and cut their K loop into `ks` pieces, each a slice of fp32 partial products that the
// next RMSNorm adds up.
//
// What bounds these kernels, measured with timing-only builds.  Every byte of both operands enters a CU through
// its vector L1 once per tile, (rows + columns) * K * 2.  A CU's loads come back in the order they were issued, whichever
// wave issued them, and some 70 KB of them are in flight at most: what stands behind a weight that comes from HBM waits as
// long as that weight.  So a CU takes 60 .. 75 GB/s of a mixed stream (gate/up at 250 rows on a quarter of the chip: the
// weights alone 18 us, the activations alone 20, both 44), where it takes 150 of the activations alone, deeper look-ahead
// changes nothing, and tiles are as square as a single round allows.  The weights' loads are therefore the work of four
// waves of their own: a stage at a time, back to back, while the four waves that multiply never wait to issue, and with
// no more stages in flight than it takes (rings of 5 and 6 stages are slower).  Before, the multiplying waves dealt the
// weights' loads out behind their matrix instructions, or, up to 192 rows, brought them to registers; now, us at
// 64 / 128 / 192 / 256 / 384 / 512 rows, before -> with waves that load:
//   Q/K/V    22.8 30.0 35.7 40.1 50.6 55.7 -> 22.4 27.2 35.0 38.4 47.1 52.0
//   gate/up  34.4 39.6 49.2 55.0 74.1      -> 31.2 39.2 46.5 49.7 65.0
//   O         9.6 12.3 16.0 18.2 22.6 25.9 ->  9.2 11.3 14.6 16.2 20.7 24.0
//   down     20.3 26.1 32.0 36.5 42.1 48.0 -> 19.5 23.4 29.3 31.1 42.3 45.2
// (gate/up at 128 and Q/K/V at 192 and 256 rows have gained again since, see pt_pairs)
// At 512 rows and more the matrix instructions
// are the larger part (gate/up at 512 rows: 98 k of 114 k cycles in the K loop) and the chip runs them at 1.6-1.8
// GHz; tiles of 256 x 192 leave no registers for a second wave per SIMD, and keep the old way.  LDS holds only the weights
// (direct loads in, 4 or 2 fragment reads per byte out); the activations go straight to registers.  With both operands in
// LDS (128 x 256 tiles, eight waves) the LDS port was busy 1.4 times as long as the matrix cores: gate/up at 512 rows
// 110 us + 16 us SwiGLU kernel against 88 us here, Q/K/V 67 + 12 against 59.
//
// v_mfma_f32_32x32x16_f16: 1.76 PFLOP/s from one wave per SIMD; the 16x16x32 form reaches 1.1.
#pragma once
#include "ll_device.h"
#include "prefill_skinny.h"

struct TileArgs {
  const half_t* A;        // activations [rows of the bucket][K] fp16, fragment-major with tb token blocks
  const half_t* Wf;       // weights, fragment-major (sk_shuffle_kernel): 1 KB per 16-row block and 32-wide K step
  const DevState* st;
  int N, K, tb;
  int mtiles, ctiles, ks; // row tiles, column tiles, pieces of the K loop
  int upt;                // 16-row weight blocks of a column tile, at most 2 NB (the rest reads as zero, without traffic)
  half_t* Hout;           // GATEUP: [rows][N] fp16, fragment-major
  half_t* Q;              // QKV: [rows][N] fp16 rotated queries
  half_t* kc;             // QKV: this layer's K cache [head][max_seq][head_dim]
  half_t* vc;
  const float2* rope;     // [max_seq][head_dim / 2] (cos, sin)
  int head_dim, max_seq;
  float* C;               // RES: slices [ks][rows][N] fp32
  size_t slice_floats;
};

// 16-row blocks a projection's tiles cover: gate/up includes the rows that fill the last 32-wide K step of the
// down projection behind it (their weights read as zero, so zeros are stored: the buffer may hold anything)
__host__ __device__ inline int pt_units(int mode, int N) {
  return mode == SK_GATEUP ? (N + 31) / 32 * 4 : skinny_units(mode, N);
}

#define PT_WAVES 4           // waves that multiply
// Tiles whose accumulators leave room for two waves per SIMD have four more waves, which load the weights
__host__ __device__ constexpr bool pt_fed(int mt, int nb) { return mt * nb <= 9; }
__host__ __device__ constexpr int pt_threads(int mt, int nb) { return (pt_fed(mt, nb) ? 2 : 1) * PT_WAVES * 64; }
#define PT_LDS_BYTES(NB, S32, NS) ((NS) * (NB) * (S32) * 2048)

// g / (1 + expf(-g)) * u at the library functions' own error (max 2.2e-7, rms 4.6e-8 of the value against 64 bits over
// |g| <= 86; infinities and NaN give the same), without what they spend on arguments that cannot occur here: a
// lane of a 256 x 192 tile finishes 96 of these.  exp(-g) = 2^t 2^f with t the nearest integer to -g log2(e) and f
// from log2(e) in two parts; past +-88.8 the exponential is infinite or nothing beside the 1.  The quotient is
// g * rcp(d) with its remainder added once; div_fixup settles infinite operands.  Gate/up of the 7B shape at 250 /
// 500 / 1000 rows 59.7 / 87.7 / 169.8 us with the library's functions, 59.2 / 85.5 / 165.5 this way (rcp(1 + __expf(-g)), up to
// 3.9e-6 off: 58.0 / 83.5 / 161.9).
__device__ __forceinline__ float pt_swiglu(float g, float u) {
  const float x = __builtin_amdgcn_fmed3f(g, -88.8f, 88.8f);
  const float t = __builtin_rintf(x * -1.44269502f);
  const float f = __builtin_fmaf(x, -1.92596303e-8f, __builtin_fmaf(x, -1.44269502f, -t));
  const float d = 1.0f + __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f(f), (int)t);
  const float r = __builtin_amdgcn_rcpf(d);
  const float q = g * r;
  return __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-d, q, g), r, q), d, g) * u;
}

// Cosines and sines of the four RoPE pairs that a lane finishes in 16-row block u of Q/K/V.  A head's blocks are a power of
// two of its rows (head_dim 64 or 128), so that no division stands between a tile's sums and its stores.
struct PtRope { f4 c, s; };
__device__ __forceinline__ int pt_head_shift(const TileArgs& a) { return a.head_dim == 128 ? 3 : 2; }     // 16-row blocks per head
__device__ __forceinline__ PtRope pt_rope(const TileArgs& a, int u, int half, int pos) {
  const int j0 = (u & ((1 << pt_head_shift(a)) - 1)) * 8 + 4 * half;
  const float* cs = reinterpret_cast<const float*>(a.rope + (size_t)pos * (a.head_dim >> 1) + j0);
  const f4 c01 = *as_global(reinterpret_cast<const f4*>(cs)), c23 = *as_global(reinterpret_cast<const f4*>(cs + 4));
  return {f4{c01[0], c01[2], c23[0], c23[2]}, f4{c01[1], c01[3], c23[1], c23[3]}};
}

// Finishes rows 4 half .. + 3 (lo) and 8 + 4 half .. + 3 (hi) of 16-row block u for one token.  Accumulator
// layout of the 32x32 product with the weights as its first operand: a lane holds token (lane % 32) and weight
// rows 8 (e / 4) + 4 (lane / 32) + e % 4.  A 32-row block is two 16-row blocks of the copy, whose rows i and
// i + 8 belong together (RoPE partners, gate and up): both are in this lane.
template <int MODE>
__device__ __forceinline__ void pt_finish(const TileArgs& a, int u, int tok, int half, int pos, int split, f4 lo, f4 hi,
                                          const PtRope& cs) {
  if (MODE == SK_GATEUP) {
    h4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = (half_t)pt_swiglu(lo[i], hi[i]);
    *reinterpret_cast<h4*>(a.Hout + act_offset(tok, u * 8 + 4 * half, a.N, a.tb)) = o;
  } else if (MODE == SK_RES) {
    float* c = a.C + split * a.slice_floats + (size_t)tok * a.N + u * 16 + 4 * half;
    *as_global(reinterpret_cast<f4*>(c)) = lo;
    *as_global(reinterpret_cast<f4*>(c + 8)) = hi;
  } else {
    const int hh = a.head_dim >> 1, per = a.N / 16, z = (u >= per) + (u >= 2 * per), v = u - z * per;
    const int head = v >> pt_head_shift(a), b = v - (head << pt_head_shift(a));
    h4 o0, o1;
    if (z == 2) {
#pragma unroll
      for (int i = 0; i < 4; ++i) { o0[i] = (half_t)lo[i]; o1[i] = (half_t)hi[i]; }
      half_t* vr = a.vc + ((size_t)head * a.max_seq + pos) * a.head_dim + b * 16 + 4 * half;
      *as_global(reinterpret_cast<h4*>(vr)) = o0;
      *as_global(reinterpret_cast<h4*>(vr + 8)) = o1;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        o0[i] = (half_t)(lo[i] * cs.c[i] - hi[i] * cs.s[i]);
        o1[i] = (half_t)(hi[i] * cs.c[i] + lo[i] * cs.s[i]);
      }
      half_t* dst = (z == 0 ? a.Q + (size_t)tok * a.N + head * a.head_dim
                            : a.kc + ((size_t)head * a.max_seq + pos) * a.head_dim) + b * 8 + 4 * half;
      *as_global(reinterpret_cast<h4*>(dst)) = o0;
      *as_global(reinterpret_cast<h4*>(dst + hh)) = o1;
    }
  }
}

// Piece idx of a refill goes out in this one of its WS slots
__host__ __device__ constexpr int pt_slot(int idx, int WS, int PP) { return idx * WS / PP; }

// How many of a wave's loads may still be in flight (they return in order) at the barriers that hand a ring stage over:
// the kernel's own order of issue, replayed.  Prologue: pieces of stage 0, its WS * MT activation loads, pieces of stages
// 1 .. NS - 2 and slot 0 of stage NS - 1.  K step ws of stage it: its products, behind them the pieces of one
// refill slot and, behind a row block's last product, that block's activation load; the hand-over of stage it + 1 in front
// of the products of the last step.  The first NS - 2 stages handed over came without activation loads between their
// pieces, so fewer loads are younger there than later on; one count serves all (the waits for the activations
// themselves, one stage old at that point, admit no more than that anyway).
struct PtWaits { int first, handover; };
__host__ __device__ constexpr PtWaits pt_waits(int NS, int PP, int WS, int MT, int NB) {
  int issued = 0, last[16] = {};              // loads so far; number of the last piece of every stage
  PtWaits w{63, 63};                          // vmcnt has 6 bits
  for (int s = 0; s < NS - 1; ++s) {
    last[s] = issued += PP;
    if (s == 0) issued += WS * MT;
  }
  for (int idx = 0; idx < PP; ++idx)
    if (pt_slot(idx, WS, PP) == 0) last[NS - 1] = ++issued;
  if (issued - last[0] < w.first) w.first = issued - last[0];
  for (int it = 0; it < 2 * NS; ++it)
    for (int ws = 0; ws < WS; ++ws) {
      if (ws == WS - 1 && issued - last[it + 1] < w.handover) w.handover = issued - last[it + 1];
      const int stage = ws == WS - 1 ? it + NS : it + NS - 1, sl = (ws + 1) % WS, first = (sl * PP + WS - 1) / WS;
      for (int t = 0; t < MT * NB; ++t) {
        if (first + t < PP && pt_slot(first + t, WS, PP) == sl) last[stage] = ++issued;
        if (t % NB == NB - 1) ++issued;
      }
    }
  return w;
}

// k16 steps by which a wave requests its activations ahead, in tiles that are fed by other waves: a stage's, where that is
// what the measured tiles wanted (gate/up at 250 rows: 8 steps 49.7 us, 4 52.6; Q/K/V at 100: 16 steps 27.2, 4 29.2), but
// 4 for the residual projections (down at 250 rows: 31.1, 8 32.3) and where three row blocks leave no registers for more
__host__ __device__ constexpr int pt_look(int mode, int wk, int mt, int s32) {
  const int ws = s32 * 2 / wk;
  return mode == SK_RES || (wk == 1 && mt >= 3) ? (ws < 4 ? ws : 4) : ws;
}
// Q/K/V and gate/up in tiles of six accumulator blocks per wave with K split between the waves have registers for two stages
// of activations: those of two steps are requested together, a stage ahead and more.  us, step by step -> in pairs: gate/up
// at 100 rows 42.2 (as 128 x 96 without the split, its best step by step) -> 36.4, Q/K/V at 180 38.2 (8 K steps a stage) -> 37.0,
// at 250 40.7 -> 38.4.  Requested in fours: 37.5, 38.6 and 39.1; whole stages at once 39.9 and 40.5 (100 and 250 rows); two stages ahead
// step by step 40.7 (250).  In the other tiles that have the registers nothing is gained (O and down at 50 .. 250 rows, Q/K/V at
// 50: within 1 %) or it loses (Q/K/V at 100 rows 28.1 -> 29.9, gate/up at 50 31.8 -> 32.2); pairs without the second set of
// registers, which are requested later, lose everywhere.
__host__ __device__ constexpr bool pt_pairs(int mode, int wk, int mt, int nb) { return mode != SK_RES && wk == 2 && mt * nb == 6; }
template <int H> struct PtHalf { static constexpr int value = H; };

// Tile of 32 WM MT rows x 32 NB columns, four waves that multiply: WM along the rows (MT row blocks of 32 each), WK = 2
// splitting every K step in half between two waves per row group (half the LDS reads; the two halves of the
// accumulators are exchanged through LDS at the end).  Weights: a ring of NS stages of S32 32-wide K steps in LDS,
// filled by direct loads, 1 KB of consecutive bytes each: by four waves of their own, a freed stage at a time, or
// dealt one behind a matrix instruction over the steps that follow a stage's release (pt_fed).  Activations: steps of MT
// fragments in registers, each re-requested for a later step (pt_look; the next stage's) as soon as its last product is
// issued.  WNT: weights used by a single row tile are loaded non-temporal.
template <int MODE, int WM, int WK, int MT, int NB, int S32, int NS, bool WNT>
__global__ __launch_bounds__(pt_threads(MT, NB), 1) void pf_tile_kernel(TileArgs a) {
  static_assert(WM * WK == PT_WAVES, "four waves");
  constexpr bool FED = pt_fed(MT, NB);
  constexpr int BM = 32 * WM * MT;                 // rows of the tile
  constexpr int WS = S32 * 2 / WK;                 // k16 steps of a wave per stage
  constexpr int PIECES = 2 * NB * S32;             // 1 KB pieces per stage
  constexpr int PP = PIECES / 4;                   // ... per wave
  static_assert(PIECES % 4 == 0, "pieces divide over the waves");
  constexpr int STAGE = PIECES * 512;              // halves per stage
  extern __shared__ __attribute__((aligned(16))) half_t pt_lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w4 = wave & 3, wm = w4 % WM, wk = w4 / WM;
  const int r = lane & 31, half = lane >> 5;

  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int run = (slot / a.mtiles) * 8 + xcd;
  const int m0 = (slot % a.mtiles) * BM;
  const int n = a.st->n_prompt;
  if (run >= a.ctiles * a.ks || m0 >= n) return;
  const int ct = run / a.ks, split = run - ct * a.ks;
  const int K = a.K, ksteps = (K + 31) >> 5;
  const int units = skinny_units(MODE, a.N), upad = min(pt_units(MODE, a.N), (ct + 1) * a.upt), u0 = ct * a.upt;
  const int stages = (ksteps + S32 - 1) / S32;
  const int q = (stages + a.ks - 1) / a.ks;
  const int sl0 = split * q, cnt = min(q, stages - sl0);

  // Piece idx of this wave in a stage: 16-row block blk and K step s of piece p = idx * 4 + w4, k-step major
  // in LDS.  Everything that does not change from stage to stage sits in registers: the byte offset of the
  // lane's 16 bytes from the stage's start in the weight copy.
  int pvoff[PP], pks[PP];
#pragma unroll
  for (int idx = 0; idx < PP; ++idx) {
    const int p = idx * 4 + w4, s = p / (2 * NB), blk = p - s * (2 * NB);
    pks[idx] = s;
    pvoff[idx] = (blk * ksteps + s) * 1024 + lane * 16;
  }
  // Operands are fetched through buffer descriptors: what lies outside (blocks past the matrix, K steps past
  // its end, stages past this piece of the K loop) reads as zero without a branch and without traffic.
  const int blocks = max(min(units - u0, a.upt), 0);
  const half_t* wbase = a.Wf + (size_t)u0 * ksteps * 512;
  const unsigned wbytes = (unsigned)blocks * ksteps * 1024u;
  const unsigned astep = (unsigned)a.tb * 1024u, abytes = (unsigned)ksteps * astep;
  auto stage_k = [&](int it) {              // first K step of stage `it`; ksteps (nothing left) past the end
    return it < cnt ? (sl0 + it) * S32 : ksteps;
  };
  auto w_rsrc = [&](int k32) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(wbase + (size_t)k32 * 512), 0,
                                             wbytes > 0 && k32 < ksteps ? wbytes - (unsigned)k32 * 1024u : 0u, 0x00027000);
  };
  auto a_rsrc = [&](int k32) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(a.A + (size_t)k32 * (astep / 2)), 0,
                                             k32 < ksteps ? abytes - (unsigned)k32 * astep : 0u, 0x00027000);
  };
  auto issue_piece = [&](__amdgpu_buffer_rsrc_t w, int left, int stage, int idx) {
    const int voff = pvoff[idx] | (pks[idx] < left ? 0 : 0x40000000);       // a K step past the end: out of range
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        w, (__attribute__((address_space(3))) void*)(pt_lds + stage * STAGE + (idx * 4 + w4) * 512), 16, voff, 0, 0,
        WNT ? 2 : 0);
  };
  if constexpr (FED) {
    // The waves that load: a stage is handed over when its pieces have landed (each wave's own come back in order) and refilled
    // when all have left it.  Behind the K loop they leave, once nothing of theirs is on its way into the ring any more.
    if (__builtin_expect(wave >= PT_WAVES, 1)) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int k32 = stage_k(s);
        const __amdgpu_buffer_rsrc_t w = w_rsrc(k32);
#pragma unroll
        for (int idx = 0; idx < PP; ++idx) issue_piece(w, ksteps - k32, s, idx);
        __builtin_amdgcn_sched_barrier(0);
      }
      static_assert(PP * (NS - 1) < 64, "vmcnt has 6 bits");
      wait_vm_at_most<PP * (NS - 1)>();
      __builtin_amdgcn_s_barrier();
      int stage = 0;
      for (int it = 0; it < cnt; ++it) {
        wait_vm_at_most<PP * (NS - 2)>();          // stage it + 1; the younger ones are on their way
        __builtin_amdgcn_s_barrier();
        const int k32 = stage_k(it + NS);
        const __amdgpu_buffer_rsrc_t w = w_rsrc(k32);
#pragma unroll
        for (int idx = 0; idx < PP; ++idx) issue_piece(w, ksteps - k32, stage, idx);
        __builtin_amdgcn_sched_barrier(0);
        stage = stage + 1 == NS ? 0 : stage + 1;
      }
      wait_vm_at_most<0>();
      if (WK == 2) __builtin_amdgcn_s_barrier();   // the exchange takes the ring's place
      return;
    }
  }
  // activation fragment of the wave's k16 step ws, row block mt
  int avoff[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int tok = m0 + (wm * MT + mt) * 32 + r;
    avoff[mt] = (tok >> 4) * 1024 + (half * 16 + (tok & 15)) * 16 + (WK == 2 ? wk * 512 : 0) +
                ((tok & ~15) < n ? 0 : 0x40000000);         // 16-row blocks past the prompt: out of range, no traffic
  }
  auto load_a = [&](__amdgpu_buffer_rsrc_t ar, int ws, int mt) -> h8 {
    const int s = WK == 1 ? ws >> 1 : ws, ks = WK == 1 ? ws & 1 : 0;
    return __builtin_bit_cast(h8, __builtin_amdgcn_raw_buffer_load_b128(ar, avoff[mt] + ks * 512 + s * (int)astep, 0, 0));
  };

  f16v acc[MT][NB];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  constexpr bool PAIRS = FED && pt_pairs(MODE, WK, MT, NB);
  constexpr int LOOK = FED && !PAIRS ? pt_look(MODE, WK, MT, S32) : WS;
  static_assert(WS % LOOK == 0, "a step's registers are the same in every stage");
  static_assert(WS % 2 == 0, "the fragment double buffer keeps its parity across stages");
  h8 fa[PAIRS ? 2 * WS : LOOK][MT], fb[2][NB];
  auto load_b = [&](int stage, int ws, h8 (&f)[NB]) {
    const int s = WK == 1 ? ws >> 1 : ws, ks = WK == 1 ? ws & 1 : wk;
    const half_t* base = pt_lds + stage * STAGE + (s * 2 * NB + (r >> 4)) * 512 + ((ks * 2 + half) * 16 + (r & 15)) * 8;
#pragma unroll
    for (int j = 0; j < NB; ++j) f[j] = *reinterpret_cast<const h8*>(base + j * 1024);
  };
  if constexpr (FED) {
    __amdgpu_buffer_rsrc_t ar = a_rsrc(stage_k(0));
#pragma unroll
    for (int ws = 0; ws < LOOK; ++ws)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) fa[ws][mt] = load_a(ar, ws, mt);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    load_b(0, 0, fb[0]);
    __builtin_amdgcn_sched_barrier(0);
    int stage = 0;
    // stage it, its activations in the registers from CUR on (PAIRS: the next stage's go to the other half)
    auto steps = [&](int it, auto half_of) {
      constexpr int CUR = decltype(half_of)::value * WS;
      const __amdgpu_buffer_rsrc_t ar1 = a_rsrc(stage_k(it + 1));
      const int nstage = stage + 1 == NS ? 0 : stage + 1;
#pragma unroll
      for (int ws = 0; ws < WS; ++ws) {
        wait_lgkm_at_most<0>();
        __builtin_amdgcn_sched_barrier(0);
        if (ws + 1 < WS) {
          load_b(stage, ws + 1, fb[(ws + 1) & 1]);
        } else {                       // this wave has left the stage, and the next one is complete
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
          load_b(nstage, 0, fb[0]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < MT * NB; ++t) {
          const int mt = t / NB, nb = t % NB;
          acc[mt][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[ws & 1][nb], fa[CUR + ws % LOOK][mt], acc[mt][nb], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          if (!PAIRS && nb == NB - 1) {
            fa[ws % LOOK][mt] = ws + LOOK < WS ? load_a(ar, ws + LOOK, mt) : load_a(ar1, ws + LOOK - WS, mt);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        if (PAIRS && (ws & 1) == 0) {
#pragma unroll
          for (int w2 = ws; w2 < ws + 2; ++w2)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) fa[WS - CUR + w2][mt] = load_a(ar1, w2, mt);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      stage = nstage;
      ar = ar1;
    };
    for (int it = 0; it < cnt; ++it) {
      steps(it, PtHalf<0>());
      if (PAIRS && ++it < cnt) steps(it, PtHalf<PAIRS>());
    }
  } else {
    auto slot_of = [](int idx) { return pt_slot(idx, WS, PP); };
    constexpr int N_SLOT0 = (PP + WS - 1) / WS;

#pragma unroll
    for (int s = 0; s < NS - 1; ++s) {
      const int k32 = stage_k(s);
      const __amdgpu_buffer_rsrc_t w = w_rsrc(k32);
#pragma unroll
      for (int idx = 0; idx < PP; ++idx) issue_piece(w, ksteps - k32, s, idx);
      __builtin_amdgcn_sched_barrier(0);      // the waits below count loads: they hold for this order of issue only
      if (s == 0) {
        const __amdgpu_buffer_rsrc_t ar = a_rsrc(k32);
#pragma unroll
        for (int ws = 0; ws < WS; ++ws)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) fa[ws][mt] = load_a(ar, ws, mt);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // the refill under way: descriptor and K steps left of the stage that is being fetched
    int rk = stage_k(NS - 1);
    __amdgpu_buffer_rsrc_t rw = w_rsrc(rk);
#pragma unroll
    for (int idx = 0; idx < PP; ++idx)
      if (slot_of(idx) == 0) issue_piece(rw, ksteps - rk, NS - 1, idx);

    constexpr PtWaits WAIT = pt_waits(NS, PP, WS, MT, NB);
    __builtin_amdgcn_sched_barrier(0);
    wait_vm_at_most<WAIT.first>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    load_b(0, 0, fb[0]);
    __builtin_amdgcn_sched_barrier(0);
    int stage = 0;
    for (int it = 0; it < cnt; ++it) {
      const __amdgpu_buffer_rsrc_t ar = a_rsrc(stage_k(it + 1));
      const int nstage = stage + 1 == NS ? 0 : stage + 1;
      const int pstage = stage == 0 ? NS - 1 : stage - 1;
#pragma unroll
      for (int ws = 0; ws < WS; ++ws) {
        wait_lgkm_at_most<0>();
        __builtin_amdgcn_sched_barrier(0);
        if (ws + 1 < WS) {
          load_b(stage, ws + 1, fb[(ws + 1) & 1]);
        } else {
          wait_vm_at_most<WAIT.handover>();
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
          load_b(nstage, 0, fb[0]);
          rk = stage_k(it + NS);
          rw = w_rsrc(rk);
        }
        __builtin_amdgcn_sched_barrier(0);
        // the refill under way: slot 0 right behind the hand-over of stage it, slot s in step s - 1 of stage it + 1
        const int rstage = ws == WS - 1 ? stage : pstage;
        const int sl = (ws + 1) % WS;
        const int first = (sl * PP + WS - 1) / WS;
#pragma unroll
        for (int t = 0; t < MT * NB; ++t) {
          const int mt = t / NB, nb = t % NB;
          acc[mt][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[ws & 1][nb], fa[ws][mt], acc[mt][nb], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          if (first + t < PP && slot_of(first + t) == sl) {
            issue_piece(rw, ksteps - rk, rstage, first + t);
            __builtin_amdgcn_sched_barrier(0);
          }
          if (nb == NB - 1) {
            fa[ws][mt] = load_a(ar, ws, mt);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        static_assert(N_SLOT0 <= MT * NB, "one piece behind each matrix instruction at most");
      }
      stage = nstage;
    }
    wait_vm_at_most<0>();     // the look-ahead loads must not outlive the workgroup's LDS
    wait_lgkm_at_most<0>();
  }

  if constexpr (WK == 2) {
    // the two K halves of a row block: every wave hands over half of its accumulators and finishes the other half
    float* xch = reinterpret_cast<float*>(pt_lds);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < MT * NB; ++t) {
      if ((t & 1) == wk) continue;
      float* dst = xch + ((size_t)(wm * MT * NB + t) * 16) * 64 + lane * 4;
      const f16v& v = acc[t / NB][t % NB];
#pragma unroll
      for (int e = 0; e < 4; ++e) *reinterpret_cast<f4*>(dst + e * 256) = f4{v[4 * e], v[4 * e + 1], v[4 * e + 2], v[4 * e + 3]};
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < MT * NB; ++t) {
      if ((t & 1) != wk) continue;
      const float* src = xch + ((size_t)(wm * MT * NB + t) * 16) * 64 + lane * 4;
      f16v& v = acc[t / NB][t % NB];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const f4 o = *reinterpret_cast<const f4*>(src + e * 256);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[4 * e + i] += o[i];
      }
    }
  }

  // The RoPE factors of all blocks of a row block are requested together, not each in front of its own stores (Q/K/V at 500
  // rows 52.2 -> 51.4 us, at 250 39.1 -> 38.6).  What is left behind the K loop is mostly the stores' way to memory: 2 to 3 us
  // of Q/K/V, and 3.5 us per 17 MB of slices.
  const int p0 = a.st->pos;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int tok = m0 + (wm * MT + mt) * 32 + r;
    PtRope cs[MODE == SK_QKV ? NB : 1][2];
    if constexpr (MODE == SK_QKV) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int hb = 0; hb < 2; ++hb)
          if (WK == 1 || ((mt * NB + nb) & 1) == wk) cs[nb][hb] = pt_rope(a, u0 + nb * 2 + hb, half, p0 + min(tok, n - 1));
      __builtin_amdgcn_sched_barrier(0);
    }
    if (tok >= n) continue;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      if (WK == 2 && ((mt * NB + nb) & 1) != wk) continue;
#pragma unroll
      for (int hb = 0; hb < 2; ++hb) {
        const int u = u0 + nb * 2 + hb;
        if (u >= upad) continue;
        f4 lo, hi;
#pragma unroll
        for (int i = 0; i < 4; ++i) { lo[i] = acc[mt][nb][hb * 8 + i]; hi[i] = acc[mt][nb][hb * 8 + 4 + i]; }
        pt_finish<MODE>(a, u, tok, half, p0 + tok, split, lo, hi, cs[MODE == SK_QKV ? nb : 0][hb]);
      }
    }
  }
}
