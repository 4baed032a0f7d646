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
// its vector L1 once per tile, (rows + columns) * K * 2, and those bytes cost 40 TB/s chip-wide ON TOP of the
// time the weights take from HBM (gate/up, 256 rows: weights alone 47 us, with the activations 58): the two do
// not overlap, so tiles are as square as a single round allows.  At 512 rows and more the matrix instructions
// are the larger part (gate/up at 512 rows: 98 k of 114 k cycles in the K loop) and the chip runs them at 1.6-1.8
// GHz.  LDS holds only the weights (direct loads in, 4 or 2 fragment reads per byte out); the
// activations go straight to registers, one stage ahead.  With both operands in LDS (128 x 256 tiles, eight
// waves) the LDS port was busy 1.4 times as long as the matrix cores: gate/up at 512 rows 110 us + 16 us SwiGLU
// kernel against 88 us here, Q/K/V 67 + 12 against 59.
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
  int upt;                // stream kernel: 16-row weight blocks of a column tile, at most 2 NB (the rest reads as zero)
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

#define PT_THREADS 256
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

// Finishes rows 4 half .. + 3 (lo) and 8 + 4 half .. + 3 (hi) of 16-row block u for one token.  Accumulator
// layout of the 32x32 product with the weights as its first operand: a lane holds token (lane % 32) and weight
// rows 8 (e / 4) + 4 (lane / 32) + e % 4.  A 32-row block is two 16-row blocks of the copy, whose rows i and
// i + 8 belong together (RoPE partners, gate and up): both are in this lane.
template <int MODE>
__device__ __forceinline__ void pt_finish(const TileArgs& a, int u, int tok, int half, int pos, int split, f4 lo, f4 hi) {
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
    const int hh = a.head_dim >> 1, per = a.N / 16, z = u / per, v = u - z * per;
    h4 o0, o1;
    if (z == 2) {
      const int c0 = v * 16, head = c0 / a.head_dim, e = c0 - head * a.head_dim + 4 * half;
#pragma unroll
      for (int i = 0; i < 4; ++i) { o0[i] = (half_t)lo[i]; o1[i] = (half_t)hi[i]; }
      half_t* vr = a.vc + ((size_t)head * a.max_seq + pos) * a.head_dim + e;
      *reinterpret_cast<h4*>(vr) = o0;
      *reinterpret_cast<h4*>(vr + 8) = o1;
    } else {
      const int bph = hh / 8, head = v / bph, j0 = (v - head * bph) * 8 + 4 * half;
      const float* cs = reinterpret_cast<const float*>(a.rope + (size_t)pos * hh + j0);
      const f4 c01 = *as_global(reinterpret_cast<const f4*>(cs)), c23 = *as_global(reinterpret_cast<const f4*>(cs + 4));
      const f4 c = {c01[0], c01[2], c23[0], c23[2]}, sn = {c01[1], c01[3], c23[1], c23[3]};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        o0[i] = (half_t)(lo[i] * c[i] - hi[i] * sn[i]);
        o1[i] = (half_t)(hi[i] * c[i] + lo[i] * sn[i]);
      }
      half_t* dst = z == 0 ? a.Q + (size_t)tok * a.N + head * a.head_dim
                           : a.kc + ((size_t)head * a.max_seq + pos) * a.head_dim;
      *reinterpret_cast<h4*>(dst + j0) = o0;
      *reinterpret_cast<h4*>(dst + j0 + hh) = o1;
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

// Tile of 32 WM MT rows x 32 NB columns, four waves: WM along the rows (MT row blocks of 32 each), WK = 2
// splitting every K step in half between two waves per row group (half the LDS reads; the two halves of the
// accumulators are exchanged through LDS at the end).  Weights: a ring of NS stages of S32 32-wide K steps in LDS,
// filled by direct loads, 1 KB of consecutive bytes each, dealt one behind a matrix instruction over the steps
// that follow a stage's release.  Activations: WS steps of MT fragments in registers, each re-requested for the
// next stage as soon as its last product is issued.  WNT: weights used by a single row tile are loaded
// non-temporal.
template <int MODE, int WM, int WK, int MT, int NB, int S32, int NS, bool WNT>
__global__ __launch_bounds__(PT_THREADS, 1) void pf_tile_kernel(TileArgs a) {
  static_assert(WM * WK == 4, "four waves");
  constexpr int BM = 32 * WM * MT;                 // rows of the tile
  constexpr int WS = S32 * 2 / WK;                 // k16 steps of a wave per stage
  constexpr int PIECES = 2 * NB * S32;             // 1 KB pieces per stage
  constexpr int PP = PIECES / 4;                   // ... per wave
  static_assert(PIECES % 4 == 0, "pieces divide over the waves");
  constexpr int STAGE = PIECES * 512;              // halves per stage
  extern __shared__ __attribute__((aligned(16))) half_t pt_lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WM, wk = wave / WM;
  const int r = lane & 31, half = lane >> 5;

  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int run = (slot / a.mtiles) * 8 + xcd;
  const int m0 = (slot % a.mtiles) * BM;
  const int n = a.st->n_prompt;
  if (run >= a.ctiles * a.ks || m0 >= n) return;
  const int ct = run / a.ks, split = run - ct * a.ks;
  const int K = a.K, ksteps = (K + 31) >> 5;
  const int units = skinny_units(MODE, a.N), upad = pt_units(MODE, a.N), u0 = ct * NB * 2;
  const int stages = (ksteps + S32 - 1) / S32;
  const int q = (stages + a.ks - 1) / a.ks;
  const int sl0 = split * q, cnt = min(q, stages - sl0);

  // Piece idx of this wave in a stage: 16-row block blk and K step s of piece p = idx * 4 + wave, k-step major
  // in LDS.  Everything that does not change from stage to stage sits in registers: the byte offset of the
  // lane's 16 bytes from the stage's start in the weight copy.
  int pvoff[PP], pks[PP];
#pragma unroll
  for (int idx = 0; idx < PP; ++idx) {
    const int p = idx * 4 + wave, s = p / (2 * NB), blk = p - s * (2 * NB);
    pks[idx] = s;
    pvoff[idx] = (blk * ksteps + s) * 1024 + lane * 16;
  }
  // Operands are fetched through buffer descriptors: what lies outside (blocks past the matrix, K steps past
  // its end, stages past this piece of the K loop) reads as zero without a branch and without traffic.
  const int blocks = max(min(units - u0, 2 * NB), 0);
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
        w, (__attribute__((address_space(3))) void*)(pt_lds + stage * STAGE + (idx * 4 + wave) * 512), 16, voff, 0, 0,
        WNT ? 2 : 0);
  };
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

  auto slot_of = [](int idx) { return pt_slot(idx, WS, PP); };
  constexpr int N_SLOT0 = (PP + WS - 1) / WS;

  h8 fa[WS][MT], fb[2][NB];
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

  auto load_b = [&](int stage, int ws, h8 (&f)[NB]) {
    const int s = WK == 1 ? ws >> 1 : ws, ks = WK == 1 ? ws & 1 : wk;
    const half_t* base = pt_lds + stage * STAGE + (s * 2 * NB + (r >> 4)) * 512 + ((ks * 2 + half) * 16 + (r & 15)) * 8;
#pragma unroll
    for (int j = 0; j < NB; ++j) f[j] = *reinterpret_cast<const h8*>(base + j * 1024);
  };
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
      static_assert(WS % 2 == 0, "the fragment double buffer keeps its parity across stages");
      static_assert(N_SLOT0 <= MT * NB, "one piece behind each matrix instruction at most");
    }
    stage = nstage;
  }
  wait_vm_at_most<0>();     // the look-ahead loads must not outlive the workgroup's LDS
  wait_lgkm_at_most<0>();

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

  const int p0 = a.st->pos;
#pragma unroll
  for (int t = 0; t < MT * NB; ++t) {
    if (WK == 2 && (t & 1) != wk) continue;
    const int mt = t / NB, nb = t % NB;
    const int tok = m0 + (wm * MT + mt) * 32 + r;
    if (tok >= n) continue;
#pragma unroll
    for (int hb = 0; hb < 2; ++hb) {
      const int u = u0 + nb * 2 + hb;
      if (u >= upad) continue;
      f4 lo, hi;
#pragma unroll
      for (int i = 0; i < 4; ++i) { lo[i] = acc[mt][nb][hb * 8 + i]; hi[i] = acc[mt][nb][hb * 8 + 4 + i]; }
      pt_finish<MODE>(a, u, tok, half, p0 + tok, split, lo, hi);
    }
  }
}

// The same product for few rows (or narrow tiles), where the weight stream is nearly all there is: the four
// waves split K, so nothing is shared and nothing is staged; every operand goes straight to registers, D steps
// of (MT + NB) KB ahead per wave, with no barrier before the partial sums meet in LDS at the end.  At 64 rows gate/up
// takes 34.3 us this way and 36.8 us with the weights in LDS, Q/K/V 26.0 and 27.5 (both in 192 workgroups); deeper
// look-ahead (D = 12) is slower (37.3 us).  A CU's own fetches set the time, so `upt` lets the host make the tiles narrower
// than 32 NB columns where that occupies CUs that would have none: Q/K/V of 50 rows 28.4 us in 192 tiles of 64
// columns, 23.4 in 256 of 48; what is left out of a tile reads as zero, without traffic.
#define PS_LDS_BYTES(MT, NB) (4 * ((MT) < 2 ? 1 : 2) * (NB) * 4096)
template <int MODE, int MT, int NB, int D, bool WNT>
__global__ __launch_bounds__(PT_THREADS, 1) void pf_stream_kernel(TileArgs a) {
  static_assert(D * (MT + NB) < 64, "vmcnt is a 6-bit counter");
  extern __shared__ __attribute__((aligned(16))) float ps_lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 31, half = lane >> 5;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int run = (slot / a.mtiles) * 8 + xcd, m0 = (slot % a.mtiles) * (32 * MT);
  const int n = a.st->n_prompt, p0 = a.st->pos;
  if (run >= a.ctiles * a.ks || m0 >= n) return;
  const int ct = run / a.ks, split = run - ct * a.ks;
  const int ksteps = (a.K + 31) >> 5, units = skinny_units(MODE, a.N), upad = min(pt_units(MODE, a.N), (ct + 1) * a.upt), u0 = ct * a.upt;
  // K range of this wave in 16-wide steps
  const int parts = 4 * a.ks, per = (ksteps + parts - 1) / parts * 2;
  const int k_begin = (split * 4 + wave) * per, k_end = min(k_begin + per, 2 * ksteps);
  const unsigned wbytes = (unsigned)max(min(units - u0, a.upt), 0) * ksteps * 1024u;
  const unsigned astep = (unsigned)a.tb * 1024u;
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<half_t*>(a.Wf + (size_t)u0 * ksteps * 512), 0, wbytes, 0x00027000);
  const __amdgpu_buffer_rsrc_t ar = __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(a.A), 0, ksteps * astep, 0x00027000);
  int wv[NB], av[MT];
#pragma unroll
  for (int j = 0; j < NB; ++j) wv[j] = (j * 2 + (r >> 4)) * ksteps * 1024 + (half * 16 + (r & 15)) * 16;
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int tok = m0 + i * 32 + r;
    av[i] = (tok >> 4) * 1024 + (half * 16 + (tok & 15)) * 16 + ((tok & ~15) < n ? 0 : 0x40000000);
  }
  auto ld = [](__amdgpu_buffer_rsrc_t rs, int off) { return __builtin_bit_cast(h8, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0)); };
  auto ldw = [](__amdgpu_buffer_rsrc_t rs, int off) { return __builtin_bit_cast(h8, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, WNT ? 2 : 0)); };
  h8 fa[D][MT], fw[D][NB];
  f16v acc[MT][NB];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  auto issue = [&](int k16, h8 (&A)[MT], h8 (&W)[NB]) {
    const bool in = k16 < k_end;
    const int wo = in ? k16 * 512 : 0x40000000;                                     // past the range: reads zero
    const int ao = in ? (k16 >> 1) * (int)astep + (k16 & 1) * 512 : 0x20000000;
#pragma unroll
    for (int j = 0; j < NB; ++j) W[j] = ldw(wr, wv[j] + wo);
#pragma unroll
    for (int i = 0; i < MT; ++i) A[i] = ld(ar, av[i] + ao);
  };
#pragma unroll
  for (int d = 0; d < D; ++d) issue(k_begin + d, fa[d], fw[d]);
  __builtin_amdgcn_sched_barrier(0);
  for (int k = k_begin; k < k_end; k += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fw[d][j], fa[d][i], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      issue(k + d + D, fa[d], fw[d]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // the waves' partial sums meet in LDS, two row blocks at a time; a wave finishes every fourth 16-row block
  constexpr int MR = MT < 2 ? 1 : 2;                 // row blocks per round
#pragma unroll
  for (int i0 = 0; i0 < MT; i0 += MR) {
    if (m0 + i0 * 32 >= n) break;
    if (i0) __syncthreads();
#pragma unroll
    for (int i = 0; i < MR; ++i) {
      if (i0 + i >= MT) continue;
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const f16v& v = acc[i0 + i][j];
          *reinterpret_cast<f4*>(ps_lds + (((wave * MR + i) * NB + j) * 4 + e) * 256 + lane * 4) =
              f4{v[4 * e], v[4 * e + 1], v[4 * e + 2], v[4 * e + 3]};
        }
    }
    __syncthreads();
    for (int h = wave; h < MR * NB * 2; h += 4) {
      const int i = h / (NB * 2), ub = h - i * (NB * 2), u = u0 + ub, tok = m0 + (i0 + i) * 32 + r;
      if (u >= upad || tok >= n || i0 + i >= MT) continue;
      f4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float* src = ps_lds + (((w * MR + i) * NB + (ub >> 1)) * 4 + (ub & 1) * 2) * 256 + lane * 4;
        lo += *reinterpret_cast<const f4*>(src);
        hi += *reinterpret_cast<const f4*>(src + 256);
      }
      pt_finish<MODE>(a, u, tok, half, p0 + tok, split, lo, hi);
    }
  }
}
