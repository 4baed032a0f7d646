// Short-prompt prefill kernels for gfx950 (prompts of 10-500 tokens, the
// paper's TTFT regime, Sec. IV-E / Table I): the same layer as the decode path
// but for n rows at positions 0..n-1: the elementwise kernels around the
// projection GEMM (prefill_gemm.h) and the causal attention on the matrix cores.
//
// Every kernel is launched on a grid sized for a prompt-length bucket Mb and
// reads the true n from DevState, so one captured graph per bucket serves all
// prompts that fit it.  Rows >= n are zero operands for the projections beyond
// 32 rows, whatever the residual stream holds there, and never reach the KV cache
// or the logits.  A prompt longer than the largest bucket is fed in
// chunks: DevState.pos holds the number of positions already cached (p0), row r
// of the chunk sits at position p0 + r, and attention also covers the p0 keys
// of the earlier chunks.
#pragma once
#include "ll_device.h"

// State block and prompt ids from the pinned staging buffer (host memory: one round trip over the bus for all of
// it, so ids are fetched for every row of the bucket without waiting for n; the rows past n are not used).  zeros:
// optionally 256 bytes to clear.  One workgroup.
__global__ __launch_bounds__(LL_WG) void pf_stage_kernel(const int* __restrict__ stage, int* __restrict__ state,
                                                         int* __restrict__ tokens, int rows, int* __restrict__ zeros) {
  constexpr int WORDS = sizeof(DevState) / 4;
  const int tid = threadIdx.x;
  if (tid < WORDS) state[tid] = stage[tid];
  for (int i = tid; i < rows; i += LL_WG) tokens[i] = stage[WORDS + i];
  if (zeros && tid < 64) zeros[tid] = 0;
}

// Sum of np split-K slices at p (slice stride in floats), four loads in flight at a time.
__device__ __forceinline__ f4 pf_slice_sum(const float* p, int np, size_t slice_floats) {
  f4 v = {0.f, 0.f, 0.f, 0.f};
  int s = 0;
  for (; s + 4 <= np; s += 4) {
    const f4 a = *reinterpret_cast<const f4*>(p + (size_t)s * slice_floats);
    const f4 b = *reinterpret_cast<const f4*>(p + (size_t)(s + 1) * slice_floats);
    const f4 c = *reinterpret_cast<const f4*>(p + (size_t)(s + 2) * slice_floats);
    const f4 e = *reinterpret_cast<const f4*>(p + (size_t)(s + 3) * slice_floats);
    v += (a + b) + (c + e);
  }
  for (; s < np; ++s) v += *reinterpret_cast<const f4*>(p + (size_t)s * slice_floats);
  return v;
}

// Row-wise RMSNorm of the fp32 residual stream into fp16 GEMM operands, one
// 1024-thread workgroup per row.  FIRST: the row is the embedding of token r, stored to X as well.  Otherwise the residual
// GEMM in front of it may have left its result as np split-K slices ([np][rows][d] at part): they are added to X
// here, X is stored back, and the norm is taken of the sum.  Rows past the prompt
// give zero operands.  frag_tb != 0 writes the operands in the short-prompt
// kernels' fragment-major layout.
// Everything it reads is requested up front and kept in registers, PF_NORM_CHUNKS pieces of a thread (d_model up to 12288; an
// instance has at most 8192).  At 50 rows it is one memory round trip and a barrier long (5.0 us a launch), at 500 the slices'
// way between XCDs (11.2, 4 TB/s); the first one takes 4.6 / 6.4 / 7.6 us at 50 / 250 / 500 rows where a gather kernel and a
// norm took 5.5 / 9.5 / 12.8.
#define PF_NORM_THREADS 1024
#define PF_NORM_CHUNKS 3
template <bool FIRST>
__global__ __launch_bounds__(PF_NORM_THREADS) void pf_rmsnorm_kernel(float* __restrict__ X, const half_t* __restrict__ emb,
                                                                     const int* __restrict__ tokens,
                                                                     const half_t* __restrict__ gain,
                                                                     half_t* __restrict__ Xn, int d, float eps,
                                                                     const DevState* __restrict__ st,
                                                                     const float* __restrict__ part, SliceMap map,
                                                                     int frag_tb) {
  __shared__ float red[PF_NORM_THREADS / 64];
  const int r = blockIdx.x, tid = threadIdx.x;
  const int n = st->n_prompt, token = FIRST ? tokens[r] : 0;      // (an id is staged for every row of the bucket)
  auto at = [&](int c) { return (c * PF_NORM_THREADS + tid) * 4; };
  if (r >= n) {
    const h4 zero = {0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < PF_NORM_CHUNKS; ++c)
      if (at(c) < d) *reinterpret_cast<h4*>(Xn + act_offset(r, at(c), d, frag_tb)) = zero;
    return;
  }
  float* xr = X + (size_t)r * d;
  const float* pr = part + (size_t)r * d;
  f4 v[PF_NORM_CHUNKS];
  h4 g[PF_NORM_CHUNKS];
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < PF_NORM_CHUNKS; ++c) {
    const int i = at(c);
    if (i >= d) continue;
    g[c] = *as_global(reinterpret_cast<const h4*>(gain + i));
    if constexpr (FIRST) {
      const h4 e = *as_global(reinterpret_cast<const h4*>(emb + (size_t)token * d + i));
      v[c] = f4{(float)e[0], (float)e[1], (float)e[2], (float)e[3]};
    } else {
      v[c] = *as_global(reinterpret_cast<const f4*>(xr + i));
      if (part) v[c] += pf_slice_sum(pr + i, map.quota == 1 ? map.nslabs : slice_count(map, i), map.slice_floats);
    }
    if (FIRST || part) *as_global(reinterpret_cast<f4*>(xr + i)) = v[c];
    ss += v[c][0] * v[c][0] + v[c][1] * v[c][1] + v[c][2] * v[c][2] + v[c][3] * v[c][3];
  }
  ss = wave_sum(ss);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();                       // (nobody waits for the rows' way back to memory here)
  asm volatile("" ::: "memory");
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < PF_NORM_THREADS / 64; ++w) tot += red[w];
  const float inv = 1.0f / sqrtf(tot / (float)d + eps);
#pragma unroll
  for (int c = 0; c < PF_NORM_CHUNKS; ++c) {
    const int i = at(c);
    if (i >= d) continue;
    h4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = (half_t)(v[c][j] * inv * (float)g[c][j]);
    *as_global(reinterpret_cast<h4*>(Xn + act_offset(r, i, d, frag_tb))) = o;
  }
}

// RoPE on the q and k thirds of the QKV projection (fp32, slices of [Mb][3d], summed here) at
// position p0 + r, then q -> fp16 Q[r], k/v -> the KV cache rows of position p0 + r.  Four rotation
// pairs per thread with 16-byte loads, every load of a thread issued before the first use
// (head_dim % 8 == 0).  grid = (Mb, ceil(n_heads * head_dim / 8 / LL_WG)), rows >= n idle.
__global__ __launch_bounds__(LL_WG) void pf_rope_kv_kernel(const float* __restrict__ QKV, SliceMap map,
                                                            const float2* __restrict__ rope,
                                                            const DevState* __restrict__ st,
                                                            half_t* __restrict__ Q,
                                                            half_t* __restrict__ kc,
                                                            half_t* __restrict__ vc, int d,
                                                            int head_dim, int max_seq) {
  const int r = blockIdx.x;
  if (r >= st->n_prompt) return;
  const int hh = head_dim >> 1, per_head = hh >> 2;
  const int item = blockIdx.y * LL_WG + threadIdx.x;
  const int head = item / per_head, j = (item - head * per_head) * 4;
  if (head * head_dim >= d) return;
  const int pos = st->pos + r;
  const int ia = head * head_dim + j, ib = ia + hh;
  const float* row = QKV + (size_t)r * 3 * d;
  const f4 c01 = *reinterpret_cast<const f4*>(rope + (size_t)pos * hh + j);       // (cos, sin) of pairs j, j + 1
  const f4 c23 = *reinterpret_cast<const f4*>(rope + (size_t)pos * hh + j + 2);
  auto val = [&](int i) { return pf_slice_sum(row + i, slice_count(map, i), map.slice_floats); };
  const f4 qa = val(ia), qb = val(ib), ka = val(d + ia), kb = val(d + ib), va = val(2 * d + ia), vb = val(2 * d + ib);
  const f4 cs = {c01[0], c01[2], c23[0], c23[2]}, sn = {c01[1], c01[3], c23[1], c23[3]};
  h4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (half_t)(qa[e] * cs[e] - qb[e] * sn[e]);
  *reinterpret_cast<h4*>(Q + (size_t)r * d + ia) = o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (half_t)(qb[e] * cs[e] + qa[e] * sn[e]);
  *reinterpret_cast<h4*>(Q + (size_t)r * d + ib) = o;
  half_t* kr = kc + ((size_t)head * max_seq + pos) * head_dim;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (half_t)(ka[e] * cs[e] - kb[e] * sn[e]);
  *reinterpret_cast<h4*>(kr + j) = o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (half_t)(kb[e] * cs[e] + ka[e] * sn[e]);
  *reinterpret_cast<h4*>(kr + j + hh) = o;
  half_t* vr = vc + ((size_t)head * max_seq + pos) * head_dim;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (half_t)va[e];
  *reinterpret_cast<h4*>(vr + j) = o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (half_t)vb[e];
  *reinterpret_cast<h4*>(vr + j + hh) = o;
}

// Causal attention of one head for a block of 64 queries, on the matrix cores.
// grid = (heads, Mb / 64), longest blocks first; 128 G threads: G groups of two waves, group g taking the key tiles
// (32 keys) g, g + G, ... of the block; each of a group's two waves owns 32 queries, with an online softmax.
//
// Both products are computed transposed so that the softmax needs no transpose:
//   S^T[key][q] = sum_d K[key][d] Q[q][d]      A = K tile (LDS), B = Q (registers)
//   O^T[d][q]  += sum_key V[key][d] P[q][key]  A = V^T tile (LDS), B = P^T (registers)
// In the 32x32 accumulator layout a lane holds ONE query column (lane % 32) and
// 16 of the 32 key rows (the other 16 sit in lane ^ 32), so the row max / sum is
// 15 register operations plus one cross-half shuffle, the rescale of O^T is a
// per-lane scalar, and the probabilities are already in B-operand position:
// k-slot j of lane half hf in k-step s holds key 16 s + 8 (j / 4) + 4 hf + j % 4.
//
// K and V tiles go global -> LDS directly, row-major, one tile ahead, and stay row-major: the V^T operand is read with
// the transposing LDS read (ds_read_b64_tr_b16: 16 lanes fetch four rows of 16 columns and each receives one
// column of the four rows, which is exactly a k-slot quad above).  Within a row of HD halves the 16-byte chunk c sits at
// c ^ swz(key), which keeps both kinds of reads off one another's banks.
//
// What bounds it: a trip of all four groups moves 64 KB into LDS and reads 128 KB from it (some 2000 cycles of the LDS
// port) around 700 cycles of vector work (softmax, rescale) and 16 matrix instructions per wave: 1.8 us.  So
// the scale is folded into the exponential's argument (one multiply-add per score), only tiles on the diagonal
// are masked, the rescale is skipped when no query's maximum moved, all operands of a tile are requested at
// once, and the groups' partial results are merged by all threads (by one group it cost as much as two tiles).
// Per layer at the 7B shape, tiles staged through registers and V transposed by 2-byte pair stores before / now:
// 50 tokens 5.9 / 5.4 us, 100: 7.7 / 6.4, 250: 13.0 / 9.3, 350: 16.0 / 10.8, 500: 20.7 / 14.5, the two chunks of
// 2000 tokens 41 and 82 / 26 and 58.  Groups (same order): one 5.8 / 8.9 / 14.5 / - / 27 us, two 5.4 / 7.1 / 10.6 /
// - / 19.5, four 5.9 / 6.4 / 9.3 / 10.8 / 14.5.
#define PF_ATTN_TILE_HALVES(HD) (2 * 32 * (HD))                       /* one K and one V tile */
#define PF_ATTN_MERGE_BYTES(HD, G) ((G) == 1 ? 0 : (G) * 128 * ((HD) / 2 + 2) * 4)
#define PF_ATTN_LDS_BYTES(HD, G) \
  ((G) * 2 * PF_ATTN_TILE_HALVES(HD) * 2 > PF_ATTN_MERGE_BYTES(HD, G) ? (G) * 2 * PF_ATTN_TILE_HALVES(HD) * 2 \
                                                                      : PF_ATTN_MERGE_BYTES(HD, G))

template <int HD, int G>
__global__ __launch_bounds__(128 * G) void pf_attn_kernel(const half_t* __restrict__ Q,
                                                          const half_t* __restrict__ kc,
                                                          const half_t* __restrict__ vc,
                                                          const DevState* __restrict__ st,
                                                          half_t* __restrict__ O, int d, int max_seq,
                                                          int frag_tb) {
  constexpr int QB = 64, TK = 32, KS = HD / 16, DT = HD / 32, CPR = HD / 8;
  constexpr int RPL = 64 / CPR;               // tile rows one 1 KB direct load covers
  constexpr int LOADS = TK / RPL;             // direct loads of a K (or V) tile: wave 0 of the group brings K, wave 1 V
  extern __shared__ __attribute__((aligned(16))) half_t pf_attn_lds[];
  const int h = blockIdx.x, q0 = (gridDim.y - 1 - blockIdx.y) * QB;
  const int n = st->n_prompt, p0 = st->pos;   // rows of this chunk, positions cached before it
  if (q0 >= n) return;
  const int tid = threadIdx.x & 127, lane = tid & 63, hf = lane >> 5, ql = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x >> 7);
  half_t* buf = pf_attn_lds + grp * 2 * PF_ATTN_TILE_HALVES(HD);      // two stages of [K tile | V tile]
  const int qi = q0 + wave * 32 + ql;
  const int wave_q = q0 + wave * 32;          // the wave's first query
  const float c2 = 1.44269504088896340736f / sqrtf((float)HD);        // scores enter exp2 scaled by log2(e) / sqrt(HD)

  // chunk swizzle of a key's row (even, so that pairs of chunks stay pairs)
  auto swz = [](int key) { return HD == 128 ? (key & 7) * 2 : ((key >> 1) & 3) * 2; };
  const half_t* src = (wave ? vc : kc) + (size_t)h * max_seq * HD;
  const int last_row = p0 + n - 1, last_key = p0 + min(q0 + QB, n) - 1;   // the block's last valid query attends it
  auto issue = [&](int k0, int stage) {
    half_t* dst = buf + stage * PF_ATTN_TILE_HALVES(HD) + wave * TK * HD;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      const int row = i * RPL + lane / CPR, c = (lane % CPR) ^ swz(row);
      __builtin_amdgcn_global_load_lds((const LL_GLOBAL void*)(src + (size_t)min(k0 + row, last_row) * HD + c * 8),
                                       (__attribute__((address_space(3))) void*)(dst + i * 512), 16, 0, 0);
    }
  };
  constexpr int STEP = G * TK;
  const int kg = grp * TK;
  if (kg <= last_key) issue(kg, 0);

  h8 qf[KS];
  {
    const half_t* qp = Q + (size_t)min(qi, n - 1) * d + h * HD + hf * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = load_h8(qp + ks * 16);
  }
  f16v acc[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
  float m = -INFINITY, l = 0.f;               // running maximum of the raw scores, running sum

  // LDS byte offsets of this lane's operand reads: K row ql (chunk 2 ks + hf), V^T quads (see above)
  const int koff = ql * HD * 2 + swz(ql) * 16 + hf * 16;
  const int vkey = 4 * hf + ((lane & 15) >> 2);
  const int voff = TK * HD * 2 + vkey * HD * 2 + ((((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) ^ swz(vkey)) * 16 + (lane & 1) * 8;
  typedef __fp16 v4f16 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) v4f16 lds_v4f16;
  // Operands of a tile: all of them are requested before the first product (and before the next tile's direct
  // loads: the compiler holds a transposing read back until every direct load in flight has landed).
  h4 fv[DT][2][2];
  h8 fk[KS];
  auto load_tile = [&](const half_t* b) {
    const char* base = reinterpret_cast<const char*>(b);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fk[ks] = *reinterpret_cast<const h8*>(base + (koff ^ (ks * 32)));
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        fv[t][i >> 1][i & 1] = __builtin_bit_cast(
            h4, __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_v4f16*)(base + ((voff ^ (t * 64)) + i * 8 * HD * 2))));
  };
  auto tile = [&](int k0) {
    f16v sc, sd;                              // two chains of products
#pragma unroll
    for (int e = 0; e < 16; ++e) sc[e] = sd[e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ks += 2) {
      sc = __builtin_amdgcn_mfma_f32_32x32x16_f16(fk[ks], qf[ks], sc, 0, 0, 0);
      sd = __builtin_amdgcn_mfma_f32_32x32x16_f16(fk[ks + 1], qf[ks + 1], sd, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) sc[e] += sd[e];
    if (k0 + TK - 1 > p0 + wave_q) {          // a tile on the wave's diagonal
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (k0 + 8 * (e >> 2) + 4 * hf + (e & 3) > p0 + qi) sc[e] = -INFINITY;
    }
    float mx = sc[0];
#pragma unroll
    for (int e = 1; e < 16; ++e) mx = fmaxf(mx, sc[e]);
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    if (__any(mx > m)) {
      // finite: p0 and the waves' first queries are multiples of 32, so a tile that is not skipped
      // holds at least one key for each of its queries
      const float mn = fmaxf(m, mx);
      const float corr = __builtin_amdgcn_exp2f((m - mn) * c2);
      m = mn;
      l *= corr;
#pragma unroll
      for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] *= corr;
    }
    const float mc = m * c2;
    float rs = 0.f;
    h8 pb[2];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float p = __builtin_amdgcn_exp2f(sc[e] * c2 - mc);
      rs += p;
      pb[e >> 3][e & 7] = (half_t)p;
    }
    l += rs + __shfl_xor(rs, 32);
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int t = 0; t < DT; ++t) {
        const h4 a0 = fv[t][s2][0], a1 = fv[t][s2][1];
        const h8 a = {a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, pb[s2], acc[t], 0, 0, 0);
      }
  };

  // every group makes the same number of trips (barriers)
  int stage = 0;
  for (int kb = 0; kb <= last_key; kb += STEP, stage ^= 1) {
    const int k0 = kb + kg;
    // this wave's half of tile k0 has landed and its reads of the other stage are over ...
    wait_vm_at_most<0>();
    wait_lgkm_at_most<0>();
    __builtin_amdgcn_s_barrier();             // ... and so for everybody
    asm volatile("" ::: "memory");
    const bool mine = k0 <= last_key && k0 <= p0 + wave_q + 31;      // not above the wave's diagonal
    if (mine) load_tile(buf + stage * PF_ATTN_TILE_HALVES(HD));
    __builtin_amdgcn_sched_barrier(0);
    if (k0 + STEP <= last_key) issue(k0 + STEP, stage ^ 1);
    __builtin_amdgcn_sched_barrier(0);
    if (mine) tile(k0);
  }

  if constexpr (G == 1) {
    if (qi < n) {
      const float rl = 1.0f / l;
#pragma unroll
      for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {   // rows 32 t + 8 g4 + 4 hf + (0..3) of O^T = 4 consecutive columns of O
          h4 o;
#pragma unroll
          for (int j = 0; j < 4; ++j) o[j] = (half_t)(acc[t][g4 * 4 + j] * rl);
          *reinterpret_cast<h4*>(O + act_offset(qi, h * HD + t * 32 + g4 * 8 + hf * 4, d, frag_tb)) = o;
        }
    }
  } else {
    // merge: every group leaves (m, l, O^T) in LDS, [group][quad of values][thread of the group][4] and [group][2][thread];
    // then group g adds up and stores its share of the quads
    constexpr int QUADS = DT * 4, SHARE = QUADS / G;
    static_assert(QUADS % G == 0, "quads divide over the groups");
    float* mo = reinterpret_cast<float*>(pf_attn_lds);
    float* ml = mo + G * QUADS * 128 * 4;
    __syncthreads();   // all tiles consumed: the tile buffers are free
#pragma unroll
    for (int i = 0; i < QUADS; ++i)
      *reinterpret_cast<f4*>(mo + ((grp * QUADS + i) * 128 + tid) * 4) =
          f4{acc[i >> 2][(i & 3) * 4], acc[i >> 2][(i & 3) * 4 + 1], acc[i >> 2][(i & 3) * 4 + 2], acc[i >> 2][(i & 3) * 4 + 3]};
    ml[grp * 256 + tid] = m;
    ml[grp * 256 + 128 + tid] = l;
    __syncthreads();
    if (qi >= n) return;
    float w[G], M = -INFINITY, L = 0.f;
#pragma unroll
    for (int g = 0; g < G; ++g) { w[g] = ml[g * 256 + tid]; M = fmaxf(M, w[g]); }      // finite: group 0 always holds key 0
#pragma unroll
    for (int g = 0; g < G; ++g) {
      w[g] = __builtin_amdgcn_exp2f((w[g] - M) * c2);          // a group without an unmasked key has m = -inf: weight 0
      L += ml[g * 256 + 128 + tid] * w[g];
    }
    const float rl = 1.0f / L;
#pragma unroll
    for (int i = 0; i < SHARE; ++i) {
      const int quad = grp * SHARE + i;
      f4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int g = 0; g < G; ++g) v += *reinterpret_cast<const f4*>(mo + ((g * QUADS + quad) * 128 + tid) * 4) * w[g];
      h4 o;
#pragma unroll
      for (int j = 0; j < 4; ++j) o[j] = (half_t)(v[j] * rl);
      *reinterpret_cast<h4*>(O + act_offset(qi, h * HD + (quad >> 2) * 32 + (quad & 3) * 8 + hf * 4, d, frag_tb)) = o;
    }
  }
}

// Hm[r][i] = silu(G[r][i]) * U[r][i] with GU = slices of [Mb][2F] fp32 (gate | up), summed here.
// grid = (Mb, ceil(F/1024))
__global__ __launch_bounds__(LL_WG) void pf_swiglu_kernel(const float* __restrict__ GU, SliceMap map,
                                                          const DevState* __restrict__ st,
                                                          half_t* __restrict__ Hm, int F) {
  const int r = blockIdx.x;
  const int i = (blockIdx.y * LL_WG + threadIdx.x) * 4;
  if (i >= F) return;
  h4 o = {0, 0, 0, 0};
  if (r < st->n_prompt) {
    const float* row = GU + (size_t)r * 2 * F;
    const f4 g = pf_slice_sum(row + i, slice_count(map, i), map.slice_floats);
    const f4 u = pf_slice_sum(row + F + i, slice_count(map, F + i), map.slice_floats);
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = (half_t)(g[j] / (1.0f + expf(-g[j])) * u[j]);
  }
  *reinterpret_cast<h4*>(Hm + (size_t)r * F + i) = o;
}
