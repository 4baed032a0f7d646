// Batched lock-step decoding over a paged KV cache: the kernels that have no counterpart in the
// single-sequence path.  The paper embeds a paged-KV attention library for its cache (Sec. II-C,
// Sec. V-A) and keeps batch 1 (Sec. V-A); this is the batch > 1 regime it leaves open, where the
// projections of a step become 16- or 32-row matrix products (the short-prompt kernels of
// prefill_skinny.h, one row per sequence) instead of GEMVs.
//
// A sequence owns pages of `page_tokens` consecutive cache rows; page_table[slot][i] is the first
// cache row of its i-th page, so position p of slot b lives in cache row
// page_table[b][p / page_tokens] + p % page_tokens of the per-layer pools [head][pool rows][head_dim].
// Free slots point at page 0, which no sequence ever owns: whatever they compute lands there.
#pragma once
#include "ll_device.h"
#include "sample_kernels.h"

#define BT_MAX_BATCH 32

struct BatchState {
  int32_t pos[BT_MAX_BATCH];         // cached positions of slot b = position of the token it feeds next
  int32_t next_token[BT_MAX_BATCH];  // token slot b feeds next
  int32_t active[BT_MAX_BATCH];      // 0: free slot
  int32_t steps[BT_MAX_BATCH];       // tokens slot b's sequence has produced (the draw index of stochastic selection)
  int32_t order[BT_MAX_BATCH];       // slots in the order in which the attention kernel takes them, see bt_order
};

// Slots 0 .. rows - 1 by falling length, every second round of `per_round` of them reversed: workgroups are dealt to the CUs in
// turn, so a CU that has one of the longest sequences first gets one of the shortest next (in slot order a CU could
// get all four of its sequences long: 32 sequences of 10 .. 560 keys 22.3 -> 19.1 us per layer, 16 of them 12.9 -> 12.4).
// All sequences grow by one a step: the order holds until one joins or leaves.
inline void bt_order(const int32_t* pos, const int32_t* active, int rows, int per_round, int32_t* order) {
  for (int b = 0; b < rows; ++b) {
    int rank = 0;
    for (int o = 0; o < rows; ++o) {
      const int lo = active[o] ? pos[o] : -1, lb = active[b] ? pos[b] : -1;
      rank += lo > lb || (lo == lb && o < b);
    }
    const int round = rank / per_round, first = round * per_round, last = (rows < first + per_round ? rows : first + per_round) - 1;
    order[round & 1 ? first + last - rank : rank] = b;
  }
}

// Attention of slot b's new query (position pos[b], already written to the cache) for one head.
// grid = (heads, rows of the step = 16 or 32: slots in bt_order's order), NT threads, four waves per SIMD (the launch bound says so: without it
// the compiler takes 143 registers at head_dim 64, and half as many workgroups fit a CU); tb = rows / 16 selects the output's
// fragment-major layout.  512 threads at 16 rows; 256 at 32, where twice as many workgroups then run side by side and
// the many short sequences of a mixed batch leave fewer lanes idle (16 sequences of 10..560 keys 12.6 -> 11.3 us per
// layer, 32 sequences 22.9 -> 19.9; 32 sequences in 512-thread workgroups: 21.3).  Two trips of 16 keys per wave are
// in flight; the kernel's time is that of the longest sequences' trips, some 225 instructions per wave and trip.  As in the single-sequence kernel a key row is read
// by HD / 8 adjacent lanes with one 16-byte load each and every lane group keeps an online-softmax
// state over the keys it is dealt; groups merge by shuffles, waves through LDS.  Output: fp16,
// in the fragment-major operand layout of the O projection.
#define BT_ATTN_THREADS(TB) ((TB) == 1 ? 512 : 256)
template <int HD, int NT>
__global__ __launch_bounds__(NT, 4) void bt_attn_kernel(
    const half_t* __restrict__ Q, const half_t* __restrict__ kc, const half_t* __restrict__ vc,
    const BatchState* __restrict__ bs, const int* __restrict__ page_table, int pt_stride, int page_tokens,
    half_t* __restrict__ O, int d, int pool_rows, int tb) {
  constexpr int LPR = HD / 8;      // lanes per key row
  constexpr int GPW = 64 / LPR;    // lane groups per wave
  constexpr int NW = NT / 64;
  constexpr int UK = 4;            // keys in flight per group
  __shared__ float s_m[NW], s_l[NW], s_acc[NW][HD];
  extern __shared__ int s_pt[];    // this slot's page-table row: a key's address then costs no global round trip
  const int h = blockIdx.x, b = bs->order[blockIdx.y];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // key positions of a trip then start from a scalar
  const int gi = lane / LPR, li = lane % LPR;
  // One round trip for everything the key loop needs: the slot's state, the query and the WHOLE page-table
  // row (entries past the sequence's end are not used; reading them saves waiting for the position first).
  const int active = bs->active[b];
  const int n_keys = bs->pos[b] + 1;
  const h8 q = load_h8(Q + (size_t)b * d + h * HD + li * 8);
  for (int i = tid; i < pt_stride; i += NT) s_pt[i] = page_table[b * pt_stride + i];
  if (!active) {
    if (tid < HD / 8) *reinterpret_cast<h8*>(O + act_offset(b, h * HD + tid * 8, d, tb)) = h8{0, 0, 0, 0, 0, 0, 0, 0};
    return;
  }
  __syncthreads();
  const float scale = 1.0f / sqrtf((float)HD);
  float qv[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) qv[e] = (float)q[e] * scale;
  const half_t* kh = kc + (size_t)h * pool_rows * HD + li * 8;
  const half_t* vh = vc + (size_t)h * pool_rows * HD + li * 8;

  // Page of a position by a reciprocal instead of an integer division per key: (u + 1/2) / page_tokens is at least
  // 1 / (2 page_tokens) away from an integer, more than its rounding error for every u < 2^20 (the limit of max_seq).
  const float rpt = 1.0f / (float)page_tokens;
  float m = -INFINITY, l = 0.f, acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
  constexpr int STRIDE = NW * GPW, TRIP = STRIDE * UK;     // keys one trip of the workgroup covers
  // Trips are double-buffered: the requests of trip t + 1 go out before trip t is used, so a long sequence
  // costs one memory round trip plus the arithmetic of its trips, not a round trip per trip.  A trip past
  // the sequence's end is still requested (every key clamped to the last one: cache hits), which keeps
  // the number of loads in flight the same on every path and the waits exact.
  auto issue = [&](int base, h8 (&kk)[UK], h8 (&vv)[UK]) {
#pragma unroll
    for (int j = 0; j < UK; ++j) {
      const int u = min(base + j * STRIDE + gi, n_keys - 1);
      const int pg = (int)(((float)u + 0.5f) * rpt);     // u / page_tokens
      const size_t row = (size_t)(s_pt[pg] + (u - pg * page_tokens));
      kk[j] = load_stream(kh + row * HD);
      vv[j] = load_stream(vh + row * HD);
    }
  };
  // One online-softmax step per trip, not per key: the trip's scores first, then one new maximum, one
  // correction of the running state and one exponential per key (branch-free: inside a branch the
  // compiler sinks a value row's load to its use and waits for it there).
  auto consume = [&](int base, const h8 (&kk)[UK], const h8 (&vv)[UK]) {
    float dot[UK], mn = m;
#pragma unroll
    for (int j = 0; j < UK; ++j) {
      float t = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) t += qv[e] * (float)kk[j][e];
      t = group_sum<LPR>(t);
      dot[j] = (base + j * STRIDE + gi < n_keys) ? t : -INFINITY;
      mn = fmaxf(mn, dot[j]);
    }
    const float corr = (m == mn) ? 1.0f : __expf(m - mn);     // also m = mn = -inf
    l *= corr;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] *= corr;
#pragma unroll
    for (int j = 0; j < UK; ++j) {
      const float p = (dot[j] > -INFINITY) ? __expf(dot[j] - mn) : 0.f;
      l += p;
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += p * (float)vv[j][e];
    }
    m = mn;
  };
  h8 ka[UK], va[UK], kb[UK], vb[UK];
  issue(wave * GPW, ka, va);
  if (n_keys <= TRIP) {
    consume(wave * GPW, ka, va);
  } else for (int base = wave * GPW; base < n_keys; base += 2 * TRIP) {
    issue(base + TRIP, kb, vb);
    __builtin_amdgcn_sched_barrier(0);
    consume(base, ka, va);
    __builtin_amdgcn_sched_barrier(0);
    issue(base + 2 * TRIP, ka, va);
    __builtin_amdgcn_sched_barrier(0);
    consume(base + TRIP, kb, vb);
    __builtin_amdgcn_sched_barrier(0);
  }
  {
    float M = m;
#pragma unroll
    for (int off = LPR; off < 64; off <<= 1) M = fmaxf(M, __shfl_xor(M, off));
    const float w = (M > -INFINITY) ? __expf(m - M) : 0.f;   // empty groups (m = -inf) weigh 0
    l *= w;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] *= w;
#pragma unroll
    for (int off = LPR; off < 64; off <<= 1) {
      l += __shfl_xor(l, off);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += __shfl_xor(acc[e], off);
    }
    if (gi == 0) {
      if (li == 0) { s_m[wave] = M; s_l[wave] = l; }
#pragma unroll
      for (int e = 0; e < 8; ++e) s_acc[wave][li * 8 + e] = acc[e];
    }
  }
  __syncthreads();
  if (tid < HD) {
    float M = -INFINITY;
#pragma unroll
    for (int i = 0; i < NW; ++i) M = fmaxf(M, s_m[i]);
    float L = 0.f, A = 0.f;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const float w = (s_m[i] > -INFINITY) ? __expf(s_m[i] - M) : 0.f;    // M is finite: key 0 is always attended
      L += s_l[i] * w;
      A += s_acc[i][tid] * w;
    }
    O[act_offset(b, h * HD + tid, d, tb)] = (half_t)(A / L);
  }
}

// Token of every slot and the slots' state advance: greedy (lowest index among equal maxima), or
// the stochastic selection of sample_kernels.h with the slot's own draw index, so a sequence draws
// the same stream in a batch as alone.  grid = rows of the step, SMP_THREADS threads, SMP_Z_BYTES(PER)
// of dynamic LDS; out = device-visible host memory, -1 for free slots.
template <int PER>
__global__ __launch_bounds__(SMP_THREADS) void bt_select_kernel(const float* __restrict__ logits, int vocab,
                                                                const SampleCfg* __restrict__ cfg,
                                                                BatchState* bs, int* out) {
  extern __shared__ float bt_z[];
  __shared__ int si[SMP_THREADS];
  __shared__ uint32_t sk[SMP_THREADS];
  __shared__ float red[2 * 3 * (SMP_THREADS / 64)];
  __shared__ int found;
  const int b = blockIdx.x, tid = threadIdx.x;
  const float* row = logits + (size_t)b * vocab;
  // (requested together: see sample_kernel)
  const float inv_temp = cfg->inv_temp, logit0 = row[min(tid, vocab - 1)];
  const int active = bs->active[b], pos = bs->pos[b], steps = bs->steps[b];
  if (!active) {
    if (tid == 0) out[b] = -1;
    return;
  }
  int tok;
  if (inv_temp == 0.f || vocab > SMP_THREADS * PER) {
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    for (int i = tid * 4; i < vocab; i += SMP_THREADS * 4) {     // vocab % 16 == 0 (checked when the batch is opened)
      const f4 v = *reinterpret_cast<const f4*>(row + i);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (v[e] > bv) { bv = v[e]; bi = i + e; }                // indices ascend: the first maximum stays
    }
    tok = smp_block_argmax(bv, bi, red, si);
    if (tok == 0x7fffffff) tok = 0;          // every logit NaN: still a valid id
  } else {
    tok = smp_draw_token<PER>(row, vocab, cfg, (uint32_t)steps, logit0, bt_z, si, sk, red, &found);
  }
  if (tid == 0) {
    bs->next_token[b] = tok;
    bs->pos[b] = pos + 1;
    bs->steps[b] = steps + 1;
    out[b] = tok;
  }
}

// After a prompt has been prefilled into the contiguous single-sequence cache: copy its rows
// 0 .. n - 1 into the pages of slot b.  grid = (n, layers * 2); a workgroup moves one cache row of
// every head of one layer's K or V.
__global__ __launch_bounds__(LL_WG) void bt_scatter_kernel(const half_t* __restrict__ src_kv, size_t src_layer_halves,
                                                           int src_rows, half_t* __restrict__ dst_kv,
                                                           size_t dst_layer_halves, int dst_rows,
                                                           const int* __restrict__ page_table, int pt_stride,
                                                           int page_tokens, int slot, int n_heads, int head_dim) {
  const int r = blockIdx.x, lk = blockIdx.y;      // lk = layer * 2 + (0: K, 1: V)
  const int pg = r / page_tokens;
  const size_t drow = (size_t)(page_table[slot * pt_stride + pg] + (r - pg * page_tokens));
  const half_t* s = src_kv + (size_t)lk * src_layer_halves;
  half_t* d = dst_kv + (size_t)lk * dst_layer_halves;
  const int per_head = head_dim / 8;
  for (int i = threadIdx.x; i < n_heads * per_head; i += LL_WG) {
    const int h = i / per_head, c = i - h * per_head;
    *reinterpret_cast<h8*>(d + ((size_t)h * dst_rows + drow) * head_dim + c * 8) =
        load_h8(s + ((size_t)h * src_rows + r) * head_dim + c * 8);
  }
}

// Slots' state (by workgroup 0) and one page-table row per workgroup, from the host's pinned mirrors: one launch where
// two copies in front of the next kernel cost 15 us more.  grid = rows, row first + blockIdx.x.  st: optionally where slot
// `first` finds its next token, that of a prefill still in the queue
__global__ __launch_bounds__(LL_WG) void bt_push_kernel(const int* __restrict__ h_state, int* __restrict__ state,
                                                        const int* __restrict__ h_table, int* __restrict__ table,
                                                        int pt_stride, int first, const DevState* __restrict__ st) {
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < (int)(sizeof(BatchState) / 4); i += LL_WG)
      state[i] = st && i == (int)(offsetof(BatchState, next_token) / 4) + first ? st->next_token : h_state[i];
  const size_t row = (size_t)(first + blockIdx.x) * pt_stride;
  for (int i = threadIdx.x; i < pt_stride; i += LL_WG) table[row + i] = h_table[row + i];
}

// Page-table entries that changed since the last step, passed by value: one small launch in
// front of the step instead of a host-to-device copy of the table.
struct PageUpdates {
  int n;
  int index[BT_MAX_BATCH];      // slot * pt_stride + page number
  int row[BT_MAX_BATCH];        // first cache row of the page
};
__global__ __launch_bounds__(64) void bt_page_update_kernel(int* __restrict__ page_table, PageUpdates u) {
  const int i = threadIdx.x;
  if (i < u.n) page_table[u.index[i]] = u.row[i];
}
