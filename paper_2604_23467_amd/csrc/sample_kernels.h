// Token selection and state advance, the last kernel of every step: greedy
// argmax, or temperature / top-k / top-p sampling with a counter-based random
// draw.  The paper leaves sampling to its host-side dynamic domain (Sec. III-A,
// III-C) and lists stochastic operations as what keeps it outside graph replay
// (Sec. VI-C); here it is one single-workgroup kernel inside the captured graph:
// its parameters and the draw index live in device memory, so replays stay
// bit-reproducible for a given seed and a reset replays the same stream.
//
// Definition (every open choice of the textbook procedure fixed as stated):
//   z_i = logit_i * float(1 / T); candidates C = the top_k largest z (ties by lower index);
//   e_i = exp(z_i - max z) over C, S = sum; nucleus F = candidates above the threshold value tau
//   plus the first n_tie equal to it (lower index first), tau = largest value whose upper set has
//   mass >= top_p * S, n_tie = ceil((top_p * S - mass above) / e_tau) >= 1; the draw walks F in
//   order of increasing INDEX and returns the first token whose running sum of e exceeds u * sum_F;
//   u = (x0 >> 8) * 2^-24, x0 = first word of Philox4x32-10(counter = (draw index, 0, 0, 0), key = seed).
//
// Nothing is sorted.  Every thread holds up to 32 consecutive tokens in registers (vocabularies up to 32768).  A top-k cut
// first finds a bound that leaves a few hundred candidates; up to 512 of them are ranked, each compared with all others,
// and the ranks give the cut and, by one prefix sum, the nucleus.  Without a cut, or with more candidates, the k-th largest
// value and the nucleus threshold are found by bisecting the 32 bits of an order-preserving integer image of z, two
// bits to a block-wide count or sum.
#pragma once
#include "ll_device.h"

#define SMP_THREADS 1024
#define SMP_PER 32                               // consecutive tokens per thread
#define SMP_MAX_VOCAB (SMP_THREADS * SMP_PER)
// tokens per thread that a selection kernel is built for, and its dynamic LDS
inline int smp_per(int vocab) { return vocab <= SMP_THREADS ? 1 : vocab <= SMP_THREADS * 8 ? 8 : SMP_PER; }
#define SMP_Z_BYTES(PER) (((PER) == 1 ? SMP_THREADS : SMP_THREADS / 32 * 33 * (PER)) * 4)

struct SampleCfg {
  float inv_temp;      // float(1 / T); 0 selects greedy argmax
  int32_t top_k;       // 0 or >= vocab: no top-k cut
  float top_p;         // 1: no nucleus cut
  uint32_t seed_lo, seed_hi;
  int32_t pad[11];
};

__device__ __forceinline__ void philox4x32_10(uint32_t (&c)[4], uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c[1] ^ k0;
    const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c[3] ^ k1;
    c[0] = n0; c[1] = (uint32_t)p1; c[2] = n2; c[3] = (uint32_t)p0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
}

// larger float <=> larger key; every real value maps above key 0, which marks "no token"
__device__ __forceinline__ uint32_t order_key(float z) {
  const uint32_t b = __builtin_bit_cast(uint32_t, z);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ __forceinline__ float key_to_float(uint32_t k) {
  return __builtin_bit_cast(float, (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// Block-wide sums of three values at once over SMP_THREADS threads; every thread gets the
// results.  `red` holds two banks of 3 x 16 wave slots used alternately (`phase` counts the
// calls), so one barrier per call is enough: a bank is rewritten only two calls later, and
// nobody can be two barriers ahead of a thread that still reads it.
struct Sum3 { float a, b, c; };
__device__ __forceinline__ Sum3 smp_block_sum3(float a, float b, float c, float* red, int& phase) {
  constexpr int NW = SMP_THREADS / 64;
  a = wave_sum(a);
  b = wave_sum(b);
  c = wave_sum(c);
  const int tid = threadIdx.x;
  float* bank = red + (phase & 1) * 3 * NW;
  ++phase;
  if ((tid & 63) == 0) { bank[tid >> 6] = a; bank[NW + (tid >> 6)] = b; bank[2 * NW + (tid >> 6)] = c; }
  __syncthreads();
  Sum3 s = {0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < NW; ++w) { s.a += bank[w]; s.b += bank[NW + w]; s.c += bank[2 * NW + w]; }
  return s;
}
__device__ __forceinline__ float smp_block_sum(float v, float* red, int& phase) {
  return smp_block_sum3(v, 0.f, 0.f, red, phase).a;
}
// counts stay below 2^24, so they are exact in the float lanes of the reduction
__device__ __forceinline__ int smp_block_sum_int(int v, float* red, int& phase) {
  return (int)(smp_block_sum(v, red, phase) + 0.5f);
}
__device__ __forceinline__ float smp_block_max(float m, float* red, int& phase) {
  constexpr int NW = SMP_THREADS / 64;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  const int tid = threadIdx.x;
  float* bank = red + (phase & 1) * 3 * NW;
  ++phase;
  if ((tid & 63) == 0) bank[tid >> 6] = m;
  __syncthreads();
  m = bank[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) m = fmaxf(m, bank[w]);
  return m;
}

// Exclusive prefix sum over the threads in thread order (and the grand total), one barrier:
// shuffle scan inside each wave, then every thread adds the totals of the waves before its own,
// always in the same order, so the result is reproducible.
__device__ __forceinline__ float smp_block_scan_excl(float v, float* red, int& phase, float* total) {
  constexpr int NW = SMP_THREADS / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const float up = __shfl_up(incl, off);
    if (lane >= off) incl += up;
  }
  float* bank = red + (phase & 1) * 3 * NW;
  ++phase;
  if (lane == 63) bank[wave] = incl;
  __syncthreads();
  float before = 0.f, all = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    if (w < wave) before += bank[w];
    all += bank[w];
  }
  *total = all;
  const float prev = __shfl_up(incl, 1);
  return before + (lane > 0 ? prev : 0.f);
}

// k-th largest key over PER slots per thread (0 marks an empty slot) by bisecting the key's 32
// bits two at a time; a wave counts with ballots, so a slot costs one compare per candidate prefix.
// Returns 0 when fewer than k slots are filled.  low_bit > 0 stops above that bit: a lower bound whose lower bits
// are zero, at fewer passes; `prefix` and high_bit go on from there.
template <int PER>
__device__ __forceinline__ uint32_t smp_kth_largest(const uint32_t (&key)[PER], int k, float* red, int& phase,
                                                    int low_bit = 0, int high_bit = 31, uint32_t prefix = 0u) {
  constexpr int NW = SMP_THREADS / 64;
  const int tid = threadIdx.x;
  for (int bit = high_bit; bit >= low_bit + 1; bit -= 2) {
    const uint32_t c1 = prefix | (1u << (bit - 1)), c2 = prefix | (2u << (bit - 1)), c3 = prefix | (3u << (bit - 1));
    int n1 = 0, n2 = 0, n3 = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      n1 += __builtin_popcountll(__ballot(key[j] >= c1));
      n2 += __builtin_popcountll(__ballot(key[j] >= c2));
      n3 += __builtin_popcountll(__ballot(key[j] >= c3));
    }
    int* bank = reinterpret_cast<int*>(red) + (phase & 1) * 3 * NW;
    ++phase;
    if ((tid & 63) == 0) { bank[tid >> 6] = n1; bank[NW + (tid >> 6)] = n2; bank[2 * NW + (tid >> 6)] = n3; }
    __syncthreads();
    int t1 = 0, t2 = 0, t3 = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) { t1 += bank[w]; t2 += bank[NW + w]; t3 += bank[2 * NW + w]; }
    prefix = t3 >= k ? c3 : t2 >= k ? c2 : t1 >= k ? c1 : prefix;
  }
  return prefix;
}

// Top-k cut over PER slots per thread (thread order = index order): slots outside the k largest
// keys (equal keys enter by lower index) get key 0; every kept slot gets e = exp(z - zmax).
// top_k = 0 keeps every filled slot.
template <int PER>
__device__ __forceinline__ void smp_apply_topk(uint32_t (&key)[PER], float (&e)[PER], int top_k, float zmax,
                                               float* red, int& phase) {
  uint32_t cut = 1u;          // kept: key > cut, or key == cut among the first tie_take ties
  int tie_take = 0x7fffffff;  // (cut = 1 with all ties taken keeps every real token: real keys are >= 0x007FFFFF)
  int seen = 0;
  if (top_k > 0) {
    cut = smp_kth_largest<PER>(key, top_k, red, phase);
    int gt = 0, mine = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) { gt += key[j] > cut; mine += key[j] == cut; }
    tie_take = top_k - smp_block_sum_int(gt, red, phase);
    float all;
    seen = (int)(smp_block_scan_excl((float)mine, red, phase, &all) + 0.5f);   // ties before this thread
  }
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    bool in = key[j] > cut;
    if (key[j] == cut && key[j] != 0u) { in = seen < tie_take; ++seen; }
    if (!in) key[j] = 0u;
    e[j] = in ? expf(key_to_float(key[j]) - zmax) : 0.f;
  }
}

// Nucleus cut and draw over PER kept-or-dropped slots per thread; slot j of a thread is token
// id0 + j and thread order is index order.  Dropped slots have key 0 and e 0.
template <int PER>
__device__ __forceinline__ int smp_nucleus_and_draw(uint32_t (&key)[PER], float (&e)[PER], int id0, float top_p,
                                                    float u, float* red, int& phase, int* found) {
  const int tid = threadIdx.x;
  auto ties_before = [&](uint32_t at) {
    int mine = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) mine += key[j] == at;
    float all;
    return (int)(smp_block_scan_excl((float)mine, red, phase, &all) + 0.5f);   // counts < 2^24: exact
  };
  // top-p: largest key whose upper set holds top_p of the mass, ties by index order
  if (top_p < 1.f) {
    float mine = 0.f;
#pragma unroll
    for (int j = 0; j < PER; ++j) mine += e[j];
    const float want = top_p * smp_block_sum(mine, red, phase);
    uint32_t prefix = 0u;
    for (int bit = 31; bit >= 1; bit -= 2) {      // two bits per pass: three candidate prefixes, one reduction
      const uint32_t c1 = prefix | (1u << (bit - 1)), c2 = prefix | (2u << (bit - 1)), c3 = prefix | (3u << (bit - 1));
      float m1 = 0.f, m2 = 0.f, m3 = 0.f;
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        m1 += key[j] >= c1 ? e[j] : 0.f;
        m2 += key[j] >= c2 ? e[j] : 0.f;
        m3 += key[j] >= c3 ? e[j] : 0.f;
      }
      const Sum3 m = smp_block_sum3(m1, m2, m3, red, phase);
      prefix = m.c >= want ? c3 : m.b >= want ? c2 : m.a >= want ? c1 : prefix;
    }
    if (prefix != 0u) {                            // prefix = 0: rounding left the total below the target, keep all
      float above = 0.f, etau = 0.f;
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        above += key[j] > prefix ? e[j] : 0.f;
        if (key[j] == prefix) etau = e[j];
      }
      above = smp_block_sum(above, red, phase);
      etau = smp_block_max(etau, red, phase);      // every tie has the same e; take it from whichever thread holds one
      int n_tie = (int)ceilf((want - above) / etau);
      if (n_tie < 1) n_tie = 1;
      int seen = ties_before(prefix);
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        bool in = key[j] > prefix;
        if (key[j] == prefix) { in = seen < n_tie; ++seen; }
        if (!in) { key[j] = 0u; e[j] = 0.f; }
      }
    }
  }

  // the draw: running sum of e in index order against u * total
  float mine = 0.f;
#pragma unroll
  for (int j = 0; j < PER; ++j) mine += e[j];
  if (tid == 0) *found = 0x7fffffff;
  float total;
  const float run0 = smp_block_scan_excl(mine, red, phase, &total);   // (its barrier also publishes *found)
  const float target = u * total;
  // every thread continues the walk from the running sum in front of its range; the lowest
  // token whose running sum exceeds the target wins, exactly as in a sequential walk
  {
    float run = run0;
    int pick = 0x7fffffff;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      if (e[j] > 0.f) {
        run += e[j];
        if (pick == 0x7fffffff && run > target) pick = id0 + j;
      }
    }
    if (pick != 0x7fffffff) atomicMin(found, pick);
  }
  __syncthreads();
  if (*found == 0x7fffffff) {
    // rounding left no running sum above the target: the last kept token
    __syncthreads();
    if (tid == 0) *found = -1;
    __syncthreads();
    int last = -1;
#pragma unroll
    for (int j = 0; j < PER; ++j) if (e[j] > 0.f) last = id0 + j;
    if (last >= 0) atomicMax(found, last);
    __syncthreads();
  }
  return *found < 0 ? 0 : *found;
}

// Top-k cut, nucleus cut and draw over n <= SMP_THREADS / TPC candidates (sk: keys, si: tokens, in index order; LDS).  All
// threads find every candidate's rank in the order (key descending, index ascending) by comparing it with all others, TPC
// threads to a candidate; the ranks ARE the top-k cut, and one wave finds the nucleus by one prefix sum over the masses in
// rank order and draws: no serial chain of one pass per key bit is left.  What bounded it was that chain.  The selection
// kernel with top-p 0.95, us, with this and the bound that each wave finds by itself (below); in brackets with the bits
// bisected by one wave (up to 256 candidates) or by all with a barrier per pass: vocabulary 500 and 1024, top-k 50 13.4 and
// 11.1 (16.6, 16.8), 1024, top-k 300 21.1 (38.9); 32000, top-k 50 22.1 (26.6).  Not gained: 32000, top-k 200 27.0 (26.7);
// 1024, top-k 600, which takes the steps it took, 39.6 (38.9).  With one thread to each of up to 1024 candidates the last wave
// holds 16 a lane, which spill: top-k 600 45.9.  scratch: SMP_THREADS words of LDS nobody reads any more.
// Returns the token in every thread.
template <int TPC>
__device__ __forceinline__ int smp_ranked_pick(const uint32_t* sk, const int* si, int n, int top_k, float zmax, float top_p,
                                               float u, float* scratch, int* found) {
  static_assert(TPC == 2 || TPC == 4, "a candidate's threads lie in one quad");
  constexpr int PER = SMP_THREADS / TPC / 64;
  const int tid = threadIdx.x, lane = tid & 63;
  int* rank_of = reinterpret_cast<int*>(scratch);
  float* sorted = scratch + SMP_THREADS / TPC;
  {
    const int c = tid / TPC, q = tid & (TPC - 1);
    const uint32_t key = c < n ? sk[c] : 0u;
    int r = 0;
#pragma unroll 4
    for (int j = q; j < n; j += TPC) {
      const uint32_t other = sk[j];
      r += other > key || (other == key && j < c);
    }
    r += __builtin_amdgcn_update_dpp(0, r, 0xB1, 0xf, 0xf, true);
    if (TPC == 4) r += __builtin_amdgcn_update_dpp(0, r, 0x4E, 0xf, 0xf, true);
    if (q == 0 && c < n) rank_of[c] = r;
  }
  __syncthreads();
  if (tid < 64) {
    int rank[PER], id[PER];
    float e[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int c = lane * PER + j;
      const bool have = c < n;
      rank[j] = have ? rank_of[c] : c;              // (places n .. of the sorted order are empty)
      id[j] = have ? si[c] : 0;
      e[j] = have && rank[j] < top_k ? expf(key_to_float(sk[c]) - zmax) : 0.f;
      sorted[rank[j]] = e[j];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // read back by other lanes of this wave
    __builtin_amdgcn_wave_barrier();
    auto scan = [&](float mine) {                   // running sum over the lanes, this one included
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const float up = __shfl_up(mine, off);
        if (lane >= off) mine += up;
      }
      return mine;
    };
    if (top_p < 1.f) {
      // smallest prefix of the rank order that holds top_p of the mass; rounding may leave the total below it: keep all
      float v[PER], mine = 0.f;
#pragma unroll
      for (int j = 0; j < PER; ++j) mine += v[j] = sorted[lane * PER + j];
      const float incl = scan(mine), want = top_p * __shfl(incl, 63);
      float run = __shfl_up(incl, 1);
      if (lane == 0) run = 0.f;
      int last = 0x7fffffff;
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        run += v[j];
        if (last == 0x7fffffff && run >= want) last = lane * PER + j;
      }
      const unsigned long long hit = __ballot(last != 0x7fffffff);
      last = hit ? __builtin_amdgcn_readlane(last, __builtin_ctzll(hit)) : n;
#pragma unroll
      for (int j = 0; j < PER; ++j)
        if (rank[j] > last) e[j] = 0.f;
    }
    // the draw: running sum of e in index order against u * total; the lowest token past it, or the last kept one
    float mine = 0.f;
#pragma unroll
    for (int j = 0; j < PER; ++j) mine += e[j];
    const float incl = scan(mine), target = u * __shfl(incl, 63);
    float run = __shfl_up(incl, 1);
    if (lane == 0) run = 0.f;
    int pick = 0x7fffffff, last = -1;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      if (e[j] > 0.f) {
        run += e[j];
        if (pick == 0x7fffffff && run > target) pick = id[j];
        last = id[j];
      }
    }
    const unsigned long long hit = __ballot(pick != 0x7fffffff), kept = __ballot(last >= 0);
    const int t = hit ? __builtin_amdgcn_readlane(pick, __builtin_ctzll(hit))
                      : kept ? __builtin_amdgcn_readlane(last, 63 - __builtin_clzll(kept)) : 0;
    if (tid == 0) *found = t;
  }
  __syncthreads();
  return *found;
}

// One draw from logits[0 .. vocab) by a workgroup of SMP_THREADS threads (all of them call this;
// vocab <= SMP_THREADS * PER, cfg->inv_temp != 0).  smp_z: SMP_Z_BYTES(PER) of LDS; si, sk: SMP_THREADS
// words each; red: 6 words per wave; found: one word; logit0: logits[thread], fetched by the caller.  Returns the token in
// every thread.
template <int PER>
__device__ __forceinline__ int smp_draw_token(const float* __restrict__ logits, int vocab,
                                           const SampleCfg* __restrict__ cfg, uint32_t draw_index, float logit0,
                                           float* smp_z, int* si, uint32_t* sk, float* red, int* found) {
  const int tid = threadIdx.x;
  const float inv_temp = cfg->inv_temp;
  int phase = 0;
  int tok;
  // Thread t holds tokens t * per .. + per - 1: every thread has some, whatever the vocabulary (with 32 each, a
  // vocabulary of 1024 sat in 32 threads, too few for the bound of (1)).  More than one each: the logits are
  // read once, coalesced, into LDS rows of 32 padded to 33 words, from which a thread takes its share almost without
  // bank conflicts (read straight from global memory, every load instruction of a wave would touch 64 cache lines).
  const int per = PER == 1 ? 1 : (vocab + SMP_THREADS - 1) / SMP_THREADS;
  if (PER > 1) {
    for (int i = tid; i < vocab; i += SMP_THREADS) smp_z[i + (i >> 5)] = logits[i];
    __syncthreads();
  }
  const int base = tid * per;
  uint32_t key[PER];
  float zmax = -INFINITY;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int i = base + j;
    const bool have = j < per && i < vocab;
    const float z = have ? __fmul_rn(PER == 1 ? logit0 : smp_z[i + (i >> 5)], inv_temp) + 0.f : 0.f;   // + 0: -0 and +0 are one value
    key[j] = have ? order_key(z) : 0u;
    if (have) zmax = fmaxf(zmax, z);
  }
  zmax = smp_block_max(zmax, red, phase);

  uint32_t ctr[4] = {draw_index, 0u, 0u, 0u};
  philox4x32_10(ctr, cfg->seed_lo, cfg->seed_hi);
  const float u = (float)(ctr[0] >> 8) * (1.0f / 16777216.0f);
  const int top_k = (cfg->top_k >= 1 && cfg->top_k < vocab) ? cfg->top_k : 0;

  // (1) With a top-k cut of at most one candidate per thread, almost all of the vocabulary can be
  // discarded cheaply first: the k-th largest of the threads' own maxima is a lower bound of the
  // k-th largest key (at least k keys reach it), found with one slot per thread.  Its upper 16 bits (1 % of the
  // value) are mostly bound enough; where more candidates reach them than the split of the ranking holds (logits that share
  // an offset much larger than their spread) the lower bits are found too (32000 logits of 100 +- 0.5 at temperature 0.8,
  // top-k 200, a step: 95.6 us without, 66.3 with).  What reaches the bound is packed in index order, and up to 512 candidates
  // are ranked; more go on with one slot per thread.
  bool done = false;
  if (top_k > 0 && top_k <= SMP_THREADS) {
    uint32_t tmax[1] = {0u};
#pragma unroll
    for (int j = 0; j < PER; ++j) tmax[0] = key[j] > tmax[0] ? key[j] : tmax[0];
    uint32_t bound = 0u;
    // candidates to go on with: as many as the smallest split of the ranking that holds top_k of them
    const int enough = top_k <= SMP_THREADS / 4 ? SMP_THREADS / 4 : SMP_THREADS / 2;
    int at, nreach = SMP_THREADS + 1;
    auto count_reach = [&]() {
      int reach = 0;
#pragma unroll
      for (int j = 0; j < PER; ++j) reach += key[j] >= bound;
      float all;
      at = (int)(smp_block_scan_excl((float)reach, red, phase, &all) + 0.5f);
      nreach = (int)(all + 0.5f);
    };
    if (top_k <= SMP_THREADS / 8 && vocab > per * (SMP_THREADS - 64)) {
      // cheaper still: every wave finds the ceil(k / 16)-th largest of its own threads' maxima, and the smallest of the 16
      // is reached by at least k keys: ballots and one barrier in place of one barrier per pass.  Only where every wave holds
      // tokens (a wave without them would make the bound 0), and up to top-k 128: past it more than 256 reach this bound, and
      // ranking those costs more than the passes (32000 tokens, top-k 200: 30.7 us against 27.0)
      constexpr int NW = SMP_THREADS / 64;
      const int kw = (top_k + NW - 1) / NW;
      uint32_t prefix = 0u;
      for (int bit = 31; bit >= 16; --bit) {
        const uint32_t c = prefix | (1u << bit);
        if (__builtin_popcountll(__ballot(tmax[0] >= c)) >= kw) prefix = c;
      }
      uint32_t* bank = reinterpret_cast<uint32_t*>(red) + (phase & 1) * 3 * NW;
      ++phase;
      if ((tid & 63) == 0) bank[tid >> 6] = prefix;
      __syncthreads();
      bound = bank[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) bound = bank[w] < bound ? bank[w] : bound;
      if (bound != 0u) count_reach();
    }
    if (nreach > enough) {                                 // uniform: what counts is the same in every thread
      bound = smp_kth_largest<1>(tmax, top_k, red, phase, 16);
      count_reach();
    }
    if (bound != 0u && nreach > enough) {
      bound = smp_kth_largest<1>(tmax, top_k, red, phase, 0, 15, bound);
      count_reach();
    }
    if (bound != 0u && nreach <= SMP_THREADS) {
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        if (key[j] >= bound) {
          sk[at] = key[j];
          si[at] = base + j;
          ++at;
        }
      }
      __syncthreads();
      if (nreach <= SMP_THREADS / 4) return smp_ranked_pick<4>(sk, si, nreach, top_k, zmax, cfg->top_p, u, smp_z, found);
      if (nreach <= SMP_THREADS / 2) return smp_ranked_pick<2>(sk, si, nreach, top_k, zmax, cfg->top_p, u, smp_z, found);
      uint32_t k1[1] = {tid < nreach ? sk[tid] : 0u};
      float e1[1];
      const int id = tid < nreach ? si[tid] : 0;
      __syncthreads();
      smp_apply_topk<1>(k1, e1, top_k, zmax, red, phase);
      tok = smp_nucleus_and_draw<1>(k1, e1, id, cfg->top_p, u, red, phase, found);
      done = true;
    }
  }
  // (2) otherwise: the cut (if any), the nucleus and the draw over all slots of a thread
  if (!done) {
    float e[PER];
    smp_apply_topk<PER>(key, e, top_k, zmax, red, phase);
    tok = smp_nucleus_and_draw<PER>(key, e, base, cfg->top_p, u, red, phase, found);
  }
  return tok;
}

// Index of the largest value over a workgroup, the lowest index among equals (v: -inf where a thread has none), in every
// thread: lane-crossing moves inside a wave, and one barrier.  sv, si: a word per wave.  (A tree over LDS takes a
// barrier per level.)
__device__ __forceinline__ int smp_block_argmax(float v, int i, float* sv, int* si) {
  constexpr int NW = SMP_THREADS / 64;
  const int tid = threadIdx.x;
  auto over_rows = [](auto x, auto op) {          // the four rows of 16 lanes
    auto at = [&](int lane) { return __builtin_bit_cast(decltype(x), __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane)); };
    return op(op(at(0), at(16)), op(at(32), at(48)));
  };
  auto big = [](float a, float b) { return fmaxf(a, b); };
  auto low = [](int a, int b) { return a < b ? a : b; };
  float top = big(v, dpp_mov<0xB1>(v));
  top = big(top, dpp_mov<0x4E>(top));
  top = big(top, dpp_mov<0x141>(top));
  top = over_rows(big(top, dpp_mov<0x140>(top)), big);
  int at = v == top ? i : 0x7fffffff;
  at = low(at, __builtin_amdgcn_update_dpp(0, at, 0xB1, 0xf, 0xf, true));
  at = low(at, __builtin_amdgcn_update_dpp(0, at, 0x4E, 0xf, 0xf, true));
  at = low(at, __builtin_amdgcn_update_dpp(0, at, 0x141, 0xf, 0xf, true));
  at = over_rows(low(at, __builtin_amdgcn_update_dpp(0, at, 0x140, 0xf, 0xf, true)), low);
  if ((tid & 63) == 0) { sv[tid >> 6] = top; si[tid >> 6] = at; }
  __syncthreads();
  top = sv[0];
  at = si[0];
#pragma unroll
  for (int w = 1; w < NW; ++w)
    if (sv[w] > top || (sv[w] == top && si[w] < at)) { top = sv[w]; at = si[w]; }
  return at;
}

//   prefill = 1: pos += n_prompt (rows of the last prompt chunk), steps := 1, ring[0] := token (draw index 0)
//   prefill = 0: pos += 1, ring[steps] := token, steps += 1   (draw index = steps before the step)
// It also gathers the selected token's embedding row into x_next (when given), the input of the next
// decode step, which therefore needs no gather kernel of its own (what x_next held, the final residual
// stream of the step or of the prompt's last row, is kept in x_keep for the read-back hook); and it reports token -1 to the host
// when a kernel of the step raised DevState::fault (the device state still advances with a valid id).
//
// A slot costs some 15 instructions, used or not, with four waves to a SIMD, and what the 32 of a large vocabulary spill costs
// every launch: built for up to 1024, 8192 and SMP_MAX_VOCAB tokens (PER = 1, 8, SMP_PER).  A step of a toy model, us, with 32
// slots for all and loads behind the choice / now: vocabulary 1024 greedy 32.1 / 31.3, top-k 50 39.6 / 36.1, with top-p 0.95
// 40.0 / 36.6, top-p 0.95 alone 50.3 / 47.5; 4096 33.1 / 32.2, 42.1 / 39.3, 42.6 / 39.6, 79.1 / 56.3; 32000 41.0 / 40.1,
// 57.8 / 57.1, 58.8 / 58.1, 99.2 / 98.8.
template <int PER>
__global__ __launch_bounds__(SMP_THREADS) void sample_kernel(const float* __restrict__ pval,
                                                             const int* __restrict__ pidx, int nparts,
                                                             const float* __restrict__ logits, int vocab,
                                                             const SampleCfg* __restrict__ cfg,
                                                             DevState* st, int* host_ring, int ring_size,
                                                             int prefill, const half_t* __restrict__ emb,
                                                             float* __restrict__ x_next, float* __restrict__ x_keep,
                                                             int d) {
  extern __shared__ float smp_z[];     // SMP_Z_BYTES(PER), used by the stochastic path only
  __shared__ int si[SMP_THREADS];
  __shared__ uint32_t sk[SMP_THREADS];
  __shared__ float red[2 * 3 * (SMP_THREADS / 64)];
  __shared__ int found;
  const int tid = threadIdx.x;
  // Nothing the kernel reads depends on anything but the token's embedding row on the token: requested up front, a memory
  // round trip instead of one behind the other.
  const float inv_temp = cfg->inv_temp, logit0 = logits[min(tid, vocab - 1)];
  const int last = min(tid, nparts - 1), pos = st->pos, n_prompt = st->n_prompt, steps = st->steps, fault = st->fault;
  const float v0 = pval[last];
  const int i0 = pidx[last];
  int tok;
  // what the step leaves in x_next is kept (d <= SMP_THREADS * 8)
  if (x_next && tid * 8 < d) {
    *as_global(reinterpret_cast<f4*>(x_keep + tid * 8)) = *as_global(reinterpret_cast<const f4*>(x_next + tid * 8));
    *as_global(reinterpret_cast<f4*>(x_keep + tid * 8 + 4)) = *as_global(reinterpret_cast<const f4*>(x_next + tid * 8 + 4));
  }

  if (inv_temp == 0.f || vocab > SMP_THREADS * PER) {
    // ---- greedy: reduce the LM head's per-workgroup (max, lowest index) candidates
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    auto offer = [&](float v, int ix) {
      if (v > bv || (v == bv && ix < bi)) { bv = v; bi = ix; }
    };
    offer(v0, i0);                                  // (a thread without a candidate offers the last one again)
    for (int i = tid + SMP_THREADS; i < nparts; i += SMP_THREADS) offer(pval[i], pidx[i]);
    tok = smp_block_argmax(bv, bi, red, si);
    if ((unsigned)tok >= (unsigned)vocab) tok = 0;   // no candidate (every logit NaN): still a valid id
  } else {
    tok = smp_draw_token<PER>(logits, vocab, cfg, (uint32_t)(prefill ? 0 : steps), logit0, smp_z, si, sk, red, &found);
  }

  tok = __builtin_amdgcn_readfirstlane(tok);        // one value for every thread, whichever path chose it
  if (x_next && tid * 8 < d) {
    const h8 e = load_h8(emb + (size_t)tok * d + tid * 8);
    *as_global(reinterpret_cast<f4*>(x_next + tid * 8)) = f4{(float)e[0], (float)e[1], (float)e[2], (float)e[3]};
    *as_global(reinterpret_cast<f4*>(x_next + tid * 8 + 4)) = f4{(float)e[4], (float)e[5], (float)e[6], (float)e[7]};
  }

  if (tid == 0) {
    const int idx = prefill ? 0 : steps;
    st->pos = pos + (prefill ? n_prompt : 1);
    st->steps = idx + 1;
    st->next_token = tok;
    if (idx < ring_size) host_ring[idx] = fault ? -1 : tok;
  }
}
