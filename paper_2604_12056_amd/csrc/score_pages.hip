// QUEST page scoring, per-query top pages and their union per KV head
// (paper: Preliminaries, Sparse Attention Algorithms for LLMs; Methodology, eq. quest_union).
//
//   page_scores   s[b,j,r,p] = sum_c max(q_c*min_c, q_c*max_c)   r = a*G + hg over the active slots a
//   select_pages  per row r: exact top-K by radix select on order-preserving keys (ties:
//                 smaller page); picks go into a union bitmap per KV head, or, where the caller wants the
//                 list, the last row of a head to finish ORs the row bitmaps and compacts them into one
//
// Everything that decides a set is integer work on float bit patterns: no float atomics,
// so the outcome does not depend on scheduling.
#include "losa_device.h"
#include "losa_internal.h"

namespace losa {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// What the scoring kernel leaves ready for the launches that follow it: the ticket counter of every (sequence, KV
// head) at zero, an empty result when no token is active, so that no selection workgroup will run, and, where the
// attention kernel ranks the union itself, what that kernel wants at addresses it knows: the head's page table with
// every page's token count, and the gathered query rows (the scoring workgroups hold them anyway).
struct ScoreAux {
  int32_t* tickets;
  int32_t* sel_count;
  int32_t* entries;       // nullable: [heads, max_pages] physical page | valid tokens << kEntryShift, by logical page
  uint16_t* q_act;        // ... and [heads, rows_max, d]
  uint32_t* union_bits;   // nullable: union bitmaps, cleared here for the selection to OR into
  int union_stride;       // words per head ...
  int union_len;          // ... of which this launch uses so many
  // every thread of one workgroup per head
  __device__ void clear_union(int head) const {
    if (union_bits)
      for (int w = threadIdx.x; w < union_len; w += 256) union_bits[(size_t)head * union_stride + w] = 0u;
  }
  __device__ void reset(int head, int M) const {
    tickets[head] = 0;
    if (M <= 0) sel_count[head] = 0;
  }
};

// In-kernel locality pruning (paper: Methodology, Locality Pruning): when `delta` is given,
// every scoring workgroup ranks the block's locality scores itself (B <= kRankTokens, ranking by
// counting as in the stand-alone kernel) instead of reading an
// active list some earlier launch produced, and the first workgroup of each sequence writes
// mask / list / count out for the kernels that follow.  This replaces the hand-over at the end
// of the locality kernel (store, wait, ticket, reload, rank) by compares here: a quarter of the block per lane and
// wavefront for blocks of up to 64 tokens, the whole block per thread beyond.
constexpr int kRankTokens = 256;
constexpr int kMaxTilesPerWg = 4;   // 64-page tiles one scoring workgroup may take
struct RankArgs {
  const float* delta;     // [batch*B] locality scores; NULL: use the active list passed to the kernel
  int mode, n;            // LOSA_SEL_TOPK / FRACTION (n = count), LOSA_SEL_THRESHOLD or LOSA_SEL_MASS (tau)
  float tau;
  uint8_t* mask;          // outputs, written by workgroup (0, 0, b)
  int32_t* active_idx;
  int32_t* active_count;
};

// Active set of a block of up to 64 tokens, a lane per token, by every wavefront of a workgroup of NW: 1 in the lanes of its
// tokens.  The wavefronts each compare every token with their share of the block, the score compared
// with held in a scalar register, and meet once, in LDS; from the ranks on every wavefront works for itself: the
// active set is a lane mask, a token's place in the list the number of lanes below it, and every wavefront keeps its
// own copy of the list, so that no further barrier is needed.  With a thread per token, the scores in LDS, a scan and
// four barriers the ranking of 32 tokens took 1.55 of the scoring kernel's 7.1 us (2048 pages, 42 rows, 4 KV heads); that
// kernel now takes 5.7.
// ranks: NW * 64 ints of LDS; sorted: 64 floats for this wavefront alone.
template <int NW>
__device__ __forceinline__ int rank_small(const RankArgs& ra, int B, float my_delta, int lane, int wave, int* ranks, float* sorted) {
  const float score = ra.mode == LOSA_SEL_THRESHOLD ? my_delta : ranked_score(my_delta);
  const float mine = lane < B ? score : -INFINITY;   // the padding never outranks a token
  int rank = 0;
  if (ra.mode != LOSA_SEL_THRESHOLD) {
    const int per = (B + NW - 1) / NW, k0 = wave * per, k1 = min(k0 + per, B);
    for (int k = k0; k < k1; ++k) {
      const float dk = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(mine), k));
      rank += (int)(dk > mine) | ((int)(dk == mine) & (int)(k < lane));   // bitwise on purpose: no branches
    }
    ranks[wave * 64 + lane] = rank;
    __syncthreads();
    rank = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) rank += ranks[w * 64 + lane];
  }
  if (ra.mode != LOSA_SEL_MASS) return (lane < B) & (ra.mode == LOSA_SEL_THRESHOLD ? (int)(mine > ra.tau) : (int)(rank < ra.n));
  // Cumulative-mass rule, as in the stand-alone kernel: the scores in descending order are summed in that order in
  // float, here by all lanes at once: lane r adds the scores of ranks 0..r and zeros after them.  A token is in A if
  // the sum before it stays below tau * total (and total and tau are positive).
  if (lane < B) sorted[rank] = mine;
  wave_lds_fence();
  const float at_rank = sorted[min(lane, B - 1)];
  float prefix = 0.f;
  for (int k = 0; k < B; ++k) {
    const float dk = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(at_rank), k));
    prefix += k <= lane ? dk : 0.f;
  }
  const float total = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(prefix), B - 1));
  wave_lds_fence();
  sorted[lane] = prefix;
  wave_lds_fence();
  const int act = (lane < B) & (total > 0.f) & (ra.tau > 0.f) & ((rank == 0) | (int)(sorted[max(rank - 1, 0)] < ra.tau * total));
  wave_lds_fence();
  return act;
}

// Float mode.  A workgroup takes 8 pages and all rows of a KV head, a thread one page and two rows at a time,
// four channels per step out of LDS; the terms of a score are added in channel order.  With 8 pages per
// workgroup a prefix of a few thousand tokens fills the chip (with 32, a quarter of it); the two rows
// share what is read of the page.  501 pages x 4 KV heads x 42 rows: 22.5 -> 7.7 us, most of it three memory
// round trips.
constexpr int kScorePages = 8;   // pages per workgroup
constexpr int kScoreRows = 64;   // query rows staged at a time

template <int D>
__global__ __launch_bounds__(256) void page_scores_f32_kernel(KvView kv, Shape sh, const float* __restrict__ q,
                                                              const int32_t* __restrict__ active_idx,
                                                              const int32_t* __restrict__ active_count,
                                                              float* __restrict__ scores, ScoreAux aux) {
  constexpr int PT = kScorePages, RC = kScoreRows, VPR = D / 4, STR = D + 4;   // STR: 16 bytes of padding spread rows over the banks
  __shared__ __attribute__((aligned(16))) float mn[PT][STR];
  __shared__ __attribute__((aligned(16))) float mx[PT][STR];
  __shared__ __attribute__((aligned(16))) float qs[RC][STR];
  const int b = blockIdx.z, j = blockIdx.y, p0 = blockIdx.x * PT, tid = threadIdx.x;
  // Three dependent memory round trips (token ids and counts; query rows and page ids; metadata rows), not one
  // per step of the code: everything is requested, clamped, before what it depends on has been checked.
  constexpr int QV = RC * VPR / 256;       // query vectors per thread and staged chunk
  constexpr int MV = PT * 2 * VPR / 256;   // metadata vectors per thread
  static_assert(RC * VPR % 256 == 0 && PT * 2 * VPR % 256 == 0, "vectors do not split evenly over the threads");
  float4 qv[QV];
  int tok[QV];
  auto load_tokens = [&](int r0) {
#pragma unroll
    for (int k = 0; k < QV; ++k) tok[k] = active_idx[(size_t)b * sh.B + row_token(sh, min(r0 + (tid + 256 * k) / VPR, sh.rows_max - 1))];
  };
  auto load_queries = [&](int r0) {
#pragma unroll
    for (int k = 0; k < QV; ++k) {
      const int r = min(r0 + (tid + 256 * k) / VPR, sh.rows_max - 1), cv = (tid + 256 * k) % VPR;
      const int tc = (unsigned)tok[k] < (unsigned)sh.B ? tok[k] : 0;
      qv[k] = reinterpret_cast<const float4*>(q + (((size_t)b * sh.B + tc) * sh.Hq + j * sh.G + (r - row_token(sh, r) * sh.G)) * D)[cv];
    }
  };
  load_tokens(0);
  int n = __builtin_amdgcn_readfirstlane(active_count[b]);
  const Sequence seq = sequence(kv, sh, b);
  asm("" : "+s"(n) : "s"(seq.tokens), "s"(kv.page_indices), "s"(kv.meta), "s"(kv.num_pages), "s"(sh.Hkv), "s"(sh.B), "s"(sh.G), "s"(q));   // (see Sequence)
  const int base = seq.base, P = seq.pages, M = min(n, sh.B) * sh.G;
  if (p0 >= P || M <= 0) {
    if (blockIdx.x == 0 && tid == 0) aux.reset(b * sh.Hkv + j, M);
    return;
  }
  int phys[MV];
#pragma unroll
  for (int k = 0; k < MV; ++k) phys[k] = kv.page_indices[base + min(p0 + (tid + 256 * k) / (2 * VPR), P - 1)];
  load_queries(0);
  __builtin_amdgcn_sched_barrier(0);
  if (blockIdx.x == 0 && tid == 0) aux.reset(b * sh.Hkv + j, M);   // (behind the loads: a wait for one of them would be one for this store)
  float4 mv[MV];   // all requested before the first is waited for
#pragma unroll
  for (int k = 0; k < MV; ++k) {
    const int v = tid + 256 * k, rem = v % (2 * VPR), which = rem / VPR, cv = rem % VPR;
    const bool ok = (unsigned)phys[k] < (unsigned)kv.num_pages;
    mv[k] = reinterpret_cast<const float4*>((const float*)kv.meta + (((size_t)(ok ? phys[k] : 0) * sh.Hkv + j) * 2 + which) * D)[cv];
  }
#pragma unroll
  for (int k = 0; k < MV; ++k) {
    const int v = tid + 256 * k, pg = v / (2 * VPR), rem = v % (2 * VPR), which = rem / VPR, cv = rem % VPR;
    const bool ok = (unsigned)phys[k] < (unsigned)kv.num_pages;
    *reinterpret_cast<float4*>(which ? &mx[pg][cv * 4] : &mn[pg][cv * 4]) = ok ? mv[k] : make_float4(0.f, 0.f, 0.f, 0.f);
  }

  const int pg = tid % PT, rs = tid / PT;   // rows rs and rs + 32 of the staged ones
  for (int r0 = 0; r0 < M; r0 += RC) {
    const int rows = min(RC, M - r0);
    if (r0) {
      load_tokens(r0);
      load_queries(r0);
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < QV; ++k) {   // (rows past M: clamped copies nobody reads)
      const bool ok = (unsigned)tok[k] < (unsigned)sh.B;
      *reinterpret_cast<float4*>(&qs[(tid + 256 * k) / VPR][(tid + 256 * k) % VPR * 4]) = ok ? qv[k] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();
    if (rs >= rows) continue;
    const bool two = rs + 32 < rows;
    const int rs2 = two ? rs + 32 : rs;
    float s0 = 0.f, s1 = 0.f;
#pragma unroll 4
    for (int cv = 0; cv < VPR; ++cv) {
      const f32x4_t lo = *reinterpret_cast<const f32x4_t*>(&mn[pg][cv * 4]), hi = *reinterpret_cast<const f32x4_t*>(&mx[pg][cv * 4]);
      const f32x4_t q0 = *reinterpret_cast<const f32x4_t*>(&qs[rs][cv * 4]), q1 = *reinterpret_cast<const f32x4_t*>(&qs[rs2][cv * 4]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s0 += fmaxf(q0[e] * lo[e], q0[e] * hi[e]);
        s1 += fmaxf(q1[e] * lo[e], q1[e] * hi[e]);
      }
    }
    if (p0 + pg < P) {
      float* dst = scores + (((size_t)b * sh.Hkv + j) * sh.rows_max + r0) * sh.max_pages + p0 + pg;
      dst[(size_t)rs * sh.max_pages] = s0;
      if (two) dst[(size_t)(rs + 32) * sh.max_pages] = s1;
    }
  }
}

// Matrix-core page scoring for bfloat16.  Since max >= min per channel,
//   max(q*min, q*max) = q+ * max + q- * min      with q+ = max(q,0), q- = min(q,0),
// and one of the two terms is exactly zero, so each channel contributes the same exact
// product either way: the score matrix of a KV head is the dense contraction
//   S^T [pages x rows] = [max | min] (pages x 2d) . [Q+ | Q-]^T (2d x rows).
// A wavefront takes 16 pages: its A operands are the 16 metadata rows read straight from
// memory (one 16-byte load per lane and k-step, 8 KiB per wavefront all in flight at once);
// the B operands are the sign-split query fragments.  Output leaves the matrix core as 4
// consecutive pages per lane and query row: one 16-byte store.
template <int D, int MAXT>
__global__ __launch_bounds__(256) void page_scores_mfma_kernel(Address delta, Address page_indptr, Address seq_lens,
                                                               Address page_indices, Address meta, int block, int kv_heads, int num_pages,
                                                               int max_pages,
                                                               KvView kv, Shape sh, const bf16_t* __restrict__ q,
                                                               const int32_t* __restrict__ active_idx,
                                                               const int32_t* __restrict__ active_count,
                                                               float* __restrict__ scores, ScoreAux aux, RankArgs ra,
                                                               int tpw) {
  ra.delta = pointer<const float>(delta);   // (leading arguments: see KvView)
  kv.page_indptr = pointer<const int32_t>(page_indptr);
  kv.seq_lens = pointer<const int32_t>(seq_lens);
  kv.page_indices = pointer<const int32_t>(page_indices);
  kv.meta = pointer<void>(meta);
  kv.num_pages = num_pages;
  sh.B = block;
  sh.Hkv = kv_heads;
  sh.max_pages = max_pages;
  // A workgroup scores tpw (<= MAXT, a template argument so that the one-tile form carries no
  // code for more) consecutive 64-page tiles: what it does before
  // the first product (ranking, query staging) is then paid once for all of them, and a
  // batch of many sequences still fits the machine in one round of workgroups.
  const int bx = blockIdx.x * tpw, j = blockIdx.y, b = blockIdx.z, head = b * sh.Hkv + j;
  constexpr int KS = D / 32;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, qd = lane >> 4;
  const bool ranked = ra.delta != nullptr;   // uniform over the launch
  const bool small = sh.B <= 64;             // a lane per token: every wavefront holds the whole block's scores
  // Everything that can be fetched before the active set is known is requested first, the locality scores ahead of
  // all (their address needs kernel arguments only; behind the page counts they came 0.5 us later).
  float my_delta = 0.f;
  if (ranked) my_delta = ra.delta[(size_t)b * sh.B + min(small ? lane : tid, sh.B - 1)];
  const Sequence seq = sequence(kv, sh, b);
  const int base = seq.base, P = seq.pages, tokens = seq.tokens;
  const int p0 = bx * 64 + wave * 16;
  __shared__ __attribute__((aligned(16))) float sdelta[kRankTokens];
  __shared__ int act_list[kRankTokens];
  __shared__ int rscan[17];
  const bool first = bx == 0;                             // this workgroup leaves what belongs to the head
  const bool writes_active = ranked && first && j == 0;   // ... and this one publishes the active set
  auto tile_page = [&](int t) { return max(0, min((bx + t) * 64 + wave * 16 + l16, P - 1)); };
  auto tile_phys = [&](int t) {   // page whose metadata rows lane l16 feeds for tile t of this workgroup; -1: outside the pool
    const int ph = P > 0 ? kv.page_indices[base + tile_page(t)] : 0;
    return (unsigned)ph < (unsigned)kv.num_pages ? ph : -1;
  };
  if (bx * 64 >= P && !first) return;   // no pages here

  // Metadata rows of this wavefront's pages: two dependent round trips (page table, then the rows), which travel
  // while the ranking runs.  A operands: rows of page p0 + l16 (a valid page is read for lanes past P, never stored).
  // The page ids of all of this workgroup's tiles are fetched at once.
  int physv[MAXT];
#pragma unroll
  for (int t = 0; t < MAXT; ++t) physv[t] = t < tpw ? tile_phys(t) : 0;
  bf16x8_t amin[KS], amax[KS];
  auto load_meta = [&](int phys, bf16x8_t (&mn)[KS], bf16x8_t (&mx)[KS]) {
    const bf16_t* mrow = (const bf16_t*)kv.meta + ((size_t)max(phys, 0) * sh.Hkv + j) * 2 * D;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      mn[ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(mrow + ks * 32 + qd * 8));
      mx[ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(mrow + D + ks * 32 + qd * 8));
    }
  };
  load_meta(physv[0], amin, amax);

  int M;
  int list_at = 0;   // where this wavefront's copy of the active list starts in act_list
  if (ranked && small) {
    const int B = sh.B;
    const int act = rank_small<4>(ra, B, my_delta, lane, wave, reinterpret_cast<int*>(sdelta),
                                  reinterpret_cast<float*>(act_list) + wave * 64);   // (free until the list is written)
    const unsigned long long set = __ballot(act);
    const int n_act = __popcll(set);
    const int pos = __builtin_amdgcn_mbcnt_hi((unsigned)(set >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)set, 0));
    list_at = wave * 64;
    if (act) act_list[list_at + pos] = lane;
    wave_lds_fence();
    if (writes_active && wave == 0) {
      if (lane < B) ra.mask[(size_t)b * B + lane] = (uint8_t)act;
      if (act) ra.active_idx[(size_t)b * B + pos] = lane;
      if (lane >= n_act && lane < B) ra.active_idx[(size_t)b * B + lane] = -1;
      if (lane == 0) ra.active_count[b] = n_act;
    }
    M = n_act * sh.G;
  } else if (ranked) {
    const int B = sh.B;   // <= kRankTokens (checked by the launcher)
    if (ra.mode != LOSA_SEL_THRESHOLD) my_delta = ranked_score(my_delta);
    sdelta[tid] = tid < B ? my_delta : -INFINITY;   // 256 threads, kRankTokens entries: the padding never outranks a token
    __syncthreads();
    int act = 0, rank = 0;
    if (tid < B && ra.mode != LOSA_SEL_THRESHOLD) {
      // four scores per LDS read
#pragma unroll 1   // (unrolled, the compare masks of 16 scores spill scalar registers to scratch in every launch)
      for (int k = 0; k < B; k += 4) {
        const f32x4_t dk = *reinterpret_cast<const f32x4_t*>(&sdelta[k]);
#pragma unroll
        for (int e = 0; e < 4; ++e)   // bitwise on purpose: the short-circuit forms compile to a branch per element
          rank += (int)(dk[e] > my_delta) | ((int)(dk[e] == my_delta) & (int)(k + e < tid));
      }
    }
    if (ra.mode == LOSA_SEL_MASS) {
      // Cumulative-mass rule, as in the stand-alone kernel: prefix sums of the scores in descending order, taken
      // in that order in float by one thread; a token is in A if the sums before it stay below tau * total.
      __shared__ __attribute__((aligned(16))) float sorted[kRankTokens], prefix[kRankTokens];
      if (tid < B) sorted[rank] = my_delta;
      if (tid < ((4 - (B & 3)) & 3)) sorted[B + tid] = 0.f;
      __syncthreads();
      if (tid == 0) sorted_prefix_sums(sorted, prefix, B);
      __syncthreads();
      if (tid < B) act = mass_takes(prefix, rank, B, ra.tau);
    } else if (tid < B) {
      act = ra.mode == LOSA_SEL_THRESHOLD ? my_delta > ra.tau : rank < ra.n;
    }
    int n_act;
    const int pos = block_exclusive_scan(act, rscan, &n_act);
    if (act) act_list[pos] = tid;
    if (writes_active) {
      if (tid < B) ra.mask[(size_t)b * B + tid] = (uint8_t)act;
      if (act) ra.active_idx[(size_t)b * B + pos] = tid;
      for (int i = n_act + tid; i < B; i += 256) ra.active_idx[(size_t)b * B + i] = -1;
      if (tid == 0) ra.active_count[b] = n_act;
    }
    __syncthreads();   // act_list is read below
    M = n_act * sh.G;
  } else {
    M = min(active_count[b], sh.B) * sh.G;
  }
  if (first) aux.clear_union(head);
  if (first && tid == 0) aux.reset(head, M);
  if (bx * 64 >= P) return;   // whole workgroup (only a head's first one gets here without pages)
  if (M <= 0) return;

  float* out_base = scores + ((size_t)b * sh.Hkv + j) * sh.rows_max * sh.max_pages;

  // Query rows go through LDS, kRows at a time, so that the four wavefronts (64 pages) fetch
  // each row once instead of once per wavefront.  A row is D bfloat16 plus 16 bytes of padding:
  // the 16 lanes that read the same 16-byte column of 16 consecutive rows then fall on
  // different banks.
  const bool table = aux.entries && M <= kUnionRows;   // the attention kernel will want the page table
  constexpr int kRows = 64, VPR = D / 8, STRIDE = D * 2 + 16;   // bytes; 64 rows cover the usual active sets in one go; with 128 channels 38 KiB of LDS, four workgroups per CU
  // Staged already split by sign (score = q+ . max + q- . min): the split is done once per
  // workgroup by the staging threads, not once per wavefront, tile and row tile.
  __shared__ __attribute__((aligned(16))) unsigned char qs[2][kRows * STRIDE];   // [0]: q+, [1]: q-
  bool staged = false;   // LDS holds rows [0, kRows) of this head's active queries
#pragma unroll
  for (int t = 0; t < MAXT; ++t) {
    if (t >= tpw || (bx + t) * 64 >= P) break;   // uniform over the workgroup
    const int p0t = p0 + t * 64;
    const bool live = p0t < P;   // a wavefront without pages still helps staging and keeps the barriers
    const bool vec_ok = (sh.max_pages & 3) == 0 && p0t + 16 <= P;
    if (table && qd == 0 && p0t + l16 < P) {
      const int page = p0t + l16, nv = max(0, min(sh.g, tokens - page * sh.g));
      aux.entries[(size_t)head * sh.max_pages + page] = physv[t] >= 0 && physv[t] < (1 << kEntryShift) ? (physv[t] | (nv << kEntryShift)) : 0;
    }
    // the next tile's metadata rows travel while this tile is scored
    bf16x8_t nmin[KS], nmax[KS];
    if (t + 1 < MAXT && t + 1 < tpw) load_meta(physv[t + 1 < MAXT ? t + 1 : t], nmin, nmax);
    for (int r0 = 0; r0 < M; r0 += kRows) {
      const int nrows = min(kRows, M - r0);
      if (!(staged && M <= kRows)) {   // with a single chunk of rows the first tile's staging serves all tiles
        if (staged) __syncthreads();   // everyone is done reading the previous chunk
        // staging: thread -> (row, 16-byte vector); token ids first, then all the row loads
        constexpr int PER = kRows * VPR / 256;
        int tok[PER], grp[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
          const int r = r0 + min((tid + 256 * k) / VPR, nrows - 1), a = row_token(sh, r);
          grp[k] = r - a * sh.G;
          tok[k] = ranked ? act_list[list_at + a] : active_idx[(size_t)b * sh.B + a];
        }
        uint4 v[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
          const int cv = (tid + 256 * k) % VPR;
          const int tc = (unsigned)tok[k] < (unsigned)sh.B ? tok[k] : 0;
          v[k] = reinterpret_cast<const uint4*>(q + (((size_t)b * sh.B + tc) * sh.Hq + j * sh.G + grp[k]) * D)[cv];
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
          const int rr = (tid + 256 * k) / VPR, cv = (tid + 256 * k) % VPR;
          if (rr < nrows) {
            typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
            typedef int16_t i16x8_t __attribute__((ext_vector_type(8)));
            const uint32_t keep = (unsigned)tok[k] < (unsigned)sh.B ? 0xFFFFFFFFu : 0u;
            const u32x4_t x = u32x4_t{v[k].x, v[k].y, v[k].z, v[k].w} & keep;
            const u32x4_t mk = __builtin_bit_cast(u32x4_t, __builtin_bit_cast(i16x8_t, x) >> 15);   // all-ones where the sign bit is set
            *reinterpret_cast<u32x4_t*>(qs[0] + rr * STRIDE + cv * 16) = x & ~mk;
            *reinterpret_cast<u32x4_t*>(qs[1] + rr * STRIDE + cv * 16) = x & mk;
            if (t == 0 && first && table)
              *reinterpret_cast<u32x4_t*>(aux.q_act + ((size_t)head * sh.rows_max + r0 + rr) * D + cv * 8) = x;
          }
        }
        __syncthreads();
        staged = true;
      }
      if (!live) continue;
      for (int t0 = 0; t0 < nrows; t0 += 16) {
        const int rr = t0 + l16;           // row of this lane inside the chunk (may be past nrows: masked below)
        uint4 qpos[KS], qneg[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          qpos[ks] = *reinterpret_cast<const uint4*>(qs[0] + min(rr, nrows - 1) * STRIDE + ks * 64 + qd * 16);
          qneg[ks] = *reinterpret_cast<const uint4*>(qs[1] + min(rr, nrows - 1) * STRIDE + ks * 64 + qd * 16);
        }
        f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(amax[ks], __builtin_bit_cast(bf16x8_t, qpos[ks]), acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(amin[ks], __builtin_bit_cast(bf16x8_t, qneg[ks]), acc, 0, 0, 0);
        }
        // acc[e] = score of page p0t + 4*qd + e for query row r0 + t0 + l16
        if (rr < nrows) {
          float* dst = out_base + (size_t)(r0 + rr) * sh.max_pages + p0t + 4 * qd;
          if (vec_ok) {
            __builtin_nontemporal_store(acc, reinterpret_cast<f32x4_t*>(dst));
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (p0t + 4 * qd + e < P) dst[e] = acc[e];
          }
        }
      }
    }
    if (t + 1 < MAXT && t + 1 < tpw) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        amin[ks] = nmin[ks];
        amax[ks] = nmax[ks];
      }
    }
  }
}

// float -> uint32 whose unsigned order is the float order (-0 and +0 made equal first).
__device__ __forceinline__ uint32_t order_key(float f) {
  f += 0.0f;
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// What the selection kernel leaves behind: a union bitmap per (sequence, KV head) that its row workgroups OR their
// picks into, or (LIST) the union as an ascending page list: every row's workgroup stores its pick bitmap,
// then takes a ticket; the workgroup that draws the last ticket of a head ORs the rows, compacts
// the union.  (How the stores are made visible to that
// workgroup is described at the hand-over.)
struct SelectOut {
  int32_t* topk_out;    // nullable [batch, B, Hq, topk]
  int32_t* sel_pages;   // [batch, Hkv, cap] logical pages of the union, ascending
  int32_t* sel_count;   // [batch, Hkv]
  int cap;
  uint32_t* rowmaps;    // workspace [heads, rows_max, words]: pick bitmap of every query row
  int32_t* tickets;     // workspace [heads], zero on entry (zeroed by the scoring kernel), zero on exit
  // union_words() | words of a copy << 16 and (copies - 1) | row shift << 8; beside the pointer, so that they arrive with
  // it: fetched where they are used, they cost a scalar round trip (0.3 us)
  uint32_t union_shape, union_rows;
  uint32_t* union_bits; // non-NULL: rows only OR their picks into a copy of this bitmap
                        // ([heads, union_words()], cleared by the scoring kernel): no hand-over, no list
};

// A bucket of at most this many keys is ranked directly instead of by further histogram passes.
constexpr int kRankMax = 64, kRankBits = 6;

// LDS state of radix_kth.  hist and cand must be all zero when radix_kth is entered (radix_clear, called early; the
// first barrier inside radix_kth orders the clear before its first use).
template <int NT>
struct RadixLds {
  // one bucket and one candidate slot per lane behind the real ones take what does not count: an address per lane is
  // cheaper than a branch around the access
  __attribute__((aligned(16))) uint32_t hist[256 + 64];
  __attribute__((aligned(16))) uint32_t cand[kRankMax + 64];
  __attribute__((aligned(16))) uint32_t lo[NT / 64], hi[NT / 64];
  __attribute__((aligned(8))) uint32_t kth, next;
  int ncand;
};
template <int NT>
__device__ __forceinline__ void radix_clear(RadixLds<NT>& L) {
  if (threadIdx.x < 256) L.hist[threadIdx.x] = 0u;
  if (threadIdx.x < kRankMax) L.cand[threadIdx.x] = 0u;
}

// Radix select.  It runs on keys relative to the row's smallest key and starts at the highest
// bit of the row's largest one (a block min/max finds both), so the first histogram is already
// spread over many buckets instead of piling every key onto the few exponent patterns the
// scores share.  As soon as the bucket that holds the K-th key has at most kRankMax keys,
// those are copied to LDS and ranked against each other directly, which replaces the remaining histogram passes.
// Four barriers for a row that needs one histogram: extremes, histogram, candidates, K-th key.  What lies between
// them is done by every wavefront for itself where that saves a hand-over (the bucket search), and spread over the
// threads where it is long (a candidate is compared with the others by four threads).
//
// The K-th largest of the workgroup's keys (thread t holds key[0..nmine)), Kp < number of keys: on return the Kp
// largest are the keys >= kth, unless `cut`: then keys > kth are among them, and of the keys == kth, of which not all
// are, the first ones in page order.  On return the keys have been rebased (the row minimum subtracted); kth is
// in the same units.  Every thread of the workgroup must call it.
template <int E, int NT>
__device__ __forceinline__ void radix_kth(uint32_t (&key)[E], int nmine, int Kp, RadixLds<NT>& L, uint32_t& kth, bool& cut) {
  const int tid = threadIdx.x, lane = tid & 63;
  constexpr int NW = NT / 64;
  static_assert(NT >= 4 * kRankMax, "four threads per candidate");
  uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
  for (int i = 0; i < E; ++i) {
    lo = min(lo, i < nmine ? key[i] : 0xFFFFFFFFu);
    hi = max(hi, i < nmine ? key[i] : 0u);
  }
  lo = wave_min_u32(lo);
  hi = wave_max_u32(hi);
  if (lane == 0) {
    L.lo[tid >> 6] = lo;
    L.hi[tid >> 6] = hi;
  }
  if (tid == 0) {
    L.ncand = 0;
    L.next = 0xFFFFFFFFu;
  }
  __syncthreads();
  lo = L.lo[0];
  hi = L.hi[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) {
    lo = min(lo, L.lo[w]);
    hi = max(hi, L.hi[w]);
  }
  // Keys are taken relative to the row minimum from here on (order is unchanged): the
  // first digit then resolves the row's actual range into 128..256 buckets wherever that
  // range lies, instead of splitting at whatever power of two happens to fall inside it.
#pragma unroll
  for (int i = 0; i < E; ++i) key[i] -= lo;   // entries past the row's pages are never looked at
  hi = __builtin_amdgcn_readfirstlane(hi - lo);
  kth = 0u;
  cut = true;
  if (hi == 0u) return;                        // every key is the same
  const int hb = 31 - __clz((int)hi);          // no key has a bit above hb
  uint32_t pmask = hb >= 31 ? 0u : ~((2u << hb) - 1u), prefix = 0u;
  int need = Kp;
  bool first_pass = true;   // the histogram was cleared by the caller (a barrier has passed since)
  for (int shift = max(hb - 7, 0);; shift = max(shift - 8, 0)) {
    if (!first_pass) {
      __syncthreads();   // everyone has read the previous pass's histogram
      if (tid < 256) L.hist[tid] = 0u;
      __syncthreads();
    }
    first_pass = false;
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const bool in = (i < nmine) & ((key[i] & pmask) == prefix);
      atomicAdd(&L.hist[in ? (key[i] >> shift) & 255u : 256u + lane], 1u);
    }
    __syncthreads();
    // Every wavefront finds the bucket where the running count from the top first reaches `need`: lane l owns buckets
    // 255-4l .. 252-4l (descending), the lane that crosses tells the others.
    const uint4 c4 = *reinterpret_cast<const uint4*>(&L.hist[252 - 4 * lane]);
    const int c[4] = {(int)c4.w, (int)c4.z, (int)c4.y, (int)c4.x};
    const int tot = (c[0] + c[1]) + (c[2] + c[3]);
    const int incl = wave_inclusive_scan(tot);
    int above = incl - tot;   // keys in buckets owned by lower lanes (= higher buckets)
    int bucket = 255 - 4 * lane, size = c[0];
#pragma unroll
    for (int k = 1; k < 4; ++k) {   // step down while the bucket does not reach `need`
      const bool below = above + size < need;
      above += below ? size : 0;
      bucket -= below;
      size = below ? c[k] : size;
    }
    const int at = __builtin_ctzll(__ballot(incl >= need));   // the last lane's count covers every key: never empty
    const uint32_t found = (uint32_t)__builtin_amdgcn_readlane(bucket, at);
    const int count = __builtin_amdgcn_readlane(size, at);
    need -= __builtin_amdgcn_readlane(above, at);
    // bits of the digit that lie above bit hb (only when hb < 7) are common to all keys
    const uint32_t dmask = 0xFFu << shift;
    prefix = (prefix & ~dmask) | (found << shift);
    pmask |= dmask;
    if (shift == 0) {
      kth = prefix;
      cut = count != need;
      return;
    }
    if (count <= kRankMax) {
      // The K-th key is the need-th largest of `count` candidates: rank them directly.  A candidate is the key's bits
      // below the digit (at most 24) over its slot number, so no two are equal and one compare ranks them.
      // They are packed wavefront by wavefront (one LDS atomic each); which slots equal keys get does not matter.
      int mine_n = 0;
#pragma unroll
      for (int i = 0; i < E; ++i) mine_n += (int)(i < nmine) & (int)((key[i] & pmask) == prefix);
      const int wincl = wave_inclusive_scan(mine_n);
      int wbase = 0;
      if (lane == 63) wbase = atomicAdd(&L.ncand, wincl);
      wbase = __builtin_amdgcn_readlane(wbase, 63);
      int put = wbase + wincl - mine_n;
#pragma unroll
      for (int i = 0; i < E; ++i) {
        const int in = (int)(i < nmine) & (int)((key[i] & pmask) == prefix);
        L.cand[in ? put : kRankMax + lane] = (key[i] & ~pmask) << kRankBits | (uint32_t)(put & (kRankMax - 1));
        put += in;
      }
      __syncthreads();
      // thread -> a candidate and a quarter of those it is compared with (unused slots are 0: above none of them)
      if (tid < 4 * kRankMax) {
        const int which = tid >> 2, quarter = tid & 3;
        const uint32_t mine = L.cand[which];
        int rank = 0;
#pragma unroll
        for (int k = 0; k < kRankMax / 16; ++k) {
          const uint4 o = *reinterpret_cast<const uint4*>(&L.cand[quarter * 4 + k * 16]);
          rank += (int)(o.x > mine) + (int)(o.y > mine) + (int)(o.z > mine) + (int)(o.w > mine);
        }
        rank += dpp_quad_xor<1>(rank);
        rank += dpp_quad_xor<2>(rank);
        if (which < count && rank == need - 1) L.kth = mine >> kRankBits;
        if (which < count && rank == need) L.next = mine >> kRankBits;
      }
      __syncthreads();
      const uint32_t low = L.kth;
      kth = prefix | low;
      cut = L.next == low;   // the next one, not among the Kp, has the same key
      return;
    }
  }
}

// Per-query top pages, register resident (thread t of NT owns the E consecutive pages
// [t*E, t*E+E); P <= NT*E: 256 threads x 8 up to 2048 pages, 512 up to 4096, 1024 threads x 8 or 16 beyond).
// LIST: the union list instead of a bitmap (SelectOut).
// 2048 pages, 42 rows x 4 heads: 5.3 -> 4.5 us (before: histogram and candidates behind branches, a candidate ranked by
// one thread, picks through LDS); 4096 pages, 9.2 us with 1024 threads and 5.7 with 512.  The query rows and the page
// table, which a workgroup of this launch per head used to gather, come from the scoring kernel.
template <int E, int NT, bool MULTI, bool LIST>
__global__ __launch_bounds__(NT) void select_pages_kernel(const float* __restrict__ scores, const int32_t* __restrict__ active_count,
                                                           Address page_indptr, Address seq_lens, int kv_heads, int rows_max,
                                                           int max_pages, int rows_known, KvView kv, Shape sh, int topk, SelectOut out, int rpw) {
  kv.page_indptr = pointer<const int32_t>(page_indptr);   // (leading arguments: see KvView)
  kv.seq_lens = pointer<const int32_t>(seq_lens);
  sh.Hkv = kv_heads;
  sh.rows_max = rows_max;
  sh.max_pages = max_pages;
  // A workgroup selects for up to rpw query rows, one after the other (the next row's
  // scores travel while the current row is selected).  rpw is 1 until further workgroups cost more than further
  // rows (launch_select_pages says where).
  // MULTI = false is the one-row form (rpw == 1) without the loop's register cost.
  constexpr int WORDS = NT * E / 32;
  constexpr int TPW = 32 / E;           // threads whose pages share a bitmap word
  __shared__ RadixLds<NT> rl;
  __shared__ int scan[17];
  // A workgroup's rows are r_first, r_first + r_step, ...: dealt round-robin over the row workgroups, so
  // that when the grid was sized for more rows than exist (a count only the device knows) the rows
  // that do exist still spread over as many workgroups as possible.
  const int r_step = MULTI ? (int)gridDim.x : 1;
  const int r_first = blockIdx.x, j = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
  const int head = b * sh.Hkv + j;
  const int p_first_all = tid * E;
  const int p_first = p_first_all;
  // When the host knows the row count (rows_known: every workgroup of the grid has a row), the row's
  // scores are fetched before anything else: the address depends on kernel arguments only,
  // so these loads travel together with the loads of the counts below (entries past the
  // sequence's pages are masked later).  Otherwise they wait until the row is known to exist.
  float raw[E];
  auto load_row = [&](float (&dst)[E], int r) {   // thread t: pages [t*E, t*E+E), 32 or 64 contiguous bytes
    const float* row = scores + ((size_t)head * sh.rows_max + min(r, sh.rows_max - 1)) * sh.max_pages;
    if (p_first + E <= sh.max_pages && (sh.max_pages & 3) == 0) {
#pragma unroll
      for (int i = 0; i < E; i += 4) {
        const f32x4_t v = *reinterpret_cast<const f32x4_t*>(row + p_first + i);
        dst[i] = v[0];
        dst[i + 1] = v[1];
        dst[i + 2] = v[2];
        dst[i + 3] = v[3];
      }
    } else {
#pragma unroll
      for (int i = 0; i < E; ++i) dst[i] = row[min(p_first + i, sh.max_pages - 1)];
    }
  };
  if (rows_known) load_row(raw, r_first);
  int n_act = active_count[b];
  const Sequence seq = sequence(kv, sh, b);
  asm("" : "+s"(n_act) : "s"(seq.tokens), "s"(sh.B), "s"(sh.G), "s"(topk), "s"(out.union_bits), "s"(out.union_shape), "s"(out.union_rows));   // (see Sequence)
  const int P = min(seq.pages, NT * E);   // (the launcher picks NT * E >= the page limit)
  const int M = min(n_act, sh.B) * sh.G;
  if (r_first >= M) return;
  if (!rows_known) load_row(raw, r_first);
  const int words = (sh.max_pages + 31) / 32;
  const int Kp = min(topk, P);
  const int nmine_all = max(0, min(E, P - p_first));   // pages of this thread that exist
  // LDS that must start at zero is cleared now, while the scores are still on their way
  radix_clear(rl);
  const int r_end = MULTI ? M : r_first + 1;
#pragma unroll 1
  for (int r = r_first; r < r_end; r += r_step) {
    // Per-thread constants are made opaque once per row: otherwise everything derived from them
    // (bit masks, predicates, addresses) is computed once ahead of the loop and kept in registers
    // across it, which costs half the kernel's occupancy.
    int p_first_r = p_first_all, nmine_r = nmine_all;
    if constexpr (MULTI) asm volatile("" : "+v"(p_first_r), "+v"(nmine_r));
    const int p_first = p_first_r, nmine = nmine_r;
    int32_t* tk = nullptr;
    if constexpr (LIST) {
      const int a = row_token(sh, r), h = j * sh.G + r - a * sh.G;
      if (out.topk_out) tk = out.topk_out + (((size_t)b * sh.B + a) * sh.Hq + h) * topk;
    }
    uint32_t key[E];
#pragma unroll
    for (int i = 0; i < E; ++i) key[i] = i < nmine ? order_key(raw[i]) : 0u;
    if (r + r_step < r_end) load_row(raw, r + r_step);   // the next row's scores, on their way during this row's selection

    // Picks: keys from the K-th up; where not all keys equal to it are picked, the first of them in page order.
    const bool all = Kp >= P;   // (Kp covers every page: nothing to find)
    uint32_t kth = 0u, bits = 0u;
    bool cut = false;
    if (!all) radix_kth<E, NT>(key, nmine, Kp, rl, kth, cut);
    if (cut) {   // block-uniform: derives from LDS values every thread read
      int my_gt = 0, my_eq = 0;
#pragma unroll
      for (int i = 0; i < E; ++i) {
        my_gt += (int)(i < nmine) & (int)(key[i] > kth);
        my_eq += (int)(i < nmine) & (int)(key[i] == kth);
      }
      int gt_total, eq_total;
      block_exclusive_scan(my_gt, scan, &gt_total);
      int eq_rank = block_exclusive_scan(my_eq, scan, &eq_total);
#pragma unroll
      for (int i = 0; i < E; ++i) {
        const int eq = key[i] == kth;
        bits |= (uint32_t)((int)(key[i] > kth) | (eq & (int)(eq_rank < Kp - gt_total))) << i;
        eq_rank += eq;   // (only the pages past the row's last come behind one that does not exist)
      }
    } else {
#pragma unroll
      for (int i = E - 1; i >= 0; --i) bits = bits + bits + (uint32_t)(key[i] >= kth);
      if (all) bits = ~0u;
    }
    bits &= (1u << nmine) - 1u;   // nmine <= E <= 16
    if (tk) {
      int total;
      int pos = block_exclusive_scan(__popc(bits), scan, &total);
#pragma unroll
      for (int i = 0; i < E; ++i)
        if ((bits >> i) & 1u) tk[pos++] = p_first + i;
      for (int k = total + tid; k < topk; k += NT) tk[k] = -1;
    }
    // the threads that share a word put it together with lane moves; the first of them writes it out
    bits <<= p_first & 31;
    bits |= (uint32_t)dpp_quad_xor<1>((int)bits);
    if constexpr (TPW == 4) bits |= (uint32_t)dpp_quad_xor<2>((int)bits);
    static_assert(TPW == 2 || TPW == 4, "a word's threads are lanes of one quad");
    const int word = p_first >> 5;
    const bool writes = tid % TPW == 0;
    if constexpr (!LIST) {
      // read by the next launch; nothing waits for the atomics here (an OR has no order)
      uint32_t* u = out.union_bits + (size_t)head * (out.union_shape & 0xFFFF) +
                    ((r >> (out.union_rows >> 8)) & (int)(out.union_rows & 0xFF)) * (int)(out.union_shape >> 16);
      if (writes && bits) __hip_atomic_fetch_or(&u[word], bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // (bits: a page < P)
    } else {
      // ---- hand-over: the last row of this (sequence, head) builds the union.
      // The row bitmap travels in agent-scope atomic stores (written through to memory, past the
      // per-die L2 slices); ordering is "my stores have completed (wait count zero), then my
      // ticket".  A full agent-scope fence would also work but writes back and invalidates whole
      // L2 slices, once per workgroup.
      uint32_t* myrow = out.rowmaps + ((size_t)head * sh.rows_max + r) * words;
      if (writes && word < words) __hip_atomic_store(&myrow[word], bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      for (int w = WORDS + tid; w < words; w += NT) __hip_atomic_store(&myrow[w], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (r + r_step < r_end) {
      // clear the LDS state of the next row (this row's last reads of it lie behind the barrier); the next row's
      // first barrier (inside radix_kth) orders these writes
      __syncthreads();
      radix_clear(rl);
    }
  }
  if constexpr (LIST) {
    const int rows_done = (r_end - 1 - r_first) / r_step + 1;
    __shared__ int s_last;
    __shared__ uint32_t ubits[WORDS];     // union of the head's rows
    for (int w = tid; w < WORDS; w += NT) ubits[w] = 0u;
    __builtin_amdgcn_s_waitcnt(0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __syncthreads();
    // the ticket counts rows: the workgroup whose rows complete the head's M builds the union
    if (tid == 0)
      s_last = __hip_atomic_fetch_add(&out.tickets[head], rows_done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + rows_done == M;
    __syncthreads();
    if (!s_last) return;
    if (tid == 0) out.tickets[head] = 0;
    // Union of the M row bitmaps -> ascending page list.
    // Pages are handled a thread each, E per thread.  A page's slot in the list is the popcount prefix of its bitmap
    // word plus the set bits below it in the word: no serial walk, stores ascend with the thread id.
    const int wordsP = (P + 31) / 32;
    int32_t* sel = out.sel_pages + (size_t)head * out.cap;
    __shared__ int wordbase[WORDS];
    const uint32_t* maps = out.rowmaps + (size_t)head * sh.rows_max * words;
    {
      // Thread t ORs bitmap word (t mod nw) of every `groups`-th row in registers, 16 independent
      // loads at a time (a loop of load-then-use would pay one memory latency per iteration),
      // and only the per-thread results meet in LDS.  Agent-scope atomic loads: they are served
      // from the coherence point, not from a line this compute unit or its die's L2 holds.  The
      // writers' stores went through to memory (agent scope) and had completed before their
      // tickets were drawn, but the bitmap regions of two (sequence, head) pairs can share a
      // cache line (rows * words * 4 need not be a multiple of the line), and the union
      // workgroup of the other pair may have fetched that line while this pair's rows were
      // still being written.
      for (int w0 = 0; w0 < wordsP; w0 += NT) {
        const int nw = min(NT, wordsP - w0);
        const int groups = NT / nw;
        const int ww = w0 + tid % nw, rg = tid / nw;
        if (rg < groups) {
          uint32_t acc = 0u;
          for (int r0 = rg; r0 < M; r0 += groups * 16) {
            uint32_t v[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
              const int rr = r0 + groups * k;
              v[k] = __hip_atomic_load(&maps[(size_t)min(rr, M - 1) * words + ww], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (int k = 0; k < 16; ++k) acc |= (r0 + groups * k < M) ? v[k] : 0u;
          }
          if (acc) atomicOr(&ubits[ww], acc);
        }
      }
    }
    __syncthreads();
    int base_out = 0;
    for (int w0 = 0; w0 < WORDS; w0 += NT) {   // exclusive popcount prefix per word
      const int w = w0 + tid;
      const int c = w < wordsP ? __popc(ubits[w]) : 0;
      int total;
      const int ex = block_exclusive_scan(c, scan, &total);
      if (w < WORDS) wordbase[w] = base_out + ex;
      base_out += total;
    }
    __syncthreads();
    // Every load of this thread has landed by now; saying so keeps the stores below from each
    // waiting for the one before it (loads and stores share one in-order counter).
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0) only
    uint32_t wd[E];
    int wb[E];
#pragma unroll
    for (int i = 0; i < E; ++i) {   // all LDS reads first: one latency, not one per page
      wd[i] = ubits[(tid + NT * i) >> 5];
      wb[i] = wordbase[(tid + NT * i) >> 5];
    }
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const int page = tid + NT * i;
      if (page < P && ((wd[i] >> (page & 31)) & 1u)) {
        const int at = wb[i] + __popc(wd[i] & ((1u << (page & 31)) - 1u));
        if (at < out.cap) sel[at] = page;
      }
    }
    const int U = min(base_out, out.cap);
    if (tid == 0) out.sel_count[head] = U;
  }
}

// One page set per (sequence, KV head) shared by all of its active queries (not in the paper:
// the other reading of a per-KV-head budget): every page takes the largest bound any active
// query of the head gives it, and the K best pages are kept, so exactly min(K, P) pages are
// read.  One workgroup per (sequence, head): the row maxima are taken in registers on the
// order-preserving keys (the same pages-per-thread layout as select_pages_kernel), the K-th
// is found by the same radix select, and the list is emitted in ascending page order by a
// prefix sum over the threads' pick counts - no hand-over between workgroups is needed.
template <int E, int NT>
__global__ __launch_bounds__(NT) void shared_select_kernel(KvView kv, Shape sh, const int32_t* __restrict__ active_count,
                                                            const float* __restrict__ scores, int topk,
                                                            int32_t* __restrict__ sel_pages,
                                                            int32_t* __restrict__ sel_count, int cap) {
  __shared__ RadixLds<NT> rl;
  __shared__ int scan[17];
  const int j = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const int head = b * sh.Hkv + j;
  const int p_first = tid * E;
  radix_clear(rl);
  const int M = min(active_count[b], sh.B) * sh.G;
  const int P = min(seq_pages(kv, sh, b), NT * E);
  if (M <= 0 || P <= 0) {
    if (tid == 0) sel_count[head] = 0;
    return;
  }
  const int nmine = max(0, min(E, P - p_first));
  const bool vec = p_first + E <= sh.max_pages && (sh.max_pages & 3) == 0;
  const float* rows = scores + (size_t)head * sh.rows_max * sh.max_pages;
  uint32_t key[E];
#pragma unroll
  for (int i = 0; i < E; ++i) key[i] = 0u;
  constexpr int RB = E >= 16 ? 2 : 4;   // rows in flight (fewer with more keys per thread: 128 registers at 1024 threads)
  for (int r0 = 0; r0 < M; r0 += RB) {
    float v[RB][E];
#pragma unroll
    for (int rr = 0; rr < RB; ++rr) {
      const float* row = rows + (size_t)min(r0 + rr, M - 1) * sh.max_pages;   // clamped: the repeat changes no maximum
      if (vec) {
#pragma unroll
        for (int i = 0; i < E; i += 4) {
          const float4 x = *reinterpret_cast<const float4*>(row + p_first + i);
          v[rr][i] = x.x;
          v[rr][i + 1] = x.y;
          v[rr][i + 2] = x.z;
          v[rr][i + 3] = x.w;
        }
      } else {
#pragma unroll
        for (int i = 0; i < E; ++i) v[rr][i] = row[min(p_first + i, sh.max_pages - 1)];
      }
    }
#pragma unroll
    for (int rr = 0; rr < RB; ++rr)
#pragma unroll
      for (int i = 0; i < E; ++i) key[i] = max(key[i], order_key(v[rr][i]));
  }
#pragma unroll
  for (int i = 0; i < E; ++i)
    if (i >= nmine) key[i] = 0u;

  const int Kp = min(topk, P);
  const bool all = Kp >= P;
  uint32_t kth = 0u;
  bool cut = false;
  if (!all) radix_kth<E, NT>(key, nmine, Kp, rl, kth, cut);

  int my_eq = 0, my_gt = 0;
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const bool in = i < nmine;
    my_gt += in && (all || key[i] > kth);
    my_eq += in && !all && key[i] == kth;
  }
  int tot_gt, tot_eq, eq_rank = 0;
  block_exclusive_scan(my_gt, scan, &tot_gt);
  const int need = Kp - tot_gt;   // keys equal to the K-th that are kept
  if (cut) eq_rank = block_exclusive_scan(my_eq, scan, &tot_eq);
  const int mine = my_gt + (cut ? max(0, min(my_eq, need - eq_rank)) : my_eq);
  int total;
  int pos = block_exclusive_scan(mine, scan, &total);
  int32_t* sel = sel_pages + (size_t)head * cap;
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const bool in = i < nmine;
    bool take = in && (all || key[i] > kth);
    if (in && !all && key[i] == kth) {
      take = !cut || eq_rank < need;
      ++eq_rank;
    }
    if (take) {
      if (pos < cap) sel[pos] = p_first + i;
      ++pos;
    }
  }
  if (tid == 0) sel_count[head] = min(total, cap);
}

// Scoring and selection in one launch, for prefixes of up to kPickPages pages.  A workgroup of 16 wavefronts takes 16 query
// rows of a KV head and every page of the sequence: it ranks the locality scores (as the scoring kernel does), scores
// all pages for its rows on the matrix cores, a wavefront per 16 pages, leaves the scores in LDS and selects a row per
// wavefront out of them.  No score matrix in memory, one launch less, and no atomics: the rows' union is put
// together in LDS and stored as the copy of the head's bitmap that belongs to the 16 rows.
// A step of 42 rows x 4 heads over 128 pages 24.2 -> 22.1 us, of 128 rows x 128 heads 98 -> 78, with the locality scores (8 rows x 1 head,
// 64 channels) 18.3 -> 16.3; where the line to the separate launches lies stands at pick_pages_serves.
// What bounds it: the dependent round trips (locality scores; query rows beside page ids and metadata rows) and, as pages
// grow, one compute unit taking all of a head's metadata (256 KiB at 512 pages and 128 channels), which is why longer
// prefixes keep the two launches.
// A row is selected by one wavefront without LDS: page 64*i + lane is key i of a lane; the K-th key is found bit by bit
// from the highest in which the row's keys differ from its smallest, the count of keys that reach the candidate coming from scalar
// population counts of the compares, until exactly K keys do (some 12 of up to 32 steps); the compares' lane masks then are the
// row's bitmap as it stands.
// The locality scores too, for hidden states of up to 64 16-byte pieces (h_cur given): a wavefront per token, sums in the order
// of the locality kernel's, whose three other wavefronts have nothing then.
template <int D, int TPW>   // TPW: 16-page tiles per wavefront
__global__ __launch_bounds__(1024) void pick_pages_kernel(Address delta, Address hidden_cur, Address hidden_prev, Address page_indptr, Address seq_lens,
                                                          int block, int hidden, KvView kv, Shape sh,
                                                          const bf16_t* __restrict__ q, ScoreAux aux, RankArgs ra, int topk) {
  ra.delta = pointer<const float>(delta);   // (leading arguments: see KvView)
  kv.page_indptr = pointer<const int32_t>(page_indptr);
  kv.seq_lens = pointer<const int32_t>(seq_lens);
  sh.B = block;
  sh.H = hidden;
  const bf16_t *h_cur = pointer<const bf16_t>(hidden_cur), *h_prev = pointer<const bf16_t>(hidden_prev);
  constexpr int NW = 16, KS = D / 32, VPR = D / 8, STRIDE = D * 2 + 16;
  constexpr int NP = NW * 16 * TPW, ROW = NP + 4;   // pages; floats per row of scores in LDS (the writes of 16 rows spread over the banks)
  constexpr int E = NP / 64, COPY = 16;             // keys per lane; words of a copy of the union bitmap
  static_assert(NP / 32 <= COPY && kUnionSpread / COPY * kPickRows == kPickMostRows, "a copy of the bitmap holds a row's, and there is one for every 16 rows");
  __shared__ __attribute__((aligned(16))) float sc[kPickRows * ROW];
  __shared__ __attribute__((aligned(16))) unsigned char qs[2][kPickRows * STRIDE];   // [0]: q+, [1]: q-
  __shared__ int ranks[NW * 64], act_list[NW * 64];
  __shared__ float sdelta[64];
  __shared__ uint32_t uw[COPY];
  const int rt = blockIdx.x, j = blockIdx.y, b = blockIdx.z, head = b * sh.Hkv + j, r0 = rt * kPickRows;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, qd = lane >> 4;
  const int B = sh.B;   // <= 64 (checked by the launcher)
  float my_delta = 0.f;
  uint4 hx[4], hy[4];
  const int nvec = sh.H / 8;
  if (h_cur) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const size_t at = ((size_t)b * B + min(wave + NW * k, B - 1)) * nvec + min(lane, nvec - 1);
      hx[k] = reinterpret_cast<const uint4*>(h_cur)[at];
      hy[k] = reinterpret_cast<const uint4*>(h_prev)[at];
    }
  } else {
    my_delta = ra.delta[(size_t)b * B + min(lane, B - 1)];
  }
  Sequence seq = sequence(kv, sh, b);
  asm("" : "+s"(seq.base) : "s"(kv.page_indices), "s"(kv.meta), "s"(kv.num_pages), "s"(sh.Hkv));   // (see Sequence)
  const int base = seq.base, P = min(seq.pages, NP), tokens = seq.tokens;
  int phys[TPW];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {   // the page whose metadata rows lane l16 feeds; -1: outside the pool
    const int ph = P > 0 ? kv.page_indices[base + max(0, min((wave + NW * t) * 16 + l16, P - 1))] : 0;
    phys[t] = (unsigned)ph < (unsigned)kv.num_pages ? ph : -1;
  }
  bf16x8_t amin[TPW][KS], amax[TPW][KS];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    if ((wave + NW * t) * 16 >= P) break;   // uniform over the wavefront
    const bf16_t* mrow = (const bf16_t*)kv.meta + ((size_t)max(phys[t], 0) * sh.Hkv + j) * 2 * D;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      amin[t][ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(mrow + ks * 32 + qd * 8));
      amax[t][ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(mrow + D + ks * 32 + qd * 8));
    }
  }
  if (tid < COPY) uw[tid] = 0u;
  if (h_cur) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float fx[8], fy[8], part = 0.f;
      widen16(hx[k], fx, bf16_t());
      widen16(hy[k], fy, bf16_t());
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float df = fx[e] - fy[e];
        part = fmaf(df, df, part);
      }
      const float sum = wave_sum(lane < nvec ? part : 0.f);
      if (lane == 0 && wave + NW * k < B) sdelta[wave + NW * k] = sum / (float)sh.H;
    }
    __syncthreads();
    my_delta = sdelta[min(lane, B - 1)];
  }

  // ---- active set; every wavefront holds it as a lane mask and keeps a list of its own
  int* list = act_list + wave * 64;
  const int act = rank_small<NW>(ra, B, my_delta, lane, wave, ranks, reinterpret_cast<float*>(list));
  const unsigned long long set = __ballot(act);
  const int n_act = __popcll(set), M = n_act * sh.G;
  const int pos = __builtin_amdgcn_mbcnt_hi((unsigned)(set >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)set, 0));
  if (act) list[pos] = lane;
  wave_lds_fence();
  if (rt == 0 && j == 0 && wave == 0) {
    if (lane < B) ra.mask[(size_t)b * B + lane] = (uint8_t)act;
    if (act) ra.active_idx[(size_t)b * B + pos] = lane;
    if (lane >= n_act && lane < B) ra.active_idx[(size_t)b * B + lane] = -1;
    if (lane == 0) ra.active_count[b] = n_act;
  }
  if (rt == 0 && tid == 0) aux.reset(head, M);
  const int nrows = min(kPickRows, M - r0);   // (of this workgroup; none: zero copies)
  const bool table = M <= kUnionRows;         // the attention kernel will want the page table and the rows

  if (nrows > 0 && P > 0) {   // uniform over the workgroup
    if (tid < kPickRows * VPR) {
      const int rr = tid / VPR, cv = tid % VPR, r = r0 + min(rr, nrows - 1), a = row_token(sh, r);
      const uint4 v = reinterpret_cast<const uint4*>(q + (((size_t)b * B + list[a]) * sh.Hq + j * sh.G + (r - a * sh.G)) * D)[cv];
      typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
      typedef int16_t i16x8_t __attribute__((ext_vector_type(8)));
      const u32x4_t x = {v.x, v.y, v.z, v.w};
      const u32x4_t mk = __builtin_bit_cast(u32x4_t, __builtin_bit_cast(i16x8_t, x) >> 15);   // all-ones where the sign bit is set
      *reinterpret_cast<u32x4_t*>(qs[0] + rr * STRIDE + cv * 16) = x & ~mk;
      *reinterpret_cast<u32x4_t*>(qs[1] + rr * STRIDE + cv * 16) = x & mk;
      if (table && rr < nrows) *reinterpret_cast<u32x4_t*>(aux.q_act + ((size_t)head * sh.rows_max + r) * D + cv * 8) = x;
    }
    if (rt == 0 && table && qd == 0) {
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        const int page = (wave + NW * t) * 16 + l16, nv = max(0, min(sh.g, tokens - page * sh.g));
        if (page < P)
          aux.entries[(size_t)head * sh.max_pages + page] = phys[t] >= 0 && phys[t] < (1 << kEntryShift) ? (phys[t] | (nv << kEntryShift)) : 0;
      }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      const int p0 = (wave + NW * t) * 16;
      if (p0 >= P) break;   // uniform over the wavefront
      f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {   // (the same products in the same order as the scoring kernel's: the same bits)
        const uint4 qpos = *reinterpret_cast<const uint4*>(qs[0] + l16 * STRIDE + ks * 64 + qd * 16);
        const uint4 qneg = *reinterpret_cast<const uint4*>(qs[1] + l16 * STRIDE + ks * 64 + qd * 16);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(amax[t][ks], __builtin_bit_cast(bf16x8_t, qpos), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(amin[t][ks], __builtin_bit_cast(bf16x8_t, qneg), acc, 0, 0, 0);
      }
      *reinterpret_cast<f32x4_t*>(&sc[l16 * ROW + p0 + 4 * qd]) = acc;   // pages p0 + 4*qd .. of row l16
    }
    __syncthreads();
    if (wave < nrows) {
      uint32_t key[E], lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
      for (int i = 0; i < E; ++i) {
        const bool in = 64 * i + lane < P;
        const uint32_t kx = order_key(sc[wave * ROW + min(64 * i + lane, P - 1)]);   // (a page that exists: no bits of earlier use)
        key[i] = kx;
        lo = min(lo, kx);
        hi = max(hi, in ? kx : 0u);
      }
      lo = __builtin_amdgcn_readfirstlane(wave_min_u32(lo));
      hi = __builtin_amdgcn_readfirstlane(wave_max_u32(hi)) - lo;
#pragma unroll
      for (int i = 0; i < E; ++i) key[i] = 64 * i + lane < P ? key[i] - lo : 0u;   // (no candidate is 0: never counted)
      const int Kp = min(topk, P);
      uint32_t kth = 0u;
      int reach = P;   // keys >= kth
      if (Kp < P && hi) {
        for (uint32_t bit = 1u << (31 - __clz((int)hi)); bit; bit >>= 1) {
          const uint32_t cand = kth | bit;
          int n = 0;
#pragma unroll
          for (int i = 0; i < E; ++i) n += __popcll(__ballot(key[i] >= cand));
          if (n >= Kp) {
            kth = cand;
            reach = n;
            if (n == Kp) break;
          }
        }
      }
      int need = 0;   // keys equal to the K-th that are picked, the first ones in page order (looked at only if not all are)
      const bool cut = reach > Kp;
      if (cut) {
        int gt = 0;
#pragma unroll
        for (int i = 0; i < E; ++i) gt += __popcll(__ballot(key[i] > kth));
        need = Kp - gt;
      }
      uint32_t mine = 0u;   // word `lane` of the row's bitmap
#pragma unroll
      for (int i = 0; i < E; ++i) {
        const bool in = 64 * i + lane < P;
        unsigned long long pick;
        if (cut) {
          const bool eq = in & (key[i] == kth);
          const unsigned long long eqs = __ballot(eq);
          const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(eqs >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)eqs, 0));
          pick = __ballot((in & (key[i] > kth)) | (eq & (before < need)));
          need -= __popcll(eqs);   // (below zero: nothing further)
        } else {
          pick = __ballot(in & (key[i] >= kth));
        }
        mine = lane == 2 * i ? (uint32_t)pick : lane == 2 * i + 1 ? (uint32_t)(pick >> 32) : mine;
      }
      if (lane < 2 * E && mine) atomicOr(&uw[lane], mine);
    }
    __syncthreads();
  }
  // copy rt of the head's bitmap, and zeros for those that no workgroup has rows for
  if (tid < kUnionSpread) {
    const int copy = tid / COPY, tiles = gridDim.x;
    if (copy == rt || (copy >= tiles && copy % tiles == rt))
      aux.union_bits[(size_t)head * aux.union_stride + tid] = copy == rt && nrows > 0 && P > 0 ? uw[tid % COPY] : 0u;
  }
}

hipError_t launch_page_scores(hipStream_t st, int dtype, const KvView& kv, const Shape& sh, int batch,
                              int max_seq_pages, const void* q, const int32_t* active_idx,
                              const int32_t* active_count, float* scores, int32_t* tickets, int32_t* sel_count,
                              int32_t* entries, uint16_t* q_act, int rows_upper, const InKernelRanking* ranking, long workgroups_per_round,
                              uint32_t* union_bits) {
  if (batch <= 0) return hipSuccess;
  if (union_bits && dtype != LOSA_BF16) return hipErrorInvalidValue;
  const int copy_words = union_copy_words(max_seq_pages);
  ScoreAux aux{tickets, sel_count, union_bits ? entries : nullptr, q_act, union_bits,
               union_words(sh.max_pages, sh.rows_max),
               union_copies(copy_words, rows_upper >= 1 && rows_upper < sh.rows_max ? rows_upper : sh.rows_max) * copy_words};
  RankArgs ra{nullptr, 0, 0, 0.f, nullptr, nullptr, nullptr};
  if (ranking) {
    if (dtype != LOSA_BF16 || sh.B > kRankTokens) return hipErrorInvalidValue;
    ra = RankArgs{ranking->delta, ranking->mode, ranking->n, ranking->tau, ranking->mask, ranking->active_idx,
                  ranking->active_count};
  }
  dim3 grid((max_seq_pages + kScorePages - 1) / kScorePages, sh.Hkv, batch);
  if (grid.x == 0) grid.x = 1;
  if (dtype == LOSA_BF16) {
    // One 64-page tile per workgroup while the grid fits the machine in one round; beyond
    // that, more tiles per workgroup rather than a second round.
    const long tiles = max((max_seq_pages + 63) / 64, 1);
    const long round = max(workgroups_per_round, 1L);
    int tpw = (int)((tiles * sh.Hkv * batch + round - 1) / round);
    tpw = max(1, min(tpw, kMaxTilesPerWg));
    dim3 mgrid((unsigned)((tiles + tpw - 1) / tpw), sh.Hkv, batch);
    auto kern = sh.d == 128 ? (tpw == 1 ? page_scores_mfma_kernel<128, 1> : page_scores_mfma_kernel<128, kMaxTilesPerWg>)
                            : (tpw == 1 ? page_scores_mfma_kernel<64, 1> : page_scores_mfma_kernel<64, kMaxTilesPerWg>);
    kern<<<mgrid, 256, 0, st>>>(address(ra.delta), address(kv.page_indptr), address(kv.seq_lens), address(kv.page_indices), address(kv.meta), sh.B,
                                sh.Hkv, kv.num_pages, sh.max_pages, kv, sh, (const bf16_t*)q, active_idx, active_count, scores, aux, ra, tpw);
  } else {
    (sh.d == 128 ? page_scores_f32_kernel<128> : page_scores_f32_kernel<64>)<<<grid, 256, 0, st>>>(
        kv, sh, (const float*)q, active_idx, active_count, scores, aux);
  }
  return hipGetLastError();
}

// Whether one launch scores and selects.  It saves a launch and the score matrix's way through memory (2 us, and more the more
// rows there are); it costs what a compute unit needs for all of a head's metadata (the separate scoring spreads the
// pages over the chip), which the number of its workgroups does not change until the chip is full.  Separate launches / this, a step
// in us, by pages and workgroups (heads x 16-row tiles; 128 channels):
//   128 pages, 12 24.2 / 22.1; 320 52.5 / 46.4; 1024 98.0 / 78.1    192, 12 24.3 / 23.1; one tile of rows, 4 18.5 / 19.0; 16 20.6 / 20.9
//   256, 8 21.4 / 21.8; 12 24.6 / 24.6; 32 24.4 / 25.1; 36 36.1 / 32.8; 44 35.4 / 35.3; 64 34.1 / 32.3; 96 36.5 / 34.1; 576 85.6 / 79.2; 2048 201 / 168
//   375, 48 34.5 / 36.7; 96 42.0 / 42.0; 128 71.7 / 69.3; 192 61.8 / 57.6
//   512, 64 51.7 / 55.2; 96 45.9 / 48.4; 128 50.3 / 51.4; 144 57.8 / 57.8; 192 69.0 / 67.4; 512 96.1 / 90.9
//   (64 channels) 256, 1 17.1 / 15.0; 16 18.9 / 16.7
// Beyond 256 pages a wavefront has two tiles of them, 1 us more in every workgroup, which few workgroups do not make up for unless
// the locality scores' launch goes as well:
//   (64 channels) 288, 1 17.0 / 17.6; 16 18.6 / 20.5; 64 24.8 / 24.5; 128 28.4 / 26.2    384, 4 19.5 / 21.7; 16 19.0 / 21.3; 64 25.7 / 26.5;
//   128 30.0 / 28.8; with ten tiles of rows 288, 10 25.2 / 24.6    384, 10 25.5 / 26.0; 40 30.9 / 30.3
//   (256 hidden channels) 288, 1 17.0 / 16.5; 16 18.4 / 18.4    384, 1 16.9 / 17.3; 16 18.9 / 19.9, and issued one by one, where the host
//   is what limits, 22.1 / 17.4; 22.3 / 20.0
// A workgroup fills a compute unit, so that a second round of them pays where it is full, the more so the more pages there are:
//   288, 288 57.0 / 56.9    352, 288 62.2 / 62.9; 384 70.6 / 67.3    384, 320 64.0 / 64.6; 640 96.1 / 96.9; 1024 143 / 137    512, 288 70.2 / 76.9;
//   384 81.0 / 82.4; 640 111 / 116; 1280 197 / 195
// Where only the device knows the count, the grid has workgroups for rows that do not exist, each holding a compute unit for a start:
//   64 pages, 56 23.4 / 21.1    128, 56 24.2 / 23.0; 896 41.6 / 47.1    192, 56 24.6 / 24.7    256, 448 38.5 / 41.5
bool pick_pages_serves(const Shape& sh, int batch, int max_seq_pages, int rows, bool rows_known) {
  const int tiles = (rows + kPickRows - 1) / kPickRows;
  if (sh.B > 64 || max_seq_pages > kPickPages || tiles * kPickRows > kPickMostRows) return false;
  const long workgroups = (long)tiles * sh.Hkv * batch, wide = ((long)max_seq_pages * sh.d + 127) / 128;   // (wide: pages of 128 channels)
  if (!rows_known) return max_seq_pages <= 128 && workgroups <= 256;
  if (max_seq_pages <= 256) return wide <= 192 || workgroups >= 40;
  if (wide <= 192) return pick_takes_hidden(sh) || workgroups >= (wide <= 160 ? 64 : 128) || (tiles >= 8 && (wide <= 160 || workgroups >= 40));
  const long rounds = (workgroups + 255) / 256, percent = workgroups * 100 / (256 * rounds);   // compute units with a workgroup
  return workgroups >= 144 && (rounds == 1 || wide <= 288 || percent >= (wide <= 352 ? 70 : 90));
}

hipError_t launch_pick_pages(hipStream_t st, const KvView& kv, const Shape& sh, int batch, int max_seq_pages, const void* q, const void* h_cur,
                             const void* h_prev, int rows, int topk, int32_t* tickets, int32_t* sel_count, int32_t* entries, uint16_t* q_act,
                             const InKernelRanking& ranking, uint32_t* union_bits) {
  if (batch <= 0) return hipSuccess;
  if (sh.B > 64 || max_seq_pages > kPickPages || rows > kPickMostRows || (h_cur && !pick_takes_hidden(sh)))
    return hipErrorInvalidValue;
  const ScoreAux aux{tickets, sel_count, entries, q_act, union_bits, union_words(sh.max_pages, sh.rows_max), 0};
  const RankArgs ra{ranking.delta, ranking.mode, ranking.n, ranking.tau, ranking.mask, ranking.active_idx, ranking.active_count};
  const dim3 grid((rows + kPickRows - 1) / kPickRows, sh.Hkv, batch);
  auto kern = sh.d == 128 ? (max_seq_pages <= 256 ? pick_pages_kernel<128, 1> : pick_pages_kernel<128, 2>)
                          : (max_seq_pages <= 256 ? pick_pages_kernel<64, 1> : pick_pages_kernel<64, 2>);
  kern<<<grid, 1024, 0, st>>>(address(ra.delta), address(h_cur), address(h_prev), address(kv.page_indptr), address(kv.seq_lens), sh.B, sh.H, kv, sh,
                              (const bf16_t*)q, aux, ra, topk);
  return hipGetLastError();
}

hipError_t launch_select_pages(hipStream_t st, const KvView& kv, const Shape& sh, int batch, int max_seq_pages,
                               const int32_t* active_count, const float* scores, int topk, int32_t* topk_out,
                               int32_t* sel_pages, int32_t* sel_count, int cap, uint32_t* rowmaps, int32_t* tickets,
                               int rows_hint, long workgroups_per_round, uint32_t* union_bits) {
  if (batch <= 0) return hipSuccess;
  if (union_bits && topk_out) return hipErrorInvalidValue;
  SelectOut out;
  out.union_bits = union_bits;
  const int copy_words = union_copy_words(max_seq_pages);
  out.topk_out = topk_out;
  out.sel_pages = sel_pages;
  out.sel_count = sel_count;
  out.cap = cap;
  out.rowmaps = rowmaps;
  out.tickets = tickets;
  const bool rows_known = rows_hint >= 1;
  // rows_hint: an upper bound on |A| * G the host happens to know (0: none); rows past it get no workgroup
  const int rows = rows_hint >= 1 && rows_hint < sh.rows_max ? rows_hint : sh.rows_max;
  out.union_shape = (uint32_t)union_words(sh.max_pages, sh.rows_max) | (uint32_t)copy_words << 16;
  out.union_rows = (uint32_t)(union_copies(copy_words, rows) - 1) | (uint32_t)union_row_shift(copy_words) << 8;
  const int pages = max_seq_pages < sh.max_pages ? max_seq_pages : sh.max_pages;
  if (pages > kMaxSelectPages) return hipErrorInvalidValue;
  const bool list = !union_bits;
  // Query rows per workgroup: one per `round` workgroups of a grid with one row each.  A second row costs its selection
  // once more, a further workgroup its start and, where it has no row, its leaving; how many workgroups outweigh a
  // second row depends on the ending and on whether every row of the grid exists.
  //   bitmaps, count known (1 / 2 / 4 rows, us): 3584 rows 13.4 / 13.7 / 16.7; 7680 26.9 / 27.1 / 28.9; 10240 31.0 / 29.7 / 29.8;
  //     14336 40.7 / 39.6 / 39.1; 3584 of 4096 pages 22.4 / 25.8 / 27.5; 896 of 8192 pages 15.0 / 19.5 / 17.8
  //   bitmaps, count on the device (1 / 2 / 4 / 8): 84 of 256 rows x 32 heads 10.0 / 9.4 / 8.8 / 9.4; 21 of 224 x 64 10.4 / 10.0 /
  //     8.1 / 7.5; 35 of 224 x 8 5.0 / 4.9 / 5.1 / 7.1; 56 of 448 x 4, 8192 pages 8.7 / 7.9 / 7.0 / 6.9.  At most four: rows may all exist.
  //   union list, whose workgroups draw tickets (1 / 2 / 4 / 8): 84 of 256 x 32 35.4 / 35.8 / 27.0 / 18.7; 70 of 224 x 64 43.1 / 43.8 /
  //     36.1 / 22.7; 14 of 224 x 64 14.2 / 12.3 / 11.7 / 11.3; 35 of 224 x 8 9.6 / 9.9 / 10.0 / 10.0.  Every row there, scoring
  //     included: 224 x 64 196 / 130 / 105 / 103; 256 x 32 125 / 83 / 66 / 62; 224 x 16 66 / 49 / 41 / 44; 256 x 8 44.8 / 35.0 / 33.4 / 39.4;
  //     224 x 4 28.9 / 26.3 / 28.3 / 36.4; 64 x 32 of 4096 pages 51.7 / 46.0 / 42.5 / 47.7; 224 x 8 of 8192 75 / 69 / 65 / 62
  const long wgs = (long)rows * sh.Hkv * batch;
  const int threads = pages <= 256 * 8 ? 256 : pages <= 512 * 8 ? 512 : 1024;
  const long round = (list ? 1024L : rows_known ? 5120L : 2048L) * 256 / threads;
  const long want = workgroups_per_round > 0 ? (wgs + workgroups_per_round - 1) / workgroups_per_round : wgs / round;
  const int rpw = (int)max(1L, min(want, list ? 8L : 4L));
  dim3 grid((rows + rpw - 1) / rpw, sh.Hkv, batch);
  // Few keys per thread keep the unrolled code small (it has to come through the instruction
  // cache on every launch) and the loads contiguous: longer sequences get more threads, not
  // more keys per thread.
#define LOSA_SELECT(E, NT)                                                                                                             \
  (rpw == 1 ? (list ? select_pages_kernel<E, NT, false, true> : select_pages_kernel<E, NT, false, false>)                              \
            : (list ? select_pages_kernel<E, NT, true, true> : select_pages_kernel<E, NT, true, false>))<<<grid, NT, 0, st>>>(          \
      scores, active_count, address(kv.page_indptr), address(kv.seq_lens), sh.Hkv, sh.rows_max, sh.max_pages, rows_known, kv, sh, topk, out, rpw)
  if (pages <= 256 * 8)
    LOSA_SELECT(8, 256);
  else if (pages <= 512 * 8)
    LOSA_SELECT(8, 512);
  else if (pages <= 1024 * 8)
    LOSA_SELECT(8, 1024);
  else
    LOSA_SELECT(16, 1024);
#undef LOSA_SELECT
  return hipGetLastError();
}

hipError_t launch_shared_select(hipStream_t st, const KvView& kv, const Shape& sh, int batch, int max_seq_pages,
                                const int32_t* active_count, const float* scores, int topk, int32_t* sel_pages,
                                int32_t* sel_count, int cap) {
  if (batch <= 0) return hipSuccess;
  dim3 grid(sh.Hkv, batch);
  const int pages = max_seq_pages < sh.max_pages ? max_seq_pages : sh.max_pages;
  if (pages <= 256 * 8)
    shared_select_kernel<8, 256><<<grid, 256, 0, st>>>(kv, sh, active_count, scores, topk, sel_pages, sel_count, cap);
  else if (pages <= 1024 * 8)
    shared_select_kernel<8, 1024><<<grid, 1024, 0, st>>>(kv, sh, active_count, scores, topk, sel_pages, sel_count, cap);
  else if (pages <= kMaxSelectPages)
    shared_select_kernel<16, 1024><<<grid, 1024, 0, st>>>(kv, sh, active_count, scores, topk, sel_pages, sel_count, cap);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace losa
