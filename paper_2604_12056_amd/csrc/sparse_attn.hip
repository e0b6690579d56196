// Paged sparse prefix attention in float mode, and the merge of split-K partials that all attention kernels share
// (paper: Preliminaries, Attention Decomposition With Online Softmax; Methodology, eq. update_rule).
//
// Float mode accumulates in float64: with outlier channels |q.k| reaches hundreds, and float summation alone
// would come within reach of the mode's 1e-4 bound.  Both contractions run on the float64 matrix
// instructions (v_mfma_f64_16x16x4_f64).  A workgroup takes 16 query rows of a KV head and a share of its page
// list; its four wavefronts deal the pages of the share out, 16 tokens at a time, and combine their states
// through LDS at the end (two workgroups per CU: one wavefront's exponentials run under another's products):
//
//   S^T = K . Q^T        A operand: key rows, B operand: the queries, both widened from float as they are used
//   O^T += V^T . P^T     A operand: channel-major values, B operand: the numerators, as S^T leaves them
//
// A result holds, per lane, rows 4*r + lane/16 (r = 0..3) of column lane % 16.  Key row m is token
// 4*(m%4) + m/4 of the 16, so that lane group qd ends up with tokens 4*qd .. 4*qd+3, one per register: k-step r
// of the second product then takes register r of S^T and element r of a 16-byte piece of 4 consecutive
// tokens of a value channel.  Channels of O are dealt the same way, so that a lane stores 16 bytes.
// Keys of the next 16 tokens are requested when the score products of the current ones have been issued, values
// when the value products have: one register set each, and the latency lies under the other half.
//
// What bounds it: the float64 products (a register-only loop of them reaches 49 TFLOP/s) and the
// wavefronts' own start and end.  42 rows x 4 KV heads over 0.9 of 8001 tokens: 25 us (14 of them products;
// 108 us on the vector ALUs with keys and values staged through LDS).
//
// attn_merge combines the chunks of a row in chunk order with the log-sum-exp rule the paper uses to merge
// prefix and block parts, normalises, and writes (o_p, lse_p) at the active token's row.  No float atomics
// anywhere: results do not depend on scheduling.
#include <math.h>

#include <type_traits>

#include "losa_device.h"
#include "losa_internal.h"

namespace losa {

constexpr int kFloatRows = 16;   // query rows per workgroup
constexpr float kLag = 16.0f;    // natural-log units
typedef __attribute__((ext_vector_type(4))) double f64x4_t;
typedef __attribute__((ext_vector_type(4))) float f32x4v_t;

template <int D, int GP>
__global__ __launch_bounds__(256, 2) void attn_f32_kernel(KvView kv, Shape sh, const float* __restrict__ q,
                                                      const int32_t* __restrict__ active_idx,
                                                      const int32_t* __restrict__ active_count,
                                                      const int32_t* __restrict__ sel_pages,
                                                      const int32_t* __restrict__ sel_count, int cap, int nchunk, int row_blocks,
                                                      Partials part) {
  constexpr int NC = D / 16;    // 16-channel groups: pieces of keys and of values per lane and 16 tokens
  constexpr int SUB = GP / 16;  // 16-token tiles per page
  extern __shared__ __attribute__((aligned(16))) double fsm[];
  double* so = fsm;                                                    // [4][NC][4][64]: O of every wavefront
  double* sl = so + 4 * NC * 4 * 64;                                   // [4][16]
  float* sm = reinterpret_cast<float*>(sl + 4 * 16);                   // [4][16]
  float* sq = sm + 4 * 16;                                             // [NC][64][4]: query pieces in operand order
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, qd = lane >> 4;
  const int chunk = blockIdx.x, j = blockIdx.y / row_blocks, b = blockIdx.z;
  const int r0 = blockIdx.y % row_blocks * kFloatRows;
  const int head = b * sh.Hkv + j;
  const int32_t* list = sel_pages ? sel_pages + (size_t)head * cap : nullptr;
  // The way to the first tile: (list entry, token of the query row, counts) -> (page id; query row) -> (keys, values), every step
  // requested whole before the next is waited for.  One value at a time it was five memory round trips and nine scalar
  // ones: a step over 8001 tokens 47.6 -> 46.2 us, with the scoring kernel's queries and page ids together.
  auto list_position = [&](int first) { return chunk + (long)((first + lane) * 4 + wave) * nchunk; };
  int first_logical = (int)min(list_position(0), (long)0x7fffffff);
  if (list) first_logical = list_position(0) < cap ? list[list_position(0)] : -1;
  const int r = r0 + l16, slot = row_token(sh, min(r, sh.rows_max - 1));
  const int tok_listed = *(active_idx ? active_idx + (size_t)b * sh.B + slot : kv.seq_lens + b);
  int n_act = __builtin_amdgcn_readfirstlane((active_count ? active_count : kv.seq_lens)[b]);
  int listed = __builtin_amdgcn_readfirstlane(*(sel_count ? sel_count + head : kv.seq_lens + b));
  const Sequence seq = sequence(kv, sh, b);
  asm("" : "+s"(n_act), "+s"(listed) : "s"(seq.tokens), "s"(kv.page_indices), "s"(kv.num_pages), "s"(kv.k_pages), "s"(kv.v_pages), "s"(q),
      "s"(part.rows), "s"(sh.Hq));   // (see Sequence)
  const int base = seq.base, P = seq.pages, L = seq.tokens;
  const int M = min((active_idx ? min(n_act, sh.B) : sh.B) * sh.G, part.rows);
  if (r0 >= M) return;
  const int U = list ? min(listed, cap) : P;
  if (chunk >= U) return;   // pages are dealt round-robin: chunk, chunk + nchunk, ...
  // ... and this wavefront's are the wave-th, (wave + 4)-th, ... of those
  const int npages = max(0, ((U - 1 - chunk) / nchunk + 1 - wave + 3) / 4);

  // pages of this workgroup, 64 at a time: lane i resolves page i (physical id, valid tokens)
  int pg_phys = 0, pg_valid = 0;
  // (no branch around the load: what joins behind one waits for it.  An empty sequence has no entry: resolve() takes none.  The
  // choice is kept in scalar registers: as two vector registers over the loop, whose 256 are full with 128 channels, it put two others
  // into scratch memory.  Steps of 1000 to 32768 tokens take the same time within 0.5 %, attention over lists alone 1 % more)
  const int32_t* table = __builtin_amdgcn_readfirstlane(P) > 0 ? kv.page_indices + base : kv.seq_lens + b;
  auto request = [&](int logical) { return table[max(0, min(logical, P - 1))]; };
  auto resolve = [&](int first, int logical, int ph) {
    const bool ok = list_position(first) < U && (unsigned)logical < (unsigned)P && (unsigned)ph < (unsigned)kv.num_pages;
    pg_phys = ok ? ph : 0;
    pg_valid = ok ? max(0, min(GP, L - logical * GP)) : 0;
  };
  const int first_phys = request(first_logical);

  // queries of row r0 + l16 (zero past M), channels 16*c + 4*qd .., shared by the wavefronts through LDS
  // (in registers they would cost the second wavefront per SIMD)
  const int tok = active_idx ? tok_listed : slot;
  const bool known_row = r < M && (unsigned)tok < (unsigned)sh.B;
  f32x4v_t qv[NC / 4];
  {
    const float* row = q + (((size_t)b * sh.B + (known_row ? tok : 0)) * sh.Hq + j * sh.G + (min(r, sh.rows_max - 1) - slot * sh.G)) * D + 4 * qd;
#pragma unroll
    for (int c = 0; c < NC / 4; ++c) qv[c] = *reinterpret_cast<const f32x4v_t*>(row + 16 * (wave * (NC / 4) + c));
  }
  __builtin_amdgcn_sched_barrier(0);   // (the queries are requested before the page id is waited for)
  resolve(0, first_logical, first_phys);

  const int turn = 4 * (l16 & 3) + (l16 >> 2);   // token / channel this lane's operand row stands for (of 16)
  f32x4v_t kf[NC], vf[NC];
  auto load_keys = [&](int ph, int sub) {
    const float* src = (const float*)kv.k_pages + (((size_t)ph * sh.Hkv + j) * GP + 16 * sub + turn) * D + 4 * qd;
#pragma unroll
    for (int c = 0; c < NC; ++c) kf[c] = *reinterpret_cast<const f32x4v_t*>(src + 16 * c);
  };
  auto load_values = [&](int ph, int sub) {
    const float* src = (const float*)kv.v_pages + (((size_t)ph * sh.Hkv + j) * D + turn) * GP + 16 * sub + 4 * qd;
#pragma unroll
    for (int c = 0; c < NC; ++c) vf[c] = *reinterpret_cast<const f32x4v_t*>(src + (size_t)16 * c * GP);
  };
  const int ntiles = npages * SUB;
  auto tile_phys = [&](int t) { return __builtin_amdgcn_readlane(pg_phys, (t / SUB) & 63); };

  float m = -INFINITY;   // running reference of the exponentials of row l16 (any value near the maximum works)
  double l = 0.0;        // sum over this lane's own tokens
  f64x4_t o[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) o[c] = (f64x4_t){0.0, 0.0, 0.0, 0.0};
  load_keys(tile_phys(0), 0);
  load_values(tile_phys(0), 0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int c = 0; c < NC / 4; ++c)
    *reinterpret_cast<f32x4v_t*>(sq + ((wave * (NC / 4) + c) * 64 + lane) * 4) = known_row ? qv[c] : (f32x4v_t){0.f, 0.f, 0.f, 0.f};
  __syncthreads();
  for (int t = 0; t < ntiles; ++t) {
    const int nv = __builtin_amdgcn_readlane(pg_valid, (t / SUB) & 63) - 16 * (t % SUB);   // valid tokens of this tile (may be <= 0 or > 16)
    f64x4_t sc = {0.0, 0.0, 0.0, 0.0};   // (dependent float64 products issue back to back: one sum is enough)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const f32x4v_t qf = *reinterpret_cast<const f32x4v_t*>(sq + (c * 64 + lane) * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        sc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)kf[c][e], (double)qf[e], sc, 0, 0, 0);
    }
    // the page batch is exhausted: the next tile's pages have to be resolved before it can be requested
    const int tn = t + 1;
    const bool more = tn < ntiles;
    if (more && tn % (64 * SUB) == 0) {
      const long lp = list_position(tn / SUB);
      const int logical = list ? list[min(lp, (long)cap - 1)] : (int)min(lp, (long)0x7fffffff);
      resolve(tn / SUB, logical, request(logical));
    }
    const int ph_next = more ? tile_phys(tn) : 0;
    if (more) load_keys(ph_next, tn % SUB);
    double s[4];
    float tmax = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s[e] = 4 * qd + e < nv ? sc[e] * (double)sh.sm_scale : -INFINITY;
      tmax = fmaxf(tmax, (float)s[e]);
    }
    tmax = __uint_as_float(across_rows(__float_as_uint(tmax), [](uint32_t x, uint32_t y) {
      return __float_as_uint(fmaxf(__uint_as_float(x), __uint_as_float(y)));
    }));
    // the reference lags the maximum by up to kLag (e^16 is nothing to float64 sums), so after the first tile it
    // hardly ever moves
    if (__any(tmax > m + kLag)) {
      const float m_new = fmaxf(m, tmax);
      const double alpha = m == -INFINITY ? 0.0 : exp((double)m - (double)m_new);
      m = m_new;
      l *= alpha;
#pragma unroll
      for (int c = 0; c < NC; ++c) o[c] *= alpha;
    }
    const double m_use = m == -INFINITY ? 0.0 : (double)m;
    double p[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p[e] = exp(s[e] - m_use);
      l += p[e];
    }
    if (nv < 16) {   // slots past the end of the sequence may hold NaN
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) vf[c][e] = 4 * qd + e < nv ? vf[c][e] : 0.f;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int c = 0; c < NC; ++c) o[c] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)vf[c][e], p[e], o[c], 0, 0, 0);
    if (more) load_values(ph_next, tn % SUB);
  }
  // the row's tokens lie in the four lane groups
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  // ---- the four wavefronts' states meet in LDS; wavefront w combines and stores the w-th quarter of the channels
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) so[((wave * NC + c) * 4 + e) * 64 + lane] = o[c][e];
  if (qd == 0) {
    sm[wave * 16 + l16] = m;
    sl[wave * 16 + l16] = l;
  }
  __syncthreads();
  if (r >= M) return;
  float m_all = sm[l16];
#pragma unroll
  for (int w = 1; w < 4; ++w) m_all = fmaxf(m_all, sm[w * 16 + l16]);
  double wgt[4], l_all = 0.0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float mw = sm[w * 16 + l16];
    wgt[w] = mw == -INFINITY ? 0.0 : exp((double)mw - (double)m_all);
    l_all += wgt[w] * sl[w * 16 + l16];
  }
  // the reference may lag the maximum by kLag: float partials of values past 1e31 would overflow at weights of e^16,
  // so they leave with weights that add up to about 1
  if (l_all > 1.0) {
    const float m_out = m_all + logf((float)l_all);
    const double f = exp((double)m_all - (double)m_out);
    m_all = m_out;
    l_all *= f;
#pragma unroll
    for (int w = 0; w < 4; ++w) wgt[w] *= f;
  }
  const size_t prow = (((size_t)b * sh.Hkv + j) * nchunk + chunk) * part.rows + r;
#pragma unroll
  for (int c0 = 0; c0 < NC / 4; ++c0) {
    const int c = wave * (NC / 4) + c0;
    double x[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] += wgt[w] * so[((w * NC + c) * 4 + e) * 64 + lane];
    *reinterpret_cast<f32x4v_t*>(part.o + prow * D + 16 * c + 4 * qd) = (f32x4v_t){(float)x[0], (float)x[1], (float)x[2], (float)x[3]};
  }
  if (wave == 0 && qd == 0) {
    part.m[prow] = m_all;
    part.l[prow] = (float)l_all;
  }
}

// Merge of partials laid out by fragments (sparse_attn_rows.hip), 32 rows x 8 channels each, every load 1 KiB
// contiguous.  PER wavefronts deal the chunks of a fragment out, KB in flight each, and meet in LDS, in wavefront
// order; a workgroup of WAVES takes WAVES / PER fragments.  `block` counts (row tile, group of fragments) pairs.
// SPECULATE: slots exist for every row and chunk of the launch, so the first batch is requested before it is known
// which of them were written, and counts(M, live) asked for behind it; otherwise M and live are known.
constexpr int kFragSlot = 256 + 64;   // floats a wavefront leaves in LDS: fragment, references, sums
template <int D, int WAVES, int PER, int KB, bool SPECULATE, typename Counts>
__device__ __forceinline__ void merge_fragments(const Shape& sh, const int32_t* __restrict__ active_idx, int b, int j, int block,
                                                int M, int live, Counts counts, int nchunk, const Partials& part,
                                                float* __restrict__ o_p, float* __restrict__ lse_p, float* lds) {
  typedef __attribute__((ext_vector_type(4))) float f32x4_t;
  constexpr int FPB = WAVES / PER;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5, share = wave % PER;
  const int tile = block / (D / 8 / FPB), frag = block % (D / 8 / FPB) * FPB + wave / PER;
  const int r = tile * kPartialTile + l32;
  float m = -1.0e30f, l = 0.f;   // ("no token seen", as the partials have it)
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  int tok = 0;
  const int last = SPECULATE ? nchunk : live;
  if constexpr (SPECULATE) live = nchunk;
  else tok = active_idx ? active_idx[(size_t)b * sh.B + min(r / sh.G, sh.B - 1)] : r / sh.G;
  // scalar addresses that move on by a constant, plus a lane offset
  const size_t row0 = (((size_t)b * sh.Hkv + j) * nchunk + min(share, nchunk - 1)) * part.rows + tile * kPartialTile;
  const uint32_t step = (uint32_t)PER * part.rows;
  const float* pm = part.m + row0;
  const float* pl = part.l + row0;
  const float* po = part.o + row0 * D + frag * 256;
  for (int c0 = share; c0 < live; c0 += PER * KB) {
    float mk[KB], lk[KB];
    f32x4_t x[KB];
#pragma unroll
    for (int k = 0; k < KB; ++k) {   // no branches: a load behind one is waited for before the next goes out
      mk[k] = pm[l32];
      lk[k] = pl[l32];
      x[k] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(po + lane * 4));
      const uint32_t on = c0 + PER * (k + 1) < last ? step : 0;   // (past the end: the last chunk again)
      pm += on;
      pl += on;
      po += (size_t)on * D;
    }
    if constexpr (SPECULATE) {
      if (c0 == share) {
        counts(M, live);
        tok = active_idx ? active_idx[(size_t)b * sh.B + min(r / sh.G, sh.B - 1)] : r / sh.G;
      }
    }
#pragma unroll
    for (int k = 0; k < KB; ++k)
      if (c0 + PER * k >= live) {   // not a chunk, or leftovers of earlier launches, NaN included
        mk[k] = -INFINITY;
        lk[k] = 0.f;
        x[k] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
      }
    float m_new = m;
#pragma unroll
    for (int k = 0; k < KB; ++k) m_new = fmaxf(m_new, mk[k]);
    const float keep = __builtin_amdgcn_exp2f(m - m_new);
    m = m_new;
    l *= keep;
    acc *= keep;
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      const float w = __builtin_amdgcn_exp2f(mk[k] - m);
      l = fmaf(lk[k], w, l);
      acc += x[k] * w;
    }
  }
  if constexpr (PER > 1) {
    float* slot = lds + wave * kFragSlot;
    if (share) {
      *reinterpret_cast<f32x4_t*>(slot + lane * 4) = acc;
      if (half == 0) {
        slot[256 + l32] = m;
        slot[256 + 32 + l32] = l;
      }
    }
    __syncthreads();
    if (share) return;
    float mw[PER], lw[PER], m_all = m;
    f32x4_t xw[PER];
#pragma unroll
    for (int w = 1; w < PER; ++w) {
      mw[w] = slot[w * kFragSlot + 256 + l32];
      lw[w] = slot[w * kFragSlot + 256 + 32 + l32];
      xw[w] = *reinterpret_cast<const f32x4_t*>(slot + w * kFragSlot + lane * 4);
    }
#pragma unroll
    for (int w = 1; w < PER; ++w) m_all = fmaxf(m_all, mw[w]);
    const float keep = __builtin_amdgcn_exp2f(m - m_all);
    m = m_all;
    l *= keep;
    acc *= keep;
#pragma unroll
    for (int w = 1; w < PER; ++w) {
      const float wt = __builtin_amdgcn_exp2f(mw[w] - m);
      l = fmaf(lw[w], wt, l);
      acc += xw[w] * wt;
    }
  }
  if (r >= M || (unsigned)tok >= (unsigned)sh.B) return;
  const size_t orow = ((size_t)b * sh.B + tok) * sh.Hq + j * sh.G + r % sh.G;
  const bool any = m > -1.0e29f;   // no valid token at all: the neutral element of the merge
  const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
  *reinterpret_cast<f32x4_t*>(o_p + orow * D + frag * 8 + half * 4) = any ? acc / l : zero;
  if (frag == 0 && half == 0) lse_p[orow] = any ? (m + log2f(l)) * 0.6931471805599453f : -INFINITY;
}

// The leading arguments of the merge kernels (see KvView) put where the code reads them.
__device__ __forceinline__ void take_leading(Address pm, Address pl, Address po, Address active_count,
                                             int part_rows, int kv_heads, int group, int block, AttnInputs& in, Shape& sh, Partials& part) {
  part.m = pointer<float>(pm);
  part.l = pointer<float>(pl);
  part.o = pointer<float>(po);
  part.rows = part_rows;
  in.active_count = pointer<const int32_t>(active_count);
  sh.Hkv = kv_heads;
  sh.G = group;
  sh.B = block;
}

// Pages the partials of a head were dealt from.
__device__ __forceinline__ int merged_pages(const AttnInputs& in, const KvView& kv, const Shape& sh, int b, int head) {
  int listed = __builtin_amdgcn_readfirstlane(*(in.sel_count ? in.sel_count + head : kv.seq_lens + b));   // (not behind a branch where there is a count)
  const Sequence seq = sequence(kv, sh, b);
  asm("" : "+s"(listed) : "s"(seq.tokens), "s"(in.cap));   // (see Sequence)
  const int all = seq.pages;
  return in.sel_count ? min(min(listed, in.cap), sh.max_pages) : all;
}

// Query rows of a KV head (up to what partials hold) and the pages they were dealt, from one scalar round trip.
struct RowsPages {
  int rows, pages;
};
__device__ __forceinline__ RowsPages rows_and_pages(const AttnInputs& in, const KvView& kv, const Shape& sh, const Partials& part, int b, int head) {
  int n = __builtin_amdgcn_readfirstlane((in.active_count ? in.active_count : kv.seq_lens)[b]);
  int listed = __builtin_amdgcn_readfirstlane(*(in.sel_count ? in.sel_count + head : kv.seq_lens + b));
  const Sequence seq = sequence(kv, sh, b);
  asm("" : "+s"(n), "+s"(listed) : "s"(seq.tokens));   // (see Sequence)
  return {min(min((in.active_count ? min(n, sh.B) : sh.B) * sh.G, sh.rows_max), part.rows),
          in.sel_count ? min(min(listed, in.cap), sh.max_pages) : seq.pages};
}

// Every head's partials are laid out by fragments.  DENSE: every row, every page.
template <int D, int WAVES, int PER, int KB, bool DENSE>
__global__ __launch_bounds__(64 * WAVES) void attn_merge_fragments_kernel(Address pm, Address pl, Address po, Address active_count,
                                                                    int part_rows, int nchunk, int kv_heads, int rows_known, int group, int block, KvView kv, Shape sh, AttnInputs in, Partials part,
                                                                          float* __restrict__ o_p, float* __restrict__ lse_p) {
  __shared__ __attribute__((aligned(16))) float lds[PER > 1 ? WAVES * kFragSlot : 4];
  take_leading(pm, pl, po, active_count, part_rows, kv_heads, group, block, in, sh, part);
  const int j = blockIdx.y, b = blockIdx.z, head = b * sh.Hkv + j;
  const auto counts = [&](int& M, int& live) {
    const RowsPages rp = rows_and_pages(in, kv, sh, part, b, head);
    M = DENSE ? min(sh.rows_max, part.rows) : rp.rows;
    const int pages = DENSE ? sequence(kv, sh, b).pages : rp.pages, pps = kManyRowStage / sh.g;
    live = min(nchunk, (pages + pps - 1) / pps);
  };
  if (!DENSE && !rows_known && (int)blockIdx.x / (D / 8 / (WAVES / PER)) * kPartialTile >= active_rows(in, kv, sh, b)) return;   // surplus workgroup
  merge_fragments<D, WAVES, PER, KB, true>(sh, DENSE ? nullptr : in.active_idx, b, j, blockIdx.x, 0, 0, counts, nchunk, part, o_p, lse_p, lds);
}

// Combine the chunk partials of one query row with the log-sum-exp rule, normalise, and
// write (o_p, lse_p) at the active token's row.  256 threads = CL chunk lanes x D/4 channel
// quads: every chunk lane sums its chunks c = lane, lane+CL, ... (independent loads), then
// the lanes are added in a fixed order, so the result does not depend on scheduling.
// LOG2: partial maxima are in log2 units (scores scaled by sm_scale*log2(e)) and sums are
// float; otherwise natural units and double sums (float mode).
// MIXED (0: no): heads with more than 64 query rows have partials laid out by fragments; their workgroups take those, MIXED
// wavefronts each (four chunks in flight, counts first: the plain form's registers and occupancy).
template <int D, bool LOG2, int MIXED>
__global__ __launch_bounds__(256) void attn_merge_kernel(Address pm, Address pl, Address po, Address active_count,
                                                         int part_rows, int nchunk, int kv_heads, int rows_known, int group, int block, KvView kv, Shape sh, AttnInputs in, Partials part,
                                                         float* __restrict__ o_p, float* __restrict__ lse_p, int few_tile, int many_tile) {
  typedef typename std::conditional<LOG2, float, double>::type Acc;
  take_leading(pm, pl, po, active_count, part_rows, kv_heads, group, block, in, sh, part);
  constexpr int C4 = D / 4, CL = 256 / C4;
  __shared__ __attribute__((aligned(16))) Acc red[CL][D];
  __shared__ Acc lred[CL];
  __shared__ float wmax[CL];
  const int r = blockIdx.x, j = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
  if constexpr (MIXED) {
    const int M = min(min(active_rows(in, kv, sh, b), sh.rows_max), part.rows);
    if (__builtin_expect(M > kUnionRows, 0)) {
      __shared__ __attribute__((aligned(16))) float frag_lds[4 * kFragSlot];
      if (r / (D / 8 / (4 / MIXED)) * kPartialTile >= M) return;
      const int U = merged_pages(in, kv, sh, b, b * sh.Hkv + j), pps = kManyRowStage / sh.g;
      merge_fragments<D, 4, MIXED, 4, false>(sh, in.active_idx, b, j, r, M, min(nchunk, (U + pps - 1) / pps), 0, nchunk, part, o_p, lse_p, frag_lds);
      return;
    }
    if (r >= M) return;
  }
  // A grid sized without knowing the row count (threshold / cumulative-mass selection) has a
  // workgroup for every possible row: those look at the count first and leave, instead of
  // fetching partials nobody wrote (a block of 224 possible rows with 35 active ones would fetch
  // six times what it needs).
  if (!MIXED && !rows_known && r >= active_rows(in, kv, sh, b)) return;
  // The first KSPEC chunks of this thread are fetched before it is known how many chunks are
  // live (slots exist for all nchunk work items): together with the counts below this makes
  // the kernel one memory round trip deep instead of three.
  constexpr int KSPEC = 8;
  float pm_s[KSPEC], pl_s[KSPEC];
  float4 po_s[KSPEC];
  {
    const int cl = tid / C4, c4 = tid % C4;
    const uint32_t item0 = (uint32_t)(b * sh.Hkv + j) * nchunk;   // (rows of partials are counted in 32 bits: fewer than the bytes of them)
#pragma unroll
    for (int k = 0; k < KSPEC; ++k) {
      const int c = min(cl + CL * k, nchunk - 1);
      const uint32_t prow = (item0 + c) * part.rows + r;
      pm_s[k] = part.m[prow];
      pl_s[k] = part.l[prow];
      po_s[k] = reinterpret_cast<const float4*>(part.o + (size_t)prow * D)[c4];
    }
  }
  __builtin_amdgcn_sched_barrier(0);   // nothing is fetched or waited for ahead of them
  // the token of this row, fetched alongside (its slot exists whatever the active count is)
  int row = min(r, sh.rows_max - 1);
  asm("" : "+s"(row) : "s"(kv.page_indptr), "s"(kv.seq_lens), "s"(in.sel_count), "s"(in.cap), "s"(in.active_idx), "s"(sh.g_magic), "s"(few_tile),
      "s"(many_tile), "s"(o_p), "s"(lse_p));   // (see Sequence)
  const int a = row_token(sh, row);
  const int tok_listed = *(in.active_idx ? in.active_idx + (size_t)b * sh.B + a : kv.seq_lens + b);   // (no branch around a load)
  const RowsPages rp = rows_and_pages(in, kv, sh, part, b, b * sh.Hkv + j);
  const int M = rp.rows, U = rp.pages;
  const int tok_early = in.active_idx ? tok_listed : a;
  if (r >= M) return;
  const int hg = r - a * sh.G;
  const int tok = tok_early;   // r < M <= B*G here, so the index above was not clamped
  if ((unsigned)tok >= (unsigned)sh.B) return;
  const int ppt = (M <= kUnionRows ? few_tile : many_tile) / sh.g;
  const int ntiles = (U + ppt - 1) / ppt;
  const int live = min(nchunk, ntiles);   // work item c exists iff tile c does
  const size_t item0 = ((size_t)b * sh.Hkv + j) * nchunk;

  // thread (cl, c4) owns chunks cl, cl+CL, ... and channel quad c4
  const int cl = tid / C4, c4 = tid % C4;
  float mk[KSPEC];
#pragma unroll
  for (int k = 0; k < KSPEC; ++k) mk[k] = cl + CL * k < live ? pm_s[k] : -INFINITY;
  float mx = -INFINITY;
#pragma unroll
  for (int k = 0; k < KSPEC; ++k) mx = fmaxf(mx, mk[k]);
  for (int c = cl + CL * KSPEC; c < live; c += CL) mx = fmaxf(mx, part.m[(item0 + c) * part.rows + r]);
  if (c4 == 0) wmax[cl] = mx;
  __syncthreads();
  float m_tot = -INFINITY;
#pragma unroll
  for (int k = 0; k < CL; ++k) m_tot = fmaxf(m_tot, wmax[k]);
  const size_t orow = ((size_t)b * sh.B + tok) * sh.Hq + j * sh.G + hg;
  if (!(m_tot > -1.0e29f)) {   // no valid token at all: the neutral element of the merge
    if (tid < C4) reinterpret_cast<float4*>(o_p + orow * D)[tid] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (tid == 0) lse_p[orow] = -INFINITY;
    return;
  }
  Acc ax = 0, ay = 0, az = 0, aw = 0, lacc = 0;
#pragma unroll
  for (int k = 0; k < KSPEC; ++k) {
    if (cl + CL * k < live) {   // slots past `live` hold leftovers of earlier launches: never touch their values
      const float dm = mk[k] - m_tot;
      const Acc w = LOG2 ? (Acc)exp2f(dm) : (Acc)exp((double)dm);
      ax += w * (Acc)po_s[k].x;
      ay += w * (Acc)po_s[k].y;
      az += w * (Acc)po_s[k].z;
      aw += w * (Acc)po_s[k].w;
      lacc += w * (Acc)pl_s[k];
    }
  }
  for (int c = cl + CL * KSPEC; c < live; c += CL) {
    const size_t prow = (item0 + c) * part.rows + r;
    const float dm = part.m[prow] - m_tot;
    const Acc w = LOG2 ? (Acc)exp2f(dm) : (Acc)exp((double)dm);
    const float4 v = reinterpret_cast<const float4*>(part.o + prow * D)[c4];
    ax += w * (Acc)v.x;
    ay += w * (Acc)v.y;
    az += w * (Acc)v.z;
    aw += w * (Acc)v.w;
    lacc += w * (Acc)part.l[prow];
  }
  red[cl][c4 * 4 + 0] = ax;
  red[cl][c4 * 4 + 1] = ay;
  red[cl][c4 * 4 + 2] = az;
  red[cl][c4 * 4 + 3] = aw;
  if (c4 == 0) lred[cl] = lacc;
  __syncthreads();
  if (tid < D) {
    Acc o = 0, l = 0;
#pragma unroll
    for (int k = 0; k < CL; ++k) {
      o += red[k][tid];
      l += lred[k];
    }
    o_p[orow * D + tid] = (float)(o / l);
    if (tid == 0)
      lse_p[orow] = LOG2 ? (m_tot + log2f((float)l)) * 0.6931471805599453f : (float)((double)m_tot + log((double)l));
  }
}

// The same for few chunks (nchunk <= KC): a wavefront takes 256 / D rows, a thread one channel quad of a row and all of its
// chunks, with no LDS and no barrier.  The form above deals the chunks out to 1024 / D lanes per row, whether there are
// that many or not, with eight loads each: with four chunks half of its threads have none and most loads are repeats.
// Rows x heads, chunks, plain form / this: 64 x 128, 2 16.9 / 5.5 us; 63 x 64, 4 10.1 / 5.0; 35 x 64, 4 7.5 / 4.9; 64 x 32, 8
// 6.8 / 4.9; 42 x 4, 8 the same.  With 11 or 12 chunks and few rows its threads' loads take longer than the plain form's
// barriers (24 x 1 3.4 / 3.9).  A thread's products are rounded and added in chunk order, as the plain form's lanes
// are, so the results are the same bits.
// MIXED, as above: a workgroup of four wavefronts then, which takes fragments of the heads that have them (63 of 224 rows
// x 64 heads, 4 chunks 10.3 / 5.1 us; 112 rows 6.6 / 6.3).
constexpr int kFewChunks = 8;
template <int D, int KC, bool MIXED>
__global__ __launch_bounds__(64 * (MIXED ? 4 : 1)) void attn_merge_few_kernel(Address pm, Address pl, Address po, Address active_count,
                                                            int part_rows, int nchunk, int kv_heads, int rows_known, int group, int block, KvView kv, Shape sh, AttnInputs in, Partials part,
                                                            float* __restrict__ o_p, float* __restrict__ lse_p, int few_tile, int many_tile) {
  constexpr int C4 = D / 4, WAVES = MIXED ? 4 : 1;
  take_leading(pm, pl, po, active_count, part_rows, kv_heads, group, block, in, sh, part);
  const int tid = threadIdx.x, c4 = tid % C4, j = blockIdx.y, b = blockIdx.z;
  const int r0 = blockIdx.x * (64 * WAVES / C4), r = r0 + tid / C4;
  if constexpr (MIXED) {
    const int M = min(min(active_rows(in, kv, sh, b), sh.rows_max), part.rows);
    if (__builtin_expect(M > kUnionRows, 0)) {
      if ((int)blockIdx.x / (D / 8 / WAVES) * kPartialTile >= M) return;
      const int U = merged_pages(in, kv, sh, b, b * sh.Hkv + j), pps = kManyRowStage / sh.g;
      merge_fragments<D, WAVES, 1, 4, false>(sh, in.active_idx, b, j, blockIdx.x, M, min(nchunk, (U + pps - 1) / pps), 0, nchunk, part, o_p, lse_p, nullptr);
      return;
    }
    if (r0 >= M) return;
  } else if (!rows_known && r0 >= active_rows(in, kv, sh, b)) {
    return;   // surplus workgroup
  }
  float mk[KC], lk[KC];
  f32x4v_t x[KC];
#pragma unroll
  for (int k = 0; k < KC; ++k) {   // before it is known how many chunks are live: slots exist for all of them
    const uint32_t prow = ((uint32_t)(b * sh.Hkv + j) * nchunk + min(k, nchunk - 1)) * part.rows + min(r, part.rows - 1);   // (32 bits hold it)
    mk[k] = part.m[prow];
    lk[k] = part.l[prow];
    x[k] = reinterpret_cast<const f32x4v_t*>(part.o + (size_t)prow * D)[c4];
  }
  __builtin_amdgcn_sched_barrier(0);   // nothing is fetched or waited for ahead of them
  int last_row = sh.rows_max - 1;
  asm("" : "+s"(last_row) : "s"(kv.page_indptr), "s"(kv.seq_lens), "s"(in.sel_count), "s"(in.cap), "s"(in.active_idx), "s"(sh.g_magic), "s"(few_tile),
      "s"(many_tile), "s"(o_p), "s"(lse_p));   // (see Sequence)
  const int a = row_token(sh, min(r, last_row));
  const int tok_listed = *(in.active_idx ? in.active_idx + (size_t)b * sh.B + a : kv.seq_lens + b);   // (no branch around a load)
  const int tok = in.active_idx ? tok_listed : a;
  const RowsPages rp = rows_and_pages(in, kv, sh, part, b, b * sh.Hkv + j);
  const int M = rp.rows, U = rp.pages;
  if (r >= M || (unsigned)tok >= (unsigned)sh.B) return;
  const int ppt = (M <= kUnionRows ? few_tile : many_tile) / sh.g;
  const int live = min(nchunk, (U + ppt - 1) / ppt);
  float m_tot = -INFINITY;
#pragma unroll
  for (int k = 0; k < KC; ++k) {
    if (k >= live) {   // not a chunk, or leftovers of earlier launches, NaN included
      mk[k] = -INFINITY;
      lk[k] = 0.f;
      x[k] = (f32x4v_t){0.f, 0.f, 0.f, 0.f};
    }
    m_tot = fmaxf(m_tot, mk[k]);
  }
  const size_t orow = ((size_t)b * sh.B + tok) * sh.Hq + j * sh.G + (r - a * sh.G);
  f32x4v_t o = {0.f, 0.f, 0.f, 0.f};
  float l = 0.f;
  if (!(m_tot > -1.0e29f)) {   // no valid token at all: the neutral element of the merge
    reinterpret_cast<f32x4v_t*>(o_p + orow * D)[c4] = o;
    if (c4 == 0) lse_p[orow] = -INFINITY;
    return;
  }
#pragma unroll
  for (int k = 0; k < KC; ++k) {
#pragma clang fp contract(off)
    const float w = exp2f(mk[k] - m_tot);
    o += x[k] * w;
    l += lk[k] * w;
  }
  reinterpret_cast<f32x4v_t*>(o_p + orow * D)[c4] = o / l;
  if (c4 == 0) lse_p[orow] = (m_tot + log2f(l)) * 0.6931471805599453f;
}

template <int D, int GP>
static hipError_t launch_f32(hipStream_t st, const KvView& kv, const Shape& sh, int batch, const float* q,
                             const int32_t* active_idx, const int32_t* active_count, const int32_t* sel_pages,
                             const int32_t* sel_count, int cap, int nchunk, const Partials& part) {
  constexpr size_t lds_bytes = 4 * (D / 16) * 4 * 64 * sizeof(double) + 4 * 16 * (sizeof(double) + sizeof(float)) + 16 * D * sizeof(float);
  const int row_blocks = (part.rows + kFloatRows - 1) / kFloatRows;
  auto kern = attn_f32_kernel<D, GP>;
  static bool attr_set = false;   // per instantiation
  if (lds_bytes > 48 * 1024 && !attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds_bytes);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  kern<<<dim3(nchunk, sh.Hkv * row_blocks, batch), 256, lds_bytes, st>>>(kv, sh, q, active_idx, active_count, sel_pages,
                                                                         sel_count, cap, nchunk, row_blocks, part);
  return hipGetLastError();
}

hipError_t launch_attn_f32(hipStream_t st, const KvView& kv, const Shape& sh, int batch, const void* q,
                           const int32_t* active_idx, const int32_t* active_count, const int32_t* sel_pages,
                           const int32_t* sel_count, int cap, int nchunk, const Partials& part) {
  if (batch <= 0 || nchunk <= 0) return hipSuccess;
  auto launch = sh.d == 128 ? (sh.g == 16 ? launch_f32<128, 16> : launch_f32<128, 32>)
                            : (sh.g == 16 ? launch_f32<64, 16> : launch_f32<64, 32>);
  return launch(st, kv, sh, batch, (const float*)q, active_idx, active_count, sel_pages, sel_count, cap, nchunk, part);
}

hipError_t launch_attn_merge(hipStream_t st, const KvView& kv, const Shape& sh, int batch, const AttnInputs& in,
                             bool bf16, int nchunk, const Partials& part, float* o_p, float* lse_p, int rows_hint, int few_tile, int many_tile) {
  if (batch <= 0) return hipSuccess;
  // rows_hint: an upper bound on the active rows per KV head the host happens to know (0: none);
  // rows past it get no workgroup (they would only fetch partials speculatively and exit)
  const int rows = rows_hint >= 1 && rows_hint < sh.rows_max ? rows_hint : sh.rows_max;
  const bool dense_step = !in.active_idx && !in.sel_count;
  const int known = rows_hint >= 1 || !in.active_idx;   // (no list of active tokens: every row exists)
  const int tiles = (rows + kPartialTile - 1) / kPartialTile, frags = sh.d / 8;
  if (few_tile == kManyRowStage) {   // every head's partials are laid out by fragments
    auto launch = [&](auto kern, int per_tile, int waves) {
      kern<<<dim3(tiles * per_tile, sh.Hkv, batch), 64 * waves, 0, st>>>(address(part.m), address(part.l), address(part.o), address(in.active_count), part.rows, nchunk, sh.Hkv, known, sh.G, sh.B, kv, sh, in, part, o_p, lse_p);
    };
#define LOSA_FRAGMENTS(W, PER, KB)                                                                                  \
  launch(sh.d == 128 ? (dense_step ? attn_merge_fragments_kernel<128, W, PER, KB, true>                             \
                                   : attn_merge_fragments_kernel<128, W, PER, KB, false>)                           \
                     : (dense_step ? attn_merge_fragments_kernel<64, W, PER, KB, true>                              \
                                   : attn_merge_fragments_kernel<64, W, PER, KB, false>), frags * PER / W, W)
    // One or two batches of loads per wavefront, no more wavefronts than that takes (the chip starts one per 10
    // cycles and die).  By chunks, this form / its neighbour: 2 (128 heads, 128 rows) 6.7 / 10.3 us; 4 5.5 / 7.0;
    // 16 (16 heads, 256 rows) 7.5 / 10.8; 32 (8 heads) 8.2 / 8.5; 64 (4 heads, 224 rows) 7.0 / 7.2; 256 (1 head) 7.0 / 8.6.
    if (nchunk <= 4) LOSA_FRAGMENTS(4, 1, 2);
    else if (nchunk <= 16) LOSA_FRAGMENTS(4, 1, 8);
    else if (nchunk <= 64) LOSA_FRAGMENTS(4, 4, 8);
    else LOSA_FRAGMENTS(8, 8, 8);
#undef LOSA_FRAGMENTS
    return hipGetLastError();
  }
  if (bf16 && nchunk <= kFewChunks) {
    const bool mixed = many_tile == kManyRowStage;
    auto kern = mixed ? (sh.d == 128 ? (nchunk <= 4 ? attn_merge_few_kernel<128, 4, true> : attn_merge_few_kernel<128, 8, true>)
                                     : (nchunk <= 4 ? attn_merge_few_kernel<64, 4, true> : attn_merge_few_kernel<64, 8, true>))
                      : (sh.d == 128 ? (nchunk <= 4 ? attn_merge_few_kernel<128, 4, false> : attn_merge_few_kernel<128, 8, false>)
                                     : (nchunk <= 4 ? attn_merge_few_kernel<64, 4, false> : attn_merge_few_kernel<64, 8, false>));
    const int waves = mixed ? 4 : 1, per_wg = waves * 256 / sh.d, few = ((mixed ? min(rows, kUnionRows) : rows) + per_wg - 1) / per_wg;
    kern<<<dim3(mixed ? max(few, tiles * frags / 4) | 1 : few, sh.Hkv, batch), 64 * waves, 0, st>>>(address(part.m), address(part.l), address(part.o), address(in.active_count), part.rows, nchunk, sh.Hkv, known, sh.G, sh.B, kv, sh, in, part, o_p, lse_p,
                                                                                                  few_tile, many_tile);
    return hipGetLastError();
  }
  // wavefronts per fragment in a mixed launch: with few chunks one, a quarter of the workgroups
  const int mixed = many_tile != kManyRowStage ? 0 : nchunk <= 16 ? 1 : 4;
  auto kern = sh.d == 128 ? (!bf16 ? attn_merge_kernel<128, false, 0> : mixed == 0 ? attn_merge_kernel<128, true, 0>
                             : mixed == 1 ? attn_merge_kernel<128, true, 1> : attn_merge_kernel<128, true, 4>)
                          : (!bf16 ? attn_merge_kernel<64, false, 0> : mixed == 0 ? attn_merge_kernel<64, true, 0>
                             : mixed == 1 ? attn_merge_kernel<64, true, 1> : attn_merge_kernel<64, true, 4>);
  // (mixed: an odd width.  Most of its workgroups leave at once, and with a multiple of 8 the ones that stay meet on a
  // few of every die's compute units: 14 of 64 rows, 40 heads 6.8 us, of 65 5.4)
  kern<<<dim3(mixed ? max(min(rows, kUnionRows), tiles * frags * mixed / 4) | 1 : rows, sh.Hkv, batch), 256, 0, st>>>(
      address(part.m), address(part.l), address(part.o), address(in.active_count), part.rows, nchunk, sh.Hkv, known, sh.G, sh.B, kv, sh, in, part, o_p, lse_p, few_tile, many_tile);
  return hipGetLastError();
}

}  // namespace losa
