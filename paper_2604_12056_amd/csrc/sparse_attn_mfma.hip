// Split-K paged sparse prefix attention on the gfx950 matrix cores, bfloat16 inputs
// (paper: Preliminaries, Attention Decomposition With Online Softmax; Methodology, eq. update_rule).
//
// One wavefront owns up to R*16 query rows of one KV head and walks 32-token tiles of that
// head's page list with v_mfma_f32_16x16x32_bf16:
//
//   S^T = K_tile . Q^T      A operand = 16 keys x 32 channels, read straight from the
//                           token-major key page (each lane one 16-byte load);
//                           B operand = the query fragment, resident in registers.
//   O^T += V_tile^T . P^T   A operand = 16 channels x 32 tokens, read straight from the
//                           channel-major value page (one 16-byte load per lane);
//                           B operand = P^T, which is exactly how S^T leaves the matrix core
//                           (lane = query column, 4+4 tokens), so probabilities never cross
//                           lanes and the per-row rescale factor is lane-local as well.
//
// The 16 rows of a score-product half are a chosen subset of the tile's 32 tokens such that
// each lane ends up with 8 consecutive tokens; both operands of the second product use that
// same token order, which is all a contraction needs.
//
// Two work shapes:
//   split-pages (rows <= 64, the sparse steps): the four wavefronts of a workgroup take
//       interleaved tiles, K/V go global -> registers in operand layout one tile ahead (no LDS
//       and no barrier in the main loop), and the four combine their (reference, sum, O)
//       through LDS at the end, so one partial leaves the workgroup;
//   many rows: four independent wavefronts of 64 rows, each loading every tile itself.  More than 64
//       rows normally take sparse_attn_rows.hip; this form is what LOSA_TUNE_SHARED_TILES = 0 selects.
// Tiles of a (sequence, head) list are dealt round-robin to its workgroups, so every
// workgroup gets the same number of tiles (within one) whatever the union size turns out to be.
#include <hip/hip_ext.h>
#include <math.h>

#include <type_traits>

#include "losa_device.h"
#include "losa_internal.h"

namespace losa {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(8))) float f32x8_t;
typedef uint32_t u32x4v_t __attribute__((ext_vector_type(4)));   // a plain vector value (stays in registers)

constexpr float kNegBig = -1.0e30f;   // finite stand-in for "no token seen yet"

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// max over the 4 lanes {l, l^16, l^32, l^48} with the gfx950 lane-swap instructions (vector ALU,
// no LDS round trip): after a swap of a register with itself the pair holds both halves.
__device__ __forceinline__ float max_over_lane_groups(float v) {
  const unsigned u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float m16 = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const unsigned w = __float_as_uint(m16);
  const auto c = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return fmaxf(__uint_as_float(c[0]), __uint_as_float(c[1]));
}
__device__ __forceinline__ float sum_over_lane_groups(float v) {
  const unsigned u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float s16 = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const unsigned w = __float_as_uint(s16);
  const auto c = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return __uint_as_float(c[0]) + __uint_as_float(c[1]);
}

template <int D, int R>
struct MergeSlot {   // LDS image of one wavefront's state: O as [row tile][channel tile][lane] 16-byte
                     // vectors (every access is lane-linear, so bank-conflict free), then ref[], sum[]
  static constexpr int kOFloats = R * (D / 16) * 64 * 4;
  static constexpr int kFloats = kOFloats + 2 * R * 16;
};

// A wavefront resolves its pages itself: list entry (logical page) -> page table -> key and value pages, with the query rows
// gathered by the active list beside it, everything that does not depend on what is still under way requested at once.
// (A launch of its own that resolved the list and gathered the rows first took 3.5 us; the two dependent
// round trips it saved here take 0.6.)
// UNION (split-pages shape only): there is no page list.  The selection kernel left the
// union of the head's picks as a bitmap, the scoring kernel the query rows and a copy of the head's page table (which the
// four wavefronts bring to LDS together); every wavefront ranks the union with a popcount prefix sum (lane = bitmap
// word), keeps words and ranks in LDS (in its own merge slot, which is idle until the combine), and finds
// the pages of its own tiles by rank: a four-way search over the word ranks, a 5-step search inside
// the word, then the page's entry from the table in LDS (from memory for pages beyond the first
// 2048).  That is more start-up work than with a list (about 1.5 us at 2048 pages), in
// exchange for the selection kernel's whole hand-over tail (about 4 us).
// By stamps (42 rows x 4 heads, 0.72 of 2048 pages; 2.45 GHz): a wavefront has its bitmap after 1550 cycles, its first pages after
// 3900, has asked for its first tile after 7400 (a compute unit takes some 22 bytes of requests a cycle), has it after 12700,
// takes 2700 to 3800 cycles a tile, the combine and the stores 4900; cached keys and values take 2 us off the step, no more.
constexpr int kMaxUnionWords = kMaxSelectPages / 32;
constexpr int kTablePagesInLds = 2048;   // the first so many entries of a head's page table are kept in LDS
// LDS of the split-pages shape, in floats: the four wavefronts' merge slots, then (UNION) the page table.
constexpr int kUnionShared = kTablePagesInLds;
template <int D, int GP, int R, bool SPLIT_PAGES, int NBUF, bool UNION = false>
__device__ __forceinline__ void attn_mfma_body(const AttnInputs& in, int nchunk, int nrbg, Shape sh, KvView kv, Partials part,
                                               float scale_log2e, int m_lo, int m_hi, UnionInKernel uni, float* lds) {
  static_assert(!UNION || SPLIT_PAGES, "the union is built in the kernel only in the split-pages shape");
  static_assert(!UNION || MergeSlot<D, R>::kFloats >= 2 * kMaxUnionWords, "the union's words and ranks do not fit a merge slot");
  constexpr int kSlotStride = MergeSlot<D, R>::kFloats;
  constexpr int KS = D / 32;    // k-steps of the score product
  constexpr int NT = D / 16;    // channel tiles of the output
  constexpr int PPT = 32 / GP;  // pages per 32-token tile
  constexpr int TPR = 64 / PPT; // tiles covered by one page-entry fetch (one entry per lane)

  // the wavefront number is the same for all lanes; saying so keeps what derives from it (tile
  // numbers, loop bounds, page ids, base addresses) in scalar registers and scalar arithmetic
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, qd = lane >> 4;
  const int chunk = blockIdx.x, b = blockIdx.z;
  const int j = SPLIT_PAGES ? blockIdx.y : blockIdx.y / nrbg;
  const int rb = SPLIT_PAGES ? 0 : (blockIdx.y % nrbg) * 4 + wave;
  const int head = b * sh.Hkv + j;

  // Tiles are dealt round-robin: workgroup `chunk` owns tiles chunk, chunk+nchunk, ... of the
  // list, and in the split-pages shape its four wavefronts deal those out again.  Which tiles
  // a wavefront owns therefore does not depend on the list length, only whether they exist.
  const int wstart = SPLIT_PAGES ? wave : 0, wstride = SPLIT_PAGES ? 4 : 1;
  const int tfirst = chunk + nchunk * wstart;   // first tile of this wavefront
  const int tstep = nchunk * wstride;           // distance between its tiles
  const int32_t* ent = UNION ? uni.entries + (size_t)head * sh.max_pages : nullptr;

  // ---- start-up.  What gates the kernel is when the first key/value load leaves, and that
  // needs only the counts and the page entries: they are fetched first, the exit tests follow,
  // and the query fragments are requested next but not waited for until after the first tiles
  // have been requested (they arrive long before the first tile does).
  [[maybe_unused]] int tok[R];   // token of row l16 of every row tile (clamped: a slot that exists)
  if constexpr (!UNION) {
#pragma unroll
    for (int mt = 0; mt < R; ++mt) {
      const int a = row_token(sh, min(rb * (R * 16) + mt * 16 + l16, sh.rows_max - 1));
      const int at = *(in.active_idx ? in.active_idx + (size_t)b * sh.B + a : kv.seq_lens + b);   // (no branch around a load: what
      tok[mt] = in.active_idx ? at : a;                                                            // joins behind one waits for it)
    }
  }
  auto list_position = [&](int first_local_tile) {
    return (tfirst + (first_local_tile + lane / PPT) * tstep) * PPT + lane % PPT;   // (below 64 x 4096 past a list of 16384)
  };
  auto listed = [&](int lp) {   // logical page at a position of the list (inside the array whatever the list's length is)
    const int at = *(in.list ? in.list + (size_t)head * in.cap + min(lp, in.cap - 1) : kv.seq_lens + b);
    return in.list ? at : min(lp, sh.max_pages);
  };
  [[maybe_unused]] int logical = 0;
  if constexpr (!UNION) logical = listed(list_position(0));
  // counts, the sequence and (lists; the union has its own place) the arguments that the way to the first tile needs: see Sequence
  int n_act = __builtin_amdgcn_readfirstlane((in.active_count ? in.active_count : kv.seq_lens)[b]), n_listed = 0;
  if constexpr (!UNION) n_listed = __builtin_amdgcn_readfirstlane(*(in.list ? in.sel_count + head : kv.seq_lens + b));
  const Sequence seq = sequence(kv, sh, b);
  if constexpr (UNION)
    asm("" : "+s"(n_act) : "s"(seq.tokens));
  else
    asm("" : "+s"(n_act), "+s"(n_listed) : "s"(seq.tokens), "s"(kv.page_indices), "s"(kv.num_pages), "s"(kv.k_pages), "s"(kv.v_pages), "s"(in.q),
        "s"(sh.rows_max), "s"(part.rows), "s"(sh.Hq), "s"(m_lo), "s"(m_hi));
  const int M_raw = (in.active_count ? min(n_act, sh.B) : sh.B) * sh.G;
  const int base = seq.base, P = seq.pages, tokens = seq.tokens;
  int U_raw;
  int pg_entry = 0;
  [[maybe_unused]] auto fetch_entry = [&]() {   // of page `logical`: its id; page and id are checked when it is decoded
    pg_entry = *(P > 0 ? kv.page_indices + base + max(0, min(logical, P - 1)) : kv.seq_lens + b);   // (an empty sequence has none)
  };
  // UNION: words and ranks of the head's union, in this wavefront's own merge slot; the page table behind the slots
  [[maybe_unused]] uint32_t* u_bits = reinterpret_cast<uint32_t*>(lds + (SPLIT_PAGES ? wave : 0) * kSlotStride);
  [[maybe_unused]] int* u_base = reinterpret_cast<int*>(u_bits) + kMaxUnionWords;
  [[maybe_unused]] int* u_tab = reinterpret_cast<int*>(lds + 4 * kSlotStride);   // entries by logical page
  [[maybe_unused]] int u_words = 0;
  // pages whose entries the LDS copy holds: whole 16-byte pieces of the table, up to what fits
  [[maybe_unused]] const int tab_lds_pages = min(sh.max_pages & ~3, kTablePagesInLds);
  if constexpr (UNION) {
    // The four wavefronts share the fetch of the page table (8 KiB; once per wavefront it would cost the
    // compute unit four times the traffic): a quarter each, one barrier.
    const bool copies = uni.copy_words <= kMostCopiedWords;
    const int words = copies ? kUnionSpread : uni.copy_words;
    // the head's page table, written by the scoring kernel at an address known here: its first
    // kTablePagesInLds entries go to LDS, so that resolving a page needs no dependent load
    // (pages beyond them are looked up in memory)
    constexpr int TPW = kTablePagesInLds / 4 / 256;   // 16-byte pieces per lane per wavefront
    u32x4v_t tabv[TPW];
#pragma unroll
    for (int k = 0; k < TPW; ++k) {
      const int i4 = min(wave * (64 * TPW) + lane + 64 * k, max(sh.max_pages / 4 - 1, 0));   // clamped inside the head's table
      tabv[k] = reinterpret_cast<const u32x4v_t*>(ent)[i4];
    }
    // the head's union bitmap: up to four words per lane in flight (8192 pages are one memory round trip); copies of
    // 16 or 32 words lie one behind the other and are ORed in the lanes
    const uint32_t* head_bits = uni.bits + (size_t)head * uni.stride;
    constexpr int kGroupsInFlight = 4;
    uint32_t ub[kGroupsInFlight];
#pragma unroll
    for (int u = 0; u < kGroupsInFlight; ++u) ub[u] = 64 * u < words ? head_bits[min(64 * u + lane, words - 1)] : 0u;
#pragma unroll
    for (int k = 0; k < TPW; ++k) reinterpret_cast<u32x4v_t*>(u_tab)[wave * (64 * TPW) + lane + 64 * k] = tabv[k];
    u_words = (P + 31) >> 5;
    // Kernel arguments that the way to the first tile needs, all fetched by now: fetched where they are used, each group
    // of them is a scalar round trip there.
    asm volatile("" ::"s"(nchunk), "s"(sh.rows_max), "s"(part.rows), "s"(kv.num_pages), "s"(kv.k_pages), "s"(kv.v_pages), "s"(uni.q_act),
                 "s"(uni.sel_count), "s"(m_lo), "s"(m_hi), "s"(sh.B), "s"(sh.G));
    __syncthreads();
    if (copies) {
      uint32_t all = (ub[0] | ub[1]) | (ub[2] | ub[3]);
      if (uni.copy_words == 16) {
        all = across_rows(all, [](uint32_t x, uint32_t y) { return x | y; });
      } else {
        const auto sw = __builtin_amdgcn_permlane32_swap(all, all, false, false);
        all = sw[0] | sw[1];
      }
      ub[0] = all;   // (lanes past the copy's words hold repeats: past u_words, so cleared below)
    }
    const int ranked = copies ? 64 : words;
    int total = 0;
    for (int g0 = 0; g0 < ranked; g0 += 64 * kGroupsInFlight) {
      if (g0) {
#pragma unroll
        for (int u = 0; u < kGroupsInFlight; ++u)
          ub[u] = g0 + 64 * u < words ? head_bits[min(g0 + 64 * u + lane, words - 1)] : 0u;
      }
#pragma unroll
      for (int u = 0; u < kGroupsInFlight; ++u) {
        if (g0 + 64 * u >= ranked) break;   // uniform
        const int w = g0 + 64 * u + lane;
        uint32_t acc = ub[u];
        // pages past the sequence's last one are never picked; the masks only keep a stale bitmap harmless
        if (w >= u_words) acc = 0u;
        if (w == u_words - 1 && (P & 31)) acc &= (1u << (P & 31)) - 1u;
        const int c = __popc(acc);
        const int incl = wave_inclusive_scan(c);
        u_bits[w] = acc;
        u_base[w] = total + incl - c;
        total += __builtin_amdgcn_readlane(incl, 63);
      }
    }
    U_raw = total;
  } else {
    U_raw = in.list ? min(n_listed, in.cap) : P;
    fetch_entry();
  }
  const int U = min(U_raw, sh.max_pages);
  const int M = min(M_raw, min(sh.rows_max, part.rows));   // (rows past the partial stride have nowhere to go: the host sizes it from an upper bound)
  const int ntiles = (U + PPT - 1) / PPT;
  // M <= 0: nothing active; chunk >= ntiles: this workgroup owns no tile; third: no rows for this
  // wavefront in the split-rows shape (which uses no barrier)
  // fourth: this launch only serves row counts in (m_lo, m_hi] (the host may not know the count
  // and then launches both work shapes, each taking its own range)
  const bool has_rows = SPLIT_PAGES || rb * (R * 16) < M;
  // the union's size, for the merge kernel and the caller's diagnostics: stored at the end, as the wait for a page entry out of
  // memory would be one for this store too
  [[maybe_unused]] auto leave_count = [&]() {
    if constexpr (UNION)
      if (chunk == 0 && threadIdx.x == 0 && M_raw > 0) uni.sel_count[head] = U_raw;
  };
  if ((M <= 0) | (chunk >= ntiles) | !has_rows | (M <= m_lo) | (M > m_hi)) {
    leave_count();
    return;
  }
  const int ntw = tfirst < ntiles ? (ntiles - 1 - tfirst) / tstep + 1 : 0;   // this wavefront's tiles

  bf16x8_t qf[R][KS];
  {
#pragma unroll
    for (int mt = 0; mt < R; ++mt) {
      const int r = min(rb * (R * 16) + mt * 16 + l16, sh.rows_max - 1);
      const bf16_t* row;
      if constexpr (UNION) {   // (gathered by the scoring kernel: the rows' tokens are one round trip less here)
        row = uni.q_act + ((size_t)head * sh.rows_max + r) * D;
      } else {
        const int t = (unsigned)tok[mt] < (unsigned)sh.B ? tok[mt] : 0;
        row = (const bf16_t*)in.q + (((size_t)b * sh.B + t) * sh.Hq + j * sh.G + (r - row_token(sh, r) * sh.G)) * D;
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        qf[mt][ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(row + ks * 32 + qd * 8));
    }
  }
  __builtin_amdgcn_sched_barrier(0);   // the query loads stay ahead of the tile loads below

  float m_run[R], l_run[R], up_thr[R];   // up_thr: the raw score above which a row's reference has to move
  const float inv_scale_log2e = 1.0f / scale_log2e;
  f32x4_t o[R][NT];
#pragma unroll
  for (int mt = 0; mt < R; ++mt) {
    m_run[mt] = kNegBig;
    up_thr[mt] = -INFINITY;
    l_run[mt] = 0.f;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) o[mt][nt] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
  }

  // ---- decoded page entries of this wavefront's next 64 pages, one per lane
  int pg_phys = 0, pg_valid = 0;
  auto decode_entries = [&](int first_local_tile) {
    const int lp = list_position(first_local_tile);
    if constexpr (UNION) {
      // the page of rank lp in the union: the last bitmap word whose rank is <= lp, then the
      // (lp - rank)-th set bit of that word; its physical id comes from the page table
      int page = 0;
      const bool want = lp < U;
      if (want) {
        int lo = 0, k = lp;
        // four ways a step (three LDS reads at once): 3 steps for 64 words; the trip count is uniform over the wavefront
        for (int step = u_words <= 64 ? 16 : u_words <= 256 ? 64 : 256; step; step >>= 2) {
          int below = 0;
#pragma unroll
          for (int i = 1; i < 4; ++i) {
            const int at = lo + i * step;
            below += (int)(at < u_words) & (int)(u_base[min(at, u_words - 1)] <= k);
          }
          lo += below * step;
        }
        const uint32_t word = u_bits[lo];
        k -= u_base[lo];
        int pos = 0;
#pragma unroll
        for (int sft = 16; sft >= 1; sft >>= 1) {
          const int c = __popc((word >> pos) & ((1u << sft) - 1u));
          if (k >= c) {
            k -= c;
            pos += sft;
          }
        }
        page = lo * 32 + pos;
      }
      // (page < P <= max_pages: inside the table either way)
      const bool from_lds = page < tab_lds_pages;
      pg_entry = !want ? 0 : (from_lds ? u_tab[page] : ent[page]);
    }
    int ph, nv;
    if constexpr (UNION) {   // the entry of the page just found
      ph = pg_entry & ((1 << kEntryShift) - 1);
      nv = (int)((unsigned)pg_entry >> kEntryShift);
    } else {
      ph = (unsigned)logical < (unsigned)P ? pg_entry : -1;
      nv = max(0, tokens - logical * GP);
    }
    const bool ok = lp < U && (unsigned)ph < (unsigned)kv.num_pages;
    pg_phys = ok ? ph : 0;
    pg_valid = ok ? min(GP, nv) : 0;
  };

  // A 32-token tile is fed to the matrix core as two 16-row halves.  Row i of half h is token
  //   tt(h, i) = 8*(i/4) + 4*h + (i%4)
  // of the tile, so that after the score product lane group qd holds tokens 8*qd .. 8*qd+7
  // (half 0 gives +0..3, half 1 gives +4..7): the 8 k-slots of the second product are 8
  // CONSECUTIVE tokens and its value operand is one 16-byte load from the channel-major page.
  struct Tile {
    bf16x8_t k[2][KS];
    uint4 v[NT];
    int nv[2];   // GP == 16: valid tokens of the tile's two pages; GP == 32: {min(nv,16), max(nv-16,0)}
  };

  // n >= ne asks for a tile that does not exist: the same number of loads is issued (so the
  // count of loads in flight stays a compile-time constant), but all lanes read the first few
  // lines of the pool, which costs a handful of cache hits instead of a tile of traffic.
  auto load_tile = [&](Tile& t, int n, int ne) {
    const bool real = n < ne;
    const int slot = (n * PPT) & 63;
    const bf16_t *k0, *k1, *vp;
    if (GP == 16) {
      const int pa = real ? __builtin_amdgcn_readlane(pg_phys, slot) : 0;
      const int pb = real ? __builtin_amdgcn_readlane(pg_phys, slot + 1) : 0;
      t.nv[0] = real ? __builtin_amdgcn_readlane(pg_valid, slot) : 0;
      t.nv[1] = real ? __builtin_amdgcn_readlane(pg_valid, slot + 1) : 0;
      // lanes l16 < 8 read rows of the first page, the others of the second; row within the page:
      // half 0 -> {0..3, 8..11}, half 1 -> {4..7, 12..15}
      const size_t tk = (size_t)(l16 < 8 ? pa : pb) * sh.Hkv + j;
      const int row0 = real ? 8 * ((l16 >> 2) & 1) + (l16 & 3) : 0;
      k0 = (const bf16_t*)kv.k_pages + tk * (GP * D) + row0 * D;
      k1 = k0 + (real ? 4 * D : 0);
      const size_t tv = (size_t)(qd < 2 ? pa : pb) * sh.Hkv + j;
      vp = (const bf16_t*)kv.v_pages + tv * (GP * D) + (real ? l16 * GP : 0) + 8 * (qd & 1);
    } else {
      const int pa = real ? __builtin_amdgcn_readlane(pg_phys, slot) : 0;
      const int nv = real ? __builtin_amdgcn_readlane(pg_valid, slot) : 0;
      t.nv[0] = nv;
      t.nv[1] = nv;
      const size_t ta = (size_t)pa * sh.Hkv + j;
      const int row0 = real ? 8 * (l16 >> 2) + (l16 & 3) : 0;
      k0 = (const bf16_t*)kv.k_pages + ta * (GP * D) + row0 * D;
      k1 = k0 + (real ? 4 * D : 0);
      vp = (const bf16_t*)kv.v_pages + ta * (GP * D) + (real ? l16 * GP : 0) + 8 * qd;
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      // (streaming loads: a key / value tile is read once per step, and keeping it out of the caches'
      // allocation measured 1 us at C1 and 10 us at C4 per step)
      t.k[0][ks] = __builtin_bit_cast(bf16x8_t, __builtin_nontemporal_load(reinterpret_cast<const u32x4v_t*>(k0 + ks * 32 + qd * 8)));
      t.k[1][ks] = __builtin_bit_cast(bf16x8_t, __builtin_nontemporal_load(reinterpret_cast<const u32x4v_t*>(k1 + ks * 32 + qd * 8)));
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) t.v[nt] = __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4v_t*>(vp + nt * 16 * GP)));
  };

  // Exponentials are taken against a reference point m_run that is allowed to lag the true
  // row maximum by up to kLag (log2 units): the accumulators are rescaled only when a row's
  // maximum overtakes its reference by more than that, which after the first tile is rare.
  // exp2(kLag) = 256 is far inside float / bfloat16 range, and (m_run, l, O) stay consistent.
  constexpr float kLag = 8.0f;

  // all score products of a tile, back to back: S^T = K_tile . Q^T for both 16-row halves
  auto score_products = [&](const bf16x8_t (&k)[2][KS], f32x4_t (&sc)[R][2]) {
#pragma unroll
    for (int mt = 0; mt < R; ++mt) {
      sc[mt][0] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
      sc[mt][1] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        sc[mt][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[0][ks], qf[mt][ks], sc[mt][0], 0, 0, 0);
        sc[mt][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[1][ks], qf[mt][ks], sc[mt][1], 0, 0, 0);
      }
    }
  };

  // softmax update and value products of a tile whose scores are given
  auto softmax_values = [&](Tile& t, f32x4_t (&sc)[R][2], bool first) {
    // valid tokens among this lane's 8 (tile tokens 8*qd .. 8*qd+7)
    int lane_valid;
    bool full;
    if (GP == 16) {
      full = (t.nv[0] == 16) && (t.nv[1] == 16);
      lane_valid = (qd < 2 ? t.nv[0] : t.nv[1]) - 8 * (qd & 1);
    } else {
      full = t.nv[0] == 32;
      lane_valid = t.nv[0] - 8 * qd;
    }
    if (!full) {
      // slots past the end of the sequence may hold anything: clear them in V (0 * NaN = NaN)
      const int cnt = max(0, min(8, lane_valid));
      const uint32_t m0 = cnt >= 2 ? ~0u : (cnt == 1 ? 0xFFFFu : 0u);
      const uint32_t m1 = cnt >= 4 ? ~0u : (cnt == 3 ? 0xFFFFu : 0u);
      const uint32_t m2 = cnt >= 6 ? ~0u : (cnt == 5 ? 0xFFFFu : 0u);
      const uint32_t m3 = cnt >= 8 ? ~0u : (cnt == 7 ? 0xFFFFu : 0u);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        t.v[nt].x &= m0;
        t.v[nt].y &= m1;
        t.v[nt].z &= m2;
        t.v[nt].w &= m3;
      }
    }
    // ---- phase 2: one lazy-rescale decision for the wavefront.  Whether some row's maximum
    // has overtaken its reference by more than kLag is decided from each lane's own maximum
    // (a row's lanes share m_run, and scaling by a positive factor keeps the order, so "some
    // lane exceeds" and "the row maximum exceeds" are the same event); the cross-lane maximum
    // itself is only taken when that happens, which after the first tile is rare.
    // (Every instruction that reads a matrix-core result here is an ordinary compiler-visible
    // one: the wait states such a read needs are inserted by the compiler, which it cannot do
    // for inline assembly.)
    // The scores are used where the matrix core left them (element e of the lane's 8 tokens is
    // sc[mt][e / 4][e % 4]); the test against the reference is one compare per row tile against a
    // threshold in score units, kept up to date with the reference.
    float tm[R];
    bool any_up = false;
#pragma unroll
    for (int mt = 0; mt < R; ++mt) {
      if (!full) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (e >= lane_valid) sc[mt][e >> 2][e & 3] = -INFINITY;
      }
      const f32x4_t a = sc[mt][0], b = sc[mt][1];
      tm[mt] = fmaxf(fmaxf(fmaxf(fmaxf(a[0], a[1]), a[2]), fmaxf(fmaxf(a[3], b[0]), b[1])), fmaxf(b[2], b[3]));
      any_up |= tm[mt] > up_thr[mt];
    }
    if (__any(any_up)) {
      float al[R];
#pragma unroll
      for (int mt = 0; mt < R; ++mt) {
        const float m_cand = max_over_lane_groups(tm[mt]) * scale_log2e;
        const bool up = m_cand > m_run[mt] + kLag;
        const float alpha = up ? fast_exp2(m_run[mt] - m_cand) : 1.0f;
        m_run[mt] = up ? m_cand : m_run[mt];
        up_thr[mt] = (m_run[mt] + kLag) * inv_scale_log2e;
        l_run[mt] *= alpha;
        al[mt] = alpha;
      }
      if (!first) {   // (a wavefront's first tile always gets here, with nothing accumulated yet)
#pragma unroll
        for (int mt = 0; mt < R; ++mt)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) o[mt][nt] *= al[mt];
      }
    }
    // ---- phase 3: numerators as a bfloat16 pair, value products.
    // P = hi + lo with hi = p truncated to its top 16 bits (exact, no conversion) and
    // lo = p - hi rounded: 16 mantissa bits in all.  A single bfloat16 would cost 2^-9 of the
    // spread of V per row, which outlier value channels push past the 2e-2 bound.
    // The hi products of a row tile are issued right after its numerators, so the matrix core
    // works while the vector ALU does the next row tile; all lo products come last, far from
    // the hi product that feeds the same accumulator.
    bf16x8_t p_lo[R];
#pragma unroll
    for (int mt = 0; mt < R; ++mt) {
      const float neg_m = -m_run[mt];
      float p[8], psum = 0.f;
      f32x8_t lo;
      uint32_t pb[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        p[e] = fast_exp2(fmaf(sc[mt][e >> 2][e & 3], scale_log2e, neg_m));
        psum += p[e];
        pb[e] = __float_as_uint(p[e]);
        lo[e] = p[e] - __uint_as_float(pb[e] & 0xFFFF0000u);
      }
      l_run[mt] += psum;
      uint4 hi_bits;
      hi_bits.x = __builtin_amdgcn_perm(pb[1], pb[0], 0x07060302u);
      hi_bits.y = __builtin_amdgcn_perm(pb[3], pb[2], 0x07060302u);
      hi_bits.z = __builtin_amdgcn_perm(pb[5], pb[4], 0x07060302u);
      hi_bits.w = __builtin_amdgcn_perm(pb[7], pb[6], 0x07060302u);
      const bf16x8_t p_hi = __builtin_bit_cast(bf16x8_t, hi_bits);
      p_lo[mt] = __builtin_convertvector(lo, bf16x8_t);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        o[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, t.v[nt]), p_hi, o[mt][nt], 0, 0, 0);
    }
#pragma unroll
    for (int mt = 0; mt < R; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        o[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, t.v[nt]), p_lo[mt], o[mt][nt], 0, 0, 0);
    // Scheduling hint for this region: alternate one matrix instruction with a few vector
    // instructions, so the numerators of the next row tile are computed while the matrix core
    // works on the products of the previous one (one wavefront per SIMD: nobody else would).
#pragma unroll
    for (int i = 0; i < 2 * R * NT; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // 1 MFMA
      __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);   // 3 VALU
    }
  };
  auto compute_tile = [&](Tile& t, bool first) {
    f32x4_t sc[R][2];
    score_products(t.k, sc);
    softmax_values(t, sc, first);
  };

  // ---- main loop: NBUF tile buffers in registers, NBUF-1 tiles of lookahead (how many: see
  // the launcher).  A wavefront has a SIMD to itself, so memory latency is hidden by its own
  // lookahead, not by occupancy.  Every load is issued unconditionally (see load_tile) so that
  // the number of loads in flight at each use is a compile-time constant: a load behind a
  // branch would force a full drain at the join.
  Tile tb[NBUF];
  decode_entries(0);
#pragma unroll
  for (int k = 0; k < NBUF - 1; ++k) load_tile(tb[k], k, min(ntw, TPR));
  __builtin_amdgcn_sched_barrier(0);
  // rows past M, and of tokens that do not exist: zero queries (first wait for them)
#pragma unroll
  for (int mt = 0; mt < R; ++mt) {
    bool keep_row = rb * (R * 16) + mt * 16 + l16 < M;
    if constexpr (!UNION) keep_row &= (unsigned)tok[mt] < (unsigned)sh.B;
    const uint32_t keep = keep_row ? 0xFFFFFFFFu : 0u;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint4 x = __builtin_bit_cast(uint4, qf[mt][ks]);
      x.x &= keep;
      x.y &= keep;
      x.z &= keep;
      x.w &= keep;
      qf[mt][ks] = __builtin_bit_cast(bf16x8_t, x);
    }
  }
  for (int nb = 0; nb < ntw; nb += TPR) {
    const int ne = min(ntw, nb + TPR);
    if (nb > 0) {
      if constexpr (!UNION) {
        logical = listed(list_position(nb));
        fetch_entry();
      }
      decode_entries(nb);
#pragma unroll
      for (int k = 0; k < NBUF - 1; ++k) load_tile(tb[k], nb + k, ne);
    }
    for (int n = nb; n < ne; n += NBUF) {
#pragma unroll
      for (int k = 0; k < NBUF; ++k) {
        load_tile(tb[(k + NBUF - 1) % NBUF], n + k + NBUF - 1, ne);
        if (n + k < ne) compute_tile(tb[k], n + k == 0);
      }
    }
  }

  leave_count();
  // each lane summed its own tokens; rows are spread over the 4 lane groups
#pragma unroll
  for (int mt = 0; mt < R; ++mt) l_run[mt] = sum_over_lane_groups(l_run[mt]);

  const uint32_t item = (uint32_t)head * nchunk + chunk;   // (32 bits hold the rows of all partials)
  if (SPLIT_PAGES) {
    // ---- one-round combine of the 4 wavefronts: wavefront w owns channel tiles {w*NTW ..} of
    // the partial.  Everyone publishes (ref, sum) and the O tiles it does NOT own in LDS (its
    // own stay in registers), then reads the three other wavefronts' versions of its tiles,
    // combines the four in wavefront order and stores its slice.  One barrier; the order is
    // fixed, so is the result.  The register file is indexed by the wavefront number, hence
    // one specialisation per wavefront behind a uniform branch.
    typedef MergeSlot<D, R> Slot;
    constexpr int NTW = NT / 4;   // channel tiles per wavefront
    auto publish = [&](auto wv) {
      constexpr int W = decltype(wv)::value;
      {
        float* so = lds + W * kSlotStride;
        float* sm = so + Slot::kOFloats;
        float* sl = sm + R * 16;
#pragma unroll
        for (int mt = 0; mt < R; ++mt) {
          const int r = mt * 16 + l16;
          if (qd == 0) {
            sm[r] = m_run[mt];
            sl[r] = l_run[mt];
          }
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            if (nt / NTW != W) *reinterpret_cast<f32x4_t*>(so + ((mt * NT + nt) * 64 + lane) * 4) = o[mt][nt];
        }
      }
    };
    auto combine = [&](auto wv) {
      constexpr int W = decltype(wv)::value;
      // all LDS reads of the combine are issued before the first is used
      float mw[R][4], lw[R][4];
      f32x4_t ov[R][NTW][4];
#pragma unroll
      for (int mt = 0; mt < R; ++mt) {
        const int r = mt * 16 + l16;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const float* sm = lds + w * kSlotStride + Slot::kOFloats;
          mw[mt][w] = sm[r];
          lw[mt][w] = sm[R * 16 + r];
#pragma unroll
          for (int k = 0; k < NTW; ++k)
            ov[mt][k][w] = w == W ? o[mt][W * NTW + k]
                                  : *reinterpret_cast<const f32x4_t*>(lds + w * kSlotStride +
                                                                      ((mt * NT + W * NTW + k) * 64 + lane) * 4);
        }
      }
#pragma unroll
      for (int mt = 0; mt < R; ++mt) {
        const float m_all = fmaxf(fmaxf(mw[mt][0], mw[mt][1]), fmaxf(mw[mt][2], mw[mt][3]));
        float wgt[4], l_all = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          wgt[w] = fast_exp2(mw[mt][w] - m_all);
          l_all = fmaf(lw[mt][w], wgt[w], l_all);
        }
        const int rg = mt * 16 + l16;
        if (rg < M) {
          const uint32_t prow = item * part.rows + rg;
          if (W == 0 && qd == 0) {
            // (streaming stores: the partials are read once, by the next launch; leaving them out of the
            // caches' write-back at the kernel's end measured 0.3 us per step at 48 MB launches)
            __builtin_nontemporal_store(m_all, &part.m[prow]);
            __builtin_nontemporal_store(l_all, &part.l[prow]);
          }
#pragma unroll
          for (int k = 0; k < NTW; ++k) {
            f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < 4; ++w) acc += ov[mt][k][w] * wgt[w];
            __builtin_nontemporal_store(acc, reinterpret_cast<f32x4_t*>(part.o + (size_t)prow * D + (W * NTW + k) * 16 + qd * 4));
          }
        }
      }
    };
    switch (wave) {
      case 0: publish(std::integral_constant<int, 0>{}); break;
      case 1: publish(std::integral_constant<int, 1>{}); break;
      case 2: publish(std::integral_constant<int, 2>{}); break;
      default: publish(std::integral_constant<int, 3>{}); break;
    }
    __syncthreads();
    switch (wave) {
      case 0: combine(std::integral_constant<int, 0>{}); break;
      case 1: combine(std::integral_constant<int, 1>{}); break;
      case 2: combine(std::integral_constant<int, 2>{}); break;
      default: combine(std::integral_constant<int, 3>{}); break;
    }
    return;
  }

  // ---- partial of this (sequence, head, chunk): un-normalised O, running max (log2 units), sum
#pragma unroll
  for (int mt = 0; mt < R; ++mt) {
    const int rg = rb * (R * 16) + mt * 16 + l16;
    if (rg < M) {
      const uint32_t prow = item * part.rows + rg;
      if (qd == 0) {
        part.m[prow] = m_run[mt];
        part.l[prow] = l_run[mt];
      }
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        *reinterpret_cast<f32x4_t*>(part.o + (size_t)prow * D + nt * 16 + qd * 4) = o[mt][nt];
    }
  }
}

// The leading arguments (see KvView) put where the code reads them: union bitmap, entries and words per head; or list,
// counts and capacity.
template <bool UNION>
__device__ __forceinline__ void take_leading(Address first, Address second, Address active_count, Address page_indptr,
                                             Address seq_lens, int stride, int copy_words, int max_pages, int kv_heads, AttnInputs& in,
                                             Shape& sh, KvView& kv, UnionInKernel& uni) {
  in.active_count = pointer<const int32_t>(active_count);
  kv.page_indptr = pointer<const int32_t>(page_indptr);
  kv.seq_lens = pointer<const int32_t>(seq_lens);
  sh.max_pages = max_pages;
  sh.Hkv = kv_heads;
  if constexpr (UNION) {
    uni.bits = pointer<const uint32_t>(first);
    uni.entries = pointer<const int32_t>(second);
    uni.stride = stride;
    uni.copy_words = copy_words;
  } else {
    in.list = pointer<const int32_t>(first);
    in.sel_count = pointer<const int32_t>(second);
    in.cap = stride;
  }
}

template <int D, int GP, int R, bool SPLIT_PAGES, int NBUF, bool UNION = false>
__global__ __launch_bounds__(256) void attn_mfma_kernel(Address first, Address second, Address active_count, Address page_indptr, Address seq_lens,
                                                        int stride, int copy_words, int max_pages, int kv_heads, AttnInputs in,
                                                        int nchunk, int nrbg, Shape sh, KvView kv,
                                                        Partials part, float scale_log2e, int m_lo, int m_hi,
                                                        UnionInKernel uni) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  take_leading<UNION>(first, second, active_count, page_indptr, seq_lens, stride, copy_words, max_pages, kv_heads, in, sh, kv, uni);
  attn_mfma_body<D, GP, R, SPLIT_PAGES, NBUF, UNION>(in, nchunk, nrbg, sh, kv, part, scale_log2e,
                                                                            m_lo, m_hi, uni, lds);
}

// The split-pages shape for launches whose row counts only the device knows (threshold / cumulative-mass selection, the
// separate calls): every (sequence, KV head) runs the body
// compiled for its own number of 16-row tiles, read from the count the selection left, so that a
// head with a few active rows does not pay for the 64 the launch has to allow.  Heads with more than
// 64 rows are not served here.
template <int D, int GP, bool UNION>
__global__ __launch_bounds__(256) void attn_mfma_rows_kernel(Address first, Address second, Address active_count, Address page_indptr, Address seq_lens,
                                                             int stride, int copy_words, int max_pages, int kv_heads, AttnInputs in,
                                                             int nchunk, Shape sh, KvView kv, Partials part,
                                                             float scale_log2e, int m_lo, int m_hi, UnionInKernel uni) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  take_leading<UNION>(first, second, active_count, page_indptr, seq_lens, stride, copy_words, max_pages, kv_heads, in, sh, kv, uni);
  const int M = active_rows(in, kv, sh, blockIdx.z);
  if (M <= 0 || M > kUnionRows) return;
  if (M <= 16)
    attn_mfma_body<D, GP, 1, true, 2, UNION>(in, nchunk, 1, sh, kv, part, scale_log2e, m_lo, m_hi, uni, lds);
  else if (M <= 32)
    attn_mfma_body<D, GP, 2, true, 2, UNION>(in, nchunk, 1, sh, kv, part, scale_log2e, m_lo, m_hi, uni, lds);
  else if (M <= 48)
    attn_mfma_body<D, GP, 3, true, 2, UNION>(in, nchunk, 1, sh, kv, part, scale_log2e, m_lo, m_hi, uni, lds);
  else
    attn_mfma_body<D, GP, 4, true, 2, UNION>(in, nchunk, 1, sh, kv, part, scale_log2e, m_lo, m_hi, uni, lds);
}

template <int D, int GP, int R, bool SPLIT, bool UNION = false>
static hipError_t launch_one(hipStream_t st, const KvView& kv, const Shape& sh, int batch, const AttnInputs& in,
                             int nchunk, const Partials& part, hipEvent_t ev_start, hipEvent_t ev_stop, int m_lo,
                             int m_hi, const UnionInKernel& uni = UnionInKernel{nullptr}) {
  const int nrbg = SPLIT ? 1 : (sh.rows_max + R * 64 - 1) / (R * 64);
  const size_t lds_bytes = SPLIT ? (4 * MergeSlot<D, R>::kFloats + (UNION ? kUnionShared : 0)) * sizeof(float)
                                 : 0;
  // Tile buffers per wavefront (one is being computed on, the others are in flight).  The sparse
  // shape wants exactly one tile of lookahead: with more, every wavefront has its whole share
  // of the list requested at once, the memory system completes those requests in no useful
  // order, and the first tile of every wavefront lands only near the end of the stream, so
  // nothing is left to overlap the arithmetic with (C1: 17.9 us with 3 tiles of lookahead,
  // 15.2 us with 1).  The dense shape has arithmetic to hide behind and keeps a deeper queue.
  constexpr int NBUF = SPLIT ? 2 : ((D == 128 && R == 4) ? 3 : 4);
  auto kern = attn_mfma_kernel<D, GP, R, SPLIT, NBUF, UNION>;
  static bool attr_set = false;   // per instantiation
  if (lds_bytes > 48 * 1024 && !attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds_bytes);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const float scale_log2e = sh.sm_scale * 1.4426950408889634f;
  dim3 grid(nchunk, sh.Hkv * nrbg, batch);
  if (ev_start && ev_stop)   // events bound to this dispatch: they read the kernel's own begin and end
    hipExtLaunchKernelGGL(kern, grid, dim3(256), (uint32_t)lds_bytes, st, ev_start, ev_stop, 0, address(UNION ? (const void*)uni.bits : in.list), address(UNION ? uni.entries : in.sel_count), address(in.active_count),
                          address(kv.page_indptr), address(kv.seq_lens),
                          UNION ? uni.stride : in.cap, uni.copy_words, sh.max_pages, sh.Hkv, in, nchunk,
                          nrbg, sh, kv, part, scale_log2e, m_lo, m_hi, uni);
  else
    kern<<<grid, 256, lds_bytes, st>>>(address(UNION ? (const void*)uni.bits : in.list), address(UNION ? uni.entries : in.sel_count), address(in.active_count),
                          address(kv.page_indptr), address(kv.seq_lens),
                          UNION ? uni.stride : in.cap, uni.copy_words, sh.max_pages, sh.Hkv, in, nchunk, nrbg, sh, kv, part, scale_log2e, m_lo, m_hi, uni);
  return hipGetLastError();
}

// rows_on_device: launch the form that takes every head's row-tile count from the device.
// More than 64 rows: 4 independent wavefronts of 64 rows.
template <int D, int GP>
static hipError_t launch_dg(hipStream_t st, const KvView& kv, const Shape& sh, int batch, const AttnInputs& in,
                            int nchunk, int rows_upper, const Partials& part, hipEvent_t e0, hipEvent_t e1, int m_lo,
                            int m_hi, bool rows_on_device, const UnionInKernel* uni) {
  if (rows_on_device) {
    auto launch = [&](auto kern, size_t lds_bytes, bool& attr_set) -> hipError_t {
      if (lds_bytes > 48 * 1024 && !attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)lds_bytes);
        if (e != hipSuccess) return e;
        attr_set = true;
      }
      const dim3 grid(nchunk, sh.Hkv, batch);
      const float scale_log2e = sh.sm_scale * 1.4426950408889634f;
      const UnionInKernel u = uni ? *uni : UnionInKernel{nullptr};
      if (e0 && e1)   // events bound to this dispatch, as in launch_one
        hipExtLaunchKernelGGL(kern, grid, dim3(256), (uint32_t)lds_bytes, st, e0, e1, 0, address(uni ? (const void*)u.bits : in.list), address(uni ? u.entries : in.sel_count), address(in.active_count),
                              address(kv.page_indptr), address(kv.seq_lens),
                              uni ? u.stride : in.cap, u.copy_words, sh.max_pages, sh.Hkv, in, nchunk, sh, kv, part, scale_log2e, m_lo,
                              m_hi, u);
      else
        kern<<<grid, 256, lds_bytes, st>>>(address(uni ? (const void*)u.bits : in.list), address(uni ? u.entries : in.sel_count), address(in.active_count),
                              address(kv.page_indptr), address(kv.seq_lens),
                              uni ? u.stride : in.cap, u.copy_words, sh.max_pages, sh.Hkv, in, nchunk, sh, kv, part, scale_log2e, m_lo, m_hi, u);
      return hipGetLastError();
    };
    constexpr size_t slots = 4 * MergeSlot<D, 4>::kFloats;
    static bool with_union = false, with_list = false;   // (attribute set) per instantiation
    return uni ? launch(attn_mfma_rows_kernel<D, GP, true>, (slots + kUnionShared) * sizeof(float), with_union)
               : launch(attn_mfma_rows_kernel<D, GP, false>, slots * sizeof(float), with_list);
  }
  if (uni && uni->bits) {   // the kernel ranks the head's union bitmap itself
    if (rows_upper <= 16) return launch_one<D, GP, 1, true, true>(st, kv, sh, batch, in, nchunk, part, e0, e1, m_lo, m_hi, *uni);
    if (rows_upper <= 32) return launch_one<D, GP, 2, true, true>(st, kv, sh, batch, in, nchunk, part, e0, e1, m_lo, m_hi, *uni);
    if (rows_upper <= 48) return launch_one<D, GP, 3, true, true>(st, kv, sh, batch, in, nchunk, part, e0, e1, m_lo, m_hi, *uni);
    if (rows_upper <= 64) return launch_one<D, GP, 4, true, true>(st, kv, sh, batch, in, nchunk, part, e0, e1, m_lo, m_hi, *uni);
    return hipErrorInvalidValue;
  }
  if (rows_upper <= 16) return launch_one<D, GP, 1, true>(st, kv, sh, batch, in, nchunk, part, e0, e1, m_lo, m_hi);
  if (rows_upper <= 32) return launch_one<D, GP, 2, true>(st, kv, sh, batch, in, nchunk, part, e0, e1, m_lo, m_hi);
  if (rows_upper <= 48) return launch_one<D, GP, 3, true>(st, kv, sh, batch, in, nchunk, part, e0, e1, m_lo, m_hi);
  if (rows_upper <= 64) return launch_one<D, GP, 4, true>(st, kv, sh, batch, in, nchunk, part, e0, e1, m_lo, m_hi);
  return launch_one<D, GP, 4, false>(st, kv, sh, batch, in, nchunk, part, e0, e1, m_lo, m_hi);
}

hipError_t launch_attn_mfma(hipStream_t st, const KvView& kv, const Shape& sh, int batch, const AttnInputs& in,
                            int nchunk, int rows_upper, const Partials& part, hipEvent_t e0, hipEvent_t e1, int m_lo,
                            int m_hi, bool rows_on_device, const UnionInKernel* uni) {
  if (batch <= 0 || nchunk <= 0) return hipSuccess;
  if (sh.d == 128) {
    if (sh.g == 16) return launch_dg<128, 16>(st, kv, sh, batch, in, nchunk, rows_upper, part, e0, e1, m_lo, m_hi, rows_on_device, uni);
    return launch_dg<128, 32>(st, kv, sh, batch, in, nchunk, rows_upper, part, e0, e1, m_lo, m_hi, rows_on_device, uni);
  }
  if (sh.g == 16) return launch_dg<64, 16>(st, kv, sh, batch, in, nchunk, rows_upper, part, e0, e1, m_lo, m_hi, rows_on_device, uni);
  return launch_dg<64, 32>(st, kv, sh, batch, in, nchunk, rows_upper, part, e0, e1, m_lo, m_hi, rows_on_device, uni);
}

}  // namespace losa
