// Internal declarations shared by the translation units of liblosa.so.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "losa.h"

namespace losa {

constexpr int kWave = 64;

// Device view of the ragged page table, passed to kernels by value.
// What a kernel's first loads need (page_indptr, seq_lens, counts, strides) also comes as plain arguments ahead of the structs, and the
// kernel puts it back into them: up to 14 dwords of leading plain arguments arrive in scalar registers with the wavefront
// (kernarg preloading, a compiler option of the build), a struct is always fetched, one scalar round trip before the first load can
// leave.  A step of 42 rows x 4 heads over 32768 tokens 31.78 -> 31.37 us, 16 sequences 115.5 -> 114.5, a block of 16 steps 581 -> 571.  (Not
// the page bounds, which gain nothing: more arguments cost the host 0.2 us a launch where it is what limits.)
struct KvView {
  const void* k_pages;
  const void* v_pages;
  void* meta;
  const int32_t* page_indptr;
  const int32_t* page_indices;
  const int32_t* seq_lens;
  int32_t num_pages;
  int32_t seq_page_limit;   // the host's upper bound on pages per sequence (grids and register tiles are sized by it)
};

// An address among a kernel's leading arguments.  The runtime looks every plain pointer argument up among its allocations at every
// launch; an integer it copies: 10 leading arguments with 5 pointers took 0.25 us of the host's time a launch, with 5 integers none that
// shows, and a step of few heads is issued no faster than it runs.
typedef uint64_t Address;
inline Address address(const void* p) { return (Address)(uintptr_t)p; }
template <typename T>
__device__ __forceinline__ T* pointer(Address a) {   // (through the global address space: a bare conversion would make every access a flat one)
  return (T*)(__attribute__((address_space(1))) T*)a;
}

// Static problem shape, passed to kernels by value.
struct Shape {
  int32_t max_pages;   // row stride of the score matrix / bitmap sizing (config.max_pages_per_seq)
  int32_t rows_max;    // B * G: rows of one KV head when every token is active
  int32_t g;           // (beside the two above, which are fetched with it)
  int32_t Hkv, Hq, G, d, H, B;
  float sm_scale;
  uint32_t g_magic;    // ceil(2^32 / G), for row_token()
};
// r / G for a query row r of a KV head (r < 4096 and G <= 4096, so the reciprocal rounded up is exact).
__device__ __forceinline__ int row_token(const Shape& sh, int r) {
  return sh.G == 1 ? r : (int)__umulhi((uint32_t)r, sh.g_magic);
}

// Pages of sequence b that the kernels look at: those the page table lists, that hold at least
// one of the sequence's tokens (a table may list pages reserved ahead of the tokens: their
// metadata was never written), and that the launch was sized for.
__device__ __forceinline__ int seq_pages(const KvView& kv, const Shape& sh, int b) {
  const int listed = kv.page_indptr[b + 1] - kv.page_indptr[b];
  const int filled = (kv.seq_lens[b] + sh.g - 1) >> (sh.g == 16 ? 4 : 5);   // g is 16 or 32
  return max(0, min(min(listed, filled), min(sh.max_pages, kv.seq_page_limit)));
}

// The same with what else is read of the page table, in one scalar round trip: the empty asm keeps the three loads ahead of
// whatever tests one of them (not a volatile one: loads behind that are vector loads).  (Kernel arguments and counts are kept together the same way: left alone, each is fetched
// where it is used, and a kernel of a few microseconds walked through four to six scalar round trips one after the other.)
struct Sequence {
  int base, tokens, pages;   // first entry of the page table, prefix length, seq_pages()
};
__device__ __forceinline__ Sequence sequence(const KvView& kv, const Shape& sh, int b) {
  int base = __builtin_amdgcn_readfirstlane(kv.page_indptr[b]), end = __builtin_amdgcn_readfirstlane(kv.page_indptr[b + 1]);
  int tokens = __builtin_amdgcn_readfirstlane(kv.seq_lens[b]);
  asm("" : "+s"(base), "+s"(end), "+s"(tokens) : "s"(sh.g), "s"(sh.max_pages), "s"(kv.seq_page_limit));
  const int filled = (tokens + sh.g - 1) >> (sh.g == 16 ? 4 : 5);
  return {base, tokens, max(0, min(min(end - base, filled), min(sh.max_pages, kv.seq_page_limit)))};
}

// Split-K partials of the attention: item = ((b*Hkv + j)*nchunk + c), row r < rows.
struct Partials {
  float* o;   // [items, rows, d]   un-normalised sum_t exp(s_t - m) v_t
  float* m;   // [items, rows]      running max of the scaled scores
  float* l;   // [items, rows]      sum_t exp(s_t - m)
  int rows;   // rows per item in this launch: an upper bound on the query rows of a KV head
};

// What the attention kernels read besides keys and values.
struct AttnInputs {
  const void* q;                 // [batch*B, Hq, d]
  const int32_t* active_idx;     // [batch, B] token of every active slot, active_count [batch]; both NULL: every token
  const int32_t* active_count;
  const int32_t* list;           // [heads, cap] logical pages, sel_count [heads] of them; NULL: every page, or the union below
  const int32_t* sel_count;
  int cap;
};
// Query rows of a KV head of sequence b.  (A load behind a branch would wait for what the branch tests and hold up what
// follows: the address is chosen instead, any valid one where there is no count.)
__device__ __forceinline__ int active_rows(const AttnInputs& in, const KvView& kv, const Shape& sh, int b) {
  const int n = (in.active_count ? in.active_count : kv.seq_lens)[b];
  return (in.active_count ? min(n, sh.B) : sh.B) * sh.G;
}
constexpr int kEntryShift = 26;   // entry = physical page id | (valid tokens << 26)
// The other way the matrix-core kernels can get their pages (sparse steps of losa_step): the selection workgroups OR
// their row's picks into one bitmap per head, and every attention workgroup ranks that union and resolves its own pages
// itself while it starts up.  That takes the selection kernel's serial tail (bitmap hand-over to one
// workgroup per head, union, list) out of the chain of launches.
constexpr int kUnionRows = 64;   // the most rows the split-pages shape serves
struct UnionInKernel {
  const uint32_t* bits;      // [heads][union_words()] union of the head's picks, in copies; NULL: no union
  const int32_t* entries;    // [heads, max_pages] the head's page table as entries, by logical page
  const uint16_t* q_act;     // [heads, rows_max, d] bfloat16: query rows of the active tokens, gathered
  int32_t* sel_count;        // [heads] out: pages in the union (written by the head's first workgroup)
  int stride, copy_words, copies;   // union_words(), union_copy_words(), union_copies()
};
// A head's union bitmap.  The rows' atomics on one word come one after the other (34 ns each), so it is kept in copies.  Up
// to 1024 pages, where all rows fall on the same few words, row r goes to copy r mod their number, and they fill
// kUnionSpread words (2 x 378-728 tokens, 32 rows: selection 7.4 us with one copy, 6.3 with 16; where a row
// does not OR at all, 6.3).  The split-pages kernel reads all of them with the four loads it has for 8192 pages.
// Beyond, the words are many enough for that kernel's rows (at 2048 pages four copies cost 0.5 us more than they
// save, 4 x 65536 tokens), and every further 64 rows get a copy of their own, up to eight.
constexpr int kUnionSpread = 256;
constexpr int kMostCopiedWords = 32;
// words of one copy, for the pages the launch was sized for (KvView::seq_page_limit)
__host__ __device__ inline int union_copy_words(int pages) {
  const int words = (pages + 31) / 32;
  return words <= 16 ? 16 : words <= kMostCopiedWords ? kMostCopiedWords : (words + 3) & ~3;
}
// their number (a power of two) for heads of up to `rows` rows, and the shift that makes a row its copy
__host__ __device__ inline int union_copies(int copy_words, int rows) {
  if (copy_words <= kMostCopiedWords) return kUnionSpread / copy_words;
  return rows <= kUnionRows ? 1 : rows <= 2 * kUnionRows ? 2 : rows <= 4 * kUnionRows ? 4 : 8;
}
__host__ __device__ inline int union_row_shift(int copy_words) { return copy_words <= kMostCopiedWords ? 0 : 6; }
// words per head, whatever the launch
__host__ __device__ inline int union_words(int max_pages, int rows_max) {
  const int copy_words = union_copy_words(max_pages), words = copy_words * union_copies(copy_words, rows_max);
  return words > kUnionSpread ? words : kUnionSpread;
}

// ---- losa_api.hip
// Sets `n` ints to zero with a small fill kernel (safe to record into a captured graph).
hipError_t launch_zero_ints(hipStream_t st, int32_t* p, int n);
// Records the error text losa_last_error(NULL) returns on this thread; returns `st`.
losa_status set_thread_error(losa_status st, const char* fmt, ...);

// ---- select_active.hip
// fused: score per token + ranking by the last workgroup of each sequence (tickets: [batch] ints, zero on entry)
hipError_t launch_locality_select(hipStream_t st, int dtype, const void* h_cur, const void* h_prev, int batch, int B,
                                  int H, int mode, int n, float tau, float* delta, uint8_t* mask, int32_t* active_idx,
                                  int32_t* active_count, int32_t* tickets);
// One shared page set per (sequence, KV head): top pages of the scores max-reduced over the head's rows.
hipError_t launch_shared_select(hipStream_t st, const KvView& kv, const Shape& sh, int batch, int max_seq_pages,
                                const int32_t* active_count, const float* scores, int topk, int32_t* sel_pages,
                                int32_t* sel_count, int cap);
// Locality scores only (no ranking): for the step whose scoring kernel ranks them itself.
hipError_t launch_locality_delta(hipStream_t st, int dtype, const void* h_cur, const void* h_prev, int batch, int B,
                                 int H, float* delta);

// ---- page_bounds.hip
hipError_t launch_page_bounds(hipStream_t st, int dtype, const KvView& kv, const Shape& sh, int batch,
                              int first_page, int num_pages_in_range);

// ---- score_pages.hip
constexpr int kMaxSelectPages = 1024 * 16;   // pages per sequence the register-resident top-k handles
// ranking != NULL (bfloat16, B <= 256): the scoring workgroups derive the
// active set from `delta` themselves and write mask / active_idx / active_count; the active_idx /
// active_count arguments are then outputs of this launch, not inputs.
struct InKernelRanking {
  const float* delta;
  int mode, n;
  float tau;
  uint8_t* mask;
  int32_t* active_idx;
  int32_t* active_count;
};
hipError_t launch_page_scores(hipStream_t st, int dtype, const KvView& kv, const Shape& sh, int batch, int max_seq_pages,
                              const void* q, const int32_t* active_idx, const int32_t* active_count,
                              float* scores, int32_t* tickets, int32_t* sel_count, int32_t* entries, uint16_t* q_act, int rows_upper,
                              const InKernelRanking* ranking, long workgroups_per_round, uint32_t* union_bits = nullptr);
hipError_t launch_select_pages(hipStream_t st, const KvView& kv, const Shape& sh, int batch, int max_seq_pages,
                               const int32_t* active_count, const float* scores, int topk, int32_t* topk_out,
                               int32_t* sel_pages, int32_t* sel_count, int cap, uint32_t* rowmaps, int32_t* tickets,
                               int rows_hint, long workgroups_per_round,
                               uint32_t* union_bits = nullptr);

// Scoring and selection of short prefixes in one launch, which also takes the locality scores' place where a hidden state is short.
// pick_pages_serves: whether it takes a step of `rows` active rows per KV head (rows_known; else up to that many).  It ranks as `ranking` says (delta is read only
// without h_cur / h_prev) and leaves what the scoring kernel would for the attention, and the union bitmap complete.
constexpr int kPickPages = 512;      // pages per sequence
constexpr int kPickRows = 16;        // query rows per workgroup
constexpr int kPickMostRows = 256;   // ... and per KV head: a copy of the union bitmap for each 16
bool pick_pages_serves(const Shape& sh, int batch, int max_seq_pages, int rows, bool rows_known);
// ... and whether it scores the tokens too: hidden states of up to 64 16-byte pieces, a wavefront's one load, which is what toy and test
// models have (a model's thousands of channels take the launch of their own).  2048 workgroups of 64 tokens of 512 channels each,
// read by all of them, cost nothing that shows: 1024 tokens, 16 sequences, 8 heads of 256 rows 63.0 us with 64 channels, 63.7 with 512.
inline bool pick_takes_hidden(const Shape& sh) { return sh.H <= 512; }
hipError_t launch_pick_pages(hipStream_t st, const KvView& kv, const Shape& sh, int batch, int max_seq_pages, const void* q, const void* h_cur,
                             const void* h_prev, int rows, int topk, int32_t* tickets, int32_t* sel_count, int32_t* entries, uint16_t* q_act,
                             const InKernelRanking& ranking, uint32_t* union_bits);

// ---- sparse_attn.hip (float mode, merge) and sparse_attn_mfma.hip (bfloat16)
// Tiles of a (sequence, KV head) page list are dealt round-robin to `nchunk` work items: tiles of 32 tokens
// (bfloat16), single pages (float mode).  launch_attn_merge: bf16 means bfloat16 partials.
hipError_t launch_attn_f32(hipStream_t st, const KvView& kv, const Shape& sh, int batch, const void* q,
                           const int32_t* active_idx, const int32_t* active_count, const int32_t* sel_pages,
                           const int32_t* sel_count, int cap, int nchunk, const Partials& part);
// e0/e1 (both or neither): events bound to the dispatch itself, for exact kernel timing.
hipError_t launch_attn_mfma(hipStream_t st, const KvView& kv, const Shape& sh, int batch, const AttnInputs& in,
                            int nchunk, int rows_upper, const Partials& part, hipEvent_t e0, hipEvent_t e1,
                            int m_lo = 0, int m_hi = 0x7fffffff,   // serves (sequence, head) pairs with m_lo < rows <= m_hi
                            bool rows_on_device = false, const UnionInKernel* uni = nullptr);   // ... up to 64, counted on the device
// sparse_attn_rows.hip: more than 64 query rows per KV head, eight wavefronts sharing stages of kManyRowStage
// tokens through LDS; serves (sequence, head) pairs with more than m_lo rows.  Its partials are laid out by
// fragments: per 32 rows (kPartialTile; part.rows is a multiple of it) and 8 channels, 64 lanes x 4 floats,
// lane = row of the tile + 32 * (second half of the 8 channels).
constexpr int kManyRowStage = 64;
constexpr int kPartialTile = 32;
hipError_t launch_attn_rows(hipStream_t st, const KvView& kv, const Shape& sh, int batch, const AttnInputs& in, int nchunk,
                            const Partials& part, hipEvent_t e0, hipEvent_t e1, int m_lo, bool half_values, int upper,
                            const UnionInKernel* uni);   // upper: the most pages a head can have
// few_tile / many_tile: tokens per tile that the partials of a head with at most / more than 64 query rows were
// dealt in (they decide which of the nchunk work items exist); kManyRowStage: partials laid out by fragments.
hipError_t launch_attn_merge(hipStream_t st, const KvView& kv, const Shape& sh, int batch, const AttnInputs& in,
                             bool bf16, int nchunk, const Partials& part, float* o_p, float* lse_p, int rows_hint, int few_tile, int many_tile);

// ---- block_merge.hip
hipError_t launch_block_merge(hipStream_t st, int dtype, const Shape& sh, int batch, const void* q, const void* k_b,
                              const void* v_b, const float* o_p, const float* lse_p, float* out, float* o_b,
                              float* lse_b);

}  // namespace losa
