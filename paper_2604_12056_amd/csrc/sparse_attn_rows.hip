// Split-K paged prefix attention for more than 64 query rows per KV head (the dense initialisation and
// large active sets), bfloat16 inputs, on the 32x32x16 matrix instructions of gfx950
// (paper: Preliminaries, Attention Decomposition With Online Softmax; Methodology, eq. update_rule).
//
// Eight wavefronts of 32 query rows walk the same stages of 64 tokens:
//
//   S^T = K . Q^T        A operand: 32 keys x 16 channels from LDS, B operand: the queries, in registers
//   O^T += V^T . P^T     A operand: 32 channels x 16 tokens from LDS, B operand: P^T, which is how the
//                        numerators of S^T lie in the registers already (lane = query row): nothing
//                        crosses lanes.
//
// Why 32x32x16 and not 16x16x32: both do 1024 flop per cycle and SIMD, but a 32x32x16 product holds the
// matrix pipe for 32 cycles at one issue slot, which leaves room behind it for about six vector
// instructions instead of two, and a tile of 32 rows x 32 tokens needs half as many instructions.  The
// softmax of a tile (16 fma, 16 exp2, conversions, sums) can then run under its 16 products.
//
// Token order.  A 32x32 result holds, per lane, rows 8*b + 4*half + e (b, e = 0..3; half = lane / 32).
// Key row m of a 32-token block is token swap(m), where swap exchanges bits 2 and 3: the lane's registers
// 8*s .. 8*s+7 are then the CONSECUTIVE tokens 16*s + 8*half .. +7, which is the B operand of k-step s
// of the second product, and its A operand is one 16-byte piece of a channel-major value page.
//
// What bounds it.  At 256 rows matrix products, exponentials, LDS traffic and the HBM stream each take time
// that adds up: of 545 thousand cycles for 256 rows over 4 x 65536 tokens the matrix cores are busy 0.48, the vector ALUs'
// issue port 0.49, both at once 0.17.  At up to 128 rows it runs at the HBM stream (5 TB/s).  Scheduling
// hints (interleaving products with vector instructions) and wavefront priorities were measured and
// change nothing.  Whole dense step against the kernel on 16x16x32 products with LDS tiles of 32 tokens:
// 4 x 65536 tokens, 8 KV heads, 256 rows 363 -> 329 us; the sparse step of 128 rows over 0.68 of 4 x 65536
// tokens 230 -> 189 us (both with the normaliser's own sum, 2 % of the kernel).
//
// Memory to LDS.  A stage's keys and values are fetched once per workgroup with perfectly linear 16-byte
// streaming loads (a page-head tile is contiguous; without the streaming hint +5%), two stages ahead in
// registers, and the permutation into operand order happens in the LDS write address.  Pieces lie in strips of 32 (one per row or channel of
// an operand) whose strides (kKeyStrip, kValStrip) are offset by 16 / 32 / 64 bytes from a multiple of the
// bank width, so that the eight lanes of a write or read phase always hit different banks.
#include <hip/hip_ext.h>
#include <math.h>

#include <type_traits>

#include "losa_device.h"
#include "losa_internal.h"

namespace losa {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(8))) float f32x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8_t;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2_t;
typedef uint32_t u32x4v_t __attribute__((ext_vector_type(4)));   // a plain vector value (stays in registers)

constexpr int kRowsPerWave = 32;
constexpr int kRowWaves = 8;
constexpr int kRowGroup = kRowsPerWave * kRowWaves;   // query rows one workgroup serves
constexpr float kNoReference = -1.0e30f;              // finite stand-in for "no token seen yet"

constexpr int kImages = 3;                            // stages in LDS at a time

template <int D, int GP>
struct StageImage {   // LDS image of one 64-token stage: two 32-token blocks of keys, then two of values
  static constexpr int kTokens = kManyRowStage;
  static constexpr int kPages = kTokens / GP;
  static constexpr int kKeyStrip = 32 * 16 + 16;                      // 32 keys x one 16-byte channel piece
  static constexpr int kKeyBlock = (D / 8) * kKeyStrip;
  static constexpr int kValStrip = 32 * 16 + (GP == 32 ? 32 : 64);    // 32 channels x one 8-token piece
  static constexpr int kValBlock = (D / 32) * 4 * kValStrip;
  static constexpr int kValBase = 2 * kKeyBlock;
  static constexpr int kBytes = 2 * (kKeyBlock + kValBlock);
};

// bfloat16 pair -> half pair, towards zero: exact inside the half range, never infinite
__device__ __forceinline__ uint32_t bf16_pair_to_half(uint32_t two_bf16) {
  const auto h = __builtin_amdgcn_cvt_pkrtz(__uint_as_float(two_bf16 << 16), __uint_as_float(two_bf16 & 0xFFFF0000u));
  return __builtin_bit_cast(uint32_t, h);
}

// Where a workgroup's pages come from: the whole page table (the dense step), a list of logical pages, or the head's
// union bitmap, out of which it has made its own list.
enum class PageSource { all, list, own };

// HALF: the value product runs in half precision.  Values are converted bfloat16 -> half while they are
// staged (exact for 2^-14 <= |v| <= 65504, truncated towards zero below that range and held at +-65504
// above it), the numerators enter as ONE half-precision operand (11 significant bits, round to nearest).
// The reference of the exponentials then sits 7 (log2 units) below where it would otherwise be, so that
// the numerators use the upper end of the half-precision range.  O is normalised with the sum of the ROUNDED
// numerators, the weights it was made with: what the roundings have in common cancels, so a row that one
// token dominates and a channel whose values are alike come out exact (with the unrounded sum they are off by up
// to 2^-11 of the value).  The log-sum-exp and the weight of a chunk among chunks take the unrounded sum.
// Otherwise P is a bfloat16 pair hi + lo and values stay bfloat16.
//
// TG token groups: with up to 128 rows four wavefronts hold all of them, and the other four take the
// second 32-token block of every stage instead of idling; the two halves meet through LDS at the end.
template <int D, int GP, bool HALF, int TG, PageSource SRC>
__device__ __forceinline__ void attn_rows_body(int nchunk, int row_group, int j, const Shape& sh,
                                               const KvView& kv, const Partials& part, float scale_log2e, int M, int U, const Sequence& seq,
                                               const AttnInputs& in, const uint16_t* own, int logical, int entry, unsigned char* lds) {
  typedef StageImage<D, GP> Img;
  constexpr int KS = D / 16;            // k-steps of the score product
  constexpr int CB = D / 32;            // 32-channel blocks of the output
  constexpr int PPS = Img::kPages;      // pages per stage
  constexpr int SPF = 64 / PPS;         // stages covered by one fetch of page entries (one entry per lane)
  constexpr int NP = Img::kTokens * D / 8 / 512;   // 16-byte pieces of keys (and of values) per thread and stage
  constexpr int PPP = GP * D / 8;       // pieces per page
  constexpr int NB = 2 / TG;            // 32-token blocks of a stage this wavefront computes on
  constexpr int PD = 2;                 // stages in flight in registers
  static_assert(PPP % 64 == 0, "a wavefront's pieces come from one page");

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int b = blockIdx.z, chunk = blockIdx.x, head = b * sh.Hkv + j;
  const int row_wave = TG == 1 ? wave : wave & 3, block0 = TG == 1 ? 0 : wave >> 2;
  const int r0 = row_group * kRowGroup + row_wave * kRowsPerWave;
  const bool has_rows = r0 < M;
  const int nstages_all = (U + PPS - 1) / PPS;
  const int ns = (nstages_all - 1 - chunk) / nchunk + 1;   // stages of this workgroup: chunk, chunk + nchunk, ... (chunk < nstages_all)

  // Page entries, one per lane and batch of SPF stages: position in the list -> logical page -> page table, each step
  // requested a stage before the next needs it.
  int next_logical = logical, next_entry = entry, pg_phys = 0, pg_valid = 0;
  const int32_t* table = kv.page_indices + seq.base;
  const int tokens = seq.tokens, P = seq.pages;
  auto list_position = [&](int first_stage) {
    return ((long)chunk + (long)(first_stage + lane / PPS) * nchunk) * PPS + lane % PPS;
  };
  [[maybe_unused]] auto fetch_logical = [&](int first_stage) {
    if constexpr (SRC == PageSource::own)   // (the last stages of a batch may not exist: any page)
      next_logical = own[min(first_stage + lane / PPS, ns - 1) * PPS + lane % PPS];
    else
      next_logical = in.list[(size_t)head * in.cap + min(list_position(first_stage), (long)in.cap - 1)];
  };
  auto fetch_entry = [&](int first_stage) {   // (an empty sequence has no entry of its own)
    if constexpr (SRC == PageSource::all) {
      const long lp = list_position(first_stage);
      next_entry = lp < U ? table[lp] : 0;
    } else {
      if (P > 0) next_entry = table[max(0, min(next_logical, P - 1))];
    }
  };
  auto decode_entries = [&](int first_stage) {
    const long lp = list_position(first_stage);
    bool ok = lp < U && (unsigned)next_entry < (unsigned)kv.num_pages;
    if constexpr (SRC == PageSource::all) {
      pg_valid = ok ? (int)min((long)GP, (long)tokens - lp * GP) : 0;
    } else {
      ok &= (unsigned)next_logical < (unsigned)P;
      pg_valid = ok ? max(0, min(GP, tokens - next_logical * GP)) : 0;
    }
    pg_phys = ok ? next_entry : 0;
  };

  // queries: B operands, lane = row l32, channels 16*ks + 8*half ..
  bf16x8_t qf[KS];
  bool known_row;
  {
    const int row = min(r0 + l32, sh.rows_max - 1), a = row_token(sh, row);
    const int tok = in.active_idx ? in.active_idx[(size_t)b * sh.B + a] : a;
    known_row = r0 + l32 < M && (unsigned)tok < (unsigned)sh.B;
    const bf16_t* qa = (const bf16_t*)in.q + (((size_t)b * sh.B + (known_row ? tok : 0)) * sh.Hq + j * sh.G + (row - a * sh.G)) * D;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qf[ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(qa + ks * 16 + half * 8));
  }

  // ---- staging: thread -> NP pieces of keys and NP of values.  Piece i is piece (i*512 + tid) of the stage
  // in memory order; which page that is is the same for the whole wavefront.
  struct Stage {
    u32x4v_t k[NP], v[NP];
    int nv[PPS];   // valid tokens of the stage's pages
  };
  Stage st[PD];
  int k_lds[NP], v_lds[NP];   // LDS byte offsets inside a stage image
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const int p = i * 512 + tid, page = p / PPP, off = p % PPP;
    const int t = page * GP + off / (D / 8), c = off % (D / 8);
    const int t32 = t & 31, row = (t32 & 0x13) | ((t32 & 4) << 1) | ((t32 & 8) >> 1);
    k_lds[i] = (t / 32) * Img::kKeyBlock + c * Img::kKeyStrip + row * 16;
    const int ch = off / (GP / 8), tv = off % (GP / 8);
    const int tok = page * GP + tv * 8;
    v_lds[i] = Img::kValBase + (tok / 32) * Img::kValBlock + ((ch / 32) * 4 + (tok & 31) / 8) * Img::kValStrip + (ch & 31) * 16;
  }
  // stage n of this workgroup -> registers.  A stage past the list's end is requested all the same (so that the
  // number of loads in flight at every wait is a compile-time constant): its entries decode to page 0, of which
  // every lane then reads the first 16 bytes (a workgroup has three such stages, however few it has of its own).
  auto gload = [&](Stage& s, int n) {
    const int slot = (n * PPS) & 63;
    const uint32_t real = n < ns ? ~0u : 0u;
#pragma unroll
    for (int k = 0; k < PPS; ++k) s.nv[k] = __builtin_amdgcn_readlane(pg_valid, slot + k);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      // scalar base address + one lane offset: no vector address arithmetic in the loop
      const int ph = __builtin_amdgcn_readlane(pg_phys, slot + (i * 512 + wave * 64) / PPP);
      const size_t at = ((size_t)ph * sh.Hkv + j) * (PPP * 16);
      const uint32_t lane_off = (uint32_t)((i * 512 + tid) % PPP) * 16u & real;
      const unsigned char* kp = reinterpret_cast<const unsigned char*>(kv.k_pages) + at;
      const unsigned char* vp = reinterpret_cast<const unsigned char*>(kv.v_pages) + at;
      s.k[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4v_t*>(kp + lane_off));
      s.v[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4v_t*>(vp + lane_off));
    }
  };
  auto is_full = [&](const int (&nv)[PPS]) {
    bool f = true;
#pragma unroll
    for (int k = 0; k < PPS; ++k) f &= nv[k] == GP;
    return f;
  };
  // value slots past the end of the sequence may hold anything: cleared once per workgroup (0 * NaN = NaN)
  auto clear_tail = [&](Stage& s) {
    if (is_full(s.nv)) return;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int page = (i * 512 + wave * 64) / PPP;
      int nvp = s.nv[0];
#pragma unroll
      for (int k = 1; k < PPS; ++k) nvp = page == k ? s.nv[k] : nvp;
      const int cnt = max(0, min(8, nvp - (((i * 512 + tid) % PPP) % (GP / 8)) * 8));
      s.v[i][0] &= cnt >= 2 ? ~0u : (cnt == 1 ? 0xFFFFu : 0u);
      s.v[i][1] &= cnt >= 4 ? ~0u : (cnt == 3 ? 0xFFFFu : 0u);
      s.v[i][2] &= cnt >= 6 ? ~0u : (cnt == 5 ? 0xFFFFu : 0u);
      s.v[i][3] &= cnt >= 8 ? ~0u : (cnt == 7 ? 0xFFFFu : 0u);
    }
  };
  auto lstore = [&](const Stage& s, int image) {
    unsigned char* base = lds + image;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      *reinterpret_cast<u32x4v_t*>(base + k_lds[i]) = s.k[i];
      u32x4v_t x = s.v[i];
      if constexpr (HALF) {
        x[0] = bf16_pair_to_half(x[0]);
        x[1] = bf16_pair_to_half(x[1]);
        x[2] = bf16_pair_to_half(x[2]);
        x[3] = bf16_pair_to_half(x[3]);
      }
      *reinterpret_cast<u32x4v_t*>(base + v_lds[i]) = x;
    }
  };

  // ---- running state of this wavefront's rows (row l32, both lane halves hold the same reference)
  float m_run = kNoReference, l_run = 0.f;   // l_run: sum over this lane's own tokens
  [[maybe_unused]] float l_half = 0.f;       // HALF: the same sum of the rounded numerators
  f32x16_t o[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[cb][e] = 0.f;

  // Numerators are exp2(s - m_run), m_run = reference - kRefBias.  The reference lags: it is moved only when
  // a lane's numerators of a block sum up to more than 2^15, so that no numerator ever exceeds 2^15 and
  // the running maximum itself need not be tracked (the sums are needed anyway; a maximum costs half a
  // vector instruction per score on top).  The first block always moves it (exp2(s + 1e30) = inf).
  constexpr float kRefBias = HALF ? 7.0f : 0.0f;
  constexpr float kMoveAbove = HALF ? 32768.0f : 256.0f;

  const int lane_k = half * Img::kKeyStrip + l32 * 16 + block0 * Img::kKeyBlock;
  const int lane_v = Img::kValBase + half * Img::kValStrip + l32 * 16 + block0 * Img::kValBlock;

  // The pieces of a stage's arithmetic.  Each of them is straight-line code; the branches (tokens past the end,
  // a reference that has to move) lie between them, so that what is meant to overlap shares a region:
  //   S(0) | S(1) with the numerators of block 0 | O += V(0) P(0) with the numerators of block 1 | O += V(1) P(1)
  auto read_keys = [&](bf16x8_t (&kf)[KS], const unsigned char* kb) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      kf[ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4v_t*>(kb + 2 * ks * Img::kKeyStrip));
  };
  auto score_products = [&](const bf16x8_t (&kf)[KS], f32x16_t& s) {
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], s, 0, 0, 0);
  };
  auto read_values = [&](u32x4v_t (&vf)[2][CB], const unsigned char* vb) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
        vf[ks][cb] = *reinterpret_cast<const u32x4v_t*>(vb + (cb * 4 + 2 * ks) * Img::kValStrip);
  };
  auto mask_tail = [&](f32x16_t& s, int t, const int (&nv)[PPS]) {
    int half_here = half;
    asm volatile("" : "+v"(half_here));   // keeps what derives from it out of the registers of the main loop
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      // element e: token 16*(e/8) + 8*half + e%8 of block block0 + t
      const int page_lo = GP == 32 ? 0 : e / 8;   // page inside the block
      int n = nv[GP == 32 ? t : 2 * t + page_lo];
      if (TG == 2) n = block0 ? nv[GP == 32 ? 1 : 2 + page_lo] : nv[GP == 32 ? 0 : page_lo];
      if (16 * (e / 8) + 8 * half_here + e % 8 - page_lo * GP >= n) s[e] = -INFINITY;
    }
  };
  auto numerators = [&](const f32x16_t& s, float (&p)[16]) {
    float sum = 0.f;
    const float neg_m = -m_run;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      p[e] = __builtin_amdgcn_exp2f(fmaf(s[e], scale_log2e, neg_m));
      sum += p[e];
    }
    return sum;
  };
  // takes the sum of a block's numerators into account; moves the reference first where that is due
  auto settle = [&](const f32x16_t& s, float (&p)[16], float sum) {
    if (__any(!(sum <= kMoveAbove))) {
      float mx = s[0];
#pragma unroll
      for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s[e]);
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
      const float m_new = fmaxf(fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * scale_log2e - kRefBias, m_run);
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
      if constexpr (HALF) l_half *= alpha;
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) o[cb] *= alpha;
      sum = numerators(s, p);
    }
    l_run += sum;
  };
  auto value_products = [&](const u32x4v_t (&vf)[2][CB], const float (&p)[16]) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      f32x8_t pv;
#pragma unroll
      for (int e = 0; e < 8; ++e) pv[e] = p[8 * ks + e];
      if constexpr (HALF) {
        const f16x8_t ph = __builtin_convertvector(pv, f16x8_t);
        // (two numerators per instruction, exact products, subnormals kept)
        const f16x2_t ones = {1, 1};
        l_half = __builtin_amdgcn_fdot2(__builtin_shufflevector(ph, ph, 0, 1), ones, l_half, false);
        l_half = __builtin_amdgcn_fdot2(__builtin_shufflevector(ph, ph, 2, 3), ones, l_half, false);
        l_half = __builtin_amdgcn_fdot2(__builtin_shufflevector(ph, ph, 4, 5), ones, l_half, false);
        l_half = __builtin_amdgcn_fdot2(__builtin_shufflevector(ph, ph, 6, 7), ones, l_half, false);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
          o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, vf[ks][cb]), ph, o[cb], 0, 0, 0);
      } else {
        // P = hi + lo: hi = p truncated to its top 16 bits (exact), lo = the remainder, rounded
        f32x8_t lo;
        uint32_t pb[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          pb[e] = __float_as_uint(pv[e]);
          lo[e] = pv[e] - __uint_as_float(pb[e] & 0xFFFF0000u);
        }
        const u32x4v_t hi_bits = {__builtin_amdgcn_perm(pb[1], pb[0], 0x07060302u), __builtin_amdgcn_perm(pb[3], pb[2], 0x07060302u),
                                  __builtin_amdgcn_perm(pb[5], pb[4], 0x07060302u), __builtin_amdgcn_perm(pb[7], pb[6], 0x07060302u)};
        const bf16x8_t p_hi = __builtin_bit_cast(bf16x8_t, hi_bits);
        const bf16x8_t p_lo = __builtin_convertvector(lo, bf16x8_t);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, vf[ks][cb]), p_hi, o[cb], 0, 0, 0);
          o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, vf[ks][cb]), p_lo, o[cb], 0, 0, 0);
        }
      }
    }
  };
  // One stage: kf holds the keys of its first block on entry and those of the next stage's on exit.  The barrier
  // stands before the last value products: they cover the latency of the next stage's first reads, and
  // whatever of the image is still read behind it is safe with three images.  The workgroup's last stage has no
  // next one to stage and to wait for (with a few pages it is also the first).
  bf16x8_t kf[KS];
  auto compute = [&](auto last_c, int cur, int next, const int (&nv)[PPS], Stage& s, int n_request) {
    constexpr bool LAST = decltype(last_c)::value;
    const unsigned char* kb = lds + cur + lane_k;
    const unsigned char* vb = lds + cur + lane_v;
    const unsigned char* kb_next = lds + next + lane_k;
    const bool full = is_full(nv);
    f32x16_t s0;
    u32x4v_t vf[2][CB];
    float p0[16], sum0;
    if constexpr (NB == 2) {
      bf16x8_t kf1[KS];
      f32x16_t s1;
      float p1[16], sum1;
      u32x4v_t vf1[2][CB];
      score_products(kf, s0);
      read_keys(kf1, kb + Img::kKeyBlock);
      if constexpr (!LAST) lstore(s, next);
      if (!full) mask_tail(s0, 0, nv);
      score_products(kf1, s1);
      sum0 = numerators(s0, p0);
      read_values(vf, vb);
      settle(s0, p0, sum0);
      if (!full) mask_tail(s1, 1, nv);
      value_products(vf, p0);
      sum1 = numerators(s1, p1);
      read_values(vf1, vb + Img::kValBlock);
      settle(s1, p1, sum1);
      if constexpr (!LAST) __syncthreads();
      value_products(vf1, p1);
      if constexpr (!LAST) {
        read_keys(kf, kb_next);
        gload(s, n_request);
      }
    } else {
      score_products(kf, s0);
      read_values(vf, vb);
      if constexpr (!LAST) lstore(s, next);
      if (!full) mask_tail(s0, 0, nv);
      sum0 = numerators(s0, p0);
      settle(s0, p0, sum0);
      if constexpr (!LAST) {
        __syncthreads();
        read_keys(kf, kb_next);
        gload(s, n_request);
      }
      value_products(vf, p0);
    }
  };

  decode_entries(0);
#pragma unroll
  for (int k = 0; k < PD; ++k) gload(st[k], k);
  // rows past M, and of tokens that do not exist: zero queries
  {
    const uint32_t keep = known_row ? 0xFFFFFFFFu : 0u;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = __builtin_bit_cast(bf16x8_t, __builtin_bit_cast(u32x4v_t, qf[ks]) & keep);
  }
  static_assert(SPF > PD + 2, "the second batch of entries is under way before it is needed");
  auto entries_for = [&](int n) {
    if (n % SPF == 0) decode_entries(n);
    if ((n + 1) % SPF == 0) fetch_entry(n + 1);
    if constexpr (SRC != PageSource::all)
      if ((n + 2) % SPF == 0) fetch_logical(n + 2);
  };
  // Stages in flight: n + 2 and n + 3 in registers while stage n is computed on and stage n + 1 moves to LDS.
  clear_tail(st[0]);
  lstore(st[0], 0);
  int nv_cur[PPS], nv_next[PPS];
#pragma unroll
  for (int i = 0; i < PPS; ++i) nv_cur[i] = st[0].nv[i];
  entries_for(PD);
  gload(st[0], PD);
  __syncthreads();
  read_keys(kf, lds + lane_k);
  int cur = 0, next = Img::kBytes;
  // iteration n: s holds stage n + 1 on entry and stage n + 1 + PD (requested) on exit
  auto iterate = [&](auto with_rows, Stage& s, int n) {
#pragma unroll
    for (int i = 0; i < PPS; ++i) nv_next[i] = s.nv[i];
    clear_tail(s);
    entries_for(n + 1 + PD);
    if constexpr (decltype(with_rows)::value) {
      compute(std::false_type{}, cur, next, nv_cur, s, n + 1 + PD);
    } else {   // staging only: this wavefront has no rows
      lstore(s, next);
      gload(s, n + 1 + PD);
      __syncthreads();
    }
    cur = next;
    next = next == (kImages - 1) * Img::kBytes ? 0 : next + Img::kBytes;
#pragma unroll
    for (int i = 0; i < PPS; ++i) nv_cur[i] = nv_next[i];
  };
  static_assert(PD == 2, "the loop below is unrolled over the register sets");
  if (has_rows) {
    for (int n = 0; n + 1 < ns; n += PD) {
      iterate(std::true_type{}, st[1], n);
      if (n + 2 >= ns) break;
      iterate(std::true_type{}, st[0], n + 1);
    }
    compute(std::true_type{}, cur, next, nv_cur, st[0], 0);
  } else {
    for (int n = 0; n + 1 < ns; n += PD) {
      iterate(std::false_type{}, st[1], n);
      if (n + 2 >= ns) break;
      iterate(std::false_type{}, st[0], n + 1);
    }
  }

  // a lane summed its own tokens; a row's tokens lie in the two lane halves
  {
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
    l_run = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  }
  if constexpr (HALF) {   // O leaves with its weights adding up to l_run
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_half), __float_as_uint(l_half), false, false);
    l_half = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    const float to_l_run = l_half > 0.f ? l_run / l_half : 1.0f;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) o[cb] *= to_l_run;
  }
  if constexpr (TG == 2) {
    // the second token group hands its state over through LDS (the stage buffers are free now):
    // O lane-linear, 16 bytes per lane, then reference and sum per row
    static_assert(kImages * Img::kBytes >= 4 * (CB * 4 * 1024 + 2 * 32 * 4), "the hand-over does not fit the stage buffers");
    float* so = reinterpret_cast<float*>(lds) + row_wave * (CB * 4 * 256 + 64);
    __syncthreads();   // (the last stage's image is read up to here)
    if (block0 && has_rows) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
          *reinterpret_cast<f32x4_t*>(so + (cb * 4 + q4) * 256 + lane * 4) =
              (f32x4_t){o[cb][4 * q4], o[cb][4 * q4 + 1], o[cb][4 * q4 + 2], o[cb][4 * q4 + 3]};
      if (half == 0) {
        so[CB * 4 * 256 + l32] = m_run;
        so[CB * 4 * 256 + 32 + l32] = l_run;
      }
    }
    __syncthreads();
    if (block0 || !has_rows) return;
    const float m2 = so[CB * 4 * 256 + l32], l2 = so[CB * 4 * 256 + 32 + l32];
    const float m_all = fmaxf(m_run, m2);
    const float w1 = __builtin_amdgcn_exp2f(m_run - m_all), w2 = __builtin_amdgcn_exp2f(m2 - m_all);
    m_run = m_all;
    l_run = l_run * w1 + l2 * w2;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const f32x4_t x = *reinterpret_cast<const f32x4_t*>(so + (cb * 4 + q4) * 256 + lane * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[cb][4 * q4 + e] = o[cb][4 * q4 + e] * w1 + x[e] * w2;
      }
  }
  if (!has_rows) return;

  // ---- partial of this (sequence, head, chunk): un-normalised O, reference (log2 units), sum.  O leaves as it
  // lies in the registers: per 32 rows, fragments of 8 channels, lane-linear (every store 1 KiB contiguous;
  // the merge kernel reads fragments the same way).  Rows past M are zero queries: stored, never read.
  const size_t prow = ((size_t)head * nchunk + chunk) * part.rows + r0;   // part.rows and r0 are multiples of 32
  if (half == 0) {
    part.m[prow + l32] = m_run;
    part.l[prow + l32] = l_run;
  }
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const f32x4_t x = {o[cb][4 * q4], o[cb][4 * q4 + 1], o[cb][4 * q4 + 2], o[cb][4 * q4 + 3]};
      *reinterpret_cast<f32x4_t*>(part.o + prow * D + (cb * 4 + q4) * 256 + lane * 4) = x;
    }
}

// The workgroup's own pages out of the head's union bitmap.  A thread ORs the copies of a word, a prefix sum over
// the population counts ranks the words, and the pages of all stages of the workgroup are found at once, a thread each, by a
// binary search of the rank over the words and one inside the word.  Against the list that the selection kernel's last
// workgroup of a head used to build (a hand-over of every row's bitmap, about 5 us), per step: 140 rows over 8192 tokens 43.9
// -> 38.2 us, 280 over 32768 86.0 -> 72.3, 160 over 2 x 2048 58.5 -> 43.3, 128 over 4 x 65536 190 -> 182.
template <int PPS>
__device__ __forceinline__ int own_pages(const UnionInKernel& uni, const KvView& kv, const Shape& sh, int b, int head, int P, int chunk, int nchunk,
                                         unsigned char* lds, uint16_t* own) {
  uint32_t* words = reinterpret_cast<uint32_t*>(lds);
  int* ranks = reinterpret_cast<int*>(words + kMaxSelectPages / 32);
  int* scan = ranks + kMaxSelectPages / 32;
  const int tid = threadIdx.x, nw = (P + 31) >> 5;
  const uint32_t* bits = uni.bits + (size_t)head * uni.stride + min(tid, uni.copy_words - 1);
  uint32_t word = 0u;
  for (int c0 = 0; c0 < uni.copies; c0 += 4) {
    uint32_t x[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) x[c] = bits[(size_t)min(c0 + c, uni.copies - 1) * uni.copy_words];
    word |= (x[0] | x[1]) | (x[2] | x[3]);
  }
  // pages past the sequence's last one are never picked; the masks only keep a stale bitmap harmless
  if (tid >= nw) word = 0u;
  if (tid == nw - 1 && (P & 31)) word &= (1u << (P & 31)) - 1u;
  int U;
  const int rank = block_exclusive_scan(__popc(word), scan, &U);
  words[tid] = word;
  ranks[tid] = rank;
  __syncthreads();
  const int stages = (U + PPS - 1) / PPS, mine = chunk < stages ? ((stages - 1 - chunk) / nchunk + 1) * PPS : 0;
  for (int i = tid; i < mine; i += 512) {
    int k = (chunk + i / PPS * nchunk) * PPS + i % PPS, page = 0;
    if (k < U) {
      int lo = 0, hi = nw;
      while (hi - lo > 1) {   // (the trip count depends on nw only)
        const int mid = (lo + hi) >> 1;
        if (ranks[mid] <= k) lo = mid; else hi = mid;
      }
      const uint32_t w = words[lo];
      k -= ranks[lo];
      int pos = 0;
#pragma unroll
      for (int sft = 16; sft >= 1; sft >>= 1) {
        const int c = __popc((w >> pos) & ((1u << sft) - 1u));
        if (k >= c) {
          k -= c;
          pos += sft;
        }
      }
      page = lo * 32 + pos;
    }
    own[i] = (uint16_t)page;
  }
  __syncthreads();
  return U;
}

template <int D, int GP, bool HALF, PageSource SRC>
__global__ __launch_bounds__(512) void attn_rows_kernel(Address first, Address active_count, Address sel_count, Address page_indptr,
                                                        Address seq_lens, int stride, int kv_heads, int nchunk, int row_groups,
                                                        AttnInputs in, Shape sh, KvView kv, Partials part,
                                                        float scale_log2e, int m_lo, UnionInKernel uni) {
  extern __shared__ __attribute__((aligned(16))) unsigned char stage_lds[];
  in.active_count = pointer<const int32_t>(active_count);   // (leading arguments: see KvView)
  in.sel_count = pointer<const int32_t>(sel_count);
  kv.page_indptr = pointer<const int32_t>(page_indptr);
  kv.seq_lens = pointer<const int32_t>(seq_lens);
  sh.Hkv = kv_heads;
  if constexpr (SRC == PageSource::list) {
    in.list = pointer<const int32_t>(first);
    in.cap = stride;
  }
  if constexpr (SRC == PageSource::own) {
    uni.bits = pointer<const uint32_t>(first);
    uni.stride = stride;
  }
  const int j = blockIdx.y / row_groups, row_group = blockIdx.y % row_groups, b = blockIdx.z;
  const int head = b * sh.Hkv + j;
  constexpr int PPS = StageImage<D, GP>::kPages;
  const int lane = threadIdx.x & 63;
  const long lp = ((long)blockIdx.x + (long)(lane / PPS) * nchunk) * PPS + lane % PPS;
  int logical = (int)min(lp, (long)sh.max_pages);
  // (the first list entries travel with the counts they are checked against)
  if constexpr (SRC == PageSource::list) logical = in.list[(size_t)head * in.cap + min(lp, (long)in.cap - 1)];
  int n = __builtin_amdgcn_readfirstlane((in.active_count ? in.active_count : kv.seq_lens)[b]), listed = 0;
  if constexpr (SRC == PageSource::list) listed = __builtin_amdgcn_readfirstlane(in.sel_count[head]);
  const Sequence seq = sequence(kv, sh, b);
  asm("" : "+s"(n), "+s"(listed) : "s"(seq.tokens), "s"(kv.page_indices), "s"(kv.k_pages), "s"(kv.v_pages), "s"(kv.num_pages), "s"(in.q),
      "s"(in.active_idx), "s"(sh.G), "s"(sh.g_magic), "s"(sh.B), "s"(part.rows), "s"(m_lo));   // (see Sequence)
  const int M = min((in.active_count ? min(n, sh.B) : sh.B) * sh.G, min(sh.rows_max, part.rows));
  const int P = seq.pages;
  int U = P;
  if constexpr (SRC == PageSource::list) U = min(min(listed, in.cap), sh.max_pages);
  // nothing active, a row count another launch serves, or no row in this group
  if (M <= max(m_lo, row_group * kRowGroup)) return;
  uint16_t* own = reinterpret_cast<uint16_t*>(stage_lds + kImages * StageImage<D, GP>::kBytes);
  if constexpr (SRC == PageSource::own) {
    static_assert(kImages * StageImage<D, GP>::kBytes >= kMaxSelectPages / 32 * 8 + 128, "the union's words and ranks do not fit the stage buffers");
    U = own_pages<PPS>(uni, kv, sh, b, head, P, blockIdx.x, nchunk, stage_lds, own);
    if (blockIdx.x == 0 && row_group == 0 && threadIdx.x == 0) uni.sel_count[head] = U;   // for the merge kernel and the caller's diagnostics
  }
  const int stages = (U + PPS - 1) / PPS;
  if ((int)blockIdx.x >= stages) return;
  if constexpr (SRC == PageSource::own) logical = own[min(lane / PPS, (stages - 1 - (int)blockIdx.x) / nchunk) * PPS + lane % PPS];
  const int entry = P > 0 ? kv.page_indices[seq.base + max(0, min(logical, P - 1))] : 0;
  if (M <= 128)
    attn_rows_body<D, GP, HALF, 2, SRC>(nchunk, row_group, j, sh, kv, part, scale_log2e, M, U, seq, in, own, logical, entry, stage_lds);
  else
    attn_rows_body<D, GP, HALF, 1, SRC>(nchunk, row_group, j, sh, kv, part, scale_log2e, M, U, seq, in, own, logical, entry, stage_lds);
}

template <int D, int GP, bool HALF, PageSource SRC>
static hipError_t launch_rows(hipStream_t st, const KvView& kv, const Shape& sh, int batch, const AttnInputs& in,
                              int nchunk, const Partials& part, hipEvent_t e0, hipEvent_t e1, int m_lo, int upper,
                              const UnionInKernel& uni) {
  // own pages: behind the stage buffers, two bytes for every page a workgroup may own
  constexpr bool OWN = SRC == PageSource::own;
  constexpr int PPS = StageImage<D, GP>::kPages;
  constexpr size_t images = kImages * StageImage<D, GP>::kBytes, most = images + (OWN ? 2 * kMaxSelectPages : 0);
  static_assert(most <= 160 * 1024, "the stage buffers and the longest list exceed the LDS");
  const size_t lds_bytes = images + (OWN ? (size_t)((upper + PPS - 1) / PPS + nchunk - 1) / nchunk * PPS * 2 : 0);
  auto kern = attn_rows_kernel<D, GP, HALF, SRC>;
  static bool attr_set = false;   // per instantiation
  if (most > 48 * 1024 && !attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)most);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int row_groups = (part.rows + kRowGroup - 1) / kRowGroup;   // part.rows: what the host knows the count cannot exceed
  const float scale_log2e = sh.sm_scale * 1.4426950408889634f;
  dim3 grid(nchunk, sh.Hkv * row_groups, batch);
  if (e0 && e1)   // events bound to this dispatch: they read the kernel's own begin and end
    hipExtLaunchKernelGGL(kern, grid, dim3(512), (uint32_t)lds_bytes, st, e0, e1, 0, address(OWN ? (const void*)uni.bits : in.list), address(in.active_count), address(in.sel_count),
                          address(kv.page_indptr), address(kv.seq_lens),
                          OWN ? uni.stride : in.cap, sh.Hkv, nchunk, row_groups, in, sh, kv,
                          part, scale_log2e, m_lo, uni);
  else
    kern<<<grid, 512, lds_bytes, st>>>(address(OWN ? (const void*)uni.bits : in.list), address(in.active_count), address(in.sel_count),
                          address(kv.page_indptr), address(kv.seq_lens),
                          OWN ? uni.stride : in.cap, sh.Hkv, nchunk, row_groups, in, sh, kv, part, scale_log2e, m_lo, uni);
  return hipGetLastError();
}

hipError_t launch_attn_rows(hipStream_t st, const KvView& kv, const Shape& sh, int batch, const AttnInputs& in, int nchunk,
                            const Partials& part, hipEvent_t e0, hipEvent_t e1, int m_lo, bool half_values, int upper,
                            const UnionInKernel* uni) {
  if (batch <= 0 || nchunk <= 0) return hipSuccess;
  auto launch = [&](auto half, auto source) {
    constexpr bool H = decltype(half)::value;
    constexpr PageSource S = decltype(source)::value;
    const UnionInKernel u = uni ? *uni : UnionInKernel{nullptr};
    auto run = sh.d == 128 ? (sh.g == 16 ? launch_rows<128, 16, H, S> : launch_rows<128, 32, H, S>)
                           : (sh.g == 16 ? launch_rows<64, 16, H, S> : launch_rows<64, 32, H, S>);
    return run(st, kv, sh, batch, in, nchunk, part, e0, e1, m_lo, upper, u);
  };
  auto launch_half = [&](auto half) {
    if (uni) return launch(half, std::integral_constant<PageSource, PageSource::own>());
    if (in.list) return launch(half, std::integral_constant<PageSource, PageSource::list>());
    return launch(half, std::integral_constant<PageSource, PageSource::all>());
  };
  return half_values ? launch_half(std::true_type()) : launch_half(std::false_type());
}

}  // namespace losa
