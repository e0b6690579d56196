// Dense in-block attention and the final online-softmax merge with the cached prefix
// statistics (paper: Methodology, Computation of the Suffix Tokens and Final Output;
// Preliminaries, eq. full_attn and Attention Decomposition With Online Softmax):
//
//   s_b = sm_scale * q_i . k_b[t]   over the B tokens of the block (bidirectional)
//   L_b = ln sum_t exp(s_b),  o_b = sum_t exp(s_b - L_b) v_b[t]
//   O_i = (e^{L_p} o_p + e^{L_b} o_b) / (e^{L_p} + e^{L_b})
//
// B << L, so this is a few KiB per head and launch-latency bound.  Two kernels: a matrix-core
// one for bfloat16 blocks of up to 64 tokens (below), and an element-generic one (vector ALUs,
// one workgroup per (sequence, query head, 32 query tokens), keys and values of the block staged
// through LDS 32 tokens at a time; float accumulation for bfloat16 inputs, double for float
// inputs) for everything else.
#include <math.h>

#include <type_traits>

#include "losa_device.h"
#include "losa_internal.h"

namespace losa {

template <typename T, int D>
__global__ __launch_bounds__(256) void block_merge_kernel(Shape sh, const T* __restrict__ q, const T* __restrict__ k_b,
                                                          const T* __restrict__ v_b, const float* __restrict__ o_p,
                                                          const float* __restrict__ lse_p, float* __restrict__ out,
                                                          float* __restrict__ o_b, float* __restrict__ lse_b) {
  typedef typename std::conditional<std::is_same<T, float>::value, double, float>::type Acc;
  constexpr int V = Vec16<T>::n, VPR = D / V, CPT = D / 8, RB = 32, TK = 32;
  __shared__ float qs[RB][D + 1];
  __shared__ float ks[TK][D + 1];
  __shared__ float vs[TK][D + 1];
  __shared__ Acc ps[RB][TK + 1];
  const int rb = blockIdx.x, h = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
  const int j = h / sh.G, r0 = rb * RB;
  if (r0 >= sh.B) return;

  for (int v = tid; v < RB * VPR; v += 256) {
    const int rr = v / VPR, cv = v % VPR, i = r0 + rr;
    float f[V];
#pragma unroll
    for (int e = 0; e < V; ++e) f[e] = 0.f;
    if (i < sh.B) {
      const uint4 raw = reinterpret_cast<const uint4*>(q + (((size_t)b * sh.B + i) * sh.Hq + h) * D)[cv];
      widen16(raw, f, T());
    }
#pragma unroll
    for (int e = 0; e < V; ++e) qs[rr][cv * V + e] = f[e];
  }
  const int row = tid / 8, sub = tid % 8;
  float m = -INFINITY;
  Acc l = 0, acc[CPT];
#pragma unroll
  for (int k = 0; k < CPT; ++k) acc[k] = 0;

  for (int t0 = 0; t0 < sh.B; t0 += TK) {
    __syncthreads();
    for (int v = tid; v < TK * VPR; v += 256) {
      const int ts = v / VPR, cv = v % VPR, t = t0 + ts;
      float fk[V], fv[V];
#pragma unroll
      for (int e = 0; e < V; ++e) fk[e] = fv[e] = 0.f;
      if (t < sh.B) {
        const size_t base = (((size_t)b * sh.B + t) * sh.Hkv + j) * D;
        widen16(reinterpret_cast<const uint4*>(k_b + base)[cv], fk, T());
        widen16(reinterpret_cast<const uint4*>(v_b + base)[cv], fv, T());
      }
#pragma unroll
      for (int e = 0; e < V; ++e) {
        ks[ts][cv * V + e] = fk[e];
        vs[ts][cv * V + e] = fv[e];
      }
    }
    __syncthreads();
    Acc s[4];
    float tmax = -INFINITY;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int ts = sub + 8 * k;
      Acc dot = 0;
#pragma unroll 8
      for (int c = 0; c < D; ++c) dot += (Acc)qs[row][c] * (Acc)ks[ts][c];
      s[k] = t0 + ts < sh.B ? dot * (Acc)sh.sm_scale : (Acc)-INFINITY;
      tmax = fmaxf(tmax, (float)s[k]);
    }
    tmax = fmaxf(tmax, __shfl_xor(tmax, 1, 64));
    tmax = fmaxf(tmax, __shfl_xor(tmax, 2, 64));
    tmax = fmaxf(tmax, __shfl_xor(tmax, 4, 64));
    const float m_new = fmaxf(m, tmax);
    const Acc alpha = exp_acc((Acc)m - (Acc)m_new);   // m_new is finite: the block holds at least one token
    Acc psum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const Acc p = exp_acc(s[k] - (Acc)m_new);
      ps[row][sub + 8 * k] = p;
      psum += p;
    }
    psum += __shfl_xor(psum, 1, 64);
    psum += __shfl_xor(psum, 2, 64);
    psum += __shfl_xor(psum, 4, 64);
    l = l * alpha + psum;
    m = m_new;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
      Acc a = acc[k] * alpha;
#pragma unroll 8
      for (int ts = 0; ts < TK; ++ts) a += (Acc)ps[row][ts] * (Acc)vs[ts][sub + 8 * k];
      acc[k] = a;
    }
  }
  const int i = r0 + row;
  if (i >= sh.B) return;
  // ---- merge with the cached prefix statistics of this row
  const size_t orow = ((size_t)b * sh.B + i) * sh.Hq + h;
  const Acc Lb = (Acc)m + log_acc(l);
  const float Lp = lse_p[orow];
  const Acc Lm = Lb > (Acc)Lp ? Lb : (Acc)Lp;
  const Acc wb = exp_acc(Lb - Lm), wp = exp_acc((Acc)Lp - Lm);   // Lp = -inf (empty prefix) gives wp = 0
  const Acc inv = (Acc)1 / (wb + wp);
#pragma unroll
  for (int k = 0; k < CPT; ++k) {
    const int c = sub + 8 * k;
    const Acc ob = acc[k] / l;
    const Acc op = wp > 0 ? (Acc)o_p[orow * D + c] : (Acc)0;
    out[orow * D + c] = (float)((ob * wb + op * wp) * inv);
    if (o_b) o_b[orow * D + c] = (float)ob;
  }
  if (lse_b && sub == 0) lse_b[orow] = (float)Lb;
}

// Matrix-core form for bfloat16 blocks of up to 64 tokens (the block sizes the paper uses:
// 16, 32, 64).  A workgroup takes CW channels of one (sequence, query head); wavefront w takes query rows
// 16w..16w+15 against all keys of the block.  Same transposed products and token order as the
// prefix kernel: S^T = K . Q^T leaves every lane with 8 consecutive tokens of its query row,
// which is the B operand of O^T += V^T . P^T; the values are staged once per workgroup into LDS
// in channel-major order (the block's V arrives token-major), so the A operand of the second
// product is one 16-byte LDS read.  All scores of a row fit in registers (NTILE tiles of 32 keys, at
// most 64 keys), so the softmax is two-pass, no running rescale.  P goes in as a bfloat16 pair hi + lo, as there.
//
// A few KiB per head, so latency is all of it: every load is requested, clamped, before anything waits, scores
// and softmax run ahead of the barrier the values are staged for, two tokens per LDS write (16-bit writes
// collided on two banks), and with few heads the channels of a head are spread over workgroups (each repeats
// the scores, a fifth of a microsecond).
// 28 heads, B = 32: 5.9 -> 3.2 us, 8 sequences 7.2 -> 5.3; 32 heads, B = 64: 8.4 -> 5.2, 8 sequences 10.5 -> 9.2.
typedef __attribute__((ext_vector_type(8))) __bf16 bm_bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float bm_f32x4_t;
typedef __attribute__((ext_vector_type(8))) float bm_f32x8_t;

template <int D, int NTILE, int CW>
__global__ __launch_bounds__(128 * NTILE) void block_merge_mfma_kernel(const bf16_t* __restrict__ q,
                                                               const bf16_t* __restrict__ k_b,
                                                               const bf16_t* __restrict__ v_b,
                                                               int block, int q_heads, int kv_heads, int group,
                                                               const float* __restrict__ o_p,
                                                               const float* __restrict__ lse_p, Shape sh, float* __restrict__ out,
                                                               float* __restrict__ o_b, float* __restrict__ lse_b) {
  sh.B = block;   // (leading arguments: see KvView)
  sh.Hq = q_heads;
  sh.Hkv = kv_heads;
  sh.G = group;
  constexpr int KS = D / 32, NT = CW / 16, PAIRS = 16 * NTILE;   // PAIRS: token pairs of the block's tiles
  constexpr int THREADS = 128 * NTILE, ITEMS = PAIRS * (CW / 8), PER = (ITEMS + THREADS - 1) / THREADS;   // (token pair, 8 channels) to stage; per thread
  __shared__ __attribute__((aligned(16))) uint32_t vT[CW][PAIRS + 4];   // [channel][token pair]; rows stay 16-byte aligned
  const int h = blockIdx.x, b = blockIdx.y, c0 = blockIdx.z * CW, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6, l16 = lane & 15, qd = lane >> 4;
  const int j = h / sh.G, B = sh.B;   // B <= 32 * NTILE (launcher)
  const int r0 = wave * 16;
  const int row = min(r0 + l16, B - 1);

  // ---- queries (B operand) and keys (A operands) straight from global memory in operand layout
  bm_bf16x8_t qf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    qf[ks] = __builtin_bit_cast(bm_bf16x8_t, *reinterpret_cast<const uint4*>(
                                                 q + (((size_t)b * B + row) * sh.Hq + h) * D + ks * 32 + qd * 8));
  // row i of half hh of a tile is its token 8*(i/4) + 4*hh + (i%4): lane group qd then ends up with
  // tokens 8*qd .. 8*qd+7 of the tile (half 0 gives +0..3, half 1 gives +4..7)
  bm_bf16x8_t kf[NTILE][2][KS];
#pragma unroll
  for (int tl = 0; tl < NTILE; ++tl)
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int t = 32 * tl + 8 * (l16 >> 2) + 4 * hh + (l16 & 3);
      const bf16_t* kr = k_b + (((size_t)b * B + min(t, B - 1)) * sh.Hkv + j) * D;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        kf[tl][hh][ks] = __builtin_bit_cast(bm_bf16x8_t, *reinterpret_cast<const uint4*>(kr + ks * 32 + qd * 8));
    }
  // ---- values of the block: two tokens x 8 channels per item
  uint4 va[PER], vb[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int idx = min(tid + THREADS * k, ITEMS - 1), t = 2 * (idx % PAIRS), cv = idx / PAIRS;
    const bf16_t* vr = v_b + ((size_t)b * B * sh.Hkv + j) * D + c0;
    va[k] = reinterpret_cast<const uint4*>(vr + (size_t)min(t, B - 1) * sh.Hkv * D)[cv];
    vb[k] = reinterpret_cast<const uint4*>(vr + (size_t)min(t + 1, B - 1) * sh.Hkv * D)[cv];
  }
  // the prefix statistics this row will be merged with: requested now, used at the very end
  const size_t orow_early = ((size_t)b * B + row) * sh.Hq + h;
  const float Lp = lse_p[orow_early];
  bm_f32x4_t op[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) op[nt] = *reinterpret_cast<const bm_f32x4_t*>(o_p + orow_early * D + c0 + nt * 16 + 4 * qd);
  __builtin_amdgcn_sched_barrier(0);   // all loads leave before the first is waited for (left alone, the values' wait for the keys)

  const float scale_log2e = sh.sm_scale * 1.4426950408889634f;
  float s[NTILE][8];
#pragma unroll
  for (int tl = 0; tl < NTILE; ++tl) {
    bm_f32x4_t sc0 = {0.f, 0.f, 0.f, 0.f}, sc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      sc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[tl][0][ks], qf[ks], sc0, 0, 0, 0);
      sc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[tl][1][ks], qf[ks], sc1, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int t0 = 32 * tl + 8 * qd + e, t1 = t0 + 4;
      s[tl][e] = t0 < B ? sc0[e] * scale_log2e : -INFINITY;       // log2 units from here on
      s[tl][4 + e] = t1 < B ? sc1[e] * scale_log2e : -INFINITY;
    }
  }
  float m = -INFINITY;
#pragma unroll
  for (int tl = 0; tl < NTILE; ++tl)
#pragma unroll
    for (int e = 0; e < 8; ++e) m = fmaxf(m, s[tl][e]);
  m = __uint_as_float(across_rows(__float_as_uint(m), [](uint32_t a, uint32_t c) {
    return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(c)));
  }));   // finite: the block holds at least one token

  // ---- stage the values, transposed; tokens past B are zero
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int idx = tid + THREADS * k, tp = idx % PAIRS, cv = idx / PAIRS;
    if (idx < ITEMS) {
      const uint32_t ma = 2 * tp < B ? ~0u : 0u, mb = 2 * tp + 1 < B ? ~0u : 0u;
      const uint32_t wa[4] = {va[k].x & ma, va[k].y & ma, va[k].z & ma, va[k].w & ma};
      const uint32_t wb[4] = {vb[k].x & mb, vb[k].y & mb, vb[k].z & mb, vb[k].w & mb};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        vT[cv * 8 + 2 * e][tp] = __builtin_amdgcn_perm(wb[e], wa[e], 0x05040100u);
        vT[cv * 8 + 2 * e + 1][tp] = __builtin_amdgcn_perm(wb[e], wa[e], 0x07060302u);
      }
    }
  }
  __syncthreads();
  if (r0 >= B) return;

  bm_f32x4_t o[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) o[nt] = (bm_f32x4_t){0.f, 0.f, 0.f, 0.f};
  float l = 0.f;
#pragma unroll
  for (int tl = 0; tl < NTILE; ++tl) {
    float pv[8];
    uint32_t pb[8];
    bm_f32x8_t lo;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      pv[e] = __builtin_amdgcn_exp2f(s[tl][e] - m);
      l += pv[e];
      pb[e] = __float_as_uint(pv[e]);
      lo[e] = pv[e] - __uint_as_float(pb[e] & 0xFFFF0000u);
    }
    uint4 hi_bits;
    hi_bits.x = __builtin_amdgcn_perm(pb[1], pb[0], 0x07060302u);
    hi_bits.y = __builtin_amdgcn_perm(pb[3], pb[2], 0x07060302u);
    hi_bits.z = __builtin_amdgcn_perm(pb[5], pb[4], 0x07060302u);
    hi_bits.w = __builtin_amdgcn_perm(pb[7], pb[6], 0x07060302u);
    const bm_bf16x8_t p_hi = __builtin_bit_cast(bm_bf16x8_t, hi_bits);
    const bm_bf16x8_t p_lo = __builtin_convertvector(lo, bm_bf16x8_t);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const bm_bf16x8_t vf = __builtin_bit_cast(
          bm_bf16x8_t, *reinterpret_cast<const uint4*>(&vT[nt * 16 + l16][16 * tl + 4 * qd]));
      o[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, p_hi, o[nt], 0, 0, 0);
      o[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, p_lo, o[nt], 0, 0, 0);
    }
  }
  l = __uint_as_float(across_rows(__float_as_uint(l), [](uint32_t a, uint32_t c) {
    return __float_as_uint(__uint_as_float(a) + __uint_as_float(c));
  }));

  // ---- merge with the cached prefix statistics of this row (lane: row l16, channels 4*qd.. of each tile)
  const int i = r0 + l16;
  if (i >= B) return;
  const size_t orow = ((size_t)b * B + i) * sh.Hq + h;
  const float Lb = (m + log2f(l)) * 0.6931471805599453f;
  const float Lm = fmaxf(Lb, Lp);
  const float wb = expf(Lb - Lm), wp = expf(Lp - Lm);   // Lp = -inf (empty prefix) gives wp = 0
  const float inv = 1.0f / (wb + wp), inv_l = 1.0f / l;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const size_t at = orow * D + c0 + nt * 16 + 4 * qd;
    bm_f32x4_t ob = o[nt] * inv_l;
    const bm_f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
    const bm_f32x4_t opv = wp > 0.f ? op[nt] : zero;   // an empty prefix may hold anything in o_p, NaN included
    *reinterpret_cast<bm_f32x4_t*>(out + at) = (ob * wb + opv * wp) * inv;
    if (o_b) *reinterpret_cast<bm_f32x4_t*>(o_b + at) = ob;
  }
  if (lse_b && qd == 0 && c0 == 0) lse_b[orow] = Lb;
}

constexpr int kSpreadChannels = 32;
constexpr long kSpreadWorkgroups = 256;

hipError_t launch_block_merge(hipStream_t st, int dtype, const Shape& sh, int batch, const void* q, const void* k_b,
                              const void* v_b, const float* o_p, const float* lse_p, float* out, float* o_b,
                              float* lse_b) {
  if (batch <= 0) return hipSuccess;
  if (dtype == LOSA_BF16 && sh.B <= 64) {
    // Channels are spread over workgroups while there is at most one per CU: 32 heads, B = 64,
    // whole against four times as many workgroups: 1 sequence 7.2 -> 5.2 us, 2 sequences 7.6 -> 5.7, 4
    // sequences (512 spread workgroups) 8.0 -> 8.7, the repeated scores and keys cost more than they save.
    // (not where lse_b replaces lse_p in place: one workgroup's store would race with another's load of it)
    const bool spread = lse_b != lse_p && (long)sh.Hq * batch * (sh.d / kSpreadChannels) <= kSpreadWorkgroups;
    const auto kernel = sh.d == 128 ? (sh.B <= 32 ? (spread ? block_merge_mfma_kernel<128, 1, kSpreadChannels> : block_merge_mfma_kernel<128, 1, 128>)
                                                  : (spread ? block_merge_mfma_kernel<128, 2, kSpreadChannels> : block_merge_mfma_kernel<128, 2, 128>))
                                    : (sh.B <= 32 ? (spread ? block_merge_mfma_kernel<64, 1, kSpreadChannels> : block_merge_mfma_kernel<64, 1, 64>)
                                                  : (spread ? block_merge_mfma_kernel<64, 2, kSpreadChannels> : block_merge_mfma_kernel<64, 2, 64>));
    const dim3 mgrid(sh.Hq, batch, spread ? sh.d / kSpreadChannels : 1);
    kernel<<<mgrid, sh.B <= 32 ? 128 : 256, 0, st>>>((const bf16_t*)q, (const bf16_t*)k_b, (const bf16_t*)v_b, sh.B, sh.Hq, sh.Hkv, sh.G, o_p, lse_p, sh,
                                                     out, o_b, lse_b);
    return hipGetLastError();
  }
  dim3 grid((sh.B + 31) / 32, sh.Hq, batch);
  if (dtype == LOSA_BF16) {
    if (sh.d == 128)
      block_merge_kernel<bf16_t, 128><<<grid, 256, 0, st>>>(sh, (const bf16_t*)q, (const bf16_t*)k_b, (const bf16_t*)v_b, o_p, lse_p, out, o_b, lse_b);
    else
      block_merge_kernel<bf16_t, 64><<<grid, 256, 0, st>>>(sh, (const bf16_t*)q, (const bf16_t*)k_b, (const bf16_t*)v_b, o_p, lse_p, out, o_b, lse_b);
  } else {
    if (sh.d == 128)
      block_merge_kernel<float, 128><<<grid, 256, 0, st>>>(sh, (const float*)q, (const float*)k_b, (const float*)v_b, o_p, lse_p, out, o_b, lse_b);
    else
      block_merge_kernel<float, 64><<<grid, 256, 0, st>>>(sh, (const float*)q, (const float*)k_b, (const float*)v_b, o_p, lse_p, out, o_b, lse_b);
  }
  return hipGetLastError();
}

}  // namespace losa
