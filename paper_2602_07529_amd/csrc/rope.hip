// dag_rope_qk: rotary position embedding (the P(i) of the paper's Eq. 2) evaluated at the adaptive
// position ids of section 4.2.  Memory-bound pre-pass, in place: each block handles a few tokens,
// computes their cos/sin tables once (fp64 angle, so that positions of tens of thousands lose no
// accuracy) and applies them to every query and key head with 16-byte loads and stores.
#include "common.h"

namespace {

// Tokens per block: four share the frequencies.  With fewer than kRopeFew tokens that leaves compute units
// idle and every thread several rows one after another: 650 tokens of 40 heads take 6.2 us, with one token a block 5.2.
// A block is a chain of frequencies, angles and rows: where a token has few pieces of rows and the batch many blocks, sixteen
// tokens share the chain (four, sixteen: 2 / 2 heads of dimension 64, 16 pieces, 20,000 tokens 9.1, 7.6 us, 76,000 24.3, 18.6; 5 / 1
// of 128, 48 pieces, 39.8, 39.1; 6 / 2, 64 pieces, 48.5, 50.4; 2 / 2 of 64, 8192 tokens 5.2, 5.1, 4000 4.2, 4.4).
constexpr int kRopeTokens = 4, kRopeManyTokens = 16;
constexpr int64_t kRopeFew = 2048, kRopeMany = 8192;
constexpr int kRopeFewPieces = 48;
constexpr int kRopeMaxHalf = 128;

template <bool BF16, int TOKENS>
__global__ void __launch_bounds__(256) k_rope(const int32_t* __restrict__ pos_ids, int64_t n_tokens,
                                              void* __restrict__ q, void* __restrict__ k, int hq, int hkv,
                                              int D, RopeTheta theta) {
  __shared__ double s_freq[kRopeMaxHalf];
  __shared__ float s_cos[TOKENS][kRopeMaxHalf];
  __shared__ float s_sin[TOKENS][kRopeMaxHalf];
  const int half = D / 2;
  const int64_t t0 = (int64_t)blockIdx.x * TOKENS;
  for (int m = threadIdx.x; m < half; m += blockDim.x)
    s_freq[m] = dag_rope_freq(theta, m, D);
  __syncthreads();
  for (int idx = threadIdx.x; idx < TOKENS * half; idx += blockDim.x) {
    const int tt = idx / half, m = idx % half;
    const int64_t t = t0 + tt;
    if (t < n_tokens) {
      double sn, cs;
      sincos((double)pos_ids[t] * s_freq[m], &sn, &cs);
      s_cos[tt][m] = (float)cs;
      s_sin[tt][m] = (float)sn;
    }
  }
  __syncthreads();
  constexpr int EPV = BF16 ? 8 : 4;          // elements per 16-byte vector
  const int upr = half / EPV;                // vectors per half row
  const int rows_q = q ? hq : 0, rows_k = k ? hkv : 0;
  const int rows = rows_q + rows_k;
  const int total = TOKENS * rows * upr;
  for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
    const int u = idx % upr;
    const int row = (idx / upr) % rows;
    const int tt = idx / (upr * rows);
    const int64_t t = t0 + tt;
    if (t >= n_tokens) continue;
    const float* cs = &s_cos[tt][u * EPV];
    const float* sn = &s_sin[tt][u * EPV];
    if (BF16) {
      uint16_t* base = row < rows_q ? (uint16_t*)q + ((size_t)t * hq + row) * D
                                    : (uint16_t*)k + ((size_t)t * hkv + (row - rows_q)) * D;
      u32x4* plo = (u32x4*)(base + u * EPV);
      u32x4* phi = (u32x4*)(base + half + u * EPV);
      u32x4 lo = *plo, hi = *phi, olo, ohi;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float l0 = dag_bf_lo(lo[w]), l1 = dag_bf_hi(lo[w]);
        const float h0 = dag_bf_lo(hi[w]), h1 = dag_bf_hi(hi[w]);
        const float c0 = cs[2 * w], c1 = cs[2 * w + 1], s0 = sn[2 * w], s1 = sn[2 * w + 1];
        olo[w] = dag_pack_bf2(l0 * c0 - h0 * s0, l1 * c1 - h1 * s1);
        ohi[w] = dag_pack_bf2(h0 * c0 + l0 * s0, h1 * c1 + l1 * s1);
      }
      *plo = olo;
      *phi = ohi;
    } else {
      float* base = row < rows_q ? (float*)q + ((size_t)t * hq + row) * D
                                 : (float*)k + ((size_t)t * hkv + (row - rows_q)) * D;
      f32x4* plo = (f32x4*)(base + u * EPV);
      f32x4* phi = (f32x4*)(base + half + u * EPV);
      f32x4 lo = *plo, hi = *phi, olo, ohi;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        olo[w] = lo[w] * cs[w] - hi[w] * sn[w];
        ohi[w] = hi[w] * cs[w] + lo[w] * sn[w];
      }
      *plo = olo;
      *phi = ohi;
    }
  }
}

}  // namespace

extern "C" int dag_rope_qk(const int32_t* pos_ids, int64_t n_tokens, void* q, void* k, int32_t hq, int32_t hkv,
                           int32_t head_dim, float theta, dag_dtype_t dtype, void* stream_) {
  if (n_tokens < 0) return DAG_ERR_BAD_LEN;
  if (dtype != DAG_F32 && dtype != DAG_BF16) return DAG_ERR_UNSUPPORTED;
  if (head_dim < 16 || head_dim > 2 * kRopeMaxHalf || head_dim % 16 != 0) return DAG_ERR_UNSUPPORTED;
  if ((q && hq < 1) || (k && hkv < 1) || !(theta > 0.f)) return DAG_ERR_UNSUPPORTED;
  if (n_tokens == 0 || (!q && !k)) return DAG_OK;
  if (!pos_ids) return DAG_ERR_NULL;
  if (!dag_aligned16(q) || !dag_aligned16(k)) return DAG_ERR_ALIGN;
  hipStream_t stream = (hipStream_t)stream_;
  const bool bf16 = dtype == DAG_BF16;
  const int pieces = ((q ? hq : 0) + (k ? hkv : 0)) * (head_dim / (bf16 ? 16 : 8));  // of a token
  const int tokens = n_tokens < kRopeFew ? 1 : n_tokens >= kRopeMany && pieces <= kRopeFewPieces ? kRopeManyTokens : kRopeTokens;
  auto* const kernel = bf16 ? (tokens == 1 ? k_rope<true, 1> : tokens == 4 ? k_rope<true, kRopeTokens> : k_rope<true, kRopeManyTokens>)
                            : (tokens == 1 ? k_rope<false, 1> : tokens == 4 ? k_rope<false, kRopeTokens> : k_rope<false, kRopeManyTokens>);
  hipLaunchKernelGGL(kernel, dim3((unsigned)dag_ceil_div(n_tokens, tokens)), dim3(256), 0, stream, pos_ids, n_tokens, q, k, hq, hkv, head_dim, dag_rope_theta(theta));
  DAG_LAUNCH_CHECK();
  return DAG_OK;
}
