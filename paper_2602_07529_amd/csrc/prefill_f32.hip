// fp32 DAG attention prefill (paper Eq. 2 + Eq. 3): the accuracy path.  fp32 everywhere: both products
// on the 16x16x4 fp32 MFMA (fused multiply-adds in fp32), exact expf.
//
// A wave owns 16 query rows of one head and works on UK keys at a time.  Nothing is staged in LDS: the
// order in which a contraction index is handed to the MFMA is free as long as both operands agree on it,
// and with the orders below every lane fetches its operands as consecutive 16-byte pieces:
//   scores   S^T = K Q^T:   lane (L, g) = (lane % 16, lane / 16) holds dimensions 16 t + 4 g + c of key L
//            (A) and of query row L (B); component c of piece t is MFMA step 4 t + c
//   output   O^T += V^T P^T: a lane holds the scores of row L for keys 4 g + e in register e, which is the
//            B operand of step e as it lies; as A operand it holds dimensions 64 x + 4 L + c of key
//            4 g + e, and component c belongs to accumulator (x, c)
// The K pieces of the next UK keys are fetched during the softmax and the P V product of the current
// ones, the V pieces during its score product.
//
// Two ways to cut the work.  SPLIT = 1: the four waves of a workgroup are the four row blocks of a
// 64-row query tile, sharing K and V through the L1.  SPLIT = 4: a workgroup is one row block and its
// waves take the key tiles of the row in turn; their results are put together through LDS.  A batch
// whose row blocks alone leave compute units idle (fewer than SPLIT_BELOW tile x head workgroups) is
// bound by the length of the serial walk over a row, which SPLIT = 4 cuts to a quarter.
//
// Measured against the plain vector kernel this replaced (four threads per row, K / V tiles in LDS):
// 448 tokens, 4 heads, D 64: 184 -> 15 us; 1024 tokens, 32 heads, D 128: 1588 -> 160 us; 3328
// tokens, 32 heads, D 128: 9180 -> 898 us = 94 TFLOP/s (a large fp32 matrix product reaches 154).
// What is left: the softmax between the two products, two waves per SIMD at 254 registers.
#include <type_traits>

#include "common.h"
#include "prefill_launch.h"

namespace {

constexpr int TM = 64, TN = 64;

__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <int D, int SPLIT>
__global__ void __launch_bounds__(256, 2) k_prefill_f32(PrefillArgs a) {
  constexpr int UK = D == 64 ? 64 : 32;  // keys per unit: K and V pieces of a unit take 128 registers
  constexpr int NB = UK / 16;            // 16-key blocks of a unit
  constexpr int NT4 = D / 16;            // pieces of a K / Q row per lane
  constexpr int X = D / 64;              // pieces of a V row per lane
  constexpr int UPT = TN / UK;           // units per key tile

  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), L = lane & 15, g = lane >> 4;
  const int x0 = SPLIT == 1 ? blockIdx.x : blockIdx.x >> 2;
  const int rb = SPLIT == 1 ? w : blockIdx.x & 3;
  const int oi = x0 / a.hq, head = x0 % a.hq;
  const int hk = head / (a.hq / a.hkv);
  const int32_t* dsc = a.qtile_desc + (size_t)oi * 8;  // heaviest query tiles first
  const int cu = dsc[0], T = dsc[1], row0 = dsc[2] + 16 * rb, c0 = dsc[3], n_tiles = dsc[4], nbase = dsc[6];
  if (row0 >= T) return;  // (all waves of a SPLIT workgroup share the row block)
  const int i = row0 + L;  // this lane's query row inside the sequence
  const int ic = min(i, T - 1);
  const uint64_t* vis_row = a.node_vis + (int64_t)(nbase + a.tok_node[cu + ic]) * a.W;
  const uint64_t vis0 = vis_row[0];

  const float* qp = (const float*)a.q + ((size_t)(cu + ic) * a.hq + head) * D + 4 * g;
  f32x4 q[NT4], O[X][4];
#pragma unroll
  for (int t = 0; t < NT4; ++t) q[t] = *(const f32x4*)(qp + 16 * t);
#pragma unroll
  for (int x = 0; x < X; ++x)
#pragma unroll
    for (int c = 0; c < 4; ++c) O[x][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;  // reference maximum of the row, this lane's share of the row sum

  const float* kbase = (const float*)a.k + ((size_t)cu * a.hkv + hk) * D + 4 * g;
  const float* vbase = (const float*)a.v + ((size_t)cu * a.hkv + hk) * D + 4 * L;
  const size_t stride = (size_t)a.hkv * D;
  f32x4 kf[NB][NT4], vf[NB][4][X];
  auto load_k = [&](int j0) {  // (keys past the end of the sequence re-read its last one and are masked)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const float* p = kbase + (size_t)min(j0 + 16 * b + L, T - 1) * stride;
#pragma unroll
      for (int t = 0; t < NT4; ++t) kf[b][t] = *(const f32x4*)(p + 16 * t);
    }
  };
  auto load_v = [&](int j0) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float* p = vbase + (size_t)min(j0 + 16 * b + 4 * g + e, T - 1) * stride;
#pragma unroll
        for (int x = 0; x < X; ++x) vf[b][e][x] = *(const f32x4*)(p + 64 * x);
      }
  };

  constexpr int STEP = SPLIT;
  int it = SPLIT == 1 ? 0 : w;  // entry of the tile's row
  if (it < n_tiles) {
    int kt = __builtin_amdgcn_readfirstlane(a.col[c0 + it]);
    load_k(kt * TN);
    int node_of_lane = a.tok_node[cu + min(kt * TN + lane, T - 1)];  // of the tile's keys, one per lane
    while (it < n_tiles) {
      const int full = __builtin_amdgcn_readfirstlane(a.flag[c0 + it]) == DAG_TILE_FULL;
      const int kt_next = it + STEP < n_tiles ? __builtin_amdgcn_readfirstlane(a.col[c0 + it + STEP]) : kt;
      // Keys of the tile that this lane's row sees, bit j for key kt TN + j: the tile is a few runs of one node each, every one
      // switched on as a whole (a test per element took 2 us a tile).
      const bool masked = !full || kt * TN + TN > T;
      uint64_t sees = ~0ull;
      if (masked) {
        auto first_bits = [](int n) { return n >= 64 ? ~0ull : n <= 0 ? 0ull : (1ull << n) - 1; };
        if (!full) {
          sees = 0;
          const int prev = __shfl_up(node_of_lane, 1);
          uint64_t starts = __builtin_amdgcn_ballot_w64(lane == 0 || node_of_lane != prev);
          while (starts != 0) {
            const int s0 = __builtin_ctzll(starts);
            starts &= starts - 1;
            const int n = __builtin_amdgcn_readlane(node_of_lane, s0);
            const uint64_t word = a.W == 1 ? vis0 : vis_row[n >> 6];
            if ((word >> (n & 63)) & 1) sees |= first_bits(starts != 0 ? __builtin_ctzll(starts) : 64) & ~first_bits(s0);
          }
        }
        sees &= first_bits((full ? T : ic + 1) - kt * TN);
      }
#pragma unroll 1
      for (int u = 0; u < UPT; ++u) {
        const int j0 = kt * TN + u * UK;
        load_v(j0);
        f32x4 S[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) S[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < NT4; ++t)
#pragma unroll
          for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int b = 0; b < NB; ++b) S[b] = mfma16(kf[b][t][c], q[t][c], S[b]);
        load_k(u + 1 < UPT ? j0 + UK : kt_next * TN);
        if (u + 1 == UPT) node_of_lane = a.tok_node[cu + min(kt_next * TN + lane, T - 1)];
#pragma unroll
        for (int b = 0; b < NB; ++b) S[b] *= a.scale;
        if (masked) {
          const uint32_t lo = (uint32_t)(sees >> (4 * g)), hi = (uint32_t)(sees >> (4 * g + 32));
#pragma unroll
          for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) {  // this lane's key u UK + 16 b + 4 g + e of the tile
              const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe((int)((UK == 64 ? b > 1 : u > 0) ? hi : lo), 16 * (b & 1) + e, 1);
              S[b][e] = __uint_as_float((__float_as_uint(S[b][e]) & keep) | (0xff800000u & ~keep));
            }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int b = 0; b < NB; ++b) mx = fmaxf(fmaxf(mx, fmaxf(S[b][0], S[b][1])), fmaxf(S[b][2], S[b][3]));
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        if (__builtin_amdgcn_ballot_w64(mx > m) != 0) {
          const float m_new = fmaxf(m, mx);
          const float alpha = m_new == -INFINITY ? 1.f : expf(m - m_new);  // expf(-inf) = 0 on the first visible key
          m = m_new;
          l *= alpha;
#pragma unroll
          for (int x = 0; x < X; ++x)
#pragma unroll
            for (int c = 0; c < 4; ++c) O[x][c] *= alpha;
        }
        const float ref = m == -INFINITY ? 0.f : m;  // (a row that has seen no key yet: every probability below is expf(-inf))
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float p = expf(S[b][e] - ref);
            l += p;
#pragma unroll
            for (int x = 0; x < X; ++x)
#pragma unroll
              for (int c = 0; c < 4; ++c) O[x][c] = mfma16(vf[b][e][x][c], p, O[x][c]);
          }
      }
      kt = kt_next;
      it += STEP;
    }
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  // A hidden key goes through the products with probability zero, and 0 x Inf or NaN is NaN: where a visited
  // tile holds a V row that is not finite, rows that do not see it would be lost.  So a wave whose outputs
  // are not numbers although its row sums are, and whose tiles with a mask hold such a V row, goes over its
  // rows again, key by key, with nothing but the visible ones; as long as every output is a number this
  // costs a maximum over them (one that, unlike fmaxf, hands a NaN on).  o(x, e, c): this lane's output dimension 64 x + 16 g + 4 (e0 + e) + c before the
  // division, set(x, e, c, value) replaces it.
  auto nan_among = [&](auto ne, auto&& o) __attribute__((always_inline)) {
    float any = 0.f;
#pragma unroll
    for (int x = 0; x < X; ++x)
#pragma unroll
      for (int e = 0; e < decltype(ne)::value; ++e)
#pragma unroll
        for (int c = 0; c < 4; c += 2) any = __builtin_elementwise_maximum(__builtin_elementwise_maximum(o(x, e, c), o(x, e, c + 1)), any);
    return any != any;
  };
  auto visible_keys_only = [&](auto ne, int e0, float m_row, auto&& o, auto&& set) __attribute__((always_inline)) {
    constexpr int NE = decltype(ne)::value;
    bool suspect = false;
#pragma unroll 1
    for (int n = 0; n < n_tiles && !suspect; ++n) {  // a key per lane
      const int j0 = a.col[c0 + n] * TN;
      if (a.flag[c0 + n] == DAG_TILE_FULL && j0 + TN <= T) continue;
      const float* vp = (const float*)a.v + ((size_t)(cu + min(j0 + lane, T - 1)) * a.hkv + hk) * D;
      bool bad = false;
#pragma unroll 4
      for (int d = 0; d < D; d += 4) {
        const f32x4 v4 = *(const f32x4*)(vp + d);
#pragma unroll
        for (int c = 0; c < 4; ++c) bad |= !(fabsf(v4[c]) < INFINITY);
      }
      suspect = __builtin_amdgcn_ballot_w64(bad) != 0;
    }
    if (!suspect) return;
#pragma unroll
    for (int x = 0; x < X; ++x)
#pragma unroll
      for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int c = 0; c < 4; ++c) set(x, e, c, 0.f);
#pragma unroll 1
    for (int n = 0; n < n_tiles; ++n) {
      const int j0 = a.col[c0 + n] * TN, j1 = min(j0 + TN, T);
#pragma unroll 1
      for (int j = j0; j < j1; ++j) {
        const int nj = a.tok_node[cu + j];
        const bool ok = j <= i && ((vis_row[nj >> 6] >> (nj & 63)) & 1);
        const float* kp = kbase + (size_t)j * stride;
        const float* vp = (const float*)a.v + ((size_t)(cu + j) * a.hkv + hk) * D + 16 * g + 4 * e0;
        float s = 0.f;
#pragma unroll
        for (int t = 0; t < NT4; ++t) {
          const f32x4 k4 = *(const f32x4*)(kp + 16 * t);
#pragma unroll
          for (int c = 0; c < 4; ++c) s = fmaf(k4[c], q[t][c], s);
        }
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        const float p = expf(s * a.scale - m_row);
#pragma unroll
        for (int x = 0; x < X; ++x)
#pragma unroll
          for (int e = 0; e < NE; ++e) {
            const f32x4 v4 = *(const f32x4*)(vp + 64 * x + 4 * e);
#pragma unroll
            for (int c = 0; c < 4; ++c) set(x, e, c, ok ? fmaf(p, v4[c], o(x, e, c)) : o(x, e, c));
          }
      }
    }
  };
  // register e of accumulator (x, c): dimension 64 x + 16 g + 4 e + c of row L
  float* out = (float*)a.out + ((size_t)(cu + ic) * a.hq + head) * D + 16 * g;
  if constexpr (SPLIT == 1) {
    auto o = [&](int x, int e, int c) __attribute__((always_inline)) { return O[x][c][e]; };
    const std::integral_constant<int, 4> ne;
    if (__builtin_amdgcn_ballot_w64(nan_among(ne, o) && l < INFINITY) != 0)
      visible_keys_only(ne, 0, m, o, [&](int x, int e, int c, float value) __attribute__((always_inline)) { O[x][c][e] = value; });
    if (i < T) {
      const float inv = 1.f / l;
#pragma unroll
      for (int x = 0; x < X; ++x)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          *(f32x4*)(out + 64 * x + 4 * e) = f32x4{O[x][0][e] * inv, O[x][1][e] * inv, O[x][2][e] * inv, O[x][3][e] * inv};
      if (a.lse && g == 0) a.lse[(size_t)(cu + i) * a.hq + head] = m + logf(l);
    }
  } else {
    __shared__ f32x4 sO[4][4 * X][64];  // [wave][4 x + e][lane]: components c
    __shared__ float sM[4][16], sL[4][16];
#pragma unroll
    for (int x = 0; x < X; ++x)
#pragma unroll
      for (int e = 0; e < 4; ++e) sO[w][4 * x + e][lane] = f32x4{O[x][0][e], O[x][1][e], O[x][2][e], O[x][3][e]};
    if (g == 0) {
      sM[w][L] = m;
      sL[w][L] = l;
    }
    __syncthreads();
    const float M = fmaxf(fmaxf(sM[0][L], sM[1][L]), fmaxf(sM[2][L], sM[3][L]));  // (every row sees at least itself)
    float f[4], lt = 0.f;
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      f[y] = expf(sM[y][L] - M);
      lt += f[y] * sL[y][L];
    }
    const float inv = 1.f / lt;
    f32x4 part[X];
#pragma unroll
    for (int x = 0; x < X; ++x) {  // wave w writes dimensions 64 x + 16 g + 4 w ..
      part[x] = f[0] * sO[0][4 * x + w][lane];
#pragma unroll
      for (int y = 1; y < 4; ++y) part[x] += f[y] * sO[y][4 * x + w][lane];
    }
    auto o = [&](int x, int, int c) __attribute__((always_inline)) { return part[x][c]; };
    const std::integral_constant<int, 1> ne;
    if (__builtin_amdgcn_ballot_w64(nan_among(ne, o) && lt < INFINITY) != 0)
      visible_keys_only(ne, w, M, o, [&](int x, int, int c, float value) __attribute__((always_inline)) { part[x][c] = value; });
    if (i < T) {
#pragma unroll
      for (int x = 0; x < X; ++x) *(f32x4*)(out + 64 * x + 4 * w) = part[x] * inv;
      if (a.lse && g == 0 && w == 0) a.lse[(size_t)(cu + i) * a.hq + head] = M + logf(lt);
    }
  }
}

// (tile x head) workgroups, SPLIT = 4 against SPLIT = 1: 28: 15 / 34 us; 144: 34 / 73; 288 (D 128): 85 / 128;
// 416 (D 128, long rows): 258 / 401; 576: 99 / 91 (D 64), 159 / 161 (D 128); 1152: 301 / 233.
constexpr int64_t SPLIT_BELOW = 512;

template <int D>
int launch_d(const PrefillArgs& a, hipStream_t stream) {
  const int64_t tiles = a.total_qtiles * a.hq;
  if (tiles < SPLIT_BELOW)
    hipLaunchKernelGGL((k_prefill_f32<D, 4>), dim3((unsigned)(4 * tiles)), dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL((k_prefill_f32<D, 1>), dim3((unsigned)tiles), dim3(256), 0, stream, a);
  DAG_LAUNCH_CHECK();
  return DAG_OK;
}

}  // namespace

int launch_prefill_f32(const PrefillArgs& a, int head_dim, hipStream_t stream) {
  return head_dim == 64 ? launch_d<64>(a, stream) : launch_d<128>(a, stream);
}
