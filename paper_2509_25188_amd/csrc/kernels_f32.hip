// fp32 path (small models, tight tolerance): products and attention on the fp32 matrix cores, fp32 everywhere.
//
// A decode of a small model is a chain of launches of a few microseconds each, so a layer is five of them: the RMSNorm
// (and, in the first layer, the embedding) is part of the product that reads it, rotation and K / V store, SiLU * up, the
// residual sum and the vocabulary reduction are epilogues.  Two layers, 96 rows, 128 wide, vocabulary of 1024: a forward is
// 56 us (135 with nine launches a layer, vector arithmetic and tiles through LDS); bound by launch, two memory round trips
// and the chain of products in every kernel (products 4.6-5.6 us, attention 5.0).
#include "gemm_common.h"

namespace l2pd {
namespace {

// C[M, N] = A[M, K] W[N, K]^T in 16 x 16 fragments of v_mfma_f32_16x16x4_f32.  Operands go from memory straight to
// registers: both are K-contiguous and the order inside K is free, so that lane group g takes elements 4g .. 4g+3 of 16
// as one 16-byte load and feeds them to four successive MFMAs.
//   K is summed in four ranges, which are added in ascending order.  A small product (KS = 4) gives every range a wavefront
// of one workgroup, 16 x 32 outputs: a chain of a quarter of the length, all loads of up to 64 K elements in flight, no
// barrier but the one before the ranges meet in LDS.  A large one (KS = 1) has 64 x 64 outputs in every wavefront, which walks
// the ranges itself: the same bits, so that a sequence's logits do not depend on the batch it is in.
//   us a forward of two layers (32 x 32 and 64 x 64 tiles of vector arithmetic before / these): 4 x 256 rows, 512 wide, FFN 2048:
// 1,324 / 425; 8 x 512 rows, 2048 wide, FFN 4096: 19,707 / 9,417 (73 TFLOP/s).
//   NORM: rows are RMS-normalised on the way: gain is multiplied in as the row is read, the row's sum of squares is formed
// beside the products, and the sums are scaled at the end.
enum { EPI_PLAIN = 0, EPI_ROPE = 1, EPI_SWIGLU = 2, EPI_LMHEAD = 3, EPI_LMHEAD_WIDE = 4 };   // LM head: parts of 32, 64 columns
constexpr bool pair_epi(int epi) { return epi == EPI_ROPE || epi == EPI_SWIGLU; }

// Weight row behind feature f (pair epilogues: side 0 or 1 of it).
template <int EPI>
__device__ __forceinline__ const float* weight_row(const F32Product& a, int f, int side) {
  f = min(f, a.N - 1);
  if constexpr (EPI == EPI_ROPE) {
    const int half = a.Dh / 2, mat = a.per_mat(f), i = f - mat * a.H * half, head = a.half(i);
    const float* W = mat == 0 ? a.W[0] : (mat == 1 ? a.W[1] : a.W[2]);
    return W + (size_t)(head * a.Dh + i - head * half + side * half) * a.K;
  } else if constexpr (EPI == EPI_SWIGLU) {
    return a.W[side] + (size_t)f * a.K;
  } else {
    return a.W[0] + (size_t)f * a.K;
  }
}
// Output of one row: columns f and, for pair epilogues, both sides of feature f.
__device__ __forceinline__ void put_plain(const F32Product& a, int row, int f, float x) {
  if (row >= a.M || f >= a.N) return;
  float* o = a.C + (size_t)row * a.N + f;
  *o = a.accumulate ? *o + x : x;
}
__device__ __forceinline__ void put_swiglu(const F32Product& a, int row, int f, float g, float u) {
  if (row < a.M && f < a.N) a.C[(size_t)row * a.N + f] = g / (1.f + expf(-g)) * u;
}
// rotate-half pairs (i, i + Dh/2): q rotated in place of the product, k rotated and v as it is into the stores
__device__ __forceinline__ void put_rope(const F32Product& a, int row, int f, float x1, float x2) {
  if (row >= a.M || f >= a.N) return;
  const int half = a.Dh / 2, mat = a.per_mat(f), i = f - mat * a.H * half, head = a.half(i), e = i - head * half;
  const int b = a.per_seq(row), pos = a.pos0 + seq_pos_offset(a.seq_gb, a.pos_per_gb, b) + row - b * a.Tq;
  const int d = a.H * a.Dh, col = head * a.Dh + e;
  float* o = mat == 0 ? a.C + (size_t)row * d + col : (mat == 1 ? a.kstore : a.vstore) + ((size_t)b * a.Tmax + pos) * d + col;
  if (mat < 2) {
    const float2 rot = a.rope[(size_t)pos * half + e];
    const float y1 = x1 * rot.x - x2 * rot.y;
    x2 = x2 * rot.x + x1 * rot.y;
    x1 = y1;
  }
  o[0] = x1;
  o[half] = x2;
}
// The row's logits of one part of the vocabulary, NF fragments of 16 columns from f0 (lane cl holds column f0 + 16 j + cl):
// logits, and the part's (max, sum exp(x - max), lowest column that has the maximum), the mask id being no candidate.
template <int NF>
__device__ __forceinline__ void put_lmhead(const F32Product& a, int row, int f0, int cl, const float* logits) {
  if (NF == 2 && f0 >= a.N) return;            // (the rest of a 64-column tile past the vocabulary)
  float x[NF];
#pragma unroll
  for (int j = 0; j < NF; ++j) x[j] = logits[j];
  const LmHeadEpilogue& e = a.lm;
  if (e.bias.value != 0.f && (unsigned)(e.bias.token_id - f0) < 16u * NF && a.gate.ctl) {   // the biased token is in this part
    const bool biased = row < a.M && a.gate.ctl[CTL_SEQ_GB + row / e.bias.block_len] * e.bias.block_len +
                                             row % e.bias.block_len >= e.bias.gen_pos_from;
#pragma unroll
    for (int j = 0; j < NF; ++j) {
#pragma clang fp contract(off)                 // (a rounding less in one of the tiles would tell them apart)
      if (biased && f0 + 16 * j + cl == e.bias.token_id) x[j] += e.bias.value;
    }
  }
  float m = -INFINITY;
#pragma unroll
  for (int j = 0; j < NF; ++j) {
    const int col = f0 + 16 * j + cl;
    if (e.logits && row < a.M && col < a.N) e.logits[(size_t)row * a.N + col] = x[j];
    if (col == e.mask_id || col >= a.N) x[j] = -INFINITY;
    m = fmaxf(m, x[j]);
  }
  if (!e.part_max) return;
  m = fmaxf(m, dppf<kDppRor + 8>(m));
  m = fmaxf(m, dppf<kDppRor + 4>(m));
  m = fmaxf(m, dppf<kDppRor + 2>(m));
  m = fmaxf(m, dppf<kDppRor + 1>(m));
  int mi = 0x7fffffff;
  float sum = 0.f;
#pragma unroll
  for (int j = NF - 1; j >= 0; --j) mi = x[j] == m && m > -INFINITY ? f0 + 16 * j + cl : mi;
#pragma unroll
  for (int j = 0; j < NF; ++j) sum += m == -INFINITY ? 0.f : exp_neg(m - x[j]);
  mi = min(mi, (int)dpp<kDppRor + 8>((unsigned)mi));
  mi = min(mi, (int)dpp<kDppRor + 4>((unsigned)mi));
  mi = min(mi, (int)dpp<kDppRor + 2>((unsigned)mi));
  mi = min(mi, (int)dpp<kDppRor + 1>((unsigned)mi));
  sum += dppf<kDppRor + 8>(sum);
  sum += dppf<kDppRor + 4>(sum);
  sum += dppf<kDppRor + 2>(sum);
  sum += dppf<kDppRor + 1>(sum);
  if (cl == 0 && row < a.M) {
    const size_t o = (size_t)row * e.n_part + f0 / (16 * NF);
    e.part_max[o] = m;
    e.part_sum[o] = sum;
    e.part_idx[o] = mi;
  }
}
// Finished values of one row: v[j] is fragment j, column lane cl.
template <int EPI, int FN>
__device__ __forceinline__ void put_row(const F32Product& a, int row, int f0, int cl, float (&v)[FN]) {
  if constexpr (EPI == EPI_LMHEAD) {
#pragma unroll
    for (int p = 0; p < FN / 2; ++p) put_lmhead<2>(a, row, f0 + 32 * p, cl, v + 2 * p);
  } else if constexpr (EPI == EPI_LMHEAD_WIDE) {
    put_lmhead<FN>(a, row, f0, cl, v);
  } else if constexpr (pair_epi(EPI)) {
#pragma unroll
    for (int p = 0; p < FN / 2; ++p) {
      if constexpr (EPI == EPI_ROPE) put_rope(a, row, f0 + 16 * p + cl, v[2 * p], v[2 * p + 1]);
      else put_swiglu(a, row, f0 + 16 * p + cl, v[2 * p], v[2 * p + 1]);
    }
  } else {
#pragma unroll
    for (int j = 0; j < FN; ++j) put_plain(a, row, f0 + 16 * j + cl, v[j]);
  }
}

template <int FM, int FN, int KS, int EPI, bool NORM, bool VEC>
__global__ void __launch_bounds__(256) k_product_f32(F32Product a) {
  const int2 gate = gate_words(a.gate);        // looked at when the first loads are on their way
  static_assert(KS == 1 || (KS == 4 && FM == 1), "four wavefronts share one row of fragments, or none");
  constexpr int U = KS == 4 ? 4 : 1;           // 16-deep K steps per round of loads
  constexpr int TN = (pair_epi(EPI) ? FN / 2 : FN) * 16;   // features of a tile
  __shared__ float s_part[KS == 4 ? 4 : 1][KS == 4 ? 4 * FN : 1][64];
  __shared__ float s_ss[KS == 4 ? 4 : 1][64];
  const int lane = threadIdx.x & 63, g = lane >> 4, cl = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // KS == 1: the four wavefronts of a workgroup are 2 x 2 neighbours
  const int tile_m = KS == 4 ? blockIdx.y : blockIdx.y * 2 + (wave >> 1);
  const int tile_n = KS == 4 ? blockIdx.x : blockIdx.x * 2 + (wave & 1);
  const int m0 = tile_m * 16 * FM, f0 = tile_n * TN;
  if (KS == 1 && (m0 >= a.M || f0 >= a.N)) return;
  const int steps = (a.K + 15) / 16, per = (steps + 3) / 4;

  const float* pa[FM];
  const float* pw[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    int r = min(m0 + i * 16 + cl, a.M - 1);
    if (a.mapped) r = map_row(a.rows, r, a.gate.ctl);
    if (a.tokens) r = a.tokens[r];
    pa[i] = a.A + (size_t)r * a.K + g * 4;
  }
#pragma unroll
  for (int j = 0; j < FN; ++j)
    pw[j] = (pair_epi(EPI) ? weight_row<EPI>(a, f0 + j / 2 * 16 + cl, j & 1) : weight_row<EPI>(a, f0 + j * 16 + cl, 0)) + g * 4;
  // a lane's four K elements of step c, zero beyond K or the range
  auto fetch = [&](const float* p, int c, int c1) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if constexpr (VEC) {
      if (c < c1 && c * 16 + g * 4 < a.K) v = *reinterpret_cast<const f32x4*>(p + c * 16);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (c < c1 && c * 16 + g * 4 + j < a.K) v[j] = p[c * 16 + j];
    }
    return v;
  };
  struct Round { f32x4 x[U][FM], w[U][FN], gain[NORM ? U : 1]; };
  auto load = [&](Round& r, int c, int c1) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < FM; ++i) r.x[u][i] = fetch(pa[i], c + u, c1);
#pragma unroll
      for (int j = 0; j < FN; ++j) r.w[u][j] = fetch(pw[j], c + u, c1);
      if constexpr (NORM) r.gain[u] = fetch(a.gain + g * 4, c + u, c1);
    }
  };
  f32x4 acc[FM][FN];
  float ss[FM];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      ss[i] = 0.f;
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  auto work = [&](Round& r, int c, int c1) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (c + u >= c1) break;
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        if (a.h_out && tile_n == 0 && m0 + i * 16 + cl < a.M) {   // embedding: the rows are the residual stream's
          float* h = a.h_out + (size_t)(m0 + i * 16 + cl) * a.K + (c + u) * 16 + g * 4;
          if constexpr (VEC) {
            if ((c + u) * 16 + g * 4 < a.K) *reinterpret_cast<f32x4*>(h) = r.x[u][i];
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if ((c + u) * 16 + g * 4 + j < a.K) h[j] = r.x[u][i][j];
          }
        }
        if constexpr (NORM) {
#pragma unroll
          for (int j = 0; j < 4; ++j) ss[i] += r.x[u][i][j] * r.x[u][i][j];
          r.x[u][i] *= r.gain[u];
        }
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(r.x[u][i][t], r.w[u][j][t], acc[i][j], 0, 0, 0);
    }
  };
  // one K range, the next round's loads in flight behind the one at work
  auto range = [&](int z) {
    const int c1 = min(steps, (z + 1) * per);
    Round r0, r1;
    load(r0, z * per, c1);
    if (gate_closed(a.gate, gate)) return false;
    for (int c = z * per; c < c1; c += 2 * U) {
      load(r1, c + U, c1);
      work(r0, c, c1);
      load(r0, c + 2 * U, c1);
      work(r1, c + U, c1);
    }
    return true;
  };
  clear();
  if constexpr (KS == 4) {
    if (!range(wave)) return;
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) s_part[wave][j * 4 + r][lane] = acc[0][j][r];
    if constexpr (NORM) s_ss[wave][lane] = ss[0];
    __syncthreads();
    // C layout: register r of a lane is row 4 g + r, column cl; wavefront w finishes the rows with r = w
    float v[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j)
      v[j] = s_part[0][j * 4 + wave][lane] + s_part[1][j * 4 + wave][lane] + s_part[2][j * 4 + wave][lane] +
             s_part[3][j * 4 + wave][lane];
    if constexpr (NORM) {
      float q = s_ss[0][lane] + s_ss[1][lane] + s_ss[2][lane] + s_ss[3][lane];   // row cl, K elements of group g
      q += __shfl_xor(q, 16, 64);
      q += __shfl_xor(q, 32, 64);
      const float inv = __shfl(rsqrtf(q / (float)a.K + a.eps), g * 4 + wave, 64);
#pragma unroll
      for (int j = 0; j < FN; ++j) v[j] *= inv;
    }
    put_row<EPI, FN>(a, m0 + g * 4 + wave, f0, cl, v);
  } else {
    f32x4 tot[FM][FN];
    float tss[FM];
    for (int z = 0; z < 4; ++z) {
      if (z > 0) clear();
      if (!range(z)) return;
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        tss[i] = z == 0 ? ss[i] : tss[i] + ss[i];
#pragma unroll
        for (int j = 0; j < FN; ++j) tot[i][j] = z == 0 ? acc[i][j] : tot[i][j] + acc[i][j];
      }
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      float inv = 1.f;
      if constexpr (NORM) {
        float q = tss[i];
        q += __shfl_xor(q, 16, 64);
        q += __shfl_xor(q, 32, 64);
        inv = rsqrtf(q / (float)a.K + a.eps);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float v[FN];
        const float s = NORM ? __shfl(inv, g * 4 + r, 64) : 1.f;
#pragma unroll
        for (int j = 0; j < FN; ++j) v[j] = NORM ? tot[i][j][r] * s : tot[i][j][r];
        put_row<EPI, FN>(a, m0 + i * 16 + g * 4 + r, f0, cl, v);
      }
    }
  }
}

// Tile choice: 64 x 64 outputs a wavefront once there are enough of them for every SIMD.
constexpr int kBigTiles = 1024;
bool big_product(int M, int cols) { return (long long)((M + 63) / 64) * ((cols + 63) / 64) >= kBigTiles; }

template <int EPI, bool NORM>
void launch_product(const F32Product& a, hipStream_t s) {
  constexpr int sides = pair_epi(EPI) ? 2 : 1;
  uintptr_t bits = reinterpret_cast<uintptr_t>(a.A) | reinterpret_cast<uintptr_t>(a.gain) | reinterpret_cast<uintptr_t>(a.h_out);
  for (const float* w : a.W) bits |= reinterpret_cast<uintptr_t>(w);
  const bool vec = a.K % 4 == 0 && bits % 16 == 0;
  if (big_product(a.M, a.N * sides)) {
    const int tn = 64 / sides;
    const dim3 grid((a.N + 2 * tn - 1) / (2 * tn), (a.M + 127) / 128);
    if (vec) hipLaunchKernelGGL((k_product_f32<4, 4, 1, EPI, NORM, true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_product_f32<4, 4, 1, EPI, NORM, false>), grid, dim3(256), 0, s, a);
  } else {
    constexpr int FN = EPI == EPI_LMHEAD_WIDE ? 4 : 2;
    const int tn = 16 * FN / sides;
    const dim3 grid((a.N + tn - 1) / tn, (a.M + 15) / 16);
    if (vec) hipLaunchKernelGGL((k_product_f32<1, FN, 4, EPI, NORM, true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_product_f32<1, FN, 4, EPI, NORM, false>), grid, dim3(256), 0, s, a);
  }
}

// Bidirectional softmax attention, 16 queries of one (sequence, head) per workgroup; its four wavefronts deal the keys
// among them in contiguous runs and join at the end (the same runs whatever the batch).  S^T = K Q^T, so that a lane holds
// scores of one query (column cl; rows 4 g + r are keys) and its exponentials are the B operand of O^T = V^T P^T as they
// are: MFMA r of a 16-key tile takes keys 4 g + r.  Operands from memory straight to registers, 32 keys a round, the values
// sent off before the scores, in heads of any size: asked for where they are needed, the 128 of a lane in heads of 256 are 16
// round trips one after the other (a step of two layers, one head of 256, 32 queries over 1984 keys: 540 us, 1362 with the values
// behind the scores, 885 with a wavefront per query).  96 rows, 4 heads of 32: 5.0 us (7.2 behind, 8.9 with a wavefront per query).
// ND: 16-wide pieces of the head, padded with zeros.
template <int ND, bool VEC>
__global__ void __launch_bounds__(256) k_attn_f32(const float* __restrict__ q, const float* __restrict__ kstore,
                                                  const float* __restrict__ vstore, float* __restrict__ out, int Tq, int Tk_all,
                                                  int Tmax, int H, int Dh, const int* __restrict__ tk_dev, Gate gate) {
  if (gate_skip(gate)) return;
  constexpr int LD = 16 * ND + 4;
  extern __shared__ __attribute__((aligned(16))) float s_o[];   // [wavefront][query][feature], then maxima and sums
  float* const s_m = s_o + 4 * 16 * LD;
  float* const s_l = s_m + 64;
  const int lane = threadIdx.x & 63, g = lane >> 4, cl = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int hh = blockIdx.y, b = blockIdx.z, d = H * Dh, q0 = blockIdx.x * 16;
  const int Tk = tk_dev ? min(Tk_all, tk_dev[b]) : Tk_all;
  const float scale = rsqrtf((float)Dh);
  auto piece = [&](const float* p, int c) {      // features 16 c + 4 g .. + 3 of a row
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    const int e = c * 16 + g * 4;
    if constexpr (VEC) {
      if (e < Dh) v = *reinterpret_cast<const f32x4*>(p + e);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (e + j < Dh) v[j] = p[e + j];
    }
    return v;
  };
  f32x4 fq[ND];
  const float* qp = q + ((size_t)b * Tq + min(q0 + cl, Tq - 1)) * d + hh * Dh;
#pragma unroll
  for (int c = 0; c < ND; ++c) fq[c] = piece(qp, c);
  const float* kb = kstore + (size_t)b * Tmax * d + hh * Dh;
  const float* vb = vstore + (size_t)b * Tmax * d + hh * Dh;

  f32x4 o[ND];
#pragma unroll
  for (int f = 0; f < ND; ++f) o[f] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  const int tiles = (Tk + 15) / 16, per = (tiles + 3) / 4;
  const int t1 = min(tiles, (wave + 1) * per);
  for (int t = wave * per; t < t1; t += 2) {
    f32x4 s[2];
    float p[2][4];
    float v[ND][2][4];      // values of the round: sent off before the scores that they wait for
#pragma unroll
    for (int f = 0; f < ND; ++f)
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          v[f][u][r] = f * 16 + cl < Dh ? vb[(size_t)min((t + u) * 16 + g * 4 + r, Tk - 1) * d + f * 16 + cl] : 0.f;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      s[u] = f32x4{0.f, 0.f, 0.f, 0.f};
      const float* kr = kb + (size_t)min((t + u) * 16 + cl, Tk - 1) * d;
#pragma unroll
      for (int c = 0; c < ND; ++c) {
        const f32x4 x = piece(kr, c);
#pragma unroll
        for (int j = 0; j < 4; ++j) s[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j], fq[c][j], s[u], 0, 0, 0);
      }
    }
    float tmax = -INFINITY;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const bool in = t + u < t1 && (t + u) * 16 + g * 4 + r < Tk;
        p[u][r] = in ? s[u][r] * scale : -INFINITY;
        tmax = fmaxf(tmax, p[u][r]);
      }
    tmax = fmaxf(tmax, __shfl_xor(tmax, 16, 64));
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
    // (m = -inf at first: alpha 0; scores of -inf alone so far: relative to the lowest number, sums of zero)
    const float mn = fmaxf(m, tmax), ref = fmaxf(mn, -3.402823466e38f), alpha = exp_neg(ref - m);
    m = mn;
    l *= alpha;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[u][r] = exp_neg(ref - p[u][r]);
        l += p[u][r];
      }
#pragma unroll
    for (int f = 0; f < ND; ++f) {
      o[f] *= alpha;
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          o[f] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[f][u][r], p[u][r], o[f], 0, 0, 0);
    }
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  // O^T fragment f: features 16 f + 4 g + r of query cl
#pragma unroll
  for (int f = 0; f < ND; ++f) *reinterpret_cast<f32x4*>(s_o + (wave * 16 + cl) * LD + f * 16 + g * 4) = o[f];
  if (g == 0) { s_m[wave * 16 + cl] = m; s_l[wave * 16 + cl] = l; }
  __syncthreads();
  const int qi = threadIdx.x >> 4;              // a query per 16 lanes
  float M = s_m[qi];
#pragma unroll
  for (int w = 1; w < 4; ++w) M = fmaxf(M, s_m[w * 16 + qi]);
  float f[4], L = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    f[w] = exp_neg(M - s_m[w * 16 + qi]);
    L += s_l[w * 16 + qi] * f[w];
  }
  if (q0 + qi >= Tq) return;
  float* ov = out + ((size_t)b * Tq + q0 + qi) * d + hh * Dh;
  for (int e = threadIdx.x & 15; e < Dh; e += 16) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) v += s_o[(w * 16 + qi) * LD + e] * f[w];
    ov[e] = v / L;
  }
}
template <int ND, bool VEC>
void launch_attn(const float* q, const float* kstore, const float* vstore, float* out, int B, int Tq, int Tk, int Tmax, int H,
                 int Dh, const int* tk_dev, Gate g, hipStream_t s) {
  auto kern = k_attn_f32<ND, VEC>;
  constexpr int smem = (4 * 16 * (16 * ND + 4) + 128) * 4;
  static DynLdsAttr attr;
  attr.ensure(reinterpret_cast<const void*>(kern), smem);
  hipLaunchKernelGGL(kern, dim3((Tq + 15) / 16, H, B), dim3(256), smem, s, q, kstore, vstore, out, Tq, Tk, Tmax, H, Dh, tk_dev, g);
}

}  // namespace

// Parts of the vocabulary reduction: by the vocabulary alone, so that a row's sums, and with them its confidence, do not depend on
// the batch it is in.  64 columns once the small tiles of 64 are a workgroup for every CU, 32 below.  us a step of two layers
// of 128 (parts of 64 / 32; tiles of 32 and 64 with a part each, by the rows: the third): vocabulary 126,464, 32 head rows 169 / 191 / 170,
// 512 rows 640 / 768 / 645; 50,000, 32 rows 83 / 88 / 88, 512 rows 348 / 404 / 349; 16,320 (- / 32 columns / by the rows), 32 rows - / 68 / 69, 512 rows - / 207 / 194.
static int head_part_cols(int V) { return V > 255 * 64 ? 64 : 32; }
int f32_lmhead_n_part(int V) { return (V + head_part_cols(V) - 1) / head_part_cols(V); }

void launch_product_f32(F32Product a, int kind, hipStream_t s) {
  a.mapped = row_map_moves(a.rows, a.M);
  if (kind == F32_QKV) { a.per_mat = Div(a.H * (a.Dh / 2)); a.half = Div(a.Dh / 2); a.per_seq = Div(a.Tq); }
  if (kind == F32_QKV) launch_product<EPI_ROPE, true>(a, s);
  else if (kind == F32_SWIGLU) launch_product<EPI_SWIGLU, true>(a, s);
  else if (kind == F32_LMHEAD && head_part_cols(a.N) == 64) launch_product<EPI_LMHEAD_WIDE, true>(a, s);
  else if (kind == F32_LMHEAD) launch_product<EPI_LMHEAD, true>(a, s);
  else launch_product<EPI_PLAIN, false>(a, s);
}

void launch_attn_f32(const float* q, const float* kstore, const float* vstore, float* out, int B, int Tq, int Tk,
                     int Tmax, int H, int Dh, const int* tk_dev, Gate g, hipStream_t s) {
#define L2PD_ATTN(ND)                                                                                         \
  (Dh % 4 == 0 ? launch_attn<ND, true>(q, kstore, vstore, out, B, Tq, Tk, Tmax, H, Dh, tk_dev, g, s)           \
               : launch_attn<ND, false>(q, kstore, vstore, out, B, Tq, Tk, Tmax, H, Dh, tk_dev, g, s))
  if (Dh <= 32) L2PD_ATTN(2);
  else if (Dh <= 64) L2PD_ATTN(4);
  else if (Dh <= 128) L2PD_ATTN(8);
  else L2PD_ATTN(16);
#undef L2PD_ATTN
}

}  // namespace l2pd
