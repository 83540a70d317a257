// fp32 path (small models, tight tolerance): plain tiled kernels, fp32 everywhere.
#include "common.h"

namespace l2pd {

// C[M,N] (+)= A[M,K] * W[N,K]^T.  64x64 tile, 16x16 threads, 4x4 outputs per thread, K tile 16.
__global__ void __launch_bounds__(256) k_gemm_f32(const float* __restrict__ A, const float* __restrict__ W,
                                                  float* __restrict__ C, int M, int N, int K, int accumulate,
                                                  Gate g) {
  if (gate_skip(g)) return;
  __shared__ float sA[16][64 + 1];
  __shared__ float sW[16][64 + 1];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += 16) {
    for (int i = tid; i < 64 * 16; i += 256) {
      int r = i >> 4, k = i & 15;
      int gm = m0 + r, gn = n0 + r, gk = k0 + k;
      sA[k][r] = (gm < M && gk < K) ? A[(size_t)gm * K + gk] : 0.f;
      sW[k][r] = (gn < N && gk < K) ? W[(size_t)gn * K + gk] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      float a[4], w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { a[i] = sA[k][ty * 4 + i]; w[i] = sW[k][tx * 4 + i]; }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += a[i] * w[j];
    }
    __syncthreads();
  }
  for (int i = 0; i < 4; ++i) {
    int gm = m0 + ty * 4 + i;
    if (gm >= M) continue;
    for (int j = 0; j < 4; ++j) {
      int gn = n0 + tx * 4 + j;
      if (gn >= N) continue;
      size_t o = (size_t)gm * N + gn;
      C[o] = accumulate ? C[o] + acc[i][j] : acc[i][j];
    }
  }
}
// Small products (the 64 x 64 tiles above would be fewer than the CUs): 32 x 32 tiles, 16 x 16 threads with 2 x 2 outputs
// each, 32 deep; the next K step waits in registers while one is worked on, so a step costs its arithmetic and not
// a round trip to memory.  VEC: rows in 16-byte pieces (K a multiple of 4, operands aligned).  Up to three products of
// one A and weights of one shape share a launch.  Every output sums over K in ascending order, as above: same bits.
// 96 x 128 x 128: 21.6 us with the 64 x 64 tiles (four of them), 7.0 with these.
struct GemmF32Set {
  const float* W[3];
  float* C[3];
};
template <bool VEC>
__global__ void __launch_bounds__(256) k_gemm_f32_small(const float* __restrict__ A, GemmF32Set set, int M, int N, int K,
                                                        int accumulate, Gate g) {
  if (gate_skip(g)) return;
  constexpr int LD = 34;
  __shared__ __attribute__((aligned(8))) float sA[32][LD], sW[32][LD];
  const float* __restrict__ W = blockIdx.z == 0 ? set.W[0] : (blockIdx.z == 1 ? set.W[1] : set.W[2]);
  float* C = blockIdx.z == 0 ? set.C[0] : (blockIdx.z == 1 ? set.C[1] : set.C[2]);
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int m0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
  const int r = tid >> 3, kq = (tid & 7) * 4;      // this thread's row and first of four K elements of a tile
  const float* pa = A + (size_t)min(m0 + r, M - 1) * K + kq;
  const float* pw = W + (size_t)min(n0 + r, N - 1) * K + kq;
  float va[4], vw[4];
  auto fetch = [&](int k0) {
    if constexpr (VEC) {
      const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
      const float4 x = k0 + kq < K ? *reinterpret_cast<const float4*>(pa + k0) : z;
      const float4 y = k0 + kq < K ? *reinterpret_cast<const float4*>(pw + k0) : z;
      va[0] = x.x; va[1] = x.y; va[2] = x.z; va[3] = x.w;
      vw[0] = y.x; vw[1] = y.y; vw[2] = y.z; vw[3] = y.w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool in = k0 + kq + i < K;
        va[i] = in ? pa[k0 + i] : 0.f;
        vw[i] = in ? pw[k0 + i] : 0.f;
      }
    }
  };
  float acc[2][2] = {};
  fetch(0);
  for (int k0 = 0; k0 < K; k0 += 32) {
#pragma unroll
    for (int i = 0; i < 4; ++i) { sA[kq + i][r] = va[i]; sW[kq + i][r] = vw[i]; }
    __syncthreads();
    if (k0 + 32 < K) fetch(k0 + 32);
#pragma unroll
    for (int k = 0; k < 32; ++k) {
      const float2 x = *reinterpret_cast<const float2*>(&sA[k][ty * 2]), y = *reinterpret_cast<const float2*>(&sW[k][tx * 2]);
      acc[0][0] += x.x * y.x; acc[0][1] += x.x * y.y;
      acc[1][0] += x.y * y.x; acc[1][1] += x.y * y.y;
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int gm = m0 + ty * 2 + i;
    if (gm >= M) continue;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int gn = n0 + tx * 2 + j;
      if (gn >= N) continue;
      const size_t o = (size_t)gm * N + gn;
      C[o] = accumulate ? C[o] + acc[i][j] : acc[i][j];
    }
  }
}
void launch_gemm_f32(const float* A, const float* const* W, float* const* C, int n, int M, int N, int K, int accumulate,
                     Gate g, hipStream_t s) {
  const long long tiles = (long long)((N + 63) / 64) * ((M + 63) / 64) * n;
  if (tiles < 256) {
    GemmF32Set set = {};
    uintptr_t bits = reinterpret_cast<uintptr_t>(A);
    for (int i = 0; i < n; ++i) {
      set.W[i] = W[i];
      set.C[i] = C[i];
      bits |= reinterpret_cast<uintptr_t>(W[i]);
    }
    const dim3 grid((N + 31) / 32, (M + 31) / 32, n);
    if (K % 4 == 0 && bits % 16 == 0)
      hipLaunchKernelGGL(k_gemm_f32_small<true>, grid, dim3(256), 0, s, A, set, M, N, K, accumulate, g);
    else
      hipLaunchKernelGGL(k_gemm_f32_small<false>, grid, dim3(256), 0, s, A, set, M, N, K, accumulate, g);
    return;
  }
  const dim3 grid((N + 63) / 64, (M + 63) / 64);
  for (int i = 0; i < n; ++i)
    hipLaunchKernelGGL(k_gemm_f32, grid, dim3(256), 0, s, A, W[i], C[i], M, N, K, accumulate, g);
}

// Rotary embedding (pairs (i, i + Dh/2)) on q in place; k rotated and v copied into the key/value
// stores at absolute position pos0 + t.
__global__ void k_rope_store_f32(float* q, const float* k, const float* v, float* kstore, float* vstore, int B,
                                 int Tq, int pos0, int Tmax, int H, int Dh, const float2* rope, const int* seq_gb, int pos_per_gb, Gate g) {
  if (gate_skip(g)) return;
  const int half = Dh / 2, d = H * Dh;
  size_t n = (size_t)B * Tq * H * half;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int e = i % half;
  int hh = (i / half) % H;
  int r = i / ((size_t)half * H);
  int b = r / Tq, t = r % Tq, pos = pos0 + seq_pos_offset(seq_gb, pos_per_gb, b) + t;
  const float2 rot = rope[pos * half + e];
  const float c = rot.x, sn = rot.y;
  size_t src = (size_t)r * d + hh * Dh + e;
  size_t dst = ((size_t)b * Tmax + pos) * d + hh * Dh + e;
  float q1 = q[src], q2 = q[src + half];
  q[src] = q1 * c - q2 * sn;
  q[src + half] = q2 * c + q1 * sn;
  float k1 = k[src], k2 = k[src + half];
  kstore[dst] = k1 * c - k2 * sn;
  kstore[dst + half] = k2 * c + k1 * sn;
  vstore[dst] = v[src];
  vstore[dst + half] = v[src + half];
}
void launch_rope_store_f32(float* q, const float* k, const float* v, float* kstore, float* vstore, int B, int Tq,
                           int pos0, int Tmax, int H, int Dh, const float2* rope, const int* seq_gb, int pos_per_gb, Gate g,
                           hipStream_t s) {
  size_t n = (size_t)B * Tq * H * (Dh / 2);
  hipLaunchKernelGGL(k_rope_store_f32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, q, k, v, kstore, vstore,
                     B, Tq, pos0, Tmax, H, Dh, rope, seq_gb, pos_per_gb, g);
}

// Bidirectional softmax attention, one wavefront per (sequence, head, query): lanes own keys for the
// scores and feature dims for the output.  Scores are staged in LDS in chunks of 1024 keys with an
// online rescale between chunks.
__global__ void __launch_bounds__(64) k_attn_f32(const float* q, const float* kstore, const float* vstore,
                                                 float* out, int B, int Tq, int Tk_all, int Tmax, int H, int Dh,
                                                 const int* tk_dev, Gate g) {
  if (gate_skip(g)) return;
  const int Tk = tk_dev ? min(Tk_all, tk_dev[blockIdx.z]) : Tk_all;   // per-sequence key count when given
  __shared__ float s_q[256];
  __shared__ float s_p[1024];
  const int lane = threadIdx.x;
  const int t = blockIdx.x, hh = blockIdx.y, b = blockIdx.z;
  const int d = H * Dh;
  const float scale = rsqrtf((float)Dh);
  const float* qv = q + ((size_t)b * Tq + t) * d + hh * Dh;
  for (int e = lane; e < Dh; e += 64) s_q[e] = qv[e];
  __syncthreads();
  float m = -INFINITY, l = 0.f;
  float o[4] = {0.f, 0.f, 0.f, 0.f};   // Dh <= 256
  for (int k0 = 0; k0 < Tk; k0 += 1024) {
    int kn = min(1024, Tk - k0);
    float cm = -INFINITY;
    for (int j = lane; j < kn; j += 64) {
      const float* kv = kstore + ((size_t)b * Tmax + k0 + j) * d + hh * Dh;
      float sc = 0.f;
      if (Dh % 4 == 0) {       // rows of the store start at multiples of Dh floats of an aligned buffer
#pragma unroll 4
        for (int e = 0; e < Dh; e += 4) {
          const float4 k4 = *reinterpret_cast<const float4*>(kv + e);
          sc += s_q[e] * k4.x; sc += s_q[e + 1] * k4.y; sc += s_q[e + 2] * k4.z; sc += s_q[e + 3] * k4.w;
        }
      } else {
        for (int e = 0; e < Dh; ++e) sc += s_q[e] * kv[e];
      }
      sc *= scale;
      s_p[j] = sc;
      cm = fmaxf(cm, sc);
    }
#pragma unroll
    for (int of = 32; of > 0; of >>= 1) cm = fmaxf(cm, __shfl_xor(cm, of, 64));
    float mn = fmaxf(m, cm);
    float alpha = (m == -INFINITY) ? 0.f : expf(m - mn);
    float ls = 0.f;
    __syncthreads();
    for (int j = lane; j < kn; j += 64) {
      float p = expf(s_p[j] - mn);
      s_p[j] = p;
      ls += p;
    }
#pragma unroll
    for (int of = 32; of > 0; of >>= 1) ls += __shfl_xor(ls, of, 64);
    l = l * alpha + ls;
    m = mn;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      int e = lane + c * 64;
      if (e < Dh) {
        float acc = o[c] * alpha;
#pragma unroll 16
        for (int j = 0; j < kn; ++j) acc += s_p[j] * vstore[((size_t)b * Tmax + k0 + j) * d + hh * Dh + e];
        o[c] = acc;
      }
    }
    __syncthreads();
  }
  float* ov = out + ((size_t)b * Tq + t) * d + hh * Dh;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    int e = lane + c * 64;
    if (e < Dh) ov[e] = o[c] / l;
  }
}
void launch_attn_f32(const float* q, const float* kstore, const float* vstore, float* out, int B, int Tq, int Tk,
                     int Tmax, int H, int Dh, const int* tk_dev, Gate g, hipStream_t s) {
  hipLaunchKernelGGL(k_attn_f32, dim3(Tq, H, B), dim3(64), 0, s, q, kstore, vstore, out, B, Tq, Tk, Tmax, H, Dh, tk_dev,
                     g);
}

__global__ void k_swiglu_f32(const float* gate, const float* up, float* act, size_t n, Gate g) {
  if (gate_skip(g)) return;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float x = gate[i];
  act[i] = x / (1.f + expf(-x)) * up[i];
}
void launch_swiglu_f32(const float* gate, const float* up, float* act, size_t n, Gate g, hipStream_t s) {
  hipLaunchKernelGGL(k_swiglu_f32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, gate, up, act, n, g);
}

}  // namespace l2pd
