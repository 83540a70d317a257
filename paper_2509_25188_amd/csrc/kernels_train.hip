// Filter training (Sec. 3.2, Eq. 6; Sec. 4.1: AdamW): full-batch epochs on the mean binary
// cross-entropy of sigmoid(W2 relu(W1 c + b1) + b2) against the EGP labels.  The model has a few thousand parameters and
// the epochs are one dependent chain.  With a workspace for partial gradients the rows of an epoch are dealt to workgroups
// and the kernel boundaries are the synchronisation (k_filter_train_rows); few rows, and calls without a workspace, stay in
// one workgroup over all epochs (k_filter_train_mfma; k_filter_train for widths that do not fit it).
#include "gemm_common.h"

#include <algorithm>

namespace l2pd {

static __host__ __device__ inline int filter_param_count_dev(int s, int hidden, int n_layers) {
  int n = 0;
  for (int k = 0; k < n_layers; ++k) {
    const int in = k == 0 ? s : hidden, out = k == n_layers - 1 ? s : hidden;
    n += out * in + out;
  }
  return n;
}
int filter_param_count(int s, int hidden, int n_layers) { return filter_param_count_dev(s, hidden, n_layers); }

// ------------------------------------------------------------------------------------------------
// Matrix-core kernel.  Forward, back-propagation and parameter gradients of a chunk of rows are products of
// 16 x 16 tiles on v_mfma_f32_16x16x4_f32 (fp32 in, fp32 accumulation), operands in LDS.  Widths are padded to 16 with zeros,
// and LDS rows are 4 floats longer than that: 16 lanes that read one float4 each of consecutive rows, or one float each of four
// rows 4 apart, then cover all 64 banks.  The order of summation inside K is free, so lane group g feeds elements 4g .. 4g+3
// of 16 to four successive MFMAs and reads them as one float4 where K runs along the row.
//   Every wavefront owns up to kSlots tiles of the parameter matrices (a bias is one more column tile, summed by vector
// adds): gradient and both AdamW moments of a tile stay in its registers over all epochs, the parameters in LDS.
//   LDS holds the parameters, the input of every layer, and the loss gradient at the last layer's pre-activation;
// the gradient at a hidden layer's pre-activation replaces that layer's output once the parameter gradient that needs
// the output is formed.  Rows that fit at once stay resident over the epochs; otherwise the next chunk's rows wait in
// registers while a chunk is worked on.
//   Bound by dependent phases (five barriers an epoch) for few rows, towards the fp32 matrix rate of one CU
// (0.6 TFLOP/s) for many: 241 rows of 32 -> 32 -> 32 take 14.1 us an epoch (4.1 at that rate), 4096 rows of
// 64 -> 128 -> 64 1.23 ms (0.55); the scalar loops below 275 us and 33 ms.  The sigmoid and the loss are written out
// (exp_neg, log1p_unit): with the library's functions every one of the 16 wavefronts spends most of a phase in them
// (19.9 us and 1.43 ms).
constexpr int kMfThreads = 1024, kMfWaves = kMfThreads / 64;
constexpr int kMaxSlots = 5;                  // parameter tiles per wavefront
// confidences and labels per thread that wait in registers: fewer where the parameter tiles take them
constexpr int row_regs(int slots) { return slots > 2 ? 4 : 8; }
constexpr int kMfLdsFloats = 40960;           // all 160 KB
static __host__ __device__ inline int pad16(int v) { return (v + 15) / 16 * 16; }
// floats of LDS before the rows (parameters, biases, the loss reduction) and per row
static void mf_sizes(int s, int h, int L, int* fixed, int* per_row, int* tiles) {
  const int sp = pad16(s), hp = L > 1 ? pad16(h) : sp;
  *fixed = 2 * kMfWaves;
  *tiles = 0;
  for (int k = 0; k < L; ++k) {
    const int in = k == 0 ? sp : hp, out = k == L - 1 ? sp : hp;
    *fixed += out * (in + 4) + out;
    *tiles += out / 16 * (in / 16 + 1);
  }
  *per_row = 2 * (sp + 4) + (L - 1) * (hp + 4);
}
// How a set of n rows is worked on: chunks of equal size, a multiple of 16 rows (0: the filter does not fit).  Rows
// that leave room for the hidden layers' gradients next to their outputs (`apart`) need fewer phases.
struct MfPlan { int rows, apart, slots, floats; };
static MfPlan mf_plan(int s, int h, int L, long long n) {
  int fixed, per_row, tiles;
  mf_sizes(s, h, L, &fixed, &per_row, &tiles);
  MfPlan p = {0, 0, (tiles + kMfWaves - 1) / kMfWaves, 0};
  if (p.slots > kMaxSlots) return p;
  const long long regs = row_regs(p.slots) * kMfThreads / s / 16 * 16;
  const int per_row_apart = per_row + (L - 1) * (pad16(h) + 4);
  long long cap = (kMfLdsFloats - fixed) / per_row_apart / 16 * 16;
  if (n <= (cap < regs ? cap : regs)) {
    p.apart = 1;
    per_row = per_row_apart;
  } else {
    cap = (kMfLdsFloats - fixed) / per_row / 16 * 16;
  }
  if (regs < cap) cap = regs;
  if (cap < 16) return p;
  const long long chunks = (n + cap - 1) / cap;
  p.rows = (int)(((n + chunks - 1) / chunks + 15) / 16 * 16);
  p.floats = fixed + p.rows * per_row;
  return p;
}

// 1 / d for d in [1, 4): the hardware's reciprocal and one Newton step
__device__ __forceinline__ float recip(float d) {
  const float r = __builtin_amdgcn_rcpf(d);
  return fmaf(fmaf(-d, r, 1.f), r, r);
}
// log(1 + e) for e in [0, 1]: 2 artanh(e / (2 + e)), the argument at most 1/3, by its series (next term 2e-8)
__device__ __forceinline__ float log1p_unit(float e) {
  const float s = e * recip(2.f + e), q = s * s;
  float p = fmaf(q, 1.f / 13.f, 1.f / 11.f);
  p = fmaf(q, p, 1.f / 9.f);
  p = fmaf(q, p, 1.f / 7.f);
  p = fmaf(q, p, 1.f / 5.f);
  p = fmaf(q, p, 1.f / 3.f);
  return fmaf(2.f * s * q, p, 2.f * s);
}

struct MfDivs {       // by the number of 16-wide tiles of the outer and the hidden width, and by one more
  Div s, h, s1, h1;
};
static MfDivs mf_divs(int s, int hidden, int L) {
  const int st = pad16(s) / 16, ht = pad16(L > 1 ? hidden : s) / 16;
  return MfDivs{Div(st), Div(ht), Div(st + 1), Div(ht + 1)};
}
// A filter in LDS: parameters (rows 4 floats longer than the padded width), biases, the rows' layer inputs, the loss
// gradient at the last pre-activation and, with `apart`, at the hidden ones.  The phases that both kernels below share.
struct MfNet {
  int L, s, h, sp, hp, R;
  bool apart;
  float *w, *bias0, *rows0, *d_last;
  MfDivs div;
  __device__ __forceinline__ int in(int k) const { return k == 0 ? s : h; }
  __device__ __forceinline__ int out(int k) const { return k == L - 1 ? s : h; }
  __device__ __forceinline__ int in_p(int k) const { return k == 0 ? sp : hp; }
  __device__ __forceinline__ int out_p(int k) const { return k == L - 1 ? sp : hp; }
  __device__ __forceinline__ int div_in(int k, int x) const { return k == 0 ? div.s(x) : div.h(x); }     // by in_p / 16
  __device__ __forceinline__ int div_out(int k, int x) const { return k == L - 1 ? div.s(x) : div.h(x); }
  __device__ __forceinline__ int off_w(int k) const {
    return k == 0 ? 0 : (L == 1 ? sp : hp) * (sp + 4) + (k - 1) * hp * (hp + 4);
  }
  __device__ __forceinline__ int n_w() const { return off_w(L - 1) + sp * (in_p(L - 1) + 4); }
  __device__ __forceinline__ float* act(int k) const {         // input of layer k
    return rows0 + (k == 0 ? 0 : R * (sp + 4) + (k - 1) * R * (hp + 4));
  }
  __device__ __forceinline__ float* grad(int k) const {        // loss gradient at layer k's pre-activation
    return k == L - 1 ? d_last : (apart ? d_last + R * (sp + 4) + k * R * (hp + 4) : act(k + 1));
  }
  __device__ __forceinline__ MfNet(const TrainArgs& a, const MfDivs& divs, int rows, bool apart_, float* lds, int reserved)
      : L(a.n_layers), s(a.s), h(a.n_layers > 1 ? a.hidden : a.s), sp(pad16(a.s)),
        hp(pad16(a.n_layers > 1 ? a.hidden : a.s)), R(rows), apart(apart_), w(lds), div(divs) {
    bias0 = lds + n_w();                                       // layer k's biases at + k * hp
    rows0 = bias0 + (L - 1) * hp + sp + reserved;
    d_last = rows0 + R * (sp + 4) + (L - 1) * R * (hp + 4);
  }
};
// every thread's LDS accesses so far are complete and visible to the workgroup; global loads stay in flight
__device__ __forceinline__ void mf_sync() {
  __builtin_amdgcn_s_waitcnt(0xc07f);         // lgkmcnt(0)
  lds_barrier();
}
// Forward, z = A W^T + b, tile by tile: layer inputs, then the loss gradient in d_last (which holds the labels before).
// Returns this thread's part of the loss.
__device__ __forceinline__ float mf_forward(const MfNet& n, int rows, float inv_m, int wave, int lane) {
  const int g = lane >> 4, cl = lane & 15, rt = (rows + 15) / 16;
  float loss = 0.f;
  for (int k = 0; k < n.L; ++k) {
    const int ldi = n.in_p(k) + 4, ldo = n.out_p(k) + 4, ot = n.out_p(k) / 16, kt = n.in_p(k) / 16;
    const float* A = n.act(k) + cl * ldi + g * 4;
    const float* W = n.w + n.off_w(k) + cl * ldi + g * 4;
    const float* B = n.bias0 + k * n.hp + cl;
    float* O = (k == n.L - 1 ? n.d_last : n.act(k + 1)) + g * 4 * ldo + cl;
    for (int t = wave; t < rt * ot; t += kMfWaves) {
      const int tr = n.div_out(k, t), to = t - tr * ot;
      const float b = B[to * 16];
      f32x4 z = {0.f, 0.f, 0.f, 0.f};
      const float *pa = A + tr * 16 * ldi, *pw = W + to * 16 * ldi;
#pragma unroll 2
      for (int kk = 0; kk < kt; ++kk) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(pa + kk * 16), w = *reinterpret_cast<const f32x4*>(pw + kk * 16);
#pragma unroll
        for (int j = 0; j < 4; ++j) z = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j], w[j], z, 0, 0, 0);
      }
      z += f32x4{b, b, b, b};
      float* o = O + tr * 16 * ldo + to * 16;
      const int row = tr * 16 + g * 4;
      if (k < n.L - 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r * ldo] = row + r < rows ? fmaxf(z[r], 0.f) : 0.f;
      } else {
        const bool col_in = to * 16 + cl < n.s;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float y = o[r * ldo], zz = z[r];
          const bool valid = col_in && row + r < rows;
          const float e = exp_neg(fabsf(zz)), inv = recip(1.f + e);
          loss += valid ? fmaxf(zz, 0.f) + log1p_unit(e) - y * zz : 0.f;   // softplus(z) - y z
          o[r * ldo] = valid ? ((zz >= 0.f ? inv : e * inv) - y) * inv_m : 0.f;
        }
      }
    }
    mf_sync();
  }
  return loss;
}
// Back through layer k and the ReLU before it.
__device__ __forceinline__ void mf_back(const MfNet& n, int k, int rt, int wave, int lane) {
  const int g = lane >> 4, cl = lane & 15;
  const int ldi = n.in_p(k) + 4, ldo = n.out_p(k) + 4, ot = n.out_p(k) / 16, it = n.in_p(k) / 16;
  for (int t = wave; t < rt * it; t += kMfWaves) {
    const int tr = n.div_in(k, t), ti = t - tr * it;
    f32x4 z = {0.f, 0.f, 0.f, 0.f};
    const float* pd = n.grad(k) + (tr * 16 + cl) * ldo + g * 4;
    const float* pw = n.w + n.off_w(k) + g * 4 * ldi + ti * 16 + cl;
#pragma unroll 2
    for (int kk = 0; kk < ot; ++kk) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(pd + kk * 16);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        z = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j], pw[(kk * 16 + j) * ldi], z, 0, 0, 0);
    }
    const int at0 = (tr * 16 + g * 4) * ldi + ti * 16 + cl;
    const float* y = n.act(k) + at0;
    float* o = n.grad(k - 1) + at0;
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r * ldi] = y[r * ldi] > 0.f ? z[r] : 0.f;
  }
  mf_sync();
}
// A parameter tile of layer k: 16 outputs from o * 16, 16 inputs from i * 16 (i == in_p / 16: the biases).
struct MfTile { int k, o, i; };
__device__ __forceinline__ int mf_tile(const MfNet& n, int t) {   // packed; layer L: none
  int k = 0;
  while (k < n.L && t >= n.out_p(k) / 16 * (n.in_p(k) / 16 + 1)) {
    t -= n.out_p(k) / 16 * (n.in_p(k) / 16 + 1);
    ++k;
  }
  const int o = k == 0 ? n.div.s1(t) : n.div.h1(t);
  return k < n.L ? (k << 16) | (o << 8) | (t - o * (n.in_p(k) / 16 + 1)) : n.L << 16;
}
// Unpacked where it is used: hidden from the compiler, which would otherwise keep every address that follows from it in
// registers over all epochs.
__device__ __forceinline__ MfTile mf_unpack(int packed) {
  asm volatile("" : "+s"(packed));
  return MfTile{packed >> 16, (packed >> 8) & 255, packed & 255};
}
// Adds the gradient of a tile over rt row tiles to z: rows g * 4 + r, column cl.  Biases: lane (g, cl) adds its rows of
// column cl, four running sums (mf_bias_sum joins them).
__device__ __forceinline__ f32x4 mf_tile_grad(const MfNet& n, const MfTile& sl, f32x4 z, int rt, int lane) {
  const int g = lane >> 4, cl = lane & 15;
  const int ldi = n.in_p(sl.k) + 4, ldo = n.out_p(sl.k) + 4;
  const float* pd = n.grad(sl.k) + g * 4 * ldo + cl + sl.o * 16;
  const float* pa = n.act(sl.k) + g * 4 * ldi + cl + sl.i * 16;
  if (sl.i == n.in_p(sl.k) / 16) {
#pragma unroll 2
    for (int tr = 0; tr < rt; ++tr) {
#pragma unroll
      for (int j = 0; j < 4; ++j) z[j] += pd[(tr * 16 + j) * ldo];
    }
  } else {
#pragma unroll 2
    for (int tr = 0; tr < rt; ++tr) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        z = __builtin_amdgcn_mfma_f32_16x16x4f32(pd[(tr * 16 + j) * ldo], pa[(tr * 16 + j) * ldi], z, 0, 0, 0);
    }
  }
  return z;
}
__device__ __forceinline__ float mf_bias_sum(const f32x4& z) {
  float t = (z[0] + z[1]) + (z[2] + z[3]);
  t += __shfl_xor(t, 16, 64);
  return t + __shfl_xor(t, 32, 64);
}
// AdamW with decoupled weight decay on one parameter; r1 = 1 / (1 - beta1^t), r2 = 1 / (1 - beta2^t)
__device__ __forceinline__ float adamw(const TrainArgs& a, float t, float& m, float& v, float gr, float r1, float r2) {
  m = a.beta1 * m + (1.f - a.beta1) * gr;
  v = a.beta2 * v + (1.f - a.beta2) * gr * gr;
  return t - a.lr * (m * r1 / (sqrtf(v * r2) + a.eps) + a.weight_decay * t);
}

template <int kSlots>
__global__ void __launch_bounds__(kMfThreads) k_filter_train_mfma(TrainArgs a, MfPlan plan, MfDivs divs) {
  constexpr int kRowRegs = row_regs(kSlots);
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int R = plan.rows;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, cl = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const MfNet n(a, divs, R, plan.apart, lds, 2 * kMfWaves);
  float* const red = n.rows0 - 2 * kMfWaves;
  const int L = n.L, s = n.s;

  for (int i = tid; i < plan.floats; i += kMfThreads) lds[i] = 0.f;
  __syncthreads();
  int n_params = 0;
#pragma unroll
  for (int k = 0; k < kFilterMaxLayers; ++k) {
    if (k >= L) break;
    for (int q = tid; q < n.out(k) * n.in(k); q += kMfThreads)
      lds[n.off_w(k) + q / n.in(k) * (n.in_p(k) + 4) + q % n.in(k)] = a.w[k][q];
    for (int q = tid; q < n.out(k); q += kMfThreads) n.bias0[k * n.hp + q] = a.b[k][q];
    n_params += n.out(k) * n.in(k) + n.out(k);
  }

  // parameter tiles of this wavefront
  int slot[kSlots];
  f32x4 mom[kSlots], var[kSlots], acc[kSlots];
#pragma unroll
  for (int i = 0; i < kSlots; ++i) {
    slot[i] = mf_tile(n, wave + kMfWaves * i);
    mom[i] = var[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // rows of a chunk on their way from memory: element i = tid + kMfThreads * u of the chunk's rows * s
  float conf[kRowRegs], label[kRowRegs];
  int at[kRowRegs];                           // its place in a [R][sp + 4] array
#pragma unroll
  for (int u = 0; u < kRowRegs; ++u) {
    const int i = tid + kMfThreads * u;
    at[u] = i < R * s ? i / s * (n.sp + 4) + i % s : -1;
  }
  auto fetch = [&](long long c0) {
    const int left = (int)min((long long)(R * s), (a.n - c0) * s);
    const float *cb = a.conf + c0 * s, *lb = a.label + c0 * s;   // uniform, so that the loads share one lane offset
#pragma unroll
    for (int u = 0; u < kRowRegs; ++u) {
      const bool have = kMfThreads * u + tid < left;
      conf[u] = have ? (cb + kMfThreads * u)[tid] : 0.f;
      label[u] = have ? (lb + kMfThreads * u)[tid] : 0.f;
    }
  };
  const bool resident = a.n <= R;
  fetch(0);
  __syncthreads();

  const float inv_m = 1.f / ((float)a.n * (float)s);
  float b1t = 1.f, b2t = 1.f;                 // beta^t
  for (int ep = 0; ep < a.epochs; ++ep) {
#pragma unroll
    for (int i = 0; i < kSlots; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    float loss = 0.f;
    for (long long c0 = 0; c0 < a.n; c0 += R) {
      const int rows = (int)min((long long)R, a.n - c0), rt = (rows + 15) / 16;
      if (c0 > 0) mf_sync();                  // the chunk before is done with its rows
#pragma unroll
      for (int u = 0; u < kRowRegs; ++u)
        if (at[u] >= 0) {
          if (!resident || ep == 0) n.rows0[at[u]] = conf[u];
          n.d_last[at[u]] = label[u];
        }
      if (!resident) fetch(c0 + R < a.n ? c0 + R : 0);
      mf_sync();
      loss += mf_forward(n, rows, inv_m, wave, lane);
      // gradients of the owned parameter tiles, of layer `only` or of all
      auto tile_grads = [&](int only) {
#pragma unroll
        for (int i = 0; i < kSlots; ++i) {
          const MfTile sl = mf_unpack(slot[i]);
          if (sl.k >= L || (only >= 0 && sl.k != only)) continue;
          acc[i] = mf_tile_grad(n, sl, acc[i], rt, lane);
        }
      };
      for (int k = L - 1; k > 0; --k) {
        if (!n.apart) {     // layer k's input is about to be replaced by the gradient there
          tile_grads(k);
          mf_sync();
        }
        mf_back(n, k, rt, wave, lane);
      }
      tile_grads(n.apart ? -1 : 0);
    }
    // loss of the epoch (before its update); two places in turn, so that nothing has to wait for the reader
    if (a.loss_out) {
#pragma unroll
      for (int of = 32; of > 0; of >>= 1) loss += __shfl_xor(loss, of, 64);
      if (lane == 0) red[(ep & 1) * kMfWaves + wave] = loss;
    }
    b1t *= a.beta1;
    b2t *= a.beta2;
    const float r1 = 1.f / (1.f - b1t), r2 = 1.f / (1.f - b2t);
#pragma unroll
    for (int i = 0; i < kSlots; ++i) {
      const MfTile sl = mf_unpack(slot[i]);
      const int k = sl.k;
      if (k >= L) continue;
      const int ldi = n.in_p(k) + 4;
      const bool is_bias = sl.i == n.in_p(k) / 16;
      if (is_bias) acc[i][0] = mf_bias_sum(acc[i]);   // lanes of group 0 own the tile's 16 biases, element 0
      const bool col_in = is_bias ? g == 0 : sl.i * 16 + cl < n.in(k);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = sl.o * 16 + (is_bias ? cl : g * 4 + r);
        if (!col_in || o >= n.out(k) || (is_bias && r > 0)) continue;
        float* th = is_bias ? n.bias0 + k * n.hp + o : lds + n.off_w(k) + o * ldi + sl.i * 16 + cl;
        float m = mom[i][r], v = var[i][r];
        *th = adamw(a, *th, m, v, acc[i][r], r1, r2);
        mom[i][r] = m;
        var[i][r] = v;
      }
    }
    mf_sync();
    if (a.loss_out && tid == 0) {
      float tot = 0.f;
      for (int w = 0; w < kMfWaves; ++w) tot += red[(ep & 1) * kMfWaves + w];
      a.loss_out[ep] = tot * inv_m;
    }
  }
  __syncthreads();
  int done = 0;                               // parameters of the layers before
#pragma unroll
  for (int k = 0; k < kFilterMaxLayers; ++k) {
    if (k >= L) break;
    const int nw = n.out(k) * n.in(k);
    for (int q = tid; q < nw; q += kMfThreads)
      a.w[k][q] = lds[n.off_w(k) + q / n.in(k) * (n.in_p(k) + 4) + q % n.in(k)];
    for (int q = tid; q < n.out(k); q += kMfThreads) a.b[k][q] = n.bias0[k * n.hp + q];
#pragma unroll
    for (int i = 0; i < kSlots; ++i) {
      const MfTile sl = mf_unpack(slot[i]);
      if (sl.k != k) continue;
      const bool is_bias = sl.i == n.in_p(k) / 16;
      const int c = sl.i * 16 + cl;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = sl.o * 16 + (is_bias ? cl : g * 4 + r);
        if (o >= n.out(k) || (is_bias ? g > 0 || r > 0 : c >= n.in(k))) continue;
        const int p = done + (is_bias ? nw + o : o * n.in(k) + c);
        a.opt_state[p] = mom[i][r];
        a.opt_state[n_params + p] = var[i][r];
      }
    }
    done += nw + n.out(k);
  }
}

// ------------------------------------------------------------------------------------------------
// Rows over workgroups.  With a workspace the rows of an epoch are dealt to up to kSplitMax workgroups, each of which
// leaves the gradient of its rows, a loss and nothing else; the kernel boundary is the only synchronisation.
//   The workspace holds everything as an image of the padded parameters (per layer [out_p][in_p], then all biases): the
// state (parameters and both moments, twice) and one partial gradient per workgroup (FUSED: twice).  What is padding has a
// gradient of exactly zero, so that parameters and moments there stay zero without a test.
//   Small images (FUSED): one launch an epoch.  Every workgroup sums the partial gradients of the epoch before, applies
// AdamW to all parameters on its way into LDS, and goes on with its rows; the first one also writes the new state.  States
// and partial gradients alternate between two places, since workgroups of one launch read the one while others write
// the other.  Larger images: a second launch sums and updates, spread over the chip.
//   Bound by the chain launch - arguments - loads - phases between barriers: 241 rows of 32 -> 32 -> 32 take 8.4 us an epoch
// (14.1 in one workgroup; half of it is the start and the update), 4096 rows of 64 -> 128 -> 64 23 us (1,204): rows 18, of
// which its matrix instructions need 4.5, update 5.
//   How many rows to a workgroup: the estimate of split_plan, from these (us an epoch with 16 / 32 / 48 / 64 rows):
// 241 x (32, 32, 32) 8.4 / 8.3 / 10.0 / 9.7, one launch each; 1500 x (32, 32, 32) 14.9 / 12.2 / 12.0 / 11.1 (one launch); 700 x
// (16, 128, 16) 11.2 / 12.1 / 15.5 (from here on one launch) / 14.8; 200 x (64, 128, 64) 14.1 / 17.7 / 20.7 / 27.7, two launches;
// 4096 x (64, 128, 64), two launches, - / 23.6 / 25.2 / 30.9 (256 workgroups of 16 rows, twice the memory: 36.0).
// One workgroup over all epochs needs no start: 40 rows of (32, 32, 32) 6.0 (split 7.6), 100 rows 8.5 (8.9), 241 rows 14.1.
struct SplitPlan {
  int groups;          // workgroups (0: not split)
  int group_rows;      // rows of each
  int chunk;           // of these at once in LDS
  int fused;
  int floats;          // dynamic LDS
  int image, stride;   // floats of an image; of a partial gradient (the image, then a loss of every wavefront)
};
constexpr int kSplitMax = 128;
constexpr int kFusedFloats = 64 * 1024;       // partial gradients that every workgroup can read: 256 KB
static SplitPlan split_plan(int s, int h, int L, long long n) {
  SplitPlan p = {};
  int fixed, per_row, tiles;
  mf_sizes(s, h, L, &fixed, &per_row, &tiles);
  if (tiles > kMaxSlots * kMfWaves) return p;
  per_row += (L - 1) * (pad16(h) + 4);
  const int cap = (kMfLdsFloats - fixed) / per_row / 16 * 16;
  if (cap < 16) return p;
  const int sp = pad16(s), hp = L > 1 ? pad16(h) : sp;
  p.image = (L - 1) * hp + sp;
  for (int k = 0; k < L; ++k) p.image += (k == 0 ? sp : hp) * (k == L - 1 ? sp : hp);
  p.stride = p.image + kMfWaves;
  int products = 0;                           // matrix instructions for 16 rows
  for (int k = 0; k < L; ++k) products += (k == 0 ? 8 : 12) * ((k == 0 ? sp : hp) / 16) * ((k == L - 1 ? sp : hp) / 16);
  const long long row_tiles = (n + 15) / 16;
  const long long most = std::min<long long>(kSplitMax, ((long long)kTrainSplitFloats - 6 * p.image) / p.stride);
  const long long least = (row_tiles + most - 1) / most;
  double best = 4. + row_tiles * products / 125.;        // one workgroup over all epochs
  long long per = row_tiles;
  p.groups = 1;
  for (long long r = least; r < least + 8; ++r) {
    const long long groups = (row_tiles + r - 1) / r;
    if (groups < 2) break;
    const double floats = (double)groups * p.stride;
    const bool fused = floats <= kFusedFloats;
    const double cost = r * products / 150. +
                        (fused ? 4.6 + 3.2 * ((p.image / 4 + kMfThreads - 1) / kMfThreads) + floats / 38400. : 10. + floats / 250000. + groups / 40.);
    if (cost < best) { best = cost; per = r; p.groups = (int)groups; p.fused = fused; }
  }
  p.group_rows = (int)std::min<long long>(per * 16, 1 << 24);
  p.chunk = std::min(cap, p.group_rows);
  p.floats = fixed + p.chunk * per_row;
  return p;
}
size_t filter_train_split_bytes(int s, int hidden, int n_layers, long long n) {
  const SplitPlan p = split_plan(s, hidden, n_layers, n);
  return p.groups > 1 ? (6 * (size_t)p.image + (p.fused ? 2 : 1) * (size_t)p.groups * p.stride) * sizeof(float) : 0;
}

struct SplitEpoch {
  const float* state;      // parameters, first and second moments: images one after the other
  float* state_out;
  const float* parts;      // partial gradients to apply first (FUSED; null in the first epoch)
  float* parts_out;
  float r1, r2;            // 1 / (1 - beta^t) of the update
  float* loss_out;         // where the loss of `parts` goes, or null
  long long group_rows;
  int chunk, groups, image, stride;
  MfDivs divs;
};
// This thread's part (of n threads) of the loss of the rows behind e.parts: 16 numbers of every workgroup, eight at a time.
__device__ __forceinline__ double split_loss(const SplitEpoch& e, int thread, int n) {
  double l = 0.;
  for (int z0 = thread >> 4; z0 < e.groups; z0 += n / 2) {
    float x[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int z = z0 + n / 16 * q;
      x[q] = z < e.groups ? e.parts[(size_t)z * e.stride + e.image + (thread & 15)] : 0.f;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) l += x[q];
  }
#pragma unroll
  for (int of = 32; of > 0; of >>= 1) l += __shfl_xor(l, of, 64);
  return l;
}
// Every launch runs its code once, so there is little of it: loops that are not unrolled, gradients straight to memory
// (a second chunk of rows reads them back and adds), and all loads of the beginning sent off before the first is needed.
template <bool FUSED>
__global__ void __launch_bounds__(kMfThreads) k_filter_train_rows(TrainArgs a, SplitEpoch e) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, cl = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const MfNet n(a, e.divs, e.chunk, true, lds, 0);
  const int L = n.L, s = n.s;
  const float inv_m = 1.f / ((float)a.n * (float)s);
  const long long r0 = blockIdx.x * e.group_rows, r1 = min((long long)a.n, r0 + e.group_rows);

  // rows of a chunk: inputs and labels, padding zero; element i of the padded rows
  struct Elem { float conf, label; };
  auto row_elem = [&](long long c0, int rows, int i) {
    const int r = n.div.s(i >> 4), c = i - r * n.sp;
    const size_t at = (size_t)(c0 + r) * s + c;
    return r < rows && c < s ? Elem{a.conf[at], a.label[at]} : Elem{0.f, 0.f};
  };
  auto rows_in = [&](long long c0, int rows, Elem next) {
    const int total = (rows + 15) / 16 * 16 * n.sp;
#pragma unroll 1
    for (int i = tid; i < total; i += kMfThreads) {
      const Elem x = next;
      if (i + kMfThreads < total) next = row_elem(c0, rows, i + kMfThreads);
      const int at = i + n.div.s(i >> 4) * 4;
      n.rows0[at] = x.conf;
      n.d_last[at] = x.label;
    }
  };
  const int first_rows = (int)min((long long)e.chunk, r1 - r0);
  const Elem first_elem = row_elem(r0, first_rows, tid);
  // the image into LDS, through the update of the epoch before
  const f32x4* st = reinterpret_cast<const f32x4*>(e.state);
  const int image4 = e.image / 4, w4 = image4 - ((L - 1) * n.hp + n.sp) / 4;
  const bool first = blockIdx.x == 0;
  auto to_lds = [&](int i, const f32x4& t) {
    int at = (int)(n.bias0 - lds) + (i - w4) * 4;
    if (i < w4) {
      int k = 0, q = i;
      while (q >= n.out_p(k) * n.in_p(k) / 4) { q -= n.out_p(k) * n.in_p(k) / 4; ++k; }
      at = n.off_w(k) + (q + n.div_in(k, q >> 2)) * 4;      // q / 4: 16-wide pieces
    }
    *reinterpret_cast<f32x4*>(lds + at) = t;
  };
  if (FUSED && e.parts) {
#pragma unroll 1
    for (int i = tid; i < image4; i += kMfThreads) {
      f32x4 t = st[i], m = st[image4 + i], v = st[2 * image4 + i];
      f32x4 gr = {0.f, 0.f, 0.f, 0.f};
      const float* pz = e.parts + 4 * i;
#pragma unroll 8
      for (int z = 0; z < e.groups; ++z, pz += e.stride) gr += *reinterpret_cast<const f32x4*>(pz);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float mj = m[j], vj = v[j];
        t[j] = adamw(a, t[j], mj, vj, gr[j], e.r1, e.r2);
        m[j] = mj;
        v[j] = vj;
      }
      if (first) {
        f32x4* o = reinterpret_cast<f32x4*>(e.state_out);
        o[i] = t;
        o[image4 + i] = m;
        o[2 * image4 + i] = v;
      }
      to_lds(i, t);
    }
  } else {
#pragma unroll 1
    for (int i0 = tid; i0 < image4; i0 += 5 * kMfThreads) {   // (20,480 parameters at once)
      f32x4 t[5];
#pragma unroll
      for (int q = 0; q < 5; ++q) t[q] = st[min(i0 + q * kMfThreads, image4 - 1)];
#pragma unroll
      for (int q = 0; q < 5; ++q)
        if (i0 + q * kMfThreads < image4) to_lds(i0 + q * kMfThreads, t[q]);
    }
  }
  rows_in(r0, first_rows, first_elem);
  if (FUSED && e.parts && e.loss_out && first && wave == kMfWaves - 1) {
    const double l = split_loss(e, lane, 64);
    if (lane == 0) *e.loss_out = (float)(l / ((double)a.n * s));
  }

  float* out = e.parts_out + (size_t)blockIdx.x * e.stride;
  float loss = 0.f;
#pragma unroll 1
  for (long long c0 = r0; c0 < r1; c0 += e.chunk) {
    const int rows = (int)min((long long)e.chunk, r1 - c0), rt = (rows + 15) / 16;
    if (c0 > r0) {
      mf_sync();                              // the chunk before is done with its rows
      rows_in(c0, rows, row_elem(c0, rows, tid));
    }
    mf_sync();
    loss += mf_forward(n, rows, inv_m, wave, lane);
#pragma unroll 1
    for (int k = L - 1; k > 0; --k) mf_back(n, k, rt, wave, lane);
    // Gradients: a wavefront takes 16 outputs of a layer by 32 inputs, two sums side by side that share the operand from
    // the outputs' side, and with the first inputs the outputs' biases.
    int k = 0, u = wave, iw = 0;              // layer, unit among its units, the layer's place in the image
#pragma unroll 1
    while (true) {
      const int ip = n.in_p(k), ot = n.out_p(k) / 16;
      if (u >= ot * ((ip + 31) / 32)) {
        u -= ot * ((ip + 31) / 32);
        iw += n.out_p(k) * ip;
        if (++k == L) break;
        continue;
      }
      const int i2 = n.div_out(k, u), o = u - i2 * ot;      // all outputs with the first inputs, then with the next
      u += kMfWaves;
      const int ldi = ip + 4, ldo = n.out_p(k) + 4;
      const bool two = i2 * 32 + 16 < ip;     // (the last piece of an odd number of them is formed twice)
      const float* pd = n.grad(k) + g * 4 * ldo + cl + o * 16;
      const float* pa = n.act(k) + g * 4 * ldi + cl + i2 * 32;
      const int second = two ? 16 : 0;
      f32x4 z0 = {0.f, 0.f, 0.f, 0.f}, z1 = z0, zb = z0;
#pragma unroll 2
      for (int tr = 0; tr < rt; ++tr, pd += 16 * ldo, pa += 16 * ldi) {
        float d[4], x0[4], x1[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) { d[j] = pd[j * ldo]; x0[j] = pa[j * ldi]; x1[j] = pa[j * ldi + second]; }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          zb[j] += d[j];
          z0 = __builtin_amdgcn_mfma_f32_16x16x4f32(d[j], x0[j], z0, 0, 0, 0);
          z1 = __builtin_amdgcn_mfma_f32_16x16x4f32(d[j], x1[j], z1, 0, 0, 0);
        }
      }
      float* po = out + iw + (o * 16 + g * 4) * ip + i2 * 32 + cl;
      const float b = mf_bias_sum(zb);
      float* pb = out + w4 * 4 + k * n.hp + o * 16 + cl;
      if (c0 > r0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) { z0[r] += po[r * ip]; z1[r] += po[r * ip + second]; }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) po[r * ip] = z0[r];
      if (two) {
#pragma unroll
        for (int r = 0; r < 4; ++r) po[r * ip + 16] = z1[r];
      }
      if (i2 == 0 && g == 0) *pb = c0 > r0 ? *pb + b : b;
    }
  }
#pragma unroll
  for (int of = 32; of > 0; of >>= 1) loss += __shfl_xor(loss, of, 64);
  if (lane == 0) out[e.image + wave] = loss;
}

// Sum of the partial gradients and AdamW: 16 lanes take 64 consecutive parameters, the 16 of a workgroup deal the
// partials among them and add up through LDS.  The last workgroup sums the loss.  `last`: the results go where the caller
// wants them.
__global__ void __launch_bounds__(256) k_filter_train_update(TrainArgs a, SplitEpoch e, int last) {
  __shared__ __attribute__((aligned(16))) float s_sum[16][64];
  const int tid = threadIdx.x, c4 = tid & 15, part = tid >> 4;
  if (blockIdx.x + 1 == gridDim.x) {
    __shared__ double s_loss[4];
    if (!e.loss_out) return;
    const double l = split_loss(e, tid, 256);
    if ((tid & 63) == 0) s_loss[tid >> 6] = l;
    __syncthreads();
    if (tid == 0) *e.loss_out = (float)((s_loss[0] + s_loss[1] + s_loss[2] + s_loss[3]) / ((double)a.n * a.s));
    return;
  }
  const int i4 = blockIdx.x * 16 + c4;
  f32x4 gr = {0.f, 0.f, 0.f, 0.f};
  if (i4 < e.image / 4) {
    const float* pz = e.parts + (size_t)part * e.stride + 4 * i4;
#pragma unroll 8
    for (int z = part; z < e.groups; z += 16, pz += (size_t)16 * e.stride) gr += *reinterpret_cast<const f32x4*>(pz);
  }
  *reinterpret_cast<f32x4*>(&s_sum[part][c4 * 4]) = gr;
  const int i = blockIdx.x * 64 + tid;
  const bool mine = tid < 64 && i < e.image;
  float t = 0.f, m = 0.f, v = 0.f;
  if (mine) { t = e.state[i]; m = e.state[e.image + i]; v = e.state[2 * e.image + i]; }
  __syncthreads();
  if (!mine) return;
  float sum = 0.f;
#pragma unroll
  for (int p = 0; p < 16; ++p) sum += s_sum[p][tid];
  t = adamw(a, t, m, v, sum, e.r1, e.r2);
  if (!last) {
    e.state_out[i] = t;
    e.state_out[e.image + i] = m;
    e.state_out[2 * e.image + i] = v;
    return;
  }
  const int L = a.n_layers, s = a.s, h = L > 1 ? a.hidden : s, sp = pad16(s), hp = pad16(h);
  const int n_params = filter_param_count_dev(s, h, L);
  int q = i, done = 0;                        // place inside the layer's weights, then among the biases
  for (int k = 0; k < L; ++k) {
    const int ip = k == 0 ? sp : hp, op = k == L - 1 ? sp : hp, in = k == 0 ? s : h, out = k == L - 1 ? s : h;
    if (q >= 0 && q < op * ip && q / ip < out && q % ip < in) {
      const int o = q / ip * in + q % ip;
      a.w[k][o] = t;
      a.opt_state[done + o] = m;
      a.opt_state[n_params + done + o] = v;
    }
    q -= op * ip;
    done += out * in + out;
  }
  done = 0;
  for (int k = 0; k < L; ++k) {               // q counts from the first bias on
    const int op = k == L - 1 ? sp : hp, in = k == 0 ? s : h, out = k == L - 1 ? s : h;
    if (q >= 0 && q < out) {
      a.b[k][q] = t;
      a.opt_state[done + out * in + q] = m;
      a.opt_state[n_params + done + out * in + q] = v;
    }
    q -= op;
    done += out * in + out;
  }
}
// The image of the parameters as they are, moments zero.
__global__ void __launch_bounds__(256) k_filter_train_image(TrainArgs a, float* state, int image) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= image) return;
  const int L = a.n_layers, s = a.s, h = L > 1 ? a.hidden : s, sp = pad16(s), hp = pad16(h);
  float v = 0.f;
  int q = i;
  for (int k = 0; k < L; ++k) {
    const int ip = k == 0 ? sp : hp, op = k == L - 1 ? sp : hp, in = k == 0 ? s : h, out = k == L - 1 ? s : h;
    if (q >= 0 && q < op * ip && q / ip < out && q % ip < in) v = a.w[k][q / ip * in + q % ip];
    q -= op * ip;
  }
  for (int k = 0; k < L; ++k) {
    const int op = k == L - 1 ? sp : hp, out = k == L - 1 ? s : h;
    if (q >= 0 && q < out) v = a.b[k][q];
    q -= op;
  }
  state[i] = v;
  state[image + i] = 0.f;
  state[2 * image + i] = 0.f;
}

// ------------------------------------------------------------------------------------------------
// The same for filters whose padded widths do not fit the matrix-core kernel (a single hidden width of several
// hundred units between narrow ends): scalar loops, every thread owns a few parameters and accumulates their
// gradient over the rows in ascending order.
constexpr int kTrainThreads = 1024;
constexpr int kTrainMaxOwn = 20;                 // parameters per thread
constexpr int kTrainLdsFloats = 36 * 1024;       // 144 KB
static int train_chunk_rows(int s, int hidden, int n_layers) {
  const int left = kTrainLdsFloats - filter_param_count(s, hidden, n_layers) - 64;
  int ch = left / (2 * (s + (n_layers - 1) * hidden));
  return ch > 64 ? 64 : ch;
}
int filter_train_supported(int s, int hidden, int n_layers) {
  return n_layers >= 1 && n_layers <= kFilterMaxLayers && s >= 1 && (n_layers == 1 || hidden >= 1) &&
         filter_param_count(s, hidden, n_layers) <= kTrainThreads * kTrainMaxOwn &&
         train_chunk_rows(s, hidden, n_layers) >= 8;
}
__global__ void __launch_bounds__(kTrainThreads) k_filter_train(TrainArgs a, int chunk) {
  extern __shared__ float lds[];
  const int s = a.s, h = a.hidden, L = a.n_layers, tid = threadIdx.x;
  // layer k maps width in(k) to width out(k); its parameters sit at off(k) (weights, then biases).
  // Closed forms rather than tables, so nothing here is indexed dynamically out of registers.
  auto in = [&](int k) { return k == 0 ? s : h; };
  auto out = [&](int k) { return k == L - 1 ? s : h; };
  const int first = h * s + h, mid = h * h + h;            // parameters of layer 0 / of a hidden->hidden layer
  auto off = [&](int k) { return k == 0 ? 0 : first + (k - 1) * mid; };
  const int n_params = off(L - 1) + s * in(L - 1) + s;
  auto layer_of = [&](int p) {
    if (L == 1 || p < first) return 0;
    const int k = 1 + (p - first) / mid;
    return k < L - 1 ? k : L - 1;
  };
  // LDS: parameters, then per chunk the input of every layer (A(0) = the confidence rows) and the
  // loss gradient at every layer's pre-activation (D), then reduction scratch
  float* th = lds;
  float* const baseA = th + n_params;
  float* const baseD = baseA + chunk * (s + (L - 1) * h);
  auto A = [&](int k) { return baseA + (k == 0 ? 0 : chunk * s + (k - 1) * chunk * h); };
  auto D = [&](int k) { return baseD + k * chunk * h; };
  float* red = baseD + chunk * ((L - 1) * h + s);          // 64 floats
  for (int p = tid; p < n_params; p += kTrainThreads) {
    const int k = layer_of(p), q = p - off(k), nw = out(k) * in(k);
    th[p] = q < nw ? a.w[k][q] : a.b[k][q - nw];
    a.opt_state[p] = 0.f;
    a.opt_state[n_params + p] = 0.f;
  }
  __syncthreads();
  const float inv_m = 1.f / ((float)a.n * (float)s);
  float b1t = 1.f, b2t = 1.f;     // beta^t
  for (int ep = 0; ep < a.epochs; ++ep) {
    float g[kTrainMaxOwn];
#pragma unroll
    for (int o = 0; o < kTrainMaxOwn; ++o) g[o] = 0.f;
    float loss = 0.f;
    for (long long c0 = 0; c0 < a.n; c0 += chunk) {
      const int rows = (int)min((long long)chunk, a.n - c0);
      for (int i = tid; i < rows * s; i += kTrainThreads) A(0)[i] = a.conf[c0 * s + i];
      __syncthreads();
      for (int k = 0; k + 1 < L; ++k) {                            // hidden activations
        const float* W = th + off(k);
        const float* Bv = W + out(k) * in(k);
        for (int i = tid; i < rows * out(k); i += kTrainThreads) {
          const int r = i / out(k), t = i % out(k);
          float acc = Bv[t];
          for (int j = 0; j < in(k); ++j) acc += W[t * in(k) + j] * A(k)[r * in(k) + j];
          A(k + 1)[i] = fmaxf(acc, 0.f);
        }
        __syncthreads();
      }
      {                                                            // logits, loss, dL/dz
        const int k = L - 1;
        const float* W = th + off(k);
        const float* Bv = W + s * in(k);
        for (int i = tid; i < rows * s; i += kTrainThreads) {
          const int r = i / s, j = i % s;
          float z = Bv[j];
          for (int t = 0; t < in(k); ++t) z += W[j * in(k) + t] * A(k)[r * in(k) + t];
          const float y = a.label[c0 * s + i];
          loss += fmaxf(z, 0.f) + log1pf(expf(-fabsf(z))) - y * z;   // softplus(z) - y z
          D(k)[i] = (1.f / (1.f + expf(-z)) - y) * inv_m;
        }
        __syncthreads();
      }
      for (int k = L - 1; k > 0; --k) {                            // back through layer k and the ReLU before it
        const float* W = th + off(k);
        for (int i = tid; i < rows * in(k); i += kTrainThreads) {
          const int r = i / in(k), t = i % in(k);
          float acc = 0.f;
          for (int j = 0; j < out(k); ++j) acc += D(k)[r * out(k) + j] * W[j * in(k) + t];
          D(k - 1)[i] = A(k)[i] > 0.f ? acc : 0.f;
        }
        __syncthreads();
      }
#pragma unroll
      for (int o = 0; o < kTrainMaxOwn; ++o) {                     // gradient of the owned parameters
        const int p = tid + o * kTrainThreads;
        if (p >= n_params) break;
        const int k = layer_of(p), q = p - off(k), nw = out(k) * in(k);
        float acc = 0.f;
        if (q < nw) {
          const int t = q / in(k), j = q % in(k);
          for (int r = 0; r < rows; ++r) acc += D(k)[r * out(k) + t] * A(k)[r * in(k) + j];
        } else {
          const int t = q - nw;
          for (int r = 0; r < rows; ++r) acc += D(k)[r * out(k) + t];
        }
        g[o] += acc;
      }
      __syncthreads();
    }
    // loss of the epoch (before its update)
    if (a.loss_out) {
#pragma unroll
      for (int of = 32; of > 0; of >>= 1) loss += __shfl_xor(loss, of, 64);
      if ((tid & 63) == 0) red[tid >> 6] = loss;
      __syncthreads();
      if (tid == 0) {
        float tot = 0.f;
        for (int w = 0; w < kTrainThreads / 64; ++w) tot += red[w];
        a.loss_out[ep] = tot * inv_m;
      }
    }
    // AdamW, decoupled weight decay
    b1t *= a.beta1;
    b2t *= a.beta2;
#pragma unroll
    for (int o = 0; o < kTrainMaxOwn; ++o) {
      const int p = tid + o * kTrainThreads;
      if (p >= n_params) break;
      const float m = a.beta1 * a.opt_state[p] + (1.f - a.beta1) * g[o];
      const float v = a.beta2 * a.opt_state[n_params + p] + (1.f - a.beta2) * g[o] * g[o];
      a.opt_state[p] = m;
      a.opt_state[n_params + p] = v;
      const float mh = m / (1.f - b1t), vh = v / (1.f - b2t);
      th[p] = th[p] - a.lr * (mh / (sqrtf(vh) + a.eps) + a.weight_decay * th[p]);
    }
    __syncthreads();
  }
  for (int p = tid; p < n_params; p += kTrainThreads) {
    const int k = layer_of(p), q = p - off(k), nw = out(k) * in(k);
    if (q < nw) a.w[k][q] = th[p];
    else a.b[k][q - nw] = th[p];
  }
}
template <int kSlots>
static void launch_mfma(const TrainArgs& a, const MfPlan& p, hipStream_t s) {
  auto kern = k_filter_train_mfma<kSlots>;
  static DynLdsAttr attr;
  attr.ensure(reinterpret_cast<const void*>(kern), kMfLdsFloats * (int)sizeof(float));
  hipLaunchKernelGGL(kern, dim3(1), dim3(kMfThreads), (size_t)p.floats * sizeof(float), s, a, p,
                     mf_divs(a.s, a.hidden, a.n_layers));
}
template <bool FUSED>
static void launch_rows(const TrainArgs& a, const SplitEpoch& e, const SplitPlan& p, hipStream_t s) {
  auto kern = k_filter_train_rows<FUSED>;
  static DynLdsAttr attr;
  attr.ensure(reinterpret_cast<const void*>(kern), kMfLdsFloats * (int)sizeof(float));
  hipLaunchKernelGGL(kern, dim3(p.groups), dim3(kMfThreads), (size_t)p.floats * sizeof(float), s, a, e);
}
static void launch_split(const TrainArgs& a, const SplitPlan& p, float* ws, hipStream_t s) {
  float* const state[2] = {ws, ws + 3 * (size_t)p.image};
  float* const parts[2] = {ws + 6 * (size_t)p.image, ws + 6 * (size_t)p.image + (size_t)p.groups * p.stride};
  hipLaunchKernelGGL(k_filter_train_image, dim3((p.image + 255) / 256), dim3(256), 0, s, a, state[0], p.image);
  SplitEpoch e = {};
  e.group_rows = p.group_rows; e.chunk = p.chunk; e.groups = p.groups; e.image = p.image; e.stride = p.stride;
  e.divs = mf_divs(a.s, a.hidden, a.n_layers);
  const dim3 update_grid((p.image + 63) / 64 + 1);
  double b1t = 1., b2t = 1.;                  // beta^t
  for (int ep = 0; ep < a.epochs; ++ep) {
    const int at = p.fused ? ep & 1 : 0;
    e.state = p.fused && ep > 0 ? state[at ^ 1] : state[0];
    e.state_out = state[at];
    e.parts = p.fused && ep > 0 ? parts[at ^ 1] : nullptr;
    e.parts_out = parts[at];
    e.loss_out = a.loss_out && ep > 0 ? a.loss_out + ep - 1 : nullptr;
    if (p.fused) launch_rows<true>(a, e, p, s);    // with the factors of the update before
    else launch_rows<false>(a, e, p, s);
    b1t *= a.beta1;
    b2t *= a.beta2;
    e.r1 = (float)(1. / (1. - b1t));
    e.r2 = (float)(1. / (1. - b2t));
    const bool last = ep + 1 == a.epochs;
    if (p.fused && !last) continue;
    e.state = e.state_out = state[at];
    e.parts = parts[at];
    e.loss_out = a.loss_out ? a.loss_out + ep : nullptr;
    hipLaunchKernelGGL(k_filter_train_update, update_grid, dim3(256), 0, s, a, e, last ? 1 : 0);
  }
}
void launch_filter_train(const TrainArgs& a, float* ws, hipStream_t s) {
  if (ws) {
    const SplitPlan sp = split_plan(a.s, a.hidden, a.n_layers, a.n);
    if (sp.groups > 1) return launch_split(a, sp, ws, s);
  }
  const MfPlan p = mf_plan(a.s, a.hidden, a.n_layers, a.n);
  if (p.rows > 0) {
    if (p.slots == 1) launch_mfma<1>(a, p, s);
    else if (p.slots == 2) launch_mfma<2>(a, p, s);
    else if (p.slots <= 3) launch_mfma<3>(a, p, s);
    else launch_mfma<kMaxSlots>(a, p, s);
    return;
  }
  const int chunk = train_chunk_rows(a.s, a.hidden, a.n_layers);
  const int n_params = filter_param_count(a.s, a.hidden, a.n_layers);
  const size_t smem =
      (size_t)(n_params + chunk * 2 * (a.s + (a.n_layers - 1) * a.hidden) + 64) * sizeof(float);
  static DynLdsAttr attr;
  attr.ensure(reinterpret_cast<const void*>(k_filter_train), kTrainLdsFloats * (int)sizeof(float));
  hipLaunchKernelGGL(k_filter_train, dim3(1), dim3(kTrainThreads), smem, s, a, chunk);
}

}  // namespace l2pd
