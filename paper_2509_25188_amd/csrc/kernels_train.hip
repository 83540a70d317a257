// Filter training (Sec. 3.2, Eq. 6; Sec. 4.1: AdamW): full-batch epochs on the mean binary
// cross-entropy of sigmoid(W2 relu(W1 c + b1) + b2) against the EGP labels.  One workgroup: the
// model has a few thousand parameters, so the epochs are one dependent chain that wants no grid
// synchronisation (and the call has no memory for partial gradients of several workgroups).
#include "gemm_common.h"

namespace l2pd {

int filter_param_count(int s, int hidden, int n_layers) {
  int n = 0;
  for (int k = 0; k < n_layers; ++k) {
    const int in = k == 0 ? s : hidden, out = k == n_layers - 1 ? s : hidden;
    n += out * in + out;
  }
  return n;
}

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
// (0.6 TFLOP/s) for many: 241 rows of 32 -> 32 -> 32 take 14.3 us an epoch (4.1 at that rate), 4096 rows of
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

template <int kSlots>
__global__ void __launch_bounds__(kMfThreads) k_filter_train_mfma(TrainArgs a, MfPlan plan) {
  constexpr int kRowRegs = row_regs(kSlots);
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int R = plan.rows;
  const bool apart = plan.apart;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, cl = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int L = a.n_layers, s = a.s, h = L > 1 ? a.hidden : a.s, sp = pad16(s), hp = pad16(h);
  auto in = [&](int k) { return k == 0 ? s : h; };
  auto out = [&](int k) { return k == L - 1 ? s : h; };
  auto in_p = [&](int k) { return k == 0 ? sp : hp; };
  auto out_p = [&](int k) { return k == L - 1 ? sp : hp; };
  const int first = (L == 1 ? sp : hp) * (sp + 4), mid = hp * (hp + 4);
  auto off_w = [&](int k) { return k == 0 ? 0 : first + (k - 1) * mid; };
  const int n_w = off_w(L - 1) + (L == 1 ? first : sp * (hp + 4));
  float* const bias0 = lds + n_w;             // layer k's biases at + k * hp
  float* const red = bias0 + (L - 1) * hp + sp;
  float* const rows0 = red + 2 * kMfWaves;
  float* const d_last = rows0 + R * (sp + 4) + (L - 1) * R * (hp + 4);
  auto act = [&](int k) { return rows0 + (k == 0 ? 0 : R * (sp + 4) + (k - 1) * R * (hp + 4)); };   // input of layer k
  // loss gradient at layer k's pre-activation
  auto grad = [&](int k) {
    return k == L - 1 ? d_last : (apart ? d_last + R * (sp + 4) + k * R * (hp + 4) : act(k + 1));
  };
  // every thread's LDS accesses so far are complete and visible to the workgroup; global loads stay in flight
  auto sync = [&]() {
    __builtin_amdgcn_s_waitcnt(0xc07f);       // lgkmcnt(0)
    lds_barrier();
  };

  for (int i = tid; i < plan.floats; i += kMfThreads) lds[i] = 0.f;
  __syncthreads();
  int n_params = 0;
#pragma unroll
  for (int k = 0; k < kFilterMaxLayers; ++k) {
    if (k >= L) break;
    for (int q = tid; q < out(k) * in(k); q += kMfThreads)
      lds[off_w(k) + q / in(k) * (in_p(k) + 4) + q % in(k)] = a.w[k][q];
    for (int q = tid; q < out(k); q += kMfThreads) bias0[k * hp + q] = a.b[k][q];
    n_params += out(k) * in(k) + out(k);
  }

  // parameter tiles of this wavefront: layer, row tile, column tile (== in_p / 16: the bias)
  int slot[kSlots];
  f32x4 mom[kSlots], var[kSlots], acc[kSlots];
#pragma unroll
  for (int i = 0; i < kSlots; ++i) {
    int t = wave + kMfWaves * i, k = 0;
    while (k < L && t >= out_p(k) / 16 * (in_p(k) / 16 + 1)) {
      t -= out_p(k) / 16 * (in_p(k) / 16 + 1);
      ++k;
    }
    slot[i] = k < L ? (k << 16) | (t / (in_p(k) / 16 + 1) << 8) | (t % (in_p(k) / 16 + 1)) : L << 16;
    mom[i] = var[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // Layer, row tile and column tile of a slot, unpacked where they are used: hidden from the compiler, which would
  // otherwise keep every address that follows from them in registers over all epochs.
  struct Slot { int k, o, i; };
  auto unpack = [&](int packed) {
    asm volatile("" : "+s"(packed));
    return Slot{packed >> 16, (packed >> 8) & 255, packed & 255};
  };

  // rows of a chunk on their way from memory: element i = tid + kMfThreads * u of the chunk's rows * s
  float conf[kRowRegs], label[kRowRegs];
  int at[kRowRegs];                           // its place in a [R][sp + 4] array
#pragma unroll
  for (int u = 0; u < kRowRegs; ++u) {
    const int i = tid + kMfThreads * u;
    at[u] = i < R * s ? i / s * (sp + 4) + i % s : -1;
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
      if (c0 > 0) sync();                     // the chunk before is done with its rows
#pragma unroll
      for (int u = 0; u < kRowRegs; ++u)
        if (at[u] >= 0) {
          if (!resident || ep == 0) rows0[at[u]] = conf[u];
          d_last[at[u]] = label[u];
        }
      if (!resident) fetch(c0 + R < a.n ? c0 + R : 0);
      sync();
      // forward: z = A W^T + b, tile by tile
      for (int k = 0; k < L; ++k) {
        const int ldi = in_p(k) + 4, ldo = out_p(k) + 4, ot = out_p(k) / 16, kt = in_p(k) / 16;
        const float* A = act(k) + cl * ldi + g * 4;
        const float* W = lds + off_w(k) + cl * ldi + g * 4;
        const float* B = bias0 + k * hp + cl;
        float* O = (k == L - 1 ? d_last : act(k + 1)) + g * 4 * ldo + cl;
        for (int t = wave; t < rt * ot; t += kMfWaves) {
          const int tr = t / ot, to = t % ot;
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
          if (k < L - 1) {
#pragma unroll
            for (int r = 0; r < 4; ++r) o[r * ldo] = row + r < rows ? fmaxf(z[r], 0.f) : 0.f;
          } else {
            const bool col_in = to * 16 + cl < s;
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
        sync();
      }
      // gradients of the owned parameter tiles, of layer `only` or of all
      auto tile_grads = [&](int only) {
#pragma unroll
        for (int i = 0; i < kSlots; ++i) {
          const Slot sl = unpack(slot[i]);
          const int k = sl.k;
          if (k >= L || (only >= 0 && k != only)) continue;
          const int ldi = in_p(k) + 4, ldo = out_p(k) + 4;
          const float* pd = grad(k) + g * 4 * ldo + cl + sl.o * 16;
          const float* pa = act(k) + g * 4 * ldi + cl + sl.i * 16;
          f32x4 z = acc[i];
          if (sl.i == in_p(k) / 16) {
            // a bias: column sums; lane (g, cl) adds its rows of column cl, four running sums in z
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
          acc[i] = z;
        }
      };
      for (int k = L - 1; k > 0; --k) {
        if (!apart) {       // layer k's input is about to be replaced by the gradient there
          tile_grads(k);
          sync();
        }
        // back through layer k and the ReLU before it
        const int ldi = in_p(k) + 4, ldo = out_p(k) + 4, ot = out_p(k) / 16, it = in_p(k) / 16;
        for (int t = wave; t < rt * it; t += kMfWaves) {
          const int tr = t / it, ti = t % it;
          f32x4 z = {0.f, 0.f, 0.f, 0.f};
          const float* pd = grad(k) + (tr * 16 + cl) * ldo + g * 4;
          const float* pw = lds + off_w(k) + g * 4 * ldi + ti * 16 + cl;
#pragma unroll 2
          for (int kk = 0; kk < ot; ++kk) {
            const f32x4 x = *reinterpret_cast<const f32x4*>(pd + kk * 16);
#pragma unroll
            for (int j = 0; j < 4; ++j)
              z = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j], pw[(kk * 16 + j) * ldi], z, 0, 0, 0);
          }
          const int at0 = (tr * 16 + g * 4) * ldi + ti * 16 + cl;
          const float* y = act(k) + at0;
          float* o = grad(k - 1) + at0;
#pragma unroll
          for (int r = 0; r < 4; ++r) o[r * ldi] = y[r * ldi] > 0.f ? z[r] : 0.f;
        }
        sync();
      }
      tile_grads(apart ? -1 : 0);
    }
    // loss of the epoch (before its update); two places in turn, so that nothing has to wait for the reader
    if (a.loss_out) {
#pragma unroll
      for (int of = 32; of > 0; of >>= 1) loss += __shfl_xor(loss, of, 64);
      if (lane == 0) red[(ep & 1) * kMfWaves + wave] = loss;
    }
    // AdamW, decoupled weight decay
    b1t *= a.beta1;
    b2t *= a.beta2;
#pragma unroll
    for (int i = 0; i < kSlots; ++i) {
      const Slot sl = unpack(slot[i]);
      const int k = sl.k;
      if (k >= L) continue;
      const int ldi = in_p(k) + 4;
      const bool is_bias = sl.i == in_p(k) / 16;
      if (is_bias) {        // lanes of group 0 own the tile's 16 biases, element 0
        float t = (acc[i][0] + acc[i][1]) + (acc[i][2] + acc[i][3]);
        t += __shfl_xor(t, 16, 64);
        acc[i][0] = t + __shfl_xor(t, 32, 64);
      }
      const bool col_in = is_bias ? g == 0 : sl.i * 16 + cl < in(k);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = sl.o * 16 + (is_bias ? cl : g * 4 + r);
        if (!col_in || o >= out(k) || (is_bias && r > 0)) continue;
        float* th = is_bias ? bias0 + k * hp + o : lds + off_w(k) + o * ldi + sl.i * 16 + cl;
        const float gr = acc[i][r];
        const float m = a.beta1 * mom[i][r] + (1.f - a.beta1) * gr;
        const float v = a.beta2 * var[i][r] + (1.f - a.beta2) * gr * gr;
        mom[i][r] = m;
        var[i][r] = v;
        const float t = *th;
        const float mh = m / (1.f - b1t), vh = v / (1.f - b2t);
        *th = t - a.lr * (mh / (sqrtf(vh) + a.eps) + a.weight_decay * t);
      }
    }
    sync();
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
    const int nw = out(k) * in(k);
    for (int q = tid; q < nw; q += kMfThreads) a.w[k][q] = lds[off_w(k) + q / in(k) * (in_p(k) + 4) + q % in(k)];
    for (int q = tid; q < out(k); q += kMfThreads) a.b[k][q] = bias0[k * hp + q];
#pragma unroll
    for (int i = 0; i < kSlots; ++i) {
      const Slot sl = unpack(slot[i]);
      if (sl.k != k) continue;
      const bool is_bias = sl.i == in_p(k) / 16;
      const int c = sl.i * 16 + cl;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int o = sl.o * 16 + (is_bias ? cl : g * 4 + r);
        if (o >= out(k) || (is_bias ? g > 0 || r > 0 : c >= in(k))) continue;
        const int p = done + (is_bias ? nw + o : o * in(k) + c);
        a.opt_state[p] = mom[i][r];
        a.opt_state[n_params + p] = var[i][r];
      }
    }
    done += nw + out(k);
  }
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
  hipLaunchKernelGGL(kern, dim3(1), dim3(kMfThreads), (size_t)p.floats * sizeof(float), s, a, p);
}
void launch_filter_train(const TrainArgs& a, hipStream_t s) {
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
