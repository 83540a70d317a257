// Bidirectional (non-causal) flash-style attention on bf16 MFMA for gfx950.
//
// Inputs are what the QKV GEMM epilogue leaves: rotated queries q [B*Tq, d], rotated keys
// kstore [B, Tpad, d] and transposed values vtstore [B, H, Dh, Tpad].  A workgroup owns 32*NQ
// queries of one (sequence, head) and splits the keys into NSPL contiguous ranges; wavefront
// (query group, key range) runs the online softmax of its 32 queries over its range, and the
// ranges are merged at the end.  Key/value tiles of 64 keys go global -> LDS directly into a ring of NST tiles
// per range (rows XOR-swizzled on the global side), one tile per range and iteration, shared by the query groups:
// one barrier per tile, after which the tiles NST - 1 ahead are sent off.
//
// The wave computes S^T = K Q^T (keys are MFMA rows, queries are columns), so that a lane holds
// scores of ONE query: the row maximum is 31 register maxima plus one cross-lane exchange, and the
// exponentiated scores are already laid out as the B operand of O^T = V^T P^T.  The key order
// inside each 16-key MFMA step is the accumulator's (keys {4h..4h+3, 8+4h..8+4h+3} for lane half h);
// V^T is read from LDS in that same order, which is legal because the contraction is a sum.
//
// Exponents are taken relative to the running maximum itself, so that the heaviest key of a row has P = 1, which bf16
// holds exactly.  (A reference that lags behind by up to 2^8 saves most rescalings of O^T, but then that key's P is
// rounded by up to 2^-9 while the sum of P is not: error of the output against float64, before its own rounding, 1.0e-3
// instead of 0.4e-3 at a score spread of 4 and 512 keys.)  The rescaling is skipped where no query's maximum has grown.
//
// Bound by vector instructions (32 exponentials a lane and tile) with two wavefronts per SIMD, by their latency
// with one; with few queries by the stream of stored keys and values.
#include "gemm_common.h"

namespace l2pd {

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

// the larger of x in the two halves of the wavefront, in every lane
__device__ __forceinline__ float max_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

template <int DH, int NQ, int NSPL, int NST>
__global__ void __launch_bounds__(NQ * NSPL * 64) k_attn_bf16(const bf16* __restrict__ q, const bf16* __restrict__ kstore,
                                                              const bf16* __restrict__ vtstore, bf16* __restrict__ out,
                                                              int B, int Tq, int Tk_all, int Tpad, int H, int n_chunks,
                                                              float* __restrict__ chunk_out,
                                                              const int* __restrict__ tk_dev, QueryRows sel, Gate g) {
  if (gate_skip(g)) return;
  constexpr int KT = 64;                       // keys per LDS tile
  constexpr int K_ROW = DH * 2;                // bytes per key row
  constexpr int K_BYTES = KT * K_ROW;
  constexpr int V_BYTES = DH * KT * 2;         // [DH rows][64 keys]
  constexpr int STAGE = K_BYTES + V_BYTES;
  constexpr int KL = K_BYTES / 1024 / NQ, VL = V_BYTES / 1024 / NQ;   // 1 KB loads per wavefront and tile
  static_assert(KL * NQ * 1024 == K_BYTES && VL * NQ * 1024 == V_BYTES, "tile/wavefronts mismatch");
  static_assert(NST >= 2 && (NST - 2) * (KL + VL) < 64, "ring depth");
  constexpr int KK = DH / 16;                  // MFMA steps over the feature dim
  constexpr int FO = DH / 32;                  // output row fragments
  constexpr int XW = FO * 16 + 2;              // floats a wave hands over per lane: O^T fragments, m, l
  // the exchange area of the final merge reuses the tile buffers; the launch sizes LDS for the larger of the two
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // [NSPL key ranges][NST tiles][K tile | V^T tile]

  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, lj = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qg = wave % NQ, sp = wave / NQ;    // query group and key range of this wavefront
  // Workgroups are dealt to the 8 XCDs round-robin by their linear id.  All query tiles of one
  // (sequence, head) read the same K / V^T, so they are given ids that land on one XCD and share
  // its L2 (T = 512: 1 MB of K/V per XCD instead of all 8 MB through every L2).
  const int per_head = gridDim.x / (H * B);     // query tiles x key chunks
  int hb, inner;
  if ((H * B) % 8 == 0) {
    const int slot = blockIdx.x >> 3;
    hb = (slot / per_head) * 8 + (blockIdx.x & 7);
    inner = slot % per_head;
  } else {
    hb = blockIdx.x / per_head;
    inner = blockIdx.x % per_head;
  }
  const int b = hb / H, h = hb % H;
  // per-sequence key count (sequences shortened by step-granular EoTP), else the launch's
  const int Tk = tk_dev ? min(Tk_all, tk_dev[b]) : Tk_all;
  const int d = H * DH;
  // With n_chunks > 1 the keys are also dealt to n_chunks workgroups per query tile (few queries,
  // many keys: one workgroup per head would leave most CUs idle); each writes its unnormalised
  // (O^T, m, l) to chunk_out and k_attn_merge combines them.
  const int qt = inner / n_chunks, ch = inner % n_chunks;
  const int q0 = qt * (32 * NQ) + qg * 32;
  const int sel_lo = sel.n > 0 ? sel.base + (sel.seq_gb ? sel.seq_gb[b] * sel.per_gb : 0) : 0;
  if (sel.n > 0 && (qt * (32 * NQ) >= sel_lo + sel.n || (qt + 1) * (32 * NQ) <= sel_lo)) return;   // no row asked for
  const int qrow = min(q0 + lj, Tq - 1);

  // Q as the B operand: lane (query lj, half hf) holds features kk*16 + hf*8 .. +7
  bf16x8_t fq[KK];
  {
    const bf16* qp = q + ((size_t)b * Tq + qrow) * d + h * DH + hf * 8;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) fq[kk] = *reinterpret_cast<const bf16x8_t*>(qp + kk * 16);
  }

  // Direct-to-LDS loads of a tile: this wavefront's pieces are qg + i * NQ, 1 KB each, lane l at byte 16 * l.
  // The 64 LDS banks sweep 256 bytes.  A K row is 256 B (DH = 128: key = row & 15 over its 16 chunks) or 128 B
  // (DH = 64: two rows per sweep, key = (row >> 1) & 7); a V^T row is 128 B.
  auto kkey = [](int r) { return DH == 128 ? (r & 15) : ((r >> 1) & 7); };
  constexpr int KC = DH / 8;                   // 16-byte chunks per key row
  const bf16* srcK[KL];
  const bf16* srcV[VL];
#pragma unroll
  for (int i = 0; i < KL; ++i) {
    const int r = (qg + i * NQ) * (64 / KC) + lane / KC, c = (lane % KC) ^ kkey(r);
    srcK[i] = kstore + ((size_t)b * Tpad + r) * d + h * DH + c * 8;
  }
#pragma unroll
  for (int i = 0; i < VL; ++i) {
    const int r = (qg + i * NQ) * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
    srcV[i] = vtstore + ((size_t)(b * H + h) * DH + r) * Tpad + c * 8;
  }
  const unsigned lds0 = __builtin_amdgcn_readfirstlane(
      (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)(smem + sp * NST * STAGE + qg * 1024));
  // The key tiles are dealt to the NSPL key ranges in contiguous runs of `per` tiles; every range
  // is walked by NQ wavefronts (one per query group), and all ranges advance together, one tile
  // per iteration.
  const int n_tiles = (Tk + KT - 1) / KT;
  const int per_chunk = (n_tiles + n_chunks - 1) / n_chunks;    // the host picks n_chunks so that no chunk is empty
  const int wg_first = ch * per_chunk, wg_count = min(per_chunk, n_tiles - wg_first);
  const int per = (wg_count + NSPL - 1) / NSPL;
  const int my_first = wg_first + sp * per, my_count = max(0, min(per, wg_first + wg_count - my_first));
  auto load_tile = [&](int t) {
    const size_t k0 = (size_t)(my_first + t) * KT;
    const unsigned dst = lds0 + (t % NST) * STAGE;
#pragma unroll
    for (int i = 0; i < KL; ++i) dma16(srcK[i] + k0 * d, dst + i * NQ * 1024);
#pragma unroll
    for (int i = 0; i < VL; ++i) dma16(srcV[i] + k0, dst + K_BYTES + i * NQ * 1024);
  };

  f32x16 o[FO];
#pragma unroll
  for (int f = 0; f < FO; ++f)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[f][r] = 0.f;
  float m = -INFINITY, lsum = 0.f;             // running maximum (scaled scores, base 2), sum of P
  const float sc = rsqrtf((float)DH) * 1.4426950408889634f;   // softmax scale folded with log2(e)
  const int keyK = kkey(lj), keyV = (lj >> 1) & 7;   // fragment rows are lj modulo 32

#pragma unroll
  for (int t = 0; t < NST - 1; ++t)
    if (t < my_count) load_tile(t);
  for (int t = 0; t < per; ++t) {
    // tile t has landed (the younger ones, if all of them were sent off, may still be on their way) ...
    if (t + NST - 2 < my_count) wait_vmcnt<(NST - 2) * (KL + VL)>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_waitcnt(0xc07f);        // ... and this wavefront's reads of tile t - 1 are complete
    if constexpr (NQ * NSPL > 1) lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if (t + NST - 1 < my_count) load_tile(t + NST - 1);   // into the place of tile t - 1
    if (t >= my_count) continue;
    const unsigned char* base = smem + (sp * NST + t % NST) * STAGE;
    const int k0 = (my_first + t) * KT;

    // S^T for the two 32-key halves of the tile
    f32x16 s[2];
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[sub][r] = 0.f;
      const unsigned char* krow = base + (sub * 32 + lj) * K_ROW;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        bf16x8_t fk = *reinterpret_cast<const bf16x8_t*>(krow + (((kk * 2 + hf) ^ keyK) << 4));
        s[sub] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fk, fq[kk], s[sub], 0, 0, 0);
      }
    }
    if (k0 + KT > Tk) {                        // the last tile: keys past the end
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (k0 + sub * 32 + (r >> 2) * 8 + hf * 4 + (r & 3) >= Tk) s[sub][r] = -INFINITY;
    }
    float tmax = -INFINITY;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, s[sub][r]);
    tmax = max_halves(tmax) * sc;
    if (__any(tmax > m)) {                     // (m = -inf on the first tile)
      const float mn = fmaxf(m, tmax);
      const float alpha = __builtin_amdgcn_exp2f(m - mn);
      m = mn;
      lsum *= alpha;
#pragma unroll
      for (int f = 0; f < FO; ++f)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[f][r] *= alpha;
    }
    float ps = 0.f;
    unsigned int pk[2][8];                     // bf16 pairs: [sub][4 per 16-key step * 2 steps]
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        // v_exp_f32 directly: arguments are <= 0 but for rounding, and a result below the normal range may flush to zero
        const float p0 = __builtin_amdgcn_exp2f(fmaf(s[sub][r], sc, -m)), p1 = __builtin_amdgcn_exp2f(fmaf(s[sub][r + 1], sc, -m));
        ps += p0 + p1;
        pk[sub][r >> 1] = pack_bf16(p0, p1);
      }
    lsum += ps;

    // O^T += V^T P^T, 16 keys per MFMA
#pragma unroll
    for (int m16 = 0; m16 < 4; ++m16) {
      const int sub = m16 >> 1, mm = m16 & 1;
      u32x4 pw = {pk[sub][mm * 4 + 0], pk[sub][mm * 4 + 1], pk[sub][mm * 4 + 2], pk[sub][mm * 4 + 3]};
      bf16x8_t fp = __builtin_bit_cast(bf16x8_t, pw);
#pragma unroll
      for (int f = 0; f < FO; ++f) {
        const unsigned char* vrow = base + K_BYTES + (f * 32 + lj) * (KT * 2) + hf * 8;
        u32x2 v0 = *reinterpret_cast<const u32x2*>(vrow + (((m16 * 2) ^ keyV) << 4));
        u32x2 v1 = *reinterpret_cast<const u32x2*>(vrow + (((m16 * 2 + 1) ^ keyV) << 4));
        u32x4 vw = {v0.x, v0.y, v1.x, v1.y};
        bf16x8_t fv = __builtin_bit_cast(bf16x8_t, vw);
        o[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fv, fp, o[f], 0, 0, 0);
      }
    }
  }

  // Merge the key ranges: range 0 of each query group folds in the others' (m, l, O^T), in range
  // order, through the tile buffers (dead now).  A range without keys hands over m = -inf, l = 0.
  if constexpr (NSPL > 1) {
    __syncthreads();
    float* xch = reinterpret_cast<float*>(smem);
    if (sp > 0) {
      float* mine = xch + (size_t)((sp - 1) * NQ + qg) * XW * 64 + lane;
#pragma unroll
      for (int f = 0; f < FO; ++f)
#pragma unroll
        for (int r = 0; r < 16; ++r) mine[(f * 16 + r) * 64] = o[f][r];
      mine[(FO * 16) * 64] = m;
      mine[(FO * 16 + 1) * 64] = lsum;
    }
    __syncthreads();
    if (sp > 0) return;
#pragma unroll
    for (int x = 1; x < NSPL; ++x) {
      const float* oth = xch + (size_t)((x - 1) * NQ + qg) * XW * 64 + lane;
      const float m2 = oth[(FO * 16) * 64], l2 = oth[(FO * 16 + 1) * 64];
      const float M = fmaxf(m, m2);   // m is finite: range 0 always holds the first tile
      const float a1 = __builtin_amdgcn_exp2f(m - M), a2 = __builtin_amdgcn_exp2f(m2 - M);
#pragma unroll
      for (int f = 0; f < FO; ++f)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[f][r] = o[f][r] * a1 + oth[(f * 16 + r) * 64] * a2;
      lsum = lsum * a1 + l2 * a2;
      m = M;
    }
  }

  const float l = lsum + __shfl_xor(lsum, 32, 64);
  if (n_chunks > 1) {
    if (q0 + lj < Tq) {
      float* po = chunk_out + ((((size_t)b * H + h) * Tq + q0 + lj) * n_chunks + ch) * (DH + 2);
#pragma unroll
      for (int f = 0; f < FO; ++f)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq)
          *reinterpret_cast<float4*>(po + f * 32 + rq * 8 + hf * 4) =
              make_float4(o[f][rq * 4 + 0], o[f][rq * 4 + 1], o[f][rq * 4 + 2], o[f][rq * 4 + 3]);
      if (hf == 0) { po[DH] = m; po[DH + 1] = l; }
    }
    return;
  }
  const float inv = 1.f / l;
  const int qi = q0 + lj, row = sel.n > 0 ? qi - sel_lo : qi, n_out = sel.n > 0 ? sel.n : Tq;   // row of the output
  if (qi < Tq && row >= 0 && row < n_out) {
    unsigned short* op = reinterpret_cast<unsigned short*>(out) + ((size_t)b * n_out + row) * d + h * DH;
#pragma unroll
    for (int f = 0; f < FO; ++f)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        u32x2 w;
        w.x = pack_bf16(o[f][rq * 4 + 0] * inv, o[f][rq * 4 + 1] * inv);
        w.y = pack_bf16(o[f][rq * 4 + 2] * inv, o[f][rq * 4 + 3] * inv);
        *reinterpret_cast<u32x2*>(op + f * 32 + rq * 8 + hf * 4) = w;
      }
  }
}

// One thread per (sequence, head, query, 4 features): combines the key chunks in ascending order.
template <int DH>
__global__ void __launch_bounds__(256) k_attn_merge(const float* __restrict__ chunk_out, bf16* __restrict__ out, int B,
                                                   int Tq, int H, int n_chunks, Gate g) {
  if (gate_skip(g)) return;
  const int t = blockIdx.x * 256 + threadIdx.x;
  const int per_q = DH / 4;
  if (t >= B * H * Tq * per_q) return;
  const int f4 = t % per_q, qi = (t / per_q) % Tq, h = (t / per_q / Tq) % H, b = t / per_q / Tq / H;
  const float* p = chunk_out + ((((size_t)b * H + h) * Tq + qi) * n_chunks) * (DH + 2);
  float M = -INFINITY;
  for (int c = 0; c < n_chunks; ++c) M = fmaxf(M, p[c * (DH + 2) + DH]);
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  float L = 0.f;
  for (int c = 0; c < n_chunks; ++c) {
    const float w = __builtin_amdgcn_exp2f(p[c * (DH + 2) + DH] - M);
    const float4 v = *reinterpret_cast<const float4*>(p + c * (DH + 2) + f4 * 4);
    acc.x += v.x * w; acc.y += v.y * w; acc.z += v.z * w; acc.w += v.w * w;
    L += p[c * (DH + 2) + DH + 1] * w;
  }
  const float inv = 1.f / L;
  u32x2 w2;
  w2.x = pack_bf16(acc.x * inv, acc.y * inv);
  w2.y = pack_bf16(acc.z * inv, acc.w * inv);
  unsigned short* op = reinterpret_cast<unsigned short*>(out) + ((size_t)b * Tq + qi) * (H * DH) + h * DH + f4 * 4;
  *reinterpret_cast<u32x2*>(op) = w2;
}

template <int DH, int NQ, int NSPL, int NST>
static void launch(const bf16* q, const bf16* kstore, const bf16* vtstore, bf16* out, int B, int Tq, int Tk,
                   int Tpad, int H, float* chunk_ws, size_t chunk_ws_bytes, const int* tk_dev, QueryRows sel, Gate g, hipStream_t s) {
  auto kern = k_attn_bf16<DH, NQ, NSPL, NST>;
  constexpr int tiles = NST * NSPL * (64 * DH * 2 + DH * 64 * 2);
  constexpr int xchg = (NSPL - 1) * NQ * ((DH / 32) * 16 + 2) * 64 * 4;
  constexpr int smem = tiles > xchg ? tiles : xchg;
  static DynLdsAttr attr;
  attr.ensure(reinterpret_cast<const void*>(kern), smem);
  const int q_tiles = (Tq + 32 * NQ - 1) / (32 * NQ), n_tiles = (Tk + 63) / 64;
  // few queries against many keys: deal the key tiles to several workgroups per query tile
  int n_chunks = 1;
  if (chunk_ws && !tk_dev && sel.n == 0 && q_tiles * H * B < 128 && n_tiles >= (Tq <= 64 ? 2 * NSPL : 8)) {   // chunks must not be empty: launch-wide key count only
    int want = (256 + q_tiles * H * B - 1) / (q_tiles * H * B);
    if (want > 16) want = 16;
    if (want > n_tiles / NSPL) want = n_tiles / NSPL;   // a tile for every key range of a chunk
    const int per_chunk = (n_tiles + want - 1) / want;
    n_chunks = (n_tiles + per_chunk - 1) / per_chunk;       // every chunk gets at least one tile
    if ((size_t)B * H * Tq * n_chunks * (DH + 2) * 4 > chunk_ws_bytes) n_chunks = 1;
  }
  dim3 grid(q_tiles * n_chunks * H * B);
  hipLaunchKernelGGL(kern, grid, dim3(NQ * NSPL * 64), smem, s, q, kstore, vtstore, out, B, Tq, Tk, Tpad, H, n_chunks,
                     chunk_ws, tk_dev, sel, g);
  if (n_chunks > 1) {
    const int n = B * H * Tq * (DH / 4);
    hipLaunchKernelGGL(k_attn_merge<DH>, dim3((n + 255) / 256), dim3(256), 0, s, chunk_ws, out, B, Tq, H, n_chunks, g);
  }
}

// The number of key ranges depends on the head size, the query rows per sequence and the head count, never on the batch
// size or the data (another number sums in another order, and a row's result must not depend on the batch it is
// part of); a wavefront's 32 queries are the same in every configuration, so how many wavefronts share the tiles may
// depend on the batch.  Measured with 32 heads of 128 (us; in brackets the kernel before: tiles through registers, four
// ranges and two barriers a tile):
//   512 rows          2 wavefronts x 2 ranges 14.1, 2 x 1 17.2, 8 x 1 22.2   (16.0)
//   8 x 512 rows      2 x 2 106, 4 x 2 69, 8 x 1 56                          (123)
//   1280 rows         4 x 2 54.7, 8 x 1 45.1                                 (70)
//   8 x 32 rows over 1280 keys   1 x 2 34.6 (4.97 TB/s), 1 x 1 37.8          (43)
//   32 x 64 rows over 768 keys   2 x 1 84.5 (5.16 TB/s), 2 x 2 94.3          (115)
//   16 heads of 64, 221 rows 2 x 2 6.2, 2 x 4 6.3 (6.3); 8 x 384 rows 4 x 2 13.6, 2 x 4 20.6 (23.7)
// Two ranges pay until one sequence by itself gives every CU a workgroup of 128 queries.
void launch_attn_bf16(const bf16* q, const bf16* kstore, const bf16* vtstore, bf16* out, int B, int Tq, int Tk,
                      int Tpad, int H, int Dh, float* chunk_ws, size_t chunk_ws_bytes, const int* tk_dev, QueryRows sel,
                      Gate g, hipStream_t s) {
#define L2PD_ATTN(DH, NQ, NSPL) \
  launch<DH, NQ, NSPL, 2>(q, kstore, vtstore, out, B, Tq, Tk, Tpad, H, chunk_ws, chunk_ws_bytes, tk_dev, sel, g, s)
#define L2PD_ATTN_DH(NQ, NSPL) (Dh == 128 ? L2PD_ATTN(128, NQ, NSPL) : L2PD_ATTN(64, NQ, NSPL))
  auto wgs = [&](int queries) { return (long long)((Tq + queries - 1) / queries) * H; };   // per sequence
  if (Tq <= 64) {      // block-only steps: bound by the stream of stored keys and values
    if (Tq <= 32) L2PD_ATTN_DH(1, 2);
    else if (wgs(64) * B >= 512) L2PD_ATTN_DH(2, 1);
    else L2PD_ATTN_DH(2, 2);
  } else if (wgs(128) <= 256) {
    if (wgs(64) * B >= 512) L2PD_ATTN_DH(4, 2);
    else L2PD_ATTN_DH(2, 2);
  } else {
    if (wgs(256) * B >= 128) L2PD_ATTN_DH(8, 1);
    else L2PD_ATTN_DH(4, 1);
  }
#undef L2PD_ATTN
#undef L2PD_ATTN_DH
}

}  // namespace l2pd
