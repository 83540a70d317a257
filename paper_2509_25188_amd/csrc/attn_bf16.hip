// Bidirectional (non-causal) flash-style attention on bf16 MFMA for gfx950.
//
// Inputs are what the QKV GEMM epilogue leaves: rotated queries q [B*Tq, d], rotated keys
// kstore [B, Tpad, d] and transposed values vtstore [B, H, Dh, Tpad].  A workgroup owns 32*NQ
// queries of one (sequence, head) and splits the keys into contiguous ranges, NSPL of them walked side by side and NSER
// one after the other; wavefront (query group, run of ranges) runs the online softmax of its 32 queries over each of its
// ranges, and the ranges are joined at the end.  Key/value tiles of 64 keys go global -> LDS directly into a ring of
// NST tiles per side (rows XOR-swizzled on the global side), one tile per side and iteration, shared by the query
// groups: one barrier per tile, after which the tiles NST - 1 ahead are sent off.
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
// with one; with few queries by the stream of stored keys and values.  The launch bounds ask for two wavefronts per SIMD
// even where LDS allows one: with the whole register file to itself the compiler puts the accumulators into AGPRs, which
// vector instructions reach by copies only (512 rows 17.3 us, 13.7 within 256 VGPRs).
#include "gemm_common.h"

namespace l2pd {

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

// the larger of x in the two halves of the wavefront, in every lane
__device__ __forceinline__ float max_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

struct AttnDivs {
  Div per_head, heads, chunks;   // by query tiles x key chunks, by H, by the chunks
  int per_head_n;
};

// Key ranges: NSPL side by side, one to a wavefront, times NSER that a wavefront walks one after the other, each with a
// maximum, a sum and an output of its own.  They are joined in ascending order however they are dealt to wavefronts.
//   ONCE: a single query tile, so that every stored key and value is read once, by one workgroup, and a pass over cold weights
// lies between two such readings (dma16_once).  64 rows of each of 32 sequences over 704 keys, four layers: a step 5,030 -> 4,964 us.
template <int DH, int NQ, int NSPL, int NSER, int NST, bool ONCE>
__global__ void __launch_bounds__(NQ * NSPL * 64, 2) k_attn_bf16(const bf16* __restrict__ q, const bf16* __restrict__ kstore,
                                                                 const bf16* __restrict__ vtstore, bf16* __restrict__ out,
                                                                 int B, int Tq, int Tk_all, int Tpad, int H, int n_chunks,
                                                                 float* __restrict__ chunk_out,
                                                                 const int* __restrict__ tk_dev, QueryRows sel, AttnDivs div, Gate g) {
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
  constexpr int FH = FO / NSPL;                // of these, how many a wavefront joins and writes at the end
  constexpr int XW = FH * 16 + 2;              // floats handed over per lane and range: O^T fragments, m, l
  static_assert(NSPL == 1 || (NSPL == 2 && NSER <= 2), "side by side, a wavefront holds at most two ranges");
  // the exchange area of the final merge reuses the tile buffers; the launch sizes LDS for the larger of the two
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // [NSPL key ranges][NST tiles][K tile | V^T tile]

  const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, lj = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qg = wave % NQ, sp = wave / NQ;    // query group and key range of this wavefront
  // Workgroups are dealt to the 8 XCDs round-robin by their linear id.  All query tiles of one
  // (sequence, head) read the same K / V^T, so they are given ids that land on one XCD and share
  // its L2 (T = 512: 1 MB of K/V per XCD instead of all 8 MB through every L2).
  const bool spread = (H * B) % 8 == 0;
  const int slot = spread ? blockIdx.x >> 3 : blockIdx.x, quot = div.per_head(slot);
  const int inner = slot - quot * div.per_head_n;
  const int hb = spread ? quot * 8 + (blockIdx.x & 7) : quot;
  const int b = div.heads(hb), h = hb - b * H;
  // per-sequence key count (sequences shortened by step-granular EoTP), else the launch's
  const int Tk = tk_dev ? min(Tk_all, tk_dev[b]) : Tk_all;
  const int d = H * DH;
  // With n_chunks > 1 the keys are also dealt to n_chunks workgroups per query tile (few queries,
  // many keys: one workgroup per head would leave most CUs idle); each writes its unnormalised
  // (O^T, m, l) to chunk_out and k_attn_merge combines them.
  const int qt = div.chunks(inner), ch = inner - qt * n_chunks;
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
  // The swizzle key repeats every 16 rows: a wavefront's pieces KP (VP) apart differ by a constant stride.
  constexpr int KP = NQ * (64 / KC) < 16 ? 16 / (NQ * (64 / KC)) : 1, VP = NQ * 8 < 16 ? 2 : 1;
  const bf16* srcK[KP];
  const bf16* srcV[VP];
#pragma unroll
  for (int i = 0; i < KP; ++i) {
    const int r = (qg + i * NQ) * (64 / KC) + lane / KC, c = (lane % KC) ^ kkey(r);
    srcK[i] = kstore + ((size_t)b * Tpad + r) * d + h * DH + c * 8;
  }
#pragma unroll
  for (int i = 0; i < VP; ++i) {
    const int r = (qg + i * NQ) * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
    srcV[i] = vtstore + ((size_t)(b * H + h) * DH + r) * Tpad + c * 8;
  }
  const unsigned lds0 = __builtin_amdgcn_readfirstlane(
      (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)(smem + sp * NST * STAGE + qg * 1024));
  // The key tiles are dealt to the NSPL * NSER key ranges in contiguous runs of `per` tiles; every range is walked by
  // NQ wavefronts (one per query group), NSPL ranges at a time, which advance together, one tile per iteration.
  const int n_tiles = (Tk + KT - 1) / KT;
  const int per_chunk = div.chunks(n_tiles + n_chunks - 1);     // the host picks n_chunks so that no chunk is empty
  const int wg_first = ch * per_chunk, wg_count = min(per_chunk, n_tiles - wg_first);
  const int per = (wg_count + NSPL * NSER - 1) / (NSPL * NSER);
  const int my_first = wg_first + sp * NSER * per, my_count = max(0, min(NSER * per, wg_first + wg_count - my_first));
  auto load_tile = [&](int t) {
    const size_t k0 = (size_t)(my_first + t) * KT;
    const unsigned dst = lds0 + (t % NST) * STAGE;
#pragma unroll
    for (int i = 0; i < KL; ++i) dma16_weights<ONCE>(srcK[i % KP] + (k0 + (i - i % KP) * NQ * (64 / KC)) * d, dst + i * NQ * 1024);
#pragma unroll
    for (int i = 0; i < VL; ++i) dma16_weights<ONCE>(srcV[i % VP] + k0 + (size_t)((i - i % VP) * NQ * 8) * Tpad, dst + K_BYTES + i * NQ * 1024);
  };

  f32x16 o[FO];
#pragma unroll
  for (int f = 0; f < FO; ++f)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[f][r] = 0.f;
  float m = -INFINITY, lsum = 0.f;             // running maximum (scaled scores, base 2), sum of P
  const float sc = rsqrtf((float)DH) * 1.4426950408889634f;   // softmax scale folded with log2(e)
  const int keyK = kkey(lj), keyV = (lj >> 1) & 7;   // fragment rows are lj modulo 32

  // Folds a later range (m2, l2, O2 by its accessor) into an earlier one, N output fragments of it.  A range without keys
  // has m = -inf, l = 0; the first range always holds a tile, so the common maximum is finite.  The operations are
  // spelled out: the same bits in every configuration.
  auto fold = [&](auto& o1, float& m1, float& l1, float m2, float l2, auto o2) {
    constexpr int N = sizeof(o1) / sizeof(f32x16);
    const float M = fmaxf(m1, m2);
    const float a1 = __builtin_amdgcn_exp2f(m1 - M), a2 = __builtin_amdgcn_exp2f(m2 - M);
#pragma unroll
    for (int f = 0; f < N; ++f)
#pragma unroll
      for (int r = 0; r < 16; ++r) o1[f][r] = __fmaf_rn(o1[f][r], a1, __fmul_rn(o2(f, r), a2));
    l1 = __fmaf_rn(l1, a1, __fmul_rn(l2, a2));
    m1 = M;
  };
  f32x16 ob[NSER > 1 ? FO : 1];                // the wavefront's finished ranges
  float mb = -INFINITY, lb = 0.f;
  int left = per;                              // tiles of the range at hand still to come

  const int2 gate = gate_words(g);             // looked at when the first loads are on their way
#pragma unroll
  for (int t = 0; t < NST - 1; ++t)
    if (t < my_count) load_tile(t);
  if (gate_closed(g, gate)) {
    wait_vmcnt<0>();                           // LDS stays this workgroup's until its loads have landed
    return;
  }
  for (int t = 0; t < NSER * per; ++t) {
    // tile t has landed (the younger ones, if all of them were sent off, may still be on their way) ...
    if (t + NST - 2 < my_count) wait_vmcnt<(NST - 2) * (KL + VL)>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_waitcnt(0xc07f);        // ... and this wavefront's reads of tile t - 1 are complete
    if constexpr (NQ * NSPL > 1) lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
    if (t + NST - 1 < my_count) load_tile(t + NST - 1);   // into the place of tile t - 1
    if constexpr (NSER > 1) {
      if (left == 0) {                         // a range ends here: bank it and start the next from nothing
        if (t == per) {
          mb = m; lb = lsum;
#pragma unroll
          for (int f = 0; f < FO; ++f) ob[f] = o[f];
        } else {
          fold(ob, mb, lb, m, lsum, [&](int f, int r) { return o[f][r]; });
        }
        m = -INFINITY; lsum = 0.f;
#pragma unroll
        for (int f = 0; f < FO; ++f)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[f][r] = 0.f;
        left = per;
      }
      --left;
    }
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

  // Join the key ranges in ascending order.  Side by side, each of the two wavefronts of a query group takes half of the
  // output features: it hands the other half of its ranges over through the tile buffers (dead now).
  f32x16 res[FH];
  float rm, rl;
  if constexpr (NSPL == 1) {
    if constexpr (NSER > 1) fold(ob, mb, lb, m, lsum, [&](int f, int r) { return o[f][r]; });
#pragma unroll
    for (int f = 0; f < FO; ++f) res[f] = NSER > 1 ? ob[NSER > 1 ? f : 0] : o[f];
    rm = NSER > 1 ? mb : m;
    rl = NSER > 1 ? lb : lsum;
  } else {
    __syncthreads();
    float* const xch = reinterpret_cast<float*>(smem) + lane;
    auto area = [&](int to, int i) { return xch + (size_t)((to * NSER + i) * NQ + qg) * XW * 64; };
    auto hand_over = [&](auto to, int i, const f32x16 (&v)[FO], float vm, float vl) {
      float* x = area(to, i);
#pragma unroll
      for (int f = 0; f < FH; ++f)
#pragma unroll
        for (int r = 0; r < 16; ++r) x[(f * 16 + r) * 64] = v[decltype(to)::value * FH + f][r];
      x[(FH * 16) * 64] = vm;
      x[(FH * 16 + 1) * 64] = vl;
    };
    auto hand_all = [&](auto to) {
      if constexpr (NSER > 1) hand_over(to, 0, ob, mb, lb);
      hand_over(to, NSER - 1, o, m, lsum);
    };
    if (sp == 0) hand_all(std::integral_constant<int, 1>{});
    else hand_all(std::integral_constant<int, 0>{});
    __syncthreads();
    auto theirs = [&](int i) {                 // folds range i of the other wavefront
      const float* x = area(sp, i);
      fold(res, rm, rl, x[(FH * 16) * 64], x[(FH * 16 + 1) * 64], [&](int f, int r) { return x[(f * 16 + r) * 64]; });
    };
    if (sp == 0) {
#pragma unroll
      for (int f = 0; f < FH; ++f) res[f] = NSER > 1 ? ob[NSER > 1 ? f : 0] : o[f];
      rm = NSER > 1 ? mb : m;
      rl = NSER > 1 ? lb : lsum;
      if constexpr (NSER > 1) fold(res, rm, rl, m, lsum, [&](int f, int r) { return o[f][r]; });
#pragma unroll
      for (int i = 0; i < NSER; ++i) theirs(i);
    } else {
      const float* x = area(1, 0);
#pragma unroll
      for (int f = 0; f < FH; ++f)
#pragma unroll
        for (int r = 0; r < 16; ++r) res[f][r] = x[(f * 16 + r) * 64];
      rm = x[(FH * 16) * 64];
      rl = x[(FH * 16 + 1) * 64];
      if constexpr (NSER > 1) {
        theirs(1);
        fold(res, rm, rl, mb, lb, [&](int f, int r) { return ob[FH + f][r]; });
      }
      fold(res, rm, rl, m, lsum, [&](int f, int r) { return o[FH + f][r]; });
    }
  }

  const float l = rl + __shfl_xor(rl, 32, 64);
  const int f0 = NSPL > 1 ? sp * FH * 32 : 0;  // first feature of this wavefront's half
  if (n_chunks > 1) {
    if (q0 + lj < Tq) {
      float* po = chunk_out + ((((size_t)b * H + h) * Tq + q0 + lj) * n_chunks + ch) * (DH + 2);
#pragma unroll
      for (int f = 0; f < FH; ++f)
#pragma unroll
        for (int rq = 0; rq < 4; ++rq)
          *reinterpret_cast<float4*>(po + f0 + f * 32 + rq * 8 + hf * 4) =
              make_float4(res[f][rq * 4 + 0], res[f][rq * 4 + 1], res[f][rq * 4 + 2], res[f][rq * 4 + 3]);
      if (hf == 0 && f0 == 0) { po[DH] = rm; po[DH + 1] = l; }
    }
    return;
  }
  const float inv = 1.f / l;
  const int qi = q0 + lj, row = sel.n > 0 ? qi - sel_lo : qi, n_out = sel.n > 0 ? sel.n : Tq;   // row of the output
  if (qi < Tq && row >= 0 && row < n_out) {
    unsigned short* op = reinterpret_cast<unsigned short*>(out) + ((size_t)b * n_out + row) * d + h * DH + f0;
#pragma unroll
    for (int f = 0; f < FH; ++f)
#pragma unroll
      for (int rq = 0; rq < 4; ++rq) {
        u32x2 w;
        w.x = pack_bf16(res[f][rq * 4 + 0] * inv, res[f][rq * 4 + 1] * inv);
        w.y = pack_bf16(res[f][rq * 4 + 2] * inv, res[f][rq * 4 + 3] * inv);
        *reinterpret_cast<u32x2*>(op + f * 32 + rq * 8 + hf * 4) = w;
      }
  }
}

// One thread per (sequence, head, query, 4 features): combines the key chunks in ascending order.  NC: the chunks rounded up,
// so that all loads are in flight together (those past the last chunk read it again and count nothing).  32 queries of
// 32 heads, 5 chunks: 4.8 us (5.2 with two loops over the chunks).
template <int DH, int NC>
__global__ void __launch_bounds__(256) k_attn_merge(const float* __restrict__ chunk_out, bf16* __restrict__ out, int n, int Tq,
                                                   int H, int n_chunks, Div queries, Div heads, Gate g) {
  const int2 gate = gate_words(g);
  const int t = blockIdx.x * 256 + threadIdx.x;
  constexpr int per_q = DH / 4;
  const int f4 = t % per_q, row = min(t / per_q, n - 1);      // row: query by query, head by head, sequence by sequence
  const float* p = chunk_out + (size_t)row * n_chunks * (DH + 2);
  float m[NC], l[NC];
  f32x4 v[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const float* pc = p + min(c, n_chunks - 1) * (DH + 2);
    const u32x2 *pv = reinterpret_cast<const u32x2*>(pc + f4 * 4), *pm = reinterpret_cast<const u32x2*>(pc + DH);
    const u32x2 lo = pv[0], hi = pv[1], ml = *pm;              // rows of DH + 2 floats: 8-byte pieces
    v[c] = f32x4{__uint_as_float(lo.x), __uint_as_float(lo.y), __uint_as_float(hi.x), __uint_as_float(hi.y)};
    m[c] = c < n_chunks ? __uint_as_float(ml.x) : -INFINITY;
    l[c] = __uint_as_float(ml.y);
  }
  if (gate_closed(g, gate) || t / per_q >= n) return;
  float M = m[0];
#pragma unroll
  for (int c = 1; c < NC; ++c) M = fmaxf(M, m[c]);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  float L = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const float w = __builtin_amdgcn_exp2f(m[c] - M);
    if (c < n_chunks) {                        // (a chunk of infinities stays out as a whole)
      acc += v[c] * w;
      L += l[c] * w;
    }
  }
  const float inv = 1.f / L;
  u32x2 w2;
  w2.x = pack_bf16(acc[0] * inv, acc[1] * inv);
  w2.y = pack_bf16(acc[2] * inv, acc[3] * inv);
  const int bh = queries(row), qi = row - bh * Tq, b = heads(bh), h = bh - b * H;
  unsigned short* op = reinterpret_cast<unsigned short*>(out) + ((size_t)b * Tq + qi) * (H * DH) + h * DH + f4 * 4;
  *reinterpret_cast<u32x2*>(op) = w2;
}

template <int DH, int NQ, int NSPL, int NSER, int NST, bool ONCE = false>
static void launch(const bf16* q, const bf16* kstore, const bf16* vtstore, bf16* out, int B, int Tq, int Tk,
                   int Tpad, int H, float* chunk_ws, size_t chunk_ws_bytes, const int* tk_dev, QueryRows sel, Gate g, hipStream_t s) {
  if constexpr (!ONCE && NQ <= 2)
    if (g.cold && Tq <= 32 * NQ)
      return launch<DH, NQ, NSPL, NSER, NST, true>(q, kstore, vtstore, out, B, Tq, Tk, Tpad, H, chunk_ws, chunk_ws_bytes, tk_dev, sel, g, s);
  auto kern = k_attn_bf16<DH, NQ, NSPL, NSER, NST, ONCE>;
  constexpr int tiles = NST * NSPL * (64 * DH * 2 + DH * 64 * 2);
  constexpr int xchg = NSPL == 1 ? 0 : NSPL * NSER * NQ * ((DH / 32 / NSPL) * 16 + 2) * 64 * 4;
  constexpr int smem = tiles > xchg ? tiles : xchg;
  static DynLdsAttr attr;
  attr.ensure(reinterpret_cast<const void*>(kern), smem);
  const int q_tiles = (Tq + 32 * NQ - 1) / (32 * NQ), n_tiles = (Tk + 63) / 64;
  // few queries against many keys: deal the key tiles to several workgroups per query tile, a tile to every key range
  constexpr int R = NSPL * NSER;
  int n_chunks = 1;
  if (chunk_ws && !tk_dev && sel.n == 0 && q_tiles * H * B < 128 && n_tiles >= 8) {   // chunks must not be empty: launch-wide key count only
    int want = (256 + q_tiles * H * B - 1) / (q_tiles * H * B);
    if (want > 16) want = 16;
    if (want > (n_tiles + R - 1) / R) want = (n_tiles + R - 1) / R;
    const int per_chunk = (n_tiles + want - 1) / want;
    n_chunks = (n_tiles + per_chunk - 1) / per_chunk;       // every chunk gets at least one tile
    if ((size_t)B * H * Tq * n_chunks * (DH + 2) * 4 > chunk_ws_bytes) n_chunks = 1;
  }
  dim3 grid(q_tiles * n_chunks * H * B);
  const AttnDivs div = {Div(q_tiles * n_chunks), Div(H), Div(n_chunks), q_tiles * n_chunks};
  hipLaunchKernelGGL(kern, grid, dim3(NQ * NSPL * 64), smem, s, q, kstore, vtstore, out, B, Tq, Tk, Tpad, H, n_chunks,
                     chunk_ws, tk_dev, sel, div, g);
  if (n_chunks > 1) {
    const int n = B * H * Tq;
    const dim3 grid((n * (DH / 4) + 255) / 256);
    if (n_chunks <= 4)
      hipLaunchKernelGGL((k_attn_merge<DH, 4>), grid, dim3(256), 0, s, chunk_ws, out, n, Tq, H, n_chunks, Div(Tq), Div(H), g);
    else if (n_chunks <= 8)
      hipLaunchKernelGGL((k_attn_merge<DH, 8>), grid, dim3(256), 0, s, chunk_ws, out, n, Tq, H, n_chunks, Div(Tq), Div(H), g);
    else
      hipLaunchKernelGGL((k_attn_merge<DH, 16>), grid, dim3(256), 0, s, chunk_ws, out, n, Tq, H, n_chunks, Div(Tq), Div(H), g);
  }
}

// The number of key ranges, and with it the order of the sums, depends on the query rows of a sequence and the head count,
// never on the batch size or the data (a row's result must not depend on the batch it is part of): four, or two where one
// sequence by itself gives every CU a workgroup of 128 queries.  More ranges are also more exact, since each has its own
// heaviest key with P = 1.  How the ranges are dealt to wavefronts and how many wavefronts share the tiles changes no bit
// and follows the batch: side by side while the launch is one round of workgroups, one after the other (half the LDS, a
// second workgroup per CU) beyond that.  Only a launch of fewer than 128 workgroups over 512 keys or more is cut up by the
// shape of the launch (n_chunks above).
// Measured (us; in brackets with tiles through registers, four wavefronts' ranges and two barriers a tile):
//   32 heads of 128        2 wavefronts x 2 ranges side by side, x 2 in turn / 4 x 1, x 4 in turn
//     512 rows             13.7 / 19.1   (16.0)          2 x 512 rows   26.1 / 21.1  (30.2)
//     8 x 512 rows         105 / 61      (128)           2 x 300 rows   21.8 / 15.0  (25.9)
//   16 heads of 64
//     221 rows             6.2 / 8.4     (6.3)           8 x 221 rows   8.9 / 9.4    (12.1)
//   few workgroups, two query wavefronts a range / one: twice the workgroups, the tiles read by each (with events around the launch)
//     32 heads of 128      100 rows 11.1 / 10.8, 200 rows 11.7 / 11.4, 256 rows 11.6 / 11.4; 64 rows over 256 stored keys 12.6 / 11.2, over
//                          384 15.7 / 14.4, four sequences of them 16.3 / 15.1 (read twice, so without the hint of ONCE)
//     16 heads of 64       40 rows 7.7 / 7.9, 64 rows 7.9 / 7.6, 221 rows 9.1 / 8.7, 4 x 64 rows 7.8 / 7.6; 8 of 128, 4 x 64 rows 9.6 / 9.2
//     8 x 384 rows         17.5 / 15.9   (24.2)          8 x 600 rows   32.5 / 28.2  (50.5)
//   two ranges in all      4 x 2 side by side / 4 x 1, x 2 in turn
//     1024 rows, 32 of 128 27.2 / 31.8   (32.0)          1280 rows      56.9 / 48.3  (68.0)
//     4 x 1280 rows        156 / 139     (199)           2 x 2200 rows, 16 of 64  74.7 / 71.6  (108)
//   block rows over a store, 32 heads of 128
//     32 over 1280 keys    15.7 (16.7; chunks and merge)  8 x 32        35.3 (44.2; 4.9 TB/s)
//     64 over 768 keys     14.2 (15.6)                    8 x 64        2 x 2 x 2 24.7, 2 x 1 x 4 25.9 (30.9)
//     32 x 64              2 x 2 x 2 93.9, 2 x 1 x 4 86.9 (114; 5.0 TB/s)
void launch_attn_bf16(const bf16* q, const bf16* kstore, const bf16* vtstore, bf16* out, int B, int Tq, int Tk,
                      int Tpad, int H, int Dh, float* chunk_ws, size_t chunk_ws_bytes, const int* tk_dev, QueryRows sel,
                      Gate g, hipStream_t s) {
#define L2PD_ATTN(DH, NQ, NSPL, NSER) \
  launch<DH, NQ, NSPL, NSER, 2>(q, kstore, vtstore, out, B, Tq, Tk, Tpad, H, chunk_ws, chunk_ws_bytes, tk_dev, sel, g, s)
#define L2PD_ATTN_DH(NQ, NSPL, NSER) (Dh == 128 ? L2PD_ATTN(128, NQ, NSPL, NSER) : L2PD_ATTN(64, NQ, NSPL, NSER))
  auto wgs = [&](int queries) { return (long long)((Tq + queries - 1) / queries) * H; };   // per sequence
  const int room = 256 * (128 / Dh);       // workgroups with two ranges' tiles that the chip holds at once (160 KB of LDS a CU)
  const bool few = wgs(32) * B <= 256 && Tk <= 7 * 64;   // (from 8 tiles on a small launch deals them to workgroups)
  if (Tq <= 32 || few) {
    L2PD_ATTN_DH(1, 2, 2);
  } else if (Tq <= 64) {
    if (wgs(64) * B <= room) L2PD_ATTN_DH(2, 2, 2);
    else L2PD_ATTN_DH(2, 1, 4);
  } else if (wgs(128) < 256) {
    if (wgs(64) * B <= room) L2PD_ATTN_DH(2, 2, 2);
    else L2PD_ATTN_DH(4, 1, 4);
  } else {
    if (wgs(128) * B <= room) L2PD_ATTN_DH(4, 2, 1);
    else L2PD_ATTN_DH(4, 1, 2);
  }
#undef L2PD_ATTN
#undef L2PD_ATTN_DH
}

}  // namespace l2pd
