// bf16 MFMA GEMM for gfx950:  C[M, N] = A[M, K] * W[N, K]^T, fp32 accumulation (up to 64 rows: launch_few below, and the split
// projections in gemm_few_rows.hip).
//
// Both operands are K-contiguous, which is the layout v_mfma_f32_16x16x32_bf16 wants: a lane feeds eight
// consecutive K elements of one row.  Tiles go global -> LDS directly (global_load_lds_dwordx4: no VGPR
// staging, no ds_write).  One such load writes 1 KB = 8 LDS rows of 64 K elements, lane i at byte 16*i, so
// the XOR swizzle of the 128-byte rows is applied on the global side: lane i fetches chunk (i & 7) ^ key(r) of
// its row.  The LDS of gfx950 sweeps 64 banks x 4 B = 256 B, i.e. two tile rows, so the key is (r >> 1) & 7:
// 16 consecutive rows then cover every bank exactly once per 16-byte read.
//
// Two wavefronts per SIMD take turns.  Wavefronts 0-3 and 4-7 of the workgroup (the hardware puts w and w + 4 on
// one SIMD) run the same program, the second four one slot later, slots being separated by workgroup barriers: in
// every slot one wavefront of a SIMD keeps the matrix pipe busy from registers alone, while the other one does
// all of its LDS reads, address arithmetic, load issue and waiting.  (Wavefronts in step, their reads slotted
// between their own MFMAs, leave the pipe idle around every barrier.)
//
// A phase (one read slot, one MFMA slot) covers the whole 64-deep K stage of half of the wavefront's rows:
// phase 0 reads the stage's B fragments (kept for phase 1) and the upper half of the A fragments, phase 1 the lower
// half.  So B(k) is free once both groups are past phase 0 of stage k, A(k) after phase 1, and with DEPTH stages
// in flight the ring holds DEPTH B tiles and DEPTH + 1 A tiles: phase 0 of stage k sends off A(k + DEPTH) into the
// place of A(k - 1), phase 1 sends off B(k + DEPTH) into the place of B(k).
//
// MFMA shape: 16x16x32 and not 32x32x16.  The part is power limited in these loops, and the smaller shape spends
// less per flop: 4096 x 4096 x 12288 with random operands 275 us (1.50 PFLOP/s) against 312 us with 32x32x16 in the
// same kernel, 202 against 225 us with all-zero operands, where power does not bind.
//
// The fused epilogues are the ones the decoding step needs: rotary embedding + K / V^T store (QKV), SiLU(gate) * up
// (FFN), fp32 split-K partials that the next RMSNorm folds into the residual stream (O and down projections), and
// the LM head's per-tile (max, sum exp, argmax) reduction so that logits are never written.  "Pair" epilogues need
// two columns in one lane (feature i and i + Dh/2 for the rotation, gate and up column for SwiGLU): the weight rows
// are dealt to the tile so that of every 32 columns the first 16 are side 0 and the next 16 side 1 of the same pairs.
#include "gemm_common.h"

namespace l2pd {

enum { EPI_PARTIAL = 0, EPI_QKV = 1, EPI_SWIGLU = 2, EPI_LMHEAD = 3, EPI_PARTIAL_SER = 4 };
// EPI_PARTIAL_SER is EPI_PARTIAL with GemmArgs::serial honoured (a kernel of its own: the second set of
// accumulators costs registers).

struct GemmArgs {
  const bf16* A;
  const bf16* B0;
  const bf16* B1;
  const bf16* B2;
  int M, N, K;          // N counts tile-space columns (for pair epilogues: both sides)
  int splits, k_len;    // K range of a workgroup
  TileMap map;
  Gate gate;
  // EPI_PARTIAL: K range z writes to parts + z * part_stride (fp32 [M, N])
  float* parts;
  size_t part_stride;
  int add;              // splits == 1: parts is the residual stream, and the sum is added to it in place
  int serial;           // EPI_PARTIAL_SER, splits == 1: the workgroup walks `serial` K ranges one after the other, each
                        // into a fresh accumulator, and writes their sum, formed in ascending order: the bits that
                        // `serial` workgroups' partials give when the RMSNorm sums them
  int serial_stages;    // 64-deep stages of such a range
  // EPI_SWIGLU
  bf16* act;
  int F;
  // EPI_QKV
  QkvEpilogue qkv;
  Div heads, rows_per_seq;   // by H, by Tq
  int group_shift;      // 16-feature groups of half a head: 1 << group_shift
  // EPI_LMHEAD
  LmHeadEpilogue lm;
};

// First element of the weight row that belongs in row r of the tile's B operand.
template <int BN, int EPI>
__device__ __forceinline__ const bf16* weight_row(const GemmArgs& a, int tile_n, int r) {
  if constexpr (EPI == EPI_QKV) {
    const int half = a.qkv.Dh / 2;
    const int G = tile_n * (BN / 32) + (r >> 5), j = r & 31;
    const int hg = G >> a.group_shift, gi = G & ((1 << a.group_shift) - 1);   // head of Q, K, V stacked; its group of 16 features
    const int mat = min(a.heads(hg), 2), head = mat == 2 && hg >= 3 * a.qkv.H ? hg - a.heads(hg) * a.qkv.H : hg - mat * a.qkv.H;
    const bf16* base = mat == 0 ? a.B0 : (mat == 1 ? a.B1 : a.B2);
    return base + (size_t)(head * a.qkv.Dh + gi * 16 + (j & 15) + (j >> 4) * half) * a.K;
  } else if constexpr (EPI == EPI_SWIGLU) {
    const int G = tile_n * (BN / 32) + (r >> 5), j = r & 31;
    return (j >> 4 ? a.B1 : a.B0) + (size_t)min(G * 16 + (j & 15), a.F - 1) * a.K;
  } else {
    return a.B0 + (size_t)min(tile_n * BN + r, a.N - 1) * a.K;
  }
}

// What a wavefront does with its FM x FN accumulator fragments.  C layout of the 16x16 MFMA: register r of a lane is
// row (lane / 16) * 4 + r, column lane % 16.  smem: the tile buffers, dead by now.
template <int BM, int BN, int WM, int WN, int EPI>
__device__ __forceinline__ void epilogue(const GemmArgs& a, f32x4 (&acc)[BM / WM / 16][BN / WN / 16],
                                         unsigned char* smem, int wm, int wn, int tile_m, int tile_n, int z) {
  constexpr int FM = BM / WM / 16, FN = BN / WN / 16;
  const int tid = threadIdx.x, lane = tid & 63;
  const int rg = lane >> 4, cl = lane & 15;
  const int lr = cl & 3;                                   // after a transpose: row within the group of four
  const int row_base = tile_m * BM + wm * (BM / WM) + rg * 4;   // + i * 16 + r
  if constexpr (EPI == EPI_PARTIAL || EPI == EPI_PARTIAL_SER) {
    float* out = a.parts + (size_t)z * a.part_stride;
    const int col0 = tile_n * BN + wn * (BN / WN) + (cl & ~3);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        unsigned w[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = __float_as_uint(acc[i][j][r]);   // (bit_cast of a vector element reads element 0)
        quad_transpose(w, lane);
        const int row = row_base + i * 16 + lr, col = col0 + j * 16;
        if (row < a.M && col < a.N) {                      // N is a multiple of 4
          float4* o = reinterpret_cast<float4*>(out + (size_t)row * a.N + col);
          float4 v = make_float4(__uint_as_float(w[0]), __uint_as_float(w[1]), __uint_as_float(w[2]), __uint_as_float(w[3]));
          if (a.add) {
            const float4 h = *o;
            v = make_float4(h.x + v.x, h.y + v.y, h.z + v.z, h.w + v.w);
          }
          *o = v;
        }
      }
  } else if constexpr (EPI == EPI_SWIGLU) {
    static_assert((FM == 1 || FM % 2 == 0) && FN % 2 == 0, "fragments in pairs");
#pragma unroll
    for (int i = 0; i < FM; i += 2)
#pragma unroll
      for (int p = 0; p < FN / 2; ++p) {
        const int col = (tile_n * (BN / 32) + wn * (FN / 2) + p) * 16 + (cl & ~3);
        unsigned w[4];                                     // two row fragments share one transpose: low / high half words
        constexpr int second = FM > 1 ? 1 : 0;             // (the only one stands in for both)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float g0 = acc[i][2 * p][r], u0 = acc[i][2 * p + 1][r];
          const float g1 = acc[i + second][2 * p][r], u1 = acc[i + second][2 * p + 1][r];
          // SiLU(g) * u with the hardware reciprocal (1 ulp) instead of an exact division; the
          // operations are spelled out so that every tile configuration rounds alike
          const float s0 = __fmul_rn(__fmul_rn(g0, __builtin_amdgcn_rcpf(__fadd_rn(1.f, __expf(-g0)))), u0);
          const float s1 = __fmul_rn(__fmul_rn(g1, __builtin_amdgcn_rcpf(__fadd_rn(1.f, __expf(-g1)))), u1);
          w[r] = pack_bf16(s0, s1);
        }
        quad_transpose(w, lane);
#pragma unroll
        for (int h2 = 0; h2 <= second; ++h2) {
          const int row = row_base + (i + h2) * 16 + lr;
          uint2 o;
          o.x = h2 ? (w[0] >> 16) | (w[1] & 0xffff0000u) : (w[0] & 0xffffu) | (w[1] << 16);
          o.y = h2 ? (w[2] >> 16) | (w[3] & 0xffff0000u) : (w[2] & 0xffffu) | (w[3] << 16);
          if (row < a.M && col < a.F)                      // F is a multiple of 4
            *reinterpret_cast<uint2*>(reinterpret_cast<unsigned short*>(a.act) + (size_t)row * a.F + col) = o;
        }
      }
  } else if constexpr (EPI == EPI_QKV) {
    static_assert(FN % 2 == 0, "fragments in pairs");
    const QkvEpilogue& e = a.qkv;
    const int half = e.Dh / 2, gmask = (1 << a.group_shift) - 1;
    // Rotation table, up to two row fragments ahead: the compiler cannot move a load above a store that might alias it, so
    // read where it is needed every pair would wait out a memory round trip of its own (Q/K/V of 4096 rows 311 us with the
    // next pair's on the way, 307 with these).
    constexpr int AHEAD = FM < 3 ? FM : 3;
    float2 cs[AHEAD][FN / 2][4];
    int seq[AHEAD][4], pos[AHEAD][4];          // sequence and position of this lane's four rows
    auto look_up = [&](int i, int buf) {
      const int row0 = row_base + i * 16;
      int b = a.rows_per_seq(row0), t = row0 - b * e.Tq;
      int off = (e.seq_gb && row0 < a.M) ? e.seq_gb[b] * e.pos_per_gb : 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        seq[buf][r] = b;
        pos[buf][r] = e.pos0 + off + t;
        if (++t == e.Tq) {   // next sequence of the batch
          t = 0;
          ++b;
          off = (e.seq_gb && row0 + r + 1 < a.M) ? e.seq_gb[b] * e.pos_per_gb : 0;
        }
      }
#pragma unroll
      for (int p = 0; p < FN / 2; ++p) {
        const int G = tile_n * (BN / 32) + wn * (FN / 2) + p;
        if ((G >> a.group_shift) >= 2 * e.H) continue;       // V (or past the last column): no rotation
        const int dim = (G & gmask) * 16 + cl;
#pragma unroll
        for (int r = 0; r < 4; ++r)            // (rows past the last one: any place of the table)
          cs[buf][p][r] = e.rope[(unsigned)(row0 + r < a.M ? pos[buf][r] : e.pos0) * (unsigned)half + (unsigned)dim];
      }
    };
#pragma unroll
    for (int i = 0; i < AHEAD - 1; ++i) look_up(i, i);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int row0 = row_base + i * 16, at = i % AHEAD;
      if (i + AHEAD - 1 < FM) look_up(i + AHEAD - 1, (i + AHEAD - 1) % AHEAD);
      const int seq_st = lr == 0 ? seq[at][0] : (lr == 1 ? seq[at][1] : (lr == 2 ? seq[at][2] : seq[at][3]));
      const int pos_st = lr == 0 ? pos[at][0] : (lr == 1 ? pos[at][1] : (lr == 2 ? pos[at][2] : pos[at][3]));
#pragma unroll
      for (int p = 0; p < FN / 2; ++p) {
        const int G = tile_n * (BN / 32) + wn * (FN / 2) + p;
        const int hg = G >> a.group_shift, gi = G & gmask, mat = a.heads(hg), head = hg - mat * e.H;   // uniform over the wavefront
        if (mat > 2) continue;
        if (mat == 2) {
          // V is stored transposed ([B, H, Dh, Tpad]) so that attention reads keys contiguously: four positions at once
          // where the lane's rows are consecutive ones of a sequence from a multiple of four on (221 rows: 14.7 -> 13.3 us
          // against a rule for the whole launch, which no odd window passed)
          unsigned short* vt = reinterpret_cast<unsigned short*>(e.vtstore);
          const int dim = gi * 16 + cl;
          if (seq[at][3] == seq[at][0] && pos[at][0] % 4 == 0 && row0 + 3 < a.M) {   // (Tpad is a multiple of 64)
            const size_t o = ((size_t)(seq[at][0] * e.H + head) * e.Dh + dim) * e.Tpad + pos[at][0];
            uint2 lo4, hi4;
            lo4.x = pack_bf16(acc[i][2 * p][0], acc[i][2 * p][1]);
            lo4.y = pack_bf16(acc[i][2 * p][2], acc[i][2 * p][3]);
            hi4.x = pack_bf16(acc[i][2 * p + 1][0], acc[i][2 * p + 1][1]);
            hi4.y = pack_bf16(acc[i][2 * p + 1][2], acc[i][2 * p + 1][3]);
            *reinterpret_cast<uint2*>(vt + o) = lo4;
            *reinterpret_cast<uint2*>(vt + o + (size_t)half * e.Tpad) = hi4;
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              if (row0 + r >= a.M) continue;
              const size_t o = ((size_t)(seq[at][r] * e.H + head) * e.Dh + dim) * e.Tpad + pos[at][r];
              vt[o] = f2bf(acc[i][2 * p][r]);
              vt[o + (size_t)half * e.Tpad] = f2bf(acc[i][2 * p + 1][r]);
            }
          }
        } else {
          unsigned short* dst = reinterpret_cast<unsigned short*>(mat == 0 ? e.q : e.kstore);
          unsigned w[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float x1 = acc[i][2 * p][r], x2 = acc[i][2 * p + 1][r];
            const float c = cs[at][p][r].x, sn = cs[at][p][r].y;
            // explicit roundings: every tile configuration must produce the same bits, whatever
            // contraction into fused multiply-adds the compiler would pick for each of them
            w[r] = pack_bf16(__fmaf_rn(x1, c, -__fmul_rn(x2, sn)), __fmaf_rn(x2, c, __fmul_rn(x1, sn)));
          }
          quad_transpose(w, lane);   // "one column, four rows" per lane into "four columns, one row"
          const int row = row0 + lr;
          if (row >= a.M) continue;
          const int c4 = gi * 16 + (cl & ~3);
          const size_t o = mat == 0 ? (size_t)row * e.d + head * e.Dh + c4
                                    : ((size_t)seq_st * e.Tpad + pos_st) * e.d + head * e.Dh + c4;
          uint2 lo, hi;   // feature c4..c4+3 and its partner c4+half..c4+half+3
          lo.x = (w[0] & 0xffffu) | (w[1] << 16);
          lo.y = (w[2] & 0xffffu) | (w[3] << 16);
          hi.x = (w[0] >> 16) | (w[1] & 0xffff0000u);
          hi.y = (w[2] >> 16) | (w[3] & 0xffff0000u);
          *reinterpret_cast<uint2*>(dst + o) = lo;
          *reinterpret_cast<uint2*>(dst + o + half) = hi;
        }
      }
    }
  } else {  // EPI_LMHEAD
    const LmHeadEpilogue& e = a.lm;
    constexpr int WPP = 128 / (BN / WN);                   // wavefronts that share a 128-column part
    static_assert(WPP >= 1 && WN % WPP == 0, "a wavefront's columns lie in one part");
    float* s_m = reinterpret_cast<float*>(smem);           // [WN][BM]
    float* s_s = s_m + WN * BM;
    int* s_i = reinterpret_cast<int*>(s_s + WN * BM);
    __syncthreads();
    const bool biased = e.bias.value != 0.f && a.gate.ctl;
    const int col0 = tile_n * BN + wn * (BN / WN);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = row_base + i * 16 + r;
        float vals[FN];
        float m = -INFINITY;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const int col = col0 + j * 16 + cl;
          float v = acc[i][j][r];
          if (biased && col == e.bias.token_id && row < a.M &&
              a.gate.ctl[CTL_SEQ_GB + row / e.bias.block_len] * e.bias.block_len + (row % e.bias.block_len) >=
                  e.bias.gen_pos_from)
            v += e.bias.value;
          if (e.logits && row < a.M && col < a.N) e.logits[(size_t)row * a.N + col] = v;
          if (col == e.mask_id || col >= a.N) v = -INFINITY;
          vals[j] = v;
          m = fmaxf(m, v);
        }
        // the row's maximum over the 16 lanes, then the lowest column that has it and the sum relative to it
        m = fmaxf(m, dppf<kDppRor + 8>(m));
        m = fmaxf(m, dppf<kDppRor + 4>(m));
        m = fmaxf(m, dppf<kDppRor + 2>(m));
        m = fmaxf(m, dppf<kDppRor + 1>(m));
        int mi = 0x7fffffff;
        float sum = 0.f;
#pragma unroll
        for (int j = FN - 1; j >= 0; --j) mi = vals[j] == m && m > -INFINITY ? col0 + j * 16 + cl : mi;
        mi = min(mi, (int)dpp<kDppRor + 8>((unsigned)mi));
        mi = min(mi, (int)dpp<kDppRor + 4>((unsigned)mi));
        mi = min(mi, (int)dpp<kDppRor + 2>((unsigned)mi));
        mi = min(mi, (int)dpp<kDppRor + 1>((unsigned)mi));
#pragma unroll
        for (int j = 0; j < FN; ++j) sum += (m == -INFINITY) ? 0.f : __expf(vals[j] - m);
        sum += dppf<kDppRor + 8>(sum);
        sum += dppf<kDppRor + 4>(sum);
        sum += dppf<kDppRor + 2>(sum);
        sum += dppf<kDppRor + 1>(sum);
        if (cl == 0) {
          const int lrow = row - tile_m * BM;
          s_m[wn * BM + lrow] = m;
          s_s[wn * BM + lrow] = sum;
          s_i[wn * BM + lrow] = mi;
        }
      }
    }
    __syncthreads();
    if (e.part_max) {
      for (int t = tid; t < BM * (BN / 128); t += WM * WN * 64) {
        const int lrow = t % BM, sub = t / BM, row = tile_m * BM + lrow, part = tile_n * (BN / 128) + sub;
        if (row >= a.M || part >= e.n_part) continue;
        const int w0 = sub * WPP;
        float m = s_m[w0 * BM + lrow], sum = s_s[w0 * BM + lrow];
        int mi = s_i[w0 * BM + lrow];
#pragma unroll
        for (int w = w0 + 1; w < w0 + WPP; ++w) {
          const float m2 = s_m[w * BM + lrow], s2 = s_s[w * BM + lrow];
          const int i2 = s_i[w * BM + lrow];
          const float M = fmaxf(m, m2);
          const float f1 = (m == -INFINITY) ? 0.f : __expf(m - M), f2 = (m2 == -INFINITY) ? 0.f : __expf(m2 - M);
          sum = sum * f1 + s2 * f2;
          if (m2 > m || (m2 == m && i2 < mi)) mi = i2;
          m = M;
        }
        const size_t o = (size_t)row * e.n_part + part;
        e.part_max[o] = m;
        e.part_sum[o] = sum;
        e.part_idx[o] = mi;
      }
    }
  }
}

template <int BM, int BN, int WM, int WN, int DEPTH, int EPI, bool COLD>
__global__ void __launch_bounds__(512) k_gemm_turns(GemmArgs a) {
  constexpr int BK = 64;
  constexpr int FM = BM / WM / 16, FN = BN / WN / 16;
  constexpr int HALF = FM / 2;                 // row fragments of a phase
  constexpr int RA = DEPTH + 1, RB = DEPTH;    // tiles in the rings
  constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
  constexpr int LA = BM / 64, LB = BN / 64;    // direct-to-LDS loads per wavefront and stage
  static_assert(WM * WN == 8 && BM % 64 == 0 && BN % 64 == 0 && FM % 2 == 0, "eight wavefronts, rows in pairs of fragments");
  static_assert(DEPTH >= 2 && (DEPTH - 1) * (LA + LB) < 64, "ring depth");
  static_assert(RA * A_BYTES + RB * B_BYTES <= 163840, "LDS");
  static_assert(EPI != EPI_LMHEAD || 3 * WN * BM * 4 <= RA * A_BYTES, "reduction scratch");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // [RA][A tile] [RB][B tile]
  unsigned char* const smemB = smem + RA * A_BYTES;

  // Up to the first load nothing is divided by hardware and little is waited for: at 221 rows of 1024 the 300 instructions of
  // integer divisions here were 0.5 us of each product's 8-14.
  int z, tile_m, tile_n;
  if (!a.map.place(blockIdx.x, &z, &tile_m, &tile_n)) return;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int k_begin = z * a.k_len, nk = a.k_len / BK;

  // Load i of a tile (this wavefront's pieces are i * 8 + wave, 8 rows each): lane l fills slot l of the 1 KB piece.
  const bf16* srcA[LA];
  const bf16* srcB[LB];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int r = (i * 8 + wave) * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
    srcA[i] = a.A + (size_t)min(tile_m * BM + r, a.M - 1) * a.K + k_begin + c * 8;
  }
#pragma unroll
  for (int i = 0; i < LB; ++i) {
    const int r = (i * 8 + wave) * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
    srcB[i] = weight_row<BN, EPI>(a, tile_n, r) + k_begin + c * 8;
  }
  const unsigned lds0 = __builtin_amdgcn_readfirstlane(
      (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)(smem + wave * 1024));
  auto load_a = [&](int k, int slot) {
#pragma unroll
    for (int i = 0; i < LA; ++i) dma16(srcA[i] + k * BK, lds0 + slot * A_BYTES + i * 8192);
  };
  auto load_b = [&](int k, int slot) {
#pragma unroll
    for (int i = 0; i < LB; ++i) dma16_weights<COLD>(srcB[i] + k * BK, lds0 + RA * A_BYTES + slot * B_BYTES + i * 8192);
  };

  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // fragment reads: lane (row lane % 16, chunk lane / 16 of the 32-deep K step kk)
  const int fr = lane & 15;
  int sw[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) sw[kk] = ((kk * 4 + (lane >> 4)) ^ ((fr >> 1) & 7)) << 4;
  const int rowA = (wm * (BM / WM) + fr) * 128, rowB = (wn * (BN / WN) + fr) * 128;
  bf16x8_t fa[HALF][2], fb[FN][2];
  auto read_a = [&](int slot, int half) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < HALF; ++i)
        fa[i][kk] = *reinterpret_cast<const bf16x8_t*>(smem + slot * A_BYTES + rowA + (half * HALF + i) * 2048 + sw[kk]);
  };
  auto read_b = [&](int slot) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        fb[j][kk] = *reinterpret_cast<const bf16x8_t*>(smemB + slot * B_BYTES + rowB + j * 2048 + sw[kk]);
  };
  // End of a read slot: this wavefront's fragment reads are complete, so what they read may be refilled
  // after the barrier.  Nothing may move across the counted waits and the barriers.
  auto reads_done = [&]() {
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  auto mfmas = [&](auto halfc) {
    constexpr int H = decltype(halfc)::value;
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < HALF; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[H * HALF + i][j] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i][kk], fb[j][kk], acc[H * HALF + i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };

  const int2 gate = gate_words(a.gate);    // looked at when the first loads are on their way
  const int lead = min(DEPTH, nk);
  for (int k = 0; k < lead; ++k) {
    load_a(k, k);
    load_b(k, k);
  }
  if (gate_closed(a.gate, gate)) {
    wait_vmcnt<0>();                       // LDS stays this workgroup's until its loads have landed
    return;
  }
  if (nk >= DEPTH) wait_vmcnt<(DEPTH - 1) * (LA + LB)>();   // stage 0 has landed
  else wait_vmcnt<0>();
  lds_barrier();
  if (wave >= 4) lds_barrier();   // the second group starts one slot later
  __builtin_amdgcn_sched_barrier(0);

  constexpr bool SERIAL = EPI == EPI_PARTIAL_SER;
  f32x4 tot[SERIAL ? FM : 1][SERIAL ? FN : 1];             // sum of the finished K ranges
  const int seg = SERIAL ? a.serial_stages : 0;            // stages per K range
  int seg_left = seg;
  if constexpr (SERIAL) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) tot[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  int sa = 0, sb = 0;             // ring places of A(k) and B(k)
  for (int k = 0; k < nk; ++k) {
    const bool more = k + DEPTH < nk;
    read_b(sb);
    read_a(sa, 0);
    if (more) load_a(k + DEPTH, sa == 0 ? RA - 1 : sa - 1);     // A(k-1)'s place
    reads_done();
    mfmas(std::integral_constant<int, 0>{});
    read_a(sa, 1);
    if (more) {
      load_b(k + DEPTH, sb);                                    // B(k)'s place
      wait_vmcnt<(DEPTH - 1) * (LA + LB)>();   // stage k+1 has landed: only the younger stages are outstanding
    } else {
      wait_vmcnt<0>();
    }
    reads_done();
    mfmas(std::integral_constant<int, 1>{});
    sa = sa + 1 == RA ? 0 : sa + 1;
    sb = sb + 1 == RB ? 0 : sb + 1;
    if constexpr (SERIAL) {
      if (--seg_left == 0) {      // a K range ends here: bank it and start the next from zero
        seg_left = seg;
        const bool first = k + 1 == seg;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            tot[i][j] = first ? acc[i][j] : tot[i][j] + acc[i][j];
            acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
      }
    }
  }
  if (wave < 4) lds_barrier();    // both groups have passed the same number of barriers
  if constexpr (SERIAL) epilogue<BM, BN, WM, WN, EPI>(a, tot, smem, wm, wn, tile_m, tile_n, z);
  else epilogue<BM, BN, WM, WN, EPI>(a, acc, smem, wm, wn, tile_m, tile_n, z);
}

// Whether a launch loads cold weights with the hint (dma16_once).  A panel's weights are read by each of its row tiles, and the hint
// lets go of them early: it is for one row tile, or for row tiles that read a panel together.  They do on one XCD (its count of
// tiles a multiple of them), if they are not two small ones to a CU (tiles of 128x128 on), and tiles of 128 rows if they are equally
// long too (the last three quarters full; those of 256 rows go at the pace of their multiplications).  Otherwise the later one
// goes to memory again.  us, loads as they are / with the hint, Q/K/V unless said:
//   together  4096 wide, 256 rows 48.0 / 47.2, 512 rows 59.1 / 58.6, gate/up 67.0 / 66.2, 304 rows 63.1 / 62.3; 8192, 256 rows 124 / 113
//   unequal   4096, 129 rows 41.5 / 47.8, gate/up 50.5 / 58.9, down 30.7 / 35.8; 5120, 129 rows 51.2 / 68.2, 257 rows 63.8 / 78.2
//   an XCD's tiles no multiple of them   3584, 224 rows (168 tiles) 41.0 / 44.1, 384 rows (252) 43.2 / 45.2; 1536, 480 rows (144)
//             22.9 / 23.9; 5120, 257 rows, gate/up (216 tiles of 256x256) 77.5 / 84.9
//   small     3584, 192 rows (64x64) 38.8 / 42.4; 2048, 368 rows, output (128x64) 13.2 / 13.8
// Beyond 512 rows equal within 1 %.  Calls, without the hint or any later change / with it up to 512 rows / as here: one sequence of 129 rows,
// three layers of 4096 x 12288 492 / 510 / 464, two of 5120 x 13824 482 / 512 / 457; 288 rows, six of 2048 x 5632 592 / 614 / 566.
bool read_once(int M, int N, int splits, int bm, int bn) {
  const int tiles_m = (M + bm - 1) / bm, last = M - (tiles_m - 1) * bm;
  if (M > 512) return false;
  if (tiles_m == 1) return true;
  const TileMap map(tiles_m, (N + bn - 1) / bn, splits);
  return bm >= 128 && bn >= 128 && (bm == 256 || 4 * last >= 3 * bm) && map.per_xcd % tiles_m == 0;
}
template <int BM, int BN, int WM, int WN, int DEPTH, int EPI, bool COLD = false>
static void launch(GemmArgs& a, hipStream_t s) {
  if constexpr (!COLD && EPI != EPI_PARTIAL_SER)
    if (a.gate.cold && read_once(a.M, a.N, a.splits, BM, BN)) return launch<BM, BN, WM, WN, DEPTH, EPI, true>(a, s);
  auto kern = k_gemm_turns<BM, BN, WM, WN, DEPTH, EPI, COLD>;
  constexpr int smem = ((DEPTH + 1) * BM + DEPTH * BN) * 128;
  static DynLdsAttr attr;
  attr.ensure(reinterpret_cast<const void*>(kern), smem);
  a.map = TileMap((a.M + BM - 1) / BM, (a.N + BN - 1) / BN, a.splits);
  a.k_len = a.K / a.splits;
  if (a.serial) a.serial_stages = a.k_len / 64 / a.serial;
  hipLaunchKernelGGL(kern, dim3((a.map.total + 7) / 8 * 8), dim3(512), smem, s, a);
}
// ------------------------------------------------------------------------------------------------
// Small tiles.  A wavefront's share of a 64-deep stage is a handful of MFMAs there, and with turns every slot lasts as long as
// a round trip to LDS: 0.33 us a stage of a 128x64 tile, whatever is loaded.  Here all wavefronts go in step, one barrier a
// stage: behind it a wavefront reads the whole next stage's fragments into a second set of registers and multiplies the ones it
// has, so a stage lasts as long as the LDS traffic (64x64: 48 KB) or the multiplications, whichever is longer.
//   64x64 tiles (80 KB of LDS, two workgroups a CU) are for outputs that 128x64 tiles would give to half of the chip, in eight
// wavefronts of 16x32: with four of 32x32 a SIMD's one wavefront waits out every round trip to LDS.  64x32 tiles, four
// wavefronts of 16x32, while they are a workgroup for each CU at most.  us, 64x64 in four / in eight / 64x32: 221 rows of 1024 (FFN
// 2816), Q/K/V 8.6 / 7.3 / 7.7 (384 tiles), output 5.1 / 4.9 / 4.3, down 6.1 / 6.0 / 6.3 (512 tiles); 100 rows, Q/K/V 8.5 / 7.2 / 6.7,
// output 4.9 / 4.8 / 4.3, down 5.9 / 5.7 / 4.9; more than 256 tiles, in four / in eight: 300 rows of 3072, output (480) 14.6 / 14.7,
// 400 of 2304, output (504) 14.3 / 14.4, down of 6144 27.1 / 26.5.
//   128x128 tiles: Q/K/V of 192 rows of 4096 47-49 / 44, 256 rows 49 / 47, down equal; gate/up 2 % slower, which keeps turns there.
// Every output sums in the order of the kernel above: the same bits.
template <int BM, int BN, int WM, int WN, int NS, int EPI, bool COLD>
__global__ void __launch_bounds__(WM * WN * 64) k_gemm_step(GemmArgs a) {
  constexpr int BK = 64, NW = WM * WN;     // a stage: [A tile | B tile], NS of them in the ring
  constexpr int FM = BM / WM / 16, FN = BN / WN / 16;
  constexpr int A_BYTES = BM * BK * 2, STAGE = (BM + BN) * BK * 2;
  constexpr int LA = BM / 8 / NW, LB = BN / 8 / NW;
  static_assert(LA * 8 * NW == BM && LB * 8 * NW == BN, "tile/wavefronts mismatch");
  static_assert(NS >= 3 && (NS - 1) * (LA + LB) < 64 && NS * STAGE <= 163840, "ring");
  static_assert(EPI != EPI_LMHEAD || 3 * WN * BM * 4 <= STAGE, "reduction scratch");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  int z, tile_m, tile_n;
  if (!a.map.place(blockIdx.x, &z, &tile_m, &tile_n)) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int k_begin = z * a.k_len, nk = a.k_len / BK;
  const bf16* srcA[LA];
  const bf16* srcB[LB];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int r = (i * NW + wave) * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
    srcA[i] = a.A + (size_t)min(tile_m * BM + r, a.M - 1) * a.K + k_begin + c * 8;
  }
#pragma unroll
  for (int i = 0; i < LB; ++i) {
    const int r = (i * NW + wave) * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
    srcB[i] = weight_row<BN, EPI>(a, tile_n, r) + k_begin + c * 8;
  }
  const unsigned lds0 = __builtin_amdgcn_readfirstlane(
      (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)(smem + wave * 1024));
  auto load = [&](int k, int slot) {
#pragma unroll
    for (int i = 0; i < LA; ++i) dma16(srcA[i] + k * BK, lds0 + slot * STAGE + i * NW * 1024);
#pragma unroll
    for (int i = 0; i < LB; ++i) dma16_weights<COLD>(srcB[i] + k * BK, lds0 + slot * STAGE + A_BYTES + i * NW * 1024);
  };
  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int fr = lane & 15;
  int sw[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) sw[kk] = ((kk * 4 + (lane >> 4)) ^ ((fr >> 1) & 7)) << 4;
  const int rowA = (wm * (BM / WM) + fr) * 128, rowB = A_BYTES + (wn * (BN / WN) + fr) * 128;
  struct Frags { bf16x8_t a[FM][2], b[FN][2]; };
  auto read = [&](Frags& f, int slot) {
    const unsigned char* base = smem + slot * STAGE;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int i = 0; i < FM; ++i) f.a[i][kk] = *reinterpret_cast<const bf16x8_t*>(base + rowA + i * 2048 + sw[kk]);
#pragma unroll
      for (int j = 0; j < FN; ++j) f.b[j][kk] = *reinterpret_cast<const bf16x8_t*>(base + rowB + j * 2048 + sw[kk]);
    }
  };
  auto mfmas = [&](Frags& f) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[i][kk], f.b[j][kk], acc[i][j], 0, 0, 0);
  };
  const int2 gate = gate_words(a.gate);    // looked at when the first loads are on their way
  const int lead = min(NS, nk);
  for (int k = 0; k < lead; ++k) load(k, k);
  if (gate_closed(a.gate, gate)) {
    wait_vmcnt<0>();                       // LDS stays this workgroup's until its loads have landed
    return;
  }
  __builtin_amdgcn_sched_barrier(0);
  if (nk >= NS) wait_vmcnt<(NS - 1) * (LA + LB)>();
  else wait_vmcnt<0>();
  lds_barrier();
  Frags f0, f1;
  read(f0, 0);
  int slot = 0;                     // of the stage at work
  // One stage: its fragments are on their way or here; wait for them and for the next stage, then send off what fills
  // this stage's place, read the next stage's fragments and multiply.
  auto stage = [&](int k, Frags& cur, Frags& nxt) {
    __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0): this stage's fragments are in registers
    // the next stage has landed: at most the loads of the NS - 2 younger stages are outstanding
    if (k + NS - 1 < nk) wait_vmcnt<(NS - 2) * (LA + LB)>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
    const int next = slot + 1 == NS ? 0 : slot + 1;
    read(nxt, next);                         // (behind the last stage: what lies there, for nobody)
    if (k + NS < nk) load(k + NS, slot);
    mfmas(cur);
    __builtin_amdgcn_sched_barrier(0);
    slot = next;
  };
  for (int k = 0; k < nk; k += 2) {
    stage(k, f0, f1);
    if (k + 1 < nk) stage(k + 1, f1, f0);
  }
  lds_barrier();
  epilogue<BM, BN, WM, WN, EPI>(a, acc, smem, wm, wn, tile_m, tile_n, z);
}
template <int BM, int BN, int WM, int WN, int NS, int EPI, bool COLD = false>
static void launch_step(GemmArgs& a, hipStream_t s) {
  if constexpr (!COLD)
    if (a.gate.cold && read_once(a.M, a.N, a.splits, BM, BN)) return launch_step<BM, BN, WM, WN, NS, EPI, true>(a, s);
  auto kern = k_gemm_step<BM, BN, WM, WN, NS, EPI, COLD>;
  constexpr int smem = NS * (BM + BN) * 128;
  static DynLdsAttr attr;
  attr.ensure(reinterpret_cast<const void*>(kern), smem);
  a.map = TileMap((a.M + BM - 1) / BM, (a.N + BN - 1) / BN, a.splits);
  a.k_len = a.K / a.splits;
  hipLaunchKernelGGL(kern, dim3((a.map.total + 7) / 8 * 8), dim3(WM * WN * 64), smem, s, a);
}
// Tile choice: rounds over the 256 CUs, each of a fixed part (first stages from HBM, epilogue) plus the K loop.
// Loop times per 4096 of K with every CU busy and weights coming from HBM, as measured (4096 rows, d_ffn 12288:
// 256x256 565 us over 6 rounds, 256x192 614 over 8, 256x128 698 over 12; 512 rows: 128x192 107 over 2, 128x128 83 over
// 2 of 12288 columns).  A larger tile moves fewer bytes per flop, so it wins whenever there are enough of them:
// 256x256 for thousands of rows; 512 rows x 24576 gate/up columns are exactly 256 tiles of 256x192, x 12288 Q/K/V
// columns 256 of 128x192; 128x64 and 64x64 are for outputs too small to occupy the chip otherwise.
// 128x128 and 128x64 tiles run in k_gemm_step, gate/up's 128x128 in k_gemm_turns; one figure stands for both, which differ
// by less than the tiles do (us a round at 1024 rows and 4096 of K, in step / in turns: 128x128 Q/K/V 43.4 / 45.7, gate/up
// 40.6 / 43.1, estimate 43; 128x64 29.4 / 30.8 and 28.6 / 29.3, estimate 30; at 256 rows equal within 1 %).  64x64: two share a CU, so
// a launch of 257 to 512 of them is a round too, and takes what one of 128x64 tiles does (kPairUs; Q/K/V of 256 rows of 2048 15.3 / 15.3 us,
// gate/up 22 / 20).  That fills row counts that 128-row tiles leave half empty: Q/K/V of 400 rows of 1536 13.5 us against
// 17.6 with 128x128, of 300 rows of 2048 16.2 / 21.2, gate/up of 300 rows of 1024 9.0 / 12.0.
struct Tile { int bm, bn; double us; };
constexpr Tile kTiles[7] = {{256, 256, 88.}, {256, 192, 71.}, {256, 128, 53.}, {128, 192, 48.}, {128, 128, 37.}, {128, 64, 24.}, {64, 64, 15.}};
constexpr double kRoundUs = 6., kPairUs = 24.5;
static double tile_cost(int t, int M, int N, int K, int splits) {
  const long long tiles = (long long)((M + kTiles[t].bm - 1) / kTiles[t].bm) * ((N + kTiles[t].bn - 1) / kTiles[t].bn) * splits;
  if (t == 6) {
    const double k = K / splits / 4096., pair = kRoundUs + kPairUs * k, one = kRoundUs + kTiles[6].us * k;
    return (double)(tiles / 512) * pair + (tiles % 512 == 0 ? 0. : (tiles % 512 <= 256 ? one : pair));
  }
  return (double)((tiles + 255) / 256) * (kRoundUs + kTiles[t].us * K / splits / 4096.);
}
static bool one_each(int M, int N, int splits = 1) {   // 64x32 tiles: one for each CU at most
  return (long long)((M + 63) / 64) * ((N + 31) / 32) * splits <= 256;
}
static int pick_tile(int M, int N, int K) {
  int best = 6;
  for (int t = 5; t >= 0; --t)
    if ((M > 128 || kTiles[t].bm <= 128) && tile_cost(t, M, N, K, 1) < tile_cost(best, M, N, K, 1)) best = t;
  return best;
}

// Up to 64 rows: bound by the weights' one way from memory, and where they are few by the chain of stages.  One row tile, no K
// ranges, the epilogues above: no partial sums to write and to read, no launch behind.  32 columns to a workgroup while that is one
// for each CU at most, more beyond; rings of four to six stages (deeper ones do nothing).  us, weights from memory once, this / K
// ranges and a finishing kernel (Q/K/V, gate/up of 1024) or tiles of 32x32x16 fragments (gate/up, LM head):
//   Q/K/V of      1024         2048         4096         5120          LM head  1024 x 32000  4096 x 32000  4096 x 126464
//     32 rows     6.6 / 8.2    9.7 / 13.1   21.7 / 24.0  29.6 / 36.0             14.1 / 23.0   54.4 / 65.0   153 / 163
//     64 rows     7.4 / 9.0    11.2 / 19.9  25.9 / 32.9  34.2 / 44.2             15.6 / 24.5   57.7 / 67.0   157 / 203
//   gate/up       1024 x 2816  2048 x 8192  4096 x 11008 4096 x 12288  4096 x 14336
//     32 rows     6.1 / 10.4   15.2 / 17.0  37.7 / 38.0  37.0 / 38.3   49.7 / 44.5     (64 columns in the second, else 32)
//     64 rows     7.7 / 11.3   16.2 / 20.9  38.0 / 41.5  40.0 / 43.0   60.8 / 47.9     (64 in the second, then 96)
// Both sides of the lines, us with a pair of events around the launch, weights from memory; 32 rows, then 64:
//   256 workgroups of 32 columns: Q/K/V of 2560 (7,680 columns), 32 columns / 64 14.7 / 18.2, 18.4 / 21.8; of 2816 (8,448) 20.6 / 18.9,
//   26.9 / 22.5; of 4096 27.8 / 25.0, 35.6 / 30.4; gate/up of 1536 x 4160 (8,320) 13.6 / 12.8, 17.3 / 14.6, of 3584 x 8192 26.0 / 23.1, 35.0 / 26.7
//   256 of 64: gate/up of 3584 x 9472 (18,944), 32 columns up to 32 rows and 96 beyond / 64 33.7 / 36.2, 32.2 / 42.9
// Where 32 columns make more than three workgroups for each CU (what their rings leave room for), or 96 more than one, gate/up
// stays with gemm_few_rows.hip; no one tile is ahead there (that kernel / tiles of 64 columns: 4096 x 14336 50.3 / 45.5, 54.4 / 65.7,
// 5120 x 13824 57.6 / 57.7 (52.4 with 128), 59.4 / 82.6, 3584 x 18944 65.2 / 53.1, 69.0 / 57.8, 8192 x 22016 164 / 132, 172 / 142).
template <int EPI, int COLS, int COLS2, int WM2, int WN2>
static void launch_few(GemmArgs& a, hipStream_t s) {
  const bool narrow = a.N <= 256 * COLS;
  if (a.M <= 32) {
    if (narrow) launch_step<32, COLS, 2, 1, 6, EPI>(a, s);
    else launch_step<32, COLS2, 2, 2, 6, EPI>(a, s);
  } else {
    if (narrow) launch_step<64, COLS, WM2, WN2, 6, EPI>(a, s);
    else launch_step<64, COLS2, 2, 2, 5, EPI>(a, s);
  }
}

void launch_gemm_qkv_bf16(const bf16* A, const bf16* wq, const bf16* wk, const bf16* wv, int M, int K,
                          const QkvEpilogue& e, Gate g, hipStream_t s) {
  GemmArgs a = {};
  a.A = A; a.B0 = wq; a.B1 = wk; a.B2 = wv;
  a.M = M; a.N = 3 * e.d; a.K = K; a.splits = 1; a.gate = g; a.qkv = e;
  a.heads = Div(e.H); a.rows_per_seq = Div(e.Tq); a.group_shift = e.Dh == 128 ? 2 : 1;   // head sizes are 64 and 128
  if (M <= kSkinnyRows) return launch_few<EPI_QKV, 32, 64, 4, 1>(a, s);
  switch (pick_tile(M, a.N, K)) {
    case 0: launch<256, 256, 2, 4, 2, EPI_QKV>(a, s); break;
    case 1: launch<256, 192, 4, 2, 2, EPI_QKV>(a, s); break;
    case 2: launch<256, 128, 4, 2, 2, EPI_QKV>(a, s); break;
    case 3: launch<128, 192, 4, 2, 3, EPI_QKV>(a, s); break;
    case 4: launch_step<128, 128, 4, 2, 5, EPI_QKV>(a, s); break;
    case 5: launch_step<128, 64, 4, 2, 6, EPI_QKV>(a, s); break;
    default:
      if (one_each(M, a.N)) launch_step<64, 32, 4, 1, 6, EPI_QKV>(a, s);
      else launch_step<64, 64, 4, 2, 5, EPI_QKV>(a, s);
  }
}

void launch_gemm_swiglu_bf16(const bf16* A, const bf16* wg, const bf16* wu, bf16* act, int M, int F, int K, Gate g,
                             hipStream_t s) {
  GemmArgs a = {};
  a.A = A; a.B0 = wg; a.B1 = wu; a.M = M; a.N = 2 * F; a.K = K; a.splits = 1; a.gate = g;
  a.act = act; a.F = F;
  if (M <= kSkinnyRows) {
    if (M > 32 && a.N > 256 * 64) return launch_step<64, 96, 4, 1, 4, EPI_SWIGLU>(a, s);
    if (a.N > 256 * 64) return launch_step<32, 32, 2, 1, 6, EPI_SWIGLU>(a, s);
    return launch_few<EPI_SWIGLU, 32, 64, 2, 1>(a, s);
  }
  switch (pick_tile(M, a.N, K)) {
    case 0: launch<256, 256, 2, 4, 2, EPI_SWIGLU>(a, s); break;
    case 1: launch<256, 192, 4, 2, 2, EPI_SWIGLU>(a, s); break;
    case 2: launch<256, 128, 4, 2, 2, EPI_SWIGLU>(a, s); break;
    case 3: launch<128, 192, 4, 2, 3, EPI_SWIGLU>(a, s); break;
    case 4: launch<128, 128, 4, 2, 3, EPI_SWIGLU>(a, s); break;
    case 5: launch_step<128, 64, 4, 2, 6, EPI_SWIGLU>(a, s); break;
    default:
      if (one_each(M, a.N)) launch_step<64, 32, 4, 1, 6, EPI_SWIGLU>(a, s);
      else launch_step<64, 64, 4, 2, 5, EPI_SWIGLU>(a, s);
  }
}

// [d, d] and [d, F] projections: tiles of these narrow outputs do not fill the chip at a few hundred rows, so K is
// split into ranges whose partial sums the next RMSNorm folds in ascending order.  Above 256 rows the number of
// ranges is a function of K alone, never of the row count: a sequence must sum its projections in the same order
// whatever batch it is decoded in (full-recompute forwards of one sequence and of a batch then give the same bits
// row by row).  Whether a workgroup per range writes its partial, or one workgroup walks the ranges and writes
// their sum (EPI_PARTIAL_SER), gives the same bits, so that and the tile may depend on the row count: at 512 rows of
// the 8B shape four workgroups per tile occupy the chip (down projection 50 us; 83 with unsplit 128x64 tiles), at 2048
// and more there is a tile per CU, and three more partials to write and to fold only cost (171 us and the RMSNorm
// 28, against 141 and 60 estimated for 256x256 tiles and four partials).  128x128 tiles walk the ranges where they fill the chip and
// 256x128 do not.
//   Four ranges from K = 8192 on, two below: two partials less to write and to fold. us, output projection of 4096 with two
// / four ranges: 512 rows 30.1 / 26.5, the RMSNorm behind it 6.5 / 10; 768 rows 45 / 43 and 8 / 14; 1024 rows 49 / 52, 1280
// rows 58 / 70. Steps: 3072 rows of 1024 (down K = 2816 too) 1233 -> 1192, 1280 rows of 4096 2050 -> 2022; 512 rows, where the
// projection loses what the norm gains, 2073 -> 2080 (within the spread of two runs).
// Up to 256 rows (batched block-only steps of the cached modes) the split may go up to eight ways, as the estimate
// says: 256 rows of the 8B shape split 4 ways, 128 rows 8 ways.
// Rows that are some of a pass's (the wanted ones behind the last layer's attention) take the number of ranges of
// the pass and choose the tile for themselves.
constexpr double kFoldUs = 0.8;   // a partial of up to 256 rows costs the RMSNorm this much
struct PartialPlan { int tile, splits, serial; };
// The ranges that the sums are formed in follow an estimate of their own: tiles may change, they stay.
static double range_cost(int t, int M, int N, int K, int splits) {
  const long long tiles = (long long)((M + kTiles[t].bm - 1) / kTiles[t].bm) * ((N + kTiles[t].bn - 1) / kTiles[t].bn) * splits;
  return (double)((tiles + 255) / 256) * (kRoundUs + (t == 6 ? 18. : kTiles[t].us) * K / splits / 4096.);
}
static PartialPlan plan_small_pass(int M, int N, int K) {
  PartialPlan best = {6, 1, 0};
  for (int t : {6, 5, 4})
    for (int S = 1; S <= 8 && K % (S * 64) == 0 && (S == 1 || K / S >= 512); S *= 2)
      if (range_cost(t, M, N, K, S) + S * kFoldUs < range_cost(best.tile, M, N, K, best.splits) + best.splits * kFoldUs)
        best = {t, S, 0};
  return best;
}
int k_ranges(int pass_rows, int N, int K) {
  if (pass_rows <= 256) return plan_small_pass(pass_rows, N, K).splits;
  if (K % 256 == 0 && K / 4 >= 2048) return 4;
  return K % 128 == 0 && K / 2 >= 512 ? 2 : 1;
}
static PartialPlan plan_partial(const int rows, int N, int K, int pass_rows) {
  const int R = k_ranges(pass_rows, N, K);
  int M = rows;
  if (pass_rows <= 256) {
    int best = 6;
    for (int t : {5, 4})
      if (tile_cost(t, M, N, K, R) < tile_cost(best, M, N, K, R)) best = t;
    return {best, R, 0};
  }
  M = (M + 127) / 128 * 128;   // a function of the count of 128-row tiles: the workspace is sized from it
  const double fold_us = (double)M * N * 8 / 5e6;    // a partial is written and read once, at about 5 TB/s
  PartialPlan best = {2, 1, R};
  double cost = tile_cost(2, M, N, K, 1) * 1.03 + fold_us;
  if (const double c = tile_cost(4, M, N, K, 1) * 1.03 + fold_us; c < cost) { cost = c; best = {4, 1, R}; }
  for (int t : {0, 1, 2, 4, 5, 6}) {
    if (M <= 128 && kTiles[t].bm > 128) continue;
    const double c = range_cost(t, M, N, K, R) + R * fold_us;
    if (c < cost) { cost = c; best = {t, R, 0}; }
  }
  if (best.serial == 1) best.serial = 0;
  if (!best.serial && best.splits == R)      // a workgroup for each range: the tile for the rows as they are
    for (int t : {0, 1, 2, 4, 5, 6})
      if ((M > 128 || kTiles[t].bm <= 128) && tile_cost(t, rows, N, K, R) < tile_cost(best.tile, rows, N, K, R)) best.tile = t;
  return best;
}
int wide_splits(int M, int N, int K, int pass_rows) { return plan_partial(M, N, K, pass_rows).splits; }

// Partials of any pass of up to `rows` rows of a [d, F] model.  Up to 64 rows: the ranges of the projections to d, and of gate/up
// where few_rows_gate_up splits it; the same for any count of rows.
// More rows: the projections to d, whose ranges depend on the rows through counts of tiles, of the smallest tile's 64 rows in
// passes of up to 256 (plan_small_pass; fewer rows may have more ranges), of 128 rows above (plan_partial): the last row
// count of every such step stands for all of it.  Rows that are some of a larger pass's take that pass's ranges.
size_t partial_floats(long long rows, int d, int F) {
  const size_t few = (size_t)std::min<long long>(rows, kSkinnyRows);
  size_t most = few * d * std::max(skinny_splits(d, d), skinny_splits(d, F));
  if (few_rows_gate_up(F, d, true) == GATE_UP_RANGES) most = std::max(most, few * 2 * F * skinny_splits(2 * F, d));
  if (rows <= kSkinnyRows) return most;
  for (long long top = 128;; top += top < 256 ? 64 : 128) {
    const int M = (int)std::min(top, rows);
    for (int k : {d, F})
      for (int pass : {M, std::max(M, 257)}) most = std::max(most, (size_t)wide_splits(M, d, k, pass) * M * d);
    if (top >= rows) break;
  }
  return most;
}

void launch_gemm_partial_bf16(const bf16* A, const bf16* W, float* parts, size_t part_stride, int M, int N, int K,
                              int pass_rows, bool add, Gate g, hipStream_t s) {
  const PartialPlan p = plan_partial(M, N, K, pass_rows);
  GemmArgs a = {};
  a.A = A; a.B0 = W; a.M = M; a.N = N; a.K = K; a.splits = p.splits; a.gate = g;
  a.parts = parts; a.part_stride = part_stride; a.serial = p.serial; a.add = add;
  if (p.serial && p.tile == 4) launch<128, 128, 4, 2, 3, EPI_PARTIAL_SER>(a, s);
  else if (p.serial) launch<256, 128, 4, 2, 2, EPI_PARTIAL_SER>(a, s);
  else if (p.tile == 0) launch<256, 256, 2, 4, 2, EPI_PARTIAL>(a, s);
  else if (p.tile == 1) launch<256, 192, 4, 2, 2, EPI_PARTIAL>(a, s);
  else if (p.tile == 2) launch<256, 128, 4, 2, 2, EPI_PARTIAL>(a, s);
  else if (p.tile == 4) launch_step<128, 128, 4, 2, 5, EPI_PARTIAL>(a, s);
  else if (p.tile == 5) launch_step<128, 64, 4, 2, 6, EPI_PARTIAL>(a, s);
  else if (one_each(M, N, p.splits)) launch_step<64, 32, 4, 1, 6, EPI_PARTIAL>(a, s);
  else launch_step<64, 64, 4, 2, 5, EPI_PARTIAL>(a, s);
}

void launch_gemm_lmhead_bf16(const bf16* A, const bf16* W, int M, int V, int K, const LmHeadEpilogue& e, Gate g,
                             hipStream_t s) {
  GemmArgs a = {};
  a.A = A; a.B0 = W; a.M = M; a.N = V; a.K = K; a.splits = 1; a.gate = g; a.lm = e;
  // The partial (max, sum, argmax) triples are per 128 logits in every configuration.  The weights are read once per row
  // tile, so from 129 rows on a 256-row tile halves the stream; up to 128 rows it would multiply empty rows (us, 128x128 /
  // 256x256 tiles; 4096 x 126464: 128 rows 225 / 228, 129 rows 334 / 227, 512 rows 649 / 412, 2048 rows 2400 / 1530;
  // 1024 x 32000: 128 rows 20 / 36, 256 rows 34 / 37, 288 rows 47 / 40, 1024 rows 116 / 75).
  if (M <= 32) launch_step<32, 128, 2, 2, 4, EPI_LMHEAD>(a, s);
  else if (M <= 64) launch_step<64, 128, 4, 1, 3, EPI_LMHEAD>(a, s);
  else if (M <= 128) launch<128, 128, 4, 2, 3, EPI_LMHEAD>(a, s);
  else launch<256, 256, 2, 4, 2, EPI_LMHEAD>(a, s);
}
int lmhead_n_part(int V) { return (V + 127) / 128; }

}  // namespace l2pd
