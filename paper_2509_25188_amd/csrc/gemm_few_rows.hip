// bf16 MFMA GEMM for few rows (a block-only step of the cached decode modes: up to 64 rows) on gfx950:
// C[M, N] = A[M, K] * W[N, K]^T, fp32 accumulation.
//
// Such a GEMM is bound by streaming its weights once, which wants several workgroups per CU with deep rings in
// flight: 32- or 64-row tiles whose operands go global -> LDS directly (global_load_lds_dwordx4: no VGPR staging, no
// ds_write) through an NS-stage ring, so that loads run NS-1 K-steps ahead of the MFMAs; the wait for a stage is
// a manual s_waitcnt vmcnt(n) that leaves the younger stages in flight.  LDS rows are swizzled as in
// gemm_bf16.hip.  K is split into fp32 partials (O and down projections, whose sums the next RMSNorm adds to the residual
// stream) or, where the output is wide enough, not at all (gate/up with SwiGLU in the epilogue).  Q/K/V, narrower gate/up and the LM
// head of few rows are small tiles of gemm_bf16.hip.
#include "gemm_common.h"

namespace l2pd {
namespace {

enum { EPI_PARTIAL = 0, EPI_SWIGLU = 2 };

struct FewArgs {
  const bf16* A;
  const bf16* B0;
  const bf16* B1;
  int M, N, K;          // N counts tile-space columns (SwiGLU: gate and up columns)
  int splits, k_len;    // K range of a workgroup
  TileMap map;
  Gate gate;
  // EPI_PARTIAL: K range z writes to parts + z * part_stride (fp32 [M, N])
  float* parts;
  size_t part_stride;
  int n_sub;            // > 0: the N rows are the rows of B0 and B1 stacked, n_sub rows each
  // EPI_SWIGLU (fragment 2p of a wavefront holds gate, fragment 2p+1 up columns of the same 32 features)
  bf16* act;
  int F;
};

template <int BM, int BN, int BK, int WM, int WN, int NS, int EPI, bool COLD>
__global__ void __launch_bounds__(WM* WN * 64) k_gemm_few_rows(FewArgs a) {
  constexpr int NW = WM * WN;
  constexpr int FM = BM / WM / 32, FN = BN / WN / 32;
  constexpr bool PAIR = EPI == EPI_SWIGLU;
  static_assert(!PAIR || (FN % 2 == 0), "pair epilogues need an even number of column fragments");
  static_assert(BK == 32 || BK == 64, "LDS tile rows hold 32 or 64 K elements");
  constexpr int CPR = BK / 8;               // 16-byte chunks per LDS row
  constexpr int RPD = 64 / CPR;             // rows filled by one direct-to-LDS wave load (1 KB)
  constexpr int KEY_SHIFT = BK == 64 ? 1 : 2;   // rows per 256-byte bank sweep = 1 << KEY_SHIFT
  constexpr int KS = BK / 16;               // MFMA K-steps per stage
  constexpr int LROWS = BM + BN;    // tile rows staged in LDS
  constexpr int LPS = LROWS / RPD / NW;     // direct-to-LDS loads per thread per stage
  static_assert(LPS * NW * RPD == LROWS && BM % (NW * RPD) == 0, "tile/threads mismatch");
  static_assert(NS >= 3 && (NS - 2) * LPS < 64, "ring depth: at least 3 stages, vmcnt is 6 bits");

  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  // [stage][A: BM rows | B: BN rows][BK bf16]
  constexpr int STAGE_BYTES = LROWS * BK * 2;

  int z, tile_m, tile_n;
  if (!a.map.place(blockIdx.x, &z, &tile_m, &tile_n)) return;
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int hf = lane >> 5, lj = lane & 31;

  const int k_begin = z * a.k_len;
  const int nk = a.k_len / BK;

  // ---- per-thread source pointers of the direct-to-LDS loads (fixed over the K loop) ----
  // Load q of a stage (q = wave + i*NW) fills combined tile rows RPD*q .. RPD*q+RPD-1 (A rows first, then B).
  const bf16* src[LPS];
#pragma unroll
  for (int i = 0; i < LPS; ++i) {
    const int q = wave + i * NW;
    const int rr = q * RPD + lane / CPR;         // row in the combined [A; B] tile
    const int c = (lane % CPR) ^ ((rr >> KEY_SHIFT) & (CPR - 1));   // global chunk that belongs at this lane's slot
    if (rr < BM) {
      int gr = min(m0 + rr, a.M - 1);
      src[i] = a.A + (size_t)gr * a.K + k_begin + c * 8;
    } else {
      const int r = rr - BM;
      const bf16* base;
      size_t grow;
      if constexpr (!PAIR) {
        int gn = min(n0 + r, a.N - 1);
        base = a.B0;
        if (a.n_sub > 0) {
          const int mat = gn >= a.n_sub;
          gn -= mat * a.n_sub;
          base = mat == 0 ? a.B0 : a.B1;
        }
        grow = (size_t)gn;
      } else {
        const int rw = r / (32 * FN), f = (r >> 5) % FN, j = r & 31;
        const int G = tile_n * (BN / 64) + rw * (FN / 2) + (f >> 1);
        base = f & 1 ? a.B1 : a.B0;
        grow = (size_t)min(G * 32 + j, a.F - 1);
      }
      src[i] = base + grow * a.K + k_begin + c * 8;
    }
  }
  // LDS byte address of this wave's first slot in stage 0 (wave-uniform, goes to M0)
  const unsigned lds0 = __builtin_amdgcn_readfirstlane(
      (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)(smem + wave * 1024));
  // Loads of one stage are issued in KS parts (load i belongs to part i % KS), one part per K-step,
  // so that they trickle into the texture-address queue behind MFMAs instead of arriving as a burst
  // from every wave right after the barrier (a burst stalls instruction issue until the queue drains).
  auto issue_part = [&](int kt, int part) {
    const unsigned dst = lds0 + (kt % NS) * STAGE_BYTES;
#pragma unroll
    for (int i = 0; i < LPS; ++i)
      if (i % KS == part) {
        if (i * NW * RPD >= BM) dma16_weights<COLD>(src[i] + kt * BK, dst + i * NW * 1024);
        else dma16(src[i] + kt * BK, dst + i * NW * 1024);
      }
  };

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // fragment row byte offsets inside a stage (row * 128) and the row's swizzle key
  int offA[FM], offB[FN];
#pragma unroll
  for (int i = 0; i < FM; ++i) offA[i] = (wm * (BM / WM) + i * 32 + lj) * (BK * 2);
#pragma unroll
  for (int j = 0; j < FN; ++j) offB[j] = BM * (BK * 2) + (wn * (BN / WN) + j * 32 + lj) * (BK * 2);
  const int key = (lj >> KEY_SHIFT) & (CPR - 1);   // row's swizzle key (fragment bases are multiples of 32)

  // Software pipeline.  Fragments are double-buffered in registers: the ds_reads of K-step kk+1 are
  // issued before the MFMAs of step kk, and the first fragments of the next stage are read during
  // the last step of the current one.  The ring advances (wait for stage kt+1, barrier, refill the
  // buffer of stage kt-1 with stage kt+NS-1) right before that last step, so a wave that waits at
  // the barrier leaves a full step of MFMAs queued behind it.
  bf16x8_t fa[2][FM], fb[2][FN];
  auto read_frags = [&](int buf, const unsigned char* base, int kk) {
    const int sw = ((kk * 2 + hf) ^ key) << 4;
#pragma unroll
    for (int i = 0; i < FM; ++i) fa[buf][i] = *reinterpret_cast<const bf16x8_t*>(base + offA[i] + sw);
#pragma unroll
    for (int j = 0; j < FN; ++j) fb[buf][j] = *reinterpret_cast<const bf16x8_t*>(base + offB[j] + sw);
  };
  // One K-step: the FM*FN MFMAs on fragment set `cur`, with the ds_reads that fetch set `cur ^ 1`
  // (K-step kk_next of the stage at `nbase`) slotted in between them, one read after each of the
  // first MFMAs, so that every read is issued while an MFMA occupies the matrix pipe.
  constexpr int NR = FM + FN;
  auto step = [&](int kk, const unsigned char* nbase, int kk_next, int dma_kt, int dma_part) {
    const int cur = kk & 1;   // fragment set of K-step kk
    const int sw = ((kk_next * 2 + hf) ^ key) << 4;
    const int nxt = cur ^ 1;
#pragma unroll
    for (int idx = 0; idx < FM * FN; ++idx) {
      const int i = idx / FN, j = idx % FN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[cur][i], fb[cur][j], acc[i][j], 0, 0, 0);
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        if ((r < FM * FN ? r : FM * FN - 1) != idx) continue;   // read r goes after MFMA min(r, last)
        if (r < FM) fa[nxt][r] = *reinterpret_cast<const bf16x8_t*>(nbase + offA[r] + sw);
        else fb[nxt][r - FM] = *reinterpret_cast<const bf16x8_t*>(nbase + offB[r - FM] + sw);
      }
      if (idx == 0 && dma_kt >= 0) issue_part(dma_kt, dma_part);   // stays in program order
    }
#pragma unroll
    for (int idx = 0; idx < FM * FN; ++idx) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA, then the LDS reads of its slot
#pragma unroll
      for (int r = 0; r < NR; ++r)
        if ((r < FM * FN ? r : FM * FN - 1) == idx) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  const int2 gate = gate_words(a.gate);    // looked at when the first loads are on their way
  // Prologue: stages 0 .. NS-2.  The wait counts loads, so nothing may move across it.
#pragma unroll
  for (int st = 0; st < NS - 1; ++st)
    if (st < nk) {
#pragma unroll
      for (int part = 0; part < KS; ++part) issue_part(st, part);
    }
  __builtin_amdgcn_sched_barrier(0);
  if (gate_closed(a.gate, gate)) {
    wait_vmcnt<0>();                       // LDS stays this workgroup's until its loads have landed
    return;
  }
  if (nk >= NS - 1) wait_vmcnt<(NS - 2) * LPS>();   // stage 0 has landed
  else wait_vmcnt<0>();
  __builtin_amdgcn_sched_barrier(0);
  lds_barrier();
  // Drain scalar loads here, so that only in-order LDS reads are pending when the loop is entered
  // and the compiler can wait for "all but the newest reads" instead of lgkmcnt(0) at its head.
  __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
  read_frags(0, smem, 0);
  __builtin_amdgcn_sched_barrier(0);
  for (int kt = 0; kt < nk; ++kt) {
    const unsigned char* base = smem + (kt % NS) * STAGE_BYTES;
    // parts 1 .. KS-1 of stage kt+NS-2 (its part 0 went out with the last K-step of iteration kt-1; the prologue
    // has issued all of stage NS-2)
    const int dma_a = (kt >= 1 && kt + NS - 2 < nk) ? kt + NS - 2 : -1;
#pragma unroll
    for (int kk = 0; kk < KS - 1; ++kk) step(kk, base, kk + 1, dma_a, kk + 1);
    if (kt + 1 < nk) {
      // stage kt+1 has landed once at most the loads of the NS-3 younger stages are outstanding
      if (kt + NS - 2 < nk) wait_vmcnt<(NS - 3) * LPS>();
      else wait_vmcnt<0>();
      lds_barrier();   // stage kt+1 visible to all; every wave is past its reads of stage kt-1
    }
    __builtin_amdgcn_sched_barrier(0);
    // The reads of the next stage's first fragments are unconditional (after the last stage they
    // fetch stale but valid LDS that nobody uses): a branch around them would make the compiler's
    // LDS wait counts conservative at the join.  The buffer of stage kt-1 is free from here on:
    // start refilling it with stage kt+NS-1.
    step(KS - 1, smem + ((kt + 1) % NS) * STAGE_BYTES, 0, (kt + NS - 1 < nk) ? kt + NS - 1 : -1, 0);
  }
  lds_barrier();

  // ------------------------------------------------------------------------------------------
  // C layout of the 32x32 MFMA: register r of a lane is row (r/4)*8 + hf*4 + r%4, column lj.
  const int row_base = m0 + wm * (BM / WM);
  if constexpr (EPI == EPI_PARTIAL) {
    float* out = a.parts + (size_t)z * a.part_stride;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        int col = n0 + wn * (BN / WN) + j * 32 + lj;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          int row = row_base + i * 32 + (r >> 2) * 8 + hf * 4 + (r & 3);
          if (row < a.M && col < a.N) out[(size_t)row * a.N + col] = acc[i][j][r];
        }
      }
  } else {
    const int lr = lj & 3, c4 = lj & ~3;   // after the transpose: row within the group, first of 4 columns
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int p = 0; p < FN / 2; ++p) {
        const int G = tile_n * (BN / 64) + wn * (FN / 2) + p;
        const int col = G * 32 + c4;
#pragma unroll
        for (int rq = 0; rq < 4; rq += 2) {   // two row groups share one transpose: low / high half words
          unsigned w[4];
#pragma unroll
          for (int rr = 0; rr < 4; ++rr) {
            const float g0 = acc[i][2 * p][rq * 4 + rr], u0 = acc[i][2 * p + 1][rq * 4 + rr];
            const float g1 = acc[i][2 * p][rq * 4 + 4 + rr], u1 = acc[i][2 * p + 1][rq * 4 + 4 + rr];
            // SiLU(g) * u with the hardware reciprocal (1 ulp) instead of an exact division; the
            // operations are spelled out so that every tile configuration rounds alike
            const float s0 = __fmul_rn(__fmul_rn(g0, __builtin_amdgcn_rcpf(__fadd_rn(1.f, __expf(-g0)))), u0);
            const float s1 = __fmul_rn(__fmul_rn(g1, __builtin_amdgcn_rcpf(__fadd_rn(1.f, __expf(-g1)))), u1);
            w[rr] = pack_bf16(s0, s1);
          }
          quad_transpose(w, lane);
#pragma unroll
          for (int h2 = 0; h2 < 2; ++h2) {
            const int row = row_base + i * 32 + (rq + h2) * 8 + hf * 4 + lr;
            uint2 o;
            o.x = h2 ? (w[0] >> 16) | (w[1] & 0xffff0000u) : (w[0] & 0xffffu) | (w[1] << 16);
            o.y = h2 ? (w[2] >> 16) | (w[3] & 0xffff0000u) : (w[2] & 0xffffu) | (w[3] << 16);
            if (row < a.M && col < a.F) {   // F is a multiple of 4, so a group of 4 columns is in or out as a whole
              *reinterpret_cast<uint2*>(reinterpret_cast<unsigned short*>(a.act) + (size_t)row * a.F + col) = o;
            }
          }
        }
      }
  }
}

template <int BM, int BN, int BK, int WM, int WN, int NS, int EPI, bool COLD = false>
void launch(FewArgs& a, hipStream_t s) {
  if constexpr (!COLD)
    if (a.gate.cold) return launch<BM, BN, BK, WM, WN, NS, EPI, true>(a, s);
  auto kern = k_gemm_few_rows<BM, BN, BK, WM, WN, NS, EPI, COLD>;
  constexpr int smem = NS * (BM + BN) * BK * 2;
  static DynLdsAttr attr;
  attr.ensure(reinterpret_cast<const void*>(kern), smem);
  a.map = TileMap((a.M + BM - 1) / BM, (a.N + BN - 1) / BN, a.splits);
  a.k_len = a.K / a.splits;
  hipLaunchKernelGGL(kern, dim3((a.map.total + 7) / 8 * 8), dim3(WM * WN * 64), smem, s, a);
}

}  // namespace

// K ranges of a step's projections, the same for all of up to 64 rows: a sequence's sums do not depend on how many others
// share its launch.  Tiles of 64 columns: ranges until there is a workgroup for every CU, and on to two for every CU while the
// last round of them is less than four fifths full; more only cost what sums them.  The four fifths, us with events around the launch,
// 32 rows, with / without: 5120 wide (eight ranges for four) output 16.3 / 18.5, down of 13824 30.8 / 36.3, the RMSNorm behind them
// 7.7 / 6.8; 3072 (16 for 8) down of 8192 15.2 / 16.0; 6144 (8 for 4) output 19.8 / 20.9, down of 24576 55.5 / 68.3, but of 16384 47.0 / 46.2.
// (64 rows: equal for the outputs and 13824 40.5 / 42.7, 8192 20.1 / 19.0, 24576 72.3 / 79.3, 16384 65.7 / 51.8.)
int skinny_splits(int N, int K) {
  const int tiles = (N + 63) / 64;
  int S = 1;
  while (S < 16 && K % (S * 2 * 64) == 0 && K / (S * 2) >= 256 &&
         (tiles * S < 256 || (tiles * S < 512 && (tiles * S + 255) / 256 * 256 * 4 > tiles * S * 5)))
    S *= 2;
  return S;
}

// Few rows (a block-only step of the cached decode modes: 32 or 64 rows): every GEMM is bound by
// streaming its weights once, which needs several workgroups per CU with deep rings in flight.
// K split `splits` ways into fp32 partials; gate and up, n_sub rows each, are stacked along N (SwiGLU runs afterwards on the
// summed partials).
//   Up to 32 rows two wavefronts take 64 columns: a ring of six stages while two workgroups to a CU are all there are, of four
// where three fit (us at 4096 / 12288 wide, these / tiles of 128 columns with four wavefronts and the ranges that those need:
// output 8.0 / 8.2 with half the partials, down 20.6 / 21.3 with half the partials; four ranges of the
// last layer's down projection 20.6 / 27.8).
//   Up to 64 rows, the same ranges: four wavefronts take 64 columns, with a ring of eight stages while there is a workgroup to
// a CU at most, of five while there are two; beyond that 128 columns.  64 rows of 4096 / 12288, these / tiles of 128 columns with
// twice the ranges: output and down 18.1 / 17.1 on average, the RMSNorm behind them 4.8 / 5.3, a step of eight layers 1451 / 1454;
// of 1024 / 2816: output and down 6.8 / 7.9, gate/up 8.0 / 7.9, RMSNorm 3.0 / 3.6, a step 464 / 480; 48 rows of 4096: a step 1361 / 1378.
void launch_gemm_skinny_bf16(const bf16* A, const bf16* w0, const bf16* w1, int n_sub, float* parts,
                             size_t part_stride, int M, int N, int K, int splits, Gate g, hipStream_t s) {
  FewArgs a = {};
  a.A = A; a.B0 = w0; a.B1 = w1; a.n_sub = w1 ? n_sub : 0;
  a.M = M; a.N = N; a.K = K; a.splits = splits; a.gate = g;
  a.parts = parts; a.part_stride = part_stride;
  const int groups = (N + 63) / 64 * splits;
  if (M > 32 && groups <= 256) launch<64, 64, 64, 2, 2, 8, EPI_PARTIAL>(a, s);
  else if (M > 32 && groups <= 512) launch<64, 64, 64, 2, 2, 5, EPI_PARTIAL>(a, s);
  else if (M > 32) launch<64, 128, 64, 2, 2, 4, EPI_PARTIAL>(a, s);
  else if (groups <= 512) launch<32, 64, 64, 1, 2, 6, EPI_PARTIAL>(a, s);
  else launch<32, 64, 64, 1, 2, 4, EPI_PARTIAL>(a, s);
}

// Which way gate/up takes.  Tiles of gemm_bf16.hip (figures at launch_few there) while all of them are on the chip at once; wider
// ones the kernel above: 64 (32 gate + 32 up) columns to a wavefront, or 128 to four above 32 rows, K unsplit.  Where even
// 32 columns leave half of the chip idle for a long chain of stages, split K and a finishing kernel, unless the rows must sum as those
// of a larger pass (`ranges` false).  us with events around the launches, 32 and 64 rows, ranges / tiles: 4096 x 1024 14.0 / 17.3,
// 16.0 / 22.4; 8192 x 1984 21.6 / 28.6, 24.6 / 38.9; 2816 x 1984 13.9 / 14.0, 15.9 / 17.6; 2048 x 1024 12.9 / 11.6, 14.0 / 14.4; 1600 x 1984
// 16.1 / 10.8, 17.1 / 13.0: even at about 32 stages.  The order of the sums is part of a result, so the line stays where it was put, at 24.
GateUpPath few_rows_gate_up(int F, int K, bool ranges) {
  if (ranges && 2 * F < 128 * 32 && K > 24 * 64) return GATE_UP_RANGES;
  return 2 * F <= 256 * 96 ? GATE_UP_TILES : GATE_UP_WIDE;   // 768 tiles of 32 columns, 256 of 96
}

void launch_gemm_few_rows_swiglu_bf16(const bf16* A, const bf16* wg, const bf16* wu, bf16* act, int M, int F, int K, Gate g,
                                      hipStream_t s) {
  FewArgs a = {};
  a.A = A; a.B0 = wg; a.B1 = wu; a.M = M; a.N = 2 * F; a.K = K; a.splits = 1; a.gate = g;
  a.act = act; a.F = F;
  if (M <= 32) launch<32, 64, 64, 1, 1, 6, EPI_SWIGLU>(a, s);   // one wavefront per workgroup, 72 KB ring
  else launch<64, 128, 64, 2, 2, 4, EPI_SWIGLU>(a, s);
}

}  // namespace l2pd
