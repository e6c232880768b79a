// Dense contractions of the exact block: out = epi(A W^T + bias) with A [M, K] (rows
// through a RowMap), W [N, K] (both K-contiguous), fp32 accumulation.
//
// bf16: 256-row workgroup tiles of v_mfma_f32_16x16x32_bf16 (k_gemm_pp) where the grid fills
// the card, 64- and 128-row tiles of v_mfma_f32_32x32x16_bf16 whose waves split K (k_gemm_ks) on
// small grids.  Both stream operands global -> LDS directly; a register-staged kernel (padded LDS
// rows, double buffer) takes large grids at K <= 256 and operand rows too far apart for the DMA.
// fp32: fp32 MFMAs on 16x16, 32x32 or 64x64 tiles, the waves of a tile splitting K.
#include "dev_common.h"
#include "gemm_plan.h"

namespace ff {

namespace {

// Template-only epilogue value: bias, plus GELU where the problem's own a.epi asks for it
// (a uniform branch per tile), so that a bias GEMM and a bias+GELU GEMM can share a launch.
constexpr int EPI_BIAS_OR_GELU = 3;


// Elements (uint16) of LDS the epilogue stages per workgroup: each wave owns 32 rows of
// its WN columns in fp32 (the worst case), rows padded by 4 floats.
template <int NW, int WN>
constexpr int epi_lds_elems() { return NW * 32 * (WN + 4) * 2; }

// Epilogue of one wavefront's TM x TN block of 32x32 MFMA tiles (acc), whose rows start at
// rbase and columns at cbase.  In the MFMA layout lane l owns row rbase + 32 i + l%32 and,
// per 32-column tile, 4 groups of 4 consecutive columns (8 q + 4 (l/32)): a store
// instruction there writes 8 bytes to each of 32 rows, which costs the memory pipeline one
// request per row.  So each 32-row block goes through the wave's own LDS region (lds):
// values are finished as far as the MFMA layout allows (bias, GELU) and staged as rows,
// as rounded bf16 when that is the output, else in fp32 (the gated residual is added to
// the unrounded value).  They are read back with consecutive lanes on consecutive
// 8-column pieces of a row, so every residual, gate and history load and every store is
// a 16-byte access and one instruction covers whole row segments.  The physical row (and
// sample) of each row is computed once by the lane that owns it in the MFMA layout and
// fetched by the storing lanes with a lane shuffle.  N % 8 == 0: a piece is in range as a
// whole.  LDS use is wave-private: the caller must have retired the main loop's LDS reads
// of all waves (barrier) before the first call.
//
// Accumulator layouts: pieces of 4 consecutive output columns held by a lane, piece p of
// 32-row block i at row row() and column col() of the block.
template <int TM_, int TN_>
struct Acc32 {   // 32x32 tiles: lane l row l%32, columns 32 j + 8 q + 4 (l/32) + 0..3
  static constexpr int TM = TM_, WN = TN_ * 32, P = TN_ * 4;
  f32x16_t t[TM_][TN_];
  __device__ __forceinline__ static int row(int, int lane) { return lane & 31; }
  __device__ __forceinline__ static int col(int p, int lane) { return p * 8 + (lane >> 5) * 4; }
  __device__ __forceinline__ float get(int i, int p, int e) const { return t[i][p / 4][4 * (p % 4) + e]; }
};
template <int TM_, int TN_>
struct Acc16 {   // 16x16 tiles (two per 32-row block): lane l row l%16, columns 16 j + 4 (l/16) + 0..3
  static constexpr int TM = TM_ / 2, WN = TN_ * 16, P = TN_ * 2;
  f32x4_t t[TM_][TN_];
  __device__ __forceinline__ static int row(int p, int lane) { return (p / TN_) * 16 + (lane & 15); }
  __device__ __forceinline__ static int col(int p, int lane) { return (p % TN_) * 16 + (lane >> 4) * 4; }
  __device__ __forceinline__ float get(int i, int p, int e) const { return t[2 * i + p / TN_][p % TN_][e]; }
};
template <int EPI, bool OUT_F32, bool RES_F32, class ACC>
__device__ __forceinline__ void epilogue_block(const GemmArgs a, int rbase, int cbase, const ACC& acc, uint16_t* lds) {
  constexpr bool kF32 = OUT_F32 || EPI == EPI_GATED;
  constexpr int TM = ACC::TM, WN = ACC::WN, CPR = WN / 8, RPP = 64 / CPR, NPASS = (32 + RPP - 1) / RPP;
  constexpr int LDW = kF32 ? WN + 4 : WN + 8;   // row pitch in staged elements
  static_assert(CPR <= 64, "row wider than a wavefront's pieces");
  constexpr bool kCache = EPI == EPI_GATED && !OUT_F32;
  const int lane = threadIdx.x & 63, fr = lane & 31;
  const uint16_t* bias = reinterpret_cast<const uint16_t*>(a.bias);
  const bool gelu = EPI == EPI_BIAS_GELU || (EPI == EPI_BIAS_OR_GELU && a.epi == EPI_BIAS_GELU);
  float* lf = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int rmine = rbase + i * 32 + fr;
    const int prow = a.omap.phys(rmine < a.M ? rmine : 0);
    const int srow = EPI == EPI_GATED ? a.omap.sample(rmine < a.M ? rmine : 0) : 0;
#pragma unroll
    for (int p = 0; p < ACC::P; ++p) {
      const int pr = ACC::row(p, lane), pc = ACC::col(p, lane), c = cbase + pc;
      const u32x2_t bw = *reinterpret_cast<const u32x2_t*>(bias + (c < a.N ? c : 0));
      float v[4] = {acc.get(i, p, 0) + __uint_as_float(bw[0] << 16), acc.get(i, p, 1) + __uint_as_float(bw[0] & 0xffff0000u),
                    acc.get(i, p, 2) + __uint_as_float(bw[1] << 16), acc.get(i, p, 3) + __uint_as_float(bw[1] & 0xffff0000u)};
      if (gelu) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = gelu_tanh_f(v[e]);
      }
      const int off = pr * LDW + pc;
      if (kF32) {
        *reinterpret_cast<f32x4_t*>(lf + off) = f32x4_t{v[0], v[1], v[2], v[3]};
      } else {
        *reinterpret_cast<u32x2_t*>(lds + off) = u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
      }
    }
    if (!kF32) {
#pragma unroll
      for (int p = 0; p < NPASS; ++p) {
        const int rr = p * RPP + lane / CPR, cc = (lane % CPR) * 8;
        const int src = rr < 32 ? rr : 0;
        const size_t pr = (size_t)__shfl(prow, src, 64);
        const int r = rbase + i * 32 + rr, c = cbase + cc;
        if (lane >= RPP * CPR || rr >= 32 || r >= a.M || c >= a.N) continue;
        *reinterpret_cast<u32x4_t*>(reinterpret_cast<uint16_t*>(a.out) + pr * a.ldo + c) =
            *reinterpret_cast<const u32x4_t*>(lds + rr * LDW + cc);
      }
      continue;
    }
    // fp32-staged rows, in groups of PG passes: every global load of a group (residual,
    // gate, and the layer input of the history refresh) is requested before the group's
    // first use.  Lanes that store nothing load row pr, column 0 (in range) and skip the
    // rest.  With the loads under the per-pass lane test, each pass waited for its own
    // loads (twice with the history refresh): up to 14 memory round trips per row block.
    constexpr int PG = NPASS < 4 ? NPASS : 4;
    const bool want_u = kCache && a.cache_out && a.cache_u;
#pragma unroll
    for (int p0 = 0; p0 < NPASS; p0 += PG) {
      size_t gpr[PG];
      int gc[PG], grr[PG], gcc[PG];
      bool ok[PG];
      f32x4_t rsf[PG][2], gg[PG][2];
      u32x4_t rsb[PG], uu[PG];
#pragma unroll
      for (int q = 0; q < PG; ++q) {
        const int p = p0 + q;
        if (p >= NPASS) break;
        const int rr = p * RPP + lane / CPR, cc = (lane % CPR) * 8;
        const int src = rr < 32 ? rr : 0;
        const size_t pr = (size_t)__shfl(prow, src, 64);
        const int sr = EPI == EPI_GATED ? __shfl(srow, src, 64) : 0;
        const int r = rbase + i * 32 + rr, c = cbase + cc;
        ok[q] = !(lane >= RPP * CPR || rr >= 32 || r >= a.M || c >= a.N);
        const int cl = ok[q] ? c : 0;
        gpr[q] = pr; gc[q] = c; grr[q] = rr; gcc[q] = cc;
        if (EPI == EPI_GATED) {
          if (RES_F32) {
            const float* rp = reinterpret_cast<const float*>(a.resid) + pr * a.ldr + cl;
            rsf[q][0] = *reinterpret_cast<const f32x4_t*>(rp);
            rsf[q][1] = *reinterpret_cast<const f32x4_t*>(rp + 4);
          } else {
            rsb[q] = *reinterpret_cast<const u32x4_t*>(reinterpret_cast<const uint16_t*>(a.resid) + pr * a.ldr + cl);
          }
          const float* gp = a.gate + (size_t)sr * a.ldg + cl;
          gg[q][0] = *reinterpret_cast<const f32x4_t*>(gp);
          gg[q][1] = *reinterpret_cast<const f32x4_t*>(gp + 4);
        }
        if (want_u) uu[q] = *reinterpret_cast<const u32x4_t*>(reinterpret_cast<const uint16_t*>(a.cache_u) + pr * a.ldo + cl);
      }
#pragma unroll
      for (int q = 0; q < PG; ++q) {
        if (p0 + q >= NPASS) break;
        if (!ok[q]) continue;
        const size_t pr = gpr[q];
        const int c = gc[q], rr = grr[q], cc = gcc[q];
        const f32x4_t x0 = *reinterpret_cast<const f32x4_t*>(lf + rr * LDW + cc);
        const f32x4_t x1 = *reinterpret_cast<const f32x4_t*>(lf + rr * LDW + cc + 4);
        float v[8] = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
        if (EPI == EPI_GATED) {
          float rs[8];
          if (RES_F32) {
#pragma unroll
            for (int e = 0; e < 4; ++e) { rs[e] = rsf[q][0][e]; rs[e + 4] = rsf[q][1][e]; }
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              rs[2 * e] = __uint_as_float(rsb[q][e] << 16);
              rs[2 * e + 1] = __uint_as_float(rsb[q][e] & 0xffff0000u);
            }
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[e] = rs[e] + gg[q][0][e] * v[e];
            v[e + 4] = rs[e + 4] + gg[q][1][e] * v[e + 4];
          }
        }
        if (OUT_F32) {
          St<DT_F32>::store(a.out, pr * a.ldo + c, v);
          St<DT_F32>::store(a.out, pr * a.ldo + c + 4, v + 4);
          continue;
        }
        St<DT_BF16>::store(a.out, pr * a.ldo + c, v);
        if (kCache && a.cache_out) {
          // history refresh from the stored (rounded) output, as the separate kernel does
          float h[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) h[e] = St<DT_BF16>::rnd(v[e]);
          if (a.cache_u) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              h[2 * e] -= __uint_as_float(uu[q][e] << 16);
              h[2 * e + 1] -= __uint_as_float(uu[q][e] & 0xffff0000u);
            }
          }
          St<DT_BF16>::store(a.cache_out, pr * a.ldo + c, h);
        }
      }
    }
  }
}

// Up to two GEMMs of the same epilogue in one launch (the text and image streams of an
// MMDiT block): workgroups [0, n0) take problem 0's tiles, the rest problem 1's.
template <int NP>
struct GemmGroup {
  GemmArgs g[NP];
  int tm[NP], tn[NP];   // tile rows / columns per problem
};

// Workgroup -> (problem, output tile).  Workgroups are dispatched round-robin over the 8
// XCDs (each with its own L2); the first floor(n/8)*8 of them are renumbered so that every
// XCD owns a contiguous range of tiles, and within a problem tiles are ordered in groups
// of kGroupM tile-rows so that an XCD's concurrent tiles share A rows and W columns in its
// L2.
constexpr int kGroupM = 8;
__device__ __forceinline__ int tile_of(int bid, int tm0, int tn0, int tm1, int tn1, int np, int& tm, int& tn) {
  const int n0 = tm0 * tn0;
  const int nwg = n0 + (np > 1 ? tm1 * tn1 : 0);
  const int full = (nwg / 8) * 8;
  int id = bid < full ? (bid % 8) * (full / 8) + bid / 8 : bid;
  int p = 0, tiles_m = tm0, tiles_n = tn0;
  if (id >= n0) { p = 1; id -= n0; tiles_m = tm1; tiles_n = tn1; }
  const int per_group = kGroupM * tiles_n;
  const int first_m = (id / per_group) * kGroupM;
  const int gsz = min(tiles_m - first_m, kGroupM);
  const int in_group = id % per_group;
  tm = first_m + in_group % gsz;
  tn = in_group / gsz;
  return p;
}

// ------------------------------------------------------------------ bf16 MFMA GEMM
// Register-staged (large grids at short K, any operand strides): BM x BN workgroup tile, BK = 64 per LDS stage
// with padded rows, wavefront tiles WM x WN of v_mfma_f32_32x32x16_bf16.
constexpr int BK = 64, LDT = BK + 8;

// 32x32x16 MFMA: A operand lane l = row (l%32), k 8*(l/32)..+7; B operand lane l = col (l%32),
// same k; D[v] at row 8*(v/4) + 4*(l/32) + v%4, col l%32.  With A = weight rows (output
// columns n) and B = activation rows (output rows m): lane l owns output row m = l%32 and
// columns n = 8*(v/4) + 4*(l/32) + (v%4), i.e. 4 groups of 4 consecutive columns.
template <int BM, int BN, int WM, int WN, int EPI, bool OUT_F32, bool RES_F32, int NP>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64) void k_gemm_bf16(GemmGroup<NP> G) {
  constexpr int NWN = BN / WN;
  constexpr int NT = (BM / WM) * NWN * 64;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int RSTEP = NT / 8;
  constexpr int CA = BM / RSTEP, CB = BN / RSTEP;
  constexpr int kMain = 2 * (BM + BN) * LDT, kEpi = epi_lds_elems<(BM / WM) * NWN, WN>();
  __shared__ __attribute__((aligned(1024))) uint16_t smem[kMain > kEpi ? kMain : kEpi];
  uint16_t (*sA)[BM * LDT] = reinterpret_cast<uint16_t (*)[BM * LDT]>(smem);
  uint16_t (*sB)[BN * LDT] = reinterpret_cast<uint16_t (*)[BN * LDT]>(smem + 2 * BM * LDT);
  // wave index in a scalar register: the per-wave LDS addresses of the DMA (M0) are then
  // computed on the scalar unit instead of with a v_readfirstlane per instruction
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tm, tn;
  // workgroup-uniform: keep the problem select and tile origin in scalar registers
  const int prob = __builtin_amdgcn_readfirstlane(tile_of(blockIdx.x, G.tm[0], G.tn[0], G.tm[NP - 1], G.tn[NP - 1], NP, tm, tn));
  tm = __builtin_amdgcn_readfirstlane(tm);
  tn = __builtin_amdgcn_readfirstlane(tn);
  const GemmArgs a = (NP > 1 && prob) ? G.g[NP - 1] : G.g[0];
  const int m0 = tm * BM, n0 = tn * BN;
  const uint16_t* A = reinterpret_cast<const uint16_t*>(a.A);
  const uint16_t* W = reinterpret_cast<const uint16_t*>(a.W);
  const int lrow = tid >> 3, kc = (tid & 7) * 8;
  size_t offa[CA], offb[CB];
  unsigned mask = 0;
#pragma unroll
  for (int i = 0; i < CA; ++i) {
    const int gm = m0 + lrow + RSTEP * i;
    if (gm < a.M) mask |= 1u << i;
    offa[i] = (size_t)(gm < a.M ? a.amap.phys(gm) : 0) * a.lda + kc;
  }
#pragma unroll
  for (int i = 0; i < CB; ++i) {
    const int gn = n0 + lrow + RSTEP * i;
    if (gn < a.N) mask |= 1u << (16 + i);
    offb[i] = (size_t)(gn < a.N ? gn : 0) * a.ldw + kc;
  }
  u32x4_t ra[CA], rb[CB];
  const u32x4_t z4 = {0u, 0u, 0u, 0u};
#define FF_GLOAD(k0)                                                                                   \
  do {                                                                                                 \
    const bool kin = (k0) + kc < a.K;                                                                  \
    _Pragma("unroll") for (int i = 0; i < CA; ++i)                                                     \
      ra[i] = (kin && (mask & (1u << i))) ? *reinterpret_cast<const u32x4_t*>(A + offa[i] + (k0)) : z4; \
    _Pragma("unroll") for (int i = 0; i < CB; ++i)                                                     \
      rb[i] = (kin && (mask & (1u << (16 + i)))) ? *reinterpret_cast<const u32x4_t*>(W + offb[i] + (k0)) : z4; \
  } while (0)
#define FF_SSTORE(buf)                                                                                 \
  do {                                                                                                 \
    _Pragma("unroll") for (int i = 0; i < CA; ++i)                                                     \
      *reinterpret_cast<u32x4_t*>(&sA[buf][(lrow + RSTEP * i) * LDT + kc]) = ra[i];                    \
    _Pragma("unroll") for (int i = 0; i < CB; ++i)                                                     \
      *reinterpret_cast<u32x4_t*>(&sB[buf][(lrow + RSTEP * i) * LDT + kc]) = rb[i];                    \
  } while (0)
  Acc32<TM, TN> accs;
  f32x16_t (&acc)[TM][TN] = accs.t;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  const int wm = (wave / NWN) * WM, wn = (wave % NWN) * WN;
  const int fr = lane & 31, fk = (lane >> 5) * 8;
  const int nk = (a.K + BK - 1) / BK;
  FF_GLOAD(0);
  FF_SSTORE(0);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < nk) FF_GLOAD((kt + 1) * BK);
#pragma unroll
    for (int kk = 0; kk < BK; kk += 16) {
      bf16x8_t fa[TM], fb[TN];
#pragma unroll
      for (int t = 0; t < TM; ++t)
        fa[t] = *reinterpret_cast<const bf16x8_t*>(&sA[cur][(wm + t * 32 + fr) * LDT + kk + fk]);
#pragma unroll
      for (int t = 0; t < TN; ++t)
        fb[t] = *reinterpret_cast<const bf16x8_t*>(&sB[cur][(wn + t * 32 + fr) * LDT + kk + fk]);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_iglp_opt(0);   // interleave the LDS fragment reads with the MFMAs
    }
    if (kt + 1 < nk) FF_SSTORE(cur ^ 1);
    __syncthreads();
  }
#undef FF_GLOAD
#undef FF_SSTORE
  // the loop ends with a barrier after every wave's last LDS read
  epilogue_block<EPI, OUT_F32, RES_F32>(a, m0 + wm, n0 + wn, accs, smem + wave * 32 * (WN + 4) * 2);
}
// ------------------------------------------------------------------ bf16 MFMA GEMM, two wave groups in turn
// 256 x 64 TN tile (TN = 2, 3, 4), 64-wide K stages, 8 waves in two groups of four, one wave
// of each group per SIMD.  A stage has four phases, one per 32 rows of a wave's 128 x 16 TN
// block; a phase is a memory part (its fragment reads and two DMA instructions per wave) and
// 4 TN MFMAs, with a barrier after each.  The second group runs half a phase behind, so that
// on every SIMD one wave's MFMAs cover the other's reads and DMA.
//
// What bounds it: on large grids the card's power limit.  With random operands the clock is 1.9 to
// 2.0 GHz of 2.4 and the MFMAs are busy 69 % of its cycles (counters at M = 4608, N = 21504, K = 3072),
// so what counts is energy per FLOP: v_mfma_f32_16x16x32_bf16 moves half the accumulator bytes per
// FLOP of the 32x32x16 form and runs 8 % faster in this same kernel (the same shape: 496 -> 460 us;
// one wait and barrier per stage with 32x32x16: 545 us).  On small grids it is bound by its
// chain of stages: 0.96 us per stage of 256x256 against 0.85 us of MFMA time at 2.4 GHz.
//
// Operands: 64-row pieces of 8 KB, each filled by one DMA instruction per wave, in two buffers
// per operand.  A piece's slot is refilled (two stages ahead) as soon as every wave is past
// its reads, one phase later, so 8 to 13 of a wave's DMAs stay in flight across every
// wait, and a piece has at least four phases (2048 cycles at TN = 4) to land.  With both buffers
// refilled only at stage ends (vmcnt(0) there) the same tile took 545 us on the shape above.
// Every wave waits for its own LDS reads and for its own share of the pieces that the next
// phase reads, then for the barrier; the phase that reads a piece starts after that barrier
// for both groups, and the DMA that overwrites one starts after a barrier that every wave
// passes with its reads of it complete.
// Reading one phase ahead (fragments double-buffered) was no faster: 1317 against 1337 TFLOP/s.
// Operand loads with sc0 | sc1 (past the L1) make no difference here or in k_gemm_ks: DiT-XL/2 block at
// batch 8 135.7 against 135.7 us, FLUX-like double block 1201 against 1201.
//
// K % 64 != 0 (K % 8 == 0): the chunks of the last stage past K are loaded from the row's
// first chunk of that stage (in bounds) and their fragments are zeroed in registers.
// DMA schedule of k_gemm_pp.  A stage's operands are 4 + TN pieces (A0-A3, B0..).  Phase p of
// stage k issues, in this order:
//   0: A3 of stage k+1, A0 of k+2    1: B0, B1 of k+2    2: A1, B2 of k+2    3: A2, B3 of k+2
// and reads: phase 0 all B of stage k, phases 1-3 A1-A3 of stage k, phase 3 also A0 of k+1.
// So a piece's slot is refilled no earlier than one phase after its last read, and a piece
// lands at least four phases after it was issued.
constexpr int kPPIssue[4][2] = {{3, 0}, {4, 5}, {1, 6}, {2, 7}};   // A0-A3 are 0-3, B0-B3 are 4-7
// How many of a wave's DMAs may still be outstanding at the end of phase p of a stage with
// `left` stages after it (2: two or more), so that what phase p + 1 reads has landed.
constexpr int pp_vm(int TN, int p, int left) {
  int n = 0, need = -1;   // DMAs issued in stages -2, -1 and 0 (this one) up to phase p; the last one needed
  for (int j = -2; j <= 0; ++j)
    for (int q = 0; q < (j == 0 ? p + 1 : 4); ++q)
      for (int i = 0; i < 2; ++i) {
        const int pc = kPPIssue[q][i], st = pc == 3 ? j + 1 : j + 2;
        if (pc >= 4 + TN || st > left) continue;
        ++n;
        const bool next = (p == 0 && pc == 1 && st == 0) || (p == 1 && pc == 2 && st == 0) ||
                          (p == 2 && ((pc == 3 && st == 0) || (pc == 0 && st == 1))) || (p == 3 && pc >= 4 && st == 1);
        if (next) need = n;
      }
  return need < 0 ? 63 : n - need;
}

#define FF_RDA(dst, off)                                             \
  do {                                                               \
    (dst)[0] = lds_rd128_at<(off)>(rda[0]);                          \
    (dst)[1] = lds_rd128_at<(off)>(rda[1]);                          \
    (dst)[2] = lds_rd128_at<(off) + 16 * 128>(rda[0]);               \
    (dst)[3] = lds_rd128_at<(off) + 16 * 128>(rda[1]);               \
  } while (0)

template <int TN, int EPI, bool OUT_F32, bool RES_F32, int NP>
__global__ __launch_bounds__(512) void k_gemm_pp(GemmGroup<NP> G) {
#ifdef __HIP_DEVICE_COMPILE__   // the host pass needs the launch stub only
  constexpr int BM = 256, BN = 64 * TN, WN = 16 * TN, BKd = 64, RB = 128;   // RB: bytes of an LDS row
  constexpr int PC = 64 * RB;                                                // bytes of a piece
  constexpr int BUFA = 4 * PC, BUFB = TN * PC, OFFB = 2 * BUFA;
  constexpr int kMain = OFFB + 2 * BUFB, kEpi = epi_lds_elems<8, WN>() * 2;
  __shared__ __attribute__((aligned(1024))) uint16_t smem[(kMain > kEpi ? kMain : kEpi) / 2];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int tm, tn;
  const int prob = __builtin_amdgcn_readfirstlane(tile_of(blockIdx.x, G.tm[0], G.tn[0], G.tm[NP - 1], G.tn[NP - 1], NP, tm, tn));
  tm = __builtin_amdgcn_readfirstlane(tm);
  tn = __builtin_amdgcn_readfirstlane(tn);
  const GemmArgs a = (NP > 1 && prob) ? G.g[NP - 1] : G.g[0];
  const int m0 = tm * BM, n0 = tn * BN;
  const int mw = wave >> 2, nw = wave & 3;
  const int nk = (a.K + BKd - 1) / BKd, kpad = nk * BKd - a.K;
  // operand bases of this tile (scalar) and per-lane byte offsets of its DMA rows: a piece is
  // 64 LDS rows, 8 per wave and instruction.  Piece Aq holds rows 32 q .. 32 q + 31 of both
  // wave rows, piece Bu columns 16 u .. 16 u + 15 of all four wave columns.  Rows past the
  // matrix read the tile's first row (in bounds); their results are never stored.
  const int p0 = a.amap.phys(m0);
  const char* Ab = reinterpret_cast<const char*>(a.A) + (size_t)p0 * a.lda * 2;
  const char* Wb = reinterpret_cast<const char*>(a.W) + (size_t)n0 * a.ldw * 2;
  __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(Ab), 0, 0xffffffffu, 0x00020000);
  __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(Wb), 0, 0xffffffffu, 0x00020000);
  const int R = wave * 8 + (lane >> 3);
  const uint32_t ch = ((lane & 7) ^ ((R >> 1) & 7)) * 16;
  uint32_t voa[4], vob[TN];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int gm = m0 + (R >> 5) * 128 + q * 32 + (R & 31);
    voa[q] = (gm < a.M ? (uint32_t)(a.amap.phys(gm) - p0) * (uint32_t)a.lda * 2u : 0u) + ch;
  }
#pragma unroll
  for (int u = 0; u < TN; ++u) {
    const int gn = (R >> 4) * WN + u * 16 + (R & 15);
    vob[u] = (n0 + gn < a.N ? (uint32_t)gn * (uint32_t)a.ldw * 2u : 0u) + ch;
  }
  // K % 64 != 0: the last stage's chunks past K load the row's chunk 0 of that stage instead
  // (in bounds), and their fragments are zeroed
  const uint32_t back = (kpad && ch >= (uint32_t)(BKd - kpad) * 2u) ? ch : 0u;
  char* const lds = reinterpret_cast<char*>(smem);
#define FF_DMA(rs, vo, dst, kb) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, FF_AS3(lds + (dst) + wave * 1024), 16, vo, kb, 0, 0)
  Acc16<8, TN> accs;
  f32x4_t (&acc)[8][TN] = accs.t;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int fr = lane & 15, fh = lane >> 4;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) const void*)smem);
  uint32_t rda[2], rdb[2];   // fragment addresses of the two 32-wide k steps, current buffers
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const uint32_t c = ((4 * s + fh) ^ (fr >> 1)) * 16;
    rda[s] = lds0 + (mw * 32 + fr) * RB + c;
    rdb[s] = lds0 + OFFB + (nw * 16 + fr) * RB + c;
  }
  bf16x8_t fa[2][4], fb[2 * TN];
  int kb = 0, ca = 0, cb = 0;   // this stage's byte offset along K, and its buffers
#define FF_MEM_END() asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory")
#define FF_MMA(q, A)                                                                                            \
  do {                                                                                                          \
    __builtin_amdgcn_sched_barrier(0);                                                                          \
    __builtin_amdgcn_s_setprio(1);                                                                              \
    _Pragma("unroll") for (int s = 0; s < 2; ++s)                                                               \
      _Pragma("unroll") for (int t = 0; t < 2; ++t)                                                             \
        _Pragma("unroll") for (int u = 0; u < TN; ++u)                                                          \
          acc[2 * (q) + t][u] =                                                                                 \
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[2 * u + s], (A)[2 * t + s], acc[2 * (q) + t][u], 0, 0, 0); \
    __builtin_amdgcn_s_setprio(0);                                                                              \
    __builtin_amdgcn_sched_barrier(0);                                                                          \
    asm volatile("s_barrier" ::: "memory");                                                                     \
  } while (0)
#define FF_TIEA(A) _Pragma("unroll") for (int i = 0; i < 4; ++i) FF_TIE((A)[i])
  // zero the fragments whose k lies past K (last stage; both operands, so that 0 * 0 is added)
  auto cut = [&](bf16x8_t& f, int s) __attribute__((always_inline)) {
    u32x4_t w = __builtin_bit_cast(u32x4_t, f);
    const bool in = (4 * s + fh) * 8 < BKd - kpad;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = in ? w[e] : 0u;
    f = __builtin_bit_cast(bf16x8_t, w);
  };
#define FF_CUTA(A)                                          \
  if (LEFT == 0 && kpad) {                                  \
    _Pragma("unroll") for (int i = 0; i < 4; ++i) cut((A)[i], i & 1); \
  }
  // one stage.  LEFT: stages after it (2: two or more)
  auto stage = [&](auto LEFTc) __attribute__((always_inline)) {
    constexpr int LEFT = decltype(LEFTc)::value;
    constexpr bool k1 = LEFT >= 1, k2 = LEFT >= 2;
    const int oa = BUFA - ca, ob = BUFB - cb;
    // phase 0
#pragma unroll
    for (int u = 0; u < TN; ++u) {
      fb[2 * u] = lds_rd128_off(rdb[0], u * PC);
      fb[2 * u + 1] = lds_rd128_off(rdb[1], u * PC);
    }
    if (k1) FF_DMA(ra, voa[3], 3 * PC + oa, kb + RB);
    if (k2) FF_DMA(ra, voa[0], ca, kb + 2 * RB);
    wait_vm<pp_vm(TN, 0, LEFT)>();
    FF_MEM_END();
#pragma unroll
    for (int i = 0; i < 2 * TN; ++i) FF_TIE(fb[i]);
    if (LEFT == 0 && kpad) {
#pragma unroll
      for (int i = 0; i < 2 * TN; ++i) cut(fb[i], i & 1);
    }
    FF_CUTA(fa[0]);
    FF_MMA(0, fa[0]);
    // phase 1
    FF_RDA(fa[1], 1 * PC);
    if (k2) {
      FF_DMA(rw, vob[0], OFFB + cb, kb + 2 * RB);
      FF_DMA(rw, vob[1], OFFB + PC + cb, kb + 2 * RB);
    }
    wait_vm<pp_vm(TN, 1, LEFT)>();
    FF_MEM_END();
    FF_TIEA(fa[1]);
    FF_CUTA(fa[1]);
    FF_MMA(1, fa[1]);
    // phase 2
    FF_RDA(fa[0], 2 * PC);
    if (k2) {
      FF_DMA(ra, voa[1], PC + ca, kb + 2 * RB);
      if (TN > 2) FF_DMA(rw, vob[TN > 2 ? 2 : 0], OFFB + 2 * PC + cb, kb + 2 * RB);
    }
    wait_vm<pp_vm(TN, 2, LEFT)>();
    FF_MEM_END();
    FF_TIEA(fa[0]);
    FF_CUTA(fa[0]);
    FF_MMA(2, fa[0]);
    // phase 3
    FF_RDA(fa[1], 3 * PC);
    rda[0] += oa - ca; rda[1] += oa - ca;
    rdb[0] += ob - cb; rdb[1] += ob - cb;
    if (k1) FF_RDA(fa[0], 0);
    if (k2) {
      FF_DMA(ra, voa[2], 2 * PC + ca, kb + 2 * RB);
      if (TN > 3) FF_DMA(rw, vob[TN > 3 ? 3 : 0], OFFB + 3 * PC + cb, kb + 2 * RB);
    }
    wait_vm<pp_vm(TN, 3, LEFT)>();
    FF_MEM_END();
    FF_TIEA(fa[1]);
    if (k1) { FF_TIEA(fa[0]); }
    FF_CUTA(fa[1]);
    FF_MMA(3, fa[1]);
    kb += RB;
    ca = oa;
    cb = ob;
  };
  // prologue: what the stages -2 and -1 would have issued, in that order
#pragma unroll
  for (int j = -2; j < 0; ++j)
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int pc = kPPIssue[q / 2][q % 2], st = pc == 3 ? j + 1 : j + 2;
      if (pc >= 4 + TN || st < 0) continue;
      if (pc < 4) FF_DMA(ra, voa[pc & 3], st * BUFA + pc * PC, st * RB);
      else FF_DMA(rw, vob[pc - 4 < TN ? pc - 4 : 0], OFFB + st * BUFB + (pc - 4) * PC, st * RB);
    }
  wait_vm<3 + TN>();   // stage 0 has landed, and stage 1 but for A3 is on its way
  asm volatile("s_barrier" ::: "memory");
  if (wave >= 4) asm volatile("s_barrier" ::: "memory");   // the second group runs half a phase behind
  FF_RDA(fa[0], 0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  FF_TIEA(fa[0]);
  for (int kt = 0; kt < nk - 3; ++kt) stage(Int<2>{});
  // the pieces issued from here on are the last stage's, but for A3 of the last but one
#pragma unroll
  for (int q = 0; q < 3; ++q) voa[q] -= back;
#pragma unroll
  for (int u = 0; u < TN; ++u) vob[u] -= back;
  stage(Int<2>{});
  voa[3] -= back;
  stage(Int<1>{});
  stage(Int<0>{});
  if (wave < 4) asm volatile("s_barrier" ::: "memory");
#undef FF_TIEA
#undef FF_CUTA
#undef FF_MEM_END
#undef FF_DMA
#undef FF_MMA
  // every wave's LDS reads and DMA ended before the last barrier
  epilogue_block<EPI, OUT_F32, RES_F32>(a, m0 + mw * 128, n0 + nw * WN, accs, smem + wave * 32 * (WN + 4) * 2);
#endif
}

// ------------------------------------------------------------------ bf16 MFMA GEMM, waves split K
// Small grids, where 256-row tiles would leave CUs idle: BM x BN tile, 64-wide stages, 8 waves on
// the two halves of the tile's rows and the four 16-wide k steps of a stage.
//
// What bounds it: the memory part of a half stage (fragment reads, DMA, waits and the barrier), one
// after the other; at long K on wide models also what the caches deliver.  A 128x96 stage takes 730
// cycles (0.307 us at 2.4 GHz), of which the MFMAs fill 386; by the counters the LDS is busy with
// fragment reads for 200, and the DMA writes 28 KB.  The kernel before it split K over two groups
// only and read a 32-row block at a time (950 cycles); deeper rings and prefetches into the L2 made
// that one slower, and fragments straight from memory (16 rows x 64 bytes per load) run at a quarter
// of the L1's rate.  Rings of four stages for 64x64 and 64x32, where five and six fit, are slower
// (DiT-XL/2 block of one image 58.6 -> 62.5 us).
// Alternation: waves 0-3 and 4-7, one of each per SIMD, run half a stage apart, a barrier after
// each half, so that one's MFMAs cover the other's fragment reads and DMA.  A stage's buffer is
// refilled from the slot after its last read on (NST - 1 stages ahead); a wave waits for its own
// DMA of the next stage before the barrier that precedes that stage's first read.  A DMA
// instruction fills 8 rows of 128 bytes, 16-byte chunks XOR-ed with row / 2 against bank conflicts.
// Measured against the former kernel's best tile, us: M = 2048 N = 1152 K = 4608 37.3 -> 29.7,
// K = 1152 15.4 -> 13.6; M = 256 K = 4608 26.7 -> 12.9; M = 1024 N = 3456 K = 1152 18.4 -> 14.1;
// M = 1536 N = 3072 K = 15360 203 -> 174 (128x192, against 256x128 tiles of the kernel above).
// SHORT: at most NST stages, all issued at once.
template <int BM, int BN, int NST, bool SHORT, int EPI, bool OUT_F32, bool RES_F32, int NP>
__global__ __launch_bounds__(512) void k_gemm_ks(GemmGroup<NP> G) {
#ifdef __HIP_DEVICE_COMPILE__   // the host pass needs the launch stub only
  constexpr int TM = BM / 64, TN = BN / 32, PN = BN <= 128 ? BN : BN / 2;   // PN: columns of an epilogue pass
  constexpr int RB = 128, STB = (BM + BN) * RB;   // bytes of a staged row, of a stage
  constexpr int LDR = PN + 4, kRed = 2 * BM * LDR * 4;
  static_assert(BM % 64 == 0 && PN % 32 == 0 && NST >= 3, "tile");
  __shared__ __attribute__((aligned(1024))) char smem[NST * STB > kRed ? NST * STB : kRed];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int tm, tn;
  const int prob = __builtin_amdgcn_readfirstlane(tile_of(blockIdx.x, G.tm[0], G.tn[0], G.tm[NP - 1], G.tn[NP - 1], NP, tm, tn));
  const GemmArgs a = (NP > 1 && prob) ? G.g[NP - 1] : G.g[0];
  const int m0 = __builtin_amdgcn_readfirstlane(tm) * BM, n0 = __builtin_amdgcn_readfirstlane(tn) * BN;
  const int half = wave & 1, kg = wave >> 1;   // this wave's rows of the tile and its k step of a stage
  const int nk = (a.K + 63) / 64, kpad = nk * 64 - a.K;
  const int fr = lane & 31, fh = lane >> 5;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) const void*)smem);
  const uint32_t chunk = (uint32_t)((2 * kg + fh) ^ ((fr >> 1) & 7)) * 16;
  uint32_t rda = lds0 + (half * (BM / 2) + fr) * RB + chunk, rdb = lds0 + (BM + fr) * RB + chunk;
  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  auto loop = [&](auto Gc) __attribute__((always_inline)) {
    constexpr int GRP = decltype(Gc)::value;              // waves 0-3 load the A rows, 4-7 the B rows
    constexpr int ROWS = GRP ? BN : BM, PER = ROWS / 32;  // DMA instructions of a wave and stage
    const int w4 = wave & 3;
    const int p0 = GRP ? 0 : a.amap.phys(m0);
    const char* base = GRP ? reinterpret_cast<const char*>(a.W) + (size_t)n0 * a.ldw * 2
                           : reinterpret_cast<const char*>(a.A) + (size_t)p0 * a.lda * 2;
    __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, 0xffffffffu, 0x00020000);
    uint32_t vo[PER], back[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int R = (w4 * PER + j) * 8 + (lane >> 3);
      const uint32_t ch = ((lane & 7) ^ ((R >> 1) & 7)) * 16;
      // rows past the matrix read the tile's first row (in bounds); their results are never stored
      if (GRP) vo[j] = (n0 + R < a.N ? (uint32_t)R * (uint32_t)a.ldw * 2u : 0u) + ch;
      else vo[j] = (m0 + R < a.M ? (uint32_t)(a.amap.phys(m0 + R) - p0) * (uint32_t)a.lda * 2u : 0u) + ch;
      // the last stage's chunks past K load the row's chunk 0 of that stage (in bounds) and are zeroed when read
      back[j] = (kpad && ch >= (uint32_t)(64 - kpad) * 2u) ? ch : 0u;
    }
    char* const dst0 = smem + (GRP ? BM * RB : 0) + w4 * PER * 1024;
    int kb = 0, ib = 0;   // the next stage to issue: byte offset along K, and its buffer
    auto issue = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < PER; ++j)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, FF_AS3(dst0 + ib + j * 1024), 16, vo[j], kb, 0, 0);
      kb += RB;
      ib = ib == (NST - 1) * STB ? 0 : ib + STB;
    };
    bf16x8_t fa[TM], fb[TN];
    int cb = 0;
    // the memory part of a stage; VM: DMAs of later stages that may stay outstanding
    auto mem = [&](bool more, bool last, auto VMc) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < TM; ++t) fa[t] = lds_rd128_off(rda, t * 32 * RB);
#pragma unroll
      for (int t = 0; t < TN; ++t) fb[t] = lds_rd128_off(rdb, t * 32 * RB);
      if (more) issue();
      const int step = cb == (NST - 1) * STB ? -(NST - 1) * STB : STB;
      cb += step;
      rda += step;
      rdb += step;
      wait_vm<decltype(VMc)::value>();
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
      for (int t = 0; t < TM; ++t) FF_TIE(fa[t]);
#pragma unroll
      for (int t = 0; t < TN; ++t) FF_TIE(fb[t]);
      if (last && kpad) {   // both operands, so that 0 * 0 is added
        const bool in = (2 * kg + fh) * 8 < 64 - kpad;
        auto cut = [&](bf16x8_t& f) __attribute__((always_inline)) {
          u32x4_t w = __builtin_bit_cast(u32x4_t, f);
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = in ? w[e] : 0u;
          f = __builtin_bit_cast(bf16x8_t, w);
        };
#pragma unroll
        for (int t = 0; t < TM; ++t) cut(fa[t]);
#pragma unroll
        for (int t = 0; t < TN; ++t) cut(fb[t]);
      }
    };
    auto mma = [&]() __attribute__((always_inline)) {
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_barrier" ::: "memory");
    };
#define FF_KS_BACK() do { _Pragma("unroll") for (int j = 0; j < PER; ++j) vo[j] -= back[j]; } while (0)
    if constexpr (SHORT) {   // nk <= NST (host check): every stage has a buffer of its own
      for (int kt = 0; kt < nk - 1; ++kt) issue();
      FF_KS_BACK();
      issue();
      wait_vm<0>();
      asm volatile("s_barrier" ::: "memory");
      if (GRP) asm volatile("s_barrier" ::: "memory");   // the second group runs half a stage behind
      for (int kt = 0; kt < nk; ++kt) {
        mem(false, kt == nk - 1, Int<0>{});
        mma();
      }
    } else {   // nk >= NST (host check): the prologue's stages are none of them the last
#pragma unroll
      for (int s = 0; s < NST - 1; ++s) issue();
      wait_vm<(NST - 2) * PER>();
      asm volatile("s_barrier" ::: "memory");
      if (GRP) asm volatile("s_barrier" ::: "memory");   // the second group runs half a stage behind
      for (int kt = 0; kt < nk - NST; ++kt) {
        mem(true, false, Int<(NST - 2) * PER>{});
        mma();
      }
      FF_KS_BACK();
      mem(true, false, Int<(NST - 2) * PER>{});   // issues the last stage
      mma();
      static_for<0, NST - 1>([&](auto ic) __attribute__((always_inline)) {
        constexpr int later = NST - 3 - decltype(ic)::value;
        mem(false, decltype(ic)::value == NST - 2, Int<(later > 0 ? later : 0) * PER>{});
        mma();
      });
    }
    if (!GRP) asm volatile("s_barrier" ::: "memory");
#undef FF_KS_BACK
  };
  if (wave < 4) loop(Int<0>{});
  else loop(Int<1>{});
  // every wave's LDS reads and DMA ended before the last barrier

  // The four k steps' sums meet in LDS, PN columns at a time: 2 and 3 go to 0 and 1, then those
  // two, from which each thread finishes pieces of 8 columns of a row.
  constexpr int CPR = PN / 8, UNITS = BM * CPR, UPT = (UNITS + 511) / 512, TP = PN / 32;
  constexpr bool kCache = EPI == EPI_GATED && !OUT_F32;
  const bool want_u = kCache && a.cache_out && a.cache_u;
  const bool gelu = EPI == EPI_BIAS_GELU || (EPI == EPI_BIAS_OR_GELU && a.epi == EPI_BIAS_GELU);
  float* const red = reinterpret_cast<float*>(smem) + (kg & 1) * BM * LDR + (half * (BM / 2) + fr) * LDR + 4 * fh;
  static_for<0, BN / PN>([&](auto passc) __attribute__((always_inline)) {
    constexpr int J0 = decltype(passc)::value * TP;
    u32x4_t bias[UPT], resb[UPT], uu[UPT];
    f32x4_t resf[UPT][2], gate[UPT][2];
    size_t po[UPT];
    bool ok[UPT];
    auto request = [&]() __attribute__((always_inline)) {   // what the pass needs from memory
#pragma unroll
      for (int q = 0; q < UPT; ++q) {
        const int p = q * 512 + threadIdx.x, r = m0 + p / CPR, c = n0 + J0 * 32 + p % CPR * 8;
        ok[q] = p < UNITS && r < a.M && c < a.N;   // N % 8 == 0: a piece is in range as a whole
        const int rr = ok[q] ? r : m0, cc = ok[q] ? c : n0;
        const size_t pr = (size_t)a.omap.phys(rr);
        po[q] = pr * a.ldo + cc;
        bias[q] = *reinterpret_cast<const u32x4_t*>(reinterpret_cast<const uint16_t*>(a.bias) + cc);
        if (EPI == EPI_GATED) {
          if (RES_F32) {
            const float* rp = reinterpret_cast<const float*>(a.resid) + pr * a.ldr + cc;
            resf[q][0] = *reinterpret_cast<const f32x4_t*>(rp);
            resf[q][1] = *reinterpret_cast<const f32x4_t*>(rp + 4);
          } else {
            resb[q] = *reinterpret_cast<const u32x4_t*>(reinterpret_cast<const uint16_t*>(a.resid) + pr * a.ldr + cc);
          }
          const float* gp = a.gate + (size_t)a.omap.sample(rr) * a.ldg + cc;
          gate[q][0] = *reinterpret_cast<const f32x4_t*>(gp);
          gate[q][1] = *reinterpret_cast<const f32x4_t*>(gp + 4);
        }
        if (want_u) uu[q] = *reinterpret_cast<const u32x4_t*>(reinterpret_cast<const uint16_t*>(a.cache_u) + po[q]);
      }
    };
    auto put = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TP; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            *reinterpret_cast<f32x4_t*>(red + i * 32 * LDR + j * 32 + 8 * v) =
                f32x4_t{acc[i][J0 + j][4 * v], acc[i][J0 + j][4 * v + 1], acc[i][J0 + j][4 * v + 2], acc[i][J0 + j][4 * v + 3]};
    };
    // the loads come before the exchange where the registers allow
    if (BN == PN) request();
    if (J0) __syncthreads();   // the last pass's reads
    if (kg >= 2) put();
    __syncthreads();
    if (kg < 2) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TP; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const f32x4_t p = *reinterpret_cast<const f32x4_t*>(red + i * 32 * LDR + j * 32 + 8 * v);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][J0 + j][4 * v + e] += p[e];
          }
      put();   // where this lane alone has read
    }
    if (BN != PN) request();
    __syncthreads();
#pragma unroll
    for (int q = 0; q < UPT; ++q) {
      if (!ok[q]) continue;
      const int p = q * 512 + threadIdx.x;
      const float* l = reinterpret_cast<const float*>(smem) + (p / CPR) * LDR + p % CPR * 8;
      float v[8];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const f32x4_t x = *reinterpret_cast<const f32x4_t*>(l + 4 * h), y = *reinterpret_cast<const f32x4_t*>(l + BM * LDR + 4 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * h + e] = x[e] + y[e];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[e] += __uint_as_float(e & 1 ? bias[q][e / 2] & 0xffff0000u : bias[q][e / 2] << 16);
        if (gelu) v[e] = gelu_tanh_f(v[e]);
        if (EPI == EPI_GATED) {
          const float rs = RES_F32 ? resf[q][e / 4][e % 4] : __uint_as_float(e & 1 ? resb[q][e / 2] & 0xffff0000u : resb[q][e / 2] << 16);
          v[e] = rs + gate[q][e / 4][e % 4] * v[e];
        }
      }
      if (OUT_F32) {
        St<DT_F32>::store(a.out, po[q], v);
        St<DT_F32>::store(a.out, po[q] + 4, v + 4);
        continue;
      }
      St<DT_BF16>::store(a.out, po[q], v);
      if (kCache && a.cache_out) {   // history refresh from the stored (rounded) output
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          v[e] = St<DT_BF16>::rnd(v[e]);
          if (want_u) v[e] -= __uint_as_float(e & 1 ? uu[q][e / 2] & 0xffff0000u : uu[q][e / 2] << 16);
        }
        St<DT_BF16>::store(a.cache_out, po[q], v);
      }
    }
  });
#endif
}

// ------------------------------------------------------------------ fp32 GEMM
// v_mfma_f32_16x16x4 / 32x32x2 (fp32 in, fp32 accumulation): the card's fp32 rate with a
// fraction of the operand traffic of plain FMAs.  The A operand holds weight rows (output
// columns n), the B operand activation rows m, so that a lane holds 4 consecutive columns of
// one output row.  Both operands take the same k for the same (lane group, step), in any order:
// a lane's 16-byte chunk of 4 consecutive k feeds 4 steps.

// 4 consecutive columns c.. of output row r
template <int EPI>
__device__ __forceinline__ void store4_f32(const GemmArgs& a, int r, int c, f32x4_t v) {
  const f32x4_t b = *reinterpret_cast<const f32x4_t*>(reinterpret_cast<const float*>(a.bias) + c);
  const size_t pr = (size_t)a.omap.phys(r);
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] += b[e];
  if (EPI == EPI_BIAS_GELU) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = gelu_tanh_f(v[e]);
  }
  if (EPI == EPI_GATED) {
    const f32x4_t rs = *reinterpret_cast<const f32x4_t*>(reinterpret_cast<const float*>(a.resid) + pr * a.ldr + c);
    const f32x4_t g = *reinterpret_cast<const f32x4_t*>(a.gate + (size_t)a.omap.sample(r) * a.ldg + c);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = rs[e] + g[e] * v[e];
  }
  *reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(a.out) + pr * a.ldo + c) = v;
}

// Small grids: a 16 x 16 output tile per workgroup, its 8 waves on interleaved 16-wide blocks of
// k, operands straight from memory into registers with up to 16 loads in flight, so that K =
// 1024 costs one memory round trip; the waves' sums are added in wave order through LDS.
template <int EPI>
__global__ __launch_bounds__(512) void k_gemm_f32_small(GemmArgs a) {
  constexpr int U = 8;   // k blocks in flight per wave
  __shared__ f32x4_t red[8][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tiles_n = (a.N + 15) / 16;
  const int m0 = (blockIdx.x / tiles_n) * 16, n0 = (blockIdx.x % tiles_n) * 16;
  const int i16 = lane & 15, g = lane >> 4;
  const int m = m0 + i16 < a.M ? m0 + i16 : m0, n = n0 + i16 < a.N ? n0 + i16 : n0;   // past the matrix: never stored
  const float* pa = reinterpret_cast<const float*>(a.A) + (size_t)a.amap.phys(m) * a.lda + 4 * g;
  const float* pw = reinterpret_cast<const float*>(a.W) + (size_t)n * a.ldw + 4 * g;
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  const f32x4_t z = acc;
  for (int k0 = wave * 16; k0 < a.K; k0 += 8 * 16 * U) {
    f32x4_t x[U], w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + u * 128;
      const bool in = k + 4 * g < a.K;
      x[u] = in ? *reinterpret_cast<const f32x4_t*>(pa + k) : z;
      w[u] = in ? *reinterpret_cast<const f32x4_t*>(pw + k) : z;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k0 + u * 128 >= a.K) break;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][e], x[u][e], acc, 0, 0, 0);
    }
  }
  red[wave][lane] = acc;
  __syncthreads();
  if (wave) return;
#pragma unroll
  for (int i = 1; i < 8; ++i) {
    const f32x4_t p = red[i][lane];
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] += p[e];
  }
  if (m0 + i16 < a.M && n0 + 4 * g < a.N) store4_f32<EPI>(a, m0 + i16, n0 + 4 * g, acc);
}

// T x T output tile (32 or 64), 8 waves: T/32 x T/32 blocks of 32 x 32, KG groups of waves on
// the k steps of a BK-wide stage; operands by DMA into a ring of four stages (rows of 128 or
// 256 bytes, 16-byte chunks rotated by the row against bank conflicts).  Two workgroups share a
// CU, so one's MFMAs cover the other's waits.  K % BK != 0: the last stage's chunks past K
// load the row's first chunk of that stage (in bounds) and are zeroed after the LDS read.
template <int T, int EPI>
__global__ __launch_bounds__(512) void k_gemm_f32(GemmArgs a) {
#ifdef __HIP_DEVICE_COMPILE__   // the host pass needs the launch stub only
  constexpr int NB = T / 32, KG = 8 / (NB * NB), BK = 8 * (KG < 4 ? 4 : KG), SUB = BK / 8 / KG, NST = 4;
  constexpr int CH = BK / 4, RPI = 64 / CH, DPW = 2 * T / RPI / 8;   // chunks per row, rows and instructions per wave
  constexpr int ROWS = 2 * T, STB = ROWS * BK * 4;
  static_assert(DPW == 2 && SUB * KG * 8 == BK, "two DMA instructions per wave and stage");
  __shared__ __attribute__((aligned(1024))) char smem[NST * STB];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tiles_n = (a.N + T - 1) / T;
  const int m0 = (blockIdx.x / tiles_n) * T, n0 = (blockIdx.x % tiles_n) * T;
  const int blk = wave % (NB * NB), grp = wave / (NB * NB);
  auto swz = [](int row) { return CH == 16 ? (row & 15) : ((row >> 1) & 7); };
  const int nk = (a.K + BK - 1) / BK, kpad = nk * BK - a.K;
  // rows 0 .. T-1 of a stage are activation rows, T .. 2T-1 weight rows
  const char* src[DPW];
  int back[DPW];
#pragma unroll
  for (int j = 0; j < DPW; ++j) {
    const int R = (wave * DPW + j) * RPI + lane / CH, c = (lane % CH) ^ swz(R);
    if (R < T) {
      const int m = m0 + R < a.M ? m0 + R : m0;
      src[j] = reinterpret_cast<const char*>(reinterpret_cast<const float*>(a.A) + (size_t)a.amap.phys(m) * a.lda + c * 4);
    } else {
      const int n = n0 + R - T < a.N ? n0 + R - T : n0;
      src[j] = reinterpret_cast<const char*>(reinterpret_cast<const float*>(a.W) + (size_t)n * a.ldw + c * 4);
    }
    back[j] = c * 4 >= BK - kpad ? c * 16 : 0;
  }
  auto issue = [&](int kt) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < DPW; ++j) {
      const char* p = src[j] + (size_t)kt * BK * 4 - (kt == nk - 1 ? back[j] : 0);
      __builtin_amdgcn_global_load_lds(FF_AS1(p), FF_AS3(smem + (kt % NST) * STB + (wave * DPW + j) * 1024), 16, 0, 0);
    }
  };
  f32x16_t acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  const int fr = lane & 31, fh = lane >> 5;
  const int ra = (blk / NB) * 32 + fr, rw = T + (blk % NB) * 32 + fr;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) const void*)smem);
#pragma unroll
  for (int s = 0; s < NST - 1; ++s)
    if (s < nk) issue(s);
  for (int kt = 0; kt < nk; ++kt) {
    const int later = nk - 1 - kt;   // stages issued after this one: min(later, 2)
    if (later >= 2) wait_vm<2 * DPW>();
    else if (later == 1) wait_vm<DPW>();
    else wait_vm<0>();
    asm volatile("s_barrier" ::: "memory");   // stage kt is in; every wave is done with stage kt - 1
    if (kt + NST - 1 < nk) issue(kt + NST - 1);
    const uint32_t st = lds0 + (kt % NST) * STB;
    bf16x8_t xa[SUB], xw[SUB];
#pragma unroll
    for (int s = 0; s < SUB; ++s) {
      const int c = (grp * SUB + s) * 2 + fh;
      xa[s] = lds_rd128_off(st + ra * BK * 4 + ((c ^ swz(ra)) * 16), 0);
      xw[s] = lds_rd128_off(st + rw * BK * 4 + ((c ^ swz(rw)) * 16), 0);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int s = 0; s < SUB; ++s) { FF_TIE(xa[s]); FF_TIE(xw[s]); }
#pragma unroll
    for (int s = 0; s < SUB; ++s) {
      f32x4_t fa = __builtin_bit_cast(f32x4_t, xa[s]), fw = __builtin_bit_cast(f32x4_t, xw[s]);
      if (kt == nk - 1 && ((grp * SUB + s) * 2 + fh) * 4 >= BK - kpad) {
        fa = f32x4_t{0.f, 0.f, 0.f, 0.f};
        fw = fa;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fw[e], fa[e], acc, 0, 0, 0);
    }
  }
  __syncthreads();   // the ring is free
  if (KG > 1) {
    float* red = reinterpret_cast<float*>(smem) + lane;
    if (grp > 0) {
#pragma unroll
      for (int v = 0; v < 16; ++v) red[(((grp - 1) * NB * NB + blk) * 16 + v) * 64] = acc[v];
    }
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int i = 0; i < KG - 1; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] += red[((i * NB * NB + blk) * 16 + v) * 64];
  }
  const int r = m0 + (blk / NB) * 32 + fr;
  if (r >= a.M) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = n0 + (blk % NB) * 32 + 8 * q + 4 * fh;
    if (c < a.N) store4_f32<EPI>(a, r, c, f32x4_t{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]});
  }
#endif
}

// The 16 x 16 tiles up to 512 of them (M = 64, N = 256, K = 1024: 6.0 us against 10.1 with 32 x 32
// and 28 with 64 x 64 tiles; 512 x 384 x 384, 768 tiles: 6.3 against 6.0).  Against the kernel
// these replaced (64 x 64 tiles of plain FMAs): M = 64, N = 256, K = 1024 76 -> 6 us, M = 512,
// N = 4608, K = 1152 202 -> 75 us.
template <int EPI>
void launch_f32(const GemmArgs& a, hipStream_t s) {
  const long t16 = (long)((a.M + 15) / 16) * ((a.N + 15) / 16), t32 = (long)((a.M + 31) / 32) * ((a.N + 31) / 32);
  const long t64 = (long)((a.M + 63) / 64) * ((a.N + 63) / 64);
  // 64 x 64 tiles take 6 + 25 us per round of 256 at K = 1152 (31 us for 72 or 216 tiles, 51 for
  // 288 or 432, 75 for 576), 32 x 32 tiles 8 us + 0.035 us each (20 us for 288, 38 for 864)
  const double c64 = 0.24 + (double)((t64 + 255) / 256), c32 = 0.32 + t32 / 714.0;
  if (t16 <= 512) FF_LAUNCH(k_gemm_f32_small<EPI>, t16, 512, 0, s, a);
  else if (c32 < c64) FF_LAUNCH((k_gemm_f32<32, EPI>), t32, 512, 0, s, a);
  else FF_LAUNCH((k_gemm_f32<64, EPI>), t64, 512, 0, s, a);
}

template <int BM, int BN, int NP>
GemmGroup<NP> make_group(const GemmArgs* a, int& nwg) {
  GemmGroup<NP> G{};
  nwg = 0;
  for (int i = 0; i < NP; ++i) {
    G.g[i] = a[i];
    G.tm[i] = (a[i].M + BM - 1) / BM;
    G.tn[i] = (a[i].N + BN - 1) / BN;
    nwg += G.tm[i] * G.tn[i];
  }
  return G;
}

// What the two streams of a block, or the two parts of a single block's first projection, share
constexpr bool grouped_epi(int epi, bool of, bool rf) { return epi == EPI_GATED ? of != rf : !of && !rf; }

// One problem, or two (only those pairs that the path groups are built)
#define FF_LAUNCH_GEMM(BM, BN, THREADS, ...)                                       \
  do {                                                                             \
    int nwg;                                                                       \
    if (n == 1) {                                                                  \
      if constexpr (EPI != EPI_BIAS_OR_GELU) {                                     \
        const GemmGroup<1> G = make_group<BM, BN, 1>(a, nwg);                      \
        FF_LAUNCH((__VA_ARGS__, EPI, OF, RF, 1>), nwg, THREADS, 0, s, G);          \
      }                                                                            \
    } else {                                                                       \
      if constexpr (grouped_epi(EPI, OF, RF)) {                                    \
        const GemmGroup<2> G = make_group<BM, BN, 2>(a, nwg);                      \
        FF_LAUNCH((__VA_ARGS__, EPI, OF, RF, 2>), nwg, THREADS, 0, s, G);          \
      }                                                                            \
    }                                                                              \
  } while (0)

template <int TN, int EPI, bool OF, bool RF>
void launch_pp(const GemmArgs* a, int n, hipStream_t s) { FF_LAUNCH_GEMM(256, 64 * TN, 512, k_gemm_pp<TN); }

template <int BM, int BN, int NST, bool SHORT, int EPI, bool OF, bool RF>
void launch_ks(const GemmArgs* a, int n, hipStream_t s) { FF_LAUNCH_GEMM(BM, BN, 512, k_gemm_ks<BM, BN, NST, SHORT); }

template <int EPI, bool OF, bool RF>
void launch_reg(const GemmArgs* a, int n, hipStream_t s) { FF_LAUNCH_GEMM(128, 128, 512, k_gemm_bf16<128, 128, 64, 32); }

GemmShape shape_of(const GemmArgs& a) { return GemmShape{a.M, a.N, a.K, a.lda, a.ldw, a.amap.n_seg, a.amap.N}; }

template <int EPI, bool OF, bool RF>
void launch_bf16(const GemmArgs* a, int n, hipStream_t s) {
  const GemmShape sh[2] = {shape_of(a[0]), shape_of(a[n - 1])};
  const int nk = min_stages(sh, n);
  switch (plan_tiles(sh, n).tile) {
    case kTileShort64: launch_ks<64, 64, kShortStages, true, EPI, OF, RF>(a, n, s); break;
    case kTileShort64x32: launch_ks<64, 32, kShortStages, true, EPI, OF, RF>(a, n, s); break;
    case kTile256: launch_pp<4, EPI, OF, RF>(a, n, s); break;
    case kTile256x192: launch_pp<3, EPI, OF, RF>(a, n, s); break;
    case kTile256x128: launch_pp<2, EPI, OF, RF>(a, n, s); break;
    case kTile128x192: launch_ks<128, 192, 4, false, EPI, OF, RF>(a, n, s); break;
    case kTile128: launch_ks<128, 128, 5, false, EPI, OF, RF>(a, n, s); break;
    case kTile128x96: launch_ks<128, 96, 4, false, EPI, OF, RF>(a, n, s); break;
    case kTile128x64: launch_ks<128, 64, 4, false, EPI, OF, RF>(a, n, s); break;
    case kTile64x96: launch_ks<64, 96, 4, false, EPI, OF, RF>(a, n, s); break;
    case kTile64:   // fewer buffers where there are fewer stages
      if (nk >= 5) launch_ks<64, 64, 5, false, EPI, OF, RF>(a, n, s);
      else launch_ks<64, 64, 4, false, EPI, OF, RF>(a, n, s);
      break;
    case kTile64x32:
      if (nk >= 6) launch_ks<64, 32, 6, false, EPI, OF, RF>(a, n, s);
      else launch_ks<64, 32, 4, false, EPI, OF, RF>(a, n, s);
      break;
    default: launch_reg<EPI, OF, RF>(a, n, s); break;
  }
}

}  // namespace

namespace {

// bf16 dispatch of n (1 or 2) problems that share epilogue, output and residual types
hipError_t gemm_bf16(const GemmArgs* a, int n, hipStream_t s) {
  const bool of = a[0].out_f32 != 0, rf = a[0].resid_f32 != 0;
  if (n == 2 && a[0].epi != a[1].epi) launch_bf16<EPI_BIAS_OR_GELU, false, false>(a, n, s);   // bias with bias+GELU
  else if (a[0].epi == EPI_BIAS && of) launch_bf16<EPI_BIAS, true, false>(a, n, s);
  else if (a[0].epi == EPI_BIAS) launch_bf16<EPI_BIAS, false, false>(a, n, s);
  else if (a[0].epi == EPI_BIAS_GELU && !of) launch_bf16<EPI_BIAS_GELU, false, false>(a, n, s);
  else if (a[0].epi == EPI_GATED && of && !rf) launch_bf16<EPI_GATED, true, false>(a, n, s);
  else if (a[0].epi == EPI_GATED && !of && rf) launch_bf16<EPI_GATED, false, true>(a, n, s);
  else if (a[0].epi == EPI_GATED && !of) launch_bf16<EPI_GATED, false, false>(a, n, s);
  else return hipErrorInvalidValue;   // no part of the path asks for it
  return hipGetLastError();
}

}  // namespace

hipError_t gemm(int dtype, const GemmArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  if (dtype == DT_F32) {
    switch (a.epi) {
      case EPI_BIAS: launch_f32<EPI_BIAS>(a, s); break;
      case EPI_BIAS_GELU: launch_f32<EPI_BIAS_GELU>(a, s); break;
      default: launch_f32<EPI_GATED>(a, s); break;
    }
    return hipGetLastError();
  }
  return gemm_bf16(&a, 1, s);
}

hipError_t gemm2(int dtype, const GemmArgs& a0, const GemmArgs& a1, hipStream_t s) {
  const bool e0 = a0.M > 0 && a0.N > 0, e1 = a1.M > 0 && a1.N > 0;
  const bool ungated = a0.epi != EPI_GATED && a1.epi != EPI_GATED;
  const bool same = (a0.epi == a1.epi || ungated) && a0.out_f32 == a1.out_f32 && a0.resid_f32 == a1.resid_f32;
  const bool built = grouped_epi(a0.epi, a0.out_f32 != 0, a0.resid_f32 != 0);
  if (dtype == DT_F32 || !same || !built || !e0 || !e1 || !plan_grouped(shape_of(a0), shape_of(a1))) {
    hipError_t e = gemm(dtype, a0, s);
    return e != hipSuccess ? e : gemm(dtype, a1, s);
  }
  const GemmArgs both[2] = {a0, a1};
  return gemm_bf16(both, 2, s);
}

}  // namespace ff
