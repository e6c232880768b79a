// Dense contractions of the exact block: out = epi(A W^T + bias) with A [M, K] (rows
// through a RowMap), W [N, K] (both K-contiguous), fp32 accumulation.
//
// bf16: 256-row workgroup tiles of v_mfma_f32_16x16x32_bf16 (k_gemm_pp) where the grid fills
// the card or K % 64 != 0, 128-row tiles of v_mfma_f32_32x32x16_bf16 (k_gemm_dl) on small
// grids.  Both stream operands global -> LDS directly; a register-staged kernel (padded LDS
// rows, double buffer) covers K <= 128 off the 64 grid (the patch embedding).
// fp32: fp32 MFMAs on 16x16, 32x32 or 64x64 tiles, the waves of a tile splitting K.
#include <algorithm>
#include "dev_common.h"

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
// Register-staged fallback (K % 32 != 0): BM x BN workgroup tile, BK = 64 per LDS stage
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
// ------------------------------------------------------------------ bf16 MFMA GEMM, direct-to-LDS
// For K % BKd == 0 (BKd = 32 or 64).  Operand tiles go global -> LDS with
// global_load_lds_dwordx4 (no VGPR staging, no ds_write), into an NST-stage ring of
// BKd-wide K slices issued NST-1 slices ahead.  Each DMA instruction fills 1 KB of LDS in
// lane order (16 rows x 64 bytes, or 8 rows x 128 bytes), so rows cannot be padded;
// instead lane l of a row loads a 16-byte chunk XOR-swizzled by the row ((l%4) ^
// ((row>>2)&3), or (l%8) ^ ((row>>1)&7)), which keeps the fragment reads free of bank
// conflicts: a 16-row group of a read spreads over all 64 banks.  (With 128-byte rows, even
// rows sit on banks 0-31 and odd rows on 32-63, so the 64-wide swizzle takes row/2; the
// first version used row&7, which put rows r and r+8 on the same banks.)
//
// Synchronisation is explicit: the compiler's barrier lowering waits for ALL outstanding
// loads (it cannot tell which stage a DMA targets), which would remove the prefetch.  So a
// stage boundary waits only for the next stage (s_waitcnt vmcnt(n) with the later stages
// still in flight) and then s_barrier, as one volatile asm that is also a compiler memory
// barrier.  Fragments are double-buffered in registers across the 16-wide k steps: the
// reads of the next step (ds_read_b128 asm) are in flight while the MFMAs of the current
// one run, each step waits with lgkmcnt(TM+TN) for the older reads only, and volatile "+v"
// asms tie the fragments to the MFMAs so that none is consumed before its wait.  The one
// barrier per stage sits between its last k step and the next stage's first.
//
// KG = 2 doubles the waves without growing the tile: waves w and w + NW accumulate the
// same output block, the first over k steps 0-1 of every 64-wide stage and the second
// over steps 2-3 (only the first issues the DMA; the second's vmcnt waits pass at once and
// the stage barrier orders it).  With two waves per SIMD, one wave's LDS reads and barrier
// waits hide behind the other's MFMAs.  After the loop the second k group hands its fp32
// sums to the first through LDS (a fixed order: group 0 + group 1), which runs the epilogue.
// Wait until at most later * PER of this wave's DMA instructions are outstanding, then
// barrier.  A later beyond the cases waits for more than needed, which is safe.
template <int PER>
__device__ __forceinline__ void wait_stage(int later) {
  static_assert(3 * PER <= 63, "vmcnt field");
  switch (later) {
    case 0: asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory"); break;
    case 1: asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(PER) : "memory"); break;
    case 2: asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * PER) : "memory"); break;
    default: asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(3 * PER) : "memory"); break;
  }
}

template <int BM, int BN, int WM, int WN, int NST, int EPI, bool OUT_F32, bool RES_F32, int NP>
__global__ __launch_bounds__(2 * (BM / WM) * (BN / WN) * 64) void k_gemm_dl(GemmGroup<NP> G) {
  constexpr int BKd = 64, KG = 2;
  constexpr int AUX = BN == 64 ? 0 : 17;   // sc0|sc1: skips the L1 (each tile streams its panels once)
  constexpr int NWN = BN / WN;
  constexpr int NW = (BM / WM) * NWN;                            // output blocks (waves per k group)
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int CH = BKd / 8, RPI = 64 / CH, KS = BKd / 16;   // chunks per row, rows per DMA, k steps
  constexpr int KPG = KS / KG;                                   // k steps per stage of one k group
  constexpr int IA = BM / RPI / NW, IB = BN / RPI / NW;        // DMA instructions per wave per stage
  static_assert(BKd == 32 || BKd == 64, "stage width");
  static_assert((KG == 1 || KG == 2) && KPG % 2 == 0, "k groups take an even number of k steps");
  static_assert(IA * RPI * NW == BM && IB * RPI * NW == BN, "every tile row loaded by one DMA lane");
  static_assert(NST >= 3 && NST <= 5 && TM + TN <= 15, "unsupported tile");
  constexpr int kMain = NST * (BM + BN) * BKd, kEpi = epi_lds_elems<NW, WN>();
  constexpr int kRed = KG > 1 ? NW * TM * TN * 16 * 64 * 2 : 0;   // k group 1's partial sums (fp32)
  __shared__ __attribute__((aligned(1024))) uint16_t smem[kMain > kEpi + kRed ? kMain : kEpi + kRed];
  uint16_t (*sA)[BM * BKd] = reinterpret_cast<uint16_t (*)[BM * BKd]>(smem);
  uint16_t (*sB)[BN * BKd] = reinterpret_cast<uint16_t (*)[BN * BKd]>(smem + NST * BM * BKd);
  // wave index in a scalar register: the per-wave LDS addresses of the DMA (M0) are then
  // computed on the scalar unit instead of with a v_readfirstlane per instruction.  With
  // KG = 2, waves w and w + NW own the same output block (cw) and split every stage's k
  // steps between them (k group grp); only k group 0 issues the DMA.
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = KG > 1 ? wave / NW : 0, cw = KG > 1 ? wave % NW : wave;
  int tm, tn;
  // workgroup-uniform: keep the problem select and tile origin in scalar registers
  const int prob = __builtin_amdgcn_readfirstlane(tile_of(blockIdx.x, G.tm[0], G.tn[0], G.tm[NP - 1], G.tn[NP - 1], NP, tm, tn));
  tm = __builtin_amdgcn_readfirstlane(tm);
  tn = __builtin_amdgcn_readfirstlane(tn);
  const GemmArgs a = (NP > 1 && prob) ? G.g[NP - 1] : G.g[0];
  const int m0 = tm * BM, n0 = tn * BN;
  const uint16_t* A = reinterpret_cast<const uint16_t*>(a.A);
  const uint16_t* W = reinterpret_cast<const uint16_t*>(a.W);
  auto swz = [](int ch, int row) { return BKd == 64 ? (ch ^ ((row >> 1) & 7)) : (ch ^ ((row >> 2) & 3)); };
  // rows past the matrix read row 0 (in bounds); their results are never stored
  const int lr = lane / CH, ls = lane % CH;
  size_t ga[IA], gb[IB];
#pragma unroll
  for (int j = 0; j < IA; ++j) {
    const int row = (cw * IA + j) * RPI + lr, gm = m0 + row;
    ga[j] = (size_t)a.amap.phys(gm < a.M ? gm : 0) * a.lda + swz(ls, row) * 8;
  }
#pragma unroll
  for (int j = 0; j < IB; ++j) {
    const int row = (cw * IB + j) * RPI + lr, gn = n0 + row;
    gb[j] = (size_t)(gn < a.N ? gn : 0) * a.ldw + swz(ls, row) * 8;
  }
#define FF_ISSUE(st, k0)                                                                                  \
  do {                                                                                                    \
    if (KG == 1 || grp == 0) {                                                                            \
      _Pragma("unroll") for (int j = 0; j < IA; ++j)                                                      \
        __builtin_amdgcn_global_load_lds(FF_AS1(A + ga[j] + (k0)), FF_AS3(&sA[st][(cw * IA + j) * RPI * BKd]), 16, 0, AUX); \
      _Pragma("unroll") for (int j = 0; j < IB; ++j)                                                      \
        __builtin_amdgcn_global_load_lds(FF_AS1(W + gb[j] + (k0)), FF_AS3(&sB[st][(cw * IB + j) * RPI * BKd]), 16, 0, AUX); \
    }                                                                                                     \
  } while (0)

  Acc32<TM, TN> accs;
  f32x16_t (&acc)[TM][TN] = accs.t;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  const int wm = (cw / NWN) * WM, wn = (cw % NWN) * WN;
  const int fr = lane & 31, fh = lane >> 5;
  // fragment offsets within a stage for this k group's 16-wide k steps
  int offa[KPG][TM], offb[KPG][TN];
#pragma unroll
  for (int kk = 0; kk < KPG; ++kk) {
    const int ks = grp * KPG + kk;
#pragma unroll
    for (int t = 0; t < TM; ++t) {
      const int row = wm + t * 32 + fr;
      offa[kk][t] = row * BKd + swz(ks * 2 + fh, row) * 8;
    }
#pragma unroll
    for (int t = 0; t < TN; ++t) {
      const int row = wn + t * 32 + fr;
      offb[kk][t] = row * BKd + swz(ks * 2 + fh, row) * 8;
    }
  }
  const int nk = a.K / BKd;
#pragma unroll
  for (int s = 0; s < NST - 1; ++s)
    if (s < nk) FF_ISSUE(s, s * BKd);
  wait_stage<IA + IB>(min(NST - 2, nk - 1));   // stage 0 landed
  bf16x8_t fa[2][TM], fb[2][TN];
#pragma unroll
  for (int t = 0; t < TM; ++t) fa[0][t] = lds_rd128(&sA[0][offa[0][t]]);
#pragma unroll
  for (int t = 0; t < TN; ++t) fb[0][t] = lds_rd128(&sB[0][offb[0][t]]);
  for (int kt = 0; kt < nk; ++kt) {
    const int st = kt % NST;
#pragma unroll
    for (int s = 0; s < KPG; ++s) {
      const int cur = s & 1, nxt = cur ^ 1;   // KPG is even: stage k step 0 is always buffer 0
      if (s + 1 < KPG) {
#pragma unroll
        for (int t = 0; t < TM; ++t) fa[nxt][t] = lds_rd128(&sA[st][offa[s + 1][t]]);
#pragma unroll
        for (int t = 0; t < TN; ++t) fb[nxt][t] = lds_rd128(&sB[st][offb[s + 1][t]]);
        asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(TM + TN) : "memory");
      } else if (kt + 1 < nk) {
        // stage kt+1 complete everywhere, and every wave is past its reads of stage kt-1,
        // whose buffer now takes stage kt+NST-1; then the first k step of stage kt+1 is
        // read while the last one of stage kt computes
        wait_stage<IA + IB>(min(NST - 3, nk - 2 - kt));
        if (kt + NST - 1 < nk) FF_ISSUE((kt + NST - 1) % NST, (kt + NST - 1) * BKd);
        const int sn = (kt + 1) % NST;
#pragma unroll
        for (int t = 0; t < TM; ++t) fa[nxt][t] = lds_rd128(&sA[sn][offa[0][t]]);
#pragma unroll
        for (int t = 0; t < TN; ++t) fb[nxt][t] = lds_rd128(&sB[sn][offb[0][t]]);
        asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(TM + TN) : "memory");
      } else {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
#pragma unroll
      for (int t = 0; t < TM; ++t) asm volatile("" : "+v"(fa[cur][t]));
#pragma unroll
      for (int t = 0; t < TN; ++t) asm volatile("" : "+v"(fb[cur][t]));
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[cur][j], fa[cur][i], acc[i][j], 0, 0, 0);
    }
  }
#undef FF_ISSUE
  __syncthreads();   // every wave's last fragment reads retired before LDS is reused
  if (KG > 1) {
    // k group 1 hands its partial sums to k group 0 through LDS (past the epilogue staging)
    float* red = reinterpret_cast<float*>(smem + kEpi) + cw * TM * TN * 16 * 64 + lane;
    if (grp == 1) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) red[((i * TN + j) * 16 + v) * 64] = acc[i][j][v];
    }
    __syncthreads();
    if (grp == 1) return;   // the epilogue has no workgroup barrier
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] += red[((i * TN + j) * 16 + v) * 64];
  }
  epilogue_block<EPI, OUT_F32, RES_F32>(a, m0 + wm, n0 + wn, accs, smem + cw * 32 * (WN + 4) * 2);
}

// ------------------------------------------------------------------ bf16 MFMA GEMM, two wave groups in turn
// 256 x 64 TN tile (TN = 2, 3, 4), 64-wide K stages, 8 waves in two groups of four, one wave
// of each group per SIMD.  A stage has four phases, one per 32 rows of a wave's 128 x 16 TN
// block; a phase is a memory part (its fragment reads and two DMA instructions per wave) and
// 4 TN MFMAs, with a barrier after each.  The second group runs half a phase behind, so that
// on every SIMD one wave's MFMAs cover the other's reads and DMA.
//
// What bounds it: on large grids the card's power limit.  With random operands the clock falls
// to about 1.7 GHz while the MFMAs are busy 84 % of the cycles, so what counts is energy per
// FLOP: v_mfma_f32_16x16x32_bf16 moves half the accumulator bytes per FLOP of the 32x32x16
// form and runs 8 % faster in this same kernel (M = 4608, N = 21504, K = 3072: 496 -> 460 us;
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

template <int BM, int BN, int WM, int WN, int EPI, bool OF, bool RF>
void launch_tile(const GemmArgs* a, int n, hipStream_t s) {
  int nwg;
  if (n == 1) {
    const GemmGroup<1> G = make_group<BM, BN, 1>(a, nwg);
    FF_LAUNCH((k_gemm_bf16<BM, BN, WM, WN, EPI, OF, RF, 1>), nwg, (BM / WM) * (BN / WN) * 64, 0, s, G);
  } else {
    const GemmGroup<2> G = make_group<BM, BN, 2>(a, nwg);
    FF_LAUNCH((k_gemm_bf16<BM, BN, WM, WN, EPI, OF, RF, 2>), nwg, (BM / WM) * (BN / WN) * 64, 0, s, G);
  }
}

template <int BM, int BN, int WM, int WN, int NST, int EPI, bool OF, bool RF>
void launch_dl(const GemmArgs* a, int n, hipStream_t s) {
  int nwg;
  if (n == 1) {
    const GemmGroup<1> G = make_group<BM, BN, 1>(a, nwg);
    FF_LAUNCH((k_gemm_dl<BM, BN, WM, WN, NST, EPI, OF, RF, 1>), nwg, 2 * (BM / WM) * (BN / WN) * 64, 0, s, G);
  } else {
    const GemmGroup<2> G = make_group<BM, BN, 2>(a, nwg);
    FF_LAUNCH((k_gemm_dl<BM, BN, WM, WN, NST, EPI, OF, RF, 2>), nwg, 2 * (BM / WM) * (BN / WN) * 64, 0, s, G);
  }
}

template <int TN, int EPI, bool OF, bool RF>
void launch_pp(const GemmArgs* a, int n, hipStream_t s) {
  int nwg;
  if (n == 1) {
    const GemmGroup<1> G = make_group<256, 64 * TN, 1>(a, nwg);
    FF_LAUNCH((k_gemm_pp<TN, EPI, OF, RF, 1>), nwg, 512, 0, s, G);
  } else {
    const GemmGroup<2> G = make_group<256, 64 * TN, 2>(a, nwg);
    FF_LAUNCH((k_gemm_pp<TN, EPI, OF, RF, 2>), nwg, 512, 0, s, G);
  }
}

// Tile choice: the candidate with the least estimated time.  A candidate's round of
// workgroups over the 256 CUs takes lat + k * K us when it is bound by its own chain of
// stages, and its tiles keep the whole card busy for pow us per 256 tiles and unit of K when
// the card's power limit binds (large grids: the clock falls to about 1.6 GHz, so that a
// grid that leaves CUs idle runs its tiles faster).  Measured on MI355X with random bf16
// data; 256 x 64 TN tiles run k_gemm_pp, 128-row tiles k_gemm_dl.  In us at K = 1152 / 4608 /
// 15360 for one round of few tiles: 256x256 31 / 85 / 230, 256x192 28 / 70 / 188, 256x128
// 21 / 57 / 159, 128x96 15 / 37 / -, 128x64 10 / 29 / -; a full round at K = 3072 (clock
// down): 77, 62, 47 us.  What the choice picks, against the kernels this replaced (256x256 and
// 256x192 of 32x32x16 MFMAs with one wait and barrier per stage, 128x128 two per CU): M = 4608,
// N = 21504, K = 3072 545 -> 460 us (1324 TFLOP/s), 4096 x 3072 x 12288 263 -> 222 us,
// 14310 x 8192 x 2048 440 -> 370 us, 8192 x 4608 x 1152 100 -> 89 us, 2048 x 3456 x 1152
// 26.1 -> 20.8 us.
enum { kTile256, kTile256x192, kTile256x128, kTile128, kTile128x96, kTile128x64, kTileCount };
struct TilePlan { int tile; double cost; };
struct TileCost { int bm, bn; double lat, k, pow; };
constexpr TileCost kTileCost[kTileCount] = {
    {256, 256, 15.0, 0.0150, 0.0245}, {256, 192, 13.0, 0.0122, 0.0192}, {256, 128, 9.0, 0.0103, 0.0145},
    {128, 128, 9.5, 0.0076, 0.0145},  {128, 96, 8.3, 0.0062, 0.0120},   {128, 64, 4.2, 0.0054, 0.0100}};

long tiles_of(const GemmArgs* a, int n, int bm, int bn) {
  long t = 0;
  for (int i = 0; i < n; ++i) t += (long)((a[i].M + bm - 1) / bm) * ((a[i].N + bn - 1) / bn);
  return t;
}

bool all_k(const GemmArgs* a, int n, int m) {
  for (int i = 0; i < n; ++i)
    if (a[i].K % m) return false;
  return true;
}

// k_gemm_pp takes three or more 64-wide stages, and its operand rows lie within a 32-bit byte
// offset of their tile's first row (256 consecutive rows of a row map span at most
// 255 / n_seg + 1 further samples).
bool pp_ok(const GemmArgs* a, int n) {
  for (int i = 0; i < n; ++i) {
    const RowMap& m = a[i].amap;
    const uint64_t span = m.n_seg == m.N ? 256 : (uint64_t)(255 / m.n_seg + 1) * m.N + 256;
    if (a[i].K <= 128 || span * a[i].lda * 2 > 0xf0000000ull || 256ull * a[i].ldw * 2 > 0xf0000000ull) return false;
  }
  return true;
}

TilePlan plan_tiles(const GemmArgs* a, int n) {
  const bool pp = pp_ok(a, n), ring = all_k(a, n, 64);
  int K = 0;
  for (int i = 0; i < n; ++i) K = std::max(K, a[i].K);
  TilePlan best{-1, 1e300};
  for (int c = 0; c < kTileCount; ++c) {
    if (c < kTile128 ? !pp : !ring) continue;
    const TileCost& t = kTileCost[c];
    const long tiles = tiles_of(a, n, t.bm, t.bn);
    const double cost = std::max((double)((tiles + 255) / 256) * (t.lat + t.k * K), tiles / 256.0 * t.pow * K);
    if (cost < best.cost) best = TilePlan{c, cost};
  }
  return best;
}

template <int EPI, bool OF, bool RF>
void launch_bf16(const GemmArgs* a, int n, hipStream_t s) {
  switch (plan_tiles(a, n).tile) {
    case kTile256: launch_pp<4, EPI, OF, RF>(a, n, s); break;
    case kTile256x192: launch_pp<3, EPI, OF, RF>(a, n, s); break;
    case kTile256x128: launch_pp<2, EPI, OF, RF>(a, n, s); break;
    case kTile128: launch_dl<128, 128, 64, 64, 4, EPI, OF, RF>(a, n, s); break;
    case kTile128x96: launch_dl<128, 96, 32, 96, 4, EPI, OF, RF>(a, n, s); break;
    case kTile128x64: launch_dl<128, 64, 32, 64, 4, EPI, OF, RF>(a, n, s); break;
    default: launch_tile<128, 128, 64, 32, EPI, OF, RF>(a, n, s); break;   // K <= 128 off the 64 grid
  }
}

}  // namespace

namespace {

// bf16 dispatch of n (1 or 2) problems that share epilogue, output and residual types
hipError_t gemm_bf16(const GemmArgs* a, int n, hipStream_t s) {
  const bool of = a[0].out_f32 != 0, rf = a[0].resid_f32 != 0;
  if (n == 2 && a[0].epi != a[1].epi) {   // bias with bias+GELU (gemm2 admits no other mix)
    if (of) launch_bf16<EPI_BIAS_OR_GELU, true, false>(a, n, s);
    else launch_bf16<EPI_BIAS_OR_GELU, false, false>(a, n, s);
    return hipGetLastError();
  }
  switch (a[0].epi) {
    case EPI_BIAS:
      if (of) launch_bf16<EPI_BIAS, true, false>(a, n, s);
      else launch_bf16<EPI_BIAS, false, false>(a, n, s);
      break;
    case EPI_BIAS_GELU:
      if (of) launch_bf16<EPI_BIAS_GELU, true, false>(a, n, s);
      else launch_bf16<EPI_BIAS_GELU, false, false>(a, n, s);
      break;
    default:
      if (of && rf) launch_bf16<EPI_GATED, true, true>(a, n, s);
      else if (of) launch_bf16<EPI_GATED, true, false>(a, n, s);
      else if (rf) launch_bf16<EPI_GATED, false, true>(a, n, s);
      else launch_bf16<EPI_GATED, false, false>(a, n, s);
      break;
  }
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
  // Grouping pays when the combined launch is estimated to take no longer than the two.
  const GemmArgs both[2] = {a0, a1};
  const TilePlan pb = plan_tiles(both, 2);
  const bool pays = pb.tile < 0 || pb.cost <= plan_tiles(&a0, 1).cost + plan_tiles(&a1, 1).cost;
  if (dtype == DT_F32 || !same || !e0 || !e1 || !pays) {
    hipError_t e = gemm(dtype, a0, s);
    return e != hipSuccess ? e : gemm(dtype, a1, s);
  }
  return gemm_bf16(both, 2, s);
}

}  // namespace ff
