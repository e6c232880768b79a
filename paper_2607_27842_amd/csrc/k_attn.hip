// Softmax attention softmax(q k^T * scale) v per (sample, head), flash-style: key/value
// tiles are staged through LDS and each wavefront keeps a running (max, sum) per query
// (online softmax), so no N x N matrix is ever stored.
//
// bf16: v_mfma_f32_16x16x32_bf16.  A wavefront owns 16 or 32 queries; the 8 wavefronts of a
// workgroup share each 64-key tile.  Scores are formed transposed, S^T = K Q^T, so every
// lane holds scores of ONE query (per 16-query tile), and the probabilities are already in the
// register layout of the B operand of O^T = V^T P^T (no shuffle).
// fp32: v_mfma_f32_16x16x4 in the same form, the waves of a workgroup splitting the keys.
#include "dev_common.h"

namespace ff {

namespace {

constexpr float kPLim = 256.0f;   // a lane's probability sum per query and tile that raises the running max

// ---------------------------------------------------------------- bf16, two wave groups in turn
// 8 waves of 16 QT queries in two groups of four (one wave of each group per SIMD), 64-key
// tiles of K and V in rings of four.  Per tile a wave has a softmax slot (the tile's
// probabilities, and the DMA of the tiles three and two ahead) and an MFMA slot (the next
// tile's scores, then this tile's P V), each ended by a barrier; the second group runs one
// slot behind, so that on every SIMD one wave's VALU work meets the other's MFMAs.
// What bounds it: the card's power limit on long sequences (N = 14566, H = 16, d = 128: clock 2.0 of
// 2.4 GHz, MFMAs busy 58 % of its cycles, VALU work beside them in 35 % of those; fewer VALU
// instructions, no bank conflicts and earlier DMA took 7 % of the cycles and none of the time).
// Against the kernel this replaced (32x32x16 MFMAs, both waves of a SIMD in phase, K and V staged
// through registers): N = 14566, H = 16, d = 128 1710 -> 1460 us (1190 TFLOP/s), N = 4608, H = 24
// 267 -> 230, N = 1536, H = 24 62 -> 40, N = 3000, H = 20, d = 96 100 -> 67, B = 2, N = 1668, H = 37,
// d = 40 105 -> 75, B = 8, N = 256, H = 16, d = 72 8.7 -> 8.0.
// v_mfma_f32_16x16x32_bf16 layouts (A lane l: row l%16, k 8*(l/16)+0..7; B lane l: column
// l%16, same k; D[v] at row 4*(l/16)+v, column l%16):
//   S^T = K Q^T: lane l holds the scores of query l%16 at keys 16 i + 4 (l/16) + v, i < 4.
//   O^T += V^T P^T, 32 keys per MFMA: k index 8 g + j stands for key 4 g + j (j < 4) of the
//     first and 4 g + j - 4 of the second 16 keys, which makes the B operand the lane's own
//     eight probabilities; the A operand is two transposed reads (4 keys of one dim each).
// Head dims are zero-padded: k steps of 32 (NC), output tiles of 16 (NE); RWB bytes per LDS row.
//
// Ring slots: the MFMA slot of tile j reads K j+1 and V j, its first K reads going out at the
// end of the softmax slot before.  A softmax slot i refills what the MFMA slot i-2 read
// (K i-1, V i-2): both groups have ended that slot before either starts this one.  Before
// the barrier that ends it, a wave waits for its DMA of the softmax slot before (K j+1 and
// V j of the next MFMA slot's reads were issued two tiles ahead).
template <int RWB, int NC, int NE, int QT>
__global__ __launch_bounds__(512) void k_attn_pp(AttnArgs a) {
#ifdef __HIP_DEVICE_COMPILE__   // the host pass needs the launch stub only
  constexpr int KB = 64, NB = 4;                 // keys per tile, ring depth
  constexpr int TB = KB * RWB;                   // bytes of a K (or V) tile
  constexpr int DPW = RWB / 128;                 // DMA instructions per wave, tile and operand
  constexpr int CPR = RWB / 16;                  // 16-byte chunks per LDS row
  static_assert(NC * 64 <= RWB && NE * 32 <= RWB, "head dim tiles fit the LDS row");
  constexpr int LDO = NE * 16 + 8;               // staged output row pitch (elements)
  constexpr int kMain = 2 * NB * TB, kOut = 8 * 16 * QT * LDO * 2;
  __shared__ __attribute__((aligned(1024))) char smem[kMain > kOut ? kMain : kOut];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  int qb, hd, b;
  {
    const int nqb = (a.N + 128 * QT - 1) / (128 * QT), n = gridDim.x, id = blockIdx.x;
    const int full = n / 8 * 8;
    const int t = id < full ? (id % 8) * (full / 8) + id / 8 : id;
    qb = __builtin_amdgcn_readfirstlane(t % nqb);
    hd = __builtin_amdgcn_readfirstlane((t / nqb) % a.H);
    b = __builtin_amdgcn_readfirstlane(t / (nqb * a.H));
  }
  const int N = a.N, d = a.d, q0 = qb * 128 * QT + wave * 16 * QT;
  const size_t rb = (size_t)b * N;
  const char* base = reinterpret_cast<const char*>(reinterpret_cast<const uint16_t*>(a.qkv) + rb * a.ldq);
  const uint32_t ldb = (uint32_t)a.ldq * 2;
  // Q^T fragments: lane holds Q[q0 + 16 t + l16][32 c + 8 g .. +7], zero past N and d
  bf16x8_t qf[QT][NC];
#pragma unroll
  for (int t = 0; t < QT; ++t)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int q = q0 + 16 * t + l16, e = 32 * c + 8 * g;
      u32x4_t v = {0u, 0u, 0u, 0u};
      if (q < N && e < d) v = *reinterpret_cast<const u32x4_t*>(base + (size_t)q * ldb + ((size_t)hd * d + e) * 2);
      qf[t][c] = __builtin_bit_cast(bf16x8_t, v);
    }
  // the rows of an LDS tile are rotated by f(row) among their 16-byte chunks, so that both the
  // K reads (16 rows, one chunk) and the transposed V reads (8 rows, one chunk pair) of a
  // pass spread over all banks
  auto swz = [](int row) {
    const int hi = (row >> 3) & 1;
    return (CPR == 16 ? ((row & 7) ^ (hi << 2)) : (((row >> 1) & 3) ^ (hi << 1))) << 1 | hi;
  };
  uint32_t vo[DPW];   // this lane's byte offsets within a K tile; past d: out of range (zeros)
#pragma unroll
  for (int j = 0; j < DPW; ++j) {
    const int idx = (wave * DPW + j) * 64 + lane, row = idx / CPR, e = ((idx % CPR) ^ swz(row)) * 8;
    vo[j] = e < d ? (uint32_t)row * ldb + (uint32_t)e * 2 : 0x80000000u;
  }
  // DMA of the next K / V tile (c0: its column in bytes) into ring slot *slot.  The tile's own
  // resource ends with the sample's last row, so that keys past N load as zeros.
  auto load = [&](int off, int* tile, int* slot, uint32_t c0) __attribute__((always_inline)) {
    const int rows = N - *tile * KB;
    const uint64_t left = rows > 0 ? (uint64_t)rows * ldb - c0 : 0;
    const uint32_t num = left < 0x7fffff00u ? (uint32_t)left : 0x7fffff00u;
    __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base) + (size_t)*tile * KB * ldb + c0, 0, num, 0x00020000);
#pragma unroll
    for (int j = 0; j < DPW; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, FF_AS3(smem + off + *slot + (wave * DPW + j) * 1024), 16, vo[j], 0, 0, 0);
    ++*tile;
    *slot = *slot == (NB - 1) * TB ? 0 : *slot + TB;
  };
  int ktile = 0, vtile = 0, kslot = 0, vslot = 0;
  const uint32_t kc = ((uint32_t)a.C + (uint32_t)hd * d) * 2, vc = kc + (uint32_t)a.C * 2;
  auto load_k = [&]() __attribute__((always_inline)) { load(0, &ktile, &kslot, kc); };
  auto load_v = [&]() __attribute__((always_inline)) { load(NB * TB, &vtile, &vslot, vc); };
  // fragment addresses within a tile (k step c and output tile e enter by xor)
  const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) const void*)smem);
  const uint32_t ka = lds0 + l16 * RWB + ((g ^ swz(l16)) * 16);
  const int vr = 4 * g + (l16 >> 2);
  const uint32_t va = lds0 + NB * TB + vr * RWB + ((((l16 & 3) >> 1) ^ swz(vr)) * 16) + (l16 & 1) * 8;
  f32x4_t o[NE][QT], sc[4][QT];
#pragma unroll
  for (int e = 0; e < NE; ++e)
#pragma unroll
    for (int t = 0; t < QT; ++t) o[e][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m[QT], l[QT], lim[QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) { m[t] = -INFINITY; l[t] = 0.f; lim[t] = -1.f; }
  const float sl2 = a.scale * 1.4426950408889634f;
  bf16x8_t pb[2][QT];
  int ks = 0, vs = 0;            // ring slots being read
  // The MFMA slot of a tile is a chain of units of two A fragments and 2 QT MFMAs: first
  // the 2 NC units of the next tile's scores (K fragments), then the NE units of this tile's
  // PV product (V^T fragments, each two transposed reads).  A unit's reads are issued UD
  // units ahead: LDS latency with four waves reading is longer than one unit's MFMAs.
  constexpr int UK = 2 * NC, UV = NE, UD = 3;
  bf16x8_t kf[UD + 1][2];
  u32x2_t vf[UD + 1][2][2] = {};
  uint32_t ka_ = ka, va_ = va;
  auto rd = [&](auto Uc) __attribute__((always_inline)) {
    constexpr int U = decltype(Uc)::value;
    if constexpr (U < UK) {
      constexpr int c = U / 2, i0 = U % 2 * 2;
      const uint32_t ad = ka_ ^ (c * 64);
      kf[U % (UD + 1)][0] = lds_rd128_at<i0 * 16 * RWB>(ad);
      kf[U % (UD + 1)][1] = lds_rd128_at<(i0 + 1) * 16 * RWB>(ad);
    } else if constexpr (U < UK + UV) {
      constexpr int f = 2 * (U - UK);
      const uint32_t a0 = va_ ^ (f % NE * 32), a1 = va_ ^ ((f + 1) % NE * 32);
      vf[U % (UD + 1)][0][0] = lds_rd64_tr(a0, f / NE * 32 * RWB);
      vf[U % (UD + 1)][0][1] = lds_rd64_tr(a0, f / NE * 32 * RWB + 16 * RWB);
      vf[U % (UD + 1)][1][0] = lds_rd64_tr(a1, (f + 1) / NE * 32 * RWB);
      vf[U % (UD + 1)][1][1] = lds_rd64_tr(a1, (f + 1) / NE * 32 * RWB + 16 * RWB);
    }
  };
  auto unit = [&](auto Uc) __attribute__((always_inline)) {
    constexpr int U = decltype(Uc)::value;
    rd(Int<U + UD>{});
    constexpr int later = (U + 1 < UK + UV ? (U + 1 < UK ? 2 : 4) : 0) + (U + 2 < UK + UV ? (U + 2 < UK ? 2 : 4) : 0) +
                          (U + 3 < UK + UV ? (U + 3 < UK ? 2 : 4) : 0);
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(later) : "memory");
    constexpr int buf = U % (UD + 1);
    if constexpr (U < UK) {
      FF_TIE(kf[buf][0]); FF_TIE(kf[buf][1]);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int t = 0; t < QT; ++t) {
          constexpr int c = U / 2, i0 = U % 2 * 2;
          sc[i0 + i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[buf][i], qf[t][c], c == 0 ? f32x4_t{0.f, 0.f, 0.f, 0.f} : sc[i0 + i][t], 0, 0, 0);
        }
    } else {
#pragma unroll
      for (int i = 0; i < 2; ++i) { FF_TIE(vf[buf][i][0]); FF_TIE(vf[buf][i][1]); }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        constexpr int f0 = 2 * (U - UK);
        const int s = (f0 + i) / NE, e = (f0 + i) % NE;
        const u32x4_t w = {vf[buf][i][0][0], vf[buf][i][0][1], vf[buf][i][1][0], vf[buf][i][1][1]};
#pragma unroll
        for (int t = 0; t < QT; ++t)
          o[e][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w), pb[s][t], o[e][t], 0, 0, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
#define FF_BAR() asm volatile("s_barrier" ::: "memory")
  const int nt = (N + KB - 1) / KB;
  load_k();
  load_k(); load_v();
  load_k(); load_v();
  wait_vm<2 * DPW>();
  FF_BAR();
  // the first tile's scores (the V reads that run ahead here are used nowhere, but hold their
  // registers until they are in)
  static_for<0, UD>(rd);
  static_for<0, UK>(unit);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
  for (int i = 0; i < (UD + 1) * 4; ++i) FF_TIE(vf[i / 4][i / 2 % 2][i % 2]);
  ks = TB;
  if (wave >= 4) FF_BAR();   // the second group runs one slot behind
  // sc -> probabilities pb (complete when it returns: nothing of it moves past the barrier)
  auto softmax = [&]() __attribute__((always_inline)) {
    // probabilities against the running maxima m (log2 units of the scaled scores).  m is
    // raised, and O and l rescaled, only when a lane's 16 probabilities of a query add up to
    // more than kPLim = 2^8 (or are not all numbers), which no tile whose scores are all at
    // most m + 4 does: most tiles form no maximum at all.  The shift cancels in O / l, and
    // p <= 2^8 stays well inside fp32.
    float p[QT][16], ps[QT];
    bool up = false;
    auto probs = [&](int t) __attribute__((always_inline)) {
      // m is still -inf only if every score so far is: those probabilities are 0, not NaN
      const float mo = m[t] == -INFINITY ? 0.f : m[t];
#pragma unroll
      for (int i = 0; i < 16; ++i) p[t][i] = __builtin_amdgcn_exp2f(fmaf(sc[i / 4][t][i % 4], sl2, -mo));
      float s4[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) s4[i] = (p[t][4 * i] + p[t][4 * i + 1]) + (p[t][4 * i + 2] + p[t][4 * i + 3]);
      ps[t] = (s4[0] + s4[1]) + (s4[2] + s4[3]);
    };
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      probs(t);
      up = up || !(ps[t] <= lim[t]);
    }
    if (__any(up)) {
#pragma unroll
      for (int t = 0; t < QT; ++t) {
        float x = -INFINITY;
#pragma unroll
        for (int i = 0; i < 16; ++i) x = fmaxf(x, sc[i / 4][t][i % 4]);
        x = fmaxf(x, __shfl_xor(x, 16, 64));         // the four lanes of a query together
        x = fmaxf(x, __shfl_xor(x, 32, 64)) * sl2;   // scale > 0: max commutes with it
        const float mn = fmaxf(m[t], ceilf(x));      // whole: the rescale is by a power of two, exact
        const float al = mn == m[t] ? 1.f : __builtin_amdgcn_exp2f(m[t] - mn);   // exp2(-inf) = 0
        m[t] = mn;
        lim[t] = mn == -INFINITY ? -1.f : kPLim;     // -1: the next tile comes here too
        l[t] *= al;
#pragma unroll
        for (int e = 0; e < NE; ++e) o[e][t] *= al;
        probs(t);
      }
    }
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      l[t] += ps[t];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const float* q = &p[t][8 * s];
        const u32x4_t w = {pack_bf16x2(q[0], q[1]), pack_bf16x2(q[2], q[3]), pack_bf16x2(q[4], q[5]), pack_bf16x2(q[6], q[7])};
        pb[s][t] = __builtin_bit_cast(bf16x8_t, w);
      }
    }
#pragma unroll
    for (int t = 0; t < QT; ++t) { FF_TIE(pb[0][t]); FF_TIE(pb[1][t]); FF_TIE(l[t]); }
    __builtin_amdgcn_sched_barrier(0);
  };
  for (int kt = 0; kt < nt - 1; ++kt) {
    load_k();
    load_v();
    __builtin_amdgcn_sched_barrier(0);
    softmax();
    ka_ = ka + ks;
    va_ = va + vs;
    static_for<0, UD>(rd);
    wait_vm<2 * DPW>();
    FF_BAR();
    __builtin_amdgcn_s_setprio(1);
    static_for<0, UK + UV>(unit);
    __builtin_amdgcn_s_setprio(0);
    FF_BAR();
    ks = ks == (NB - 1) * TB ? 0 : ks + TB;
    vs = vs == (NB - 1) * TB ? 0 : vs + TB;
  }
  // the last tile: keys past N get probability 0
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int t = 0; t < QT; ++t)
        if ((nt - 1) * KB + 16 * i + 4 * g + v >= N) sc[i][t][v] = -INFINITY;
  softmax();
  va_ = va + vs;
  static_for<UK, UK + UD>(rd);
  wait_vm<0>();
  FF_BAR();
  static_for<UK, UK + UV>(unit);
  FF_BAR();
  if (wave < 4) FF_BAR();
#undef FF_BAR
  // o[e][t][v] = O[query q0 + 16 t + l16][16 e + 4 g + v], staged through the wave's own LDS
  // region and stored as 16-byte row pieces; every wave's tile reads and DMA ended before
  // the last barrier
  uint16_t* stg = reinterpret_cast<uint16_t*>(smem) + wave * 16 * QT * LDO;
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    float s = l[t] + __shfl_xor(l[t], 16, 64);
    s += __shfl_xor(s, 32, 64);
    const float inv = 1.0f / s;
#pragma unroll
    for (int e = 0; e < NE; ++e)
      *reinterpret_cast<u32x2_t*>(stg + (16 * t + l16) * LDO + 16 * e + 4 * g) =
          u32x2_t{pack_bf16x2(o[e][t][0] * inv, o[e][t][1] * inv), pack_bf16x2(o[e][t][2] * inv, o[e][t][3] * inv)};
  }
  uint16_t* out = reinterpret_cast<uint16_t*>(a.out);
  const int ppr = d / 8;
  for (int idx = lane; idx < 16 * QT * ppr; idx += 64) {
    const int row = idx / ppr, pc = idx - row * ppr;
    if (q0 + row < N)
      *reinterpret_cast<u32x4_t*>(out + (rb + q0 + row) * a.ldo + (size_t)hd * d + pc * 8) =
          *reinterpret_cast<const u32x4_t*>(stg + row * LDO + pc * 8);
  }
#endif
}

// ---------------------------------------------------------------- fp32
// v_mfma_f32_16x16x4 in the same transposed form: a workgroup's 4 waves share 16 QT queries and
// split the keys in blocks of 32; q, K and V go from memory to registers in operand layout
// (S^T = K Q^T takes 4 dims of a row per 16-byte chunk, one per step; in O^T = V^T P^T step
// v takes keys 4 g + v, so the B operand is the lane's own probability), and the waves'
// (m, l, O) are merged in wave order through LDS.  Everything stays fp32.  Bound by the fp32
// MFMA rate and the latency of its loads; against one thread per query: N = 64, H = 4, d = 64
// 71 -> 5 us, B = 2, N = 256, H = 16, d = 72 762 -> 16 us.
// ND: 16-wide pieces of the head dim.
template <int ND, int QT>
__global__ __launch_bounds__(256) void k_attn_f32(AttnArgs a) {
  constexpr int PF = ND * QT * 4 + 2 * QT;   // floats per lane of a merge entry
  __shared__ float xch[3][PF][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  int qb, hd, b;
  {
    const int nqb = (a.N + 16 * QT - 1) / (16 * QT), n = gridDim.x, id = blockIdx.x;
    const int full = n / 8 * 8;
    const int t = id < full ? (id % 8) * (full / 8) + id / 8 : id;
    qb = t % nqb; hd = (t / nqb) % a.H; b = t / (nqb * a.H);
  }
  const int N = a.N, d = a.d, q0 = qb * 16 * QT;
  const size_t rb = (size_t)b * N;
  const float* base = reinterpret_cast<const float*>(a.qkv) + rb * a.ldq + (size_t)hd * d;
  const f32x4_t z4 = {0.f, 0.f, 0.f, 0.f};
  f32x4_t qf[QT][ND], o[ND][QT];
#pragma unroll
  for (int t = 0; t < QT; ++t)
#pragma unroll
    for (int c = 0; c < ND; ++c) {
      const int q = q0 + 16 * t + l16, e = 16 * c + 4 * g;
      qf[t][c] = q < N && e < d ? *reinterpret_cast<const f32x4_t*>(base + (size_t)q * a.ldq + e) : z4;
      o[c][t] = z4;
    }
  float m[QT], l[QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) { m[t] = -INFINITY; l[t] = 0.f; }
  for (int k0 = wave * 32; k0 < N; k0 += 128) {
    f32x4_t kf[2][ND];
    float vv[2][4][ND];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int c = 0; c < ND; ++c) {
        const int k = k0 + 16 * i + l16, e = 16 * c + 4 * g;
        kf[i][c] = k < N && e < d ? *reinterpret_cast<const f32x4_t*>(base + (size_t)k * a.ldq + a.C + e) : z4;
      }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int c = 0; c < ND; ++c) {
          const int k = k0 + 16 * i + 4 * g + v, e = 16 * c + l16;
          vv[i][v][c] = k < N && e < d ? base[(size_t)k * a.ldq + 2 * (size_t)a.C + e] : 0.f;
        }
    f32x4_t sc[2][QT];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int t = 0; t < QT; ++t) sc[i][t] = z4;
#pragma unroll
    for (int c = 0; c < ND; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int t = 0; t < QT; ++t) sc[i][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i][c][j], qf[t][c][j], sc[i][t], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      float x = -INFINITY;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          sc[i][t][v] = k0 + 16 * i + 4 * g + v < N ? sc[i][t][v] * a.scale : -INFINITY;
          x = fmaxf(x, sc[i][t][v]);
        }
      x = fmaxf(x, __shfl_xor(x, 16, 64));
      x = fmaxf(x, __shfl_xor(x, 32, 64));
      const float mn = fmaxf(m[t], x), mo = mn == -INFINITY ? 0.f : mn;
      const float al = expf(m[t] - mo);   // exp(-inf) = 0
      m[t] = mn;
      l[t] *= al;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          sc[i][t][v] = expf(sc[i][t][v] - mo);
          l[t] += sc[i][t][v];
        }
#pragma unroll
      for (int c = 0; c < ND; ++c) o[c][t] *= al;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int c = 0; c < ND; ++c)
#pragma unroll
          for (int t = 0; t < QT; ++t) o[c][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[i][v][c], sc[i][t][v], o[c][t], 0, 0, 0);
  }
  // l is per lane: the four lanes of a query add up after the merge (m is common to them)
  if (wave > 0) {
    float (*x)[64] = xch[wave - 1];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
#pragma unroll
      for (int c = 0; c < ND; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) x[(t * ND + c) * 4 + v][lane] = o[c][t][v];
      x[ND * QT * 4 + 2 * t][lane] = m[t];
      x[ND * QT * 4 + 2 * t + 1][lane] = l[t];
    }
  }
  __syncthreads();
  if (wave > 0) return;
#pragma unroll
  for (int t = 0; t < QT; ++t) {
#pragma unroll
    for (int w = 0; w < 3; ++w) {
      const float m2 = xch[w][ND * QT * 4 + 2 * t][lane], l2 = xch[w][ND * QT * 4 + 2 * t + 1][lane];
      const float mn = fmaxf(m[t], m2), mo = mn == -INFINITY ? 0.f : mn;
      const float a1 = expf(m[t] - mo), a2 = expf(m2 - mo);
      m[t] = mn;
      l[t] = l[t] * a1 + l2 * a2;
#pragma unroll
      for (int c = 0; c < ND; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) o[c][t][v] = o[c][t][v] * a1 + xch[w][(t * ND + c) * 4 + v][lane] * a2;
    }
    float s = l[t] + __shfl_xor(l[t], 16, 64);
    s += __shfl_xor(s, 32, 64);
    const float inv = 1.0f / s;
    const int q = q0 + 16 * t + l16;
    if (q < N) {
      float* out = reinterpret_cast<float*>(a.out) + (rb + q) * a.ldo + (size_t)hd * d;
#pragma unroll
      for (int c = 0; c < ND; ++c)
        if (16 * c + 4 * g < d) *reinterpret_cast<f32x4_t*>(out + 16 * c + 4 * g) = o[c][t] * inv;
    }
  }
}

}  // namespace

hipError_t attention(int dtype, const AttnArgs& a, hipStream_t s) {
  if (a.N <= 0) return hipSuccess;
  if (dtype == DT_BF16) {
    // a lane's byte offset within a 64-key tile stays below 2^31
    if ((uint64_t)a.ldq * 2 * 64 > 0x7fffff00ull) return hipErrorInvalidValue;
    // 16 queries per wave for d <= 64: two workgroups then share a CU (64 KB of LDS and at most
    // 128 VGPRs each) and take 0.83 of the time of one with 32 queries (B = 2, N = 2000, H =
    // 24, d = 64: 65 against 78 us).  For larger d 16 or 32 (QT = 2), whichever needs the
    // shorter sum of rounds over the 256 CUs: a round with 16 takes 0.63 of one with 32 (d =
    // 128: 1.14 against 1.80 us per 64 keys).
    const long hb = (long)a.H * a.B, w2 = (a.N + 255) / 256 * hb, w1 = (a.N + 127) / 128 * hb;
    const bool two = a.d > 64 && (double)((w2 + 255) / 256) <= 0.63 * ((w1 + 255) / 256);
    const long nwg = two ? w2 : w1;
    if (nwg > 0x7fffffffL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nwg);   // one dimension: the kernel maps it to (sample, head, query block)
#define FF_ATTN(RWB, NC, NE)                                                          \
    do {                                                                              \
      if constexpr (RWB > 128)                                                        \
        if (two) { FF_LAUNCH((k_attn_pp<RWB, NC, NE, 2>), grid, 512, 0, s, a); break; } \
      FF_LAUNCH((k_attn_pp<RWB, NC, NE, 1>), grid, 512, 0, s, a);                     \
    } while (0)
    if (a.d <= 48) FF_ATTN(128, 2, 3);
    else if (a.d <= 64) FF_ATTN(128, 2, 4);
    else if (a.d <= 80) FF_ATTN(256, 3, 5);
    else if (a.d <= 96) FF_ATTN(256, 3, 6);
    else FF_ATTN(256, 4, 8);
#undef FF_ATTN
  } else {
    // 32 queries per workgroup (each K / V load feeds two query tiles) when that still gives
    // four workgroups per CU
    const long hb = (long)a.H * a.B;
    const bool two = (a.N + 31) / 32 * hb >= 1024;
    const long nwg = two ? (a.N + 31) / 32 * hb : (a.N + 15) / 16 * hb;
    if (nwg > 0x7fffffffL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nwg);
#define FF_ATTN32(ND)                                                       \
    do {                                                                    \
      if (two) FF_LAUNCH((k_attn_f32<ND, 2>), grid, 256, 0, s, a);          \
      else FF_LAUNCH((k_attn_f32<ND, 1>), grid, 256, 0, s, a);              \
    } while (0)
    if (a.d <= 32) FF_ATTN32(2);
    else if (a.d <= 64) FF_ATTN32(4);
    else if (a.d <= 80) FF_ATTN32(5);
    else if (a.d <= 96) FF_ATTN32(6);
    else FF_ATTN32(8);
#undef FF_ATTN32
  }
  return hipGetLastError();
}

}  // namespace ff
