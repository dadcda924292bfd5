// Prefill GEMM of the quantized linear on small tiles: the launches (more
// than 64 tokens) whose 256 x 256 tiles would leave most of the chip idle,
// e.g. one prompt of a few hundred tokens.
#include "ot_gemm_common.h"

namespace ot {
namespace detail {

// ---------------------------------------------------------------------------
// Deep-ring tile GEMM (v_mfma_i32_32x32x32_i8)
// ---------------------------------------------------------------------------
// Workgroup tile BN (weight rows) x BM (token rows), K tile BK bytes, waves
// arranged WN x WM x WK: WN x WM blocks of (BN/WN) x (BM/WM), each worked on
// by WK waves that take 1/WK of every K tile's 32-byte steps.
//
// What bounds it, from builds with one part of the K loop taken out (us, the
// weights from HBM; whole, without MFMAs and fragment reads, without loads).
// Up to a few hundred tokens, staging the operands: 512 x 5120, K = 20480 on
// 128 x 96 tiles 75, 73, 44; 512 x 15360, K = 5120 on 256 x 128 46, 45, 28;
// 131 x 6150, K = 4112 on 64 x 128 17, 17, 10.  A CU stages 43-61 GB/s there
// ((BN + BM) bytes per BN * BM products), where loads that all hit the L2 reach
// 145; with the weights in the last-level cache the loads alone take 57 of the
// 73 us.  With many tokens no part alone: 2048 x 4096, K = 16384 on 256 x 128
// tiles 118, 96, 83 (a fragment read and 0.375 loads per MFMA, which cost the
// matrix core issue cycles).  So:
//   - the ring is as deep as the LDS allows (3-8 stages): a K tile takes less
//     time than a load's latency, and the two stages that suffice for the
//     large tiles left the loads exposed (256 x 128 tiles, 2048 x 4096,
//     K = 16384: 148 us with 2 stages, 122 with 3);
//   - a stage holds the tile's rows once and no wave reads a fragment that
//     another reads too where WK splits the K steps instead (64 x 64 tile:
//     4 waves of the whole tile), which halves the LDS reads;
//   - the tile is the one that stages least per CU among those that fill the
//     CUs (the launch plan, ot_prefill.hip).
// Against the large tiles, one launch each, weights rotating through HBM:
// 512 x 5120 with K = 5120 22 us (37 before), K = 20480 78 (171); 300 x 4096,
// K = 11008 31 (100); 128 x 7168, K = 7168 22 (70); 131 x 6150, K = 4112 17 (41).
//
// Loads, swizzle, K walk and epilogue arithmetic are those of the large
// tiles (ot_prefill.hip); the sums are exact integers, so the results are
// the same bits.  A stage is [BN weight rows | BM token rows][BK], its 1 KiB
// blocks dealt to the waves in turn.
template <int BN, int BM, int BK, int WN, int WM, int WK, int S>
struct RingCfg {
  static constexpr int kWaves = WN * WM * WK;
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kChunks = BK / 16;
  static constexpr int kTN = BN / WN, kTM = BM / WM;
  static constexpr int kFN = kTN / 32, kFM = kTM / 32;
  static constexpr int kMfma = kFN * kFM;         // 32x32 blocks of a wave
  static constexpr int kSteps = BK / 32 / WK;     // K steps per wave and K tile
  static constexpr int kStage = (BN + BM) * BK;
  static constexpr int kBlocksA = BN * BK / 1024;  // 1 KiB blocks of weights in a stage
  static constexpr int kLoads = kStage / 1024 / kWaves;
  // after the loop the ring's bytes hold the K groups' partial sums, the fp16
  // output tile and the epilogue's parameters, side by side.  Block b of a
  // wave position is finished by K group b mod WK.
  static constexpr int kOwn = (kMfma + WK - 1) / WK;
  static constexpr int kRed = WN * WM * WK * (WK - 1) * kOwn * 4096;
  static constexpr int kOut = BN * BM * 2;
  static constexpr int kParams = 12 * BN + 4 * BM;        // sW, b', zW; sX
  static constexpr int kSums = kWaves * kFM * 32 * 4;     // token code sums
  static constexpr int kTail = kRed + kOut + kParams + kSums;
  static constexpr int kSmem = S * kStage > kTail ? S * kStage : kTail;
  static_assert(BK == 128 || BK == 256, "BK");
  static_assert(kLoads * kWaves * 1024 == kStage, "a stage splits evenly over the waves");
  static_assert(kTN % 32 == 0 && kTM % 32 == 0, "32x32 blocks");
  static_assert(kSteps >= 2 && kSteps % 2 == 0, "the fragment buffers alternate within a K tile");
  static_assert(S >= 2 && (S - 2) * kLoads <= 63, "vmcnt range");
  static_assert(kThreads >= BN && kThreads >= BM, "one thread per channel and token parameter");
  static_assert(kSmem <= 160 * 1024, "LDS");
};

// Chunk c (16 bytes) of stage row r sits at chunk c ^ swz_ring(r): the 16
// rows of a fragment read then cover distinct 16-byte banks groups.
template <int kChunks>
__device__ __forceinline__ int swz_ring(int r) {
  if constexpr (kChunks == 8) return (r & 7) ^ ((r >> 3) & 1);
  else return r & 15;
}

template <int BN, int BM, int BK, int WN, int WM, int WK, int S, int EPI>
__device__ __forceinline__ void ring_body(
    int8_t *smem, const int8_t *__restrict__ Xq, const int8_t *__restrict__ Wq,
    const float *__restrict__ sX, const int32_t *__restrict__ zW, const float *__restrict__ sW,
    const float *__restrict__ bp, int M, int N, int K, uint16_t *__restrict__ Y,
    int32_t *__restrict__ acc_out, int tiles_m, int tiles_n) {
  using C = RingCfg<BN, BM, BK, WN, WM, WK, S>;
  constexpr int kMfma = C::kMfma, kReads = C::kFN + C::kFM;

  // ---- tile schedule: as the large tiles (each XCD a contiguous range of
  // tiles, walked in groups of 8 token tiles) --------------------------------
  constexpr int kGroupM = 8;
  const int nwg = gridDim.x, bid = blockIdx.x;
  const int xcd = bid & 7, local = bid >> 3;
  const int per = nwg >> 3, rem = nwg & 7;
  const int lid = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + local;
  const int group_size = kGroupM * tiles_n;
  const int first_m = (lid / group_size) * kGroupM;
  const int gm = min(tiles_m - first_m, kGroupM);
  const int tm = first_m + (lid % group_size) % gm;
  const int tn = (lid % group_size) / gm;
  const int n0 = tn * BN, m0 = tm * BM;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pos = wave % (WN * WM), kg = wave / (WN * WM);
  const int wn = pos % WN, wm = pos / WN;

  // the epilogue's parameters, one channel and one token per thread, loaded
  // now so that their latency passes during the K loop
  float p_s = 0.f, p_b = 0.f, p_x = 0.f;
  int p_z = 0;
  if (tid < BN && n0 + tid < N) {
    p_s = sW[n0 + tid];
    p_b = bp[n0 + tid];
    if constexpr (EPI == kEpiAsym) p_z = zW[n0 + tid];
  }
  if constexpr (EPI == kEpiToken) {
    if (tid < BM && m0 + tid < M) p_x = sX[m0 + tid];
  }

  // ---- global -> LDS addressing ---------------------------------------------
  const __amdgpu_buffer_rsrc_t ra =
      make_rsrc(Wq + (int64_t)n0 * K, (uint32_t)(min(BN, N - n0) * K));
  const __amdgpu_buffer_rsrc_t rb =
      make_rsrc(Xq + (int64_t)m0 * K, (uint32_t)(min(BM, M - m0) * K));
  // Lane i of load j fetches the chunk that belongs at stage row
  // (j kWaves + wave) kRowsPerLoad + i / kChunks, position i mod kChunks.  The
  // rows of a lane's loads are multiples of 16 apart, the swizzle's period, so
  // one chunk offset serves them all.
  constexpr int kRowsPerLoad = 64 / C::kChunks;
  static_assert(C::kWaves * kRowsPerLoad % 16 == 0, "one swizzle per lane");
  const int row0 = wave * kRowsPerLoad + lane / C::kChunks;
  const int gck = 16 * ((lane % C::kChunks) ^ swz_ring<C::kChunks>(row0));
  uint32_t goff[C::kLoads];
#pragma unroll
  for (int j = 0; j < C::kLoads; ++j) {
    const int row = row0 + j * C::kWaves * kRowsPerLoad;
    goff[j] = (uint32_t)((row < BN ? row : row - BN) * K + gck);
  }
  const int KT = (K + BK - 1) / BK;
  const int phi = (tm + tn) & 1;  // neighbouring tiles walk K one tile apart
  // The tile being loaded: its number, what it adds to a lane's offsets (its
  // first K byte, or out of range past the end of K: zeros) and its stage.
  // Worked out once per tile: with the address arithmetic at each load the K
  // loop spends issue slots that its MFMAs and loads need (OPT-6.7B asymmetric
  // block at 2048 tokens 457.8 -> 450.1 us, 131 x 6150 linear 19.3 -> 19.0).
  int l_kt = 0;
  uint32_t l_add = 0;
  int8_t *l_dst = smem + wave * 1024;
  int l_slot = 0;
  auto aim = [&]() {  // l_add for tile l_kt
    int kr = l_kt + phi;
    if (kr >= KT) kr -= KT;
    const int k0 = kr * BK;
    l_add = l_kt < KT && k0 + gck < K ? (uint32_t)k0 : kOobOffset;
  };
  auto next_tile = [&]() {
    ++l_kt;
    l_slot = l_slot + 1 == S ? 0 : l_slot + 1;
    l_dst = smem + l_slot * C::kStage + wave * 1024;
    aim();
  };
  auto issue_one = [&](int j) {
    const int q = j * C::kWaves + wave;  // 1 KiB block of the stage (wave-uniform)
    int8_t *dst = l_dst + j * C::kWaves * 1024;
    if ((j + 1) * C::kWaves <= C::kBlocksA || (j * C::kWaves < C::kBlocksA && q < C::kBlocksA))
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void *)dst, 16, goff[j] + l_add, 0, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_void *)dst, 16, goff[j] + l_add, 0, 0, 0);
  };

  // ---- LDS -> register fragments ---------------------------------------------
  const int fr = lane & 31, fh = lane >> 5;
  int frag_off[C::kSteps];
#pragma unroll
  for (int s = 0; s < C::kSteps; ++s)
    frag_off[s] = fr * BK + 16 * ((2 * (kg * C::kSteps + s) + fh) ^ swz_ring<C::kChunks>(fr));
  const int a_base = wn * C::kTN * BK;
  const int b_base = (BN + wm * C::kTM) * BK;
  v4i fa[2][C::kFN], fb[2][C::kFM];
  v16i acc[C::kFN][C::kFM];
#pragma unroll
  for (int f = 0; f < C::kFN; ++f)
#pragma unroll
    for (int g = 0; g < C::kFM; ++g) acc[f][g] = v16i{};
  // asymmetric weights: token code sums over this wave's share of its K steps
  // (the WN waves of a token block take them in turn)
  static_assert(EPI != kEpiAsym || C::kSteps % WN == 0, "K steps split over the WN waves");
  int rs[C::kFM];
#pragma unroll
  for (int g = 0; g < C::kFM; ++g) rs[g] = 0;

  // A K tile's loads are spread evenly over the MFMAs from the previous
  // tile's last step to its own last but one; upto(u) of them go out before
  // the u-th of these kSlots MFMAs.
  constexpr int kSlots = kMfma * C::kSteps;
  auto upto = [](int u) {
    const int n = (u * C::kLoads + kSlots - 1) / kSlots;
    return n < C::kLoads ? n : C::kLoads;
  };
  // One K step: MFMAs on fragment buffer cb, reads of step rstep of the tile in
  // stage st into buffer nb, the aimed tile's loads from slot u0 on.
  auto kstep = [&](int cb, int step, const int8_t *st, int rstep, int nb, int u0) {
    constexpr int kN = kMfma > kReads ? kMfma : kReads;
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      if (i < C::kFN)
        fa[nb][i] = *reinterpret_cast<const v4i *>(st + a_base + i * 32 * BK + frag_off[rstep]);
      else if (i < kReads)
        fb[nb][i - C::kFN] =
            *reinterpret_cast<const v4i *>(st + b_base + (i - C::kFN) * 32 * BK + frag_off[rstep]);
      if (i < kMfma) {
        const int f = i / C::kFM, g = i % C::kFM;
        acc[f][g] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[cb][f], fb[cb][g], acc[f][g], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < C::kLoads; ++j)
          if (j >= upto(u0 + i) && j < upto(u0 + i + 1)) issue_one(j);
      }
    }
    if constexpr (EPI == kEpiAsym) {
      if (step % WN == wn) {
#pragma unroll
        for (int g = 0; g < C::kFM; ++g) rs[g] = byte_sum16(fb[cb][g], rs[g]);
      }
    }
    constexpr int kMaskMfma = 0x008, kMaskVmemRead = 0x020, kMaskDsRead = 0x100;
#pragma unroll
    for (int i = 0; i < kN; ++i) {
      if (i < kReads) __builtin_amdgcn_sched_group_barrier(kMaskDsRead, 1, 0);
      if (i < kMfma) {
        __builtin_amdgcn_sched_group_barrier(kMaskMfma, 1, 0);
#pragma unroll
        for (int j = 0; j < C::kLoads; ++j)
          if (j >= upto(u0 + i) && j < upto(u0 + i + 1))
            __builtin_amdgcn_sched_group_barrier(kMaskVmemRead, 1, 0);
      }
    }
  };

  // ---- main loop (the waits and the barrier as in the large tiles) -------------
  aim();
#pragma unroll
  for (int t = 0; t < S - 1; ++t) {
#pragma unroll
    for (int j = 0; j < C::kLoads; ++j) issue_one(j);
    next_tile();
  }
  wait_vmcnt<(S - 2) * C::kLoads>();  // K tile 0 (and the parameters) have landed
  lds_barrier();
  // keeps the compiler from sinking the parameter loads past the loop
  asm volatile("" : "+v"(p_s), "+v"(p_b), "+v"(p_x), "+v"(p_z));
#pragma unroll
  for (int j = 0; j < C::kLoads; ++j)
    if (j < upto(kMfma)) issue_one(j);
#pragma unroll
  for (int f = 0; f < C::kFN; ++f)
    fa[0][f] = *reinterpret_cast<const v4i *>(smem + a_base + f * 32 * BK + frag_off[0]);
#pragma unroll
  for (int g = 0; g < C::kFM; ++g)
    fb[0][g] = *reinterpret_cast<const v4i *>(smem + b_base + g * 32 * BK + frag_off[0]);
  int r_slot = 0;  // stage of tile kt
  for (int kt = 0; kt < KT; ++kt) {
    const int8_t *st = smem + r_slot * C::kStage;
#pragma unroll
    for (int s = 0; s + 1 < C::kSteps; ++s)
      kstep(s & 1, s, st, s + 1, (s + 1) & 1, kMfma * (s + 1));
    r_slot = r_slot + 1 == S ? 0 : r_slot + 1;
    next_tile();
    // this wave's reads of tile kt are done once lgkmcnt drains, tile kt+1 has
    // landed once at most S-2 younger tiles are in flight; after the barrier
    // tile kt's stage takes tile kt+S
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    wait_vmcnt<(S - 2) * C::kLoads>();
    lds_barrier();
    kstep(1, C::kSteps - 1, smem + r_slot * C::kStage, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
  wait_vmcnt<0>();                     // the trailing out-of-range loads
  __builtin_amdgcn_s_waitcnt(0xC07F);  // this wave's last fragment reads
  lds_barrier();                       // every wave is done with the ring

  // ---- K groups' partial sums, parameters and token sums through LDS -----------
  v4i *red = reinterpret_cast<v4i *>(smem);
  uint16_t *tile = reinterpret_cast<uint16_t *>(smem + C::kRed);
  float *par = reinterpret_cast<float *>(smem + C::kRed + C::kOut);
  float *l_s = par, *l_b = par + BN, *l_x = par + 3 * BN;
  int *l_z = reinterpret_cast<int *>(par + 2 * BN);
  int *sums = reinterpret_cast<int *>(smem + C::kRed + C::kOut + C::kParams);
#pragma unroll
  for (int b = 0; b < kMfma; ++b) {
    const int o = b % WK, n = b / WK;  // owning K group and its n-th block
    if (WK == 1 || o == kg) continue;
    const int w = kg < o ? kg : kg - 1;  // this group among the owner's writers
    v4i *dst = red + (((pos * WK + o) * (WK - 1) + w) * C::kOwn + n) * 256 + lane;
    const v16i a = acc[b / C::kFM][b % C::kFM];
#pragma unroll
    for (int r = 0; r < 4; ++r)
      dst[r * 64] = v4i{a[4 * r], a[4 * r + 1], a[4 * r + 2], a[4 * r + 3]};
  }
  if (tid < BN) {
    l_s[tid] = p_s;
    l_b[tid] = p_b;
    if constexpr (EPI == kEpiAsym) l_z[tid] = p_z;
  }
  if constexpr (EPI == kEpiToken) {
    if (tid < BM) l_x[tid] = p_x;
  }
  if constexpr (EPI == kEpiAsym) {
#pragma unroll
    for (int g = 0; g < C::kFM; ++g) {
      const int t = rs[g] + __shfl_xor(rs[g], 32);  // the two halves of a K step
      if (lane < 32) sums[(wave * C::kFM + g) * 32 + lane] = t;
    }
  }
  __builtin_amdgcn_s_waitcnt(0xC07F);
  lds_barrier();

  // ---- dequantize this wave's blocks into the fp16 output tile ------------------
  // Lane l of a 32x32 block holds token l mod 32 and, in registers 4j..4j+3,
  // channels 8j + 4 (l / 32) .. +3.  The 8-byte unit u of tile row r sits at
  // unit u ^ h(r), which spreads the lanes of a write over the banks.
  constexpr int kUnits = BN / 4;
  constexpr int kSwz = kUnits % 16 == 0 ? 16 : 8;
  static_assert(kUnits % kSwz == 0, "the swizzle permutes whole groups of units");
  auto stage_swz = [](int r) { return kSwz == 16 ? (r & 15) : ((r >> 1) & 7); };
#pragma unroll
  for (int n = 0; n < C::kOwn; ++n) {
    if (kMfma % WK != 0 && n * WK + kg >= kMfma) continue;
    const int b = n * WK + kg;
    v16i a = acc[n * WK / C::kFM][n * WK % C::kFM];
#pragma unroll
    for (int w = 1; w < WK; ++w)
      if (n * WK + w < kMfma && kg == w) a = acc[(n * WK + w) / C::kFM][(n * WK + w) % C::kFM];
#pragma unroll
    for (int w = 0; w < WK - 1; ++w)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const v4i v = red[(((pos * WK + kg) * (WK - 1) + w) * C::kOwn + n) * 256 + r * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) a[4 * r + e] += v[e];
      }
    const int row = wm * C::kTM + (b % C::kFM) * 32 + fr;  // token within the tile
    const float sx = EPI == kEpiToken ? l_x[row] : 0.f;
    int tsum = 0;
    if constexpr (EPI == kEpiAsym) {
#pragma unroll
      for (int k = 0; k < WK; ++k)
#pragma unroll
        for (int w = 0; w < WN; ++w)
          tsum += sums[(((k * WM + wm) * WN + w) * C::kFM + b % C::kFM) * 32 + fr];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int nl = wn * C::kTN + (b / C::kFM) * 32 + 8 * j + 4 * fh;  // channel within the tile
      const float4 s4 = *reinterpret_cast<const float4 *>(l_s + nl);
      const float4 b4 = *reinterpret_cast<const float4 *>(l_b + nl);
      int a0 = a[4 * j], a1 = a[4 * j + 1], a2 = a[4 * j + 2], a3 = a[4 * j + 3];
      if constexpr (EPI == kEpiAsym) {
        const int4 z4 = *reinterpret_cast<const int4 *>(l_z + nl);
        a0 -= z4.x * tsum;
        a1 -= z4.y * tsum;
        a2 -= z4.z * tsum;
        a3 -= z4.w * tsum;
      }
      if (acc_out != nullptr && m0 + row < M) {  // test path: the raw sums too
        int32_t *dst = acc_out + (int64_t)(m0 + row) * N + n0 + nl;
        if (n0 + nl + 0 < N) dst[0] = a0;
        if (n0 + nl + 1 < N) dst[1] = a1;
        if (n0 + nl + 2 < N) dst[2] = a2;
        if (n0 + nl + 3 < N) dst[3] = a3;
      }
      uint2 h;
      h.x = (uint32_t)dequant_x<EPI>(a0, sx, s4.x, b4.x) |
            ((uint32_t)dequant_x<EPI>(a1, sx, s4.y, b4.y) << 16);
      h.y = (uint32_t)dequant_x<EPI>(a2, sx, s4.z, b4.z) |
            ((uint32_t)dequant_x<EPI>(a3, sx, s4.w, b4.w) << 16);
      *reinterpret_cast<uint2 *>(tile + row * BN + 4 * ((nl >> 2) ^ stage_swz(row))) = h;
    }
  }
  __builtin_amdgcn_s_waitcnt(0xC07F);
  lds_barrier();

  // ---- whole token rows out, 16 bytes per lane -----------------------------------
  constexpr int kCpr = BN / 8;  // 16-byte chunks per row
#pragma unroll 2
  for (int c = tid; c < BM * kCpr; c += C::kThreads) {
    const int r = c / kCpr, cc = c % kCpr;
    const int x = stage_swz(r);
    uint4 v = *reinterpret_cast<const uint4 *>(tile + r * BN + (cc ^ (x >> 1)) * 8);
    if (x & 1) {  // the two 8-byte units of the pair are stored swapped
      const uint32_t t0 = v.x, t1 = v.y;
      v.x = v.z; v.y = v.w; v.z = t0; v.w = t1;
    }
    const int n = n0 + cc * 8;
    if (m0 + r < M) {
      uint16_t *dst = Y + (int64_t)(m0 + r) * N + n;
      if ((N & 7) == 0 && n + 7 < N) {
        *reinterpret_cast<uint4 *>(dst) = v;
      } else {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
        for (int i = 0; i < 8; ++i)
          if (n + i < N) dst[i] = (uint16_t)(w[i >> 1] >> (16 * (i & 1)));
      }
    }
  }
}

// One workgroup per CU: the ring takes the LDS.
template <int BN, int BM, int BK, int WN, int WM, int WK, int S, int EPI>
__global__ __launch_bounds__(64 * WN * WM * WK, 1) void qgemm_ring_kernel(
    const int8_t *__restrict__ Xq, const int8_t *__restrict__ Wq, const float *__restrict__ sX,
    const int32_t *__restrict__ zW, const float *__restrict__ sW, const float *__restrict__ bp,
    int M, int N, int K, uint16_t *__restrict__ Y, int32_t *__restrict__ acc_out, int tiles_m,
    int tiles_n) {
  __shared__ __attribute__((aligned(1024)))
  int8_t smem[RingCfg<BN, BM, BK, WN, WM, WK, S>::kSmem];
  ring_body<BN, BM, BK, WN, WM, WK, S, EPI>(smem, Xq, Wq, sX, zW, sW, bp, M, N, K, Y, acc_out,
                                            tiles_m, tiles_n);
}

template <int BN, int BM, int BK, int WN, int WM, int WK, int S>
hipError_t launch_ring(const int8_t *Xq, const int8_t *Wq, const float *sX, const int32_t *zW,
                       const float *sW, const float *bp, int64_t M, int64_t N, int64_t K,
                       uint16_t *Y, int32_t *acc_out, hipStream_t st) {
  const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (int)((N + BN - 1) / BN);
  const unsigned grid = (unsigned)(tiles_m * tiles_n);
  const dim3 block(64 * WN * WM * WK);
  if (sX)
    qgemm_ring_kernel<BN, BM, BK, WN, WM, WK, S, kEpiToken><<<grid, block, 0, st>>>(
        Xq, Wq, sX, zW, sW, bp, (int)M, (int)N, (int)K, Y, acc_out, tiles_m, tiles_n);
  else if (zW)
    qgemm_ring_kernel<BN, BM, BK, WN, WM, WK, S, kEpiAsym><<<grid, block, 0, st>>>(
        Xq, Wq, sX, zW, sW, bp, (int)M, (int)N, (int)K, Y, acc_out, tiles_m, tiles_n);
  else
    qgemm_ring_kernel<BN, BM, BK, WN, WM, WK, S, kEpiChannel><<<grid, block, 0, st>>>(
        Xq, Wq, sX, zW, sW, bp, (int)M, (int)N, (int)K, Y, acc_out, tiles_m, tiles_n);
  return hipGetLastError();
}

}  // namespace detail

using namespace detail;

// Tiles and their rings: waves WN x WM x WK, K tile, stages.  From a sweep of
// 23 configurations of 17 tile shapes; of two shapes that win in turn within
// 1 % the smaller set is kept.
hipError_t launch_qgemm_ring(int bn, int bm, const int8_t *Xq, const int8_t *Wq, const float *sX,
                             const int32_t *zW, const float *sW, const float *bp, int64_t M,
                             int64_t N, int64_t K, uint16_t *Y, int32_t *acc_out,
                             hipStream_t st) {
#define OT_RING(BN, BM, BK, WN, WM, WK, S) \
  if (bn == BN && bm == BM)                \
  return launch_ring<BN, BM, BK, WN, WM, WK, S>(Xq, Wq, sX, zW, sW, bp, M, N, K, Y, acc_out, st)
  OT_RING(256, 128, 128, 4, 2, 1, 3);
  OT_RING(192, 128, 128, 2, 2, 2, 3);
  OT_RING(128, 128, 128, 2, 2, 2, 4);
  OT_RING(128, 96, 128, 2, 1, 2, 5);
  OT_RING(64, 128, 256, 1, 2, 4, 3);
  OT_RING(64, 64, 256, 1, 1, 4, 4);
  OT_RING(32, 64, 256, 1, 1, 4, 5);
  OT_RING(32, 32, 256, 1, 1, 4, 8);
#undef OT_RING
  return hipErrorInvalidValue;
}

}  // namespace ot
