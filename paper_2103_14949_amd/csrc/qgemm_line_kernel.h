// (The file that includes this has said which kind of results it is for: kOut.)
// Dense int8 GEMM on large tiles: operands stream from global memory straight into LDS in k-stages of 128 bytes.
//
// D[i][j] = sum_k P[i][k] Q[j][k], P = weights [N,K], Q = activations [M,K]; LDS layout, zero-point term and epilogue as in
// qgemm_dma.hip, whose ring of four 64-byte stages served these tiles before.
//
// What bounds it.  A 192 x 256 tile of K = 768 fetches 344 KB from L2 into one CU's LDS while its SIMDs have 9 216 cycles of
// matrix instructions (5.8 us at the 1.6 GHz that the board holds under them).  What the L2 holds reaches the LDS at
// 130 GB/s per CU, but most of a line's first readers wait for it to come from memory: with 64-byte stages, which fetch a
// line in two halves and have a barrier for each, the main loop took 8.15 us, 42 GB/s per CU.
// Two slots of 128-byte stages (112 KB of LDS for 192 rows of weights and 256 of activations) leave a stage's loads almost
// a whole stage of matrix instructions to land in.  For that the wavefronts must be done with a slot early: fragments are
// double-buffered by 32-k groups, the reads of a group go out behind the matrix instructions of the one before, so that
// before its last group a stage has been read completely.  The one barrier per stage lies there, half as many per k.
// (Lanes beyond K are masked in both operands, stream_offset.h: 4096 x 784 -> 3072 17.5 us, 17.7 with the weights alone masked.)
// us, 64-byte stages and here (u8, both with the present epilogue): 4096 x 768 -> 3072 15.5, 14.6; -> 2304 13.4, 12.6;
// 4096 x 4096 -> 4096 (256 x 256 tiles) 65, 62.  128 x 256 tiles serve layers that fill the chip with neither larger ones nor
// one round of 128 x 128: 2048 x 768 -> 3072 10.1 (13.6), 2048 x 1024 -> 4096 13.5 (21.6), 3000 x 512 -> 2048 8.2 (11.2).  Now the main loop is 7.6 of 13.0 us of a workgroup at N = 3072, start 1.3,
// channel terms 0.8, requantize 1.7, copy-out 0.5, and 2.3 lie between two launches.
#pragma once

#include "qgemm_dma.h"
#include "qgemm_stream.h"

namespace hago {

namespace {

template <int WP, int WQ, int TP, int TQ, bool FLIP, int OUT>
__global__ __launch_bounds__(64 * WP * WQ, 1) void qgemm_line_kernel(QgemmParams p) {
  constexpr int BK = 128, NH = 4;   // bytes and 32-k groups of a stage
  constexpr int RPI = 8, CPR = 8;   // rows of a DMA instruction, 16-byte chunks of a row
  constexpr int NW = WP * WQ, NT = 64 * NW;
  constexpr int BP = WP * TP * 32, BQ = WQ * TQ * 32;
  constexpr int STAGE = (BP + BQ) * BK;
  constexpr int GP = BP / RPI, G = (BP + BQ) / RPI;  // row groups (one DMA instruction each): of P, in all
  constexpr int L = G / NW;                          // a wavefront issues groups wave, wave + NW, ...
  static_assert(GP % NW == 0 && G % NW == 0, "a slot's operand is the same in every wavefront");
  constexpr int NM = TP * TQ;                        // matrix instructions of a 32-k group
  constexpr int WBLK = BP / 32;                      // 32-row blocks of the weight tile
  static_assert(WBLK <= NW, "one wavefront sums a block's rows");
  HAGO_STAMP(p, 7);

  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  int32_t* s_corr = reinterpret_cast<int32_t*>(smem + 2 * STAGE);
  int32_t* s_mult = s_corr + BP;
  int32_t* s_shift = s_mult + BP;
  int64_t* s_c64 = reinterpret_cast<int64_t*>(s_shift + BP);
  int32_t* s_shm1 = reinterpret_cast<int32_t*>(s_c64 + BP);  // shift - 1
  __shared__ int32_t s_vote;

  const int t = threadIdx.x;
  if (t == 0) s_vote = 0;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wp = wave % WP, wq = wave / WP;
  int tile_p, tile_q;
  panel_tile((int)xcd_run(blockIdx.x, gridDim.x), (p.N + BP - 1) / BP, (p.M + BQ - 1) / BQ, tile_p, tile_q);
  const int p0 = tile_p * BP, q0 = tile_q * BQ;

  const v4i rs_w = make_rsrc(p.wgt, (uint32_t)p.N * (uint32_t)p.K);
  const v4i rs_a = make_rsrc(p.act, (uint32_t)p.M * (uint32_t)p.K);
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t*)smem;
  const uint32_t wave_lds = lds0 + (uint32_t)wave * 1024u;

  // the lane's byte offset of every DMA slot: its row's start and its chunk of a stage (every group of a wavefront has the
  // wavefront's parity, so the chunk is the same in every slot)
  const int lrow = lane / CPR;
  const int lck = ((lane % CPR) ^ swz<BK>((wave & 1) * 8 + lrow)) * 16;
  uint32_t voff[L];
#pragma unroll
  for (int d = 0; d < L; ++d) {
    const bool isq = d >= GP / NW;
    const int row = (isq ? q0 - BP : p0) + (wave + NW * d) * RPI + lrow;
    voff[d] = stream_row_offset(row, isq ? p.M : p.N, p.K, lck);
  }
  const int KT = (p.K + BK - 1) / BK;
  // DMA instructions lo .. hi - 1 of a stage.  Lanes beyond K, in the stage that K ends inside and in the ones behind it, get
  // an offset beyond the tensor and write zeros.
  auto issue = [&](int stage, auto slot, auto lo, auto hi) {
    const int k0 = stage * BK;
    [&]<int... I>(std::integer_sequence<int, I...>) {
      ([&] {
        constexpr int d = decltype(lo)::value + I;
        dma16s(d >= GP / NW ? rs_a : rs_w, wave_lds + (uint32_t)(decltype(slot)::value * STAGE + NW * d * 1024),
               stream_lane_offset(voff[d], k0, lck, p.K), stream_scalar_offset(k0, p.K));
      }(), ...);
    }(std::make_integer_sequence<int, decltype(hi)::value - decltype(lo)::value>{});
  };
  template_int<0> i0;
  template_int<1> i1;
  HAGO_STAMP(p, 0);
  issue(0, i0, i0, template_int<L>{});
  issue(1, i1, i0, template_int<L>{});
  HAGO_STAMP(p, 1);
  __builtin_amdgcn_sched_barrier(0);
  ChannelRegs<NT, BP> chregs;
  load_channel_regs<NT, BP>(p, p0, chregs);

  v16i acc[TP][TQ];
#pragma unroll
  for (int i = 0; i < TP; ++i)
#pragma unroll
    for (int j = 0; j < TQ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

  // fragment addresses inside a stage: one register per operand and 32-k group
  const int frow = lane & 31, fhalf = lane >> 5;
  int pa[NH], qa[NH], sa[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    const int chunk = ((h * 2 + fhalf) ^ swz<BK>(frow & 15)) * 16;
    pa[h] = (wp * TP * 32 + frow) * BK + chunk;
    qa[h] = BP * BK + (wq * TQ * 32 + frow) * BK + chunk;
    sa[h] = ((wave < WBLK ? wave : WBLK - 1) * 32 + frow) * BK + chunk;  // the 32 weight rows this wavefront sums
  }
  constexpr int kFrag = 32 * BK;
  v4i pf[2][TP], qf[2][TQ], sd;
  uint32_t wsum = 0;  // biased: every byte counts as w + 128
  auto flip1 = [&](v4i& f, int u) {
    int x = f[u];
    asm volatile("v_xor_b32 %0, %1, %0" : "+v"(x) : "s"(p.act_xor4));
    f[u] = x;
  };
  auto sum1 = [&](int u) { wsum = __builtin_amdgcn_sad_u8((uint32_t)sd[u] ^ 0x80808080u, 0u, wsum); };
  // read r of the NR of a group's operands: activations (which are flipped), weights, the rows to sum
  constexpr int NR = TQ + TP + 1;
  auto read = [&](const uint8_t* base, auto set, auto group, int r) {
    constexpr int S = decltype(set)::value, H = decltype(group)::value;
    if (r < TQ) qf[S][r] = *reinterpret_cast<const v4i*>(base + qa[H] + r * kFrag);
    else if (r < TQ + TP) pf[S][r - TQ] = *reinterpret_cast<const v4i*>(base + pa[H] + (r - TQ) * kFrag);
    else sd = *reinterpret_cast<const v4i*>(base + sa[H]);
  };
  // Group H of a stage: multiply its set of fragments.  Behind the matrix instructions go the reads of the next group's set
  // (from `next`), then its flips and sums, and in the last group of a stage the DMA instructions of stage `dma_stage`.
  auto multiply = [&](auto hconst, const uint8_t* next, int dma_stage, auto dma_slot) {
    constexpr int H = decltype(hconst)::value, S = H & 1, HN = (H + 1) % NH;
    [&]<int... Mi>(std::integer_sequence<int, Mi...>) {
      ([&] {
        constexpr int m = Mi, j = m / TP, i = m % TP;
        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(pf[S][i], qf[S][j], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        // two reads behind each of the first instructions
#pragma unroll
        for (int r = 2 * m; r < 2 * m + 2 && r < NR; ++r) read(next, template_int<(S ^ 1)>{}, template_int<HN>{}, r);
        constexpr int lo = NM / 2;
        if constexpr (FLIP && m >= lo) {
#pragma unroll
          for (int e = 4 * TQ * (m - lo) / (NM - lo); e < 4 * TQ * (m - lo + 1) / (NM - lo); ++e) flip1(qf[S ^ 1][e / 4], e % 4);
        }
        if constexpr (m >= NM - 2) {
          sum1(2 * (m - (NM - 2)));
          sum1(2 * (m - (NM - 2)) + 1);
        }
        if constexpr (H == NH - 1)
          issue(dma_stage, dma_slot, template_int<m * L / NM>{}, template_int<(m + 1) * L / NM>{});
        __builtin_amdgcn_sched_barrier(0);
      }(), ...);
    }(std::make_integer_sequence<int, NM>{});
  };
  // Stage kt in slot R.  Before its last group every wavefront has all of its fragments, and the next stage has landed: the
  // barrier says both, the next group's fragments come from the other slot, and this slot takes stage kt + 2.  (After the last
  // stage follows one of zeros, whose first group is read and not multiplied.)
  auto stage_body = [&](int kt, auto ring) {
    constexpr int R = decltype(ring)::value;
    const uint8_t* here = smem + R * STAGE;
    const uint8_t* other = smem + (R ^ 1) * STAGE;
    multiply(template_int<0>{}, here, 0, ring);
    multiply(template_int<1>{}, here, 0, ring);
    multiply(template_int<2>{}, here, 0, ring);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    multiply(template_int<3>{}, other, kt + 2, ring);
  };

  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(L) : "memory");  // stage 0
  __syncthreads();
  HAGO_STAMP(p, 2);
#pragma unroll
  for (int r = 0; r < NR; ++r) read(smem, i0, i0, r);
  if constexpr (FLIP) {
#pragma unroll
    for (int e = 0; e < 4 * TQ; ++e) flip1(qf[0][e / 4], e % 4);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) sum1(u);
  for (int kt = 0; kt < KT; kt += 2) {
    stage_body(kt, i0);
    if (kt + 1 < KT) stage_body(kt + 1, i1);
  }
  HAGO_STAMP(p, 3);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the stage beyond K; before LDS is reused)

  // the two 32-lane halves hold the two halves of each 32-k group of a row
  int32_t v = (int32_t)(wsum - (uint32_t)(KT * NH + 1) * (uint32_t)(16 * 128));
  v += __shfl_xor(v, 32);
  if (wave < WBLK && fhalf == 0) s_corr[wave * 32 + frow] = v;
  __syncthreads();
  const int form = finish_channel_terms<NT, BP, OUT>(p, chregs, s_corr, s_mult, s_shift, s_c64, &s_vote, nullptr, s_shm1);
  HAGO_STAMP(p, 4);
  static_assert(BQ * (BP + 16) <= 2 * STAGE && (BQ * BP / 16) % NT == 0, "the results are staged in the ring's place");
  if constexpr (OUT == kOutOther) {
    qgemm_epilogue<WP, WQ, TP, TQ, false>(p, acc, p0, q0, s_corr, s_mult, s_shift);
  } else {
    constexpr int kFast = OUT == kOutFull ? kRqSat : kRqFolded;
    if (form == kFast)
      qgemm_epilogue_dense_staged<WP, WQ, TP, TQ, kFast>(p, acc, p0, q0, s_corr, s_mult, s_shift, s_c64, s_shm1, smem);
    else if (OUT == kOutFull && form == kRqFolded)
      qgemm_epilogue_dense_staged<WP, WQ, TP, TQ, kRqFolded>(p, acc, p0, q0, s_corr, s_mult, s_shift, s_c64, s_shm1, smem);
    else
      qgemm_epilogue_dense_staged<WP, WQ, TP, TQ, kRqGeneral>(p, acc, p0, q0, s_corr, s_mult, s_shift, s_c64, s_shm1, smem);
  }
}

template <int WP, int WQ, int TP, int TQ>
hipError_t launch_line(const QgemmParams& p, hipStream_t st) {
  constexpr int BP = WP * TP * 32, BQ = WQ * TQ * 32;
  constexpr size_t lds = 2 * (size_t)(BP + BQ) * 128 + 6 * BP * sizeof(int32_t);
  const int64_t tiles = (int64_t)((p.N + BP - 1) / BP) * ((p.M + BQ - 1) / BQ);
  auto run = [&]<bool FLIP>() {
    const auto kern = qgemm_line_kernel<WP, WQ, TP, TQ, FLIP, kOut>;
    static std::atomic<uint64_t> attr_set{0};  // per kernel: the devices whose dynamic-LDS limit is raised
    const hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), (int)lds, attr_set);
    if (e != hipSuccess) return e;
    return launch_kernel(kern, dim3((unsigned)tiles), dim3(64 * WP * WQ), lds, st, p);
  };
  return p.act_xor4 ? run.template operator()<true>() : run.template operator()<false>();
}

}  // namespace

template <>
hipError_t qdense_line<kOut>(const QgemmParams& p, int shape, hipStream_t st) {
  switch (shape) {
    case 1: return launch_line<2, 4, 3, 2>(p, st);   // 192 x 256
    case 5: return launch_line<2, 4, 2, 2>(p, st);   // 128 x 256
    default: return launch_line<2, 4, 4, 2>(p, st);  // 256 x 256
  }
}

}  // namespace hago
