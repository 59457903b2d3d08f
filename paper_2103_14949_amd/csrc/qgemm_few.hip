// Dense GEMM for few output tiles: operands of any size and alignment, int8 and int16.  A workgroup owns ONE 32 x 32 tile and its
// wavefronts split the reduction: wavefront w takes blocks w, w + NW, ... of 128 bytes of all 64 rows, which it loads into an
// LDS slot of its own (two, so one block is under way behind the one in use), with no barrier until the partial sums meet.
//
// What bounds it is one chain: launch, arguments, first load, reduction, partial sums, requantize, store.
//   * Loads go to LDS (eight rows of 128 contiguous bytes each, 25 cycles of the CU's memory pipe) and not straight into the
//     fragments' registers, where every lane has a row of its own (64 cycles, 256 off four bytes); that form took 7.7 us for
//     128 x 3072 -> 768, this one 4.3.  Four loads share a value of m0, whose write behind a load into LDS holds the wavefront
//     for about 110 cycles.
//   * A wavefront that is alone on its SIMD issues an instruction every four to five cycles, so set-up counts: one offset per
//     load is kept and blocks add to it, rows beyond the operands come out of the descriptors' range check (which is exact to
//     the dword, also where the last row ends inside a block), and K needs a mask only in its last 32 elements.
//   * What the first loads need is in scalar registers at the start; the other arguments are fetched in one go behind them.
//   * No barrier in the loop: a form in which all wavefronts shared the stage and had a quarter of the tile each took 6.4 us for
//     128 x 3072 -> 768.
// Rows off a multiple of four bytes (MIS) are loaded from the aligned dwords that hold them, one dword more per row and block, and
// shifted into place behind the LDS (512 x 1283 -> 512 4.5 us, 8.7 by 64 x 64 tiles through registers).
#include "qgemm_any.h"
#include "qgemm_stream.h"

namespace hago {

namespace {

constexpr int kBlock = (int)kRunBlock;           // bytes of a row that a wavefront takes at a time
constexpr int kDepth = 2;                        // such blocks that it has under way
constexpr int kPitch = 576;                      // LDS bytes of the partial sums of four channels (32 rows): no bank conflicts either way

template <bool MIS>
constexpr int slot_bytes() { return 64 * kBlock + (MIS ? 512 : 0); }

// Eight rows of a block per load, four loads per value of m0: window i takes the instruction offset i KB, which counts on both
// sides (the lane offsets take it back, run_offset).
__device__ __forceinline__ void load_run(const v4i& r, uint32_t lds_addr, uint32_t o0, uint32_t o1, uint32_t o2, uint32_t o3) {
  asm volatile(
      "s_mov_b32 m0, %0\n\ts_nop 0\n\t"
      "buffer_load_dwordx4 %1, %5, 0 offen lds\n\t"
      "buffer_load_dwordx4 %2, %5, 0 offen offset:1024 lds\n\t"
      "buffer_load_dwordx4 %3, %5, 0 offen offset:2048 lds\n\t"
      "buffer_load_dwordx4 %4, %5, 0 offen offset:3072 lds"
      :
      : "s"(lds_addr), "v"(o0), "v"(o1), "v"(o2), "v"(o3), "s"(r)
      : "memory", "m0");
}
__device__ __forceinline__ void load_dword(const v4i& r, uint32_t lds_addr, uint32_t o) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" : : "s"(lds_addr), "v"(o), "s"(r) : "memory", "m0");
}

// What the kernel needs of a layer's parameters: with the scalars in front of them the arguments are 108 bytes (kCheapArguments).
struct FewParams {
  const int32_t* bias;
  void* out;
  const int32_t* mult;
  const int32_t* shift;
  int32_t corr_coef, z_out, lo_rel, hi_rel;
  uint32_t flags;
};
static_assert(56 + sizeof(FewParams) <= kCheapArguments);
enum : uint32_t { kPerChannel = 1, kHalfAway = 2, kFlip = 4, kHalves = 8 };  // and, from bit 8 on, acc_wrap_shift

inline FewParams few_params(const QgemmParams& p) {
  return FewParams{p.bias, p.out, p.mult, p.shift, p.corr_coef, p.rs.z_out, p.rs.lo_rel, p.rs.hi_rel,
                   (p.per_channel ? kPerChannel : 0u) | (p.rs.half_away ? kHalfAway : 0u) | (p.act_xor4 ? kFlip : 0u) | (p.out_mode == 2 ? kHalves : 0u) |
                       (uint32_t)p.acc_wrap_shift << 8};
}

// The first 14 dwords of the arguments are in scalar registers when a wavefront starts; the others, in `q`, take as long as a
// load from memory.  KB: bytes of a row.  minor: tiles of the index that runs first, bit 31: that is the channels'.  KIND: bit 0: int16,
// bit 1: codes go out, else sums (one number, as the tests of the routes know a kernel by the third); us in one kernel for both and so: 8081 x 112 ->
// 123 4.05, 3.8; 128 x 3072 -> 768 4.45, 4.32; 64 x 256 -> 128 2.77, 2.68, raw 2.60, 2.53.
template <int KIND, bool MIS, int NW>
__global__ __launch_bounds__(64 * NW, 2) void qgemm_few_kernel(const uint8_t* act, const int8_t* wgt, int M, int N, uint32_t KB,
                                                                    int blocks, uint32_t count, uint32_t minor, uint32_t inv_minor,
                                                                    uint32_t size_w, uint32_t size_a, FewParams q) {
  constexpr bool I16 = KIND & 1, RQ = KIND & 2;
  constexpr int SLOT = slot_bytes<MIS>(), L = MIS ? 10 : 8;  // loads of a block
  constexpr int GB = I16 ? 64 : 32, NG = kBlock / GB;        // bytes of 32 elements; 32-k groups of a block
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  uint32_t m0, n0;
  {
    const uint32_t id = xcd_run(blockIdx.x, count), of = minor & 0x7fffffffu;
    const uint32_t major = inv_minor ? __umulhi(id, inv_minor) : id, rest = id - major * of;
    m0 = (minor >> 31 ? major : rest) * 32;
    n0 = (minor >> 31 ? rest : major) * 32;
  }
  // Descriptors of the whole dwords that hold the operands: rows beyond them, and what lies behind the last, read as zeros.
  // A block reaches into the next row where KB ends inside it: there the weights are cleared.
  const uint32_t w_at = MIS ? (uint32_t)reinterpret_cast<uintptr_t>(wgt) & 3u : 0u;
  const uint32_t a_at = MIS ? (uint32_t)reinterpret_cast<uintptr_t>(act) & 3u : 0u;
  const v4i rs_w = make_run_rsrc(reinterpret_cast<const uint8_t*>(wgt) - w_at, size_w);
  const v4i rs_a = make_run_rsrc(act - a_at, size_a);
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t*)smem + (uint32_t)wave * SLOT;
  // the lane's offsets: rows 8 i + lane / 8 of either operand; MIS: of the dwords behind a block, row lane % 32
  uint32_t off_w[4], off_a[4], more_w = 0, more_a = 0;
  {
    const uint32_t base_w = n0 * KB + w_at, base_a = m0 * KB + a_at;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      off_w[i] = run_offset(base_w, KB, (uint32_t)lane, i, MIS);
      off_a[i] = run_offset(base_a, KB, (uint32_t)lane, i, MIS);
    }
    if constexpr (MIS) {
      more_w = run_behind_offset(base_w, KB, (uint32_t)lane);
      more_a = run_behind_offset(base_a, KB, (uint32_t)lane);
    }
  }
  auto issue = [&](int b, int slot) {
    const uint32_t k = (uint32_t)b * kBlock, dst = lds0 + (uint32_t)(slot * NW * SLOT);
    load_run(rs_w, dst, off_w[0] + k, off_w[1] + k, off_w[2] + k, off_w[3] + k);
    load_run(rs_a, dst + 32 * kBlock, off_a[0] + k, off_a[1] + k, off_a[2] + k, off_a[3] + k);
    if constexpr (MIS) {
      load_dword(rs_w, dst + 64 * kBlock, more_w + k);
      load_dword(rs_a, dst + 64 * kBlock + 256, more_a + k);
    }
  };
  // (kept, so that a later block's loads need nothing but an addition each)
#pragma unroll
  for (int i = 0; i < 4; ++i) asm("" : "+v"(off_w[i]), "+v"(off_a[i]));
  if constexpr (MIS) asm("" : "+v"(more_w), "+v"(more_a));
  if (wave < blocks) issue(wave, 0);
  if (wave + NW < blocks) issue(wave + NW, 1);
  __builtin_amdgcn_sched_barrier(0);

  // while the first loads are under way: what needs no further argument, and the other arguments
  const int frow = lane & 31, fhalf = lane >> 5;
  int place = frow * kBlock + ((frow >> 1) & 7) * 16;  // chunk c of the lane's row lies at place ^ 16 c
  uint32_t sh_w = MIS ? (n0 + frow) * KB + w_at : 0u, sh_a = MIS ? (m0 + frow) * KB + a_at : 0u;
  Tile32<I16> acc;
  acc.clear();
#pragma unroll
  for (v16i& a : acc.a) asm volatile("" : "+v"(a));
  asm volatile("" : "+v"(place), "+v"(sh_w), "+v"(sh_a));
  fetch_arguments<56 + sizeof(FewParams)>();
  QgemmParams p{};
  p.bias = q.bias, p.out = q.out, p.mult = q.mult, p.shift = q.shift, p.N = N;
  p.per_channel = q.flags & kPerChannel ? 1 : 0;
  p.acc_wrap_shift = (int32_t)(q.flags >> 8);
  p.out_mode = RQ ? 0 : (q.flags & kHalves ? 2 : 1);
  p.act_xor4 = q.flags & kFlip ? 0x80808080u : 0u;
  p.corr_coef = q.corr_coef;
  p.rs = RequantScalars{q.z_out, q.lo_rel, q.hi_rel, q.flags & kHalfAway ? 1 : 0};
  // finishing threads: row t / 8, channels 4 (t % 8) ..
  const int fr = t >> 3, fc = t & 7, m = (int)m0 + fr, n = (int)n0 + 4 * fc;
  v4i c_bias = {0, 0, 0, 0};
  if (wave < 4) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(p.bias), 0, p.bias ? 4 * N : 0, 0x00020000);
    c_bias = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(r, 4 * n, 0, 0));
  }
  // Multipliers and shifts: a dword per lane, by one wavefront for all through its slot.  (16 bytes per finishing thread, as the
  // bias, are eight loads of a tile for these two, which the operands of the CU's other tiles wait for: 8081 x 112 -> 123 4.6 us, 4.2 so;
  // 5523 x 128 -> 34 3.7, 3.4; 13945 x 42 -> 42 4.5, 4.0; over 1300 layers 0.98 where requantized.  The bias so too: raw layers 3 % slower.)
  int32_t c_mult = 0, c_shift = 0;
  if (RQ && wave == 0) {
    const int bytes = p.per_channel ? 4 * N : 4, at = p.per_channel ? 4 * ((int)n0 + frow) : 0;
    const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(p.mult), 0, p.mult ? bytes : 0, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(p.shift), 0, bytes, 0x00020000);
    c_mult = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rm, at, 0, 0);
    c_shift = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, at, 0, 0);
  }
  const uint32_t x4 = p.act_xor4;
  const bool need_wsum = I16 || p.corr_coef != 0;
  int32_t wsum = 0, asum = 0;
  constexpr int NV = GB / 32;   // 16-byte chunks of a lane and group
  struct Group { v4i w[NV], a[NV]; uint32_t mw, ma; };
  auto read = [&](const uint8_t* s, int h, Group& x) {
    const int c0 = (2 * h + fhalf) * NV;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      x.w[i] = *reinterpret_cast<const v4i*>(s + (place ^ (16 * (c0 + i))));
      x.a[i] = *reinterpret_cast<const v4i*>(s + (place ^ (16 * (c0 + i))) + 32 * kBlock);
    }
    if constexpr (MIS) {
      const bool inside = h < NG - 1 || fhalf == 0;
      const int next = inside ? place ^ (16 * (c0 + NV)) : 64 * kBlock + 4 * frow;
      x.mw = *reinterpret_cast<const uint32_t*>(s + next);
      x.ma = *reinterpret_cast<const uint32_t*>(s + next + (inside ? 32 * kBlock : 256));
    }
  };
  auto settle = [&](Group& x) {
    if constexpr (MIS) {
#pragma unroll
      for (int i = 0; i < 4 * NV; ++i) {
        const int d = i & 3, v = i >> 2;
        const uint32_t nw = i + 1 < 4 * NV ? (uint32_t)x.w[(i + 1) >> 2][(i + 1) & 3] : x.mw, na = i + 1 < 4 * NV ? (uint32_t)x.a[(i + 1) >> 2][(i + 1) & 3] : x.ma;
        x.w[v][d] = (int)__builtin_amdgcn_alignbyte(nw, (uint32_t)x.w[v][d], sh_w);
        x.a[v][d] = (int)__builtin_amdgcn_alignbyte(na, (uint32_t)x.a[v][d], sh_a);
      }
    }
    if constexpr (!I16) x.a[0] = xor4(x.a[0], x4);
  };
  // weights beyond the row are zeros; left: bytes of the row from this group on, fewer than it has
  auto cut = [&](Group& x, int left) {
    const int mine = left - GB / 2 * fhalf;
#pragma unroll
    for (int i = 0; i < 4 * NV; ++i) {
      const int bytes = mine - 4 * i, by = bytes > 0 && bytes < 4 ? 32 - 8 * bytes : 0;
      const uint32_t w = (uint32_t)x.w[i >> 2][i & 3] << by >> by;
      x.w[i >> 2][i & 3] = bytes > 0 ? (int)w : 0;
    }
  };
  auto sums = [&](const Group& x) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      wsum = plain_sum<I16>(x.w[i], wsum);
      if constexpr (I16) asum = plain_sum<true>(x.a[i], asum);
    }
  };
  auto multiply = [&](const Group& x) {
    if constexpr (I16) {
      v4i wh, wl, ah, al;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        int h, l;
        split16(x.w[e >> 1][2 * (e & 1)], x.w[e >> 1][2 * (e & 1) + 1], h, l);
        wh[e] = h;
        wl[e] = l;
        split16(x.a[e >> 1][2 * (e & 1)], x.a[e >> 1][2 * (e & 1) + 1], h, l);
        ah[e] = h;
        al[e] = l;
      }
      acc.a[0] = mfma(wh, ah, acc.a[0]);
      acc.a[1] = mfma(wh, al, acc.a[1]);
      acc.a[2] = mfma(wl, al, acc.a[2]);
      acc.a[1] = mfma(wl, ah, acc.a[1]);
    } else {
      acc.a[0] = mfma(x.w[0], x.a[0], acc.a[0]);
    }
  };

  for (int b = wave, slot = 0; b < blocks; b += NW, slot ^= 1) {
    if (b + NW < blocks) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(L) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const uint8_t* const s = smem + (slot * NW + wave) * SLOT;
    const int left = (int)KB - b * kBlock;
    Group x[NG];
#pragma unroll
    for (int h = 0; h < NG; ++h) read(s, h, x[h]);
    if (left >= kBlock) {
#pragma unroll
      for (int h = 0; h < NG; ++h) settle(x[h]);
      if (need_wsum) {  // (uniform)
#pragma unroll
        for (int h = 0; h < NG; ++h) sums(x[h]);
      }
#pragma unroll
      for (int h = 0; h < NG; ++h) multiply(x[h]);
    } else {
#pragma unroll
      for (int h = 0; h < NG; ++h) {
        if (left <= GB * h) break;
        settle(x[h]);
        if (left < GB * (h + 1)) cut(x[h], left - GB * h);
        if (need_wsum) sums(x[h]);
        multiply(x[h]);
      }
    }
    if (b + 2 * NW < blocks) {  // the slot has been read
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      issue(b + 2 * NW, slot);
    }
  }
  // partial sums, four channels by four (channels 8 g + 4 fhalf .. of row frow), and the weights' sums behind them
  const int parts = NW < blocks ? NW : blocks;
  constexpr int kScales = 8 * kPitch + 128;
  if (RQ && wave == 0) *reinterpret_cast<int32_t*>(smem + kScales + 4 * lane) = fhalf ? c_shift : c_mult;
  if (wave < parts) {
    if constexpr (I16) asum += __shfl_xor(asum, 32);
    uint8_t* const s = smem + wave * SLOT + fhalf * kPitch + frow * 16;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      v4i v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = I16 ? (int32_t)((uint32_t)acc.value(4 * g + e) + 128u * (uint32_t)asum) : acc.value(4 * g + e);
      *reinterpret_cast<v4i*>(s + 2 * g * kPitch) = v;
    }
    if (need_wsum) {
      wsum += __shfl_xor(wsum, 32);
      if (fhalf == 0) *reinterpret_cast<int32_t*>(smem + wave * SLOT + 8 * kPitch + 4 * frow) = wsum;
    }
  }
  __syncthreads();
  if (t >= 256 || m >= M || n >= N) return;
  v4i v = c_bias;
  {
    const uint8_t* const s = smem + fc * kPitch + fr * 16;
    for (int w = 0; w < parts; ++w) v += *reinterpret_cast<const v4i*>(s + w * SLOT);
    if (need_wsum) {
      v4i ws = {0, 0, 0, 0};
      for (int w = 0; w < parts; ++w) ws += *reinterpret_cast<const v4i*>(smem + w * SLOT + 8 * kPitch + 16 * fc);
      const uint32_t kpad = (KB + (GB - 1)) / GB * 32u;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = (int32_t)((uint32_t)v[e] + (uint32_t)channel_term<I16>(p, 0, ws[e], (int32_t)kpad));
    }
  }
  if (p.acc_wrap_shift) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = wrap_acc_bits(v[e], p.acc_wrap_shift);
  }
  if constexpr (RQ) {
    const v4i mult = *reinterpret_cast<const v4i*>(smem + kScales + 16 * fc), shift = *reinterpret_cast<const v4i*>(smem + kScales + 128 + 16 * fc);
    const int32_t away = p.rs.half_away ? -1 : 0, lo = p.rs.lo_rel, hi = p.rs.hi_rel, z = p.rs.z_out;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int32_t sh = shift[e] - (p.mult ? 0 : 1), mu = p.mult ? mult[e] : 1 << 30;
      const int64_t pr = (int64_t)v[e] * (int64_t)mu + ((int64_t)1 << (30 + sh)) + (int64_t)((v[e] >> 31) & away);
      v[e] = med3((int32_t)(pr >> (31 + sh)), lo, hi) + z;
    }
  }
  const int32_t out[4] = {v[0], v[1], v[2], v[3]};
  store_four<RQ>(p, m, n, out);
}

}  // namespace

// Its offsets are 32 bits wide, those of the rows of a tile that lie beyond the matrix too.
bool qgemm_few_ok(const QgemmParams& p, bool i16) {
  const int64_t most = (1ll << 31) - (1 << 16), kb = (int64_t)p.K * (i16 ? 2 : 1);
  const int64_t tiles_m = (p.M + 31) / 32, tiles_n = (p.N + 31) / 32;
  return p.K > 0 && ((int64_t)p.N + 32) * kb < most && ((int64_t)p.M + 32) * kb < most &&
         tiles_m * tiles_n * (tiles_m < tiles_n ? tiles_m : tiles_n) < (1ll << 32) && tiles_m * tiles_n <= max_blocks(512);
}

// One round of tiles over the chip, or two workgroups of four wavefronts on a CU, beats the tiles of 64 rows and more at every
// length of the reduction.  With more tiles the larger ones reuse what they load, and only short reductions, whose time is not
// the loads', are faster here; the lines lie higher for rows of no whole 16 bytes, whose other kernel is the slower one, more so
// where a quarter or half of its 64 x 64 tiles is empty, and int16 has none (four products for one).  Over 600 layers of other rows and more
// than 512 tiles the kernel so chosen is 1.2 % from the better one.  Us, here and there:
//   aligned   256 x 768 -> 768 3.1, 4.5; 128 x 3072 -> 768 4.5, 7.8; 512 x 768 -> 768 3.8, 4.55; 986 x 2880 -> 377 6.8, 8.85;
//             972 x 640 -> 759 4.55, 4.8; 1097 x 208 -> 859 3.9, 4.3; but 12465 x 64 -> 50 4.0, 3.4, 12754 x 800 -> 61 6.6, 6.1,
//             1854 x 3072 -> 296 9.2, 8.2, 324 x 64 -> 3208 4.5, 3.8
//   others    512 x 1283 -> 512 4.75, 9.05; 700 x 333 -> 700 3.65, 5.4; 720 x 2163 -> 366 7.8, 10.9; 373 x 471 -> 2901 6.4, 7.9;
//             52673 x 180 -> 4 5.8, 7.85; 5 x 515 -> 16859 4.5, 7.3; 11 x 2853 -> 21142 13.7, 22.7; 7225 x 926 -> 66 raw 7.0, 8.0; but
//             118 x 1769 -> 4294 10.2, 9.7, 20680 x 1023 -> 61 12.2, 10.15, 1481 x 740 -> 1272 9.9, 8.5, 1307 x 1272 -> 433 8.35, 7.2
//   int16     106 x 711 -> 1693 5.4, 6.2; 474 x 2000 -> 659 11.2, 14.2; 119 x 18 -> 2714 3.7, 4.55; but 3591 x 48 -> 192 5.8, 4.3
bool qgemm_few_wins(const QgemmParams& p, bool i16) {
  if (!qgemm_few_ok(p, i16)) return false;
  const int64_t tiles = (int64_t)((p.M + 31) / 32) * ((p.N + 31) / 32), tiles64 = (int64_t)((p.M + 63) / 64) * ((p.N + 63) / 64);
  if (tiles <= 512) return true;
  if (i16) return false;
  const bool whole = p.K % 16 == 0 && ptr_aligned(p.act, 16) && ptr_aligned(p.wgt, 16);
  if (whole) return tiles <= 1024 && p.K > 64 && p.K <= 640;
  return tiles <= 2048 && (p.K <= 512 || (p.K <= 768 && tiles <= 1024) || tiles <= (p.K <= 1024 ? 3 : 2) * tiles64);
}

// Requires qgemm_few_ok.  waves: 4 or 8, 0: by the length of the reduction.
hipError_t launch_qgemm_few(const QgemmParams& p, bool i16, int waves, hipStream_t st) {
  const int64_t kb = (int64_t)p.K * (i16 ? 2 : 1);
  const bool mis = kb % 4 != 0 || !ptr_aligned(p.act, 4) || !ptr_aligned(p.wgt, 4);
  const int blocks = (int)((kb + kBlock - 1) / kBlock);
  const int64_t tiles_m = (p.M + 31) / 32, tiles_n = (p.N + 31) / 32, tiles = tiles_m * tiles_n;
  const bool channels_first = p.M >= p.N;  // an XCD's run of tiles keeps the longer operand's rows
  const int64_t minor = channels_first ? tiles_n : tiles_m;
  const uint32_t inv = minor > 1 ? (uint32_t)(((1ull << 32) + minor - 1) / minor) : 0u;
  auto size = [&](const void* ptr, int64_t rows) { return run_size(rows, kb, (uint32_t)(reinterpret_cast<uintptr_t>(ptr) & 3)); };
  const FewParams q = few_params(p);
  auto run = [&]<bool I16, bool MIS, int NW>() {
    const int slots = blocks < kDepth * NW ? blocks : kDepth * NW;
    const auto kern = p.has_rq ? qgemm_few_kernel<I16 + 2, MIS, NW> : qgemm_few_kernel<I16, MIS, NW>;
    static std::atomic<uint64_t> attr_set[2];  // per kernel: the devices whose dynamic-LDS limit is raised
    const hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), kDepth * NW * slot_bytes<MIS>(), attr_set[p.has_rq != 0]);
    if (e != hipSuccess) return e;
    return launch_kernel(kern, dim3((unsigned)tiles), dim3(64 * NW), slots * slot_bytes<MIS>(), st, p.act, p.wgt, p.M, p.N, (uint32_t)kb, blocks,
                       (uint32_t)tiles, (uint32_t)minor | (channels_first ? 0x80000000u : 0u), inv, size(p.wgt, p.N), size(p.act, p.M), q);
  };
  auto by_form = [&]<bool I16, bool MIS>() {
    // eight wavefronts for tiles that are alone on their CU and have blocks for them (128 x 3072 -> 768 4.3 us, 4.7 with
    // four; 256 x 768 -> 3072 4.6 with four, 5.5 with eight, whose LDS leaves no room for a second tile)
    const bool eight = waves ? waves == 8 : blocks > 4 && tiles <= 256;
    return eight ? run.template operator()<I16, MIS, 8>() : run.template operator()<I16, MIS, 4>();
  };
  if (i16) return mis ? by_form.template operator()<true, true>() : by_form.template operator()<true, false>();
  return mis ? by_form.template operator()<false, true>() : by_form.template operator()<false, false>();
}

}  // namespace hago
