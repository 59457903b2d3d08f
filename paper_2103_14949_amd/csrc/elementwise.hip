// Bandwidth-bound elementwise kernels: fp32 simulated_quantize, the standalone
// integer requantize and the max-abs calibration reduction.  The first two stream
// [outer, channels, inner] tensors once (read) and once (write); the only reuse is
// the per-channel parameter, which is block-uniform in the row kernels and so lives
// in scalar registers.  The reduction reads the tensor once.
//
// Three launch shapes per operator, all with 128-bit accesses:
//   rows     : one workgroup per (row = outer*channels index, segment of inner); the channel's
//              parameters are fetched once per workgroup.  Aligned rows of 512 elements or more.
//   periodic : short or ragged rows (channel-last tensors among them) whose pattern of channels comes
//              back within the tensor: a lane keeps the same four channels' parameters over many vectors.
//   flat     : the rest (the pattern comes back fewer than four times): four consecutive elements per
//              vector, their channels found with one multiply-high division.
#include "hago_device.h"
#include "launch.h"
#include "span_split.h"

#include <type_traits>

namespace hago {

namespace {

constexpr int kThreads = kSpanThreads;
constexpr int kVecPerLane = 4;  // 128-bit vectors per lane and job of the row kernels

typedef float v4f __attribute__((ext_vector_type(4)));
typedef int32_t v4i32 __attribute__((ext_vector_type(4)));
typedef int16_t v4i16 __attribute__((ext_vector_type(4)));

// A row of inner_vec vectors is cut into nseg jobs of seg_len vectors, as even as possible.
inline void split_row(int64_t inner_vec, int u, int32_t* nseg, int32_t* seg_len) {
  const int64_t per_job = (int64_t)kThreads * u;
  const int64_t n = (inner_vec + per_job - 1) / per_job;
  *nseg = (int32_t)n;
  *seg_len = (int32_t)((inner_vec + n - 1) / n);
}

// Row and channel of a row kernel's job (job = row * nseg + segment).  A job streams a dozen
// kilobytes, so its bookkeeping counts: jobs below 2^32, the usual case, are divided with the
// host's reciprocals floor(2^32 / d) (a multiply-high and at most two corrections, all on
// wavefront-uniform values, i.e. scalar instructions) instead of the 25 vector instructions of an
// integer division each.
struct JobDiv {
  uint32_t inv_nseg, inv_channels;
};
inline uint32_t reciprocal32(int64_t d) { return d <= 1 ? 0xffffffffu : (uint32_t)((1ull << 32) / (uint64_t)d); }

__device__ __forceinline__ uint32_t div32(uint32_t n, uint32_t d, uint32_t inv, uint32_t& rem) {
  uint32_t q = __umulhi(n, inv);   // q - 2 <= this <= q
  uint32_t r = n - q * d;
  if (r >= d) { ++q; r -= d; }
  if (r >= d) { ++q; r -= d; }
  rem = r;
  return q;
}

__device__ __forceinline__ void job_row_channel(int64_t job, int32_t nseg, int32_t channels, int per_channel,
                                                JobDiv jd, int64_t& row, int32_t& c) {
  if (job <= 0xffffffffll) {
    uint32_t seg, cc;
    const uint32_t r32 = div32((uint32_t)job, (uint32_t)nseg, jd.inv_nseg, seg);
    row = r32;
    div32(r32, (uint32_t)channels, jd.inv_channels, cc);
    c = per_channel ? (int32_t)cc : 0;
  } else {
    row = job / nseg;
    c = per_channel ? (int32_t)(row % channels) : 0;
  }
}

// u = rintf(x / s), the rounded quotient of Eq. 3 (correctly rounded binary32 division, then
// round half to even), for a divisor that many elements share.  The division expands to about
// fifteen vector instructions, which made the row kernels issue-bound; this takes five on
// almost every element and gives the SAME value on every element:
//   rc = RN(1 / s), computed once per row with |s| in [2^-100, 2^100] (so rc is normal and within
//   2^-24 of 1 / s, relatively); qt = RN(x * rc) is within |x / s| * (2^-23 + 2^-48) of the
//   exact quotient, and so is RN(x / s) within |x / s| * 2^-24: the two differ by less than
//   |qt| * 2^-22.  With n = rintf(qt) and d = qt - n (exact: |qt| < 2^23 here), both lie strictly
//   inside (n - 1/2, n + 1/2) whenever |d| + |qt| * 2^-22 < 1/2, and then rintf of either is n
//   (an underflowing qt has n = 0, as the quotient has).  The test below asks for twice that margin,
//   which also covers the rounding of the threshold itself.
//   Anything else takes the division: quotients within about 2^-21 |qt| of a tie (one element in
//   2^14 for |qt| near 32), |qt| >= 2^20, infinities and NaN (every comparison false), and, through
//   rc = NaN, scales outside the range above.
__device__ __forceinline__ float quotient_reciprocal(float s) {
  const float a = fabsf(s);
  return (a >= 0x1p-100f && a <= 0x1p100f) ? 1.0f / s : __builtin_nanf("");
}

// Four elements at once, so that a kernel branches once per 128-bit vector: true when all four
// pass the test, and then n[e] = rintf(x[e] / s), all finite; otherwise the caller redoes the four
// with the division.
__device__ __forceinline__ bool fast_quotient4(v4f x, float rc, v4f& n) {
  bool ok = true;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float qt = x[e] * rc;
    n[e] = rintf(qt);
    const float d = qt - n[e];
    const float thr = __builtin_fmaf(fabsf(qt), -0x1p-21f, 0.5f);
    ok = ok && (fabsf(d) < thr);
  }
  return ok;
}

// Eq. 3 with zero point and saturation, in binary32, from the rounded quotient u.  The scalar
// definition clips with two compare-selects, (v < lo) ? lo : ((v > hi) ? hi : v), under which NaN
// stays NaN; for every other v (lo <= hi, both finite) that is the median of the three, one
// instruction, and v is never -0 here (a sum that is zero is +0), so no zero changes sign.
__device__ __forceinline__ float simquant_of(float u, float s, float zf, float lo, float hi) {
  const float v = u + zf;
  const float c = (v != v) ? v : __builtin_amdgcn_fmed3f(v, lo, hi);
  return (c - zf) * s;
}

// The same for a finite u (what fast_quotient4 hands out): no NaN to keep.
__device__ __forceinline__ float simquant_of_finite(float u, float s, float zf, float lo, float hi) {
  return (__builtin_amdgcn_fmed3f(u + zf, lo, hi) - zf) * s;
}

__device__ __forceinline__ float simquant_one(float x, float s, float zf, float lo, float hi) {
  return simquant_of(rintf(x / s), s, zf, lo, hi);
}


// The same with the overflow of the simulated integer type (Sec. 5.2 of the paper: the third error
// source): the code is reduced modulo 2^wrap_bits before the clip, into the two's-complement range
// (wrap_signed) or into 0 .. 2^wrap_bits - 1.  A code of magnitude 4e18 or more, or an infinite one,
// reduces to 0 (every binary32 number that large is a multiple of 2^32); NaN stays NaN.
__device__ __forceinline__ float simquant_wrap_of(float u, float s, float zf, float lo, float hi,
                                                  int wrap_bits, int wrap_signed) {
  float v = u + zf;
  if (v == v) {
    long long code = 0;
    if (v > -4.0e18f && v < 4.0e18f) {
      code = (long long)v;  // v holds an integer below 2^62
      const int sh = 64 - wrap_bits;
      const unsigned long long low = (unsigned long long)code << sh;
      code = wrap_signed ? ((long long)low >> sh) : (long long)(low >> sh);
    }
    v = (float)code;  // exact up to 25 bits, round to nearest beyond
  }
  v = (v < lo) ? lo : ((v > hi) ? hi : v);
  return (v - zf) * s;
}

// U: 128-bit vectors per lane and job; all of a job's loads are issued before the first
// result is computed.  Loads carry the nontemporal hint (without it the copy rate of this chip is about 10 % lower), stores
// go through the L2 (`store_through`; us, nontemporal and so: simquant of 8 x 144 x 784 3.95, 3.45, of 32 x 144 x 3136 19.1, 16.3 and with
// its codes 22.2, 18.9, but on buffers that the last-level cache does not hold 20.6, 21.3 and 23.4, 24.1; dequantize of 4096 x 768, per channel, 4.5, 3.95).
// WRAP: the overflow-simulating form (wrap_bits, wrap_signed).
template <int U, bool WRAP = false>
__global__ __launch_bounds__(kThreads) void simquant_rows_kernel(
    const v4f* __restrict__ x, v4f* __restrict__ y, int64_t rows, int32_t channels,
    int64_t inner_vec, int32_t nseg, int32_t seg_len, const float* __restrict__ scale,
    const int32_t* __restrict__ zp, int per_channel, JobDiv jd, float lo, float hi, int wrap_bits = 0,
    int wrap_signed = 0) {
  for (int64_t job = blockIdx.x; job < rows * nseg; job += gridDim.x) {
    int64_t row;
    int32_t c;
    job_row_channel(job, nseg, channels, per_channel, jd, row, c);
    const int32_t seg = (int32_t)(job - row * nseg);
    const float s = scale[c];
    const float zf = (float)zp[c];
    const float rc = quotient_reciprocal(s);
    auto of = [&](float u, float s, float zf) {
      if constexpr (WRAP) return simquant_wrap_of(u, s, zf, lo, hi, wrap_bits, wrap_signed);
      else return simquant_of(u, s, zf, lo, hi);
    };
    const int64_t v0 = (int64_t)seg * seg_len;
    const int64_t v1 = (v0 + seg_len < inner_vec) ? v0 + seg_len : inner_vec;
    const v4f* xr = x + row * inner_vec;
    v4f* yr = y + row * inner_vec;
    for (int64_t vb = v0 + threadIdx.x; vb < v1; vb += (int64_t)kThreads * U) {
      v4f a[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (vb + u * kThreads < v1) a[u] = __builtin_nontemporal_load(xr + vb + u * kThreads);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (vb + u * kThreads < v1) {
          v4f n, r;
          if (__builtin_expect(fast_quotient4(a[u], rc, n), 1)) {
            if constexpr (WRAP) r = v4f{of(n.x, s, zf), of(n.y, s, zf), of(n.z, s, zf), of(n.w, s, zf)};
            else r = v4f{simquant_of_finite(n.x, s, zf, lo, hi), simquant_of_finite(n.y, s, zf, lo, hi),
                         simquant_of_finite(n.z, s, zf, lo, hi), simquant_of_finite(n.w, s, zf, lo, hi)};
          } else {  // IEEE division (correctly rounded)
            r = v4f{of(rintf(a[u].x / s), s, zf), of(rintf(a[u].y / s), s, zf), of(rintf(a[u].z / s), s, zf),
                    of(rintf(a[u].w / s), s, zf)};
          }
          store_through(yr + vb + u * kThreads, r);
        }
      }
    }
  }
}

// Batched candidates (Sec. 6.3): x is read ONCE and every candidate b writes its own
// y[b][...] with scale[b][c], zero_point[b][c] and clip range b.  4 + 4 B bytes per element
// instead of 8 B for B separate launches.
constexpr int kMaxCandidates = 16;
struct CandidateClips {
  float lo[kMaxCandidates], hi[kMaxCandidates];
};

template <int U, bool THROUGH>
__global__ __launch_bounds__(kThreads) void simquant_batched_rows_kernel(
    const v4f* __restrict__ x, v4f* __restrict__ y, int64_t rows, int32_t channels,
    int64_t inner_vec, int32_t nseg, int32_t seg_len, int32_t nbatch, int32_t nparam,
    const float* __restrict__ scale, const int32_t* __restrict__ zp, int per_channel, JobDiv jd,
    CandidateClips clips) {
  const int64_t batch_stride = rows * inner_vec;  // vectors per candidate output
  for (int64_t job = blockIdx.x; job < rows * nseg; job += gridDim.x) {
    int64_t row;
    int32_t c;
    job_row_channel(job, nseg, channels, per_channel, jd, row, c);
    const int32_t seg = (int32_t)(job - row * nseg);
    const int64_t v0 = (int64_t)seg * seg_len;
    const int64_t v1 = (v0 + seg_len < inner_vec) ? v0 + seg_len : inner_vec;
    const v4f* xr = x + row * inner_vec;
    v4f* yr = y + row * inner_vec;
    for (int64_t vb = v0 + threadIdx.x; vb < v1; vb += (int64_t)kThreads * U) {
      v4f a[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (vb + u * kThreads < v1) a[u] = __builtin_nontemporal_load(xr + vb + u * kThreads);
      for (int b = 0; b < nbatch; ++b) {
        const float s = scale[(int64_t)b * nparam + c];
        const float zf = (float)zp[(int64_t)b * nparam + c];
        const float lo = clips.lo[b], hi = clips.hi[b];
        const float rc = quotient_reciprocal(s);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (vb + u * kThreads < v1) {
            v4f n, r;
            if (__builtin_expect(fast_quotient4(a[u], rc, n), 1)) {
              r = v4f{simquant_of_finite(n.x, s, zf, lo, hi), simquant_of_finite(n.y, s, zf, lo, hi),
                      simquant_of_finite(n.z, s, zf, lo, hi), simquant_of_finite(n.w, s, zf, lo, hi)};
            } else {
              r = v4f{simquant_one(a[u].x, s, zf, lo, hi), simquant_one(a[u].y, s, zf, lo, hi),
                      simquant_one(a[u].z, s, zf, lo, hi), simquant_one(a[u].w, s, zf, lo, hi)};
            }
            if constexpr (THROUGH) store_through(yr + b * batch_stride + vb + u * kThreads, r);
            else __builtin_nontemporal_store(r, yr + b * batch_stride + vb + u * kThreads);
          }
        }
      }
    }
  }
}

// AWAY: the launch's tie rule is halves away from zero (the general form); else the plain one.
template <bool AWAY>
__device__ __forceinline__ int32_t requant_pick(int32_t acc, int32_t mult, int32_t sh, const RequantScalars& rs) {
  if constexpr (AWAY) return requant_half_away(acc, mult, sh, rs);
  else return requant_one(acc, mult, sh, rs);
}

// rows: 4 accumulators -> 4 output bytes per step, 128-bit loads for int32; U steps per lane
// and job with all loads issued first, nontemporal as above.
// POW2: no multiplier array (power-of-two scales): the rounding shift alone, no multiplication.
template <typename AccT, int U, bool AWAY, bool POW2 = false>
__global__ __launch_bounds__(kThreads) void requant_rows_kernel(
    const AccT* __restrict__ acc, uint32_t* __restrict__ out, int64_t rows, int32_t channels,
    int64_t inner_vec, int32_t nseg, int32_t seg_len, const int32_t* __restrict__ mult,
    const int32_t* __restrict__ shift, int per_channel, JobDiv jd, RequantScalars rs) {
  using VecT = typename std::conditional<sizeof(AccT) == 4, v4i32, v4i16>::type;
  for (int64_t job = blockIdx.x; job < rows * nseg; job += gridDim.x) {
    int64_t row;
    int32_t c;
    job_row_channel(job, nseg, channels, per_channel, jd, row, c);
    const int32_t seg = (int32_t)(job - row * nseg);
    const int32_t m = POW2 ? 0 : rq_mult(mult, c);
    const int32_t sh = POW2 ? shift[c] : rq_shift(mult, shift, c);
    auto one = [&](int32_t a) {
      if constexpr (POW2) return med3(shift_round(a, sh), rs.lo_rel, rs.hi_rel) + rs.z_out;
      else return requant_pick<AWAY>(a, m, sh, rs);
    };
    const int64_t v0 = (int64_t)seg * seg_len;
    const int64_t v1 = (v0 + seg_len < inner_vec) ? v0 + seg_len : inner_vec;
    const VecT* ar = reinterpret_cast<const VecT*>(acc) + row * inner_vec;
    uint32_t* orow = out + row * inner_vec;
    for (int64_t vb = v0 + threadIdx.x; vb < v1; vb += (int64_t)kThreads * U) {
      VecT q[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (vb + u * kThreads < v1) q[u] = __builtin_nontemporal_load(ar + vb + u * kThreads);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (vb + u * kThreads < v1) {
          const uint32_t r = pack4(one((int32_t)q[u].x), one((int32_t)q[u].y), one((int32_t)q[u].z), one((int32_t)q[u].w));
          store_through(orow + vb + u * kThreads, r);
        }
      }
    }
  }
}

// ---- quantize / dequantize (the two halves of Eq. 3; Sec. 6.1): the code is formed exactly as in
// simulated_quantize (binary32 division, round half to even, zero point added as a float,
// compare-select clip), then stored in the integer container; NaN takes the code of real zero.
__device__ __forceinline__ int32_t quantize_of(float u, float zf, float lo, float hi) {
  const float v = (u != u) ? zf : u + zf;                  // never NaN from here on
  return (int32_t)__builtin_amdgcn_fmed3f(v, lo, hi);      // the clip; integral and within +-2^24
}

__device__ __forceinline__ int32_t quantize_of_finite(float u, float zf, float lo, float hi) {
  return (int32_t)__builtin_amdgcn_fmed3f(u + zf, lo, hi);
}

__device__ __forceinline__ int32_t quantize_one(float x, float s, float zf, float lo, float hi) {
  return quantize_of(rintf(x / s), zf, lo, hi);
}

__device__ __forceinline__ float dequantize_one(int32_t q, float s, float zf) {
  return ((float)q - zf) * s;
}

template <typename Q> struct QVec;  // four codes of a container as one store / load
template <> struct QVec<int8_t> { typedef uint32_t T; };
template <> struct QVec<uint8_t> { typedef uint32_t T; };
template <> struct QVec<int16_t> { typedef v4i16 T; };
template <> struct QVec<int32_t> { typedef v4i32 T; };

template <typename Q>
__device__ __forceinline__ typename QVec<Q>::T pack_codes(int32_t a, int32_t b, int32_t c, int32_t d) {
  if constexpr (sizeof(Q) == 1) return pack4(a, b, c, d);
  else if constexpr (sizeof(Q) == 2) return v4i16{(int16_t)a, (int16_t)b, (int16_t)c, (int16_t)d};
  else return v4i32{a, b, c, d};
}

template <typename Q>
__device__ __forceinline__ void unpack_codes(typename QVec<Q>::T v, int32_t (&q)[4]) {
  if constexpr (sizeof(Q) == 1) {
#pragma unroll
    for (int e = 0; e < 4; ++e) q[e] = (int32_t)(Q)((v >> (8 * e)) & 0xffu);
  } else {
    q[0] = (int32_t)v.x; q[1] = (int32_t)v.y; q[2] = (int32_t)v.z; q[3] = (int32_t)v.w;
  }
}

// Row kernels as for simulated_quantize.  OP 0: fp32 -> codes; 1: codes -> fp32; 2: fp32 -> codes
// (out) and the simulated_quantize value (out2) in one pass over x.
template <typename Q, int OP, int U>
__global__ __launch_bounds__(kThreads) void quant_rows_kernel(
    const void* __restrict__ in, void* __restrict__ out, float* __restrict__ out2, int64_t rows, int32_t channels,
    int64_t inner_vec, int32_t nseg, int32_t seg_len, const float* __restrict__ scale,
    const int32_t* __restrict__ zp, int per_channel, JobDiv jd, float lo, float hi) {
  using VQ = typename QVec<Q>::T;
  for (int64_t job = blockIdx.x; job < rows * nseg; job += gridDim.x) {
    int64_t row;
    int32_t c;
    job_row_channel(job, nseg, channels, per_channel, jd, row, c);
    const int32_t seg = (int32_t)(job - row * nseg);
    const float s = scale[c];
    const float zf = (float)zp[c];
    const float rc = OP == 1 ? 0.0f : quotient_reciprocal(s);
    const int64_t v0 = (int64_t)seg * seg_len;
    const int64_t v1 = (v0 + seg_len < inner_vec) ? v0 + seg_len : inner_vec;
    for (int64_t vb = v0 + threadIdx.x; vb < v1; vb += (int64_t)kThreads * U) {
      if constexpr (OP == 1) {
        const VQ* qr = static_cast<const VQ*>(in) + row * inner_vec;
        v4f* yr = static_cast<v4f*>(out) + row * inner_vec;
        VQ a[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (vb + u * kThreads < v1) a[u] = __builtin_nontemporal_load(qr + vb + u * kThreads);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (vb + u * kThreads < v1) {
            int32_t q[4];
            unpack_codes<Q>(a[u], q);
            const v4f r = {dequantize_one(q[0], s, zf), dequantize_one(q[1], s, zf),
                           dequantize_one(q[2], s, zf), dequantize_one(q[3], s, zf)};
            store_through(yr + vb + u * kThreads, r);
          }
        }
      } else {
        const v4f* xr = static_cast<const v4f*>(in) + row * inner_vec;
        VQ* qr = static_cast<VQ*>(out) + row * inner_vec;
        v4f a[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (vb + u * kThreads < v1) a[u] = __builtin_nontemporal_load(xr + vb + u * kThreads);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (vb + u * kThreads < v1) {
            v4f n, y;
            VQ r;
            if (__builtin_expect(fast_quotient4(a[u], rc, n), 1)) {   // four finite quotients
              r = pack_codes<Q>(quantize_of_finite(n.x, zf, lo, hi), quantize_of_finite(n.y, zf, lo, hi),
                                quantize_of_finite(n.z, zf, lo, hi), quantize_of_finite(n.w, zf, lo, hi));
              if constexpr (OP == 2)
                y = v4f{simquant_of_finite(n.x, s, zf, lo, hi), simquant_of_finite(n.y, s, zf, lo, hi),
                        simquant_of_finite(n.z, s, zf, lo, hi), simquant_of_finite(n.w, s, zf, lo, hi)};
            } else {
              r = pack_codes<Q>(quantize_one(a[u].x, s, zf, lo, hi), quantize_one(a[u].y, s, zf, lo, hi),
                                quantize_one(a[u].z, s, zf, lo, hi), quantize_one(a[u].w, s, zf, lo, hi));
              if constexpr (OP == 2)
                y = v4f{simquant_one(a[u].x, s, zf, lo, hi), simquant_one(a[u].y, s, zf, lo, hi),
                        simquant_one(a[u].z, s, zf, lo, hi), simquant_one(a[u].w, s, zf, lo, hi)};
            }
            store_through(qr + vb + u * kThreads, r);
            if constexpr (OP == 2) {
              store_through(reinterpret_cast<v4f*>(out2) + row * inner_vec + vb + u * kThreads, y);
            }
          }
        }
      }
    }
  }
}

// ---- short, ragged and channel-last rows.  An operator of this section names how four consecutive
// elements are loaded, what a channel's parameters are and how they are applied; the two kernels below
// find the channels.  The vectors carry the element type's alignment only, so a tensor that starts
// anywhere takes the same code (global accesses of gfx950 may be unaligned).
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
typedef int32_t v4i32_any __attribute__((ext_vector_type(4), aligned(4)));
typedef int16_t v4i16_any __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32_any __attribute__((aligned(1)));

template <typename T> struct AnyVec;  // four T as one access of T's alignment
template <> struct AnyVec<float> { typedef v4f_any T; };
template <> struct AnyVec<int32_t> { typedef v4i32_any T; };
template <> struct AnyVec<int16_t> { typedef v4i16_any T; };
template <> struct AnyVec<int8_t> { typedef u32_any T; };
template <> struct AnyVec<uint8_t> { typedef u32_any T; };

template <typename T>
__device__ __forceinline__ auto load4(const T* p, int64_t i) {
  return __builtin_nontemporal_load(reinterpret_cast<const typename AnyVec<T>::T*>(p + i));
}
template <bool THROUGH = true, typename T, typename V>
__device__ __forceinline__ void store4(T* p, int64_t i, V v) {
  if constexpr (THROUGH) store_through(p + i, v);
  else __builtin_nontemporal_store((typename AnyVec<T>::T)v, reinterpret_cast<typename AnyVec<T>::T*>(p + i));
}

// s, z and (RC) the reciprocal of s for fast_quotient4; without it the division is taken at once.
struct ScaleZero {
  float s, zf, rc;
};

template <bool RC>
__device__ __forceinline__ ScaleZero scale_zero(const float* scale, const int32_t* zp, int64_t c) {
  const float s = scale[c];
  return ScaleZero{s, (float)zp[c], RC ? quotient_reciprocal(s) : 0.0f};
}

// Parameters of four channels; run: they are consecutive ones (channel-last tensors), read as one vector.
__device__ __forceinline__ void scale_zero4(const float* scale, const int32_t* zp, const int64_t (&c)[4], bool run, float (&s)[4],
                                            int32_t (&z)[4]) {
  if (run) {
    const v4f sv = *reinterpret_cast<const v4f_any*>(scale + c[0]);
    const v4i32 zv = *reinterpret_cast<const v4i32_any*>(zp + c[0]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s[e] = sv[e];
      z[e] = zv[e];
    }
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    s[e] = scale[c[e]];
    z[e] = zp[c[e]];
  }
}
template <bool RC>
struct ScaleZero4 {
  ScaleZero p[4];
  __device__ void read(const float* scale, const int32_t* zp, const int64_t (&c)[4], bool run) {
    float s[4];
    int32_t z[4];
    scale_zero4(scale, zp, c, run, s, z);
#pragma unroll
    for (int e = 0; e < 4; ++e) p[e] = ScaleZero{s[e], (float)z[e], RC ? quotient_reciprocal(s[e]) : 0.0f};
  }
};

// The four rounded quotients; returns whether all are known to be finite.
template <bool RC>
__device__ __forceinline__ bool quotients4(v4f x, const ScaleZero (&p)[4], v4f& n) {
  if constexpr (RC) {
    bool ok = true;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float qt = x[e] * p[e].rc;
      n[e] = rintf(qt);
      ok = ok && (fabsf(qt - n[e]) < __builtin_fmaf(fabsf(qt), -0x1p-21f, 0.5f));  // as in fast_quotient4
    }
    if (__builtin_expect(ok, 1)) return true;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) n[e] = rintf(x[e] / p[e].s);
  return false;
}

// THROUGH: results go through the L2.
template <bool WRAP, bool RC, bool THROUGH = true>
struct SimquantOp {
  typedef v4f Vec;
  typedef ScaleZero Par;
  typedef ScaleZero4<RC> Kept;  // what a lane of the periodic kernel keeps of its four channels
  const float* x;
  float* y;
  const float* scale;
  const int32_t* zp;
  float lo, hi;
  int wrap_bits, wrap_signed;
  __device__ Par par(int64_t c) const { return scale_zero<RC>(scale, zp, c); }
  __device__ void keep(Kept& k, const int64_t (&c)[4], bool run) const { k.read(scale, zp, c, run); }
  __device__ void four(int64_t i, Vec v, const Kept& k) const { four(i, v, k.p); }
  __device__ Vec load(int64_t i) const { return load4(x, i); }
  __device__ float of(float u, const Par& p) const {
    if constexpr (WRAP) return simquant_wrap_of(u, p.s, p.zf, lo, hi, wrap_bits, wrap_signed);
    else return simquant_of(u, p.s, p.zf, lo, hi);
  }
  __device__ void four(int64_t i, Vec v, const Par (&p)[4]) const {
    v4f n;
    quotients4<RC>(v, p, n);
    store4<THROUGH>(y, i, v4f{of(n.x, p[0]), of(n.y, p[1]), of(n.z, p[2]), of(n.w, p[3])});
  }
  __device__ void one(int64_t i, const Par& p) const { y[i] = of(rintf(x[i] / p.s), p); }
};

// OP as in quant_rows_kernel.
template <typename Q, int OP, bool RC, bool THROUGH = true>
struct QuantOp {
  typedef typename std::conditional<OP == 1, typename QVec<Q>::T, v4f>::type Vec;
  typedef ScaleZero Par;
  typedef ScaleZero4<RC && OP != 1> Kept;
  const void* in;
  void* out;
  float* out2;
  const float* scale;
  const int32_t* zp;
  float lo, hi;
  __device__ Par par(int64_t c) const { return scale_zero<RC && OP != 1>(scale, zp, c); }
  __device__ void keep(Kept& k, const int64_t (&c)[4], bool run) const { k.read(scale, zp, c, run); }
  __device__ void four(int64_t i, Vec v, const Kept& k) const { four(i, v, k.p); }
  __device__ Vec load(int64_t i) const {
    if constexpr (OP == 1) return load4(static_cast<const Q*>(in), i);
    else return load4(static_cast<const float*>(in), i);
  }
  __device__ void four(int64_t i, Vec v, const Par (&p)[4]) const {
    if constexpr (OP == 1) {
      int32_t q[4];
      unpack_codes<Q>(v, q);
      store4(static_cast<float*>(out), i, v4f{dequantize_one(q[0], p[0].s, p[0].zf), dequantize_one(q[1], p[1].s, p[1].zf),
                                              dequantize_one(q[2], p[2].s, p[2].zf), dequantize_one(q[3], p[3].s, p[3].zf)});
    } else {
      v4f n;
      quotients4<RC>(v, p, n);
      store4<THROUGH>(static_cast<Q*>(out), i, pack_codes<Q>(quantize_of(n.x, p[0].zf, lo, hi), quantize_of(n.y, p[1].zf, lo, hi),
                                                             quantize_of(n.z, p[2].zf, lo, hi), quantize_of(n.w, p[3].zf, lo, hi)));
      if constexpr (OP == 2)
        store4<THROUGH>(out2, i, v4f{simquant_of(n.x, p[0].s, p[0].zf, lo, hi), simquant_of(n.y, p[1].s, p[1].zf, lo, hi),
                                     simquant_of(n.z, p[2].s, p[2].zf, lo, hi), simquant_of(n.w, p[3].s, p[3].zf, lo, hi)});
    }
  }
  __device__ void one(int64_t i, const Par& p) const {
    if constexpr (OP == 1) {
      static_cast<float*>(out)[i] = dequantize_one((int32_t)static_cast<const Q*>(in)[i], p.s, p.zf);
    } else {
      const float u = rintf(static_cast<const float*>(in)[i] / p.s);
      static_cast<Q*>(out)[i] = (Q)quantize_of(u, p.zf, lo, hi);
      if constexpr (OP == 2) out2[i] = simquant_of(u, p.s, p.zf, lo, hi);
    }
  }
};

template <typename AccT, bool AWAY>
struct RequantOp {
  typedef typename std::conditional<sizeof(AccT) == 4, v4i32, v4i16>::type Vec;
  struct Par {
    int32_t m, sh;
  };
  // Kept: rounding term and output zero point in one constant where every lane's shifts allow it and the clip is the
  // container's whole range (products are below 2^62, the constant below 2^61 + 2^51): the packing then saturates.
  struct Kept {
    Par p[4];
    int64_t k64[4];
    bool sat;
  };
  const AccT* acc;
  void* out;
  const int32_t* mult;
  const int32_t* shift;
  RequantScalars rs;
  __device__ Par par(int64_t c) const { return Par{rq_mult(mult, c), rq_shift(mult, shift, c)}; }
  __device__ void keep(Kept& k, const int64_t (&c)[4], bool run) const {
    if (run) {
      const v4i32 sv = *reinterpret_cast<const v4i32_any*>(shift + c[0]);
      v4i32 mv = {1 << 30, 1 << 30, 1 << 30, 1 << 30};  // (as rq_mult, rq_shift)
      if (mult) mv = *reinterpret_cast<const v4i32_any*>(mult + c[0]);
#pragma unroll
      for (int e = 0; e < 4; ++e) k.p[e] = Par{mv[e], sv[e] - (mult ? 0 : 1)};
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) k.p[e] = par(c[e]);
    }
    bool ok = !AWAY && sat_range(rs) && rs.z_out >= -128 && rs.z_out <= 255;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int32_t sh = k.p[e].sh;
      ok = ok && sh >= 1 && sh <= 21;
      k.k64[e] = ((int64_t)1 << (30 + (sh & 31))) + ((int64_t)(rs.z_out + sat_bias(rs)) << (31 + (sh & 31)));
    }
    k.sat = __builtin_amdgcn_ballot_w64(!ok) == 0;  // wavefront-uniform
  }
  __device__ void four(int64_t i, Vec v, const Kept& k) const {
    if (!k.sat) return four(i, v, k.p);
    int32_t r[4];
    uint32_t dw;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = (int32_t)(((int64_t)v[e] * (int64_t)k.p[e].m + k.k64[e]) >> 32) >> (k.p[e].sh - 1);
    ashr_sat_pair<0>(dw, r[0], r[1], 0);
    ashr_sat_pair<1>(dw, r[2], r[3], 0);
    store4(static_cast<uint8_t*>(out), i, dw ^ sat_flip(rs));
  }
  __device__ Vec load(int64_t i) const { return load4(acc, i); }
  __device__ int32_t of(int32_t a, const Par& p) const { return requant_pick<AWAY>(a, p.m, p.sh, rs); }
  __device__ void four(int64_t i, Vec v, const Par (&p)[4]) const {
    store4(static_cast<uint8_t*>(out), i, pack4(of(v.x, p[0]), of(v.y, p[1]), of(v.z, p[2]), of(v.w, p[3])));
  }
  __device__ void one(int64_t i, const Par& p) const { static_cast<uint8_t*>(out)[i] = (uint8_t)of(acc[i], p); }
};

// The channel of flat element i = (o * channels + c) * inner + k, and k.
struct ChannelDiv {
  int64_t inner, channels;
  uint32_t inv_inner, inv_channels;
  int32_t narrow;  // the whole tensor has fewer than 2^32 elements
};

inline ChannelDiv channel_div(int64_t total, int64_t channels, int64_t inner) {
  return ChannelDiv{inner, channels, reciprocal32(inner), reciprocal32(channels), total < (1ll << 32) ? 1 : 0};
}

__device__ __forceinline__ int64_t channel_at(const ChannelDiv& d, int64_t i, int64_t& k) {
  if (d.narrow) {
    uint32_t r, c;
    const uint32_t q = div32((uint32_t)i, (uint32_t)d.inner, d.inv_inner, r);
    div32(q, (uint32_t)d.channels, d.inv_channels, c);
    k = r;
    return c;
  }
  const int64_t q = i / d.inner;
  k = i - q * d.inner;
  return q % d.channels;
}

// Channels of four consecutive elements from i on.
__device__ __forceinline__ void channels4(const ChannelDiv& d, int64_t i, int64_t (&c)[4]) {
  int64_t k;
  c[0] = channel_at(d, i, k);
#pragma unroll
  for (int e = 1; e < 4; ++e) {
    c[e] = c[e - 1];
    if (++k == d.inner) {
      k = 0;
      if (++c[e] == d.channels) c[e] = 0;
    }
  }
}

// One workgroup of a tensor's division into spans (span_split.h).
template <class Op, int U>
__global__ __launch_bounds__(kThreads) void periodic_kernel(Op op, SpanArgs g, ChannelDiv d) {
  const int t = threadIdx.x;
  const int32_t rg = (int32_t)(blockIdx.x / (uint32_t)g.nseg);
  const int32_t j = (int32_t)(blockIdx.x - (uint32_t)rg * (uint32_t)g.nseg) * g.seg_len + t;
  const int64_t nvec = g.total >> 2;
  if (blockIdx.x == 0 && t < (int)(g.total & 3)) {  // the last, incomplete vector
    int64_t k;
    const int64_t i = 4 * nvec + t;
    op.one(i, op.par(channel_at(d, i, k)));
  }
  if (t >= g.seg_len || j >= g.span) return;
  int64_t v = (int64_t)rg * g.rows * g.span + j;
  const int64_t end = v + (int64_t)g.rows * g.span < nvec ? v + (int64_t)g.rows * g.span : nvec;
  // the first vectors are requested before the channels' parameters, which are a chain of loads and divisions (a channel-last
  // tensor of 4096 x 768, back to back: simquant 5.0 us, 6.1 before; dequantize 4.4, 5.4; quantize 4.6, 4.8)
  typename Op::Vec a[U];
  auto load = [&](int64_t v0) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (v0 + (int64_t)u * g.span < end) a[u] = op.load(4 * (v0 + (int64_t)u * g.span));
  };
  load(v);
  __builtin_amdgcn_sched_barrier(0);
  int64_t c[4];
  channels4(d, 4ll * j, c);
  typename Op::Kept p;
  op.keep(p, c, d.inner == 1 && (d.channels & 3) == 0);
  while (v < end) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (v + (int64_t)u * g.span < end) op.four(4 * (v + (int64_t)u * g.span), a[u], p);
    v += (int64_t)U * g.span;
    load(v);
  }
}

// MULTI: inner < 4, every element of a vector may have its own channel; else at most two.
template <class Op, int U, bool MULTI>
__global__ __launch_bounds__(kThreads) void flat_kernel(Op op, int64_t total, ChannelDiv d, int64_t block0) {
  const int64_t nvec = total >> 2;
  const int64_t v0 = (block0 + blockIdx.x) * (kThreads * U) + threadIdx.x;
  if (v0 < (total & 3)) {  // the last, incomplete vector (v0 < 4: threads of the first workgroup)
    int64_t k;
    const int64_t i = 4 * nvec + v0;
    op.one(i, op.par(channel_at(d, i, k)));
  }
  HAGO_SPARE_REGISTER("v47");  // (48 registers: still eight wavefronts on a SIMD)
  typename Op::Vec a[U];
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (v0 + u * kThreads < nvec) a[u] = op.load(4 * (v0 + u * kThreads));
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t v = v0 + u * kThreads;
    if (v >= nvec) break;
    if constexpr (MULTI) {
      int64_t c[4];
      channels4(d, 4 * v, c);
      const typename Op::Par p[4] = {op.par(c[0]), op.par(c[1]), op.par(c[2]), op.par(c[3])};
      op.four(4 * v, a[u], p);
    } else {
      int64_t k;
      const int64_t c0 = channel_at(d, 4 * v, k);
      const int64_t left = d.inner - k;  // elements before the next channel
      const int64_t c1 = left < 4 ? (c0 + 1 == d.channels ? 0 : c0 + 1) : c0;
      const typename Op::Par p0 = op.par(c0), p1 = op.par(c1);
      const typename Op::Par p[4] = {p0, left > 1 ? p0 : p1, left > 2 ? p0 : p1, left > 3 ? p0 : p1};
      op.four(4 * v, a[u], p);
    }
  }
}

// Periodic / flat launch of an operator; OpP keeps reciprocals for the periodic kernel, OpF does not; OpN is OpP with results that do not go
// through the L2, where there is such a form.  (As a member of the operator the choice made the arguments of a launch more than kCheapArguments.)
template <class OpP, class OpF, class OpN, class... A>
hipError_t launch_ragged(int64_t total, int64_t channels, int64_t inner, hipStream_t st, A... args) {
  constexpr int U = kVecPerLane;
  static_assert(sizeof(OpP) + sizeof(SpanArgs) + sizeof(ChannelDiv) <= kCheapArguments && sizeof(OpN) <= sizeof(OpP));
  const ChannelDiv d = channel_div(total, channels, inner);
  SpanArgs g;
  if (periodic_split(total, channels, inner, U, WholeLines::kAlways, &g)) {
    const int64_t wgs = ((g.spans + g.rows - 1) / g.rows) * g.nseg;
    // fp32 to fp32, with codes or without, in spans that end inside lines: such lines cost the write through the L2 more than it gains once 10 MB and more
    // are read beside it (channel-last 50000 x 65 simquant 7.9 us through it, 7.2 nontemporal; 30000 x 66 4.8, 5.7)
    if (g.seg_len % 4 == 0 || total < 2500000)
      return launch_kernel(periodic_kernel<OpP, U>, dim3((unsigned)wgs), dim3(kThreads), 0, st, OpP{args...}, g, d);
    return launch_kernel(periodic_kernel<OpN, U>, dim3((unsigned)wgs), dim3(kThreads), 0, st, OpN{args...}, g, d);
  }
  // one vector per lane while that does not fill the chip, four beyond
  const int64_t nvec = total / 4 > 0 ? total / 4 : 1;
  const int64_t w1 = (nvec + kThreads - 1) / kThreads, w4 = (nvec + kThreads * U - 1) / (kThreads * U);
  // (more than one launch from 2^36 elements on)
  constexpr int64_t most = max_blocks(kThreads);
  auto flat = [&](auto kern, int64_t wgs) {
    for (int64_t b0 = 0; b0 < wgs; b0 += most) {
      const hipError_t e = launch_kernel(kern, dim3((unsigned)(wgs - b0 < most ? wgs - b0 : most)), dim3(kThreads), 0, st, OpF{args...}, total, d, b0);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  };
  if (w1 <= 1024) return inner < 4 ? flat(flat_kernel<OpF, 1, true>, w1) : flat(flat_kernel<OpF, 1, false>, w1);
  return inner < 4 ? flat(flat_kernel<OpF, U, true>, w4) : flat(flat_kernel<OpF, U, false>, w4);
}

// Batched candidates over such rows: the lane's channels stay, the candidates' parameters are read per
// candidate (from the cache) and x is kept in registers, as in the row kernel.
template <int U, bool PERIODIC>
__global__ __launch_bounds__(kThreads) void simquant_batched_ragged_kernel(
    const float* __restrict__ x, float* __restrict__ y, SpanArgs g, ChannelDiv d, int32_t nbatch, int32_t nparam,
    const float* __restrict__ scale, const int32_t* __restrict__ zp, CandidateClips clips, int64_t block0) {
  const int t = threadIdx.x;
  const int64_t total = g.total, nvec = total >> 2;
  if (block0 + blockIdx.x == 0 && t < (int)(total & 3)) {
    int64_t k;
    const int64_t i = 4 * nvec + t;
    const int64_t c = channel_at(d, i, k);
    for (int b = 0; b < nbatch; ++b)
      y[(int64_t)b * total + i] = simquant_one(x[i], scale[(int64_t)b * nparam + c], (float)zp[(int64_t)b * nparam + c],
                                               clips.lo[b], clips.hi[b]);
  }
  int64_t v0, step, end;
  if constexpr (PERIODIC) {
    const int32_t rg = (int32_t)(blockIdx.x / (uint32_t)g.nseg);
    const int32_t j = (int32_t)(blockIdx.x - (uint32_t)rg * (uint32_t)g.nseg) * g.seg_len + t;
    if (t >= g.seg_len || j >= g.span) return;
    v0 = (int64_t)rg * g.rows * g.span + j;
    step = g.span;
    end = v0 + (int64_t)g.rows * g.span < nvec ? v0 + (int64_t)g.rows * g.span : nvec;
  } else {
    v0 = (block0 + blockIdx.x) * (kThreads * U) + t;
    step = kThreads;
    end = v0 + kThreads * U < nvec ? v0 + kThreads * U : nvec;
  }
  if (v0 >= end) return;
  int64_t c[4];
  if constexpr (PERIODIC) channels4(d, 4 * v0, c);
  for (int64_t v = v0; v < end; v += U * step) {
    v4f a[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (v + u * step < end) a[u] = load4(x, 4 * (v + u * step));
    auto params = [&](int b, ScaleZero (&p)[4]) {
      const float* sb = scale + (int64_t)b * nparam;
      const int32_t* zb = zp + (int64_t)b * nparam;
#pragma unroll
      for (int e = 0; e < 4; ++e) p[e] = scale_zero<PERIODIC>(sb, zb, c[e]);
    };
    auto write = [&](int b, int u, const ScaleZero (&p)[4]) {
      v4f n;
      quotients4<PERIODIC>(a[u], p, n);
      const float lo = clips.lo[b], hi = clips.hi[b];
      store4<false>(y + (int64_t)b * total, 4 * (v + u * step),
             v4f{simquant_of(n.x, p[0].s, p[0].zf, lo, hi), simquant_of(n.y, p[1].s, p[1].zf, lo, hi),
                 simquant_of(n.z, p[2].s, p[2].zf, lo, hi), simquant_of(n.w, p[3].s, p[3].zf, lo, hi)});
    };
    if constexpr (PERIODIC) {
      for (int b = 0; b < nbatch; ++b) {
        ScaleZero p[4];
        params(b, p);
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (v + u * step < end) write(b, u, p);
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (v + u * step >= end) break;
        channels4(d, 4 * (v + u * step), c);
        for (int b = 0; b < nbatch; ++b) {
          ScaleZero p[4];
          params(b, p);
          write(b, u, p);
        }
      }
    }
  }
}

inline hipError_t launch_batched_ragged(const float* x, float* y, int64_t total, int64_t channels, int64_t inner,
                                        int32_t nbatch, const float* scale, const int32_t* zp, const CandidateClips& clips,
                                        hipStream_t st) {
  constexpr int U = 2;
  const ChannelDiv d = channel_div(total, channels, inner);
  SpanArgs g;
  if (periodic_split(total, channels, inner, U, WholeLines::kRounds, &g, nbatch)) {
    const int64_t wgs = ((g.spans + g.rows - 1) / g.rows) * g.nseg;
    return launch_kernel(simquant_batched_ragged_kernel<U, true>, dim3((unsigned)wgs), dim3(kThreads), 0, st, x, y, g, d,
                         nbatch, (int32_t)channels, scale, zp, clips, (int64_t)0);
  }
  g = SpanArgs{};
  g.total = total;
  const int64_t nvec = total / 4 > 0 ? total / 4 : 1;
  if (nvec <= 1024 * kThreads)
    return launch_kernel(simquant_batched_ragged_kernel<1, false>, dim3((unsigned)((nvec + kThreads - 1) / kThreads)),
                         dim3(kThreads), 0, st, x, y, g, d, nbatch, (int32_t)channels, scale, zp, clips, (int64_t)0);
  constexpr int64_t most = max_blocks(kThreads);
  const int64_t wgs = (nvec + kThreads * U - 1) / (kThreads * U);
  for (int64_t b0 = 0; b0 < wgs; b0 += most) {  // (more than one launch from 2^35 elements on)
    const hipError_t e = launch_kernel(simquant_batched_ragged_kernel<U, false>, dim3((unsigned)(wgs - b0 < most ? wgs - b0 : most)),
                                       dim3(kThreads), 0, st, x, y, g, d, nbatch, (int32_t)channels, scale, zp, clips, b0);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// ---- max-abs calibration (Eq. 2): thr[c] = max |x[o, c, i]| over o, i.  NaN never wins a
// comparison and is therefore ignored; the result is never negative zero.  |x| of a non-NaN
// float orders like its bit pattern as an unsigned integer, so partial results are merged with
// one integer atomic max per workgroup (order-independent: the result is exact).
__device__ __forceinline__ float absmax_step(float m, float v) {
  const float a = fabsf(v);
  return a > m ? a : m;
}

__device__ __forceinline__ float wave_max(float m) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const float o = __shfl_xor(m, d);
    m = o > m ? o : m;
  }
  return m;
}

// SOLE: the workgroup's maximum is the result; otherwise it is merged into *thr_c (zeroed beforehand).
template <bool SOLE>
__device__ __forceinline__ void block_merge_max(float m, uint32_t* thr_c) {
  __shared__ float s_m[kThreads / 64];
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) s_m[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < kThreads / 64; ++w) m = s_m[w] > m ? s_m[w] : m;
    if constexpr (SOLE) *thr_c = __float_as_uint(m);
    else if (m > 0.0f) atomicMax(thr_c, __float_as_uint(m));
  }
  __syncthreads();
}

__global__ __launch_bounds__(kThreads) void fill_zero_kernel(uint32_t* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) p[i] = 0u;
}

// rows: as the other row kernels (row = outer * channels index, 128-bit nontemporal loads, U
// vectors per lane in flight), for rows of any length and alignment.  A job is (channel, row
// segment, group of outer indices): the workgroup walks the rows o = og, og + ogroups, ... of its
// channel and merges once, so the barriers and the atomic are paid once per several rows.
// SOLE: one job per channel, which stores its result (the thresholds need not be zeroed first).
template <int U, bool SOLE>
__global__ __launch_bounds__(kThreads) void absmax_rows_kernel(
    const float* __restrict__ x, int64_t outer, int32_t channels, int64_t inner, int32_t nseg,
    int32_t seg_len, int32_t ogroups, int per_channel, uint32_t* __restrict__ thr) {
  // per tensor the "row" is the whole tensor: outer == 1, channels == 1
  const int64_t jobs = (int64_t)channels * nseg * ogroups;
  const int64_t inner_vec = inner >> 2;
  for (int64_t job = blockIdx.x; job < jobs; job += gridDim.x) {
    // job = og * (channels * nseg) + c * nseg + seg: neighbouring workgroups, neighbouring rows
    int32_t og, seg, c;
    const int64_t per_group = (int64_t)channels * nseg;
    if (jobs <= 0xffffffffll) {  // the usual case: 32-bit divisions
      og = (int32_t)((uint32_t)job / (uint32_t)per_group);
      const uint32_t cs = (uint32_t)job - (uint32_t)og * (uint32_t)per_group;
      c = (int32_t)(cs / (uint32_t)nseg);
      seg = (int32_t)(cs - (uint32_t)c * (uint32_t)nseg);
    } else {
      og = (int32_t)(job / per_group);
      const int64_t cs = job - og * per_group;
      c = (int32_t)(cs / nseg);
      seg = (int32_t)(cs - (int64_t)c * nseg);
    }
    const int64_t v0 = (int64_t)seg * seg_len;
    const int64_t v1 = (v0 + seg_len < inner_vec) ? v0 + seg_len : inner_vec;
    float m = 0.0f;
    for (int64_t o = og; o < outer; o += ogroups) {
      const float* xr = x + (o * channels + c) * inner;
      if (seg == 0 && threadIdx.x < (unsigned)(inner & 3)) m = absmax_step(m, xr[4 * inner_vec + threadIdx.x]);
      for (int64_t vb = v0 + threadIdx.x; vb < v1; vb += (int64_t)kThreads * U) {
        v4f a[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          a[u] = vb + u * kThreads < v1 ? (v4f)load4(xr, 4 * (vb + u * kThreads)) : v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int u = 0; u < U; ++u) {
          m = absmax_step(m, a[u].x); m = absmax_step(m, a[u].y);
          m = absmax_step(m, a[u].z); m = absmax_step(m, a[u].w);
        }
      }
    }
    block_merge_max<SOLE>(m, thr + (per_channel ? c : 0));
  }
}

// Short rows that come back often (channel-last tensors among them; see SpanArgs): a lane keeps a
// maximum for each of its four elements over the workgroup's spans, the lanes merge in an LDS table,
// one integer maximum per channel goes out (more channels than the table holds: straight from the
// lanes).  SOLE: one workgroup does all, and stores.
constexpr int kTableChannels = 8192;

template <bool SOLE, bool TABLE = true>
__global__ __launch_bounds__(kThreads) void absmax_periodic_kernel(const float* __restrict__ x, SpanArgs g, ChannelDiv d,
                                                                   uint32_t* __restrict__ thr) {
  extern __shared__ uint32_t s_max[];
  const int t = threadIdx.x;
  const int32_t channels = (int32_t)d.channels;
  if constexpr (TABLE) {
    for (int32_t c = t; c < channels; c += kThreads) s_max[c] = 0u;
    __syncthreads();
  }
  auto merge = [&](int64_t c, float m) {
    if (m > 0.0f) atomicMax((TABLE ? s_max : thr) + c, __float_as_uint(m));
  };
  const int32_t rg = (int32_t)(blockIdx.x / (uint32_t)g.nseg);
  const int32_t j = (int32_t)(blockIdx.x - (uint32_t)rg * (uint32_t)g.nseg) * g.seg_len + t;
  const int64_t nvec = g.total >> 2;
  if (blockIdx.x == 0 && t < (int)(g.total & 3)) {
    int64_t k;
    const int64_t i = 4 * nvec + t;
    const int64_t c = channel_at(d, i, k);
    merge(c, absmax_step(0.0f, x[i]));
  }
  if (t < g.seg_len && j < g.span) {
    constexpr int U = kVecPerLane;
    float m[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    int64_t v = (int64_t)rg * g.rows * g.span + j;
    const int64_t end = v + (int64_t)g.rows * g.span < nvec ? v + (int64_t)g.rows * g.span : nvec;
    for (; v < end; v += (int64_t)U * g.span) {
      v4f a[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        a[u] = v + (int64_t)u * g.span < end ? (v4f)load4(x, 4 * (v + (int64_t)u * g.span)) : v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) m[e] = absmax_step(m[e], a[u][e]);
    }
    int64_t c[4];
    channels4(d, 4ll * j, c);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      // (a run of elements of one channel merges in registers first)
      if (e + 1 < 4 && c[e + 1] == c[e]) m[e + 1] = absmax_step(m[e + 1], m[e]);
      else merge(c[e], m[e]);
    }
  }
  if constexpr (TABLE) {
    __syncthreads();
    for (int32_t c = t; c < channels; c += kThreads) {
      const uint32_t m = s_max[c];
      if constexpr (SOLE) thr[c] = m;
      else if (m) atomicMax(thr + c, m);
    }
  }
}

// The same for patterns of more than 32 vectors: a workgroup owns 16 vectors of the pattern (a run of up to 64 channels, 256
// bytes of a row) and 16 rows of it at a time.  With a whole pattern per workgroup every workgroup ends with an atomic for
// every channel, 256 of them on each address
// (4096 x 768, channel-last: 13.9 us, 5.9 so; 1024 x 4000 9.4, 7.1; 65536 x 220 20.0, 17.6).  Lanes of a column merge by lane exchange and through LDS, runs of one
// channel by lane exchange, and one integer maximum per channel goes out.
template <int U>
__global__ __launch_bounds__(kThreads) void absmax_slab_kernel(const float* __restrict__ x, int64_t total, int32_t lv, int32_t nslab,
                                                               int32_t groups, ChannelDiv d, uint32_t* __restrict__ thr) {
  __shared__ float s_m[kThreads / 64][64];
  const int t = threadIdx.x, jj = t & 15;
  const int32_t grp = (int32_t)(blockIdx.x / (uint32_t)nslab), slab = (int32_t)(blockIdx.x - (uint32_t)grp * (uint32_t)nslab);
  const int32_t j = slab * 16 + jj;
  const int64_t nvec = total >> 2;
  if (blockIdx.x == 0 && t < (int)(total & 3)) {
    int64_t k;
    const int64_t i = 4 * nvec + t;
    const float m = absmax_step(0.0f, x[i]);
    if (m > 0.0f) atomicMax(thr + channel_at(d, i, k), __float_as_uint(m));
  }
  float m[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  const int64_t step = (int64_t)groups * 16 * lv;
  if (j < lv) {
    for (int64_t v = ((int64_t)grp * 16 + (t >> 4)) * lv + j; v < nvec; v += U * step) {
      v4f a[U];
#pragma unroll
      for (int u = 0; u < U; ++u) a[u] = v + u * step < nvec ? (v4f)load4(x, 4 * (v + u * step)) : v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) m[e] = absmax_step(m[e], a[u][e]);
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
#pragma unroll
    for (int s = 16; s <= 32; s <<= 1) {
      const float o = __shfl_xor(m[e], s);
      m[e] = o > m[e] ? o : m[e];
    }
    if ((t & 63) < 16) s_m[t >> 6][4 * jj + e] = m[e];
  }
  __syncthreads();
  if (t >= 64) return;
  // lane t: element t of the slab
  float r = s_m[0][t];
#pragma unroll
  for (int w = 1; w < kThreads / 64; ++w) r = s_m[w][t] > r ? s_m[w][t] : r;
  int64_t k;
  const int32_t c = slab * 16 + (t >> 2) < lv ? (int32_t)channel_at(d, 64ll * slab + t, k) : -1;
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) {
    const float o = __shfl_down(r, s);
    const int32_t oc = __shfl_down(c, s);  // (by every lane; values of one channel may always merge)
    if (t + s < 64 && oc == c) r = o > r ? o : r;
  }
  const int32_t before = __shfl_up(c, 1);
  if (c >= 0 && (t == 0 || before != c) && r > 0.0f) atomicMax(thr + c, __float_as_uint(r));
}

// Few elements per channel: `lanes` (a power of two up to 64) lanes own a channel and store its result.
__global__ __launch_bounds__(kThreads) void absmax_lanes_kernel(const float* __restrict__ x, int64_t outer,
                                                                int64_t channels, int64_t inner, int32_t lanes,
                                                                float* __restrict__ thr) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t c = i / lanes;
  const int sub = (int)(i - c * lanes);
  float m = 0.0f;
  if (c < channels) {
    for (int64_t o = 0; o < outer; ++o) {
      const float* xr = x + (o * channels + c) * inner;
      for (int64_t k = sub; k < inner; k += 4 * lanes) {
        float a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = k + u * lanes < inner ? xr[k + u * lanes] : 0.0f;
#pragma unroll
        for (int u = 0; u < 4; ++u) m = absmax_step(m, a[u]);
      }
    }
  }
  for (int s = lanes >> 1; s >= 1; s >>= 1) {
    const float o = __shfl_xor(m, s);
    m = o > m ? o : m;
  }
  if (c < channels && sub == 0) thr[c] = m;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline int grid_for(int64_t jobs) {
  const int64_t cap = max_blocks(kThreads);  // one job per workgroup; the kernels loop beyond this
  return (int)(jobs < cap ? (jobs > 0 ? jobs : 1) : cap);
}

}  // namespace

hipError_t launch_simquant(const float* x, float* y, int64_t outer, int64_t channels, int64_t inner,
                           const float* scale, const int32_t* zp, int per_channel, int32_t clip_lo,
                           int32_t clip_hi, hipStream_t st) {
  const int64_t total = outer * channels * inner;
  if (total == 0) return hipSuccess;
  const float lo = (float)clip_lo, hi = (float)clip_hi;
  // Per-tensor parameters: the whole tensor is one row.
  int64_t rows = per_channel ? outer * channels : 1;
  int64_t row_len = per_channel ? inner : total;
  if (row_len % 4 == 0 && row_len >= 512 && aligned16(x) && aligned16(y)) {
    const int64_t inner_vec = row_len / 4;
    int32_t nseg, seg_len;
    split_row(inner_vec, kVecPerLane, &nseg, &seg_len);
    return launch_kernel((simquant_rows_kernel<kVecPerLane, false>), dim3(grid_for(rows * nseg)), dim3(kThreads), 0, st,
                       reinterpret_cast<const v4f*>(x), reinterpret_cast<v4f*>(y), rows,
                       (int32_t)(per_channel ? channels : 1), inner_vec, nseg, seg_len, scale, zp,
                       per_channel, JobDiv{reciprocal32(nseg), reciprocal32(per_channel ? channels : 1)}, lo, hi, 0, 0);
  }
  return launch_ragged<SimquantOp<false, true>, SimquantOp<false, false>, SimquantOp<false, true, false>>(
      total, per_channel ? channels : 1, per_channel ? inner : total, st, x, y, scale, zp, lo, hi, 0, 0);
}

hipError_t launch_simquant_wrap(const float* x, float* y, int64_t outer, int64_t channels, int64_t inner,
                                const float* scale, const int32_t* zp, int per_channel, int32_t wrap_bits,
                                int32_t wrap_signed, int32_t clip_lo, int32_t clip_hi, hipStream_t st) {
  const int64_t total = outer * channels * inner;
  if (total == 0) return hipSuccess;
  const float lo = (float)clip_lo, hi = (float)clip_hi;
  int64_t rows = per_channel ? outer * channels : 1;
  int64_t row_len = per_channel ? inner : total;
  if (row_len % 4 == 0 && row_len >= 512 && aligned16(x) && aligned16(y)) {
    const int64_t inner_vec = row_len / 4;
    int32_t nseg, seg_len;
    split_row(inner_vec, kVecPerLane, &nseg, &seg_len);
    return launch_kernel((simquant_rows_kernel<kVecPerLane, true>), dim3(grid_for(rows * nseg)), dim3(kThreads), 0, st,
                       reinterpret_cast<const v4f*>(x), reinterpret_cast<v4f*>(y), rows,
                       (int32_t)(per_channel ? channels : 1), inner_vec, nseg, seg_len, scale, zp,
                       per_channel, JobDiv{reciprocal32(nseg), reciprocal32(per_channel ? channels : 1)}, lo, hi,
                       wrap_bits, wrap_signed);
  }
  return launch_ragged<SimquantOp<true, true>, SimquantOp<true, false>, SimquantOp<true, true, false>>(
      total, per_channel ? channels : 1, per_channel ? inner : total, st, x, y, scale, zp, lo, hi, wrap_bits, wrap_signed);
}

hipError_t launch_simquant_batched(const float* x, float* y, int64_t outer, int64_t channels,
                                   int64_t inner, int32_t nbatch, const float* scale,
                                   const int32_t* zp, int per_channel, const int32_t* clip_lo,
                                   const int32_t* clip_hi, hipStream_t st) {
  const int64_t total = outer * channels * inner;
  if (total == 0 || nbatch == 0) return hipSuccess;
  if (nbatch > kMaxCandidates) return hipErrorInvalidValue;
  CandidateClips clips{};
  for (int b = 0; b < nbatch; ++b) {
    clips.lo[b] = (float)clip_lo[b];
    clips.hi[b] = (float)clip_hi[b];
  }
  const int32_t nparam = (int32_t)(per_channel ? channels : 1);
  const int64_t rows = per_channel ? outer * channels : 1;
  const int64_t row_len = per_channel ? inner : total;
  if (row_len % 4 == 0 && row_len >= 512 && aligned16(x) && aligned16(y)) {
    const int64_t inner_vec = row_len / 4;
    constexpr int kU = 2;  // fewer vectors in flight per lane: every one is stored nbatch times
    int32_t nseg, seg_len;
    split_row(inner_vec, kU, &nseg, &seg_len);
    auto run = [&](auto kern) {
      return launch_kernel(kern, dim3(grid_for(rows * nseg)), dim3(kThreads), 0, st, reinterpret_cast<const v4f*>(x),
                           reinterpret_cast<v4f*>(y), rows, nparam, inner_vec, nseg, seg_len, nbatch, nparam, scale, zp, per_channel,
                           JobDiv{reciprocal32(nseg), reciprocal32(nparam)}, clips);
    };
    // Several streams that go through the L2 reach memory less well than lines written back from it once they are too large for
    // the last-level cache (256 MB): 2 x 58 MB 28.2 us, nontemporal 30.2; 8 x 58 MB 99.0, 95.9.
    return total * nbatch <= (1 << 26) ? run(simquant_batched_rows_kernel<kU, true>) : run(simquant_batched_rows_kernel<kU, false>);
  }
  return launch_batched_ragged(x, y, total, nparam, per_channel ? inner : total, nbatch, scale, zp, clips, st);
}

template <typename Q, int OP>
static hipError_t launch_quant_t(const void* in, void* out, float* out2, int64_t outer, int64_t channels,
                                 int64_t inner, const float* scale, const int32_t* zp,
                                 int per_channel, int32_t clip_lo, int32_t clip_hi, hipStream_t st) {
  const int64_t total = outer * channels * inner;
  if (total == 0) return hipSuccess;
  const float lo = (float)clip_lo, hi = (float)clip_hi;
  const int64_t rows = per_channel ? outer * channels : 1;
  const int64_t row_len = per_channel ? inner : total;
  if (row_len % 4 == 0 && row_len >= 512 && aligned16(in) && aligned16(out) && aligned16(out2)) {
    const int64_t inner_vec = row_len / 4;
    int32_t nseg, seg_len;
    split_row(inner_vec, kVecPerLane, &nseg, &seg_len);
    return launch_kernel((quant_rows_kernel<Q, OP, kVecPerLane>), dim3(grid_for(rows * nseg)),
                       dim3(kThreads), 0, st, in, out, out2, rows, (int32_t)(per_channel ? channels : 1),
                       inner_vec, nseg, seg_len, scale, zp, per_channel,
                       JobDiv{reciprocal32(nseg), reciprocal32(per_channel ? channels : 1)}, lo, hi);
  }
  return launch_ragged<QuantOp<Q, OP, OP != 1>, QuantOp<Q, OP, false>, QuantOp<Q, OP, OP != 1, OP != 2>>(
      total, per_channel ? channels : 1, per_channel ? inner : total, st, in, out, out2, scale, zp, lo, hi);
}

// container: 0 int8, 1 uint8, 2 int16, 3 int32.  op 0: fp32 -> codes; 1: codes -> fp32;
// 2: fp32 -> codes and the simulated_quantize value (out2).
hipError_t launch_quant(const void* in, void* out, float* out2, int container, int op, int64_t outer,
                        int64_t channels, int64_t inner, const float* scale, const int32_t* zp,
                        int per_channel, int32_t clip_lo, int32_t clip_hi, hipStream_t st) {
#define HAGO_QUANT_CASE(ID, T)                                                                       \
  case ID:                                                                                           \
    return op == 1 ? launch_quant_t<T, 1>(in, out, nullptr, outer, channels, inner, scale, zp,       \
                                          per_channel, clip_lo, clip_hi, st)                         \
         : op == 2 ? launch_quant_t<T, 2>(in, out, out2, outer, channels, inner, scale, zp,          \
                                          per_channel, clip_lo, clip_hi, st)                         \
                   : launch_quant_t<T, 0>(in, out, nullptr, outer, channels, inner, scale, zp,       \
                                          per_channel, clip_lo, clip_hi, st);
  switch (container) {
    HAGO_QUANT_CASE(0, int8_t)
    HAGO_QUANT_CASE(1, uint8_t)
    HAGO_QUANT_CASE(2, int16_t)
    HAGO_QUANT_CASE(3, int32_t)
    default: return hipErrorInvalidValue;
  }
#undef HAGO_QUANT_CASE
}

hipError_t launch_absmax(const float* x, int64_t outer, int64_t channels, int64_t inner,
                         int per_channel, float* thr, hipStream_t st) {
  const int64_t nthr = per_channel ? channels : 1;
  if (nthr == 0) return hipSuccess;
  uint32_t* t = reinterpret_cast<uint32_t*>(thr);
  auto zero_first = [&] {
    // (a fill kernel, not hipMemsetAsync: the call may be captured into a graph)
    return launch_kernel(fill_zero_kernel, dim3(grid_for((nthr + kThreads - 1) / kThreads)), dim3(kThreads), 0, st, t, nthr);
  };
  const int64_t total = outer * channels * inner;
  if (total == 0) return zero_first();
  const int64_t nchan = per_channel ? channels : 1;
  const int64_t nouter = nchan > 1 ? outer : 1, row_len = nchan > 1 ? inner : total;  // one channel: one row
  // Rows shorter than a workgroup's 1024 elements: merged in LDS where their channels come back often ...
  SpanArgs g;
  if (row_len < 4 * kThreads && periodic_split(total, nchan, row_len, kVecPerLane, WholeLines::kNever, &g)) {
    const bool table = nchan <= kTableChannels;
    const size_t lds = table ? (size_t)nchan * sizeof(uint32_t) : 0;
    if (table && total <= 16384 && g.nseg == 1) {  // one workgroup: no second launch to zero the thresholds
      g.rows = (int32_t)g.spans;
      return launch_kernel((absmax_periodic_kernel<true>), dim3(1), dim3(kThreads), lds, st, x, g, channel_div(total, nchan, row_len), t);
    }
    const int64_t lv = channel_period(nchan, row_len), nvec = total / 4, nslab = (lv + 15) / 16;
    if (lv > 32 && nchan * row_len >= 128 && nchan < (1ll << 31) && nslab <= 65536) {  // (no channel twice in a slab)
      // about 1.5 workgroups per CU, each with at least one round of 4 x 16 rows
      const int64_t prows = (nvec + lv - 1) / lv;
      int64_t groups = 384 / nslab, most = (prows + 63) / 64;
      groups = groups < 1 ? 1 : (groups > most ? most : groups);
      if (const hipError_t e = zero_first(); e != hipSuccess) return e;
      return launch_kernel((absmax_slab_kernel<kVecPerLane>), dim3((unsigned)(nslab * groups)), dim3(kThreads), 0, st, x, total,
                         (int32_t)lv, (int32_t)nslab, (int32_t)groups, channel_div(total, nchan, row_len), t);
    }
    g.rows = absmax_span_rows(g);
    if (const hipError_t e = zero_first(); e != hipSuccess) return e;
    const int64_t wgs = ((g.spans + g.rows - 1) / g.rows) * g.nseg;
    auto kern = table ? absmax_periodic_kernel<false, true> : absmax_periodic_kernel<false, false>;
    return launch_kernel(kern, dim3((unsigned)wgs), dim3(kThreads), lds, st, x, g, channel_div(total, nchan, row_len), t);
  }
  // ... a few lanes per channel where they do not.
  if (row_len < 4 * kThreads && nouter * row_len <= 65536) {
    int32_t lanes = 1;
    while (lanes < 64 && lanes * 4 < row_len) lanes *= 2;
    const int64_t wgs = (nchan * lanes + kThreads - 1) / kThreads;
    if (wgs <= max_blocks(kThreads)) {
      return launch_kernel(absmax_lanes_kernel, dim3((unsigned)wgs), dim3(kThreads), 0, st, x, nouter, nchan, row_len, lanes, thr);
    }
  }
  int32_t nseg, seg_len;
  split_row(row_len / 4 > 0 ? row_len / 4 : 1, kVecPerLane, &nseg, &seg_len);
  if (nchan >= (1ll << 31) || row_len / 4 / kThreads >= (1ll << 31)) return hipErrorInvalidValue;
  // A channel of up to 64 KB, or enough channels to fill the chip: one workgroup each, which stores.
  if (nouter * row_len <= 16384 || nchan >= 1024) {
    const int64_t cap = 256 * 32;
    return launch_kernel((absmax_rows_kernel<kVecPerLane, true>), dim3((unsigned)(nchan < cap ? nchan : cap)), dim3(kThreads), 0,
                       st, x, nouter, (int32_t)nchan, row_len, 1, (int32_t)(row_len / 4), 1, per_channel, t);
  }
  // about four workgroups per CU: rows of one channel beyond that share a workgroup (config 4
  // tensor: 12.8 us with 8 rows per workgroup, 15.8 us with one)
  int64_t rows_per_wg = nouter * nchan * nseg / (256 * 4);
  if (rows_per_wg < 1) rows_per_wg = 1;
  const int64_t ogroups = (nouter + rows_per_wg - 1) / rows_per_wg;
  const int64_t jobs = nchan * nseg * ogroups;
  const int64_t cap = 256 * 32;
  if (const hipError_t e = zero_first(); e != hipSuccess) return e;
  return launch_kernel((absmax_rows_kernel<kVecPerLane, false>), dim3((unsigned)(jobs < cap ? jobs : cap)),
                     dim3(kThreads), 0, st, x, nouter, (int32_t)nchan, row_len, nseg, seg_len, (int32_t)ogroups,
                     per_channel, t);
}

template <typename AccT>
static hipError_t launch_requantize_t(const AccT* acc, int64_t outer, int64_t channels,
                                      int64_t inner, const RequantArgs& rq, void* out,
                                      hipStream_t st) {
  const int64_t total = outer * channels * inner;
  if (total == 0) return hipSuccess;
  const RequantScalars rs{rq.z_out, rq.clip_lo - rq.z_out, rq.clip_hi - rq.z_out, rq.half_away};
  const int pc = rq.per_channel;
  int64_t rows = pc ? outer * channels : 1;
  int64_t row_len = pc ? inner : total;
  const bool io_aligned = aligned16(acc) && aligned16(out);
  if (row_len % 4 == 0 && row_len >= 512 && io_aligned) {
    const int64_t inner_vec = row_len / 4;
    int32_t nseg, seg_len;
    split_row(inner_vec, kVecPerLane, &nseg, &seg_len);
    auto kern = rq.half_away ? requant_rows_kernel<AccT, kVecPerLane, true>
                : (rq.multiplier ? requant_rows_kernel<AccT, kVecPerLane, false>
                                 : requant_rows_kernel<AccT, kVecPerLane, false, true>);
    return launch_kernel(kern, dim3(grid_for(rows * nseg)), dim3(kThreads), 0, st,
                       acc, reinterpret_cast<uint32_t*>(out), rows, (int32_t)(pc ? channels : 1),
                       inner_vec, nseg, seg_len, rq.multiplier, rq.shift, pc,
                       JobDiv{reciprocal32(nseg), reciprocal32(pc ? channels : 1)}, rs);
  }
  const int64_t ch = pc ? channels : 1, in = pc ? inner : total;
  if (rq.half_away)
    return launch_ragged<RequantOp<AccT, true>, RequantOp<AccT, true>, RequantOp<AccT, true>>(total, ch, in, st, acc, out, rq.multiplier, rq.shift, rs);
  return launch_ragged<RequantOp<AccT, false>, RequantOp<AccT, false>, RequantOp<AccT, false>>(total, ch, in, st, acc, out, rq.multiplier, rq.shift, rs);
}

hipError_t launch_requantize(const void* acc, int acc16, int64_t outer, int64_t channels,
                             int64_t inner, const RequantArgs& rq, void* out, hipStream_t st) {
  if (acc16)
    return launch_requantize_t(static_cast<const int16_t*>(acc), outer, channels, inner, rq, out, st);
  return launch_requantize_t(static_cast<const int32_t*>(acc), outer, channels, inner, rq, out, st);
}

}  // namespace hago
