// How the elementwise kernels for short, ragged and channel-last rows divide a tensor.  Plain C++, so that a host program can go
// through it.
//
// The channels of consecutive vectors (of four elements) come back every lv vectors (channels * inner elements, taken two
// or four times where that is not a multiple of four).  `span` is a multiple of lv of about a workgroup's
// width where lv is small, lv itself where it is large; vector j of every span has the same four channels.  A
// workgroup owns the vectors [seg * seg_len, ...) of `rows` consecutive spans: the lane's parameters
// stay in registers, what is left per element is the operator itself.
#pragma once

#include <cstdint>

namespace hago {

constexpr int kSpanThreads = 256;  // of a workgroup

struct SpanArgs {
  int64_t total;  // elements
  int64_t spans;
  int32_t span, nseg, seg_len, rows;
};

// Vectors after which the channels of a vector come back.
inline int64_t channel_period(int64_t channels, int64_t inner) {
  const int64_t p = channels * inner;
  return p % 4 == 0 ? p / 4 : (p % 2 == 0 ? p / 2 : p);
}

// Spans of whole 64-byte lines (four vectors of fp32) where that keeps five eighths of the lanes:
//   kAlways: for results that go through the L2, which then are whole lines (65536 x 45 channel-last: quantize 5.7 -> 5.3 us, dequantize 4.3 -> 3.9;
//     20000 x 33, 132 lanes of 231: 3.3 -> 3.6);
//   kRounds: for the batched candidates, whose results do not.  Their time goes in rounds of a workgroup per CU.  Up to five candidates
//     gain by whole lines where the rounds get a tenth shorter by them (ratios of the times: 3 channels of 9, 20000 rows, rounds 0.89, one to four candidates 0.88 to
//     0.95; rounds as long: 7 of 7, 40000, 1.04 to 1.12, 12 of 17, 20000, 1.04 to 1.23).  From six on the stores are most of it: of channels with more than one element in
//     a row they gain with rounds up to 1.07 as long, too (eight: 3 of 9, 100000, 1.04, 0.88; 2 of 13, 300000, 1.05, 0.84; 12 of 17, 60000, 1.07, 0.91; 5 of 5, 60000,
//     1.07, 1.07; 7 of 7, 100000, 1.12, 1.17; 5 of 5, 200000, 1.12, 1.28), and where whole lines leave next to no lane idle (3 channels last, 70000 to 4000000, 0.82
//     to 0.97).  Else every workgroup looks up four times the parameters for fewer elements (eight, 45 channels last, 65536, 1.04; 51, 50000, 1.39; 50, 60000, 1.24);
//   kNever: for max-abs, which stores nothing (37 channels last, 3000 5.7, 6.5, 700000 24.5, 28.7).
enum class WholeLines { kAlways, kRounds, kNever };

// Whether the pattern comes back often enough (four times) for the periodic form, and its split: workgroups
// own at least u spans each and, beyond eight workgroups per CU, more of them.
inline bool periodic_split(int64_t total, int64_t channels, int64_t inner, int u, WholeLines lines, SpanArgs* g, int candidates = 1) {
  const int64_t nvec = total / 4, lv = channel_period(channels, inner);
  if (channels == 1 || nvec / lv < 4 || lv >= (1ll << 30)) return false;
  auto split = [&](int64_t span) {
    SpanArgs a;
    a.total = total;
    a.span = (int32_t)span;
    a.spans = (nvec + span - 1) / span;
    a.nseg = (int32_t)((span + kSpanThreads - 1) / kSpanThreads);
    a.seg_len = (int32_t)((span + a.nseg - 1) / a.nseg);
    int64_t rows = a.spans * a.nseg / (256 * 8);
    rows = (rows + u - 1) / u * u;
    if (rows < u) rows = u;
    while (rows > 1 && ((a.spans + rows - 1) / rows) * a.nseg < 256) rows /= 2;  // small tensors: spread over the CUs
    a.rows = (int32_t)rows;
    return a;
  };
  auto workgroups = [](const SpanArgs& a) { return ((a.spans + a.rows - 1) / a.rows) * a.nseg; };
  const int64_t most = lv <= kSpanThreads ? kSpanThreads / lv : 1;
  const int64_t line = lv % 4 == 0 ? 1 : (lv % 2 == 0 ? 2 : 4), whole = most / line * line;
  const bool cuttable = lv <= kSpanThreads && whole < most && 8 * whole >= 5 * most;
  *g = split(lv * (cuttable && lines == WholeLines::kAlways ? whole : most));
  if (cuttable && lines == WholeLines::kRounds) {
    const SpanArgs cut = split(lv * whole);
    auto length = [&](const SpanArgs& a) { return (workgroups(a) + 255) / 256 * a.rows * a.span; };
    const int percent = candidates < 6 ? 90 : inner > 1 ? 107 : 64 * (most - whole) <= most ? 100 : 90;
    if (100 * length(cut) <= percent * length(*g)) *g = cut;
  }
  return workgroups(*g) < (1ll << 31);
}

// Spans of a workgroup of max-abs.  Every workgroup ends with an atomic per channel, one after another on each address, which is most of a
// small tensor's time, while a large one needs workgroups that load: as many as the root of its vectors, over four, from 128 to 512.  Us with 128, 192, 256, 320, 384 and 512 of
// them: 51 channels last, 20000 rows, 6.7, 7.3, 8.4, 8.4, 9.9, 13.0; 45, 65536, 9.4, 8.8, 9.3, 9.3, 10.2, 11.0; 64, 100000, 14.4, 13.3, 13.1, 12.9, 13.9, 15.4; 64, 200000, 24.2, 19.6, 18.2,
// 17.3, 17.8, 18.7; 37, 700000, 49.2, 35.1, 29.7, 26.5, 24.6, 23.9; 64, 2000000, 197, 140, 111, 92.6, 83.6, 79.6.  Spans go by fours, so few of them are a multiple of it (37, 700000, 57
// and 56 spans 23.9, 23.3).
inline int32_t absmax_span_rows(const SpanArgs& g) {
  const int64_t all = g.spans * g.nseg, root = (int64_t)(__builtin_sqrt((double)(g.total / 4)) / 4), wgs = root < 128 ? 128 : root > 512 ? 512 : root;
  const int64_t rows = all / wgs;
  return (int32_t)(rows < 8 ? (all + wgs - 1) / wgs : rows < 32 ? (rows + 2) / 4 * 4 : rows);
}

}  // namespace hago
