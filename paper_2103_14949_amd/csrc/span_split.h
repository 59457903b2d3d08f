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
//   kFewerRounds: for the batched candidates, whose results do not, only as a shorter span: their time goes in rounds of a workgroup per CU, and fewer lanes
//     and a round more are a loss, fewer lanes in as many rounds a gain (eight candidates, us, all lanes and whole lines: 45 channels last, 12000 10.9, 9.9,
//     20000 12.1, 12.9, 24000 15.0, 13.1, 28000 14.9, 14.9, 32000 17.9, 15.0, 50000 23.0, 27.4; 37, 4000 7.9, 7.2, 20000 10.5, 11.5, 60000 22.2, 24.2).
//     Where every element of a vector has a channel of its own, each workgroup also looks up four times the parameters, and it takes a tenth fewer (as
//     many rounds: 200 channels last, 9000 20.9, 21.8; 10 channels of 9, 20000 16.9, 14.8; 2 of 45, 20000 16.5, 14.7);
//   kNever: for max-abs, which stores nothing (37 channels last, 3000 5.7, 6.5, 700000 24.5, 28.7).
enum class WholeLines { kAlways, kFewerRounds, kNever };

// Whether the pattern comes back often enough (four times) for the periodic form, and its split: workgroups
// own at least u spans each and, beyond eight workgroups per CU, more of them.
inline bool periodic_split(int64_t total, int64_t channels, int64_t inner, int u, WholeLines lines, SpanArgs* g) {
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
  if (cuttable && lines == WholeLines::kFewerRounds) {
    const SpanArgs cut = split(lv * whole);
    auto length = [&](const SpanArgs& a) { return (workgroups(a) + 255) / 256 * a.rows * a.span; };
    if (inner > 1 ? length(cut) <= length(*g) : 10 * length(cut) < 9 * length(*g)) *g = cut;
  }
  return workgroups(*g) < (1ll << 31);
}

// Spans of a workgroup of max-abs.  Every workgroup ends with an atomic per channel, one after another on each address, which is most of a
// small tensor's time: 320 workgroups at most (us with up to 547 of them, with 320, 200 and 128: 37 channels last, 20000 9.8, 7.9, 6.6, 6.0, 65536 12.0,
// 8.8, 7.7, 7.3, but 200000 14.1, 13.3, 14.5, 17.8; 100 channels, 200000 21.7, 21.6, 25.2, 34.3).
inline int32_t absmax_span_rows(const SpanArgs& g) { return (int32_t)((g.spans * g.nseg + 319) / 320); }

}  // namespace hago
