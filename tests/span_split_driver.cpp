// Goes through the division of channel-last and ragged tensors of all sizes into spans: every vector has its workgroup and lane, results
// through the L2 are whole lines where that keeps enough lanes, and an operator that has nothing of lines keeps all of them.
#include "span_split.h"

#include <cstdio>

using namespace hago;

namespace {

int failures = 0;
void expect(bool ok, const char* what, int64_t outer, int64_t channels, int64_t inner) {
  if (!ok && failures++ < 20) std::printf("%s: %lld x %lld x %lld\n", what, (long long)outer, (long long)channels, (long long)inner);
}

}  // namespace

int main() {
  const int64_t inners[] = {1, 2, 3, 9, 20, 49, 255}, outers[] = {1, 7, 64, 900, 3000, 12000, 20000, 65536, 700001};
  const WholeLines rules[] = {WholeLines::kAlways, WholeLines::kRounds, WholeLines::kNever};
  int64_t cut = 0, kept = 0;
  for (int64_t channels = 1; channels <= 600; ++channels)
    for (int64_t inner : inners)
      for (int64_t outer : outers) {
        const int64_t total = outer * channels * inner, nvec = total / 4, lv = channel_period(channels, inner);
        if (total >= 1ll << 32) continue;
        auto is = [&](bool ok, const char* what) { expect(ok, what, outer, channels, inner); };
        is(lv * 4 % (channels * inner) == 0, "the channels come back");
        for (WholeLines lines : rules)
          for (int u = 2; u <= 4; u += 2) {
            SpanArgs g;
            if (!periodic_split(total, channels, inner, u, lines, &g)) {
              is(channels == 1 || nvec / lv < 4, "periodic");
              continue;
            }
            is(g.total == total && g.rows >= 1 && g.nseg >= 1, "sizes");
            is(g.span % lv == 0 && g.spans * g.span >= nvec && (g.spans - 1) * g.span < nvec, "spans");
            is(g.seg_len <= kSpanThreads && (int64_t)g.seg_len * g.nseg >= g.span && (int64_t)g.seg_len * (g.nseg - 1) < g.span, "segments");
            is((g.spans + g.rows - 1) / g.rows * g.nseg < 1ll << 31, "one launch");
            if (lv > kSpanThreads) continue;
            const int64_t lanes = kSpanThreads / lv * lv, fewer = kSpanThreads / lv / 4 * 4 * lv;
            if (g.span != lanes) {
              is(lines != WholeLines::kNever && g.span % 4 == 0 && 8 * g.span >= 5 * lanes, "whole lines");
              ++cut;
            } else {
              is(lines != WholeLines::kAlways || g.span % 4 == 0 || 8 * fewer < 5 * lanes, "all lanes");
              ++kept;
            }
            if (lines == WholeLines::kRounds) {  // rounds of a workgroup per CU, by lanes, against those with all lanes
              SpanArgs all, many;
              periodic_split(total, channels, inner, u, WholeLines::kNever, &all);
              periodic_split(total, channels, inner, u, lines, &many, 8);
              auto rounds = [](const SpanArgs& a) { return ((a.spans + a.rows - 1) / a.rows * a.nseg + 255) / 256 * a.rows * a.span; };
              is(g.span == lanes || 10 * rounds(g) <= 9 * rounds(all), "rounds of few candidates");
              is(many.span == lanes || many.span == fewer || many.span % 4 == 0, "lanes of many candidates");
              is(many.span == lanes || 100 * rounds(many) <= (inner > 1 ? 107 : 100) * rounds(all), "rounds of many candidates");
              is(g.span == lanes || many.span == g.span, "what is whole lines for few is for many");
              is(many.spans * many.span >= nvec && (many.spans - 1) * many.span < nvec, "spans of many candidates");
            }
            if (lines == WholeLines::kNever) {
              g.rows = absmax_span_rows(g);
              const int64_t workgroups = (g.spans + g.rows - 1) / g.rows * g.nseg;
              is(g.rows >= 1 && workgroups <= 640 && (g.spans * g.nseg < 128 || workgroups >= 64), "workgroups of max-abs");
              is(nvec < 1 << 23 || workgroups >= 480, "workgroups of a large max-abs");
            }
          }
      }
  std::printf("span split: %s (%lld cut, %lld of all lanes)\n", failures ? "FAILED" : "ok", (long long)cut, (long long)kept);
  return failures != 0 || !cut || !kept;
}
