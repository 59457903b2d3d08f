// What every entry point says of a runtime that refuses.  Of each call of the library: with nothing refused it is fine, also where an
// earlier error of somebody else's is pending, which stays theirs; with any one of its calls refused it reports the device, makes no
// further launch, and leaves no error behind for the next caller.
#include "fake_runtime.h"

#include <cstdio>
#include <functional>
#include <string>

#include "hago.h"

using namespace fake;

namespace {

const hago_qtype u8{HAGO_U8, 8, 0, 128}, i8{HAGO_I8, 8, 1, 0}, i16{HAGO_I16, 16, 1, -11};
const hago_requant rq{at<int32_t>(8), at<int32_t>(9), 1, {HAGO_I8, 8, 1, 0}, -128, 127, HAGO_ROUND_UPWARD};

int check(const std::string& name, const std::function<hago_status()>& call) {
  int bad = 0;
  auto expect = [&](bool ok, const char* what, int n) {
    if (!ok) std::printf("%s, call %d refused: %s\n", name.c_str(), n, what), ++bad;
  };
  // (each kernel's LDS limit is raised by its first call only: calls are refused from the first on)
  for (int n = 0;; ++n) {
    calls = launches_after = 0;
    refused = n;
    pending = hipSuccess;
    const hago_status s = call();
    if (calls <= n) {
      expect(n > 0, "the call reaches no kernel", -1);
      break;
    }
    expect(s == HAGO_ERR_DEVICE, "not reported", n);
    expect(pending == hipSuccess, "the error is left behind", n);
    expect(launches_after == 0, "a launch behind it", n);
    if (n > 16) break;
  }
  refused = -1;
  pending = hipErrorInvalidValue;
  expect(call() == HAGO_OK, "another's error is reported", -1);
  expect(pending == hipErrorInvalidValue, "another's error is taken", -1);
  return bad;
}

}  // namespace

int main() {
  int bad = 0;
  auto dense = [&](const char* name, const hago_qtype& a, const hago_qtype& w, int64_t M, int64_t K, int64_t N, int off, int path = 0, int tile = -1) {
    bad += check(name, [=] {
      hago_set_test_hook(HAGO_HOOK_GEMM_PATH, path);
      hago_set_test_hook(HAGO_HOOK_GENERAL_TILE, tile);
      const hago_status s = hago_qdense(at<char>(0) + off, a, at(1), w, at<int32_t>(2), M, N, K, HAGO_I32, &rq, at(3), 0, nullptr);
      hago_set_test_hook(HAGO_HOOK_GEMM_PATH, 0);
      hago_set_test_hook(HAGO_HOOK_GENERAL_TILE, -1);
      return s;
    });
  };
  hago_qtype w16 = i16;
  w16.zero_point = 0;
  dense("few tiles", u8, i8, 64, 256, 128, 0);
  dense("few tiles, unaligned", u8, i8, 64, 251, 128, 1);
  dense("few tiles, int16", i16, w16, 64, 256, 128, 0);
  dense("streaming tiles", u8, i8, 4096, 768, 768, 0);
  dense("large streaming tiles", i8, i8, 8192, 4096, 4096, 0);
  dense("any size, 64", u8, i8, 1021, 1283, 1001, 0);
  dense("any size, 128", i8, i8, 4099, 1283, 4099, 0);
  dense("any size, int16", i16, w16, 1024, 768, 768, 0);
  dense("any size, of many launches", i8, i8, 1 << 30, 1, 3, 0, 1, 3);

  enum { kPlain, kKeep, kReady, kStatic };
  auto conv = [&](const char* name, const hago_qtype& a, hago_layout layout, int B, int C, int H, int O, int k, int stride, int mode, int path = 0,
                  const hago_qtype* w = nullptr, int groups = 1, bool raw = false) {
    bad += check(name, [=] {
      hago_set_test_hook(HAGO_HOOK_GEMM_PATH, path);
      const hago_requant* r = raw ? nullptr : &rq;
      const int64_t need = hago_qconv2d_workspace_bytes(layout, B, C, H, H, O, k, k, stride, stride, k / 2, k / 2, groups);
      const hago_qtype& wt = w ? *w : i8;
      hago_status s;
      if (mode == kPlain)
        s = hago_qconv2d(at(0), a, at(1), wt, at<int32_t>(2), layout, B, C, H, H, O, k, k, stride, stride, k / 2, k / 2, groups, HAGO_I32, r, at(3), 0, nullptr);
      else if (mode == kStatic)
        s = hago_qconv2d_static(at(0), a, at(1), wt, at<int32_t>(2), layout, B, C, H, H, O, k, k, stride, stride, k / 2, k / 2, groups, HAGO_I32, r, at(3), 0, nullptr);
      else
        s = hago_qconv2d_ws(at(0), a, at(1), wt, at<int32_t>(2), layout, B, C, H, H, O, k, k, stride, stride, k / 2, k / 2, groups, HAGO_I32, r, at(3), at(4), need,
                            mode == kReady ? HAGO_WS_WEIGHTS_READY : 0, nullptr);
      hago_set_test_hook(HAGO_HOOK_GEMM_PATH, 0);
      return s;
    });
  };
  conv("3x3 NCHW", u8, HAGO_NCHW, 1, 64, 56, 64, 3, 1, kPlain);
  conv("stem", u8, HAGO_NCHW, 8, 3, 224, 64, 7, 2, kPlain);
  conv("one launch, channel-last", u8, HAGO_NHWC, 57, 30, 56, 224, 5, 1, kPlain);
  conv("one launch, weights kept", u8, HAGO_NCHW, 32, 64, 56, 128, 3, 2, kKeep);
  conv("rewrite, NCHW", u8, HAGO_NCHW, 4, 256, 56, 256, 5, 1, kKeep);
  conv("rewrite, weights ready", u8, HAGO_NCHW, 4, 256, 56, 256, 5, 1, kReady);
  conv("rewrite, odd rows", u8, HAGO_NCHW, 4, 250, 55, 256, 5, 1, kKeep, 2);
  conv("rewrite, channel-last", u8, HAGO_NHWC, 4, 250, 56, 256, 5, 1, kKeep, 2);
  conv("static scratch", u8, HAGO_NCHW, 2, 250, 28, 256, 5, 1, kStatic);
  conv("gathered", i8, HAGO_NHWC, 1, 24, 14, 64, 3, 1, kPlain, 4);
  conv("gathered, NCHW", u8, HAGO_NCHW, 1, 24, 14, 64, 5, 1, kPlain, 4);
  conv("streamed, channel-last", i8, HAGO_NHWC, 4, 128, 55, 128, 3, 1, kPlain, 5);
  conv("streamed, weights kept", i8, HAGO_NHWC, 4, 128, 55, 128, 3, 1, kKeep);
  conv("1x1 NCHW", i8, HAGO_NCHW, 32, 24, 56, 144, 1, 1, kPlain);
  conv("1x1 NCHW, 64 channels, raw", i8, HAGO_NCHW, 32, 64, 56, 144, 1, 1, kPlain, 0, nullptr, 1, true);
  conv("1x1 NCHW, 96 channels", i8, HAGO_NCHW, 32, 96, 9, 144, 1, 1, kPlain);
  conv("1x1 NCHW, many channels", i8, HAGO_NCHW, 32, 480, 56, 80, 1, 1, kPlain);
  conv("1x1 NCHW, four wavefronts", i8, HAGO_NCHW, 1, 480, 14, 80, 1, 1, kPlain);
  conv("1x1 channel-last", i8, HAGO_NHWC, 16, 256, 28, 64, 1, 1, kPlain);
  conv("general, NCHW", u8, HAGO_NCHW, 2, 20, 28, 64, 3, 1, kPlain, 1);
  conv("general, channel-last", u8, HAGO_NHWC, 2, 20, 28, 64, 3, 1, kPlain, 1);
  conv("int16", i16, HAGO_NCHW, 2, 20, 28, 64, 3, 1, kPlain, 0, &w16);
  conv("int16, no zero point", w16, HAGO_NHWC, 2, 20, 28, 64, 3, 1, kPlain, 0, &w16);
  conv("depthwise, rows", i8, HAGO_NCHW, 8, 144, 56, 144, 3, 1, kPlain, 0, nullptr, 144);
  conv("depthwise, matrix", i8, HAGO_NCHW, 8, 144, 28, 144, 3, 1, kPlain, 0, nullptr, 144);
  conv("depthwise, channel-last", i8, HAGO_NHWC, 8, 144, 28, 144, 3, 2, kPlain, 0, nullptr, 144);
  conv("depthwise, any", i8, HAGO_NCHW, 8, 144, 28, 144, 5, 1, kPlain, 0, nullptr, 144);

  struct Shape { int64_t outer, channels, inner; };
  const int32_t lo[2] = {-128, -64}, hi[2] = {127, 63};
  for (const Shape& s : {Shape{32, 144, 3136}, {4096, 768, 1}, {3, 5, 7}, {40, 300, 50}, {2, 100003, 3}, {1 << 20, 1, 33}, {16, 3, 12544 * 7}})
    for (int pc = 0; pc < 2; ++pc) {
      const std::string shape = " " + std::to_string(s.outer) + " x " + std::to_string(s.channels) + " x " + std::to_string(s.inner) + (pc ? " by channel" : "");
      const auto [o, c, i] = s;
      auto* x = at<float>(0);
      auto* y = at<float>(1);
      auto* scale = at<float>(2);
      auto* zp = at<int32_t>(3);
      bad += check("simquant" + shape, [=] { return hago_simquant(x, y, o, c, i, scale, zp, pc, i8, -128, 127, nullptr); });
      bad += check("simquant_wrap" + shape, [=] { return hago_simquant_wrap(x, y, o, c, i, scale, zp, pc, i8, -128, 127, nullptr); });
      bad += check("simquant_batched" + shape, [=] { return hago_simquant_batched(x, y, o, c, i, 2, scale, zp, pc, i8, lo, hi, nullptr); });
      bad += check("quantize" + shape, [=] { return hago_quantize(x, y, o, c, i, scale, zp, pc, i16, -128, 127, nullptr); });
      bad += check("dequantize" + shape, [=] { return hago_dequantize(x, i8, y, o, c, i, scale, zp, pc, nullptr); });
      bad += check("simquant_codes" + shape, [=] { return hago_simquant_codes(x, y, at(5), o, c, i, scale, zp, pc, i8, -128, 127, nullptr); });
      bad += check("absmax" + shape, [=] { return hago_absmax(x, o, c, i, pc, y, nullptr); });
      hago_requant r = rq;
      for (int away = 0; away < 2; ++away) {
        r.per_channel = pc;
        r.rounding = away ? HAGO_ROUND_HALF_AWAY : HAGO_ROUND_UPWARD;
        bad += check("requantize" + shape, [=] { return hago_requantize(x, HAGO_I32, o, c, i, &r, y, nullptr); });
      }
    }
  bad += check("absmax of nothing", [] { return hago_absmax(nullptr, 0, 7, 5, 1, at<float>(0), nullptr); });
  bad += check("probe, matrix", [] { return hago_probe_mfma_i8(at(0), at(1), 4, 4, nullptr); });
  bad += check("probe, copy", [] { return hago_probe_copy(at(0), at(1), 4096, nullptr); });
  if (!bad) std::printf("launch statuses: ok\n");
  return bad != 0;
}
