// Which kernels serve a call: reads one call a line,
//   dense <act> <M> <K> <N> <raw> <byte offset of the activations> [<accumulator bits>, 32 unless given]
//   conv <act> <nhwc> <B> <C> <H> <W> <O> <KH> <KW> <stride_h> <stride_w> <pad_h> <pad_w> <raw> <path> <shape>
// (act: u8, i8 or i16; path and shape: the test hooks) and prints the kernels that it launches on a line, separated by tabs.
#include "fake_runtime.h"

#include <iostream>
#include <sstream>

#include "hago.h"

int main() {
  const hago_qtype w8{HAGO_I8, 8, 1, 0}, w16{HAGO_I16, 16, 1, 0};
  const hago_requant rq{fake::at<int32_t>(8), fake::at<int32_t>(9), 1, {HAGO_I8, 8, 1, 0}, -128, 127, HAGO_ROUND_UPWARD};
  std::string line;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    std::string what, act;
    in >> what >> act;
    const hago_qtype a = act == "u8" ? hago_qtype{HAGO_U8, 8, 0, 121} : act == "i16" ? hago_qtype{HAGO_I16, 16, 1, -7} : hago_qtype{HAGO_I8, 8, 1, 3};
    const hago_qtype& w = act == "i16" ? w16 : w8;
    fake::launched.clear();
    hago_status s = HAGO_ERR_PARAM;
    if (what == "dense") {
      int64_t M, K, N, raw, off, bits = 32;
      in >> M >> K >> N >> raw >> off;
      if (in && !(in >> bits)) in.clear(), bits = 32;
      const hago_dtype acc = bits == 16 ? HAGO_I16 : bits == 24 ? HAGO_I24 : HAGO_I32;
      s = hago_qdense(fake::at<char>(0) + off, a, fake::at(1), w, fake::at<int32_t>(2), M, N, K, acc, raw ? nullptr : &rq, fake::at(3), 0, nullptr);
    } else if (what == "conv") {
      int64_t nhwc, B, C, H, W, O, KH, KW, sh, sw, ph, pw, raw, path, shape;
      in >> nhwc >> B >> C >> H >> W >> O >> KH >> KW >> sh >> sw >> ph >> pw >> raw >> path >> shape;
      hago_set_test_hook(HAGO_HOOK_GEMM_PATH, (int32_t)path);
      hago_set_test_hook(HAGO_HOOK_GENERAL_TILE, (int32_t)shape);
      s = hago_qconv2d(fake::at(0), a, fake::at(1), w, fake::at<int32_t>(2), nhwc ? HAGO_NHWC : HAGO_NCHW, B, C, H, W, O, (int32_t)KH, (int32_t)KW,
                       (int32_t)sh, (int32_t)sw, (int32_t)ph, (int32_t)pw, 1, HAGO_I32, raw ? nullptr : &rq, fake::at(3), 0, nullptr);
    }
    if (s != HAGO_OK || !in) {
      std::cerr << line << ": " << hago_status_string(s) << "\n";
      return 1;
    }
    for (char& c : fake::launched)
      if (c == '\n') c = '\t';
    std::cout << fake::launched << "\n";
  }
  return 0;
}
