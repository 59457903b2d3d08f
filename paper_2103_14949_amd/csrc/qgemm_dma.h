// The streaming dense kernels by their kinds of results (qgemm_common.h).  Each kind is compiled in a file of its own (qgemm_dma.hip,
// qgemm_dma_clipped.hip, qgemm_dma_other.hip, and the qgemm_line files so too), since a process that calls one loads all kernels of its file
// (the first calls of the encoder's four layers, all kinds in one file 6.7 ms, 2.2 so).
#pragma once

#include "qgemm_common.h"

namespace hago {

// Require: K % 16 == 0, K >= 16, 16-byte aligned operands, N*K and M*K below 2^31.
template <int OUT>
hipError_t qdense_dma(const QgemmParams& p, int shape, hipStream_t st);
template <int OUT>
hipError_t qdense_line(const QgemmParams& p, int shape, hipStream_t st);

// The same over the caller's channel-last operands (C % 16 == 0, 16-byte aligned, tensors below 2^31 bytes).
template <int OUT>
hipError_t qconv_dma_direct(const QgemmParams& p, int shape, hipStream_t st);

// Implicit-GEMM convolution over the prepacked operands (p.act: padded NHWC copy, p.wgt:
// [O][KH*KW*C] copy, p.g: geometry of the padded copy, p.K = KH*KW*C with C % 16 == 0).
// nchw_out: output [B,O,OH,OW] (activations are the P operand; kOutOther only) else [B,OH,OW,O].
template <int OUT>
hipError_t qconv_dma(const QgemmParams& p, bool nchw_out, hipStream_t st);

template <>
hipError_t qdense_dma<kOutFull>(const QgemmParams&, int, hipStream_t);
template <>
hipError_t qdense_line<kOutFull>(const QgemmParams&, int, hipStream_t);
template <>
hipError_t qconv_dma_direct<kOutFull>(const QgemmParams&, int, hipStream_t);
template <>
hipError_t qconv_dma<kOutFull>(const QgemmParams&, bool, hipStream_t);
template <>
hipError_t qdense_dma<kOutClipped>(const QgemmParams&, int, hipStream_t);
template <>
hipError_t qdense_line<kOutClipped>(const QgemmParams&, int, hipStream_t);
template <>
hipError_t qconv_dma_direct<kOutClipped>(const QgemmParams&, int, hipStream_t);
template <>
hipError_t qconv_dma<kOutClipped>(const QgemmParams&, bool, hipStream_t);
template <>
hipError_t qdense_dma<kOutOther>(const QgemmParams&, int, hipStream_t);
template <>
hipError_t qdense_line<kOutOther>(const QgemmParams&, int, hipStream_t);
template <>
hipError_t qconv_dma_direct<kOutOther>(const QgemmParams&, int, hipStream_t);
template <>
hipError_t qconv_dma<kOutOther>(const QgemmParams&, bool, hipStream_t);

}  // namespace hago
