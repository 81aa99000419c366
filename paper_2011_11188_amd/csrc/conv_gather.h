// Forward convolutions with a short reduction (conv_gather.hip).
#pragma once

#include "gemm_core.h"
#include "internal.h"

namespace mdnn {

// *done: whether the layer was taken: r runs of s * c_in elements, padded to
// 8 (16-bit) or 4 (fp32) each, of at most 192 (96) in all; above 64 (fp32:
// 96) only channel counts that are no multiple of 8.
mdnn_status_t conv_gather_fwd(const ConvGeom& g, const void* x, const void* w, const Epilogue& ep, mdnn_dtype_t io,
                              mdnn_dtype_t out, hipStream_t st, bool* done);

}  // namespace mdnn
