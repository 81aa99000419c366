// Implicit-GEMM convolutions on the register-staged mainloop (conv_reg.hip):
// fp32 data and channel counts or alignments the direct-to-LDS loaders do
// not take.  *done is false when a size limit leaves the layer to the
// general kernels.
#pragma once

#include "gemm_core.h"
#include "internal.h"

namespace mdnn {

mdnn_status_t conv_reg_fwd(const ConvGeom& g, const void* x, const void* w, const Epilogue& ep, mdnn_dtype_t io,
                           mdnn_dtype_t out, hipStream_t st, bool* done);
mdnn_status_t conv_reg_bwd_data(const ConvGeom& g, const void* dy, const void* w, const Epilogue& ep,
                                mdnn_dtype_t io, mdnn_dtype_t out, hipStream_t st, bool* done);
// Splits of the filter gradient's K (0: not taken).
SplitPlan conv_reg_filter_plan(const ConvGeom& g, mdnn_dtype_t io);
mdnn_status_t conv_reg_bwd_filter(const ConvGeom& g, const void* x, const void* dy, float* dw, void* ws,
                                  mdnn_dtype_t io, hipStream_t st, bool* done, ReduceBatch* defer);

}  // namespace mdnn
