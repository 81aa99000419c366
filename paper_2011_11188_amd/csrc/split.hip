// fp32 matrix products on the fp16 matrix cores: section 3.2's Eq. (1).
//
// An fp32 matrix X at a power-of-two scale s is split into fp16 matrices
//   X1 = RNE16(X / s),  X2 = RNE16((X / s - X1) * 2^11),
// so that X ~ s*X1 + s*2^-11*X2 to about 22 significant bits (X / s - X1 is
// exact in fp32, and scaling by powers of two is exact).  A product of two
// split matrices keeps three fp16 products,
//   A B ~ a b [ A1 B1 + 2^-11 (A1 B2 + A2 B1) ],
// which run on the MFMA GEMM engine as two launches: the two correction
// products as one GEMM over the concatenated depth [A1 | A2] x [B2 ; B1]
// (fp32 result, with beta*C folded in), then the leading product whose
// epilogue adds that result.  Both accumulate in fp32.
#include <cmath>

#include "common.h"
#include "internal.h"

namespace mdnn {
namespace {

constexpr float SHIFT_UP = 2048.0f;  // 2^11 = s / s2

// Automatic scale (the paper does not say how to pick a1): the power of two
// s = 2^(floor(log2 max|x|) - 14), which puts max|x| / s in [2^14, 2^15),
// inside fp16's range with its leading bits in the normal range; s = 1 when
// max|x| is 0, Inf or NaN; s >= 2^-126.  Pass 1: max |x| as fp32 bit
// patterns (ordered like the magnitudes; NaN above Inf), one atomic max per
// block into a word that starts at 0.
struct AbsmaxOp {
  const float* x;
  int64_t rows, cols, ldx, chunks;  // chunks: 1024-column pieces per row
  uint32_t* bits;                   // null: not this operand
};
// (a few hundred blocks in all, each over many row pieces: with a block and an
// atomic per 256 elements the serialised atomics took 200 us on 704 x 2420)
__global__ void __launch_bounds__(256) absmax_bits_kernel(AbsmaxOp a, AbsmaxOp b) {
  const AbsmaxOp& o = blockIdx.y == 0 ? a : b;
  if (!o.bits) return;
  uint32_t m = 0;
  auto take = [&](float f) {
    const uint32_t u = __float_as_uint(f) & 0x7fffffffu;
    m = u > m ? u : m;
  };
  const int64_t n = o.rows * o.chunks;
  for (int64_t q0 = blockIdx.x; q0 < n; q0 += 4 * (int64_t)gridDim.x) {
    // four pieces in flight (a piece past the end repeats the first)
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
    f4 t[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t q = q0 + u * (int64_t)gridDim.x < n ? q0 + u * (int64_t)gridDim.x : q0;
      const int64_t row = q / o.chunks, c = (q - row * o.chunks) * 1024 + threadIdx.x * 4;
      const float* p = o.x + row * o.ldx;
      t[u] = (f4){0.f, 0.f, 0.f, 0.f};
      if (c + 4 <= o.cols) {
        t[u] = *(const __attribute__((address_space(1))) f4*)(p + c);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (c + e < o.cols) take(p[c + e]);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) take(t[u].x), take(t[u].y), take(t[u].z), take(t[u].w);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint32_t w = (uint32_t)__shfl_xor((int)m, off);
    m = w > m ? w : m;
  }
  __shared__ uint32_t wmax[4];
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) m = wmax[w] > m ? wmax[w] : m;
    m = wmax[0] > m ? wmax[0] : m;
    if (m) atomicMax(o.bits, m);
  }
}

__device__ float auto_scale(uint32_t bits) {
  if (bits == 0 || bits >= 0x7f800000u) return 1.0f;
  int e = ilogbf(__uint_as_float(bits)) - 14;  // floor(log2 max|x|) - 14
  if (e < -126) e = -126;
  return ldexpf(1.0f, e);
}

// One operand: rows x cols fp32 (leading dimension ldx) -> hi / lo fp16.
// inv_scale = 1/s (a power of two, so
// x * inv_scale is exact for normal results), or 1 / *scale_dev, or from the
// bit maximum in *bits when the scale is chosen on the device.
struct SplitOp {
  const float* x;
  int64_t rows, cols, ldx;
  uint16_t *hi, *lo;
  int64_t ldh, ldl;
  float inv_scale;
  const float* scale_dev;
  const uint32_t* bits;
  int32_t lanes_log2;  // threads per row piece, four columns each
  int64_t chunks;      // pieces per row
  int64_t blocks;      // blocks of this operand
};
constexpr int SPLIT_LANES_LOG2 = 8;  // a piece has at most a block's 256 threads

// Blocks of both operands of a product in one launch (op b may be empty).
// HBM-bound (4 B read, 4 B written per element): four elements per thread by
// unaligned 16- and 8-byte accesses; element by element, one launch per
// operand, two 2048 x 2048 operands took 21 us.  A block holds as many rows as
// their pieces leave room for: with one row per block tall narrow matrices are
// bound by block launches (56512 x 114 38.5 -> 11.4 us, 184512 x 31 119 -> 13).
// ab_scale (nullable) receives
// the product of the two automatic or fixed scales.
__global__ void __launch_bounds__(256) split_f16_kernel(SplitOp a, SplitOp b, float* ab_scale) {
  for (int64_t g = blockIdx.x; g < a.blocks + b.blocks; g += gridDim.x) {
    const bool first = g < a.blocks;
    const SplitOp& o = first ? a : b;
    const int64_t blk = first ? g : g - a.blocks;
    float inv = o.inv_scale;
    if (o.scale_dev) inv = 1.0f / *o.scale_dev;  // exact: a power of two in [2^-126, 2^113]
    if (o.bits) inv = 1.0f / auto_scale(*o.bits);
    if (ab_scale && g == 0 && threadIdx.x == 0)
      *ab_scale = (a.bits ? auto_scale(*a.bits) : 1.0f / a.inv_scale) * (b.bits ? auto_scale(*b.bits) : 1.0f / b.inv_scale);
    const int64_t grp = blk / o.chunks, piece = blk - grp * o.chunks;
    const int lane = threadIdx.x & ((1 << o.lanes_log2) - 1), sub = threadIdx.x >> o.lanes_log2;
    const int64_t row = (grp << (SPLIT_LANES_LOG2 - o.lanes_log2)) + sub, c = ((piece << o.lanes_log2) + lane) * 4;
    if (row >= o.rows || c >= o.cols) continue;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    const float* p = o.x + row * o.ldx + c;
    if (c + 4 <= o.cols) {
      typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
      const f4 t = *(const __attribute__((address_space(1))) f4*)p;
      v[0] = t.x, v[1] = t.y, v[2] = t.z, v[3] = t.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c + e < o.cols) v[e] = p[e];
    }
    uint16_t h[4], l[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float w = v[e] * inv;
      h[e] = f32_to_f16(w);
      const float r = w - f16_to_f32(h[e]);  // exact: w and h agree in their leading 11 bits
      l[e] = f32_to_f16(r * SHIFT_UP);
    }
    uint16_t* dh = o.hi + row * o.ldh + c;
    uint16_t* dl = o.lo + row * o.ldl + c;
    if (c + 4 <= o.cols) {
      typedef uint32_t u2 __attribute__((ext_vector_type(2), aligned(2)));
      *(__attribute__((address_space(1))) u2*)dh =
          (u2){(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16)};
      *(__attribute__((address_space(1))) u2*)dl =
          (u2){(uint32_t)l[0] | ((uint32_t)l[1] << 16), (uint32_t)l[2] | ((uint32_t)l[3] << 16)};
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c + e < o.cols) dh[e] = h[e], dl[e] = l[e];
    }
  }
}

// the automatic scale of one matrix, in place (word 0 only)
__global__ void scale_one_kernel(uint32_t* word) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  *(float*)word = auto_scale(*word);
}

bool power_of_two(float s) {
  if (!(s > 0.0f) || !std::isfinite(s)) return false;
  int e;
  return std::frexp(s, &e) == 0.5f && e > -125 && e < 126;
}

size_t seg(size_t bytes) { return (bytes + 255) & ~(size_t)255; }

SplitOp split_op(int64_t rows, int64_t cols, const float* x, int64_t ldx, float scale, const float* scale_dev,
                 const uint32_t* bits, uint16_t* hi, int64_t ldh, uint16_t* lo, int64_t ldl) {
  SplitOp o{x, rows, cols, ldx, hi, lo, ldh, ldl, scale_dev || bits ? 1.0f : 1.0f / scale, scale_dev,
            bits, 0, 0, 0};
  while (o.lanes_log2 < SPLIT_LANES_LOG2 && ((int64_t)4 << o.lanes_log2) < cols) ++o.lanes_log2;
  o.chunks = ceil_div(cols, (int64_t)4 << o.lanes_log2);
  o.blocks = ceil_div(rows, (int64_t)1 << (SPLIT_LANES_LOG2 - o.lanes_log2)) * o.chunks;
  return o;
}
mdnn_status_t launch_split(const SplitOp& a, const SplitOp& b, float* ab_scale, hipStream_t st) {
  const int64_t blocks = a.blocks + b.blocks;
  if (blocks == 0) return MDNN_SUCCESS;
  // a launch holds fewer than 2^32 threads; the kernel loops past the grid
  const unsigned grid = blocks > ((int64_t)1 << 20) ? 1u << 20 : (unsigned)blocks;
  hipLaunchKernelGGL(split_f16_kernel, dim3(grid), dim3(256), 0, st, a, b, ab_scale);
  return check_launch("split_f16_kernel");
}

// atomic max of |x|'s bit patterns into the operands' words (pass 1 of the
// automatic scale); an operand with a fixed scale has no word
AbsmaxOp absmax_op(int64_t rows, int64_t cols, const float* x, int64_t ldx, uint32_t* bits) {
  return AbsmaxOp{x, rows, cols, ldx, ceil_div(cols, (int64_t)1024), rows > 0 && cols > 0 ? bits : nullptr};
}
mdnn_status_t launch_absmax(const AbsmaxOp& a, const AbsmaxOp& b, hipStream_t st) {
  if (!a.bits && !b.bits) return MDNN_SUCCESS;
  const int64_t na = a.bits ? a.rows * a.chunks : 0, nb = b.bits ? b.rows * b.chunks : 0;
  int64_t blocks = ceil_div(na > nb ? na : nb, 4);
  if (blocks > 256) blocks = 256;
  hipLaunchKernelGGL(absmax_bits_kernel, dim3((unsigned)blocks, b.bits ? 2 : 1), dim3(256), 0, st, a, b);
  return check_launch("absmax_bits_kernel");
}

}  // namespace
}  // namespace mdnn

using namespace mdnn;

extern "C" mdnn_status_t mdnn_split_f16(int64_t rows, int64_t cols, const float* x, int64_t ldx, float scale,
                                        float* scale_out, void* hi, int64_t ldh, void* lo, int64_t ldl,
                                        mdnn_stream_t stream) {
  if (rows < 0 || cols < 0) return fail(MDNN_ERR_SHAPE, "split: negative size");
  const bool automatic = scale == 0.0f;
  if (!automatic && !power_of_two(scale))
    return fail(MDNN_ERR_SHAPE, "split: scale must be a positive power of two, or 0 (chosen on the device)");
  if (automatic && !scale_out) return fail(MDNN_ERR_NULL, "split: scale 0 needs scale_out");
  if (scale_out && !aligned(scale_out, 4)) return fail(MDNN_ERR_MISALIGNED, "split: scale_out is misaligned");
  if ((rows == 0 || cols == 0) && !automatic) return MDNN_SUCCESS;
  if ((rows > 0 && cols > 0) && (!x || !hi || !lo)) return fail(MDNN_ERR_NULL, "split: x, hi and lo are required");
  if (rows > 0 && cols > 0 && (ldx < cols || ldh < cols || ldl < cols))
    return fail(MDNN_ERR_LAYOUT, "split: leading dimension < cols");
  if ((x && !aligned(x, 4)) || (hi && !aligned(hi, 2)) || (lo && !aligned(lo, 2)))
    return fail(MDNN_ERR_MISALIGNED, "split: misaligned base pointer");
  clear_error();
  hipStream_t st = as_stream(stream);
  SplitOp op = split_op(rows, cols, x, ldx, scale, automatic ? scale_out : nullptr, nullptr, (uint16_t*)hi, ldh,
                        (uint16_t*)lo, ldl);
  if (!automatic) return launch_split(op, SplitOp{}, nullptr, st);
  uint32_t* w = (uint32_t*)scale_out;
  MDNN_TRY(fill_zero(w, 4, st));
  MDNN_TRY(launch_absmax(absmax_op(rows, cols, x, ldx, w), AbsmaxOp{}, st));
  hipLaunchKernelGGL(scale_one_kernel, dim3(1), dim3(64), 0, st, w);
  MDNN_TRY(check_launch("scale_one_kernel"));
  return launch_split(op, SplitOp{}, nullptr, st);
}

// Workspace: [A1 | A2] (2 M K fp16), [B2 ; B1] (2 K N fp16), the fp32
// correction product (M N), and three scale words (the bit maxima of A and
// B, and s_a s_b), each 256-byte aligned.
extern "C" size_t mdnn_gemm_split3_workspace(int64_t M, int64_t N, int64_t K) {
  if (M < 0 || N < 0 || K < 0) return 0;
  return seg((size_t)2 * M * K * 2) + seg((size_t)2 * K * N * 2) + seg((size_t)M * N * 4) + 256;
}

extern "C" mdnn_status_t mdnn_gemm_split3(mdnn_layout_t layout, int64_t M, int64_t N, int64_t K, float alpha,
                                          const float* A, int64_t lda, float a_scale, const float* B, int64_t ldb,
                                          float b_scale, float beta, const float* C, int64_t ldc, float* D,
                                          int64_t ldd, void* workspace, size_t ws_bytes, mdnn_stream_t stream) {
  if (layout != MDNN_NN && layout != MDNN_NT && layout != MDNN_TN)
    return fail(MDNN_ERR_LAYOUT, "gemm_split3: unknown layout %d", (int)layout);
  if (M < 0 || N < 0 || K < 0) return fail(MDNN_ERR_SHAPE, "gemm_split3: negative size");
  if ((a_scale != 0.0f && !power_of_two(a_scale)) || (b_scale != 0.0f && !power_of_two(b_scale)))
    return fail(MDNN_ERR_SHAPE, "gemm_split3: scales must be positive powers of two, or 0 (chosen on the device)");
  if (M == 0 || N == 0) return MDNN_SUCCESS;
  if (!D) return fail(MDNN_ERR_NULL, "gemm_split3: D is NULL");
  if (K > 0 && (!A || !B)) return fail(MDNN_ERR_NULL, "gemm_split3: A or B is NULL");
  if (beta != 0.0f && !C) return fail(MDNN_ERR_NULL, "gemm_split3: beta != 0 but C is NULL");
  const int64_t a_w = layout == MDNN_TN ? M : K, b_w = layout == MDNN_NT ? K : N;
  if (K > 0 && (lda < a_w || lda < 1)) return fail(MDNN_ERR_LAYOUT, "gemm_split3: lda < %lld", (long long)a_w);
  if (K > 0 && (ldb < b_w || ldb < 1)) return fail(MDNN_ERR_LAYOUT, "gemm_split3: ldb < %lld", (long long)b_w);
  if (ldd < N) return fail(MDNN_ERR_LAYOUT, "gemm_split3: ldd < N");
  if (beta != 0.0f && ldc < N) return fail(MDNN_ERR_LAYOUT, "gemm_split3: ldc < N");
  if ((A && !aligned(A, 4)) || (B && !aligned(B, 4)) || !aligned(D, 4) || (C && !aligned(C, 4)))
    return fail(MDNN_ERR_MISALIGNED, "gemm_split3: a base pointer is not 4-byte aligned");
  const size_t need = mdnn_gemm_split3_workspace(M, N, K);
  if (!workspace || ws_bytes < need || !aligned(workspace, 256))
    return fail(MDNN_ERR_WORKSPACE, "gemm_split3: needs %zu bytes of 256-byte aligned workspace", need);
  clear_error();
  hipStream_t st = as_stream(stream);
  char* ws = (char*)workspace;
  uint16_t* ah = (uint16_t*)ws;                                  // [A1 | A2]
  uint16_t* bh = (uint16_t*)(ws + seg((size_t)2 * M * K * 2));  // [B2 ; B1]
  float* dlo = (float*)((char*)bh + seg((size_t)2 * K * N * 2));
  // scales chosen on the device (a_scale or b_scale 0): the split kernel
  // derives them from the bit maxima and leaves s_a s_b, which the products'
  // epilogues multiply into alpha
  const bool automatic = a_scale == 0.0f || b_scale == 0.0f;
  uint32_t* words = (uint32_t*)((char*)dlo + seg((size_t)M * N * 4));
  const uint32_t* wa = a_scale == 0.0f ? words : nullptr;
  const uint32_t* wb = b_scale == 0.0f ? words + 1 : nullptr;
  const bool a_t = layout == MDNN_TN, b_t = layout != MDNN_NT;  // stored [K][M], [K][N]
  const int64_t ar = a_t ? K : M, ac = a_t ? M : K, br = b_t ? K : N, bc = b_t ? N : K;
  if (automatic) {
    MDNN_TRY(fill_zero(words, 16, st));
    MDNN_TRY(launch_absmax(absmax_op(ar, ac, A, lda, (uint32_t*)wa), absmax_op(br, bc, B, ldb, (uint32_t*)wb), st));
  }
  // concatenated operands: K-contiguous ones side by side along the row,
  // MN-contiguous ones stacked by rows
  const int64_t ld_ah = a_t ? M : 2 * K, ld_bh = b_t ? N : 2 * K;
  uint16_t* a2 = ah + (a_t ? K * M : K);
  uint16_t* b1 = bh + (b_t ? K * N : K);
  const uint16_t* a1 = ah;
  float* ab_dev = automatic ? (float*)(words + 2) : nullptr;
  MDNN_TRY(launch_split(split_op(ar, ac, A, lda, a_scale, nullptr, wa, ah, ld_ah, a2, ld_ah),
                        split_op(br, bc, B, ldb, b_scale, nullptr, wb, b1, ld_bh, bh, ld_bh),
                        ab_dev, st));
  const float ab = automatic ? alpha : alpha * a_scale * b_scale;
  // corrections: alpha a b 2^-11 (A1 B2 + A2 B1) + beta C
  MDNN_TRY(gemm_mixed_ws(layout, M, N, 2 * K, ab / SHIFT_UP, ah, ld_ah, bh, ld_bh, MDNN_F16, beta, C, ldc, dlo, N,
                         MDNN_F32, nullptr, MDNN_ACT_NONE, nullptr, 0, nullptr, 0, stream, nullptr, ab_dev));
  // leading product plus the corrections
  return gemm_mixed_ws(layout, M, N, K, ab, a1, ld_ah, b1, ld_bh, MDNN_F16, 1.0f, dlo, N, D, ldd, MDNN_F32, nullptr,
                       MDNN_ACT_NONE, nullptr, 0, nullptr, 0, stream, nullptr, ab_dev);
}
