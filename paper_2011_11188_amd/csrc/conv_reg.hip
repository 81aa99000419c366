// Convolutions on the register-staged mainloop (gemm_reg.h): any channel
// count, fp32 or 16-bit data.  The reduction of each pass is walked as runs
// of memory (see the loaders), padded to whole 16-byte chunks: a 3-channel
// 7x7 layer reduces over 7 runs of 24 (of 21) elements.
#include "conv_reg.h"

#include "conv_pipe.h"
#include "gemm_reg.h"

namespace mdnn {

namespace {

constexpr int64_t LIM = (int64_t)1 << 30;  // elements of a tensor, rows and columns of a product
constexpr size_t FILTER_WS_MAX = 64ull << 20;

uint32_t magic_of(int64_t d) { return d == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); }
bool div_ok(int64_t x, int64_t d) { return x < LIM && x * (d - 1) < ((int64_t)1 << 32); }
int64_t round_up(int64_t x, int64_t e) { return ceil_div(x, e) * e; }

template <class T, class OutT, class TL, int NR, template <class, int, int> class LA, template <class, int, int> class LB>
void launch(const reg::RunArgs& a, const reg::RunArgs& b, int64_t M, int64_t N, int64_t K, const Epilogue& ep,
            hipStream_t st) {
  hipLaunchKernelGGL((reg::gemm_reg_kernel<T, OutT, TL, NR, LA<T, TL::BM, TL::LA>, LB<T, TL::BN, TL::LB>>),
                     dim3((unsigned)(ceil_div(M, TL::BM) * ceil_div(N, TL::BN))), dim3(TL::NT), 0, st, a, b, M, N, K,
                     ep);
}

// Tiles: 128 x 128 when they give two workgroups per CU (one for 16-bit
// data, whose steps are four times shorter), 128 x 64 for narrow outputs,
// else 64 x 64.
template <class T, class OutT, template <class, int, int> class LA, template <class, int, int> class LB>
void run(const reg::RunArgs& a, const reg::RunArgs& b, int64_t M, int64_t N, int64_t K, const Epilogue& ep,
         hipStream_t st) {
  const int64_t full = reg::El<T>::ES == 4 ? 512 : 256;
  if (N <= 64 && ceil_div(M, 128) >= 512)
    launch<T, OutT, reg::TileR128x64, 2, LA, LB>(a, b, M, N, K, ep, st);
  else if (N > 64 && ceil_div(M, 128) * ceil_div(N, 128) >= full)
    launch<T, OutT, reg::TileR128, 2, LA, LB>(a, b, M, N, K, ep, st);
  else
    launch<T, OutT, reg::TileR64, 4, LA, LB>(a, b, M, N, K, ep, st);
}

template <template <class, int, int> class LA, template <class, int, int> class LB>
mdnn_status_t run_typed(const reg::RunArgs& a, const reg::RunArgs& b, int64_t M, int64_t N, int64_t K,
                        const Epilogue& ep, mdnn_dtype_t io, mdnn_dtype_t out, hipStream_t st) {
  if (io == MDNN_F32) run<F32, F32, LA, LB>(a, b, M, N, K, ep, st);
  else if (io == MDNN_F16 && out == MDNN_F32) run<F16, F32, LA, LB>(a, b, M, N, K, ep, st);
  else if (io == MDNN_F16) run<F16, F16, LA, LB>(a, b, M, N, K, ep, st);
  else if (out == MDNN_F32) run<BF16, F32, LA, LB>(a, b, M, N, K, ep, st);
  else run<BF16, BF16, LA, LB>(a, b, M, N, K, ep, st);
  return check_launch("gemm_reg_kernel");
}

struct Sizes {
  int64_t E, x, y, w;  // elements per chunk, of the input, of the output, of the filter
  explicit Sizes(const ConvGeom& g, mdnn_dtype_t io)
      : E(16 / (int64_t)dtype_size(io)), x((int64_t)g.n * g.h * g.w * g.c), y((int64_t)g.n * g.ho * g.wo * g.k),
        w((int64_t)g.k * g.r * g.s * g.c) {}
  bool ok() const { return x >= E && x < LIM && y >= E && y < LIM && w >= E && w < LIM; }
};

}  // namespace

mdnn_status_t conv_reg_fwd(const ConvGeom& g, const void* x, const void* w, const Epilogue& ep, mdnn_dtype_t io,
                           mdnn_dtype_t out, hipStream_t st, bool* done) {
  *done = false;
  const Sizes z(g, io);
  const int64_t len = (int64_t)g.s * g.c, lp = round_up(len, z.E), K = g.r * lp, M = (int64_t)g.n * g.ho * g.wo;
  if (!z.ok() || !div_ok(K + 128, lp)) return MDNN_SUCCESS;
  const reg::RunArgs a{x,   (int32_t)z.x, g.r,  (int32_t)len, (int32_t)lp, magic_of(lp), g.h, g.w * g.c, g.c,
                       g.ho, g.wo,        g.pad, g.pad,        0,           M};
  const reg::RunArgs b{w, (int32_t)z.w, g.r, (int32_t)len, (int32_t)lp, magic_of(lp), 0, 0, 0, 0, 0, 0, 0, 0, g.k};
  MDNN_TRY((run_typed<reg::RunRowsLoader, reg::RunFilterLoader>(a, b, M, g.k, K, ep, io, out, st)));
  *done = true;
  return MDNN_SUCCESS;
}

mdnn_status_t conv_reg_bwd_data(const ConvGeom& g, const void* dy, const void* w, const Epilogue& ep,
                                mdnn_dtype_t io, mdnn_dtype_t out, hipStream_t st, bool* done) {
  *done = false;
  const Sizes z(g, io);
  const int64_t len = (int64_t)g.s * g.k, lp = round_up(len, z.E), K = g.r * lp, M = (int64_t)g.n * g.h * g.w;
  if (!z.ok() || !div_ok(K + 128, lp) || !div_ok(lp, g.k)) return MDNN_SUCCESS;
  // fp32 layers of one chunk's reduction and many 16-byte outputs are stores: a
  // K step of 32 before them costs more than the general kernel's of 16 (192 ->
  // 2 channels, 1x1, 14 x 63 x 63: 31.6 us here, 25.0 there; with 5 to 16 within
  // a tenth of each other)
  if (io == MDNN_F32 && (int64_t)g.r * g.s * g.k <= 4 && g.c % 4 == 0 && M * g.c >= (1 << 22)) return MDNN_SUCCESS;
  const reg::RunArgs a{dy,  (int32_t)z.y, g.r,           (int32_t)len,    (int32_t)lp, magic_of(lp), g.ho, g.wo * g.k, g.k,
                       g.h, g.w,          g.r - 1 - g.pad, g.s - 1 - g.pad, 0,           M};
  const reg::RunArgs b{w, (int32_t)z.w, g.r, (int32_t)len, (int32_t)lp,      magic_of(lp), g.k, g.s,
                       g.c, 0,          0,   0,            0,                magic_of(g.k), 0};
  MDNN_TRY((run_typed<reg::RunRowsLoader, reg::RunFilterTLoader>(a, b, M, g.c, K, ep, io, out, st)));
  *done = true;
  return MDNN_SUCCESS;
}

SplitPlan conv_reg_filter_plan(const ConvGeom& g, mdnn_dtype_t io) {
  SplitPlan p{0, 0};
  const Sizes z(g, io);
  const int64_t len = (int64_t)g.s * g.c, lp = round_up(len, z.E), M = g.k, N = g.r * lp,
                K = (int64_t)g.n * g.ho * g.wo, bk = 8 * z.E;
  if (!z.ok() || M < z.E || N >= LIM || K + 128 >= LIM) return p;
  // at most 512 workgroups, which is two per CU at once (one more would run
  // alone after them: 513 took 41 us where 510 take 34), each split at least
  // four steps deep
  const int64_t tiles = ceil_div(M, 64) * ceil_div(N, 64), steps = ceil_div(K, bk);
  if (tiles > 0x7fffffffLL) return p;
  int64_t s = 512 / tiles;
  if (s > steps / 4) s = steps / 4;
  while (s > 1 && (size_t)s * z.w * 4 > FILTER_WS_MAX) --s;
  if (s < 1) s = 1;
  p.k_per_split = ceil_div(steps, s) * bk;
  p.splits = (int)ceil_div(K, p.k_per_split);
  return p;
}

namespace {

template <class T>
void filter_launch(const reg::MatArgs& a, const reg::RunArgs& b, int64_t M, int64_t N, int64_t K, const Epilogue& ep,
                   int splits, hipStream_t st) {
  typedef reg::TileR64 TL;
  const dim3 grid((unsigned)(ceil_div(M, TL::BM) * ceil_div(N, TL::BN)), (unsigned)splits);
  hipLaunchKernelGGL((reg::gemm_reg_kernel<T, F32, TL, 4, reg::MatLoader<T, false, TL::BM, TL::LA>,
                                           reg::RunColsLoader<T, TL::BN, TL::LB>>),
                     grid, dim3(TL::NT), 0, st, a, b, M, N, K, ep);
}

}  // namespace

mdnn_status_t conv_reg_bwd_filter(const ConvGeom& g, const void* x, const void* dy, float* dw, void* ws,
                                  mdnn_dtype_t io, hipStream_t st, bool* done, ReduceBatch* defer) {
  *done = false;
  const SplitPlan p = conv_reg_filter_plan(g, io);
  if (p.splits == 0 || (p.splits > 1 && !ws)) return MDNN_SUCCESS;
  const Sizes z(g, io);
  const int64_t len = (int64_t)g.s * g.c, lp = round_up(len, z.E), M = g.k, N = g.r * lp,
                K = (int64_t)g.n * g.ho * g.wo;
  const reg::MatArgs a{dy, g.k, g.k, K};
  const reg::RunArgs b{x,    (int32_t)z.x, g.r,   (int32_t)len, (int32_t)lp,     magic_of(lp),    g.h, g.w * g.c, g.c,
                       g.ho, g.wo,         g.pad, g.pad,        0,               0};
  Epilogue ep{};
  ep.alpha = 1.0f;
  ep.D = dw;
  ep.ldd = len * g.r;
  ep.k_per_split = K;
  if (p.splits > 1) {
    ep.partial = (float*)ws;
    ep.k_per_split = p.k_per_split;
  }
  if (io == MDNN_F32) filter_launch<F32>(a, b, M, N, K, ep, p.splits, st);
  else if (io == MDNN_F16) filter_launch<F16>(a, b, M, N, K, ep, p.splits, st);
  else filter_launch<BF16>(a, b, M, N, K, ep, p.splits, st);
  MDNN_TRY(check_launch("gemm_reg_kernel"));
  if (p.splits > 1) MDNN_TRY(reduce_splits((const float*)ws, p.splits, M, (int64_t)g.r * len, dw, st, defer));
  *done = true;
  return MDNN_SUCCESS;
}

}  // namespace mdnn
