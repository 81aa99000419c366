// Host build of the register-staged loaders' address arithmetic: every chunk
// that a workgroup's lanes would fetch from an operand is computed by the
// loader's own code and compared with the operand's extent, without a GPU.
#include "../paper_2011_11188_amd/csrc/gemm_reg.h"

using namespace mdnn;

namespace {

// The K-contiguous loader over its last tile and last K step: the number of
// chunks outside the operand's (MN - 1) * ld + K elements.
template <class T, int W, int L, int WAVES>
int64_t mat_last_outside(int64_t MN, int64_t ld, int64_t K) {
  typedef reg::MatLoader<T, true, W, L> Loader;
  const reg::MatArgs a{nullptr, ld, MN, K};
  const int64_t total = (MN - 1) * ld + K, kz = (K - 1) / Loader::BK * Loader::BK;
  int64_t n = 0;
  for (int wave = 0; wave < WAVES; ++wave)
    for (int lane = 0; lane < 64; ++lane) {
      Loader ld_;
      ld_.init(a, (MN - 1) / W * W, kz, K, wave, lane);
      for (int i = 0; i < L; ++i) {
        const int64_t at = kz + (int64_t)(ld_.off[i] / Loader::ES) - ld_.last_back(i);
        n += at < 0 || at + Loader::E > total;
      }
    }
  return n;
}

}  // namespace

extern "C" int64_t host_mat_last_outside(int dtype, int64_t MN, int64_t ld, int64_t K) {
  typedef reg::TileR64 S;
  typedef reg::TileR128 B;
  if (dtype == MDNN_F32)
    return mat_last_outside<F32, S::BM, S::LA, S::NW>(MN, ld, K) + mat_last_outside<F32, B::BM, B::LA, B::NW>(MN, ld, K);
  return mat_last_outside<F16, S::BM, S::LA, S::NW>(MN, ld, K) + mat_last_outside<F16, B::BM, B::LA, B::NW>(MN, ld, K);
}

namespace {

// Chunk shifts of a whole or longer chunk (undefined shifts) over all K steps
// and tiles of a convolution's operands (fp16 or fp32, 64-wide tiles).
template <class Loader, int L>
int64_t run_bad_shifts(const reg::RunArgs& a, int64_t rows, int64_t K) {
  int64_t n = 0;
  for (int64_t mn0 = 0; mn0 < rows; mn0 += 64)
    for (int wave = 0; wave < 4; ++wave)
      for (int lane = 0; lane < 64; ++lane) {
        Loader ld;
        ld.init(a, mn0, 0, K, wave, lane);
        for (int t = 0; t < (int)ceil_div(K, Loader::BK); ++t)
          for (int i = 0; i < L; ++i) {
            const int d = ld.shift(t, i);
            n += d <= -Loader::E || d >= Loader::E;
          }
      }
  return n;
}

uint32_t magic(int64_t d) { return d == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); }

template <class T>
int64_t conv_bad_shifts(int n, int h, int w, int c, int k, int r, int pad) {
  constexpr int L = reg::TileR64::LA;
  const int ho = h + 2 * pad - r + 1, wo = w + 2 * pad - r + 1, E = reg::El<T>::E;
  const int len = r * c, lp = (int)ceil_div(len, E) * E, lent = r * k, lpt = (int)ceil_div(lent, E) * E;
  const int64_t px = (int64_t)n * ho * wo;
  const reg::RunArgs x{nullptr, n * h * w * c, r, len, lp, magic(lp), h, w * c, c, ho, wo, pad, pad, 0, px};
  const reg::RunArgs f{nullptr, k * r * len, r, len, lp, magic(lp), 0, 0, 0, 0, 0, 0, 0, 0, k};
  const reg::RunArgs ft{nullptr, k * r * len, r, lent, lpt, magic(lpt), k, r, c, 0, 0, 0, 0, magic(k), 0};
  return run_bad_shifts<reg::RunRowsLoader<T, 64, L>, L>(x, px, (int64_t)r * lp) +
         run_bad_shifts<reg::RunFilterLoader<T, 64, L>, L>(f, k, (int64_t)r * lp) +
         run_bad_shifts<reg::RunFilterTLoader<T, 64, L>, L>(ft, c, (int64_t)r * lpt);
}

}  // namespace

extern "C" int64_t host_conv_bad_shifts(int dtype, int n, int h, int w, int c, int k, int r, int pad) {
  return dtype == MDNN_F32 ? conv_bad_shifts<F32>(n, h, w, c, k, r, pad) : conv_bad_shifts<F16>(n, h, w, c, k, r, pad);
}
