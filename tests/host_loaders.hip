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
