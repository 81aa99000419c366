// Plain-matrix products on the register-staged mainloop (gemm_reg.h).
#include "gemm_reg.h"

#include "internal.h"

namespace mdnn {

namespace {

template <class T, class OutT, class TL, int NR, bool A_KC, bool B_KC>
void launch(const reg::MatArgs& a, const reg::MatArgs& b, int64_t M, int64_t N, int64_t K, const Epilogue& ep,
            int splits, hipStream_t st) {
  const dim3 grid((unsigned)(ceil_div(M, TL::BM) * ceil_div(N, TL::BN)), (unsigned)splits);
  hipLaunchKernelGGL((reg::gemm_reg_kernel<T, OutT, TL, NR, reg::MatLoader<T, A_KC, TL::BM, TL::LA>,
                                           reg::MatLoader<T, B_KC, TL::BN, TL::LB>>),
                     grid, dim3(TL::NT), 0, st, a, b, M, N, K, ep);
}

// 128 x 128 tiles from one per CU on, else 64 x 64 (four times the
// workgroups, four register sets: their steps are shorter than a load).
// Products of at most two 16-bit K steps are all first load and stores: as many
// 64 x 64 workgroups per CU as registers allow (bf16 TN 2176 x 1024 x 38 8.3 ->
// 6.5 us, 320 x 6784 x 70 9.4 -> 6.8; under larger outputs the 128 x 128 tiles
// are up to a fifth quicker).
// fp32 ones of two to four whole steps take 64 x 64 tiles also where the 128 x 128
// ones would be just over one per CU (NT 663 x 5440 x 128 26.3 -> 17.2 us, NN 939
// x 4160 x 88 22.5 -> 15.7; from 385 tiles on, and below K of 64, the large ones
// are level or ahead).
template <class T, class OutT, bool A_KC, bool B_KC>
void run(const reg::MatArgs& a, const reg::MatArgs& b, int64_t M, int64_t N, int64_t K, const Epilogue& ep,
         int splits, hipStream_t st) {
  constexpr bool H = reg::El<T>::ES == 2;
  const int64_t tiles = ceil_div(M, 128) * ceil_div(N, 128) * splits;
  const bool shallow = K <= 128 && splits == 1;
  if (M > 64 && N > 64 && tiles >= (!H && shallow && K >= 64 ? 385 : 256)) {
    launch<T, OutT, reg::TileR128, 2, A_KC, B_KC>(a, b, M, N, K, ep, splits, st);
    return;
  }
  if constexpr (H) {
    if (shallow && M * N >= (1 << 18)) {
      launch<T, OutT, reg::TileR64Shallow, 2, A_KC, B_KC>(a, b, M, N, K, ep, splits, st);
      return;
    }
  }
  launch<T, OutT, reg::TileR64, 4, A_KC, B_KC>(a, b, M, N, K, ep, splits, st);
}

template <class T, class OutT>
void run_layout(mdnn_layout_t layout, const reg::MatArgs& a, const reg::MatArgs& b, int64_t M, int64_t N, int64_t K,
                const Epilogue& ep, int splits, hipStream_t st) {
  if (layout == MDNN_NN) run<T, OutT, true, false>(a, b, M, N, K, ep, splits, st);
  else if (layout == MDNN_NT) run<T, OutT, true, true>(a, b, M, N, K, ep, splits, st);
  else run<T, OutT, false, false>(a, b, M, N, K, ep, splits, st);
}

// one operand: chunks of 16 bytes along its contiguous dimension lie inside
// it, byte offsets (within the operand, or within one K step) in 32 bits.  A
// K step's chunks reach bk elements from a row's start also where K is
// shorter, and their offsets are formed before they are moved back inside.
bool operand_ok(int64_t es, bool kc, int64_t MN, int64_t ld, int64_t K) {
  const int64_t e = 16 / es, bk = 128 / es;
  if (kc) return K >= e && (MN - 1) * ld + (K > bk ? K : bk) < ((int64_t)1 << 32) / es;
  return MN >= e && bk * ld + MN < ((int64_t)1 << 32) / es;
}

}  // namespace

bool gemm_reg_ok(mdnn_dtype_t ab, mdnn_layout_t layout, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb,
                 int splits) {
  const int64_t es = (int64_t)dtype_size(ab);
  return M > 0 && N > 0 && K > 0 && operand_ok(es, layout != MDNN_TN, M, lda, K) &&
         operand_ok(es, layout == MDNN_NT, N, ldb, K) && ceil_div(M, 64) * ceil_div(N, 64) <= 0x7fffffffLL &&
         K <= 0x7fffffffLL && splits <= 65535;
}

mdnn_status_t gemm_reg(mdnn_dtype_t ab, mdnn_dtype_t d, mdnn_layout_t layout, int64_t M, int64_t N, int64_t K,
                       const void* A, int64_t lda, const void* B, int64_t ldb, const Epilogue& ep, int splits,
                       hipStream_t st) {
  const reg::MatArgs a{A, lda, M, K}, b{B, ldb, N, K};
  if (ab == MDNN_F32) run_layout<F32, F32>(layout, a, b, M, N, K, ep, splits, st);
  else if (ab == MDNN_F16 && d == MDNN_F32) run_layout<F16, F32>(layout, a, b, M, N, K, ep, splits, st);
  else if (ab == MDNN_F16) run_layout<F16, F16>(layout, a, b, M, N, K, ep, splits, st);
  else if (d == MDNN_F32) run_layout<BF16, F32>(layout, a, b, M, N, K, ep, splits, st);
  else run_layout<BF16, BF16>(layout, a, b, M, N, K, ep, splits, st);
  return check_launch("gemm_reg_kernel");
}

}  // namespace mdnn
