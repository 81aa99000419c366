// Forward convolutions with a short reduction (a network's first layers:
// 1 to 4 channels, 3x3 to 7x7) on the matrix cores without LDS: a wave keeps
// the filter's fragments of up to 64 output channels in registers and walks
// groups of 16 output pixels, each lane loading its own fragment chunks
// straight from the image (gemm_reg.h's runs: one filter row's s * c elements
// are one run of memory; chunks at any element address, image edges cleared
// in registers), the next group's chunks in flight behind the current
// group's MFMAs and stores.
#include "conv_gather.h"

#include "gemm_reg.h"

namespace mdnn {
namespace {

using reg::El;
using reg::end_shift;
using reg::keep_bits;
using reg::keep_chunk;
using reg::load_chunk;
using reg::run_keep;
using reg::shift_chunk;

struct GatherArgs {
  const void *x, *w;
  int32_t x_total, w_total;
  int32_t M, N;            // output pixels, channels
  int32_t rows, len, lp;   // filter rows, elements per run, padded
  int32_t hs, wsC, C;      // image rows, elements per image row, channels
  int32_t ho, wo, pad;
  uint32_t magic_w, magic_h;
};

template <int KS>
struct Group {
  uint4 v[KS];
  uint32_t keep[KS];
  int32_t base;  // of the lane's pixel
  bool shift;
};

// Elements o .. o + E - 1 of a tensor that holds no whole chunk, zeros outside it.
template <class T>
__device__ __forceinline__ uint4 tiny_chunk(const void* p, int o, int total) {
  uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
  for (int e = 0; e < El<T>::E; ++e) {
    const int i = o + e;
    if (i < 0 || i >= total) continue;
    if constexpr (El<T>::ES == 2)
      w[e / 2] |= (uint32_t)((const uint16_t*)p)[i] << (16 * (e & 1));
    else
      w[e] = ((const uint32_t*)p)[i];
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// TINY: the filter (1) or filter and image (2) are read by elements, for tensors
// of less than one chunk (6 -> 1 channels, 1x1, 222 x 31 x 31: 5 us, 91 in the
// general kernel, which would be left).
template <class T, class OutT, int KS, int NF, int TINY = 0>
__global__ void __launch_bounds__(256, 2) conv_gather_kernel(GatherArgs a, Epilogue ep) {
  typedef typename OutT::storage DS;
  constexpr int ES = El<T>::ES, E = El<T>::E;
  constexpr uint32_t ALL = (1u << E) - 1u;
  const int lane = threadIdx.x & 63, l15 = lane & 15, q4 = lane >> 4;
  const char* x = (const char*)a.x;
  const int n0 = (int)blockIdx.y * (16 * NF);

  // this lane's chunk of each step: filter row, position in the run, and the
  // offset of both in the image
  int32_t row[KS], pos[KS], rel[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    const int k = (s * 4 + q4) * E;
    row[s] = k / a.lp;
    pos[s] = k - row[s] * a.lp;
    rel[s] = row[s] * a.wsC + pos[s];
  }
  // filter fragments (channels past N repeat the last one: never stored)
  uint4 wf[KS][NF];
#pragma unroll
  for (int s = 0; s < KS; ++s)
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      const int n = n0 + j * 16 + l15 < a.N ? n0 + j * 16 + l15 : a.N - 1;
      const int o = (n * a.rows + row[s]) * a.len + pos[s], from = reg::clampi(o, 0, a.w_total - E);
      const uint32_t keep = row[s] < a.rows ? keep_bits(0, reg::clampi(a.len - pos[s], 0, E)) : 0u;
      uint4 c;
      if (TINY == 1 || (TINY == 2 && a.w_total < E)) {
        c = tiny_chunk<T>(a.w, o, a.w_total);
      } else {
        c = load_chunk<ES>((const char*)a.w + (uint32_t)from * (uint32_t)ES);
        if (__any(o != from)) c = shift_chunk<ES>(c, end_shift<E>(o, a.w_total));
      }
      wf[s][j] = keep_chunk<ES>(c, keep, 0);
    }
  float bias[NF][4];
#pragma unroll
  for (int j = 0; j < NF; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = n0 + j * 16 + 4 * q4 + e;
      bias[j][e] = ep.bias ? ep.bias[n < a.N ? n : a.N - 1] : 0.0f;
    }
#pragma unroll
  for (int s = 0; s < KS; ++s)
    if (row[s] >= a.rows) row[s] = 1 << 30;  // past the filter: outside every image

  const int groups = (a.M + 15) / 16, stride = (int)gridDim.x * 4;
  auto load = [&](int g, Group<KS>& G) {
    const int m = g * 16 + l15 < a.M ? g * 16 + l15 : a.M - 1;
    const int q1 = (int)lds::fast_div((uint32_t)m, a.magic_w), j = m - q1 * a.wo;
    const int img = (int)lds::fast_div((uint32_t)q1, a.magic_h), i = q1 - img * a.ho;
    const int y0 = i - a.pad, x0 = (j - a.pad) * a.C;
    G.base = (img * a.hs + y0) * a.wsC + x0;
    bool any = false;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int o = G.base + rel[s], from = reg::clampi(o, 0, a.x_total - E);
      if constexpr (TINY == 2)
        G.v[s] = tiny_chunk<T>(a.x, o, a.x_total);
      else
        G.v[s] = load_chunk<ES>(x + (uint32_t)from * (uint32_t)ES);
      G.keep[s] = run_keep<E>((uint32_t)(y0 + row[s]) < (uint32_t)a.hs, x0 + pos[s], a.wsC, a.len - pos[s]);
      any |= TINY < 2 && o != from && G.keep[s] != 0;
    }
    G.shift = __any(any);
  };
  auto finish = [&](auto full, int g, Group<KS>& G) {
    constexpr bool FULL = decltype(full)::value;
    if (G.shift) {
#pragma unroll
      for (int s = 0; s < KS; ++s) G.v[s] = shift_chunk<ES>(G.v[s], end_shift<E>(G.base + rel[s], a.x_total));
    }
    float4_t acc[1][1][NF];
#pragma unroll
    for (int j = 0; j < NF; ++j) acc[0][0][j] = (float4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      uint4 af[1] = {__any(G.keep[s] != ALL) ? keep_chunk<ES>(G.v[s], G.keep[s], 0) : G.v[s]};
      reg::mfma_step<T, 1>(af, wf[s], acc);
    }
    const int m = g * 16 + l15;
    if (!FULL && m >= a.M) return;
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      const int n = n0 + j * 16 + 4 * q4;
      DS h[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float v = acc[0][0][j][e] + bias[j][e];
        if (ep.act == MDNN_ACT_RELU) v = relu_f(v);
        h[e] = from_f<OutT>(v);
      }
      DS* d = (DS*)ep.D + (int64_t)m * ep.ldd + n;
      if (FULL || n + 4 <= a.N) {
        Quad<OutT> q;
        if constexpr (sizeof(DS) == 2) {
          q.q[0] = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
          q.q[1] = (uint32_t)h[2] | ((uint32_t)h[3] << 16);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) q.q[e] = __builtin_bit_cast(uint32_t, h[e]);
        }
        q.store(d);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n + e < a.N) d[e] = h[e];
      }
    }
  };
  // two groups in turn, the next one's loads ahead of this one's products.
  // Whole groups of whole channel blocks store without a branch: stores count
  // with the loads, and behind a branch the wait for the next group's loads
  // would wait for them too.
  auto walk = [&](auto full, int g, int end) {
    Group<KS> A, B;
    if (g < end) load(g, A);
    while (g < end) {
      if (g + stride < end) load(g + stride, B);
      finish(full, g, A);
      g += stride;
      if (g >= end) break;
      if (g + stride < end) load(g + stride, A);
      finish(full, g, B);
      g += stride;
    }
    return g;
  };
  int g = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (n0 + 16 * NF <= a.N) g = walk(std::true_type{}, g, a.M / 16);
  walk(std::false_type{}, g, groups);
}

template <class T, class OutT, int KS>
void launch_nf(const GatherArgs& a, const Epilogue& ep, hipStream_t st) {
  const int groups = (a.M + 15) / 16;
  // as many channels per wave as its registers hold (each chunk is gathered
  // once per 16 nf channels), fewer while that leaves CUs idle; at most the
  // workgroups that fit at once (two per CU with 96 registers of filter)
  int nf = a.N <= 16 ? 1 : a.N <= 32 ? 2 : 4;
  while (nf > 1 && ceil_div(groups, 4) * ceil_div(a.N, 16 * nf) < 256) nf /= 2;
  const int64_t cols = ceil_div(a.N, 16 * nf), most = KS * nf > 16 ? 512 : 1024;
  int64_t bx = ceil_div(groups, 4);
  if (bx * cols > most) bx = ceil_div(most, cols);
  const dim3 grid((unsigned)bx, (unsigned)ceil_div(a.N, 16 * nf));
  if (nf == 1) hipLaunchKernelGGL((conv_gather_kernel<T, OutT, KS, 1>), grid, dim3(256), 0, st, a, ep);
  else if (nf == 2) hipLaunchKernelGGL((conv_gather_kernel<T, OutT, KS, 2>), grid, dim3(256), 0, st, a, ep);
  else hipLaunchKernelGGL((conv_gather_kernel<T, OutT, KS, 4>), grid, dim3(256), 0, st, a, ep);
}

template <class T, class OutT>
void launch(const GatherArgs& a, int ks, const Epilogue& ep, hipStream_t st) {
  // (a filter below a chunk has at most 7 rows and 56 padded elements)
  if (a.x_total < El<T>::E || a.w_total < El<T>::E) {
    const int64_t by = ceil_div((int64_t)a.N, 16), most = ceil_div((int64_t)1024, by), all = ceil_div((int64_t)a.M, 64);
    const dim3 grid((unsigned)(all < most ? all : most), (unsigned)by);
    if (a.x_total >= El<T>::E && ks <= 1)
      hipLaunchKernelGGL((conv_gather_kernel<T, OutT, 1, 1, 1>), grid, dim3(256), 0, st, a, ep);
    else if (a.x_total >= El<T>::E)
      hipLaunchKernelGGL((conv_gather_kernel<T, OutT, 2, 1, 1>), grid, dim3(256), 0, st, a, ep);
    else if (ks <= 1) hipLaunchKernelGGL((conv_gather_kernel<T, OutT, 1, 1, 2>), grid, dim3(256), 0, st, a, ep);
    else hipLaunchKernelGGL((conv_gather_kernel<T, OutT, 6, 1, 2>), grid, dim3(256), 0, st, a, ep);
  } else if (ks <= 1) launch_nf<T, OutT, 1>(a, ep, st);
  else if (ks == 2) launch_nf<T, OutT, 2>(a, ep, st);
  else if (ks == 3) launch_nf<T, OutT, 3>(a, ep, st);
  else if (ks == 4) launch_nf<T, OutT, 4>(a, ep, st);
  else launch_nf<T, OutT, 6>(a, ep, st);
}

uint32_t magic_of(int64_t d) { return d == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); }

}  // namespace

mdnn_status_t conv_gather_fwd(const ConvGeom& g, const void* x, const void* w, const Epilogue& ep, mdnn_dtype_t io,
                              mdnn_dtype_t out, hipStream_t st, bool* done) {
  *done = false;
  const int64_t E = 16 / (int64_t)dtype_size(io), len = (int64_t)g.s * g.c, lp = ceil_div(len, E) * E, K = g.r * lp;
  const int64_t M = (int64_t)g.n * g.ho * g.wo, xt = (int64_t)g.n * g.h * g.w * g.c, wt = (int64_t)g.k * g.r * len;
  const int64_t LIM = (int64_t)1 << 30;
  // Against the kernels behind this one (register-staged, direct-to-LDS), 4 to
  // 1024 output channels, 6 to 200 thousand pixels: 0.3-1.0 of their time up to
  // 64 output channels and for channel counts that are multiples of 4 (3 -> 64,
  // 3x3, 64 x 56 x 56 fp16 10 against 16 us); up to 1.2 for 64 channels, 1x1, on 128
  // to 512 (32 x 28 x 28 fp16 -> 256: 11.5 and 9.7) and up to 1.5 for 16-bit rows
  // on odd elements with a reduction above 128 (3 -> 64, 7x7, 16 x 64 x 64: 20 and
  // 13.5, but 64 x 64 x 64 34 and 48): a wave's filter loads wait for each other,
  // which few pixel groups per wave do not make up for.
  if (K > 24 * E || (K > 64 && E == 8 && g.c % 8 == 0)) return MDNN_SUCCESS;
  if (xt >= LIM || wt >= LIM || M + 32 >= LIM || ceil_div(g.k, 16) > 65535 ||
      (M + 32) * (g.wo - 1) >= ((int64_t)1 << 32) || ((M + 32) / g.wo + 1) * (g.ho - 1) >= ((int64_t)1 << 32))
    return MDNN_SUCCESS;
  const GatherArgs a{x,   w,     (int32_t)xt, (int32_t)wt,  (int32_t)M, g.k,  g.r,  (int32_t)len,  (int32_t)lp,
                     g.h, g.w * g.c, g.c,     g.ho, g.wo, g.pad, magic_of(g.wo), magic_of(g.ho)};
  const int ks = (int)ceil_div(K, 4 * E);
  if (io == MDNN_F32) launch<F32, F32>(a, ks, ep, st);
  else if (io == MDNN_F16 && out == MDNN_F32) launch<F16, F32>(a, ks, ep, st);
  else if (io == MDNN_F16) launch<F16, F16>(a, ks, ep, st);
  else if (out == MDNN_F32) launch<BF16, F32>(a, ks, ep, st);
  else launch<BF16, BF16>(a, ks, ep, st);
  *done = true;
  return check_launch("conv_gather_kernel");
}

}  // namespace mdnn
