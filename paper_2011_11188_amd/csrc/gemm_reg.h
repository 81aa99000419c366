// Register-staged GEMM mainloop for gfx950: the products whose operands the
// direct-to-LDS mainloop (gemm_lds.h) cannot fetch -- rows that start on any
// element (odd leading dimensions and sizes, any K), and fp32 operands --
// on the matrix cores (v_mfma_f32_16x16x32_{f16,bf16} and
// v_mfma_f32_16x16x4_f32), fp32 accumulation.
//
// An operand tile is 128 bytes of k per row (64 16-bit or 32 fp32 elements),
// fetched as 16-byte chunks of E consecutive elements along the operand's
// contiguous dimension: global memory -> registers (one unaligned 16-byte
// load per chunk; gfx950 takes any element address) -> LDS (16-byte writes)
// -> fragments.  NR register sets keep the loads of NR - 1 tiles in flight
// behind the MFMAs of the current one; LDS holds two tiles, so a K step has
// one barrier.
//
// Every load stays inside the operand: a chunk that would run past the end
// starts earlier and is shifted into place, and elements outside the valid
// range (k past the end, zero padding of an image) are cleared, both in
// registers before the LDS write and only in waves that hold such a chunk
// (Fix).  Chunks past M or N of an operand whose contiguous dimension
// is M or N are fetched from inside the row: they feed outputs that are
// never stored.
//
// What bounds it: fp32 products the matrix cores (137 TFLOP/s at 4096^3; busy
// 62-64% of the time at 1024 x 2048 x 2048, 114 TFLOP/s, where the launch and
// the first loads show); 16-bit ones the LDS writes and their barrier (4001 x
// 3999 x 4003: 676-694 TFLOP/s, about half of the direct-to-LDS kernel on
// aligned operands).  Reading the second half step's fragments ahead of the
// first half's MFMAs spilled registers and gained nothing.
//
// LDS layouts: as in gemm_lds.h for 16-bit elements and for K-contiguous
// fp32 tiles (128-byte rows, 16-byte chunk c of row r at c ^ ((r >> 1) & 7));
// an MN-contiguous fp32 tile is stored k-row by k-row, its 64-byte block b at
// b ^ ((k >> 2) & 3), so that the four k-rows one fragment read touches lie
// in different banks.  An fp32 fragment is 16 rows x 16 k: lane group g
// holds k = 4g .. 4g + 3, one MFMA per k mod 4 (both operands alike).
#pragma once

#include "gemm_lds.h"

namespace mdnn {
namespace reg {

using lds::LoadPos;

template <class T>
struct El {
  static constexpr int ES = (int)sizeof(typename T::storage);
  static constexpr int E = 16 / ES;    // elements per chunk
  static constexpr int BK = 128 / ES;  // k per step
};

// One chunk at any element address.
typedef uint32_t u32x4_a2 __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
template <int ES>
__device__ __forceinline__ uint4 load_chunk(const char* p) {
  typedef std::conditional_t<ES == 2, u32x4_a2, u32x4_a4> V;
  const V v = *(const __attribute__((address_space(1))) V*)p;
  return make_uint4(v.x, v.y, v.z, v.w);
}

// How loaded chunks become the wanted ones: chunk i keeps the elements whose
// bits are set in byte i of `keep` (all: keep_all), and where some lane of the
// wave has a chunk at the operand's end (`shift`, uniform) element e of it is
// loaded element e + d, d from the loader.
struct Fix {
  uint32_t keep;
  bool shift;
};
// The last step's: also each chunk's d, a byte each (d + 16).
struct LastFix {
  uint32_t keep, shift;
};
__device__ __forceinline__ uint32_t pack_shift(int d, int i) { return (uint32_t)(d + 16) << (8 * i); }
template <int E, int L>
constexpr uint32_t keep_all() {
  uint32_t k = 0;
  for (int i = 0; i < L; ++i) k |= ((1u << E) - 1u) << (8 * i);
  return k;
}
// bits lo .. hi - 1
__device__ __forceinline__ uint32_t keep_bits(int lo, int hi) {
  return lo < hi ? ((1u << hi) - 1u) & ~((1u << lo) - 1u) : 0u;
}
// (|d| below the chunk's elements)
template <int ES>
__device__ __forceinline__ uint4 shift_chunk(uint4 v, int d) {
  constexpr int B = 8 * ES;
  typedef unsigned __int128 u128;
  u128 x = ((u128)(((uint64_t)v.w << 32) | v.z) << 64) | (((uint64_t)v.y << 32) | v.x);
  x = d >= 0 ? x >> (B * (d & 15)) : x << (B * (-d & 15));
  const uint64_t l = (uint64_t)x, h = (uint64_t)(x >> 64);
  return make_uint4((uint32_t)l, (uint32_t)(l >> 32), (uint32_t)h, (uint32_t)(h >> 32));
}
template <int ES>
__device__ __forceinline__ uint4 keep_chunk(uint4 v, uint32_t keep, int i) {
  uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if constexpr (ES == 2) {
      const uint32_t a = (uint32_t)__builtin_amdgcn_sbfe((int)keep, 8 * i + 2 * j, 1),
                     b = (uint32_t)__builtin_amdgcn_sbfe((int)keep, 8 * i + 2 * j + 1, 1);
      w[j] &= __builtin_amdgcn_perm(b, a, 0x05040100u);
    } else {
      w[j] &= (uint32_t)__builtin_amdgcn_sbfe((int)keep, 8 * i + j, 1);
    }
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// What load i of this lane fetches (as lds::load_pos, for either element size).
template <class T, bool KC, int W, int L>
__host__ __device__ __forceinline__ LoadPos load_pos(int wave, int lane, int i) {
  if constexpr (sizeof(typename T::storage) == 2) {
    return lds::load_pos<KC, W, L>(wave, lane, i);
  } else if constexpr (KC) {
    const int r = (wave * L + i) * 8 + (lane >> 3);
    return {r, ((lane & 7) ^ ((r >> 1) & 7)) * 4};
  } else {
    constexpr int LPR = W / 4;     // lanes per k-row
    constexpr int KPB = 64 / LPR;  // k-rows per 1 KB
    const int k = (wave * L + i) * KPB + lane / LPR, pc = lane % LPR;
    return {k, (((pc >> 2) ^ ((k >> 2) & 3)) << 4) + (pc & 3) * 4};
  }
}

// ---------------------------------------------------------------- loaders

struct MatArgs {
  const void* p;
  int64_t ld, MN, K;
};

// Plain matrix, K-contiguous ([MN][ld >= K]) or MN-contiguous ([K][ld >= MN]).
// K >= E, and MN >= E when MN-contiguous; byte offsets within the operand
// (K-contiguous: and one whole step past the start of its last row, where a
// shorter K's last chunks lie before they are moved back) or within one step
// (MN-contiguous) below 2^32.
template <class T, bool KC_, int W, int L>
struct MatLoader {
  static constexpr bool KC = KC_;
  static constexpr bool ANY_STEP = false;  // only the last step's chunks may need fixing
  static constexpr bool RUNS = false;      // the operand's columns are the product's
  static constexpr int ES = El<T>::ES, E = El<T>::E, BK = El<T>::BK;
  typedef MatArgs Args;
  const char* base;
  int64_t step, ld, MN, K, kbeg, kend;
  uint32_t off[L];
  int32_t kpos[L];  // KC: k of the chunk within a step; else its k-row

  __host__ __device__ __forceinline__ void init(const MatArgs& a, int64_t mn0, int64_t kb, int64_t ke, int wave,
                                                int lane) {
    ld = a.ld, MN = a.MN, K = a.K, kbeg = kb, kend = ke;
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const LoadPos q = load_pos<T, KC, W, L>(wave, lane, i);
      if constexpr (KC) {
        int64_t row = mn0 + q.r;
        if (row >= MN) row = MN - 1;
        kpos[i] = q.c;
        off[i] = (uint32_t)((row * ld + q.c) * ES);
      } else {
        int64_t mn = mn0 + q.c;
        if (mn >= MN) mn = MN - E;
        kpos[i] = q.r;
        off[i] = (uint32_t)(((int64_t)q.r * ld + mn) * ES);
      }
    }
    step = (KC ? (int64_t)BK : BK * ld) * ES;
    base = (const char*)a.p + (KC ? kbeg : kbeg * ld) * ES;
  }
  __device__ __forceinline__ void load(int t, uint4 (&v)[L], Fix&) {
    const char* kb = base + (int64_t)t * step;
#pragma unroll
    for (int i = 0; i < L; ++i) v[i] = load_chunk<ES>(kb + off[i]);
  }
  // elements by which chunk i of the last step (from kbeg) is moved back to lie in the operand
  __host__ __device__ __forceinline__ int64_t last_back(int i) const {
    const int64_t over = KC ? kbeg + kpos[i] + E - K : (int64_t)(off[i] / ES) - ((K - 1 - kbeg) * ld + MN - E);
    return over > 0 ? over : 0;
  }
  // the last step (from kbeg): k past kend is cleared, chunks past the
  // operand's end are fetched from inside it
  __device__ __forceinline__ void load_last(uint4 (&v)[L], LastFix& f) {
    f.keep = f.shift = 0;
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const int64_t d = last_back(i), left = kend - (kbeg + kpos[i]);
      v[i] = load_chunk<ES>(base + ((int64_t)off[i] - d * ES));
      const int hi = left <= 0 ? 0 : !KC || left > E ? E : (int)left;
      f.keep |= keep_bits(0, hi) << (8 * i);
      f.shift |= pack_shift(hi ? (int)d : 0, i);
    }
  }
};

// Convolutions (NHWC, stride 1): for one filter row the S * C elements under
// an output pixel are one run of memory in the image row, and one run of the
// filter.  The reduction is walked run by run, each padded to Lp, a multiple
// of the chunk, so that a chunk is a piece of one run for any channel count;
// elements past the run and left or right of the image are cleared.

// x / d for x * (d - 1) < 2^32 (magic: ceil(2^32 / d), 0 for d = 1).
using lds::fast_div;

struct RunArgs {
  const void* p;
  int32_t total;           // elements of p
  int32_t rows, L, Lp;     // filter rows, elements per run, padded
  uint32_t magic_lp;
  int32_t hs, wsC, C;      // image rows, elements per image row, channels
  int32_t ho, wo;          // output grid
  int32_t padr, pads;      // rows above, pixels left
  uint32_t magic_a;        // RunFilterTLoader: of the filters
  int64_t M;               // output pixels (RunRowsLoader), filters (RunFilter)
};

__host__ __device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : v > hi ? hi : v; }

// How far a chunk wanted at element o of `total` is shifted after it was
// fetched from inside: 0 where nothing of it is kept (shift_chunk takes less
// than a chunk).
template <int E>
__host__ __device__ __forceinline__ int end_shift(int o, int total) {
  const int d = o - clampi(o, 0, total - E);
  return d > -E && d < E ? d : 0;
}

// elements kept of an image chunk: x position q of its first element in the
// image row (wsC elements), `left` elements left in the run
template <int E>
__device__ __forceinline__ uint32_t run_keep(bool ok, int q, int wsC, int left) {
  const int lo = q < 0 ? (q < -E ? E : -q) : 0, hi = clampi(wsC - q < left ? wsC - q : left, 0, E);
  return ok ? keep_bits(lo, hi) : 0u;
}

// the last step of a run loader (set up at that step)
template <class Loader, int L>
__device__ __forceinline__ void run_load_last(Loader& ld, uint4 (&v)[L], LastFix& f) {
  Fix g;
  ld.load(0, v, g);
  f.keep = g.keep;
  f.shift = 0;
#pragma unroll
  for (int i = 0; i < L; ++i) f.shift |= pack_shift(ld.shift(0, i), i);
}

// Rows = output pixels, k = (filter row, run): forward x, and dy of backward
// data (whose runs are the filter's mirrored).
template <class T, int W, int L>
struct RunRowsLoader {
  static constexpr bool KC = true, ANY_STEP = true, RUNS = false;
  static constexpr int ES = El<T>::ES, E = El<T>::E, BK = El<T>::BK;
  static_assert(L == 1 || L % 2 == 0, "a lane's k within a step depends on its load's parity");
  static constexpr int P = L >= 2 ? 2 : 1;
  typedef RunArgs Args;
  const char* p;
  int32_t total, rows, len, lp, hs, wsC, k0;
  uint32_t magic;
  int32_t base[L], iy[L], jc[L], kc[P];

  __host__ __device__ __forceinline__ void init(const RunArgs& a, int64_t mn0, int64_t kb, int64_t, int wave, int lane) {
    p = (const char*)a.p, total = a.total, rows = a.rows, len = a.L, lp = a.Lp, hs = a.hs, wsC = a.wsC;
    magic = a.magic_lp, k0 = (int32_t)kb;
    const int32_t hw = a.ho * a.wo;
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const LoadPos q = load_pos<T, true, W, L>(wave, lane, i);
      if (i < P) kc[i] = q.c;
      const int64_t m = mn0 + q.r;
      if (m < a.M) {
        const int32_t mi = (int32_t)m, n = mi / hw, rem = mi - n * hw, i0 = rem / a.wo, j0 = rem - i0 * a.wo;
        iy[i] = i0 - a.padr;
        jc[i] = (j0 - a.pads) * a.C;
        base[i] = (n * a.hs + iy[i]) * a.wsC + jc[i];
      } else {
        iy[i] = -(1 << 20);  // outside the image for every filter row
        jc[i] = 0;
        base[i] = 0;
      }
    }
  }
  __host__ __device__ __forceinline__ void where(int t, int par, int& r, int& e) {
    const uint32_t k = (uint32_t)(k0 + t * BK + kc[par]);
    r = (int)fast_div(k, magic);
    e = (int)k - r * lp;
  }
  __device__ __forceinline__ void load(int t, uint4 (&v)[L], Fix& f) {
    int r[P], e[P], rel[P];
#pragma unroll
    for (int q = 0; q < P; ++q) {
      where(t, q, r[q], e[q]);
      rel[q] = r[q] * wsC + e[q];
      if (r[q] >= rows) r[q] = 1 << 30;  // past the filter: outside every image
    }
    bool any = false;
    f.keep = 0;
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const int par = i % P, o = base[i] + rel[par], from = clampi(o, 0, total - E);
      v[i] = load_chunk<ES>(p + (uint32_t)from * (uint32_t)ES);
      const uint32_t k = run_keep<E>((uint32_t)(iy[i] + r[par]) < (uint32_t)hs, jc[i] + e[par], wsC, len - e[par]);
      f.keep |= k << (8 * i);
      any |= o != from && k != 0;
    }
    f.shift = __any(any);
  }
  __device__ __forceinline__ void load_last(uint4 (&v)[L], LastFix& f) { run_load_last(*this, v, f); }
  __host__ __device__ __forceinline__ int shift(int t, int i) {
    int r, e;
    where(t, i % P, r, e);
    return end_shift<E>(base[i] + r * wsC + e, total);
  }
};

// The filter [filters][rows][L], K-contiguous with padded runs (forward).
template <class T, int W, int L>
struct RunFilterLoader {
  static constexpr bool KC = true, ANY_STEP = true, RUNS = false;
  static constexpr int ES = El<T>::ES, E = El<T>::E, BK = El<T>::BK;
  static constexpr int P = L >= 2 ? 2 : 1;
  typedef RunArgs Args;
  const char* p;
  int32_t total, rows, len, lp, k0;
  uint32_t magic;
  int32_t base[L], kc[P];

  __host__ __device__ __forceinline__ void init(const RunArgs& a, int64_t mn0, int64_t kb, int64_t, int wave, int lane) {
    p = (const char*)a.p, total = a.total, rows = a.rows, len = a.L, lp = a.Lp, magic = a.magic_lp, k0 = (int32_t)kb;
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const LoadPos q = load_pos<T, true, W, L>(wave, lane, i);
      if (i < P) kc[i] = q.c;
      int64_t m = mn0 + q.r;
      if (m >= a.M) m = a.M - 1;
      base[i] = (int32_t)m * a.rows * a.L;
    }
  }
  __host__ __device__ __forceinline__ void where(int t, int par, int& r, int& e) {
    const uint32_t k = (uint32_t)(k0 + t * BK + kc[par]);
    r = (int)fast_div(k, magic);
    e = (int)k - r * lp;
  }
  __device__ __forceinline__ void load(int t, uint4 (&v)[L], Fix& f) {
    int rel[P];
    uint32_t k[P];
#pragma unroll
    for (int q = 0; q < P; ++q) {
      int r, e;
      where(t, q, r, e);
      rel[q] = r * len + e;
      k[q] = r < rows ? keep_bits(0, clampi(len - e, 0, E)) : 0u;
    }
    bool any = false;
    f.keep = 0;
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const int o = base[i] + rel[i % P], from = clampi(o, 0, total - E);
      v[i] = load_chunk<ES>(p + (uint32_t)from * (uint32_t)ES);
      f.keep |= k[i % P] << (8 * i);
      any |= o != from && k[i % P] != 0;
    }
    f.shift = __any(any);
  }
  __device__ __forceinline__ void load_last(uint4 (&v)[L], LastFix& f) { run_load_last(*this, v, f); }
  __host__ __device__ __forceinline__ int shift(int t, int i) {
    int r, e;
    where(t, i % P, r, e);
    return end_shift<E>(base[i] + r * len + e, total);
  }
};

// The filter [filters][rows][S][C] of backward data as the MN-contiguous
// operand: k = (mirrored row, run of (mirrored tap, filter)), columns C.
// L here is S * filters.
template <class T, int W, int L>
struct RunFilterTLoader {
  static constexpr bool KC = false, ANY_STEP = true, RUNS = false;
  static constexpr int ES = El<T>::ES, E = El<T>::E, BK = El<T>::BK;
  typedef RunArgs Args;  // C: columns; hs: filters; wsC: taps per row (S); magic_a: of the filters
  const char* p;
  int32_t total, rows, len, lp, nf, S, C, k0;
  uint32_t magic, magic_f;
  int32_t col[L], krow[L];

  __host__ __device__ __forceinline__ void init(const RunArgs& a, int64_t mn0, int64_t kb, int64_t, int wave, int lane) {
    p = (const char*)a.p, total = a.total, rows = a.rows, len = a.L, lp = a.Lp, nf = a.hs, S = a.wsC, C = a.C;
    magic = a.magic_lp, magic_f = a.magic_a, k0 = (int32_t)kb;
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const LoadPos q = load_pos<T, false, W, L>(wave, lane, i);
      const int64_t mn = mn0 + q.c;
      col[i] = mn < a.C ? (int32_t)mn : 0;
      krow[i] = q.r;
    }
  }
  __host__ __device__ __forceinline__ bool where(int t, int i, int& o) {
    const uint32_t k = (uint32_t)(k0 + t * BK + krow[i]);
    const int r = (int)fast_div(k, magic), e = (int)k - r * lp;
    const int s = (int)fast_div((uint32_t)e, magic_f), f = e - s * nf;
    o = ((f * rows + rows - 1 - r) * S + S - 1 - s) * C + col[i];
    return r < rows && e < len;
  }
  __device__ __forceinline__ void load(int t, uint4 (&v)[L], Fix& f) {
    bool any = false;
    f.keep = 0;
#pragma unroll
    for (int i = 0; i < L; ++i) {
      int o;
      const bool ok = where(t, i, o);
      const int from = clampi(o, 0, total - E);
      v[i] = load_chunk<ES>(p + (uint32_t)from * (uint32_t)ES);
      f.keep |= (ok ? (1u << E) - 1u : 0u) << (8 * i);
      any |= ok && o != from;
    }
    f.shift = __any(any);
  }
  __device__ __forceinline__ void load_last(uint4 (&v)[L], LastFix& f) { run_load_last(*this, v, f); }
  __host__ __device__ __forceinline__ int shift(int t, int i) {
    int o;
    where(t, i, o);
    return end_shift<E>(o, total);
  }
};

// Shifted image columns of the filter gradient: k = output pixel, columns =
// (filter row, padded run).  Steps are loaded in order: each lane's pixel
// (image, row, column) moves on by one step's pixels with carries, where two
// divisions per chunk had bound the kernel (3 channels, 7x7).
template <class T, int W, int L>
struct RunColsLoader {
  static constexpr bool KC = false, ANY_STEP = true, RUNS = true;
  static constexpr int ES = El<T>::ES, E = El<T>::E, BK = El<T>::BK;
  typedef RunArgs Args;
  const char* p;
  int32_t total, hs, wsC, ho, wo;
  // per step: rows and the offset they and the columns move on by; carries
  int32_t dj, di, doff, dqs, woC, row_gap, img_gap;
  int32_t n0, lp, k0, padr, pads, C;  // for shift()
  // next step's pixels left, column, row (less the padding), x position and
  // offset of each chunk; elements left in its run
  int32_t pleft[L], j[L], i_[L], y0[L], q[L], o[L], left[L];

  __device__ __forceinline__ void init(const RunArgs& a, int64_t mn0, int64_t kb, int64_t ke, int wave, int lane) {
    p = (const char*)a.p, total = a.total, hs = a.hs, wsC = a.wsC, ho = a.ho, wo = a.wo;
    n0 = (int32_t)mn0, lp = a.Lp, k0 = (int32_t)kb, padr = a.padr, pads = a.pads, C = a.C;
    const int32_t rows = BK / wo, dn = rows / ho;
    dj = BK - rows * wo;
    di = rows - dn * ho;
    dqs = dj * a.C;
    doff = (dn * hs + di) * wsC + dqs;
    woC = wo * a.C;
    row_gap = wsC - woC;        // a carry from the last column to the next row
    img_gap = (hs - ho) * wsC;  // and from the last row to the next image
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const LoadPos c = load_pos<T, false, W, L>(wave, lane, i);
      const int32_t nn = (int32_t)mn0 + c.c, r = nn / a.Lp, e = nn - r * a.Lp;
      const int32_t px = (int32_t)kb + c.r, q1 = px / wo, n = q1 / ho;
      pleft[i] = (int32_t)ke - px;
      j[i] = px - q1 * wo;
      i_[i] = q1 - n * ho;
      y0[i] = r < a.rows ? r - a.padr : -(1 << 24);  // (outside every image)
      q[i] = (j[i] - a.pads) * a.C + e;
      left[i] = a.L - e;
      o[i] = (int32_t)(((uint32_t)n * (uint32_t)hs + (uint32_t)(i_[i] + r - a.padr)) * (uint32_t)wsC + (uint32_t)q[i]);
    }
  }
  __device__ __forceinline__ void load(int, uint4 (&v)[L], Fix& f) {
    bool any = false;
    f.keep = 0;
#pragma unroll
    for (int i = 0; i < L; ++i) {
      const uint32_t k = run_keep<E>(pleft[i] > 0 && (uint32_t)(i_[i] + y0[i]) < (uint32_t)hs, q[i], wsC, left[i]);
      const int from = clampi(o[i], 0, total - E);
      v[i] = load_chunk<ES>(p + (uint32_t)from * (uint32_t)ES);
      f.keep |= k << (8 * i);
      any |= o[i] != from && k != 0;
      pleft[i] -= BK;
      j[i] += dj;
      q[i] += dqs;
      o[i] += doff;
      i_[i] += di;
      if (j[i] >= wo) {
        j[i] -= wo;
        q[i] -= woC;
        o[i] += row_gap;
        ++i_[i];
      }
      if (i_[i] >= ho) {
        i_[i] -= ho;
        o[i] += img_gap;
      }
    }
    f.shift = __any(any);
  }
  __device__ __forceinline__ void load_last(uint4 (&v)[L], LastFix& f) { run_load_last(*this, v, f); }
  // (rare: the first and last pixels' chunks) the offset again, by division
  __device__ __forceinline__ int shift(int t, int i) {
    const LoadPos c =
        load_pos<T, false, W, L>(__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), (int)threadIdx.x & 63, i);
    const int32_t nn = n0 + c.c, r = nn / lp, e = nn - r * lp;
    const int32_t px = k0 + t * BK + c.r, q1 = px / wo, n = q1 / ho;
    const int32_t at = (int32_t)(((uint32_t)n * (uint32_t)hs + (uint32_t)(q1 - n * ho + r - padr)) * (uint32_t)wsC +
                                 (uint32_t)((px - q1 * wo - pads) * C + e));
    return end_shift<E>(at, total);
  }
};

// ------------------------------------------------------------- fragments

template <class T, bool KC, int W>
__device__ __forceinline__ lds::LaneFrag lane_frag(int lane) {
  if constexpr (KC || sizeof(typename T::storage) == 2) {
    return lds::lane_frag<KC, W>(lane);
  } else {
    lds::LaneFrag f;
    f.swz = (uint32_t)(lane >> 4);
    f.row_off = (uint32_t)(lane >> 4) * (4u * W * 4u) + (uint32_t)(lane & 15) * 4u;
    f.c = 0;
    return f;
  }
}

// 16 rows (mn) from tile row r0, half step kk (0 or 1): 32 16-bit or 16 fp32 k.
template <class T, bool KC, int W>
__device__ __forceinline__ uint4 fragment(const char* tile, int r0, int kk, const lds::LaneFrag& f) {
  if constexpr (KC || sizeof(typename T::storage) == 2) {
    return lds::fragment<KC, W>(tile, r0, kk, f);
  } else {
    const char* p = tile + (uint32_t)kk * (16u * W * 4u) + f.row_off + (((uint32_t)(r0 >> 4) ^ f.swz) << 6);
    return make_uint4(*(const uint32_t*)p, *(const uint32_t*)(p + W * 4), *(const uint32_t*)(p + 2 * W * 4),
                      *(const uint32_t*)(p + 3 * W * 4));
  }
}

__device__ __forceinline__ uint32_t dword(const uint4& v, int q) {
  return q == 0 ? v.x : q == 1 ? v.y : q == 2 ? v.z : v.w;
}

// NA accumulator sets (fp32: 1 or 4, set q for k mod 4 = q).
template <class T, int NA, int FM, int FN>
__device__ __forceinline__ void mfma_step(const uint4 (&a)[FM], const uint4 (&b)[FN], float4_t (&acc)[NA][FM][FN]) {
  if constexpr (sizeof(typename T::storage) == 2) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[0][i][j] = Mfma<T>::run(b[j], a[i], acc[0][i][j]);
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
          acc[q % NA][i][j] =
              __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, dword(b[j], q)),
                                                   __builtin_bit_cast(float, dword(a[i], q)), acc[q % NA][i][j], 0, 0, 0);
  }
}

template <class T, class TL, int NR>
struct Sets {
  uint4 a[NR][TL::LA], b[NR][TL::LB];
  Fix fa[NR], fb[NR];
};

// Tile t of one operand: registers -> LDS.  A loader that may need to fix
// any step's chunks (image edges) is tested per wave.
template <int ES, class Loader, int L>
__device__ __forceinline__ void commit(char* dst, int t, const uint4 (&v)[L], const Fix& f, Loader& ld) {
  if constexpr (Loader::ANY_STEP) {
    if (__any(f.keep != keep_all<16 / ES, L>()) || f.shift) {
#pragma unroll
      for (int i = 0; i < L; ++i) {
        uint4 c = v[i];
        if (f.shift) c = shift_chunk<ES>(c, ld.shift(t, i));
        *(uint4*)(dst + i * 1024) = keep_chunk<ES>(c, f.keep, i);
      }
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < L; ++i) *(uint4*)(dst + i * 1024) = v[i];
}
template <int ES, int L>
__device__ __forceinline__ void commit_last(char* dst, const uint4 (&v)[L], const LastFix& f) {
#pragma unroll
  for (int i = 0; i < L; ++i) {
    uint4 c = v[i];
    const int d = (int)((f.shift >> (8 * i)) & 0xffu) - 16;
    if (__any(d != 0)) c = shift_chunk<ES>(c, d);
    *(uint4*)(dst + i * 1024) = keep_chunk<ES>(c, f.keep, i);
  }
}

// The products of the tile in one LDS stage.
template <class T, class TL, class LA, class LB, int NA>
__device__ __forceinline__ void tile_products(const char* ta, const char* tb, int wm, int wn, const lds::LaneFrag& fa,
                                              const lds::LaneFrag& fb, float4_t (&acc)[NA][TL::FM][TL::FN]) {
  uint4 a0[TL::FM], b0[TL::FN], a1[TL::FM], b1[TL::FN];
#pragma unroll
  for (int i = 0; i < TL::FM; ++i) a0[i] = fragment<T, LA::KC, TL::BM>(ta, wm * TL::WTM + i * 16, 0, fa);
#pragma unroll
  for (int j = 0; j < TL::FN; ++j) b0[j] = fragment<T, LB::KC, TL::BN>(tb, wn * TL::WTN + j * 16, 0, fb);
#pragma unroll
  for (int i = 0; i < TL::FM; ++i) a1[i] = fragment<T, LA::KC, TL::BM>(ta, wm * TL::WTM + i * 16, 1, fa);
#pragma unroll
  for (int j = 0; j < TL::FN; ++j) b1[j] = fragment<T, LB::KC, TL::BN>(tb, wn * TL::WTN + j * 16, 1, fb);
  mfma_step<T, NA>(a0, b0, acc);
  mfma_step<T, NA>(a1, b1, acc);
}

// Steps t + J .. t + U - 1 of one unrolled round; tile t + J is in LDS stage
// J % 2, the tiles after it in register sets (J + 1) % NR, ...
// CHECK = false: the round's loads and tiles all exist.
template <class T, class TL, int NR, class LA, class LB, int J, int U, bool CHECK, int NA>
__device__ __forceinline__ void steps(int t, int n1, char* const (&sa)[2], char* const (&sb)[2], uint32_t wa,
                                      uint32_t wb, int wm, int wn, const lds::LaneFrag& fa, const lds::LaneFrag& fb,
                                      LA& la, LB& lb, Sets<T, TL, NR>& s, float4_t (&acc)[NA][TL::FM][TL::FN]) {
  if constexpr (J < U) {
    if (CHECK && t + J >= n1) return;
    constexpr int S = J % NR, S1 = (J + 1) % NR;
    if (!CHECK || t + J + NR < n1) {
      la.load(t + J + NR, s.a[S], s.fa[S]);
      lb.load(t + J + NR, s.b[S], s.fb[S]);
    }
    tile_products<T, TL, LA, LB, NA>(sa[J & 1], sb[J & 1], wm, wn, fa, fb, acc);
    if (!CHECK || t + J + 1 < n1) {
      commit<El<T>::ES>(sa[(J + 1) & 1] + wa, t + J + 1, s.a[S1], s.fa[S1], la);
      commit<El<T>::ES>(sb[(J + 1) & 1] + wb, t + J + 1, s.b[S1], s.fb[S1], lb);
    }
    __syncthreads();
    steps<T, TL, NR, LA, LB, J + 1, U, CHECK, NA>(t, n1, sa, sb, wa, wb, wm, wn, fa, fb, la, lb, s, acc);
  }
}

template <class T, class OutT, class TL, int NR, class LA, class LB>
__global__ void __launch_bounds__(TL::NT, TL::OCC)
gemm_reg_kernel(typename LA::Args aa, typename LB::Args ba, int64_t M, int64_t N, int64_t K, Epilogue ep) {
  constexpr int FM = TL::FM, FN = TL::FN, ES = El<T>::ES, BK = El<T>::BK;
  __shared__ __attribute__((aligned(1024))) char a0[TL::A_BYTES];
  __shared__ __attribute__((aligned(1024))) char b0[TL::B_BYTES];
  __shared__ __attribute__((aligned(1024))) char a1[TL::A_BYTES];
  __shared__ __attribute__((aligned(1024))) char b1[TL::B_BYTES];
  char* const sa[2] = {a0, a1};
  char* const sb[2] = {b0, b1};
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / TL::WN, wn = wave % TL::WN;

  int tm, tn, split;
  split_tile_coords(ceil_div(M, TL::BM), ceil_div(N, TL::BN), tm, tn, split);
  const int64_t m0 = (int64_t)tm * TL::BM, n0 = (int64_t)tn * TL::BN;
  int64_t kbeg = 0, kend = K;
  if (ep.partial) {
    kbeg = (int64_t)split * ep.k_per_split;
    kend = kbeg + ep.k_per_split < K ? kbeg + ep.k_per_split : K;
  }
  const int nk = (int)ceil_div(kend - kbeg, BK);

  LA la;
  LB lb;
  la.init(aa, m0, kbeg, kend, wave, lane);
  lb.init(ba, n0, kbeg, kend, wave, lane);
  const uint32_t wa = (uint32_t)(wave * TL::LA) * 1024u + (uint32_t)lane * 16u;
  const uint32_t wb = (uint32_t)(wave * TL::LB) * 1024u + (uint32_t)lane * 16u;
  const lds::LaneFrag fa = lane_frag<T, LA::KC, TL::BM>(lane), fb = lane_frag<T, LB::KC, TL::BN>(lane);

  // fp32 sums of a wave tile of few fragments run in four chains (k mod 4)
  // that are added at the end: a quarter of the roundings in a row, and
  // enough independent MFMAs to hide their latency
  constexpr int NA = ES == 4 && FM * FN <= 4 ? 4 : 1;
  float4_t accs[NA][FM][FN];
#pragma unroll
  for (int q = 0; q < NA; ++q)
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) accs[q][i][j] = (float4_t){0.f, 0.f, 0.f, 0.f};

  // Tiles 0 .. n1 - 1 are pipelined; the last one, which may end inside a step
  // and at the operands' ends, is fetched beside the final rounds and
  // multiplied after them, so that only it carries the code for that (code of
  // 38-95 KB was 14-34 KB without it in every round: 1000 x 777 x 1531 bf16
  // 17.7 -> 15.4 us).  Two loaders that fix any step's chunks need no such step.
  constexpr bool LAST = !(LA::ANY_STEP && LB::ANY_STEP);
  const int n1 = LAST ? nk - 1 : nk;
  Sets<T, TL, NR> s;
#pragma unroll
  for (int r = 0; r < NR; ++r)
    if (r < n1) {
      la.load(r, s.a[r], s.fa[r]);
      lb.load(r, s.b[r], s.fb[r]);
    }
  if (n1 > 0) {
    commit<ES>(sa[0] + wa, 0, s.a[0], s.fa[0], la);
    commit<ES>(sb[0] + wb, 0, s.b[0], s.fb[0], lb);
  }
  __syncthreads();
  constexpr int U = NR % 2 == 0 ? NR : 2 * NR;
  int t = 0;
  // Everything fetched so far has landed before the steady loop: with loads of
  // the branches above outstanding at its head the compiler waits there for
  // every load in flight, once per round (fp32 NN 1024 x 2048 x 2048 takes a tenth longer).
  if (U + NR <= n1) __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
  for (; t + U + NR <= n1; t += U)
    steps<T, TL, NR, LA, LB, 0, U, false, NA>(t, n1, sa, sb, wa, wb, wm, wn, fa, fb, la, lb, s, accs);
  uint4 za[TL::LA], zb[TL::LB];
  LastFix ga, gb;
  if (LAST && nk > 0) {
    const int64_t kz = kbeg + (int64_t)n1 * BK;
    LA qa;
    LB qb;
    qa.init(aa, m0, kz, kend, wave, lane);
    qb.init(ba, n0, kz, kend, wave, lane);
    qa.load_last(za, ga);
    qb.load_last(zb, gb);
  }
  for (; t < n1; t += U)
    steps<T, TL, NR, LA, LB, 0, U, true, NA>(t, n1, sa, sb, wa, wb, wm, wn, fa, fb, la, lb, s, accs);
  if (LAST && nk > 0) {
    char* const ta = n1 & 1 ? sa[1] : sa[0];
    char* const tb = n1 & 1 ? sb[1] : sb[0];
    commit_last<ES>(ta + wa, za, ga);
    commit_last<ES>(tb + wb, zb, gb);
    __syncthreads();
    tile_products<T, TL, LA, LB, NA>(ta, tb, wm, wn, fa, fb, accs);
  }
  float4_t(&acc)[FM][FN] = accs[0];
  if constexpr (NA == 4) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = (accs[0][i][j] + accs[1][i][j]) + (accs[2][i][j] + accs[3][i][j]);
  }

  const int64_t mb = m0 + wm * TL::WTM + (lane & 15);
  const int64_t nb = n0 + wn * TL::WTN + 4 * (lane >> 4);
  if constexpr (LB::RUNS) {
    // filter gradients: columns run through padded filter rows (Lp columns
    // for L elements); plain fp32 results or split partials
    const int64_t NR_ = (int64_t)ba.rows * ba.L;
    float* P = ep.partial ? ep.partial + (int64_t)split * M * NR_ : (float*)ep.D;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int32_t n = (int32_t)(nb + j * 16), r = n / ba.Lp, e = n - r * ba.Lp;
      if (n >= N) continue;
      const bool v4 = (ba.L & 3) == 0 && ((uintptr_t)P & 15) == 0 && e + 4 <= ba.L;
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        const int64_t m = mb + i * 16;
        if (m >= M) continue;
        float* p = P + m * NR_ + (int64_t)r * ba.L + e;
        if (v4) {
          *(float4*)p = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (e + q < ba.L) p[q] = acc[i][j][q];
        }
      }
    }
    return;
  }
  if (ep.partial) {
    float* P = ep.partial + (int64_t)split * M * N;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int64_t m = mb + i * 16, n = nb + j * 16;
        if (m >= M) continue;
        float* p = P + m * N + n;
        if ((N & 3) == 0 && n + 4 <= N) {
          *(float4*)p = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (n + e < N) p[e] = acc[i][j][e];
        }
      }
    return;
  }
  epilogue_any<T, OutT, FM, FN>(ep, M, N, mb, nb, acc);
}

// 128 x 128 with waves of 64 x 64; 128 x 64 and 64 x 64 for narrow products
// and small grids; 64 x 64 in at most 128 registers for 16-bit products of one
// or two K steps
typedef lds::Tile<128, 128, 2, 2, 2> TileR128;
typedef lds::Tile<128, 64, 2, 2, 2> TileR128x64;
typedef lds::Tile<64, 64, 2, 2, 2> TileR64;
typedef lds::Tile<64, 64, 2, 2, 4> TileR64Shallow;

}  // namespace reg
}  // namespace mdnn
