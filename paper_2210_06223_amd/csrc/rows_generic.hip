// The row schedule for every shape and type without a matrix-core kernel of its own: fp32, and bf16 at any width.
#include "bottleneck_rows.hpp"

namespace lasnet {
namespace {

// Whether the convolutions read the caller's weights.  Read in their natural layout -- 64-byte pieces of 16 rows, which lie a
// power of two apart at the usual widths -- they cost more per fragment than packed ones, and a tile's reduction that is long
// stands for them, so it pays where the fragments that the call reads (every pixel active) are few and conv1's reduction is short (fp32 from
// 12 k-steps on, it never did).  Direct / with a plan, r=0.5 if not noted, us:
//   bf16, up to six k-steps:      26k  24 x 32x32x128 mid 32 26.8 / 30.5              28k  5 x 40x40x160 mid 40 24.1 / 26.6 (r=1 29.4 / 33.3)
//     31k  32 x 32x32x96 mid 24 28.6 / 32.3 (r=1 38.3 / 41.1)  35k  32 x 32x32x128 30.8 / 34.4 (r=1 37.3 / 40.4)
//     beyond  38k  18 x 28x20x192 mid 48 31.7 / 31.7           41k  16 x 56x56x64 mid 16 41.1 / 41.0 (47k  16 x 28x28x192, S=7 31.5 / 33.0, r=1 40.9 / 41.5)
//   bf16, more:  2k  20x20x320 mid 80 21.9 / 24.5               15k  40x40x384 mid 96 23.6 / 25.1
//     beyond  31k  2 x 40x40x384, r=0.6 27.5 / 27.9, r=1 30.3 / 30.2           46k  3 x 40x40x384, r=0.3 28.0 / 28.0, r=0.6 32.1 / 31.3
//       of seven to nine k-steps it would still pay there: 29k  7 x 32x32x224 mid 56 25.5 / 26.8, 33k  8 of them 25.7 / 27.1 (r=1 30.9 / 33.1),
//       35k  4 x 32x32x288 mid 72 25.4 / 27.6 (r=1 27.9 / 29.3)
//   fp32, up to six:  4k  4 x 32x32x128 21.8 / 23.5             12k  4 x 28x28x192 25.1 / 26.0         13k  12 x 32x32x128 26.6 / 28.7
//     beyond  15k  16 x 32x32x96 26.8 / 28.9 but r=1 33.9 / 32.9  17k  16 x 32x32x128 28.9 / 29.7 but r=1 36.3 / 33.2
//   fp32, 7 to 11:  3k  20x20x320 25.3 / 26.2                   7k  28x28x320 mid 80 25.5 / 26.4, 2 x 28x28x256 mid 64 24.2 / 24.5
//     beyond  13k  2 x 40x40x224 mid 56 26.9 / 26.4, 56x56x256 26.2 / 25.6 (r=1 29.9 / 28.4)
//   fp32, 12:  1k  8x8x384 mid 96 26.2 / 25.5                   5k  24x24x384 27.2 / 26.6              11k  2 x 24x24x384 28.2 / 26.8
template <class F>
bool direct_is_faster(const Geom& g) {
  const long long tiles = ((long long)g.N * g.H * g.W + 15) / 16, pairs1 = (g.M + 31) / 32, pairs3 = (g.C + 31) / 32;
  const long long fragments = tiles * (2 * pairs1 * pairs3 + 9 * pairs1 * pairs1);
  const long long few = F::ES == 2 ? (pairs3 <= 6 ? 36000 : 28000) : pairs3 <= 6 ? 14000 : pairs3 < 12 ? 7000 : 0;
  return g.P <= kDirectCells && pairs1 <= 3 && fragments <= few;
}

template <class F, bool VEC>
hipError_t run_rows(const Geom& g, const void* x, const int32_t* idx, const int32_t* count, const BlockWeights& w, void* out,
                    bool post_relu, bool copy, void* workspace, hipStream_t st) {
  typedef typename F::T T;
  RowsLayout l;
  if (!rows_layout<F>(g, l)) return hipErrorInvalidValue;
  const bool direct = VEC && l.images == g.N && g.M % F::EPP == 0 &&
                      (((uintptr_t)w.W1 | (uintptr_t)w.W2 | (uintptr_t)w.W3) & 15) == 0 && direct_is_faster<F>(g);
  const bool rides = copy && VEC && g.P <= kDirectCells;     // the copy is a part of the first launch
  if (copy && !rides)
    if (hipError_t e = launch_copy(x, out, (size_t)g.N * g.H * g.W * g.C * F::ES, st); e != hipSuccess) return e;
  unsigned char* wp1 = (unsigned char*)workspace;
  unsigned char* wp2 = wp1 + rows_round(l.w1);
  unsigned char* wp3 = wp2 + rows_round(l.w2);
  uint8_t* need = wp3 + rows_round(l.w3);
  unsigned char* y1 = need + l.need;
  unsigned char* y2 = y1 + l.y;
  RowsArgs a;
  a.g = g;
  a.ks1 = a.pairs3 = (g.C + 31) / 32;
  a.ksm = a.pairs1 = (g.M + 31) / 32;
  a.idx = idx;
  a.count = count;
  a.need = idx ? need : nullptr;
  constexpr unsigned kStep = 2 * F::KPL * 1024;
  a.w1 = RowsWeights{a.ks1 * kStep, kStep};
  a.w2 = RowsWeights{9 * a.ksm * kStep, kStep};
  a.w3 = RowsWeights{a.ksm * kStep, kStep};
  a.w1_bytes = (unsigned)l.w1;
  a.w2_bytes = (unsigned)l.w2;
  a.w3_bytes = (unsigned)l.w3;
  a.cpi = div31((unsigned)(g.G * g.GW));
  a.gw = div31((unsigned)g.GW);
  a.s2 = div31((unsigned)(g.S * g.S));
  a.s = div31((unsigned)g.S);
  a.conv_blocks = 0;
  const int hw = g.H * g.W;
  if constexpr (VEC)
    if (direct) {
      a.px0 = 0;
      a.npx = g.N * hw;
      a.need = nullptr;
      a.w1_bytes = a.w3_bytes = (unsigned)((size_t)g.M * g.C * F::ES);
      a.w2_bytes = (unsigned)((size_t)9 * g.M * g.M * F::ES);
      return launch_rows_convs<F, true, call_weights>(a, a.npx, x, (const unsigned char*)w.W1, (const unsigned char*)w.W2, (const unsigned char*)w.W3,
                                              w.b1, w.b2, w.b3, y1, y2, out, post_relu, copy, st);
    }
  for (int n0 = 0; n0 < g.N; n0 += l.images) {
    const int n = g.N - n0 < l.images ? g.N - n0 : l.images;
    a.px0 = n0 * hw;
    a.npx = n * hw;
    const long long fragments = (long long)a.pairs1 * a.ks1 + (long long)a.pairs1 * 9 * a.ksm + (long long)a.pairs3 * a.ksm;
    const int pack_blocks = n0 == 0 ? (int)((fragments * 128 + kRowsThreads - 1) / kRowsThreads) : 0;
    const int need_blocks = idx ? (a.npx + kNeedPixels - 1) / kNeedPixels : 0;
    const int copy_blocks = rides && n0 == 0 ? rows_copy_blocks<F>(g) : 0;
    if (pack_blocks + need_blocks + copy_blocks > 0)
      hipLaunchKernelGGL(rows_plan_kernel<F>, dim3(pack_blocks + need_blocks + copy_blocks), dim3(kRowsThreads), 0, st, a, pack_blocks,
                         need_blocks, (int)(g.P <= kScanCells), (const T*)x, (T*)out, (const T*)w.W1, (const T*)w.W2, (const T*)w.W3, wp1, need);
    if (idx && g.P > kScanCells) {
      const long long blocks = ((long long)g.P * (g.S + 2) + kRowsThreads - 1) / kRowsThreads;
      hipLaunchKernelGGL(rows_need_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(kRowsThreads), 0, st, a, need);
    }
    if (hipError_t e = launch_rows_convs<F, VEC, plan_weights>(a, l.images * hw, x, wp1, wp2, wp3, w.b1, w.b2, w.b3, y1, y2, out, post_relu, false, st); e != hipSuccess)
      return e;
  }
  return hipSuccess;
}

// Whether the scalar kernel is the faster one (then no workspace is asked for): where one launch of it is over before three
// or four short ones are, and where its work per pixel is so small that the row schedule, whose MFMAs and y rows are 32 channels
// wide, does several times as much.  `chain` is the FMAs that a thread does one after the other for a patch (45 to 90 ns each),
// 2048 the patches that run at once (half of the cells are active).  Where it says so the scalar kernel is the faster one, but for the calls marked *; it
// would be in others too, of many cells and little work (marked +).  Block alone on a drawn list, scalar / row schedule, us, fp32 (bf16):
//   8x8x16 M=4 S=2      7.1 / 13.0 (6.9 / 15.1)     28x28x32 M=8 S=2       11.2 / 13.1 (10.9 / 12.6)    4 x 28x28x32 M=8 S=4*  15.3 / 13.1 (14.4 / 12.7)
//   16 x 28x28x16 M=4 S=2 8.3 / 19.0 (8.3 / 18.5)   256 x 28x28x16 M=4 S=4 34.4 / 69.3 (31.4 / 48.6)    64 x 112x112x16 M=4 S=7 100 / 220 (86 / 179)
//   beyond: 2 x 8x8x48 M=12 S=2 16.2 / 12.8 (15.6 / 15.0)    8x8x48 M=12 S=4 22.2 / 12.3 (21.5 / 14.7)     16x16x64 M=16 S=2 25.2 / 13.3 (25.3 / 12.6)
//     256 x 28x28x16 M=4 S=2 105 / 71 (106 / 51)             64 x 112x112x32 M=8 S=4 730 / 247 (504 / 200)
//     8 x 28x28x32 M=8 S=2+ 12.8 / 17.7 (11.8 / 17.2)        16 x 28x28x32 M=8 S=2+ 17.6 / 19.1 (15.5 / 18.5)   64 x 28x28x64 M=4 S=4+ 25.8 / 36.3 (23.2 / 31.4)
//     32 x 28x28x16 M=4 S=2+ 14.1 / 22.6 (14.2 / 21.1)
bool scalar_is_faster(const Geom& g) {
  const double S2 = (double)g.S * g.S, W2 = (double)(g.S + 2) * (g.S + 2), M = g.M, C = g.C;
  const auto rounds = [](double n) { return (double)(long long)((n + 255) / 256); };       // of a workgroup's 256 threads
  const double chain = rounds(W2 * M) * C + rounds(S2 * M) * 9 * M + rounds(S2 * C) * M;
  const double fmas = W2 * M * C + S2 * 9 * M * M + S2 * M * C;                             // of a patch
  return chain * (1 + g.P / 2048.0) <= 170 || fmas <= 400 * S2;
}

}  // namespace

size_t rows_workspace_bytes(int dtype, const Geom& g) {
  if (scalar_is_faster(g)) return 0;
  RowsLayout l;
  return (dtype == LASNET_BF16 ? rows_layout<Bf16Wide>(g, l) : rows_layout<Fp32>(g, l)) ? l.total : 0;
}

hipError_t launch_rows(int dtype, const Geom& g, const void* x, const int32_t* idx, const int32_t* count,
                       const BlockWeights& w, void* out, bool post_relu, bool copy, void* workspace, hipStream_t st) {
  if (g.P == 0) return hipSuccess;
  const uintptr_t low = (uintptr_t)x | (uintptr_t)out;
  if (dtype == LASNET_BF16) {
    if (low % 16 == 0 && g.C % 8 == 0) return run_rows<Bf16Wide, true>(g, x, idx, count, w, out, post_relu, copy, workspace, st);
    return run_rows<Bf16Wide, false>(g, x, idx, count, w, out, post_relu, copy, workspace, st);
  }
  if (low % 16 == 0 && g.C % 4 == 0) return run_rows<Fp32, true>(g, x, idx, count, w, out, post_relu, copy, workspace, st);
  return run_rows<Fp32, false>(g, x, idx, count, w, out, post_relu, copy, workspace, st);
}

}  // namespace lasnet
