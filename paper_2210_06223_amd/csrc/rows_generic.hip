// The row schedule for every shape and type without a matrix-core kernel of its own: fp32, and bf16 at any width.
#include "bottleneck_rows.hpp"

#include <type_traits>

namespace lasnet {
namespace {

// How a convolution is cut: NB row blocks per wave, KS waves to a tile's reduction, nsl channel slices per row tile.
// 1024 waves are one per SIMD.  More rows per wave read the weights less often, so NB is as large as leaves the chip
// that many tiles; with fewer even at NB = 1 the waves of a workgroup share a tile's reduction.
struct RowsCut { int nb, ks, units, nsl; };
RowsCut rows_cut(long long rows_max, long long rows_expected, int pairs, int ksteps) {
  RowsCut c;
  c.nb = 4;
  while (c.nb > 1 && (rows_expected + 16 * c.nb - 1) / (16 * c.nb) * pairs < 1024) c.nb /= 2;
  const long long tiles = (rows_expected + 16 * c.nb - 1) / (16 * c.nb);
  c.ks = tiles * pairs < 1024 && ksteps >= 8 ? 4 : 1;
  c.units = (int)((rows_max + 16 * c.nb - 1) / (16 * c.nb));
  const int wc = 4 / c.ks, most = (pairs + wc - 1) / wc;
  c.nsl = (int)((1024 + tiles - 1) / tiles);
  if (c.nsl > most) c.nsl = most;
  return c;
}

#define ROWS_DISPATCH(c, CALL)                                             \
  if (c.ks == 4) {                                                         \
    if (c.nb == 1) CALL(1, 4); else if (c.nb == 2) CALL(2, 4); else CALL(4, 4); \
  } else {                                                                 \
    if (c.nb == 1) CALL(1, 1); else if (c.nb == 2) CALL(2, 1); else CALL(4, 1); \
  }

template <class F, bool VEC>
hipError_t run_rows(const Geom& g, const void* x, const int32_t* idx, const int32_t* count, const BlockWeights& w, void* out,
                    bool post_relu, void* workspace, hipStream_t st) {
  typedef typename F::T T;
  RowsLayout l;
  if (!rows_layout<F>(g, l)) return hipErrorInvalidValue;
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
  a.w1_bytes = (unsigned)l.w1;
  a.w2_bytes = (unsigned)l.w2;
  a.w3_bytes = (unsigned)l.w3;
  const int hw = g.H * g.W;
  for (int n0 = 0; n0 < g.N; n0 += l.images) {
    const int n = g.N - n0 < l.images ? g.N - n0 : l.images;
    a.px0 = n0 * hw;
    a.npx = n * hw;
    const long long fragments = (long long)a.pairs1 * a.ks1 + (long long)a.pairs1 * 9 * a.ksm + (long long)a.pairs3 * a.ksm;
    const int pack_blocks = n0 == 0 ? (int)((fragments * 128 + kRowsThreads - 1) / kRowsThreads) : 0;
    const int need_blocks = idx ? (a.npx + kNeedPixels - 1) / kNeedPixels : 0;
    if (pack_blocks + need_blocks > 0)
      hipLaunchKernelGGL(rows_plan_kernel<F>, dim3(pack_blocks + need_blocks), dim3(kRowsThreads), 0, st, a, pack_blocks,
                         (const T*)w.W1, (const T*)w.W2, (const T*)w.W3, wp1, need);
    // the list's rows of this chunk are not known here: half of the pixels is a middling activation ratio
    const long long rows = (long long)g.P * g.S * g.S, likely = idx ? (a.npx + 1) / 2 : a.npx;
    RowsCut c = rows_cut(a.npx, a.npx, a.pairs1, a.ks1);
#define ROWS_CONV1(NB, KS)                                                                                               \
  hipLaunchKernelGGL((rows_conv1_kernel<F, VEC, NB, KS>), dim3(rows_grid(c.units, c.nsl)), dim3(kRowsThreads), 0, st, a, \
                     c.nsl, (const T*)x, wp1, w.b1, y1)
    ROWS_DISPATCH(c, ROWS_CONV1)
    c = rows_cut(rows, likely, a.pairs1, 9 * a.ksm);
#define ROWS_CONV2(NB, KS)                                                                                               \
  hipLaunchKernelGGL((rows_conv2_kernel<F, NB, KS>), dim3(rows_grid(c.units, c.nsl)), dim3(kRowsThreads), 0, st, a,      \
                     c.nsl, wp2, w.b2, y1, y2)
    ROWS_DISPATCH(c, ROWS_CONV2)
    c = rows_cut(rows, likely, a.pairs3, a.ksm);
#define ROWS_CONV3(NB, KS)                                                                                               \
  hipLaunchKernelGGL((rows_conv3_kernel<F, VEC, NB, KS>), dim3(rows_grid(c.units, c.nsl)), dim3(kRowsThreads), 0, st, a, \
                     c.nsl, (const T*)x, wp3, w.b3, y2, (T*)out, (int)post_relu)
    ROWS_DISPATCH(c, ROWS_CONV3)
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

size_t rows_workspace_bytes(int dtype, const Geom& g) {
  RowsLayout l;
  return (dtype == LASNET_BF16 ? rows_layout<Bf16Wide>(g, l) : rows_layout<Fp32>(g, l)) ? l.total : 0;
}

hipError_t launch_rows(int dtype, const Geom& g, const void* x, const int32_t* idx, const int32_t* count,
                       const BlockWeights& w, void* out, bool post_relu, void* workspace, hipStream_t st) {
  if (g.P == 0) return hipSuccess;
  const uintptr_t low = (uintptr_t)x | (uintptr_t)out;
  if (dtype == LASNET_BF16) {
    if (low % 16 == 0 && g.C % 8 == 0) return run_rows<Bf16Wide, true>(g, x, idx, count, w, out, post_relu, workspace, st);
    return run_rows<Bf16Wide, false>(g, x, idx, count, w, out, post_relu, workspace, st);
  }
  if (low % 16 == 0 && g.C % 4 == 0) return run_rows<Fp32, true>(g, x, idx, count, w, out, post_relu, workspace, st);
  return run_rows<Fp32, false>(g, x, idx, count, w, out, post_relu, workspace, st);
}

}  // namespace lasnet
