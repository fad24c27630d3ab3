// The row schedule for every shape and type without a matrix-core kernel of its own: fp32, and bf16 at any width.
#include "bottleneck_rows.hpp"

namespace lasnet {
namespace {

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
  constexpr unsigned kStep = 2 * F::KPL * 1024;
  a.w1 = RowsWeights{a.ks1 * kStep, kStep};
  a.w2 = RowsWeights{9 * a.ksm * kStep, kStep};
  a.w3 = RowsWeights{a.ksm * kStep, kStep};
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
                         (int)(g.P <= kScanCells), (const T*)w.W1, (const T*)w.W2, (const T*)w.W3, wp1, need);
    if (idx && g.P > kScanCells) {
      const long long blocks = ((long long)g.P * (g.S + 2) + kRowsThreads - 1) / kRowsThreads;
      hipLaunchKernelGGL(rows_need_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(kRowsThreads), 0, st, a, need);
    }
    if (hipError_t e = launch_rows_convs<F, VEC>(a, l.images * hw, x, wp1, wp2, wp3, w.b1, w.b2, w.b3, y1, y2, out, post_relu, st); e != hipSuccess)
      return e;
  }
  return hipSuccess;
}

// Whether the scalar kernel is the faster one (then no workspace is asked for): where one launch of it is over before three
// or four short ones are, and where its work per pixel is so small that the row schedule, whose MFMAs and y rows are 32 channels
// wide, does several times as much.  `chain` is the FMAs that a thread does one after the other for a patch (45 to 90 ns each),
// 2048 the patches that run at once (half of the cells are active).  Measured, scalar / row schedule, us, fp32:
//   8x8x16 M=4 S=2      10 / 18   28x28x32 M=8 S=2     11 / 18   4 x 28x28x32 M=8 S=4   15 / 18   16 x 28x28x16 M=4 S=2  12 / 21
//   2 x 8x8x48 M=12 S=2 16 / 19   8x8x48 M=12 S=4      22 / 18   16 x 28x28x32 M=8 S=2  26 / 21   64 x 28x28x64 M=4 S=4  36 / 33
//   64 x 112x112x16 M=4 S=7 109 / 274   256 x 28x28x16 M=4 S=4 36 / 82   S=2 417 / 278   64 x 112x112x32 M=8 S=4 677 / 274
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
