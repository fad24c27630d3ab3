// The slab schedule's instantiations: the deep ResNet-101 stages.
#include "bottleneck_slab.hpp"

namespace lasnet {
namespace {

size_t round256(size_t v) { return (v + 255) / 256 * 256; }
int small_div_magic(int d) { return 65536 / d + 1; }
constexpr int imax(int a, int b) { return a > b ? a : b; }
constexpr int kSlabLds = 152 * 1024;             // most a workgroup may take (its tables are static LDS beside it)

// What a way to cut a convolution costs, in clocks.  A round of workgroups takes its chain of dependent accesses (about
// 3 us; workgroups that fit a CU together wait together), then every workgroup of a CU reads its weights and its slab at
// the 50 bytes a clock that a CU gets while all of them read, and its waves run their MFMAs.
double cut_cost(int tiles, int slices, int lds, double bytes, int nst, int nb) {
  const int wgs = tiles * slices, fit = lds > 76 * 1024 ? 1 : 2;
  return (wgs + 256 * fit - 1) / (256 * fit) * 7000.0 + (wgs + 255) / 256 * (bytes / 50.0 + nst * nb * 2 * 16.0);
}

template <int C, int M, int NB, int KS>
struct Conv1 {
  static constexpr int slices = M / 32 * KS / 4;
  static int tiles(const SlabArgs& a) { return (a.npx + NB * 16 - 1) / (NB * 16); }
  static double cost(const SlabArgs& a) { return cut_cost(tiles(a), slices, NB * 32 * C, NB * 32.0 * C + 4 / KS * 64.0 * C, C / 32 / KS, NB); }
  static hipError_t run(SlabArgs a, const void* x, const __bf16* wp, const float* b1, __bf16* y1, hipStream_t st) {
    static std::atomic<unsigned long long> done;
    auto k = slab_conv1_kernel<C, M, NB, KS>;
    constexpr int lds = imax(NB * 32 * C, Slab<C, 1, NB, KS, kConv1Ring>::PART_BYTES);
    static_assert(lds <= kSlabLds, "LDS");
    if (hipError_t e = allow_dynamic_lds((const void*)k, lds, done); e != hipSuccess) return e;
    a.nsl = slices;
    hipLaunchKernelGGL(k, dim3(slab_grid(tiles(a), slices)), dim3(kSlabThreads), lds, st, a, (const __bf16*)x, wp, b1, y1);
    return hipGetLastError();
  }
};

template <int M, int NB, int KS>
struct Conv2 {
  static constexpr int slices = M / 32 * KS / 4;
  static int ppt(const SlabArgs& a) { return NB * 16 / (a.g.S * a.g.S); }
  static int lds(const SlabArgs& a) {
    return imax((slab_zero_row<M>(ppt(a) * (a.g.S + 2) * (a.g.S + 2)) + 1) * M * 2, Slab<M, 9, NB, KS, kConv2Ring>::PART_BYTES);
  }
  static bool fits(const SlabArgs& a) { return ppt(a) > 0 && lds(a) <= kSlabLds; }
  static int tiles(const SlabArgs& a, int patches) { return (patches + ppt(a) - 1) / ppt(a); }
  static double cost(const SlabArgs& a) {
    if (!fits(a)) return 1e30;
    const int patches = a.idx ? (a.g.P + 1) / 2 : a.g.P;
    return cut_cost(tiles(a, patches), slices, lds(a), lds(a) + 4 / KS * 64.0 * 9 * M, 9 * M / 32 / KS, NB);
  }
  static hipError_t run(SlabArgs a, const __bf16* wp, const float* b2, const __bf16* y1, __bf16* y2, hipStream_t st) {
    static std::atomic<unsigned long long> done;
    auto k = slab_conv2_kernel<M, NB, KS>;
    if (hipError_t e = allow_dynamic_lds((const void*)k, kSlabLds, done); e != hipSuccess) return e;
    a.nsl = slices;
    a.ppt = ppt(a);
    hipLaunchKernelGGL(k, dim3(slab_grid(tiles(a, a.g.P), slices)), dim3(kSlabThreads), lds(a), st, a, wp, b2, y1, y2);
    return hipGetLastError();
  }
};

template <int C, int M, int NB>
struct Conv3 {
  static constexpr int slices = C / 128;
  static int tiles(int rows) { return (rows + NB * 16 - 1) / (NB * 16); }
  static double cost(const SlabArgs& a) {
    return cut_cost(tiles(a.idx ? (a.npx + 1) / 2 : a.npx), slices, NB * 32 * M, NB * 32.0 * M + 256.0 * M + NB * 16 * 512.0, M / 32, NB);
  }
  static hipError_t run(SlabArgs a, const void* x, const __bf16* wp, const float* b3, const __bf16* y2, void* out, bool post_relu,
                        hipStream_t st) {
    static std::atomic<unsigned long long> done;
    auto k = slab_conv3_kernel<C, M, NB>;
    constexpr int lds = NB * 32 * M;
    if (hipError_t e = allow_dynamic_lds((const void*)k, lds, done); e != hipSuccess) return e;
    a.nsl = slices;
    hipLaunchKernelGGL(k, dim3(slab_grid(tiles(a.npx), slices)), dim3(kSlabThreads), lds, st, a, (const __bf16*)x, wp, b3, y2,
                       (__bf16*)out, (int)post_relu);
    return hipGetLastError();
  }
};

// Runs the cheapest of Cs.
template <class... Cs, class... Args>
hipError_t cheapest(const SlabArgs& a, Args... args) {
  double best = 1e30;
  hipError_t (*run)(SlabArgs, Args...) = nullptr;
  ((Cs::cost(a) < best ? (void)(best = Cs::cost(a), run = &Cs::run) : (void)0), ...);
  return run ? run(a, args...) : hipErrorInvalidValue;
}

template <int C, int M>
hipError_t launch(const SlabArgs& a, const void* x, const __bf16* wp, const float* b1, const float* b2, const float* b3,
                  __bf16* y1, __bf16* y2, void* out, bool relu, hipStream_t st) {
  const __bf16 *w2 = wp + (size_t)M * C, *w3 = w2 + (size_t)9 * M * M;
  hipError_t e = cheapest<Conv1<C, M, 1, 4>, Conv1<C, M, 1, 2>, Conv1<C, M, 1, 1>, Conv1<C, M, 2, 4>, Conv1<C, M, 2, 2>,
                          Conv1<C, M, 2, 1>>(a, x, wp, b1, y1, st);
  if (e != hipSuccess) return e;
  e = cheapest<Conv2<M, 1, 4>, Conv2<M, 1, 2>, Conv2<M, 1, 1>, Conv2<M, 2, 4>, Conv2<M, 2, 2>, Conv2<M, 2, 1>, Conv2<M, 4, 4>,
               Conv2<M, 4, 2>, Conv2<M, 4, 1>>(a, w2, b2, (const __bf16*)y1, y2, st);
  if (e != hipSuccess) return e;
  return cheapest<Conv3<C, M, 1>, Conv3<C, M, 2>, Conv3<C, M, 4>>(a, x, w3, b3, (const __bf16*)y2, out, relu, st);
}

}  // namespace

// y1 and y2, one bf16 row of M channels per pixel each.
size_t slab_workspace_bytes(const Geom& g) { return 2 * round256((size_t)g.N * g.H * g.W * g.M * 2); }

// Where it is the faster one, by the pixels of the map (block alone, us, iid lists at activation ratio 0.5 and 0.9):
//   14x14x1024, S=2   N=1 fused 20.9 / 20.9, slab 14.4 / 14.3    N=16 24.7 / 24.6, 18.8 / 26.3    N=20 24.5 / 25.2, 25.5 / 27.5
//               S=7   N=1 fused 29.7 / 30.7, slab 14.6 / 14.4    N=32 32.9 / 33.7, 25.7 / 31.7    N=40 33.2 / 35.1, 29.7 / 38.6
//               dense N=1 fused 37.4, slab 19.1                  N=32 39.1, 37.4                  N=40 39.4, 44.9
//   7x7x2048, S=1     N=1 tiled 35.2 / 38.5, slab 17.9 / 18.2    N=40 54.4 / 62.0, 34.4 / 51.8    N=48 54.3 / 64.8, 56.6 / 80.8
// (the fused kernel's larger tiles of S = 7 leave it fewer workgroups, so its end of the range is farther out).
bool slab_takes(const Geom& g) {
  const long long px = (long long)g.N * g.H * g.W;
  if (g.S * g.S > 64) return false;              // (a patch is at most four blocks of rows)
  if (g.C == 1024 && g.M == 256) return px <= (g.S >= 7 ? 32 * 196 : 16 * 196);
  if (g.C == 2048 && g.M == 512) return px <= 40 * 49;
  return false;
}

hipError_t launch_slab(const Geom& g, const void* x, const int32_t* idx, const int32_t* count, const void* packed,
                       const float* b1, const float* b2, const float* b3, void* out, bool post_relu, void* workspace,
                       hipStream_t st) {
  SlabArgs a;
  a.g = g;
  a.idx = idx;
  a.count = count;
  a.npx = g.N * g.H * g.W;
  a.nsl = a.ppt = 0;
  a.m_t2 = small_div_magic((g.S + 2) * (g.S + 2));
  a.m_t = small_div_magic(g.S + 2);
  a.m_s2 = small_div_magic(g.S * g.S);
  a.m_s = small_div_magic(g.S);
  __bf16* y1 = (__bf16*)workspace;
  __bf16* y2 = (__bf16*)((unsigned char*)workspace + round256((size_t)a.npx * g.M * 2));
  if (g.M == 256) return launch<1024, 256>(a, x, (const __bf16*)packed, b1, b2, b3, y1, y2, out, post_relu, st);
  return launch<2048, 512>(a, x, (const __bf16*)packed, b1, b2, b3, y1, y2, out, post_relu, st);
}

}  // namespace lasnet
