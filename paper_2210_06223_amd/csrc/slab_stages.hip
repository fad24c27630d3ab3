// The slab schedule's instantiations: the deep ResNet-101 stages.
#include "bottleneck_slab.hpp"

namespace lasnet {
namespace {

size_t round256(size_t v) { return (v + 255) / 256 * 256; }
int small_div_magic(int d) { return 65536 / d + 1; }
constexpr int kSlabLds = 152 * 1024;             // most a workgroup may take (its tables are static LDS beside it)

// What a way to cut a convolution costs, in clocks.  A round of workgroups takes its chain of dependent accesses (about
// 3 us; workgroups that fit a CU together wait together), then every workgroup of a CU reads its weights and its slab at
// the 50 bytes a clock that a CU gets while all of them read, and its waves run their MFMAs.
double cut_cost(int tiles, int slices, int nw, int lds, double bytes, int nst, int mfmas) {
  const int by_lds = 160 * 1024 / (lds + 4096), by_waves = 8 / nw;      // (two waves per SIMD: 130 to 180 registers)
  const int wgs = tiles * slices, fit = by_lds < by_waves ? by_lds : by_waves;
  return (wgs + 256 * fit - 1) / (256 * fit) * 7000.0 + (wgs + 255) / 256 * (bytes / 50.0 + nst * mfmas * 16.0);
}

// The same over the activation ratios, which are not known here: two parts of a half, one of one.  (For a half alone, 7x7x2048,
// 8 images go out in two rounds at one: 35.5 us instead of 24; for equal parts, 14x14x1024, S=2, 4 images take 13.7 us at a half
// instead of 11.4.)
template <class Fn>
double over_ratios(const SlabArgs& a, int all, Fn&& cost) {
  return a.idx ? (2 * cost((all + 1) / 2) + cost(all)) / 3 : cost(all);
}

template <int C, int M, int NB, int NW, int TJ>
struct Conv1 {
  static constexpr int pairs = SlabWave<NW, TJ>::PAIRS, slices = M / 32 / pairs;
  static int tiles(const SlabArgs& a) { return (a.npx + NB * 16 - 1) / (NB * 16); }
  static double cost(const SlabArgs& a) { return cut_cost(tiles(a), slices, NW, NB * 32 * C, NB * 32.0 * C + pairs * 64.0 * C, C / 32, NB * TJ); }
  static constexpr int lds = NB * 32 * C;
  static_assert(lds <= kSlabLds, "LDS");
  static constexpr auto k = slab_conv1_kernel<C, M, NB, NW, TJ>;
  static hipError_t prepare() {
    static std::atomic<unsigned long long> done;
    return allow_dynamic_lds((const void*)k, lds, done);
  }
  static hipError_t run(SlabArgs a, const void* x, const __bf16* wp, const float* b1, __bf16* y1, hipStream_t st) {
    a.nsl = slices;
    hipLaunchKernelGGL(k, dim3((unsigned)sliced_grid(tiles(a), slices)), dim3(NW * 64), lds, st, a, (const __bf16*)x, wp, b1, y1);
    return hipGetLastError();
  }
};

template <int M, int NB, int NW, int TJ>
struct Conv2 {
  static constexpr int pairs = SlabWave<NW, TJ>::PAIRS, slices = M / 32 / pairs;
  static int ppt(const SlabArgs& a) { return NB * 16 / (a.g.S * a.g.S); }
  static int lds(const SlabArgs& a) {
    return (slab_zero_row<M>(ppt(a) * (a.g.S + 2) * (a.g.S + 2)) + 1) * M * 2;
  }
  static bool fits(const SlabArgs& a) { return ppt(a) > 0 && lds(a) <= kSlabLds; }
  static int tiles(const SlabArgs& a, int patches) { return (patches + ppt(a) - 1) / ppt(a); }
  static double cost(const SlabArgs& a) {
    if (!fits(a)) return 1e30;
    return over_ratios(a, a.g.P, [&](int patches) {
      return cut_cost(tiles(a, patches), slices, NW, lds(a), lds(a) + pairs * 64.0 * 9 * M, 9 * M / 32, NB * TJ);
    });
  }
  static constexpr auto k = slab_conv2_kernel<M, NB, NW, TJ>;
  static hipError_t prepare() {
    static std::atomic<unsigned long long> done;
    return allow_dynamic_lds((const void*)k, kSlabLds, done);
  }
  static hipError_t run(SlabArgs a, const __bf16* wp, const float* b2, const __bf16* y1, __bf16* y2, hipStream_t st) {
    a.nsl = slices;
    a.ppt = ppt(a);
    hipLaunchKernelGGL(k, dim3((unsigned)sliced_grid(tiles(a, a.g.P), slices)), dim3(NW * 64), lds(a), st, a, wp, b2, y1, y2);
    return hipGetLastError();
  }
};

template <int C, int M, int NB>
struct Conv3 {
  static constexpr int slices = C / 128;
  static int tiles(int rows) { return (rows + NB * 16 - 1) / (NB * 16); }
  static double cost(const SlabArgs& a) {
    return over_ratios(a, a.npx, [&](int rows) {
      return cut_cost(tiles(rows), slices, 4, NB * 32 * M, NB * 32.0 * M + 256.0 * M + NB * 16 * 512.0, M / 32, NB * 2);
    });
  }
  static constexpr int lds = NB * 32 * M;
  static constexpr auto k = slab_conv3_kernel<C, M, NB>;
  static hipError_t prepare() {
    static std::atomic<unsigned long long> done;
    return allow_dynamic_lds((const void*)k, lds, done);
  }
  static hipError_t run(SlabArgs a, const void* x, const __bf16* wp, const float* b3, const __bf16* y2, void* out, bool post_relu,
                        hipStream_t st) {
    a.nsl = slices;
    hipLaunchKernelGGL(k, dim3((unsigned)sliced_grid(tiles(a.npx), slices)), dim3(256), lds, st, a, (const __bf16*)x, wp, b3, y2,
                       (__bf16*)out, (int)post_relu);
    return hipGetLastError();
  }
};

// The ways to cut one convolution: prepare() and run() take the cheapest.
template <class... Cs>
struct Cuts {
  static hipError_t prepare(const SlabArgs& a) {
    hipError_t (*p)() = pick<hipError_t (*)()>(a, &Cs::prepare...);
    return p ? p() : hipErrorInvalidValue;
  }
  template <class... Args>
  static hipError_t run(const SlabArgs& a, Args... args) {
    auto r = pick<hipError_t (*)(SlabArgs, Args...)>(a, &Cs::run...);
    return r ? r(a, args...) : hipErrorInvalidValue;
  }

 private:
  template <class Fn, class... Fns>
  static Fn pick(const SlabArgs& a, Fns... fns) {
    double best = 1e30;
    Fn f = nullptr;
    ((Cs::cost(a) < best ? (void)(best = Cs::cost(a), f = fns) : (void)0), ...);
    return f;
  }
};

// The cuts of a stage: those that some map in slab_takes' range is cheapest with.
template <int C, int M>
struct Stage {
  typedef Cuts<Conv1<C, M, 1, 2, 1>, Conv1<C, M, 2, 2, 1>, Conv1<C, M, 2, 4, 1>, Conv1<C, M, 2, 4, 2>> Cuts1;
  typedef Cuts<Conv3<C, M, 1>, Conv3<C, M, 2>, Conv3<C, M, 4>> Cuts3;
  // (512, S = 1: the windows of 32 pixels exceed the LDS)
  typedef std::conditional_t<M == 512, Cuts<Conv2<M, 1, 2, 1>, Conv2<M, 1, 4, 1>, Conv2<M, 1, 4, 2>>,
                             Cuts<Conv2<M, 1, 2, 1>, Conv2<M, 2, 2, 1>, Conv2<M, 2, 4, 1>, Conv2<M, 4, 2, 1>, Conv2<M, 4, 4, 1>,
                                  Conv2<M, 4, 4, 2>>> Cuts2;

  static hipError_t prepare(const SlabArgs& a) {
    hipError_t e = Cuts1::prepare(a);
    if (e == hipSuccess) e = Cuts2::prepare(a);
    return e == hipSuccess ? Cuts3::prepare(a) : e;
  }
  static hipError_t launch(const SlabArgs& a, const void* x, const __bf16* wp, const float* b1, const float* b2, const float* b3,
                           __bf16* y1, __bf16* y2, void* out, bool relu, hipStream_t st) {
    const __bf16 *w2 = wp + (size_t)M * C, *w3 = w2 + (size_t)9 * M * M;
    hipError_t e = Cuts1::run(a, x, wp, b1, y1, st);
    if (e == hipSuccess) e = Cuts2::run(a, w2, b2, (const __bf16*)y1, y2, st);
    return e == hipSuccess ? Cuts3::run(a, x, w3, b3, (const __bf16*)y2, out, relu, st) : e;
  }
};

SlabArgs slab_args(const Geom& g, const int32_t* idx, const int32_t* count) {
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
  return a;
}

}  // namespace

// y1 and y2, one bf16 row of M channels per pixel each.
size_t slab_workspace_bytes(const Geom& g) { return 2 * round256((size_t)g.N * g.H * g.W * g.M * 2); }

// Where it is the faster one, at every activation ratio, by the pixels of the map (us on the GPU, iid lists at ratio 0.5 / 0.9 / 1):
//   14x14x1024, S=2   N=1 fused 20.9 / 21.1 / 21.1, slab 10.6 / 10.7 / 10.7   N=16 23.9 / 23.7 / 23.7, 17.4 / 22.4 / 22.5
//               S=1   N=1 20.8 / 22.6 / 23.0, 11.5 / 11.5 / 11.5              N=10 23.8 / 23.4 / 23.4, 16.7 / 16.9 / 16.6
//                                                                             N=12 24.3 / 24.7 / 24.7, 18.1 / 25.8 / 26.3
//               S=7   N=1 30.4 / 31.1 / 31.1, 14.0 / 14.3 / 14.4              N=32 32.6 / 34.3 / 34.4, 25.1 / 33.3 / 33.9
//               dense N=1 31.1, slab 14.2                                     N=32 34.1, 33.5
//   50x60x1024, S=2   N=1 23.6 / 24.1 / 23.5, 17.2 / 22.6 / 22.7
//   7x7x2048, S=1     N=1 tiled 34.4 / 38.3 / 44.0, slab 19.3 / 19.7 / 19.9   N=40 54.7 / 63.2 / 67.5, 33.3 / 48.2 / 49.1
//   25x42x2048, S=1   N=1 fused 119 / 120 / 123, slab 30.3 / 31.9 / 45.2
// (with S = 1 a workgroup's windows take the most LDS, so its rounds are full first; the fused kernel's larger tiles of S = 7 leave
// it fewer workgroups, so its end of the range is farther out.)
bool slab_takes(const Geom& g) {
  const long long px = (long long)g.N * g.H * g.W;
  if (g.S * g.S > 64) return false;              // (a patch is at most four blocks of rows)
  if (g.C == 1024 && g.M == 256) return px <= (g.S >= 7 ? 32 * 196 : g.S > 1 ? 16 * 196 : 10 * 196);
  if (g.C == 2048 && g.M == 512) return px <= 40 * 49;
  return false;
}

hipError_t prepare_slab(const Geom& g, const int32_t* idx) {
  const SlabArgs a = slab_args(g, idx, nullptr);
  return g.M == 256 ? Stage<1024, 256>::prepare(a) : Stage<2048, 512>::prepare(a);
}

hipError_t launch_slab(const Geom& g, const void* x, const int32_t* idx, const int32_t* count, const void* packed,
                       const float* b1, const float* b2, const float* b3, void* out, bool post_relu, void* workspace,
                       hipStream_t st) {
  const SlabArgs a = slab_args(g, idx, count);
  __bf16* y1 = (__bf16*)workspace;
  __bf16* y2 = (__bf16*)((unsigned char*)workspace + round256((size_t)a.npx * g.M * 2));
  if (g.M == 256) return Stage<1024, 256>::launch(a, x, (const __bf16*)packed, b1, b2, b3, y1, y2, out, post_relu, st);
  return Stage<2048, 512>::launch(a, x, (const __bf16*)packed, b1, b2, b3, y1, y2, out, post_relu, st);
}

}  // namespace lasnet
