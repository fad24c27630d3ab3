// The row schedule of the sparse bottleneck: the three convolutions as three GEMMs over rows of pixels, y1 and y2
// through a workspace, for shapes and types without a kernel of their own (all of fp32, and bf16 at any width).
//
//   plan   (a) the weights -> MFMA A-fragments in the order a wave reads them, zero-padded to whole fragments
//          (b) one byte per pixel: does some active patch's (S+2)x(S+2) window hold it
//          (calls with few cells and small weights have none, direct_is_faster: the convolutions read the caller's weights, and
//          conv1 finds its needed pixels in the list; with few cells the copy of x to out is a part of the first launch)
//   conv1  rows = the needed pixels of a run of consecutive pixels           y1[pixel] = ReLU(b1 + W1 x)
//   conv2  rows = the list's pixels, S*S per entry, in the list's order      y2[pixel] = ReLU(b2 + W2 * y1 around it)
//   conv3  the same rows                                                     out[pixel] = x + b3 + W3 y2
//
// What bounds it: the matrix cores at batch size (fp32: 256 FLOP per clock and CU), launches and load latency
// at a few images.  So the work is cut fine -- a wave computes NB blocks of 16 pixels times 32 output channels,
// and nothing but the four waves of a workgroup has to meet -- and a wave loads both operands for itself, D
// k-steps ahead, the weights into registers and the rows through LDS of its own: a 32-deep fp32 k-step is 8 MFMAs of 32 clocks per
// 16x16 tile, so with no reuse between its four waves a CU asks its L1 for 48, 32 and 24 of the 64 bytes a clock it delivers with 1, 2 and 4 row
// blocks per wave (4 KiB of weights and 2 KiB of rows per block in each k-step).  When the rows are too few to fill the chip the four waves share one tile and split its reduction (KS = 4, partial sums
// added in a fixed order through LDS); else they take four neighbouring groups of 32 channels (KS = 1).
//
// Measured, whole call sequence (masker, list, block) against the scalar one-kernel path: fp32 56x56x256, S=4, r=0.6, one
// image 672 -> 25 us; fp32 14x14x1024, S=2, r=0.5, 16 images 7900 -> 74 us (conv1 20, conv2 24, conv3 15 us: 71 TFLOP/s
// of the 154 that a large fp32 matrix product reaches); bf16 28x20x192, mid 48, S=4, 13 images 371 -> 24 us.
//
// Number formats (products and sums are never narrower than fp32, and nothing is rounded between the convolutions):
//   Fp32     v_mfma_f32_16x16x4_f32 throughout
//   Bf16Wide bf16 x and weights: conv1 multiplies them as they are (a bf16 product is exact in fp32); y1 and y2 are kept
//            as three bf16 terms whose sum is the fp32 value (8 + 8 + 8 significant bits), so conv2 and
//            conv3 run on the bf16 matrix cores, three MFMAs of 16 clocks where fp32 ones would take 256
#pragma once
#include "common.hpp"

#include <type_traits>

namespace lasnet {
namespace {

// (the global and LDS address spaces are named: through generic pointers these would be FLAT accesses)
#define ROWS_LDS __attribute__((address_space(3)))

constexpr int kRowsThreads = 256;                 // four waves
constexpr unsigned kOutOfRange = 0x80000000u;     // a buffer offset past every descriptor's end: such a load returns zeros

typedef __amdgpu_buffer_rsrc_t rows_rsrc_t;
__device__ __forceinline__ int rows_uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ rows_rsrc_t rows_rsrc(const void* p, unsigned bytes) {
  const unsigned long long v = (unsigned long long)p;
  const unsigned lo = rows_uni((int)(unsigned)v), hi = rows_uni((int)(unsigned)(v >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void*)(((unsigned long long)hi << 32) | lo), 0, rows_uni((int)bytes), 0x00020000);
}
template <class V>
__device__ __forceinline__ V rows_load16(rows_rsrc_t r, unsigned lane_bytes, unsigned uniform_bytes) {
  return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_bytes, (int)uniform_bytes, 0));
}

// Where the fragments of the groups of 32 output channels lie: `group` bytes apart, the two tiles of a k-step next to each
// other and the k-steps `step` bytes apart.
struct RowsWeights { unsigned group, step; };

// One call (or one chunk of images of it), by value into every kernel.
struct RowsArgs {
  Geom g;
  int px0, npx;            // pixels [px0, px0 + npx) of the map are this chunk's; y1, y2 and `need` are relative to px0
  int ks1, ksm;            // 32-deep k-steps of the C and the M channels
  int pairs1, pairs3;      // groups of 32 output channels of conv1 / conv2, and of conv3
  const int32_t* idx;      // nullptr: every cell
  const int32_t* count;
  const uint8_t* need;     // nullptr: every pixel
  unsigned w1_bytes, w2_bytes, w3_bytes;    // as they lie in memory: packed, or in a direct call the caller's
  RowsWeights w1, w2, w3;                   // (packed)
  Div31 cpi, gw, s2, s;    // cells per image and per row of cells, S*S, S
  int conv_blocks;         // conv1 in a direct call: workgroups that are the convolution's; the others copy x to out
};

// The active list as rows: row r is pixel (r mod S*S) of entry r / (S*S).
__device__ __forceinline__ int rows_active(const RowsArgs& a) {
  return rows_uni(a.idx ? max(min(*a.count, a.g.P), 0) : a.g.P) * (a.g.S * a.g.S);     // (P * S * S < 2^31)
}
// Its pixel, or -1: past the end of the list, not a cell of the map, or not of this chunk.  The entry is read beside the count, not after
// it (row_cell comes before rows_active; the list has storage for every cell of the map).
struct RowPixel { int px, h, w; };
__device__ __forceinline__ int row_cell(const RowsArgs& a, int r) {
  const int e = div31_by(r, a.s2);
  return e < a.g.P ? (a.idx ? a.idx[e] : e) : -1;
}
__device__ __forceinline__ RowPixel row_pixel(const RowsArgs& a, int cell, int r, int nrows) {
  RowPixel p{-1, 0, 0};
  if (r >= nrows || (unsigned)cell >= (unsigned)a.g.P) return p;
  const int S = a.g.S, q = r - div31_by(r, a.s2) * (S * S);
  const int n = div31_by(cell, a.cpi), rem = cell - n * (a.g.G * a.g.GW), gy = div31_by(rem, a.gw), gx = rem - gy * a.g.GW;
  const int qy = div31_by(q, a.s);
  p.h = gy * S + qy;
  p.w = gx * S + q - qy * S;
  const int px = (n * a.g.H + p.h) * a.g.W + p.w;
  if (px >= a.px0 && px < a.px0 + a.npx) p.px = px;
  return p;
}

// ---- number formats -----------------------------------------------------------------------------------
// KPL pieces of 16 bytes a lane holds of one 32-deep fragment; YP terms a y value is stored as.  Lane (i = lane % 16,
// lg = lane / 16) holds row i, and the k of its piece h, element e are 16*h + 4*lg + e (fp32) or 8*lg + e
// (bf16), for A and B alike: one load instruction then reads 64 contiguous bytes of each of 16 rows.
struct Fp32 {
  typedef float T;
  typedef floatx4 V;
  static constexpr int ES = 4, KPL = 2, XP = 1, YP = 1, EPP = 4;     // EPP: elements per piece
  static constexpr int STEP = 128;                                   // bytes of a 32-deep k-step of one row
  struct Frag { V v[KPL]; };
  static __device__ __forceinline__ void mma(floatx4& acc, const Frag& a, const Frag& b, int h, int e) {
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[h][e], b.v[h][e], acc, 0, 0, 0);
  }
  static constexpr int SUB = 4;                                      // MFMAs per piece
};
struct Bf16Wide {
  typedef uint16_t T;
  typedef bf16x8 V;
  static constexpr int ES = 2, KPL = 1, XP = 1, YP = 3, EPP = 8;
  static constexpr int STEP = 64;
  struct Frag { V v[KPL]; };
  static __device__ __forceinline__ void mma(floatx4& acc, const Frag& a, const Frag& b, int, int) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v[0], b.v[0], acc, 0, 0, 0);
  }
  static constexpr int SUB = 1;
};

__device__ __forceinline__ float rows_widen(float v) { return v; }
__device__ __forceinline__ float rows_widen(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }

// Channel of a lane's accumulator element: tiles 0 and 1 of a group of 32 channels give lane group lg the 8 consecutive
// channels 8*lg .. 8*lg+7 (tile j: + 4*j + v), so that a lane stores whole 16-byte pieces.
__device__ __forceinline__ int rows_channel(int pair, int lg) { return pair * 32 + lg * 8; }

// y rows: YP terms of [ksm * 32] elements each.
template <class F>
__device__ __host__ __forceinline__ unsigned y_pitch(int ksm) { return (unsigned)ksm * 32 * F::ES * F::YP; }

template <class F>
__device__ __forceinline__ void store_y(unsigned char* row, int ch, int ksm, const float (&v)[8]);
template <>
__device__ __forceinline__ void store_y<Fp32>(unsigned char* row, int ch, int, const float (&v)[8]) {
  floatx4* p = reinterpret_cast<floatx4*>(row + ch * 4);
  p[0] = floatx4{v[0], v[1], v[2], v[3]};
  p[1] = floatx4{v[4], v[5], v[6], v[7]};
}
template <>
__device__ __forceinline__ void store_y<Bf16Wide>(unsigned char* row, int ch, int ksm, const float (&v)[8]) {
  bf16x8 t[3];
#pragma unroll
  for (int i = 0; i < 8; ++i) {                  // v = t0 + t1 + t2, v >= 0: each term takes the next 8 significant bits
    // Truncated, so that no term is negative, and no term of a v > 0 is zero (the smallest normal number stands in, 30
    // decimal places below what fp32 resolves of ordinary values): an infinite weight then gives an infinity, as it
    // does with v itself, and not the NaN of 0 * inf or of inf - inf.
    float r = v[i];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float top = __uint_as_float(__float_as_uint(r) & 0xffff0000u);
      t[k][i] = (__bf16)(k > 0 && v[i] > 0.f ? fmaxf(top, 0x1p-126f) : top);
      r = __builtin_isfinite(r) ? r - top : 0.f;            // (an infinite y stays one)
    }
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) *reinterpret_cast<bf16x8*>(row + (k * ksm * 32 + ch) * 2) = t[k];
}

// ---- weights ------------------------------------------------------------------------------------------
// One group of 32 output channels (`pair`) of a convolution with nch of them, K channels in per tap and kpt k-steps per tap.
// Packed by the plan: the fragments of a k-step are consecutive KiB.
struct plan_weights {
  static constexpr bool direct = false;
  rows_rsrc_t rs;
  unsigned lane16, base, step;
  template <class F>
  __device__ __forceinline__ void open(const unsigned char* wp, unsigned bytes, RowsWeights w, int pair, int, int, int, int, int lane) {
    rs = rows_rsrc(wp, bytes);
    lane16 = lane * 16;
    base = pair * w.group;
    step = w.step;
  }
  template <class F>
  __device__ __forceinline__ void load(typename F::Frag (&a)[2], int s) {
    const unsigned so = base + (unsigned)s * step;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int h = 0; h < F::KPL; ++h) a[j].v[h] = rows_load16<typename F::V>(rs, lane16 + (j * F::KPL + h) * 1024, so);
  }
};
// The caller's, [nch][taps][K]: a lane reads its 16-byte pieces of its channel's row, zeros past the last channel and past K.
struct call_weights {
  static constexpr bool direct = true;
  rows_rsrc_t rs;
  unsigned off[2];
  int K, kpt, lg, at, in_tap, tap;         // (k-steps are asked for in order, as by YRows)
  template <class F>
  __device__ __forceinline__ void open(const unsigned char* wp, unsigned bytes, RowsWeights, int pair, int nch, int k, int ksteps, int s0,
                                       int lane) {
    rs = rows_rsrc(wp, bytes);
    K = k;
    kpt = ksteps;
    lg = lane >> 4;
    const unsigned pitch = bytes / (unsigned)nch;
    const int ch = pair * 32 + ((lane & 15) >> 2) * 8 + (lane & 3);
#pragma unroll
    for (int j = 0; j < 2; ++j) off[j] = ch + j * 4 < nch ? (unsigned)(ch + j * 4) * pitch : kOutOfRange;
    at = s0;
    tap = s0 / kpt;
    in_tap = s0 - tap * kpt;
  }
  template <class F>
  __device__ __forceinline__ void load(typename F::Frag (&a)[2], int s) {
    if (s != at) {
      at = s;
      if (++in_tap == kpt) {
        in_tap = 0;
        ++tap;
      }
    }
#pragma unroll
    for (int h = 0; h < F::KPL; ++h) {
      const int k = in_tap * 32 + h * 16 * (F::KPL - 1) + lg * F::EPP;
#pragma unroll
      for (int j = 0; j < 2; ++j)
        a[j].v[h] = rows_load16<typename F::V>(rs, k < K ? off[j] + (unsigned)(tap * K + k) * F::ES : kOutOfRange, 0);
    }
  }
};

// Calls f(integral_constant<j>) for j = 0 .. N-1.
template <int N, int J = 0, class Fn>
__device__ __forceinline__ void rows_each(Fn&& f) {
  if constexpr (J < N) {
    f(std::integral_constant<int, J>{});
    rows_each<N, J + 1>(static_cast<Fn&&>(f));
  }
}
// Calls f(integral_constant<n>) for the run-time n in [LO, HI].
template <int LO, int HI, class Fn>
__device__ __forceinline__ void rows_count(int n, Fn&& f) {
  if constexpr (LO == HI) f(std::integral_constant<int, LO>{});
  else if (n == LO) f(std::integral_constant<int, LO>{});
  else rows_count<LO + 1, HI>(n, static_cast<Fn&&>(f));
}

// ---- the wave's ring of rows ------------------------------------------------------------------------------
// A wave's B rows come through LDS of its own: the next D k-steps are requested by direct loads that nobody but the wave waits for.
// What it saves is lookups: a CU's L1 takes the addresses of four lanes at a time, and in a fragment's lanes (lane % 16 the row) those are
// four rows', so a load of 1 KiB costs 64 lookups.  Here four lanes in a row load one row's 64 bytes: 16 lookups, as for the weights, and
// the fragment's lanes find their pieces in LDS.  (fp32, per k-step and wave, one row block: 192 of them against 512 clocks of MFMAs,
// and there are four waves to a CU's L1; now 96.)  Four row blocks would take 64 KiB (fp32) or 96 (bf16) of LDS for two k-steps and need the fewest lookups
// to begin with, 576 per 2048 clocks: they read straight into registers.
// The compiler does not count these loads, so where the MFMAs of a k-step wait for its weights it leaves (D-1) * NA operations outstanding
// and not (D-1) * (NA + NL): by then the next k-step's rows have landed too (in bf16's conv2 and conv3, one block, a third of those after it as well).  So
// of the D k-steps' distance a row has D-1 in the steady loop, the depths below were measured with that, and the ring's own counts decide only what a reduction's
// first k-step and its ends read.
// Piece lg of row i lies at place i*4 + (lg ^ i/4): the 16 rows that are read together are in different banks.
// Call sequences, rows straight into registers / through LDS, us: fp32 14x14x1024, S=2, 16 images, r=0.1 55.4 / 54.8, r=0.5 79.4 / 74.2, r=0.9
// 100.9 / 91.0, static block 107.5 / 97.3; 28x28x512, S=4, 16 images 88.0 / 80.9; 56x56x256, S=4, 4 images 43.1 / 40.7, 12 images (four blocks)
// 85.9 / 85.5; 7x7x2048, 16 images 90.1 / 79.8; bf16 28x20x192, mid 48, S=4, 13 images 27.2 / 24.8, r=1 33.8 / 30.2; 40x40x192, 40
// images 92.9 / 86.8; 32x32x96, mid 24, 2 images 19.7 / 19.1.  Rings of 4 k-steps and 2 (one block): 75.0 and 79.8 where 3 take 73.3.
constexpr bool rows_through_lds(int nb) { return nb <= 2; }
constexpr int rows_depth(int nb, int pl) { return nb == 1 ? 3 : nb == 2 ? (pl == 3 ? 2 : 3) : 2; }
template <class F>
constexpr int rows_ring_bytes(int nb, int pl) {              // of one wave, for up to nb row blocks
  const int one = rows_depth(1, pl) * pl * F::KPL * 1024, two = rows_depth(2, pl) * 2 * pl * F::KPL * 1024;
  return nb == 1 || one > two ? one : two;
}
__device__ __forceinline__ int ring_row(int lane) { return lane >> 2; }                        // what lane loads
__device__ __forceinline__ int ring_piece(int lane) { return (lane & 3) ^ (lane >> 4); }
__device__ __forceinline__ int ring_place(int l16, int lg) { return l16 * 4 + (lg ^ (l16 >> 2)); }

// 64 x 16 bytes from base + the lanes' offsets to 1 KiB of LDS.  (asm: the compiler must not know that it writes LDS, or it waits for
// everything before each read.)
__device__ __forceinline__ void ring_load(const unsigned char* base, unsigned off, unsigned to) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(to) : "memory");
}
// All but the youngest VM of the wave's memory operations have ended.  (With LASNET_DRAIN_AT_BARRIERS all have: the check build.)
template <int VM>
__device__ __forceinline__ void ring_wait() {
  static_assert(VM >= 0 && VM < 64, "vmcnt is 6 bits");
  __builtin_amdgcn_sched_barrier(0);
#ifdef LASNET_DRAIN_AT_BARRIERS
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#else
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(VM) : "memory");
#endif
  __builtin_amdgcn_sched_barrier(0);
}

// ---- the GEMM of one wave: NB blocks of 16 rows x one group of 32 channels ------------------------------
// k-steps [s0, s1).  A fragments by `weights`, B rows by `rows`; RING: through the wave's ring, else into registers.  `meanwhile` runs once
// the first loads have gone out (what it loads only makes the waits for them longer).
struct RowsNothing {
  __device__ __forceinline__ void operator()() const {}
};
template <class F, int NB, int PL, bool RING, class Weights, class Rows, class Meanwhile = RowsNothing>
__device__ __forceinline__ void rows_gemm(floatx4 (&acc)[NB][2], Weights& weights, Rows& rows, int s0, int s1, ROWS_LDS unsigned char* ring,
                                          int lane, Meanwhile meanwhile = Meanwhile{}) {
  using Frag = typename F::Frag;
  constexpr int D = RING ? rows_depth(NB, PL) : 2;
  constexpr int NA = 2 * F::KPL, NL = NB * PL * F::KPL;      // a k-step's loads of weights and of rows
  Frag a[D][2], b[RING ? 1 : D][NB][PL];
  const unsigned ring0 = (unsigned)rows_uni((int)(unsigned)(size_t)ring);
  const int mine = ring_place(lane & 15, lane >> 4) * 16;
  auto load = [&](int d, int s) {
    if constexpr (RING) {
      // the place's last k-step has been read: not only its reads requested, which a load that finds its rows in L1 could overtake
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      rows.template direct<F, NB, PL>(ring0 + d * NL * 1024, s);
      __builtin_amdgcn_sched_barrier(0);         // (before the weights: the waits are counted so)
    }
    weights.template load<F>(a[d], s);
    if constexpr (!RING) rows.template load<F, NB, PL>(b[d], s);
  };
  auto read = [&](int d, int p, int h) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
      b[0][i][p].v[h] = *reinterpret_cast<const ROWS_LDS typename F::V*>(ring + (d * NL + (p * NB + i) * F::KPL + h) * 1024 + mine);
  };
  // k-step d of the ring, behind which `after` k-steps have been requested.  (Reading each fragment of the next one into the registers that
  // the MFMAs have just left: 1 to 2 % faster for a few images, as much slower for more, whose SIMDs then hold a wave less.)
  auto compute = [&](int d, auto after) {
    if constexpr (RING) {
      ring_wait<NA + decltype(after)::value * (NA + NL)>();
#pragma unroll
      for (int p = 0; p < PL; ++p)
#pragma unroll
        for (int h = 0; h < F::KPL; ++h) read(d, p, h);
    }
    Frag(&bd)[NB][PL] = b[RING ? 0 : d];
#pragma unroll
    for (int p = 0; p < PL; ++p)
#pragma unroll
      for (int h = 0; h < F::KPL; ++h)
#pragma unroll
        for (int e = 0; e < F::SUB; ++e)
#pragma unroll
          for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) F::mma(acc[i][j], a[d][j], bd[i][p], h, e);
  };
  typedef std::integral_constant<int, D - 1> All;
  if constexpr (NB == 4) {
    // (256 registers do not hold four blocks beside the ends below: past the end the last step is requested again, unused)
#pragma unroll
    for (int d = 0; d < D; ++d) load(d, min(s0 + d, s1 - 1));
    meanwhile();
    int s = s0;
    for (; s + D <= s1; s += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        compute(d, All{});
        load(d, min(s + D + d, s1 - 1));
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
      if (s + d < s1) compute(d, All{});
    return;
  }
  // Nothing is requested past the end (a CU's L1 is near its rate, and what is loaded to fill a round up delays what follows it): the
  // steady loop leaves 1 to 2D-1 k-steps, whose number is a constant in each of as many straight-line ends.  Against a ring that is
  // filled up with repeats of the last step (2 of 10 k-steps where four waves share 36), call sequences, us: bf16 28x20x192, mid 48, S=4, 13 images
  // 29.6 -> 27.0, r=1 38.3 -> 33.3; fp32 56x56x256, S=4, 4 images 46.3 -> 43.3; 14x14x1024, S=2, 16 images 82.8 -> 79.7; 28x28x512, S=4,
  // r=0.9, 16 images 115.5 -> 112.1.
  int s = s0;
  auto end = [&](auto left) {
    constexpr int L = decltype(left)::value;
    if constexpr (L < D) {                       // (the whole reduction: nothing has been requested yet)
#pragma unroll
      for (int d = 0; d < L; ++d) {
        load(d, s + d);
        __builtin_amdgcn_sched_barrier(0);
      }
      meanwhile();
      __builtin_amdgcn_sched_barrier(0);
    }
    rows_each<L>([&](auto j) {                   // step j of those left: the steps up to j + D have been requested
      constexpr int J = decltype(j)::value;
      compute(J % D, std::integral_constant<int, (J + D < L ? J + D : L) - 1 - J>{});
      if constexpr (J + D < L) load(J % D, s + D + J);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  if (s1 - s0 >= D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      load(d, s + d);
      __builtin_amdgcn_sched_barrier(0);         // (in the loop's order: what it waits for is counted)
    }
    meanwhile();
    __builtin_amdgcn_sched_barrier(0);
    for (; s + 2 * D <= s1; s += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        compute(d, All{});
        load(d, s + D + d);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  rows_count<1, 2 * D - 1>(s1 - s, end);
}

// B rows of conv1: pixels of x.  VEC: 16-byte pieces (C and the pointers allow them), else element by element; the
// pieces past channel C are zeros (the next pixel's values, which may be anything, must not meet the zero weights).
template <bool VEC>
struct XRows {
  rows_rsrc_t rs;
  unsigned off[4];         // byte offset of the lane's row in the chunk, kOutOfRange for rows that do not exist
  int C, lg;
  const unsigned char* base;             // for direct(): the chunk's first pixel; off is of the row and piece that the lane loads there
  // (rows that do not exist are some row that does, and C is a whole number of k-steps)
  template <class F, int NB, int PL>
  __device__ __forceinline__ void direct(unsigned to, int s) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int h = 0; h < F::KPL; ++h) ring_load(base + (unsigned)(s * F::STEP + h * 64), off[i], to + (i * F::KPL + h) * 1024);
  }
  template <class F, int NB, int PL>
  __device__ __forceinline__ void load(typename F::Frag (&b)[NB][PL], int s) {
    static_assert(PL == 1, "x is one term");
#pragma unroll
    for (int h = 0; h < F::KPL; ++h) {
      const int k = s * 32 + h * 16 * (F::KPL - 1) + lg * F::EPP;    // first channel of the lane's piece
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        if constexpr (VEC) {
          b[i][0].v[h] = rows_load16<typename F::V>(rs, k < C ? off[i] + (unsigned)k * F::ES : kOutOfRange, 0);
        } else {
#pragma unroll
          for (int e = 0; e < F::EPP; ++e) {
            const unsigned o = k + e < C ? off[i] + (unsigned)(k + e) * F::ES : kOutOfRange;
            if constexpr (F::ES == 4)
              b[i][0].v[h][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)o, 0, 0));
            else
              b[i][0].v[h][e] = __builtin_bit_cast(__bf16, (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, (int)o, 0, 0));
          }
        }
      }
    }
  }
};

// B rows of conv3: the row's own y2; of conv2: y1 of the pixel that tap s / ksm names, zeros outside the image.  RING: by direct(), then
// px, h and w are of the row that the lane loads, and outside the image, where a buffer load gives zeros, is y1's row of zeros.
template <bool TAPS, bool RING>
struct YRows {
  rows_rsrc_t rs;
  const unsigned char* base;
  unsigned outside;
  unsigned off[4];         // TAPS: of the current tap
  unsigned pitch;
  int ksm, lg;
  int px[4], h[4], w[4], H, W;
  int at, in_tap, tap;     // the k-step last loaded = tap * ksm + in_tap (k-steps are asked for in order)
  __device__ __forceinline__ void set_tap(int nb) {
    const int dy = tap / 3 - 1, dx = tap - tap / 3 * 3 - 1;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < nb) {
        const bool in = px[i] >= 0 && (unsigned)(h[i] + dy) < (unsigned)H && (unsigned)(w[i] + dx) < (unsigned)W;
        off[i] = in ? (unsigned)(px[i] + dy * W + dx) * pitch + lg * 16 : outside;
      }
  }
  // (to the k-step after the last one, or the last one again: its place within the tap)
  __device__ __forceinline__ int advance(int s, int nb) {
    if constexpr (!TAPS) return s;
    if (s != at) {
      at = s;
      if (++in_tap == ksm) {
        in_tap = 0;
        ++tap;
        set_tap(nb);
      }
    }
    return in_tap;
  }
  template <class F, int NB, int PL>
  __device__ __forceinline__ void direct(unsigned to, int s) {
    const int so = advance(s, NB);
#pragma unroll
    for (int p = 0; p < PL; ++p)
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int h2 = 0; h2 < F::KPL; ++h2)
          ring_load(base + (unsigned)(so * F::STEP + p * ksm * F::STEP + h2 * 64), off[i], to + ((p * NB + i) * F::KPL + h2) * 1024);
  }
  __device__ __forceinline__ void seek(int s, int nb) {
    at = s;
    tap = s / ksm;
    in_tap = s - tap * ksm;
    set_tap(nb);
  }
  template <class F, int NB, int PL>
  __device__ __forceinline__ void load(typename F::Frag (&b)[NB][PL], int s) {
    const int so = advance(s, NB);
#pragma unroll
    for (int p = 0; p < PL; ++p)
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int h2 = 0; h2 < F::KPL; ++h2)
          b[i][p].v[h2] = rows_load16<typename F::V>(rs, off[i], (unsigned)(so * F::STEP + p * ksm * F::STEP + h2 * 64));
  }
};

// Biases of a lane's 8 channels (zeros past n), as the accumulators' start.
template <int NB>
__device__ __forceinline__ void start_at_bias(floatx4 (&acc)[NB][2], const float* bias, int n, int ch, bool mine) {
  const rows_rsrc_t rs = rows_rsrc(bias, (unsigned)n * 4);
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float b = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, mine ? (ch + j * 4 + v) * 4 : (int)kOutOfRange, 0, 0));
#pragma unroll
      for (int i = 0; i < NB; ++i) acc[i][j][v] = b;
    }
}

// Adds the partial sums of the KS waves that share a tile, in the order of the waves; wave k is left with the row
// blocks i = k, k + KS, ..
template <int NB, int KS>
__device__ __forceinline__ void reduce_over_waves(floatx4 (&acc)[NB][2], ROWS_LDS float* part, int wave, int lane) {
  if constexpr (KS > 1) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        *reinterpret_cast<ROWS_LDS floatx4*>(part + (((wave * NB + i) * 2 + j) * 64 + lane) * 4) = acc[i][j];
    __syncthreads();
    const int w0 = wave / KS * KS;
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if (i % KS == wave % KS)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          floatx4 t = *reinterpret_cast<ROWS_LDS floatx4*>(part + (((w0 * NB + i) * 2 + j) * 64 + lane) * 4);
#pragma unroll
          for (int k = 1; k < KS; ++k)
            t += *reinterpret_cast<ROWS_LDS floatx4*>(part + ((((w0 + k) * NB + i) * 2 + j) * 64 + lane) * 4);
          acc[i][j] = t;
        }
    __syncthreads();
  }
}

// Calls f(integral_constant<n>) for the run-time n in [1, HI] (2 and 3 blocks share an instantiation of 4's size class).
template <int HI, class Fn>
__device__ __forceinline__ void rows_blocks(int n, Fn&& f) {
  if constexpr (HI == 1) {
    f(std::integral_constant<int, 1>{});
  } else {
    if (n <= HI / 2) rows_blocks<HI / 2>(n, static_cast<Fn&&>(f));
    else f(std::integral_constant<int, HI>{});
  }
}

// ---- calls with few cells --------------------------------------------------------------------------------
// What bounds them is their launches, 2 to 5 us each of a chain of dependent kernels.  So the copy of x to out, where there is one, has
// no launch of its own but a part of the next one's workgroups; and where the weights are small too (direct_is_faster) there is
// no plan: the convolutions read the caller's weights, and a workgroup of conv1 finds the needed pixels of its own run by
// going through the list itself.  Call sequences (rows straight into registers; through LDS each is 3 to 4 us shorter), us: fp32 56x56x256, S=4, r=0.6, one image (copy with the plan) 31.0 -> 29.0; bf16
// 28x20x192, mid 48, S=4, 13 images (no plan) 30.9 -> 28.4; bf16 20x20x320, mid 80, S=2, one image (neither) 31.6 -> 25.7.
constexpr int kDirectCells = 512;

// Workgroup `block` of `blocks` that copy the whole map (16-byte pieces).
template <class F>
__device__ __forceinline__ void rows_copy(const RowsArgs& a, int block, int blocks, const typename F::T* __restrict__ from,
                                          typename F::T* __restrict__ to) {
  const size_t n = (size_t)a.g.N * a.g.H * a.g.W * a.g.C * F::ES / 16, step = (size_t)blocks * kRowsThreads;
  for (size_t i = (size_t)block * kRowsThreads + threadIdx.x; i < n; i += step)
    reinterpret_cast<uint4*>(to)[i] = reinterpret_cast<const uint4*>(from)[i];
}
// (four pieces per thread, to four workgroups per CU.  Up to 512 / 1024 / 2048 workgroups, a launch of its own, us: fp32 128 images of
// 14x14x2048, mid 64, S=7 264.2 / 254.4 / 263.8, 259.3; 14x14x4096 492.9 / 471.6 / 497.5, 488.1; 32 of 112x112x256, mid 24, S=28
// 555.9 / 535.6 / 563.2, 584.2; maps to 50 MB the same with any of the three, 2 to 18 % slower with a launch of its own.)
template <class F>
int rows_copy_blocks(const Geom& g) {
  const long long blocks = ((long long)g.N * g.H * g.W * g.C * F::ES / 16 + 4 * kRowsThreads - 1) / (4 * kRowsThreads);
  return (int)(blocks < 1024 ? blocks : 1024);
}

// Bit i: pixel p0 + i (i < n <= 64) lies in the window of an entry of the list.  Its entries are read together with the count (the
// list has storage for every cell).
__device__ __forceinline__ unsigned long long rows_near(const RowsArgs& a, int p0, int n, ROWS_LDS unsigned* near, int tid) {
  int cells[kDirectCells / kRowsThreads];
#pragma unroll
  for (int u = 0; u < kDirectCells / kRowsThreads; ++u) {
    const int e = tid + u * kRowsThreads;
    cells[u] = e < a.g.P ? a.idx[e] : -1;
  }
  if (tid < 2) near[tid] = 0;
  const int nact = rows_uni(*a.count), S = a.g.S, H = a.g.H, W = a.g.W;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kDirectCells / kRowsThreads; ++u) {
    const int cell = cells[u];
    if (tid + u * kRowsThreads >= nact || (unsigned)cell >= (unsigned)a.g.P) continue;
    const int img = div31_by(cell, a.cpi), rem = cell - img * (a.g.G * a.g.GW), gy = div31_by(rem, a.gw), gx = rem - gy * a.g.GW;
    const int h0 = max(gy * S - 1, 0), h1 = min(gy * S + S, H - 1), w0 = max(gx * S - 1, 0), w1 = min(gx * S + S, W - 1);
    const int base = img * H * W - p0;
    if (base + h1 * W + w1 < 0 || base + h0 * W + w0 >= n) continue;
    unsigned long long m = 0;
    for (int h = h0; h <= h1; ++h) {
      const int first = max(base + h * W + w0, 0), last = min(base + h * W + w1, n - 1);
      if (first <= last) m |= ((2ull << (last - first)) - 1) << first;
    }
    if ((unsigned)m) __hip_atomic_fetch_or(near, (unsigned)m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (m >> 32) __hip_atomic_fetch_or(near + 1, (unsigned)(m >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __syncthreads();
  return near[0] | (unsigned long long)near[1] << 32;
}

// ---- conv1 -----------------------------------------------------------------------------------------------
// (Three waves per SIMD where four row blocks come straight into registers: what hides their loads is other waves.  Call sequences, two / three, us:
// fp32 56x56x256, S=4, 12 images 94.7 / 85.8, 16 images r=0.1 67.2 / 64.3, r=0.5 118.7 / 110.3, r=1 157.8 / 149.8; 40x40x192, 32 images 108.9 / 102.8; bf16, which
// has them anyway, the same.)
template <class F, bool VEC, int NB, int KS, class Weights>
__global__ __launch_bounds__(kRowsThreads, VEC && NB == 4 ? 3 : 2) void rows_conv1_kernel(RowsArgs a, int nsl, const typename F::T* __restrict__ x,
                                                                     const unsigned char* __restrict__ wp,
                                                                     const float* __restrict__ b1,
                                                                     unsigned char* __restrict__ y1,
                                                                     typename F::T* __restrict__ copy_to) {
  if (Weights::direct && (int)blockIdx.x >= a.conv_blocks) {
    rows_copy<F>(a, (int)blockIdx.x - a.conv_blocks, (int)gridDim.x - a.conv_blocks, x, copy_to);
    return;
  }
  __shared__ int rowpx[NB * 16];
  __shared__ __attribute__((aligned(16))) float part[KS > 1 ? 4 * NB * 2 * 64 * 4 : 4];
  constexpr int RINGB = VEC && rows_through_lds(NB) ? rows_ring_bytes<F>(NB, F::XP) : 4;
  __shared__ __attribute__((aligned(1024))) unsigned char rings[4 * RINGB];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4, wave = rows_uni(tid >> 6);
  int unit, slice;
  if (!unit_and_slice((a.npx + NB * 16 - 1) / (NB * 16), nsl, unit, slice)) return;
  if (unit == 0 && slice == 0)                   // the row of zeros behind y1's last
    for (unsigned i = tid; i < y_pitch<F>(a.ksm) / 4; i += kRowsThreads)
      reinterpret_cast<unsigned*>(y1 + (size_t)a.npx * y_pitch<F>(a.ksm))[i] = 0;
  const int p0 = unit * NB * 16;
  // the needed pixels of this run, ascending
  static_assert(NB * 16 <= 64, "one ballot");
  bool on = lane < NB * 16 && p0 + lane < a.npx;
  if constexpr (Weights::direct) {
    __shared__ unsigned near[2];
    if (a.idx) {
      const unsigned long long needed = rows_near(a, p0, NB * 16, (ROWS_LDS unsigned*)near, tid);      // (by every thread)
      on = on && (needed >> lane & 1);
    }
  } else {
    on = on && (!a.need || a.need[p0 + lane] != 0);
  }
  const unsigned long long b = __ballot(on);
  const int U = __popcll(b);
  if (U == 0) return;                            // uniform over the workgroup
  if (wave == 0) {
    if (on) rowpx[__popcll(b & ((1ull << lane) - 1ull))] = p0 + lane;
    if (lane < NB * 16 && lane >= U) rowpx[lane] = -1;
  }
  __syncthreads();
  constexpr int WC = 4 / KS;
  rows_blocks<NB>((U + 15) >> 4, [&](auto nbc) {
    constexpr int N = decltype(nbc)::value;
    XRows<VEC> rows;
    rows.rs = rows_rsrc(x + (size_t)a.px0 * a.g.C, (unsigned)a.npx * a.g.C * F::ES);
    rows.base = (const unsigned char*)(x + (size_t)a.px0 * a.g.C);
    rows.C = a.g.C;
    rows.lg = lg;
    // (the next pixel's values must not meet the zero weights past channel C)
    constexpr bool MAY_RING = VEC && rows_through_lds(NB);     // (fewer blocks in a kernel of four read as its four do: its registers)
    const bool ring = MAY_RING && a.g.C % 32 == 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int px = rowpx[i * 16 + (ring ? ring_row(lane) : l16)];
      rows.off[i] = ring ? (unsigned)max(px, p0) * a.g.C * F::ES + ring_piece(lane) * 16 : px >= 0 ? (unsigned)px * a.g.C * F::ES : kOutOfRange;
    }
    const int kq = (a.ks1 + KS - 1) / KS, s0 = min(wave % KS * kq, a.ks1), s1 = min(s0 + kq, a.ks1);
    for (int pair = slice * WC + wave / KS; pair < (KS > 1 ? (a.pairs1 + WC - 1) / WC * WC : a.pairs1); pair += nsl * WC) {
      floatx4 acc[N][2];
      start_at_bias<N>(acc, b1, a.g.M, rows_channel(pair, lg), wave % KS == 0);
      if (s0 < s1 && pair < a.pairs1) {
        Weights weights;
        weights.template open<F>(wp, a.w1_bytes, a.w1, pair, a.g.M, a.g.C, a.ks1, s0, lane);
        ROWS_LDS unsigned char* mine = (ROWS_LDS unsigned char*)rings + wave * RINGB;
        if constexpr (MAY_RING) {
          if (ring) rows_gemm<F, N, F::XP, true>(acc, weights, rows, s0, s1, mine, lane);
          else rows_gemm<F, N, F::XP, false>(acc, weights, rows, s0, s1, mine, lane);
        } else {
          rows_gemm<F, N, F::XP, false>(acc, weights, rows, s0, s1, mine, lane);
        }
      }
      reduce_over_waves<N, KS>(acc, (ROWS_LDS float*)part, wave, lane);
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int px = rowpx[i * 16 + l16];
        if ((KS == 1 || i % KS == wave % KS) && pair < a.pairs1 && px >= 0) {
          float v[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) v[u] = fmaxf(acc[i][u / 4][u % 4], 0.f);
          store_y<F>(y1 + (size_t)px * y_pitch<F>(a.ksm), rows_channel(pair, lg), a.ksm, v);
        }
      }
    }
  });
}

// ---- conv2 -----------------------------------------------------------------------------------------------
template <class F, int NB, int KS, class Weights>
__global__ __launch_bounds__(kRowsThreads, 2) void rows_conv2_kernel(RowsArgs a, int nsl, const unsigned char* __restrict__ wp,
                                                                     const float* __restrict__ b2,
                                                                     const unsigned char* __restrict__ y1,
                                                                     unsigned char* __restrict__ y2) {
  __shared__ __attribute__((aligned(16))) float part[KS > 1 ? 4 * NB * 2 * 64 * 4 : 4];
  constexpr bool RING = rows_through_lds(NB);
  constexpr int RINGB = RING ? rows_ring_bytes<F>(NB, F::YP) : 4;
  __shared__ __attribute__((aligned(1024))) unsigned char rings[4 * RINGB];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4, wave = rows_uni(tid >> 6);
  int unit, slice, cell[NB];
  unit_and_slice(0, nsl, unit, slice);           // (a unit past the last has no rows)
  const int r0 = unit * NB * 16, rl = RING ? ring_row(lane) : l16;         // rl: row of a block that the lane loads
#pragma unroll
  for (int i = 0; i < NB; ++i) cell[i] = row_cell(a, r0 + i * 16 + rl);
  const int nrows = rows_active(a);
  if (r0 >= nrows) return;
  YRows<true, RING> rows;
  const unsigned pitch = y_pitch<F>(a.ksm);
  int px[NB];                                    // of the lane's row of the result
  bool any = false;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const RowPixel p = row_pixel(a, cell[i], r0 + i * 16 + rl, nrows);
    rows.px[i] = p.px < 0 ? -1 : p.px - a.px0;
    rows.h[i] = p.h;
    rows.w[i] = p.w;
    any |= p.px >= 0;
    px[i] = RING ? __shfl(rows.px[i], l16 * 4) : rows.px[i];
  }
  if (!__any(any)) return;                       // (the same rows in every wave)
  rows.rs = rows_rsrc(y1, (unsigned)a.npx * pitch);
  rows.base = y1;
  rows.pitch = pitch;
  rows.ksm = a.ksm;
  rows.lg = RING ? ring_piece(lane) : lg;
  rows.outside = RING ? (unsigned)a.npx * pitch + ring_piece(lane) * 16 : kOutOfRange;
  rows.H = a.g.H;
  rows.W = a.g.W;
  constexpr int WC = 4 / KS;
  const int total = 9 * a.ksm, kq = (total + KS - 1) / KS, s0 = min(wave % KS * kq, total), s1 = min(s0 + kq, total);
  for (int pair = slice * WC + wave / KS; pair < (KS > 1 ? (a.pairs1 + WC - 1) / WC * WC : a.pairs1); pair += nsl * WC) {
    floatx4 acc[NB][2];
    start_at_bias<NB>(acc, b2, a.g.M, rows_channel(pair, lg), wave % KS == 0);
    rows.seek(min(s0, total - 1), NB);
    if (s0 < s1 && pair < a.pairs1) {
      Weights weights;
      weights.template open<F>(wp, a.w2_bytes, a.w2, pair, a.g.M, a.g.M, a.ksm, s0, lane);
      rows_gemm<F, NB, F::YP, RING>(acc, weights, rows, s0, s1, (ROWS_LDS unsigned char*)rings + wave * RINGB, lane);
    }
    reduce_over_waves<NB, KS>(acc, (ROWS_LDS float*)part, wave, lane);
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if ((KS == 1 || i % KS == wave % KS) && pair < a.pairs1 && px[i] >= 0) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = fmaxf(acc[i][u / 4][u % 4], 0.f);
        store_y<F>(y2 + (size_t)px[i] * pitch, rows_channel(pair, lg), a.ksm, v);
      }
  }
}

// ---- conv3 + residual ------------------------------------------------------------------------------------
template <class F, bool VEC, int NB, int KS, class Weights>
__global__ __launch_bounds__(kRowsThreads, 2) void rows_conv3_kernel(RowsArgs a, int nsl, const typename F::T* __restrict__ x,
                                                                     const unsigned char* __restrict__ wp,
                                                                     const float* __restrict__ b3,
                                                                     const unsigned char* __restrict__ y2,
                                                                     typename F::T* __restrict__ out, int post_relu) {
  __shared__ __attribute__((aligned(16))) float part[KS > 1 ? 4 * NB * 2 * 64 * 4 : 4];
  typedef typename F::T T;
  constexpr bool RING = rows_through_lds(NB);
  constexpr int RINGB = RING ? rows_ring_bytes<F>(NB, F::YP) : 4;
  __shared__ __attribute__((aligned(1024))) unsigned char rings[4 * RINGB];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4, wave = rows_uni(tid >> 6);
  int unit, slice, cell[NB];
  unit_and_slice(0, nsl, unit, slice);           // (a unit past the last has no rows)
  const int r0 = unit * NB * 16;
#pragma unroll
  for (int i = 0; i < NB; ++i) cell[i] = row_cell(a, r0 + i * 16 + l16);
  const int nrows = rows_active(a);
  if (r0 >= nrows) return;
  YRows<false, RING> rows;
  const unsigned pitch = y_pitch<F>(a.ksm);
  int px[NB], some = -1;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    px[i] = row_pixel(a, cell[i], r0 + i * 16 + l16, nrows).px;
    some = max(some, px[i]);
  }
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) some = max(some, __shfl_xor(some, o, 16));
  if (some < 0) return;                          // (the same rows in every wave)
#pragma unroll
  for (int i = 0; i < NB; ++i)                   // (a row that does not exist loads one that does, unused)
    rows.off[i] = RING ? (unsigned)__shfl((px[i] < 0 ? some : px[i]) - a.px0, ring_row(lane)) * pitch + ring_piece(lane) * 16
                       : px[i] < 0 ? kOutOfRange : (unsigned)(px[i] - a.px0) * pitch + lg * 16;
  rows.base = y2;
  rows.rs = rows_rsrc(y2, (unsigned)a.npx * pitch);
  rows.ksm = a.ksm;
  rows.lg = lg;
  constexpr int WC = 4 / KS;
  const int C = a.g.C, kq = (a.ksm + KS - 1) / KS, s0 = min(wave % KS * kq, a.ksm), s1 = min(s0 + kq, a.ksm);
  for (int pair = slice * WC + wave / KS; pair < (KS > 1 ? (a.pairs3 + WC - 1) / WC * WC : a.pairs3); pair += nsl * WC) {
    floatx4 acc[NB][2];
    const int ch = rows_channel(pair, lg);
    start_at_bias<NB>(acc, b3, C, ch, wave % KS == 0);
    // The residual of the row blocks that this wave will store, requested behind the first k-steps (four blocks have no registers
    // for it): after the reduction it would be one more access to memory in the chain.
    typedef T Piece __attribute__((ext_vector_type(16 / F::ES)));
    constexpr int E = 16 / F::ES;
    constexpr bool EARLY = VEC && NB <= 2;
    Piece res[NB][8 / E];
    const auto request = [&] {
      if constexpr (EARLY) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int q = 0; q < 8 / E; ++q)        // (rows and channels that do not exist read x's first, unused)
            if (KS == 1 || i % KS == wave % KS)
              res[i][q] = reinterpret_cast<const Piece*>(x + (px[i] >= 0 && ch + q * E < C ? (size_t)px[i] * C + ch : 0))[px[i] >= 0 && ch + q * E < C ? q : 0];
      }
    };
    if (s0 < s1 && pair < a.pairs3) {
      Weights weights;
      weights.template open<F>(wp, a.w3_bytes, a.w3, pair, C, a.g.M, a.ksm, s0, lane);
      rows_gemm<F, NB, F::YP, RING>(acc, weights, rows, s0, s1, (ROWS_LDS unsigned char*)rings + wave * RINGB, lane, request);
    } else {
      request();
    }
    reduce_over_waves<NB, KS>(acc, (ROWS_LDS float*)part, wave, lane);
#pragma unroll
    for (int i = 0; i < NB; ++i)
      if ((KS == 1 || i % KS == wave % KS) && px[i] >= 0 && ch < C) {
        const T* xp = x + (size_t)px[i] * C + ch;
        T* op = out + (size_t)px[i] * C + ch;
        auto result = [&](int u, T xv) {
          float r = rows_widen(xv) + acc[i][u / 4][u % 4];
          if (post_relu) r = fmaxf(r, 0.f);
          if constexpr (F::ES == 4) return r;
          else return __builtin_bit_cast(uint16_t, (__bf16)r);
        };
        if constexpr (VEC) {                     // (C is then a whole number of the lane's 16-byte pieces)
#pragma unroll
          for (int q = 0; q < 8 / E; ++q)
            if (q == 0 || ch + q * E < C) {
              Piece xv;
              if constexpr (EARLY) xv = res[i][q];
              else xv = reinterpret_cast<const Piece*>(xp)[q];
              Piece o;
#pragma unroll
              for (int u = 0; u < E; ++u) o[u] = result(q * E + u, xv[u]);
              reinterpret_cast<Piece*>(op)[q] = o;
            }
        } else {
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (ch + u < C) op[u] = result(u, xp[u]);
        }
      }
  }
}

// ---- plan ------------------------------------------------------------------------------------------------
constexpr int kNeedPixels = 16384;                // pixels whose bytes one workgroup of the plan makes (in LDS)
// Every such workgroup scans the whole list, which is a launch less than clearing the bytes and scattering into them
// (1.3 us at a few hundred cells) but grows with pixels times cells: to this many cells of the map.  (64 images of
// 224x224x16, S=1, a list of 1.6 M entries: fp32 12.3 ms by scans, 1.9 ms scattered; bf16 14.9 and 1.8.  3136 cells: 29 and 21 us.)
constexpr int kScanCells = 1024;

// Blocks [0, pack_blocks): the weight fragments, one 8-element lane share per thread.  The next need_blocks: the need
// bytes of kNeedPixels pixels each, by a scan of the list (it may be in any order), or cleared for rows_need_kernel.  The others
// copy x to out.
template <class F>
__global__ __launch_bounds__(kRowsThreads) void rows_plan_kernel(RowsArgs a, int pack_blocks, int need_blocks, int scan,
                                                                 const typename F::T* __restrict__ x, typename F::T* __restrict__ out,
                                                                 const typename F::T* __restrict__ W1,
                                                                 const typename F::T* __restrict__ W2,
                                                                 const typename F::T* __restrict__ W3,
                                                                 unsigned char* __restrict__ wp, uint8_t* __restrict__ need) {
  typedef typename F::T T;
  const int tid = threadIdx.x, C = a.g.C, M = a.g.M;
  if ((int)blockIdx.x < pack_blocks) {
    const int n1 = a.pairs1 * a.ks1, n2 = a.pairs1 * 9 * a.ksm, n3 = a.pairs3 * a.ksm;   // k-steps of 2 tiles
    const int t = (int)blockIdx.x * kRowsThreads + tid;
    const int lane = t & 63, j = (t >> 6) & 1;
    int f = t >> 7;
    if (f >= n1 + n2 + n3) return;
    const int i = lane & 15, lg = lane >> 4;
    unsigned char* dst = wp + (size_t)(t >> 6) * (F::KPL * 1024) + lane * 16;
    const T* src;
    int rows, kmax, pair, k0;
    if (f < n1) {
      pair = f / a.ks1;
      k0 = (f - pair * a.ks1) * 32;
      src = W1; rows = M; kmax = C;
    } else if (f < n1 + n2) {
      f -= n1;
      pair = f / (9 * a.ksm);
      const int s = f - pair * 9 * a.ksm, tap = s / a.ksm;
      k0 = (s - tap * a.ksm) * 32;
      src = W2 + (size_t)tap * M; rows = M; kmax = M;
    } else {
      f -= n1 + n2;
      pair = f / a.ksm;
      k0 = (f - pair * a.ksm) * 32;
      src = W3; rows = C; kmax = M;
    }
    const size_t pitch = src == W1 ? (size_t)C : src == W3 ? (size_t)M : (size_t)9 * M;
    const int ch = rows_channel(pair, i >> 2) + j * 4 + (i & 3);
    const T* row = src + (size_t)ch * pitch;
#pragma unroll
    for (int h = 0; h < F::KPL; ++h) {
      T v[F::EPP];
#pragma unroll
      for (int e = 0; e < F::EPP; ++e) {
        const int k = k0 + h * 16 * (F::KPL - 1) + lg * F::EPP + e;
        v[e] = ch < rows && k < kmax ? row[k] : T(0);
      }
      typename F::V o;
      __builtin_memcpy(&o, v, 16);
      *reinterpret_cast<typename F::V*>(dst + h * 1024) = o;
    }
    return;
  }
  if ((int)blockIdx.x >= pack_blocks + need_blocks) {
    rows_copy<F>(a, (int)blockIdx.x - pack_blocks - need_blocks, (int)gridDim.x - pack_blocks - need_blocks, x, out);
    return;
  }
  __shared__ __attribute__((aligned(16))) uint8_t flag[kNeedPixels];
  const int q0 = ((int)blockIdx.x - pack_blocks) * kNeedPixels, nq = min(kNeedPixels, a.npx - q0);
  for (int i = tid; i < kNeedPixels / 16; i += kRowsThreads) reinterpret_cast<uint4*>(flag)[i] = uint4{0, 0, 0, 0};
  __syncthreads();
  const int nact = scan ? rows_uni(min(*a.count, a.g.P)) : 0, S = a.g.S, H = a.g.H, W = a.g.W, cpi = a.g.G * a.g.GW;
  for (int e = tid; e < nact; e += kRowsThreads) {
    const int cell = a.idx[e];
    if ((unsigned)cell >= (unsigned)a.g.P) continue;
    const int n = cell / cpi, rem = cell - n * cpi, gy = rem / a.g.GW, gx = rem - gy * a.g.GW;
    const int h0 = max(gy * S - 1, 0), h1 = min(gy * S + S, H - 1), w0 = max(gx * S - 1, 0), w1 = min(gx * S + S, W - 1);
    const int base = n * H * W - a.px0 - q0;     // of the image, relative to this workgroup's pixels
    if (base + h1 * W + w1 < 0 || base + h0 * W + w0 >= nq) continue;
    for (int h = h0; h <= h1; ++h)
      for (int w = w0; w <= w1; ++w)
        if ((unsigned)(base + h * W + w) < (unsigned)nq) flag[base + h * W + w] = 1;
  }
  __syncthreads();
  // (need has room for whole workgroups' pixels)
  for (int i = tid; i * 16 < nq; i += kRowsThreads) reinterpret_cast<uint4*>(need + q0)[i] = reinterpret_cast<uint4*>(flag)[i];
}

// The need bytes of a chunk (cleared by the plan) from a long list: one thread per row of an entry's window.
__global__ __launch_bounds__(kRowsThreads) void rows_need_kernel(RowsArgs a, uint8_t* __restrict__ need) {
  const int S = a.g.S, H = a.g.H, W = a.g.W, cpi = a.g.G * a.g.GW;
  const unsigned T = S + 2;
  const long long n = (long long)rows_uni(min(*a.count, a.g.P)) * T;
  for (long long i = (long long)blockIdx.x * kRowsThreads + threadIdx.x; i < n; i += (long long)gridDim.x * kRowsThreads) {
    const int e = (int)(i / T), cell = a.idx[e];
    if ((unsigned)cell >= (unsigned)a.g.P) continue;
    const int img = cell / cpi, rem = cell - img * cpi, gy = rem / a.g.GW, gx = rem - gy * a.g.GW;
    const int h = gy * S - 1 + (int)(i - (long long)e * T);
    if ((unsigned)h >= (unsigned)H) continue;
    const int w0 = max(gx * S - 1, 0), w1 = min(gx * S + S, W - 1), row = (img * H + h) * W - a.px0;
    for (int w = w0; w <= w1; ++w)
      if ((unsigned)(row + w) < (unsigned)a.npx) need[row + w] = 1;
  }
}

// ---- host ------------------------------------------------------------------------------------------------
// Bytes a chunk of images may take for y1 and y2: a larger batch runs chunk after chunk (at 256 MiB every ResNet-101
// stage at batch 128 is one chunk in fp32, and a chunk is thousands of row tiles, so nothing is lost by the cut).
constexpr size_t kRowsYBytes = (size_t)256 << 20;

struct RowsLayout {
  int images;                       // per chunk
  size_t w1, w2, w3, need, y, total; // bytes: packed weights, need bytes of a chunk, y1 (= y2) of a chunk
};
inline size_t rows_round(size_t v) { return (v + 255) / 256 * 256; }

// How a convolution is cut: NB row blocks per wave, KS waves to a tile's reduction, nsl channel slices per row tile.
// 1024 waves are one per SIMD.  More rows per wave read the weights less often, so NB is as large as leaves the chip
// that many tiles (NB = 2: `two`); with fewer even at NB = 1 the waves of a workgroup share a tile's reduction.
struct RowsCut { int nb, ks, units, nsl; };
inline RowsCut rows_cut(long long rows_max, long long rows_expected, int pairs, int ksteps, long long two = 1024) {
  RowsCut c;
  c.nb = 4;
  while (c.nb > 1 && (rows_expected + 16 * c.nb - 1) / (16 * c.nb) * pairs < (c.nb == 2 ? two : 1024)) c.nb /= 2;
  const long long tiles = (rows_expected + 16 * c.nb - 1) / (16 * c.nb);
  c.ks = c.nb == 1 && tiles * pairs < 1024 && ksteps >= 8 ? 4 : 1;
  c.units = (int)((rows_max + 16 * c.nb - 1) / (16 * c.nb));
  const int wc = 4 / c.ks, most = (pairs + wc - 1) / wc;
  c.nsl = (int)((1024 + tiles - 1) / tiles);
  if (c.nsl > most) c.nsl = most;
  return c;
}

// conv1, whose rows are known.  1200 to 2047 waves of one row block take as long as half as many of two -- some SIMDs have two of the former --
// and ask the L1 for 6 KiB of weights and rows (fp32, per two k-steps' MFMAs of a block) where two blocks share the weights.  Before the rows
// came through LDS two blocks were 3 to 5 % faster from this line on; now, call sequences, r=0.5 if not noted, one block / two, us, they are 0.2 to 0.4 faster at
// 14x14 and 0.2 slower at 7x7: bf16 14x14x1024, S=2, mid 200, 16 images 48.1 / 47.8, 17 48.7 / 48.3, 20 51.8 / 51.7, mid 224, 16 images 48.3 / 48.1; fp32 mid 256, 14
// images 70.6 / 70.3, 16 74.3 / 74.1, 16 at r=1 101.0 / 100.8, 20 76.5 / 76.4; 7x7x2048, 28 images 120.5 / 120.7.  Below it, down to 544 tiles, there is as little:
// fp32 11 images 68.3 / 68.2, 28x28x512, S=4, 8 images 51.1 / 50.7; and under 512 one is the faster: 14x14x1024, 10 images 53.2 / 59.1,
// 7x7x2048, 16 images 80.2 / 94.5, 20 79.9 / 93.9, 28x28x512, 5 images 38.4 / 41.3, 56x56x256, 4 images 40.7 / 43.8.
inline RowsCut rows_cut_conv1(long long pixels, long long chunk, int pairs, int ksteps) {
  const bool one_round = (chunk + 31) / 32 * ((pairs + 3) / 4) <= 256;
  return rows_cut(pixels, chunk, pairs, ksteps, ksteps >= 32 && one_round ? 600 : 1024);
}

// false: even one image does not fit (or exceeds the 32-bit offsets of the loads), or a launch would have 2^32 threads.
template <class F>
bool rows_layout(const Geom& g, RowsLayout& l) {
  const size_t pairs1 = (g.M + 31) / 32, pairs3 = (g.C + 31) / 32, ks1 = pairs3, ksm = pairs1;
  const size_t hw = (size_t)g.H * g.W, ypx = y_pitch<F>((int)ksm), xpx = (size_t)g.C * F::ES;
  l.w1 = pairs1 * ks1 * 2 * F::KPL * 1024;
  l.w2 = pairs1 * 9 * ksm * 2 * F::KPL * 1024;
  l.w3 = pairs3 * ksm * 2 * F::KPL * 1024;
  const size_t lim = (size_t)1 << 31;            // every descriptor stays below kOutOfRange
  if (hw * 2 * ypx > kRowsYBytes || hw * xpx >= lim || l.w1 >= lim || l.w2 >= lim || l.w3 >= lim) return false;
  size_t n = kRowsYBytes / (hw * 2 * ypx), nx = (lim - 1) / (hw * xpx);
  if (n > nx) n = nx;
  if (n > (size_t)g.N) n = (size_t)g.N;
  if (n == 0) return false;
  l.images = (int)n;
  const long long all = (long long)g.P * g.S * g.S, chunk = (long long)(n * hw);
  for (const RowsCut& c : {rows_cut_conv1(chunk, chunk, (int)pairs1, (int)ks1), rows_cut(all, (chunk + 1) / 2, (int)pairs1, 9 * (int)ksm),
                           rows_cut(all, chunk, (int)pairs1, 9 * (int)ksm), rows_cut(all, (chunk + 1) / 2, (int)pairs3, (int)ksm),
                           rows_cut(all, chunk, (int)pairs3, (int)ksm)})
    if (sliced_grid(c.units, c.nsl) * kRowsThreads >= 1ll << 32) return false;
  l.need = (n * hw + kNeedPixels - 1) / kNeedPixels * kNeedPixels;
  l.y = rows_round((n * hw + 1) * ypx);          // (a row of zeros behind the last)
  l.total = rows_round(l.w1) + rows_round(l.w2) + rows_round(l.w3) + l.need + 2 * l.y;
  return true;
}

// (several waves to a tile only with one row block: with more there are tiles enough)
#define ROWS_DISPATCH(c, CALL) \
  if (c.ks == 4) CALL(1, 4); else if (c.nb == 1) CALL(1, 1); else if (c.nb == 2) CALL(2, 1); else CALL(4, 1);

// The three convolutions of the chunk that `a` describes.
template <class F, bool VEC, class Weights>
hipError_t launch_rows_convs(RowsArgs a, int chunk, const void* x, const unsigned char* wp1, const unsigned char* wp2,
                             const unsigned char* wp3, const float* b1, const float* b2, const float* b3, unsigned char* y1,
                             unsigned char* y2, void* out, bool post_relu, bool copy, hipStream_t st) {
  typedef typename F::T T;
  const Geom& g = a.g;
  // the list's rows of this chunk are not known here: half of the pixels is a middling activation ratio
  // (and every chunk is cut like the full one, which rows_layout has checked)
  const long long rows = (long long)g.P * g.S * g.S, likely = a.idx ? (chunk + 1) / 2 : chunk;
  RowsCut c = rows_cut_conv1(a.npx, chunk, a.pairs1, a.ks1);
  long long grid = sliced_grid(c.units, c.nsl);
  a.conv_blocks = (int)grid;
  if (Weights::direct && copy) grid += rows_copy_blocks<F>(g);
#define ROWS_CONV1(NB, KS)                                                                                               \
  hipLaunchKernelGGL((rows_conv1_kernel<F, VEC, NB, KS, Weights>), dim3((unsigned)grid), dim3(kRowsThreads), 0, st, a, \
                     c.nsl, (const T*)x, wp1, b1, y1, (T*)out)
  ROWS_DISPATCH(c, ROWS_CONV1)
  c = rows_cut(rows, likely, a.pairs1, 9 * a.ksm);
#define ROWS_CONV2(NB, KS)                                                                                               \
  hipLaunchKernelGGL((rows_conv2_kernel<F, NB, KS, Weights>), dim3((unsigned)sliced_grid(c.units, c.nsl)), dim3(kRowsThreads), 0, st, a,      \
                     c.nsl, wp2, b2, y1, y2)
  ROWS_DISPATCH(c, ROWS_CONV2)
  c = rows_cut(rows, likely, a.pairs3, a.ksm);
#define ROWS_CONV3(NB, KS)                                                                                               \
  hipLaunchKernelGGL((rows_conv3_kernel<F, VEC, NB, KS, Weights>), dim3((unsigned)sliced_grid(c.units, c.nsl)), dim3(kRowsThreads), 0, st, a, \
                     c.nsl, (const T*)x, wp3, b3, y2, (T*)out, (int)post_relu)
  ROWS_DISPATCH(c, ROWS_CONV3)
#undef ROWS_CONV1
#undef ROWS_CONV2
#undef ROWS_CONV3
  return hipGetLastError();
}

}  // namespace
}  // namespace lasnet
