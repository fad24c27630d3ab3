// The slab schedule: the sparse bottleneck for a few images of a deep ResNet-101 stage (bf16), where the fused kernel
// leaves most of the chip idle -- it has a workgroup per run of patches, and each streams all weights through one
// CU, which takes 20 us whatever little there is to compute.  Three launches instead, each cut into (16 * NB rows of
// pixels) x (a few groups of 32 output channels) per workgroup, so that hundreds of CUs read a slice of the weights each:
//
//   conv1  rows = 16 * NB consecutive pixels of the whole map (it then depends on no list)     y1[pixel]
//   conv2  rows = the list's pixels, S*S per entry, in the list's order                        y2[pixel]
//   conv3  the same rows                                                                       out
//
// What bounds it is the chain of dependent memory accesses (~1 us each), so a workgroup makes as few as it can: the
// count, the list entries (requested together with the count: the list has storage for every cell) and its first
// weights at once; then its whole activation operand -- every row over the full reduction, conv2's with all nine
// taps -- as one burst of direct global->LDS loads; then the reduction from LDS, with weights D k-steps ahead in registers.
// The waves of a workgroup (NW) share the slab and take TJ tiles of 16 channels each: four waves with a group of 32 channels
// (TJ = 2) where there are many rows, four or two with half a group each where there are few.  A wave sums over the whole
// reduction, in the order of the fused and the tiled kernels: splitting it over the waves gave other bits than theirs (a relative
// 2.6e-4 of the output, from roundings of y1 and y2 that flip).
//
// Measured (the block's three launches on the GPU, against the schedule that ran before): 14x14x1024, S=2, one image 20.9 -> 10.6 us,
// 16 images 23.9 -> 17.4; S=7, 24 images 32.4 -> 24.4; 7x7x2048, one image 34 -> 19.3 us, 40 images 55 -> 33.  In conv2 the chain
// of accesses takes about 3 us; past that a CU streams its weights.
//
// Rounding points, order of the sums, weight layout (lasnet_pack_weights') and results are the fused kernel's, bit for bit.
#pragma once
#include "bottleneck_mfma.hpp"

namespace lasnet {
namespace {

struct SlabArgs {
  Geom g;
  const int32_t* idx;              // nullptr: every cell
  const int32_t* count;
  int npx, nsl;                    // pixels of the map; channel slices per row tile
  int ppt;                         // conv2: patches per workgroup
  int m_t2, m_t, m_s2, m_s;        // small_div's multipliers for (S+2)^2, S+2, S*S and S
};

__device__ __forceinline__ void slab_load(const AS_GLOBAL __bf16* src, AS_LDS __bf16* dst) {     // 64 x 16 bytes -> 1 KiB at dst
  const unsigned a = uni((int)(unsigned)(size_t)dst);
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(a) : "memory");
}
// Every load of every wave has landed in LDS.
__device__ __forceinline__ void slab_ready() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// One convolution's reduction: K channels per tap, TAPS taps, TJ tiles of output channels; D k-steps of weights in flight.
// The slab is rows of K channels whose 16-byte chunks are XOR-swizzled with the row's key, so that the 16 rows that a
// fragment read touches lie in different banks.
template <int K, int TAPS, int NB, int TJ, int D>
struct Slab {
  static constexpr int MS = K / 32, NST = TAPS * MS;
  static_assert(NST % D == 0, "whole rings");
  static constexpr int KEYS = K / 8 - 1 < 15 ? K / 8 - 1 : 15;
  bf16x8 w[D][TJ];

  __device__ __forceinline__ void fetch(rsrc_t wrs, int lane16, unsigned base, unsigned step, int slot, int s) {
#pragma unroll
    for (int j = 0; j < TJ; ++j) w[slot][j] = buf_load16(wrs, lane16 + j * 1024, (int)(base + (unsigned)s * step));
  }
  // the first D k-steps
  __device__ __forceinline__ void start(rsrc_t wrs, int lane16, unsigned base, unsigned step) {
#pragma unroll
    for (int d = 0; d < D; ++d) fetch(wrs, lane16, base, step, d, d);
  }
  // where(i, tap, row, key): slab row of the lane's row in block i
  template <class Where>
  __device__ __forceinline__ void run(floatx4 (&acc)[NB][TJ], rsrc_t wrs, int lane16, unsigned base, unsigned step,
                                      const AS_LDS __bf16* slab, int lg, Where&& where) {
    // One wave per SIMD issues an instruction every four clocks at best, and a k-step has as few as one MFMA of 16, so it may
    // hold little else: the swizzle flips bits 4 .. 7 of a chunk's byte offset, so four addresses per row (k-steps 0 .. 3 of
    // a tap) serve the others through the immediate offset.  (With the address worked out for every k-step, a k-step took 85 to
    // 100 clocks: 14x14x1024, S=2, one image 13.1 us; so 10.6.)
    const AS_LDS char* at[NB][4];
    int tap = 0;
    auto enter = [&] {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        int row, k;
        where(i, tap, row, k);
#pragma unroll
        for (int m = 0; m < 4; ++m)
          at[i][m] = reinterpret_cast<const AS_LDS char*>(slab) + row * (K * 2) + ((m * 64) ^ ((lg ^ (k & KEYS)) << 4));
      }
    };
    enter();
    // k-step s of the ring (s >= D: of the next one)
    static_assert(TAPS == 1 || D % MS == 0, "a tap begins at the same places of every ring");
    auto read = [&](bf16x8 (&b)[NB], int s) {
      if (TAPS > 1 && s > 0 && s % MS == 0) {
        ++tap;
        enter();
      }
      const int ms = TAPS > 1 ? s % MS : s;
#pragma unroll
      for (int i = 0; i < NB; ++i) b[i] = *reinterpret_cast<const AS_LDS bf16x8*>(at[i][ms & 3] + (ms >> 2) * 256);
    };
    // Fragments are read R - 1 k-steps ahead: with one or two waves per SIMD nothing else hides the LDS latency, which is
    // several k-steps' MFMAs.  (Rolled over whole rings of weights, or this would be tens of KB of code.)
    constexpr int R = NB * TJ <= 2 ? 8 : 4;
    static_assert(D % R == 0, "the fragment ring turns over with the weights' ring");
    bf16x8 b[R][NB];
#pragma unroll
    for (int d = 0; d < R - 1; ++d) read(b[d], d);
    auto ring = [&](int g, auto last) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        if (!last.value || d + R - 1 < D) read(b[(d + R - 1) % R], d + R - 1);
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int j = 0; j < TJ; ++j) acc[i][j] = mfma16(w[d][j], b[d % R][i], acc[i][j]);
        if (!last.value) fetch(wrs, lane16, base, step, d, g + d + D);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (TAPS == 1)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int m = 0; m < 4; ++m) at[i][m] += D * 64;
    };
#pragma nounroll
    for (int g = 0; g < NST - D; g += D) ring(g, std::false_type{});
    ring(NST - D, std::true_type{});
  }
};

// Lane -> (row of the piece, chunk position in it) for the 1 KiB pieces of a slab with K channels per row: RPI whole rows, or
// a part of one.
template <int K>
__device__ __forceinline__ void slab_piece(int piece, int lane, int& row, int& pos) {
  constexpr int CPR = K / 8;                     // 16-byte chunks per row
  static_assert(CPR % 64 == 0 || 64 % CPR == 0, "whole rows or whole pieces");
  if constexpr (CPR <= 64) {
    row = piece * (64 / CPR) + lane / CPR;
    pos = lane % CPR;
  } else {
    row = piece / (CPR / 64);
    pos = piece % (CPR / 64) * 64 + lane;
  }
}

// Weights in flight, in k-steps of TJ tiles: conv2's in whole taps.  2048x512, whose weights exceed an XCD's L2, has three
// times as many where a wave takes one tile (one image: 20.5 -> 19.3 us); at 1024x256 more measured the same or slower.
constexpr int conv1_ring(int c, int tj) { return tj == 2 ? 8 : c == 2048 ? 32 : 16; }
constexpr int conv2_ring(int m, int tj) { return m == 512 ? (tj == 2 ? 16 : 48) : tj == 2 ? 8 : 24; }

// Which group of 32 channels a wave works on, and the first of its tiles there.
template <int NW, int TJ>
struct SlabWave {
  static constexpr int WPP = 2 / TJ, PAIRS = NW / WPP;     // waves per group; groups per workgroup
  static_assert(NW % WPP == 0, "whole groups");
  int pair, ch;                                            // group; first channel of the lane's
  unsigned tile;                                           // byte offset of the wave's first tile in a k-step
  __device__ __forceinline__ SlabWave(int slice, int wave, int lg) {
    pair = slice * PAIRS + wave / WPP;
    tile = (unsigned)(wave % WPP) * 1024;
    ch = pair * 32 + lg * 8 + wave % WPP * 4;
  }
};

// The accumulators' start: the bias.
template <int NB, int TJ>
__device__ __forceinline__ void slab_bias(floatx4 (&acc)[NB][TJ], const float* b, int ch) {
#pragma unroll
  for (int j = 0; j < TJ; ++j) {
    floatx4 v;
    __builtin_memcpy(&v, b + ch + j * 4, 16);
#pragma unroll
    for (int i = 0; i < NB; ++i) acc[i][j] = v;
  }
}

// ReLU, bf16, the lane's 4 * TJ channels (tiles 0 and 1 of a group of 32 give lane group lg the channels 8*lg ..) as one store.
template <int TJ>
__device__ __forceinline__ void slab_store_y(__bf16* dst, const floatx4 (&t)[TJ]) {
  typedef __bf16 V __attribute__((ext_vector_type(4 * TJ)));
  V o;
#pragma unroll
  for (int u = 0; u < 4 * TJ; ++u) o[u] = (__bf16)fmaxf(t[u / 4][u % 4], 0.f);
  *reinterpret_cast<AS_GLOBAL V*>((AS_GLOBAL __bf16*)dst) = o;
}

// Cell e of the list: its image's first pixel and its own first row and column, or n < 0.  The entry is read together with
// the count, not after it (e < P keeps it inside the list's storage).
struct SlabCell { int n, h, w; };
__device__ __forceinline__ SlabCell slab_cell(const SlabArgs& a, int e) {
  SlabCell c{-1, 0, 0};
  if (e >= a.g.P) return c;
  const int cell = a.idx ? a.idx[e] : e;
  const int nact = a.idx ? min(*a.count, a.g.P) : a.g.P;
  if (e >= nact || (unsigned)cell >= (unsigned)a.g.P) return c;
  const int cpi = a.g.G * a.g.GW, n = cell / cpi, rem = cell - n * cpi, gy = rem / a.g.GW;
  c.n = n;
  c.h = gy * a.g.S;
  c.w = (rem - gy * a.g.GW) * a.g.S;
  return c;
}
// a / d for the small a of a slab (a * d < 2^16): a multiply and a shift, m = 65536 / d + 1
__device__ __forceinline__ int small_div(int a, int m) { return (a * m) >> 16; }

// ---- conv1 -----------------------------------------------------------------------------------------------
template <int C, int M, int NB, int NW, int TJ>
__global__ __launch_bounds__(NW * 64, NW / 2) void slab_conv1_kernel(SlabArgs a, const __bf16* __restrict__ x,
                                                                     const __bf16* __restrict__ wp, const float* __restrict__ b1,
                                                                     __bf16* __restrict__ y1) {
  using L = Slab<C, 1, NB, TJ, conv1_ring(C, TJ)>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  AS_LDS __bf16* slab = (AS_LDS __bf16*)smem;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4, wave = uni(tid >> 6);
  int unit, slice;
  if (!unit_and_slice((a.npx + NB * 16 - 1) / (NB * 16), a.nsl, unit, slice)) return;
  const int p0 = unit * NB * 16;
  // the lane reads the chunk that belongs at the position it writes
#pragma unroll
  for (int u = 0; u < NB * 32 * C / 1024 / NW; ++u) {
    int row, pos;
    slab_piece<C>(u * NW + wave, lane, row, pos);
    slab_load((const AS_GLOBAL __bf16*)x + (size_t)min(p0 + row, a.npx - 1) * C + ((pos ^ (row & L::KEYS)) << 3),
              slab + (u * NW + wave) * 512);
  }
  const SlabWave<NW, TJ> me(slice, wave, lg);
  const rsrc_t wrs = make_rsrc((g_bf16_p)wp, (unsigned)M * C * 2);
  const unsigned wbase = me.pair * 2048 + me.tile;
  L l;
  l.start(wrs, lane * 16, wbase, M * 64);
  floatx4 acc[NB][TJ];
  slab_bias<NB, TJ>(acc, b1, me.ch);
  slab_ready();
  l.run(acc, wrs, lane * 16, wbase, M * 64, slab, lg, [&](int i, int, int& row, int& key) { row = i * 16 + l16; key = l16; });
#pragma unroll
  for (int i = 0; i < NB; ++i)
    if (p0 + i * 16 + l16 < a.npx) slab_store_y<TJ>(y1 + (size_t)(p0 + i * 16 + l16) * M + me.ch, acc[i]);
}

// ---- conv2 -----------------------------------------------------------------------------------------------
// A workgroup takes a.ppt patches (a.ppt * S*S <= NB * 16 output rows); its slab is their (S+2)x(S+2) windows, one after
// the other, then an all-zero row for what lies outside the image.  Output row q of patch p reads window row
// (i + dy, j + dx): the key p*S*S + wy*S + wx of a window row makes that q + dy*S + dx, so the 16 rows of a
// block always have 16 different keys.
constexpr int kSlabMaxPatches = 64, kSlabMaxRows = 304;   // (304 rows of 256 channels, the zero row among them, are 152 KB)
// the all-zero row comes after whole 1 KiB pieces of window rows
template <int M>
__device__ __host__ __forceinline__ int slab_zero_row(int wrows) {
  constexpr int RPP = M * 2 < 1024 ? 1024 / (M * 2) : 1;
  return (wrows + RPP - 1) / RPP * RPP;
}
template <int M, int NB, int NW, int TJ>
__global__ __launch_bounds__(NW * 64, 1) void slab_conv2_kernel(SlabArgs a, const __bf16* __restrict__ wp,
                                                                     const float* __restrict__ b2, const __bf16* __restrict__ y1,
                                                                     __bf16* __restrict__ y2) {
  using L = Slab<M, 9, NB, TJ, conv2_ring(M, TJ)>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ int cells[kSlabMaxPatches * 4];
  __shared__ int source[kSlabMaxRows];           // of every window row: pixel | key << 27
  AS_LDS __bf16* slab = (AS_LDS __bf16*)smem;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4, wave = uni(tid >> 6);
  int unit, slice;
  unit_and_slice(0, a.nsl, unit, slice);       // (a unit past the last has no entries)
  const int S = a.g.S, T = S + 2, T2 = T * T, H = a.g.H, W = a.g.W, ppt = a.ppt, wrows = ppt * T2;
  const int zrow = slab_zero_row<M>(wrows);
  const SlabWave<NW, TJ> mine(slice, wave, lg);
  SlabCell me{-1, 0, 0};
  if (lane < ppt) me = slab_cell(a, unit * ppt + lane);
  if (!__any(me.n >= 0)) return;                 // (the same patches in every wave)
  if (wave == 0 && lane < ppt) {
    cells[lane * 4 + 0] = me.n < 0 ? -1 : me.n * H * W;
    cells[lane * 4 + 1] = me.h;
    cells[lane * 4 + 2] = me.w;
  }
  const rsrc_t wrs = make_rsrc((g_bf16_p)wp, (unsigned)M * M * 18);
  const unsigned wbase = mine.pair * 2048 + mine.tile;
  L l;
  l.start(wrs, lane * 16, wbase, M * 64);
  floatx4 acc[NB][TJ];
  slab_bias<NB, TJ>(acc, b2, mine.ch);
  for (int i = tid; i < M / 8; i += NW * 64)
    *reinterpret_cast<AS_LDS bf16x8*>(slab + zrow * M + i * 8) = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
  __syncthreads();
  // where every window row comes from: one that lies outside the image, or of a patch that does not exist, is loaded
  // from pixel 0 and never read (rows past the last fill up the last piece)
  for (int r = tid; r < zrow; r += NW * 64) {
    const int row = min(r, wrows - 1);
    const int p = small_div(row, a.m_t2), wpos = row - p * T2, wy = small_div(wpos, a.m_t), wx = wpos - wy * T;
    const int img = cells[p * 4], h = cells[p * 4 + 1] + wy - 1, w = cells[p * 4 + 2] + wx - 1;
    const bool in = img >= 0 && (unsigned)h < (unsigned)H && (unsigned)w < (unsigned)W;
    source[r] = (in ? img + h * W + w : 0) | ((p * S * S + wy * S + wx) & L::KEYS) << 27;
  }
  __syncthreads();
  // (four pieces' table entries are read at once: the loads then go out back to back)
  const int npiece = zrow * (M / 8) / 64;
  for (int first = wave; first < npiece; first += 4 * NW) {
    int src[4], pos[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      int row;
      slab_piece<M>(min(first + NW * k, npiece - 1), lane, row, pos[k]);
      src[k] = source[row];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (first + NW * k < npiece)
        slab_load((const AS_GLOBAL __bf16*)y1 + (size_t)(src[k] & 0x7ffffff) * M + ((pos[k] ^ (int)((unsigned)src[k] >> 27)) << 3),
                  slab + (first + NW * k) * 512);
  }
  int px[NB], ok[NB], row0[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int q = i * 16 + l16, p = small_div(q, a.m_s2), r = q - p * S * S, iy = small_div(r, a.m_s), ix = r - iy * S;
    const int img = p < ppt ? cells[p * 4] : -1;
    px[i] = -1;
    ok[i] = 0;
    row0[i] = p * T2 + iy * T + ix;
    if (img >= 0) {
      const int h = cells[p * 4 + 1] + iy, w = cells[p * 4 + 2] + ix;
      px[i] = img + h * W + w;
#pragma unroll
      for (int tap = 0; tap < 9; ++tap)
        ok[i] |= (unsigned)(h + tap / 3 - 1) < (unsigned)H && (unsigned)(w + tap % 3 - 1) < (unsigned)W ? 1 << tap : 0;
    }
  }
  slab_ready();
  l.run(acc, wrs, lane * 16, wbase, M * 64, slab, lg, [&](int i, int tap, int& row, int& key) {
    const int dy = tap / 3, dx = tap - dy * 3;
    const bool in = (ok[i] >> tap) & 1;
    row = in ? row0[i] + dy * T + dx : zrow;
    key = i * 16 + l16 + dy * S + dx;
  });
#pragma unroll
  for (int i = 0; i < NB; ++i)
    if (px[i] >= 0) slab_store_y<TJ>(y2 + (size_t)px[i] * M + mine.ch, acc[i]);
}

// ---- conv3 + residual ------------------------------------------------------------------------------------
// Rows are the list's pixels, S*S per entry.  (In place, out == x, is safe: a lane reads and writes the same elements.)
template <int C, int M, int NB>
__global__ __launch_bounds__(256, 2) void slab_conv3_kernel(SlabArgs a, const __bf16* x, const __bf16* __restrict__ wp,
                                                                     const float* __restrict__ b3, const __bf16* __restrict__ y2,
                                                                     __bf16* out, int post_relu) {
  using L = Slab<M, 1, NB, 2, 8>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ int rowpx[NB * 16];
  AS_LDS __bf16* slab = (AS_LDS __bf16*)smem;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4, wave = uni(tid >> 6);
  int unit, slice;
  unit_and_slice(0, a.nsl, unit, slice);       // (a unit past the last has no entries)
  const int S = a.g.S, pair = slice * 4 + wave, ch = pair * 32 + lg * 8;
  int mine = -1;
  if (lane < NB * 16) {
    const int r = unit * NB * 16 + lane, e = r / (S * S), q = r - e * S * S, iy = q / S;
    const SlabCell c = slab_cell(a, e);
    if (c.n >= 0) mine = (c.n * a.g.H + c.h + iy) * a.g.W + c.w + q - iy * S;
  }
  if (!__any(mine >= 0)) return;
  if (wave == 0 && lane < NB * 16) rowpx[lane] = mine;
  // packed in passes of four tiles: two groups of 32 channels
  const rsrc_t wrs = make_rsrc((g_bf16_p)wp, (unsigned)M * C * 2);
  const unsigned wbase = (unsigned)(pair >> 1) * (M / 32) * 4096 + (pair & 1) * 2048;
  L l;
  l.start(wrs, lane * 16, wbase, 4096);
  floatx4 acc[NB][2];
  slab_bias<NB, 2>(acc, b3, ch);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < NB * 16 * M * 2 / 4096; ++u) {
    int row, pos;
    slab_piece<M>(u * 4 + wave, lane, row, pos);
    slab_load((const AS_GLOBAL __bf16*)y2 + (size_t)max(rowpx[row], 0) * M + ((pos ^ (row & L::KEYS)) << 3), slab + (u * 4 + wave) * 512);
  }
  int px[NB];
  bf16x8 res[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    px[i] = rowpx[i * 16 + l16];
    res[i] = *reinterpret_cast<const AS_GLOBAL bf16x8*>((const AS_GLOBAL __bf16*)x + (size_t)max(px[i], 0) * C + ch);
  }
  slab_ready();
  l.run(acc, wrs, lane * 16, wbase, 4096, slab, lg, [&](int i, int, int& row, int& key) { row = i * 16 + l16; key = l16; });
  const float floor_ = post_relu ? 0.f : -__builtin_inff();
#pragma unroll
  for (int i = 0; i < NB; ++i)
    if (px[i] >= 0) {
      bf16x8 o;
#pragma unroll
      for (int u = 0; u < 8; ++u) o[u] = (__bf16)fmaxf((float)res[i][u] + acc[i][u / 4][u % 4], floor_);
      *reinterpret_cast<AS_GLOBAL bf16x8*>((AS_GLOBAL __bf16*)out + (size_t)px[i] * C + ch) = o;
    }
}

}  // namespace
}  // namespace lasnet
