// Specialised instance for the cluster
//     out = add5(p, gather(N, p), gather(S, p), gather(W, p), gather(E, p))  [+ m = fold(max) p]
// where p = F(in) is a producer shared by consumers that read it in five
// different traversal orders (section 3.3, `simple5`: one array read in several
// orders inside one loop) and N, S, W, E are clamped unit shifts of a 2-D index.
//
// The generic element program would evaluate F five times per point and do
// integer division for every index.  Here a wave takes units of four rows and 256
// columns: a lane owns four adjacent columns, reads the unit's rows and the rows above
// and below it, evaluates F once per loaded element, and takes its west / east neighbours
// from the adjacent lanes with DPP wave shifts.  The column left of the strip and
// the one right of it are read by lanes 0 and 63 with one extra 4-byte load per
// row.  Rows may start on any 4-byte boundary: the 128-bit accesses of global memory need
// no more.
//
// Bound by memory.  The rows above and below a unit, and the halo columns, are being read
// by neighbouring waves at about the same time and come from the cache (ordinary loads;
// F is evaluated 1.5 times per point, which the idle half of the issue slots takes).  Bands
// as low as four rows keep what is in flight close together and give small grids enough
// waves; before, a wave walked down 32 to 128 rows with three of them in registers: 8192 x 8192
// 112 -> 98 us, 4096 x 4096 30.6 -> 22.4, 1024 x 1024 15.1 -> 6.3, 64 x 64 13.8 -> 5.1 (and grids
// whose rows are no multiple of four went through the generic element program: 8192 x 8191
// 269 -> 109 us, 1531 x 2477 22.4 -> 9.3).  Results are stored non-temporally: ordinary stores
// leave dirty lines in the memory-side cache that the next kernel waits for.  What the choice costs depends on what ran
// before (8192 x 8192, us, before / now / now with ordinary stores): grids in turn 110 / 94 / 105, after idle 113 / 98
// / 105, after a compaction 115 / 105 / 110; but right after a kernel that leaves dirty lines of its own
// (a copy of 512 MiB) 95 / 119 / 101, where the two together take 316 / 306 / 300, with a fill 197 / 209 / 193; the
// output the next call's input 98 / 97 / 108, 5800 x 5800 53 / 58 / 49, 4096 x 4096 31 / 32 / 24.
#pragma once

#include "kernels.hpp"
#include "launchers.hpp"
#include "registry.hpp"

namespace fc {

constexpr int kStripCols = kWave * kVec;         // 256 output columns per wave
constexpr int kBandRows = 4;                     // output rows of a unit

struct Quad { float x, y, z, w; };

// Row r (clamped to the grid) of the input at columns c .. c+3, before F; the 128-bit
// read is taken at min(c, W-4) and so always inside the row (W >= 4, c >= 0).  Nothing
// here depends on the loaded value, so the row reads of a step are issued back to back
// and are in flight together.
using RawRow = float __attribute__((ext_vector_type(4)));
using RowInMemory = Quad128<float>;              // rows start on any 4-byte boundary
__device__ __forceinline__ RawRow load_row(const float *g, int r, int c, int H, int W) {
  r = min(max(r, 0), H - 1);
  return *reinterpret_cast<const RowInMemory *>(g + (size_t)r * (size_t)W + min(c, W - kVec));
}

// p = F(row).  `past` = how far (0 .. 3) the read was moved left to stay inside the row: columns right
// of the grid stand for the clamped column W-1.
template <class F>
__device__ __forceinline__ Quad apply_row(const Slot &s, RawRow t, bool ragged, int past) {
  if (ragged) {                                  // the same for the whole wave: its strip reaches past the grid
    if (past & 1) { t.x = t.y; t.y = t.z; t.z = t.w; }
    if (past & 2) { t.x = t.z; t.y = t.w; t.z = t.w; }
  }
  return {F::apply(s, t.x), F::apply(s, t.y), F::apply(s, t.z), F::apply(s, t.w)};
}

// p at the column left of the strip (lane 0) or right of it (lane 63), clamped to the grid
// Only the load sits under the lane condition; F is applied by the caller on
// all lanes, so that no wait for the load is needed inside the branch and the
// loads of a step stay in flight together.
__device__ __forceinline__ float load_halo(const float *g, int r, int c0, int lane, int H, int W) {
  float v = 0.0f;
  if (lane == 0 || lane == kWave - 1) {
    r = min(max(r, 0), H - 1);
    const int c = lane == 0 ? max(c0 - 1, 0) : min(c0 + kStripCols, W - 1);
    v = g[(size_t)r * (size_t)W + c];
  }
  return v;
}

// F: element function of the shared producer (FnExpNeg, or FnIdentF when p is
// read from memory).  WithMax: also fold(max) over p into out[1].
template <class F, int FSlot, bool WithMax>
__global__ __launch_bounds__(kBlock) void stencil5_kernel(const Packed<kHeadH | kHeadW | kHeadFlags, WithMax ? 3u : 1u, In<0, float>> packed,
                                                          Control *ctl, unsigned long long *partials, int n_strips, int n_units) {
  static_assert(SlotUse<F>::value == 0, "the shared producer takes no parameters");
  const KArgs &a = packed.open();
  const int H = a.h, W = a.w;
  const float *g = static_cast<const float *>(a.in[0]);
  float *out = static_cast<float *>(a.out[0]);
  const Slot &fs = a.p[FSlot];
  const unsigned epoch = WithMax ? epoch_at_start(ctl) : 0u;
  const int lane = lane_id();

  // workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous
  // range of units (unit = band, strip), a wave a unit at a time, so that
  // halo rows are re-read from its own L2
  const int per_xcd = ((n_units + kWavesPerBlock - 1) / kWavesPerBlock + 7) / 8 * kWavesPerBlock;
  const int first = (int)(blockIdx.x % 8) * per_xcd, end = min(first + per_xcd, n_units);
  const int stride = (int)(a.grid / 8) * kWavesPerBlock;
  RawRow raw[kBandRows + 2];                     // rows r0-1 .. r0+kBandRows of the unit that is worked on next
  float hraw[kBandRows];
  auto fetch = [&](int unit) {
    const int band = unit / n_strips, strip = unit - band * n_strips, r0 = band * kBandRows;
    const int c0 = strip * kStripCols, c = c0 + lane * kVec;
#pragma unroll
    for (int k = 0; k < kBandRows; ++k) hraw[k] = load_halo(g, r0 + k, c0, lane, H, W);
#pragma unroll
    for (int k = 0; k < kBandRows + 2; ++k) raw[k] = load_row(g, r0 + k - 1, c, H, W);
  };
  float m = -__builtin_inff();
  const int unit0 = __builtin_amdgcn_readfirstlane(first + (int)(blockIdx.x / 8) * kWavesPerBlock + wave_id());
  if (unit0 < end) fetch(unit0);
  with_keep(a.keeps(0), [&](auto keep) {
    for (int unit = unit0; unit < end; unit += stride) {
      const int band = unit / n_strips, strip = unit - band * n_strips, r0 = band * kBandRows;
      const int c0 = strip * kStripCols, c = c0 + lane * kVec;
      const int mine = min(W - c, kVec);           // columns of the lane inside the grid (less than one: none)
      const bool ragged = c0 + kStripCols > W;
      const int past = min(max(c - (W - kVec), 0), kVec - 1);
      Quad p[kBandRows + 2];
      float h[kBandRows];
#pragma unroll
      for (int k = 0; k < kBandRows + 2; ++k) p[k] = apply_row<F>(fs, raw[k], ragged, past);
#pragma unroll
      for (int k = 0; k < kBandRows; ++k) h[k] = F::apply(fs, hraw[k]);
      if (unit + stride < end) fetch(unit + stride);
#pragma unroll
      for (int k = 0; k < kBandRows; ++k) {
        const Quad &up = p[k], &cur = p[k + 1], &down = p[k + 2];
        const float left = lane_prev(h[k], cur.w);     // lane 0 keeps its halo value
        const float right = lane_next(h[k], cur.x);    // lane 63 keeps its halo value
        // (((p + N) + S) + W) + E, the order of add5
        RawRow o;
        o.x = (((cur.x + up.x) + down.x) + left) + cur.y;
        o.y = (((cur.y + up.y) + down.y) + cur.x) + cur.z;
        o.z = (((cur.z + up.z) + down.z) + cur.y) + cur.w;
        o.w = (((cur.w + up.w) + down.w) + cur.z) + right;
        if (r0 + k < H) {
          float *to = out + (size_t)(r0 + k) * (size_t)W + c;
          if (mine == kVec) {
            if (decltype(keep)::value) *reinterpret_cast<RowInMemory *>(to) = o; else __builtin_nontemporal_store(o, reinterpret_cast<RowInMemory *>(to));
          } else {
#pragma unroll
            for (int q = 0; q < kVec - 1; ++q) if (q < mine) to[q] = o[q];
          }
          // columns past the grid repeat its last column
          if (WithMax) m = fmaxf(fmaxf(fmaxf(m, cur.x), fmaxf(cur.y, cur.z)), cur.w);
        }
      }
    }
  });
  if (WithMax) fold_finish<MaxF32>(m, a, 1, ctl, partials, epoch);
}

template <class F, int FSlot, bool WithMax, int G0, int GStride>
bool stencil5_accept(const KArgs &a) {
  static const int want[4][2] = {{-1, 0}, {1, 0}, {0, -1}, {0, 1}};
  if (a.h < 1 || a.w < kVec || a.w > 0x7fffffff - 4 * kStripCols) return false;     // columns past the row's end are counted in int
  // A narrow grid leaves most lanes of a strip idle, and the generic element program, which takes points in storage
  // order, is faster there: 4.2 x 10^6 points in rows of 4 take 242 us here and 20 there, of 17 66 and 21, of 33 41 and 21,
  // of 66 (3.9 columns of the strip for one of the grid) 21 and 21, of 129 13 and 20.  Unless the units are few enough to run all at
  // once: 2.6 x 10^5 points in rows of 33 (1986 units) take 6.7 us here and 8.4 there, of 17 (3855) 8.4 and 8.2.
  const long long strips = (a.w + kStripCols - 1) / kStripCols, units = strips * ((a.h + kBandRows - 1) / kBandRows);
  if (units > 2048 && strips * kStripCols * 2 > 7LL * a.w) return false;
  for (int k = 0; k < 4; ++k) {
    const Slot &s = a.p[G0 + k * GStride];
    if (s.i[0] != want[k][0] || s.i[1] != want[k][1] || s.ext[0] != a.h || s.ext[1] != a.w) return false;
  }
  return true;
}

template <class F, int FSlot, bool WithMax>
hipError_t launch_stencil5(const KArgs &a, const LaunchCtx &c) {
  if (a.n == 0 && !WithMax) return hipSuccess;
  const int strips = (a.w + kStripCols - 1) / kStripCols;
  const int units = strips * ((a.h + kBandRows - 1) / kBandRows);
  // A unit per wave, up to a round of the XCDs fewer workgroups than the fold has partials (the form without the fold
  // keeps to the same number): the hardware hands the next workgroup out as one ends, and what runs at a time is one
  // front of adjacent units per XCD; in larger grids a wave takes several units, a grid's length apart.  8192 workgroups, which
  // give every wave of 8192 x 8192 two units, are slower than these 8184, which leave eight units per XCD for a
  // third turn: 99.5 us against 94.7.  With 4 workgroups per compute unit that walk over the units 8192 x 8192 takes 98 us,
  // but 7000 x 8001 100 us instead of 91 and 4096 x 4096 24 us instead of 22.4.
  const int blocks = std::min(std::max(8, ((units + kWavesPerBlock - 1) / kWavesPerBlock + 7) / 8 * 8), kMaxPartials - 8);
  return launch_k(&stencil5_kernel<F, FSlot, WithMax>, (unsigned)blocks, c, a, c.ctl, c.partials, strips, units);
}

}  // namespace fc
