// The kernels of interpreted elementwise clusters: for element programs that are short (at most kShortDepth values below
// the top of the value stack and one gather at a time) and for the others.
//
// Short programs were bound by the instructions of the interpreter and are bound by memory where nothing is looked up (sum of exp(-x)^2 + 1, 2^24
// elements: 54 vector instructions an element and 35 us before, 25 now; exp(-d) * t stored and summed 54 and 40 us, of 200 MB;
// exp(-d)^2 + 1 stored 34.5 and 28; a * b + exp(-c) stored, 2^22: 18.1 and 14.1).  The value stack is named rows of registers
// that every instruction works on from its top, not an array indexed at run time (three instructions to reach a register); the
// rows are vectors of four, which the compiler moves in pairs where the branches of the interpreter meet (elements on their own: 24.9
// against 26.8 us for the first of these sums); the arrays of the next tile are on their way while a tile is worked on,
// and results really go past the caches.  Short arrays last as long as one program: every piece of code that one
// workgroup runs after another is fetched for the first time, so the end of the array is a group like the others (42034
// elements with a lookup 9.3 us before, with two passes more for what was left, 6.4 now).
#pragma once

#include "kernels.hpp"

namespace fc {

constexpr int kShortDepth = 2;        // values below the top of the stack

// The elements a lane works on: G groups, `apart` elements from each other, the first at `first`.  Single groups (G = 1) may be
// cut off by the end of the array: of theirs the first `valid` exist, and the others stand for the first once more (so
// that no index is made up); they are neither stored nor folded.  base: the workgroup's first element, n: of the array.
template <int G> struct Span {
  unsigned first, apart;
  __device__ __forceinline__ Span(unsigned, unsigned first_, unsigned apart_, unsigned) : first(first_), apart(apart_) {}
  __device__ __forceinline__ unsigned offset(int e) const { return (e / kVec) * apart + e % kVec; }
  __device__ __forceinline__ bool exists(int) const { return true; }
  __device__ __forceinline__ void read(const void *array, Words4 (&x)[G]) const {
    const unsigned *p = static_cast<const unsigned *>(array) + first;
#pragma unroll
    for (int g = 0; g < G; ++g) x[g] = __builtin_nontemporal_load(reinterpret_cast<const Quad128<unsigned> *>(p + g * apart));
  }
  template <bool Keep> __device__ __forceinline__ void write(void *array, const Words4 (&x)[G]) const {
    using Raw = Quad128<unsigned>;
    unsigned *p = static_cast<unsigned *>(array) + first;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const Raw v = x[g];
      if (Keep) *reinterpret_cast<Raw *>(p + g * apart) = v; else __builtin_nontemporal_store(v, reinterpret_cast<Raw *>(p + g * apart));
    }
  }
};
template <> struct Span<1> {
  using Raw = int __attribute__((ext_vector_type(4)));
  unsigned base, first, valid, bytes;                  // bytes: of the array from `base` on, as many as the lanes reach
  __device__ __forceinline__ Span(unsigned base_, unsigned first_, unsigned, unsigned n)
      : base(base_), first(first_), valid(min(n - first_, (unsigned)kVec)), bytes(min(n - base_, 1u << 16) * 4u) {}
  __device__ __forceinline__ unsigned offset(int e) const { return (unsigned)e < valid ? e : 0; }
  __device__ __forceinline__ bool exists(int e) const { return (unsigned)e < valid; }
  // a 32-bit word past the end reads as zero, and is not written
  template <bool Stream = true> __device__ __forceinline__ void read(const void *array, Words4 (&x)[1]) const {
    const __amdgpu_buffer_rsrc_t buf =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned *>(static_cast<const unsigned *>(array) + base), 0, (int)bytes, 0x00020000);
    const Raw v = __builtin_amdgcn_raw_buffer_load_b128(buf, (int)((first - base) * 4u), 0, Stream ? 0x2 : 0);
#pragma unroll
    for (int e = 0; e < kVec; ++e) x[0][e] = (unsigned)(exists(e) ? v[e] : v[0]);
  }
  template <bool Keep> __device__ __forceinline__ void write(void *array, const Words4 (&x)[1]) const {
    const __amdgpu_buffer_rsrc_t buf = __builtin_amdgcn_make_buffer_rsrc(static_cast<unsigned *>(array) + base, 0, (int)bytes, 0x00020000);
    const Raw v = __builtin_bit_cast(Raw, x[0]);
    __builtin_amdgcn_raw_buffer_store_b128(v, buf, (int)((first - base) * 4u), 0, Keep ? 0 : 0x2);
  }
};

// The programs that are not short: a group a lane at a time, the end of the array as a group like the others.  Single elements
// for it were a pass of their own behind a workgroup's tiles, all of its code fetched for the first time (x = exp(-a), add3(x, b, add3(b,
// c, d * e)) stored and summed, us a pass before / now: 4099 elements 12.9 / 9.0, 300001 13.0 / 9.5, 1000003 13.3 / 11.6, 2^24 113).  All groups
// as if they could be cut off take more instructions: 2^24 elements 118.6 us, 60000 9.8 instead of 9.0.
__global__ __launch_bounds__(kBlock, 1) void interp_kernel(const KArgs a, Control *ctl, unsigned long long *partials) {
  const unsigned n = (unsigned)a.n;
  const unsigned epoch = epoch_at_start(ctl);
  unsigned acc[kInterpFolds] = {interp_identity(a.fold_op[0]), interp_identity(a.fold_op[1])};
  constexpr unsigned kTileOf = kBlock * kVec;
  unsigned none[kVec], base = blockIdx.x * kTileOf;
  const unsigned mine = threadIdx.x * kVec;
  for (; base + kTileOf <= n; base += a.grid * kTileOf)
    interp_run<1, kBlock>(a, 0, base + mine, acc, none);
  if (base + mine < n)                                   // one workgroup's, and for short arrays all that it does
    interp_run<1, kBlock>(a, 0, base + mine, acc, none, Span<1>(base, base + mine, 0u, n));
  interp_finish<kWavesPerBlock>(a, acc, ctl, partials, epoch);
}

// The first D arrays that the program reads at the elements' own positions, read ahead of the run.
template <int G, int D> struct ShortAhead {
  static_assert(D == 2 || D == 4, "arrays read ahead");
  Words4 v[D][G];
  __device__ __forceinline__ void read(const KArgs &a, const Span<G> span) {
#pragma unroll
    for (int k = 0; k < D; ++k)
      if (a.ahead[k]) span.read(a.ahead[k], v[k]);
  }
};

// The first `len` elements of the array that kCodeTable looks up, in LDS, with room for one more behind them; more: the
// array goes on in memory.
struct TableView { const unsigned *slice; unsigned len; bool more; };

// Runs the program for the elements of `span`.  The value stack is three named rows of registers, and every instruction
// works on its top in place.  `ahead` holds what the program reads at the elements' own positions.  table: where kCodeTable looks up.
template <int G, int D, int Depth, bool Enter, bool Table>
__device__ __forceinline__ void interp_short(const KArgs &a, const Span<G> span, const ShortAhead<G, D> &ahead, const TableView &table,
                                             unsigned (&acc)[kInterpFolds]) {
  constexpr int V = G * kVec;                          // elements a lane
  // worked out where it is needed: kept from instruction to instruction, the positions would take V registers
  auto own = [&](int e) {
    unsigned first = span.first;
    asm volatile("" : "+v"(first));
    return (int)(first + span.offset(e));
  };
  Words4 top[G], second[G], third[Depth > 1 ? G : 1];    // vectors of four: the compiler moves them in pairs of registers
  int at[Enter ? V : 1];                               // the positions a gather's source is read at
  int count = 0;                                       // values on the stack: the same in every lane, as is all that branches
  bool inside = false;                                 // below a gather: the position is `at`
  auto push = [&]() {
    if (Depth > 1 && count == 2) {
#pragma unroll
      for (int g = 0; g < G; ++g) third[Depth > 1 ? g : 0] = second[g];
    }
    if (count != 0) {
#pragma unroll
      for (int g = 0; g < G; ++g) second[g] = top[g];
    }
    ++count;
  };
  auto pop = [&]() {
    --count;
    if (count != 0) {
#pragma unroll
      for (int g = 0; g < G; ++g) top[g] = second[g];
    }
    if (Depth > 1 && count == 2) {
#pragma unroll
      for (int g = 0; g < G; ++g) second[g] = third[Depth > 1 ? g : 0];
    }
  };
  // array number k of those read ahead
  auto take = [&](int k) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const Words4 v0 = ahead.v[0][g], v1 = ahead.v[1][g], v2 = ahead.v[2 % D][g], v3 = ahead.v[3 % D][g];   // values: a choice of addresses would put v into memory
      top[g] = k == 0 ? v0 : D == 2 || k == 1 ? v1 : k == 2 ? v2 : v3;
    }
  };
  int pc = 0;
  for (Code c = a.code_word(0), following; c.op != kCodeEnd; c = following) {
    following = a.code_word(++pc);                     // the last entry is kCodeEnd
    switch (c.op & ~kCodeStays) {
      case kCodeIn: {
        push();
        if (c.b != 0) {
          take(c.b - 1);
        } else {
          const unsigned *p = static_cast<const unsigned *>(a.in[c.a]);
          if (Enter && inside) {
#pragma unroll
            for (int e = 0; e < V; ++e) top[e / kVec][e % kVec] = p[at[Enter ? e : 0]];
          } else {
#pragma unroll
            for (int e = 0; e < V; ++e) top[e / kVec][e % kVec] = p[own(e)];
          }
        }
        break;
      }
      case kCodeLookup: {
        push();
        take(c.b - 1);
        const unsigned *p = static_cast<const unsigned *>(a.in[c.a]);
#pragma unroll
        for (int e = 0; e < V; ++e) top[e / kVec][e % kVec] = p[(int)top[e / kVec][e % kVec]];
        break;
      }
      case kCodeTable:
        if constexpr (Table) {
          push();
          take(c.b - 1);
          unsigned x[V];
#pragma unroll
          for (int e = 0; e < V; ++e) x[e] = table.slice[min(top[e / kVec][e % kVec], table.len)];
          if (table.more) {
            const unsigned *p = static_cast<const unsigned *>(a.in[c.a]);
#pragma unroll
            for (int e = 0; e < V; ++e)
              if (top[e / kVec][e % kVec] >= table.len) x[e] = p[(int)top[e / kVec][e % kVec]];
          }
#pragma unroll
          for (int e = 0; e < V; ++e) top[e / kVec][e % kVec] = x[e];
        }
        break;
      case kCodeGen: {
        push();
        int where[V];
#pragma unroll
        for (int e = 0; e < V; ++e) where[e] = Enter && inside ? at[Enter ? e : 0] : own(e);
        unsigned x[V];
        interp_gen<V>(c.a, a.p[c.b], a, where, x);
#pragma unroll
        for (int e = 0; e < V; ++e) top[e / kVec][e % kVec] = x[e];
        break;
      }
      case kCodeMap:
        if (c.c == 1) {
          unsigned x[V];
#pragma unroll
          for (int e = 0; e < V; ++e) x[e] = top[e / kVec][e % kVec];
          interp_map1<V>(c.a, a.p[c.b], x);
#pragma unroll
          for (int e = 0; e < V; ++e) top[e / kVec][e % kVec] = x[e];
        } else if (c.c == 2) {
          if (c.a == FC_FN_MUL2) {
#pragma unroll
            for (int e = 0; e < V; ++e) top[e / kVec][e % kVec] = (unsigned)as_bits(FnMul2::apply(a.p[0], from_bits<float>((int)second[e / kVec][e % kVec]), from_bits<float>((int)top[e / kVec][e % kVec])));
          } else {
#pragma unroll
            for (int e = 0; e < V; ++e) top[e / kVec][e % kVec] = (unsigned)as_bits(FnAdd2::apply(a.p[0], from_bits<float>((int)second[e / kVec][e % kVec]), from_bits<float>((int)top[e / kVec][e % kVec])));
          }
          --count;
          if (Depth > 1 && count == 2) {
#pragma unroll
            for (int g = 0; g < G; ++g) second[g] = third[Depth > 1 ? g : 0];
          }
        } else if (Depth > 1) {                         // three arguments: add3, from the left
#pragma unroll
          for (int e = 0; e < V; ++e)
            top[e / kVec][e % kVec] = (unsigned)as_bits(FnAdd3::apply(a.p[0], from_bits<float>((int)third[Depth > 1 ? e / kVec : 0][e % kVec]), from_bits<float>((int)second[e / kVec][e % kVec]), from_bits<float>((int)top[e / kVec][e % kVec])));
          count -= 2;
        }
        break;
      case kCodeEnter:
        if constexpr (Enter) {
#pragma unroll
          for (int e = 0; e < V; ++e) at[e] = (int)top[e / kVec][e % kVec];
          inside = true;
          pop();
        }
        break;
      case kCodeLeave:
        inside = false;
        break;
      case kCodeStore: {
        if (a.keeps(c.a)) {
          asm volatile("; kept in the caches");        // differs from the other branch's: the two stores stay two
          span.template write<true>(a.out[c.a], top);
          asm volatile("; kept in the caches");
        } else {
          asm volatile("; past the caches");
          span.template write<false>(a.out[c.a], top);
          asm volatile("; past the caches");
        }
        if (!(c.op & kCodeStays)) pop();
        break;
      }
      default: {                                        // kCodeFold
        auto into = [&](unsigned &sum) {
          switch (c.b) {
#define FC_EACH(Op) _Pragma("unroll") for (int e = 0; e < V; ++e) sum = (unsigned)as_bits(Op::apply(from_bits<Op::T>((int)sum), span.exists(e) ? from_bits<Op::T>((int)top[e / kVec][e % kVec]) : Op::identity())); break
            case kFoldAddF32: FC_EACH(AddF32);
            case kFoldMaxF32: FC_EACH(MaxF32);
            case kFoldMulF32: FC_EACH(MulF32);
            case kFoldAddI32: FC_EACH(AddI32);
            default: FC_EACH(MaxI32);
#undef FC_EACH
          }
        };
        unsigned sum = c.c == 0 ? acc[0] : acc[1];
        into(sum);
        if (c.c == 0) acc[0] = sum; else acc[1] = sum;
        if (!(c.op & kCodeStays)) pop();
        break;
      }
    }
  }
}

// G groups a lane at a time, single groups for the rest.  The widest form (two groups, four arrays, Enter) needs two registers more than
// four workgroups a compute unit leave it, and spills them (12 bytes a lane): a * b + exp(-c) stored and summed, 2^20 elements 10.9 us, 2^24 59,
// where the general interpreter took 16.1 and 70.
template <int G, int D, int Depth, bool Enter, bool Next>
__global__ __launch_bounds__(kBlock, 4) void interp_short_kernel(const KArgs a, Control *ctl, unsigned long long *partials) {
  const unsigned n = (unsigned)a.n;
  const unsigned epoch = epoch_at_start(ctl);
  unsigned acc[kInterpFolds] = {interp_identity(a.fold_op[0]), interp_identity(a.fold_op[1])};
  const TableView none = {nullptr, 0u, false};
  constexpr unsigned kGroup = kBlock * kVec, kTileOf = kGroup * G;
  const unsigned mine = threadIdx.x * kVec;
  if constexpr (G == 1) {
    for (unsigned base = blockIdx.x * kGroup; base < n; base += a.grid * kGroup) {
      if (base + mine >= n) break;
      const Span<1> span(base, base + mine, 0u, n);
      ShortAhead<1, D> ahead;
      ahead.read(a, span);
      interp_short<1, D, Depth, Enter, false>(a, span, ahead, none, acc);
    }
  } else {
    const unsigned whole = n / kTileOf * kTileOf, stride = a.grid * kTileOf;
    if (blockIdx.x * kTileOf < whole) {
      ShortAhead<G, D> ahead;
      unsigned i = blockIdx.x * kTileOf + mine;
      ahead.read(a, Span<G>(0u, i, kGroup, n));
      for (unsigned base = blockIdx.x * kTileOf; base < whole; base += stride, i += stride) {
        const Span<G> span(0u, i, kGroup, n), after(0u, i + stride, kGroup, n);
        if constexpr (Next) {
          ShortAhead<G, D> next;
          if (base + stride < whole) next.read(a, after);
          interp_short<G, D, Depth, Enter, false>(a, span, ahead, none, acc);
          ahead = next;
        } else {
          interp_short<G, D, Depth, Enter, false>(a, span, ahead, none, acc);
          if (base + stride < whole) ahead.read(a, after);
        }
      }
    }
    // What is left is less than a tile: a group a lane for the G workgroups whose turn it would be.
    const unsigned turn = whole / kTileOf % a.grid, k = blockIdx.x - turn + (blockIdx.x < turn ? a.grid : 0u), base = whole + k * kGroup;
    if (k < (unsigned)G && base + mine < n) {
      const Span<1> span(base, base + mine, 0u, n);
      ShortAhead<1, D> ahead;
      ahead.read(a, span);
      interp_short<1, D, Depth, Enter, false>(a, span, ahead, none, acc);
    }
  }
  interp_finish<kWavesPerBlock>(a, acc, ctl, partials, epoch);
}

// ------------------------------------------------------------------ lookups from LDS
// The same for a program whose first lookup (kCodeLookup: an element of a table at the index another array holds) goes to
// kCodeTable: the first kTableSlice elements of the table are kept in LDS, the others are read from memory.  Lookups that hit
// L2 are bound by the rate at which it takes requests (2.4 x 10^11 a second: 2^22 of them 17.6 us, whatever else the kernel does),
// those from LDS by memory again: exp(-d) * t[i] stored and summed, tables of 256 KiB, 2^22 elements 28.9 us before, 27.4 with the short
// program's kernel, 20.0 this way (10.4 of it fixed: launch, table, the hand-over of the sums), 2^24 95 / 93 / 65; of 156 KiB 92 / 90 / 43.
// The whole table in pieces, one after the other, with the indices kept in registers takes 2.7 us a piece and step (256 KiB: 29.9 and 90 us).
constexpr int kTableBlock = 1024;                      // threads of the one workgroup a compute unit holds
constexpr unsigned kTableSlab = kTableBlock * kVec;    // elements of a group a lane
constexpr unsigned kTableSlice = 39936;                // elements of the table in LDS: 156 KiB

__global__ __launch_bounds__(kTableBlock) void interp_table_kernel(const KArgs a, Control *ctl, unsigned long long *partials, int table_array,
                                                                   unsigned elems) {
  using RawI = int __attribute__((ext_vector_type(4)));
  constexpr int D = 2, Depth = 1;                        // of the programs that it takes
  __shared__ unsigned slice[kTableSlice + kVec];
  const unsigned n = (unsigned)a.n;
  const unsigned epoch = epoch_at_start(ctl);
  unsigned acc[kInterpFolds] = {interp_identity(a.fold_op[0]), interp_identity(a.fold_op[1])};
  const unsigned *array = static_cast<const unsigned *>(a.in[table_array]);
  const unsigned mine = threadIdx.x * kVec;
  const TableView table = {slice, min(elems, kTableSlice), elems > kTableSlice};
  // Two slabs at a time while there are that many for every workgroup, then one (the array's last one perhaps not whole): a
  // stretch of the array each would put the workgroups' accesses a power of two apart.
  const unsigned all = (n + kTableSlab - 1u) / kTableSlab, pairs = n / kTableSlab / (2u * a.grid);
  ShortAhead<2, D> ahead;
  const unsigned stride = a.grid * (2u * kTableSlab);
  unsigned base = blockIdx.x * (2u * kTableSlab);
  if (pairs != 0u) ahead.read(a, Span<2>(base, base + mine, kTableSlab, n));
  {
    // buffer loads: what lies past the end reads as zero without a condition in front of it, which would leave a wave
    // with one read in flight
    const unsigned len4 = table.len & ~3u;
    const __amdgpu_buffer_rsrc_t table_buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned *>(array), 0, (int)(len4 * 4u), 0x00020000);
    constexpr int kReads = (kTableSlice + kTableSlab - 1) / kTableSlab;
    RawI v[kReads];
#pragma unroll
    for (int u = 0; u < kReads; ++u) v[u] = __builtin_amdgcn_raw_buffer_load_b128(table_buf, (int)((mine + u * kTableSlab) * 4u), 0, 0);
#pragma unroll
    for (int u = 0; u < kReads; ++u)
      if (mine + u * kTableSlab < len4) *reinterpret_cast<RawI *>(&slice[mine + u * kTableSlab]) = v[u];
    if (threadIdx.x < table.len - len4) slice[len4 + threadIdx.x] = array[len4 + threadIdx.x];
  }
  __syncthreads();
  for (unsigned k = 0; k < pairs; ++k, base += stride) {
    ShortAhead<2, D> next;
    if (k + 1u < pairs) next.read(a, Span<2>(base + stride, base + stride + mine, kTableSlab, n));
    interp_short<2, D, Depth, false, true>(a, Span<2>(base, base + mine, kTableSlab, n), ahead, table, acc);
    ahead = next;
  }
  for (unsigned s = pairs * 2u * a.grid + blockIdx.x; s < all; s += a.grid) {
    const unsigned slab = s * kTableSlab;
    if (slab + mine < n) {
      const Span<1> span(slab, slab + mine, 0u, n);
      ShortAhead<1, D> own;
      own.read(a, span);
      interp_short<1, D, Depth, false, true>(a, span, own, table, acc);
    }
  }
  interp_finish<kTableBlock / kWave>(a, acc, ctl, partials, epoch);
}

}  // namespace fc
