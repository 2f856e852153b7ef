// The kernels of interpreted elementwise clusters: for element programs that are short (at most kShortDepth values below
// the top of the value stack and one gather at a time) and for the others.
//
// Short programs were bound by the instructions of the interpreter and are bound by memory where nothing is looked up (sum of exp(-x)^2 + 1, 2^24
// elements: 54 vector instructions an element and 35 us before, 25 now; exp(-d) * t stored and summed 54 and 40 us, of 200 MB;
// exp(-d)^2 + 1 stored 34.5 and 28).  The value stack is named rows of registers that every instruction works on from its top,
// not an array indexed at run time (three instructions to reach a register), the arrays of the next tile are on their way while a tile is
// worked on, and results really go past the caches.
#pragma once

#include "kernels.hpp"

namespace fc {

// A group a lane at a time, single elements for the rest.
__global__ __launch_bounds__(kBlock, 1) void interp_kernel(const KArgs a, Control *ctl, unsigned long long *partials) {
  const unsigned n = (unsigned)a.n, n4 = n & ~3u;
  const unsigned epoch = epoch_at_start(ctl);
  unsigned acc[kInterpFolds] = {interp_identity(a.fold_op[0]), interp_identity(a.fold_op[1])};
  constexpr unsigned kTileOf = kBlock * kVec;
  unsigned none[kVec], none1[1];
  for (unsigned base = blockIdx.x * kTileOf; base < n4; base += a.grid * kTileOf) {
    const unsigned i = base + threadIdx.x * kVec;
    if (i >= n4) break;
    interp_run<1, kInterpDepth, kInterpGathers, kBlock, false>(a, 0, i, kTileOf, InterpAhead<1, false>(), acc, none);
  }
  if (blockIdx.x == 0 && threadIdx.x < n - n4)
    interp_run<0, kInterpDepth, kInterpGathers, kBlock, false>(a, 0, n4 + threadIdx.x, 0u, InterpAhead<0, false>(), acc, none1);
  interp_finish<kWavesPerBlock>(a, acc, ctl, partials, epoch);
}

constexpr int kShortDepth = 2;        // values below the top of the stack

// The first D arrays that the program reads at the elements' own positions, read ahead of the run: G groups a lane (G = 0:
// one element), `apart` elements from each other.
template <int G, int D> struct ShortAhead {
  static_assert(D == 2 || D == 4, "arrays read ahead");
  static constexpr int V = G ? G * kVec : 1;
  unsigned v[D][V];
  template <bool Stream> __device__ __forceinline__ void read(const KArgs &a, unsigned first, unsigned apart) {
#pragma unroll
    for (int k = 0; k < D; ++k)
      if (a.ahead[k]) InterpAhead<G, true>::template read_one<Stream>(a.ahead[k], first, apart, v[k]);
  }
};

// The first `len` elements of the array that kCodeTable looks up, in LDS, with room for one more behind them; more: the
// array goes on in memory.
struct TableView { const unsigned *slice; unsigned len; bool more; };

// Runs the program for G groups a lane (G = 0: one element), `apart` elements from each other, the lane's first one at
// `first`.  The value stack is three named rows of registers, and every instruction works on its top in place.
// `ahead` holds what the program reads at the elements' own positions.
// table: where kCodeTable looks up.
template <int G, int D, int Depth, bool Enter, bool Table>
__device__ __forceinline__ void interp_short(const KArgs &a, unsigned first, unsigned apart, const ShortAhead<G, D> &ahead, 
                                             const TableView &table, unsigned (&acc)[kInterpFolds]) {
  using Raw = Quad128<unsigned>;
  constexpr int V = ShortAhead<G, D>::V;
  // worked out where it is needed: kept from instruction to instruction, the positions would take V registers
  auto own = [&](int e) {
    unsigned f = first;
    asm volatile("" : "+v"(f));
    return (int)(f + (e / kVec) * apart + e % kVec);
  };
  unsigned top[V], second[V], third[Depth > 1 ? V : 1];
  int at[Enter ? V : 1];                               // the positions a gather's source is read at
  int count = 0;                                       // values on the stack: the same in every lane, as is all that branches
  bool inside = false;                                 // below a gather: the position is `at`
  auto push = [&]() {
    if (Depth > 1 && count == 2) {
#pragma unroll
      for (int e = 0; e < V; ++e) third[Depth > 1 ? e : 0] = second[e];
    }
    if (count != 0) {
#pragma unroll
      for (int e = 0; e < V; ++e) second[e] = top[e];
    }
    ++count;
  };
  auto pop = [&]() {
    --count;
    if (count != 0) {
#pragma unroll
      for (int e = 0; e < V; ++e) top[e] = second[e];
    }
    if (Depth > 1 && count == 2) {
#pragma unroll
      for (int e = 0; e < V; ++e) second[e] = third[Depth > 1 ? e : 0];
    }
  };
  // array number k of those read ahead
  auto take = [&](int k) {
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const unsigned v0 = ahead.v[0][e], v1 = ahead.v[1][e], v2 = ahead.v[2 % D][e], v3 = ahead.v[3 % D][e];   // values: a choice of addresses would put v into memory
      top[e] = k == 0 ? v0 : D == 2 || k == 1 ? v1 : k == 2 ? v2 : v3;
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
            for (int e = 0; e < V; ++e) top[e] = p[at[Enter ? e : 0]];
          } else {
#pragma unroll
            for (int e = 0; e < V; ++e) top[e] = p[own(e)];
          }
        }
        break;
      }
      case kCodeLookup: {
        push();
        take(c.b - 1);
        const unsigned *p = static_cast<const unsigned *>(a.in[c.a]);
#pragma unroll
        for (int e = 0; e < V; ++e) top[e] = p[(int)top[e]];
        break;
      }
      case kCodeTable:
        if constexpr (Table) {
          push();
          take(c.b - 1);
          unsigned x[V];
#pragma unroll
          for (int e = 0; e < V; ++e) x[e] = table.slice[min(top[e], table.len)];
          if (table.more) {
            const unsigned *p = static_cast<const unsigned *>(a.in[c.a]);
#pragma unroll
            for (int e = 0; e < V; ++e)
              if (top[e] >= table.len) x[e] = p[(int)top[e]];
          }
#pragma unroll
          for (int e = 0; e < V; ++e) top[e] = x[e];
        }
        break;
      case kCodeGen: {
        push();
        int where[V];
#pragma unroll
        for (int e = 0; e < V; ++e) where[e] = Enter && inside ? at[Enter ? e : 0] : own(e);
        interp_gen<V>(c.a, a.p[c.b], a, where, top);
        break;
      }
      case kCodeMap:
        if (c.c == 1) {
          interp_map1<V>(c.a, a.p[c.b], top);
        } else if (c.c == 2) {
          if (c.a == FC_FN_MUL2) {
#pragma unroll
            for (int e = 0; e < V; ++e) top[e] = (unsigned)as_bits(FnMul2::apply(a.p[0], from_bits<float>((int)second[e]), from_bits<float>((int)top[e])));
          } else {
#pragma unroll
            for (int e = 0; e < V; ++e) top[e] = (unsigned)as_bits(FnAdd2::apply(a.p[0], from_bits<float>((int)second[e]), from_bits<float>((int)top[e])));
          }
          --count;
          if (Depth > 1 && count == 2) {
#pragma unroll
            for (int e = 0; e < V; ++e) second[e] = third[Depth > 1 ? e : 0];
          }
        } else if (Depth > 1) {                         // three arguments: add3, from the left
#pragma unroll
          for (int e = 0; e < V; ++e)
            top[e] = (unsigned)as_bits(FnAdd3::apply(a.p[0], from_bits<float>((int)third[Depth > 1 ? e : 0]), from_bits<float>((int)second[e]), from_bits<float>((int)top[e])));
          count -= 2;
        }
        break;
      case kCodeEnter:
        if constexpr (Enter) {
#pragma unroll
          for (int e = 0; e < V; ++e) at[e] = (int)top[e];
          inside = true;
          pop();
        }
        break;
      case kCodeLeave:
        inside = false;
        break;
      case kCodeStore: {
        unsigned *p = static_cast<unsigned *>(a.out[c.a]) + first;
        const bool keep = a.keeps(c.a);
        if (G == 0) p[0] = top[0];
        if (G > 0 && keep) {
          asm volatile("; kept in the caches");        // differs from the other branch's: the two stores stay two
#pragma unroll
          for (int g = 0; g < G; ++g)
            *reinterpret_cast<Raw *>(p + g * apart) = Raw{top[g * kVec % V], top[(g * kVec + 1) % V], top[(g * kVec + 2) % V], top[(g * kVec + 3) % V]};
          asm volatile("; kept in the caches");
        } else if (G > 0) {
          asm volatile("; past the caches");
#pragma unroll
          for (int g = 0; g < G; ++g)
            __builtin_nontemporal_store(Raw{top[g * kVec % V], top[(g * kVec + 1) % V], top[(g * kVec + 2) % V], top[(g * kVec + 3) % V]},
                                        reinterpret_cast<Raw *>(p + g * apart));
          asm volatile("; past the caches");
        }
        if (!(c.op & kCodeStays)) pop();
        break;
      }
      default: {                                        // kCodeFold
        auto into = [&](unsigned &sum) {
          switch (c.b) {
#define FC_EACH(Op) _Pragma("unroll") for (int e = 0; e < V; ++e) sum = (unsigned)as_bits(Op::apply(from_bits<Op::T>((int)sum), from_bits<Op::T>((int)top[e]))); break
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

// G groups a lane at a time where there are that many elements, single groups and elements for the rest.
template <int G, int D, int Depth, bool Enter, bool Next>
__global__ __launch_bounds__(kBlock, 4) void interp_short_kernel(const KArgs a, Control *ctl, unsigned long long *partials) {
  const unsigned n = (unsigned)a.n, n4 = n & ~3u;
  const unsigned epoch = epoch_at_start(ctl);
  unsigned acc[kInterpFolds] = {interp_identity(a.fold_op[0]), interp_identity(a.fold_op[1])};
  const TableView none = {nullptr, 0u, false};
  constexpr unsigned kGroup = kBlock * kVec, kTileOf = kGroup * G;
  const unsigned whole = n4 / kTileOf * kTileOf, stride = a.grid * kTileOf;
  if (blockIdx.x * kTileOf < whole) {
    ShortAhead<G, D> ahead;
    unsigned i = blockIdx.x * kTileOf + threadIdx.x * kVec;
    ahead.template read<true>(a, i, kGroup);
    for (unsigned base = blockIdx.x * kTileOf; base < whole; base += stride, i += stride) {
      if constexpr (Next) {
        ShortAhead<G, D> next;
        if (base + stride < whole) next.template read<true>(a, i + stride, kGroup);
        interp_short<G, D, Depth, Enter, false>(a, i, kGroup, ahead, none, acc);
        ahead = next;
      } else {
        interp_short<G, D, Depth, Enter, false>(a, i, kGroup, ahead, none, acc);
        if (base + stride < whole) ahead.template read<true>(a, i + stride, kGroup);
      }
    }
  }
  // what is left is less than a tile: the first G workgroups take a group a lane of it
  {
    const unsigned i = whole + blockIdx.x * kGroup + threadIdx.x * kVec;
    if (i < n4) {
      ShortAhead<1, D> ahead;
      ahead.template read<true>(a, i, kGroup);
      interp_short<1, D, Depth, Enter, false>(a, i, kGroup, ahead, none, acc);
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < n - n4) {
    ShortAhead<0, D> ahead;
    ahead.template read<false>(a, n4 + threadIdx.x, 0u);
    interp_short<0, D, Depth, Enter, false>(a, n4 + threadIdx.x, 0u, ahead, none, acc);
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
  const unsigned n = (unsigned)a.n, n4 = n & ~3u;
  const unsigned epoch = epoch_at_start(ctl);
  unsigned acc[kInterpFolds] = {interp_identity(a.fold_op[0]), interp_identity(a.fold_op[1])};
  const unsigned *array = static_cast<const unsigned *>(a.in[table_array]);
  const unsigned mine = threadIdx.x * kVec;
  const TableView table = {slice, min(elems, kTableSlice), elems > kTableSlice};
  // Two slabs at a time while there are that many for every workgroup, then one (the array's last one perhaps not whole): a
  // stretch of the array each would put the workgroups' accesses a power of two apart.
  const unsigned all = (n4 + kTableSlab - 1) / kTableSlab, pairs = n4 / kTableSlab / (2u * a.grid);
  ShortAhead<2, D> ahead;
  unsigned i = blockIdx.x * (2u * kTableSlab) + mine;
  const unsigned stride = a.grid * (2u * kTableSlab);
  if (pairs != 0u) ahead.template read<true>(a, i, kTableSlab);
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
  for (unsigned k = 0; k < pairs; ++k, i += stride) {
    ShortAhead<2, D> next;
    if (k + 1u < pairs) next.template read<true>(a, i + stride, kTableSlab);
    interp_short<2, D, Depth, false, true>(a, i, kTableSlab, ahead, table, acc);
    ahead = next;
  }
  for (unsigned s = pairs * 2u * a.grid + blockIdx.x; s < all; s += a.grid) {
    const unsigned at = s * kTableSlab + mine;
    if (at < n4) {
      ShortAhead<1, D> own;
      own.template read<true>(a, at, 0u);
      interp_short<1, D, Depth, false, true>(a, at, 0u, own, table, acc);
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < n - n4) {
    ShortAhead<0, D> own;
    own.template read<false>(a, n4 + threadIdx.x, 0u);
    interp_short<0, D, Depth, false, true>(a, n4 + threadIdx.x, 0u, own, table, acc);
  }
  interp_finish<kTableBlock / kWave>(a, acc, ctl, partials, epoch);
}

}  // namespace fc
