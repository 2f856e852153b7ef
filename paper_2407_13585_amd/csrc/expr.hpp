// Element-level programs of a fused cluster as expression types.
//
// A cluster's producers (map / zipWith, generate, gather; Table 1) form a tree
// that is evaluated in registers for one iteration index.  A gather pushes its
// index through the producers of its source (section 3.3, `simple1`,
// `simple2`): Gather<EI, ES> evaluates ES at the index EI yields, so a producer
// below a gather is recomputed at the gathered position and never stored.
//
// Every expression type offers
//   eval(args, i)     value at iteration index i
//   eval4(args, i)    values at i .. i+3, 128-bit loads on leaves (i may be any position: 128-bit
//                     accesses of global memory need 4-byte alignment only, see Quad128)
//   sig(std::string&) the textual signature the host matcher compares against
//   kNodes            number of combinator nodes in the tree (parameter slots)
//   kMirror           the tree reads an array through `reverse` as well (tile order, kernels.hpp)
//   eval4_pair(args, i, ip, at_i, at_ip)   values at the groups of four i and ip, where ip is
//                     the mirror image of i (ip = n - 4 - i); see for_each_mirrored_pair
//   mirrors_whole(args, n)   every `reverse` of the tree runs over exactly n elements
// Parameter slots are numbered in pre-order, leaves included.
#pragma once

#include <hip/hip_runtime.h>

#include <string>
#include <tuple>
#include <type_traits>
#include <utility>

#include "prim.hpp"

namespace fc {

constexpr int kMaxIn = 8;
constexpr int kMaxOut = 4;
constexpr int kMaxSlots = 24;

struct Slot {     // parameters of one combinator node
  float f[2];
  int i[2];       // the node's own integer parameters
  int ext[2];     // the node's own extents (outer, inner); inner is 1 for 1-D arrays
  unsigned m[3];  // constants the host derives from the parameters (mod_eq_constants, div_constants)
};

// x mod k == r for x >= 0 without a division.  With k = 2^s * d, d odd, and
// inv = d^-1 mod 2^32: t is a multiple of k exactly if rotr(t * inv, s) <= (2^32-1) / k
// (test for a zero remainder by multiplying with the inverse of the odd part);
// apply it to t = x - r, which needs x >= r.  A residue outside [0, k) matches no x.
inline void mod_eq_constants(Slot &s) {
  const unsigned k = (unsigned)s.i[0];
  if (s.i[0] <= 0 || s.i[1] < 0 || s.i[1] >= s.i[0]) {
    s.i[1] = (int)0x80000000u;                // no non-negative int32 reaches it
    s.m[0] = s.m[1] = s.m[2] = 0;
    return;
  }
  unsigned shift = 0, d = k;
  while ((d & 1u) == 0) { d >>= 1; ++shift; }
  unsigned inv = d;                            // Newton steps double the number of correct low bits (3 to start with)
  for (int it = 0; it < 5; ++it) inv *= 2u - d * inv;
  s.m[0] = inv;
  s.m[1] = shift;
  s.m[2] = 0xffffffffu / k;
}

// The element programs of a cluster once more, as code for the interpreting kernel
// (interp_kernel), which runs clusters that no compiled instance matches.  A stack
// machine in post-order: a value per array read, generated or computed, consumed by the
// map, store or fold above it; a gather evaluates its index, then its source with the
// index as the position (kCodeEnter / kCodeLeave).
constexpr int kMaxCode = 64;
constexpr int kMaxRoots = 4;          // element programs of one cluster that yield a value each
constexpr int kInterpDepth = 6;       // values below the top of the interpreter's stack
constexpr int kInterpGathers = 3;     // nesting of gathers it follows
enum : unsigned char {
  kCodeEnd = 0,
  kCodeIn,      // a = external array: push its element at the position; b = 1 + k: it is array direct[k] of its
                // element program, read at the element's own position (KArgs::direct)
  kCodeGen,     // a = index function, b = slot: push its value at the position
  kCodeMap,     // a = element function, b = slot, c = number of arguments: replace them by the result
  kCodeEnter,   // pop an index and make it the position
  kCodeLeave,   // back to the position before the matching kCodeEnter
  kCodeLookup,  // a = external array, b = 1 + k: push its element at the index that array direct[k] (c) holds
  kCodeStore,   // a = output array: pop a value into it at the element's own position
  kCodeFold,    // a = output array, b = reducer (kFold...), c = accumulator: pop a value into it
  kCodeYield,   // the value on the stack is the result of this element program (Interp<K, T>)
  kCodeTable    // push what kCodeLookup would, from where the kernel has left it (interp_table_kernel)
};
// in Code::op of a store or a fold: the value stays on the stack (an array with several consumers is computed once)
constexpr unsigned char kCodeStays = 0x80;
constexpr int kInterpFolds = 2;       // folds of one interpreted cluster
constexpr int kInterpDirect = 4;      // arrays of an element program that are read ahead of its run
enum : unsigned char { kFoldAddF32 = 0, kFoldMaxF32, kFoldMulF32, kFoldAddI32, kFoldMaxI32 };
struct Code { unsigned char op, a, b, c; };

// What an interpreted program needs before its first read of an array comes first, in as few cache lines as it fits: a
// launch finds its arguments in no cache.
struct KArgs {    // arguments of one cluster launch
  int n;                    // iteration size
  unsigned grid;            // workgroups of the launch (see below, kernel arguments)
  unsigned flags;           // kSinglePass: a fold of the cluster carries FC_NODE_SINGLE_PASS;
                            // kKeepOut << k: out[k] is read back by a later cluster of the program
  unsigned char n_folds, fold_op[kInterpFolds], fold_out[kInterpFolds];   // of a cluster that interp_kernel runs
  unsigned char code_depth, code_gathers;   // values below the top of the stack and nested gathers that `code` needs
  const void *ahead[kInterpDirect];         // the arrays direct[0] names, where the kernel's launch has put them
  const void *in[kMaxIn];   // external arrays read by the cluster
  void *out[kMaxOut];       // arrays the cluster writes
  Code code[kMaxCode];      // kCodeEnd after the last instruction
  int w;                    // inner extent of 2-D index functions (1 for 1-D)
  int h;                    // outer extent
  int aux;                  // skeleton specific (rows of a segmented fold, ...)
  unsigned lookup_elems;    // elements of the array that the first kCodeLookup reads from, 0: there is none
  Slot p[kMaxSlots];
  unsigned root[kMaxRoots];        // where element program K of a cluster with another consumer starts in `code`
  // External arrays that element program K reads at the element's own position (the first kInterpDirect of
  // them): known before the program runs, so their reads are issued together and ahead of it.
  unsigned char direct[kMaxRoots][kInterpDirect], n_direct[kMaxRoots];
  // An instruction as one word: at an index that is the same for all lanes a scalar read, where the compiler may read
  // four bytes through the vector unit (row scans of 2^24 interpreted elements 107 us, with words 101).
  __device__ __forceinline__ Code code_word(int pc) const {
    unsigned word;
    __builtin_memcpy(&word, __builtin_assume_aligned(&code[pc], 4), sizeof(word));
    return {(unsigned char)word, (unsigned char)(word >> 8), (unsigned char)(word >> 16), (unsigned char)(word >> 24)};
  }
  void set_grid(unsigned workgroups) { grid = workgroups; }
  __host__ __device__ bool keeps(int k) const { return (flags >> (8 + k)) & 1u; }
};
constexpr unsigned kSinglePass = 1u;
constexpr unsigned kKeepOut = 1u << 8;

template <class T> struct Vec4 { T v[4]; };
// Four elements in memory, at any 4-byte boundary: one 128-bit access.  A typedef: the compiler drops `aligned`
// from an alias declaration, and the type would promise 16 bytes.
template <class T> struct Quad128Of { typedef T type __attribute__((ext_vector_type(4), aligned(4))); };
template <class T> using Quad128 = typename Quad128Of<T>::type;
static_assert(alignof(Quad128<float>) == 4 && alignof(Quad128<int>) == 4 && alignof(Quad128<unsigned>) == 4, "any 4-byte boundary");

template <class T> struct DtypeName;
template <> struct DtypeName<float> { static const char *s() { return "f32"; } };
template <> struct DtypeName<int> { static const char *s() { return "i32"; } };

// ------------------------------------------------------------------ element functions
struct FnIdentF { using R = float; static constexpr int kFn = FC_FN_IDENT;
  static __device__ __forceinline__ R apply(const Slot &, float x) { return x; } };
struct FnIdentI { using R = int; static constexpr int kFn = FC_FN_IDENT;
  static __device__ __forceinline__ R apply(const Slot &, int x) { return x; } };
struct FnAffine { using R = float; static constexpr int kFn = FC_FN_AFFINE;
  static __device__ __forceinline__ R apply(const Slot &s, float x) { float t = s.f[0] * x; return t + s.f[1]; } };
struct FnSinXMulX { using R = float; static constexpr int kFn = FC_FN_SIN_X_MUL_X;
  static __device__ __forceinline__ R apply(const Slot &, float x) { return sinf(x) * x; } };
struct FnSqPlusOne { using R = float; static constexpr int kFn = FC_FN_SQ_PLUS_ONE;
  static __device__ __forceinline__ R apply(const Slot &, float x) { float t = x * x; return t + 1.0f; } };
struct FnMul2 { using R = float; static constexpr int kFn = FC_FN_MUL2;
  static __device__ __forceinline__ R apply(const Slot &, float a, float b) { return a * b; } };
struct FnAdd2 { using R = float; static constexpr int kFn = FC_FN_ADD2;
  static __device__ __forceinline__ R apply(const Slot &, float a, float b) { return a + b; } };
struct FnAdd3 { using R = float; static constexpr int kFn = FC_FN_ADD3;
  static __device__ __forceinline__ R apply(const Slot &, float a, float b, float c) { return (a + b) + c; } };
struct FnAdd5 { using R = float; static constexpr int kFn = FC_FN_ADD5;
  static __device__ __forceinline__ R apply(const Slot &, float a, float b, float c, float d, float e) {
    return (((a + b) + c) + d) + e; } };
struct FnExpNeg { using R = float; static constexpr int kFn = FC_FN_EXP_NEG;
  static __device__ __forceinline__ R apply(const Slot &, float x) { return expf(-x); } };
struct FnModEq { using R = int; static constexpr int kFn = FC_FN_MOD_EQ;
  static __device__ __forceinline__ R apply(const Slot &s, int x) {
    const unsigned t = (unsigned)x - (unsigned)s.i[1];
    const unsigned p = t * s.m[0];
    const unsigned q = __builtin_amdgcn_alignbit(p, p, s.m[1]);     // rotate right
    return (int)((unsigned)((unsigned)x >= (unsigned)s.i[1]) & (unsigned)(q <= s.m[2])); } };   // no branch: both tests always

// i / d for 0 <= i < 2^31 and a divisor that is fixed for the launch, without a
// division: with L = ceil(log2 d) and M = ceil(2^(31+L) / d) < 2^32 the quotient is
// (i * M) >> (31 + L) (division by an invariant integer through multiplication).
// The index functions divide every element index by a row length; the compiler
// turns a division by a run-time value into some forty instructions.
inline void div_constants(Slot &s, int d) {
  unsigned L = 0;
  while ((1ull << L) < (unsigned long long)(d > 0 ? d : 1)) ++L;
  const unsigned long long two = 1ull << (31 + L), dd = (unsigned long long)(d > 0 ? d : 1);
  s.m[0] = (unsigned)((two + dd - 1) / dd);
  s.m[1] = 31 + L;
}
__device__ __forceinline__ int fast_div(const Slot &s, int i) {
  return (int)(((unsigned long long)(unsigned)i * s.m[0]) >> s.m[1]);
}

// element functions whose result is 0 or 1
template <class E> struct YieldsZeroOne { static constexpr bool value = false; };

// index functions of generate
struct GenIota { static constexpr int kFn = FC_FN_IOTA;
  static __device__ __forceinline__ int apply(const Slot &, const KArgs &, int i) { return i; } };
struct GenIotaRev { static constexpr int kFn = FC_FN_IOTA_REV;
  static __device__ __forceinline__ int apply(const Slot &s, const KArgs &, int i) { return s.ext[0] * s.ext[1] - 1 - i; } };
struct GenClampShift2D { static constexpr int kFn = FC_FN_CLAMP_SHIFT_2D;
  static __device__ __forceinline__ int apply(const Slot &s, const KArgs &, int i) {
    const int h = s.ext[0], w = s.ext[1];
    int r = fast_div(s, i), c = i - r * w;
    r = min(max(r + s.i[0], 0), h - 1);
    c = min(max(c + s.i[1], 0), w - 1);
    return r * w + c; } };
struct GenRowOf2D { static constexpr int kFn = FC_FN_ROW_OF_2D;
  static __device__ __forceinline__ int apply(const Slot &s, const KArgs &, int i) { return fast_div(s, i); } };
struct GenConst { static constexpr int kFn = FC_FN_CONST_I32;
  static __device__ __forceinline__ int apply(const Slot &s, const KArgs &, int) { return s.i[0]; } };

// ------------------------------------------------------------------ expression nodes
// external array number K of the cluster, element type T
template <int K, class T>
struct In {
  using R = T;
  static constexpr int kNodes = 1;
  static constexpr bool kMirror = false;
  // Stream: the element is read once, in order (non-temporal: it does not displace
  // gathered arrays from the caches); a gather turns it off for its source
  template <int Base, bool Stream = false> static __device__ __forceinline__ T eval(const KArgs &a, int i) {
    const T *p = static_cast<const T *>(a.in[K]) + i;
    return Stream ? __builtin_nontemporal_load(p) : *p;
  }
  template <int Base> static __device__ __forceinline__ Vec4<T> eval4(const KArgs &a, int i) {
    const Quad128<T> v = __builtin_nontemporal_load(reinterpret_cast<const Quad128<T> *>(static_cast<const T *>(a.in[K]) + i));
    return Vec4<T>{{v.x, v.y, v.z, v.w}};
  }
  template <int Base>
  static __device__ __forceinline__ void eval4_pair(const KArgs &a, int i, int ip, Vec4<T> &at_i, Vec4<T> &at_ip) {
    at_i = eval4<Base>(a, i);
    at_ip = eval4<Base>(a, ip);
  }
  template <int Base> static __device__ __forceinline__ bool mirrors_whole(const KArgs &, int) { return true; }
  static void sig(std::string &s) { s += "in" + std::to_string(K) + ":" + DtypeName<T>::s(); }
};

template <int Base, int K, class... E> struct ChildBase;
template <int Base, class E0, class... E> struct ChildBase<Base, 0, E0, E...> { static constexpr int value = Base; };
template <int Base, int K, class E0, class... E> struct ChildBase<Base, K, E0, E...> {
  static constexpr int value = ChildBase<Base + E0::kNodes, K - 1, E...>::value;
};

template <class F, class... E>
struct Map {
  using R = typename F::R;
  static constexpr int kNodes = 1 + (E::kNodes + ... + 0);
  static constexpr bool kMirror = (E::kMirror || ... || false);
  template <int Base, bool Stream, int... K>
  static __device__ __forceinline__ R eval_(const KArgs &a, int i, std::integer_sequence<int, K...>) {
    return F::apply(a.p[Base], E::template eval<ChildBase<Base + 1, K, E...>::value, Stream>(a, i)...);
  }
  template <int Base, bool Stream = false> static __device__ __forceinline__ R eval(const KArgs &a, int i) {
    return eval_<Base, Stream>(a, i, std::make_integer_sequence<int, sizeof...(E)>());
  }
  template <int Base, int... K>
  static __device__ __forceinline__ Vec4<R> eval4_(const KArgs &a, int i, std::integer_sequence<int, K...>) {
    auto t = std::make_tuple(E::template eval4<ChildBase<Base + 1, K, E...>::value>(a, i)...);
    Vec4<R> r;
#pragma unroll
    for (int c = 0; c < 4; ++c) r.v[c] = F::apply(a.p[Base], std::get<K>(t).v[c]...);
    return r;
  }
  template <int Base> static __device__ __forceinline__ Vec4<R> eval4(const KArgs &a, int i) {
    return eval4_<Base>(a, i, std::make_integer_sequence<int, sizeof...(E)>());
  }
  template <int Base, int... K>
  static __device__ __forceinline__ void eval4_pair_(const KArgs &a, int i, int ip, Vec4<R> &at_i, Vec4<R> &at_ip,
                                                     std::integer_sequence<int, K...>) {
    std::tuple<Vec4<typename E::R>...> x, xp;
    (E::template eval4_pair<ChildBase<Base + 1, K, E...>::value>(a, i, ip, std::get<K>(x), std::get<K>(xp)), ...);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      at_i.v[c] = F::apply(a.p[Base], std::get<K>(x).v[c]...);
      at_ip.v[c] = F::apply(a.p[Base], std::get<K>(xp).v[c]...);
    }
  }
  template <int Base>
  static __device__ __forceinline__ void eval4_pair(const KArgs &a, int i, int ip, Vec4<R> &at_i, Vec4<R> &at_ip) {
    eval4_pair_<Base>(a, i, ip, at_i, at_ip, std::make_integer_sequence<int, sizeof...(E)>());
  }
  template <int Base, int... K>
  static __device__ __forceinline__ bool mirrors_whole_(const KArgs &a, int n, std::integer_sequence<int, K...>) {
    return (E::template mirrors_whole<ChildBase<Base + 1, K, E...>::value>(a, n) && ... && true);
  }
  template <int Base> static __device__ __forceinline__ bool mirrors_whole(const KArgs &a, int n) {
    return mirrors_whole_<Base>(a, n, std::make_integer_sequence<int, sizeof...(E)>());
  }
  static void sig(std::string &s) {
    s += "map" + std::to_string(F::kFn) + "(";
    bool first = true;
    ((s += (first ? "" : ","), first = false, E::sig(s)), ...);
    s += ")";
  }
};

template <class... E> struct YieldsZeroOne<Map<FnModEq, E...>> { static constexpr bool value = true; };

template <class G>
struct Gen {
  using R = int;
  static constexpr int kNodes = 1;
  static constexpr bool kMirror = false;
  template <int Base, bool Stream = false> static __device__ __forceinline__ int eval(const KArgs &a, int i) {
    return G::apply(a.p[Base], a, i);
  }
  template <int Base> static __device__ __forceinline__ Vec4<int> eval4(const KArgs &a, int i) {
    Vec4<int> r;
#pragma unroll
    for (int c = 0; c < 4; ++c) r.v[c] = G::apply(a.p[Base], a, i + c);
    return r;
  }
  template <int Base>
  static __device__ __forceinline__ void eval4_pair(const KArgs &a, int i, int ip, Vec4<int> &at_i, Vec4<int> &at_ip) {
    at_i = eval4<Base>(a, i);
    at_ip = eval4<Base>(a, ip);
  }
  template <int Base> static __device__ __forceinline__ bool mirrors_whole(const KArgs &, int) { return true; }
  static void sig(std::string &s) { s += "gen" + std::to_string(G::kFn); }
};

// the constant 1: stands for the flag of a scatter that has none (takes no parameter slot)
struct AlwaysOne {
  using R = int;
  static constexpr int kNodes = 0;
  static constexpr bool kMirror = false;
  template <int Base, bool Stream = false> static __device__ __forceinline__ int eval(const KArgs &, int) { return 1; }
  template <int Base> static __device__ __forceinline__ Vec4<int> eval4(const KArgs &, int) { return Vec4<int>{{1, 1, 1, 1}}; }
  template <int Base>
  static __device__ __forceinline__ void eval4_pair(const KArgs &, int, int, Vec4<int> &at_i, Vec4<int> &at_ip) {
    at_i = at_ip = Vec4<int>{{1, 1, 1, 1}};
  }
  template <int Base> static __device__ __forceinline__ bool mirrors_whole(const KArgs &, int) { return true; }
  static void sig(std::string &s) { s += "1"; }
};

// EI yields the index, ES is evaluated there
template <class EI, class ES>
struct Gather {
  using R = typename ES::R;
  static constexpr int kNodes = 1 + EI::kNodes + ES::kNodes;
  static constexpr bool kMirror = EI::kMirror || ES::kMirror;
  template <int Base, bool Stream = false> static __device__ __forceinline__ R eval(const KArgs &a, int i) {
    int j = EI::template eval<Base + 1, Stream>(a, i);
    return ES::template eval<Base + 1 + EI::kNodes>(a, j);
  }
  template <int Base> static __device__ __forceinline__ Vec4<R> eval4(const KArgs &a, int i) {
    Vec4<int> j = EI::template eval4<Base + 1>(a, i);
    Vec4<R> r;
#pragma unroll
    for (int c = 0; c < 4; ++c) r.v[c] = ES::template eval<Base + 1 + EI::kNodes>(a, j.v[c]);
    return r;
  }
  template <int Base>
  static __device__ __forceinline__ void eval4_pair(const KArgs &a, int i, int ip, Vec4<R> &at_i, Vec4<R> &at_ip) {
    at_i = eval4<Base>(a, i);
    at_ip = eval4<Base>(a, ip);
  }
  // a `reverse` below an arbitrary gather is evaluated at gathered positions: it pairs with nothing
  template <int Base> static __device__ __forceinline__ bool mirrors_whole(const KArgs &a, int n) {
    return EI::template mirrors_whole<Base + 1>(a, n) && !ES::kMirror;
  }
  static void sig(std::string &s) {
    s += "gather(";
    EI::sig(s);
    s += ",";
    ES::sig(s);
    s += ")";
  }
};

// `reverse` (section 2, gather: the index is generate(n-1-i)): the source is read
// backwards, so four consecutive results are one 128-bit read of the source,
// taken in the opposite order.
template <class ES>
struct Gather<Gen<GenIotaRev>, ES> {
  using R = typename ES::R;
  using EI = Gen<GenIotaRev>;
  static constexpr int kNodes = 1 + EI::kNodes + ES::kNodes;
  static constexpr bool kMirror = true;
  template <int Base, bool Stream = false> static __device__ __forceinline__ R eval(const KArgs &a, int i) {
    int j = EI::template eval<Base + 1, Stream>(a, i);
    return ES::template eval<Base + 1 + EI::kNodes>(a, j);
  }
  template <int Base> static __device__ __forceinline__ Vec4<R> eval4(const KArgs &a, int i) {
    const int total = a.p[Base + 1].ext[0] * a.p[Base + 1].ext[1];
    Vec4<R> r;
    const Vec4<R> v = ES::template eval4<Base + 1 + EI::kNodes>(a, total - 4 - i);
#pragma unroll
    for (int c = 0; c < 4; ++c) r.v[c] = v.v[3 - c];
    return r;
  }
  // Over exactly n elements (mirrors_whole) the group that `reverse` reads
  // for position i is the one at ip taken backwards, and the other way round: the source is
  // evaluated at the same two groups as a direct read of it, with the roles swapped, so that the
  // reads of an array which the program takes forwards and backwards coincide (same addresses in
  // the same registers: each is issued once).
  template <int Base>
  static __device__ __forceinline__ void eval4_pair(const KArgs &a, int i, int ip, Vec4<R> &at_i, Vec4<R> &at_ip) {
    Vec4<R> v, vp;
    ES::template eval4_pair<Base + 1 + EI::kNodes>(a, ip, i, v, vp);     // v: source at ip, vp: source at i
#pragma unroll
    for (int c = 0; c < 4; ++c) { at_i.v[c] = v.v[3 - c]; at_ip.v[c] = vp.v[3 - c]; }
  }
  template <int Base> static __device__ __forceinline__ bool mirrors_whole(const KArgs &a, int n) {
    return a.p[Base + 1].ext[0] * a.p[Base + 1].ext[1] == n && ES::template mirrors_whole<Base + 1 + EI::kNodes>(a, n);
  }
  static void sig(std::string &s) {
    s += "gather(";
    EI::sig(s);
    s += ",";
    ES::sig(s);
    s += ")";
  }
};

// Does the element program read at positions that an array holds (any gather but `reverse`)?
template <class E> struct ReadsAnywhere { static constexpr bool value = false; };
template <class F, class... E> struct ReadsAnywhere<Map<F, E...>> { static constexpr bool value = (ReadsAnywhere<E>::value || ... || false); };
template <class EI, class ES> struct ReadsAnywhere<Gather<EI, ES>> { static constexpr bool value = true; };
template <class ES> struct ReadsAnywhere<Gather<Gen<GenIotaRev>, ES>> { static constexpr bool value = ReadsAnywhere<ES>::value; };

// GatherChain<E> describes an element program that is a chain of one-argument maps over one
// gather whose index is an external array read in order and whose source is again a chain of
// one-argument maps over one external array (the table).  Its value at a position depends on
// the index found there and on nothing else, which lets a commutative consumer visit the
// positions in any order.  leaf() reads the table, from_leaf<Base>() applies the maps to what
// was read, so a kernel can issue many table reads before it uses the first.
template <class E> struct GatherChain;            // only the shapes below
template <int K, class T> struct GatherChain<In<K, T>> {
  using Leaf = T;
  static constexpr int kTable = K;
  static constexpr int kIndex = -1;               // no gather at or below this node
  template <int Base> static constexpr int source_slot() { return -1; }
  static __device__ __forceinline__ T leaf(const KArgs &a, int j) { return static_cast<const T *>(a.in[K])[j]; }
  template <int Base> static __device__ __forceinline__ T from_leaf(const KArgs &, T x) { return x; }
};
template <class F, class E0> struct GatherChain<Map<F, E0>> {
  using Inner = GatherChain<E0>;
  using Leaf = typename Inner::Leaf;
  static constexpr int kTable = Inner::kTable;
  static constexpr int kIndex = Inner::kIndex;
  template <int Base> static constexpr int source_slot() { return Inner::template source_slot<Base + 1>(); }
  static __device__ __forceinline__ Leaf leaf(const KArgs &a, int j) { return Inner::leaf(a, j); }
  template <int Base> static __device__ __forceinline__ typename F::R from_leaf(const KArgs &a, Leaf x) {
    return F::apply(a.p[Base], Inner::template from_leaf<Base + 1>(a, x));
  }
};
template <int KI, class ES> struct GatherChain<Gather<In<KI, int>, ES>> {
  using Inner = GatherChain<ES>;
  using Leaf = typename Inner::Leaf;
  static constexpr int kTable = Inner::kTable;
  static constexpr int kIndex = KI;
  template <int Base> static constexpr int source_slot() { return Base + 2; }     // gather, its index, then its source
  static __device__ __forceinline__ Leaf leaf(const KArgs &a, int j) { return Inner::leaf(a, j); }
  template <int Base> static __device__ __forceinline__ typename ES::R from_leaf(const KArgs &a, Leaf x) {
    return Inner::template from_leaf<Base + 2>(a, x);
  }
};

// ------------------------------------------------------------------ kernel arguments
// A launch writes its arguments across the bus a cache line at a time, and a small program's pass costs little
// else: a kernel of 48 bytes of arguments takes the host 2.6 us to launch, one of 376 bytes 3.3 to 3.7, one of 1432 (KArgs
// as a whole) 3.3 to 3.9.  So the kernels whose element programs are compiled take the parts of KArgs
// these programs use, as Packed<...>, and open() puts them back where the program looks for them (registers:
// every index is known when the kernel is compiled).  The number of workgroups is one of the arguments: a kernel that
// asks for gridDim has another 256 bytes of arguments that the launch fills in (an empty kernel of 48 bytes of arguments
// 2.42 us a launch without and 2.85 with them, of 64 bytes 2.42 and 3.07).
template <int K, class T, int Threads, int Columns> struct Interp;        // kernels.hpp: reads KArgs::code, needs all of it

// the fields of a Slot as words: f[0], f[1], i[0], i[1], ext[0], ext[1], m[0], m[1], m[2]
constexpr int kSlotWords = 9;
constexpr unsigned kWordsF = 3u, kWordsI = 3u << 2, kWordsExt = 3u << 4, kWordsM01 = 3u << 6, kWordM2 = 1u << 8;
template <class F> struct SlotUse { static constexpr unsigned value = 0; };
template <> struct SlotUse<FnAffine> { static constexpr unsigned value = kWordsF; };
template <> struct SlotUse<FnModEq> { static constexpr unsigned value = 1u << 3 | kWordsM01 | kWordM2; };
template <> struct SlotUse<GenIotaRev> { static constexpr unsigned value = kWordsExt; };
template <> struct SlotUse<GenClampShift2D> { static constexpr unsigned value = kWordsI | kWordsExt | kWordsM01; };
template <> struct SlotUse<GenRowOf2D> { static constexpr unsigned value = kWordsM01; };
template <> struct SlotUse<GenConst> { static constexpr unsigned value = 1u << 2; };

struct WordList {
  int n = 0;
  short at[kMaxSlots * kSlotWords + 8] = {};
  constexpr void add(int w) { at[n++] = (short)w; }
  constexpr void add_slot(int slot, unsigned use) {
    for (int k = 0; k < kSlotWords; ++k) if (use >> k & 1u) add(slot * kSlotWords + k);
  }
};

// what element program E reads: external arrays 0 .. ins-1, words of its slots, or everything
template <class E> struct Needs {
  static constexpr int ins = 0;
  static constexpr bool all = false;
  template <int Base> static constexpr void words(WordList &) {}
};
template <int K, class T, int N, int C> struct Needs<Interp<K, T, N, C>> : Needs<void> { static constexpr bool all = true; };
template <int K, class T> struct Needs<In<K, T>> : Needs<void> { static constexpr int ins = K + 1; };
template <class G> struct Needs<Gen<G>> : Needs<void> {
  template <int Base> static constexpr void words(WordList &l) { l.add_slot(Base, SlotUse<G>::value); }
};
constexpr int most_of() { return 0; }
template <class... I> constexpr int most_of(int a, I... b) { const int m = most_of(b...); return a > m ? a : m; }
template <class F, class... E> struct Needs<Map<F, E...>> {
  static constexpr int ins = most_of(Needs<E>::ins...);
  static constexpr bool all = (Needs<E>::all || ... || false);
  template <int Base, int... K> static constexpr void words_(WordList &l, std::integer_sequence<int, K...>) {
    (Needs<E>::template words<ChildBase<Base + 1, K, E...>::value>(l), ...);
  }
  template <int Base> static constexpr void words(WordList &l) {
    l.add_slot(Base, SlotUse<F>::value);
    words_<Base>(l, std::make_integer_sequence<int, sizeof...(E)>());
  }
};
template <class EI, class ES> struct Needs<Gather<EI, ES>> {
  static constexpr int ins = most_of(Needs<EI>::ins, Needs<ES>::ins);
  static constexpr bool all = Needs<EI>::all || Needs<ES>::all;
  template <int Base> static constexpr void words(WordList &l) {
    Needs<EI>::template words<Base + 1>(l);
    Needs<ES>::template words<Base + 1 + EI::kNodes>(l);
  }
};

// Head: numbers of KArgs the kernel itself reads.  Outs: bit k = it writes out[k].  E: its element programs, whose slots
// follow each other.
constexpr unsigned kHeadN = 1u, kHeadW = 2u, kHeadH = 4u, kHeadAux = 8u, kHeadFlags = 16u, kHeadOffsets = 32u;
template <unsigned Head, unsigned Outs, bool All, class... E> struct PackedArgs {
  static constexpr int kIns = most_of(Needs<E>::ins...) + ((Head & kHeadOffsets) ? 1 : 0);
  static constexpr int kOuts = __builtin_popcount(Outs);
  static constexpr int kHeadWord = kMaxSlots * kSlotWords;
  template <int Base, class E0, class... R> static constexpr void add_programs(WordList &l) {
    Needs<E0>::template words<Base>(l);
    if constexpr (sizeof...(R) != 0) add_programs<Base + E0::kNodes, R...>(l);
  }
  static constexpr WordList make_list() {
    WordList l;
    for (int k = 0; k < 5; ++k) if (Head >> k & 1u) l.add(kHeadWord + k);
    if constexpr (sizeof...(E) != 0) add_programs<0, E...>(l);
    return l;
  }
  static constexpr WordList kList = make_list();
  const void *in[kIns ? kIns : 1];
  void *out[kOuts ? kOuts : 1];
  unsigned grid;
  unsigned word[kList.n ? kList.n : 1];

  // word W of KArgs, read or written
  template <int W, class A, class V> static __host__ __device__ __forceinline__ void visit(A &a, V &&v) {
    if constexpr (W >= kHeadWord) {
      constexpr int k = W - kHeadWord;
      if constexpr (k == 0) v(a.n); else if constexpr (k == 1) v(a.w); else if constexpr (k == 2) v(a.h); else if constexpr (k == 3) v(a.aux); else v(a.flags);
    } else {
      constexpr int s = W / kSlotWords, k = W % kSlotWords;
      if constexpr (k < 2) v(a.p[s].f[k]); else if constexpr (k < 4) v(a.p[s].i[k - 2]); else if constexpr (k < 6) v(a.p[s].ext[k - 4]); else v(a.p[s].m[k - 6]);
    }
  }
  template <int... I> void pack_words(const KArgs &a, std::integer_sequence<int, I...>) {
    (visit<kList.at[I]>(a, [&](const auto &x) { word[I] = __builtin_bit_cast(unsigned, x); }), ...);
  }
  template <int... I> __device__ __forceinline__ void open_words(KArgs &a, std::integer_sequence<int, I...>) const {
    (visit<kList.at[I]>(a, [&](auto &x) { x = __builtin_bit_cast(typename std::remove_reference<decltype(x)>::type, word[I]); }), ...);
  }
  PackedArgs(const KArgs &a) {
    for (int k = 0; k < kIns; ++k) in[k] = a.in[k];
    if (Head & kHeadOffsets) in[kIns - 1] = a.in[kMaxIn - 1];
    for (int k = 0, o = 0; k < kMaxOut; ++k) if (Outs >> k & 1u) out[o++] = a.out[k];
    pack_words(a, std::make_integer_sequence<int, kList.n>());
  }
  void set_grid(unsigned workgroups) { grid = workgroups; }
  __device__ __forceinline__ KArgs open() const {
    KArgs a;
#pragma unroll
    for (int k = 0; k < kIns; ++k) a.in[(Head & kHeadOffsets) && k == kIns - 1 ? kMaxIn - 1 : k] = in[k];
    int o = 0;
#pragma unroll
    for (int k = 0; k < kMaxOut; ++k) if (Outs >> k & 1u) a.out[k] = out[o++];
    a.grid = grid;
    open_words(a, std::make_integer_sequence<int, kList.n>());
    return a;
  }
  __device__ __forceinline__ KArgs in_place() const { return open(); }
};
template <unsigned Head, unsigned Outs, class... E> struct PackedArgs<Head, Outs, true, E...> {
  KArgs args;
  PackedArgs(const KArgs &a) : args(a) {}
  void set_grid(unsigned workgroups) { args.set_grid(workgroups); }
  __device__ __forceinline__ const KArgs &open() const { return args; }
  // The same, where the launch has put them (every kernel that takes one has it as its first argument).  From a parameter that
  // a kernel reads at more than some 300 places, as the scatters do, every lane has a copy of it made in its own memory (1336 bytes;
  // us a pass with the copy / in place, permuted by an index array: 5003 elements 18.7 / 6.8, 2^22 164 / 64, 2^24 546 / 225).
  // For the other skeletons the parameter is the better one (compaction of 3 x 10^6 elements 42.3 us, in place 44.1).
  static __device__ __forceinline__ const KArgs &in_place() {
    return *(const KArgs *)(const __attribute__((address_space(4))) KArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  }
};
template <unsigned Head, unsigned Outs, class... E> using Packed = PackedArgs<Head, Outs, (Needs<E>::all || ... || false), E...>;

}  // namespace fc
