// Instances for elementwise clusters that no compiled one matches: their element programs are interpreted.
#include "interp.hpp"
#include "launchers.hpp"

#include <algorithm>

namespace fc {

namespace {

template <class... P> hipError_t launch_interp_as(void (*kernel)(P...), int tile, unsigned least, const KArgs &a, const LaunchCtx &c) {
  // a fold of the cluster keeps a partial per workgroup; there may be kInterpFolds of them
  const unsigned cap = std::min<unsigned>(resident_grid(kernel), kMaxPartials / kInterpFolds);
  return launch_k(kernel, std::max<unsigned>(grid_for(a.n, tile, cap), least), c, a, c.ctl, c.partials);
}
// Whether a program of kShortDepth or less whose first lookup goes to `elems` elements, n of them, is to take them from LDS.
// Filling the LDS of every compute unit costs about 3 us, and a lookup that hits L2 costs 1 us for 2.4 x 10^5 of them: worth
// it from 1.25 x 10^6 lookups on that find their element there (us a pass, from memory / from LDS: 2^20 lookups in 39000
// elements 10.1 / 9.7, 2^21 in 16384 12.5 / 11.9, in 65536 15.6 / 13.9, in 110000 (0.76 x 10^6 of them in LDS) 16.4 / 16.4, in 150000 (0.56)
// 16.7 / 17.4; 2^22 in 39000 26.1 / 18.5, in 65536 27.4 / 20.0, in 262144 28.6 / 28.5; 2^24 in 39000 90 / 43, in 65536 94 / 64).  Tables of
// less than 32 KiB are in the caches of the compute units as they are (1024 elements: 2^22 17.6 / 17.9, 2^23 27.3 / 26.6, 2^24 45.6 / 42.4).
// The lookups that find nothing there cost what they did, so their share does not matter: of 2^23 in 262144 elements 50.1 / 48.8, in
// 500000 (0.67 x 10^6 found) 50.4 / 51.6; 2^24 in 500000 96.3 / 96.2, in 10^6 (0.67) 113.8 / 112.9; 2^25 in 10^6 224 / 219; 2^27 in 4 x 10^6 (one
// in a hundred found) 1882 / 1855, in 8 x 10^6 2238 / 2208.
bool table_pays(unsigned n, unsigned elems) {
  const double found = (double)n * std::min(1.0, (double)kTableSlice / elems);
  return found >= (elems < 8192u ? 8.0e6 : 1.25e6);
}
// The kernel for a program, and where its first lookup stands (kMaxCode: it has none).
enum class Form { Long, General, Table, Short };
struct Choice { Form form; int lookup; };
Choice choose(const KArgs &a) {
  if (a.code_depth > kShortDepth || a.code_gathers > 1) return {Form::Long, kMaxCode};
  bool enters = false;
  int lookup = kMaxCode;
  for (int k = kMaxCode - 1; k >= 0; --k) {
    enters |= a.code[k].op == kCodeEnter;
    if (a.code[k].op == kCodeLookup) lookup = k;
  }
  // Programs of two arrays at most, one value below the top of the stack and no other gathers than lookups leave the registers for
  // the next tile's arrays; the others have them read when the tile before is done.
  if (a.n_direct[0] > 2 || a.code_depth > 1 || enters) return {Form::General, lookup};
  return {lookup < kMaxCode && table_pays((unsigned)a.n, a.lookup_elems) ? Form::Table : Form::Short, lookup};
}
hipError_t launch_interp(const KArgs &args, const LaunchCtx &c) {
  KArgs a = args;
  for (int k = 0; k < a.n_direct[0]; ++k) a.ahead[k] = a.in[a.direct[0][k]];
  const Choice choice = choose(a);
  // two groups a lane where the chip is full: the sharing of an instruction's cost begins to count there
  const bool two = a.n >= (1 << 20);
  switch (choice.form) {
    case Form::Long: return launch_interp_as(&interp_kernel, kBlock * kVec, 1, a, c);
    case Form::General:
      return two ? launch_interp_as(&interp_short_kernel<2, 4, 2, true, false>, kBlock * kVec * 2, 3, a, c)
                 : launch_interp_as(&interp_short_kernel<1, 4, 2, true, false>, kBlock * kVec, 1, a, c);
    case Form::Table: {
      a.code[choice.lookup].op = kCodeTable;
      const int cus = device_compute_units();
      const unsigned slabs = ((unsigned)a.n + kTableSlab - 1) / kTableSlab;
      return launch_threads(&interp_table_kernel, std::min(slabs, (unsigned)(cus > 0 ? cus : 256)), c, kTableBlock, a, c.ctl, c.partials,
                            (int)a.code[choice.lookup].a, a.lookup_elems);
    }
    default:
      return two ? launch_interp_as(&interp_short_kernel<2, 2, 1, false, true>, kBlock * kVec * 2, 3, a, c)
                 : launch_interp_as(&interp_short_kernel<1, 2, 1, false, true>, kBlock * kVec, 1, a, c);
  }
}
const char *form_name(const KArgs &a) {
  switch (choose(a).form) {
    case Form::Long: return "interpreted, long";
    case Form::Table: return "interpreted, lookups from LDS";
    default: return "interpreted";
  }
}

}  // namespace

const Instance *interpreter_instance() {
  static const Instance inst = [] {
    Instance i{"", &launch_interp};
    i.form = &form_name;
    return i;
  }();
  return &inst;
}

}  // namespace fc
