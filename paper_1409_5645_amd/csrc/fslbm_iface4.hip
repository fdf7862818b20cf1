// Interface cells of the step with four lanes per cell (a quad), for the
// rules and forms of the plain step (no moving walls, surface tension, PLIC or
// solid cells, no adjoint record; those take k_iface).  Run before the sweep
// (SweepArgs::order), it takes the list the step before built and writes the
// populations into a list-ordered buffer that the sweep stores with its rows,
// instead of 19 scattered 2-, 4- or 8-byte stores per cell.
//
// The cell's update itself is iface4_cell (fslbm_iface4.hpp).
#include "fslbm_iface4.hpp"

#include <algorithm>

namespace fslbm {


constexpr int QBLOCK = 256;               // threads per block
constexpr int QCELLS = QBLOCK / QUAD;     // cells per block
constexpr unsigned IFACE4_GRID = 16384;   // blocks at most (grid-stride beyond); a multiple of NXCD

template <class F, int RULE, bool REC = false>
__global__ __launch_bounds__(QBLOCK) void k_iface4(SweepArgs a) {
  const Grid g = a.c.grid;
  const int n_i = a.counters[C_I];
  // before the sweep (order 1) this kernel opens the counters of the next step
  if (a.order && blockIdx.x == 0 && threadIdx.x == 0) {
#pragma unroll
    for (int c = 0; c < NCOUNT; ++c) a.counters_next[c] = 0;
  }
  iface4_list<F, RULE, REC>(a, g, n_i, QCELLS, (int)blockIdx.x, (int)gridDim.x, a.order != 0);
}

template <class F, int RULE, bool REC = false>
static void iface4_go(const StepLaunch& L) {
  // a window step's list is fixed and its length (rec_cap) known here
  const size_t cells = REC ? (size_t)L.sweep.rec_cap : (size_t)L.sweep.c.grid.N;
  unsigned nb = std::min<unsigned>(IFACE4_GRID, (unsigned)std::max<size_t>(1, (cells + QCELLS - 1) / QCELLS));
  nb = (nb + NXCD - 1) / NXCD * NXCD;
  k_iface4<F, RULE, REC><<<nb, QBLOCK, 0, (hipStream_t)L.stream>>>(L.sweep);
}

template <class F>
static void iface4_form(const StepLaunch& L, int rule) {
  if (L.sweep.rec_f) {  // a window step (rules 0 and 1)
    if (rule == 0) iface4_go<F, 0, true>(L);
    else iface4_go<F, 1, true>(L);
    return;
  }
  switch (rule) {
    case 0: iface4_go<F, 0>(L); break;
    case 1: iface4_go<F, 1>(L); break;
    case 2: iface4_go<F, 2>(L); break;
    case 3: iface4_go<F, 3>(L); break;
    case 4: iface4_go<F, 4>(L); break;
    default: iface4_go<F, 5>(L); break;
  }
}

hipError_t launch_iface4(const StepLaunch& L, int precision, int rule) {
  if (precision == 0) iface4_form<FormF64>(L, rule);
  else if (precision == 1) iface4_form<FormF32>(L, rule);
  else iface4_form<FormF16>(L, rule);
  return hipGetLastError();
}

}  // namespace fslbm
