// Resident steps of small lattices: many time steps of the plain step (no
// moving walls, surface tension, PLIC, solid walls or prescribed surface) in
// one launch.
//
// A small lattice's step is a handful of microseconds of work behind five
// kernel launches, each with its own start, drain and gap.  Here a few
// workgroups stay on the device for a run of steps and meet at barriers in
// memory instead: one per step, after the interface and liquid cells (they
// read only time t, so they need no order between them), and more only where
// cells convert.  The interface cells come from a list that the conversions
// extend (an entry counts while its cell is an interface cell and islot points
// back at it); it is made anew when it could outgrow its 2 N entries.
//
// Every cell goes through the code of the kernels of the step-by-step form
// (iface4_cell, the conversion passes) or the same operations (bulk_cell), so
// the two give the same bits.
#include "fslbm_barrier.hpp"
#include "fslbm_convert.hpp"
#include "fslbm_iface4.hpp"

#include <algorithm>

namespace fslbm {

// Threads and workgroups: at most 16384 threads; more did not help lattices of
// this size (12,000 cells: 9.9 us a step with 32 workgroups and with 64).  The
// FP64 kernels with a boundary shear from the bulk take smaller workgroups,
// whose threads may hold the 350 registers they need: a compute unit each.  How
// many of them are on the device at once is found out by the kernel (join_team).
constexpr int RTHREADS = 16384;
template <class F, int RULE>
constexpr int rblock() {
  return sizeof(typename F::R) == 8 && (RULE & 2) ? 256 : 512;
}

// Element offsets of the 18 pulls of a cell: the source population, or beyond
// a wall the cell's own opposite one (halfway bounce-back).
__device__ __forceinline__ void pull_offsets(const Grid& g, int idx, unsigned (&off)[Q]) {
  Nbr n;
  coords(g, idx, n.x, n.y, n.z);
  n.xm = step_axis(n.x, -1, g.nx, g.px);
  n.xp = step_axis(n.x, 1, g.nx, g.px);
  n.ym = step_axis(n.y, -1, g.ny, g.py);
  n.yp = step_axis(n.y, 1, g.ny, g.py);
  n.zm = step_axis(n.z, -1, g.nz, g.pz);
  n.zp = step_axis(n.z, 1, g.nz, g.pz);
  const unsigned N = (unsigned)g.N;
  off[0] = (unsigned)idx;
#define FSLBM_ROFF(q)                                                                          \
  {                                                                                            \
    const int s = pull_source<q>(g, n);                                                        \
    off[q] = s >= 0 ? (unsigned)q * N + (unsigned)s : (unsigned)OPP[q] * N + (unsigned)idx;     \
  }
  FSLBM_LINKS(FSLBM_ROFF)
#undef FSLBM_ROFF
}

// Stream and collide of one liquid cell: the operations of k_sweep.
template <class F>
__device__ __forceinline__ void bulk_cell(const SweepArgs& a, const Grid& g, int idx, const unsigned (&off)[Q]) {
  using R = typename F::R;
  using S = typename F::S;
  const unsigned N = (unsigned)g.N;
  const S* fin = reinterpret_cast<const S*>(a.fin);
  S* fout = reinterpret_cast<S*>(a.fout);
  R f[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) f[q] = F::load_raw(fin + off[q]);
  const Consts<R>& k = pick_consts<R>(a.c);
  const bool incomp = a.c.incomp, stokes = a.c.stokes;
  R rho_s, u[3];
  if constexpr (sizeof(R) == 4)
    collide_f32_scaled<F::shifted, F::scaled>(f, k, incomp, stokes, a.c.scale, a.c.inv_scale, rho_s, u);
  else
    collide<R, F::shifted>(f, k, incomp, stokes, rho_s, u);
#pragma unroll
  for (int q = 0; q < Q; ++q) F::store_raw(fout + ((unsigned)q * N + (unsigned)idx), f[q]);
}

template <class F, int RULE>
__global__ __launch_bounds__((rblock<F, RULE>())) void k_resident(ResidentArgs r) {
  constexpr int RBLOCK = rblock<F, RULE>();
  const Grid g = r.sweep[0].c.grid;
  const uint8_t* flags = r.sweep[0].flags;
  const QuadLane<typename F::R> ql(g);
  if (blockIdx.x == 0 && threadIdx.x == 0) r.bar_next[0] = r.bar_next[TEAM_WORD] = 0ull;
  const Team team = join_team(r.bar + TEAM_WORD, min((unsigned)r.team, gridDim.x), r.team_wait, [&] {
    __hip_atomic_store(&r.len[C_I], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  });
  if (team.size == 0u) return;
  GridBarrier grid(r.bar, team);
  const int tid = (int)team.rank * RBLOCK + (int)threadIdx.x, nth = (int)team.size * RBLOCK;
  // threads for interface cells at most: half of the workgroups, or of the only one
  const int most = team.size > 1u ? (int)(team.size / 2u) * RBLOCK : RBLOCK / 2;
  int len = 0;
  bool rebuild = true;
  // The cell a thread works on and where it pulls from, kept from step to step
  // while the classes stay and a thread has one cell only (loading them anew
  // puts three dependent loads before the first population)
  bool changed = true;
  int idx = -1;
  QuadTopo tp;
  unsigned off[Q];
  for (int t = 0; t < r.n; ++t) {
    if (rebuild) {  // the interface cells of the current classes (uniform over the grid)
      if (t > 0) {
        grid.meet(false);  // every workgroup has read the old length
        if (tid == 0) __hip_atomic_store(&r.len[C_I], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        grid.meet(false);
      }
      for (int i0 = 0; i0 < g.N; i0 += nth) {
        const int i = i0 + tid;
        const bool it = i < g.N && flags[i] == IFACE;
        const int pos = wave_append_at(it, &r.len[C_I], r.list, i);
        if (it) r.islot[i] = pos;
      }
      grid.meet(false);
      len = peek(&r.len[C_I]);
      rebuild = false;
    }
    const SweepArgs& a = r.sweep[t & 1];
    const ConvArgs& v = r.conv[t & 1];
    const int step = r.step + t;
    if (tid < NCOUNT) a.counters_next[tid] = 0;
    // the interface cells to the first workgroups, four lanes each, the others
    // the liquid cells
    const int ni = min((QUAD * len + RBLOCK - 1) / RBLOCK * RBLOCK, most);
    bool conv = false;
    if (__builtin_amdgcn_readfirstlane(tid) < ni) {
      const int stride = ni / QUAD;
      for (int i = tid >> 2; i < len; i += stride) {
        if (changed || len > stride) {
          idx = r.list[i];
          // an entry whose cell left the interface since (quad-uniform)
          if (flags[idx] != IFACE || r.islot[idx] != i) idx = -1;
          else iface4_topo(a, g, ql, idx, tp);
        }
        if (idx < 0) continue;
        bool filled, emptied;
        iface4_cell<F, RULE, false>(a, g, ql, tp, step, i, idx, filled, emptied);
        if (!a.freeze) {
          wave_append(filled, &a.counters[C_F], a.listF, idx);
          wave_append(emptied, &a.counters[C_E], a.listE, idx);
          conv = conv || filled || emptied;
        }
      }
    } else {
      const int stride = nth - ni;
      for (int i = tid - ni; i < g.N; i += stride) {
        if (changed || g.N > stride) {
          idx = flags[i] == LIQ ? i : -1;
          if (idx >= 0) pull_offsets(g, idx, off);
        }
        if (idx >= 0) bulk_cell<F>(a, g, idx, off);
      }
    }
    changed = false;
    if (grid.meet(conv)) {
      convert_all<F, RBLOCK, false>(v, step, peek(&a.counters[C_F]), peek(&a.counters[C_E]), grid);
      grid.meet(false);
      len = peek(&r.len[C_I]);
      rebuild = len > g.N;
      changed = true;
    }
  }
}

template <class F, int RULE>
static void resident_go(const ResidentArgs& r, hipStream_t st) {
  constexpr unsigned B = rblock<F, RULE>();
  const unsigned cells = ((unsigned)r.sweep[0].c.grid.N + B - 1) / B;
  const unsigned nb = std::max(2u, std::min(RTHREADS / B, 2 * cells));
  k_resident<F, RULE><<<nb, B, 0, st>>>(r);
}

template <class F>
static void resident_form(const ResidentArgs& r, int rule, hipStream_t st) {
  switch (rule) {
    case 0: resident_go<F, 0>(r, st); break;
    case 1: resident_go<F, 1>(r, st); break;
    case 2: resident_go<F, 2>(r, st); break;
    case 3: resident_go<F, 3>(r, st); break;
    case 4: resident_go<F, 4>(r, st); break;
    default: resident_go<F, 5>(r, st); break;
  }
}

hipError_t launch_resident(const ResidentArgs& r, int precision, int rule, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (precision == 0) resident_form<FormF64>(r, rule, st);
  else if (precision == 1) resident_form<FormF32>(r, rule, st);
  else return hipErrorInvalidValue;  // FP16 storage has no resident form
  return hipGetLastError();
}

}  // namespace fslbm
