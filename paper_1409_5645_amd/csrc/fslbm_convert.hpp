// The conversions of a step after its interface cells are done (lists F and E
// built): three passes, each over the lists the passes before it made, with a
// barrier between them.
//
//   mark    E' = E minus N(F); claims the new interface cells: gas cells next
//           to filled cells, liquid cells next to E' cells.
//   share   excess of the filled and E' cells split over the neighbours that
//           are interface cells after the conversions (receivers listed); the
//           new interface cells initialised.
//   gather  receivers add their shares in ascending link order, fill refresh;
//           new cell classes.
//
// Thirty-two lanes take one listed cell, lane q its link q: a cell's eighteen
// neighbours are loaded by eighteen lanes at once, and what is needed of all
// of them is a ballot.  Few cells convert in a step, so the passes are chains
// of memory round trips through code that is not in the instruction cache:
// each pass is one or two trips and a few hundred instructions.  (With one
// thread per cell and link, every thread walking the eighteen neighbours in
// unrolled code, the passes took 8, 5 and 4 us for five converted cells.)
//
// A few converted cells are left to one workgroup (SOLO: list lengths in LDS,
// atomics that need not leave its L2), many are spread over a team of
// workgroups (convert_team).
#pragma once

#include "fslbm_barrier.hpp"
#include "fslbm_device.hpp"
#include "fslbm_internal.hpp"
#include "fslbm_quad.hpp"
#include "fslbm_stencil.hpp"

namespace fslbm {

constexpr int CLANES = 32;  // lanes per listed cell

template <bool SOLO>
__device__ __forceinline__ int exchange(int32_t* p, int v) {
  return __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, SOLO ? __HIP_MEMORY_SCOPE_WORKGROUP : __HIP_MEMORY_SCOPE_AGENT);
}

// The lane of a link: q = lane, its direction (0 for the rest lane and the
// idle lanes 19 .. 31) and that of the odd link of its pair.
struct LinkLane {
  int q, c[3], d[3];
  bool link;
  __device__ __forceinline__ LinkLane() {
    q = (int)threadIdx.x & (CLANES - 1);
    link = q >= 1 && q < Q;
    pair_dir(link ? (q - 1) >> 1 : 0, d);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      d[k] = link ? d[k] : 0;
      c[k] = (q & 1) ? d[k] : -d[k];
    }
  }
  // the lane's neighbour of cell idx (-1 beyond a wall, and for lanes without a link)
  __device__ __forceinline__ int neighbour(const Grid& g, int idx) const {
    int x, y, z;
    coords(g, idx, x, y, z);
    return link ? neighbor(g, x, y, z, c[0], c[1], c[2]) : -1;
  }
};

// ballot over the lanes of the cell
__device__ __forceinline__ uint32_t cell_ballot(bool p) {
  return (uint32_t)(__ballot(p) >> (threadIdx.x & (unsigned)CLANES));
}

// value of lane i of the cell's lanes
template <class T>
__device__ __forceinline__ T cell_lane(T v, int i) {
  return __shfl(v, i, CLANES);
}

// Mark of an E' cell in new_epoch: below every step stamp (>= 0) and the
// initial -1, and distinct for every step.  E' cells are interface cells and
// new_epoch's step stamps go to gas and liquid cells only.
__device__ __forceinline__ int ep_stamp(int step) { return -2 - step; }

// value[l] into list l (of L, whose counters are neighbours in cnt) for the lanes
// with pred[l] set.  BLOCK = 0: an atomic per wavefront and list; else one for the
// workgroup of BLOCK threads, the lists' at once, which every thread calls: the
// device serves atomics on one address one after another, and with one per
// wavefront a surface that converts as a whole queued there.
template <int BLOCK, int L>
__device__ __forceinline__ void append_to(const bool (&pred)[L], int32_t* cnt, int32_t* const (&list)[L], const int (&value)[L]) {
  if constexpr (BLOCK == 0) {
#pragma unroll
    for (int l = 0; l < L; ++l) wave_append(pred[l], &cnt[l], list[l], value[l]);
  } else {
    constexpr int WAVES = BLOCK / 64;
    __shared__ int32_t n[L][WAVES], first[L];
    const int w = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
    unsigned long long b[L];
#pragma unroll
    for (int l = 0; l < L; ++l) {
      b[l] = __ballot(pred[l]);
      if (lane == 0) n[l][w] = __popcll(b[l]);
    }
    __syncthreads();
    if (threadIdx.x < L) {
      int total = 0;
#pragma unroll
      for (int v = 0; v < WAVES; ++v) total += n[threadIdx.x][v];
      first[threadIdx.x] = total ? atomicAdd(&cnt[threadIdx.x], total) : 0;
    }
    __syncthreads();
#pragma unroll
    for (int l = 0; l < L; ++l) {
      if (!pred[l]) continue;
      int at = first[l] + __popcll(b[l] & ((1ull << lane) - 1ull));
#pragma unroll
      for (int v = 0; v < WAVES; ++v) at += v < w ? n[l][v] : 0;
      list[l][at] = value[l];
    }
    __syncthreads();  // (the next round's counts)
  }
}

// The passes: `first` is the workgroup's first group of lanes in the team,
// `groups` the team's; every workgroup's threads go through the same rounds.
// SOLO: one workgroup alone; BLOCK: see append_to.
template <bool SOLO, int BLOCK>
__device__ __forceinline__ void mark_pass(const ConvArgs& a, int step, int32_t* cnt, int nF, int nE, int first,
                                          int groups) {
  const Grid& g = a.c.grid;
  const LinkLane ln;
  const int n = nF + nE;
  static_assert(C_NI == C_EP + 1 && C_NL == C_EP + 2, "lists marked here");
  int32_t* const lists[3] = {a.listEP, a.listNI, a.listNL};
  const int mine = (int)threadIdx.x / CLANES;
  for (int e0 = first; e0 + (BLOCK == 0 ? mine : 0) < n; e0 += groups) {
    const int e = e0 + mine;
    const bool on = BLOCK == 0 || e < n, filled = e < nF;
    const int c = !on ? 0 : (filled ? a.listF[e] : a.listE[e - nF]);
    const int s = on ? ln.neighbour(g, c) : -1;
    const uint8_t ts = s >= 0 ? a.flags[s] : (uint8_t)SOLID;
    const int fe = s >= 0 ? a.f_epoch[s] : -1;
    // E' = E minus N(F)
    const bool drop = !filled && cell_ballot(fe == step) != 0u;
    const bool ep = on && !filled && !drop;
    if (ep && ln.q == 0) a.new_epoch[c] = ep_stamp(step);
    // Which lane wins a new cell's mark does not change the result
    bool win = false;
    if (on && (filled ? ts == GAS : (ep && ts == LIQ))) win = exchange<SOLO>(&a.new_epoch[s], step) != step;
    append_to<BLOCK>({ep && ln.q == 0, win && filled, win && !filled}, cnt + C_EP, lists, {c, s, s});
  }
}

// Whether cell t is an interface cell after this step's conversions: a new
// interface cell, or an interface cell of time t that neither filled nor is in
// E'.
__device__ __forceinline__ bool iface_after(const ConvArgs& a, int step, int t) {
  const int ne = a.new_epoch[t];
  const int fe = a.f_epoch[t];
  const uint8_t fl = a.flags[t];
  return (ne == step) | ((fl == IFACE) & (fe != step) & (ne != ep_stamp(step)));
}

// Excess of a converted cell c: split over its eligible neighbours (or handed
// to the reservoir).  Whether the lane's neighbour s is a receiver not yet listed.
template <bool SOLO>
__device__ __forceinline__ bool share_cell(const ConvArgs& a, int step, const LinkLane& ln, int c, bool filled,
                                           int& s) {
  s = ln.neighbour(a.c.grid, c);
  const bool el = (s >= 0) & iface_after(a, step, s >= 0 ? s : c);
  const double m = a.mass[c], r = a.aux[4 * (size_t)c];
  const int n_elig = __popc(cell_ballot(el));
  if (ln.q == 0) {
    const double ex = filled ? m - r : m;
    if (n_elig == 0) {
      atomicAdd(a.reservoir, ex);
      if (filled) a.mass[c] = ex;
    } else {
      a.mass[c] = ex / (double)n_elig;
      a.conv_epoch[c] = step;
    }
  }
  return el && exchange<SOLO>(&a.recv_epoch[s], step) != step;
}

// New interface cell from gas: f = f^eq of the mean collision density and
// velocity of the non-gas neighbours (summed in link order), mass 0.
template <class F>
__device__ __forceinline__ void init_from_gas(const ConvArgs& a, const LinkLane& ln, int c) {
  using R = typename F::R;
  using S = typename F::S;
  constexpr bool SH = F::shifted;
  const int s = ln.neighbour(a.c.grid, c);
  const uint8_t ts = s >= 0 ? a.flags[s] : (uint8_t)GAS;
  const double4 v = *reinterpret_cast<const double4*>(a.aux + 4 * (size_t)(s >= 0 ? s : c));
  uint32_t m = cell_ballot(ts != GAS && ts != SOLID);
  double rs = 0.0, us[3] = {0.0, 0.0, 0.0};
  const int cnt = __popc(m);
  for (; m != 0u; m &= m - 1u) {
    const int i = __ffs((int)m) - 1;
    rs = rs + cell_lane(v.x, i);
    us[0] = us[0] + cell_lane(v.y, i);
    us[1] = us[1] + cell_lane(v.z, i);
    us[2] = us[2] + cell_lane(v.w, i);
  }
  const double rbar = rs / (double)cnt;
  const Consts<R>& k = pick_consts<R>(a.c);
  const bool incomp = a.c.incomp, stokes = a.c.stokes;
  const R rho_s = SH ? (R)(rbar - 1.0) : (R)rbar;
  const R rho0 = rho0_of<R, SH>(rho_s, incomp);
  R u[3], w[3], d[3];  // equilibrium_post, a link per lane
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    u[i] = (R)(us[i] / (double)cnt);
    w[i] = u[i] + k.hg[i];
    d[i] = R(ln.d[i]);
  }
  const R wq = R(ln.q == 0 ? WD[0] : (ln.q <= 6 ? WD[1] : WD[7]));
  const R ep = e_plus_w(wq, ddot(d, u), rho_s, rho0, incomp, stokes, usq_of(u));
  R cu = ddot(d, w);
  if (!incomp) cu = rho0 * cu;
  const R em = R(ln.q <= 6 ? W3D[1] : W3D[7]) * cu;
  const R out = ln.q == 0 ? ep : ((ln.q & 1) ? ep + em : ep - em);
  if (ln.q < Q) F::store(reinterpret_cast<S*>(a.fout) + ((size_t)ln.q * a.c.grid.N + c), out, a.c.scale);
  if (ln.q == 0) {
    a.mass[c] = 0.0;
    a.aux[4 * (size_t)c] = rbar;
  }
}

// A new interface cell from liquid keeps its populations (of time t+1); m = rho.
template <class F>
__device__ __forceinline__ void init_from_liquid(const ConvArgs& a, const LinkLane& ln, int c) {
  using R = typename F::R;
  using S = typename F::S;
  const int q = ln.q < Q ? ln.q : 0;
  const R f = F::load(reinterpret_cast<const S*>(a.fout) + ((size_t)q * a.c.grid.N + c), a.c.inv_scale);
  double r = F::shifted ? 0.0 : (double)cell_lane(f, 0);
  for (int i = F::shifted ? 0 : 1; i < Q; ++i) r = r + (double)cell_lane(f, i);
  if (F::shifted) r = 1.0 + r;
  if (ln.q == 0) {
    a.mass[c] = r;
    a.aux[4 * (size_t)c] = r;
  }
}

template <class F, bool SOLO, int BLOCK>
__device__ __forceinline__ void share_pass(const ConvArgs& a, int step, int32_t* cnt, int nF, int nEP, int nNI,
                                           int nNL, int first, int groups) {
  const LinkLane ln;
  const int n0 = nF + nEP, n1 = n0 + nNI, n2 = n1 + nNL;
  int32_t* const lists[1] = {a.listR};
  const int mine = (int)threadIdx.x / CLANES;
  for (int e0 = first; e0 + (BLOCK == 0 ? mine : 0) < n2; e0 += groups) {
    const int e = e0 + mine;
    bool recv = false;
    int s = -1;
    if (e < n0) recv = share_cell<SOLO>(a, step, ln, e < nF ? a.listF[e] : a.listEP[e - nF], e < nF, s);
    else if (e < n1) init_from_gas<F>(a, ln, a.listNI[e - n0]);
    else if (e < n2) init_from_liquid<F>(a, ln, a.listNL[e - n1]);
    if (BLOCK == 0 || e0 < n0) append_to<BLOCK>({recv}, cnt + C_R, lists, {s});
  }
}

// Receivers, and the new cell classes (with the interface kernel first, the
// new interface cells also join the next list).
__device__ __forceinline__ void gather_pass(const ConvArgs& a, int step, int nR, int nF, int nEP, int nNI, int nNL,
                                            int len, unsigned tid, unsigned nth) {
  const LinkLane ln;
  for (int e = (int)(tid / CLANES); e < nR; e += (int)(nth / CLANES)) {
    const int r = a.listR[e];
    const int s = ln.neighbour(a.c.grid, r);
    const int ep = s >= 0 ? a.conv_epoch[s] : -1;
    const double mn = a.mass[s >= 0 ? s : r];
    const double rho = a.aux[4 * (size_t)r];
    double m = cell_lane(mn, 0);  // the rest lane has the receiver's own
    for (uint32_t b = cell_ballot(ep == step); b != 0u; b &= b - 1u) m = m + cell_lane(mn, __ffs((int)b) - 1);
    if (ln.q == 0) {
      a.mass[r] = m;
      a.phi_out[r] = m / rho;
    }
  }
  const int n1 = nF + nEP, n2 = n1 + nNI, n3 = n2 + nNL;
  for (int j = (int)tid; j < n3; j += (int)nth) {
    const int cell = j < nF ? a.listF[j] : (j < n1 ? a.listEP[j - nF] : (j < n2 ? a.listNI[j - n1] : a.listNL[j - n2]));
    bool join = j >= n1;
    a.flags[cell] = j < nF ? LIQ : (j < n1 ? GAS : IFACE);
    if (a.order == 2 && join) {
      // a cell that was on the list (len entries) before has its entry still;
      // what islot says proves itself, so it needs no first value
      const unsigned p = (unsigned)a.islot[cell];
      join = !(p < (unsigned)len && a.listI[p] == cell);
    }
    if (a.order) {
      const int pos = wave_append_at(join, &a.counters_next[C_I], a.listI, cell);
      if (join) a.islot[cell] = pos;
    }
  }
}

// All the conversions of a step by the threads of a team, after its lists F and
// E are complete and visible (nF, nE their lengths, the same in every thread).
// Up to SOLO_CELLS converted cells the first workgroup does them alone, the
// others pass: its barriers are cheap, those of the team (and its atomics,
// which leave the L2) are not.  WIDE: lists by one atomic per workgroup, for
// teams that may do many cells.
template <class F, int BLOCK, bool WIDE>
__device__ __forceinline__ void convert_all(const ConvArgs& v, int step, int nF, int nE, GridBarrier& grid) {
  __shared__ int32_t sc[NCOUNT];
  constexpr int GROUPS = BLOCK / CLANES;
  const unsigned lid = threadIdx.x;
  const int len = v.order == 2 ? peek(&v.counters_next[C_I]) : 0;  // nothing joins before the last barrier
  if (nF + nE <= SOLO_CELLS) {
    if (grid.team.rank != 0u) return;
    if (lid < NCOUNT) sc[lid] = 0;
    __syncthreads();
    mark_pass<true, 0>(v, step, sc, nF, nE, 0, GROUPS);
    block_meet();
    const int nEP = sc[C_EP], nNI = sc[C_NI], nNL = sc[C_NL];
    share_pass<F, true, 0>(v, step, sc, nF, nEP, nNI, nNL, 0, GROUPS);
    block_meet();
    const int nR = sc[C_R];
    gather_pass(v, step, nR, nF, nEP, nNI, nNL, len, lid, BLOCK);
    if (lid == 0) {
      v.counters[C_EP] = nEP;
      v.counters[C_NI] = nNI;
      v.counters[C_NL] = nNL;
      v.counters[C_R] = nR;
    }
    return;
  }
  const unsigned tid = grid.team.rank * BLOCK + lid, nth = grid.team.size * BLOCK;
  const int first = (int)grid.team.rank * GROUPS, groups = (int)grid.team.size * GROUPS;
  mark_pass<false, WIDE ? BLOCK : 0>(v, step, v.counters, nF, nE, first, groups);
  grid.meet(false);
  const int nEP = peek(&v.counters[C_EP]), nNI = peek(&v.counters[C_NI]), nNL = peek(&v.counters[C_NL]);
  share_pass<F, false, WIDE ? BLOCK : 0>(v, step, v.counters, nF, nEP, nNI, nNL, first, groups);
  grid.meet(false);
  gather_pass(v, step, peek(&v.counters[C_R]), nF, nEP, nNI, nNL, len, tid, nth);
}

}  // namespace fslbm
