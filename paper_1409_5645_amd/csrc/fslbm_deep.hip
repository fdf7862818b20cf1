// Two time steps at once below the surface: the rows at the lattice's low y end
// that are liquid throughout go from time t to t + 2 in one pass over memory.
//
// The step's sweep streams 38 populations a cell at the rate the memory gives
// that pattern (5.1 - 5.3 TB/s), so a step costs its bytes.  Here a workgroup
// takes a tile of TX x TY cells and walks it along z: each thread pulls and
// collides one cell of the tile with a halo of one cell (time t + 1) and leaves
// it in LDS, where the planes z - 1, z and z + 1 that the next step pulls from
// are kept as far as they are needed (three planes of the links with c_z = 1,
// two of the others: 43 values a cell); then the tile's own cells are pulled from
// there, collided and stored (time t + 2).  The loads of the next plane are in
// flight meanwhile.  Reads grow by the halo (14 rows for 12, and shared lines in
// x), writes halve: 512 x 512 x 160 rows, two steps, FP64 4.79 -> 3.20 ms
// against two sweeps, FP32 2.39 -> 1.35 ms.  Tiles: TY as LDS allows (FP64 8, 10,
// 12 rows: 3.58, 3.34, 3.20 ms; FP32 8, 10, 12: 1.59, 1.34, 1.47 ms); two planes
// of loads in flight spilled or gained nothing; in FP16 storage the arithmetic
// bounds it (1.02 ms against 1.22; two cells a lane 1.32), not enough to pay for
// the rows it leaves to the sweeps.
//
// Workgroups go to the eight XCDs round robin; each XCD takes a run of strips
// (the tiles along x of one row of tiles), so that the tiles that share lines
// and halo rows run beside one another on one L2.
//
// The same operations in the same order as k_sweep: the same bits.
#include "fslbm_deep_index.hpp"
#include "fslbm_device.hpp"
#include "fslbm_internal.hpp"
#include "fslbm_stencil.hpp"

#include <type_traits>

namespace fslbm {

template <class F>
struct DeepTile {
  static constexpr int TX = deep_tx((int)sizeof(typename F::S));
  static constexpr int TY = deep_ty((int)sizeof(typename F::S));
  static constexpr int W = TX + 2, H = TY + 2;
  static constexpr int CELLS = W * H;
  static constexpr int THREADS = deep_threads((int)sizeof(typename F::S));
  static_assert(2 * H <= 64, "edge cells in one wavefront");
  // planes of the middle state kept, of the links with c_z = 1, 0 and -1
  static constexpr int NP = 3, NZ = 2, NM = 2;
  static constexpr int UNITS = 5 * NP + 9 * NZ + 5 * NM;
};

// rank of link q among the links of its c_z
constexpr int cz_rank(int q) {
  int n = 0;
  for (int p = 0; p < q; ++p) n += CZ[p] == CZ[q] ? 1 : 0;
  return n;
}

// first unit of link q (the slot of a plane is added)
template <class T>
constexpr int deep_unit(int q) {
  return CZ[q] == 1 ? T::NP * cz_rank(q)
                    : (CZ[q] == 0 ? 5 * T::NP + T::NZ * cz_rank(q) : 5 * T::NP + 9 * T::NZ + T::NM * cz_rank(q));
}

template <class F>
__global__ __launch_bounds__(DeepTile<F>::THREADS) void k_deep(DeepArgs a) {
  using R = typename F::R;
  using S = typename F::S;
  using T = DeepTile<F>;
  extern __shared__ __align__(16) unsigned char smem[];
  S* lds = reinterpret_cast<S*>(smem);
  const Grid g = a.c.grid;
  const int xcd = (int)blockIdx.x % 8, kk = (int)blockIdx.x / 8;
  const int strip = xcd * a.per + kk / a.ntx;
  if (kk / a.ntx >= a.per || strip >= a.nty * a.nzc) return;
  const int x0 = (kk % a.ntx) * T::TX;
  const int y0 = (strip % a.nty) * T::TY;
  const int z0 = (strip / a.nty) * a.zlen, z1 = min(g.nz, z0 + a.zlen);
  const int t = (int)threadIdx.x;
  // The thread's cell of the halo tile.  A thread whose cell lies beyond the
  // lattice (or the rows needed) works on a cell inside it, for nothing.
  const DeepHalo hc = deep_halo(t, T::TX, T::H);
  const int hx = hc.hx, hy = hc.hy;
  const bool out = hx >= 1 && hx <= T::TX && x0 + hx - 1 < g.nx && hy >= 1 && hy <= T::TY && y0 + hy - 1 < a.yd;
  const int x = deep_wrap(x0 + hx - 1, g.nx, g.px);
  const int y = deep_row(y0 + hy - 1, a.yd);
  const int ci = hy * T::W + hx;
  // in-plane sources
  const int xm = step_axis(x, -1, g.nx, g.px), xp = step_axis(x, 1, g.nx, g.px);
  const int ym = y > 0 ? y - 1 : -1, yp = y + 1;
  const unsigned N = (unsigned)g.N, nxy = (unsigned)g.nx * (unsigned)g.ny;
  const unsigned self = (unsigned)(x + g.nx * y);
  const S* __restrict__ fin = reinterpret_cast<const S*>(a.fin);
  S* __restrict__ fout = reinterpret_cast<S*>(a.fout);
  const Consts<R>& k = pick_consts<R>(a.c);
  R r[Q];
  auto plane = [&](int z) __attribute__((always_inline)) -> int { return deep_wrap(z, g.nz, g.pz); };
  // a wavefront off the lattice's x and y faces reaches every source at the same
  // distance from its own cell: one lane offset, scalar bases
  const bool inner = __ballot(x == 0 || x == g.nx - 1 || y == 0) == 0ull;
  const unsigned sb = self * (unsigned)sizeof(S);
  auto load = [&](int z) __attribute__((always_inline)) {  // pulls of plane z
    const int zm = step_axis(z, -1, g.nz, g.pz), zp = step_axis(z, 1, g.nz, g.pz);
    if (inner && (zm | zp) >= 0) {
      const unsigned om = (unsigned)zm * nxy, o0 = (unsigned)z * nxy, op = (unsigned)zp * nxy;
#define FSLBM_DPULL(q)                                                                                      \
  {                                                                                                         \
    const long long b = deep_base(q, CX[q], CY[q], CZ[q] == 1 ? om : (CZ[q] == -1 ? op : o0), g.nx, N);      \
    r[q] = F::load_raw(reinterpret_cast<const S*>(reinterpret_cast<const char*>(fin + b) + sb));            \
  }
      FSLBM_DPULL(0)
      FSLBM_LINKS(FSLBM_DPULL)
#undef FSLBM_DPULL
    } else {
#define FSLBM_DPULL(q)                                                                              \
  {                                                                                                 \
    const int sx = CX[q] == 1 ? xm : (CX[q] == -1 ? xp : x);                                        \
    const int sy = CY[q] == 1 ? ym : (CY[q] == -1 ? yp : y);                                        \
    const int sz = CZ[q] == 1 ? zm : (CZ[q] == -1 ? zp : z);                                        \
    r[q] = F::load_raw(fin + deep_source(q, OPP[q], sx, sy, sz, self, z, g.nx, nxy, N));             \
  }
      FSLBM_DPULL(0)
      FSLBM_LINKS(FSLBM_DPULL)
#undef FSLBM_DPULL
    }
  };
  auto collide_it = [&](R (&f)[Q]) __attribute__((always_inline)) {
    R rho_s, u[3];
    if constexpr (sizeof(R) == 4)
      collide_f32_scaled<F::shifted, F::scaled>(f, k, true, false, a.c.scale, a.c.inv_scale, rho_s, u);
    else
      collide<R, F::shifted>(f, k, true, false, rho_s, u);
  };
  const bool wxm = xm < 0, wxp = xp < 0, wym = ym < 0;
  int sp = 0, s0 = 0, sm = 0;  // slots of the plane being put, for the links with c_z = 1, 0, -1
  auto put = [&](int zi) __attribute__((always_inline)) {
    collide_it(r);
    S* const wp = lds + (sp * T::CELLS + ci);
    S* const w0 = lds + (s0 * T::CELLS + ci);
    S* const wm = lds + (sm * T::CELLS + ci);
#define FSLBM_DPUT(q) F::store_raw((CZ[q] == 1 ? wp : (CZ[q] == 0 ? w0 : wm)) + deep_unit<T>(q) * T::CELLS, r[q]);
    FSLBM_DPUT(0)
    FSLBM_LINKS(FSLBM_DPUT)
#undef FSLBM_DPUT
    load(plane(zi + 1));
  };
  auto next = [&]() __attribute__((always_inline)) {
    sp = sp == T::NP - 1 ? 0 : sp + 1;
    s0 = s0 == T::NZ - 1 ? 0 : s0 + 1;
    sm = sm == T::NM - 1 ? 0 : sm + 1;
  };
  auto back = [](int s, int d, int n) __attribute__((always_inline)) -> int { return s >= d ? s - d : s - d + n; };
  // ALL: every lane of the wavefront stores (no branch around the stores: the
  // waits for the loads of the next plane then need not wait for them)
  auto planes = [&](auto all) __attribute__((always_inline)) {
    constexpr bool ALL = decltype(all)::value;
    load(plane(z0 - 1));
    put(z0 - 1);
    next();
    put(z0);
    next();
    for (int z = z0; z < z1; ++z) {
      put(z + 1);
      __syncthreads();
      if (ALL || out) {
        const int bp = back(sp, 2, T::NP), cp = back(sp, 1, T::NP);  // planes z - 1, z
        const int c0 = back(s0, 1, T::NZ), cm = back(sm, 1, T::NM);  // plane z
        const bool wzm = z == 0 && !g.pz, wzp = z == g.nz - 1 && !g.pz;
        R f[Q];
        if (inner && !wzm && !wzp) {
          const S* const gp = lds + (bp * T::CELLS + ci - (T::W + 1));
          const S* const g0 = lds + (c0 * T::CELLS + ci - (T::W + 1));
          const S* const gm = lds + (sm * T::CELLS + ci - (T::W + 1));
#define FSLBM_DGET(q)                                                                            \
  f[q] = F::load_raw((CZ[q] == 1 ? gp : (CZ[q] == 0 ? g0 : gm)) +                                  \
                     (deep_unit<T>(q) * T::CELLS + T::W + 1 - CX[q] - T::W * CY[q]));
          FSLBM_DGET(0)
          FSLBM_LINKS(FSLBM_DGET)
#undef FSLBM_DGET
        } else {
#define FSLBM_DGET(q)                                                                              \
  {                                                                                                \
    constexpr int o = OPP[q];                                                                      \
    const bool w = (CX[q] == 1 && wxm) || (CX[q] == -1 && wxp) || (CY[q] == 1 && wym) ||           \
                   (CZ[q] == 1 && wzm) || (CZ[q] == -1 && wzp);                                    \
    const int us = deep_unit<T>(q) + (CZ[q] == 1 ? bp : (CZ[q] == 0 ? c0 : sm));                   \
    const int uo = deep_unit<T>(o) + (CZ[o] == 1 ? cp : (CZ[o] == 0 ? c0 : cm));                   \
    f[q] = F::load_raw(lds + (w ? uo * T::CELLS + ci : us * T::CELLS + ci - (CX[q] + T::W * CY[q]))); \
  }
          FSLBM_DGET(0)
          FSLBM_LINKS(FSLBM_DGET)
#undef FSLBM_DGET
        }
        collide_it(f);
        S* const fo = fout + (size_t)((unsigned)z * nxy);
#pragma unroll
        for (int q = 0; q < Q; ++q)
          F::store_raw(reinterpret_cast<S*>(reinterpret_cast<char*>(fo + (size_t)((unsigned)q * N)) + sb), f[q]);
      }
      __syncthreads();
      next();
    }
  };
  if (__ballot(!out) == 0ull) planes(std::true_type{});
  else planes(std::false_type{});
}

template <class T, class S, class K>
static hipError_t deep_go(DeepArgs a, K kernel, hipStream_t st) {
  const Grid& g = a.c.grid;
  const DeepPlan p = deep_plan(g.nx, g.nz, a.yd, T::TX, T::TY);
  a.ntx = p.ntx;
  a.nty = p.nty;
  a.nzc = p.nzc;
  a.zlen = p.zlen;
  a.per = p.per;
  constexpr size_t bytes = (size_t)T::UNITS * T::CELLS * sizeof(S);
  static_assert(bytes <= 160 * 1024, "LDS");
  hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e != hipSuccess) return e;
  kernel<<<8 * a.per * a.ntx, T::THREADS, bytes, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_deep(const DeepArgs& a, int precision, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (precision == 0) return deep_go<DeepTile<FormF64>, double>(a, k_deep<FormF64>, st);
  if (precision == 1) return deep_go<DeepTile<FormF32>, float>(a, k_deep<FormF32>, st);
  return hipErrorInvalidValue;  // FP16 storage takes its sweeps
}

}  // namespace fslbm
