// Internal interface between the C-ABI host code and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "fslbm_device.hpp"

namespace fslbm {

// list counters of one step (two sets, selected by step parity)
enum { C_F = 0, C_E = 1, C_EP = 2, C_NI = 3, C_NL = 4, C_I = 5, C_R = 6, NCOUNT = 8 };

struct Common {
  Grid grid;
  Consts<double> kd;
  Consts<float> kf;
  int incomp, stokes;
  float scale, inv_scale;  // FP16 storage scaling (powers of two)
  int moving;              // some wall face moves (then SweepArgs::wall_t holds the terms)
  double shear_b[6];       // prescribed S^b [xx, yy, zz, xy, xz, yz] (rules 4, 5)
  double sigma;            // surface tension coefficient (0: none)
  double rho_gas;          // gas density rho_b (actual, not in storage convention)
  int plic;                // FSL link distances from the PLIC plane instead of phi - 1/2
  int solid;               // solid cells present (SweepArgs carries their wall table)
  int surface;             // a prescribed surface plane per interface cell (SweepArgs surf_n, surf_d)
};

template <class R>
__device__ __forceinline__ const Consts<R>& pick_consts(const Common& c);
template <>
__device__ __forceinline__ const Consts<double>& pick_consts<double>(const Common& c) {
  return c.kd;
}
template <>
__device__ __forceinline__ const Consts<float>& pick_consts<float>(const Common& c) {
  return c.kf;
}

struct SweepArgs {
  Common c;
  const void* fin;
  void* fout;
  const uint8_t* flags;
  const double* mass_in;  // interface mass of time t (may equal mass)
  double* mass;           // interface mass of time t+1
  const double* phi_in;
  double* phi_out;
  // collision density and velocity of the interface cells of the step, [N][4]
  // (rho, u_x, u_y, u_z; 32 bytes per cell, one store)
  double* aux;
  int32_t* f_epoch;
  int32_t* listF;
  int32_t* listE;
  int32_t* listI;  // interface cells of time t (built by the sweep)
  int32_t* counters;
  int32_t* counters_next;
  double thr_hi, thr_lo;
  int step;
  int freeze;
  int hold;   // fill levels and interface masses held
  int cpr;   // blocks per lattice row (set by the launcher)
  // box of rows the sweep launches (box != 0): y in [by0, by0 + bny), z in
  // [bz0, bz0 + bnz); every liquid cell lies inside it.  0: every row.
  int box, by0, bny, bz0, bnz;
  int shell; // the box leaves the rows below to the two-step kernel
  int pairs; // FP16 form: two cells per lane when rows have even length
  int quad;  // interface cells of the plain step with four lanes per cell (k_iface4); 2: XCD-aware order
  // order != 0: the interface kernel runs before the sweep.  It takes the
  // list of time t that the previous step built (listI, counters[C_I]; with
  // holes where a cell has left the interface) and writes the populations of
  // t+1 of list entry i to rbuf[q * rcap + i] (i < rcap; beyond that straight
  // into fout).  The sweep then stores them with the rows it writes whole,
  // lists the interface cells of time t for the next step (counters_next,
  // islot: cell -> list entry) and leaves the counter zeroing to the
  // interface kernel.
  // order 2 (k_together): the interface cells in the sweep's own launch, from
  // the list listI of *len entries (with holes) that the conversions keep.
  int order;
  const int32_t* len;
  int nbi;   // order 2: blocks of the launch for the list (set by the launcher)
  int32_t* islot;
  void* rbuf;
  int rcap;
  void* u_out;  // optional (FP64 / FP32 forms): collision velocity of liquid cells, [3][N] compute type
  // optional per-step record of the interface cells (list order, capacity
  // rec_cap): pulled and own populations of time t (compute type, [Q][cap]),
  // fill and mass of time t, collision velocity ([3][cap], compute type) and
  // density of the step
  void* rec_f;
  void* rec_own;
  double* rec_phi;
  double* rec_m;
  void* rec_u;
  double* rec_rho;
  int rec_cap;
  double* kappa;  // surface tension: 3 sigma kappa per listed interface cell (list order)
  double* khf;    // surface tension with plic = 2: height-function kappa per cell (NaN: none)
  const double* wall_t;  // moving walls: [6 faces][19 links] bounce-back terms 2 w_q (c_q.u_w)/c_s^2
  // solid walls: ascending list of the non-solid cells next to a solid cell,
  // per listed cell i and link p the wall distance delta[p*nwall + i] and
  // velocity uw[(a*19 + p)*nwall + i] of the wall point x + delta c_p
  // prescribed surface: unit normal towards the gas [3][N] and plane offset
  // from the node [N] of the interface cells (caller's device memory)
  const double* surf_n;
  const double* surf_d;
  const int32_t* wcells;
  const double* wdelta;
  const double* wuw;
  int nwall;
  int nbw;   // blocks of the interface kernel for the wall list (set by the launcher)
};

struct ConvArgs {
  Common c;
  void* fout;  // populations of time t+1
  uint8_t* flags;
  double* mass;
  double* phi_out;
  double* aux;  // [N][4] as in SweepArgs
  int32_t* f_epoch;
  int32_t* new_epoch;
  int32_t* recv_epoch;
  int32_t* conv_epoch;
  int32_t *listF, *listE, *listEP, *listNI, *listNL, *listR;
  int32_t* counters;
  double* reservoir;
  int step;
  // order != 0 (SweepArgs::order): the new interface cells join the list of
  // the next step (listI, counters_next[C_I], islot); 2: unless they are still
  // on it
  int order;
  int32_t* listI;
  int32_t* islot;
  int32_t* counters_next;
  unsigned long long* bar;       // barrier and team words, zero
  unsigned long long* bar_next;  // those of the next launch (zeroed by this one)
  int team, team_wait;           // most workgroups of a team and how long it stays open (fslbm_barrier.hpp)
};

struct StepLaunch {
  SweepArgs sweep;
  ConvArgs conv;
  void* stream;
};

// A run of n plain steps of a small lattice in one launch (fslbm_resident.hip).
// sweep[k], conv[k]: arguments of the even and the odd steps of the run (the
// buffers and counter sets alternate; the step stamp is step + t); conv's
// order, listI, islot and counters_next name the kernel's own list.
struct ResidentArgs {
  SweepArgs sweep[2];
  ConvArgs conv[2];
  int32_t* list;   // interface cells, 2 N entries
  int32_t* islot;  // cell -> its entry
  int32_t* len;    // NCOUNT values, [C_I] the length of the list
  unsigned long long* bar;       // as in ConvArgs
  unsigned long long* bar_next;
  int team, team_wait;
  int step, n;
};
static_assert(sizeof(ResidentArgs) <= 4096, "kernel arguments");
// Where runs of steps are resident: lattices of up to RESIDENT_CELLS cells, and
// up to so many interface cells (as the classes at init have them) for a call of
// n steps.  What the launches cost is saved; a surface that takes more than a
// part of the resident workgroups, or that converts at every step, loses by its
// barriers.  us a step, kernels (from eight steps on with the interface cells in
// the sweep's launch) / resident:
//   64 interface cells (8 x 48 x 8 film, FP64)  n = 1 16.9 / 15.5, 2 16.8 / 11.4, 8 11.8 / 7.9, 64 12.3 / 6.9
//   216 (181 x 181 x 1, FP64)                   1 22.8 / 25.8, 2 22.6 / 21.9, 4 22.5 / 19.9, 64 18.8 / 18.1
//   408 (16 x 12 x 16, FP64)                    1 23.3 / 26.0, 2 23.4 / 22.5, 4 23.3 / 20.4, 64 18.5 / 18.5
//   555 (20^3, FP32)                            1 22.6 / 25.0, 2 22.3 / 21.0, 4 22.2 / 18.6, 64 16.6 / 15.6
//   665 (16 x 128 x 16, FP32)                   1 25.8 / 29.4, 2 25.9 / 25.5, 4 25.7 / 22.9, 64 18.5 / 20.6
//   809 (24^3, FP64, bulk shear)                1 29.9 / 36.1, 2 29.9 / 31.2, 4 29.8 / 28.4, 64 23.9 / 25.6
//   1,436 (32^3, FP64)                          1 32.3 / 37.7, 2 32.3 / 33.3, 4 32.2 / 30.5, 64 26.1 / 30.8
//   2,249 (45 x 6 x 45, FP64)                   1 30.8 / 41.4, 2 30.7 / 37.0, 4 30.7 / 34.6, 64 24.6 / 31.8
//   4,170 (64 x 8 x 64, calm, FP64)             1 17.3 / 31.0, 2 17.5 / 26.9, 4 17.3 / 24.9, 64 14.3 / 24.5
// `kept`: the kernels would take the interface cells in the sweep's launch.
// Steps per launch: see GridBarrier.
inline int resident_interface(int n, bool kept) {
  if (n == 1) return 128;
  return n == 2 || (kept && n >= 8) ? 600 : 1536;
}
constexpr int RESIDENT_CELLS = 32768;
constexpr int RESIDENT_STEPS = 256;
// Where the interface cells and the sweep share a launch (k_together): calls of
// at least TOGETHER_STEPS steps (the list is built anew for each call, about
// 20 us, so that classes a caller changed between calls are seen) on lattices
// whose two population buffers take at most TOGETHER_MAX_BYTES.  Above that the
// sweep loses by its partly written lines and by the interface cells'
// scattered traffic what the interface kernel's launch costs (us a step of a
// tank, separate / together: 40^3 FP64 24.0 / 16.8, FP32 20.6 / 14.5, FP16 23.9
// / 15.2; 96x72x96 FP64 40.8 / 31.8, FP32 35.9 / 22.1, FP16 36.0 / 22.2;
// 128x96x128 FP64 81.6 / 70.6, FP32 56.3 / 36.9, FP16 45.4 / 30.1; 160x120x160
// FP32 78.0 / 71.4, FP16 61.9 / 56.9; 253x159x131 FP16 90.6 / 87.9; 256x160x256
// FP16 144.8 / 145.4; 512x320x512 FP16 865 / 941).  The list is built anew
// after TOGETHER_REBUILD steps: cells that have left it stay as holes till
// then.
constexpr int TOGETHER_STEPS = 8;
constexpr int TOGETHER_REBUILD = 64;
constexpr double TOGETHER_MAX_BYTES = 600e6;
// Converted cells of a step that one workgroup takes (convert_all): its 16
// groups of lanes do up to about eight cells and their neighbours in one or
// two rounds.  101,565-cell tank with about 5 conversions a step (FP32): 29.0 us
// a step with 8, 30.5 with every step on the grid; 61,440 cells with about 20
// conversions: 32.4 us with 8, 35.3 with 64.
constexpr int SOLO_CELLS = 8;

// Two steps of the rows y < yd (every cell of the rows y <= yd is liquid).
struct DeepArgs {
  Common c;
  const void* fin;
  void* fout;
  int yd;
  int ntx, nty, nzc, zlen, per;  // tiles, set by the launcher
};
// Where the two-step kernel runs: the FP64 and FP32 forms, lattices whose
// population buffers have left the 256 MB cache (us a step of a tank, one step
// after the other / two at once: 128x96x128 FP64 85 / 85, FP32 47 / 57;
// 160x120x160 FP64 136 / 128, FP32 80 / 84; 192x128x192 FP64 212 / 173, FP32
// 111 / 104; 256x160x256 FP64 460 / 371, FP32 239 / 185; 512x320x512 FP64 2917
// / 2289, FP32 1564 / 1170), up to 17 GB a buffer (a third one of it is needed),
// and from two tiles of rows on.  FP16 storage is bound by its arithmetic there:
// 512x320x512 848 / 832, 256x160x256 144 / 159.
constexpr double DEEP_MIN_BYTES = 300e6;
constexpr double DEEP_MAX_BYTES = 17e9;
constexpr int DEEP_ROWS = 24;

struct InitArgs {
  Common c;
  void* f;
  const uint8_t* flags;
  double* mass;
  double* phi;
  // collision density and velocity of the interface cells of the step, [N][4]
  // (rho, u_x, u_y, u_z; 32 bytes per cell, one store)
  double* aux;
};

struct FieldArgs {
  Common c;
  const void* f;
  const uint8_t* flags;
  const double* mass;
  const double* phi;
  const double* aux;  // [N][4] as in SweepArgs
  double* rho_out;
  double* u_out;
  double* phi_out;
  uint8_t* flags_out;
  double* f_out;
  double* mass_out;
  double* rhoc_out;
  double* uc_out;
};

struct StatArgs {
  Common c;
  const void* f;
  const uint8_t* flags;
  const double* mass;
  double* acc;    // [0] mass sum
  // [0] liquid cells, [1] cells with a NaN or non-positive density, [2]
  // interface cells, [3] unused here, [4] cells with |u| above the bound (or
  // a NaN velocity), [5] cells breaking the class rule (unknown class, or a
  // liquid cell next to a gas cell)
  int32_t* cnt;
  double u_max2;  // square of the |u| bound
};

// One reverse step t+1 -> t of a window with frozen cell classes.
struct AdjArgs {
  Common c;
  // record of the step t -> t+1 (written by the forward step)
  const void* u;          // collision velocity at liquid cells ([3][N], compute type)
  const void* rec_f;      // interface cells: pulled populations ([Q][cap], compute type)
  const void* rec_own;    // interface cells: own post-collision populations of time t
  const double* rec_phi;  // interface cells: fill of time t
  const double* rec_m;    // interface cells: mass of time t
  const void* rec_u;      // interface cells: collision velocity ([3][cap], compute type)
  const double* rec_rho;  // interface cells: collision density
  // fixed topology of the interface cells (list order)
  const uint64_t* ncls;   // class of the pull source of each link, 2 bits per link (gas, interface, liquid, wall)
  const int32_t* nslot;   // [Q][cap] list position of an interface pull source, else the cell's own
  const uint8_t* flags;   // cell classes (fixed over the window)
  const void* lam_in;     // dL/dft of time t+1 (compute type)
  void* lam_out;          // dL/dft of time t (compute type)
  double* lam_m;          // dL/dm: time t+1 on entry, time t on exit (interface cells)
  const double* lphi_in;  // dL/dphi of time t+1 (interface cells)
  double* lphi_out;       // dL/dphi of time t (interface cells)
  const int32_t* listI;   // interface cells, ascending
  const int32_t* islot;   // cell -> position in listI (interface cells only)
  void* own;              // [Q][cap] own-population adjoint terms (compute type)
  double* phic;           // [Q][cap] fill adjoint terms per pull source (0: the cell itself)
  double* part_sweep;     // [sweep wavefronts][3] dL/dg partial sums
  double* part_iface;     // [interface blocks][4] dL/drho_b, dL/dg partial sums
  int n_i, cap, cpr;
};

hipError_t launch_sweep(const StepLaunch& L, int precision, int rule);
hipError_t launch_together(const StepLaunch& L, int precision, int rule);
// y and z extent of the fluid cells, and the lowest y of a cell that is not
// liquid, into ext = (ymin, ymax, zmin, zmax, ynot); (INT_MAX, -1, ..., INT_MAX) if none
constexpr int EXT_VALUES = 5;
// partial extents of k_extent (ext holds (1 + EXT_COPIES) lines of 32 int32:
// the result in the first, the partials after it)
constexpr int EXT_COPIES = 64;
constexpr size_t EXT_BYTES = (size_t)(1 + EXT_COPIES) * 32 * sizeof(int32_t);
hipError_t launch_extent_init(int32_t* ext, void* stream);
hipError_t launch_extent(const uint8_t* flags, const Grid& g, int y0, int ny, int z0, int nz, int32_t* ext,
                         void* stream);
hipError_t launch_iface(const StepLaunch& L, int precision, int rule);
hipError_t launch_iface4(const StepLaunch& L, int precision, int rule);  // fslbm_iface4.hip
// geometry of the listed cells that needs more than the interface kernel loads:
// curvature (sigma != 0), height functions (plic = 2); nothing without either
hipError_t launch_geometry(const StepLaunch& L, int rule);
hipError_t launch_convert(const StepLaunch& L, int precision);
hipError_t launch_resident(const ResidentArgs& r, int precision, int rule, void* stream);
// interface cells of the current classes -> list, islot, *counter (a step with
// the interface kernel first after a new state)
hipError_t launch_list_append(const uint8_t* flags, const Grid& g, int32_t* counter, int32_t* list, int32_t* islot,
                              void* stream);
hipError_t launch_fill_i32(int32_t* p, size_t n, int32_t v, void* stream);
hipError_t launch_fill_f64(double* p, size_t n, double v, void* stream);
hipError_t launch_check_flags(const uint8_t* flags, const Grid& g, int32_t* err, bool count, void* stream);
hipError_t launch_deep(const DeepArgs& a, int precision, void* stream);
hipError_t launch_check_walls(const uint8_t* flags, const Grid& g, const int32_t* cells, int n, const double* delta,
                              const double* uw, int32_t* err, int32_t* count, void* stream);
hipError_t launch_set_equilibrium(const InitArgs& a, int precision, const double* rho, const double* u,
                                  const double* fill, void* stream);
hipError_t launch_set_state(const InitArgs& a, int precision, const double* f, const double* mass,
                            const double* fill, void* stream);
hipError_t launch_fields(const FieldArgs& a, int precision, void* stream);
hipError_t launch_stats(const StatArgs& a, int precision, void* stream);

// adjoint window (fslbm_adjoint.hip)
unsigned adj_sweep_blocks(const Grid& g);
unsigned adj_sweep_slots(const Grid& g);  // dL/dg partial-sum slots of the sweep (one per wavefront)
unsigned adj_iface_blocks(int n_i);
unsigned list_blocks(const Grid& g);
hipError_t launch_count_iface(const uint8_t* flags, const Grid& g, int32_t* out, void* stream);
hipError_t launch_adj_topo(const uint8_t* flags, const Grid& g, const int32_t* list, const int32_t* islot, int n_i,
                           int cap, uint64_t* ncls, int32_t* nslot, void* stream);
hipError_t launch_iface_list(const uint8_t* flags, const Grid& g, int32_t* bcount, int32_t* list, int32_t* islot,
                             int32_t* n_out, void* stream);
hipError_t launch_adj_seed(const Common& c, const uint8_t* flags, int precision, const double* dLdf,
                           const double* dLdm, const double* dLdphi, void* lam, void* lam_other, double* lam_m,
                           double* lphi, double* lphi_other, void* stream);
// one reverse step = adj_sweep (liquid cells) and adj_iface (interface cells;
// independent of adj_sweep, may run concurrently), then adj_iface2 after both
hipError_t launch_adj_sweep(const AdjArgs& a, int precision, void* stream);
hipError_t launch_adj_iface(const AdjArgs& a, int precision, int rule, void* stream);
hipError_t launch_adj_iface2(const AdjArgs& a, int precision, void* stream);
hipError_t launch_adj_out(const Common& c, const uint8_t* flags, int precision, const void* lam,
                          const double* lam_m, const double* lphi, double* dLdf, double* dLdm, double* dLdphi,
                          void* stream);
hipError_t launch_adj_reduce(const double* part_sweep, int nb_sweep, const double* part_iface, int nb_iface,
                             double* out4, void* stream);

}  // namespace fslbm
