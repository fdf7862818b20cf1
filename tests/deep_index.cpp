// Evaluates every load of the two-step kernel (csrc/fslbm_deep_index.hpp, the
// kernel's own expressions) over a lattice: arguments bytes nx ny nz px pz yd.
// Prints the number of loads outside the 19 N elements of a buffer and of loads
// that a result needs but that read another element than the pull's.
#include <cstdio>
#include <cstdlib>
#include <set>
#include <tuple>

#include "fslbm_deep_index.hpp"

using namespace fslbm;

static const int C[19][3] = {{0, 0, 0},  {1, 0, 0},   {-1, 0, 0}, {0, 1, 0},  {0, -1, 0}, {0, 0, 1},  {0, 0, -1},
                             {1, 1, 0},  {-1, -1, 0}, {1, -1, 0}, {-1, 1, 0}, {1, 0, 1},  {-1, 0, -1}, {1, 0, -1},
                             {-1, 0, 1}, {0, 1, 1},   {0, -1, -1}, {0, 1, -1}, {0, -1, 1}};

static int step(int v, int d, int n, bool per) {
  v += d;
  if (v >= 0 && v < n) return v;
  return per ? (v + n) % n : -1;
}

int main(int, char** a) {
  const int s = atoi(a[1]), nx = atoi(a[2]), ny = atoi(a[3]), nz = atoi(a[4]), yd = atoi(a[7]);
  const bool px = atoi(a[5]), pz = atoi(a[6]);
  const int TX = deep_tx(s), TY = deep_ty(s), H = TY + 2;
  const DeepPlan p = deep_plan(nx, nz, yd, TX, TY);
  const long long N = (long long)nx * ny * nz, nxy = (long long)nx * ny;
  long long out = 0, wrong = 0;
  std::set<std::tuple<int, int, int>> stored;
  for (int block = 0; block < 8 * p.per * p.ntx; ++block) {
    const int xcd = block % 8, kk = block / 8, strip = xcd * p.per + kk / p.ntx;
    if (kk / p.ntx >= p.per || strip >= p.nty * p.nzc) continue;
    const int x0 = (kk % p.ntx) * TX, y0 = (strip % p.nty) * TY;
    const int z0 = (strip / p.nty) * p.zlen, z1 = nz < z0 + p.zlen ? nz : z0 + p.zlen;
    for (int w = 0; w < deep_threads(s); w += 64) {
      bool inner = true;
      for (int t = w; t < w + 64; ++t) {
        const DeepHalo h = deep_halo(t, TX, H);
        const int x = deep_wrap(x0 + h.hx - 1, nx, px);
        inner = inner && x != 0 && x != nx - 1 && deep_row(y0 + h.hy - 1, yd) != 0;
      }
      for (int t = w; t < w + 64; ++t) {
        const DeepHalo h = deep_halo(t, TX, H);
        const int X = x0 + h.hx - 1, Y = y0 + h.hy - 1;  // before wrapping
        const int x = deep_wrap(X, nx, px), y = deep_row(Y, yd);
        // what a result of the tile's rows reads, in the plane and across its faces
        const bool used = (X >= 0 || px) && (X < nx || (px && X == nx)) && Y >= 0 && Y <= yd;
        for (int Z = z0 - 1; Z <= z1 + 1; ++Z) {  // the planes put, and the one loaded ahead of the last
          const int z = deep_wrap(Z, nz, pz);
          const int zm = step(z, -1, nz, pz), zp = step(z, 1, nz, pz);
          for (int q = 0; q < 19; ++q) {
            const int *c = C[q], opp = q == 0 ? 0 : (q & 1 ? q + 1 : q - 1);
            const int sx = step(x, -c[0], nx, px), sy = y - c[1] < 0 ? -1 : y - c[1], sz = c[2] == 1 ? zm : (c[2] == -1 ? zp : z);
            long long e;
            if (inner && (zm | zp) >= 0)
              e = deep_base(q, c[0], c[1], (unsigned)(sz * nxy), nx, (unsigned)N) + x + (long long)nx * y;
            else
              e = deep_source(q, opp, sx, sy, sz, (unsigned)(x + nx * y), z, nx, (unsigned)nxy, (unsigned)N);
            if (e < 0 || e >= 19 * N) ++out;
            // the pull, from the unwrapped cell
            if (used && Z <= z1 && (Z >= 0 || pz) && (Z < nz || pz)) {
              const int wx = (X + nx) % nx, wz = (Z + nz) % nz;
              const int ux = step(wx, -c[0], nx, px), uy = Y - c[1], uz = step(wz, -c[2], nz, pz);
              const bool wall = ux < 0 || uy < 0 || uz < 0;
              const long long want = wall ? (long long)opp * N + wz * nxy + wx + (long long)nx * Y
                                          : (long long)q * N + uz * nxy + ux + (long long)nx * uy;
              if (e != want) ++wrong;
            }
          }
        }
        if (h.hx >= 1 && h.hx <= TX && X < nx && h.hy >= 1 && h.hy <= TY && Y < yd)
          for (int z = z0; z < z1; ++z) wrong += stored.insert(std::make_tuple(X, Y, z)).second ? 0 : 1;
      }
    }
  }
  wrong += (long long)stored.size() != (long long)nx * yd * nz ? 1 : 0;
  printf("%lld %lld\n", out, wrong);
}
