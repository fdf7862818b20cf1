// The cells and elements that the two-step kernel (fslbm_deep.hip) works on, as
// plain expressions that a CPU program can evaluate too: every load of the
// kernel goes through them, also those whose value nothing reads (a thread
// beyond the lattice works on a cell inside it).
#pragma once

namespace fslbm {

// Tile of the form with populations of s bytes (the largest that LDS allows, see
// fslbm_deep.hip).
constexpr int deep_tx(int s) { return s == 8 ? 32 : 64; }
constexpr int deep_ty(int s) { return s == 8 ? 12 : 10; }
constexpr int deep_threads(int s) { return deep_tx(s) * (deep_ty(s) + 2) + 64; }

// Tiles of tx x ty cells over the rows y < yd: ntx along x, nty along y, nzc
// chunks of zlen planes; per strips (tiles along x of one row of tiles and one
// chunk) for each of the eight XCDs.
struct DeepPlan {
  int ntx, nty, nzc, zlen, per;
};

// The chunks along z are those with the fewest plane steps on the busiest of
// an XCD's 32 compute units.
constexpr DeepPlan deep_plan(int nx, int nz, int yd, int tx, int ty) {
  DeepPlan p{(nx + tx - 1) / tx, (yd + ty - 1) / ty, 1, nz, 1};
  long long best = -1;
  const int most = nz / 8 > 1 ? nz / 8 : 1;
  for (int n = 1; n <= most; ++n) {
    const int len = (nz + n - 1) / n;
    const int chunks = (nz + len - 1) / len;
    const int per = (p.nty * chunks + 7) / 8;
    const long long rounds = ((long long)per * p.ntx + 31) / 32;
    const long long cost = rounds * (len + 2);
    if (best < 0 || cost < best) {
      best = cost;
      p.nzc = chunks;
      p.zlen = len;
      p.per = per;
    }
  }
  return p;
}

// The thread's cell of the halo tile of w x h cells, w = tx + 2: rows of tx
// threads, then the two edge columns.
struct DeepHalo {
  int hx, hy;
};
constexpr DeepHalo deep_halo(int t, int tx, int h) {
  if (t < tx * h) return DeepHalo{1 + t % tx, t / tx};
  const int e = t - tx * h < 2 * h - 1 ? t - tx * h : 2 * h - 1;
  return DeepHalo{(e & 1) ? tx + 1 : 0, e >> 1};
}

// Column x (or plane z) v >= -1 of a tile on an axis of n cells: v inside the
// lattice, the cell across a periodic face one beyond it; everything else (past
// a wall, or further out, as a tile wider than the lattice reaches) is not read
// by any result and takes an edge cell.
constexpr int deep_wrap(int v, int n, bool periodic) {
  if (v < 0) return periodic ? n - 1 : 0;
  if (v < n) return v;
  return periodic && v == n ? 0 : n - 1;
}

// Row y of a tile: the rows -1 and beyond yd are not read by any result.
constexpr int deep_row(int y, int yd) { return y < 0 ? 0 : (y < yd ? y : yd); }

// Element that the pull of a link reads: from the cell x - c, or (a coordinate
// of it is -1: beyond a wall) the cell's own population opp.  self = x + nx y.
constexpr unsigned deep_source(int q, int opp, int sx, int sy, int sz, unsigned self, int z, int nx, unsigned nxy,
                               unsigned N) {
  return (sx | sy | sz) < 0 ? (unsigned)opp * N + (unsigned)z * nxy + self
                            : (unsigned)q * N + (unsigned)sz * nxy + (unsigned)(sx + nx * sy);
}

// The same where no link of the wavefront wraps or leaves the lattice within
// its plane, which begins at element `plane` of a population: the element is this
// base (uniform) plus self.
constexpr long long deep_base(int q, int cx, int cy, unsigned plane, int nx, unsigned N) {
  return (long long)((unsigned)q * N + plane) - (cx + nx * cy);
}

}  // namespace fslbm
