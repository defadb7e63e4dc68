// Host check of the t-marching form's plan and staging: for every cross-section in a range that gets a
// tile, the staged sites (thread tid: tile site tid, face site tid) hold each of the six neighbours of
// every tile site at the index the step reads it from, within the workgroup's LDS; and the workgroups
// of an item cover every (right-hand side, tile, t) once.
#include <cstdio>
#include <cstring>
#include <vector>

#include "../../paper_1510_06897_amd/csrc/march.hpp"

using namespace ovl;

static Geom geom(int x, int y, int z, int t) {
  Geom g{{x, y, z, t}, {1, x, x * y, x * y * z}, x * y * z * t};
  return g;
}
static Ext4 extents(const Geom &g) {
  Ext4 e{g.L[0], g.L[1], g.L[2], g.L[3], g.stride[1], g.stride[2], g.stride[3], g.V};
  return e;
}

static bool check(const Geom &g, int nrhs, int mgroup, int nt) {
  StepItem it;
  std::memset(&it, 0, sizeof(it));
  it.g = g;
  it.nrhs = nrhs;
  const int n = march_tile(g, it.mty, it.mtz);
  if (!n) return true;
  it.mgroup = mgroup;
  it.nt = nt;
  const Ext4 ex = extents(g);
  const int ntile = g.L[1] / it.mty * (g.L[2] / it.mtz);
  const int blocks = nrhs * ntile * nt;
  std::vector<int> seen((size_t)nrhs * ntile * g.L[3], 0);
  for (int lb = 0; lb < blocks; ++lb) {
    const MarchPlace p = march_place(it, ex, lb);
    if (p.r < 0 || p.r >= nrhs || p.tile < 0 || p.tile >= ntile || p.n != n || n > kMarchThreads) return false;
    for (int t = p.t0; t < p.t1; ++t) ++seen[((size_t)p.r * ntile + p.tile) * g.L[3] + t];
    if (p.t1 <= p.t0 || p.t1 - p.t0 > (g.L[3] + nt - 1) / nt) return false;
    if (p.r || p.t0) continue;  // the staging depends on the tile alone
    std::vector<int> stage(2 * kMarchThreads, -1);
    for (int tid = 0; tid < kMarchThreads; ++tid) {
      if (p.tile_lane(tid)) stage.at(tid) = march_staged(p, it, ex, tid);
      if (p.face_lane(tid)) stage.at(n + tid) = march_staged(p, it, ex, n + tid);
    }
    for (int sj = 0; sj < n; ++sj) {
      const MarchSite m = march_site(p, it, ex, sj);
      const int x = m.s3 % ex.lx, y = m.s3 / ex.sy % ex.ly, z = m.s3 / ex.sz;
      auto at = [&](int a, int b, int c) {
        return (a + ex.lx) % ex.lx + ex.sy * ((b + ex.ly) % ex.ly) + ex.sz * ((c + ex.lz) % ex.lz);
      };
      if (stage.at(sj) != m.s3 || m.xm3 != at(x - 1, y, z) || m.ym3 != at(x, y - 1, z) ||
          m.zm3 != at(x, y, z - 1) || stage.at(m.jxp) != at(x + 1, y, z) || stage.at(m.jxm) != m.xm3 ||
          stage.at(m.jyp) != at(x, y + 1, z) || stage.at(m.jym) != m.ym3 ||
          stage.at(m.jzp) != at(x, y, z + 1) || stage.at(m.jzm) != m.zm3)
        return false;
    }
  }
  for (int s : seen)
    if (s != 1) return false;
  return true;
}

// slices of the busiest eighth of a planned launch's workgroups (an XCD's range) over the mean
static double imbalance(const Geom &g, int nrhs) {
  StepItem it;
  std::memset(&it, 0, sizeof(it));
  it.g = g;
  it.nrhs = nrhs;
  const int blocks = march_plan(&it, 1);
  const Ext4 ex = extents(g);
  double most = 0.0, all = 0.0;
  for (int x = 0; x < 8; ++x) {
    double sum = 0.0;
    for (int lb = blocks * x / 8; lb < blocks * (x + 1) / 8; ++lb) {
      const MarchPlace p = march_place(it, ex, lb);
      sum += p.t1 - p.t0;
    }
    all += sum;
    most = sum > most ? sum : most;
  }
  return most / (all / 8);
}

int main() {
  int tiles = 0, more_faces = 0, bad = 0;
  for (int x = 1; x <= 36; ++x)
    for (int y = 1; y <= 36; ++y)
      for (int z = 1; z <= 36; ++z) {
        const Geom g = geom(x, y, z, 1);
        int ty, tz;
        const int n = march_tile(g, ty, tz);
        if (!n) continue;
        ++tiles;
        more_faces += (ty < y ? 2 * x * tz : 0) + (tz < z ? 2 * x * ty : 0) > n;
        if (!check(g, 1, 1, 1)) {
          ++bad;
          std::printf("%d x %d x %d: tile %d x %d\n", x, y, z, ty, tz);
        }
      }
  for (const Geom &g : {geom(64, 64, 64, 1), geom(64, 5, 5, 2), geom(128, 1, 3, 1), geom(48, 48, 48, 1)})
    bad += !check(g, 1, 1, 1);
  for (int nrhs : {1, 2, 5, 40})
    for (int mgroup : {1, 2, 8, 32})
      for (int nt : {1, 2, 4, 5, 9}) bad += !check(geom(16, 8, 8, 9), nrhs, mgroup, nt);
  // ragged t extents: chunks of two lengths, spread evenly
  for (int lt : {5, 7, 9, 13, 17, 31, 33, 47})
    for (int nrhs : {6, 11, 14, 21, 40}) {
      const double x = imbalance(geom(16, 16, 16, lt), nrhs);
      if (x > 1.04) {
        ++bad;
        std::printf("16^3 x %d, %d vectors: the busiest XCD has %.2f times the mean\n", lt, nrhs, x);
      }
    }
  std::printf("%d cross-sections with a tile, %d with more face sites than tile sites, %d wrong\n", tiles,
              more_faces, bad);
  return bad || !tiles || !more_faces;
}
