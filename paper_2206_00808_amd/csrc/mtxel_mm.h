// Spinor matrix elements by dense transforms on the matrix cores: the tables of one
// (valence, conduction, eps) sphere triple, and the launchers (mtxel_mm.hip).
#pragma once

#include <memory>

#include "common.h"

namespace gw {

// One device allocation
struct DevBuf {
  char* p = nullptr;
  size_t bytes = 0;
  ~DevBuf();
};

// What depends on the eps sphere and the axis order alone: kept (|g1|, |g2|) quads and
// the compact index map of the last transform.
struct MmEps {
  DevBuf dev;
  int nq = 0, nq4 = 0;                  // quads, padded to 4
  size_t o_qpos = 0, o_tab = 0;
};

// Spheres, grid and tables of one triple.  Axes are internal: 0 the planes' axis, 1
// the rows of a plane, 2 the entries of a row; perm[a] is the caller's axis.
struct MmTables {
  bool dbl = true;
  int nspinor = 2;
  int perm[3] = {0, 1, 2};
  int n[3] = {1, 1, 1};                 // alias-free grid: gv + gc + geps + 1 points
  int gv[3], gc[3], ge[3];              // largest |g| of each sphere
  long long sv[3], sc[3];               // strides of the spheres' compact cubes
  const int *cube_v = nullptr, *cube_c = nullptr;  // owned by the context's sphere maps
  int neps = 0;
  int rt = 1, ks = 1, jt = 1;           // row tiles of 16, K steps of 4, groups of 16 entries
  int ncz = 1, nry = 1, nx = 1;         // tiles of 8 kept |g| per axis 2, 1, 0
  int kx = 1;                           // K steps of the last transform
  bool rows = false;                    // pair planes by rows
  size_t plane = 0;                     // elements of a plane of one band, all spinor components
  size_t o_zc = 0, o_yc = 0, o_xc = 0;
  struct Band {
    int kx, ky, ntz, ncol;              // K steps over axes 0 and 1, tiles over axis 2, columns
    size_t bx, by, bz;                  // coefficient tables
  } bv{}, bc{};
  std::shared_ptr<DevBuf> grid;         // coefficients: they depend on the largest |g| alone
  std::shared_ptr<MmEps> eps;
};

// Tables for the triple, from the context's caches or new; null when no kernel is
// built for these sizes.  Allocates when an extent of the spheres or an eps sphere is
// first met, also while the stream is captured; geps is read during the call.
gw_status mm_tables(gw_ctx* c, const SphereMap* sv, const SphereMap* sc, const SphereMap* se,
                    const int32_t* geps, int nspinor, bool dbl, std::shared_ptr<MmTables>* out);
size_t mm_workspace(const MmTables& t, int nv, int nc);
gw_status mm_mtxel(gw_ctx* c, const MmTables& t, int nv, int ngv, const void* cv, int nc, int ngc,
                   const void* cc, void* mtxel, void* ws);

}  // namespace gw
