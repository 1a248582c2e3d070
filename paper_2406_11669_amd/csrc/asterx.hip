// asterx.hip -- HIP kernels (gfx950, FP64) and the C ABI of the Valencia GRMHD right-hand side.
//
// One block, one GPU.  Per RK stage the caller runs: asterx_c2p -> asterx_fill_ghosts(prim)
// -> asterx_rhs -> asterx_rk_stage -> asterx_fill_ghosts(state).  asterx_rhs itself is
//   bcent, vertex: the field at the centres; gauge quantities G_A and F_Psi at vertices;
//   faces:         reconstruction + prim->cons + fluxes + speeds + HLLE, one lane per face;
//   cell:          flux divergence + geometric sources + div B, LDS-tiled metric;
//   edge:          FCT electric field, dA/dt and dPsi/dt,
// where phases that don't depend on each other share launches (do_rhs).
// Threads map to x fastest so every stencil load is coalesced across a wavefront; the
// block -> tile map keeps neighbouring tiles on one XCD (shared L2).  The same bodies run in
// persistent launches over work lists of (patch, tile) items for batches of patches, and the
// reverse-mode (adjoint) kernels at the end of the file transpose one stage.
// Section/equation references are to AsterX, arXiv 2406.11669.

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstring>
#include <algorithm>
#include <mutex>
#include <string>
#include <vector>

#include "asterx.h"
#include "grmhd_device.h"
#include "host_internal.h"
#include "mlp_device.h"

using namespace ax;

namespace {

thread_local std::string g_err;

// rhs workspace: centre field (3) + face fluxes (3 directions x 7) + G_A (1) + F_Psi (3)
// right-hand side workspace: centre field 3, face fluxes 21, G_A 1, F_Psi 3, upwind-CT speeds and face
// fields 9
constexpr int WS_FIELDS = 3 + 21 + 1 + 3 + 9;

int fail(int code, const char* msg) {
  g_err = msg;
  return code;
}

// ---------------------------------------------------------------------------------------
// Grid description passed by value to kernels.
struct GD {
  int n[3];
  int ng;
  int ld0, ld1;
  int sy, sz;  // strides of j and k
  size_t N;    // points per field
  double idx[3];
};

GD make_gd(const asterx_grid* g) {
  GD d;
  for (int a = 0; a < 3; ++a) {
    d.n[a] = g->n[a];
    d.idx[a] = 1.0 / g->dx[a];
  }
  d.ng = g->ng;
  d.ld0 = g->ld[0];
  d.ld1 = g->ld[1];
  d.sy = g->ld[0];
  d.sz = g->ld[0] * g->ld[1];
  d.N = (size_t)g->ld[0] * g->ld[1] * g->ld[2];
  return d;
}

DEV int at(const GD& g, int i, int j, int k) { return ((k + g.ng) * g.ld1 + (j + g.ng)) * g.ld0 + (i + g.ng); }

// Element i >= 0 of a field whose base is the same for the whole wavefront: the address is
// formed by the load from the scalar base and a 32-bit per-lane byte offset (fields hold fewer
// than 2^29 points, checked on the host), instead of a 64-bit vector add per access.
template <class T>
DEV T ldu(const T* base, int i) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + (unsigned)i * (unsigned)sizeof(T));
}

// Blocks are dispatched round-robin over the 8 XCDs; remap the linear block id so that
// each XCD walks a contiguous range of tiles (neighbouring tiles share its L2).
DEV unsigned xcd_block(unsigned bid, unsigned nblocks) {
  const unsigned nx = 8;
  unsigned per = nblocks / nx, rem = nblocks % nx;
  unsigned x = bid % nx, r = bid / nx;
  // XCD x owns tiles [start_x, start_x + per + (x < rem))
  unsigned start = x * per + (x < rem ? x : rem);
  return start + r;
}

// Linear tile decomposition of a 3-D box of extents e[3] into tiles of TX x TY x 1; `tile`
// is the logical tile index, `tid` the thread's index inside the tile.
template <int TX, int TY>
DEV bool box_at(const int e[3], unsigned tile, unsigned tid, int& a, int& b, int& c) {
  unsigned nbx = (e[0] + TX - 1) / TX, nby = (e[1] + TY - 1) / TY;
  unsigned bx = tile % nbx;
  unsigned t = tile / nbx;
  unsigned by = t % nby;
  c = (int)(t / nby);
  a = (int)(bx * TX + tid % TX);
  b = (int)(by * TY + tid / TX);
  return a < e[0] && b < e[1] && c < e[2];
}

// Linear decomposition of a 3-D box into tiles of 256 consecutive points (x fastest): for
// per-point kernels over extents that are not multiples of a tile row (n + 2, n + 2 ng).
DEV bool lin_at(const int e[3], unsigned tile, unsigned tid, int& a, int& b, int& c) {
  const unsigned q = tile * 256 + tid, t = q / (unsigned)e[0];  // below 2^29 points
  a = (int)(q % (unsigned)e[0]);
  b = (int)(t % (unsigned)e[1]);
  c = (int)(t / (unsigned)e[1]);
  return c < e[2];
}
inline unsigned lin_blocks(const int e[3]) { return (unsigned)(((long long)e[0] * e[1] * e[2] + 255) / 256); }

// Face tiles of the adjoint (two lanes per face; the figures were measured when the forward kernels had this
// form).  Face grids are n + 1 wide (129 for n = 128), so 32-wide tile rows would leave
// up to 31 of every 160 lanes idle.  In each z plane, the x range rounded down to a multiple
// of 32 is tiled 32 x 4 (x, y); the remaining x columns (fewer than 32) follow in the same
// plane, 128 faces per tile, x fastest.  Keeping them beside their plane's main tiles spreads
// these slower, uncoalesced tiles evenly over the XCDs.  Rows narrower than 32 are tiled whole.
struct FacePlan {
  int e0m, r;           // main x range [0, e0m), remainder width r
  unsigned nbx, nby;    // main tiles per plane: nbx x nby
  unsigned pm, per;     // main tiles per plane, all tiles per plane
};
__host__ __device__ inline FacePlan face_plan(const int e[3]) {
  FacePlan P;
  P.e0m = e[0] >= 32 ? (e[0] & ~31) : e[0];
  P.r = e[0] - P.e0m;
  P.nbx = (unsigned)((P.e0m + 31) / 32);
  P.nby = (unsigned)((e[1] + 3) / 4);
  P.pm = P.nbx * P.nby;
  P.per = P.pm + (unsigned)((P.r * e[1] + 127) / 128);
  return P;
}
inline unsigned face_tiles(const int e[3]) { return face_plan(e).per * (unsigned)e[2]; }
// Tile order: groups of ZG consecutive planes; inside a group, plane-tile by plane-tile (main
// tiles, then the remainder tiles) with the plane index fastest (ZG = 1: plane by plane).  For y
// and z faces (ZG = FACE_ZG) consecutive tiles of one XCD are then z-neighbours: a z face's
// stencil cells and a y face's metric rows at four z levels are shared by the next tiles and found
// in that XCD's L2, where plane by plane they were fetched again a whole plane later (reads per
// launch 0.96 -> 0.49 GB for y faces, 1.06 -> 0.50 GB for z faces; y neighbours stay FACE_ZG * nbx
// tiles apart).  x faces keep the plane order: their stencils run along x inside the tile and
// their metric is read once per face, and they measured slower in groups.
constexpr int FACE_ZG = 8;

template <int D>
constexpr int face_zg() { return D == 0 ? 1 : FACE_ZG; }
// Face f (0..127) of `tile`: position (a, b, c), whether the tile is a remainder tile (the
// same for the whole workgroup), and a main tile's origin (ax0, by0) in its plane c.
template <int ZG>
DEV bool face_at(const int e[3], unsigned tile, unsigned f, int& a, int& b, int& c, bool& rest, int& ax0,
                 int& by0) {
  const FacePlan P = face_plan(e);
  const unsigned gsz = P.per * ZG, g = tile / gsz, tl = tile - g * gsz;
  const unsigned zg = min((unsigned)ZG, (unsigned)e[2] - g * ZG);  // planes in this group
  const unsigned w = tl / zg;
  c = (int)(g * ZG + tl % zg);
  rest = w >= P.pm;
  if (!rest) {
    ax0 = (int)(w % P.nbx) * 32;
    by0 = (int)(w / P.nbx) * 4;
    a = ax0 + (int)(f % 32);
    b = by0 + (int)(f / 32);
    return a < P.e0m && b < e[1] && c < e[2];
  }
  ax0 = by0 = 0;
  const int q = (int)(w - P.pm) * 128 + (int)f;
  a = P.e0m + q % P.r;
  b = q / P.r;
  return b < e[1] && c < e[2];
}

// Logical tile of a one-tile-per-workgroup launch.
DEV unsigned my_tile() { return xcd_block(blockIdx.x, gridDim.x); }

template <int TX, int TY>
unsigned box_blocks(const int e[3]) {
  return (unsigned)((e[0] + TX - 1) / TX) * (unsigned)((e[1] + TY - 1) / TY) * (unsigned)e[2];
}

// ---------------------------------------------------------------------------------------
// Wavefront reductions (64 lanes): max of non-negative doubles, then at most one device atomic
// per wavefront.  Max is order independent, so results are deterministic.
// Atomics to one address serialize in L2 (tens of thousands of wavefronts per launch would
// cost about a millisecond), so a maximum is only pushed when it exceeds the running value,
// read first with a device-scope load: the running value only grows, so skipping is exact.
DEV double wave_max(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

DEV void atomic_max_u64(unsigned long long* addr, unsigned long long v) {
  if (__hip_atomic_load(addr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < v) atomicMax(addr, v);
}

DEV void atomic_max_pos(double* addr, double v) {
  // non-negative doubles order like their bit patterns
  atomic_max_u64((unsigned long long*)addr, (unsigned long long)__double_as_longlong(v));
}

DEV int wave_max_int(int v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  return v;
}

// ---------------------------------------------------------------------------------------
// Vertex -> centre/face interpolation of spacetime data (Sec. 3.2: fourth-order Lagrange).
// The centre of cell i lies midway between vertices i and i+1; stencil i-1..i+2.
DEV double lag(double a, double b, double c, double d) { return 0.5625 * (b + c) - 0.0625 * (a + d); }
DEV double dlag(double a, double b, double c, double d) { return (27.0 * (c - b) - (d - a)) * (1.0 / 24.0); }

// Value at the centre whose lower-corner vertex stencil starts at p (vertex i-1,j-1,k-1).
DEV double centre_val(const double* __restrict__ p, int sy, int sz) {
  double zz[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    double yy[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const double* r = p + b * sy + c * sz;
      yy[b] = lag(r[0], r[1], r[2], r[3]);
    }
    zz[c] = lag(yy[0], yy[1], yy[2], yy[3]);
  }
  return lag(zz[0], zz[1], zz[2], zz[3]);
}

DEV void centre_metric(const double* __restrict__ metric, size_t N, int base, int sy, int sz, double m[10]) {
#pragma unroll
  for (int c = 0; c < 10; ++c) m[c] = centre_val(metric + c * N + base, sy, sz);
}

// ---------------------------------------------------------------------------------------
// Staggered field (Secs. 2.3, 3.1): face Btilde = curl of the edge potential; centre value
// = average of the two faces.
DEV double faceBx(const double* Ay, const double* Az, int id, int sy, int sz, const GD& g) {
  return (Az[id + sy] - Az[id]) * g.idx[1] - (Ay[id + sz] - Ay[id]) * g.idx[2];
}
DEV double faceBy(const double* Ax, const double* Az, int id, int sy, int sz, const GD& g) {
  return (Ax[id + sz] - Ax[id]) * g.idx[2] - (Az[id + 1] - Az[id]) * g.idx[0];
}
DEV double faceBz(const double* Ax, const double* Ay, int id, int sy, int sz, const GD& g) {
  (void)sz;
  return (Ay[id + 1] - Ay[id]) * g.idx[0] - (Ax[id + sy] - Ax[id]) * g.idx[1];
}

DEV void centre_B(const double* __restrict__ A, const GD& g, int id, double Bt[3]) {
  const double* Ax = A;
  const double* Ay = A + g.N;
  const double* Az = A + 2 * g.N;
  Bt[0] = 0.5 * (faceBx(Ay, Az, id, g.sy, g.sz, g) + faceBx(Ay, Az, id + 1, g.sy, g.sz, g));
  Bt[1] = 0.5 * (faceBy(Ax, Az, id, g.sy, g.sz, g) + faceBy(Ax, Az, id + g.sy, g.sy, g.sz, g));
  Bt[2] = 0.5 * (faceBz(Ax, Ay, id, g.sy, g.sz, g) + faceBz(Ax, Ay, id + g.sz, g.sy, g.sz, g));
}

C2PParams make_c2p_params(const asterx_params* p) {
  C2PParams c;
  c.gam = p->gamma;
  c.rho_atm = p->rho_atm;
  c.k_atm = p->k_atm;
  c.tol = p->c2p_tol;
  c.wmax = p->wmax;
  c.maxit = p->c2p_maxit;
  c.brent_maxit = p->brent_maxit;
  c.method = p->c2p_method;
  return c;
}

// ---------------------------------------------------------------------------------------
// Cell tiles of 16 x 4 x 4 with the spacetime data staged in LDS.  The vertex tile
// (19 x 7 x 7) of one component is loaded once, then interpolated separably -- z, then y,
// then x -- with each pass shared by all cells of the tile (Sec. 3.2 Lagrange weights).
constexpr int CTX = 16, CTY = 4, CTZ = 4;
constexpr int VX = CTX + 3, VY = CTY + 3, VZ = CTZ + 3;
constexpr int NV = VX * VY * VZ;    // vertex tile
constexpr int NZP = VX * VY * CTZ;  // after the z pass
constexpr int NYP = VX * CTY * CTZ; // after the y pass

struct TileLDS {
  double v[NV];
  double z[2 * NZP];
  double y[3 * NYP];
};

struct TileCell {
  int i0, j0, k0, cx, cy, cz;
  bool valid;
};

DEV TileCell tile_cell(const GD& g, unsigned bid) {
  TileCell t;
  int ntx = (g.n[0] + CTX - 1) / CTX, nty = (g.n[1] + CTY - 1) / CTY;
  t.i0 = (int)(bid % ntx) * CTX;
  t.j0 = (int)((bid / ntx) % nty) * CTY;
  t.k0 = (int)(bid / (ntx * nty)) * CTZ;
  t.cx = threadIdx.x % CTX;
  t.cy = (threadIdx.x / CTX) % CTY;
  t.cz = threadIdx.x / (CTX * CTY);
  t.valid = t.i0 + t.cx < g.n[0] && t.j0 + t.cy < g.n[1] && t.k0 + t.cz < g.n[2];
  return t;
}

unsigned tile_blocks(const GD& g) {
  return (unsigned)(((g.n[0] + CTX - 1) / CTX) * ((g.n[1] + CTY - 1) / CTY) * ((g.n[2] + CTZ - 1) / CTZ));
}

// The vertex tile of one component spans vertices i0-1 .. i0+CTX+1 (etc.).  Each thread
// fetches its (at most four) points into registers first, so that the global loads of the
// next component are in flight while the current one is interpolated; vertices no owned
// cell needs (beyond n+1, in a ragged last tile) are not read.  All per-thread offsets of
// the fetch and of the three passes are computed once per tile.
constexpr int NFETCH = (NV + 255) / 256;
constexpr int NZR = (NZP + 255) / 256;
constexpr int NYR = (NYP + 255) / 256;

struct TileIdx {
  int fetch[NFETCH];  // point index of the fetched vertex, -1 if none
  int zsrc[NZR];      // z pass: first source in S.v, -1 if no item
  int ysrc[NYR];      // y pass: first source in S.z, -1 if no item
  int xsrc;           // x pass: first source in S.y
};

DEV TileIdx tile_index(const GD& g, const TileCell& t) {
  TileIdx x;
#pragma unroll
  for (int r = 0; r < NFETCH; ++r) {
    int q = threadIdx.x + 256 * r;
    int vx = q % VX, vy = (q / VX) % VY, vz = q / (VX * VY);
    int i = t.i0 - 1 + vx, j = t.j0 - 1 + vy, k = t.k0 - 1 + vz;
    bool in = q < NV && i <= g.n[0] + 1 && j <= g.n[1] + 1 && k <= g.n[2] + 1;
    x.fetch[r] = in ? at(g, i, j, k) : (q < NV ? -2 : -1);
  }
#pragma unroll
  for (int r = 0; r < NZR; ++r) {
    int q = threadIdx.x + 256 * r;
    int vx = q % VX, vy = (q / VX) % VY, z = q / (VX * VY);
    x.zsrc[r] = q < NZP ? vx + VX * (vy + VY * z) : -1;
  }
#pragma unroll
  for (int r = 0; r < NYR; ++r) {
    int q = threadIdx.x + 256 * r;
    int vx = q % VX, y = (q / VX) % CTY, z = q / (VX * CTY);
    x.ysrc[r] = q < NYP ? vx + VX * (y + VY * z) : -1;
  }
  x.xsrc = t.cx + VX * (t.cy + CTY * t.cz);
  return x;
}

// Points a tile does not need (fetch < 0) load the component's first element instead: the
// loads stay unconditional (a load under a branch is joined by a copy that waits for it, which
// would stall the interpolation pass it was meant to overlap), and such points only feed
// cells outside the block, whose results are discarded.
DEV void tile_fetch(const double* __restrict__ f, const TileIdx& x, double pre[NFETCH]) {
#pragma unroll
  for (int r = 0; r < NFETCH; ++r) pre[r] = ldu(f, x.fetch[r] >= 0 ? x.fetch[r] : 0);
}

DEV void tile_store(const TileIdx& x, const double pre[NFETCH], double* sv) {
#pragma unroll
  for (int r = 0; r < NFETCH; ++r)
    if (x.fetch[r] != -1) sv[threadIdx.x + 256 * r] = pre[r];
}

// Centre value of the staged component (every thread of the block must call it).
DEV double tile_value(TileLDS& S, const TileIdx& x) {
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NZR; ++r)
    if (x.zsrc[r] >= 0) {
      const double* p = S.v + x.zsrc[r];
      S.z[threadIdx.x + 256 * r] = lag(p[0], p[VX * VY], p[2 * VX * VY], p[3 * VX * VY]);
    }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NYR; ++r)
    if (x.ysrc[r] >= 0) {
      const double* p = S.z + x.ysrc[r];
      S.y[threadIdx.x + 256 * r] = lag(p[0], p[VX], p[2 * VX], p[3 * VX]);
    }
  __syncthreads();
  const double* p = S.y + x.xsrc;
  return lag(p[0], p[1], p[2], p[3]);
}

// Two components per round (values only): the passes of both run between the same three
// barriers, halving the barrier count of the value rounds.
struct TileLDS2 {
  double v[2][NV];
  double z[2][NZP];
  double y[2][NYP];
};

DEV void tile_store2(const TileIdx& x, const double pre[2][NFETCH], TileLDS2& S) {
#pragma unroll
  for (int r = 0; r < NFETCH; ++r)
    if (x.fetch[r] != -1) {
      S.v[0][threadIdx.x + 256 * r] = pre[0][r];
      S.v[1][threadIdx.x + 256 * r] = pre[1][r];
    }
}

DEV void tile_value2(TileLDS2& S, const TileIdx& x, double& v0, double& v1) {
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NZR; ++r)
    if (x.zsrc[r] >= 0)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const double* p = S.v[c] + x.zsrc[r];
        S.z[c][threadIdx.x + 256 * r] = lag(p[0], p[VX * VY], p[2 * VX * VY], p[3 * VX * VY]);
      }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NYR; ++r)
    if (x.ysrc[r] >= 0)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const double* p = S.z[c] + x.ysrc[r];
        S.y[c][threadIdx.x + 256 * r] = lag(p[0], p[VX], p[2 * VX], p[3 * VX]);
      }
  __syncthreads();
  const double* p = S.y[0] + x.xsrc;
  v0 = lag(p[0], p[1], p[2], p[3]);
  p = S.y[1] + x.xsrc;
  v1 = lag(p[0], p[1], p[2], p[3]);
}

// Derivatives of two staged components per round (cell kernel): 2 x (value, d/dz) after the z
// pass and 2 x (value, d/dy, d/dz-carry) after the y pass.
// The y-pass output reuses the staged values' storage (dead after the z pass), so a round must not
// store new values before every wave has finished the previous round's x pass.
struct TileLDS2D {
  union {
    double v[2][NV];
    double y[6][NYP];
  };
  double z[4][NZP];
};
static_assert(6 * NYP <= 2 * NV, "y-pass output must fit in the staged values' storage");

DEV void tile_store2d(const TileIdx& x, const double pre[2][NFETCH], TileLDS2D& S) {
#pragma unroll
  for (int r = 0; r < NFETCH; ++r)
    if (x.fetch[r] != -1) {
      S.v[0][threadIdx.x + 256 * r] = pre[0][r];
      S.v[1][threadIdx.x + 256 * r] = pre[1][r];
    }
}

// xf: the two components' values after the z and y passes at the vertex x positions on both sides
// of the thread's cell, i.e. at its lower and upper x faces (the x-face metric, interpolated across z
// then y as the x-face kernel does).
DEV void tile_derivs2(TileLDS2D& S, const TileIdx& x, const GD& g, double d0[3], double d1[3], double xf[2][2]) {
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NZR; ++r)
    if (x.zsrc[r] >= 0)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const double* p = S.v[c] + x.zsrc[r];
        double a = p[0], b = p[VX * VY], cc = p[2 * VX * VY], e = p[3 * VX * VY];
        S.z[2 * c][threadIdx.x + 256 * r] = lag(a, b, cc, e);
        S.z[2 * c + 1][threadIdx.x + 256 * r] = dlag(a, b, cc, e);
      }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NYR; ++r)
    if (x.ysrc[r] >= 0)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const double* p = S.z[2 * c] + x.ysrc[r];
        const double* q = S.z[2 * c + 1] + x.ysrc[r];
        double a = p[0], b = p[VX], cc = p[2 * VX], e = p[3 * VX];
        S.y[3 * c][threadIdx.x + 256 * r] = lag(a, b, cc, e);
        S.y[3 * c + 1][threadIdx.x + 256 * r] = dlag(a, b, cc, e);
        S.y[3 * c + 2][threadIdx.x + 256 * r] = lag(q[0], q[VX], q[2 * VX], q[3 * VX]);
      }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    double* d = c ? d1 : d0;
    const double* p = S.y[3 * c] + x.xsrc;
    const double* q = S.y[3 * c + 1] + x.xsrc;
    const double* w = S.y[3 * c + 2] + x.xsrc;
    d[0] = dlag(p[0], p[1], p[2], p[3]) * g.idx[0];
    d[1] = lag(q[0], q[1], q[2], q[3]) * g.idx[1];
    d[2] = lag(w[0], w[1], w[2], w[3]) * g.idx[2];
    xf[c][0] = p[1];
    xf[c][1] = p[2];
  }
}

// Centre derivatives (d/dx, d/dy, d/dz, scaled) of the staged component.
DEV void tile_derivs(TileLDS& S, const TileIdx& x, const GD& g, double d[3]) {
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NZR; ++r)
    if (x.zsrc[r] >= 0) {
      const double* p = S.v + x.zsrc[r];
      double a = p[0], b = p[VX * VY], c = p[2 * VX * VY], e = p[3 * VX * VY];
      S.z[threadIdx.x + 256 * r] = lag(a, b, c, e);
      S.z[NZP + threadIdx.x + 256 * r] = dlag(a, b, c, e);
    }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NYR; ++r)
    if (x.ysrc[r] >= 0) {
      const double* p = S.z + x.ysrc[r];
      const double* q = p + NZP;
      double a = p[0], b = p[VX], c = p[2 * VX], e = p[3 * VX];
      S.y[threadIdx.x + 256 * r] = lag(a, b, c, e);
      S.y[NYP + threadIdx.x + 256 * r] = dlag(a, b, c, e);
      S.y[2 * NYP + threadIdx.x + 256 * r] = lag(q[0], q[VX], q[2 * VX], q[3 * VX]);
    }
  __syncthreads();
  const double* p = S.y + x.xsrc;
  d[0] = dlag(p[0], p[1], p[2], p[3]) * g.idx[0];
  d[1] = lag(p[NYP], p[NYP + 1], p[NYP + 2], p[NYP + 3]) * g.idx[1];
  d[2] = lag(p[2 * NYP], p[2 * NYP + 1], p[2 * NYP + 2], p[2 * NYP + 3]) * g.idx[2];
}

// T^{mu nu} = (rho h + b^2) u u + (p + b^2/2) g^{mu nu} - b b   (eq. tmunu): T^00, T^0i, T^ij (symmetric)
DEV void tmunu_upper(const Geo& G, const State& St, double& T00, double T0[3], double Tk[6]) {
  double ia = 1.0 / G.alp, ia2 = ia * ia;
  double u0 = St.W * ia, u[3], b0 = St.W * St.Bv * ia, bu[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    u[a] = St.W * (St.v[a] - G.beta[a] * ia);
    bu[a] = (St.B[a] + G.alp * b0 * u[a]) / St.W;
  }
  double e = St.rhoh + St.bsq, pt = St.p + 0.5 * St.bsq;
  T00 = e * u0 * u0 - pt * ia2 - b0 * b0;
#pragma unroll
  for (int a = 0; a < 3; ++a) T0[a] = e * u0 * u[a] + pt * G.beta[a] * ia2 - b0 * bu[a];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = a; b < 3; ++b)
      Tk[sym(a, b)] = e * u[a] * u[b] + pt * (G.gu[sym(a, b)] - G.beta[a] * G.beta[b] * ia2) - bu[a] * bu[b];
}

// Geometric sources at a cell (eq. grmhdsrc in the 3+1 form): the momentum source
// 1/2 T^{mu nu} d_j g_{mu nu} is linear in the derivatives of the ten stored metric components,
// sum_c w_c d_j m_c, with weights w_c built from T, beta and gamma; the energy source is
// sum_q kc_q K_q over the six stored components of the extrinsic curvature (kc from T and beta)
// plus wa_j d_j alpha.  as = alpha sqrt(gamma) densitizes.  The weights need the state and the
// centre metric only, so they are formed before the curvature is interpolated.
struct SrcW {
  double w[10], wa[3], kc[6], as;
};

DEV void src_weights(const Geo& G, const double pr[5], const double Bt[3], double gam, SrcW& s) {
  State St;
  state_make(G, pr, Bt, gam, St);
  double T00, T0[3], Tk[6];
  tmunu_upper(G, St, T00, T0, Tk);
  double bl[3];
  lower(G.g, G.beta, bl);
  s.as = G.alp * G.sqrtg;
  // weights of d_j alpha, d_j beta^k, d_j gamma_ab in 1/2 T^{mu nu} d_j g_{mu nu}
  s.w[0] = -T00 * G.alp;
#pragma unroll
  for (int k = 0; k < 3; ++k)
    s.w[1 + k] = T00 * bl[k] + T0[0] * G.g[sym(0, k)] + T0[1] * G.g[sym(1, k)] + T0[2] * G.g[sym(2, k)];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = a; b < 3; ++b) {
      if (a == b)
        s.w[4 + sym(a, b)] = 0.5 * T00 * G.beta[a] * G.beta[a] + T0[a] * G.beta[a] + 0.5 * Tk[sym(a, a)];
      else
        s.w[4 + sym(a, b)] = T00 * G.beta[a] * G.beta[b] + T0[a] * G.beta[b] + T0[b] * G.beta[a] + Tk[sym(a, b)];
    }
  // energy source: (T00 beta^a beta^b + 2 T^{0a} beta^b + T^{ab}) K_ab summed over a, b, the two
  // orders of an off-diagonal pair joined; the lapse-gradient terms go with the derivatives of alpha
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = a; b < 3; ++b) {
      const double ab = T00 * G.beta[a] * G.beta[b] + 2.0 * T0[a] * G.beta[b] + Tk[sym(a, b)];
      s.kc[sym(a, b)] = a == b ? ab : ab + (T00 * G.beta[b] * G.beta[a] + 2.0 * T0[b] * G.beta[a] + Tk[sym(a, b)]);
    }
#pragma unroll
  for (int a = 0; a < 3; ++a) s.wa[a] = -(T00 * G.beta[a] + T0[a]);
}

// The extrinsic-curvature part of the energy source.
DEV double src_curv(const SrcW& s, const double K[6]) {
  double se = 0.0;
#pragma unroll
  for (int q = 0; q < 6; ++q) se += s.kc[q] * K[q];
  return se;
}

// Value rounds of the ten metric components at the tile's centres, two per round, round r+1's
// vertex tiles fetched during round r.  Every thread of the block must call it; the caller's
// previous LDS readers must be done (a fresh block, or a barrier since).
DEV void metric_values10(const GD& g, const double* metric, const TileIdx& x, double m[10], TileLDS2& S2) {
  double pre[2][NFETCH];
  tile_fetch(metric, x, pre[0]);
  tile_fetch(metric + g.N, x, pre[1]);
#pragma unroll
  for (int c = 0; c < 10; c += 2) {
    // the previous pair's passes no longer read S2.v (three barriers ago)
    tile_store2(x, pre, S2);
    if (c < 8) {
      tile_fetch(metric + (c + 2) * g.N, x, pre[0]);
      tile_fetch(metric + (c + 3) * g.N, x, pre[1]);
    }
    tile_value2(S2, x, m[c], m[c + 1]);
  }
}

// Value rounds of the ten metric and six curvature components at the tile's centres, two
// components per round (one set of barriers per pair), round r+1's vertex tiles fetched during
// round r.  Returns with the first metric component's tile fetched again into pre (the first
// derivative round's).  The rolled loop keeps the register footprint of one round, values
// landing by select chains (no dynamically indexed register arrays).  The leading barrier keeps
// a persistent workgroup's previous item reading the buffer the first round writes.  Every
// thread of the block must call it.
DEV void value_rounds16(const GD& g, const double* metric, const double* curv, const TileIdx& x, double m[10],
                        double K[6], double pre[NFETCH], TileLDS2& S2) {
  auto comp = [&](int r) { return r < 10 ? metric + r * g.N : (r < 16 ? curv + (r - 10) * g.N : metric); };
  double pp[2][NFETCH];
  tile_fetch(comp(0), x, pp[0]);
  tile_fetch(comp(1), x, pp[1]);
  __syncthreads();
#pragma unroll 1
  for (int c = 0; c < 16; c += 2) {
    tile_store2(x, pp, S2);
    tile_fetch(comp(c + 2), x, pp[0]);
    if (c < 14) tile_fetch(comp(c + 3), x, pp[1]);
    double v0, v1;
    tile_value2(S2, x, v0, v1);
#pragma unroll
    for (int q = 0; q < 10; ++q) m[q] = c == q ? v0 : (c + 1 == q ? v1 : m[q]);
#pragma unroll
    for (int q = 0; q < 6; ++q) K[q] = c == 10 + q ? v0 : (c + 1 == 10 + q ? v1 : K[q]);
  }
  // comp(16) (metric component 0, the first derivative round's) is already in pp[0]
#pragma unroll
  for (int r = 0; r < NFETCH; ++r) pre[r] = pp[0][r];
}

// Value rounds of the six curvature components alone (the pairs of value_rounds16, so the same
// arithmetic), then metric component 0's vertex tile fetched into pre.  Leading barrier: the
// block's previous LDS readers are done.  Every thread of the block must call it.
DEV void curv_rounds(const GD& g, const double* metric, const double* curv, const TileIdx& x, double K[6],
                     double pre[NFETCH], TileLDS2& S2) {
  double pp[2][NFETCH];
  tile_fetch(curv, x, pp[0]);
  tile_fetch(curv + g.N, x, pp[1]);
  __syncthreads();
#pragma unroll 1
  for (int c = 0; c < 6; c += 2) {
    tile_store2(x, pp, S2);
    tile_fetch(c < 4 ? curv + (c + 2) * g.N : metric, x, pp[0]);
    if (c < 4) tile_fetch(curv + (c + 3) * g.N, x, pp[1]);
    double v0, v1;
    tile_value2(S2, x, v0, v1);
#pragma unroll
    for (int q = 0; q < 6; ++q) K[q] = c == q ? v0 : (c + 1 == q ? v1 : K[q]);
  }
#pragma unroll
  for (int r = 0; r < NFETCH; ++r) pre[r] = pp[0][r];
}

// Derivative rounds of the ten metric components, two per round, accumulated into the sources:
// src[1 + j] += w_c d_j m_c and, with alpha's, src[4] += wa_j d_j alpha.  pre0: metric
// component 0's vertex tile, already fetched.  Every thread of the block must call it.
// xfm (or NULL): the x-face metric of the tile's cells' faces is stored there, ten fields indexed like
// the fluxes (the face between cells i-1 and i at cell i): each cell its lower face, the last cell of
// a row also its upper one.  cell: the thread's cell (i, j, k), valid with `valid`.
DEV void src_deriv_rounds(const GD& g, const double* metric, const TileIdx& x, bool valid, const double pre0[NFETCH],
                          const SrcW& s, double src[5], TileLDS2D& SD, double* xfm = nullptr, int fid = 0,
                          bool last_x = false) {
  double pp[2][NFETCH];
#pragma unroll
  for (int r = 0; r < NFETCH; ++r) pp[0][r] = pre0[r];
  tile_fetch(metric + g.N, x, pp[1]);
#pragma unroll 1
  for (int c = 0; c < 10; c += 2) {
    __syncthreads();
    tile_store2d(x, pp, SD);
    if (c < 8) {
      tile_fetch(metric + (c + 2) * g.N, x, pp[0]);
      tile_fetch(metric + (c + 3) * g.N, x, pp[1]);
    }
    double d0[3], d1[3], xf[2][2];
    tile_derivs2(SD, x, g, d0, d1, xf);
    if (xfm && valid) {
      xfm[(size_t)c * g.N + fid] = xf[0][0];
      xfm[(size_t)(c + 1) * g.N + fid] = xf[1][0];
      if (last_x) {
        xfm[(size_t)c * g.N + fid + 1] = xf[0][1];
        xfm[(size_t)(c + 1) * g.N + fid + 1] = xf[1][1];
      }
    }
    if (valid) {
      double w0 = s.w[0], w1 = s.w[1];
#pragma unroll
      for (int q = 2; q < 10; ++q) {
        w0 = c == q ? s.w[q] : w0;
        w1 = c + 1 == q ? s.w[q] : w1;
      }
      src[1] += w0 * d0[0];
      src[2] += w0 * d0[1];
      src[3] += w0 * d0[2];
      if (c == 0) src[4] += s.wa[0] * d0[0] + s.wa[1] * d0[1] + s.wa[2] * d0[2];
      src[1] += w1 * d1[0];
      src[2] += w1 * d1[1];
      src[3] += w1 * d1[2];
    }
  }
}

// Derivative rounds of the ten metric components, two per round, contracted with a cotangent:
// E[c] = sum_j r[j] d_j m_c at the tile's centres (derivatives scaled by 1/dx_j), dal[j] = d_j alpha,
// and flat = every derivative is zero.  pre0: metric component 0's vertex tile, already fetched.
// Every thread of the block must call it.
DEV void metric_derivs_dot(const GD& g, const double* metric, const TileIdx& x, const double pre0[NFETCH],
                           const double r[3], double E[10], double dal[3], bool& flat, TileLDS2D& SD) {
  double pp[2][NFETCH];
#pragma unroll
  for (int q = 0; q < NFETCH; ++q) pp[0][q] = pre0[q];
  tile_fetch(metric + g.N, x, pp[1]);
  flat = true;
#pragma unroll 1
  for (int c = 0; c < 10; c += 2) {
    __syncthreads();
    tile_store2d(x, pp, SD);
    if (c < 8) {
      tile_fetch(metric + (c + 2) * g.N, x, pp[0]);
      tile_fetch(metric + (c + 3) * g.N, x, pp[1]);
    }
    double d0[3], d1[3], xf[2][2];
    tile_derivs2(SD, x, g, d0, d1, xf);
    const double e0 = r[0] * d0[0] + r[1] * d0[1] + r[2] * d0[2];
    const double e1 = r[0] * d1[0] + r[1] * d1[1] + r[2] * d1[2];
#pragma unroll
    for (int q = 0; q < 10; ++q) E[q] = c == q ? e0 : (c + 1 == q ? e1 : E[q]);
    if (c == 0) {
      dal[0] = d0[0];
      dal[1] = d0[1];
      dal[2] = d0[2];
    }
    flat = flat && d0[0] == 0.0 && d0[1] == 0.0 && d0[2] == 0.0 && d1[0] == 0.0 && d1[1] == 0.0 && d1[2] == 0.0;
  }
}

// =======================================================================================
// prim -> cons on owned cells.
DEV void prim2con_body(const GD& g, double gam, const double* __restrict__ metric, const double* __restrict__ A,
                       const double* __restrict__ prim, double* __restrict__ cons, unsigned tile) {
  int i, j, k;
  if (!box_at<64, 4>(g.n, tile, threadIdx.x, i, j, k)) return;
  int id = at(g, i, j, k);
  double m[10];
  centre_metric(metric, g.N, id - 1 - g.sy - g.sz, g.sy, g.sz, m);
  Geo G;
  geo_from(m, G);
  double Bt[3], pr[5];
  centre_B(A, g, id, Bt);
#pragma unroll
  for (int c = 0; c < 5; ++c) pr[c] = prim[c * g.N + id];
  State S;
  state_make(G, pr, Bt, gam, S);
  double U[5];
  cons_of(G, S, U);
#pragma unroll
  for (int c = 0; c < 5; ++c) cons[c * g.N + id] = U[c];
}

// LDS written by this wavefront and read back by it only: its accesses execute in order, and a
// wavefront barrier keeps the compiler from moving the reads above the writes.
DEV void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// c2p on owned cells, tiled: the ten metric components are interpolated to the centres
// through LDS (Sec. 3.2), then each thread recovers its cell (Secs. 3.5, 3.6).
struct C2PArgs {
  const double* metric;
  const double* A;
  double* cons;
  double* prim;
  uint8_t* flags;
  unsigned long long* stats;
  const float* mlp;  // learned guess (LEARNED instantiation only)
  mlpd::Stdz z;
  const double* curv;  // SRC instantiation: curvature at vertices
  double* src;         // SRC instantiation: densitized sources out, [4] (S_x, S_y, S_z, tau)
};

// A wavefront with cells that have no usable warm start (previous primitives that are not a physical
// state: the first recovery of a block, reset or prolonged cells) evaluates the learned guess's network on
// its 64 cells (through F and Y, LDS of its own) and seeds Noble's iteration of those cells with it; the
// other cells, and wavefronts without such cells, start from their previous primitives as in the plain
// form.  Returns whether zw holds a seed.  Every lane of the wavefront must call it.
DEV bool learned_seed(const C2PArgs& a, const C2PParams& P, const Geo& G, const double U[5], const double Bt[3],
                      const double prev[5], bool valid, float (*F)[mlpd::NI], float (*Y)[mlpd::NO], double zw[2]) {
  using namespace mlpd;
  const int l = __lane_id(), lr = l & 15, lg = l >> 4;
  float f[NI];
  bool usable = false;
  C2PIn c;
  bool in = valid && isfinite(U[0]) && isfinite(U[1]) && isfinite(U[2]) && isfinite(U[3]) && isfinite(U[4]) &&
            U[0] >= G.sqrtg * P.rho_atm;
  if (in) in = !warm_usable(G, prev, P);
  // the network runs for whole wavefronts only (matrix instructions), and only where it is needed
  if (__ballot(in) == 0) return false;
  if (in) {
    c2p_input(G, U, Bt, c);
    features(G, c, P.gam, f, usable);
  }
#pragma unroll
  for (int k = 0; k < NI; ++k) F[l][k] = usable ? (f[k] - a.z.is[k]) * a.z.isc[k] : 0.0f;
  wave_lds_sync();
  f4 y[4];
  mlp_fwd<false>(a.mlp, F, y, nullptr);
  if (lg == 0)
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
      for (int q = 0; q < NO; ++q) Y[nt * 16 + lr][q] = a.z.os[q] + y[nt][q] / a.z.osc[q];
  wave_lds_sync();
  if (!usable) return false;
  const double W = (double)__expf(Y[l][0]);
  const double wcap = 1.0 - 1.0 / (P.wmax * P.wmax);
  zw[0] = c.D * (double)__expf(Y[l][1]);
  zw[1] = fmin(fmax(1.0 - 1.0 / (W * W), 0.0), wcap);
  return isfinite(zw[0]) && zw[0] > 0.0;
}

// Recovery counters of a workgroup: one push, all counters in one instruction (they share a cache line).
// Pushes to one line serialize in L2, and where most cells fail or are reset (a star in vacuum: 97%) one
// atomic per wavefront and counter took 4 of the 4.6 ms of a 160^3 launch.  Every thread must call it.
DEV void c2p_count(uint32_t fl, int iters, unsigned long long* stats) {
  __shared__ unsigned cnt[4][6];
  const unsigned it = (unsigned)wave_max_int(iters);
  const unsigned b[6] = {(unsigned)__popcll(__ballot(fl & 1u)),  (unsigned)__popcll(__ballot(fl & 2u)),
                         (unsigned)__popcll(__ballot(fl & 4u)),  (unsigned)__popcll(__ballot(fl & 8u)),
                         (unsigned)__popcll(__ballot(fl & 16u)), it};
  if (__lane_id() == 0)
#pragma unroll
    for (int q = 0; q < 6; ++q) cnt[threadIdx.x >> 6][q] = b[q];
  __syncthreads();
  if (threadIdx.x < 6) {
    const int q = threadIdx.x;
    const unsigned c0 = cnt[0][q], c1 = cnt[1][q], c2 = cnt[2][q], c3 = cnt[3][q];
    const unsigned v = q < 5 ? c0 + c1 + c2 + c3 : max(max(c0, c1), max(c2, c3));
    if (q < 5 && v) atomicAdd(stats + q, (unsigned long long)v);
    if (q == 5 && v) atomic_max_u64(stats + 5, v);
  }
}

// LEARNED: see learned_seed.
// SRC: the cell's geometric sources (eq. grmhdsrc) follow from the recovered state, with the
// centre metric of the recovery's own value rounds (the six curvature components join them) and
// the metric derivative rounds after it; stored densitized, alpha sqrt(gamma) S (rounded on its own).
template <bool LEARNED, bool SRC = false>
DEV void c2p_body(const GD& g, const C2PParams& P, const C2PArgs& a, TileLDS& S, unsigned tile) {
  const double* __restrict__ metric = a.metric;
  const double* __restrict__ A = a.A;
  double* __restrict__ cons = a.cons;
  double* __restrict__ prim = a.prim;
  uint8_t* __restrict__ flags = a.flags;
  const TileCell t = tile_cell(g, tile);
  const TileIdx x = tile_index(g, t);
  double m[10];
  double K[6], pre0[NFETCH];  // SRC only
  TileLDS2& S2 = *reinterpret_cast<TileLDS2*>(&S);
  metric_values10(g, metric, x, m, S2);
  uint32_t fl = 0;
  int iters = 0;
  const int id = t.valid ? at(g, t.i0 + t.cx, t.j0 + t.cy, t.k0 + t.cz) : 0;
  Geo G;
  double Bt[3], U[5], prev[5], out[5];
  if (t.valid) {
    geo_from(m, G);
    centre_B(A, g, id, Bt);
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      U[c] = cons[c * g.N + id];
      prev[c] = prim[c * g.N + id];
    }
  }
  double zw[2] = {0.0, 0.0};
  bool use_guess = false;
  if constexpr (LEARNED) {
    // F and Y (one part per wavefront) lie in TileLDS's z and y arrays, i.e. over the value rounds'
    // staged vertices and z-pass output, which every thread has finished reading at the barrier
    // before the last x pass; that x pass reads the y-pass output, which lies beyond both
    const int w = threadIdx.x >> 6;
    use_guess = learned_seed(a, P, G, U, Bt, prev, t.valid, reinterpret_cast<float(*)[64][mlpd::NI]>(S.z)[w],
                             reinterpret_cast<float(*)[64][mlpd::NO]>(S.y)[w], zw);
  }
  if (t.valid) {
    fl = c2p_point(G, U, Bt, prev, P, out, iters, use_guess ? zw : nullptr);
#pragma unroll
    for (int c = 0; c < 5; ++c) prim[c * g.N + id] = out[c];
    if (fl & 4u) {
#pragma unroll
      for (int c = 0; c < 5; ++c) cons[c * g.N + id] = U[c];
    }
    if (flags) flags[id] = (uint8_t)fl;
  }
  if constexpr (SRC) {
    SrcW sw;
    sw.as = 0.0;
    double src[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    if (t.valid) src_weights(G, out, Bt, P.gam, sw);
    // curvature rounds after the recovery and the weights (fewer live registers); the tile's LDS
    // offsets are formed again (from an opaque copy of the tile id, so they are not held across the
    // recovery)
    const TileIdx x2 = tile_index(g, tile_cell(g, (unsigned)__builtin_amdgcn_readfirstlane((int)tile)));
    curv_rounds(g, metric, a.curv, x2, K, pre0, S2);
    if (t.valid) src[4] = src_curv(sw, K);
    src_deriv_rounds(g, metric, x2, t.valid, pre0, sw, src, *reinterpret_cast<TileLDS2D*>(&S), a.src + 4 * g.N, id,
                     t.i0 + t.cx == g.n[0] - 1);
    if (t.valid)
#pragma unroll
      for (int c = 1; c < 5; ++c) a.src[(c - 1) * g.N + id] = __dmul_rn(sw.as, src[c]);
  }
  if (a.stats) c2p_count(fl, iters, a.stats);
}

// The recovery and the cell's sources with the interpolated spacetime data given (asterx_geometry): one
// thread per owned cell, x fastest, no LDS passes and no barriers before the counters.  Per cell it reads
// 46 interpolated values, 13 of the state and the potential, and writes nine: a streaming kernel.
struct C2PGeoLDS {
  float F[4][64][mlpd::NI], Y[4][64][mlpd::NO];
};
template <bool LEARNED>
DEV void c2p_geo_body(const GD& g, const C2PParams& P, const C2PArgs& a, const double* __restrict__ cen, unsigned tile,
                      C2PGeoLDS* L) {
  int i, j, k;
  const bool valid = lin_at(g.n, tile, threadIdx.x, i, j, k);
  const int id = valid ? at(g, i, j, k) : at(g, 0, 0, 0);
  uint32_t fl = 0;
  int iters = 0;
  Geo G;
  double m[10], Bt[3], U[5], prev[5], out[5];
#pragma unroll
  for (int c = 0; c < 10; ++c) m[c] = ldu(cen + (size_t)c * g.N, id);
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    U[c] = ldu(a.cons + (size_t)c * g.N, id);
    prev[c] = ldu(a.prim + (size_t)c * g.N, id);
  }
  centre_B(a.A, g, id, Bt);
  geo_from(m, G);
  double zw[2] = {0.0, 0.0};
  bool use_guess = false;
  if constexpr (LEARNED) {
    const int w = threadIdx.x >> 6;
    use_guess = learned_seed(a, P, G, U, Bt, prev, valid, L->F[w], L->Y[w], zw);
  }
  if (valid) {
    fl = c2p_point(G, U, Bt, prev, P, out, iters, use_guess ? zw : nullptr);
#pragma unroll
    for (int c = 0; c < 5; ++c) a.prim[(size_t)c * g.N + id] = out[c];
    if (fl & 4u) {
#pragma unroll
      for (int c = 0; c < 5; ++c) a.cons[(size_t)c * g.N + id] = U[c];
    }
    if (a.flags) a.flags[id] = (uint8_t)fl;
    SrcW sw;
    src_weights(G, out, Bt, P.gam, sw);
    double src[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < 10; ++c) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const double v = ldu(cen + (size_t)(10 * (d + 1) + c) * g.N, id);
        src[d] += sw.w[c] * v;
        if (c == 0) src[3] += sw.wa[d] * v;
      }
    }
#pragma unroll
    for (int q = 0; q < 6; ++q) src[3] += sw.kc[q] * ldu(cen + (size_t)(40 + q) * g.N, id);
#pragma unroll
    for (int c = 0; c < 4; ++c) a.src[(size_t)c * g.N + id] = sw.as * src[c];
  }
  if (a.stats) c2p_count(fl, iters, a.stats);
}

// Ghost points along axis d: the ghost index set of axis d times the full extents of the other two axes.
__host__ __device__ inline long long fill_points(const GD& g, int d) {
  long long cnt = 2 * g.ng + 1;
  for (int t = 0; t < 3; ++t)
    if (t != d) cnt *= (g.n[t] + 2 * g.ng + 1);
  return cnt;
}

// Ghost fill in one pass: the ghost points of x (all y, z), of y (owned x, all z) and of z (owned x, y), one
// thread per point.  Defined as axis passes (x, then y, then z), each over the full extents of the others; every
// ghost value is then a function of owned points: one per axis whose kind copies or wraps, two per axis that
// extrapolates, combined in x, y, z order as the passes would, so the result is theirs bit for bit (no
// contraction: linear extrapolation is one multiply, then one add; periodic offsets are added axis by axis).
// Up to three groups of consecutive fields with kinds of their own, so that a state is one launch: small blocks
// pay for the launches (a state with an extrapolated potential took five: 16^3, two stages per step, 181 -> 148 us
// per step), and in batches the ghosts' index arithmetic is done once (64 patches: 190 -> 125 us per stage).
struct FillArgs {
  double* f;
  int ngroup;
  int end[3];        // fields [end[q - 1], end[q])
  int kind[3][3];    // [group][axis]
  int shifted;       // the group of at most three fields whose periodic wraps add shift, or -1
  double shift[3][3];  // [field of the group][axis]
};

// The values K fields (st apart) get at a ghost point where some axes extrapolate (bits of lin): o0 the source
// offsets per axis, o1 the second ones, c their weights.
template <int K>
struct FillVals {
  double v[K];
};
template <int K>
DEV FillVals<K> fill_values(const double* F, size_t st, const int o0[3], const int o1[3], const double c[3], int lin) {
#pragma clang fp contract(off)
  auto mix = [](const FillVals<K>& a, const FillVals<K>& b, double w) {
    FillVals<K> r;
#pragma unroll
    for (int k = 0; k < K; ++k) r.v[k] = a.v[k] + w * (b.v[k] - a.v[k]);
    return r;
  };
  auto f = [&](int o) {
    FillVals<K> r;
#pragma unroll
    for (int k = 0; k < K; ++k) r.v[k] = F[k * st + o];
    return r;
  };
  auto fx = [&](int o) { return lin & 1 ? mix(f(o + o0[0]), f(o + o1[0]), c[0]) : f(o + o0[0]); };
  auto fy = [&](int o) { return lin & 2 ? mix(fx(o + o0[1]), fx(o + o1[1]), c[1]) : fx(o + o0[1]); };
  return lin & 4 ? mix(fy(o0[2]), fy(o1[2]), c[2]) : fy(o0[2]);
}

template <bool LIN>
DEV void fill_body(const GD& g, const FillArgs& a, double* __restrict__ u, unsigned tile) {
#pragma clang fp contract(off)
  const int ng = g.ng, G = 2 * ng + 1;
  const int E1 = g.n[1] + 2 * ng + 1;
  const long long s0 = (long long)G * E1 * (g.n[2] + 2 * ng + 1), s1 = (long long)g.n[0] * G * (g.n[2] + 2 * ng + 1),
                  s2 = (long long)g.n[0] * g.n[1] * G;
  long long t = (long long)tile * 256 + threadIdx.x;
  auto gh = [&](int q, int n) { return q < ng ? q - ng : n + (q - ng); };
  int idx[3];
  if (t < s0) {
    idx[0] = gh((int)(t % G), g.n[0]);
    const long long r = t / G;
    idx[1] = (int)(r % E1) - ng;
    idx[2] = (int)(r / E1) - ng;
  } else if ((t -= s0) < s1) {
    idx[0] = (int)(t % g.n[0]);
    const long long r = t / g.n[0];
    idx[1] = gh((int)(r % G), g.n[1]);
    idx[2] = (int)(r / G) - ng;
  } else if ((t -= s1) < s2) {
    idx[0] = (int)(t % g.n[0]);
    const long long r = t / g.n[0];
    idx[1] = (int)(r % g.n[1]);
    idx[2] = gh((int)(r / g.n[1]), g.n[2]);
  } else {
    return;
  }
  const int dst = at(g, idx[0], idx[1], idx[2]), st[3] = {1, g.sy, g.sz}, org = at(g, 0, 0, 0);
  int begin = 0;
#pragma unroll 1
  for (int q = 0; q < a.ngroup; ++q) {
    const int end = a.end[q];
    int o0[3], o1[3], wrap[3], lin = 0;
    double c[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int s = idx[d], n = g.n[d], kind = a.kind[q][d];
      int src = s, second = s;
      wrap[d] = 0;
      c[d] = 0.0;
      if (s < 0 || s >= n) {
        if (kind == ASTERX_BC_PERIODIC) {
          src = ((s % n) + n) % n;
          wrap[d] = (s - src) / n;
        } else {
          src = s < 0 ? 0 : n - 1;
          if (LIN && kind == ASTERX_BC_LINEAR) {
            // f(0) + s (f(1) - f(0)); f(n-1) + (n - 1 - s) (f(n-2) - f(n-1))
            second = s < 0 ? 1 : n - 2;
            c[d] = (double)(s < 0 ? s : n - 1 - s);
            lin |= 1 << d;
          }
        }
      }
      o0[d] = src * st[d] + (d == 0 ? org : 0);
      o1[d] = second * st[d] + (d == 0 ? org : 0);
    }
    const int so = o0[0] + o0[1] + o0[2];
    if (LIN && lin) {
      int f = begin;
#pragma unroll 1
      for (; f + 3 <= end; f += 3) {
        const FillVals<3> v = fill_values<3>(u + (size_t)f * g.N, g.N, o0, o1, c, lin);
#pragma unroll
        for (int k = 0; k < 3; ++k) u[(size_t)(f + k) * g.N + dst] = v.v[k];
      }
#pragma unroll 1
      for (; f < end; ++f) u[(size_t)f * g.N + dst] = fill_values<1>(u + (size_t)f * g.N, g.N, o0, o1, c, lin).v[0];
    } else if (q == a.shifted) {
      for (int f = begin; f < end; ++f) {
        double* F = u + (size_t)f * g.N;
        double v = F[so];
#pragma unroll
        for (int d = 0; d < 3; ++d)
          if (wrap[d] != 0 && a.shift[f - begin][d] != 0.0) v = v + (double)wrap[d] * a.shift[f - begin][d];
        F[dst] = v;
      }
    } else {
      // the loads of several fields in flight together: a field's store may not be overtaken by the next loads
      int f = begin;
#pragma unroll 1
      for (; f + 5 <= end; f += 5) {
        double v[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) v[k] = u[(size_t)(f + k) * g.N + so];
#pragma unroll
        for (int k = 0; k < 5; ++k) u[(size_t)(f + k) * g.N + dst] = v[k];
      }
#pragma unroll 1
      for (; f < end; ++f) u[(size_t)f * g.N + dst] = u[(size_t)f * g.N + so];
    }
    begin = end;
  }
}

// Centre field of every cell in [-ng, n+ng-1]^3 (read by the face stencils).
DEV void bcent_body(const GD& g, const double* __restrict__ A, double* __restrict__ bc, unsigned tile) {
  int e[3] = {g.n[0] + 2 * g.ng, g.n[1] + 2 * g.ng, g.n[2] + 2 * g.ng};
  int a, b, c;
  if (!lin_at(e, tile, threadIdx.x, a, b, c)) return;
  int id = at(g, a - g.ng, b - g.ng, c - g.ng);
  double Bt[3];
  centre_B(A, g, id, Bt);
  bc[id] = Bt[0];
  bc[g.N + id] = Bt[1];
  bc[2 * g.N + id] = Bt[2];
}

// ---------------------------------------------------------------------------------------
// Spacetime data interpolated once and stored (Sec. 3.2 Lagrange weights): the metric at the faces of
// each direction, and for the recovery and the sources its centre values and derivatives and the centre
// curvature.  One lane per x position and R rows (y) marches along z with the last four planes of every pass
// in registers: per plane the pass along x of the R + 3 vertex rows the rows' y stencils span, the pass along
// y, then the pass along z.  No LDS and no barriers.  Several rows per lane share their vertex rows.
// Bound by its 76 streams of stores (128^3, everything: 0.50 ms; stores alone 0.39 to 0.45, loads and arithmetic
// alone 0.20 to 0.25; one row per lane 0.53, cached instead of nontemporal stores 0.55), once per step, where the
// four stages' recoveries and faces gathered the same values from the vertices: recovery 0.404 -> 0.271 ms, x, y
// and z faces 0.214, 0.241, 0.247 -> 0.150, 0.180, 0.198 ms per stage (with the face kernels below).
// Points: x, y, z in [-lo, n + max(lo - 2, 0)]; a face direction's own index in [0, n], centres owned.
struct GeomArgs {
  const double* metric;
  const double* curv;
  // face metric along each direction: components 0..6 from fa, 7..9 from fb (a field apart each)
  double* fa[3];
  double* fb[3];
  double* cen;  // ten values, then d/dx, d/dy, d/dz of the ten, then six curvature values
  int lo, zl;   // transverse reach of the faces, planes per work item
};
enum { GM_X = 1, GM_Y = 2, GM_Z = 4, GM_C = 8 };
constexpr int GEO_FIELDS = ASTERX_GEO_FIELDS, GEO_CEN = 30;

__host__ __device__ inline void geom_box(const int n[3], int lo, int e[3]) {
  for (int a = 0; a < 3; ++a) e[a] = n[a] + 2 * lo - 1 + (lo < 2 ? 1 : 0);
}
// Planes per item: long marches reload the three planes before their first output less often, short ones
// fill the chip: with few columns a march of one or two dozen planes is a serial chain of that many loads.
__host__ __device__ inline int geom_planes(const int e[3]) {
  const long long waves = ((long long)e[0] * e[1] + 63) / 64 * e[2];
  return waves >= 16384 ? 16 : (waves >= 2048 ? 8 : 4);
}
// Rows per lane: four, or two where the centre data's five rolling quantities leave registers for no more.
template <int MASK>
constexpr int geom_rows() { return (MASK & GM_C) ? 2 : 4; }
inline unsigned geom_items(const GD& g, int lo, int comps, int rows) {
  int e[3];
  geom_box(g.n, lo, e);
  const int zl = geom_planes(e);
  return (unsigned)(((long long)g.ld0 * ((e[1] + rows - 1) / rows) + 63) / 64 * ((e[2] + zl - 1) / zl) * comps);
}

// One wavefront's item: component comp of 64 positions (along the stored rows, padding included, so that its
// loads and stores are whole cache lines) times R rows over zl planes.
template <int MASK>
DEV void geom_wave(const GD& g, const GeomArgs& ga, unsigned item) {
  constexpr int R = geom_rows<MASK>();
  constexpr bool X = MASK & GM_X, Y = MASK & GM_Y, Z = MASK & GM_Z, C = MASK & GM_C, MARCH = X || Y || C;
  int e[3];
  geom_box(g.n, ga.lo, e);
  const unsigned nrow = (unsigned)(e[1] + R - 1) / R;
  const unsigned ncol = ((unsigned)g.ld0 * nrow + 63) / 64, nch = (unsigned)(e[2] + ga.zl - 1) / ga.zl;
  const unsigned col = item % ncol, ch = (item / ncol) % nch, comp = item / (nch * ncol);
  const int lo = ga.lo;
  const unsigned q = col * 64 + __lane_id();
  const int xs = (int)(q % (unsigned)g.ld0) - g.ng, ys = (int)(q / (unsigned)g.ld0) * R - lo;
  const bool in = xs >= -lo && xs < e[0] - lo && ys < e[1] - lo;
  const int x = in ? xs : 0, y = in ? ys : 0;
  const int z0 = (int)ch * ga.zl - lo, z1 = min(z0 + ga.zl, e[2] - lo);
  const bool curv = C && comp >= 10;
  const double* f = curv ? ga.curv + (size_t)(comp - 10) * g.N : ga.metric + (size_t)comp * g.N;
  auto dst = [&](int d) { return comp < 7 ? ga.fa[d] + (size_t)comp * g.N : ga.fb[d] + (size_t)(comp - 7) * g.N; };
  // rows of the x faces, of the y faces, of the z faces and of the centres
  const int ty = g.n[1] + lo - 2, tx = g.n[0] + lo - 2;
  bool fx[R], fy[R], fz[R], own[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    fx[r] = in && !curv && x >= 0 && x <= g.n[0] && y + r <= ty;
    fy[r] = in && !curv && x <= tx && y + r >= 0 && y + r <= g.n[1];
    fz[r] = in && !curv && x <= tx && y + r <= ty;
    own[r] = in && (unsigned)x < (unsigned)g.n[0] && (unsigned)(y + r) < (unsigned)g.n[1];
  }
  // the last vertex row a lane's rows need may lie beyond the stored ones where its last rows have no output
  const int rmax = g.n[1] + g.ng - y;
  const int base = at(g, x, y, 0);
  // the last four planes: raw values' y pass, x pass, and the x pass's and its derivative's y passes
  double wv[R][4], wx[R][4], wy[R][4], wdx[R][4], wdy[R][4];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int k = 0; k < 4; ++k) wv[r][k] = wx[r][k] = wy[r][k] = wdx[r][k] = wdy[r][k] = 0.0;
#pragma unroll 4
  for (int p = MARCH ? z0 - 1 : z0; p < (MARCH ? z1 + 2 : z1); ++p) {
    const int id = base + p * g.sz;
    double raw[R + 3], vx[R + 3], dx[R + 3];
#pragma unroll
    for (int r = 0; r < R + 3; ++r) {
      const int o = id + min(r - 1, rmax) * g.sy;
      const double v0 = ldu(f - 1, o), v1 = ldu(f, o), v2 = ldu(f + 1, o), v3 = ldu(f + 2, o);
      raw[r] = v1;
      vx[r] = lag(v0, v1, v2, v3);
      if constexpr (C) dx[r] = dlag(v0, v1, v2, v3);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        wv[r][k] = wv[r][k + 1];
        wx[r][k] = wx[r][k + 1];
        wy[r][k] = wy[r][k + 1];
        wdx[r][k] = wdx[r][k + 1];
        wdy[r][k] = wdy[r][k + 1];
      }
      if constexpr (X) wv[r][3] = lag(raw[r], raw[r + 1], raw[r + 2], raw[r + 3]);
      if constexpr (Y) wx[r][3] = vx[r + 1];
      if constexpr (Z || C) wy[r][3] = lag(vx[r], vx[r + 1], vx[r + 2], vx[r + 3]);
      if constexpr (C) {
        wdx[r][3] = lag(dx[r], dx[r + 1], dx[r + 2], dx[r + 3]);
        wdy[r][3] = dlag(vx[r], vx[r + 1], vx[r + 2], vx[r + 3]);
      }
      if constexpr (Z)
        if (fz[r] && p >= 0 && p <= g.n[2] && p >= z0 && p < z1)
          __builtin_nontemporal_store(wy[r][3], dst(2) + id + r * g.sy);
    }
    if constexpr (MARCH) {
      const int z = p - 2;
      if (z < z0) continue;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int o = id - 2 * g.sz + r * g.sy;
        if (z <= g.n[2] + lo - 2) {
          if constexpr (X)
            if (fx[r]) __builtin_nontemporal_store(lag(wv[r][0], wv[r][1], wv[r][2], wv[r][3]), dst(0) + o);
          if constexpr (Y)
            if (fy[r]) __builtin_nontemporal_store(lag(wx[r][0], wx[r][1], wx[r][2], wx[r][3]), dst(1) + o);
        }
        if constexpr (C)
          if (own[r] && z >= 0 && z < g.n[2]) {
            const double val = lag(wy[r][0], wy[r][1], wy[r][2], wy[r][3]);
            if (curv) {
              __builtin_nontemporal_store(val, ga.cen + (size_t)(40 + comp - 10) * g.N + o);
            } else {
              double* c = ga.cen + (size_t)comp * g.N + o;
              __builtin_nontemporal_store(val, c);
              __builtin_nontemporal_store(lag(wdx[r][0], wdx[r][1], wdx[r][2], wdx[r][3]) * g.idx[0], c + 10 * g.N);
              __builtin_nontemporal_store(lag(wdy[r][0], wdy[r][1], wdy[r][2], wdy[r][3]) * g.idx[1], c + 20 * g.N);
              __builtin_nontemporal_store(dlag(wy[r][0], wy[r][1], wy[r][2], wy[r][3]) * g.idx[2], c + 30 * g.N);
            }
          }
      }
    }
  }
}

template <int kind, class T>
DEV T recon_right_face(const T a[5], double eps, double q) {
  if (kind == ASTERX_RECON_MINMOD) return a[2] + 0.5 * mm(a[2] - a[1], a[3] - a[2]);
  if (kind == ASTERX_RECON_PPM) {
    T s1 = mc_slope(a[0], a[1], a[2]);
    T s2 = mc_slope(a[1], a[2], a[3]);
    T s3 = mc_slope(a[2], a[3], a[4]);
    const double sixth = 1.0 / 6.0;
    T fl = 0.5 * (a[1] + a[2]) - (s2 - s1) * sixth;
    T fr = 0.5 * (a[2] + a[3]) - (s3 - s2) * sixth;
    ppm_limit(a[2], fl, fr);
    return fr;
  }
  if (kind == ASTERX_RECON_MP5) return mp5_face(a[0], a[1], a[2], a[3], a[4]);
  return wenoz_face(a[0], a[1], a[2], a[3], a[4], eps, q);
}

// Transpose of mp5_face on its active branch: ab[k] = xb d(face value) / d(a[k]); a side whose cotangent is zero
// sends nothing, whatever its slopes.
DEV void mp5_face_vjp(const double a[5], double xb, double ab[5]) {
  Lin5 s[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    s[k] = Lin5(a[k]);
    s[k].c[k] = 1.0;
  }
  const Lin5 r = mp5_face(s[0], s[1], s[2], s[3], s[4]);
#pragma unroll
  for (int k = 0; k < 5; ++k) ab[k] = xb != 0.0 ? xb * r.c[k] : 0.0;
}

// Both face values of a cell from its five-cell stencil: lo at its lower face (the right state there), hi at
// its upper one (the left state there).  hi is recon_right_face of the stencil, lo of its mirror image; the
// two share their slopes (MINMOD, PPM), smoothness indicators and ratios (WENO-Z) and curvatures (MP5).
template <int kind>
DEV void recon_cell(const double a[5], double eps, double q, double& lo, double& hi) {
  if constexpr (kind == ASTERX_RECON_MINMOD) {
    const double h = 0.5 * mm(a[2] - a[1], a[3] - a[2]);
    lo = a[2] - h;
    hi = a[2] + h;
  } else if constexpr (kind == ASTERX_RECON_PPM) {
    const double s1 = mc_slope(a[0], a[1], a[2]), s2 = mc_slope(a[1], a[2], a[3]), s3 = mc_slope(a[2], a[3], a[4]);
    const double sixth = 1.0 / 6.0;
    lo = 0.5 * (a[1] + a[2]) - (s2 - s1) * sixth;
    hi = 0.5 * (a[2] + a[3]) - (s3 - s2) * sixth;
    ppm_limit(a[2], lo, hi);
  } else if constexpr (kind == ASTERX_RECON_WENOZ) {
    wenoz_cell(a[0], a[1], a[2], a[3], a[4], eps, q, lo, hi);
  } else {
    mp5_cell(a[0], a[1], a[2], a[3], a[4], lo, hi);
  }
}

// ---------------------------------------------------------------------------------------
// Face fluxes along D.  Face (i,j,k), index along D in [0, n_D], transverse in [-1, n-1]
// (the extra layer feeds the edge averages of the electric field); UCT: transverse in [-3, n+1]
// (the upwind edge field reconstructs face values three faces beyond each edge), and the upwind
// transverse velocities (slots 5, 6 in place of the induction fluxes) and the two speeds are stored too.
struct FaceArgs {
  const double* metric;
  const double* prim;
  const double* A;
  const double* bc;
  double* flux;
  double* red;
  double gam, weno_eps, weno_q, gfac;
  int recon, speeds, riemann;
  double* apm;  // UCT: a_+, a_- and the normal field per direction
  // face metric per direction, components 0..6 from fma, 7..9 from fmb; NULL: gathered from the vertices
  const double* fma[3];
  const double* fmb[3];
  int rows[3];  // faces per march along y and z
  bool xown;    // the x faces' stored metric covers the owned rows only
};

// One lane per face.  A cell's parabola gives the right state at its lower face and the left state at its
// upper one, so each cell is reconstructed once: x faces with the lanes of a wavefront along x, the left
// state taken from the lane below (63 faces per wavefront); y and z faces in wavefronts that march along
// their direction.  Transverse positions are numbered through the whole plane (x faces: the whole block), so
// rows of any length leave no lanes idle.  The face metric is read as stored.  Against two lanes per face
// (one per side, each with its own reconstruction, geometry and flux combination): half the
// reconstructions, inverse metrics and exchanges (128^3, PPM, with the metric read as stored: x, y, z faces 0.214,
// 0.241, 0.247 -> 0.150, 0.180, 0.198 ms; WENO-Z 0.260, 0.314, 0.308 -> 0.177, 0.218, 0.217).  Bound by FP64 issue:
// about 1850 vector instructions per face, 0.1 ms of each direction at 128^3.  More wavefronts per SIMD spill, and a
// workgroup sharing windows through LDS waits at its barriers longer than it saves (both measured slower).
template <int D>
DEV void cell_faces_load(const GD& g, const FaceArgs& fa, int v, int id, double s[5]) {
  constexpr int t1 = (D + 1) % 3, t2 = (D + 2) % 3;
  const int sD = D == 0 ? 1 : (D == 1 ? g.sy : g.sz);
  const double* f = v < 5 ? fa.prim + (size_t)v * g.N : fa.bc + (size_t)(v == 5 ? t1 : t2) * g.N;
#pragma unroll
  for (int q = 0; q < 5; ++q) s[q] = ldu(f, id + (q - 2) * sD);
}

// The seven reconstructed variables of cell id at its two D faces: at the lower face into registers, at the
// upper one into this lane's column of hi (LDS; the left state of the face above).
typedef double FaceVals[7][64];
template <int D, int RECON>
DEV void cell_faces(const GD& g, const FaceArgs& fa, int id, double lo[7], FaceVals& Lhi, FaceVals& Llo) {
  const int l = __lane_id();
  if constexpr (RECON != ASTERX_RECON_MINMOD) {
    // one variable at a time (those of seven interleaved would not fit the registers), the next two variables'
    // stencils loading meanwhile
    double n1[5], n2[5];
    cell_faces_load<D>(g, fa, 0, id, n1);
    cell_faces_load<D>(g, fa, 1, id, n2);
#pragma unroll 1
    for (int v = 0; v < 7; ++v) {
      double s[5], x, y;
#pragma unroll
      for (int q = 0; q < 5; ++q) {
        s[q] = n1[q];
        n1[q] = n2[q];
      }
      if (v < 5) cell_faces_load<D>(g, fa, v + 2, id, n2);
      recon_cell<RECON>(s, fa.weno_eps, fa.weno_q, x, y);
      Llo[v][l] = x;
      Lhi[v][l] = y;
    }
#pragma unroll
    for (int v = 0; v < 7; ++v) lo[v] = Llo[v][l];
  } else {
    // all 35 stencil values are loaded before the first reconstruction
    double s[7][5];
#pragma unroll
    for (int v = 0; v < 7; ++v) cell_faces_load<D>(g, fa, v, id, s[v]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int v = 0; v < 7; ++v) {
      double y;
      recon_cell<RECON>(s[v], fa.weno_eps, fa.weno_q, lo[v], y);
      Lhi[v][l] = y;
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  wave_lds_sync();
}

// State, fluxes and speeds of one side; an unphysical reconstructed state falls back to the values of the
// side's own cell, read again (rare) rather than kept in registers.
template <int D>
DEV void face_side(const GD& g, const FaceArgs& fa, const Geo& G, double Bn, int own, double X[7], double U[7],
                   double F[7], double& cm, double& cp) {
  constexpr int t1 = (D + 1) % 3, t2 = (D + 2) % 3;
  double Bt[3];
  Bt[D] = Bn;
  Bt[t1] = X[5];
  Bt[t2] = X[6];
  State S;
  state_make(G, X, Bt, fa.gam, S, fa.gfac);
  if (!(X[0] > 0.0) || !(X[1] > 0.0) || !(S.iW2 > 0.0)) {
#pragma unroll
    for (int q = 0; q < 7; ++q) X[q] = ldu(q < 5 ? fa.prim + (size_t)q * g.N : fa.bc + (size_t)(q == 5 ? t1 : t2) * g.N, own);
    Bt[t1] = X[5];
    Bt[t2] = X[6];
    state_make(G, X, Bt, fa.gam, S, fa.gfac);
  }
  flux_of<D>(G, S, U, F);
  speeds_of<D>(G, S, fa.gam, fa.speeds, cm, cp);
}

// What a face reads besides its cells' values: its metric and the normal field from the potential around it.
// x faces load it before the reconstruction, so that it arrives meanwhile (152 -> 148 us at 128^3; y and z
// faces, whose marches hold more registers, measured slower so).
struct FaceIn {
  double m[10], Bn;
};
// Without stored metric: gathered from the 16 vertices around the face, in geom_wave's order of passes (the lower
// axis first), so that both give the same bits and blocks may choose by size.
// NQ components are gathered together.
template <int D, int NQ>
DEV void face_load(const GD& g, const FaceArgs& fa, int id, FaceIn& f, bool stored = true) {
  if (fa.fma[D] && stored) {
#pragma unroll
    for (int q = 0; q < 10; ++q) f.m[q] = ldu(q < 7 ? fa.fma[D] + (size_t)q * g.N : fa.fmb[D] + (size_t)(q - 7) * g.N, id);
  } else {
    const int s1 = D == 0 ? g.sy : 1, s2 = D == 2 ? g.sy : g.sz;
#pragma unroll NQ
    for (int q = 0; q < 10; ++q) {
      const double* p = fa.metric + (size_t)q * g.N + (id - s1 - s2);
      double r[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double* row = p + k * s2;
        r[k] = lag(row[0], row[s1], row[2 * s1], row[3 * s1]);
      }
      const double v = lag(r[0], r[1], r[2], r[3]);
#pragma unroll
      for (int k = 0; k < 10; ++k) f.m[k] = k == q ? v : f.m[k];
    }
  }
  const double* Ax = fa.A;
  const double* Ay = fa.A + g.N;
  const double* Az = fa.A + 2 * g.N;
  f.Bn = D == 0 ? faceBx(Ay, Az, id, g.sy, g.sz, g)
                : (D == 1 ? faceBy(Ax, Az, id, g.sy, g.sz, g) : faceBz(Ax, Ay, id, g.sy, g.sz, g));
}

// The face between the cells of states XL (below) and XR (above), stored at point id; returns the larger speed.
template <int D, bool UCT>
DEV double face_solve(const GD& g, const FaceArgs& fa, int id, const FaceIn& in, double XL[7], double XR[7]) {
  constexpr int t1 = (D + 1) % 3, t2 = (D + 2) % 3;
  const int st[3] = {1, g.sy, g.sz};
  const double Bn = in.Bn;
  Geo G;
  geo_from(in.m, G);
  double UL[7], FL[7], UR[7], FR[7], cmL, cpL, cmR, cpR;
  face_side<D>(g, fa, G, Bn, id - st[D], XL, UL, FL, cmL, cpL);
  __builtin_amdgcn_sched_barrier(0);
  face_side<D>(g, fa, G, Bn, id, XR, UR, FR, cmR, cpR);
  const double cmax = fmax(0.0, fmax(cpL, cpR)), cmin = -fmin(0.0, fmin(cmL, cmR));
  const double den = cmax + cmin;
  // HLLE (eq. HLLEfluxes): (cmin F_R + cmax F_L - cmax cmin (U_R - U_L)) / (cmax + cmin); LxF (eq. LxFfluxes):
  // (F_R + F_L - c_wave (U_R - U_L)) / 2, c_wave = max(cmax, cmin)
  double wl = 0.5, wr = 0.5, wu = 0.0;
  if (fa.riemann == ASTERX_RIEMANN_LXF) {
    wu = 0.5 * fmax(cmax, cmin);
  } else if (den > 0.0) {
    const double r = recip(den);
    wl = cmax * r;
    wr = cmin * r;
    wu = cmax * cmin * r;
  }
  double* out = fa.flux + (size_t)(D * 7) * g.N;
#pragma unroll
  for (int q = 0; q < (UCT ? 5 : 7); ++q) out[(size_t)q * g.N + id] = wl * FL[q] + wr * FR[q] + wu * (UL[q] - UR[q]);
  if constexpr (UCT) {
    // upwind transverse velocities (eq. uct1) with a_+ = cmax, a_- = cmin (eq. uct2)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int t = k ? t2 : t1;
      const double vl = G.alp * XL[2 + t] - G.beta[t], vr = G.alp * XR[2 + t] - G.beta[t];
      out[(size_t)(5 + k) * g.N + id] = den > 0.0 ? (cmax * vl + cmin * vr) / den : 0.5 * (vl + vr);
    }
    fa.apm[(size_t)(D * 3) * g.N + id] = cmax;
    fa.apm[(size_t)(D * 3 + 1) * g.N + id] = cmin;
    fa.apm[(size_t)(D * 3 + 2) * g.N + id] = Bn;
  }
  return fmax(cmax, cmin);
}

// Wavefront items.  x faces: 63 consecutive faces of the sequence of cells -1..n0 of every row.  y and z
// faces: 64 transverse columns times a march of `rows` faces, the marches of a column group one after another
// (the rows that two of them read are then in one XCD's L2).
__host__ __device__ inline unsigned face_items(const int n[3], int D, int lo, int rows) {
  int e[3];
  for (int a = 0; a < 3; ++a) e[a] = n[a] + 2 * lo - 1;
  if (D == 0) return (unsigned)(((long long)(n[0] + 2) * e[1] * e[2] - 1 + 62) / 63);
  const long long cols = (long long)e[0] * e[D == 1 ? 2 : 1];
  return (unsigned)((cols + 63) / 64 * ((n[D] + rows) / rows));
}
// Faces per march.  A march of r faces costs r + 1 reconstructions and r solutions (which cost about the same),
// and its five-row windows have to stay in L2 with those of all marches in flight: at most three, MINMOD, whose
// reconstruction is the shortest, two (RK4 steps, marches of at most 1, 2, 3, 4: 128^3, PPM, 5.21, 5.02, 4.98,
// 5.03 ms; 96^3, WENO-Z, 2.50, 2.39, 2.38, 2.38; 80^3, MINMOD, 1.281, 1.284, 1.295, 1.297).  Blocks whose marches
// fill the chip's wavefront slots only a few times take the length whose rounds cost least (97 x 61 x 45, MP5,
// upwind CT: single faces 1.112 ms, by the rule 1.058).
template <int R>
constexpr int face_march() { return R == ASTERX_RECON_MINMOD ? 2 : 3; }
constexpr unsigned FACE_SLOTS = 256 * 4 * 3;  // 256 CUs of four SIMDs, three wavefronts each
// Batches: two, or one where all patches' single faces fit the slots at once (Heun steps, MP5: four patches of 16^3 305
// and 272 us; two of 64^3, three rounds of single faces, 1196 and 1275).
constexpr int FACE_BATCH_ROWS = 2;
inline int face_rows(const int n[3], int D, int lo, int march) {
  int best = 1;
  unsigned least = ~0u;
  for (int r = 1; r <= march; ++r) {
    const unsigned cost = (face_items(n, D, lo, r) + FACE_SLOTS - 1) / FACE_SLOTS * (unsigned)(2 * r + 1);
    if (cost <= least) {
      least = cost;
      best = r;
    }
  }
  return best;
}

// Faces with owned transverse indices report their speed.
template <int D>
DEV bool face_owned(const GD& g, const int c[3]) {
  constexpr int t1 = (D + 1) % 3, t2 = (D + 2) % 3;
  return (unsigned)c[t1] < (unsigned)g.n[t1] && (unsigned)c[t2] < (unsigned)g.n[t2];
}
DEV void face_report(const FaceArgs& fa, double smax) {
  if (!fa.red) return;
  const double w = wave_max(smax);
  if (__lane_id() == 0) atomic_max_pos(fa.red, w);
}

struct FaceLDS {
  FaceVals hi, lo;
};
template <int RECON, bool UCT, int NQ>
DEV void face_wave_x(const GD& g, const FaceArgs& fa, unsigned item, FaceLDS& L) {
  constexpr int lo = UCT ? 3 : 1;
  const unsigned e1 = g.n[1] + 2 * lo - 1, e2 = g.n[2] + 2 * lo - 1;
  const unsigned rl = (unsigned)g.n[0] + 2, total = rl * e1 * e2;
  const unsigned q = min(item * 63 + __lane_id(), total - 1);
  const unsigned row = q / rl;
  const int c[3] = {(int)(q % rl) - 1, (int)(row % e1) - lo, (int)(row / e1) - lo};
  const int id = at(g, c[0], c[1], c[2]);
  double XL[7], XR[7], smax = 0.0;
  FaceIn fin;
  face_load<0, NQ>(g, fa, id, fin, !fa.xown || (c[1] >= 0 && c[2] >= 0));
  cell_faces<0, RECON>(g, fa, id, XR, L.hi, L.lo);
  wave_lds_sync();
  if (__lane_id() > 0 && item * 63 + __lane_id() < total && c[0] >= 0) {
#pragma unroll
    for (int v = 0; v < 7; ++v) XL[v] = L.hi[v][__lane_id() - 1];
    const double s = face_solve<0, UCT>(g, fa, id, fin, XL, XR);
    if (face_owned<0>(g, c)) smax = s;
  }
  face_report(fa, smax);
}

template <int D, int RECON, bool UCT, int NQ>
DEV void face_wave_yz(const GD& g, const FaceArgs& fa, unsigned item, FaceLDS& L) {
  constexpr int lo = UCT ? 3 : 1, E = D == 1 ? 2 : 1;
  const int rows = fa.rows[D], l = __lane_id();
  const unsigned nch = (unsigned)(g.n[D] + rows) / rows, ch = item % nch;
  const unsigned e0 = g.n[0] + 2 * lo - 1, eE = g.n[E] + 2 * lo - 1;
  const unsigned q = min((item / nch) * 64 + l, e0 * eE - 1);
  const bool in = (item / nch) * 64 + l < e0 * eE;
  const int j0 = (int)ch * rows, j1 = min(j0 + rows, g.n[D] + 1);
  int c[3];
  c[0] = (int)(q % e0) - lo;
  c[E] = (int)(q / e0) - lo;
  c[D] = j0 - 1;
  const int sD = D == 1 ? g.sy : g.sz;
  int id = at(g, c[0], c[1], c[2]);
  double smax = 0.0;
  // from the cell below the first face, whose own lower face is left out: one copy of the reconstruction's
  // code, so that a face's result does not depend on where its march begins
#pragma unroll 1
  for (int j = j0 - 1; j < j1; ++j, id += sD) {
    double XL[7], XR[7];
#pragma unroll
    for (int v = 0; v < 7; ++v) XL[v] = L.hi[v][l];
    wave_lds_sync();
    cell_faces<D, RECON>(g, fa, id, XR, L.hi, L.lo);
    wave_lds_sync();
    if (j >= j0 && in) {
      FaceIn fin;
      face_load<D, NQ>(g, fa, id, fin);
      smax = fmax(smax, face_solve<D, UCT>(g, fa, id, fin, XL, XR));
    }
  }
  face_report(fa, face_owned<D>(g, c) ? smax : 0.0);
}

// Swap of a lane pair's values (lanes 2f and 2f + 1, one per side of a face in the adjoint): a DPP quad
// permutation (1, 0, 3, 2) of the two 32-bit halves, a VALU move; both lanes of a pair are always active
// together.
DEV double shfl1(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, 0xB1, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0xB1, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// ---------------------------------------------------------------------------------------
// Cells: flux divergence (eq. fluxconseqs) + geometric sources (eq. grmhdsrc) + div B.
// Runge-Kutta stage outputs written in place of the right-hand side: per owned point,
// out = b_dt rhs + sum_m a[m] u[m], with the products and sums in the order of the
// stage-combine kernel (so the two paths agree bit for bit).
struct RKOut {
  const double* u[2];
  double a[2];
  double b_dt;
  double* out;
  int nterms;
};
struct Combine {
  RKOut o[2];
  int nout;  // 0: the right-hand side itself is stored
};

template <int MAXT>
DEV double rk_point(double b_dt, double r, const double* const* u, const double* a, int nterms, size_t o) {
  double s = b_dt * r;
#pragma unroll
  for (int m = 0; m < MAXT; ++m)
    if (m < nterms) s = fma(a[m], u[m][o], s);
  return s;
}

DEV void emit(const Combine& cb, double* rhs, size_t o, double v) {
  if (cb.nout == 0) {
    rhs[o] = v;
    return;
  }
#pragma unroll
  for (int k = 0; k < 2; ++k)
    if (k < cb.nout) cb.o[k].out[o] = rk_point<2>(cb.o[k].b_dt, v, cb.o[k].u, cb.o[k].a, cb.o[k].nterms, o);
}

struct CellArgs {
  const double* metric;
  const double* curv;
  const double* prim;
  const double* A;
  const double* bc;
  const double* flux;
  double* rhs;
  double* red;
  double gam;
  Combine cmb;
};

// Tiled cell kernel.  Pass 1 interpolates the values of the 10 metric and 6 curvature
// components through LDS; the stress tensor follows.  The momentum source
// 1/2 T^{mu nu} d_j g_{mu nu} is linear in the derivatives of the stored components,
// sum_c w_c d_j m_c with weights w_c built from T, beta and gamma, so pass 2 takes one
// component's three derivatives at a time and accumulates them (few live registers).
DEV void cell_body(const GD& g, const CellArgs& ca, TileLDS& S, unsigned tile) {
  const TileCell t = tile_cell(g, tile);
  const TileIdx x = tile_index(g, t);
  double m[10], K[6], pre[NFETCH];
  value_rounds16(g, ca.metric, ca.curv, x, m, K, pre, *reinterpret_cast<TileLDS2*>(&S));
  const int id = t.valid ? at(g, t.i0 + t.cx, t.j0 + t.cy, t.k0 + t.cz) : 0;
  SrcW sw;
  sw.as = 0.0;
  double src[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (t.valid) {
    Geo G;
    geo_from(m, G);
    double pr[5], Bt[3];
#pragma unroll
    for (int c = 0; c < 5; ++c) pr[c] = ca.prim[c * g.N + id];
    Bt[0] = ca.bc[id];
    Bt[1] = ca.bc[g.N + id];
    Bt[2] = ca.bc[2 * g.N + id];
    src_weights(G, pr, Bt, ca.gam, sw);
    src[4] = src_curv(sw, K);
  }
  src_deriv_rounds(g, ca.metric, x, t.valid, pre, sw, src, *reinterpret_cast<TileLDS2D*>(&S));
  double divb = 0.0;
  if (t.valid) {
    const int st[3] = {1, g.sy, g.sz};
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      double sdiv = 0.0;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const double* F = ca.flux + (size_t)(d * 7 + c) * g.N;
        sdiv += (ldu(F, id + st[d]) - ldu(F, id)) * g.idx[d];
      }
      // the densitized source rounded on its own, as the recovery kernel with sources stores it
      emit(ca.cmb, ca.rhs, (size_t)c * g.N + id, __dmul_rn(sw.as, src[c]) - sdiv);
    }
    if (ca.red) {
      const double* Ax = ca.A;
      const double* Ay = ca.A + g.N;
      const double* Az = ca.A + 2 * g.N;
      double dB = (faceBx(Ay, Az, id + 1, g.sy, g.sz, g) - faceBx(Ay, Az, id, g.sy, g.sz, g)) * g.idx[0] +
                  (faceBy(Ax, Az, id + g.sy, g.sy, g.sz, g) - faceBy(Ax, Az, id, g.sy, g.sz, g)) * g.idx[1] +
                  (faceBz(Ax, Ay, id + g.sz, g.sy, g.sz, g) - faceBz(Ax, Ay, id, g.sy, g.sz, g)) * g.idx[2];
      divb = fabs(dB);
    }
  }
  if (ca.red) {
    double wm = wave_max(divb);
    if (__lane_id() == 0) atomic_max_pos(ca.red + 1, wm);
  }
}

// ---------------------------------------------------------------------------------------
// Cells with their sources given (stored by the recovery kernel with sources): flux divergence
// (eq. fluxconseqs) plus the densitized source, div B, and the stage outputs, with the cell
// kernel's arithmetic (bitwise the same results).  One thread per owned cell, x fastest, no LDS:
// a streaming kernel over the fluxes, sources and stage states.
struct DivArgs {
  const double* src;  // [4] alpha sqrt(gamma) times the S_x, S_y, S_z, tau sources
  const double* flux;
  const double* A;
  double* rhs;
  double* red;
  Combine cmb;
};

DEV void div_body(const GD& g, const DivArgs& da, unsigned tile) {
  int i, j, k;
  const bool in = box_at<64, 4>(g.n, tile, threadIdx.x, i, j, k);
  double divb = 0.0;
  if (in) {
    const int id = at(g, i, j, k);
    const int st[3] = {1, g.sy, g.sz};
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      double sdiv = 0.0;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const double* F = da.flux + (size_t)(d * 7 + c) * g.N;
        sdiv += (ldu(F, id + st[d]) - ldu(F, id)) * g.idx[d];
      }
      const double sc = c ? ldu(da.src + (size_t)(c - 1) * g.N, id) : 0.0;
      emit(da.cmb, da.rhs, (size_t)c * g.N + id, sc - sdiv);
    }
    if (da.red) {
      const double* Ax = da.A;
      const double* Ay = da.A + g.N;
      const double* Az = da.A + 2 * g.N;
      double dB = (faceBx(Ay, Az, id + 1, g.sy, g.sz, g) - faceBx(Ay, Az, id, g.sy, g.sz, g)) * g.idx[0] +
                  (faceBy(Ax, Az, id + g.sy, g.sy, g.sz, g) - faceBy(Ax, Az, id, g.sy, g.sz, g)) * g.idx[1] +
                  (faceBz(Ax, Ay, id + g.sz, g.sy, g.sz, g) - faceBz(Ax, Ay, id, g.sy, g.sz, g)) * g.idx[2];
      divb = fabs(dB);
    }
  }
  if (da.red) {
    double wm = wave_max(divb);
    if (__lane_id() == 0) atomic_max_pos(da.red + 1, wm);
  }
}

// ---------------------------------------------------------------------------------------
// Covariant stress-energy tensor at the vertices [0, n]^3 (Sec. 3.1: stored with the spacetime
// variables, for a spacetime solver): the vertex fluid state is the mean of the primitives and
// centre fields of the 8 cells sharing the vertex, the metric the vertex's own;
// T_{mu nu} = g_{mu a} g_{nu b} T^{ab}.  Output fields 00, 0x, 0y, 0z, xx, xy, xz, yy, yz, zz.
struct TmunuArgs {
  const double* metric;
  const double* prim;
  const double* A;
  double* out;
  double gam;
};

// Tiles of 16 x 4 x 4 vertices: the primitives and centre fields of the 17 x 5 x 5 cells they share are
// staged through LDS once (the centre field from the curl of A), then each vertex averages its 8 cells.
constexpr int TV_X = 16, TV_Y = 4, TV_Z = 4, TC_X = TV_X + 1, TC_Y = TV_Y + 1, TC_Z = TV_Z + 1;
constexpr int TC_N = TC_X * TC_Y * TC_Z;
struct TmunuLDS {
  double c[8][TC_N];
};

unsigned tmunu_tiles(const GD& g) {
  return (unsigned)(((g.n[0] + TV_X) / TV_X) * ((g.n[1] + TV_Y) / TV_Y) * ((g.n[2] + TV_Z) / TV_Z));
}

DEV void tmunu_body(const GD& g, const TmunuArgs& ta, unsigned tile, TmunuLDS& L) {
  const int nbx = (g.n[0] + TV_X) / TV_X, nby = (g.n[1] + TV_Y) / TV_Y;
  const int i0 = (int)(tile % nbx) * TV_X, j0 = (int)((tile / nbx) % nby) * TV_Y, k0 = (int)(tile / (nbx * nby)) * TV_Z;
  for (int q = threadIdx.x; q < TC_N; q += 256) {
    const int ci = i0 - 1 + q % TC_X, cj = j0 - 1 + (q / TC_X) % TC_Y, ck = k0 - 1 + q / (TC_X * TC_Y);
    // cells -1 .. n serve the vertices 0 .. n; cells beyond are not staged (no vertex reads them)
    if (ci <= g.n[0] && cj <= g.n[1] && ck <= g.n[2]) {
      const int c = at(g, ci, cj, ck);
#pragma unroll
      for (int v = 0; v < 5; ++v) L.c[v][q] = ta.prim[v * g.N + c];
      double b[3];
      centre_B(ta.A, g, c, b);
#pragma unroll
      for (int v = 0; v < 3; ++v) L.c[5 + v][q] = b[v];
    }
  }
  __syncthreads();
  const int vx = threadIdx.x % TV_X, vy = (threadIdx.x / TV_X) % TV_Y, vz = threadIdx.x / (TV_X * TV_Y);
  const int i = i0 + vx, j = j0 + vy, k = k0 + vz;
  if (i > g.n[0] || j > g.n[1] || k > g.n[2]) return;
  double pr[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, Bt[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int dk = -1; dk <= 0; ++dk)
#pragma unroll
    for (int dj = -1; dj <= 0; ++dj)
#pragma unroll
      for (int di = -1; di <= 0; ++di) {
        const int q = (vx + 1 + di) + TC_X * ((vy + 1 + dj) + TC_Y * (vz + 1 + dk));
#pragma unroll
        for (int v = 0; v < 5; ++v) pr[v] += L.c[v][q];
#pragma unroll
        for (int v = 0; v < 3; ++v) Bt[v] += L.c[5 + v][q];
      }
#pragma unroll
  for (int q = 0; q < 5; ++q) pr[q] *= 0.125;
#pragma unroll
  for (int q = 0; q < 3; ++q) Bt[q] *= 0.125;
  const int id = at(g, i, j, k);
  double m[10];
#pragma unroll
  for (int q = 0; q < 10; ++q) m[q] = ta.metric[q * g.N + id];
  Geo G;
  geo_from(m, G);
  State St;
  state_make(G, pr, Bt, ta.gam, St);
  double T00, T0[3], Tk[6];
  tmunu_upper(G, St, T00, T0, Tk);
  double bl[3];
  lower(G.g, G.beta, bl);
  double g4[4][4], Tu[4][4];
  g4[0][0] = -G.alp * G.alp + bl[0] * G.beta[0] + bl[1] * G.beta[1] + bl[2] * G.beta[2];
  Tu[0][0] = T00;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    g4[0][a + 1] = g4[a + 1][0] = bl[a];
    Tu[0][a + 1] = Tu[a + 1][0] = T0[a];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      g4[a + 1][b + 1] = G.g[sym(a, b)];
      Tu[a + 1][b + 1] = Tk[sym(a, b)];
    }
  }
  double X[4][4];  // T^{a}_{nu}
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int n = 0; n < 4; ++n) X[a][n] = Tu[a][0] * g4[0][n] + Tu[a][1] * g4[1][n] + Tu[a][2] * g4[2][n] + Tu[a][3] * g4[3][n];
  const int mu[10] = {0, 0, 0, 0, 1, 1, 1, 2, 2, 3}, nu[10] = {0, 1, 2, 3, 1, 2, 3, 2, 3, 3};
#pragma unroll
  for (int c = 0; c < 10; ++c) {
    const int a = mu[c], b = nu[c];
    ta.out[(size_t)c * g.N + id] = g4[a][0] * X[0][b] + g4[a][1] * X[1][b] + g4[a][2] * X[2][b] + g4[a][3] * X[3][b];
  }
}

// ---------------------------------------------------------------------------------------
// Factor-2 inter-level operators (refinement boundaries, Sec. 3.9 and the AMR tests of Sec. 4).  The
// fine grid's vertex 0 sits on coarse vertex c0; each axis of a field is cell- (stag 0) or
// vertex-centred (stag 1).  Prolongation per axis: vertex directions inject on coincident points
// and take (-1, 9, 9, -1)/16 at midpoints; cell directions give the children of coarse cell c the
// conservative quadratic values u_c -+ (u_{c+1} - u_{c-1})/8; tensor product.  Cell fields fall
// back per coarse cell to minmod-limited linear children when a third-order child leaves the
// [min, max] of the 27 coarse cells around it.  Restriction: children's mean along cell
// directions, injection along vertex directions.
struct InterArgs {
  GD gc, gf;
  int c0[3], stag[3], lo[3], hi[3];
  int nf;
  const double* src;
  double* dst;
};

DEV int fdiv2(int f) { return f >= 0 ? f / 2 : -((1 - f) / 2); }

// The two children along x of one coarse point, at fine point (f0, f1, f2), f0 even: one 16-byte store (rows start
// at any 8-byte address; against single children's, 16 bytes apart: 11.6 and 12.5 us), or the one in the box.
typedef double pair8 __attribute__((ext_vector_type(2), aligned(8)));
DEV void store_children(const InterArgs& a, double* o, int f0, int f1, int f2, double c0, double c1) {
  if (f1 < a.lo[1] || f1 > a.hi[1] || f2 < a.lo[2] || f2 > a.hi[2]) return;
  double* p = o + at(a.gf, f0, f1, f2);
  if (f0 >= a.lo[0] && f0 < a.hi[0]) {
    *(pair8*)p = pair8{c0, c1};
  } else if (f0 >= a.lo[0] && f0 <= a.hi[0]) {
    p[0] = c0;
  } else if (f0 + 1 >= a.lo[0] && f0 < a.hi[0]) {
    p[1] = c1;
  }
}

// Both children of a coarse point along one axis from its 1-D stencil u (cell: c-1, c, c+1; vertex: c-1 .. c+2,
// the first child on the point itself).
template <bool VERTEX>
DEV void children(const double* u, double& c0, double& c1) {
  if constexpr (VERTEX) {
    c0 = u[1];
    c1 = (9.0 * (u[1] + u[2]) - (u[0] + u[3])) * (1.0 / 16.0);
  } else {
    const double h = (u[2] - u[0]) * 0.125;
    c0 = u[1] - h;
    c1 = u[1] + h;
  }
}

// Fields vertex-centred along at least one axis (bits of STAG): one thread per coarse point, its eight children by
// passes along x, y and z, the children inside the fine box stored.  The stencils reach from c - 1 to c + 2 at most,
// also where a box ends on a first child (the reach that is checked on the host).  Eight children share 36 to 64
// loads; one thread per child with run-time stencils took up to 64 for each (134^3 points: 50 us per field, now 12).
template <int STAG>
DEV void prolong_body(const InterArgs& a, unsigned tile) {
  constexpr bool VX = STAG & 1, VY = STAG & 2, VZ = STAG & 4;
  constexpr int NX = VX ? 4 : 3, NY = VY ? 4 : 3, NZ = VZ ? 4 : 3;
  int pl[3], e[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    pl[d] = a.c0[d] + fdiv2(a.lo[d]);
    e[d] = a.c0[d] + fdiv2(a.hi[d]) - pl[d] + 1;
  }
  int i, j, k;
  if (!lin_at(e, tile, threadIdx.x, i, j, k)) return;
  const int cc[3] = {pl[0] + i, pl[1] + j, pl[2] + k};
  const int id = at(a.gc, cc[0] - 1, cc[1] - 1, cc[2] - 1);
  const int f[3] = {2 * (cc[0] - a.c0[0]), 2 * (cc[1] - a.c0[1]), 2 * (cc[2] - a.c0[2])};
  for (int q = 0; q < a.nf; ++q) {
    const double* c = a.src + (size_t)q * a.gc.N;
    double z[4][NZ];  // x and y children, planes
#pragma unroll
    for (int r = 0; r < NZ; ++r) {
      double y[2][NY];
#pragma unroll
      for (int p = 0; p < NY; ++p) {
        double u[NX];
#pragma unroll
        for (int m = 0; m < NX; ++m) u[m] = c[id + m + p * a.gc.sy + r * a.gc.sz];
        children<VX>(u, y[0][p], y[1][p]);
      }
      children<VY>(y[0], z[0][r], z[2][r]);
      children<VY>(y[1], z[1][r], z[3][r]);
    }
    double* o = a.dst + (size_t)q * a.gf.N;
#pragma unroll
    for (int h = 0; h < 4; h += 2) {
      double l[2], r[2];
      children<VZ>(z[h], l[0], l[1]);
      children<VZ>(z[h + 1], r[0], r[1]);
#pragma unroll
      for (int m = 0; m < 2; ++m) store_children(a, o, f[0], f[1] + (h >> 1), f[2] + m, l[m], r[m]);
    }
  }
}

// Cell fields: one thread per coarse parent of the fine box; the 27 parent-centred values, the fallback
// decision and all 8 children computed once, the children inside the box stored (134^3 points, five fields: 40 us,
// 2.4 TB/s of stores; the children by axis passes as above would take 37 us, but round a child that lies on the
// extremes differently, and with it the fallback).
DEV void prolong_cells_body(const InterArgs& a, unsigned tile, int q) {
  int pl[3], e[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    pl[d] = a.c0[d] + fdiv2(a.lo[d]);
    e[d] = a.c0[d] + fdiv2(a.hi[d]) - pl[d] + 1;
  }
  int i, j, k;
  if (!lin_at(e, tile, threadIdx.x, i, j, k)) return;
  const int cc[3] = {pl[0] + i, pl[1] + j, pl[2] + k};
  const size_t Nc = a.gc.N, Nf = a.gf.N;
  const double* c = a.src + (size_t)q * Nc;
  double u[27];
#pragma unroll
  for (int r = 0; r < 27; ++r) u[r] = c[at(a.gc, cc[0] - 1 + r % 3, cc[1] - 1 + (r / 3) % 3, cc[2] - 1 + r / 9)];
  double mn = u[13], mx = u[13];
#pragma unroll
  for (int r = 0; r < 27; ++r) {
    mn = fmin(mn, u[r]);
    mx = fmax(mx, u[r]);
  }
  double ch[8];
  bool fall = false;
#pragma unroll
  for (int h = 0; h < 8; ++h) {
    const int cx = h & 1, cy = (h >> 1) & 1, cz = h >> 2;
    const double wx[3] = {cx ? -0.125 : 0.125, 1.0, cx ? 0.125 : -0.125};
    const double wy[3] = {cy ? -0.125 : 0.125, 1.0, cy ? 0.125 : -0.125};
    const double wz[3] = {cz ? -0.125 : 0.125, 1.0, cz ? 0.125 : -0.125};
    double sum = 0.0;
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int p2 = 0; p2 < 3; ++p2)
#pragma unroll
        for (int p1 = 0; p1 < 3; ++p1) sum += wx[p1] * wy[p2] * wz[r] * u[p1 + 3 * p2 + 9 * r];
    ch[h] = sum;
    fall = fall || sum < mn || sum > mx;
  }
  if (fall) {
    const double uc = u[13];
    const double sx = mm(u[14] - uc, uc - u[12]), sy = mm(u[16] - uc, uc - u[10]), sz = mm(u[22] - uc, uc - u[4]);
#pragma unroll
    for (int h = 0; h < 8; ++h)
      ch[h] = uc + ((h & 1) ? 0.25 : -0.25) * sx + (((h >> 1) & 1) ? 0.25 : -0.25) * sy + ((h >> 2) ? 0.25 : -0.25) * sz;
  }
  double* o = a.dst + (size_t)q * Nf;
#pragma unroll
  for (int h = 0; h < 8; h += 2)
    store_children(a, o, 2 * (cc[0] - a.c0[0]), 2 * (cc[1] - a.c0[1]) + ((h >> 1) & 1), 2 * (cc[2] - a.c0[2]) + (h >> 2),
                   ch[h], ch[h + 1]);
}

DEV void restrict_body(const InterArgs& a, unsigned tile) {
  const int e[3] = {a.hi[0] - a.lo[0] + 1, a.hi[1] - a.lo[1] + 1, a.hi[2] - a.lo[2] + 1};
  int i, j, k;
  if (!lin_at(e, tile, threadIdx.x, i, j, k)) return;
  const int c[3] = {a.lo[0] + i, a.lo[1] + j, a.lo[2] + k};
  int n[3], b[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    b[d] = 2 * (c[d] - a.c0[d]);
    n[d] = a.stag[d] ? 1 : 2;
  }
  const double inv = 1.0 / (double)(n[0] * n[1] * n[2]);
  for (int q = 0; q < a.nf; ++q) {
    const double* f = a.src + (size_t)q * a.gf.N;
    double s = 0.0;
    for (int r = 0; r < n[2]; ++r)
      for (int p2 = 0; p2 < n[1]; ++p2)
        for (int p1 = 0; p1 < n[0]; ++p1) s += f[at(a.gf, b[0] + p1, b[1] + p2, b[2] + r)];
    a.dst[(size_t)q * a.gc.N + at(a.gc, c[0], c[1], c[2])] = s * inv;
  }
}

// ---------------------------------------------------------------------------------------
// Vertices in [-1, n]^3: G_A = alpha Psi / sqrt(gamma) - beta^j A_j and
// F_Psi^j = alpha sqrt(gamma) gamma^jk A_k - beta^j Psi, with A averaged to the vertex
// along its own direction (Sec. 3.4).
struct VertexArgs {
  const double* metric;
  const double* A;
  const double* psi;
  double* ga;
  double* fp;
};

DEV void vertex_body(const GD& g, const VertexArgs& va, unsigned tile) {
  const double* __restrict__ metric = va.metric;
  const double* __restrict__ A = va.A;
  const double* __restrict__ psi = va.psi;
  double* __restrict__ ga = va.ga;
  double* __restrict__ fp = va.fp;
  int e[3] = {g.n[0] + 2, g.n[1] + 2, g.n[2] + 2};
  int a, b, c;
  if (!lin_at(e, tile, threadIdx.x, a, b, c)) return;
  const int id = at(g, a - 1, b - 1, c - 1);
  double m[10];
#pragma unroll
  for (int q = 0; q < 10; ++q) m[q] = metric[q * g.N + id];
  Geo G;
  geo_from(m, G);
  double Av[3];
  Av[0] = 0.5 * (A[id - 1] + A[id]);
  Av[1] = 0.5 * (A[g.N + id - g.sy] + A[g.N + id]);
  Av[2] = 0.5 * (A[2 * g.N + id - g.sz] + A[2 * g.N + id]);
  double ps = psi[id];
  ga[id] = G.alp * ps / G.sqrtg - (G.beta[0] * Av[0] + G.beta[1] * Av[1] + G.beta[2] * Av[2]);
  double as = G.alp * G.sqrtg;
  fp[id] = as * (G.gu[0] * Av[0] + G.gu[1] * Av[1] + G.gu[2] * Av[2]) - G.beta[0] * ps;
  fp[g.N + id] = as * (G.gu[1] * Av[0] + G.gu[3] * Av[1] + G.gu[4] * Av[2]) - G.beta[1] * ps;
  fp[2 * g.N + id] = as * (G.gu[2] * Av[0] + G.gu[4] * Av[1] + G.gu[5] * Av[2]) - G.beta[2] * ps;
}

// Owned edges and vertices: E by flux-CT (average of the four face induction fluxes around
// each edge; E = -vt x Btilde), dA/dt = -E - grad G_A, dPsi/dt = -div F_Psi - xi alpha Psi.
struct EdgeArgs {
  const double* metric;
  const double* psi;
  const double* flux;
  const double* ga;
  const double* fp;
  double* rhs;
  double xi;
  int gauge;
  Combine cmb;
  const double* apm;  // UCT: a_+, a_- and the normal field per face direction (stored by the face kernel)
};

// One term of the upwind edge field (Sec. 3.4, eq. eq3.20) at the edge owned by point id: the 1-D
// Riemann problem along DIR, from the FD-faces in the row through the edge along DIR (their upwind
// velocity component DIR and normal field, both stored by the UCT face kernel, PPM-reconstructed to
// the edge from below (L) and above (R)), with the larger speeds of the two DIR-faces meeting at the
// edge (offset along SDIR).
template <int DIR, int FD, int SDIR>
DEV double uct_term(const GD& g, const EdgeArgs& ea, int id) {
  const int st[3] = {1, g.sy, g.sz};
  const int sd = st[DIR];
  constexpr int slot = DIR == (FD + 1) % 3 ? 5 : 6;
  const double* vb = ea.flux + (size_t)(FD * 7 + slot) * g.N;
  const double* bn = ea.apm + (size_t)(FD * 3 + 2) * g.N;
  double v6[6], b6[6];
#pragma unroll
  for (int s = 0; s < 6; ++s) {
    v6[s] = vb[id + (s - 3) * sd];
    b6[s] = bn[id + (s - 3) * sd];
  }
  const double vm[5] = {v6[5], v6[4], v6[3], v6[2], v6[1]}, bm[5] = {b6[5], b6[4], b6[3], b6[2], b6[1]};
  const double vl = recon_right_face<ASTERX_RECON_PPM>(v6, 0.0, 1.0), vr = recon_right_face<ASTERX_RECON_PPM>(vm, 0.0, 1.0);
  const double bl = recon_right_face<ASTERX_RECON_PPM>(b6, 0.0, 1.0), br = recon_right_face<ASTERX_RECON_PPM>(bm, 0.0, 1.0);
  const double* ap = ea.apm + (size_t)(DIR * 3) * g.N;
  const double* am = ea.apm + (size_t)(DIR * 3 + 1) * g.N;
  const int o = st[SDIR];
  const double a_p = fmax(ap[id], ap[id - o]), a_m = fmax(am[id], am[id - o]);
  const double den = a_p + a_m;
  if (!(den > 0.0)) return 0.5 * (vl * bl + vr * br);
  return (a_p * vl * bl + a_m * vr * br - a_p * a_m * (br - bl)) / den;
}

template <bool UCT = false>
DEV void edge_body(const GD& g, const EdgeArgs& ea, unsigned tile) {
  int i, j, k;
  if (!box_at<64, 4>(g.n, tile, threadIdx.x, i, j, k)) return;
  const int id = at(g, i, j, k);
  const int sy = g.sy, sz = g.sz;
  double Ex, Ey, Ez;
  if constexpr (UCT) {
    // E_c = -(term along c+1 from the (c+2)-faces) + (term along c+2 from the (c+1)-faces)
    Ex = -uct_term<1, 2, 2>(g, ea, id) + uct_term<2, 1, 1>(g, ea, id);
    Ey = -uct_term<2, 0, 0>(g, ea, id) + uct_term<0, 2, 2>(g, ea, id);
    Ez = -uct_term<0, 1, 1>(g, ea, id) + uct_term<1, 0, 0>(g, ea, id);
  } else {
    const double* Fx_By = ea.flux + (size_t)(0 * 7 + 5) * g.N;
    const double* Fx_Bz = ea.flux + (size_t)(0 * 7 + 6) * g.N;
    const double* Fy_Bz = ea.flux + (size_t)(1 * 7 + 5) * g.N;
    const double* Fy_Bx = ea.flux + (size_t)(1 * 7 + 6) * g.N;
    const double* Fz_Bx = ea.flux + (size_t)(2 * 7 + 5) * g.N;
    const double* Fz_By = ea.flux + (size_t)(2 * 7 + 6) * g.N;
    Ez = 0.25 * (-Fx_By[id] - Fx_By[id - sy] + Fy_Bx[id] + Fy_Bx[id - 1]);
    Ex = 0.25 * (-Fy_Bz[id] - Fy_Bz[id - sz] + Fz_By[id] + Fz_By[id - sy]);
    Ey = 0.25 * (-Fz_Bx[id] - Fz_Bx[id - 1] + Fx_Bz[id] + Fx_Bz[id - sz]);
  }
  double* r = ea.rhs;
  const size_t N = g.N;
  if (ea.gauge == ASTERX_GAUGE_LORENZ) {
    double G0 = ea.ga[id];
    const double* f0 = ea.fp;
    const double* f1 = ea.fp + g.N;
    const double* f2 = ea.fp + 2 * g.N;
    double div = (f0[id + 1] - f0[id - 1]) * (0.5 * g.idx[0]) + (f1[id + sy] - f1[id - sy]) * (0.5 * g.idx[1]) +
                 (f2[id + sz] - f2[id - sz]) * (0.5 * g.idx[2]);
    emit(ea.cmb, r, 5 * N + id, -Ex - (ea.ga[id + 1] - G0) * g.idx[0]);
    emit(ea.cmb, r, 6 * N + id, -Ey - (ea.ga[id + sy] - G0) * g.idx[1]);
    emit(ea.cmb, r, 7 * N + id, -Ez - (ea.ga[id + sz] - G0) * g.idx[2]);
    emit(ea.cmb, r, 8 * N + id, -div - ea.xi * ea.metric[id] * ea.psi[id]);
  } else {
    emit(ea.cmb, r, 5 * N + id, -Ex);
    emit(ea.cmb, r, 6 * N + id, -Ey);
    emit(ea.cmb, r, 7 * N + id, -Ez);
    emit(ea.cmb, r, 8 * N + id, 0.0);
  }
}

// ---------------------------------------------------------------------------------------
// RK combine on owned points of 9 fields.
struct RKArgs {
  const double* u[4];
  double a[4];
  int nterms;
  double b_dt;
  const double* rhs;
  double* out;
};

DEV void rk_body(const GD& g, const RKArgs& ra, unsigned tile) {
  int i, j, k;
  if (!box_at<64, 4>(g.n, tile, threadIdx.x, i, j, k)) return;
  const int id = at(g, i, j, k);
#pragma unroll
  for (int f = 0; f < 9; ++f) {
    size_t o = (size_t)f * g.N + id;
    ra.out[o] = rk_point<4>(ra.b_dt, ra.rhs[o], ra.u, ra.a, ra.nterms, o);
  }
}

// =======================================================================================
// Kernels.  Single block: one workgroup per logical tile of the block.  Batched: a
// persistent grid of workgroups walks a list of (patch, tile) items; every patch is a grid
// descriptor plus a base offset into field-major pools whose field stride is the total
// point count of all patches, so the same bodies run unchanged.
struct PatchDesc {
  GD g;
  long long off;
};
struct Item {
  int patch;
  int tile;
};

template <class T>
DEV T* shifted(T* p, long long off) {
  return p ? p + off : p;
}
DEV Combine shifted(const Combine& c, long long off) {
  Combine r = c;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    r.o[k].out = shifted(c.o[k].out, off);
#pragma unroll
    for (int m = 0; m < 2; ++m) r.o[k].u[m] = shifted(c.o[k].u[m], off);
  }
  return r;
}

__global__ __launch_bounds__(256) void k_prim2con(GD g, double gam, const double* metric, const double* A,
                                                  const double* prim, double* cons) {
  prim2con_body(g, gam, metric, A, prim, cons, my_tile());
}
__global__ __launch_bounds__(256) void kb_prim2con(const PatchDesc* __restrict__ P, const Item* __restrict__ it,
                                                   int nit, double gam, const double* metric, const double* A,
                                                   const double* prim, double* cons) {
  for (int w = blockIdx.x; w < nit; w += gridDim.x) {
    const Item m = it[w];
    const PatchDesc d = P[m.patch];
    prim2con_body(d.g, gam, metric + d.off, A + d.off, prim + d.off, cons + d.off, (unsigned)m.tile);
  }
}

// c2p stages two components per value round (TileLDS2); the learned guess reuses the buffer
union C2PLDS {
  TileLDS t;
  TileLDS2 t2;
};
// the cell kernel's value and derivative rounds share one buffer
union CellLDS {
  TileLDS t;
  TileLDS2 t2;
  TileLDS2D t2d;
};

__global__ __launch_bounds__(256) void k_c2p(GD g, C2PParams cp, C2PArgs a) {
  __shared__ C2PLDS S;
  c2p_body<false>(g, cp, a, S.t, my_tile());
}
__global__ __launch_bounds__(256) void k_c2p_learned(GD g, C2PParams cp, C2PArgs a) {
  __shared__ C2PLDS S;
  c2p_body<true>(g, cp, a, S.t, my_tile());
}
// 3 waves per SIMD: the stress tensor and the source weights after the recovery take about 160
// registers; held at 4 waves the kernel spills across the recovery and measured slower.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_c2p_src(GD g, C2PParams cp, C2PArgs a) {
  __shared__ CellLDS S;
  c2p_body<false, true>(g, cp, a, S.t, my_tile());
}
__global__ __launch_bounds__(256) void k_c2p_learned_src(GD g, C2PParams cp, C2PArgs a) {
  __shared__ CellLDS S;
  c2p_body<true, true>(g, cp, a, S.t, my_tile());
}
__global__ __launch_bounds__(256) void k_c2p_geo(GD g, C2PParams cp, C2PArgs a, const double* cen) {
  c2p_geo_body<false>(g, cp, a, cen, my_tile(), nullptr);
}
__global__ __launch_bounds__(256) void k_c2p_learned_geo(GD g, C2PParams cp, C2PArgs a, const double* cen) {
  __shared__ C2PGeoLDS L;
  c2p_geo_body<true>(g, cp, a, cen, my_tile(), &L);
}
__global__ __launch_bounds__(256) void kb_c2p(const PatchDesc* __restrict__ P, const Item* __restrict__ it, int nit,
                                              C2PParams cp, C2PArgs a) {
  __shared__ C2PLDS S;
  for (int w = blockIdx.x; w < nit; w += gridDim.x) {
    const Item m = it[w];
    const PatchDesc d = P[m.patch];
    C2PArgs b = a;
    b.metric = a.metric + d.off;
    b.A = a.A + d.off;
    b.cons = a.cons + d.off;
    b.prim = a.prim + d.off;
    b.flags = shifted(a.flags, d.off);
    c2p_body<false>(d.g, cp, b, S.t, (unsigned)m.tile);
  }
}

template <bool LIN>
__global__ __launch_bounds__(256) void k_fill(GD g, FillArgs a) { fill_body<LIN>(g, a, a.f, blockIdx.x); }
template <bool LIN>
__global__ __launch_bounds__(256) void kb_fill(const PatchDesc* __restrict__ P, const Item* __restrict__ it, int nit,
                                               FillArgs a) {
  for (int w = blockIdx.x; w < nit; w += gridDim.x) {
    const Item m = it[w];
    const PatchDesc d = P[m.patch];
    fill_body<LIN>(d.g, a, a.f + d.off, (unsigned)m.tile);
  }
}

__global__ __launch_bounds__(256) void k_bcent(GD g, const double* A, double* bc) { bcent_body(g, A, bc, my_tile()); }
__global__ __launch_bounds__(256) void kb_bcent(const PatchDesc* __restrict__ P, const Item* __restrict__ it, int nit,
                                                const double* A, double* bc) {
  for (int w = blockIdx.x; w < nit; w += gridDim.x) {
    const Item m = it[w];
    const PatchDesc d = P[m.patch];
    bcent_body(d.g, A + d.off, bc + d.off, (unsigned)m.tile);
  }
}

template <int MASK>
__global__ __launch_bounds__(64) void k_geom(GD g, GeomArgs ga) { geom_wave<MASK>(g, ga, my_tile()); }
// Batches: the wavefronts of a workgroup take items of their own.
DEV int first_wave_item() { return (int)(blockIdx.x * 4 + (threadIdx.x >> 6)); }
template <int MASK>
__global__ __launch_bounds__(256) void kb_geom(const PatchDesc* __restrict__ P, const Item* __restrict__ it, int nit,
                                               GeomArgs ga) {
  for (int w = __builtin_amdgcn_readfirstlane(first_wave_item()); w < nit; w += gridDim.x * 4) {
    const Item m = it[w];
    const PatchDesc d = P[m.patch];
    GeomArgs b = ga;
    b.metric = ga.metric + d.off;
    b.curv = shifted(ga.curv, d.off);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      b.fa[a] = shifted(ga.fa[a], d.off);
      b.fb[a] = shifted(ga.fb[a], d.off);
    }
    int e[3];
    geom_box(d.g.n, ga.lo, e);
    b.zl = geom_planes(e);
    geom_wave<MASK>(d.g, b, (unsigned)m.tile);
  }
}

// 3 wavefronts per SIMD: both sides' states and fluxes of a face are live together (146-168 registers); held
// at 4 the kernels spill (128^3, PPM: x faces 0.15 -> 0.21 ms, y 0.19 -> 0.24).
// NQ: two components of a gathered face metric in flight where the reconstruction leaves registers for them
// (asterx_rhs, 64^3: MINMOD 166 -> 162 us; PPM 168 -> 176, MP5 192 -> 201).  Batches, which never gather, take one:
// their kernels are what they would be without (64 patches, MINMOD, with two: 4928 -> 4955 us per step).
template <int R>
constexpr int face_nq() { return R == ASTERX_RECON_MINMOD ? 2 : 1; }
template <int D, int R, bool UCT, int NQ = face_nq<R>()>
DEV void face_wave(const GD& g, const FaceArgs& fa, unsigned item, FaceLDS& L) {
  if constexpr (D == 0) face_wave_x<R, UCT, NQ>(g, fa, item, L);
  else face_wave_yz<D, R, UCT, NQ>(g, fa, item, L);
}
template <int D, int R, bool UCT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3))) void k_face(GD g, FaceArgs fa) {
  __shared__ FaceLDS L;
  face_wave<D, R, UCT>(g, fa, my_tile(), L);
}
// The three directions in one launch: c0 and c1 x and y items, then the z items.
template <int R, bool UCT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3))) void k_faces(GD g, FaceArgs fa, unsigned c0,
                                                                                     unsigned c1) {
  __shared__ FaceLDS L;
  const unsigned w = blockIdx.x;
  if (w < c0) face_wave<0, R, UCT>(g, fa, xcd_block(w, c0), L);
  else if (w < c0 + c1) face_wave<1, R, UCT>(g, fa, xcd_block(w - c0, c1), L);
  else face_wave<2, R, UCT>(g, fa, xcd_block(w - c0 - c1, gridDim.x - c0 - c1), L);
}
template <int D, int R>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void kb_face(
    const PatchDesc* __restrict__ P, const Item* __restrict__ it, int nit, FaceArgs fa) {
  __shared__ FaceLDS L[4];
  for (int w = __builtin_amdgcn_readfirstlane(first_wave_item()); w < nit; w += gridDim.x * 4) {
    const Item m = it[w];
    const PatchDesc d = P[m.patch];
    FaceArgs b = fa;
    b.metric = fa.metric + d.off;
    b.prim = fa.prim + d.off;
    b.A = fa.A + d.off;
    b.bc = fa.bc + d.off;
    b.flux = fa.flux + d.off;
    b.fma[D] = shifted(fa.fma[D], d.off);
    b.fmb[D] = shifted(fa.fmb[D], d.off);
    wave_lds_sync();  // the previous item's reads come before this one's writes
    face_wave<D, R, false, 1>(d.g, b, (unsigned)m.tile, L[threadIdx.x >> 6]);
  }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_cell(GD g, CellArgs ca) {
  __shared__ CellLDS S;
  cell_body(g, ca, S.t, my_tile());
}
__global__ __launch_bounds__(256) void kb_cell(const PatchDesc* __restrict__ P, const Item* __restrict__ it, int nit,
                                               CellArgs ca) {
  __shared__ CellLDS S;
  for (int w = blockIdx.x; w < nit; w += gridDim.x) {
    const Item m = it[w];
    const PatchDesc d = P[m.patch];
    CellArgs b = ca;
    b.metric = ca.metric + d.off;
    b.curv = ca.curv + d.off;
    b.prim = ca.prim + d.off;
    b.A = ca.A + d.off;
    b.bc = ca.bc + d.off;
    b.flux = ca.flux + d.off;
    b.rhs = shifted(ca.rhs, d.off);
    b.cmb = shifted(ca.cmb, d.off);
    cell_body(d.g, b, S.t, (unsigned)m.tile);
  }
}

__global__ __launch_bounds__(256) void k_vertex(GD g, VertexArgs va) { vertex_body(g, va, my_tile()); }
__global__ __launch_bounds__(256) void k_tmunu(GD g, TmunuArgs ta) {
  __shared__ TmunuLDS L;
  tmunu_body(g, ta, my_tile(), L);
}
template <int STAG>
__global__ __launch_bounds__(256) void k_prolong(InterArgs a) { prolong_body<STAG>(a, my_tile()); }
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_prolong_cells(InterArgs a) {
  const unsigned per = gridDim.x / (unsigned)a.nf;
  prolong_cells_body(a, xcd_block(blockIdx.x % per, per), (int)(blockIdx.x / per));
}
__global__ __launch_bounds__(256) void k_restrict(InterArgs a) { restrict_body(a, my_tile()); }
__global__ __launch_bounds__(256) void kb_vertex(const PatchDesc* __restrict__ P, const Item* __restrict__ it, int nit,
                                                 VertexArgs va) {
  for (int w = blockIdx.x; w < nit; w += gridDim.x) {
    const Item m = it[w];
    const PatchDesc d = P[m.patch];
    VertexArgs b{va.metric + d.off, va.A + d.off, va.psi + d.off, va.ga + d.off, va.fp + d.off};
    vertex_body(d.g, b, (unsigned)m.tile);
  }
}

__global__ __launch_bounds__(256) void k_edge(GD g, EdgeArgs ea) { edge_body(g, ea, my_tile()); }
__global__ __launch_bounds__(256) void k_edge_uct(GD g, EdgeArgs ea) { edge_body<true>(g, ea, my_tile()); }
// Two phases that don't depend on each other in one launch, the first n0 workgroups for the first: the centre
// field and the gauge quantities before the faces, the divergence and the edges after them.  RK4 steps from a graph,
// PPM, the first pair apart, the second pair apart, both in one launch: 16^3 0.163, 0.173, 0.154 ms; 64^3 0.722, 0.725,
// 0.709; 128^3 4.959, 4.944, 4.925; 192^3 15.80, 15.80, 15.78.
__global__ __launch_bounds__(256) void k_bcent_vertex(GD g, const double* A, double* bc, VertexArgs va, unsigned n0) {
  if (blockIdx.x < n0) bcent_body(g, A, bc, xcd_block(blockIdx.x, n0));
  else vertex_body(g, va, xcd_block(blockIdx.x - n0, gridDim.x - n0));
}
template <bool UCT>
__global__ __launch_bounds__(256) void k_div_edge(GD g, DivArgs da, EdgeArgs ea, unsigned n0) {
  if (blockIdx.x < n0) div_body(g, da, xcd_block(blockIdx.x, n0));
  else edge_body<UCT>(g, ea, xcd_block(blockIdx.x - n0, gridDim.x - n0));
}
__global__ __launch_bounds__(256) void kb_edge(const PatchDesc* __restrict__ P, const Item* __restrict__ it, int nit,
                                               EdgeArgs ea) {
  for (int w = blockIdx.x; w < nit; w += gridDim.x) {
    const Item m = it[w];
    const PatchDesc d = P[m.patch];
    EdgeArgs b = ea;
    b.metric = ea.metric + d.off;
    b.psi = ea.psi + d.off;
    b.flux = ea.flux + d.off;
    b.ga = ea.ga + d.off;
    b.fp = ea.fp + d.off;
    b.rhs = shifted(ea.rhs, d.off);
    b.cmb = shifted(ea.cmb, d.off);
    edge_body(d.g, b, (unsigned)m.tile);
  }
}

__global__ __launch_bounds__(256) void k_rk(GD g, RKArgs ra) { rk_body(g, ra, my_tile()); }
__global__ __launch_bounds__(256) void kb_rk(const PatchDesc* __restrict__ P, const Item* __restrict__ it, int nit,
                                             RKArgs ra) {
  for (int w = blockIdx.x; w < nit; w += gridDim.x) {
    const Item m = it[w];
    const PatchDesc d = P[m.patch];
    RKArgs b = ra;
#pragma unroll
    for (int q = 0; q < 4; ++q) b.u[q] = shifted(ra.u[q], d.off);
    b.rhs = ra.rhs + d.off;
    b.out = ra.out + d.off;
    rk_body(d.g, b, (unsigned)m.tile);
  }
}

// =======================================================================================
// Adjoint (vector-Jacobian products) of one right-hand side evaluation with its c2p.
// The linear parts (flux divergence, FCT averages, gauge terms, staggered curl and averages,
// periodic ghost fills) are transposed exactly; the face physics of each side runs one
// hand-written reverse sweep (side_vjp), the other pointwise nonlinear parts (reconstruction,
// sources) build local Jacobians with dual numbers (forward mode) and contract them with the
// incoming cotangents; converged iterations (quartic roots, c2p) are differentiated through
// the implicit-function theorem.  Non-smooth points take the active branch; an exact tie of
// the two sides in the HLLE max/min splits the cotangent equally (the central derivative).

// Adjoint workspace: fields of the block's index space.
enum {
  AW_CONS = 0, AW_PRIM = 5, AW_BC = 10, AW_PBAR = 13, AW_BCBAR = 18, AW_BFBAR = 21, AW_ABAR = 24, AW_PSIBAR = 27,
  AW_AVBAR = 28, AW_FBAR = 31, AW_FIELDS = 52,
  AW_XBAR = AW_ABAR  // seven fields that hold nothing until the faces are done
};
// The Gamma cotangent is accumulated into GSLOTS workspace slots (workgroup id modulo GSLOTS):
// per-wavefront FP64 atomics to one address would serialize in L2.  The slots are summed in a
// fixed order into the caller's gamma_bar at the end of each adjoint call.
constexpr int GSLOTS = 64;

DEV void gslots_body(const double* __restrict__ slots, double* __restrict__ gamma_bar) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    double t = 0.0;
    for (int q = 0; q < GSLOTS; ++q) t += slots[q];
    gamma_bar[0] += t;
  }
}

DEV bool owned3(const GD& g, int i, int j, int k) {
  return i >= 0 && j >= 0 && k >= 0 && i < g.n[0] && j < g.n[1] && k < g.n[2];
}

// Cotangent of one field at (i, j, k) if that point is owned, else 0.
DEV double rb_at(const GD& g, const double* r, int i, int j, int k) {
  return owned3(g, i, j, k) ? r[at(g, i, j, k)] : 0.0;
}

// Face-flux cotangents from the right-hand-side cotangent rbar (9 fields, owned points):
// hydro components through the divergence (rhs[i] = -(F[i+e] - F[i]) / dx, so
// Fbar[f] = (rbar[f] - rbar[f-e]) / dx), induction components through the FCT averages.
struct FluxBarArgs {
  const double* rbar;
  double* fbar;
};

DEV void fluxbar_body(const GD& g, const FluxBarArgs& a, unsigned tile) {
  int e[3] = {g.n[0] + 2, g.n[1] + 2, g.n[2] + 2};
  int p, q, r;
  if (!box_at<64, 4>(e, tile, threadIdx.x, p, q, r)) return;
  const int i = p - 1, j = q - 1, k = r - 1;  // every index in [-1, n]
  const int id = at(g, i, j, k);
  const double* R = a.rbar;
  auto rc = [&](int c, int ii, int jj, int kk) { return rb_at(g, R + (size_t)c * g.N, ii, jj, kk); };
  const int off[3][3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}};
  for (int d = 0; d < 3; ++d) {
    const int il = i - off[d][0], jl = j - off[d][1], kl = k - off[d][2];
#pragma unroll
    for (int c = 0; c < 5; ++c)
      a.fbar[(size_t)(d * 7 + c) * g.N + id] = (rc(c, i, j, k) - rc(c, il, jl, kl)) * g.idx[d];
  }
  // dA/dt = -E: Ebar = -rbar_A; E components are quarter-sums of induction fluxes
  double* fb = a.fbar;
  fb[(size_t)(0 * 7 + 5) * g.N + id] = 0.25 * (rc(7, i, j, k) + rc(7, i, j + 1, k));   // Fx_By <- E_z
  fb[(size_t)(0 * 7 + 6) * g.N + id] = -0.25 * (rc(6, i, j, k) + rc(6, i, j, k + 1));  // Fx_Bz <- E_y
  fb[(size_t)(1 * 7 + 5) * g.N + id] = 0.25 * (rc(5, i, j, k) + rc(5, i, j, k + 1));   // Fy_Bz <- E_x
  fb[(size_t)(1 * 7 + 6) * g.N + id] = -0.25 * (rc(7, i, j, k) + rc(7, i + 1, j, k));  // Fy_Bx <- E_z
  fb[(size_t)(2 * 7 + 5) * g.N + id] = 0.25 * (rc(6, i, j, k) + rc(6, i + 1, j, k));   // Fz_Bx <- E_y
  fb[(size_t)(2 * 7 + 6) * g.N + id] = -0.25 * (rc(5, i, j, k) + rc(5, i, j + 1, k));  // Fz_By <- E_x
}

struct FaceAdjArgs {
  const double* metric;
  const double* prim;
  const double* A;
  const double* bc;
  double* fbar;
  double* xbar;  // seven fields
  double* pbar;
  double* bcbar;
  double* bfbar;
  double* gbar;
  double gam, weno_eps, weno_q;
  int speeds, riemann;
  int rows = 0;  // points per march of the transposed reconstruction along y and z
};

template <int D, int RECON>
DEV void face_adj_body(const GD& g, const FaceAdjArgs& fa, unsigned tile) {
  constexpr int t1 = (D + 1) % 3, t2 = (D + 2) % 3;
  const int side = threadIdx.x & 1;
  int e[3] = {g.n[0] + 1, g.n[1] + 1, g.n[2] + 1};
  int a, b, c;
  bool rest;
  int ax0, by0;
  bool valid = face_at<face_zg<D>()>(e, tile, threadIdx.x >> 1, a, b, c, rest, ax0, by0);
  double gsum = 0.0;
  if (valid) {
    int ijk[3] = {a - 1, b - 1, c - 1};
    ijk[D] += 1;
    const int id = at(g, ijk[0], ijk[1], ijk[2]);
    const int st[3] = {1, g.sy, g.sz};
    const int sD = st[D], s1 = st[t1], s2 = st[t2];
    const int o0 = side ? 2 : -3, os = side ? -1 : 1;
    // forward recomputation of this lane's side
    auto field = [&](int v) { return v < 5 ? fa.prim + v * g.N : fa.bc + (v == 5 ? t1 : t2) * g.N; };
    double X[7];
#pragma unroll
    for (int v = 0; v < 7; ++v) {
      double sten[5];
#pragma unroll
      for (int q = 0; q < 5; ++q) sten[q] = field(v)[id + (o0 + os * q) * sD];
      X[v] = recon_right_face<RECON>(sten, fa.weno_eps, fa.weno_q);
    }
    double mine[5];
    const int mb = id - s1 - s2;
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      const double* p = fa.metric + (size_t)(5 * side + q) * g.N + mb;
      double rr[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double* row = p + r * s2;
        rr[r] = lag(row[0], row[s1], row[2 * s1], row[3 * s1]);
      }
      mine[q] = lag(rr[0], rr[1], rr[2], rr[3]);
    }
    double m[10];
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      double other = shfl1(mine[q]);
      m[q] = side ? other : mine[q];
      m[5 + q] = side ? mine[q] : other;
    }
    Geo G;
    geo_from(m, G);
    const double* Ax = fa.A;
    const double* Ay = fa.A + g.N;
    const double* Az = fa.A + 2 * g.N;
    double Bn = D == 0 ? faceBx(Ay, Az, id, g.sy, g.sz, g)
                       : (D == 1 ? faceBy(Ax, Az, id, g.sy, g.sz, g) : faceBz(Ax, Ay, id, g.sy, g.sz, g));
    bool fallback;
    {
      double vl[3], v[3] = {X[2], X[3], X[4]};
      lower(G.g, v, vl);
      double v2 = v[0] * vl[0] + v[1] * vl[1] + v[2] * vl[2];
      fallback = !(X[0] > 0.0) || !(X[1] > 0.0) || !(v2 < 1.0);
      if (fallback) {
        // this side's own cell (stencil point 2)
#pragma unroll
        for (int q = 0; q < 7; ++q) X[q] = field(q)[id + (o0 + os * 2) * sD];
      }
    }
    double Bt[3];
    Bt[D] = Bn;
    Bt[t1] = X[5];
    Bt[t2] = X[6];
    State S;
    state_make(G, X, Bt, fa.gam, S);
    double U[7], F[7], cm, cp;
    flux_of<D>(G, S, U, F);
    speeds_of<D>(G, S, fa.gam, fa.speeds, cm, cp);
    double Uo[7], Fo[7];
#pragma unroll
    for (int q = 0; q < 7; ++q) {
      Uo[q] = shfl1(U[q]);
      Fo[q] = shfl1(F[q]);
    }
    double cmo = shfl1(cm), cpo = shfl1(cp);
    double cmax = fmax(0.0, fmax(cp, cpo));
    double cmin = -fmin(0.0, fmin(cm, cmo));
    double den = cmax + cmin;
    // HLLE transposed for this lane's side
    double fbar[7];
#pragma unroll
    for (int q = 0; q < 7; ++q) fbar[q] = fa.fbar[(size_t)(D * 7 + q) * g.N + id];
    double Ub[7], Fb[7], cmb = 0.0, cpb = 0.0;
    if (fa.riemann == ASTERX_RIEMANN_LXF) {
      // (F_L + F_R - c_wave (U_R - U_L)) / 2 transposed; c_wave = max(cmax, cmin)
      const double cw = fmax(cmax, cmin);
      double dcw = 0.0;
#pragma unroll
      for (int q = 0; q < 7; ++q) {
        Fb[q] = 0.5 * fbar[q];
        Ub[q] = (side ? -0.5 : 0.5) * cw * fbar[q];
        const double UL = side ? Uo[q] : U[q], UR = side ? U[q] : Uo[q];
        dcw -= 0.5 * fbar[q] * (UR - UL);
      }
      double dcmax = cmax > cmin ? dcw : (cmax == cmin ? 0.5 * dcw : 0.0);
      double dcmin = cmin > cmax ? dcw : (cmax == cmin ? 0.5 * dcw : 0.0);
      if (cmax > 0.0) {
        if (cp == cpo) cpb = 0.5 * dcmax;
        else if (cp > cpo) cpb = dcmax;
      }
      if (cmin > 0.0) {
        if (cm == cmo) cmb = -0.5 * dcmin;
        else if (cm < cmo) cmb = -dcmin;
      }
    } else if (den > 0.0) {
      double id_ = 1.0 / den, cc = cmax * cmin;
      double wF = (side ? cmin : cmax) * id_, wU = (side ? -cc : cc) * id_;
      double dcmax = 0.0, dcmin = 0.0;
#pragma unroll
      for (int q = 0; q < 7; ++q) {
        Fb[q] = fbar[q] * wF;
        Ub[q] = fbar[q] * wU;
        double FL = side ? Fo[q] : F[q], FR = side ? F[q] : Fo[q];
        double UL = side ? Uo[q] : U[q], UR = side ? U[q] : Uo[q];
        double fo = (cmin * FR + cmax * FL - cc * (UR - UL)) * id_;
        dcmax += fbar[q] * (FL - cmin * (UR - UL) - fo) * id_;
        dcmin += fbar[q] * (FR - cmax * (UR - UL) - fo) * id_;
      }
      // cmax = max(0, c+_L, c+_R), cmin = -min(0, c-_L, c-_R): to the active side, half each on a tie
      if (cmax > 0.0) {
        if (cp == cpo) cpb = 0.5 * dcmax;
        else if (cp > cpo) cpb = dcmax;
      }
      if (cmin > 0.0) {
        if (cm == cmo) cmb = -0.5 * dcmin;
        else if (cm < cmo) cmb = -dcmin;
      }
    } else {
#pragma unroll
      for (int q = 0; q < 7; ++q) {
        Fb[q] = 0.5 * fbar[q];
        Ub[q] = 0.0;
      }
    }
    // local VJP through (X, Bn, Gamma) -> (U, F, c-, c+): one reverse sweep
    double Xb[7], Bnb, gb;
    side_vjp<D>(G, X, Bn, fa.gam, fa.speeds, cp, cm, Ub, Fb, cmb, cpb, Xb, Bnb, gb);
    // The cotangents of the two states: the left one's into xbar, the right one's in place of the flux
    // cotangent (read by both lanes of the pair above).  Unphysical reconstructions used the own cell's values.
    double* xb = side ? fa.fbar + (size_t)(D * 7) * g.N : fa.xbar;
#pragma unroll
    for (int v = 0; v < 7; ++v) {
      if (fallback) {
        double* dst = v < 5 ? fa.pbar + v * g.N : fa.bcbar + (v == 5 ? t1 : t2) * g.N;
        atomicAdd(dst + id + (o0 + os * 2) * sD, Xb[v]);
        Xb[v] = 0.0;
      }
      xb[(size_t)v * g.N + id] = Xb[v];
    }
    // the normal field is shared by both sides: sum the pair, one store per face
    double bn_total = Bnb + shfl1(Bnb);
    if (side == 0) fa.bfbar[(size_t)D * g.N + id] += bn_total;
    gsum = gb;
  }
  double w = gsum;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) w += __shfl_xor(w, o, 64);
  if (__lane_id() == 0 && w != 0.0) atomicAdd(fa.gbar + (blockIdx.x & (GSLOTS - 1)), w);
}

// Reconstruction transposed: the cotangents of the states at a direction's faces (left ones in fa.xbar, right
// ones in fa.fbar) to the cells of their stencils.  Each point gathers what the five cells around it send it,
// in a fixed order.  As a scatter at the end of the face adjoint, 70 FP64 atomics per face, it set that kernel's
// time: 64^3, PPM, x/y/z faces 341/222/240 us with the scatter, 72/61/61 us without, and 19/26/26 us here.  The
// slopes are selected without branches (as branches, whose targets went through scratch: 97/139/137 us).
// A wavefront takes one variable.  x: 64 consecutive stored points, of which the middle 60 are complete, with
// the exchange through LDS.  y and z: 64 columns, a march over `rows` points of each (and the two cells
// before and after them) with the five running sums in registers.
// Cells in [-1, n] along D have a face of [0, n]; their stencils reach [-3, n + 2], inside the ghosts.
__host__ __device__ inline unsigned recon_adj_items(const GD& g, int D, int rows) {
  if (D == 0) return (unsigned)(((long long)g.ld0 * (g.n[1] + 1) * (g.n[2] + 1) + 59) / 60 * 7);
  const long long cols = (long long)(g.n[0] + 1) * (g.n[D == 1 ? 2 : 1] + 1);
  return (unsigned)((cols + 63) / 64 * ((g.n[D] + 6 + rows - 1) / rows) * 7);
}
// Points per march: a march of r points transposes r + 4 cells one after another, so that blocks whose marches leave
// the chip idle take the length whose rounds of wavefronts cost least (asterx_rhs_adjoint with marches of 8, 4, 2, 1
// points: 16^3, MP5, 225, 208, 202, 196 us; 32^3, PPM, 225, 221, 220, 225; 48^3, MP5, 380, 370, 386, 431; 64^3, PPM, 534,
// 538, 553, 588).
inline int recon_adj_rows(const GD& g, int D) {
  int best = 8;
  unsigned least = ~0u;
  for (int r = 8; r >= 1; r /= 2) {
    const unsigned cost = (recon_adj_items(g, D, r) + FACE_SLOTS - 1) / FACE_SLOTS * (unsigned)(r + 4);
    if (cost < least) {
      least = cost;
      best = r;
    }
  }
  return best;
}

// Transpose of both face values of the cell of stencil a: ab[k] goes to the point k - 2 from it.
template <int RECON>
DEV void recon_cell_vjp(const FaceAdjArgs& fa, const double a[5], double lb, double hb, double ab[5]) {
  if constexpr (RECON == ASTERX_RECON_MINMOD) {
    // centre -+ half the smaller difference, or the centre at an extremum
    const double x = a[2] - a[1], y = a[3] - a[2], h = 0.5 * (hb - lb);
    const bool up = x * y > 0.0, left = fabs(x) <= fabs(y);
    const double hl = up && left ? h : 0.0, hr = up && !left ? h : 0.0;
    ab[0] = ab[4] = 0.0;
    ab[1] = -hl;
    ab[2] = hb + lb + hl - hr;
    ab[3] = hr;
  } else if constexpr (RECON == ASTERX_RECON_PPM) {
    ppm_cell_vjp(a, lb, hb, ab);
  } else if constexpr (RECON == ASTERX_RECON_WENOZ) {
    wenoz_cell_vjp(a, fa.weno_eps, fa.weno_q, lb, hb, ab);
  } else {
    const double b[5] = {a[4], a[3], a[2], a[1], a[0]};
    double r[5];
    mp5_face_vjp(a, hb, ab);
    mp5_face_vjp(b, lb, r);
#pragma unroll
    for (int k = 0; k < 5; ++k) ab[k] += r[4 - k];
  }
}

template <int D, int RECON>
DEV void recon_adj_wave(const GD& g, const FaceAdjArgs& fa, unsigned item, double (*L)[64]) {
  constexpr int t1 = (D + 1) % 3, t2 = (D + 2) % 3;
  const int sD = D == 0 ? 1 : (D == 1 ? g.sy : g.sz), n = g.n[D];
  const int v = (int)(item % 7);
  const unsigned w = item / 7;
  const double* f = v < 5 ? fa.prim + (size_t)v * g.N : fa.bc + (size_t)(v == 5 ? t1 : t2) * g.N;
  double* out = v < 5 ? fa.pbar + (size_t)v * g.N : fa.bcbar + (size_t)(v == 5 ? t1 : t2) * g.N;
  const double* xl = fa.xbar + (size_t)v * g.N;
  const double* xr = fa.fbar + (size_t)(D * 7 + v) * g.N;
  if constexpr (D == 0) {
    const int l = __lane_id();
    const long long q = (long long)w * 60 + l - 2;
    const unsigned rows = (unsigned)(g.n[1] + 1) * (g.n[2] + 1);
    const bool in = q >= 0 && q < (long long)g.ld0 * rows;
    const unsigned row = in ? (unsigned)q / g.ld0 : 0;
    const int c = in ? (int)((unsigned)q % g.ld0) - g.ng : -g.ng;
    const int id = at(g, c, (int)(row % (g.n[1] + 1)) - 1, (int)(row / (g.n[1] + 1)) - 1);
    double ab[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    if (in && c >= -1 && c <= n) {
      double a[5];
#pragma unroll
      for (int k = 0; k < 5; ++k) a[k] = f[id + k - 2];
      recon_cell_vjp<RECON>(fa, a, c >= 0 ? xr[id] : 0.0, c < n ? xl[id + 1] : 0.0, ab);
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) L[k][l] = ab[k];
    wave_lds_sync();
    // the cell k - 2 below sends its k-th contribution here; rows end in points that get none
    if (in && l >= 2 && l < 62 && c >= -3 && c <= n + 2) {
      double t = 0.0;
#pragma unroll
      for (int k = 0; k < 5; ++k) t += L[k][l - k + 2];
      out[id] += t;
    }
  } else {
    const unsigned nx = (unsigned)g.n[0] + 1, cols = nx * (unsigned)(g.n[D == 1 ? 2 : 1] + 1);
    const unsigned nch = (unsigned)(n + 6 + fa.rows - 1) / fa.rows;
    const unsigned col = w / nch * 64 + __lane_id();
    if (col >= cols) return;
    const int p0 = (int)(w % nch) * fa.rows - 3, p1 = min(p0 + fa.rows, n + 3);
    const int x = (int)(col % nx) - 1, o = (int)(col / nx) - 1;
    const int base = D == 1 ? at(g, x, 0, o) : at(g, x, o, 0);
    // points inside [-3, n + 2]
    auto val = [&](int c) { return c >= -3 && c <= n + 2 ? f[base + c * sD] : 0.0; };
    double a[5], acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 1; k < 5; ++k) a[k] = val(p0 - 5 + k);
#pragma unroll 4
    for (int c = p0 - 2; c < p1 + 2; ++c) {
      const int id = base + c * sD;
#pragma unroll
      for (int k = 0; k < 4; ++k) a[k] = a[k + 1];
      a[4] = val(c + 2);
      double ab[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
      if (c >= -1 && c <= n)
        recon_cell_vjp<RECON>(fa, a, c >= 0 ? xr[id] : 0.0, c < n ? xl[id + sD] : 0.0, ab);
      // acc[k] gathers for point c - 2 + k
#pragma unroll
      for (int k = 0; k < 5; ++k) acc[k] += ab[k];
      if (c - 2 >= p0) out[id - 2 * sD] += acc[0];
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[k] = acc[k + 1];
      acc[4] = 0.0;
    }
  }
}

// Geometric sources transposed, one owned cell per thread, over the cell tiles of the forward
// kernels: the metric's centre values and derivatives and the curvature come from the same
// LDS-staged separable passes (metric_values10 / value_rounds16, metric_derivs_dot).
struct CellAdjArgs {
  const double* metric;
  const double* curv;
  const double* prim;
  const double* bc;
  const double* rbar;
  double* pbar;
  double* bcbar;
  double* gbar;
  double gam;
};

// sum_k rb_k src_k of the densitized sources alpha sqrt(gamma) (1/2 T^{mu nu} d_j g_{mu nu}, energy
// term) of one state, in dual numbers (the formulas of the forward cell kernel).  The momentum source
// along j is linear in the metric derivatives along j, so its contraction with rb_{1+j} is the
// momentum formula evaluated once on E_c = sum_j rb_{1+j} d_j m_c; dal = d_j alpha, K the curvature.
DEV Dual sources_dot_dual(const Geo& G, const double E[10], const double dal[3], const double K[6], double rb4,
                          const Dual pr[5], const Dual Bt[3], Dual gam) {
  StateT<Dual> St;
  state_make(G, pr, Bt, gam, St, gam / (gam - 1.0));
  double ia = 1.0 / G.alp, ia2 = ia * ia;
  Dual u0 = St.W * ia, b0 = St.W * St.Bv * ia, u[3], bu[3];
  for (int a = 0; a < 3; ++a) {
    u[a] = St.W * (St.v[a] - G.beta[a] * ia);
    bu[a] = (St.B[a] + G.alp * b0 * u[a]) / St.W;
  }
  Dual e = St.rhoh + St.bsq, pt = St.p + 0.5 * St.bsq;
  Dual T00 = e * u0 * u0 - pt * ia2 - b0 * b0;
  Dual T0[3], Tk[6];
  for (int a = 0; a < 3; ++a) T0[a] = e * u0 * u[a] + pt * G.beta[a] * ia2 - b0 * bu[a];
  for (int a = 0; a < 3; ++a)
    for (int b = a; b < 3; ++b)
      Tk[sym(a, b)] = e * u[a] * u[b] + pt * (G.gu[sym(a, b)] - G.beta[a] * G.beta[b] * ia2) - bu[a] * bu[b];
  double bl[3];
  lower(G.g, G.beta, bl);
  double as = G.alp * G.sqrtg;
  // momentum, contracted
  const double* dg = &E[4];
  const double dalE = E[0], db[3] = {E[1], E[2], E[3]};
  double bbdg = 0.0;
  Dual Tdg(0.0);
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b) {
      bbdg += G.beta[a] * G.beta[b] * dg[sym(a, b)];
      Tdg += Tk[sym(a, b)] * dg[sym(a, b)];
    }
  double d00 = -2.0 * G.alp * dalE + bbdg + 2.0 * (bl[0] * db[0] + bl[1] * db[1] + bl[2] * db[2]);
  Dual s0k(0.0);
  for (int a = 0; a < 3; ++a) {
    double d0a = 0.0;
    for (int b = 0; b < 3; ++b) d0a += G.beta[b] * dg[sym(a, b)] + G.g[sym(a, b)] * db[b];
    s0k += T0[a] * d0a;
  }
  Dual mom = 0.5 * T00 * d00 + s0k + 0.5 * Tdg;
  // energy
  double bK[3];
  for (int a = 0; a < 3; ++a) bK[a] = G.beta[0] * K[sym(a, 0)] + G.beta[1] * K[sym(a, 1)] + G.beta[2] * K[sym(a, 2)];
  Dual se = T00 * (G.beta[0] * bK[0] + G.beta[1] * bK[1] + G.beta[2] * bK[2] -
                   (G.beta[0] * dal[0] + G.beta[1] * dal[1] + G.beta[2] * dal[2]));
  for (int a = 0; a < 3; ++a) se += T0[a] * (2.0 * bK[a] - dal[a]);
  for (int a = 0; a < 3; ++a)
    for (int b = 0; b < 3; ++b) se += Tk[sym(a, b)] * K[sym(a, b)];
  return as * (mom + rb4 * se);
}

DEV void cell_adj_body(const GD& g, const CellAdjArgs& ca, CellLDS& S, unsigned tile) {
  const TileCell t = tile_cell(g, tile);
  const TileIdx x = tile_index(g, t);
  const int id = t.valid ? at(g, t.i0 + t.cx, t.j0 + t.cy, t.k0 + t.cz) : 0;
  double rb[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (t.valid)
    for (int c = 0; c < 5; ++c) rb[c] = ca.rbar[(size_t)c * g.N + id];
  double m[10], K[6], pre[NFETCH], E[10], dal[3];
  bool flat;
  value_rounds16(g, ca.metric, ca.curv, x, m, K, pre, S.t2);
  metric_derivs_dot(g, ca.metric, x, pre, rb + 1, E, dal, flat, S.t2d);
  for (int c = 0; c < 6; ++c) flat = flat && K[c] == 0.0;
  double gsum = 0.0;
  // a metric with no derivatives and no curvature has no sources
  if (t.valid && !flat && (rb[1] != 0.0 || rb[2] != 0.0 || rb[3] != 0.0 || rb[4] != 0.0)) {
    Geo G;
    geo_from(m, G);
    double pr[5], Bt[3];
    for (int c = 0; c < 5; ++c) pr[c] = ca.prim[c * g.N + id];
    for (int c = 0; c < 3; ++c) Bt[c] = ca.bc[c * g.N + id];
#pragma unroll 1
    for (int dir = 0; dir < 9; ++dir) {
      Dual pd[5], bd[3];
      for (int c = 0; c < 5; ++c) pd[c] = Dual(pr[c], dir == c ? 1.0 : 0.0);
      for (int c = 0; c < 3; ++c) bd[c] = Dual(Bt[c], dir == 5 + c ? 1.0 : 0.0);
      const double s = sources_dot_dual(G, E, dal, K, rb[4], pd, bd, Dual(ca.gam, dir == 8 ? 1.0 : 0.0)).d;
      if (dir < 5) ca.pbar[(size_t)dir * g.N + id] += s;
      else if (dir < 8) ca.bcbar[(size_t)(dir - 5) * g.N + id] += s;
      else gsum = s;
    }
  }
  double w = gsum;
  for (int o = 32; o >= 1; o >>= 1) w += __shfl_xor(w, o, 64);
  if (__lane_id() == 0 && w != 0.0) atomicAdd(ca.gbar + (blockIdx.x & (GSLOTS - 1)), w);
}

// Gauge terms transposed at vertices [-1, n]^3: G_A and F_Psi cotangents from the A and Psi
// right-hand-side cotangents, then to Psi and to the vertex-averaged potential.
struct VertexAdjArgs {
  const double* metric;
  const double* rbar;
  double* psibar;
  double* avbar;
  double xi;
  int gauge;
};

DEV void vertex_adj_body(const GD& g, const VertexAdjArgs& va, unsigned tile) {
  int e[3] = {g.n[0] + 2, g.n[1] + 2, g.n[2] + 2};
  int p, q, r;
  if (!box_at<64, 4>(e, tile, threadIdx.x, p, q, r)) return;
  const int i = p - 1, j = q - 1, k = r - 1;
  const int id = at(g, i, j, k);
  const double* R = va.rbar;
  auto rc = [&](int c, int ii, int jj, int kk) { return rb_at(g, R + (size_t)c * g.N, ii, jj, kk); };
  double mm_[10];
  for (int c = 0; c < 10; ++c) mm_[c] = va.metric[(size_t)c * g.N + id];
  Geo G;
  geo_from(mm_, G);
  double psb = 0.0, avb[3] = {0.0, 0.0, 0.0};
  if (va.gauge == ASTERX_GAUGE_LORENZ) {
    // dA_d/dt[edge] -= (G_A[edge + e_d] - G_A[edge]) / dx_d, so G_A's cotangent at vertex v is
    // sum_d (rbar_A_d[v] - rbar_A_d[v - e_d]) / dx_d
    double gb = (rc(5, i, j, k) - rc(5, i - 1, j, k)) * g.idx[0] + (rc(6, i, j, k) - rc(6, i, j - 1, k)) * g.idx[1] +
                (rc(7, i, j, k) - rc(7, i, j, k - 1)) * g.idx[2];
    // dPsi/dt[v] = -(F[v + e] - F[v - e]) / (2 dx) - xi alpha Psi[v]
    double fb[3] = {(rc(8, i + 1, j, k) - rc(8, i - 1, j, k)) * 0.5 * g.idx[0],
                    (rc(8, i, j + 1, k) - rc(8, i, j - 1, k)) * 0.5 * g.idx[1],
                    (rc(8, i, j, k + 1) - rc(8, i, j, k - 1)) * 0.5 * g.idx[2]};
    double as = G.alp * G.sqrtg;
    psb = gb * G.alp / G.sqrtg - (fb[0] * G.beta[0] + fb[1] * G.beta[1] + fb[2] * G.beta[2]) -
          va.xi * G.alp * rc(8, i, j, k);
    for (int kk = 0; kk < 3; ++kk)
      avb[kk] = -gb * G.beta[kk] +
                as * (fb[0] * G.gu[sym(0, kk)] + fb[1] * G.gu[sym(1, kk)] + fb[2] * G.gu[sym(2, kk)]);
  }
  va.psibar[id] += psb;
  for (int c = 0; c < 3; ++c) va.avbar[(size_t)c * g.N + id] = avb[c];
}

// Edge potential from the vertex averages (A^v_d[v] = (A_d[v - e_d] + A_d[v]) / 2), edges
// [-2, n]^3 (gather, one edge per thread).
DEV void edge_adj_body(const GD& g, const double* __restrict__ avbar, double* __restrict__ abar, unsigned tile) {
  int e[3] = {g.n[0] + 3, g.n[1] + 3, g.n[2] + 3};
  int p, q, r;
  if (!box_at<64, 4>(e, tile, threadIdx.x, p, q, r)) return;
  const int i = p - 2, j = q - 2, k = r - 2;
  const int id = at(g, i, j, k);
  const int st[3] = {1, g.sy, g.sz};
  const int ijk[3] = {i, j, k};
  for (int d = 0; d < 3; ++d) {
    auto inv = [&](int dd) {  // vertex index shifted by dd along d within [-1, n]^3
      for (int a = 0; a < 3; ++a) {
        int v = ijk[a] + (a == d ? dd : 0);
        if (v < -1 || v > g.n[a]) return false;
      }
      return true;
    };
    double s = 0.0;
    if (inv(0)) s += 0.5 * avbar[(size_t)d * g.N + id];
    if (inv(1)) s += 0.5 * avbar[(size_t)d * g.N + id + st[d]];
    abar[(size_t)d * g.N + id] += s;
  }
}

// Periodic ghost fill transposed along axis d: every ghost cotangent is added to its image
// and cleared (axes are undone in the reverse order of the fill).
struct FillTArgs {
  double* f;
  int nf;
  int d;
};

DEV void fillT_body(const GD& g, const FillTArgs& a, unsigned tile) {
  const int d = a.d;
  int cnt[3] = {g.n[0] + 2 * g.ng + 1, g.n[1] + 2 * g.ng + 1, g.n[2] + 2 * g.ng + 1};
  cnt[d] = 2 * g.ng + 1;
  long long tid = (long long)tile * 256 + threadIdx.x;
  if (tid >= (long long)cnt[0] * cnt[1] * cnt[2]) return;
  int q0 = (int)(tid % cnt[0]);
  long long r = tid / cnt[0];
  int q1 = (int)(r % cnt[1]);
  int q2 = (int)(r / cnt[1]);
  int idx[3] = {q0 - g.ng, q1 - g.ng, q2 - g.ng};
  int n = g.n[d];
  int q = idx[d] + g.ng;
  int s = q < g.ng ? q - g.ng : n + (q - g.ng);
  idx[d] = s;
  int dst = at(g, idx[0], idx[1], idx[2]);
  int stride = d == 0 ? 1 : (d == 1 ? g.sy : g.sz);
  int src = ((s % n) + n) % n;
  for (int f = 0; f < a.nf; ++f) {
    double* F = a.f + (size_t)f * g.N;
    double v = F[dst];
    if (v != 0.0) atomicAdd(F + dst + (src - s) * stride, v);
    F[dst] = 0.0;
  }
}

// c2p transposed at owned cells: cons = f(prim, Btilde, Gamma) at the recovered state, so
// prim_bar -> lambda = J_prim^{-T} prim_bar, cons_bar += lambda, Btilde_bar -= J_B^T lambda,
// Gamma_bar -= J_Gamma^T lambda.  Atmosphere cells (constant primitives) pass nothing.
struct C2PAdjArgs {
  const double* metric;
  const double* prim;
  const double* bc;
  const uint8_t* flags;
  const double* pbar;
  double* consbar;
  double* bcbar;
  double* gbar;
  double gam;
  int mode;  // 0: c2p (solve with J_prim^T), 1: prim -> cons (multiply by J^T)
};

DEV void c2p_adj_body(const GD& g, const C2PAdjArgs& ca, TileLDS2& S2, unsigned tile) {
  const TileCell t = tile_cell(g, tile);
  const TileIdx x = tile_index(g, t);
  double m[10];
  metric_values10(g, ca.metric, x, m, S2);
  double gsum = 0.0;
  if (t.valid) {
    const int id = at(g, t.i0 + t.cx, t.j0 + t.cy, t.k0 + t.cz);
    double pb[5];
    bool any = false;
    for (int c = 0; c < 5; ++c) {
      pb[c] = ca.pbar[(size_t)c * g.N + id];
      any = any || pb[c] != 0.0;
    }
    bool atmo = ca.mode == 0 && ca.flags && (ca.flags[id] & 4u);
    if (any && !atmo) {
      Geo G;
      geo_from(m, G);
      double pr[5], Bt[3];
      for (int c = 0; c < 5; ++c) pr[c] = ca.prim[(size_t)c * g.N + id];
      for (int c = 0; c < 3; ++c) Bt[c] = ca.bc[(size_t)c * g.N + id];
      double J[5][9];
      for (int dir = 0; dir < 9; ++dir) {
        Dual pd[5], bd[3];
        for (int c = 0; c < 5; ++c) pd[c] = Dual(pr[c], dir == c ? 1.0 : 0.0);
        for (int c = 0; c < 3; ++c) bd[c] = Dual(Bt[c], dir == 5 + c ? 1.0 : 0.0);
        Dual gd(ca.gam, dir == 8 ? 1.0 : 0.0);
        StateT<Dual> S;
        state_make(G, pd, bd, gd, S, gd / (gd - 1.0));
        Dual U[5];
        cons_of(G, S, U);
        for (int c = 0; c < 5; ++c) J[c][dir] = U[c].d;
      }
      double lam[5];
      if (ca.mode == 0) {
        // solve J_prim^T lam = pb (Gaussian elimination with partial pivoting)
        double M[5][6];
        for (int r = 0; r < 5; ++r) {
          for (int c = 0; c < 5; ++c) M[r][c] = J[c][r];
          M[r][5] = pb[r];
        }
        // partial pivoting by row swaps with fixed indices (the first largest |M[r][c]|, r >= c, ends
        // in row c), so that M stays in registers
#pragma unroll
        for (int c = 0; c < 5; ++c) {
#pragma unroll
          for (int r = c + 1; r < 5; ++r) {
            const bool sw = fabs(M[r][c]) > fabs(M[c][c]);
#pragma unroll
            for (int q = c; q < 6; ++q) {
              const double a = M[c][q], b = M[r][q];
              M[c][q] = sw ? b : a;
              M[r][q] = sw ? a : b;
            }
          }
          const double inv = 1.0 / M[c][c];
#pragma unroll
          for (int r = c + 1; r < 5; ++r) {
            const double f = M[r][c] * inv;
#pragma unroll
            for (int q = c; q < 6; ++q) M[r][q] -= f * M[c][q];
          }
        }
#pragma unroll
        for (int r = 4; r >= 0; --r) {
          double s = M[r][5];
#pragma unroll
          for (int q = r + 1; q < 5; ++q) s -= M[r][q] * lam[q];
          lam[r] = s / M[r][r];
        }
        for (int c = 0; c < 5; ++c) ca.consbar[(size_t)c * g.N + id] += lam[c];
        for (int b = 0; b < 3; ++b) {
          double s = 0.0;
          for (int c = 0; c < 5; ++c) s += J[c][5 + b] * lam[c];
          ca.bcbar[(size_t)b * g.N + id] -= s;
        }
        double s = 0.0;
        for (int c = 0; c < 5; ++c) s += J[c][8] * lam[c];
        gsum = -s;
      } else {
        // cons = f(prim, B, Gamma): prim_bar' += J_prim^T cons_bar (pbar holds cons_bar here)
        for (int r = 0; r < 5; ++r) {
          double s = 0.0;
          for (int c = 0; c < 5; ++c) s += J[c][r] * pb[c];
          ca.consbar[(size_t)r * g.N + id] += s;  // consbar holds prim_bar in this mode
        }
        for (int b = 0; b < 3; ++b) {
          double s = 0.0;
          for (int c = 0; c < 5; ++c) s += J[c][5 + b] * pb[c];
          ca.bcbar[(size_t)b * g.N + id] += s;
        }
        double s = 0.0;
        for (int c = 0; c < 5; ++c) s += J[c][8] * pb[c];
        gsum = s;
      }
    }
  }
  double w = gsum;
  for (int o = 32; o >= 1; o >>= 1) w += __shfl_xor(w, o, 64);
  if (__lane_id() == 0 && w != 0.0) atomicAdd(ca.gbar + (blockIdx.x & (GSLOTS - 1)), w);
}

// Centre-field cotangents to face-field cotangents (gather over the two adjacent cells),
// faces [-ng+1, n+ng]^3.
DEV void bcface_adj_body(const GD& g, const double* __restrict__ bcbar, double* __restrict__ bfbar, unsigned tile) {
  // faces [-ng, n+ng]^3: the centre of cell c (in [-ng, n+ng-1]) averages faces c and c + e_d
  int e[3] = {g.n[0] + 2 * g.ng + 1, g.n[1] + 2 * g.ng + 1, g.n[2] + 2 * g.ng + 1};
  int p, q, r;
  if (!box_at<64, 4>(e, tile, threadIdx.x, p, q, r)) return;
  const int i = p - g.ng, j = q - g.ng, k = r - g.ng;
  const int id = at(g, i, j, k);
  const int st[3] = {1, g.sy, g.sz};
  const int ijk[3] = {i, j, k};
  for (int d = 0; d < 3; ++d) {
    double s = 0.0;
    if (ijk[d] <= g.n[d] + g.ng - 1) s += 0.5 * bcbar[(size_t)d * g.N + id];
    if (ijk[d] - 1 >= -g.ng) s += 0.5 * bcbar[(size_t)d * g.N + id - st[d]];
    bfbar[(size_t)d * g.N + id] += s;
  }
}

// Face-field cotangents to the edge potential (transposed curl, gather), edges [-ng, n+ng]^3
// (a face f feeds the edges f and f + e_t of its two transverse directions t).
DEV void curlT_body(const GD& g, const double* __restrict__ bf, double* __restrict__ abar, unsigned tile) {
  int e[3] = {g.n[0] + 2 * g.ng + 1, g.n[1] + 2 * g.ng + 1, g.n[2] + 2 * g.ng + 1};
  int p, q, r;
  if (!box_at<64, 4>(e, tile, threadIdx.x, p, q, r)) return;
  const int i = p - g.ng, j = q - g.ng, k = r - g.ng;
  const int id = at(g, i, j, k);
  const double* Bx = bf;
  const double* By = bf + g.N;
  const double* Bz = bf + 2 * g.N;
  const int sy = g.sy, sz = g.sz;
  const bool im = i > -g.ng, jm = j > -g.ng, km = k > -g.ng;  // the face below exists
  auto F = [](const double* f, int o, bool ok) { return ok ? f[o] : 0.0; };
  abar[id] += (F(By, id - sz, km) - By[id]) * g.idx[2] + (Bz[id] - F(Bz, id - sy, jm)) * g.idx[1];
  abar[g.N + id] += (Bx[id] - F(Bx, id - sz, km)) * g.idx[2] + (F(Bz, id - 1, im) - Bz[id]) * g.idx[0];
  abar[2 * g.N + id] += (F(Bx, id - sy, jm) - Bx[id]) * g.idx[1] + (By[id] - F(By, id - 1, im)) * g.idx[0];
}

// dst[owned] += src[owned] for nf fields.
struct AccumArgs {
  const double* src;
  double* dst;
  int nf;
};

DEV void accum_body(const GD& g, const AccumArgs& a, unsigned tile) {
  int i, j, k;
  if (!box_at<64, 4>(g.n, tile, threadIdx.x, i, j, k)) return;
  const int id = at(g, i, j, k);
  for (int f = 0; f < a.nf; ++f) a.dst[(size_t)f * g.N + id] += a.src[(size_t)f * g.N + id];
}

template <class T>
DEV void copy_body(const GD& g, const T* __restrict__ src, T* __restrict__ dst, long long n, unsigned tile) {
  long long t = (long long)tile * 256 + threadIdx.x;
  if (t < n) dst[t] = src[t];
}

__global__ __launch_bounds__(256) void k_fluxbar(GD g, FluxBarArgs a) { fluxbar_body(g, a, my_tile()); }
// At the 2-wave floor (256 registers) the kernel spills 24-32 doubles per lane (PPM, WENO-Z, MP5)
// yet hides more latency: one wavefront per SIMD leaves every load and FP64 dependency chain exposed.
template <int D, int R>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_face_adj(GD g, FaceAdjArgs fa) {
  face_adj_body<D, R>(g, fa, my_tile());
}
template <int D, int R>
__global__ __launch_bounds__(64) void k_recon_adj(GD g, FaceAdjArgs fa) {
  __shared__ double L[D == 0 ? 5 : 1][64];
  recon_adj_wave<D, R>(g, fa, my_tile(), L);
}
__global__ __launch_bounds__(256) void k_cell_adj(GD g, CellAdjArgs ca) {
  __shared__ CellLDS S;
  cell_adj_body(g, ca, S, my_tile());
}
__global__ __launch_bounds__(256) void k_vertex_adj(GD g, VertexAdjArgs va) { vertex_adj_body(g, va, my_tile()); }
__global__ __launch_bounds__(256) void k_edge_adj(GD g, const double* avbar, double* abar) {
  edge_adj_body(g, avbar, abar, my_tile());
}
__global__ __launch_bounds__(256) void k_fillT(GD g, FillTArgs a) { fillT_body(g, a, blockIdx.x); }
__global__ __launch_bounds__(256) void k_c2p_adj(GD g, C2PAdjArgs ca) {
  __shared__ TileLDS2 S2;
  c2p_adj_body(g, ca, S2, my_tile());
}
__global__ __launch_bounds__(64) void k_gslots(const double* slots, double* gamma_bar) { gslots_body(slots, gamma_bar); }
__global__ __launch_bounds__(256) void k_bcface_adj(GD g, const double* bcbar, double* bfbar) {
  bcface_adj_body(g, bcbar, bfbar, my_tile());
}
__global__ __launch_bounds__(256) void k_curlT(GD g, const double* bf, double* abar) { curlT_body(g, bf, abar, my_tile()); }
__global__ __launch_bounds__(256) void k_accum(GD g, AccumArgs a) { accum_body(g, a, my_tile()); }
__global__ __launch_bounds__(256) void k_copy(GD g, const double* src, double* dst, long long n) {
  copy_body(g, src, dst, n, blockIdx.x);
}

__global__ void k_zero(double* p, long long n) {
  long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) p[t] = 0.0;
}

// ---------------------------------------------------------------------------------------
int check_grid(const asterx_grid* g, int min_ng) {
  if (!g) return fail(ASTERX_EARG, "grid is NULL");
  for (int a = 0; a < 3; ++a) {
    if (g->n[a] < 1) return fail(ASTERX_EARG, "grid: n must be >= 1");
    if (g->ld[a] < g->n[a] + 2 * g->ng + 1) return fail(ASTERX_EARG, "grid: ld must be >= n + 2 ng + 1");
    if (!(g->dx[a] > 0.0)) return fail(ASTERX_EARG, "grid: dx must be > 0");
  }
  if (g->ng < min_ng) return fail(ASTERX_EARG, "grid: too few ghost layers for this stencil");
  double npts = (double)g->ld[0] * g->ld[1] * g->ld[2];
  if (npts >= 536870912.0) return fail(ASTERX_EARG, "grid: ld[0]*ld[1]*ld[2] must be below 2^29");
  return 0;
}

int check_params(const asterx_params* p) {
  if (!p) return fail(ASTERX_EARG, "params is NULL");
  if (!(p->gamma > 1.0)) return fail(ASTERX_EARG, "params: gamma must be > 1");
  if (p->recon < 0 || p->recon > 3) return fail(ASTERX_EARG, "params: unknown reconstruction");
  if (p->riemann < 0 || p->riemann > 1) return fail(ASTERX_EARG, "params: unknown Riemann solver");
  if (p->ct < 0 || p->ct > 1) return fail(ASTERX_EARG, "params: unknown electric-field scheme");
  if (p->gauge < 0 || p->gauge > 1) return fail(ASTERX_EARG, "params: unknown gauge");
  if (p->speeds < 0 || p->speeds > 1) return fail(ASTERX_EARG, "params: unknown speed estimate");
  if (p->c2p_method < 0 || p->c2p_method > 2) return fail(ASTERX_EARG, "params: unknown c2p method");
  if (!(p->wmax > 1.0)) return fail(ASTERX_EARG, "params: wmax must be > 1");
  if (p->c2p_maxit < 1 || p->brent_maxit < 1) return fail(ASTERX_EARG, "params: iteration caps must be >= 1");
  if (!(p->rho_atm >= 0.0)) return fail(ASTERX_EARG, "params: rho_atm must be >= 0");
  return 0;
}

int launched() {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    g_err = std::string("launch failed: ") + hipGetErrorString(e);
    return ASTERX_ELAUNCH;
  }
  return 0;
}

// ---------------------------------------------------------------------------------------
// Optional per-kernel timing: when enabled, every launch is bracketed by two HIP events on
// its own stream; asterx_timing_read waits for them and accumulates elapsed times.  Not for
// use while a stream is being captured into a graph.
enum {
  KT_PRIM2CON, KT_C2P, KT_FILL, KT_BCENT, KT_FACE_X, KT_FACE_Y, KT_FACE_Z, KT_CELL, KT_VERTEX, KT_EDGE, KT_RK,
  KT_ZERO, KT_ADJ, KT_TMUNU, KT_INTER, KT_GEOM, KT_FACES, KT_BCENT_VERTEX, KT_DIV_EDGE, KT_N
};
const char* const kt_names[KT_N] = {"prim2con", "c2p", "fill_ghosts", "centre_B", "face_x", "face_y",
                                    "face_z", "cell", "vertex", "edge", "rk_stage", "zero", "adjoint", "tmunu",
                                    "inter_level", "geometry", "faces", "centre_B+vertex", "divergence+edge"};
struct Pending {
  hipEvent_t a, b;
  int kind;
};
bool g_timing = false;
std::vector<Pending> g_pending;
std::vector<hipEvent_t> g_free_events;
double g_ms[KT_N];
long long g_count[KT_N];

hipEvent_t take_event() {
  if (!g_free_events.empty()) {
    hipEvent_t e = g_free_events.back();
    g_free_events.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

template <class F>
int timed(int kind, hipStream_t s, F&& launch) {
  if (!g_timing) {
    launch();
    return launched();
  }
  hipEvent_t a = take_event(), b = take_event();
  bool ok = a && b && hipEventRecord(a, s) == hipSuccess;
  launch();
  int rc = launched();
  ok = ok && hipEventRecord(b, s) == hipSuccess;
  if (ok) {
    g_pending.push_back(Pending{a, b, kind});
  } else {
    if (a) g_free_events.push_back(a);
    if (b) g_free_events.push_back(b);
  }
  return rc;
}

// ---------------------------------------------------------------------------------------
// Launch targets.  A single block launches one workgroup per tile of each phase; a batch
// of patches launches a persistent grid over that phase's (patch, tile) work list.
enum { PH_P2C, PH_C2P, PH_FILL, PH_BCENT, PH_FACEX, PH_FACEY, PH_FACEZ, PH_CELL, PH_VERTEX, PH_EDGE,
       PH_RK, PH_GEOM, PH_N };

unsigned host_tile_blocks(const GD& g) {
  return (unsigned)(((g.n[0] + CTX - 1) / CTX) * ((g.n[1] + CTY - 1) / CTY) * ((g.n[2] + CTZ - 1) / CTZ));
}

// rows: faces per march along y and z in a batch (single blocks choose their own).
unsigned tiles_for(int phase, const GD& g, const int* rows = nullptr) {
  int e[3];
  switch (phase) {
    case PH_C2P:
    case PH_CELL:
      return host_tile_blocks(g);
    case PH_BCENT:
      for (int a = 0; a < 3; ++a) e[a] = g.n[a] + 2 * g.ng;
      return lin_blocks(e);
    case PH_FILL: {
      const long long G = 2 * g.ng + 1, E1 = g.n[1] + 2 * g.ng + 1, E2 = g.n[2] + 2 * g.ng + 1;
      const long long cnt = G * E1 * E2 + (long long)g.n[0] * G * E2 + (long long)g.n[0] * g.n[1] * G;
      return (unsigned)((cnt + 255) / 256);
    }
    case PH_FACEX:
    case PH_FACEY:
    case PH_FACEZ:
      return face_items(g.n, phase - PH_FACEX, 1, rows[phase - PH_FACEX]);
    case PH_GEOM:  // of one component
      return geom_items(g, 1, 10, geom_rows<GM_Z>());
    case PH_VERTEX:
      for (int a = 0; a < 3; ++a) e[a] = g.n[a] + 2;
      return lin_blocks(e);
    default:
      return box_blocks<64, 4>(g.n);
  }
}

}  // namespace

struct asterx_batch {
  int np = 0;
  long long ntot = 0;
  int blocks = 0;
  std::vector<GD> gds;
  std::vector<long long> off;
  PatchDesc* d_patches = nullptr;
  Item* d_items[PH_N] = {};
  int nitems[PH_N] = {};
  int rows[3] = {1, 1, 1};  // faces per march along each direction
};

namespace {

unsigned bgrid(const asterx_batch* b, int phase) {
  return (unsigned)(b->nitems[phase] < b->blocks ? b->nitems[phase] : b->blocks);
}

// One phase on either target: KS(g, args...) one workgroup per tile, or
// KB(patches, items, nitems, args...) persistent over the batch's work list.
#define RUN_PHASE(KT, PHASE, KS, KB, ...)                                                                     \
  (b ? (b->nitems[PHASE] ? timed(KT, s,                                                                      \
                                 [&] {                                                                       \
                                   hipLaunchKernelGGL(KB, dim3(bgrid(b, PHASE)), dim3(256), 0, s,           \
                                                      b->d_patches, b->d_items[PHASE], b->nitems[PHASE],     \
                                                      __VA_ARGS__);                                          \
                                 })                                                                          \
                         : 0)                                                                                \
     : timed(KT, s, [&] { hipLaunchKernelGGL(KS, dim3(tiles_for(PHASE, g)), dim3(256), 0, s, g, __VA_ARGS__); }))

// Phases whose items are wavefronts: single blocks launch workgroups of one wavefront (count of them), batches
// persistent workgroups of four whose wavefronts walk the work list.
#define RUN_WAVES(KT, PHASE, COUNT, KS, KB, ...)                                                              \
  (b ? (b->nitems[PHASE] ? timed(KT, s,                                                                      \
                                 [&] {                                                                       \
                                   const int nw = (b->nitems[PHASE] + 3) / 4;                                \
                                   hipLaunchKernelGGL(KB, dim3(nw < b->blocks ? nw : b->blocks), dim3(256), 0, s, \
                                                      b->d_patches, b->d_items[PHASE], b->nitems[PHASE],     \
                                                      __VA_ARGS__);                                          \
                                 })                                                                          \
                         : 0)                                                                                \
     : timed(KT, s, [&] { hipLaunchKernelGGL(KS, dim3(COUNT), dim3(64), 0, s, g, __VA_ARGS__); }))

template <int D, int R>
int face_launch(const GD& g, const asterx_batch* b, FaceArgs fa, bool uct, hipStream_t s) {
  const int lo = uct ? 3 : 1;
  fa.rows[D] = b ? b->rows[D] : face_rows(g.n, D, lo, face_march<R>());
  const unsigned count = b ? 0 : face_items(g.n, D, lo, fa.rows[D]);
  if (uct) return timed(KT_FACE_X + D, s, [&] { hipLaunchKernelGGL((k_face<D, R, true>), dim3(count), dim3(64), 0, s, g, fa); });
  return RUN_WAVES(KT_FACE_X + D, PH_FACEX + D, count, (k_face<D, R, false>), (kb_face<D, R>), fa);
}

template <int D>
int faces(const GD& g, const asterx_batch* b, const FaceArgs& fa, bool uct, hipStream_t s) {
  if (fa.recon == ASTERX_RECON_MINMOD) return face_launch<D, ASTERX_RECON_MINMOD>(g, b, fa, uct, s);
  if (fa.recon == ASTERX_RECON_PPM) return face_launch<D, ASTERX_RECON_PPM>(g, b, fa, uct, s);
  if (fa.recon == ASTERX_RECON_MP5) return face_launch<D, ASTERX_RECON_MP5>(g, b, fa, uct, s);
  return face_launch<D, ASTERX_RECON_WENOZ>(g, b, fa, uct, s);
}

// The first nd directions in one launch: no direction waits for another's last wavefronts.  RK4 steps from a graph
// with stored geometry, the directions apart and in one launch: 32^3, PPM, 0.275 and 0.203 ms; 64^3 0.798 and 0.709;
// 96^3 2.276 and 2.188; 128^3 5.018 and 4.925; 192^3 15.82 and 15.78; 64^3, MP5, upwind CT, 1.098 and 0.978.
template <int R>
int faces_joint(const GD& g, FaceArgs fa, bool uct, hipStream_t s, int nd) {
  const int lo = uct ? 3 : 1;
  unsigned c[3];
  for (int d = 0; d < 3; ++d) {
    fa.rows[d] = face_rows(g.n, d, lo, face_march<R>());
    c[d] = d < nd ? face_items(g.n, d, lo, fa.rows[d]) : 0;
  }
  return timed(KT_FACES, s, [&] {
    const dim3 all(c[0] + c[1] + c[2]);
    if (uct) hipLaunchKernelGGL((k_faces<R, true>), all, dim3(64), 0, s, g, fa, c[0], c[1]);
    else hipLaunchKernelGGL((k_faces<R, false>), all, dim3(64), 0, s, g, fa, c[0], c[1]);
  });
}
int first_faces(const GD& g, const FaceArgs& fa, bool uct, hipStream_t s, int nd) {
  if (fa.recon == ASTERX_RECON_MINMOD) return faces_joint<ASTERX_RECON_MINMOD>(g, fa, uct, s, nd);
  if (fa.recon == ASTERX_RECON_PPM) return faces_joint<ASTERX_RECON_PPM>(g, fa, uct, s, nd);
  if (fa.recon == ASTERX_RECON_MP5) return faces_joint<ASTERX_RECON_MP5>(g, fa, uct, s, nd);
  return faces_joint<ASTERX_RECON_WENOZ>(g, fa, uct, s, nd);
}

// Whether a block without stored geometry gathers its face metric instead of interpolating it into the workspace
// first: then nothing waits for the interpolation, all directions and the centre field with the gauge quantities share
// launches, but every face reads 160 values.  Small blocks are bound by the launches, large ones by those reads: the
// line is at a count of faces (asterx_rhs from a graph, interpolated and gathered: PPM, 24^3, 73 and 56 us; 64^3 187
// and 172; 88^3, 2.12e6 faces, 444 and 428; 96^3, 2.74e6, 557 and 562; 128^3 1253 and 1385; upwind CT, PPM, 80^3,
// 1.76e6, 397 and 389; 88^3, 2.31e6, 526 and 525; 400 x 200 x 6, 2.38e6, 484 and 505; MINMOD, whose faces cost less
// beside the reads, 64^3, 0.82e6, 169 and 166; 80^3, 1.59e6, 307 and 315; 128^3 1174 and 1433).
bool face_gather(const GD& g, const asterx_params* p) {
  const int lo = p->ct == ASTERX_CT_UCT ? 3 : 1;
  long long e[3], f[3];
  for (int a = 0; a < 3; ++a) {
    e[a] = g.n[a] + 2 * lo - 1;
    f[a] = g.n[a] + 1;
  }
  const long long faces = f[0] * e[1] * e[2] + e[0] * f[1] * e[2] + e[0] * e[1] * f[2];
  return faces <= (p->recon == ASTERX_RECON_MINMOD ? 5LL << 18 : 9LL << 18);
}

// Interpolated spacetime data of the sets in MASK.
template <int MASK>
int geometry(const GD& g, const asterx_batch* b, GeomArgs ga, hipStream_t s) {
  int e[3];
  geom_box(g.n, ga.lo, e);
  ga.zl = geom_planes(e);
  return RUN_WAVES(KT_GEOM, PH_GEOM, geom_items(g, ga.lo, (MASK & GM_C) ? 16 : 10, geom_rows<MASK>()), (k_geom<MASK>), (kb_geom<MASK>), ga);
}

// ---- the phases, shared by the single-block and the batched entry points ----
int do_prim2con(const GD& g, const asterx_batch* b, const asterx_params* p, const double* metric, const double* A,
                const double* prim, double* cons, hipStream_t s) {
  return RUN_PHASE(KT_PRIM2CON, PH_P2C, k_prim2con, kb_prim2con, p->gamma, metric, A, prim, cons);
}

int do_c2p(const GD& g, const asterx_batch* b, const asterx_params* p, const double* metric, const double* A,
           double* cons, double* prim, uint8_t* flags, asterx_c2p_stats* stats, hipStream_t s) {
  C2PParams cp = make_c2p_params(p);
  C2PArgs a{metric, A, cons, prim, flags, (unsigned long long*)stats, nullptr, {}};
  return RUN_PHASE(KT_C2P, PH_C2P, k_c2p, kb_c2p, cp, a);
}

int do_c2p_learned(const GD& g, const asterx_params* p, const double* metric, const double* A, double* cons,
                   double* prim, uint8_t* flags, asterx_c2p_stats* stats, const float* mlp, const mlpd::Stdz& z,
                   hipStream_t s) {
  C2PParams cp = make_c2p_params(p);
  C2PArgs a{metric, A, cons, prim, flags, (unsigned long long*)stats, mlp, z};
  return timed(KT_C2P, s, [&] {
    hipLaunchKernelGGL(k_c2p_learned, dim3(tiles_for(PH_C2P, g)), dim3(256), 0, s, g, cp, a);
  });
}

int do_c2p_src(const GD& g, const asterx_params* p, const double* metric, const double* curv, const double* A,
               double* cons, double* prim, uint8_t* flags, asterx_c2p_stats* stats, const float* mlp,
               const mlpd::Stdz& z, double* src, hipStream_t s) {
  C2PParams cp = make_c2p_params(p);
  C2PArgs a{metric, A, cons, prim, flags, (unsigned long long*)stats, mlp, z, curv, src};
  return timed(KT_C2P, s, [&] {
    if (mlp)
      hipLaunchKernelGGL(k_c2p_learned_src, dim3(tiles_for(PH_C2P, g)), dim3(256), 0, s, g, cp, a);
    else
      hipLaunchKernelGGL(k_c2p_src, dim3(tiles_for(PH_C2P, g)), dim3(256), 0, s, g, cp, a);
  });
}

// The network's standardisation from an asterx_mlp (scales must be positive).
int make_stdz(const asterx_mlp* mlp, mlpd::Stdz& z, const char* who) {
  for (int k = 0; k < mlpd::NI; ++k) {
    if (!(mlp->in_scale[k] > 0.0f)) return fail(ASTERX_EARG, (std::string(who) + ": network scales must be > 0").c_str());
    z.is[k] = mlp->in_shift[k];
    z.isc[k] = mlp->in_scale[k];
  }
  for (int k = 0; k < mlpd::NO; ++k) {
    if (!(mlp->out_scale[k] > 0.0f)) return fail(ASTERX_EARG, (std::string(who) + ": network scales must be > 0").c_str());
    z.os[k] = mlp->out_shift[k];
    z.osc[k] = 1.0f / mlp->out_scale[k];
  }
  return 0;
}

int run_fill(const GD& g, const asterx_batch* b, const FillArgs& fa, hipStream_t s) {
  bool lin = false;
  for (int q = 0; q < fa.ngroup; ++q)
    for (int a = 0; a < 3; ++a) lin = lin || fa.kind[q][a] == ASTERX_BC_LINEAR;
  if (lin) return RUN_PHASE(KT_FILL, PH_FILL, k_fill<true>, kb_fill<true>, fa);
  return RUN_PHASE(KT_FILL, PH_FILL, k_fill<false>, kb_fill<false>, fa);
}

int do_fill(const GD& g, const asterx_batch* b, double* f, int nf, const int32_t* kinds, hipStream_t s,
            const double* shift = nullptr) {
  FillArgs fa{};
  fa.f = f;
  fa.ngroup = 1;
  fa.end[0] = nf;
  for (int a = 0; a < 3; ++a) fa.kind[0][a] = kinds[a];
  fa.shifted = shift ? 0 : -1;
  if (shift)
    for (int q = 0; q < 3 && q < nf; ++q)
      for (int a = 0; a < 3; ++a) fa.shift[q][a] = shift[q * 3 + a];
  return run_fill(g, b, fa, s);
}

// A state's nine fields: the conserved variables and Psi by kinds_cell, the potential by kinds_A or, with shift,
// periodic with an offset per wrap.
int do_fill_state(const GD& g, const asterx_batch* b, double* u, const int32_t* kinds_cell, const int32_t* kinds_A,
                  const double* shift, hipStream_t s) {
  FillArgs fa{};
  fa.f = u;
  fa.ngroup = 3;
  fa.end[0] = 5;
  fa.end[1] = 8;
  fa.end[2] = 9;
  for (int a = 0; a < 3; ++a) {
    fa.kind[0][a] = fa.kind[2][a] = kinds_cell[a];
    fa.kind[1][a] = shift ? ASTERX_BC_PERIODIC : kinds_A[a];
  }
  fa.shifted = shift ? 1 : -1;
  if (shift)
    for (int q = 0; q < 3; ++q)
      for (int a = 0; a < 3; ++a) fa.shift[q][a] = shift[q * 3 + a];
  return run_fill(g, b, fa, s);
}

int do_bcent(const GD& g, const double* A, double* bc, hipStream_t s) {
  const asterx_batch* b = nullptr;
  return RUN_PHASE(KT_BCENT, PH_BCENT, k_bcent, kb_bcent, A, bc);
}

// src (single blocks): densitized sources stored by a recovery with sources; the cell phase is
// then the divergence kernel instead of the cell kernel.  The face metric comes from geo (all directions,
// as stored by asterx_geometry), for x faces from xfm (as stored by asterx_c2p_src), is gathered by the faces
// (face_gather), or is interpolated here into parts of the workspace that hold nothing at that time: the fluxes of
// directions not yet done, the gauge quantities (written after the faces) and, under flux CT, the nine fields of
// upwind CT.  Phases of a single block that don't depend on each other share launches.
int do_rhs(const GD& g, const asterx_batch* b, const asterx_params* p, const double* metric, const double* curv,
           const double* prim, const double* A, const double* psi, double dt_max, double* rhs, double* red,
           double* ws, hipStream_t s, const Combine& cmb = Combine{}, const double* src = nullptr,
           const double* xfm = nullptr, const double* geo = nullptr) {
  int rc;
  double* bc = ws;
  double* flux = ws + 3 * g.N;
  double* ga = ws + 24 * g.N;
  double* fp = ws + 25 * g.N;
  double* apm = ws + 28 * g.N;
  const bool uct = p->ct == ASTERX_CT_UCT, lorenz = p->gauge == ASTERX_GAUGE_LORENZ;
  const bool gather = !b && !geo && face_gather(g, p);
  const bool staged = !geo && !gather;  // the workspace holds face metric until the faces are done
  const VertexArgs va{metric, A, psi, ga, fp};
  const bool gauge_first = lorenz && !b && !staged;
  if (gauge_first) {
    const unsigned n0 = tiles_for(PH_BCENT, g), n1 = tiles_for(PH_VERTEX, g);
    rc = timed(KT_BCENT_VERTEX, s, [&] {
      hipLaunchKernelGGL(k_bcent_vertex, dim3(n0 + n1), dim3(256), 0, s, g, A, bc, va, n0);
    });
  } else {
    rc = RUN_PHASE(KT_BCENT, PH_BCENT, k_bcent, kb_bcent, A, bc);
  }
  if (rc) return rc;
  FaceArgs fa{metric, prim, A, bc, flux, red, p->gamma, p->weno_eps, p->weno_q, p->gamma / (p->gamma - 1.0),
              p->recon, p->speeds, p->riemann, apm, {nullptr, nullptr, nullptr}, {nullptr, nullptr, nullptr}, {1, 1, 1}, false};
  GeomArgs gm{metric, nullptr, {nullptr, nullptr, nullptr}, {nullptr, nullptr, nullptr}, nullptr, uct ? 3 : 1, 0};
  auto put = [&](int d, int f0, int f1) {  // components 0..6 into workspace fields from f0, 7..9 from f1
    gm.fa[d] = ws + (size_t)f0 * g.N;
    gm.fb[d] = ws + (size_t)f1 * g.N;
    fa.fma[d] = gm.fa[d];
    fa.fmb[d] = gm.fb[d];
  };
  if (xfm && !uct) {
    fa.xown = true;
    fa.fma[0] = xfm;
    fa.fmb[0] = xfm + 7 * g.N;
  }
  // workspace fields: x fluxes 3..9, y 10..16, z 17..23, gauge 24..27, upwind CT 28..30 (x), 31..33 (y), 34..36 (z)
  bool later_z = false;
  if (geo) {
    for (int d = 0; d < 3; ++d) {
      fa.fma[d] = geo + (size_t)(10 * d) * g.N;
      fa.fmb[d] = fa.fma[d] + 7 * g.N;
    }
  } else if (gather) {
  } else if (uct) {
    put(0, 10, 17);
    put(1, 20, 34);
    if ((rc = geometry<GM_X | GM_Y>(g, b, gm, s))) return rc;  // z faces gather theirs: no ten fields are free then
  } else if (xfm) {
    put(1, 17, 34);
    put(2, 24, 31);
    if ((rc = geometry<GM_Y | GM_Z>(g, b, gm, s))) return rc;
  } else {
    put(0, 24, 31);
    put(1, 17, 34);
    later_z = true;
    if ((rc = geometry<GM_X | GM_Y>(g, b, gm, s))) return rc;
  }
  if (!b && !staged) {
    if ((rc = first_faces(g, fa, uct, s, 3))) return rc;
  } else {
    // x and y faces share a launch where neither's output lies over the other's metric
    if (!b && !uct) {
      if ((rc = first_faces(g, fa, uct, s, 2))) return rc;
    } else {
      if ((rc = faces<0>(g, b, fa, uct, s))) return rc;
      if ((rc = faces<1>(g, b, fa, uct, s))) return rc;
    }
    if (later_z) {
      put(2, 24, 31);
      if ((rc = geometry<GM_Z>(g, b, gm, s))) return rc;
    }
    if ((rc = faces<2>(g, b, fa, uct, s))) return rc;
  }
  EdgeArgs ea{metric, psi, flux, ga, fp, rhs, p->xi / dt_max, p->gauge, cmb, apm};
  auto gauge = [&] { return RUN_PHASE(KT_VERTEX, PH_VERTEX, k_vertex, kb_vertex, va); };
  if (src) {
    if (lorenz && !gauge_first && (rc = gauge())) return rc;
    const DivArgs da{src, flux, A, rhs, red, cmb};
    const unsigned n0 = box_blocks<64, 4>(g.n), n1 = tiles_for(PH_EDGE, g);
    return timed(KT_DIV_EDGE, s, [&] {
      if (uct) hipLaunchKernelGGL(k_div_edge<true>, dim3(n0 + n1), dim3(256), 0, s, g, da, ea, n0);
      else hipLaunchKernelGGL(k_div_edge<false>, dim3(n0 + n1), dim3(256), 0, s, g, da, ea, n0);
    });
  }
  CellArgs ca{metric, curv, prim, A, bc, flux, rhs, red, p->gamma, cmb};
  if ((rc = RUN_PHASE(KT_CELL, PH_CELL, k_cell, kb_cell, ca))) return rc;
  if (lorenz && !gauge_first && (rc = gauge())) return rc;
  if (uct)
    return timed(KT_EDGE, s, [&] {
      hipLaunchKernelGGL(k_edge_uct, dim3(tiles_for(PH_EDGE, g)), dim3(256), 0, s, g, ea);
    });
  return RUN_PHASE(KT_EDGE, PH_EDGE, k_edge, kb_edge, ea);
}

bool overlap(const void* a, size_t na, const void* b, size_t nb) {
  const char *pa = (const char*)a, *pb = (const char*)b;
  return a && b && pa < pb + nb && pb < pa + na;
}

// Checks of the stage outputs against the right-hand side's inputs and each other; npts is the
// per-field stride (the block's points, or a batch's pool).
int make_combine(int32_t nout, const asterx_rk_out* outs, size_t npts, const double* const* ins, const size_t* nin,
                 int nins, Combine& cmb) {
  if (nout < 1 || nout > 2 || !outs) return fail(ASTERX_EARG, "rhs_rk: nout must be 1 or 2");
  const size_t st = 9 * npts * sizeof(double);
  cmb = Combine{};
  cmb.nout = nout;
  for (int k = 0; k < nout; ++k) {
    const asterx_rk_out& o = outs[k];
    if (o.nterms < 1 || o.nterms > 2 || !o.out) return fail(ASTERX_EARG, "rhs_rk: bad output");
    for (int m = 0; m < o.nterms; ++m)
      if (!o.u[m]) return fail(ASTERX_EARG, "rhs_rk: NULL state");
    for (int i = 0; i < nins; ++i)
      if (overlap(o.out, st, ins[i], nin[i] * sizeof(double)))
        return fail(ASTERX_EARG, "rhs_rk: an output overlaps an input of the right-hand side");
    for (int m = 0; m < o.nterms; ++m)
      if (o.u[m] != o.out && overlap(o.out, st, o.u[m], st))
        return fail(ASTERX_EARG, "rhs_rk: an output partially overlaps one of its own states");
    for (int j = 0; j < nout; ++j) {
      if (j == k) continue;
      if (overlap(o.out, st, outs[j].out, st)) return fail(ASTERX_EARG, "rhs_rk: outputs overlap");
      for (int m = 0; m < outs[j].nterms; ++m)
        if (overlap(o.out, st, outs[j].u[m], st))
          return fail(ASTERX_EARG, "rhs_rk: an output overlaps a state the other output reads");
    }
    RKOut& r = cmb.o[k];
    r.nterms = o.nterms;
    r.b_dt = o.b_dt;
    r.out = o.out;
    for (int m = 0; m < 2; ++m) {
      r.u[m] = m < o.nterms ? o.u[m] : nullptr;
      r.a[m] = m < o.nterms ? o.a[m] : 0.0;
    }
  }
  return 0;
}

int do_rk(const GD& g, const asterx_batch* b, int32_t nterms, const double* a, const double* const* u, double b_dt,
          const double* rhs, double* out, hipStream_t s) {
  if (nterms < 1 || nterms > 4 || !a || !u || !rhs || !out) return fail(ASTERX_EARG, "rk_stage: bad arguments");
  RKArgs ra;
  for (int m = 0; m < 4; ++m) {
    ra.u[m] = m < nterms ? u[m] : nullptr;
    ra.a[m] = m < nterms ? a[m] : 0.0;
    if (m < nterms && !u[m]) return fail(ASTERX_EARG, "rk_stage: NULL state");
  }
  ra.nterms = nterms;
  ra.b_dt = b_dt;
  ra.rhs = rhs;
  ra.out = out;
  return RUN_PHASE(KT_RK, PH_RK, k_rk, kb_rk, ra);
}

int check_batch_kinds(const asterx_batch* b, const int32_t* kinds) {
  for (int a = 0; a < 3; ++a) {
    if (kinds[a] < 0 || kinds[a] > 2) return fail(ASTERX_EARG, "fill_ghosts: unknown boundary kind");
    for (int q = 0; q < b->np; ++q)
      if (kinds[a] == ASTERX_BC_LINEAR && b->gds[q].n[a] < 2)
        return fail(ASTERX_EARG, "fill_ghosts: LINEAR needs n >= 2");
  }
  return 0;
}

int check_kinds(const asterx_grid* gr, const int32_t* kinds) {
  for (int a = 0; a < 3; ++a) {
    if (kinds[a] < 0 || kinds[a] > 2) return fail(ASTERX_EARG, "fill_ghosts: unknown boundary kind");
    if (kinds[a] == ASTERX_BC_LINEAR && gr->n[a] < 2) return fail(ASTERX_EARG, "fill_ghosts: LINEAR needs n >= 2");
  }
  return 0;
}

}  // namespace

// =======================================================================================
namespace axh {
int set_error(int code, const char* msg) { return fail(code, msg); }
}  // namespace axh

// ---------------------------------------------------------------------------------------
// Library-held right-hand side workspace of asterx_rhs_rk_noalloc, for callers that cannot
// allocate.  Each device holds its own copy of the array until the process ends; host code
// reaches it only through the device address hipGetSymbolAddress returns with that device
// current (the array's name in host code is not a device address).  Every call on a device
// shares its copy, so calls that overlap on one device race.
static __device__ __align__(256) double scratch[ASTERX_NOALLOC_WS_BYTES / sizeof(double)];

namespace {
constexpr int SCRATCH_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[SCRATCH_MAX_DEVICES] = {};

// Device address of the current device's copy of `scratch`, looked up once per device.
int scratch_address(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return fail(ASTERX_ELAUNCH, "rhs_rk_noalloc: no current device");
  if (dev >= SCRATCH_MAX_DEVICES) return fail(ASTERX_EARG, "rhs_rk_noalloc: device index beyond 63");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) {
      g_err = std::string("rhs_rk_noalloc: hipGetSymbolAddress failed: ") + hipGetErrorString(e);
      return ASTERX_ELAUNCH;
    }
    g_scratch_dev[dev] = ptr;
  }
  *out = g_scratch_dev[dev];
  return 0;
}
}  // namespace

extern "C" {

int asterx_timing_enable(int32_t on) {
  g_timing = on != 0;
  return 0;
}

int asterx_timing_read(double* ms, long long* counts, int32_t n) {
  for (const Pending& p : g_pending) {
    float t = 0.f;
    if (hipEventSynchronize(p.b) == hipSuccess && hipEventElapsedTime(&t, p.a, p.b) == hipSuccess) {
      g_ms[p.kind] += t;
      g_count[p.kind] += 1;
    }
    g_free_events.push_back(p.a);
    g_free_events.push_back(p.b);
  }
  g_pending.clear();
  for (int k = 0; k < n && k < KT_N; ++k) {
    if (ms) ms[k] = g_ms[k];
    if (counts) counts[k] = g_count[k];
  }
  return KT_N;
}

int asterx_timing_reset(void) {
  asterx_timing_read(nullptr, nullptr, 0);
  for (int k = 0; k < KT_N; ++k) {
    g_ms[k] = 0.0;
    g_count[k] = 0;
  }
  return 0;
}

const char* asterx_timing_name(int32_t k) { return (k >= 0 && k < KT_N) ? kt_names[k] : ""; }

int asterx_version(void) { return 8; }

const char* asterx_last_error(void) { return g_err.c_str(); }

size_t asterx_rhs_workspace_size(const asterx_grid* g) {
  if (!g) return 0;
  size_t N = (size_t)g->ld[0] * g->ld[1] * g->ld[2];
  return (size_t)WS_FIELDS * N * sizeof(double);
}

int asterx_prim2con(const asterx_grid* gr, const asterx_params* p, const double* metric, const double* A,
                    const double* prim, double* cons, void* stream) {
  int rc;
  if ((rc = check_grid(gr, 2)) || (rc = check_params(p))) return rc;
  if (!metric || !A || !prim || !cons) return fail(ASTERX_EARG, "prim2con: NULL array");
  GD g = make_gd(gr);
  const asterx_batch* b = nullptr;
  return do_prim2con(g, b, p, metric, A, prim, cons, (hipStream_t)stream);
}

int asterx_c2p(const asterx_grid* gr, const asterx_params* p, const double* metric, const double* A, double* cons,
               double* prim, uint8_t* flags, asterx_c2p_stats* stats, void* stream) {
  int rc;
  if ((rc = check_grid(gr, 2)) || (rc = check_params(p))) return rc;
  if (!metric || !A || !prim || !cons) return fail(ASTERX_EARG, "c2p: NULL array");
  GD g = make_gd(gr);
  const asterx_batch* b = nullptr;
  return do_c2p(g, b, p, metric, A, cons, prim, flags, stats, (hipStream_t)stream);
}

int asterx_c2p_learned(const asterx_grid* gr, const asterx_params* p, const double* metric, const double* A,
                       double* cons, double* prim, uint8_t* flags, asterx_c2p_stats* stats, const asterx_mlp* mlp,
                       void* stream) {
  int rc;
  if ((rc = check_grid(gr, 2)) || (rc = check_params(p))) return rc;
  if (!metric || !A || !prim || !cons || !mlp || !mlp->params) return fail(ASTERX_EARG, "c2p_learned: NULL array");
  mlpd::Stdz z;
  if ((rc = make_stdz(mlp, z, "c2p_learned"))) return rc;
  GD g = make_gd(gr);
  return do_c2p_learned(g, p, metric, A, cons, prim, flags, stats, mlp->params, z, (hipStream_t)stream);
}

int asterx_c2p_src(const asterx_grid* gr, const asterx_params* p, const double* metric, const double* curv,
                   const double* A, double* cons, double* prim, uint8_t* flags, asterx_c2p_stats* stats,
                   const asterx_mlp* mlp, double* src, void* stream) {
  int rc;
  if ((rc = check_grid(gr, 2)) || (rc = check_params(p))) return rc;
  if (!metric || !curv || !A || !prim || !cons || !src) return fail(ASTERX_EARG, "c2p_src: NULL array");
  mlpd::Stdz z{};
  if (mlp) {
    if (!mlp->params) return fail(ASTERX_EARG, "c2p_src: NULL network parameters");
    if ((rc = make_stdz(mlp, z, "c2p_src"))) return rc;
  }
  GD g = make_gd(gr);
  return do_c2p_src(g, p, metric, curv, A, cons, prim, flags, stats, mlp ? mlp->params : nullptr, z, src,
                    (hipStream_t)stream);
}

int asterx_fill_ghosts(const asterx_grid* gr, double* f, int32_t nf, const int32_t* kinds, void* stream) {
  int rc;
  if ((rc = check_grid(gr, 1))) return rc;
  if (!f || !kinds || nf < 1) return fail(ASTERX_EARG, "fill_ghosts: bad arguments");
  if ((rc = check_kinds(gr, kinds))) return rc;
  GD g = make_gd(gr);
  const asterx_batch* b = nullptr;
  return do_fill(g, b, f, nf, kinds, (hipStream_t)stream);
}

int asterx_fill_state(const asterx_grid* gr, double* u, const int32_t* kinds_cell, const int32_t* kinds_A,
                      const double* shift, void* stream) {
  int rc;
  if ((rc = check_grid(gr, 1))) return rc;
  if (!u || !kinds_cell || (!kinds_A && !shift)) return fail(ASTERX_EARG, "fill_state: bad arguments");
  if ((rc = check_kinds(gr, kinds_cell)) || (!shift && (rc = check_kinds(gr, kinds_A)))) return rc;
  const asterx_batch* b = nullptr;
  return do_fill_state(make_gd(gr), b, u, kinds_cell, kinds_A, shift, (hipStream_t)stream);
}

int asterx_fill_ghosts_shift(const asterx_grid* gr, double* f, int32_t nf, const double* shift, void* stream) {
  int rc;
  if ((rc = check_grid(gr, 1))) return rc;
  if (!f || !shift || nf < 1 || nf > 3) return fail(ASTERX_EARG, "fill_ghosts_shift: bad arguments");
  GD g = make_gd(gr);
  const asterx_batch* b = nullptr;
  const int32_t per[3] = {ASTERX_BC_PERIODIC, ASTERX_BC_PERIODIC, ASTERX_BC_PERIODIC};
  return do_fill(g, b, f, nf, per, (hipStream_t)stream, shift);
}

int asterx_rhs(const asterx_grid* gr, const asterx_params* p, const double* metric, const double* curv,
               const double* prim, const double* A, const double* psi, double dt_max, double* rhs, double* red,
               void* workspace, size_t ws_bytes, void* stream) {
  int rc;
  if ((rc = check_params(p))) return rc;
  // the face kernels load a six-cell stencil (i-3..i+2) for every scheme
  if ((rc = check_grid(gr, 3))) return rc;
  if (p->ct == ASTERX_CT_UCT && gr->ng < 4) return fail(ASTERX_EARG, "rhs: upwind CT needs ng >= 4");
  if (!metric || !curv || !prim || !A || !psi || !rhs || !workspace) return fail(ASTERX_EARG, "rhs: NULL array");
  if (ws_bytes < asterx_rhs_workspace_size(gr)) return fail(ASTERX_EARG, "rhs: workspace too small");
  if (!(dt_max > 0.0)) return fail(ASTERX_EARG, "rhs: dt_max must be > 0");
  GD g = make_gd(gr);
  const asterx_batch* b = nullptr;
  return do_rhs(g, b, p, metric, curv, prim, A, psi, dt_max, rhs, red, (double*)workspace, (hipStream_t)stream);
}

int asterx_rk_stage(const asterx_grid* gr, int32_t nterms, const double* a, const double* const* u, double b_dt,
                    const double* rhs, double* out, void* stream) {
  int rc;
  if ((rc = check_grid(gr, 1))) return rc;
  GD g = make_gd(gr);
  const asterx_batch* b = nullptr;
  return do_rk(g, b, nterms, a, u, b_dt, rhs, out, (hipStream_t)stream);
}

int asterx_rhs_rk(const asterx_grid* gr, const asterx_params* p, const double* metric, const double* curv,
                  const double* prim, const double* A, const double* psi, double dt_max, int32_t nout,
                  const asterx_rk_out* outs, double* red, void* workspace, size_t ws_bytes, void* stream) {
  int rc;
  if ((rc = check_params(p)) || (rc = check_grid(gr, 3))) return rc;
  if (p->ct == ASTERX_CT_UCT && gr->ng < 4) return fail(ASTERX_EARG, "rhs_rk: upwind CT needs ng >= 4");
  if (!metric || !curv || !prim || !A || !psi || !workspace) return fail(ASTERX_EARG, "rhs_rk: NULL array");
  if (ws_bytes < asterx_rhs_workspace_size(gr)) return fail(ASTERX_EARG, "rhs_rk: workspace too small");
  if (!(dt_max > 0.0)) return fail(ASTERX_EARG, "rhs_rk: dt_max must be > 0");
  GD g = make_gd(gr);
  const double* ins[6] = {metric, curv, prim, A, psi, (const double*)workspace};
  const size_t nin[6] = {10 * g.N, 6 * g.N, 5 * g.N, 3 * g.N, g.N, ws_bytes / sizeof(double)};
  Combine cmb;
  if ((rc = make_combine(nout, outs, g.N, ins, nin, 6, cmb))) return rc;
  return do_rhs(g, nullptr, p, metric, curv, prim, A, psi, dt_max, nullptr, red, (double*)workspace,
                (hipStream_t)stream, cmb);
}

int asterx_rhs_rk_src(const asterx_grid* gr, const asterx_params* p, const double* metric, const double* prim,
                      const double* A, const double* psi, const double* src, double dt_max, int32_t nout,
                      const asterx_rk_out* outs, double* red, void* workspace, size_t ws_bytes, void* stream) {
  int rc;
  if ((rc = check_params(p)) || (rc = check_grid(gr, 3))) return rc;
  if (p->ct == ASTERX_CT_UCT && gr->ng < 4) return fail(ASTERX_EARG, "rhs_rk_src: upwind CT needs ng >= 4");
  if (!metric || !prim || !A || !psi || !src || !workspace) return fail(ASTERX_EARG, "rhs_rk_src: NULL array");
  if (ws_bytes < asterx_rhs_workspace_size(gr)) return fail(ASTERX_EARG, "rhs_rk_src: workspace too small");
  if (!(dt_max > 0.0)) return fail(ASTERX_EARG, "rhs_rk_src: dt_max must be > 0");
  GD g = make_gd(gr);
  const double* ins[6] = {metric, prim, A, psi, src, (const double*)workspace};
  const size_t nin[6] = {10 * g.N, 5 * g.N, 3 * g.N, g.N, ASTERX_SRC_FIELDS * g.N, ws_bytes / sizeof(double)};
  Combine cmb;
  if ((rc = make_combine(nout, outs, g.N, ins, nin, 6, cmb))) return rc;
  return do_rhs(g, nullptr, p, metric, nullptr, prim, A, psi, dt_max, nullptr, red, (double*)workspace,
                (hipStream_t)stream, cmb, src, p->ct == ASTERX_CT_UCT ? nullptr : src + 4 * g.N);
}

int asterx_geometry(const asterx_grid* gr, const asterx_params* p, const double* metric, const double* curv, double* geo,
                    void* stream) {
  int rc;
  if ((rc = check_params(p)) || (rc = check_grid(gr, 3))) return rc;
  if (p->ct == ASTERX_CT_UCT && gr->ng < 4) return fail(ASTERX_EARG, "geometry: upwind CT needs ng >= 4");
  if (!metric || !curv || !geo) return fail(ASTERX_EARG, "geometry: NULL array");
  GD g = make_gd(gr);
  GeomArgs ga{metric, curv, {}, {}, geo + (size_t)GEO_CEN * g.N, p->ct == ASTERX_CT_UCT ? 3 : 1, 0};
  for (int d = 0; d < 3; ++d) {
    ga.fa[d] = geo + (size_t)(10 * d) * g.N;
    ga.fb[d] = ga.fa[d] + 7 * g.N;
  }
  return geometry<GM_X | GM_Y | GM_Z | GM_C>(g, nullptr, ga, (hipStream_t)stream);
}

int asterx_c2p_geo(const asterx_grid* gr, const asterx_params* p, const double* geo, const double* A, double* cons,
                   double* prim, uint8_t* flags, asterx_c2p_stats* stats, const asterx_mlp* mlp, double* src,
                   void* stream) {
  int rc;
  if ((rc = check_grid(gr, 2)) || (rc = check_params(p))) return rc;
  if (!geo || !A || !prim || !cons || !src) return fail(ASTERX_EARG, "c2p_geo: NULL array");
  mlpd::Stdz z{};
  if (mlp) {
    if (!mlp->params) return fail(ASTERX_EARG, "c2p_geo: NULL network parameters");
    if ((rc = make_stdz(mlp, z, "c2p_geo"))) return rc;
  }
  GD g = make_gd(gr);
  hipStream_t s = (hipStream_t)stream;
  const C2PParams cp = make_c2p_params(p);
  const C2PArgs a{nullptr, A, cons, prim, flags, (unsigned long long*)stats, mlp ? mlp->params : nullptr, z, nullptr, src};
  const double* cen = geo + (size_t)GEO_CEN * g.N;
  return timed(KT_C2P, s, [&] {
    if (mlp)
      hipLaunchKernelGGL(k_c2p_learned_geo, dim3(lin_blocks(g.n)), dim3(256), 0, s, g, cp, a, cen);
    else
      hipLaunchKernelGGL(k_c2p_geo, dim3(lin_blocks(g.n)), dim3(256), 0, s, g, cp, a, cen);
  });
}

int asterx_rhs_rk_geo(const asterx_grid* gr, const asterx_params* p, const double* metric, const double* geo,
                      const double* prim, const double* A, const double* psi, const double* src, double dt_max,
                      int32_t nout, const asterx_rk_out* outs, double* red, void* workspace, size_t ws_bytes,
                      void* stream) {
  int rc;
  if ((rc = check_params(p)) || (rc = check_grid(gr, 3))) return rc;
  if (p->ct == ASTERX_CT_UCT && gr->ng < 4) return fail(ASTERX_EARG, "rhs_rk_geo: upwind CT needs ng >= 4");
  if (!metric || !geo || !prim || !A || !psi || !src || !workspace) return fail(ASTERX_EARG, "rhs_rk_geo: NULL array");
  if (ws_bytes < asterx_rhs_workspace_size(gr)) return fail(ASTERX_EARG, "rhs_rk_geo: workspace too small");
  if (!(dt_max > 0.0)) return fail(ASTERX_EARG, "rhs_rk_geo: dt_max must be > 0");
  GD g = make_gd(gr);
  const double* ins[7] = {metric, prim, A, psi, src, (const double*)workspace, geo};
  const size_t nin[7] = {10 * g.N, 5 * g.N, 3 * g.N, g.N, 4 * g.N, ws_bytes / sizeof(double), ASTERX_GEO_FIELDS * g.N};
  Combine cmb;
  if ((rc = make_combine(nout, outs, g.N, ins, nin, 7, cmb))) return rc;
  return do_rhs(g, nullptr, p, metric, nullptr, prim, A, psi, dt_max, nullptr, red, (double*)workspace,
                (hipStream_t)stream, cmb, src, nullptr, geo);
}

int asterx_rhs_rk_noalloc(const asterx_grid* gr, const asterx_params* p, const double* metric, const double* curv,
                          const double* prim, const double* A, const double* psi, double dt_max, int32_t nout,
                          const asterx_rk_out* outs, double* red, void* stream) {
  int rc;
  if ((rc = check_params(p)) || (rc = check_grid(gr, 3))) return rc;
  const size_t need = asterx_rhs_workspace_size(gr);
  if (need > ASTERX_NOALLOC_WS_BYTES)
    return fail(ASTERX_EARG, "rhs_rk_noalloc: the grid needs more workspace than the library holds (64 MiB)");
  void* ws = nullptr;
  if ((rc = scratch_address(&ws))) return rc;
  return asterx_rhs_rk(gr, p, metric, curv, prim, A, psi, dt_max, nout, outs, red, ws, need, stream);
}

int asterx_tmunu(const asterx_grid* gr, const asterx_params* p, const double* metric, const double* prim,
                 const double* A, double* tmunu, void* stream) {
  int rc;
  if ((rc = check_params(p)) || (rc = check_grid(gr, 2))) return rc;
  if (!metric || !prim || !A || !tmunu) return fail(ASTERX_EARG, "tmunu: NULL array");
  GD g = make_gd(gr);
  TmunuArgs ta{metric, prim, A, tmunu, p->gamma};
  hipStream_t s = (hipStream_t)stream;
  return timed(KT_TMUNU, s, [&] { hipLaunchKernelGGL(k_tmunu, dim3(tmunu_tiles(g)), dim3(256), 0, s, g, ta); });
}

// Coarse index range reached by prolonging fine indices [lo, hi] along one axis.
void prolong_reach(int lo, int hi, int c0, int vertex, int& cmin, int& cmax) {
  auto fd = [](int f) { return f >= 0 ? f / 2 : -((1 - f) / 2); };
  cmin = c0 + fd(lo) - 1;
  cmax = c0 + fd(hi) + (vertex ? 2 : 1);
}

int check_inter(const asterx_grid* gc, const asterx_grid* gf, const int32_t* c0, const int32_t* stag, int32_t nf,
                const void* src, const void* dst, const int32_t* lo, const int32_t* hi, bool prolong) {
  int rc;
  if ((rc = check_grid(gc, 2)) || (rc = check_grid(gf, 2))) return rc;
  if (!c0 || !stag || !lo || !hi || !src || !dst || nf < 1) return fail(ASTERX_EARG, "inter-level: bad arguments");
  for (int d = 0; d < 3; ++d) {
    if (stag[d] != 0 && stag[d] != 1) return fail(ASTERX_EARG, "inter-level: stag must be 0 (cell) or 1 (vertex)");
    if (lo[d] > hi[d]) return fail(ASTERX_EARG, "inter-level: empty box");
    const asterx_grid* out = prolong ? gf : gc;
    if (lo[d] < -out->ng || hi[d] > out->n[d] + out->ng) return fail(ASTERX_EARG, "inter-level: box outside the target grid");
    int rmin, rmax;
    const asterx_grid* in = prolong ? gc : gf;
    if (prolong) {
      prolong_reach(lo[d], hi[d], c0[d], stag[d], rmin, rmax);
    } else {
      rmin = 2 * (lo[d] - c0[d]);
      rmax = 2 * (hi[d] - c0[d]) + 1;
    }
    if (rmin < -in->ng || rmax > in->n[d] + in->ng) return fail(ASTERX_EARG, "inter-level: stencil outside the source grid");
  }
  return 0;
}

int inter_launch(const asterx_grid* gc, const asterx_grid* gf, const int32_t* c0, const int32_t* stag, int32_t nf,
                 const double* src, double* dst, const int32_t* lo, const int32_t* hi, bool prolong, void* stream) {
  InterArgs a;
  a.gc = make_gd(gc);
  a.gf = make_gd(gf);
  for (int d = 0; d < 3; ++d) {
    a.c0[d] = c0[d];
    a.stag[d] = stag[d];
    a.lo[d] = lo[d];
    a.hi[d] = hi[d];
  }
  a.nf = nf;
  a.src = src;
  a.dst = dst;
  int e[3] = {hi[0] - lo[0] + 1, hi[1] - lo[1] + 1, hi[2] - lo[2] + 1};
  if (prolong)
    for (int d = 0; d < 3; ++d) {
      auto fd = [](int f) { return f >= 0 ? f / 2 : -((1 - f) / 2); };
      e[d] = fd(hi[d]) - fd(lo[d]) + 1;  // coarse parents of the fine box
    }
  hipStream_t s = (hipStream_t)stream;
  void (*kern)(InterArgs) = k_restrict;
  if (prolong) {
    void (*const by_stag[8])(InterArgs) = {k_prolong_cells, k_prolong<1>, k_prolong<2>, k_prolong<3>,
                                           k_prolong<4>,    k_prolong<5>, k_prolong<6>, k_prolong<7>};
    kern = by_stag[stag[0] + 2 * stag[1] + 4 * stag[2]];
  }
  const unsigned nb = lin_blocks(e) * (kern == k_prolong_cells ? (unsigned)nf : 1u);
  return timed(KT_INTER, s, [&] { hipLaunchKernelGGL(kern, dim3(nb), dim3(256), 0, s, a); });
}

int asterx_prolong(const asterx_grid* coarse, const asterx_grid* fine, const int32_t* c0, const int32_t* stag,
                   int32_t nf, const double* cf, double* ff, const int32_t* lo, const int32_t* hi, void* stream) {
  int rc;
  if ((rc = check_inter(coarse, fine, c0, stag, nf, cf, ff, lo, hi, true))) return rc;
  return inter_launch(coarse, fine, c0, stag, nf, cf, ff, lo, hi, true, stream);
}

int asterx_restrict(const asterx_grid* coarse, const asterx_grid* fine, const int32_t* c0, const int32_t* stag,
                    int32_t nf, const double* ff, double* cf, const int32_t* lo, const int32_t* hi, void* stream) {
  int rc;
  if ((rc = check_inter(coarse, fine, c0, stag, nf, ff, cf, lo, hi, false))) return rc;
  return inter_launch(coarse, fine, c0, stag, nf, ff, cf, lo, hi, false, stream);
}

int asterx_zero(double* buf, int64_t count, void* stream) {
  if (!buf || count < 1) return fail(ASTERX_EARG, "zero: bad arguments");
  hipStream_t s = (hipStream_t)stream;
  return timed(KT_ZERO, s, [&] {
    hipLaunchKernelGGL(k_zero, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, buf, (long long)count);
  });
}

// ---- batches of patches -------------------------------------------------------------------

int asterx_batch_create(int32_t npatches, const asterx_grid* grids, const asterx_batch_tuning* tuning,
                        asterx_batch** out) {
  if (!out || npatches < 1 || !grids) return fail(ASTERX_EARG, "batch_create: bad arguments");
  *out = nullptr;
  int order = tuning ? tuning->order : 1;
  int per_cu = tuning ? tuning->blocks_per_cu : 4;
  if (order < 0 || order > 2 || per_cu < 1 || per_cu > 64) return fail(ASTERX_EARG, "batch_create: bad tuning");
  asterx_batch* b = new asterx_batch();
  b->np = npatches;
  long long tot = 0;
  for (int q = 0; q < npatches; ++q) {
    int rc = check_grid(&grids[q], 3);
    if (rc) {
      delete b;
      return rc;
    }
    b->off.push_back(tot);
    tot += (long long)grids[q].ld[0] * grids[q].ld[1] * grids[q].ld[2];
  }
  b->ntot = tot;
  std::vector<PatchDesc> pd(npatches);
  for (int q = 0; q < npatches; ++q) {
    GD g = make_gd(&grids[q]);
    g.N = (size_t)tot;  // field stride of the pools
    b->gds.push_back(g);
    pd[q].g = g;
    pd[q].off = b->off[q];
  }
  int dev = 0, ncu = 256;
  if (hipGetDevice(&dev) == hipSuccess) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) ncu = v;
  }
  b->blocks = per_cu * ncu;
  for (int d = 1; d < 3; ++d) {
    long long single = 0;
    for (const GD& g : b->gds) single += face_items(g.n, d, 1, 1);
    b->rows[d] = single <= FACE_SLOTS ? 1 : FACE_BATCH_ROWS;
  }
  const auto tiles = [b](int ph, int q) { return tiles_for(ph, b->gds[q], b->rows); };
  std::vector<std::vector<Item>> lists(PH_N);
  for (int ph = 0; ph < PH_N; ++ph) {
    std::vector<int> porder(npatches);
    for (int q = 0; q < npatches; ++q) porder[q] = q;
    if (order == 1)
      std::stable_sort(porder.begin(), porder.end(),
                       [&](int x, int y) { return tiles(ph, x) > tiles(ph, y); });
    std::vector<Item>& L = lists[ph];
    if (order == 2) {  // round robin over patches, largest first
      std::stable_sort(porder.begin(), porder.end(),
                       [&](int x, int y) { return tiles(ph, x) > tiles(ph, y); });
      unsigned maxt = 0;
      for (int q = 0; q < npatches; ++q) maxt = std::max(maxt, tiles(ph, q));
      for (unsigned t = 0; t < maxt; ++t)
        for (int q : porder)
          if (t < tiles(ph, q)) L.push_back(Item{q, (int)t});
    } else {
      for (int q : porder)
        for (unsigned t = 0; t < tiles(ph, q); ++t) L.push_back(Item{q, (int)t});
    }
    b->nitems[ph] = (int)L.size();
  }
  bool ok = hipMalloc((void**)&b->d_patches, sizeof(PatchDesc) * npatches) == hipSuccess &&
            hipMemcpy(b->d_patches, pd.data(), sizeof(PatchDesc) * npatches, hipMemcpyHostToDevice) == hipSuccess;
  for (int ph = 0; ph < PH_N && ok; ++ph) {
    ok = hipMalloc((void**)&b->d_items[ph], sizeof(Item) * lists[ph].size()) == hipSuccess &&
         hipMemcpy(b->d_items[ph], lists[ph].data(), sizeof(Item) * lists[ph].size(), hipMemcpyHostToDevice) ==
             hipSuccess;
  }
  if (!ok) {
    asterx_batch_destroy(b);
    return fail(ASTERX_ELAUNCH, "batch_create: device allocation failed");
  }
  *out = b;
  return 0;
}

int asterx_batch_destroy(asterx_batch* b) {
  if (!b) return 0;
  if (b->d_patches) (void)hipFree(b->d_patches);
  for (int ph = 0; ph < PH_N; ++ph)
    if (b->d_items[ph]) (void)hipFree(b->d_items[ph]);
  delete b;
  return 0;
}

int64_t asterx_batch_points(const asterx_batch* b) { return b ? b->ntot : -1; }

int64_t asterx_batch_offset(const asterx_batch* b, int32_t p) {
  return (b && p >= 0 && p < b->np) ? b->off[p] : -1;
}

size_t asterx_batch_workspace_size(const asterx_batch* b) {
  return b ? (size_t)WS_FIELDS * (size_t)b->ntot * sizeof(double) : 0;
}

int asterx_batch_prim2con(const asterx_batch* b, const asterx_params* p, const double* metric, const double* A,
                          const double* prim, double* cons, void* stream) {
  int rc;
  if (!b) return fail(ASTERX_EARG, "batch is NULL");
  if ((rc = check_params(p))) return rc;
  if (!metric || !A || !prim || !cons) return fail(ASTERX_EARG, "batch_prim2con: NULL array");
  const GD& g = b->gds[0];
  return do_prim2con(g, b, p, metric, A, prim, cons, (hipStream_t)stream);
}

int asterx_batch_c2p(const asterx_batch* b, const asterx_params* p, const double* metric, const double* A,
                     double* cons, double* prim, uint8_t* flags, asterx_c2p_stats* stats, void* stream) {
  int rc;
  if (!b) return fail(ASTERX_EARG, "batch is NULL");
  if ((rc = check_params(p))) return rc;
  if (!metric || !A || !prim || !cons) return fail(ASTERX_EARG, "batch_c2p: NULL array");
  const GD& g = b->gds[0];
  return do_c2p(g, b, p, metric, A, cons, prim, flags, stats, (hipStream_t)stream);
}

int asterx_batch_fill_state(const asterx_batch* b, double* u, const int32_t* kinds_cell, const int32_t* kinds_A,
                            void* stream) {
  if (!b || !u || !kinds_cell || !kinds_A) return fail(ASTERX_EARG, "batch_fill_state: bad arguments");
  int rc;
  if ((rc = check_batch_kinds(b, kinds_cell)) || (rc = check_batch_kinds(b, kinds_A))) return rc;
  return do_fill_state(b->gds[0], b, u, kinds_cell, kinds_A, nullptr, (hipStream_t)stream);
}

int asterx_batch_fill_ghosts(const asterx_batch* b, double* f, int32_t nf, const int32_t* kinds, void* stream) {
  if (!b || !f || !kinds || nf < 1) return fail(ASTERX_EARG, "batch_fill_ghosts: bad arguments");
  int rc;
  if ((rc = check_batch_kinds(b, kinds))) return rc;
  const GD& g = b->gds[0];
  return do_fill(g, b, f, nf, kinds, (hipStream_t)stream);
}

int asterx_batch_rhs(const asterx_batch* b, const asterx_params* p, const double* metric, const double* curv,
                     const double* prim, const double* A, const double* psi, double dt_max, double* rhs, double* red,
                     void* workspace, size_t ws_bytes, void* stream) {
  int rc;
  if (!b) return fail(ASTERX_EARG, "batch is NULL");
  if ((rc = check_params(p))) return rc;
  if (p->ct == ASTERX_CT_UCT) return fail(ASTERX_EARG, "batch: upwind CT is available for single blocks only");
  if (!metric || !curv || !prim || !A || !psi || !rhs || !workspace) return fail(ASTERX_EARG, "rhs: NULL array");
  if (ws_bytes < asterx_batch_workspace_size(b)) return fail(ASTERX_EARG, "rhs: workspace too small");
  if (!(dt_max > 0.0)) return fail(ASTERX_EARG, "rhs: dt_max must be > 0");
  const GD& g = b->gds[0];
  return do_rhs(g, b, p, metric, curv, prim, A, psi, dt_max, rhs, red, (double*)workspace, (hipStream_t)stream);
}

int asterx_batch_rhs_rk(const asterx_batch* b, const asterx_params* p, const double* metric, const double* curv,
                        const double* prim, const double* A, const double* psi, double dt_max, int32_t nout,
                        const asterx_rk_out* outs, double* red, void* workspace, size_t ws_bytes, void* stream) {
  int rc;
  if (!b) return fail(ASTERX_EARG, "batch is NULL");
  if ((rc = check_params(p))) return rc;
  if (p->ct == ASTERX_CT_UCT) return fail(ASTERX_EARG, "batch: upwind CT is available for single blocks only");
  if (!metric || !curv || !prim || !A || !psi || !workspace) return fail(ASTERX_EARG, "rhs_rk: NULL array");
  if (ws_bytes < asterx_batch_workspace_size(b)) return fail(ASTERX_EARG, "rhs_rk: workspace too small");
  if (!(dt_max > 0.0)) return fail(ASTERX_EARG, "rhs_rk: dt_max must be > 0");
  const size_t n = (size_t)b->ntot;
  const double* ins[6] = {metric, curv, prim, A, psi, (const double*)workspace};
  const size_t nin[6] = {10 * n, 6 * n, 5 * n, 3 * n, n, ws_bytes / sizeof(double)};
  Combine cmb;
  if ((rc = make_combine(nout, outs, n, ins, nin, 6, cmb))) return rc;
  const GD& g = b->gds[0];
  return do_rhs(g, b, p, metric, curv, prim, A, psi, dt_max, nullptr, red, (double*)workspace, (hipStream_t)stream,
                cmb);
}

int asterx_batch_rk_stage(const asterx_batch* b, int32_t nterms, const double* a, const double* const* u,
                          double b_dt, const double* rhs, double* out, void* stream) {
  if (!b) return fail(ASTERX_EARG, "batch is NULL");
  const GD& g = b->gds[0];
  return do_rk(g, b, nterms, a, u, b_dt, rhs, out, (hipStream_t)stream);
}

}  // extern "C"

// ---- adjoint -------------------------------------------------------------------------------

namespace {

unsigned pts_blocks(long long n) { return (unsigned)((n + 255) / 256); }

int adj_fillT(const GD& g, double* f, int nf, hipStream_t s) {
  int rc;
  for (int a = 2; a >= 0; --a) {
    FillTArgs fa{f, nf, a};
    unsigned nb = (unsigned)((fill_points(g, a) + 255) / 256);
    if ((rc = timed(KT_ADJ, s, [&] { hipLaunchKernelGGL(k_fillT, dim3(nb), dim3(256), 0, s, g, fa); }))) return rc;
  }
  return 0;
}

template <int D, int R>
int adj_faces_d(const GD& g, FaceAdjArgs fa, hipStream_t s) {
  int rc;
  fa.rows = recon_adj_rows(g, D);
  const int e[3] = {g.n[0] + 1, g.n[1] + 1, g.n[2] + 1};
  if ((rc = timed(KT_ADJ, s, [&] { hipLaunchKernelGGL((k_face_adj<D, R>), dim3(face_tiles(e)), dim3(256), 0, s, g, fa); })))
    return rc;
  return timed(KT_ADJ, s, [&] { hipLaunchKernelGGL((k_recon_adj<D, R>), dim3(recon_adj_items(g, D, fa.rows)), dim3(64), 0, s, g, fa); });
}

template <int R>
int adj_faces_r(const GD& g, const FaceAdjArgs& fa, hipStream_t s) {
  int rc;
  if ((rc = adj_faces_d<0, R>(g, fa, s)) || (rc = adj_faces_d<1, R>(g, fa, s))) return rc;
  return adj_faces_d<2, R>(g, fa, s);
}

int check_adjoint(const asterx_grid* gr, const asterx_params* p, size_t ws_bytes) {
  int rc;
  if ((rc = check_params(p)) || (rc = check_grid(gr, 3))) return rc;
  for (int a = 0; a < 3; ++a)
    if (gr->n[a] < gr->ng + 1) return fail(ASTERX_EARG, "adjoint: periodic blocks need n > ng on every axis");
  if (ws_bytes < asterx_adjoint_workspace_size(gr)) return fail(ASTERX_EARG, "adjoint: workspace too small");
  return 0;
}

// Zero workspace fields [AW_PBAR, zero_end), copy the stage input, recompute c2p (flags in the workspace tail) and
// the centre field.  The fields before are written here; the flux cotangents and, in a stage's adjoint, those that
// the left faces' cotangents take first, are written before they are read (64^3: clearing all 52 took 17 us a call).
int adj_prologue(const GD& g, const asterx_params* p, const double* metric, const double* cons,
                 const double* prim_guess, const double* A, double* ws, uint8_t* flags, hipStream_t s, bool with_c2p,
                 int zero_end) {
  int rc;
  long long nzero = (long long)(zero_end - AW_PBAR) * (long long)g.N;
  if ((rc = timed(KT_ZERO, s, [&] {
         hipLaunchKernelGGL(k_zero, dim3(pts_blocks(nzero)), dim3(256), 0, s, ws + AW_PBAR * g.N, nzero);
       })))
    return rc;
  if ((rc = do_bcent(g, A, ws + AW_BC * g.N, s))) return rc;
  if (!with_c2p) return 0;
  long long n5 = 5LL * (long long)g.N;
  if ((rc = timed(KT_ADJ, s, [&] {
         hipLaunchKernelGGL(k_copy, dim3(pts_blocks(n5)), dim3(256), 0, s, g, cons, ws + AW_CONS * g.N, n5);
       })))
    return rc;
  if ((rc = timed(KT_ADJ, s, [&] {
         hipLaunchKernelGGL(k_copy, dim3(pts_blocks(n5)), dim3(256), 0, s, g, prim_guess, ws + AW_PRIM * g.N, n5);
       })))
    return rc;
  const asterx_batch* b = nullptr;
  if ((rc = do_c2p(g, b, p, metric, A, ws + AW_CONS * g.N, ws + AW_PRIM * g.N, flags, nullptr, s))) return rc;
  const int32_t per[3] = {ASTERX_BC_PERIODIC, ASTERX_BC_PERIODIC, ASTERX_BC_PERIODIC};
  return do_fill(g, b, ws + AW_PRIM * g.N, 5, per, s);
}

// Gamma cotangent slots: after the flags in the workspace tail.
double* gamma_slots(const GD& g, double* ws) { return ws + (size_t)AW_FIELDS * g.N + ((size_t)g.N + 7) / 8; }

int gslots_zero(double* slots, hipStream_t s) {
  return timed(KT_ZERO, s, [&] { hipLaunchKernelGGL(k_zero, dim3(1), dim3(256), 0, s, slots, (long long)GSLOTS); });
}

int gslots_finish(const double* slots, double* gamma_bar, hipStream_t s) {
  return timed(KT_ADJ, s, [&] { hipLaunchKernelGGL(k_gslots, dim3(1), dim3(64), 0, s, slots, gamma_bar); });
}

// Centre-field and face-field cotangents to the edge potential, fold ghosts, add to A_bar.
int adj_epilogue(const GD& g, double* ws, double* A_bar, double* psi_bar, hipStream_t s) {
  int rc;
  int ef[3] = {g.n[0] + 2 * g.ng + 1, g.n[1] + 2 * g.ng + 1, g.n[2] + 2 * g.ng + 1};
  unsigned nb = box_blocks<64, 4>(ef);
  if ((rc = timed(KT_ADJ, s, [&] {
         hipLaunchKernelGGL(k_bcface_adj, dim3(nb), dim3(256), 0, s, g, ws + AW_BCBAR * g.N, ws + AW_BFBAR * g.N);
       })))
    return rc;
  if ((rc = timed(KT_ADJ, s, [&] {
         hipLaunchKernelGGL(k_curlT, dim3(nb), dim3(256), 0, s, g, ws + AW_BFBAR * g.N, ws + AW_ABAR * g.N);
       })))
    return rc;
  // Psi's cotangent is the field after the potential's three
  if ((rc = adj_fillT(g, ws + AW_ABAR * g.N, psi_bar ? 4 : 3, s))) return rc;
  unsigned no = tiles_for(PH_RK, g);
  if (A_bar) {
    AccumArgs aa{ws + AW_ABAR * g.N, A_bar, 3};
    if ((rc = timed(KT_ADJ, s, [&] { hipLaunchKernelGGL(k_accum, dim3(no), dim3(256), 0, s, g, aa); }))) return rc;
  }
  if (psi_bar) {
    AccumArgs pa{ws + AW_PSIBAR * g.N, psi_bar, 1};
    if ((rc = timed(KT_ADJ, s, [&] { hipLaunchKernelGGL(k_accum, dim3(no), dim3(256), 0, s, g, pa); }))) return rc;
  }
  return 0;
}

}  // namespace

extern "C" {

size_t asterx_adjoint_workspace_size(const asterx_grid* g) {
  if (!g) return 0;
  size_t N = (size_t)g->ld[0] * g->ld[1] * g->ld[2];
  return (size_t)AW_FIELDS * N * sizeof(double) + ((N + 7) / 8) * 8 + GSLOTS * sizeof(double);
}

int asterx_rhs_adjoint(const asterx_grid* gr, const asterx_params* p, const double* metric, const double* curv,
                       const double* cons, const double* prim_guess, const double* A, const double* psi,
                       double dt_max, const double* rhs_bar, double* cons_bar, double* A_bar, double* psi_bar,
                       double* gamma_bar, void* workspace, size_t ws_bytes, void* stream) {
  int rc;
  if ((rc = check_adjoint(gr, p, ws_bytes))) return rc;
  if (p->ct == ASTERX_CT_UCT) return fail(ASTERX_EARG, "rhs_adjoint: upwind CT is not differentiated");
  if (!metric || !curv || !cons || !prim_guess || !A || !psi || !rhs_bar || !cons_bar || !A_bar || !psi_bar ||
      !gamma_bar || !workspace)
    return fail(ASTERX_EARG, "rhs_adjoint: NULL array");
  if (!(dt_max > 0.0)) return fail(ASTERX_EARG, "rhs_adjoint: dt_max must be > 0");
  hipStream_t s = (hipStream_t)stream;
  GD g = make_gd(gr);
  double* ws = (double*)workspace;
  uint8_t* flags = (uint8_t*)(ws + (size_t)AW_FIELDS * g.N);
  double* slots = gamma_slots(g, ws);
  if ((rc = adj_prologue(g, p, metric, cons, prim_guess, A, ws, flags, s, true, AW_XBAR))) return rc;
  if ((rc = gslots_zero(slots, s))) return rc;
  unsigned nb;
  // fluxbar and vertex_adj tile the (n + 2)^3 vertex box 64 x 4
  int ev[3] = {g.n[0] + 2, g.n[1] + 2, g.n[2] + 2};
  FluxBarArgs fb{rhs_bar, ws + AW_FBAR * g.N};
  nb = box_blocks<64, 4>(ev);
  if ((rc = timed(KT_ADJ, s, [&] { hipLaunchKernelGGL(k_fluxbar, dim3(nb), dim3(256), 0, s, g, fb); }))) return rc;
  FaceAdjArgs fa{metric, ws + AW_PRIM * g.N, A, ws + AW_BC * g.N, ws + AW_FBAR * g.N, ws + AW_XBAR * g.N,
                 ws + AW_PBAR * g.N, ws + AW_BCBAR * g.N, ws + AW_BFBAR * g.N, slots, p->gamma, p->weno_eps, p->weno_q, p->speeds,
                 p->riemann};
  if (p->recon == ASTERX_RECON_MINMOD) rc = adj_faces_r<ASTERX_RECON_MINMOD>(g, fa, s);
  else if (p->recon == ASTERX_RECON_PPM) rc = adj_faces_r<ASTERX_RECON_PPM>(g, fa, s);
  else if (p->recon == ASTERX_RECON_MP5) rc = adj_faces_r<ASTERX_RECON_MP5>(g, fa, s);
  else rc = adj_faces_r<ASTERX_RECON_WENOZ>(g, fa, s);
  if (rc) return rc;
  const long long nx = 7LL * (long long)g.N;
  if ((rc = timed(KT_ZERO, s, [&] {
         hipLaunchKernelGGL(k_zero, dim3(pts_blocks(nx)), dim3(256), 0, s, ws + AW_XBAR * g.N, nx);
       })))
    return rc;
  CellAdjArgs ca{metric, curv, ws + AW_PRIM * g.N, ws + AW_BC * g.N, rhs_bar, ws + AW_PBAR * g.N,
                 ws + AW_BCBAR * g.N, slots, p->gamma};
  if ((rc = timed(KT_ADJ, s, [&] {
         hipLaunchKernelGGL(k_cell_adj, dim3(tiles_for(PH_CELL, g)), dim3(256), 0, s, g, ca);
       })))
    return rc;
  VertexAdjArgs va{metric, rhs_bar, ws + AW_PSIBAR * g.N, ws + AW_AVBAR * g.N, p->xi / dt_max, p->gauge};
  nb = box_blocks<64, 4>(ev);
  if ((rc = timed(KT_ADJ, s, [&] { hipLaunchKernelGGL(k_vertex_adj, dim3(nb), dim3(256), 0, s, g, va); }))) return rc;
  int ee[3] = {g.n[0] + 3, g.n[1] + 3, g.n[2] + 3};
  nb = box_blocks<64, 4>(ee);
  if ((rc = timed(KT_ADJ, s, [&] {
         hipLaunchKernelGGL(k_edge_adj, dim3(nb), dim3(256), 0, s, g, ws + AW_AVBAR * g.N, ws + AW_ABAR * g.N);
       })))
    return rc;
  if ((rc = adj_fillT(g, ws + AW_PBAR * g.N, 5, s))) return rc;
  C2PAdjArgs cpa{metric, ws + AW_PRIM * g.N, ws + AW_BC * g.N, flags, ws + AW_PBAR * g.N, cons_bar,
                 ws + AW_BCBAR * g.N, slots, p->gamma, 0};
  if ((rc = timed(KT_ADJ, s, [&] {
         hipLaunchKernelGGL(k_c2p_adj, dim3(tiles_for(PH_C2P, g)), dim3(256), 0, s, g, cpa);
       })))
    return rc;
  if ((rc = adj_epilogue(g, ws, A_bar, psi_bar, s))) return rc;
  return gslots_finish(slots, gamma_bar, s);
}

int asterx_c2p_adjoint(const asterx_grid* gr, const asterx_params* p, const double* metric, const double* cons,
                       const double* prim_guess, const double* A, const double* prim_bar, double* cons_bar,
                       double* A_bar, double* gamma_bar, void* workspace, size_t ws_bytes, void* stream) {
  int rc;
  if ((rc = check_adjoint(gr, p, ws_bytes))) return rc;
  if (!metric || !cons || !prim_guess || !A || !prim_bar || !cons_bar || !A_bar || !gamma_bar || !workspace)
    return fail(ASTERX_EARG, "c2p_adjoint: NULL array");
  hipStream_t s = (hipStream_t)stream;
  GD g = make_gd(gr);
  double* ws = (double*)workspace;
  uint8_t* flags = (uint8_t*)(ws + (size_t)AW_FIELDS * g.N);
  double* slots = gamma_slots(g, ws);
  if ((rc = adj_prologue(g, p, metric, cons, prim_guess, A, ws, flags, s, true, AW_PSIBAR))) return rc;
  if ((rc = gslots_zero(slots, s))) return rc;
  unsigned no = tiles_for(PH_RK, g);
  AccumArgs cp{prim_bar, ws + AW_PBAR * g.N, 5};
  if ((rc = timed(KT_ADJ, s, [&] { hipLaunchKernelGGL(k_accum, dim3(no), dim3(256), 0, s, g, cp); }))) return rc;
  C2PAdjArgs cpa{metric, ws + AW_PRIM * g.N, ws + AW_BC * g.N, flags, ws + AW_PBAR * g.N, cons_bar,
                 ws + AW_BCBAR * g.N, slots, p->gamma, 0};
  if ((rc = timed(KT_ADJ, s, [&] {
         hipLaunchKernelGGL(k_c2p_adj, dim3(tiles_for(PH_C2P, g)), dim3(256), 0, s, g, cpa);
       })))
    return rc;
  if ((rc = adj_epilogue(g, ws, A_bar, nullptr, s))) return rc;
  return gslots_finish(slots, gamma_bar, s);
}

int asterx_prim2con_adjoint(const asterx_grid* gr, const asterx_params* p, const double* metric, const double* A,
                            const double* prim, const double* cons_bar, double* prim_bar, double* A_bar,
                            double* gamma_bar, void* workspace, size_t ws_bytes, void* stream) {
  int rc;
  if ((rc = check_adjoint(gr, p, ws_bytes))) return rc;
  if (!metric || !A || !prim || !cons_bar || !prim_bar || !A_bar || !gamma_bar || !workspace)
    return fail(ASTERX_EARG, "prim2con_adjoint: NULL array");
  hipStream_t s = (hipStream_t)stream;
  GD g = make_gd(gr);
  double* ws = (double*)workspace;
  double* slots = gamma_slots(g, ws);
  if ((rc = adj_prologue(g, p, metric, nullptr, nullptr, A, ws, nullptr, s, false, AW_PSIBAR))) return rc;
  if ((rc = gslots_zero(slots, s))) return rc;
  unsigned no = tiles_for(PH_RK, g);
  AccumArgs cp{cons_bar, ws + AW_PBAR * g.N, 5};
  if ((rc = timed(KT_ADJ, s, [&] { hipLaunchKernelGGL(k_accum, dim3(no), dim3(256), 0, s, g, cp); }))) return rc;
  C2PAdjArgs cpa{metric, prim, ws + AW_BC * g.N, nullptr, ws + AW_PBAR * g.N, prim_bar, ws + AW_BCBAR * g.N,
                 slots, p->gamma, 1};
  if ((rc = timed(KT_ADJ, s, [&] {
         hipLaunchKernelGGL(k_c2p_adj, dim3(tiles_for(PH_C2P, g)), dim3(256), 0, s, g, cpa);
       })))
    return rc;
  if ((rc = adj_epilogue(g, ws, A_bar, nullptr, s))) return rc;
  return gslots_finish(slots, gamma_bar, s);
}

}  // extern "C"
