// projection.h - the pressure-correction steps on either side of the
// Poisson solve (Sec. 2: the right-hand side of Eq. (poi_ns) and the two
// updates that follow it), on the staggered grid.
//
// Layout: Phi, p and the right-hand side at cell centres (nx*ny*nz, x
// fastest).  The velocity component along an axis on the faces normal to
// it: n faces along a periodic axis (face f between cells f-1, cyclically,
// and f), n + 1 along a walled one (face 0 the low wall, face n the high
// wall); the other two extents are those of the cells.
//
// Face gradient of a cell field: (Phi_f - Phi_{f-1}) / dc_f, dc_f the
// distance of the two centres.  Walls use the ghost cells of the solve's
// boundary rule: a Neumann wall has zero gradient (the projection leaves
// its velocity untouched), a Dirichlet wall (Phi = 0 on it) has
// 2 Phi_edge / h_edge towards the inside.  The divergence of the gradient
// is then the solve's seven-point operator row for row, so the projected
// velocity is divergence-free up to rounding.
//
// Both kernels are one HBM sweep over the cells (x fastest across the
// threads): the right-hand side reads three face arrays and writes one
// cell array (32 B per cell), the update reads Phi, the three face arrays
// and p and writes the face arrays (in place or into a second set) and p
// (72 B per cell).
#pragma once
#include "refine_kernels.h"

namespace poisson_dev {

// One axis of the projection: n cells; walled (n + 1 faces) or periodic;
// wall kinds (0 Neumann, 1 Dirichlet); inv_h[n] = 1 / cell width;
// inv_dc[faces] = 1 / centre distance (at a wall: 1 / edge width).
struct ProjAxis {
  const double* inv_h;
  const double* inv_dc;
  int n;
  int walled;
  int lo_dirichlet;
  int hi_dirichlet;
};

struct ProjGeom {
  ProjAxis ax[3];
  long long npts;
};

static constexpr int PROJ_NT = 256;

// rhs = div(u, v, w) * inv_gdt at every cell.  z-marching like the update
// below (tiles of 64 x 4 columns, PROJ_KC planes): w on the high face of a
// cell is w on the low face of the cell above, so each plane reads one new
// w face per cell and keeps it for the next; the next plane's faces are
// read before this plane's result is stored.
static constexpr int PROJ_TX = 64, PROJ_TY = 4, PROJ_KC = 32;

__global__ __launch_bounds__(PROJ_NT) void proj_rhs_kernel(const double* __restrict__ u,
                                                           const double* __restrict__ v,
                                                           const double* __restrict__ w,
                                                           double inv_gdt, double* __restrict__ rhs,
                                                           ProjGeom G) {
  const int nx = G.ax[0].n, ny = G.ax[1].n, nz = G.ax[2].n;
  const int ux = nx + G.ax[0].walled;          // faces along x
  const int vy = ny + G.ax[1].walled;          // faces along y
  const long long plane = (long long)nx * ny;
  const int i = blockIdx.x * PROJ_TX + (threadIdx.x & (PROJ_TX - 1));
  const int j = blockIdx.y * PROJ_TY + threadIdx.x / PROJ_TX;
  const int k0 = (int)((long long)blockIdx.z * nz / gridDim.z);
  const int kend = (int)((long long)(blockIdx.z + 1) * nz / gridDim.z);
  if (i >= nx || j >= ny) return;
  const int ip = G.ax[0].walled || i + 1 < nx ? i + 1 : 0;     // high x face
  const int jp = G.ax[1].walled || j + 1 < ny ? j + 1 : 0;     // high y face
  const long long col = i + (long long)nx * j;
  const double ihx = G.ax[0].inv_h[i], ihy = G.ax[1].inv_h[j];
  struct In {
    double u0, u1, v0, v1, w1;
  };
  // the faces of plane k other than its low z face (the high z face of the plane below)
  auto load = [&](int k) {
    In r;
    const long long ur = (long long)ux * (j + (long long)ny * k);
    r.u0 = u[ur + i];
    r.u1 = u[ur + ip];
    const long long vb = i + (long long)nx * vy * k;
    r.v0 = v[vb + (long long)nx * j];
    r.v1 = v[vb + (long long)nx * jp];
    const int kp = G.ax[2].walled || k + 1 < nz ? k + 1 : 0;
    r.w1 = w[col + plane * kp];
    return r;
  };
  double w0 = w[col + plane * k0];
  In cur = load(k0);
  for (int k = k0; k < kend; ++k) {
    In nxt = cur;
    if (k + 1 < kend) nxt = load(k + 1);
    const double du = cur.u1 - cur.u0, dv = cur.v1 - cur.v0, dw = cur.w1 - w0;
    rhs[col + plane * k] = (du * ihx + dv * ihy + dw * G.ax[2].inv_h[k]) * inv_gdt;
    w0 = cur.w1;
    cur = nxt;
  }
}

// u = u_in - gdt grad(phi) on every face, p += phi at every cell; in place
// when u_in == u (each face is read before it is written, by the same
// thread, and by no other).  z-marching: a block owns a 64 x 4 tile of
// (i, j) columns and at most PROJ_KC consecutive planes; each thread walks its
// column upward with Phi of the cell below in a register, so the z
// gradient reads no other plane (the x and y neighbours come from the
// lines the adjacent lanes and rows load).  The face values and p, each
// read and written by one thread only, take the nontemporal hint; Phi,
// which the neighbouring lanes read again, does not.  At a wall the
// neighbour's address is the cell's own and the gradient is selected, and the
// high wall faces are read behind uniform branches, so that no lane skips a
// load; only the last column's store of its high wall face is its own.  A
// plane's waits then leave the next plane's reads and the stores in flight.
// Bound by HBM.  Measured, branches per lane -> selects: 114 -> 92 us on 512 x
// 128 x 128 (P, NN, NN; 6.5 TB/s), 329 -> 307 us on 512 x 256 x 192 (P, P, NN;
// 5.9 TB/s), 128 -> 101 us on 270 x 150 x 162 (NN, P, ND; 97 with the shorter z
// ranges of proj_tiles), 1.63 -> 1.60 ms on the periodic 512^3 (6.0 TB/s; out
// of place, at the end of a time step, 1.82 -> 1.83).
__global__ __launch_bounds__(PROJ_NT) void proj_update_zmarch_kernel(
    const double* __restrict__ phi, double gdt, const double* u_in, const double* v_in,
    const double* w_in, double* u, double* v, double* w, double* __restrict__ p, ProjGeom G) {
  const int nx = G.ax[0].n, ny = G.ax[1].n, nz = G.ax[2].n;
  const int ux = nx + G.ax[0].walled;
  const int vy = ny + G.ax[1].walled;
  const long long plane = (long long)nx * ny;
  const int i = blockIdx.x * PROJ_TX + (threadIdx.x & (PROJ_TX - 1));
  const int j = blockIdx.y * PROJ_TY + threadIdx.x / PROJ_TX;
  const int k0 = (int)((long long)blockIdx.z * nz / gridDim.z);
  const int kend = (int)((long long)(blockIdx.z + 1) * nz / gridDim.z);
  if (i >= nx || j >= ny) return;
  const ProjAxis& X = G.ax[0];
  const ProjAxis& Y = G.ax[1];
  const ProjAxis& Z = G.ax[2];
  const long long col = i + (long long)nx * j;
  // columns on a wall: the low wall face's gradient is 2 Phi / h (Dirichlet)
  // or none (Neumann), and the last column also owns the high wall face,
  // which a Neumann wall leaves as it is (nothing to do in place)
  const bool xl = X.walled && i == 0, yl = Y.walled && j == 0;
  const bool xkeep = xl && !X.lo_dirichlet, ykeep = yl && !Y.lo_dirichlet;
  const bool xwall = X.walled && (X.hi_dirichlet || u_in != u), xh = xwall && i == nx - 1;
  const bool ywall = Y.walled && (Y.hi_dirichlet || v_in != v), yh = ywall && j == ny - 1;
  const bool zwall = Z.walled && (Z.hi_dirichlet || w_in != w);
  const int dx = i > 0 ? -1 : X.walled ? 0 : nx - 1;           // the low x and y neighbours of Phi
  const long long dy = j > 0 ? -nx : Y.walled ? 0 : plane - nx;
  const double idx = X.inv_dc[i], idy = Y.inv_dc[j];
  // the inputs of one plane; the next plane's are read before this one's
  // results are stored, so a thread keeps two planes' reads in flight
  struct In {
    double ph, phx, phy, u0, v0, w0, p0, uh, vh, wh;
  };
  auto face_u = [&](int k) { return (long long)ux * (j + (long long)ny * k) + i; };
  auto face_v = [&](int k) { return i + (long long)nx * (j + (long long)vy * k); };
  auto load = [&](int k) {
    In r;
    const long long c = col + plane * k;
    r.ph = phi[c];
    r.phx = phi[c + dx];
    r.phy = phi[c + dy];
    const long long fu = face_u(k), fv = face_v(k);
    r.u0 = __builtin_nontemporal_load(&u_in[fu]);
    r.v0 = __builtin_nontemporal_load(&v_in[fv]);
    r.w0 = __builtin_nontemporal_load(&w_in[c]);
    r.p0 = __builtin_nontemporal_load(&p[c]);
    r.uh = r.vh = r.wh = 0.0;
    if (xwall) r.uh = u_in[fu + (xh ? 1 : 0)];
    if (ywall) r.vh = v_in[fv + (yh ? nx : 0)];
    if (zwall && k == nz - 1) r.wh = w_in[c + plane];
    return r;
  };
  // Phi below the first plane: the plane under it, the periodic wrap, or none (a wall)
  double below = 0.0;
  if (k0 > 0) below = phi[col + plane * (k0 - 1)];
  else if (!Z.walled) below = phi[col + plane * (nz - 1)];
  In cur = load(k0);
  for (int k = k0; k < kend; ++k) {
    In nxt = cur;
    if (k + 1 < kend) nxt = load(k + 1);
    const long long c = col + plane * k;
    const double ph = cur.ph;
    // low-face gradients; a Neumann wall face keeps its velocity
    const bool zl = Z.walled && k == 0;
    const double gx = (xl ? 2.0 * ph : ph - cur.phx) * idx;
    const double gy = (yl ? 2.0 * ph : ph - cur.phy) * idy;
    const double gz = (zl ? 2.0 * ph : ph - below) * Z.inv_dc[k];
    const long long fu = face_u(k), fv = face_v(k);
    __builtin_nontemporal_store(xkeep ? cur.u0 : cur.u0 - gdt * gx, &u[fu]);
    __builtin_nontemporal_store(ykeep ? cur.v0 : cur.v0 - gdt * gy, &v[fv]);
    __builtin_nontemporal_store(zl && !Z.lo_dirichlet ? cur.w0 : cur.w0 - gdt * gz, &w[c]);
    // high wall faces: Dirichlet gradient -2 phi_edge / h_edge; Neumann unchanged
    if (xwall && xh) u[fu + 1] = X.hi_dirichlet ? cur.uh - gdt * (-2.0 * ph * X.inv_dc[nx]) : cur.uh;
    if (ywall && yh) v[fv + nx] = Y.hi_dirichlet ? cur.vh - gdt * (-2.0 * ph * Y.inv_dc[ny]) : cur.vh;
    if (zwall && k == nz - 1)
      w[c + plane] = Z.hi_dirichlet ? cur.wh - gdt * (-2.0 * ph * Z.inv_dc[nz]) : cur.wh;
    __builtin_nontemporal_store(cur.p0 + ph, &p[c]);
    below = ph;
    cur = nxt;
  }
}

}  // namespace poisson_dev
