// Many steps of one tiny domain in a single workgroup (included by
// hlbm_device.hpp after the walls).
//
// A domain of a thousand nodes leaves the row sweeps nothing to overlap: a step
// is one launch of a few workgroups that wait on their own pipeline, and a second
// launch with walls (Couette 2 x 100 FP64: 13.6 us a step; here 2.4).  One workgroup
// keeps the whole domain, populations in registers and what neighbours read in
// LDS, and runs all steps of a call: moments, a barrier, collision, a barrier,
// streaming and entropy, a barrier (and the walls with one more).  One compute
// unit's instruction rate and the chain of dependent operations of a step bound
// it; it is used up to kResidentNodes nodes.
//
// Clamped axes: a ghost node beyond an edge carries the state of the nearest
// node, and its collision sees ghosts in turn, so the ghosts at distance one
// are nodes of the collision stage ("extended" nodes), listed after the domain's
// own.  The per-node arithmetic is the sweeps', in the same order.
#pragma once

namespace hlbm {
namespace HLBM_NS {

constexpr int kResidentThreads = 512;

struct ResidentArgs {
  DomainArgs d;
  const real *src;
  real *dst;           // may be src: a thread reads and writes its own nodes only
  unsigned *status;
  int steps, next;  // next: extended nodes
};

// Arrays of one domain, moments by node (row-major nx x ny), populations 1..8
// after collision by extended node (row-major over the domain grown by one on
// its clamped axes).
template <int CAP>
struct ResidentLDS {
  real ux[CAP], uy[CAP], gx[CAP], gy[CAP], lap[CAP], s[CAP];
  real dr[CAP], pxx[CAP], pyy[CAP], pxy[CAP];
  real f[8][CAP];
};

template <int K>
__global__ __launch_bounds__(kResidentThreads) __attribute__((amdgpu_waves_per_eu(2)))
void k_resident(ResidentArgs a) {
  __shared__ ResidentLDS<K * kResidentThreads> L;
  const DomainArgs &d = a.d;
  const int nx = d.nx, ny = d.ny, N = nx * ny;
  const int gx = d.bcx != 0, gy = d.bcy != 0;  // ghost columns and rows
  const int EX = nx + 2 * gx;                  // extended row
  const bool walls = d.bcy == kBcWall;
  // per slot: coordinates (ghosts: -1, nx, ny), and the neighbours' rows and
  // columns (rows as offsets) for the moments; columns and rows of the extended
  // grid for the populations
  int px[K], py[K];
  bool node[K], ext[K];
  real F[K][kPlanes];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int i = (int)threadIdx.x + k * kResidentThreads;
    node[k] = i < N;
    ext[k] = i < a.next;
    px[k] = py[k] = 0;
    if (node[k]) {
      py[k] = i / nx;
      px[k] = i - py[k] * nx;
      const long long o = (long long)py[k] * d.pitch + px[k];
#pragma unroll
      for (int q = 0; q < kPlanes; ++q) F[k][q] = a.src[q * d.plane + o];
    } else if (ext[k]) {  // rows -1 and ny (whole extended rows), then columns -1 and nx
      int r = i - N;
      if (gy && r < 2 * EX) {
        py[k] = r < EX ? -1 : ny;
        px[k] = (r < EX ? r : r - EX) - gx;
      } else {
        r -= gy ? 2 * EX : 0;
        px[k] = r < ny ? -1 : nx;
        py[k] = r < ny ? r : r - ny;
      }
    }
  }
  auto col = [&](int x) { return map_index(x, nx, d.bcx); };
  auto row = [&](int y) { return map_index(y, ny, d.bcy) * nx; };
  auto fcol = [&](int x) { return gx ? x + 1 : map_index(x, nx, 0); };
  auto frow = [&](int y) { return (gy ? y + 1 : map_index(y, ny, 0)) * EX; };
  int cw[K], cc[K], ce[K], rs[K], rc[K], rn[K];      // moments
  int cww[K], cee[K], rss[K], rnn[K];                // s two nodes away
  int fw[K], fc[K], fe[K], fs[K], fr[K], fn[K];      // populations
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int x = px[k], y = py[k];
    cww[k] = col(x - 2);
    cw[k] = col(x - 1);
    cc[k] = col(x);
    ce[k] = col(x + 1);
    cee[k] = col(x + 2);
    rss[k] = row(y - 2);
    rs[k] = row(y - 1);
    rc[k] = row(y);
    rn[k] = row(y + 1);
    rnn[k] = row(y + 2);
    fw[k] = node[k] ? fcol(x - 1) : 0;
    fc[k] = ext[k] ? fcol(x) : 0;
    fe[k] = node[k] ? fcol(x + 1) : 0;
    fs[k] = node[k] ? frow(y - 1) : 0;
    fr[k] = ext[k] ? frow(y) : 0;
    fn[k] = node[k] ? frow(y + 1) : 0;
  }
  Health health;
  for (int step = 0; step < a.steps; ++step) {
    // ---------------- A: moments of the domain's nodes
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (!node[k]) continue;
      real Fk[kQ], gam_x, gam_y;
#pragma unroll
      for (int q = 0; q < kQ; ++q) Fk[q] = F[k][q];
      const NodeState o = node_state(d, Fk, F[k][9], health, gam_x, gam_y);
      const int i = rc[k] + cc[k];
      L.ux[i] = o.ux;
      L.uy[i] = o.uy;
      L.gx[i] = gam_x;
      L.gy[i] = gam_y;
      L.lap[i] = o.lapv;
      L.s[i] = F[k][9];
      L.dr[i] = o.dr;
      L.pxx[i] = o.pxx;
      L.pyy[i] = o.pyy;
      L.pxy[i] = o.pxy;
    }
    __syncthreads();
    // ---------------- B: collision of the extended nodes
    real f0[K], heat[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (!ext[k]) continue;
      const int c = rc[k] + cc[k], e = rc[k] + ce[k], w = rc[k] + cw[k];
      const int n = rn[k] + cc[k], s = rs[k] + cc[k];
      const NodeState o{L.dr[c], L.ux[c], L.uy[c], L.lap[c], L.pxx[c], L.pyy[c], L.pxy[c]};
      const NodeStencil st{L.ux[e], L.ux[w], L.ux[n], L.ux[s], L.uy[e], L.uy[w], L.uy[n],
                           L.uy[s], L.gx[e], L.gx[c], L.gx[w], L.gy[n], L.gy[c], L.gy[s]};
      const bool wall_row = walls && (py[k] == 0 || py[k] == ny - 1);
      real f[kQ], phi, pt;
      collide(d, o, st, wall_row ? real(1) : d.sigma, wall_row ? real(0) : d.sigma1, f, phi, pt);
      const int j = fr[k] + fc[k];
#pragma unroll
      for (int q = 1; q < kQ; ++q) L.f[q - 1][j] = f[q];
      f0[k] = f[0];
      heat[k] = heat_term(d, laplacian(L.lap[c], L.lap[e], L.lap[w], L.lap[n], L.lap[s]), phi, pt);
    }
    __syncthreads();
    // ---------------- C: streaming and entropy
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (!node[k]) continue;
      F[k][0] = f0[k];
      F[k][1] = L.f[0][fr[k] + fw[k]];
      F[k][2] = L.f[1][fs[k] + fc[k]];
      F[k][3] = L.f[2][fr[k] + fe[k]];
      F[k][4] = L.f[3][fn[k] + fc[k]];
      F[k][5] = L.f[4][fs[k] + fw[k]];
      F[k][6] = L.f[5][fs[k] + fe[k]];
      F[k][7] = L.f[6][fn[k] + fe[k]];
      F[k][8] = L.f[7][fn[k] + fw[k]];
      const int c = rc[k] + cc[k];
      const real sc = F[k][9];
      const real sw = L.s[rc[k] + cw[k]], se = L.s[rc[k] + ce[k]];
      const real ss = L.s[rs[k] + cc[k]], sn = L.s[rn[k] + cc[k]];
      const real ax = muscl(L.ux[c], sw - L.s[rc[k] + cww[k]], sc - sw, se - sc,
                            L.s[rc[k] + cee[k]] - se);
      const real ay = muscl(L.uy[c], ss - L.s[rss[k] + cc[k]], sc - ss, sn - sc,
                            L.s[rnn[k] + cc[k]] - sn);
      F[k][9] = sc - (ax + ay) + heat[k];
    }
    __syncthreads();
    if (walls) {
      // the new velocities of the two rows inside each wall (in the arrays of u,
      // which the next A writes anew), then the wall rows
#pragma unroll
      for (int k = 0; k < K; ++k) {
        if (!node[k]) continue;
        const int y = py[k];
        if (y == 1 || y == 2 || y == ny - 2 || y == ny - 3) {
          real G[kQ];
#pragma unroll
          for (int q = 0; q < kQ; ++q) G[q] = F[k][q];
          const NodeMoments m = node_moments(G, d);
          L.ux[rc[k] + cc[k]] = m.jx / m.rho;
          L.uy[rc[k] + cc[k]] = m.jy / m.rho;
        }
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < K; ++k) {
        if (!node[k]) continue;
        const int y = py[k];
        if (y == 0 || y == ny - 1) {
          const int side = y == 0 ? 0 : 1, dir = side ? -1 : 1;
          const int i1 = (y + dir) * nx + cc[k], i2 = (y + 2 * dir) * nx + cc[k];
          wall_rebuild(d, side, F[k], L.ux[i1], L.uy[i1], L.ux[i2], L.uy[i2]);
        }
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (!node[k]) continue;
    const long long o = (long long)py[k] * d.pitch + px[k];
#pragma unroll
    for (int q = 0; q < kPlanes; ++q) a.dst[q * d.plane + o] = F[k][q];
  }
  if (health.bad()) atomicOr(a.status, 1u);
}

}  // namespace HLBM_NS
}  // namespace hlbm
