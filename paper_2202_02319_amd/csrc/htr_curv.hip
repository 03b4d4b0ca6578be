// General curvilinear grids (Methods › Numerical method, the mapped equations): metric terms,
// sensor, mapped face fluxes and the stage update of a single-grid context.
//
// The equations are mapped to a uniform index space with U~ = U/J and
// F~_d = (d xi_d / d x) . (F, G, H) / J along each index direction,
// J = det(d xi / d x), index spacing 1.  Metric terms are evaluated in the
// conservative form of Thomas & Lombard,
//   (d xi_d / d x_c) / J = D_f[(D_e x_c1) x_c2] - D_e[(D_f x_c1) x_c2],
// (d, e, f) and (c, c1, c2) cyclic, D the sixth-order central difference,
// with the face values at i+1/2 the six-point interpolation whose face
// difference is D: the sum over directions of face-metric differences is a
// sum of commuting second differences, so a uniform flow stays uniform.
//
// Per stage: k_point (CURV variant: laser over lattice images, contravariant
// dt limit, volume 1/J) -> sensor -> convective face kernel (the hybrid scheme
// on the metric-projected flux, one launch per direction) -> diffusive flux by
// the chain rule with the flux differences and the stage update, on tiles.
#include <hip/hip_runtime.h>

#include "htr_dev.h"
#include "htr_flux.h"

namespace htr {

__device__ __forceinline__ long long lin(const Member& G, int i, int j, int k) {
  return ((long long)k * G.n[1] + j) * G.n[0] + i;
}

// Coordinate c of lattice node (i, j, k), any integers (a node n[a] cells
// further along a is displaced by P[a]), minus x0.
__device__ __forceinline__ double lat(const Member& G, const CurvGeom& g, int c, int i, int j, int k, double x0) {
  const int id[3] = {i, j, k};
  int w[3];
  double sh = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    w[a] = wrapi(id[a], G.n[a]);
    sh += (double)((id[a] - w[a]) / G.n[a]) * g.P[a][c];
  }
  return (g.xyz[c * G.N + lin(G, w[0], w[1], w[2])] + sh) - x0;
}

__device__ __forceinline__ void step(int p[3], const int b[3], int e, int m) {
  p[0] = b[0];
  p[1] = b[1];
  p[2] = b[2];
  p[e] += m;
}

// D6 along e of coordinate c (relative to x0) at lattice point b.
__device__ double d6x(const Member& G, const CurvGeom& g, int c, const int b[3], int e, double x0) {
  const double w[3] = {45.0, -9.0, 1.0};
  double s = 0.0;
  for (int m = 1; m <= 3; ++m) {
    int pp[3], pm[3];
    step(pp, b, e, m);
    step(pm, b, e, -m);
    s += w[m - 1] * (lat(G, g, c, pp[0], pp[1], pp[2], x0) - lat(G, g, c, pm[0], pm[1], pm[2], x0));
  }
  return s / 60.0;
}

// D6 along o of the product (D6_e x_c1) x_c2 at lattice point b.
__device__ double d6prod(const Member& G, const CurvGeom& g, int c1, int c2, const int b[3], int e, int o,
                         const double x0[3]) {
  const double w[3] = {45.0, -9.0, 1.0};
  double s = 0.0;
  for (int m = 1; m <= 3; ++m) {
    int pp[3], pm[3];
    step(pp, b, o, m);
    step(pm, b, o, -m);
    const double fp = d6x(G, g, c1, pp, e, x0[c1]) * lat(G, g, c2, pp[0], pp[1], pp[2], x0[c2]);
    const double fm = d6x(G, g, c1, pm, e, x0[c1]) * lat(G, g, c2, pm[0], pm[1], pm[2], x0[c2]);
    s += w[m - 1] * (fp - fm);
  }
  return s / 60.0;
}

// J = 1 / det(d x / d xi) at row 9, or 0 where the determinant is not
// positive and finite (the host checks every node before accepting the grid).
__global__ __launch_bounds__(BLK) void k_curv_metrics(const Member* __restrict__ mem, CurvGeom g,
                                                      double* __restrict__ mt) {
  const Member& G = mem[0];
  const long long q = (long long)blockIdx.x * BLK + threadIdx.x;
  if (q >= G.N) return;
  const long long N = G.N;
  const int b[3] = {(int)(q % G.n[0]), (int)((q / G.n[0]) % G.n[1]), (int)(q / ((long long)G.n[0] * G.n[1]))};
  double x0[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) x0[c] = g.xyz[c * N + q];
  for (int d = 0; d < 3; ++d) {
    const int e = (d + 1) % 3, f = (d + 2) % 3;
    for (int c = 0; c < 3; ++c) {
      const int c1 = (c + 1) % 3, c2 = (c + 2) % 3;
      mt[(3 * d + c) * N + q] = d6prod(G, g, c1, c2, b, e, f, x0) - d6prod(G, g, c1, c2, b, f, e, x0);
    }
  }
  double A[3][3];
  for (int c = 0; c < 3; ++c)
    for (int e = 0; e < 3; ++e) A[c][e] = d6x(G, g, c, b, e, x0[c]);
  const double det = A[0][0] * (A[1][1] * A[2][2] - A[1][2] * A[2][1]) -
                     A[0][1] * (A[1][0] * A[2][2] - A[1][2] * A[2][0]) +
                     A[0][2] * (A[1][0] * A[2][1] - A[1][1] * A[2][0]);
  mt[9 * N + q] = (det > 0.0 && isfinite(det)) ? 1.0 / det : 0.0;
}

// Face values along d at row 9 d: mf the metric vector, gf the face mean of
// d xi_e / d x_b (row 9 d + 3 k + b, axes e = d, d + 1, d + 2 in turn).
__global__ __launch_bounds__(BLK) void k_curv_face_metrics(const Member* __restrict__ mem,
                                                           const double* __restrict__ mt, double* __restrict__ mf,
                                                           double* __restrict__ gf) {
  const Member& G = mem[0];
  const long long q = (long long)blockIdx.x * BLK + threadIdx.x;
  if (q >= G.N) return;
  const long long N = G.N;
  const int b[3] = {(int)(q % G.n[0]), (int)((q / G.n[0]) % G.n[1]), (int)(q / ((long long)G.n[0] * G.n[1]))};
  const double cw[6] = {1.0, -8.0, 37.0, 37.0, -8.0, 1.0};
  for (int d = 0; d < 3; ++d) {
    long long st[6];
    for (int m = 0; m < 6; ++m) {
      int p[3] = {b[0], b[1], b[2]};
      p[d] = wrapi(b[d] - 2 + m, G.n[d]);
      st[m] = lin(G, p[0], p[1], p[2]);
    }
    for (int c = 0; c < 3; ++c) {
      double s = 0.0;
      for (int m = 0; m < 6; ++m) s += cw[m] * mt[(3 * d + c) * N + st[m]];
      mf[(3 * d + c) * N + q] = s / 60.0;
    }
    const double Ja = mt[9 * N + q], Jb = mt[9 * N + st[3]];
    for (int k = 0; k < 3; ++k) {
      const int e = (d + k) % 3;
      for (int c = 0; c < 3; ++c)
        gf[(9 * d + 3 * k + c) * N + q] = 0.5 * (Ja * mt[(3 * e + c) * N + q] + Jb * mt[(3 * e + c) * N + st[3]]);
    }
  }
}

// theta = (div u)^2 / ((div u)^2 + |curl u|^2 + 1e-300), second-order central
// differences through the chain rule d/dx_b = sum_a J mt[3a + b] d/d xi_a.
__global__ __launch_bounds__(BLK) void k_curv_sensor(const Member* __restrict__ mem, CurvGeom g,
                                                     const double* __restrict__ aux,
                                                     unsigned char* __restrict__ flag, double theta_c,
                                                     double* __restrict__ theta_out, int nq) {
  const Member& G = mem[0];
  const long long q = (long long)blockIdx.x * BLK + threadIdx.x;
  if (q >= G.N) return;
  const long long N = G.N;
  const double* vel = aux + 4 * N;
  const int c[3] = {(int)(q % G.n[0]), (int)((q / G.n[0]) % G.n[1]), (int)(q / ((long long)G.n[0] * G.n[1]))};
  const long long stride[3] = {1, G.n[0], (long long)G.n[0] * G.n[1]};
  const double Jq = g.mt[9 * N + q];
  double gr[3][3];
#pragma unroll
  for (int b = 0; b < 3; ++b)
#pragma unroll
    for (int m = 0; m < 3; ++m) gr[b][m] = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (!G.act[a]) continue;
    const long long qp = q + (wrapi(c[a] + 1, G.n[a]) - c[a]) * stride[a];
    const long long qm = q + (wrapi(c[a] - 1, G.n[a]) - c[a]) * stride[a];
    double du[3];
#pragma unroll
    for (int m = 0; m < 3; ++m) du[m] = vel[m * N + qp] - vel[m * N + qm];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const double mab = Jq * g.mt[(3 * a + b) * N + q];
#pragma unroll
      for (int m = 0; m < 3; ++m) gr[b][m] += mab * du[m] / 2.0;
    }
  }
  const double div = gr[0][0] + gr[1][1] + gr[2][2];
  const double wx = gr[1][2] - gr[2][1], wy = gr[2][0] - gr[0][2], wz = gr[0][1] - gr[1][0];
  const double d2 = div * div;
  const double th = d2 / (d2 + wx * wx + wy * wy + wz * wz + 1e-300);
  flag[q] = th > theta_c ? 1 : 0;
  if (theta_out) theta_out[(nq - 1) * N + q] = th;
}

// Mapped convective flux through face i+1/2 along d, stored at node i: the
// hybrid switch of the rectilinear sweep (TENO where a stencil node's sensor
// is set or the pressure jump across the face is large), central six-point
// flux or TENO6 / WENO3-Z on the local Lax-Friedrichs split with
// alpha = max |u . n| + c |n| over the stencil, of the physical flux
// projected on the face metric vector n (held fixed on the stencil).
//
// One block per tile of faces: CA faces along d by CB along the companion
// axis o (x, or y when d is x), one plane r of the remaining axis.  The
// tile's nodes and a 2 + 3 node halo along d are staged in LDS in one pass,
// the conserved variables with velocity, p, c and the sensor flags, behind
// a single barrier (staging the variables one at a time through a double
// buffer, one barrier each, took 1.05 against 0.78 ms at 128^3 then: the block
// waited on each variable's loads in turn).  Each face then keeps u . n, p,
// the switch and alpha in registers and works through the variables from
// LDS.  Every node value is loaded once per block, coalesced along x.
template <int NS, int CA, int CB, bool DX>
__global__ __launch_bounds__(BLK) void k_curv_conv(const Member* __restrict__ mem, CurvGeom g, int d, unsigned flags,
                                                   const double* __restrict__ U, const double* __restrict__ aux,
                                                   const unsigned char* __restrict__ flg, double* __restrict__ ffc,
                                                   double psi_c, double CT) {
  static_assert(CA * CB == BLK, "one face per thread");
  constexpr int NV = NS + 4;
  constexpr int NA = CA + 5;   // staged nodes along d
  constexpr int NB = NA * CB;  // staged nodes
  __shared__ double s_un[3][NB];   // velocity
  __shared__ double s_p[NB], s_c[NB];
  __shared__ unsigned char s_f[NB];
  __shared__ double s_U[NS + 4][NB];
  __shared__ double s_tab[16][6];   // TENO6 coefficients of every cut-off pattern
  teno6_table(threadIdx.x, s_tab);
  const Member& G = mem[0];
  const long long N = G.N;
  // axes: d (faces), o (companion), r (plane)
  const int o = DX ? 1 : 0;
  const int r = 3 - d - o;
  const int nto = (G.n[o] + CB - 1) / CB;
  const int nta = (G.n[d] + CA - 1) / CA;
  // each XCD a contiguous run of tiles (blocks are dealt to the eight of them
  // round-robin), so that neighbours share its L2: the three launches of a
  // stage 598 -> 568 us at 128^3 cells, nine species
  const int per = gridDim.x >> 3;
  int b = (int)blockIdx.x < 8 * per ? (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
  const int to = b % nto;
  b /= nto;
  const int ta = b % nta;
  const int pr = b / nta;
  const int a0 = ta * CA, o0 = to * CB;
  const long long stride[3] = {1, G.n[0], (long long)G.n[0] * G.n[1]};
  // staged slot of node (k along d, j along o): x-consecutive threads read
  // consecutive slots (DX: k is along x; otherwise j is)
  auto slot = [](int k, int j) { return DX ? j * NA + k : k * CB + j; };
  auto node = [&](int k, int j) -> long long {
    const int ad = wrapi(a0 - 2 + k, G.n[d]);
    const int ao = wrapi(o0 + j, G.n[o]);
    return (long long)ad * stride[d] + (long long)ao * stride[o] + (long long)pr * stride[r];
  };
  for (int e = threadIdx.x; e < NB; e += BLK) {
    const int k = DX ? e % NA : e / CB, j = DX ? e / NA : e % CB;
    const long long q = node(k, j);
    const int sl = slot(k, j);
#pragma unroll
    for (int v = 0; v < NV; ++v) s_U[v][sl] = U[v * N + q];
    s_un[0][sl] = aux[4 * N + q];
    s_un[1][sl] = aux[5 * N + q];
    s_un[2][sl] = aux[6 * N + q];
    s_p[sl] = aux[q];
    s_c[sl] = aux[N + q];
    s_f[sl] = flg[q];
  }
  // this thread's face
  const int fa = DX ? threadIdx.x % CA : threadIdx.x / CB;
  const int fo = DX ? threadIdx.x / CA : threadIdx.x % CB;
  const bool live = a0 + fa < G.n[d] && o0 + fo < G.n[o];
  const long long qf = (long long)(a0 + fa) * stride[d] + (long long)(o0 + fo) * stride[o] + (long long)pr * stride[r];
  double n0 = 0.0, n1 = 0.0, n2 = 0.0;
  if (live) {
    n0 = g.mf[(3 * d) * N + qf];
    n1 = g.mf[(3 * d + 1) * N + qf];
    n2 = g.mf[(3 * d + 2) * N + qf];
  }
  __syncthreads();
  double un[6], pm[6];
  bool anyflag = false;
  double alpha = -1.0;
  const double nn = sqrt(n0 * n0 + n1 * n1 + n2 * n2);
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    const int sl = slot(fa + m, fo);
    un[m] = s_un[0][sl] * n0 + s_un[1][sl] * n1 + s_un[2][sl] * n2;
    pm[m] = s_p[sl];
    anyflag = anyflag || s_f[sl] != 0;
    alpha = fmax(alpha, fabs(un[m]) + s_c[sl] * nn);
  }
  bool teno;
  if (flags & HTR_FORCE_TENO) teno = true;
  else if (flags & HTR_FORCE_CENTRAL) teno = false;
  else teno = anyflag || (fabs(pm[3] - pm[2]) / fmin(pm[2], pm[3]) > psi_c);
  const bool weno = (flags & HTR_WENO3Z) != 0;
  double* out = ffc + (long long)d * NV * N;
#pragma unroll 1
  for (int v = 0; v < NV; ++v) {
    if (live) {
      double f[6], Uv[6];
#pragma unroll
      for (int m = 0; m < 6; ++m) {
        Uv[m] = s_U[v][slot(fa + m, fo)];
        if (v < NS) f[m] = Uv[m] * un[m];
        else if (v < NS + 3) f[m] = Uv[m] * un[m] + pm[m] * (v == NS ? n0 : (v == NS + 1 ? n1 : n2));
        else f[m] = (Uv[m] + pm[m]) * un[m];
      }
      double res;
      if (!teno) {
        const double cc[6] = {1.0, -8.0, 37.0, 37.0, -8.0, 1.0};
        double sacc = 0.0;
#pragma unroll
        for (int m = 0; m < 6; ++m) sacc += cc[m] * f[m];
        res = sacc / 60.0;
      } else {
        double hp[6], hmr[6];
#pragma unroll
        for (int m = 0; m < 6; ++m) {
          hp[m] = fma(alpha, Uv[m], f[m]);
          hmr[5 - m] = fma(-alpha, Uv[m], f[m]);
        }
        res = weno ? weno3z_h(hp) + weno3z_h(hmr) : teno6_face(s_tab, hp, hmr, CT);
      }
      out[v * N + qf] = res;
    }
  }
}

constexpr int CBOX = 10 * 10 * 6;   // a tile with its layer: 3-D the largest (2-D 18 x 18, 1-D 258)

// Tile of the diffusive kernel: BLK cells over the active axes.  On a 3-D grid
// the shape of least tiles, those with rows of four counted a quarter more
// (83x61x37 cells, nine species: 101 us a launch in 840 tiles of 4 x 8 x 8, 82
// in 880 of 8 x 8 x 4; 2x256x256 70 us in 1024 and 124 in 2048).  A grid of at
// most four cells along every axis but one fills few of a tile's threads, and
// takes the longest tile that the block can stage (BLK nodes beside its faces,
// 64 faces of a last layer, CBOX nodes): 16384x2x2 cells 58 us in 31 x 2 x 2,
// 117 in 8 x 8 x 4; 16384x2 25 us in 64 x 2, 51 in 16 x 16.
static void curv_tile(const int act[3], const int n[3], int T[3]) {
  const int na = (act[0] != 0) + (act[1] != 0) + (act[2] != 0);
  for (int a = 0; a < 3; ++a) T[a] = act[a] ? (na == 2 ? 16 : BLK) : 1;
  if (na == 0) T[0] = BLK;
  if (na < 2) return;
  auto tiles = [&](const int t[3]) {
    long long w = 1;
    for (int a = 0; a < 3; ++a) w *= (n[a] + t[a] - 1) / t[a];
    return w;
  };
  constexpr int shapes[3][3] = {{8, 8, 4}, {8, 4, 8}, {4, 8, 8}}, weight[3] = {4, 4, 5};
  long long best = 4 * tiles(T);
  for (int k = 0; k < 3 && na == 3; ++k) {
    const long long w = weight[k] * tiles(shapes[k]);
    if (k > 0 && w >= best) continue;
    best = w;
    for (int a = 0; a < 3; ++a) T[a] = shapes[k][a];
  }
  for (int d = 0; d < 3; ++d) {
    int t[3];
    bool thin = act[d];
    for (int a = 0; a < 3; ++a) {
      thin = thin && (a == d || n[a] <= 4);
      t[a] = act[a] ? n[a] : 1;
    }
    if (!thin) continue;
    auto fits = [&] {
      const int cells = t[0] * t[1] * t[2];
      int beside = 0, box = 1, most = 0;
      for (int a = 0; a < 3; ++a)
        if (act[a]) {
          beside += 2 * (cells / t[a]);
          box *= t[a] + 2;
          most = cells / t[a] > most ? cells / t[a] : most;
        }
      return cells <= BLK && beside <= BLK && box <= CBOX && most <= 64;
    };
    for (t[d] = 64; t[d] > 1 && !fits();) --t[d];
    if (4 * tiles(t) < best) {
      best = 4 * tiles(t);
      for (int a = 0; a < 3; ++a) T[a] = t[a];
    }
  }
}

// Mapped diffusive fluxes, their and the convective ones' differences, and the
// stage update: dU/dt = src + J sum_d (F_d(i) - F_d(i - e_d)), F the diffusive
// minus the convective flux; out = dU/dt (rhs_only) or the stage combination
// ca U^n + cb (U + dt dU/dt).  The diffusive flux at a face: index-space
// derivatives (normal from the two nodes, tangential the mean of the two nodal
// central differences), physical gradients by the chain rule with gf, the flux
// vector projected on the face metric vector; arithmetic-mean coefficients.
//
// One block per tile, one cell per thread: thread t has the lower face of its
// cell along every axis, and the lanes of wavefront d + 1 the upper faces of
// the tile's last layer along d.  The fields pass through LDS on the tile and
// one layer around it (with its edges: the tangential differences), a few rows
// at a time.  A species' normal derivatives are kept until the correction flux
// is known, so its mole fraction is staged once.
//
// Bound by the latency of its staged phases at two blocks per CU (250
// registers, 61 KB of LDS); each group of loads is issued a group ahead (766 us
// at 128^3 cells and nine species, 858 with each waited for in its turn; the
// metrics a face ahead as well: no change).
// Mole fractions, index-space differences, face fluxes and update as four
// launches through memory (about 330 values a cell written and read back) took
// 65 + 258 + 1450 + 446 us.
template <int NS>
__global__ __launch_bounds__(BLK, 2) void k_curv_diff(const MechTables* __restrict__ M, const Member* __restrict__ mem,
                                                      CurvGeom g, CallArgs A, int3 tile,
                                                      const double* __restrict__ U,
                                                      const double* Un, const double* __restrict__ Tf,
                                                      const double* __restrict__ aux, const double* __restrict__ src,
                                                      const double* __restrict__ ffc, double* out, double ca,
                                                      double cb, int rhs_only) {
  constexpr int NV = NS + 4;
  __shared__ double s_n[8][CBOX], s_F[3][3][DFACE];
  const Member& G = mem[0];
  const int t = threadIdx.x;
  const long long N = G.N;
  const bool act[3] = {G.act[0] != 0, G.act[1] != 0, G.act[2] != 0};
  const int T[3] = {tile.x, tile.y, tile.z}, cells = T[0] * T[1] * T[2];
  int nt[3], o[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) nt[a] = (G.n[a] + T[a] - 1) / T[a];
  tile_origin_of(T, nt, gridDim.x, blockIdx.x, o);
  const int tc = t < cells ? t : 0;   // threads past a long tile's cells repeat its first
  const int l[3] = {tc % T[0], (tc / T[0]) % T[1], tc / (T[0] * T[1])};
  const int gc[3] = {o[0] + l[0], o[1] + l[1], o[2] + l[2]};
  const bool valid = t < cells && gc[0] < G.n[0] && gc[1] < G.n[1] && gc[2] < G.n[2];
  // grid index of the node at h in the tile (-1 .. T along an active axis)
  auto node = [&](int h0, int h1, int h2) {
    return lin(G, wrapi(o[0] + h0, G.n[0]), wrapi(o[1] + h1, G.n[1]), wrapi(o[2] + h2, G.n[2]));
  };
  const long long qc = node(l[0], l[1], l[2]);
  const double Jc = g.mt[9 * N + qc], dt = rhs_only ? 0.0 : A.dt_dev[0];
  struct Row { double s, u, un; };
  auto row = [&](int v) {
    return Row{v < NS ? src[v * N + qc] : (v == NS + 3 ? src[NS * N + qc] : 0.0), U[v * N + qc],
               !rhs_only && ca != 0.0 ? Un[v * N + qc] : 0.0};
  };
  auto finish = [&](int v, const Row& r, double acc) {
    if (!valid) return;
    const double L = r.s + Jc * acc;
    if (rhs_only) {
      out[v * N + qc] = L;
    } else {
      const double base = r.u + dt * L;
      out[v * N + qc] = ca != 0.0 ? ca * r.un + cb * base : cb * base;
    }
  };
  // lower nodes of this thread's faces: 0-2 along each axis, 3 the extra one
  long long qf[4];
#pragma unroll
  for (int d = 0; d < 3; ++d) qf[d] = node(l[0] - (d == 0), l[1] - (d == 1), l[2] - (d == 2));
  if (A.flags & HTR_VISC_OFF) {
#pragma unroll 1
    for (int v = 0; v < NV; ++v) {
      const Row r = row(v);
      double acc = 0.0;
#pragma unroll
      for (int d = 0; d < 3; ++d)
        if (act[d]) acc -= ffc[(d * NV + v) * N + qc] - ffc[(d * NV + v) * N + qf[d]];
      finish(v, r, acc);
    }
    return;
  }
  // box: strides, this cell's slot, and this thread's nodes of the layer: one
  // beside a face of the tile and one on its edges
  const int p[3] = {act[0] ? 1 : 0, act[1] ? 1 : 0, act[2] ? 1 : 0};
  const int st[3] = {p[0], p[1] ? T[0] + 2 * p[0] : 0, p[2] ? (T[0] + 2 * p[0]) * (T[1] + 2 * p[1]) : 0};
  auto slot = [&](int h0, int h1, int h2) {
    return p[0] * (h0 + 1) + st[1] * (h1 + 1) + st[2] * (h2 + 1);
  };
  const int sc = slot(l[0], l[1], l[2]);
  int sh = sc, se = sc;
  long long qh = qc, qe = qc;
  bool has_h = false, has_e = false;
  {
    int k = t;   // the layers below and above along each axis
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int S = cells / T[d], cnt = p[d] ? 2 * S : 0;
      if (k >= 0 && k < cnt) {
        const int x = k % S, w = k < S ? -1 : T[d], Te = d == 0 ? T[1] : T[0];
        const int x0 = x % Te, x1 = x / Te;
        const int h0 = d == 0 ? w : x0, h1 = d == 1 ? w : (d == 0 ? x0 : x1), h2 = d == 2 ? w : x1;
        qh = node(h0, h1, h2);
        sh = slot(h0, h1, h2);
        has_h = true;
      }
      k -= cnt;
    }
    k = t;   // the four edges along axis d, where the two others are active
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int a = d == 0 ? 1 : 0, b = d == 2 ? 1 : 2;
      const int cnt = p[a] && p[b] ? 4 * T[d] : 0;
      if (k >= 0 && k < cnt) {
        const int x = k % T[d], c = k / T[d];
        const int ha = c & 1 ? T[a] : -1, hb = c & 2 ? T[b] : -1;
        const int h0 = d == 0 ? x : ha, h1 = d == 1 ? x : (d == 0 ? ha : hb), h2 = d == 2 ? x : hb;
        qe = node(h0, h1, h2);
        se = slot(h0, h1, h2);
        has_e = true;
      }
      k -= cnt;
    }
  }
  // the extra face's direction (one per wavefront), its slots and strides
  const int xd = __builtin_amdgcn_readfirstlane(t >> 6) - 1, lane = t & 63;
  const bool has_x = xd >= 0 && (xd == 0 ? act[0] : (xd == 1 ? act[1] : act[2])) &&
                     lane < cells / (xd == 0 ? T[0] : (xd == 1 ? T[1] : T[2]));
  int sx = 0, xn = 0, x1 = 0, x2 = 0;
  qf[3] = qc;
  if (has_x) {
    const int Te = xd == 0 ? T[1] : T[0];
    const int y0 = lane % Te, y1 = lane / Te;
    const int h0 = xd == 0 ? T[0] - 1 : y0, h1 = xd == 1 ? T[1] - 1 : (xd == 0 ? y0 : y1),
              h2 = xd == 2 ? T[2] - 1 : y1;
    sx = slot(h0, h1, h2);
    qf[3] = node(h0, h1, h2);
    xn = xd == 0 ? st[0] : (xd == 1 ? st[1] : st[2]);
    x1 = xd == 0 ? st[1] : (xd == 1 ? st[2] : st[0]);
    x2 = xd == 0 ? st[2] : (xd == 1 ? st[0] : st[1]);
  }
  const int pos[3] = {l[1] + T[1] * l[2], l[0] + T[0] * l[2], l[0] + T[0] * l[1]};
  // where the upper face of this cell along d is in s_F[.][d]
  const int up[3] = {l[0] + 1 < T[0] ? t + 1 : BLK + pos[0], l[1] + 1 < T[1] ? t + T[0] : BLK + pos[1],
                     l[2] + 1 < T[2] ? t + T[0] * T[1] : BLK + pos[2]};
  auto on = [&](int k) { return k < 3 ? act[k] : has_x; };
  auto axis = [&](int k) { return k < 3 ? k : xd; };
  // upper node's slot and the strides normal and tangential to face k
  const int sB[4] = {sc, sc, sc, sx + xn};
  const int sn[4] = {st[0], st[1], st[2], xn}, s1[4] = {st[1], st[2], st[0], x1}, s2[4] = {st[2], st[0], st[1], x2};
  // derivative of a staged row along the face's three index axes
  auto dxi = [&](const double* r, int k, double de[3]) {
    const int b = sB[k], a = b - sn[k];
    de[0] = r[b] - r[a];
    de[1] = 0.25 * ((r[a + s1[k]] - r[a - s1[k]]) + (r[b + s1[k]] - r[b - s1[k]]));
    de[2] = 0.25 * ((r[a + s2[k]] - r[a - s2[k]]) + (r[b + s2[k]] - r[b - s2[k]]));
  };
  auto mean = [&](const double* r, int k) { return 0.5 * (r[sB[k] - sn[k]] + r[sB[k]]); };
  // rounds x before it meets another value (no operation of its own)
  auto rounded = [](double x) {
    asm("" : "+v"(x));
    return x;
  };
  auto put = [&](int z, auto val) {
#pragma unroll
    for (int d = 0; d < 3; ++d)
      if (act[d]) s_F[z][d][t] = val(d);
    if (has_x) s_F[z][xd][BLK + lane] = val(3);
  };
  auto difference = [&](int z, auto F) {
    double acc = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d)
      if (act[d]) acc += s_F[z][d][up[d]] - F(d);
    return acc;
  };
  // convective flux of row v at face k
  auto conv = [&](int v, int k) { return on(k) ? ffc[((long long)axis(k) * NV + v) * N + qf[k]] : 0.0; };
  auto stage = [&](double* r, const double* f, bool edges) {
    r[sc] = f[qc];
    if (has_h) r[sh] = f[qh];
    if (edges && has_e) r[se] = f[qe];
  };
  // velocity and viscosity
#pragma unroll
  for (int m = 0; m < 3; ++m) stage(s_n[m], aux + (4 + m) * N, true);
  stage(s_n[3], aux + 2 * N, false);
  double rc[NS], rh[NS], re[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    rc[s] = U[s * N + qc];
    rh[s] = U[s * N + qh];
    re[s] = U[s * N + qe];
  }
  double rhoc = 0.0, rhoh = 0.0, nc = 0.0, nh = 0.0, ne = 0.0;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    rhoc += rc[s];
    rhoh += rh[s];
    nc += rc[s] * M->iW[s];
    nh += rh[s] * M->iW[s];
    ne += re[s] * M->iW[s];
  }
  const double inc = 1.0 / nc, inh = 1.0 / nh, ine = 1.0 / ne, irc = 1.0 / rhoc, irh = 1.0 / rhoh;
  const double Tc = Tf[qc], Th = Tf[qh];
  __syncthreads();
  // a: the metric vector's components along the index gradients, so that
  // n . grad phi = sum a d phi / d xi; tau: n . stress
  double a[4][3], tau[4][3], en[4] = {}, k1[4] = {}, corr[4] = {};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    a[k][0] = a[k][1] = a[k][2] = tau[k][0] = tau[k][1] = tau[k][2] = 0.0;
    if (!on(k)) continue;
    const double* mf = g.mf + 3LL * axis(k) * N + qf[k];
    const double* gp = g.gf + 9LL * axis(k) * N + qf[k];
    double n[3], Gf[3][3], gu[3][3];   // gu[b][m] = d u_m / d x_b
#pragma unroll
    for (int b = 0; b < 3; ++b) n[b] = mf[b * N];
#pragma unroll
    for (int e = 0; e < 3; ++e) {
#pragma unroll
      for (int b = 0; b < 3; ++b) Gf[e][b] = gp[(3 * e + b) * N];
      a[k][e] = Gf[e][0] * n[0] + Gf[e][1] * n[1] + Gf[e][2] * n[2];
    }
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      double de[3];
      dxi(s_n[m], k, de);
#pragma unroll
      for (int b = 0; b < 3; ++b) gu[b][m] = Gf[0][b] * de[0] + Gf[1][b] * de[1] + Gf[2][b] * de[2];
    }
    const double mu = mean(s_n[3], k), divu = gu[0][0] + gu[1][1] + gu[2][2];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      double x = 0.0;
#pragma unroll
      for (int b = 0; b < 3; ++b) x += n[b] * (gu[b][m] + gu[m][b]);
      x = mu * (x - n[m] * ((2.0 / 3.0) * divu));
      en[k] += x * mean(s_n[m], k);
      tau[k][m] = rounded(x - conv(NS + m, k));
    }
  }
  // conduction and the species' face factor rho / W
  stage(s_n[4], Tf, true);
  stage(s_n[5], aux + 3 * N, false);
  s_n[6][sc] = rhoc;
  s_n[7][sc] = rhoc * inc;
  if (has_h) {
    s_n[6][sh] = rhoh;
    s_n[7][sh] = rhoh * inh;
  }
  Row mrow[3];
#pragma unroll
  for (int m = 0; m < 3; ++m) mrow[m] = row(NS + m);
  // a group's loads are issued before the one ahead of it is worked on
  double Dc[NS], Dh[NS];
  auto fetchD = [&](int s) {
    Dc[s] = aux[(7 + s) * N + qc];
    Dh[s] = aux[(7 + s) * N + qh];
  };
  fetchD(0);
  if (NS > 1) fetchD(1);
#pragma unroll
  for (int m = 0; m < 3; ++m) put(m, [&](int k) { return tau[k][m]; });
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (!on(k)) continue;
    double de[3];
    dxi(s_n[4], k, de);
    en[k] += mean(s_n[5], k) * (a[k][0] * de[0] + a[k][1] * de[1] + a[k][2] * de[2]);
    k1[k] = mean(s_n[6], k) / mean(s_n[7], k);
  }
#pragma unroll
  for (int m = 0; m < 3; ++m) finish(NS + m, mrow[m], difference(m, [&](int d) { return tau[d][m]; }));
  // species in twos, in alternating halves of the rows: rho D W_s / W n . grad X_s and their sum
  double gx[NS][4];
#pragma unroll
  for (int s0 = 0; s0 < NS; s0 += 2) {
    double(*R)[CBOX] = &s_n[(2 * s0) % 8];
#pragma unroll
    for (int j = 0; j < 2 && s0 + j < NS; ++j) {
      const int s = s0 + j;
      R[2 * j][sc] = rc[s] * M->iW[s] * inc;
      if (has_h) R[2 * j][sh] = rh[s] * M->iW[s] * inh;
      if (has_e) R[2 * j][se] = re[s] * M->iW[s] * ine;
      R[2 * j + 1][sc] = Dc[s];
      if (has_h) R[2 * j + 1][sh] = Dh[s];
    }
    __syncthreads();
#pragma unroll
    for (int j = 2; j < 4 && s0 + j < NS; ++j) fetchD(s0 + j);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
      for (int j = 0; j < 2 && s0 + j < NS; ++j) {
        gx[s0 + j][k] = 0.0;
        if (!on(k)) continue;
        double de[3];
        dxi(R[2 * j], k, de);
        gx[s0 + j][k] = k1[k] * (M->W[s0 + j] * mean(R[2 * j + 1], k)) *
                        (a[k][0] * de[0] + a[k][1] * de[1] + a[k][2] * de[2]);
        corr[k] += gx[s0 + j][k];
      }
    }
  }
  // each species' flux and its enthalpy; the energy row goes with the last ones
  const double iTc = 1.0 / Tc, iTh = 1.0 / Th;
  Row sr[NS];
  double fc[NS][4];
  auto fetch = [&](int s) {
    sr[s] = row(s);
#pragma unroll
    for (int k = 0; k < 4; ++k) fc[s][k] = conv(s, k);
  };
  fetch(0);
  if (NS > 1) fetch(1);
#pragma unroll
  for (int s0 = 0; s0 < NS; s0 += 2) {
    const bool last = s0 + 2 >= NS;
    double(*R)[CBOX] = &s_n[(2 * (s0 + NS + (NS & 1))) % 8];
    Row er{};
    double fe[4] = {};
#pragma unroll
    for (int j = 2; j < 4 && s0 + j < NS; ++j) fetch(s0 + j);
    if (last) {
      er = row(NS + 3);
#pragma unroll
      for (int k = 0; k < 4; ++k) fe[k] = conv(NS + 3, k);
    }
#pragma unroll
    for (int j = 0; j < 2 && s0 + j < NS; ++j) {
      const int s = s0 + j;
      R[2 * j][sc] = rc[s] * irc;
      R[2 * j + 1][sc] = M->RW[s] * Tc * hRTi(M, s, Tc, iTc);
      if (has_h) {
        R[2 * j][sh] = rh[s] * irh;
        R[2 * j + 1][sh] = M->RW[s] * Th * hRTi(M, s, Th, iTh);
      }
    }
    __syncthreads();
    double F[2][4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
      for (int j = 0; j < 2 && s0 + j < NS; ++j) {
        F[j][k] = 0.0;
        if (!on(k)) continue;
        const double f = gx[s0 + j][k] - mean(R[2 * j], k) * corr[k];
        en[k] += f * mean(R[2 * j + 1], k);
        F[j][k] = rounded(f - fc[s0 + j][k]);
      }
    }
#pragma unroll
    for (int j = 0; j < 2 && s0 + j < NS; ++j) put(j, [&](int k) { return F[j][k]; });
    if (last) {
#pragma unroll
      for (int k = 0; k < 4; ++k) en[k] = rounded(en[k] - fe[k]);
      put(2, [&](int k) { return en[k]; });
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2 && s0 + j < NS; ++j)
      finish(s0 + j, sr[s0 + j], difference(j, [&](int d) { return F[j][d]; }));
    if (last) finish(NS + 3, er, difference(2, [&](int d) { return en[d]; }));
  }
}

// ---------------------------------------------------------------- launchers
static inline int blocks_of(long long N) { return (int)((N + BLK - 1) / BLK); }

hipError_t launch_curv_metrics(const Member* mem, const Member& host, const CurvGeom& g, double* mt, double* mf,
                               double* gf, hipStream_t s) {
  const int nb = blocks_of(host.N);
  hipLaunchKernelGGL(k_curv_metrics, dim3(nb), dim3(BLK), 0, s, mem, g, mt);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_curv_face_metrics, dim3(nb), dim3(BLK), 0, s, mem, mt, mf, gf);
  return hipGetLastError();
}

hipError_t launch_curv_sensor(const Member* mem, int nblocks, const CurvGeom& g, const double* aux, int ns,
                              unsigned char* flag, double theta_c, double* theta_out, hipStream_t s) {
  hipLaunchKernelGGL(k_curv_sensor, dim3(nblocks), dim3(BLK), 0, s, mem, g, aux, flag, theta_c, theta_out,
                     5 + 2 * ns + 3);
  return hipGetLastError();
}

// Tiles of the convective face kernel: 64 x 4 faces in (x, y) when d is x,
// 16 along d by 16 along x otherwise.
template <int NS>
static hipError_t conv_t(const Member& host, const Member* mem, const CurvGeom& g, unsigned flags, const double* U,
                         const double* aux, const unsigned char* flag, double* ffc, double psi_c, double CT,
                         hipStream_t s) {
  for (int d = 0; d < 3; ++d) {
    if (!host.act[d]) continue;
    if (d == 0) {
      const int o = 1, r = 2;
      const int nb = ((host.n[0] + 63) / 64) * ((host.n[o] + 3) / 4) * host.n[r];
      hipLaunchKernelGGL((k_curv_conv<NS, 64, 4, true>), dim3(nb), dim3(BLK), 0, s, mem, g, d, flags, U, aux, flag,
                         ffc, psi_c, CT);
    } else {
      const int o = 0, r = 3 - d;
      const int nb = ((host.n[d] + 15) / 16) * ((host.n[o] + 15) / 16) * host.n[r];
      hipLaunchKernelGGL((k_curv_conv<NS, 16, 16, false>), dim3(nb), dim3(BLK), 0, s, mem, g, d, flags, U, aux,
                         flag, ffc, psi_c, CT);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_curv_conv(int ns, const Member& host, const Member* mem, const CurvGeom& g, const CallArgs& a,
                            const double* U, const double* aux, const unsigned char* flag, double* ffc, double psi_c,
                            double teno_CT, hipStream_t s) {
#define C_(NS) conv_t<NS>(host, mem, g, a.flags, U, aux, flag, ffc, psi_c, teno_CT, s)
  HTR_NS_SWITCH(ns, C_)
#undef C_
}

template <int NS>
static hipError_t diff_t(const MechTables* M, const Member& host, const Member* mem, const CurvGeom& g,
                         const CallArgs& a, const double* U, const double* Un, const double* T, const double* aux,
                         const double* src, const double* ffc, double* out, double ca, double cb, int rhs_only,
                         hipStream_t s) {
  int td[3], nb = 1;
  curv_tile(host.act, host.n, td);
  for (int k = 0; k < 3; ++k) nb *= (host.n[k] + td[k] - 1) / td[k];
  hipLaunchKernelGGL(k_curv_diff<NS>, dim3(nb), dim3(BLK), 0, s, M, mem, g, a, int3{td[0], td[1], td[2]}, U, Un, T, aux, src, ffc, out, ca, cb,
                     rhs_only);
  return hipGetLastError();
}

hipError_t launch_curv_diff(int ns, const MechTables* M, const Member& host, const Member* mem, const CurvGeom& g,
                            const CallArgs& a, const double* U, const double* Un, const double* T, const double* aux,
                            const double* src, const double* ffc, double* out, double ca, double cb, int rhs_only,
                            hipStream_t s) {
#define C_(NS) diff_t<NS>(M, host, mem, g, a, U, Un, T, aux, src, ffc, out, ca, cb, rhs_only, s)
  HTR_NS_SWITCH(ns, C_)
#undef C_
}

}  // namespace htr
