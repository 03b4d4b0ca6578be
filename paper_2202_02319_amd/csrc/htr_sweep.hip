// Flux sweep: for every cell, the flux differences along every active
// direction of the hybrid TENO6/central convective flux and of the
// second-order diffusive flux, plus the chemistry and laser sources, fused
// with the SSP-RK3 stage combination (or written as dU/dt).
//
// Paper (arXiv 2202.02319) Methods › Numerical method: conservative finite differences of the
// mapped equations (rectilinear metrics), TENO6 for the inviscid fluxes,
// second-order central differences for the diffusive fluxes; Methods › Solver eqs.
// (1)-(3), (5), (6) for the flux vectors.
//
// Two tiled sweeps per stage: k_conv (sources and convective flux
// differences, one block per 256-cell tile with the tile and its halo staged
// in LDS), with k_conv_lean for the tiles without TENO faces; and k_diff
// (diffusive flux differences and the stage update, one block per 256-cell
// tile of its own, on 3-D grids) or k_diff_flat (tiles of 192 cells, on grids
// of fewer axes and thin ones).  Every face is evaluated once, so the scheme is
// exactly conservative.  k_bnd does the cells next to bounded boundaries.

#include <math.h>

#include <type_traits>

#include "htr_dev.h"
#include "htr_flux.h"

namespace htr {


// Tile shapes of the tiled kernels: 256 cells.  Default 16 x 4 x 4 on 3-D
// grids, 16 x 16 over the two active axes of 2-D grids, 256 along a 1-D
// grid; other shapes are accepted if every staging buffer holds them.
// In 3-D the shape whose tiles cost least in all, a ragged tile as much as a
// whole one: the weights are a step's time at 128^3 cells, where every shape
// divides the grid, against 16x4x4 (7.09 ms; 7.24, 7.27 and 7.67 ms: shorter
// rows along x).  83x61x37 cells have 960 tiles of 16x4x4 and 880 of 8x8x4: a
// step takes 2.17 against 1.98 ms; 64 members of 12 to 24 cells an axis, 8.0
// against 7.35 ms.
void default_tile_shape(const int act[3], const int n[3], int t[3]) {
  const int na = act[0] + act[1] + act[2];
  t[0] = t[1] = t[2] = 1;
  if (na == 3) {
    constexpr int shapes[4][3] = {{16, 4, 4}, {8, 8, 4}, {8, 4, 8}, {4, 8, 8}};
    constexpr int weight[4] = {100, 102, 103, 108};
    long long best = 0;
    for (int k = 0; k < 4; ++k) {
      long long w = weight[k];
      for (int a = 0; a < 3; ++a) w *= (n[a] + shapes[k][a] - 1) / shapes[k][a];
      if (k > 0 && w >= best) continue;
      best = w;
      for (int a = 0; a < 3; ++a) t[a] = shapes[k][a];
    }
  } else if (na == 2) {
    for (int a = 0; a < 3; ++a) t[a] = act[a] ? 16 : 1;
  } else if (na == 1) {
    for (int a = 0; a < 3; ++a) t[a] = act[a] ? 256 : 1;
  } else {
    t[0] = 256;
  }
}

bool tile_shape_ok(const int act[3], const int t[3], const char** why) {
  const char* w = nullptr;
  const int na = act[0] + act[1] + act[2];
  if (t[0] < 1 || t[1] < 1 || t[2] < 1 || t[0] * t[1] * t[2] != BLK) w = "tile must have 256 cells";
  for (int a = 0; a < 3 && !w; ++a)
    if (na > 0 && !act[a] && t[a] != 1) w = "tile extends along an inactive axis";
  if (!w) {
    long box = 0, arms = 0, faces = 0;
    for (int d = 0; d < 3; ++d) {
      if (!act[d]) continue;
      const long cs = BLK / t[d];   // cross-section of the tile normal to d
      box += cs * (t[d] + 6);
      arms += 6 * cs;
      faces += cs * (t[d] + 1);
      if (!w && (cs * (t[d] + 10) > EXTA || cs * (t[d] + 5) > FACEA))
        w = "halo box too large for the convective adjoint";
    }
    if (!w && (box > XBOX_MAX || arms > XARM_MAX || faces > XFACE_MAX))
      w = "cross staging too large for the convective sweep";
  }
  if (why) *why = w;
  return w == nullptr;
}

// The diffusive sweep's tile.  On 3-D grids the shape of least tiles among
// k_diff's (8 x 8 x 4, 8 x 4 x 8, 4 x 8 x 8: their 256 halo nodes are one per
// thread) and the 16 x 4 x 3 of k_diff_flat: tiles of a thin grid are mostly
// empty and cost as much.  Nine species: 16384x2x2 cells 38 us a launch in
// 16 x 4 x 3, 80 in 8 x 8 x 4; 256x2x256 47 us in 8 x 4 x 8, 83 in 8 x 8 x 4;
// 4x256x256 53 us in 1024 tiles of 4 x 8 x 8, 84 in 2048 of 8 x 8 x 4: with
// rows of four a tile costs a quarter more.  16 x 4 x 3 needs a fifth less,
// since ensembles whose members take either pay for both kernels (64 members of
// 12 to 24 cells an axis: 7.9 against 7.3 ms a five-step run if ties are its),
// or a tie where an axis is shorter than a tile (256x256x5 cells, one species:
// 32 against 44 us).
// On 2-D grids 16 x 12 over the two active axes (204 and 208 faces) and on 1-D
// grids 192, for k_diff_flat.
static void diff_tile_shape(const int act[3], const int n[3], int t[3]) {
  const int na = act[0] + act[1] + act[2];
  default_tile_shape(act, n, t);
  if (na == 3) {
    const bool thin = n[0] < 8 || n[1] < 8 || n[2] < 8;
    constexpr int shapes[4][3] = {{8, 8, 4}, {8, 4, 8}, {4, 8, 8}, {16, 4, 3}};
    const int weight[4] = {4, 4, 5, thin ? 4 : 5};
    long long best = 0;
    for (int k = 0; k < 4; ++k) {
      long long w = weight[k];
      for (int a = 0; a < 3; ++a) w *= (n[a] + shapes[k][a] - 1) / shapes[k][a];
      if (k > 0 && (k == 3 && thin ? w > best : w >= best)) continue;
      best = w;
      for (int a = 0; a < 3; ++a) t[a] = shapes[k][a];
    }
  } else if (na == 2) {
    int k = 0;
    for (int a = 0; a < 3; ++a)
      if (act[a]) t[a] = k++ == 0 ? 16 : 12;
  } else {
    for (int a = 0; a < 3; ++a)
      if (t[a] > 1) t[a] = DTILE;
  }
}

void set_tiles(Member& M, const int* shape, int* tblocks, int* dtblocks) {
  const int act[3] = {M.act[0], M.act[1], M.act[2]};
  int t[3];
  if (shape) {
    t[0] = shape[0]; t[1] = shape[1]; t[2] = shape[2];
  } else {
    default_tile_shape(act, M.n, t);
  }
  int nb = 1;
  for (int a = 0; a < 3; ++a) {
    M.tdim[a] = t[a];
    M.ntile[a] = (M.n[a] + t[a] - 1) / t[a];
    nb *= M.ntile[a];
  }
  M.tblock_begin = *tblocks;
  M.ntblocks = nb;
  *tblocks += nb;
  int dt[3];
  diff_tile_shape(act, M.n, dt);
  int nd = 1;
  for (int a = 0; a < 3; ++a) {
    M.dtdim[a] = dt[a];
    M.dntile[a] = (M.n[a] + dt[a] - 1) / dt[a];
    nd *= M.dntile[a];
  }
  M.dtblock_begin = *dtblocks;
  M.ndtblocks = nd;
  *dtblocks += nd;
}

__device__ __forceinline__ long long lin(const Member& G, const int g[3]) {
  return ((long long)g[2] * G.n[1] + g[1]) * G.n[0] + g[0];
}

// Cross staging of the convective sweep: the tile plus a 3-cell halo on both
// sides along every active axis.  Each staged value is loaded once and
// written into the line-contiguous box of every direction that uses it (the
// tile's own cells into all of them).
constexpr int APT = (XARM_MAX + BLK - 1) / BLK;
constexpr int XFPT = (XFACE_MAX + BLK - 1) / BLK;

// Sources plus convective flux differences of every active direction, per
// cell, into part[nv][N] (TENO6, or WENO3-Z with HTR_WENO3Z, at the faces the
// hybrid switch marks).  The sensor flag, pressure and LF node speed of the
// cross are staged once and every face of the tile takes its hybrid decision
// and Lax-Friedrichs speed once for all variables.  Then, per conserved
// variable, each staged cell's value and its node flux along each axis are
// written once (the loading thread keeps that cell's velocity and pressure
// in registers), and every face flux is evaluated once from them, all
// directions together.
//
// v0, v1: the variables to do (a launch of few tiles deals a tile's variables
// to several blocks).
// KIND 0: every tile.  KIND 1 (the lean variant): a tile none of whose faces
// takes the TENO path is done here with the central faces alone (no staged
// conserved values, no TENO state, so fewer registers and more waves per
// SIMD); a tile with any TENO face is only marked in tcls[bl].  KIND 2: the
// marked tiles, in full; the others return at once.
template <int NS, bool TAPE, int KIND>
__device__ __forceinline__ void conv_tile(int bl, const Member* __restrict__ mem, int nmem, const CallArgs& A,
                                          const double* __restrict__ Ub, const double* __restrict__ auxb,
                                          const double* __restrict__ srcb, const unsigned char* __restrict__ flagb,
                                          double* __restrict__ partb, unsigned char* __restrict__ bitsb, double psi_c,
                                          double CT, unsigned char* __restrict__ tcls, int v0, int v1) {
  constexpr int NV = NS + 4, NAUX = 7 + NS;
  constexpr bool LEAN = KIND == 1;
  static_assert(!(TAPE && KIND != 0), "the taped sweep runs every tile in full");
  if constexpr (KIND == 2) {
    if (tcls[bl] == 0) return;   // the lean variant has done this tile
  }
  // one spare slot past every box: a write target for threads without a halo cell
  __shared__ double s_U[LEAN ? 1 : XBOX_MAX + 1], s_Fn[XBOX_MAX + 1], s_F[XFACE_MAX];
  __shared__ double s_al[LEAN ? 1 : XFACE_MAX];   // LF speed of the TENO faces, in list order
  // the tile's faces, those with TENO first and the central ones from the
  // end: stencil start slot (bits 0-11), face index (12-21) and stencil
  // stride in its box (22-31)
  __shared__ unsigned s_tl[LEAN ? 1 : XFACE_MAX];
  __shared__ int s_tq[TAPE ? XFACE_MAX : 1];             // taped: the face's tape index (upper cell)
  __shared__ unsigned char s_td[TAPE ? XFACE_MAX : 1];   // taped: the face's axis
  __shared__ int s_nt, s_nc;
  __shared__ double s_tab[LEAN ? 1 : 16][6];   // TENO6 coefficients of every cut-off pattern
  // before the variable loop the same memory holds the LF node speed, the
  // pressure and the sensor flags
  double* s_spd = s_U;
  double* s_p = s_Fn;
  unsigned char* s_fl = reinterpret_cast<unsigned char*>(&s_F[0]);
  const int m = find_member_tiled(mem, nmem, bl);
  const Member& G = mem[m];
  const int t = threadIdx.x;
  int o[3];
  tile_origin(G, bl - G.tblock_begin, o);
  const int T[3] = {G.tdim[0], G.tdim[1], G.tdim[2]};
  const int TT = T[0] * T[1] * T[2];
  const bool act[3] = {G.act[0] != 0, G.act[1] != 0, G.act[2] != 0};
  // layout of the boxes, the halo cells and the faces
  int boff[3], foff[3], aoff[3];
  int Ftot, Atot;
  {
    int eo = 0, fo = 0, ao = 0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      boff[d] = eo;
      foff[d] = fo;
      aoff[d] = ao;
      if (act[d]) {
        eo += TT / T[d] * (T[d] + 6);
        fo += TT / T[d] * (T[d] + 1);
        ao += 6 * (TT / T[d]);
      }
    }
    Ftot = fo;
    Atot = ao;
  }
  // slot of box position b in box d
  auto bslot = [&](int d, int b0, int b1, int b2) {
    const int B0 = T[0] + (d == 0 ? 6 : 0), B1 = T[1] + (d == 1 ? 6 : 0);
    return boff[d] + b0 + B0 * (b1 + B1 * b2);
  };
  // this thread's cell
  const int l[3] = {t % T[0], (t / T[0]) % T[1], t / (T[0] * T[1])};
  const int gc[3] = {o[0] + l[0], o[1] + l[1], o[2] + l[2]};
  const bool valid = gc[0] < G.n[0] && gc[1] < G.n[1] && gc[2] < G.n[2];
  const long long N = G.N;
  const double* U = Ub + NV * G.off;
  const double* aux = auxb + NAUX * G.off;
  const unsigned char* flag = flagb + G.off;
  const double* src = srcb + (NS + 1) * G.off;
  // TENO cut-off patterns per axis, variable and face (indexed by the face's
  // upper cell), when a forward tape asks for them
  unsigned char* bits = TAPE ? bitsb + 3LL * NV * G.off : nullptr;
  long long qc;
  {
    int g[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) g[a] = wrapi(gc[a], G.n[a]);
    qc = lin(G, g);
  }
  if constexpr (LEAN) {
    // a tile with a flagged cell of its own is left to the full variant before
    // its halo is looked at (most tiles of a shear layer: 107 against 63 us
    // for the pass over 256x128x128 cells, 99.6% of its tiles marked)
    if (!(A.flags & HTR_FORCE_CENTRAL) && __syncthreads_or((A.flags & HTR_FORCE_TENO) != 0 || flag[qc] != 0)) {
      if (t == 0) tcls[bl] = 1;
      return;
    }
  }
  int cs[3];
#pragma unroll
  for (int d = 0; d < 3; ++d)
    cs[d] = act[d] ? bslot(d, l[0] + (d == 0 ? 3 : 0), l[1] + (d == 1 ? 3 : 0), l[2] + (d == 2 ? 3 : 0))
                   : XBOX_MAX;
  // this thread's halo cells (box slot, global index, axis)
  int as[APT], ax[APT];
  long long aq[APT];
#pragma unroll
  for (int k = 0; k < APT; ++k) {
    const int a = t + k * BLK;
    as[k] = XBOX_MAX;
    aq[k] = qc;
    ax[k] = 0;
    if (a < Atot) {
      const int d = a < aoff[1] ? 0 : (a < aoff[2] ? 1 : 2);
      const int r = a - aoff[d], S = TT / T[d];
      const int j6 = r / S, cidx = r % S;
      const int side = j6 / 3, j = j6 - 3 * side;
      int lc[3];
      lc[d] = side == 0 ? j - 3 : T[d] + j;
      const int e1 = d == 0 ? 1 : 0, e2 = d == 2 ? 1 : 2;   // the two other axes, in order
      lc[e1] = cidx % T[e1];
      lc[e2] = cidx / T[e1];
      int g[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) g[c] = wrapi(o[c] + lc[c], G.n[c]);
      aq[k] = lin(G, g);
      ax[k] = d;
      int b[3] = {lc[0], lc[1], lc[2]};
      b[d] += 3;
      as[k] = bslot(d, b[0], b[1], b[2]);
    }
  }
  if constexpr (LEAN) {
    // every node of the cross lies in the stencil of one of the tile's faces,
    // so a flagged node means a TENO face: such tiles are left to the full
    // variant after one barrier (the pressure-jump test follows below)
    int any = 0;
    if (!(A.flags & HTR_FORCE_CENTRAL)) {
#pragma unroll
      for (int k = 0; k < APT; ++k) any |= flag[aq[k]];
    }
    if (__syncthreads_or(any)) {
      if (t == 0) tcls[bl] = 1;
      return;
    }
  }
  // velocity along the box axis and pressure of every staged cell, kept in
  // registers by the thread that stages it
  double cu[3], cp, hu[APT], hp[APT];
  {
    cp = aux[qc];
    const double cc = aux[N + qc];
    const unsigned char fc = flag[qc];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      cu[d] = aux[(4 + d) * N + qc];
      if constexpr (!LEAN) s_spd[cs[d]] = fabs(cu[d]) + cc;
      s_p[cs[d]] = cp;
      s_fl[cs[d]] = fc;
    }
#pragma unroll
    for (int k = 0; k < APT; ++k) {
      hu[k] = aux[(4 + ax[k]) * N + aq[k]];
      hp[k] = aux[aq[k]];
      if constexpr (!LEAN) s_spd[as[k]] = fabs(hu[k]) + aux[N + aq[k]];
      s_p[as[k]] = hp[k];
      s_fl[as[k]] = flag[aq[k]];
    }
    (void)cc;
  }
  if (t == 0) s_nt = s_nc = 0;
  if constexpr (!LEAN) teno6_table(t, s_tab);
  __syncthreads();
  // face f of the list: axis, stencil start slot (stencil positions j-3..j+2
  // of the tile = box positions j..j+5 along d), stride along the axis, and
  // tile position of the face's upper cell
  auto face = [&](int f, int& d, int& e0, int& bs, int fb[3]) {
    d = f < foff[1] ? 0 : (f < foff[2] ? 1 : 2);
    const int r = f - foff[d];
    const int F0 = T[0] + (d == 0 ? 1 : 0), F1 = T[1] + (d == 1 ? 1 : 0);
    fb[0] = r % F0;
    fb[1] = (r / F0) % F1;
    fb[2] = r / (F0 * F1);
    e0 = bslot(d, fb[0], fb[1], fb[2]);
    const int B0 = T[0] + (d == 0 ? 6 : 0), B1 = T[1] + (d == 1 ? 6 : 0);
    bs = d == 0 ? 1 : (d == 1 ? B0 : B0 * B1);
  };
  // a stride is at most T[0] T[1] <= BLK cells
  static_assert(XBOX_MAX < (1 << 12) && XFACE_MAX < (1 << 10) && BLK < (1 << 10), "TENO list packing");
  // this thread's faces: stencil start slot, stride, hybrid decision.  The
  // full variant lists every face (the TENO ones with their Lax-Friedrichs
  // speed), so that each variable's work is spread evenly over the block: a
  // wave takes whole runs of 64 faces of one kind, where a thread's own
  // central faces would cost every wave all four of its slots.  The lean
  // variant keeps its faces in registers.
  int fe0[LEAN ? XFPT : 1], fst[LEAN ? XFPT : 1];
  const unsigned flags = A.flags;
#pragma unroll
  for (int k = 0; k < XFPT; ++k) {
    const int f = t + k * BLK;
    if constexpr (LEAN) {
      fe0[k] = -1;
      fst[k] = 1;
    }
    if (f < Ftot) {
      int d, e0, bs, fb[3];
      face(f, d, e0, bs, fb);
      if constexpr (LEAN) {
        fe0[k] = e0;
        fst[k] = bs;
      }
      bool te;
      if (flags & HTR_FORCE_TENO) te = true;
      else if (flags & HTR_FORCE_CENTRAL) te = false;
      else {
        int any = 0;
#pragma unroll
        for (int mm = 0; mm < 6; ++mm) any |= s_fl[e0 + mm * bs];
        const double pa = s_p[e0 + 2 * bs], pb = s_p[e0 + 3 * bs];
        const double psi = fabs(pb - pa) / fmin(pa, pb);
        te = any != 0 || psi > psi_c;
      }
      if constexpr (LEAN) {
        if (te) atomicOr(&s_nt, 1);
      } else {
        const unsigned pk = (unsigned)e0 | (unsigned)f << 12 | (unsigned)bs << 22;
        if (te) {
          double al = s_spd[e0];
#pragma unroll
          for (int mm = 1; mm < 6; ++mm) al = fmax(al, s_spd[e0 + mm * bs]);
          const int slot = atomicAdd(&s_nt, 1);
          s_al[slot] = al;
          s_tl[slot] = pk;
          if (TAPE) {
            int g[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) g[c] = wrapi(o[c] + fb[c], G.n[c]);
            s_tq[slot] = (int)lin(G, g);
            s_td[slot] = (unsigned char)d;
          }
        } else {
          s_tl[Ftot - 1 - atomicAdd(&s_nc, 1)] = pk;
        }
      }
    }
  }
  // this cell's two faces per axis in the face list, and the metric
  int fL[3], fR[3];
  double xi[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    int lf[3] = {l[0], l[1], l[2]};
    const int F0 = T[0] + (d == 0 ? 1 : 0), F1 = T[1] + (d == 1 ? 1 : 0);
    fL[d] = foff[d] + lf[0] + F0 * (lf[1] + F1 * lf[2]);
    lf[d] += 1;
    fR[d] = foff[d] + lf[0] + F0 * (lf[1] + F1 * lf[2]);
    xi[d] = (valid && act[d]) ? G.xin[d][gc[d]] : 0.0;
  }
  const long long q = valid ? qc : 0;
  // software pipeline: the next variable's staging loads (and source) are in
  // flight while the current variable's faces are evaluated
  auto source = [&](int v) {
    const int sv = v < NS ? v : (v == NS + 3 ? NS : -1);
    return (valid && sv >= 0) ? src[sv * N + q] : 0.0;
  };
  double ncore = U[v0 * N + qc], narm[APT];
#pragma unroll
  for (int k = 0; k < APT; ++k) narm[k] = U[v0 * N + aq[k]];
  double nsrc = source(v0);
  double* part = partb + NV * G.off;
  __syncthreads();   // the decisions have read the node speeds, pressures and flags
  const int nteno = s_nt;
  if constexpr (LEAN) {
    if (t == 0) tcls[bl] = nteno != 0;
    if (nteno != 0) return;   // uniform: the full variant does this tile
  }
#pragma unroll 1
  for (int v = v0; v < v1; ++v) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      if constexpr (!LEAN) s_U[cs[d]] = ncore;
      s_Fn[cs[d]] = node_flux<NS>(v, d, ncore, cu[d], cp);
    }
#pragma unroll
    for (int k = 0; k < APT; ++k) {
      if constexpr (!LEAN) s_U[as[k]] = narm[k];
      s_Fn[as[k]] = node_flux<NS>(v, ax[k], narm[k], hu[k], hp[k]);
    }
    const double acc0 = nsrc;
    if (v + 1 < v1) {
      ncore = U[(v + 1) * N + qc];
#pragma unroll
      for (int k = 0; k < APT; ++k) narm[k] = U[(v + 1) * N + aq[k]];
      nsrc = source(v + 1);
    }
    __syncthreads();
    // one face buffer: every thread has taken its differences of the last
    // variable before the barrier above
    double* sF = s_F;
    // a face value goes through LDS before it is differenced, so its last
    // rounding cannot be fused into the difference
    auto central = [&](int e0, int bs) {
      double f6[6];
#pragma unroll
      for (int mm = 0; mm < 6; ++mm) f6[mm] = s_Fn[e0 + mm * bs];
      return (f6[0] - 8.0 * f6[1] + 37.0 * f6[2] + 37.0 * f6[3] - 8.0 * f6[4] + f6[5]) * (1.0 / 60.0);
    };
    if constexpr (LEAN) {
#pragma unroll
      for (int k = 0; k < XFPT; ++k)
        if (fe0[k] >= 0) sF[t + k * BLK] = central(fe0[k], fst[k]);
    } else {
      // the tile's list, dealt round-robin over the block
      for (int i = t; i < Ftot; i += BLK) {
        const unsigned pk = s_tl[i];
        const int e0 = pk & 0xfffu, f = (pk >> 12) & 0x3ffu, bs = pk >> 22;
        if (i >= nteno) {
          sF[f] = central(e0, bs);
          continue;
        }
        const double al = s_al[i];
        // the two sides of the split, without their factor 1/2
        double hp[6], hm[6];
#pragma unroll
        for (int mm = 0; mm < 6; ++mm) {
          const double f6 = s_Fn[e0 + mm * bs], u6 = s_U[e0 + mm * bs];
          hp[mm] = fma(al, u6, f6);
          hm[5 - mm] = fma(-al, u6, f6);
        }
        if (flags & HTR_WENO3Z) {
          sF[f] = weno3z_h(hp) + weno3z_h(hm);
          continue;
        }
        const unsigned pp = teno6_decide(hp, CT), pm = teno6_decide(hm, CT);
        sF[f] = teno6_value(s_tab, pp, hp) + teno6_value(s_tab, pm, hm);
        if (TAPE) {
          // the cut-off pattern: bits 0-3 the + side's kept candidates, 4-7 the - side's
          const unsigned pat = pp | pm << 4;
          bits[(long long)(s_td[i] * NV + v) * N + s_tq[i]] = (unsigned char)pat;
        }
      }
    }
    __syncthreads();
    if (valid) {
      double acc = acc0;
#pragma unroll
      for (int d = 0; d < 3; ++d)
        if (act[d]) acc -= xi[d] * (sF[fR[d]] - sF[fL[d]]);
      part[v * N + q] = acc;
    }
  }
}

// Bound by FP64 instructions where TENO faces are many (77% of the faces of the
// 256x128x128 mixing layer): with the expanded indicators, four candidates
// per side, central faces in each thread's own slots and two blocks per CU
// (64 KB of LDS, 183 registers) a launch took 2834 us; with the shared
// differences, one coefficient row per pattern, one list of faces and three
// blocks per CU (48 KB, 150 registers) 1857 us.
// MODE 0: one block per tile; 1: persistent blocks striding over the nlog
// tiles; 2: one block per tile, also writing the TENO cut-off patterns;
// 3: one block per tile, the tiles that k_conv_lean marked in tcls.
template <int NS, int MODE>
__global__ __launch_bounds__(BLK, 3) void k_conv(const MechTables* __restrict__ M, const Member* __restrict__ mem,
                                              int nmem, int nlog, CallArgs A, const double* __restrict__ Ub,
                                              const double* __restrict__ auxb, const double* __restrict__ srcb,
                                              const unsigned char* __restrict__ flagb, double* __restrict__ partb,
                                              unsigned char* __restrict__ bitsb, double psi_c, double CT,
                                              unsigned char* __restrict__ tcls) {
  if constexpr (MODE == 1) {
    for (int bl = blockIdx.x; bl < nlog; bl += gridDim.x) {
      conv_tile<NS, false, 0>(bl, mem, nmem, A, Ub, auxb, srcb, flagb, partb, bitsb, psi_c, CT, tcls, 0, NS + 4);
      __syncthreads();   // the next tile reuses the LDS
    }
  } else if constexpr (MODE == 2) {
    conv_tile<NS, true, 0>(blockIdx.x, mem, nmem, A, Ub, auxb, srcb, flagb, partb, bitsb, psi_c, CT, tcls, 0, NS + 4);
  } else if constexpr (MODE == 3) {
    conv_tile<NS, false, 2>(blockIdx.x, mem, nmem, A, Ub, auxb, srcb, flagb, partb, bitsb, psi_c, CT, tcls, 0, NS + 4);
  } else {
    // the variables in gridDim.y runs
    const int run = (NS + 4 + gridDim.y - 1) / gridDim.y, v0 = blockIdx.y * run;
    conv_tile<NS, false, 0>(blockIdx.x, mem, nmem, A, Ub, auxb, srcb, flagb, partb, bitsb, psi_c, CT, tcls, v0,
                            min(v0 + run, NS + 4));
  }
}

// The lean convective sweep: the tiles without TENO faces (central fluxes
// only), at up to four blocks per CU; marks the other tiles in tcls for
// k_conv<NS, 3>.  gridDim.y: as in k_conv<NS, 0>.
template <int NS>
__global__ __launch_bounds__(BLK, 4) void k_conv_lean(const MechTables* __restrict__ M,
                                                      const Member* __restrict__ mem, int nmem, CallArgs A,
                                                      const double* __restrict__ Ub, const double* __restrict__ auxb,
                                                      const double* __restrict__ srcb,
                                                      const unsigned char* __restrict__ flagb,
                                                      double* __restrict__ partb, double psi_c,
                                                      unsigned char* __restrict__ tcls) {
  const int run = (NS + 4 + gridDim.y - 1) / gridDim.y, v0 = blockIdx.y * run;
  conv_tile<NS, false, 1>(blockIdx.x, mem, nmem, A, Ub, auxb, srcb, flagb, partb, nullptr, psi_c, 0.0, tcls, v0,
                          min(v0 + run, NS + 4));
}

// Diffusive flux at the face between nodes qA and qB = A + e_d, in the sign
// with which it enters the right-hand side.  Tangential velocity derivatives
// at the face are the mean of the nodal central differences (grad).  Every
// input is loaded before any arithmetic so that all of the face's loads are
// in flight together (the kernel is bound by their latency).
template <int NS, int d>
__device__ __forceinline__ void diff_face(const MechTables* __restrict__ M, const Member& G, int cAd, long long qA,
                                          long long qB, long long N, const double* __restrict__ U,
                                          const double* __restrict__ T, const double* __restrict__ aux,
                                          const double* __restrict__ grad, double* Fd) {
  constexpr int t1 = (d + 1) % 3, t2 = (d + 2) % 3;
  const bool a1 = G.act[t1], a2 = G.act[t2];
  double uA[3], uB[3], g1A[3], g1B[3], g2A[3], g2B[3];
#pragma unroll
  for (int mm = 0; mm < 3; ++mm) {
    uA[mm] = aux[(4 + mm) * N + qA];
    uB[mm] = aux[(4 + mm) * N + qB];
    g1A[mm] = a1 ? grad[(3 * t1 + mm) * N + qA] : 0.0;
    g1B[mm] = a1 ? grad[(3 * t1 + mm) * N + qB] : 0.0;
    g2A[mm] = a2 ? grad[(3 * t2 + mm) * N + qA] : 0.0;
    g2B[mm] = a2 ? grad[(3 * t2 + mm) * N + qB] : 0.0;
  }
  const double muA = aux[2 * N + qA], muB = aux[2 * N + qB];
  const double laA = aux[3 * N + qA], laB = aux[3 * N + qB];
  const double TA = T[qA], TB = T[qB];
  const double xf = G.xif[d][cAd];
  // velocity gradient at the face, g[a][mm] = d u_mm / d x_a
  double g[3][3];
#pragma unroll
  for (int mm = 0; mm < 3; ++mm) {
    g[d][mm] = xf * (uB[mm] - uA[mm]);
    g[t1][mm] = a1 ? 0.5 * (g1A[mm] + g1B[mm]) : 0.0;
    g[t2][mm] = a2 ? 0.5 * (g2A[mm] + g2B[mm]) : 0.0;
  }
  const double muf = 0.5 * (muA + muB);
  const double lamf = 0.5 * (laA + laB);
  const double divu = g[0][0] + g[1][1] + g[2][2];
  double tau[3];
#pragma unroll
  for (int mm = 0; mm < 3; ++mm) {
    tau[mm] = muf * (g[d][mm] + g[mm][d]);
    if (mm == d) tau[mm] -= (2.0 / 3.0) * muf * divu;
  }
  // species: mixture quantities at both nodes
  double rA = 0.0, rB = 0.0, nA = 0.0, nB = 0.0;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const double ra = U[s * N + qA], rb = U[s * N + qB];
    rA += ra;
    rB += rb;
    nA += ra * M->iW[s];
    nB += rb * M->iW[s];
  }
  const double rhof = 0.5 * (rA + rB);
  const double inA = 1.0 / nA, inB = 1.0 / nB, irA = 1.0 / rA, irB = 1.0 / rB;
  const double iWf = 1.0 / (0.5 * (rA * inA + rB * inB));
  // two passes over the species (the correction flux, then each flux),
  // reloading per-species inputs rather than holding them in registers
  auto term = [&](int s) -> double {
    const double Df = 0.5 * (aux[(7 + s) * N + qA] + aux[(7 + s) * N + qB]);
    // both mole fractions rounded before differencing (no FMA across the
    // difference), so a uniform composition gives exactly zero flux
    double XA, XB;
    {
#pragma clang fp contract(off)
      XA = U[s * N + qA] * M->iW[s] * inA;
      XB = U[s * N + qB] * M->iW[s] * inB;
    }
    const double dX = xf * (XB - XA);
    return rhof * Df * (M->W[s] * iWf) * dX;
  };
  double corr = 0.0;
#pragma unroll
  for (int s = 0; s < NS; ++s) corr += term(s);
  const double iTA = 1.0 / TA, iTB = 1.0 / TB;
  double qn = -lamf * xf * (TB - TA);
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const double Yf = 0.5 * (U[s * N + qA] * irA + U[s * N + qB] * irB);
    const double J = -term(s) + Yf * corr;
    const double hf = 0.5 * (M->RW[s] * TA * hRTi(M, s, TA, iTA) + M->RW[s] * TB * hRTi(M, s, TB, iTB));
    qn += J * hf;
    Fd[s] = -J;
  }
  double work = 0.0;
#pragma unroll
  for (int mm = 0; mm < 3; ++mm) {
    Fd[NS + mm] = tau[mm];
    work += tau[mm] * (0.5 * (uA[mm] + uB[mm]));
  }
  Fd[NS + 3] = work - qn;
}

// One direction of the diffusive sweep: every face of the tile (one per
// thread) into LDS, then each node adds its flux difference.
template <int NS, int d>
__device__ __forceinline__ void diff_dir(const MechTables* __restrict__ M, const Member& G, const int o[3],
                                         const int l[3], const int gc[3], bool valid, long long N,
                                         const double* __restrict__ U, const double* __restrict__ T,
                                         const double* __restrict__ aux, const double* __restrict__ grad,
                                         double (*s_Fd)[BLKF], double* acc) {
  constexpr int NV = NS + 4;
  const int t = threadIdx.x;
  int FB[3] = {G.dtdim[0], G.dtdim[1], G.dtdim[2]};
  FB[d] += 1;
  const int F = FB[0] * FB[1] * FB[2];
  if (t < F) {
    const int fb[3] = {t % FB[0], (t / FB[0]) % FB[1], t / (FB[0] * FB[1])};
    int gA[3], gB[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int c0 = o[a] + fb[a] - (a == d ? 1 : 0);
      gA[a] = wrapi(c0, G.n[a]);
      gB[a] = a == d ? wrapi(c0 + 1, G.n[a]) : gA[a];
    }
    double Fd[NV];
    diff_face<NS, d>(M, G, gA[d], lin(G, gA), lin(G, gB), N, U, T, aux, grad, Fd);
#pragma unroll
    for (int v = 0; v < NV; ++v) s_Fd[v][t] = Fd[v];
  }
  __syncthreads();
  if (valid) {
    int lf[3] = {l[0], l[1], l[2]};
    const int fL = lf[0] + FB[0] * (lf[1] + FB[1] * lf[2]);
    lf[d] += 1;
    const int fR = lf[0] + FB[0] * (lf[1] + FB[1] * lf[2]);
    const double xi = G.xin[d][gc[d]];
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] += xi * (s_Fd[v][fR] - s_Fd[v][fL]);
  }
  __syncthreads();
}

// Members with tiles of BLK cells are k_diff's, the others k_diff_flat's; each
// kernel passes over the blocks of the other's.
__device__ __forceinline__ bool staged(const Member& G) { return G.dtdim[0] * G.dtdim[1] * G.dtdim[2] == BLK; }

// The sweep of grids with one or two active axes, and of thin ones: diffusive flux
// differences (each face once, exchanged through LDS) added to part, then the
// SSP-RK3 stage combination (or dU/dt when rhs_only).  Tiles of DTILE cells in
// BLKF threads, the first DTILE own the cells, and every thread owns one face
// per direction (a tile has at most BLKF faces along any axis: 16 x 4 x 3 has
// 204, 240 and 256), whose nodes' fields it reads itself.  With one or two directions that costs fewer loads
// than the staged species of k_diff cost barriers: 6.0 against 10.0 us on 256
// cells along a line (five species), 20.0 against 23.6 us on 384x250 (nine).
template <int NS>
__device__ __forceinline__ void diff_flat_tile(int bl, const MechTables* __restrict__ M, const Member* __restrict__ mem,
                                          int nmem, const CallArgs& A, const double* __restrict__ Ub,
                                          const double* Unb, const double* __restrict__ Tb,
                                          const double* __restrict__ auxb, const double* __restrict__ gradb,
                                          const double* __restrict__ partb, double* outb, double ca, double cb,
                                          int rhs_only) {
  constexpr int NV = NS + 4, NAUX = 7 + NS;
  __shared__ double s_Fd[NV][BLKF];
  const int m = find_member_dtiled(mem, nmem, bl);
  const Member& G = mem[m];
  const int t = threadIdx.x;
  int o[3];
  tile_origin_of(G.dtdim, G.dntile, G.ndtblocks, bl - G.dtblock_begin, o);
  const int T0 = G.dtdim[0], T1 = G.dtdim[1];
  const int l[3] = {t % T0, (t / T0) % T1, t / (T0 * T1)};
  const int gc[3] = {o[0] + l[0], o[1] + l[1], o[2] + l[2]};
  const bool valid = t < DTILE && gc[0] < G.n[0] && gc[1] < G.n[1] && gc[2] < G.n[2];
  const long long N = G.N;
  const double* U = Ub + NV * G.off;
  const double* T = Tb + G.off;
  const double* aux = auxb + NAUX * G.off;
  const double* grad = gradb + 9 * G.off;
  const long long q = valid ? lin(G, gc) : 0;
  double acc[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) acc[v] = 0.0;
  if (!(A.flags & HTR_VISC_OFF)) {
    if (G.act[0]) diff_dir<NS, 0>(M, G, o, l, gc, valid, N, U, T, aux, grad, s_Fd, acc);
    if (G.act[1]) diff_dir<NS, 1>(M, G, o, l, gc, valid, N, U, T, aux, grad, s_Fd, acc);
    if (G.act[2]) diff_dir<NS, 2>(M, G, o, l, gc, valid, N, U, T, aux, grad, s_Fd, acc);
  }
  if (!valid) return;
  // next to a non-periodic boundary part[] holds the whole right-hand side
  // (the boundary kernel's): no diffusive term is added here
  if (in_boundary_slab(G, gc)) {
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = 0.0;
  }
  // every load before the first store: out may be the same array as U^n, so
  // the compiler could not otherwise move a later variable's loads above an
  // earlier variable's store, and each variable would cost a memory round trip
  const double* part = partb + NV * G.off;
  double* out = outb + NV * G.off;
  double pv[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) pv[v] = part[v * N + q];
  if (rhs_only) {
#pragma unroll
    for (int v = 0; v < NV; ++v) out[v * N + q] = pv[v] + acc[v];
  } else {
    const double dt = A.dt_dev[m];
    const double* Un = Unb + NV * G.off;
    double uv[NV], unv[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      uv[v] = U[v * N + q];
      unv[v] = ca != 0.0 ? Un[v * N + q] : 0.0;
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const double base = uv[v] + dt * (pv[v] + acc[v]);
      out[v * N + q] = ca != 0.0 ? ca * unv[v] + cb * base : cb * base;
    }
  }
}

template <int NS, bool PERSIST>
__global__ __launch_bounds__(BLKF, 3) void k_diff_flat(const MechTables* __restrict__ M, const Member* __restrict__ mem,
                                                  int nmem, int nlog, CallArgs A, const double* __restrict__ Ub,
                                                  const double* Unb, const double* __restrict__ Tb,
                                                  const double* __restrict__ auxb, const double* __restrict__ gradb,
                                                  const double* __restrict__ partb, double* outb, double ca,
                                                  double cb, int rhs_only) {
  if (!PERSIST) {
    if (staged(mem[find_member_dtiled(mem, nmem, blockIdx.x)])) return;   // k_diff's
    diff_flat_tile<NS>(blockIdx.x, M, mem, nmem, A, Ub, Unb, Tb, auxb, gradb, partb, outb, ca, cb, rhs_only);
    return;
  }
  for (int bl = blockIdx.x; bl < nlog; bl += gridDim.x) {
    if (staged(mem[find_member_dtiled(mem, nmem, bl)])) continue;
    diff_flat_tile<NS>(bl, M, mem, nmem, A, Ub, Unb, Tb, auxb, gradb, partb, outb, ca, cb, rhs_only);
    __syncthreads();   // the next tile reuses the LDS
  }
}

// Diffusive flux differences added to part, then the SSP-RK3 stage
// combination (or dU/dt when rhs_only), on the diffusive sweep's own tiles
// (dtdim, BLK cells, one per thread; three active axes: only their tiles have
// BLK cells.  The tests of act all hold, and stay: without them the compiler
// moves every row's loads up and spills 1 KB a thread, 1305 us at 128^3).
//
// Thread t owns cell t, its box node and one halo node, and the lower face of
// its cell along every axis; the upper faces of the tile's last layer along
// axis d go to the lanes of wavefront d + 1.  The nodes' fields are loaded
// once, and what a node contributes to its faces (mole and mass fraction,
// enthalpy, 1/rho) is formed once and passed through LDS one species at a
// time, so no per-variable array is held: the species' correction flux
// first, then each species' flux, whose differences finish that row.
// Every value that two faces or cells difference has been through LDS, so its
// last rounding cannot be fused into the difference.
//
// Bound by the rate at which the address and data units of L1 take its loads
// (the data unit is busy 84% of the time).  One face per thread reading both of
// its nodes' thirty fields (about 320 loads a cell) took 592 us at 128^3 cells
// and nine species, 1145 us at 256x128x128; this order (about 110) takes 452
// and 876 us at two blocks per CU.  At three blocks (168 registers) 13 values
// spill and it takes 582 us; a deeper prefetch of the rows and twice as many
// barriers change nothing.
template <int NS>
__device__ __forceinline__ void diff_tile(int bl, const MechTables* __restrict__ M, const Member* __restrict__ mem,
                                          int nmem, const CallArgs& A, const double* __restrict__ Ub,
                                          const double* Unb, const double* __restrict__ Tb,
                                          const double* __restrict__ auxb, const double* __restrict__ gradb,
                                          const double* __restrict__ partb, double* outb, double ca, double cb,
                                          int rhs_only) {
  constexpr int NV = NS + 4, NAUX = 7 + NS;
  // node records (cell t at slot t, halo node h at BLK + h, so that lanes of
  // a row read consecutive banks): first thirteen of the velocity, viscosity
  // and velocity gradient, then four of the conduction, then four each of two
  // species; behind the first eight, per axis a value for each lower face and
  // each upper one of the last layer, for up to three rows at once
  __shared__ double s_mem[8 * DNODE + 9 * DFACE];
  double (*s_n)[DNODE] = reinterpret_cast<double (*)[DNODE]>(s_mem);
  double (*s_F)[3][DFACE] = reinterpret_cast<double (*)[3][DFACE]>(s_mem + 8 * DNODE);
  static_assert(13 * DNODE <= 8 * DNODE + 9 * DFACE, "the gradient records fit");
  const int m = find_member_dtiled(mem, nmem, bl);
  const Member& G = mem[m];
  const int t = threadIdx.x;
  int o[3];
  tile_origin_of(G.dtdim, G.dntile, G.ndtblocks, bl - G.dtblock_begin, o);
  const int T[3] = {G.dtdim[0], G.dtdim[1], G.dtdim[2]};
  const bool act[3] = {G.act[0] != 0, G.act[1] != 0, G.act[2] != 0};
  const int l[3] = {t % T[0], (t / T[0]) % T[1], t / (T[0] * T[1])};
  const int gc[3] = {o[0] + l[0], o[1] + l[1], o[2] + l[2]};
  const bool valid = gc[0] < G.n[0] && gc[1] < G.n[1] && gc[2] < G.n[2];
  const long long N = G.N;
  const double* U = Ub + NV * G.off;
  const double* part = partb + NV * G.off;
  const double* Un = Unb + NV * G.off;
  double* out = outb + NV * G.off;
  int gw[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) gw[a] = wrapi(gc[a], G.n[a]);
  const long long qc = lin(G, gw);
  const double dt = rhs_only ? 0.0 : A.dt_dev[m];
  // row v of the update; its loads come before the row's face work (out may
  // be the array U^n, so they could not move above an earlier row's store)
  struct Row { double p, u, un; };
  const double* un_or_part = !rhs_only && ca != 0.0 ? Un : part;   // U^n where it enters
  auto row = [&](int v, double u) { return Row{part[v * N + qc], u, un_or_part[v * N + qc]}; };
  // next to a non-periodic boundary part[] holds the whole right-hand side
  // (the boundary kernel's): no diffusive term is added there
  const bool slab = in_boundary_slab(G, gc);
  auto finish = [&](int v, const Row& r, double acc) {
    if (!valid) return;
    if (slab) acc = 0.0;
    if (rhs_only) {
      out[v * N + qc] = r.p + acc;
    } else {
      const double base = r.u + dt * (r.p + acc);
      out[v * N + qc] = ca != 0.0 ? ca * r.un + cb * base : cb * base;
    }
  };
  if (A.flags & HTR_VISC_OFF) {
    Row r[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) r[v] = row(v, U[v * N + qc]);
#pragma unroll
    for (int v = 0; v < NV; ++v) finish(v, r[v], 0.0);
    return;
  }
  const double* Tf = Tb + G.off;
  const double* aux = auxb + NAUX * G.off;
  const double* grad = gradb + 9 * G.off;
  // halo nodes: per axis the layer below the tile, then the one above, each
  // by the two other axes in order; this thread's one
  int hoff[3];
  hoff[0] = BLK;
  hoff[1] = hoff[0] + (act[0] ? 2 * (BLK / T[0]) : 0);
  hoff[2] = hoff[1] + (act[1] ? 2 * (BLK / T[1]) : 0);
  const int nhalo = hoff[2] + (act[2] ? 2 * (BLK / T[2]) : 0) - BLK;
  const int sh = BLK + t;
  long long qh = qc;
  int dh = 0;   // the halo node's axis
  if (t < nhalo) {
    const int d = sh < hoff[1] ? 0 : (sh < hoff[2] ? 1 : 2);
    const int Td = d == 0 ? T[0] : (d == 1 ? T[1] : T[2]), S = BLK / Td;
    const int r = sh - (d == 0 ? hoff[0] : (d == 1 ? hoff[1] : hoff[2]));
    const int x = r % S, w = r < S ? -1 : Td;
    const int Te = d == 0 ? T[1] : T[0];
    const int x0 = x % Te, x1 = x / Te;
    const int h[3] = {d == 0 ? w : x0, d == 1 ? w : (d == 0 ? x0 : x1), d == 2 ? w : x1};
    int g[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) g[a] = wrapi(o[a] + h[a], G.n[a]);
    qh = lin(G, g);
    dh = d;
  }
  // slot of the lower neighbour of this cell along each axis
  const int pos[3] = {l[1] + T[1] * l[2], l[0] + T[0] * l[2], l[0] + T[0] * l[1]};
  const int lo[3] = {l[0] > 0 ? t - 1 : hoff[0] + pos[0], l[1] > 0 ? t - T[0] : hoff[1] + pos[1],
                     l[2] > 0 ? t - T[0] * T[1] : hoff[2] + pos[2]};
  double rc[NS], rh[NS], Dc[NS], Dh[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    rc[s] = U[s * N + qc];
    rh[s] = U[s * N + qh];
  }
  const double Tc = Tf[qc], Th = Tf[qh];
  // this cell's record: u, v, w, mu, the nine velocity derivatives; a halo
  // node serves the faces of its own axis only, with the six derivatives
  // tangential to them
  double nd[13], lamc, lamh;
  {
    double hd[10];
    const int h1 = 3 * ((dh + 1) % 3), h2 = 3 * ((dh + 2) % 3);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int a = k < 3 ? 4 + k : 2;
      nd[k] = aux[a * N + qc];
      hd[k] = aux[a * N + qh];
    }
    lamc = aux[3 * N + qc];
    lamh = aux[3 * N + qh];
#pragma unroll
    for (int k = 0; k < 9; ++k) nd[4 + k] = grad[k * N + qc];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      hd[4 + k] = grad[(h1 + k) * N + qh];
      hd[7 + k] = grad[(h2 + k) * N + qh];
    }
#pragma unroll
    for (int k = 0; k < 13; ++k) s_n[k][t] = nd[k];
#pragma unroll
    for (int k = 0; k < 4; ++k) s_n[k][sh] = hd[k];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      s_n[4 + h1 + k][sh] = hd[4 + k];
      s_n[4 + h2 + k][sh] = hd[7 + k];
    }
  }
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    Dc[s] = aux[(7 + s) * N + qc];
    Dh[s] = aux[(7 + s) * N + qh];
  }
  double rhoc = 0.0, rhoh = 0.0, nc = 0.0, nh = 0.0;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    rhoc += rc[s];
    rhoh += rh[s];
    nc += rc[s] * M->iW[s];
    nh += rh[s] * M->iW[s];
  }
  const double inc = 1.0 / nc, inh = 1.0 / nh, irc = 1.0 / rhoc, irh = 1.0 / rhoh;
  // faces: 0-2 the lower face of this cell along each axis (its upper node's
  // values in registers), 3 (wavefront d + 1) an upper face of the last layer
  // along d, between slots sx and ux
  const int xd = __builtin_amdgcn_readfirstlane(t >> 6) - 1, lane = t & 63;
  const bool has_x = xd >= 0 && act[xd < 0 ? 0 : xd] && lane < BLK / T[xd < 0 ? 0 : xd];
  int sx = 0, ux = 0;
  double xfx = 0.0;   // metric of that face
  if (has_x) {
    const int Te = xd == 0 ? T[1] : T[0];
    const int x0 = lane % Te, x1 = lane / Te;
    const int h[3] = {xd == 0 ? T[0] - 1 : x0, xd == 1 ? T[1] - 1 : (xd == 0 ? x0 : x1), xd == 2 ? T[2] - 1 : x1};
    xfx = G.xif[xd][wrapi(o[xd] + T[xd] - 1, G.n[xd])];
    sx = h[0] + T[0] * (h[1] + T[1] * h[2]);
    ux = (xd == 0 ? hoff[0] : (xd == 1 ? hoff[1] : hoff[2])) + BLK / T[xd] + lane;
  }
  // where the upper face of this cell along d is in s_F[.][d]
  const int up[3] = {l[0] + 1 < T[0] ? t + 1 : BLK + pos[0], l[1] + 1 < T[1] ? t + T[0] : BLK + pos[1],
                     l[2] + 1 < T[2] ? t + T[0] * T[1] : BLK + pos[2]};
  double xi[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) xi[d] = act[d] ? G.xin[d][gw[d]] : 0.0;
  // flux difference of a row: the upper faces from s_F[z], the lower ones F
  auto difference = [&](int z, auto F) {
    double acc = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d)
      if (act[d]) acc += xi[d] * (s_F[z][d][up[d]] - F(d));
    return acc;
  };
  // rounds x before it meets another value (no operation of its own)
  auto rounded = [](double x) {
    asm("" : "+v"(x));
    return x;
  };
  double k1[4] = {}, corr[4] = {}, en[4] = {}, tau[4][3];
  double xf[4];
#pragma unroll
  for (int d = 0; d < 3; ++d) xf[d] = act[d] ? G.xif[d][gw[d] > 0 ? gw[d] - 1 : G.n[d] - 1] : 0.0;
  xf[3] = xfx;
  Row mrow[3], srow[NS];
#pragma unroll
  for (int mm = 0; mm < 3; ++mm) mrow[mm] = row(NS + mm, U[(NS + mm) * N + qc]);
  __syncthreads();
  // viscous stress of face k along d (lower node in slot sa, upper node's
  // record B) and its work
  auto viscous = [&](auto dc, int sa, auto B, int k) {
    constexpr int d = decltype(dc)::value, t1 = (d + 1) % 3, t2 = (d + 2) % 3;
    double g[3][3], uf[3];
#pragma unroll
    for (int mm = 0; mm < 3; ++mm) {
      g[t1][mm] = 0.5 * (s_n[4 + 3 * t1 + mm][sa] + B(4 + 3 * t1 + mm));
      g[t2][mm] = 0.5 * (s_n[4 + 3 * t2 + mm][sa] + B(4 + 3 * t2 + mm));
      const double uA = s_n[mm][sa], uB = B(mm);
      g[d][mm] = xf[k] * (uB - uA);
      uf[mm] = 0.5 * (uA + uB);
    }
    const double muf = 0.5 * (s_n[3][sa] + B(3));
    const double divu = g[0][0] + g[1][1] + g[2][2];
    double work = 0.0;
#pragma unroll
    for (int mm = 0; mm < 3; ++mm) {
      double tm = muf * (g[d][mm] + g[mm][d]);
      if (mm == d) tm -= (2.0 / 3.0) * muf * divu;
      tau[k][mm] = rounded(tm);
      work += tau[k][mm] * uf[mm];
    }
    en[k] = work;
  };
  constexpr std::integral_constant<int, 0> d0{};
  constexpr std::integral_constant<int, 1> d1{};
  constexpr std::integral_constant<int, 2> d2{};
  auto own = [&](int k) { return nd[k]; };
  auto above = [&](int k) { return s_n[k][ux]; };
  if (act[0]) viscous(d0, lo[0], own, 0);
  if (act[1]) viscous(d1, lo[1], own, 1);
  if (act[2]) viscous(d2, lo[2], own, 2);
  if (has_x) {
    if (xd == 0) viscous(d0, sx, above, 3);
    else if (xd == 1) viscous(d1, sx, above, 3);
    else viscous(d2, sx, above, 3);
  }
  __syncthreads();
  // conduction and the species' face factor rho xf / W
  {
    const double c[4] = {lamc, Tc, rhoc, rhoc * inc}, h[4] = {lamh, Th, rhoh, rhoh * inh};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      s_n[k][t] = c[k];
      s_n[k][sh] = h[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (k < 3 ? !act[k] : !has_x) continue;
      const int a = k < 3 ? lo[k] : sx;
      double B[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) B[j] = k < 3 ? c[j] : s_n[j][ux];
      en[k] += 0.5 * (s_n[0][a] + B[0]) * xf[k] * (B[1] - s_n[1][a]);
      k1[k] = 0.5 * (s_n[2][a] + B[2]) * xf[k] / (0.5 * (s_n[3][a] + B[3]));
    }
  }
  // the first species' rows
#pragma unroll
  for (int s = 0; s < 2 && s < NS; ++s) srow[s] = row(s, rc[s]);
  // every face's value of one row into s_F[z]
  auto put = [&](int z, auto val) {
#pragma unroll
    for (int d = 0; d < 3; ++d)
      if (act[d]) s_F[z][d][t] = val(d);
    if (has_x) s_F[z][xd][BLK + lane] = val(3);
  };
#pragma unroll
  for (int mm = 0; mm < 3; ++mm) put(mm, [&](int k) { return tau[k][mm]; });
  __syncthreads();
#pragma unroll
  for (int mm = 0; mm < 3; ++mm) finish(NS + mm, mrow[mm], difference(mm, [&](int d) { return tau[d][mm]; }));
  // species in twos: the correction flux first, the records in alternating halves
#pragma unroll
  for (int s0 = 0; s0 < NS; s0 += 2) {
    double (*R)[DNODE] = &s_n[(4 + 2 * s0) % 8];
    double X[2];
#pragma unroll
    for (int j = 0; j < 2 && s0 + j < NS; ++j) {
      const int s = s0 + j;
      X[j] = rounded(rc[s] * M->iW[s] * inc);
      R[2 * j][t] = X[j];
      R[2 * j][sh] = rh[s] * M->iW[s] * inh;
      R[2 * j + 1][t] = Dc[s];
      R[2 * j + 1][sh] = Dh[s];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (k < 3 ? !act[k] : !has_x) continue;
      const int a = k < 3 ? lo[k] : sx;
#pragma unroll
      for (int j = 0; j < 2 && s0 + j < NS; ++j) {
        const double Xb = k < 3 ? X[j] : R[2 * j][ux], Db = k < 3 ? Dc[s0 + j] : R[2 * j + 1][ux];
        corr[k] += k1[k] * (0.5 * M->W[s0 + j] * (R[2 * j + 1][a] + Db)) * (Xb - R[2 * j][a]);
      }
    }
  }
  __syncthreads();
  // each species' flux and its enthalpy; the energy row goes with the last ones
  const double iTc = 1.0 / Tc, iTh = 1.0 / Th;
  Row er{};
#pragma unroll
  for (int s0 = 0; s0 < NS; s0 += 2) {
    const bool last = s0 + 2 >= NS;
    // the next rows' loads, ahead of this group's stores: a wavefront's
    // memory operations complete in order
#pragma unroll
    for (int j = 2; j < 4; ++j)
      if (s0 + j < NS) srow[s0 + j] = row(s0 + j, rc[s0 + j]);
    if (last) er = row(NS + 3, U[(NS + 3) * N + qc]);
    double X[2], Y[2], H[2];
#pragma unroll
    for (int j = 0; j < 2 && s0 + j < NS; ++j) {
      const int s = s0 + j;
      X[j] = rounded(rc[s] * M->iW[s] * inc);
      Y[j] = rounded(rc[s] * irc);
      H[j] = rounded(M->RW[s] * Tc * hRTi(M, s, Tc, iTc));
      s_n[4 * j][t] = X[j];
      s_n[4 * j][sh] = rh[s] * M->iW[s] * inh;
      s_n[4 * j + 1][t] = Dc[s];
      s_n[4 * j + 1][sh] = Dh[s];
      s_n[4 * j + 2][t] = Y[j];
      s_n[4 * j + 2][sh] = rh[s] * irh;
      s_n[4 * j + 3][t] = H[j];
      s_n[4 * j + 3][sh] = M->RW[s] * Th * hRTi(M, s, Th, iTh);
    }
    __syncthreads();
    double F[2][4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      F[0][k] = F[1][k] = 0.0;
      if (k < 3 ? !act[k] : !has_x) continue;
      const int a = k < 3 ? lo[k] : sx;
#pragma unroll
      for (int j = 0; j < 2 && s0 + j < NS; ++j) {
        const double (*R)[DNODE] = &s_n[4 * j];
        const double Xb = k < 3 ? X[j] : R[0][ux], Db = k < 3 ? Dc[s0 + j] : R[1][ux];
        const double Yb = k < 3 ? Y[j] : R[2][ux], Hb = k < 3 ? H[j] : R[3][ux];
        F[j][k] = rounded(k1[k] * (0.5 * M->W[s0 + j] * (R[1][a] + Db)) * (Xb - R[0][a]) -
                          0.5 * (R[2][a] + Yb) * corr[k]);
        en[k] += F[j][k] * (0.5 * (R[3][a] + Hb));
      }
    }
#pragma unroll
    for (int j = 0; j < 2 && s0 + j < NS; ++j) put(j, [&](int k) { return F[j][k]; });
    if (last) {
#pragma unroll
      for (int k = 0; k < 4; ++k) en[k] = rounded(en[k]);
      put(2, [&](int k) { return en[k]; });
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2 && s0 + j < NS; ++j)
      finish(s0 + j, srow[s0 + j], difference(j, [&](int d) { return F[j][d]; }));
    if (last) finish(NS + 3, er, difference(2, [&](int d) { return en[d]; }));
  }
}

template <int NS, bool PERSIST>
__global__ __launch_bounds__(BLK, 2) void k_diff(const MechTables* __restrict__ M, const Member* __restrict__ mem,
                                                 int nmem, int nlog, CallArgs A, const double* __restrict__ Ub,
                                                 const double* Unb, const double* __restrict__ Tb,
                                                 const double* __restrict__ auxb, const double* __restrict__ gradb,
                                                 const double* __restrict__ partb, double* outb, double ca,
                                                 double cb, int rhs_only) {
  if (!PERSIST) {
    if (!staged(mem[find_member_dtiled(mem, nmem, blockIdx.x)])) return;   // k_diff_flat's
    diff_tile<NS>(blockIdx.x, M, mem, nmem, A, Ub, Unb, Tb, auxb, gradb, partb, outb, ca, cb, rhs_only);
    return;
  }
  for (int bl = blockIdx.x; bl < nlog; bl += gridDim.x) {
    if (!staged(mem[find_member_dtiled(mem, nmem, bl)])) continue;
    diff_tile<NS>(bl, M, mem, nmem, A, Ub, Unb, Tb, auxb, gradb, partb, outb, ca, cb, rhs_only);
    __syncthreads();   // the next tile reuses the LDS
  }
}

// ----------------------------------------------------- non-periodic boundaries
// Cells within three nodes of a bounded boundary (in_boundary_slab) get
// their whole right-hand side here, each cell's faces evaluated on their own
// (the tiled sweeps assume periodic wrap).  On a
// bounded axis the first and last nodes lie on the boundary; a face whose
// six-point stencil does not fit takes the widest centred interpolation that
// does ((-1, 7, 7, -1)/12 or (1, 1)/2), or, where the hybrid switch marks
// it, the local Lax-Friedrichs (Rusanov) flux of its two nodes.  Boundary
// nodes take the locally one-dimensional characteristic treatment of
// Poinsot & Lele (the paper's NSCBC, Methods › Diffusion flame › Physical
// model and numerical setup): the normal convective terms as wave
// amplitudes from one-sided differences, entering waves prescribed
// (outflow: the acoustic one relaxes p to p_inf; walls and inflows hold u
// and T, inflows also Y, with the entering acoustic wave equal to the
// leaving one; Methods › Model rocket combustor › Numerical setup).

constexpr int BNDC = 64;   // slab cells of a block: one wavefront per face

__device__ __forceinline__ double cpR_b(const MechTables* __restrict__ M, int s, double T) {
  const double* a = M->cp[s];
  return a[0] + T * (a[1] + T * (a[2] + T * (a[3] + T * a[4])));
}

// Convective flux through face i+1/2 along d (i = c[d] with the other
// coordinates of c), variable by variable, into out[v * BNDC].  The six slots
// of the full stencil are all loaded (on a bounded axis clamped to the grid);
// a face of m < 6 points uses the middle m of them.
template <int NS>
__device__ __forceinline__ void bnd_conv_face(const Member& G, int d, const int c[3], const double* __restrict__ U,
                                              const double* __restrict__ aux, const unsigned char* __restrict__ flag,
                                              unsigned flags, double psi_c, double CT, const double (*tab)[6], double* out) {
  constexpr int NV = NS + 4;
  const long long N = G.N;
  const int i = c[d], n = G.n[d];
  const bool bnd = G.bc[d][0] != 0;
  const int m = !bnd || (i >= 2 && i <= n - 4) ? 6 : ((i == 0 || i == n - 2) ? 2 : 4);
  const int lo = (6 - m) / 2;
  long long st[6];
  double ud[6], p[6];
  double al = 0.0;
  int any = 0;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    int g[3] = {c[0], c[1], c[2]};
    const int j = i - 2 + k;
    const int w = bnd ? (j < 0 ? 0 : (j >= n ? n - 1 : j)) : wrapi(j, n);
    g[0] = d == 0 ? w : g[0];
    g[1] = d == 1 ? w : g[1];
    g[2] = d == 2 ? w : g[2];
    st[k] = lin(G, g);
    ud[k] = aux[(4 + d) * N + st[k]];
    p[k] = aux[st[k]];
    if (k >= lo && k < 6 - lo) {
      any |= flag[st[k]];
      al = fmax(al, fabs(ud[k]) + aux[N + st[k]]);
    }
  }
  bool te;
  if (flags & HTR_FORCE_TENO) te = true;
  else if (flags & HTR_FORCE_CENTRAL) te = false;
  else te = any != 0 || fabs(p[3] - p[2]) / fmin(p[2], p[3]) > psi_c;
#pragma unroll 1
  for (int v = 0; v < NV; ++v) {
    double u6[6], f6[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      u6[k] = U[v * N + st[k]];
      f6[k] = node_flux<NS>(v, d, u6[k], ud[k], p[k]);
    }
    double f;
    if (!te) {
      if (m == 6)
        f = (f6[0] - 8.0 * f6[1] + 37.0 * f6[2] + 37.0 * f6[3] - 8.0 * f6[4] + f6[5]) * (1.0 / 60.0);
      else if (m == 4)
        f = (-f6[1] + 7.0 * f6[2] + 7.0 * f6[3] - f6[4]) * (1.0 / 12.0);
      else
        f = 0.5 * (f6[2] + f6[3]);
    } else if (m == 6) {
      double hp[6], hm[6];
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        hp[k] = fma(al, u6[k], f6[k]);
        hm[5 - k] = fma(-al, u6[k], f6[k]);
      }
      f = (flags & HTR_WENO3Z) ? weno3z_h(hp) + weno3z_h(hm) : teno6_face(tab, hp, hm, CT);
    } else {
      f = 0.5 * (f6[2] + f6[3]) - 0.5 * al * (u6[3] - u6[2]);
    }
    out[v * BNDC] = f;
  }
}

template <int NS>
__device__ __forceinline__ void bnd_diff_face(const MechTables* __restrict__ M, const Member& G, int d, const int c[3],
                                              const double* __restrict__ U, const double* __restrict__ T,
                                              const double* __restrict__ aux, const double* __restrict__ grad,
                                              double* out) {
  const int w = G.bc[d][0] != 0 ? c[d] + 1 : wrapi(c[d] + 1, G.n[d]);
  const int cb[3] = {d == 0 ? w : c[0], d == 1 ? w : c[1], d == 2 ? w : c[2]};
  const long long qA = lin(G, c), qB = lin(G, cb);
  double fd[NS + 4];
  if (d == 0) diff_face<NS, 0>(M, G, c[0], qA, qB, G.N, U, T, aux, grad, fd);
  else if (d == 1) diff_face<NS, 1>(M, G, c[1], qA, qB, G.N, U, T, aux, grad, fd);
  else diff_face<NS, 2>(M, G, c[2], qA, qB, G.N, U, T, aux, grad, fd);
#pragma unroll
  for (int v = 0; v < NS + 4; ++v) out[v * BNDC] = fd[v];
}

// The slab cells in a dense order: axis by axis the six layers next to its
// two sides (the layer fastest on x, x otherwise), without the layers of the
// bounded axes before it.  Cells of axis a's part:
__host__ __device__ inline long long slab_cells(const int n[3], const int bc[3][2], int a) {
  if (bc[a][0] == 0) return 0;
  long long k = 6;
  for (int b = 0; b < 3; ++b)
    if (b != a) k *= n[b] - (b < a && bc[b][0] != 0 ? 6 : 0);
  return k;
}
__device__ __forceinline__ bool slab_cell(const Member& G, long long k, int c[3]) {
  int a = 0;
  for (; a < 3; ++a) {
    const long long m = slab_cells(G.n, G.bc, a);
    if (k < m) break;
    k -= m;
  }
  if (a == 3) return false;
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    const bool in = b < a && G.bc[b][0] != 0;   // inside the earlier axes' layers
    const int ext = b == a ? 6 : G.n[b] - (in ? 6 : 0);
    const int r = (int)(k % ext);
    k /= ext;
    c[b] = b == a ? (r < 3 ? r : G.n[b] - 6 + r) : (in ? r + 3 : r);
  }
  return true;
}

// One block: BNDC slab cells by six waves, wave r evaluating face r of every
// cell (axis r / 2, upper face when r is even), so the axis is uniform in a
// wave and a cell's faces are evaluated side by side; convective and
// diffusive fluxes pass through LDS in turn.  Bound by one wave's chain of
// thirteen TENO faces.  One thread per grid cell (a few active lanes in each
// wave, each with all of its cell's faces in turn, 456 registers) took 1554 us on
// 100x72x48 cells with two bounded axes (14% of them in the slab); this order
// takes 176 us (252 registers and no scratch, one block per CU: 180 us).
template <int NS>
__global__ __launch_bounds__(6 * BNDC, 3) void k_bnd(const MechTables* __restrict__ M, const Member* __restrict__ mem,
                                                  CallArgs A, const double* __restrict__ U,
                                                  const double* __restrict__ T, const double* __restrict__ aux,
                                                  const double* __restrict__ src,
                                                  const unsigned char* __restrict__ flag,
                                                  const double* __restrict__ grad, double* __restrict__ part,
                                                  double psi_c, double CT) {
  constexpr int NV = NS + 4, VPT = (NV + 5) / 6;
  __shared__ double s_f[6][NV][BNDC], s_acc[NV][BNDC];
  __shared__ double s_tab[16][6];   // TENO6 coefficients of every cut-off pattern
  teno6_table(threadIdx.x, s_tab);
  __syncthreads();
  const Member& G = mem[0];
  const long long N = G.N;
  const int lane = threadIdx.x % BNDC, role = __builtin_amdgcn_readfirstlane(threadIdx.x / BNDC);
  int c[3] = {0, 0, 0};
  const bool valid = slab_cell(G, (long long)blockIdx.x * BNDC + lane, c);
  const long long q = lin(G, c);
  const unsigned flags = A.flags;
  const int a = role / 2;
  const bool lower = role & 1;
  bool edge[3];   // on that axis's boundary
#pragma unroll
  for (int b = 0; b < 3; ++b) edge[b] = G.act[b] && G.bc[b][0] != 0 && (c[b] == 0 || c[b] == G.n[b] - 1);
  // this thread's face: its lower node
  int cf[3] = {c[0], c[1], c[2]};
  if (lower) {
    const int ca = a == 0 ? c[0] : (a == 1 ? c[1] : c[2]);
    const int w = G.bc[a][0] != 0 ? ca - 1 : wrapi(ca - 1, G.n[a]);
    cf[0] = a == 0 ? w : cf[0];
    cf[1] = a == 1 ? w : cf[1];
    cf[2] = a == 2 ? w : cf[2];
  }
  const bool on_edge = a == 0 ? edge[0] : (a == 1 ? edge[1] : edge[2]);
  const bool inner = valid && G.act[a] && !on_edge;
  if (inner) bnd_conv_face<NS>(G, a, cf, U, aux, flag, flags, psi_c, CT, s_tab, &s_f[role][0][lane]);
  __syncthreads();
  // variables role, role + 6, ...: the convective differences
  double cd[3][VPT];
#pragma unroll
  for (int k = 0; k < VPT; ++k) {
    const int v = role + 6 * k;
#pragma unroll
    for (int b = 0; b < 3; ++b)
      cd[b][k] = v < NV && G.act[b] && !edge[b] ? s_f[2 * b][v][lane] - s_f[2 * b + 1][v][lane] : 0.0;
  }
  __syncthreads();
  // the face inside the domain of a wall node too: the wall's species diffusion
  const int side_a = (a == 0 ? c[0] : (a == 1 ? c[1] : c[2])) == 0 ? 0 : 1;
  const bool wall_in = valid && on_edge && G.bc[a][side_a] == HTR_BC_WALL && (side_a == 1) == lower;
  if (!(flags & HTR_VISC_OFF) && (inner || wall_in))
    bnd_diff_face<NS>(M, G, a, cf, U, T, aux, grad, &s_f[role][0][lane]);
  __syncthreads();
  const bool onb = edge[0] || edge[1] || edge[2];
#pragma unroll
  for (int k = 0; k < VPT; ++k) {
    const int v = role + 6 * k;
    if (!valid || v >= NV) continue;
    double r = v < NS ? src[v * N + q] : (v == NS + 3 ? src[NS * N + q] : 0.0);
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      if (!G.act[b] || edge[b]) continue;
      const double fd = flags & HTR_VISC_OFF ? 0.0 : s_f[2 * b][v][lane] - s_f[2 * b + 1][v][lane];
      r += G.xin[b][c[b]] * (fd - cd[b][k]);
    }
    if (onb) s_acc[v][lane] = r;
    else part[v * N + q] = r;
  }
  __syncthreads();
  if (role != 0 || !valid || !onb) return;
  double acc[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) acc[v] = s_acc[v][lane];
  {
    // boundary node: characteristic treatment along every bounded axis it lies on
    double Y[NS], rho = 0.0;
    for (int s = 0; s < NS; ++s) rho += U[s * N + q];
    for (int s = 0; s < NS; ++s) Y[s] = U[s * N + q] / rho;
    const double Tq = T[q], pq = aux[q], cc = aux[N + q];
    const double uq[3] = {aux[4 * N + q], aux[5 * N + q], aux[6 * N + q]};
    double cpm = 0.0, iW = 0.0, hs[NS];
    const double iT = 1.0 / Tq;
    for (int s = 0; s < NS; ++s) {
      cpm += Y[s] * M->RW[s] * cpR_b(M, s, Tq);
      iW += Y[s] * M->iW[s];
      hs[s] = M->RW[s] * Tq * hRTi(M, s, Tq, iT);
    }
    const double W = 1.0 / iW;
    const double cv = cpm - RU * iW, gam = cpm / cv, cc2 = cc * cc;
    bool held = false, holdY = false;
    double add[NV];
    for (int v = 0; v < NV; ++v) add[v] = 0.0;
    const long long stride[3] = {1, G.n[0], (long long)G.n[0] * G.n[1]};
    for (int a = 0; a < 3; ++a) {
      if (!G.act[a] || G.bc[a][0] == 0 || !(c[a] == 0 || c[a] == G.n[a] - 1)) continue;
      const int side = c[a] == 0 ? 0 : 1;
      const int type = G.bc[a][side];
      const double sgn = side ? 1.0 : -1.0;
      const long long s1 = side ? -stride[a] : stride[a];
      const double xi = G.xin[a][c[a]];
      // one-sided second-order derivative along a (inward)
      auto D = [&](double f0, double f1, double f2) {
        return side ? xi * (3.0 * f0 - 4.0 * f1 + f2) / 2.0 : xi * (-3.0 * f0 + 4.0 * f1 - f2) / 2.0;
      };
      double r1 = 0.0, r2 = 0.0;
      for (int s = 0; s < NS; ++s) {
        r1 += U[s * N + q + s1];
        r2 += U[s * N + q + 2 * s1];
      }
      const double Dp = D(pq, aux[q + s1], aux[q + 2 * s1]);
      const double Dr = D(rho, r1, r2);
      double Du[3];
      for (int mm = 0; mm < 3; ++mm)
        Du[mm] = D(uq[mm], aux[(4 + mm) * N + q + s1], aux[(4 + mm) * N + q + 2 * s1]);
      const double un = uq[a];
      double L1 = (un - cc) * (Dp - rho * cc * Du[a]);
      double L5 = (un + cc) * (Dp + rho * cc * Du[a]);
      if (type == HTR_BC_WALL || type == HTR_BC_INFLOW) {
        held = true;
        if (type == HTR_BC_INFLOW) holdY = true;
        const double Lout = side ? L5 : L1;
        const double drho = (type == HTR_BC_INFLOW ? -(gam / cc2) : -(1.0 / cc2)) * Lout;
        for (int s = 0; s < NS; ++s) add[s] += Y[s] * drho;
        if (type == HTR_BC_WALL && !(flags & HTR_VISC_OFF)) {
          const double x2 = 2.0 * xi;
          for (int s = 0; s < NS; ++s) add[s] += (side ? -x2 : x2) * s_f[2 * a + side][s][lane];
        }
        continue;
      }
      // outflow
      double L2 = un * (cc2 * Dr - Dp);
      double L3 = un * Du[(a + 1) % 3], L4 = un * Du[(a + 2) % 3];
      const double Ld = fabs(G.xnode[a][G.n[a] - 1] - G.xnode[a][0]);
      const double Mn = fabs(un) / cc;
      const double K = G.relax[a][side] * cc * (1.0 - Mn * Mn) / Ld;
      const double relaxp = K * (pq - G.pinf[a][side]);
      if (sgn * (un - cc) < 0) L1 = relaxp;
      if (sgn * (un + cc) < 0) L5 = relaxp;
      const bool backflow = sgn * un < 0;
      if (backflow) { L2 = 0.0; L3 = 0.0; L4 = 0.0; }
      const double rho_t = -(L2 + 0.5 * (L5 + L1)) / cc2;
      const double p_t = -0.5 * (L5 + L1);
      double u_t[3];
      u_t[a] = -(L5 - L1) / (2.0 * rho * cc);
      u_t[(a + 1) % 3] = -L3;
      u_t[(a + 2) % 3] = -L4;
      double ke = 0.0, udu = 0.0;
      for (int mm = 0; mm < 3; ++mm) { ke += uq[mm] * uq[mm]; udu += uq[mm] * u_t[mm]; }
      double dE = (cpm * W / RU - 1.0) * p_t + 0.5 * ke * rho_t + rho * udu;
      for (int s = 0; s < NS; ++s) {
        const double LY = backflow ? 0.0 : un * D(Y[s], U[s * N + q + s1] / r1, U[s * N + q + 2 * s1] / r2);
        const double drs = Y[s] * rho_t - rho * LY;
        add[s] += drs;
        dE += (hs[s] - cpm * Tq * W * M->iW[s]) * drs;
      }
      for (int mm = 0; mm < 3; ++mm) add[NS + mm] += uq[mm] * rho_t + rho * u_t[mm];
      add[NS + 3] += dE;
    }
    if (!held) {
      for (int v = 0; v < NV; ++v) acc[v] += add[v];
    } else {
      double drs[NS], drho = 0.0;
      for (int s = 0; s < NS; ++s) {
        drs[s] = acc[s] + add[s];
        drho += drs[s];
      }
      if (holdY)
        for (int s = 0; s < NS; ++s) drs[s] = Y[s] * drho;
      double ke = 0.0;
      for (int mm = 0; mm < 3; ++mm) ke += uq[mm] * uq[mm];
      double dE = 0.0;
      for (int s = 0; s < NS; ++s) {
        acc[s] = drs[s];
        dE += (hs[s] - RU * Tq * M->iW[s] + 0.5 * ke) * drs[s];
      }
      for (int mm = 0; mm < 3; ++mm) acc[NS + mm] = uq[mm] * drho;
      acc[NS + 3] = dE;
    }
  }
  for (int v = 0; v < NV; ++v) part[v * N + q] = acc[v];
}

template <int NS>
static hipError_t bnd_t(const MechTables* M, const Member* mem, const Member& host, const CallArgs& a, const double* U,
                        const double* T, const double* aux, const double* src, const unsigned char* flag,
                        const double* grad, double* part, double psi_c, double CT, hipStream_t s) {
  // the blocks of the slab there is; under capture those of the largest one, as
  // the launch keeps its size while htr_set_boundaries may bound another axis
  // before a replay (the kernel takes the types from the device's member, and
  // its blocks past the slab do nothing)
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  hipError_t e = hipStreamIsCapturing(s, &capture);
  if (e != hipSuccess) return e;
  int bc[3][2];
  for (int b = 0; b < 3; ++b) bc[b][0] = bc[b][1] = capture == hipStreamCaptureStatusNone ? host.bc[b][0] : host.n[b] >= BNDMIN;
  long long cells = 0;
  for (int b = 0; b < 3; ++b) cells += slab_cells(host.n, bc, b);
  const unsigned nblocks = (unsigned)((cells + BNDC - 1) / BNDC);
  hipLaunchKernelGGL(k_bnd<NS>, dim3(nblocks), dim3(6 * BNDC), 0, s, M, mem, a, U, T, aux, src, flag, grad, part, psi_c, CT);
  return hipGetLastError();
}

hipError_t launch_bnd(int ns, const MechTables* M, const Member* mem, const Member& host, const CallArgs& a, const double* U,
                      const double* T, const double* aux, const double* src, const unsigned char* flag,
                      const double* grad, double* part, double psi_c, double CT, hipStream_t s) {
#define C_(NS) bnd_t<NS>(M, mem, host, a, U, T, aux, src, flag, grad, part, psi_c, CT, s)
  HTR_NS_SWITCH(ns, C_);
#undef C_
}

// Blocks of the full convective sweep that the 256 CUs hold at once (three each).
constexpr int CONV_RESIDENT = 768;

static int grid_of(int nblocks, int grid) { return (grid <= 0 || grid > nblocks) ? nblocks : grid; }

template <int NS>
static hipError_t conv_t(const MechTables* M, const Member* mem, int nmem, int ntblocks, int grid, const CallArgs& a,
                         const double* U, const double* aux, const double* src, const unsigned char* flag,
                         double* part, unsigned char* bits, double psi_c, double CT, unsigned char* tcls,
                         hipStream_t s) {
  if (bits) {   // taped: one block per tile, every tile in full
    hipLaunchKernelGGL((k_conv<NS, 2>), dim3(ntblocks), dim3(BLK), 0, s, M, mem, nmem, ntblocks, a, U, aux, src, flag,
                       part, bits, psi_c, CT, tcls);
  } else if (grid < ntblocks) {
    hipLaunchKernelGGL((k_conv<NS, 1>), dim3(grid), dim3(BLK), 0, s, M, mem, nmem, ntblocks, a, U, aux, src, flag,
                       part, bits, psi_c, CT, tcls);
  } else {
    // of few tiles, each one's variables are dealt to several blocks, whose
    // chains of barriers then run side by side
    int runs = CONV_RESIDENT / ntblocks;
    runs = runs < 1 ? 1 : (runs > NS + 4 ? NS + 4 : runs);
    const int run = (NS + 4 + runs - 1) / runs;
    runs = (NS + 4 + run - 1) / run;   // no empty run
    const bool central = a.flags & HTR_FORCE_CENTRAL;
    if (!tcls || (!central && runs > 1)) {
      // every tile in the full sweep: asked for, or few enough to be dealt.  In
      // one run each that would save a launch, and cost smooth tiles the lean
      // variant: 43 against 29 us on 52^3 smooth cells of five species (117
      // against 123 us where all faces are TENO's, nine species)
      hipLaunchKernelGGL((k_conv<NS, 0>), dim3(ntblocks, runs), dim3(BLK), 0, s, M, mem, nmem, ntblocks, a, U, aux, src, flag,
                         part, bits, psi_c, CT, tcls);
    } else {
      // central tiles in the lean variant, then the tiles with TENO faces if
      // there can be any.  Where all are central, however few: 160^2 cells and
      // nine species 13 us, 26 in the full sweep and 21 in two launches of one run
      hipLaunchKernelGGL((k_conv_lean<NS>), dim3(ntblocks, runs), dim3(BLK), 0, s, M, mem, nmem, a, U, aux, src, flag,
                         part, psi_c, tcls);
      if (!central)
        hipLaunchKernelGGL((k_conv<NS, 3>), dim3(ntblocks), dim3(BLK), 0, s, M, mem, nmem, ntblocks, a, U, aux, src, flag,
                           part, bits, psi_c, CT, tcls);
    }
  }
  return hipGetLastError();
}

template <int NS>
static hipError_t diff_t(const MechTables* M, const Member* mem, int nmem, int ntblocks, int grid, unsigned kinds,
                         const CallArgs& a,
                         const double* U, const double* Un, const double* T, const double* aux, const double* grad,
                         const double* part, double* out, double ca, double cb, int rhs_only, hipStream_t s) {
#define D_(KERNEL, PERSIST, GRID, THREADS)                                                                            \
  hipLaunchKernelGGL((KERNEL<NS, PERSIST>), dim3(GRID), dim3(THREADS), 0, s, M, mem, nmem, ntblocks, a, U, Un, T, aux, \
                     grad, part, out, ca, cb, rhs_only)
  if (kinds & DIFF_FLAT) {
    if (grid < ntblocks) D_(k_diff_flat, true, grid, BLKF);
    else D_(k_diff_flat, false, ntblocks, BLKF);
  }
  if (kinds & DIFF_STAGED) {
    if (grid < ntblocks) D_(k_diff, true, grid, BLK);
    else D_(k_diff, false, ntblocks, BLK);
  }
#undef D_
  return hipGetLastError();
}

hipError_t launch_conv(int ns, const MechTables* M, const Member* mem, int nmem, int ntblocks, int grid,
                       const CallArgs& a, const double* U, const double* aux, const double* src,
                       const unsigned char* flag, double* part, unsigned char* bits, double psi_c, double CT,
                       unsigned char* tcls, hipStream_t s) {
  grid = grid_of(ntblocks, grid);
#define C_(NS) conv_t<NS>(M, mem, nmem, ntblocks, grid, a, U, aux, src, flag, part, bits, psi_c, CT, tcls, s)
  HTR_NS_SWITCH(ns, C_);
#undef C_
}

hipError_t launch_diff(int ns, const MechTables* M, const Member* mem, int nmem, int ntblocks, int grid, unsigned kinds,
                       const CallArgs& a, const double* U, const double* Un, const double* T, const double* aux,
                       const double* grad, const double* part, double* out, double ca, double cb, int rhs_only,
                       hipStream_t s) {
  grid = grid_of(ntblocks, grid);
#define C_(NS) diff_t<NS>(M, mem, nmem, ntblocks, grid, kinds, a, U, Un, T, aux, grad, part, out, ca, cb, rhs_only, s)
  HTR_NS_SWITCH(ns, C_);
#undef C_
}

}  // namespace htr
