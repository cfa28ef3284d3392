// Residual-form iteration kernels of libfftc (FP32 fields, FP64 displacement) for CDNA4.
#include "fftc_internal.h"
#include "fftc_launch.h"
#include "fftc_common.h"
#include "fftc_march.h"

#include <math.h>
#include <algorithm>
#include <atomic>
#include <type_traits>

namespace fftc {

// ===========================================================================
// Residual-form iteration (FP32 fields, FP64 displacement).  The same fixed point as
// above with ACV_P, rearranged exactly: with y_i = p_i + K0 u_i the Green input of the
// paper's iteration, e_i = x_i - K0 u_i is residual-sized, u_{i+1} = Pi u_i + K0^+ e_i,
// and Anderson runs in difference form on
//   R_i = p_i + K0 delta_i - e_{i-1},  dR = R_i - R_{i-1},  dY = p_i - p_{i-1} + K0 delta_i,
//   e_i = p_i - sum_j gamma_j dY_j,  gamma = argmin |R_i - sum_j gamma_j dR_j|.
// Only residual-sized quantities pass through FP32 transforms.
// ===========================================================================

// K0 f at a node for the three components (Paux stencil, mirrored neighbours)
template <typename T>
__device__ __forceinline__ void stencil_k0(const Geo& g, const T* __restrict__ f, int i, int j, int k, T out[3]) {
  const int Nx = g.N[0], Ny = g.N[1];
  const long long Nn = g.Nn;
  const int xs[3] = {mirror_coord(g, i - 1, 0), i, mirror_coord(g, i + 1, 0)};
  const int ys[3] = {mirror_coord(g, j - 1, 1), j, mirror_coord(g, j + 1, 1)};
  const int zs[3] = {mirror_coord(g, k - 1, 2), k, mirror_coord(g, k + 1, 2)};
  auto at = [&](int c, int dx, int dy, int dz) {
    return f[c * Nn + (long long)xs[dx + 1] + (long long)Nx * ((long long)ys[dy + 1] + (long long)Ny * zs[dz + 1])];
  };
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const T sxy = at(c, -1, -1, 0) + at(c, 1, -1, 0) + at(c, -1, 1, 0) + at(c, 1, 1, 0);
    const T sxz = at(c, -1, 0, -1) + at(c, 1, 0, -1) + at(c, -1, 0, 1) + at(c, 1, 0, 1);
    const T syz = at(c, 0, -1, -1) + at(c, 0, 1, -1) + at(c, 0, -1, 1) + at(c, 0, 1, 1);
    out[c] = T(g.st[c][0]) * at(c, 0, 0, 0) + T(g.st[c][1]) * sxy + T(g.st[c][2]) * sxz + T(g.st[c][3]) * syz;
  }
}

// p = 2^b div_D(sigma) from an FP64 displacement: neighbour differences are formed in
// FP64 and rounded once to TS, the stress and divergence arithmetic is in TS (T, or FP64 for
// the refining passes of the FP32 form), and p is rounded to T.
template <typename T, bool SIG, bool FS = false, typename TS = T>
__device__ __forceinline__ void node_eval_d(const Geo& g, const double* __restrict__ u, const T* __restrict__ lam,
                                            const T* __restrict__ mu, int i, int j, int k, T p[3], double& sn,
                                            double ms[6]) {
  const int Nx = g.N[0], Ny = g.N[1];
  const long long Nn = g.Nn;
  const int xs[3] = {mirror_coord(g, i - 1, 0), i, mirror_coord(g, i + 1, 0)};
  const int ys[3] = {mirror_coord(g, j - 1, 1), j, mirror_coord(g, j + 1, 1)};
  const int zs[3] = {mirror_coord(g, k - 1, 2), k, mirror_coord(g, k + 1, 2)};
  const long long self = (long long)i + (long long)Nx * ((long long)j + (long long)Ny * k);
  double u0[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) u0[c] = u[c * Nn + self];
  TS nb[27][3];
#pragma unroll
  for (int dz = -1; dz <= 1; ++dz)
#pragma unroll
    for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
      for (int dx = -1; dx <= 1; ++dx) {
        const int nrm = (dx != 0) + (dy != 0) + (dz != 0);
        if (nrm != 2) continue;
        const long long idx = (long long)xs[dx + 1] + (long long)Nx * ((long long)ys[dy + 1] + (long long)Ny * zs[dz + 1]);
        const int q = (dx + 1) + 3 * (dy + 1) + 9 * (dz + 1);
#pragma unroll
        for (int c = 0; c < 3; ++c) nb[q][c] = (TS)(u[c * Nn + idx] - u0[c]);
      }
#pragma unroll
  for (int c = 0; c < 3; ++c) nb[13][c] = TS(0);
  TS F[3] = {TS(0), TS(0), TS(0)};
#pragma unroll
  for (int a = 0; a < 8; ++a) {
    const int ax = a & 1, ay = (a >> 1) & 1, az = (a >> 2) & 1;
    int vx = i - ax, vy = j - ay, vz = k - az;
    bool inside = true;
    if (g.periodic[0]) { if (vx < 0) vx += g.n[0]; } else inside &= (vx >= 0 && vx < g.n[0]);
    if (g.periodic[1]) { if (vy < 0) vy += g.n[1]; } else inside &= (vy >= 0 && vy < g.n[1]);
    if (g.periodic[2]) { if (vz < 0) vz += g.n[2]; } else inside &= (vz >= 0 && vz < g.n[2]);
    if (!inside) continue;
    const long long vid = (long long)vx + (long long)g.n[0] * ((long long)vy + (long long)g.n[1] * vz);
    const TS l = (TS)lam[vid], m = (TS)mu[vid];
    TS G[3][3];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int s = 0; s < 3; ++s) G[r][s] = TS(0);
    const int par = (ax + ay + az) & 1;
#pragma unroll
    for (int cc = 0; cc < 8; ++cc) {
      const int cx = cc & 1, cy = (cc >> 1) & 1, cz = (cc >> 2) & 1;
      if (((cx + cy + cz) & 1) != par) continue;
      const int q = (cx - ax + 1) + 3 * (cy - ay + 1) + 9 * (cz - az + 1);
      const TS sx = TS(cx ? 0.5 : -0.5), sy = TS(cy ? 0.5 : -0.5), sz = TS(cz ? 0.5 : -0.5);
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        G[r][0] += sx * nb[q][r];
        G[r][1] += sy * nb[q][r];
        G[r][2] += sz * nb[q][r];
      }
    }
    const TS bx = TS(ax ? 0.25 : -0.25), by = TS(ay ? 0.25 : -0.25), bz = TS(az ? 0.25 : -0.25);
    if constexpr (FS) {
      TS P[3][3];
      svk_pk1<TS>(G, l, m, P);
#pragma unroll
      for (int r = 0; r < 3; ++r) F[r] += bx * P[r][0] + by * P[r][1] + bz * P[r][2];
      if (SIG && (a == 0 || a == 1)) {
        double q = 0.0;
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
          for (int c = 0; c < 3; ++c) q += (double)P[r][c] * (double)P[r][c];
        sn += 0.5 * q;
        ms[0] += 0.5 * (double)P[0][0]; ms[1] += 0.5 * (double)P[1][1]; ms[2] += 0.5 * (double)P[2][2];
        ms[3] += 0.5 * (double)P[1][2]; ms[4] += 0.5 * (double)P[0][2]; ms[5] += 0.5 * (double)P[0][1];
      }
      continue;
    }
    const TS tr = G[0][0] + G[1][1] + G[2][2];
    const TS s00 = l * tr + TS(2) * m * G[0][0];
    const TS s11 = l * tr + TS(2) * m * G[1][1];
    const TS s22 = l * tr + TS(2) * m * G[2][2];
    const TS s01 = m * (G[0][1] + G[1][0]);
    const TS s02 = m * (G[0][2] + G[2][0]);
    const TS s12 = m * (G[1][2] + G[2][1]);
    F[0] += bx * s00 + by * s01 + bz * s02;
    F[1] += bx * s01 + by * s11 + bz * s12;
    F[2] += bx * s02 + by * s12 + bz * s22;
    if (SIG && (a == 0 || a == 1)) {
      const double d00 = s00, d11 = s11, d22 = s22, d01 = s01, d02 = s02, d12 = s12;
      sn += 0.5 * (d00 * d00 + d11 * d11 + d22 * d22 + 2.0 * (d01 * d01 + d02 * d02 + d12 * d12));
      ms[0] += 0.5 * d00; ms[1] += 0.5 * d11; ms[2] += 0.5 * d22;
      ms[3] += 0.5 * d12; ms[4] += 0.5 * d02; ms[5] += 0.5 * d01;
    }
  }
  const int xyz[3] = {i, j, k};
  const TS w2b = TS(1 << bcount(g, xyz));
#pragma unroll
  for (int c = 0; c < 3; ++c) p[c] = is_antisym(g, c, xyz) ? T(0) : (T)(-w2b * F[c]);
}

// forward-transform weight of a node in the singular coefficients (DCT1 ends 1, interior 2; DFT 1)
__device__ __forceinline__ double sing_weight(const Geo& g, const int xyz[3]) {
  double w = 1.0;
#pragma unroll
  for (int J = 0; J < 3; ++J)
    if (!g.periodic[J] && xyz[J] > 0 && xyz[J] < g.n[J]) w *= 2.0;
  return w;
}

// Per-node part of the residual pass of the residual-form iteration, once p is known:
// singular-mode coefficients of u, contact bookkeeping or constraint masking, the norm of
// p, p itself, and (ACV_P, from the second iteration on) dY_i = p_i - p_{i-1} + K0 delta_i and
// R_i = p_i + K0 delta_i - e_{i-1} = dY_i + c_{i-1}, with c = p - e the correction of the last
// Anderson combination (0 after a plain iteration).  R_i goes to a ring of four, from which the
// Gram pass forms the differences with the same FP32 subtraction.  kd = K0 delta at the node
// (read only when kd_used).
// INC: p holds the increment dp_i (the divergence term of the stresses of delta_i) and p_i is
// p_{i-1} + dp_i; dY and R are formed from dp_i itself, so that they carry no cancellation
// against |p| (p_i - p_{i-1} in FP32 is rounding noise once the iteration stagnates).
// Node inputs of the tail that do not depend on p: mask, c_{i-1}, p_{i-1}.
template <typename T>
struct TailIn {
  uint8_t m;
  T c[3], pp[3];   // c after an accelerating iteration, else p_{i-1} in its place (the tail weighs it 0)
};

template <typename T>
__device__ __forceinline__ void tail_load(const DeltaBufs<T>& D, long long Nn, bool kd_used, bool inc, int ecomb,
                                          const T* pp, long long node, TailIn<T>& t) {
  t.m = D.mask[node];
  // a uniform choice of source (no branch around the loads): after a plain iteration c is 0
  // and the second load of p_{i-1} is served by the cache.  The weight is applied in the tail, so
  // the loads stay in flight over the layer's stresses.
  const T* cs = ecomb ? D.e : pp;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    t.c[c] = T(0);
    t.pp[c] = T(0);
    if (kd_used || inc) t.pp[c] = pp[c * Nn + node];
    if (kd_used) t.c[c] = cs[c * Nn + node];
  }
}

// GEN = false: no rigid obstacle and no singular modes (both checked by the launcher).
template <typename T, bool GEN, bool INC = false>
__device__ __forceinline__ void delta_tail(const Geo& g, const DeltaBufs<T>& D, const ContactDev& ct, int cur,
                                           bool kd_used, int il, int slot, T* pc, T* Rc, int i, int j, int k,
                                           long long node, T p[3], const T kd[3], const TailIn<T>& tin, T cw,
                                           double* acc) {
  static_assert(!(GEN && INC), "the incremental pass has no contact or singular modes");
  const long long Nn = g.Nn;
  const int xyz[3] = {i, j, k};
  // singular-mode coefficients of u (projection Pi of the update)
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if (!GEN || !g.sing[c]) continue;
    const double wu = sing_weight(g, xyz) * D.u[c * Nn + node];
    acc[8 + 2 * c] += wu;
    if (g.sing[c] & 2) acc[9 + 2 * c] += ((i + j + k) & 1) ? -wu : wu;
  }
  const uint8_t m = tin.m;
  // dp: p_i - p_{i-1} as formed (INC: the increment itself, after the masking below)
  T dp[3];
  if (GEN && ct.on && (m & M_FACE)) {
    const long long f = (long long)xyz[ct.b1] + (long long)g.N[ct.b1] * xyz[ct.b2];
    const double X0 = i + D.u[node], X1 = j + D.u[Nn + node], X2 = k + D.u[2 * Nn + node];
    const double d0 = X0 - ct.center[0], d1 = X1 - ct.center[1], d2 = X2 - ct.center[2];
    const double rr = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
    const double gap = rr - ct.radius;
    const double n0 = -d0 / rr, n1 = -d1 / rr, n2 = -d2 / rr;
    const double pn = (double)p[0] * n0 + (double)p[1] * n1 + (double)p[2] * n2;
    const double fnc = -pn / (double)(1 << bcount(g, xyz));
    const uint8_t inC = ct.C[f];
    if (inC) {
      p[0] = (T)((double)p[0] - pn * n0);
      p[1] = (T)((double)p[1] - pn * n1);
      p[2] = (T)((double)p[2] - pn * n2);
    }
    ct.V[cur][f] = (uint8_t)(((!inC) && gap < 0.0) ? 1 : 0) | (uint8_t)((inC && fnc > 0.0) ? 2 : 0);
    ct.fnc[f] = fnc;
    ct.gap[f] = gap;
    acc[0] += (double)p[0] * p[0] + (double)p[1] * p[1] + (double)p[2] * p[2];
#pragma unroll
    for (int c = 0; c < 3; ++c) dp[c] = p[c] - tin.pp[c];
  } else {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if (m & (M_STRONG << c)) p[c] = T(0);
      if constexpr (INC) {
        dp[c] = p[c];
        p[c] = tin.pp[c] + dp[c];
      } else {
        dp[c] = p[c] - tin.pp[c];
      }
      if (!(m & (M_WEAK << c))) acc[0] += (double)p[c] * p[c];
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) pc[c * Nn + node] = p[c];
  if (kd_used) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const long long e = c * Nn + node;
      // At a DOF held at 0 by a Dirichlet face p is 0 and K0 delta is taken from the
      // symmetric image; the transforms drop these entries, but they stay in the Gram matrix
      // of the differences (measured: zeroing them makes the FP32 least squares less robust).
      const T y = dp[c] + kd[c];
      Rc[e] = y + cw * tin.c[c];
      if (il >= 2) D.dY[slot][e] = y;
    }
  }
}

// TS: stress arithmetic (T, or FP64 once the residual is below the refinement threshold);
// the instance whose kind is not the state's pass of this iteration returns at once (this
// untiled pass has no incremental form: its problems take the full pass every iteration).
template <typename T, bool FS, typename TS>
__global__ __launch_bounds__(kBlock) void k_residual_d(Geo g, DeltaBufs<T> D, ContactDev ct, DevState* st,
                                                       double* __restrict__ part) {
  __shared__ double sh[kPartStrideD * 16];
  if (st->done || res_pass(st) != (sizeof(TS) == 8 ? PASS_U64 : PASS_U)) return;
  double acc[kPartStrideD];
#pragma unroll
  for (int q = 0; q < kPartStrideD; ++q) acc[q] = 0.0;
  const int Nx = g.N[0], Ny = g.N[1];
  const long long Nn = g.Nn;
  const int cur = ct.on ? st->vpar : 0;
  const int il = st->i_local, par = st->it & 1, acvp = (st->acv == 2), ecomb = st->accel_ok;
  const int slot = (il + 1) % 3;   // (il - 2) mod 3
  const bool kd_used = acvp && il >= 1;
  T* pc = D.p[par];
  const T* pp = D.p[par ^ 1];
  T* Rc = D.R[il & 3];
  long long lo, hi;
  xcd_chunk(Nn, lo, hi);
  for (long long node = lo + threadIdx.x; node < hi; node += blockDim.x) {
    const int nd = (int)node;
    const int r = nd / Nx;
    const int i = nd - r * Nx;
    const int k = r / Ny, j = r - k * Ny;
    T p[3];
    double sn = 0.0, ms[6] = {0, 0, 0, 0, 0, 0};
    node_eval_d<T, true, FS, TS>(g, D.u, D.lam, D.mu, i, j, k, p, sn, ms);
    acc[1] += sn;
    T kd[3] = {T(0), T(0), T(0)};
    if (kd_used) stencil_k0<T>(g, D.delta, i, j, k, kd);
    TailIn<T> tin;
    tail_load<T>(D, Nn, kd_used, false, ecomb, pp, node, tin);
    delta_tail<T, true>(g, D, ct, cur, kd_used, il, slot, pc, Rc, i, j, k, node, p, kd, tin, ecomb ? T(1) : T(0), acc);
  }
  block_sum<kPartStrideD>(acc, sh);
  if (threadIdx.x == 0)
#pragma unroll
    for (int q = 0; q < kPartStrideD; ++q) part[q * kPartRows + blockIdx.x] = acc[q];
}

// The tiled residual pass (see fftc_march.h).  Fields: u (FP64, passes from u) gives the stresses,
// delta the reference-medium term K0 delta and, in the incremental pass (INC: small strain, no
// contact or singular modes), the stresses: p_i = p_{i-1} + their divergence term; u is then not
// read and no stress norm is formed (the control keeps the last full pass's).
//
// K0 delta at a node is a stencil over three planes; with A = st0 delta + st1 (its four in-plane
// diagonal neighbours) and S = st2 (x neighbours) + st3 (y neighbours) formed once per plane it is
// A_z + S_{z-1} + S_{z+1}: 9 LDS reads per component and step, four of them the voxel's corners.
//
// Bound by LDS and VALU issue and the latency of a step about equally: at 256^3 the incremental pass
// moves 1.36 GB after a plain iteration and 1.62 GB after an accelerating one, in 427 us on average,
// 3.5 TB/s (about 520 us with every node forming its 24 corner forces from stresses passed through
// LDS, two barriers per step); with the launches around it at 128^3 60 us (89), at 64^3 26 us (36).
// Registers set the blocks per CU: held to four, the incremental pass spills 6 of them and takes
// 70 us at 128^3; at three nothing spills, which the passes with T stresses are held to as well
// (those with contact or singular modes would spill).
template <typename T, bool GEN, typename TS, bool INC>
struct MarchLds {
  static constexpr int NS = GEN ? kPartStrideD : 2;   // partial sums (INC leaves the second 0)
  double su[INC ? 1 : 2][INC ? 1 : 3][INC ? 1 : kHY][INC ? 1 : kHX];
  double sh[NS * 16];
  TS sx[2][9][kVY][kVX];   // exchanged corner forces
  T sdl[3][3][kHY][kHX];   // three planes: read in both halves of a step
};
template <typename T, bool FS, bool GEN, typename TS, bool INC>
__device__ __forceinline__ void residual_march(const Geo& g, const DeltaBufs<T>& D, const ContactDev& ct,
                                               const DevState* st, double* __restrict__ part, const TileGrid& tg,
                                               MarchLds<T, GEN, TS, INC>& lds) {
  static_assert(!INC || (!FS && !GEN && sizeof(TS) == sizeof(T)), "incremental pass: small strain, T stresses");
  using TU = std::conditional_t<INC, T, double>;
  constexpr int NS = MarchLds<T, GEN, TS, INC>::NS;
  auto &su = lds.su;
  auto &sdl = lds.sdl;
  auto &sx = lds.sx;
  double* const sh = lds.sh;
  const int tid = threadIdx.x;
  const int b = xcd_tile(blockIdx.x, gridDim.x);
  const int bx = b % tg.tx, by = (b / tg.tx) % tg.ty, bz = b / (tg.tx * tg.ty);
  const int x0 = bx * kTX, y0 = by * kTY;
  const int Nx = g.N[0], Ny = g.N[1], Nz = g.N[2];
  const int nx = g.n[0], ny = g.n[1], nz = g.n[2];
  const int zb = bz * tg.seg;
  const int ze = min(zb + tg.seg, Nz);
  const int NxNy = Nx * Ny;
  const int cur = ct.on ? st->vpar : 0;
  const int il = st->i_local, par = st->it & 1, acvp = (st->acv == 2), ecomb = st->accel_ok;
  const int slot = (il + 1) % 3;
  const bool kd_used = acvp && il >= 1;
  const bool dl = INC || kd_used;   // delta planes staged
  T* pc = D.p[par];
  const T* pp = D.p[par ^ 1];
  T* Rc = D.R[il & 3];
  double acc[NS];
#pragma unroll
  for (int q = 0; q < NS; ++q) acc[q] = 0.0;

  int off[kPR];
  plane_offsets(g, x0, y0, tid, off);
  double ru[INC ? 1 : kPR];
  T rd[kPR];
  auto fetch = [&](int pz) {
    const int mz = mirror_coord(g, pz, 2);
    const bool okz = mz >= 0 && mz < Nz;
#pragma unroll
    for (int r = 0; r < kPR; ++r) {
      const bool ok = okz && off[r] >= 0;
      const int a = off[r] + NxNy * mz;
      if constexpr (!INC) ru[r] = ok ? D.u[a] : 0.0;
      rd[r] = T(0);
      if (dl && ok) rd[r] = D.delta[a];
    }
  };
  auto commit = [&](int pz) {
#pragma unroll
    for (int r = 0; r < kPR; ++r) {
      const int e = tid + 256 * r;
      if (e < kPlane) {
        if constexpr (!INC) (&su[pz & 1][0][0][0])[e] = ru[r];
        if (dl) (&sdl[ring3(pz)][0][0][0])[e] = rd[r];
      }
    }
  };
  const int lx = tid & (kVX - 1), ly = tid / kVX;
  const int i = x0 - 1 + lx, j = y0 - 1 + ly;   // the thread's node, and its voxel's corner 000
  const bool nact = lx >= 1 && ly >= 1 && i < Nx && j < Ny;
  const VoxelXY vox = voxel_xy(g, i, j);
  const bool own = !INC && lx >= 1 && ly >= 1 && i < nx && j < ny;   // voxel whose norm this block counts
  const NodeXY nxy = node_xy(g, i, j);
  const int wx = lx >= 1 ? lx - 1 : 0, sy = ly >= 1 ? ly - 1 : 0;   // (unused values of the halo threads)
  // corners of the thread's voxel in plane pz
  auto read_corners = [&](int pz, TU (&cn)[4][3]) {
    const int s = pz & 1, r = ring3(pz);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      if constexpr (INC) {
        cn[0][c] = sdl[r][c][ly][lx];
        cn[1][c] = sdl[r][c][ly][lx + 1];
        cn[2][c] = sdl[r][c][ly + 1][lx];
        cn[3][c] = sdl[r][c][ly + 1][lx + 1];
      } else {
        cn[0][c] = su[s][c][ly][lx];
        cn[1][c] = su[s][c][ly][lx + 1];
        cn[2][c] = su[s][c][ly + 1][lx];
        cn[3][c] = su[s][c][ly + 1][lx + 1];
      }
    }
  };
  // A and S of K0 delta in plane pz at the thread's node (INC: cn are the plane's corners)
  auto read_stencil = [&](int pz, const TU (&cn)[4][3], T (&A)[3], T (&S)[3]) {
    const int r = ring3(pz);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      A[c] = S[c] = T(0);
      if (!kd_used) continue;
      const T d0 = INC ? (T)cn[0][c] : sdl[r][c][ly][lx], de = INC ? (T)cn[1][c] : sdl[r][c][ly][lx + 1];
      const T dn = INC ? (T)cn[2][c] : sdl[r][c][ly + 1][lx], dne = INC ? (T)cn[3][c] : sdl[r][c][ly + 1][lx + 1];
      const T dw = sdl[r][c][ly][wx], ds = sdl[r][c][sy][lx];
      const T dsw = sdl[r][c][sy][wx], dse = sdl[r][c][sy][lx + 1], dnw = sdl[r][c][ly + 1][wx];
      A[c] = T(g.st[c][0]) * d0 + T(g.st[c][1]) * ((dsw + dse) + (dnw + dne));
      S[c] = T(g.st[c][2]) * (dw + de) + T(g.st[c][3]) * (ds + dn);
    }
  };
  TailIn<T> tin;
  auto tail_at = [&](int z, TailIn<T>& t) {
    tail_load<T>(D, g.Nn, kd_used, INC, ecomb, pp, (long long)i + (long long)Nx * j + (long long)NxNy * z, t);
  };

  T lam, mu;
  TU lo[4][3];   // corners of the lower plane of the current layer
  TS fu[4][3];   // forces of the layer below on its upper corners
  T Kz[3], S0[3];   // A_z + S_{z-1}, S_z
  fetch(zb - 1);
  commit(zb - 1);
  fetch(zb);
  commit(zb);
  fetch(zb + 1);
  voxel_lame(g, vox, zb - 1, D.lam, D.mu, lam, mu);
  if (nact) tail_at(zb, tin);
  __syncthreads();
  {
    TU up[4][3];
    TS fl[4][3], vs = TS(0), ms[6];
    read_corners(zb - 1, lo);
    read_corners(zb, up);
    T A[3], S[3];
    read_stencil(zb - 1, lo, A, S);
    read_stencil(zb, up, A, S0);
#pragma unroll
    for (int c = 0; c < 3; ++c) Kz[c] = A[c] + S[c];
    voxel_forces<TU, TS, FS, false>(lo, up, (TS)lam, (TS)mu, fl, fu, vs, ms);
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int c = 0; c < 3; ++c) lo[k][c] = up[k][c];
  }
  voxel_lame(g, vox, zb, D.lam, D.mu, lam, mu);
  __syncthreads();
  commit(zb + 1);
  if (zb + 1 < ze) fetch(zb + 2);
  __syncthreads();
  for (int z = zb; z < ze; ++z) {
    TS (*ex)[kVY][kVX] = sx[z & 1];
    TS F0[3];   // forces on the thread's own corner (0, 0)
    {
      TU up[4][3];
      TS fl[4][3], fn[4][3];
      TS vs = TS(0), ms[6] = {TS(0), TS(0), TS(0), TS(0), TS(0), TS(0)};
      read_corners(z + 1, up);
      voxel_forces<TU, TS, FS, !INC>(lo, up, (TS)lam, (TS)mu, fl, fn, vs, ms);
      if (own) acc[1] += 8.0 * (double)vs;   // (1/2) sigma : sigma
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        F0[c] = fl[0][c] + fu[0][c];
#pragma unroll
        for (int k = 1; k < 4; ++k) ex[3 * (k - 1) + c][ly][lx] = fl[k][c] + fu[k][c];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          fu[k][c] = fn[k][c];
          lo[k][c] = up[k][c];
        }
      }
    }
    // the next layer's and the next node's inputs are requested as soon as their registers are free
    if (z + 1 < ze) {
      voxel_lame(g, vox, z + 1, D.lam, D.mu, lam, mu);
      commit(z + 2);
    }
    if (z + 2 < ze) fetch(z + 3);
    __syncthreads();
    T A1[3], S1[3];
    read_stencil(z + 1, lo, A1, S1);
    if (nact) {
      const NodeXY nz_ = node_z(g, z);
      const TS w2b = TS(1 << (nxy.b + nz_.b));
      const int anti = nxy.anti | nz_.anti;
      T p[3], kd[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const TS F = (F0[c] + ex[c][ly][lx - 1]) + (ex[3 + c][ly - 1][lx] + ex[6 + c][ly - 1][lx - 1]);
        p[c] = ((anti >> c) & 1) ? T(0) : (T)(-w2b * F);
        kd[c] = Kz[c] + S1[c];
      }
      const long long node = (long long)i + (long long)Nx * j + (long long)NxNy * z;
      delta_tail<T, GEN, INC>(g, D, ct, cur, kd_used, il, slot, pc, Rc, i, j, z, node, p, kd, tin, ecomb ? T(1) : T(0), acc);
      if (z + 1 < ze) tail_at(z + 1, tin);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      Kz[c] = A1[c] + S0[c];
      S0[c] = S1[c];
    }
  }
  block_sum<NS>(acc, sh);
  if (threadIdx.x == 0)
#pragma unroll
    for (int q = 0; q < NS; ++q) part[q * kPartRows + blockIdx.x] = acc[q];
  // rows the control sums beyond this grid (another instance's larger grid): cleared
  if (blockIdx.x == 0)
    for (int q = 0; q < NS; ++q)
      for (int r = (int)gridDim.x + tid; r < tg.rows; r += 256) part[q * kPartRows + r] = 0.0;
}

template <typename T, bool FS, bool GEN, typename TS, bool INC = false>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(!GEN && sizeof(TS) == 4 ? 3 : 1)))
void k_residual_dt(Geo g, DeltaBufs<T> D, ContactDev ct, DevState* st, double* __restrict__ part, TileGrid tg) {
  __shared__ MarchLds<T, GEN, TS, INC> lds;
  if (st->done || res_pass(st) != (INC ? PASS_INC : (sizeof(TS) == 8 ? PASS_U64 : PASS_U))) return;
  residual_march<T, FS, GEN, TS, INC>(g, D, ct, st, part, tg, lds);
}

// Contact or singular modes, in a solve that may switch to FP64 stresses: both passes in one launch
// (both run at two waves a SIMD, so neither loses by it; the launch that returned at once took
// 4.5 us of 87 an iteration on a 64x64x48 indentation).
template <typename T, bool FS>
__global__ __launch_bounds__(256) void k_residual_dg(Geo g, DeltaBufs<T> D, ContactDev ct, DevState* st,
                                                     double* __restrict__ part, TileGrid tg) {
  using L32 = MarchLds<T, true, T, false>;
  using L64 = MarchLds<T, true, double, false>;
  __shared__ __align__(16) unsigned char lds[sizeof(L64) > sizeof(L32) ? sizeof(L64) : sizeof(L32)];
  if (st->done) return;
  if (res_pass(st) == PASS_U64)
    residual_march<T, FS, true, double, false>(g, D, ct, st, part, tg, *reinterpret_cast<L64*>(lds));
  else
    residual_march<T, FS, true, T, false>(g, D, ct, st, part, tg, *reinterpret_cast<L32*>(lds));
}

// Mean stress of the residual-form iterate, once, when the solve is reported: per voxel the
// stresses of its two tetrahedra as the tiled residual pass forms them (differences of the
// FP64 displacement against corner 000, rounded to T; the stress arithmetic in T), added in T
// and weighted by the integration-point weight 1/2 into FP64 block sums.  Components in the
// order xx, yy, zz, yz, xz, xy (first Piola-Kirchhoff for finite strain).
// A thread owns a column of voxels over a segment of z: the upper corners of a layer are the
// lower ones of the next (12 loads a voxel, requested a layer ahead), and nothing is divided.
// Bound by the 540 MB and the loads in flight: 256^3 181 us (one voxel per thread and step, with 24
// loads and three 64-bit divisions: 290 us).
constexpr int kMSX = 64, kMSY = kBlock / kMSX;
template <typename T, bool FS>
__global__ __launch_bounds__(kBlock) void k_mean_stress_d(Geo g, const double* __restrict__ u,
                                                          const T* __restrict__ lam, const T* __restrict__ mu,
                                                          double* __restrict__ part, int tx, int ty, int seg) {
  __shared__ double sh[6 * 16];
  double acc[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  const int nx = g.n[0], ny = g.n[1], Nx = g.N[0], NxNy = g.N[0] * g.N[1];
  const int units = tx * ty * ((g.n[2] + seg - 1) / seg), per = (units + gridDim.x - 1) / gridDim.x;
  const int first = xcd_tile(blockIdx.x, gridDim.x) * per;
  for (int b = first; b < min(first + per, units); ++b) {
    const int vx = (b % tx) * kMSX + (int)threadIdx.x % kMSX, vy = (b / tx) % ty * kMSY + (int)threadIdx.x / kMSX;
    const int zb = b / (tx * ty) * seg, ze = vx < nx && vy < ny ? min(zb + seg, g.n[2]) : zb;
    int at[4];   // corners (0,0), (1,0), (0,1), (1,1) in a plane (on a periodic axis there are n nodes)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int x = vx + (q & 1), y = vy + (q >> 1);
      at[q] = (x == g.N[0] ? 0 : x) + Nx * (y == g.N[1] ? 0 : y);
    }
    double nxt[4][3], uc[8][3];
    auto fetch = [&](int z) {
      const double* pl = u + (long long)NxNy * (z == g.N[2] ? 0 : z);
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) nxt[q][c] = pl[c * g.Nn + at[q]];
    };
    auto take = [&](int h) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int c = 0; c < 3; ++c) uc[h + q][c] = nxt[q][c];
    };
    T l = T(0), m = T(0);
    const int col = vx + nx * vy, nxny = nx * ny;
    if (zb < ze) {
      fetch(zb);
      take(4);
      fetch(zb + 1);
      l = lam[col + nxny * zb];
      m = mu[col + nxny * zb];
    }
    for (int vz = zb; vz < ze; ++vz) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int c = 0; c < 3; ++c) uc[q][c] = uc[4 + q][c];
      take(4);
      const T l0 = l, m0 = m;
      if (vz + 1 < ze) {
        fetch(vz + 2);
        l = lam[col + nxny * (vz + 1)];
        m = mu[col + nxny * (vz + 1)];
      }
      T vs[6] = {T(0), T(0), T(0), T(0), T(0), T(0)};
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        T G[3][3];
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
          for (int b = 0; b < 3; ++b) G[a][b] = T(0);
#pragma unroll
        for (int cc = 1; cc < 8; ++cc) {
          const int cx = cc & 1, cy = (cc >> 1) & 1, cz = (cc >> 2) & 1;
          if (((cx + cy + cz) & 1) != t) continue;
          const T sx = T(cx ? 0.5 : -0.5), sy = T(cy ? 0.5 : -0.5), sz = T(cz ? 0.5 : -0.5);
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            const T d = (T)(uc[cc][a] - uc[0][a]);
            G[a][0] += sx * d;
            G[a][1] += sy * d;
            G[a][2] += sz * d;
          }
        }
        if constexpr (FS) {
          T P[3][3];
          svk_pk1<T>(G, l0, m0, P);
          vs[0] += P[0][0];
          vs[1] += P[1][1];
          vs[2] += P[2][2];
          vs[3] += P[1][2];
          vs[4] += P[0][2];
          vs[5] += P[0][1];
        } else {
          const T tr = G[0][0] + G[1][1] + G[2][2];
          vs[0] += l0 * tr + T(2) * m0 * G[0][0];
          vs[1] += l0 * tr + T(2) * m0 * G[1][1];
          vs[2] += l0 * tr + T(2) * m0 * G[2][2];
          vs[3] += m0 * (G[1][2] + G[2][1]);
          vs[4] += m0 * (G[0][2] + G[2][0]);
          vs[5] += m0 * (G[0][1] + G[1][0]);
        }
      }
#pragma unroll
      for (int q = 0; q < 6; ++q) acc[q] += 0.5 * (double)vs[q];
    }
  }
  block_sum<6>(acc, sh);
  if (threadIdx.x == 0)
#pragma unroll
    for (int q = 0; q < 6; ++q) part[blockIdx.x * 6 + q] = acc[q];
}

// proj_P of the relations on several nodes (eq 14, eq 17) on p and on the quantities linear
// in p (R, and the difference dY): one wavefront per relation, one lane per support node.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_weak_d(Geo g, DeltaBufs<T> D, WeakDev w, DevState* st) {
  if (st->done) return;
  const long long r = (blockIdx.x * (long long)blockDim.x + threadIdx.x) >> 6;
  if (r >= w.m) return;   // uniform over the wavefront
  const int lane = threadIdx.x & 63;
  const int c = w.comp[r];
  const int il = st->i_local, par = st->it & 1, acvp = (st->acv == 2);
  const int slot = (il + 1) % 3;
  const long long o0 = w.off[r];
  const bool act = lane < w.off[r + 1] - o0;
  long long node = 0;
  double wa = 0.0, wb = 0.0, q = 0.0, scale = 1.0;
  if (act) {
    node = w.nodes[o0 + lane];
    wa = w.wa[o0 + lane];
    wb = w.wb[o0 + lane];
    const int i = (int)(node % g.N[0]);
    const long long t = node / g.N[0];
    const int j = (int)(t % g.N[1]), k = (int)(t / g.N[1]);
    T p[3];
    double sn = 0.0, ms[6];
    // the stresses in the precision the residual pass of this iteration used
    if (st->fine) {
      if (g.fs) node_eval_d<T, false, true, double>(g, D.u, D.lam, D.mu, i, j, k, p, sn, ms);
      else node_eval_d<T, false, false, double>(g, D.u, D.lam, D.mu, i, j, k, p, sn, ms);
    } else {
      if (g.fs) node_eval_d<T, false, true>(g, D.u, D.lam, D.mu, i, j, k, p, sn, ms);
      else node_eval_d<T, false, false>(g, D.u, D.lam, D.mu, i, j, k, p, sn, ms);
    }
    const int xyz[3] = {i, j, k};
    scale = (double)(1 << bcount(g, xyz));
    q = (double)p[c] / scale;
  }
  const double num = wave_sum(wa * q), den = wave_sum(wa * wb), sb = wave_sum(wb);
  const double f = num / den;
  const double pnew = (q - wb * f) * scale;
  const double pn = wave_sum(act ? pnew * pnew : 0.0);
  if (act) {
    const long long e = c * g.Nn + node;
    const T sh = (T)(wb * f * scale);
    D.p[par][e] = (T)pnew;
    if (acvp && il >= 1) {
      D.R[il & 3][e] -= sh;
      if (il >= 2) D.dY[slot][e] -= sh;
    }
  }
  if (lane == 0) {
    w.part[r] = pn;
    w.react[r] = -f * sb;
  }
}

// Gram matrix of the R differences and their products with R_i (accelerating iterations).
// The difference formed at local iteration j >= 2, R_j - R_{j-1} (FP32), pairs with the Y
// difference in slot (j + 1) mod 3; the three latest, j = i, i-1, i-2, come from the ring of
// four R fields (acceleration starts at i = 4, so all four are of the current run).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_gram3(DeltaBufs<T> D, long long n3, DevState* st, double* __restrict__ gpart) {
  __shared__ double sh[9 * 16];
  if (st->done || !st->accel) return;
  const int il = st->i_local;
  // d_k = R_{i-k} - R_{i-k-1}, k = 0, 1, 2: four fields, each read once
  const T *r0 = D.R[il & 3], *r1 = D.R[(il + 3) & 3], *r2 = D.R[(il + 2) & 3], *r3 = D.R[(il + 1) & 3];
  double acc[9];
#pragma unroll
  for (int q = 0; q < 9; ++q) acc[q] = 0.0;
  auto add = [&](T a, T b, T c, T d) {
    const double r = a, d0 = (T)(a - b), d1 = (T)(b - c), d2 = (T)(c - d);
    acc[0] += d0 * d0; acc[1] += d0 * d1; acc[2] += d0 * d2;
    acc[3] += d1 * d1; acc[4] += d1 * d2; acc[5] += d2 * d2;
    acc[6] += d0 * r; acc[7] += d1 * r; acc[8] += d2 * r;
  };
  typedef T T4 __attribute__((ext_vector_type(4)));
  const long long n4 = n3 / 4, step = (long long)gridDim.x * blockDim.x;   // (fields are 256-byte aligned)
  const long long t0 = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  for (long long e = t0; e < n4; e += step) {
    const T4 a = ((const T4*)r0)[e], b = ((const T4*)r1)[e], c = ((const T4*)r2)[e], d = ((const T4*)r3)[e];
#pragma unroll
    for (int k = 0; k < 4; ++k) add(a[k], b[k], c[k], d[k]);
  }
  if (t0 < n3 - 4 * n4) {
    const long long e = 4 * n4 + t0;
    add(r0[e], r1[e], r2[e], r3[e]);
  }
  block_sum<9>(acc, sh);
  if (threadIdx.x == 0) {
    // column of the pair of slots (s, t), s <= t, is s (5 - s) / 2 + t; of slot s with R_i 6 + s
    int k = 0;
    for (int a = 0; a < 3; ++a) {
      const int sa = (il - a + 1) % 3;
      for (int b = a; b < 3; ++b, ++k) {
        const int sb = (il - b + 1) % 3, lo = sa < sb ? sa : sb, hi = sa < sb ? sb : sa;
        gpart[(lo * (5 - lo) / 2 + hi) * kPartRows + blockIdx.x] = acc[k];
      }
      gpart[(6 + sa) * kPartRows + blockIdx.x] = acc[6 + a];
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_alpha3(DevState* st, const double* __restrict__ gpart, int nblk) {
  __shared__ double acc[9];
  if (st->done || !st->accel) return;
  col_sums(gpart, kPartRows, nblk, 9, acc);
  if (threadIdx.x != 0) return;
  double G[3][4] = {{acc[0], acc[1], acc[2], acc[6]}, {acc[1], acc[3], acc[4], acc[7]}, {acc[2], acc[4], acc[5], acc[8]}};
  const double tr = G[0][0] + G[1][1] + G[2][2];
  for (int a = 0; a < 3; ++a) G[a][a] += 1e-14 * tr / 3.0;
  double y[3];
  bool ok = solve_pivoted<3>(G, y);
  if (ok) ok = isfinite(y[0]) && isfinite(y[1]) && isfinite(y[2]);
  if (ok)
    for (int a = 0; a < 3; ++a) st->gamma[a] = y[a];
  st->accel_ok = ok ? 1 : 0;
}

// The iteration counters move on in the last kernel of an iteration (its first thread; the
// other threads of that kernel read only the done flag), which saves a launch.
__device__ __forceinline__ void advance_iteration(DevState* st, int advance) {
  if (advance && blockIdx.x == 0 && threadIdx.x == 0) {
    st->it += 1;
    st->i_local += 1;
  }
}

// proj_U of the residual-form path on the FP64 displacement; the increment follows
template <typename T>
__global__ __launch_bounds__(kBlock) void k_proj_d(Geo g, DeltaBufs<T> D, StrongDev s, WeakDev w, ContactDev ct,
                                                   DevState* st, int force, int advance) {
  if (!force && st->done) return;
  advance_iteration(st, advance);
  const long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  // strong DOFs
  if (e < s.m) {
    const long long idx = s.comp[e] * g.Nn + s.node[e];
    const double old = D.u[idx];
    D.u[idx] = s.val[e];
    D.delta[idx] = (T)((double)D.delta[idx] + (s.val[e] - old));
  }
  // contact nodes: radial projection onto the sphere
  if (ct.on && e < ct.nface && ct.C[e]) {
    int xyz[3];
    xyz[ct.axis] = ct.side ? g.n[ct.axis] : 0;
    xyz[ct.b1] = (int)(e % g.N[ct.b1]);
    xyz[ct.b2] = (int)(e / g.N[ct.b1]);
    const long long node = xyz[0] + (long long)g.N[0] * (xyz[1] + (long long)g.N[1] * xyz[2]);
    double d[3], r2 = 0.0;
    for (int c = 0; c < 3; ++c) {
      d[c] = xyz[c] + D.u[c * g.Nn + node] - ct.center[c];
      r2 += d[c] * d[c];
    }
    const double rr = sqrt(r2);
    for (int c = 0; c < 3; ++c) {
      const long long idx = c * g.Nn + node;
      const double nw = ct.center[c] + ct.radius * d[c] / rr - xyz[c];
      D.delta[idx] = (T)((double)D.delta[idx] + (nw - D.u[idx]));
      D.u[idx] = nw;
    }
  }
}

// proj_U of the relations (eq 11, eq 15) on the FP64 displacement, the increment follows
template <typename T>
__global__ __launch_bounds__(kBlock) void k_proj_rel_d(Geo g, DeltaBufs<T> D, WeakDev w, DevState* st, int force,
                                                       int advance) {
  if (!force && st->done) return;
  advance_iteration(st, advance);
  const long long r = (blockIdx.x * (long long)blockDim.x + threadIdx.x) >> 6;
  if (r >= w.m) return;
  const int lane = threadIdx.x & 63;
  const long long o0 = w.off[r];
  const bool act = lane < w.off[r + 1] - o0;
  long long e = 0;
  double wa = 0.0, wd = 0.0, v = 0.0;
  if (act) {
    e = w.comp[r] * g.Nn + w.nodes[o0 + lane];
    wa = w.wa[o0 + lane];
    wd = w.wd[o0 + lane];
    v = D.u[e];
  }
  const double num = wave_sum(wa * v), den = wave_sum(wa * wd);
  const double corr = (w.val[r] - num) / den;
  if (act) {
    D.u[e] = v + wd * corr;
    D.delta[e] = (T)((double)D.delta[e] + wd * corr);
  }
}

template <typename T>
__global__ void k_advance(DevState* st) {
  if (st->done) return;
  st->it += 1;
  st->i_local += 1;
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_reactions_d(Geo g, DeltaBufs<T> D, StrongDev s, double* out) {
  const long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (e >= s.m) return;
  const long long node = s.node[e];
  const int i = (int)(node % g.N[0]);
  const long long q = node / g.N[0];
  const int j = (int)(q % g.N[1]), k = (int)(q / g.N[1]);
  // reactions are multipliers: the stresses here are formed in FP64 (p rounded once)
  T p[3];
  double sn = 0.0, ms[6];
  if (g.fs) node_eval_d<T, false, true, double>(g, D.u, D.lam, D.mu, i, j, k, p, sn, ms);
  else node_eval_d<T, false, false, double>(g, D.u, D.lam, D.mu, i, j, k, p, sn, ms);
  const int xyz[3] = {i, j, k};
  out[e] = -(double)p[s.comp[e]] / (double)(1 << bcount(g, xyz));
}

// ---------------------------------------------------------------------------
// launch wrappers
// ---------------------------------------------------------------------------

template <typename T, typename TS>
void launch_delta_residual_ts(const Geo& g, const DeltaBufs<T>& D, const ContactDev& ct, DevState* st, double* part,
                              int nblk, const TileGrid& tg, bool gen, hipStream_t s) {
  if (tg.tx > 0) {
    const dim3 grid(tg.tx * tg.ty * tg.nseg), block(256);
    if constexpr (sizeof(TS) == 4) {
      if (gen) {
        if (g.fs) hipLaunchKernelGGL((k_residual_dt<T, true, true, TS>), grid, block, 0, s, g, D, ct, st, part, tg);
        else hipLaunchKernelGGL((k_residual_dt<T, false, true, TS>), grid, block, 0, s, g, D, ct, st, part, tg);
        return;
      }
    }
    if (g.fs) hipLaunchKernelGGL((k_residual_dt<T, true, false, TS>), grid, block, 0, s, g, D, ct, st, part, tg);
    else hipLaunchKernelGGL((k_residual_dt<T, false, false, TS>), grid, block, 0, s, g, D, ct, st, part, tg);
  } else {
    if (g.fs) hipLaunchKernelGGL((k_residual_d<T, true, TS>), dim3(nblk), dim3(kBlock), 0, s, g, D, ct, st, part);
    else hipLaunchKernelGGL((k_residual_d<T, false, TS>), dim3(nblk), dim3(kBlock), 0, s, g, D, ct, st, part);
  }
}

// The pass with T stresses, (refine) the pass with FP64 stresses and (inc) the incremental
// pass; the device state selects the one that works, the others return at once.  All write
// the partial rows the control step reads (the returned count).  inc is taken only for tiled
// small-strain problems without contact or singular modes (the caller's eligibility test).
template <typename T>
int launch_delta_residual(const Geo& g, const DeltaBufs<T>& D, const ContactDev& ct, DevState* st, double* part,
                          int nblk, int refine, int inc, int which, hipStream_t s) {
  const bool gen = ct.on || g.sing[0] || g.sing[1] || g.sing[2];
  const bool use_inc = inc && !g.fs && !gen;
  // each pass on the grid for its own resident count; the control sums the largest count of rows,
  // and a pass on a smaller grid clears the rows beyond it
  TileGrid tf = residual_tiles(g, gen, false);
  TileGrid ti = use_inc ? residual_tiles(g, false, true) : tf;
  TileGrid tu = refine ? residual_tiles_fp64(g, gen) : tf;
  if (tf.tx > 0) {
    const int rows = std::max(tf.rows, std::max(ti.rows, tu.rows));
    tf.rows = ti.rows = tu.rows = rows;
  }
  if (gen && refine && tu.tx > 0) {
    const dim3 grid(tu.tx * tu.ty * tu.nseg), block(256);
    tu.rows = grid.x;
    if (g.fs) hipLaunchKernelGGL((k_residual_dg<T, true>), grid, block, 0, s, g, D, ct, st, part, tu);
    else hipLaunchKernelGGL((k_residual_dg<T, false>), grid, block, 0, s, g, D, ct, st, part, tu);
    return tu.rows;
  }
  if (which & L_U) launch_delta_residual_ts<T, T>(g, D, ct, st, part, nblk, tf, gen, s);
  if (refine && (which & L_U64)) launch_delta_residual_ts<T, double>(g, D, ct, st, part, nblk, tu, gen, s);
  if (use_inc && ti.tx > 0 && (which & L_INC))
    hipLaunchKernelGGL((k_residual_dt<T, false, false, T, true>), dim3(ti.tx * ti.ty * ti.nseg), dim3(256), 0, s, g, D,
                       ct, st, part, ti);
  return tf.tx > 0 ? tf.rows : nblk;
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_diff(const T* __restrict__ a, const T* __restrict__ b, T* __restrict__ out,
                                                 long long n) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x)
    out[e] = a[e] - b[e];
}

template <typename T>
void launch_diff(const T* a, const T* b, T* out, long long n, hipStream_t s) {
  const int nblk = (int)std::max<long long>(1, std::min<long long>(4096, (n + kBlock - 1) / kBlock));
  hipLaunchKernelGGL(k_diff<T>, dim3(nblk), dim3(kBlock), 0, s, a, b, out, n);
}

template <typename T>
int launch_mean_stress_d(const Geo& g, const DeltaBufs<T>& D, double* part, hipStream_t s) {
  // segments of z for up to 1024 blocks (four a CU)
  const int tx = (g.n[0] + kMSX - 1) / kMSX, ty = (g.n[1] + kMSY - 1) / kMSY;
  const int want = std::max(1, std::min(g.n[2], 1024 / std::max(1, tx * ty)));
  const int seg = (g.n[2] + want - 1) / want;
  const int nblk = std::min(1024, tx * ty * ((g.n[2] + seg - 1) / seg));
  const dim3 grid(nblk), block(kBlock);
  if (g.fs) hipLaunchKernelGGL((k_mean_stress_d<T, true>), grid, block, 0, s, g, D.u, D.lam, D.mu, part, tx, ty, seg);
  else hipLaunchKernelGGL((k_mean_stress_d<T, false>), grid, block, 0, s, g, D.u, D.lam, D.mu, part, tx, ty, seg);
  return nblk;
}

template <typename T>
void launch_delta_control(const Geo& g, const DeltaBufs<T>& D, const ContactDev& ct, const WeakDev& w, DevState* st,
                          const double* part, const double* wpart, int nblk, hipStream_t s) {
  if (w.m > 0) hipLaunchKernelGGL(k_weak_d<T>, dim3(rel_grid(w.m)), dim3(kBlock), 0, s, g, D, w, st);
  // the tiled passes without contact or singular modes leave the two norms only
  const bool gen = ct.on || g.sing[0] || g.sing[1] || g.sing[2] || residual_tiles(g, false, false).tx <= 0;
  launch_control(st, part, nblk, wpart, w.m, ct, gen ? kPartStrideD : 2, s);
}

// Blocks of a residual pass instance resident on the current device at once (blocks per CU at
// its register and LDS use, times the CU count), queried once per device and instance.
int resident_blocks(const void* kernel, std::atomic<int> (&cache)[64]) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 512;
  int r = cache[dev].load(std::memory_order_relaxed);
  if (!r) {
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 256, 0) != hipSuccess || per_cu < 1) per_cu = 1;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 1;
    r = per_cu * cus;
    cache[dev].store(r, std::memory_order_relaxed);   // every thread computes the same value
  }
  return r;
}
template <bool FS, bool GEN, typename TS, bool INC>
static int residual_resident() {
  static std::atomic<int> cache[64] = {};
  return resident_blocks((const void*)k_residual_dt<float, FS, GEN, TS, INC>, cache);
}

// segment length with the fewest (rounds x planes per block) for a resident count; ties go to
// fewer segments
static int tile_split(const Geo& g, int tx, int ty, long long resident) {
  const int Nz = g.N[2];
  const int maxseg = std::max(1, std::min(Nz, kPartRows / (tx * ty)));
  long long best = -1;
  int bseg = Nz;
  for (int ns = 1; ns <= maxseg; ++ns) {
    const int seg = (Nz + ns - 1) / ns;
    const long long blocks = (long long)tx * ty * ((Nz + seg - 1) / seg);
    const long long cost = (blocks + resident - 1) / resident * (seg + 2);
    if (best < 0 || cost < best) {
      best = cost;
      bseg = seg;
    }
  }
  return bseg;
}

// Tile grid of a residual pass instance with this many resident blocks: tiles of kTX x kTY node
// columns, z split into segments, at most kPartRows blocks (the partial-sum rows); tx = 0 when the
// node plane alone needs more tiles than that.  A block marches its segment's planes plus two
// planes of prologue, and the blocks run in rounds of the resident count, so the split taken is
// the one with the fewest (rounds x planes per block); ties go to fewer segments.  Every instance
// has its own split: on another's grid it may run in two rounds.
TileGrid tile_grid_for(const Geo& g, int resident) {
  const int tx = (g.N[0] + kTX - 1) / kTX, ty = (g.N[1] + kTY - 1) / kTY;
  if ((long long)tx * ty > kPartRows) return TileGrid{0, 0, 0, 0, 0};
  TileGrid t{tx, ty, 0, tile_split(g, tx, ty, resident), 0};
  t.nseg = (g.N[2] + t.seg - 1) / t.seg;
  t.rows = tx * ty * t.nseg;
  return t;
}

// gen: the instance for contact or singular modes; inc: the incremental pass
TileGrid residual_tiles(const Geo& g, bool gen, bool inc) {
  if (inc) return tile_grid_for(g, residual_resident<false, false, float, true>());
  if (g.fs)
    return tile_grid_for(g, gen ? residual_resident<true, true, float, false>() : residual_resident<true, false, float, false>());
  return tile_grid_for(g, gen ? residual_resident<false, true, float, false>() : residual_resident<false, false, float, false>());
}
// the pass with FP64 stresses (gen: both passes in one launch)
TileGrid residual_tiles_fp64(const Geo& g, bool gen) {
  static std::atomic<int> cache[2][64] = {};
  if (gen)
    return tile_grid_for(g, g.fs ? resident_blocks((const void*)k_residual_dg<float, true>, cache[1])
                                 : resident_blocks((const void*)k_residual_dg<float, false>, cache[0]));
  return tile_grid_for(g, g.fs ? residual_resident<true, false, double, false>() : residual_resident<false, false, double, false>());
}

template <typename T>
void launch_delta_anderson(const DeltaBufs<T>& D, long long n3, DevState* st, double* gpart, int nblk, hipStream_t s) {
  // four values per thread and step, two steps at least: on small grids the block sums set the time
  nblk = (int)std::max<long long>(1, std::min<long long>(nblk, n3 / (8 * kBlock)));
  hipLaunchKernelGGL(k_gram3<T>, dim3(nblk), dim3(kBlock), 0, s, D, n3, st, gpart);
  hipLaunchKernelGGL(k_alpha3, dim3(1), dim3(kBlock), 0, s, st, gpart, nblk);
}

template <typename T>
void launch_delta_proj(const Geo& g, const DeltaBufs<T>& D, const StrongDev& sd, const WeakDev& w,
                       const ContactDev& ct, DevState* st, int force, int advance, hipStream_t s) {
  long long m = sd.m;
  if (ct.on && ct.nface > m) m = ct.nface;
  const int rel = w.m > 0;
  if (m > 0)
    hipLaunchKernelGGL(k_proj_d<T>, dim3(grid_for(m, 1 << 30)), dim3(kBlock), 0, s, g, D, sd, w, ct, st, force,
                       advance && !rel);
  if (rel) hipLaunchKernelGGL(k_proj_rel_d<T>, dim3(rel_grid(w.m)), dim3(kBlock), 0, s, g, D, w, st, force, advance);
  if (advance && m == 0 && !rel) hipLaunchKernelGGL(k_advance<T>, dim3(1), dim3(1), 0, s, st);
}

template <typename T>
void launch_reactions_d(const Geo& g, const DeltaBufs<T>& D, const StrongDev& sd, double* out, hipStream_t s) {
  if (sd.m == 0) return;
  hipLaunchKernelGGL(k_reactions_d<T>, dim3(grid_for(sd.m, 1 << 30)), dim3(kBlock), 0, s, g, D, sd, out);
}

template <typename T>
void launch_weak_d_stage(const Geo& g, const DeltaBufs<T>& D, const WeakDev& w, DevState* st, hipStream_t s) {
  if (w.m > 0) hipLaunchKernelGGL(k_weak_d<T>, dim3(rel_grid(w.m)), dim3(kBlock), 0, s, g, D, w, st);
}

template int launch_delta_residual<float>(const Geo&, const DeltaBufs<float>&, const ContactDev&, DevState*, double*,
                                          int, int, int, int, hipStream_t);
template void launch_delta_control<float>(const Geo&, const DeltaBufs<float>&, const ContactDev&, const WeakDev&,
                                          DevState*, const double*, const double*, int, hipStream_t);
template void launch_delta_anderson<float>(const DeltaBufs<float>&, long long, DevState*, double*, int, hipStream_t);
template void launch_delta_proj<float>(const Geo&, const DeltaBufs<float>&, const StrongDev&, const WeakDev&,
                                       const ContactDev&, DevState*, int, int, hipStream_t);
template void launch_diff<float>(const float*, const float*, float*, long long, hipStream_t);
template int launch_mean_stress_d<float>(const Geo&, const DeltaBufs<float>&, double*, hipStream_t);
template void launch_reactions_d<float>(const Geo&, const DeltaBufs<float>&, const StrongDev&, double*, hipStream_t);

}  // namespace fftc
