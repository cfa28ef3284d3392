// Shared parts of the tiled residual passes (fftc_residual.hip, fftc_kernels.hip): a block owns a
// kTX x kTY column of nodes and marches along z over a segment of node planes.
//
// Thread (lx, ly) of the 32 x 8 block owns the voxel whose corner 000 is the node (x0 - 1 + lx,
// y0 - 1 + ly), and, for lx, ly >= 1, that node.  Per step the next node plane sits in LDS with a
// one-node halo; a thread reads its voxel's four upper corners (the lower ones are the last
// step's, in registers), forms both tetrahedra's stresses and from them the forces on the
// eight corners, adds the forces on its lower corners to what the layer below left on them, and
// passes three of the four corners' sums to its neighbours through LDS.  Against passing the
// stresses (12 written and 48 read per thread and step, every corner force formed by the node)
// this exchanges 9 values, forms each force once, and needs one barrier per step: planes are rings
// of two or three, the exchange a double buffer, each rewritten only after the barrier that
// follows its last read.
#pragma once

#include <atomic>

#include "fftc_internal.h"
#include "fftc_common.h"

namespace fftc {

constexpr int kTX = 31, kTY = 7;              // nodes of a tile; 32 x 8 = 256 voxels per layer
constexpr int kVX = kTX + 1, kVY = kTY + 1;   // voxels x0-1 .. x0+kTX-1
constexpr int kHX = kTX + 2, kHY = kTY + 2;   // node tile with halo: x0-1 .. x0+kTX
constexpr int kPlane = 3 * kHY * kHX;         // values of one staged node plane
constexpr int kPR = (kPlane + 255) / 256;     // of them per thread

int resident_blocks(const void* kernel, std::atomic<int> (&cache)[64]);
TileGrid tile_grid_for(const Geo& g, int resident);

// slot of node plane pz (>= -1) in a ring of three
__device__ __forceinline__ int ring3(int pz) { return (pz + 3) % 3; }

// Offsets of the plane values thread tid stages, within a node plane (component and (x, y), the
// stencil's mirror or periodic image outside the grid); -1: none
__device__ __forceinline__ void plane_offsets(const Geo& g, int x0, int y0, int tid, int (&off)[kPR]) {
#pragma unroll
  for (int r = 0; r < kPR; ++r) {
    const int e = tid + 256 * r;
    const int c = e / (kHY * kHX), q = e - c * (kHY * kHX);
    const int hy = q / kHX, hx = q - hy * kHX;
    const int mx = mirror_coord(g, x0 - 1 + hx, 0), my = mirror_coord(g, y0 - 1 + hy, 1);
    const bool ok = e < kPlane && mx >= 0 && mx < g.N[0] && my >= 0 && my < g.N[1];
    off[r] = ok ? (int)(c * g.Nn) + mx + g.N[0] * my : -1;
  }
}

// Corner forces of one voxel (times -1, without the boundary weight) from its corner values:
// lo and up hold the corners (0,0), (1,0), (0,1), (1,1) of the lower and upper plane.  The
// tetrahedra are {000, 110, 101, 011} and {100, 010, 001, 111}: each corner belongs to one.  The
// gradient's halves and the force's quarters are folded into the Lame values (exact); differences
// are formed in TU and rounded once to TS.  vs gains the voxel's sum of sigma : sigma / 16, ms the
// components xx, yy, zz, yz, xz, xy of sigma / 4 summed over the tetrahedra, both in TA.
template <typename TU, typename TS, bool FS, bool SIG, typename TA>
__device__ __forceinline__ void voxel_forces(const TU (&lo)[4][3], const TU (&up)[4][3], TS l, TS m, TS (&fl)[4][3],
                                             TS (&fu)[4][3], TA& vs, TA (&ms)[6]) {
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    TS G[3][3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      // t = 0: 000, 110, 101, 011; t = 1: 100, 010, 001, 111
      const TU a = t ? lo[1][r] : lo[0][r], b = t ? lo[2][r] : lo[3][r];
      const TU c = t ? up[0][r] : up[1][r], d = t ? up[3][r] : up[2][r];
      const TU p = t ? a - b : b - a, q = t ? d - c : c - d;
      G[r][0] = (TS)(p + q);
      G[r][1] = t ? (TS)(q - p) : (TS)(p - q);
      G[r][2] = (TS)((c - a) + (d - b));
    }
    TS s[3][3];   // sigma / 4
    if constexpr (FS) {
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int q = 0; q < 3; ++q) G[r][q] *= TS(0.5);
      svk_pk1<TS>(G, TS(0.25) * l, TS(0.25) * m, s);
    } else {
      const TS l8 = TS(0.125) * l, m8 = TS(0.125) * m;
      const TS tr = l8 * (G[0][0] + G[1][1] + G[2][2]);
      s[0][0] = tr + TS(2) * m8 * G[0][0];
      s[1][1] = tr + TS(2) * m8 * G[1][1];
      s[2][2] = tr + TS(2) * m8 * G[2][2];
      s[0][1] = s[1][0] = m8 * (G[0][1] + G[1][0]);
      s[0][2] = s[2][0] = m8 * (G[0][2] + G[2][0]);
      s[1][2] = s[2][1] = m8 * (G[1][2] + G[2][1]);
    }
    if constexpr (SIG) {
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int q = 0; q < 3; ++q)
          if (FS || q >= r) vs += ((!FS && q > r) ? TA(2) : TA(1)) * ((TA)s[r][q] * (TA)s[r][q]);
      ms[0] += (TA)s[0][0];
      ms[1] += (TA)s[1][1];
      ms[2] += (TA)s[2][2];
      ms[3] += (TA)s[1][2];
      ms[4] += (TA)s[0][2];
      ms[5] += (TA)s[0][1];
    }
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const TS al = s[r][0] + s[r][1], be = s[r][0] - s[r][1], z = s[r][2];
      if (t == 0) {
        fl[0][r] = -(al + z);
        fl[3][r] = al - z;
        fu[1][r] = be + z;
        fu[2][r] = z - be;
      } else {
        fl[1][r] = be - z;
        fl[2][r] = -(be + z);
        fu[0][r] = z - al;
        fu[3][r] = al + z;
      }
    }
  }
}

// The voxel whose corner 000 is node (i, j), within a layer
struct VoxelXY {
  int at;
  bool ok;   // inside the grid
};
__device__ __forceinline__ VoxelXY voxel_xy(const Geo& g, int i, int j) {
  const int nx = g.n[0], ny = g.n[1];
  bool ok = true;
  if (g.periodic[0]) i = (i + nx) % nx;
  else ok = i >= 0 && i < nx;
  if (g.periodic[1]) j = (j + ny) % ny;
  else ok = ok && j >= 0 && j < ny;
  return VoxelXY{i + nx * j, ok};
}
// its Lame values in layer lz; 0 outside the grid
template <typename T>
__device__ __forceinline__ void voxel_lame(const Geo& g, const VoxelXY& v, int lz, const T* __restrict__ lam,
                                           const T* __restrict__ mu, T& l, T& m) {
  bool ok = v.ok;
  const int nz = g.n[2];
  int vz = lz;
  if (g.periodic[2]) vz = (lz + nz) % nz;
  else ok = ok && lz >= 0 && lz < nz;
  l = m = T(0);
  if (ok) {
    const int at = v.at + g.n[0] * g.n[1] * vz;
    l = lam[at];
    m = mu[at];
  }
}

// What a thread knows of its node before the march: in-plane part of the boundary count and of the
// components held at 0
struct NodeXY {
  int b, anti;
};
__device__ __forceinline__ NodeXY node_xy(const Geo& g, int i, int j) {
  NodeXY n{0, 0};
  const int xy[2] = {i, j};
#pragma unroll
  for (int J = 0; J < 2; ++J) {
    if (g.periodic[J]) continue;
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      if (xy[J] != (f ? g.n[J] : 0)) continue;
      n.b += 1;
#pragma unroll
      for (int c = 0; c < 3; ++c) n.anti |= ((g.aface >> (c * 6 + J * 2 + f)) & 1) << c;
    }
  }
  return n;
}
// the z part, uniform over the block
__device__ __forceinline__ NodeXY node_z(const Geo& g, int z) {
  NodeXY n{0, 0};
  if (g.periodic[2]) return n;
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    if (z != (f ? g.n[2] : 0)) continue;
    n.b += 1;
#pragma unroll
    for (int c = 0; c < 3; ++c) n.anti |= ((g.aface >> (c * 6 + 4 + f)) & 1) << c;
  }
  return n;
}

}  // namespace fftc
