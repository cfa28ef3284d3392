// Transforms as matrix products on the FP64 matrix cores: per axis for the lengths that have no
// compile-time FFT (fftc_dtt_kernels.h) and the short ones of small grids, and on small grids of
// whole (y, z) planes (k_plane).
//
// Every transform of Table 2, and the half-complex DFT of a periodic axis, is a fixed N x N matrix
// applied to the lines of the axis; k_dense_mats writes it once per binding in the order the
// lanes load it.  v_mfma_f64_16x16x4_f64, lane = r + 16 q (r < 16, q < 4):
//   A (16 x 4):  row r, column q     B (4 x 16):  row q, column r
//   D (16 x 16): row 4 e + q, column r (e < 4)
// so one layout of the matrix serves as A (y and z passes: columns are 16 consecutive x, the
// order of memory) and as B (x pass: columns are nodes along x, the order of memory).
//
// Why not an FFT: a line of length n costs 2 n^2 operations instead of about 5 n log2 n, but
// on the matrix cores, with one barrier instead of one per radix, no index arithmetic and no
// twiddles, and every length runs alike.  The runtime-length FFT took 18 to 21 us per pass on a
// 30x22x26 grid (33 blocks on 256 CUs, two or three radix stages with a barrier, divisions and
// twiddle loads each) whatever the work.  The products and sums are FP64 in the FP32 form too: the
// rounding that remains is that of the stored coefficient.
#include "fftc_internal.h"
#include "fftc_launch.h"
#include "fftc_common.h"

#include <math.h>
#include <algorithm>

namespace fftc {

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ d4 mfma64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Entry (out, in) of a transform matrix; angles are multiples of pi / 2n, reduced modulo 4n
__device__ double dense_entry(int type, int inv, int n, int out, int in) {
  auto C = [n](long long t) { return cospi((double)(t % (4ll * n)) / (2.0 * n)); };
  auto S = [n](long long t) { return sinpi((double)(t % (4ll * n)) / (2.0 * n)); };
  const long long o = out, i = in;
  switch (type) {
    case T_DCT1: {
      const double w = (in == 0 || in == n) ? 1.0 : 2.0;
      return w * C(2 * o * i) * (inv ? 1.0 / (2.0 * n) : 1.0);
    }
    case T_DST1:
      if (in == 0 || in == n || out == 0 || out == n) return 0.0;
      return 2.0 * S(2 * o * i) * (inv ? 1.0 / (2.0 * n) : 1.0);
    case T_DCT3:   // node n held at 0, coefficients 0..n-1
      if (out == n || in == n) return 0.0;
      return inv ? C(o * (2 * i + 1)) / n : (in == 0 ? 1.0 : 2.0) * C(i * (2 * o + 1));
    case T_DST3:   // node 0 held at 0
      if (inv) return (out == 0 || in == n) ? 0.0 : S(o * (2 * i + 1)) / n;
      return (in == 0 || out == n) ? 0.0 : (in == n ? 1.0 : 2.0) * S(i * (2 * o + 1));
    default: {     // half-complex DFT: real parts up to n / 2, then imaginary parts
      if (inv) {
        if (in == 0) return 1.0 / n;
        if (2 * in == n) return C(4 * o * i) / n;
        return 2.0 * (2 * in < n ? C(4 * o * i) : S(4 * o * i)) / n;
      }
      return 2 * out <= n ? C(4 * o * i) : S(4 * o * i);
    }
  }
}

// mat[tile][pair][lane][h] = entry (16 tile + lane mod 16, 8 pair + 4 h + lane / 16), zero outside: a
// lane loads its operands of two depth steps at once
__global__ __launch_bounds__(256) void k_dense_mats(int type, int n, int N, double* fwd, double* inv) {
  const int np = dense_depth(N) / 8, nt = (N + 15) / 16;
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= nt * np * 128) return;
  const int h = e & 1, lane = (e >> 1) & 63, kp = (e >> 7) % np, t = (e >> 7) / np;
  const int out = 16 * t + (lane & 15), in = 8 * kp + 4 * h + (lane >> 4);
  const bool ok = out < N && in < N;
  fwd[e] = ok ? dense_entry(type, 0, n, out, in) : 0.0;
  inv[e] = ok ? dense_entry(type, 1, n, out, in) : 0.0;
}

void launch_dense_mats(int type, int n, int N, double* fwd, double* inv, hipStream_t s) {
  const int total = (int)dense_mat_doubles(N);
  hipLaunchKernelGGL(k_dense_mats, dim3((total + 255) / 256), dim3(256), 0, s, type, n, N, fwd, inv);
}

// One pass over 16 LT lines per block.  XL: x lines (A = lines, B = matrix), else y or z lines (A =
// matrix, B = lines).  GREEN: forward, symbol, inverse on z lines, the coefficients staying in LDS
// in FP64.
// Bound by the chain load - LDS - products - store on small grids (4 to 5 us a pass) and by
// the FP64 matrix rate on large ones.
// TO: x lines stored as [x][z][y] (plane route), the roles of the operands exchanged so that 16 lanes
// hold consecutive y.
template <typename T, bool XL, bool GREEN, int LT, bool TO = false>
__global__ __launch_bounds__(256) void k_dense(DttArgs<T> a) {
  extern __shared__ __align__(16) unsigned char smem[];
  if (!a.force && a.st->done) return;
  constexpr int LB = 16 * LT;
  // blocks renumbered as in the compile-time passes: contiguous ranges per XCD
  unsigned bxi, byi, c;
  {
    const unsigned G = gridDim.x * gridDim.y * gridDim.z;
    const unsigned p = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const unsigned q = G / 8, r = G % 8, xcd = p % 8, slot = p / 8;
    const unsigned L = xcd * q + (xcd < r ? xcd : r) + slot;
    bxi = L % gridDim.x;
    byi = (L / gridDim.x) % gridDim.y;
    c = L / (gridDim.x * gridDim.y);
  }
  const int Nx = a.g.N[0], Ny = a.g.N[1], N = a.ap.N;
  const int nt = (N + 15) / 16, K = dense_depth(N), np = K / 8;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, r = lane & 15, q = lane >> 4;
  long long base;
  int nl, ls, es;   // lines of the block inside the grid, strides between lines and along them
  const int l0 = (int)bxi * LB;
  if (XL) {
    nl = Ny - l0;
    base = ((long long)(int)byi * Ny + l0) * Nx;
    ls = Nx;
    es = 1;
  } else if (a.axis == 1) {
    nl = Nx - l0;
    base = (long long)(int)byi * Nx * Ny + l0;
    ls = 1;
    es = Nx;
  } else {
    nl = Nx - l0;
    base = (long long)(int)byi * Nx + l0;
    ls = 1;
    es = Nx * Ny;
  }
  nl = min(nl, LB);
  base += (long long)c * a.g.Nn;
  // line l, node k in LDS: x lines at l KS + k, with KS = 4 mod 32 so that 16 lines' four
  // consecutive nodes fall on distinct banks; the others at k LB + l
  const int KS = dense_line_stride(N);
  T* sx = (T*)smem;
  auto at = [&](int l, int k) { return XL ? l * KS + k : k * LB + l; };
  // plane route: x lines stored to, or read from, [x][z][y]
  const bool tr_in = XL && a.plane && a.mode == PASS_INV;
  T* const trf = XL && a.plane ? plane_field(a) + (long long)c * a.g.Nn + (long long)byi * Ny + l0 : nullptr;
  const int tes = Ny * a.g.N[2];
  auto gather = [&](auto fetch, auto keep) {
    constexpr int U = 8;   // loads in flight per thread
    // element w of the block: x lines node by node, the others line by line
    const int total = LB * K;
    const float rk = 1.0f / (float)K;
    for (int w0 = tid; w0 < total; w0 += U * 256) {
      T v[U], s[U];
      unsigned off[U];
      int to[U];
      bool ok[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int w = w0 + u * 256;
        const bool by_l = !XL || tr_in;
        const int l = by_l ? w % LB : (int)(((float)w + 0.5f) * rk);   // w < 2^14: the quotient is exact
        const int k = by_l ? w / LB : w - l * K;
        ok[u] = w < total && l < nl && k < N;
        off[u] = tr_in ? (unsigned)(l + k * tes) : (unsigned)(l * ls) + (unsigned)(k * es);
        to[u] = w < total ? at(l, k) : -1;
        v[u] = s[u] = T(0);
        if (ok[u]) v[u] = fetch(off[u], s[u]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (ok[u]) keep(off[u], v[u], s[u]);
        if (to[u] >= 0) sx[to[u]] = v[u];
      }
    }
  };
  if (XL && a.src == SRC_ANDERSON) {
    const int acc_ok = a.st->accel_ok;
    double al[4] = {0, 0, 0, 0};
    if (acc_ok)
      for (int k = 0; k < 4; ++k) al[k] = a.st->alpha[k];
    const T* X = a.B.S[a.st->it & 3] + base;
    T* Sout = a.B.X + base;
    gather(
        [&](unsigned off, T&) -> T {
          if (!acc_ok) return X[off];
          double s = 0.0;
#pragma unroll
          for (int k = 0; k < 4; ++k) s += al[k] * (double)(a.B.S[(k + 1) & 3] + base)[off];
          return (T)s;
        },
        [&](unsigned off, T v, T) {
          if (acc_ok) Sout[off] = v;
        });
  } else if (XL && a.src == SRC_DELTA) {
    const T* pc = a.dp2[a.st->it & 1] + base;
    const int acc_ok = a.st->accel_ok;
    const T g0 = acc_ok ? (T)a.st->gamma[0] : T(0), g1 = acc_ok ? (T)a.st->gamma[1] : T(0),
            g2 = acc_ok ? (T)a.st->gamma[2] : T(0);
    const T *y0 = a.dY[0] + base, *y1 = a.dY[1] + base, *y2 = a.dY[2] + base;
    T* de = a.de + base;
    gather(
        [&](unsigned off, T& k) -> T {
          T v = pc[off];
          if (acc_ok) {
            k = g0 * y0[off] + g1 * y1[off] + g2 * y2[off];
            v = v - k;
          }
          return v;
        },
        [&](unsigned off, T, T k) {
          if (acc_ok) de[off] = k;
        });
  } else {
    const T* in = tr_in ? trf : a.in + base;
    gather([&](unsigned off, T&) -> T { return in[off]; }, [&](unsigned, T, T) {});
  }
  __syncthreads();
  // Output tile t of every line tile: acc = matrix tile x lines.  The matrix comes from the caches,
  // kU pairs of depth steps (1 KB each) requested while the previous ones are used: with four
  // single steps in flight and no look-ahead the loads' latency set the time (y pass at
  // 140^3 in FP64 142 us for 31 us of matrix work).
  constexpr int kU = 6;
  // Four partial sums per output, added in pairs: a quarter of the additions in a row halves the
  // rounding of the sum, to that of the FFT.
  auto product = [&](const double* mat, const auto* src, int t, d4 (&acc)[LT]) {
    d4 ps[LT][4];
#pragma unroll
    for (int u = 0; u < LT; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) ps[u][i] = d4{0.0, 0.0, 0.0, 0.0};
    const double2* mp = (const double2*)mat + (size_t)t * np * 64 + lane;
    double2 nxt[kU];
#pragma unroll
    for (int i = 0; i < kU; ++i) nxt[i] = i < np ? mp[(size_t)i * 64] : make_double2(0.0, 0.0);
    for (int kp = 0; kp < np; kp += kU) {
      double2 cur[kU];
#pragma unroll
      for (int i = 0; i < kU; ++i) {
        cur[i] = nxt[i];
        if (kp + kU + i < np) nxt[i] = mp[(size_t)(kp + kU + i) * 64];
      }
#pragma unroll
      for (int i = 0; i < kU; ++i) {
        if (kp + i >= np) break;
#pragma unroll
        for (int u = 0; u < LT; ++u) {
          const double v0 = (double)src[at(16 * u + r, 8 * (kp + i) + q)];
          const double v1 = (double)src[at(16 * u + r, 8 * (kp + i) + 4 + q)];
          d4 &p0 = ps[u][2 * (i & 1)], &p1 = ps[u][2 * (i & 1) + 1];
          p0 = XL && !TO ? mfma64(v0, cur[i].x, p0) : mfma64(cur[i].x, v0, p0);
          p1 = XL && !TO ? mfma64(v1, cur[i].y, p1) : mfma64(cur[i].y, v1, p1);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < LT; ++u) acc[u] = (ps[u][0] + ps[u][1]) + (ps[u][2] + ps[u][3]);
  };
  const double* mat = a.mat[c][a.mode == PASS_INV];
  if constexpr (GREEN) {
    double* sz = (double*)(smem + sizeof(T) * (size_t)K * LB);   // rows up to 16 nt
    const double* tab = a.cosT + (size_t)c * 6 * a.maxN;
    const double a0 = a.g.ac[c][0], a1 = a.g.ac[c][1], a2 = a.g.ac[c][2], hx = a.g.hex ? 0.0 : 1.0;
    const double sy = tab[2 * a.maxN + byi], qy = tab[3 * a.maxN + byi];
    for (int t = wv; t < nt; t += 4) {
      d4 acc[LT];
      product(mat, sx, t, acc);
#pragma unroll
      for (int u = 0; u < LT; ++u) {
        const int l = min(16 * u + r, nl - 1);
        const double sxv = tab[l0 + l], qxv = tab[a.maxN + l0 + l];
        // the factored Paux symbol (paux_symbol of the FFT passes)
        const double A = 4.0 * (a0 * sxv * qy + a1 * sy * qxv + hx * a2 * sxv * sy);
        const double B = 4.0 * (hx * a0 * qxv * sy + hx * a1 * qy * sxv + a2 * qxv * qy);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int m = 16 * t + 4 * e + q, mc = min(m, N - 1);
          const double M = tab[5 * a.maxN + mc] * A + tab[4 * a.maxN + mc] * B;
          if (m < K) sz[m * LB + 16 * u + r] = (m < N && M > a.thr[c]) ? acc[u][e] / M : 0.0;
        }
      }
    }
    __syncthreads();
    for (int t = wv; t < nt; t += 4) {
      d4 acc[LT];
      product(a.mat[c][1], sz, t, acc);
#pragma unroll
      for (int u = 0; u < LT; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int m = 16 * t + 4 * e + q, l = 16 * u + r;
          if (m < N && l < nl) a.buf[base + l * ls + (long long)m * es] = (T)acc[u][e];
        }
    }
  } else {
    const int upd = XL && a.dst == DST_UPDATE;
    const int sg = upd ? a.g.sing[c] : 0;
    const double s0 = sg ? a.st->sing[2 * c] : 0.0, s1 = sg ? a.st->sing[2 * c + 1] : 0.0;
    for (int t = wv; t < nt; t += 4) {
      d4 acc[LT];
      product(mat, sx, t, acc);
#pragma unroll
      for (int u = 0; u < LT; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          constexpr bool LR = XL && !TO;   // D rows are lines
          const int m = 16 * t + (LR ? r : 4 * e + q), l = 16 * u + (LR ? 4 * e + q : r);
          if (m >= N || l >= nl) continue;
          if (TO) {
            trf[l + (long long)m * tes] = (T)acc[u][e];
            continue;
          }
          const long long addr = base + (long long)l * ls + (long long)m * es;
          if (!upd) {
            a.buf[addr] = (T)acc[u][e];
            continue;
          }
          // residual form, last inverse pass: delta = K0^+ e - (I - Pi) u, u += delta
          double d = (double)(T)acc[u][e];
          if (sg) {
            const int parity = (m + l0 + l + (int)byi) & 1;
            d -= a.g.sing_scale[c] * (s0 + ((sg & 2) ? (parity ? -s1 : s1) : 0.0));
          }
          a.u64[addr] += d;
          a.delta[addr] = (T)d;
        }
    }
  }
}

template <typename T, bool XL, bool GREEN, int LT, bool TO = false>
static void launch_dense_lt(const DttArgs<T>& a, hipStream_t s) {
  const int Nx = a.g.N[0], Ny = a.g.N[1], Nz = a.g.N[2], N = a.ap.N, K = dense_depth(N);
  constexpr int LB = 16 * LT;
  const dim3 grid = XL ? dim3((Ny + LB - 1) / LB, Nz, 3) : dim3((Nx + LB - 1) / LB, a.axis == 1 ? Nz : Ny, 3);
  size_t sm = sizeof(T) * (XL ? (size_t)LB * dense_line_stride(N) : (size_t)K * LB);
  if (GREEN) sm += sizeof(double) * (size_t)K * LB;
  hipLaunchKernelGGL((k_dense<T, XL, GREEN, LT, TO>), grid, dim3(256), sm, s, a);
}

template <typename T>
void launch_dense(const DttArgs<T>& a, hipStream_t s) {
  // 32 lines per block (each matrix value loaded for two tiles of lines) once the grid fills the
  // chip several times over with 16
  const long long lines = a.axis == 0 ? (long long)a.g.N[1] * a.g.N[2]
                                      : (long long)a.g.N[0] * (a.axis == 1 ? a.g.N[2] : a.g.N[1]);
  // (and the lines, with the coefficients of the Green step, fit 64 KB of LDS)
  const int N = a.ap.N, green = a.mode == PASS_FWD_GREEN_INV;
  const size_t sm = a.axis == 0 ? sizeof(T) * 32 * (size_t)dense_line_stride(N)
                                : (sizeof(T) + (green ? 8 : 0)) * 32 * (size_t)dense_depth(N);
  const bool two = 3 * lines / 16 >= 2048 && sm <= 65536;
  if (a.axis == 0 && a.plane && a.mode == PASS_FWD) {
    if (two) launch_dense_lt<T, true, false, 2, true>(a, s);
    else launch_dense_lt<T, true, false, 1, true>(a, s);
  } else if (a.axis == 0) {
    if (two) launch_dense_lt<T, true, false, 2>(a, s);
    else launch_dense_lt<T, true, false, 1>(a, s);
  } else if (a.mode == PASS_FWD_GREEN_INV) {
    if (two) launch_dense_lt<T, false, true, 2>(a, s);
    else launch_dense_lt<T, false, true, 1>(a, s);
  } else {
    if (two) launch_dense_lt<T, false, false, 2>(a, s);
    else launch_dense_lt<T, false, false, 1>(a, s);
  }
}

// --------------------------------------------------------------------------
// y forward, z forward, symbol, z inverse and y inverse of one (y, z) plane per block
// --------------------------------------------------------------------------
// Block (x, component): the plane [z][y] in LDS as FP64, products from one buffer into the other, so
// that a transform costs one barrier and the three passes one launch and one read and write of
// the field.  A product unit is one matrix tile against LT tiles of lines.  The x passes lay the
// field out as [x][z][y] for it (their blocks hold 16 or more y of one z, so both orders are
// stored in whole sectors).
// Bound by the chain load - four products, each after a barrier - store: 5 us at 16^3 (y, z and y
// passes before: 12 us and two gaps), 6 us at 30x22x26 (10 and two gaps), 17 us at 48^3 in FP32 (18 and
// two gaps), where the matrix rate begins to tell.
template <typename T, int LT>
__global__ __launch_bounds__(512) void k_plane(DttArgs<T> a, PlaneMats pm) {
  extern __shared__ __align__(16) unsigned char smem[];
  if (!a.force && a.st->done) return;
  const int Ny = a.g.N[1], Nz = a.g.N[2], SY = plane_stride(Ny);
  const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, wv = tid >> 6, nw = nthr >> 6;
  const int r = lane & 15, q = lane >> 4;
  const int b = xcd_tile(blockIdx.x, gridDim.x);
  const int c = b / a.g.N[0], x = b - c * a.g.N[0];
  double* P0 = (double*)smem;
  double* P1 = P0 + (size_t)Nz * SY;
  T* f = plane_field(a) + (long long)c * a.g.Nn + (long long)x * Ny * Nz;
  const float ry = 1.0f / (float)Ny;
  const int total = Ny * Nz;
  constexpr int U = 4;
  for (int w0 = tid; w0 < total; w0 += U * nthr) {
    T v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = w0 + u * nthr < total ? f[w0 + u * nthr] : T(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int w = w0 + u * nthr;
      if (w >= total) continue;
      const int z = (int)(((float)w + 0.5f) * ry);   // w < 2^15: the quotient is exact
      P0[z * SY + (w - z * Ny)] = (double)v[u];
    }
  }
  // transform along an axis of length N and element stride sk, its M lines sl apart; put(m, l, value)
  auto pass = [&](const double* mat, const double* src, int N, int sk, int M, int sl, auto put) {
    const int nt = (N + 15) / 16, np = dense_depth(N) / 8, nu = (M + 16 * LT - 1) / (16 * LT);
    __syncthreads();
    for (int unit = wv; unit < nt * nu; unit += nw) {
      const int t = unit / nu, u0 = (unit - t * nu) * 16 * LT;
      const double2* mp = (const double2*)mat + (size_t)t * np * 64 + lane;
      const double* ln[LT];
#pragma unroll
      for (int u = 0; u < LT; ++u) ln[u] = src + min(u0 + 16 * u + r, M - 1) * sl;
      // four partial sums per output, as in k_dense
      d4 ps[LT][4];
#pragma unroll
      for (int u = 0; u < LT; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) ps[u][i] = d4{0.0, 0.0, 0.0, 0.0};
      constexpr int kU = 4;
      double2 nxt[kU];
#pragma unroll
      for (int i = 0; i < kU; ++i) nxt[i] = i < np ? mp[(size_t)i * 64] : make_double2(0.0, 0.0);
      for (int kp = 0; kp < np; kp += kU) {
        double2 cur[kU];
#pragma unroll
        for (int i = 0; i < kU; ++i) {
          cur[i] = nxt[i];
          if (kp + kU + i < np) nxt[i] = mp[(size_t)(kp + kU + i) * 64];
        }
#pragma unroll
        for (int i = 0; i < kU; ++i) {
          if (kp + i >= np) break;
          // (beyond the line the matrix is 0: any finite value of the line serves)
          const int k0 = min(8 * (kp + i) + q, N - 1) * sk, k1 = min(8 * (kp + i) + 4 + q, N - 1) * sk;
#pragma unroll
          for (int u = 0; u < LT; ++u) {
            ps[u][2 * (i & 1)] = mfma64(cur[i].x, ln[u][k0], ps[u][2 * (i & 1)]);
            ps[u][2 * (i & 1) + 1] = mfma64(cur[i].y, ln[u][k1], ps[u][2 * (i & 1) + 1]);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < LT; ++u) {
        const d4 acc = (ps[u][0] + ps[u][1]) + (ps[u][2] + ps[u][3]);
        const int l = u0 + 16 * u + r;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int m = 16 * t + 4 * e + q;
          if (m < N && l < M) put(m, l, acc[e]);
        }
      }
    }
  };
  pass(pm.y[c][0], P0, Ny, 1, Nz, SY, [&](int m, int l, double v) { P1[l * SY + m] = v; });
  const double* tab = a.cosT + (size_t)c * 6 * a.maxN;
  const double a0 = a.g.ac[c][0], a1 = a.g.ac[c][1], a2 = a.g.ac[c][2], hx = a.g.hex ? 0.0 : 1.0;
  const double sx = tab[x], qx = tab[a.maxN + x], thr = a.thr[c];
  pass(pm.z[c][0], P1, Nz, SY, Ny, 1, [&](int m, int l, double v) {
    // the factored Paux symbol (paux_symbol of the FFT passes)
    const double sy = tab[2 * a.maxN + l], qy = tab[3 * a.maxN + l];
    const double A = 4.0 * (a0 * sx * qy + a1 * sy * qx + hx * a2 * sx * sy);
    const double B = 4.0 * (hx * a0 * qx * sy + hx * a1 * qy * sx + a2 * qx * qy);
    const double S = tab[5 * a.maxN + m] * A + tab[4 * a.maxN + m] * B;
    P0[m * SY + l] = S > thr ? v / S : 0.0;
  });
  pass(pm.z[c][1], P0, Nz, SY, Ny, 1, [&](int m, int l, double v) { P1[m * SY + l] = v; });
  pass(pm.y[c][1], P1, Ny, 1, Nz, SY, [&](int m, int l, double v) { P0[l * SY + m] = v; });
  __syncthreads();
  for (int w = tid; w < total; w += nthr) {
    const int z = (int)(((float)w + 0.5f) * ry);
    f[w] = (T)P0[z * SY + (w - z * Ny)];
  }
}

template <typename T>
void launch_plane(const DttArgs<T>& a, const PlaneMats& pm, hipStream_t s) {
  const int Ny = a.g.N[1], Nz = a.g.N[2];
  const size_t sm = plane_lds(Ny, Nz);
  const int tiles = ((Ny + 15) / 16) * ((Nz + 15) / 16);
  const dim3 grid(3 * a.g.N[0]), block(tiles <= 4 ? 256 : 512);
  if (tiles <= 9) hipLaunchKernelGGL((k_plane<T, 1>), grid, block, sm, s, a, pm);
  else hipLaunchKernelGGL((k_plane<T, 2>), grid, block, sm, s, a, pm);
}
template void launch_plane<float>(const DttArgs<float>&, const PlaneMats&, hipStream_t);
template void launch_plane<double>(const DttArgs<double>&, const PlaneMats&, hipStream_t);

template void launch_dense<float>(const DttArgs<float>&, hipStream_t);
template void launch_dense<double>(const DttArgs<double>&, hipStream_t);

}  // namespace fftc
