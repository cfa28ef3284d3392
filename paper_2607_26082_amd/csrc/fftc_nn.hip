// Warm-start network: input channels, forward, backward and Adam on gfx950.
//
// The GEMM-shaped steps use v_mfma_f32_16x16x32_bf16 (BF16 operands, FP32 accumulation).
// Operand layout of that instruction for a 64-lane wave, with lane = r + 16 q (r < 16, q < 4) and
// element e of the vector:
//   A (16 x 32, row i, column k):  i = r, k = 8 q + e
//   B (32 x 16, row k, column j):  k = 8 q + e, j = r
//   D (16 x 16 FP32, row i, col j): i = 4 q + e, j = r
// The network runs in two kernels per block: k_line takes x lines of the grid through a layer
// (pointwise map, spectral term, epilogue) and forms its output's share of the next analysis
// and, backward, of the weight gradient; k_mid, between the layers, ends the analysis onto the
// cosine modes, mixes the modes and begins the synthesis.  k_last runs the last block together
// with the output layers (and, in training, the loss and the way back through them).  Partial
// sums are written per workgroup and added in a fixed order.
#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <type_traits>

#include "../../include/fftc_nn.h"
#include "fftc_nn_internal.h"

namespace nnk {

constexpr int kW = FFTC_NN_WIDTH;     // 32
constexpr int kH = FFTC_NN_HIDDEN;    // 64
constexpr int kCh = FFTC_NN_CHANNELS; // 16
constexpr int kCin = 12;
constexpr int kCout = 3;
constexpr int kMaxN = 257;
constexpr int kMaxM = 6;
constexpr int kLines = 16;                  // most x lines of a workgroup
constexpr int kHiddenGrid = 256;            // workgroups of the hidden layer's weight gradient
constexpr int kSqGrid = 512;                // blocks of the loss scale

typedef short s8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mfma32(s8 a, s8 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b), c, 0, 0, 0);
}

__device__ __host__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u;
  memcpy(&u, &f, 4);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// Upper tail of the normal law, Q(a) = erfc(a / sqrt 2) / 2 for a >= 0, as exp(-a^2 / 2) t p(t) with
// t = 1 / (1 + 0.3 a): p fitted for the smallest relative error on a <= 13.5 (1.3e-7).  E
// returns the exponential.  GELU(z) = max(z, 0) - |z| Q(|z|) keeps its relative accuracy for
// negative z (1.5e-6 down to z = -5, where 1 + erf cancels to 5e-2) at the absolute error of
// the erf form (2.4e-7 against 4.5e-7), in half its instructions and with no branch; its
// derivative shares the exponential.
__device__ __forceinline__ float normal_tail(float a, float& E) {
  const float t = __builtin_amdgcn_rcpf(1.0f + 0.3f * a);
  float s = 0.035931916f;
  s = s * t - 0.15827669f;
  s = s * t + 0.20820768f;
  s = s * t - 0.055394738f;
  s = s * t + 0.12946963f;
  s = s * t + 0.099637378f;
  s = s * t + 0.12079837f;
  s = s * t + 0.11962639f;
  E = __builtin_amdgcn_exp2f(-0.72134752f * (a * a));
  return s * t * E;
}

// beyond |z| = 16 the tail is 0 in FP32; NaN stays NaN (the first select passes it on)
__device__ __forceinline__ float gelu(float z) {
  const float a = fminf(fabsf(z), 16.0f);
  float E;
  const float q = normal_tail(a, E);
  return (z <= 0.0f ? 0.0f : z) - a * q;
}

__device__ __forceinline__ float gelu_grad(float z) {
  const float a = fminf(fabsf(z), 16.0f);
  float E;
  const float q = normal_tail(a, E);
  return (z > 0.0f ? 1.0f - q : q) + z * (0.39894228040143268f * E);
}

// Node grid and its split into workgroups: lines are the x lines (y, z) of the grid; a
// workgroup takes up to kLines consecutive lines of one z plane ("chunk"), its four waves
// taking lines in turn, 32 nodes of a line at a time.
struct Dims {
  int N[3];
  int Nn;
  int m, M3;
  int pairs;           // 32-node pieces of an x line (the last one padded)
  int chunks, lines;   // chunks per z plane, lines per chunk
};

// --------------------------------------------------------------------------
// layers on x lines
// --------------------------------------------------------------------------
// Activations [Nn][32] are stored with channel c at place 2 (c mod 16) + c / 16, so that the
// two channels r and r + 16 that a lane holds after the MFMAs are one dword, and a row of 16
// lanes writes whole 64-byte nodes; [Nn][64] fields likewise with c at 4 (c mod 16) + c / 16.
//
// The spectral term of a node (x, y, z) is separable: with G[z][ky][kx][o] = sum_kz cz P (k_mid)
// and, per line, H[kx][o] = sum_ky cy(y, ky) G, it is sum_kx cx(x, kx) H[kx][o], a contraction
// over m <= 6 values.  It rides in one MFMA of depth 32 per output tile: cos and H are split
// into BF16 high and low parts (c ~ ch + cl, H ~ Hh + Hl), and the 3 m products ch Hh + ch Hl +
// cl Hh take 18 of the 32 slots (error 2^-17 of the product; the basis values and
// coefficients rounded to BF16 before had 2^-9).  The x part of the analysis of the layer's own
// output, sum_x cx(x, kx) out[x][c], is formed from the output registers (D rows are nodes,
// which are the depth of the next MFMA): cos in three BF16 parts (24 bits, as the FP32 table),
// the activation exact.  The y part follows from LDS at the end of the chunk, and one row of
// m^2 x 32 partial sums per workgroup leaves it for k_mid.  In the backward pass the weight
// gradient sum_node dz[o] x[c] is formed from the same registers.
struct LineArgs {
  Dims d;
  const uint16_t* in;    // IN_FEAT [Nn][16], else [Nn][32]
  const s8* w;           // weight operands [tile][64 lanes]
  const float* bias;     // [32] or null
  const float* G;        // [Nz][m^2][32] (SYN)
  const float* tab;      // cosine tables x | y | z, each [N][m]
  const uint16_t* syn;   // [32 pairs][32]: cos operand of the spectral term per node of a line
  const uint16_t* ana;   // [pairs][3][m][32]: cos operand of the analysis
  const uint16_t* zaux;  // [Nn][32] pre-activation (EPI_DGELU)
  const uint16_t* aux;   // AUX_X [Nn][32], AUX_FEAT [Nn][16]: input of the layer whose dz this forms
  uint16_t* out;         // [Nn][32]
  uint16_t* zout;        // [Nn][32] (EPI_GELU_Z)
  float* a2;             // [workgroups][m^2][32] (ANA)
  float* dw;             // [workgroups][32 x (32 or 12) + 32]: weight and bias gradient
};

enum { IN_FEAT = 0, IN_X = 1, IN_D = 2 };   // IN_D: no layer, the stored field itself
enum { EPI_NONE = 0, EPI_GELU = 1, EPI_GELU_Z = 2, EPI_DGELU = 3 };
enum { AUX_NONE = 0, AUX_X = 1, AUX_FEAT = 2 };

// LDS of k_line in bytes: operand tables, G, the lines' H / analysis values, or (at the end)
// the four waves' weight gradients
inline size_t line_smem(const Dims& d, bool syn, bool ana, bool dw) {
  size_t s = 4 * (size_t)d.lines * d.m * kW;
  if (syn) s += 64 * (size_t)(32 * d.pairs) + 4 * (size_t)d.m * d.m * kW;
  if (ana) s += 64 * (size_t)(d.pairs * 3 * d.m);
  if (dw) s = std::max(s, 4 * (size_t)4 * (kW * kW + kW));
  return s;
}

typedef __bf16 bf2 __attribute__((ext_vector_type(2)));

// two values rounded to nearest even in one instruction (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf(float a, float b) {
  return __builtin_bit_cast(uint32_t, bf2{(__bf16)a, (__bf16)b});
}

__device__ __forceinline__ s8 as_s8(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  union {
    uint32_t u[4];
    s8 v;
  } r;
  r.u[0] = a;
  r.u[1] = b;
  r.u[2] = c;
  r.u[3] = d;
  return r.v;
}

// the eight node values (rows 4 q + e of tile 0, then of tile 1) of one channel as an operand
__device__ __forceinline__ s8 node_vec(const uint32_t (&P)[2][4], int t) {
  const uint32_t sel = t ? 0x07060302u : 0x05040100u;
  return as_s8(__builtin_amdgcn_perm(P[0][1], P[0][0], sel), __builtin_amdgcn_perm(P[0][3], P[0][2], sel),
               __builtin_amdgcn_perm(P[1][1], P[1][0], sel), __builtin_amdgcn_perm(P[1][3], P[1][2], sel));
}

// y cosines of a chunk's lines, 8 floats a line (zero past m)
__device__ __forceinline__ void line_cy(const Dims& d, const float* tab, float* sCy, int y0, int nl, int tid) {
  const float* cy = tab + (size_t)(d.N[0] + y0) * d.m;
  if (tid < 8 * nl) sCy[tid] = (tid & 7) < d.m ? cy[(tid >> 3) * d.m + (tid & 7)] : 0.0f;
}

// H[kx][o] of a chunk's lines as (high, low) BF16 pairs.  From LDS only, loops unrolled: with
// the cosines read from memory in a rolled loop this phase took most of a workgroup's time.
__device__ __forceinline__ void line_h(int m, const float* sCy, const float* sG, uint32_t* sH, int nl, int tid) {
  const int row = m * kW;
  for (int i = tid; i < nl * row; i += 256) {
    const int l = i / row, kc = i - l * row;
    float s = 0.0f;
#pragma unroll
    for (int ky = 0; ky < kMaxM; ++ky)
      if (ky < m) s += sCy[8 * l + ky] * sG[ky * row + kc];
    sH[i] = pack_bf(s, s - (float)(__bf16)s);
  }
}

// operand of the spectral term for output column o: slots 8 q + s of H (see above)
__device__ __forceinline__ s8 h_operand(const uint32_t* sHl, int m, int q, int o) {
  s8 v;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int slot = 8 * q + s;
    const int part = slot < m ? 0 : slot < 2 * m ? 1 : 2;
    const int kx = slot - part * m;
    uint32_t h = 0u;
    if (slot < 3 * m) h = sHl[kx * kW + o];
    v[s] = (short)(part == 1 ? h >> 16 : h & 0xffffu);
  }
  return v;
}

// Bound by VALU issue: per 32 nodes about 550 instructions a wave, most of them the GELU's 16
// values per lane, at half the SIMDs' rate (the rest is the start of a workgroup and the last
// tile of a line, which holds one node on 2^k + 1 grids).  Before, one kernel formed the m^3
// basis values of every node on the fly and three more took the analysis: a block of the
// network took 111 us at 65^3 and 564 us at 129^3 in five launches; k_line and k_mid take
// 33 us and about 118 us, 0.28 GB of it moved at 2.7 TB/s.
template <int IN, bool SYN, int EPI, bool OUT, bool ANA, int AUX>
__global__ __launch_bounds__(256) void k_line(LineArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ float sCy[8 * kLines];
  const Dims& d = a.d;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, r = lane & 15, q = lane >> 4;
  const int m = d.m, Nx = d.N[0], Ny = d.N[1];
  const int z = blockIdx.x / d.chunks, y0 = (blockIdx.x % d.chunks) * d.lines;
  const int nl = min(d.lines, Ny - y0);
  uint32_t* sH = (uint32_t*)smem;
  unsigned char* sp = smem + 4 * d.lines * m * kW;
  const uint16_t* sSyn = (const uint16_t*)sp;
  if (SYN) sp += 64 * 32 * d.pairs;
  const float* sG = (const float*)sp;
  if (SYN) sp += 4 * m * m * kW;
  const uint16_t* sAna = (const uint16_t*)sp;
  if (SYN || ANA) line_cy(d, a.tab, sCy, y0, nl, tid);
  if (SYN) {
    const uint4* g = (const uint4*)a.syn;
    for (int i = tid; i < 4 * 32 * d.pairs; i += 256) ((uint4*)sSyn)[i] = g[i];
    const float* Gz = a.G + (size_t)z * m * m * kW;
    for (int i = tid; i < m * m * kW; i += 256) ((float*)sG)[i] = Gz[i];
  }
  if (ANA) {
    const uint4* g = (const uint4*)a.ana;
    for (int i = tid; i < 4 * d.pairs * 3 * m; i += 256) ((uint4*)sAna)[i] = g[i];
  }
  s8 bw[2];
  float bias[2] = {0.0f, 0.0f};
  if constexpr (IN != IN_D) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      bw[t] = a.w[t * 64 + lane];
      if (a.bias) bias[t] = a.bias[16 * t + r];
    }
  }
  __syncthreads();
  if (SYN) {
    line_h(m, sCy, sG, sH, nl, tid);
    __syncthreads();
  }
  constexpr int DT = AUX == AUX_X ? 2 : 1;   // column tiles of the weight gradient
  f4 dw[2][DT], db[2];
  if constexpr (AUX != AUX_NONE) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      db[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < DT; ++u) dw[t][u] = f4{0.f, 0.f, 0.f, 0.f};
    }
  }
  const s8 ones = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
  const s8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
  const uint32_t* in32 = (const uint32_t*)a.in;
  const uint32_t* z32 = (const uint32_t*)a.zaux;
  const uint32_t* aux32 = (const uint32_t*)a.aux;
  // input of a piece, fetched one piece ahead (the next of the line, or the next line's first)
  s8 xn[2] = {zero8, zero8};
  auto fetch = [&](int l, int p) {
    if constexpr (IN == IN_D) return;
    const int base = (z * Ny + y0 + l) * Nx;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int x = 32 * p + 16 * h + r;
      xn[h] = zero8;
      if (x >= Nx) continue;
      if constexpr (IN == IN_FEAT) {
        if (q < 2) xn[h] = *(const s8*)(a.in + (size_t)(base + x) * kCh + 8 * q);
      } else {
        xn[h] = *(const s8*)(a.in + (size_t)(base + x) * kW + 8 * q);
      }
    }
  };
  if (wv < nl) fetch(wv, 0);
  for (int l = wv; l < nl; l += 4) {
    const int base = (z * Ny + y0 + l) * Nx;   // first node of the line
    s8 bh[2];
    if (SYN) {
      bh[0] = h_operand(sH + l * m * kW, m, q, r);
      bh[1] = h_operand(sH + l * m * kW, m, q, r + 16);
    }
    f4 an[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
    for (int p = 0; p < d.pairs; ++p) {
      uint32_t P[2][4], Z[2][4], X[2][4];
      s8 ax[2] = {xn[0], xn[1]};
      // all loads of the piece first
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int x = 32 * p + 16 * h;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int xe = x + 4 * q + e;
          const bool ok = xe < Nx;
          const size_t nd = (size_t)(base + xe);
          P[h][e] = 0u;
          if constexpr (IN == IN_D) P[h][e] = ok ? in32[nd * 16 + r] : 0u;
          if constexpr (EPI == EPI_DGELU) Z[h][e] = ok ? z32[nd * 16 + r] : 0u;
          if constexpr (AUX == AUX_X) X[h][e] = ok ? aux32[nd * 16 + r] : 0u;
          if constexpr (AUX == AUX_FEAT) X[h][e] = ok ? (uint32_t)a.aux[nd * kCh + r] : 0u;
        }
      }
      if (p + 1 < d.pairs) fetch(l, p + 1);
      else if (l + 4 < nl) fetch(l + 4, 0);
      if constexpr (IN != IN_D) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int x = 32 * p + 16 * h;
          if (x >= Nx) break;   // uniform: the line ends before this half
          f4 acc[2];
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            acc[t] = f4{bias[t], bias[t], bias[t], bias[t]};
            acc[t] = mfma32(ax[h], bw[t], acc[t]);
          }
          if (SYN) {
            const s8 cs = *(const s8*)(sSyn + (x + r) * 32 + 8 * q);
#pragma unroll
            for (int t = 0; t < 2; ++t) acc[t] = mfma32(cs, bh[t], acc[t]);
          }
          uint32_t Zo[4];
          auto finish = [&](auto first) {
#pragma unroll
            for (int e = 0; e < decltype(first)::value; ++e) {
              float v0 = acc[0][e], v1 = acc[1][e];
              if constexpr (EPI == EPI_GELU_Z) Zo[e] = pack_bf(v0, v1);
              if constexpr (EPI == EPI_GELU || EPI == EPI_GELU_Z) {
                v0 = gelu(v0);
                v1 = gelu(v1);
              } else if constexpr (EPI == EPI_DGELU) {
                v0 *= gelu_grad(bf2f((uint16_t)Z[h][e]));
                v1 *= gelu_grad(bf2f((uint16_t)(Z[h][e] >> 16)));
              }
              P[h][e] = pack_bf(v0, v1);
            }
          };
          // a last tile of one node (a line of 2^k + 1) has it in the first element: the other three
          // values a lane would take through the GELU are left out
          if (x + 1 == Nx) finish(std::integral_constant<int, 1>{});
          else finish(std::integral_constant<int, 4>{});
          // stores: unguarded on whole tiles (the guard is uniform there)
          const size_t nd = (size_t)(base + x + 4 * q);
          if (x + 16 <= Nx) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              if constexpr (EPI == EPI_GELU_Z) ((uint32_t*)a.zout)[(nd + e) * 16 + r] = Zo[e];
              if (OUT) ((uint32_t*)a.out)[(nd + e) * 16 + r] = P[h][e];
            }
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              if (x + 4 * q + e < Nx) {
                if constexpr (EPI == EPI_GELU_Z) ((uint32_t*)a.zout)[(nd + e) * 16 + r] = Zo[e];
                if (OUT) ((uint32_t*)a.out)[(nd + e) * 16 + r] = P[h][e];
              } else {
                P[h][e] = 0u;
              }
            }
          }
        }
      }
      if constexpr (ANA || AUX != AUX_NONE) {
        const s8 v0 = node_vec(P, 0), v1 = node_vec(P, 1);
        if constexpr (ANA) {
#pragma unroll
          for (int s = 0; s < 3; ++s) {
            s8 c = zero8;
            if (r < m) c = *(const s8*)(sAna + ((p * 3 + s) * m + r) * 32 + 8 * q);
            an[0] = mfma32(c, v0, an[0]);
            an[1] = mfma32(c, v1, an[1]);
          }
        }
        if constexpr (AUX != AUX_NONE) {
#pragma unroll
          for (int u = 0; u < DT; ++u) {
            const s8 xv = node_vec(X, u);
            dw[0][u] = mfma32(v0, xv, dw[0][u]);
            dw[1][u] = mfma32(v1, xv, dw[1][u]);
          }
          db[0] = mfma32(v0, ones, db[0]);
          db[1] = mfma32(v1, ones, db[1]);
        }
      }
    }
    if (ANA) {
      // the line's H is spent: its place takes the line's x analysis
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (4 * q + e < m) ((float*)sH)[(l * m + 4 * q + e) * kW + 16 * t + r] = an[t][e];
    }
  }
  if (ANA) {
    __syncthreads();
    const int row = m * kW;
    if (tid < row) {
      float s[kMaxM];
#pragma unroll
      for (int ky = 0; ky < kMaxM; ++ky) s[ky] = 0.0f;
      for (int l = 0; l < nl; ++l) {
        const float v = ((const float*)sH)[l * row + tid];
#pragma unroll
        for (int ky = 0; ky < kMaxM; ++ky) s[ky] += sCy[8 * l + ky] * v;
      }
#pragma unroll
      for (int ky = 0; ky < kMaxM; ++ky)
        if (ky < m) a.a2[((size_t)blockIdx.x * m + ky) * row + tid] = s[ky];
    }
  }
  if constexpr (AUX != AUX_NONE) {
    // the waves' gradients, added in order: [32][C] then the 32 bias entries
    constexpr int C = AUX == AUX_X ? kW : kCin, TOT = kW * C + kW;
    float* sW = (float*)smem;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int o = 16 * t + 4 * q + e;
#pragma unroll
        for (int u = 0; u < DT; ++u)
          if (16 * u + r < C) sW[wv * TOT + o * C + 16 * u + r] = dw[t][u][e];
        if (r == 0) sW[wv * TOT + kW * C + o] = db[t][e];
      }
    __syncthreads();
    for (int i = tid; i < TOT; i += 256)
      a.dw[(size_t)blockIdx.x * TOT + i] = (sW[i] + sW[TOT + i]) + (sW[2 * TOT + i] + sW[3 * TOT + i]);
  }
}

// --------------------------------------------------------------------------
// between the layers: end of the analysis, mode mixing, z part of the synthesis
// --------------------------------------------------------------------------
// One block per (ky, kx): xh[k][c] = scale sum over z and the chunks' rows of cz(z, kz) a2; then
//   forward:  P[kz][o] = sum_c Ws[k][o][c] xh[k][c], xh kept for the backward pass;
//   backward: (xh is dyh) dWs[k][o][c] = dyh[k][o] xh_fwd[k][c],
//             P[kz][c] = (1 / Nn) sum_o Ws[k][o][c] dyh[k][o];
// P rounded to BF16 (the mode coefficients' type), and G[z][ky][kx][o] = sum_kz cz(z, kz) P[kz][o],
// all else in FP32.  36 blocks of 1024 threads: a
// chain of a few dependent loads each, which is what bounds it (five kernels before).
struct MidArgs {
  Dims d;
  int rows;            // workgroups of the line kernel
  unsigned zmul;       // row / chunks = umulhi(row, zmul) (chunks > 1)
  const float* a2;     // [rows][m^2][32]
  const float* tab;
  float scale;
  const float* Ws;     // [m^3][32][32]
  float* xh;           // forward: out [m^3][32]; backward: the forward's values
  float* dWs;          // backward
  float inv_nn;
  float* G;            // [Nz][m^2][32]
};

template <bool BWD>
__global__ __launch_bounds__(1024) void k_mid(MidArgs a) {
  __shared__ __align__(16) float sCz[8 * kMaxN];
  __shared__ float sR[32 * kMaxM * kW];
  __shared__ float sX[kMaxM * kW];
  __shared__ float sP[kMaxM * kW];
  const Dims& d = a.d;
  const int m = d.m, Nz = d.N[2], tid = threadIdx.x, c = tid & 31, g = tid >> 5;
  const int b = blockIdx.x, mm = m * m;
  const float* cz = a.tab + (d.N[0] + d.N[1]) * m;
  // the mixing weights and the first rows are requested before anything waits
  float w[8];
  const int part = BWD ? (tid >> 5) & 3 : tid & 3, oc = BWD ? c : (tid >> 2) & 31, kz = tid >> 7;
  if (kz < m) {
    const float* ws = a.Ws + (size_t)(kz * mm + b) * kW * kW;
#pragma unroll
    for (int j = 0; j < 8; ++j) w[j] = BWD ? ws[(8 * part + j) * kW + oc] : ws[oc * kW + 8 * part + j];
  }
  constexpr int U = 12;   // rows in flight per thread
  const float* src = a.a2 + (size_t)b * kW + c;
  const size_t step = (size_t)mm * kW;
  float v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) v[u] = g + 32 * u < a.rows ? src[(size_t)(g + 32 * u) * step] : 0.0f;
  for (int i = tid; i < 8 * Nz; i += 1024) sCz[i] = (i & 7) < m ? cz[(i >> 3) * m + (i & 7)] : 0.0f;
  __syncthreads();
  float s[kMaxM];
#pragma unroll
  for (int k = 0; k < kMaxM; ++k) s[k] = 0.0f;
  for (int r0 = g;;) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int row = r0 + 32 * u;
      if (row < a.rows) {
        const int z = d.chunks > 1 ? (int)__umulhi((unsigned)row, a.zmul) : row;
#pragma unroll
        for (int k = 0; k < kMaxM; ++k)
          s[k] += sCz[8 * z + k] * v[u];
      }
    }
    r0 += 32 * U;
    if (r0 >= a.rows) break;
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = r0 + 32 * u < a.rows ? src[(size_t)(r0 + 32 * u) * step] : 0.0f;
  }
#pragma unroll
  for (int k = 0; k < kMaxM; ++k)
    if (k < m) sR[(g * m + k) * kW + c] = s[k];
  __syncthreads();
  // the 32 groups in two steps: four eighths per value, then their sum
  const int vals = m * kW;
  float t4 = 0.0f;
  if (tid < 4 * vals)
#pragma unroll
    for (int j = 0; j < 8; ++j) t4 += sR[(tid / vals * 8 + j) * vals + tid % vals];
  __syncthreads();
  if (tid < 4 * vals) sR[tid] = t4;
  __syncthreads();
  if (tid < vals) {
    const float t = a.scale * ((sR[tid] + sR[vals + tid]) + (sR[2 * vals + tid] + sR[3 * vals + tid]));
    sX[tid] = t;
    if (!BWD) a.xh[((tid / kW) * mm + b) * kW + tid % kW] = t;
  }
  __syncthreads();
  if constexpr (!BWD) {
    if (kz < m) {
      float t = 0.0f;
#pragma unroll
      for (int j = 0; j < 8; ++j) t += w[j] * sX[kz * kW + 8 * part + j];
      t += __shfl_xor(t, 1, 64);
      t += __shfl_xor(t, 2, 64);
      if (part == 0) sP[kz * kW + oc] = (float)(__bf16)t;
    }
  } else {
    for (int i = tid; i < m * kW * kW; i += 1024) {
      const int kq = i / (kW * kW), o = (i / kW) % kW, k = kq * mm + b;
      a.dWs[(size_t)k * kW * kW + i % (kW * kW)] = sX[kq * kW + o] * a.xh[k * kW + i % kW];
    }
    if (kz < m) {
      float t = 0.0f;
#pragma unroll
      for (int j = 0; j < 8; ++j) t += w[j] * sX[kz * kW + 8 * part + j];
      sR[tid] = t;
    }
    __syncthreads();
    if (tid < vals) {
      const int k = tid / kW;
      const float t = sR[k * 128 + c] + sR[k * 128 + 32 + c] + (sR[k * 128 + 64 + c] + sR[k * 128 + 96 + c]);
      sP[tid] = (float)(__bf16)(a.inv_nn * t);
    }
  }
  __syncthreads();
  for (int i = tid; i < Nz * kW; i += 1024) {
    const int z = i / kW, o = i % kW;
    float t = 0.0f;
#pragma unroll
    for (int k = 0; k < kMaxM; ++k)
      if (k < m) t += sCz[8 * z + k] * sP[k * kW + o];
    a.G[((size_t)z * mm + b) * kW + o] = t;
  }
}

// --------------------------------------------------------------------------
// last block and output layers
// --------------------------------------------------------------------------
// Here the MFMA rows are channels and the columns nodes, so that each layer's output registers
// are the next layer's operand (the depth order of two chained MFMAs is free as long as both
// operands agree): last spectral block (BLK; else the stored x itself), hidden layer, output
// layer, and in training the loss and the gradients back to the block's pre-activation (or to
// x when there is no block) without leaving the registers.  What the hidden layer's weight
// gradient needs (x, dhpre) is stored; the output layer's is accumulated per lane in FP32.
// Bound by VALU issue (24 GELUs per lane and 16 nodes, in training their derivatives too):
// 34 us at 65^3 in inference (hidden layer and output kernels plus the block: 87 us before), 84 us
// in training (about 290 us in nine launches before).
struct LastArgs {
  Dims d;
  const uint16_t* in;    // [Nn][32]
  const s8* w;           // block's operands [tile][64 lanes]
  const s8* wo;          // the output layers' operands (OP_P ..)
  const float* bias;     // [32]
  const float* G;
  const float* tab;
  const uint16_t* syn;
  const float* bp1;      // [64]
  const float* w2;       // Wp2[3][64] then bp2[3]
  float* y;              // [Nn][3] or null
  double* u0;            // [3][Nn] or null
  const double* base;    // [3][Nn] or null: u0 = base + s_u y
  double s_u;
  // training
  const float* target;   // [3][Nn]
  const float* tinv;     // 1 / (sum t^2 + sum b^2)
  uint16_t* xout;        // [Nn][32] (BLK)
  uint16_t* dhpre;       // [Nn][64]
  uint16_t* dz;          // [Nn][32]
  float* dw2;            // [workgroups][3 x 64 + 3]
  double* lpart;         // [workgroups]
};

// Operands of k_last in LDS, 1 KB each (16 bytes per lane), read in every tile: kept in registers
// they would leave one wave per SIMD.  High and low parts of the weights as in k_line; the
// output layer's FP32 weights in three parts (24 bits).
enum { OP_W = 0, OP_P = 4, OP_W2 = 12, OP_T = 14, OP_W2T = 22, OP_N = 26 };
constexpr int kOpLift = 2, kOpBlock = 4;   // operands of the lift and of a block
// (up to 60.5 KB, with the static arrays 64.5 KB: 257 nodes a line, 16 lines, training)
inline size_t last_smem(const Dims& d, bool blk, bool train) {
  return 1024 * (size_t)(train ? OP_N : OP_T) + (blk ? line_smem(d, true, false, false) : 0);
}

template <bool BLK, bool TRAIN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(TRAIN ? 2 : 4)))
void k_last(LastArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ float sB[kW + kH + kCout], sCy[8 * kLines];
  __shared__ float sD[TRAIN ? 4 * (kCout * kH + kCout) : 1];
  __shared__ double sL[4];
  const Dims& d = a.d;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, r = lane & 15, q = lane >> 4;
  const int m = d.m, Nx = d.N[0], Ny = d.N[1];
  const int z = blockIdx.x / d.chunks, y0 = (blockIdx.x % d.chunks) * d.lines;
  const int nl = min(d.lines, Ny - y0);
  s8* sOp = (s8*)smem;
  unsigned char* sp = smem + 1024 * (TRAIN ? OP_N : OP_T);
  uint32_t* sH = (uint32_t*)sp;
  uint16_t* sSyn = (uint16_t*)(sp + 4 * d.lines * m * kW);
  float* sG = (float*)(sp + 4 * d.lines * m * kW + 64 * 32 * d.pairs);
  if (tid < kH) sB[kW + tid] = a.bp1[tid];
  if (tid < kCout) sB[kW + kH + tid] = a.w2[kCout * kH + tid];
  if (BLK) {
    if (tid < kW) sB[tid] = a.bias[tid];
    line_cy(d, a.tab, sCy, y0, nl, tid);
    const uint4* g = (const uint4*)a.syn;
    for (int i = tid; i < 4 * 32 * d.pairs; i += 256) ((uint4*)sSyn)[i] = g[i];
    const float* Gz = a.G + (size_t)z * m * m * kW;
    for (int i = tid; i < m * m * kW; i += 256) sG[i] = Gz[i];
  }
  for (int i = tid; i < 64 * (TRAIN ? OP_N : OP_T); i += 256)
    if (BLK || i >= 64 * OP_P) sOp[i] = i < 64 * OP_P ? a.w[i] : a.wo[i - 64 * OP_P];
  __syncthreads();
  if (BLK) {
    line_h(m, sCy, sG, sH, nl, tid);
    __syncthreads();
  }
  const s8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
  const float ti = TRAIN ? *a.tinv : 0.0f;
  double loss = 0.0;
  float g2[TRAIN ? kCout : 1][TRAIN ? 16 : 1], gb[kCout] = {0.f, 0.f, 0.f};
  if (TRAIN)
#pragma unroll
    for (int c = 0; c < kCout; ++c)
#pragma unroll
      for (int j = 0; j < 16; ++j) g2[c][j] = 0.0f;
  for (int l = wv; l < nl; l += 4) {
    const int base = (z * Ny + y0 + l) * Nx;
    s8 ah[2];
    if (BLK) {
      ah[0] = h_operand(sH + l * m * kW, m, q, r);
      ah[1] = h_operand(sH + l * m * kW, m, q, r + 16);
    }
    s8 xn = zero8;
    if (r < Nx) xn = *(const s8*)(a.in + (size_t)(base + r) * kW + 8 * q);
    for (int x0 = 0; x0 < Nx; x0 += 16) {
      const bool ok = x0 + r < Nx;
      const size_t nd = (size_t)(base + x0 + r);
      // opaque to the compiler, so that the operand reads stay in the loop
      int oi = lane;
      asm volatile("" : "+v"(oi));
      const s8* op = sOp + oi;
      const float* sb = sB + (oi - lane);
      s8 xv = xn;   // fetched one tile ahead
      xn = zero8;
      if (x0 + 16 + r < Nx) xn = *(const s8*)(a.in + (nd + 16) * kW + 8 * q);
      float tg[kCout] = {0.f, 0.f, 0.f};
      if (TRAIN && ok)
#pragma unroll
        for (int c = 0; c < kCout; ++c) tg[c] = a.target[(size_t)c * d.Nn + nd];
      f4 zv[2];
      if (BLK) {
        const s8 cs = *(const s8*)(sSyn + (x0 + r) * 32 + 8 * q);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          f4 v = *(const f4*)(sb + 16 * t + 4 * q);
          v = mfma32(op[64 * (OP_W + t)], xv, v);
          zv[t] = mfma32(ah[t], cs, v);
        }
        uint32_t P[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) P[e] = pack_bf(gelu(zv[0][e]), gelu(zv[1][e]));
        xv = as_s8(P[0], P[1], P[2], P[3]);
        if (TRAIN && ok) *(s8*)(a.xout + nd * kW + 8 * q) = xv;
      }
      f4 hp[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        hp[t] = *(const f4*)(sb + kW + 16 * t + 4 * q);
        hp[t] = mfma32(op[64 * (OP_P + t)], xv, hp[t]);
      }
      uint32_t H[8];   // h rounded to BF16, at places 16 q + 4 e + t
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        H[2 * e] = pack_bf(gelu(hp[0][e]), gelu(hp[1][e]));
        H[2 * e + 1] = pack_bf(gelu(hp[2][e]), gelu(hp[3][e]));
      }
      // output layer: rows 4 c + part, so that lane group q < 3 holds the parts of y_q
      f4 yp = f4{0.f, 0.f, 0.f, 0.f};
      yp = mfma32(op[64 * OP_W2], as_s8(H[0], H[1], H[2], H[3]), yp);
      yp = mfma32(op[64 * (OP_W2 + 1)], as_s8(H[4], H[5], H[6], H[7]), yp);
      const float yq = (yp[2] + yp[1]) + yp[0] + sb[kW + kH + (q < kCout ? q : 0)];
      if constexpr (!TRAIN) {
        if (ok && q < kCout) {
          if (a.y) a.y[nd * kCout + q] = yq;
          if (a.u0)
            a.u0[(size_t)q * d.Nn + nd] = (a.base ? a.base[(size_t)q * d.Nn + nd] : 0.0) + a.s_u * (double)yq;
        }
      } else {
        // dy in three BF16 parts: slots high 0..2, mid 0..2, low 0, low 1 (group 3: low 2)
        float dy[kCout], pt[kCout];
        uint32_t dp[3][kCout];
#pragma unroll
        for (int c = 0; c < kCout; ++c) {
          const float dd = ok ? __shfl(yq, 16 * c + r, 64) - tg[c] : 0.0f;
          if (q == 0) loss += (double)dd * dd;
          dy[c] = 2.0f * dd * ti;
          gb[c] += dy[c];
          pt[c] = dy[c];
#pragma unroll
          for (int i = 0; i < 3; ++i) {
            const __bf16 b = (__bf16)pt[c];
            dp[i][c] = (uint32_t)__builtin_bit_cast(uint16_t, b);
            pt[c] -= (float)b;
          }
        }
        const s8 dv = as_s8(dp[0][0] | dp[0][1] << 16, dp[0][2] | dp[1][0] << 16, dp[1][1] | dp[1][2] << 16,
                            (q == 3 ? dp[2][2] : dp[2][0]) | dp[2][1] << 16);
        f4 dh[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) dh[t] = mfma32(op[64 * (OP_W2T + t)], dv, f4{0.f, 0.f, 0.f, 0.f});
        uint32_t D[8];   // dhpre at places 16 q + 4 e + t
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const uint32_t hw = H[2 * e + (t >> 1)];
            const float hv = __uint_as_float((t & 1) ? hw & 0xffff0000u : hw << 16);
#pragma unroll
            for (int c = 0; c < kCout; ++c) g2[c][4 * e + t] += dy[c] * hv;
            dh[t][e] *= gelu_grad(hp[t][e]);
          }
          D[2 * e] = pack_bf(dh[0][e], dh[1][e]);
          D[2 * e + 1] = pack_bf(dh[2][e], dh[3][e]);
        }
        const s8 d0 = as_s8(D[0], D[1], D[2], D[3]), d1 = as_s8(D[4], D[5], D[6], D[7]);
        if (ok) {
          *(s8*)(a.dhpre + nd * kH + 16 * q) = d0;
          *(s8*)(a.dhpre + nd * kH + 16 * q + 8) = d1;
        }
        f4 dx[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          dx[t] = f4{0.f, 0.f, 0.f, 0.f};
          dx[t] = mfma32(op[64 * (OP_T + 2 * t)], d0, dx[t]);
          dx[t] = mfma32(op[64 * (OP_T + 2 * t + 1)], d1, dx[t]);
        }
        uint32_t P[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float v0 = dx[0][e], v1 = dx[1][e];
          if (BLK) {
            v0 *= gelu_grad(zv[0][e]);
            v1 *= gelu_grad(zv[1][e]);
          }
          P[e] = pack_bf(v0, v1);
        }
        if (ok) *(s8*)(a.dz + nd * kW + 8 * q) = as_s8(P[0], P[1], P[2], P[3]);
      }
    }
  }
  if constexpr (TRAIN) {
    constexpr int TOT = kCout * kH + kCout;
    // sums over the 16 node lanes, then over the waves, in a fixed order
#pragma unroll
    for (int c = 0; c < kCout; ++c) {
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        float v = g2[c][j];
        for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (r == 0) sD[wv * TOT + c * kH + 16 * (j & 3) + 4 * q + (j >> 2)] = v;
      }
      float v = gb[c];
      for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
      if (lane == 0) sD[wv * TOT + kCout * kH + c] = v;
    }
    for (int o = 8; o > 0; o >>= 1) loss += __shfl_xor(loss, o, 64);
    if (lane == 0) sL[wv] = loss;
    __syncthreads();
    for (int i = tid; i < TOT; i += 256)
      a.dw2[(size_t)blockIdx.x * TOT + i] = (sD[i] + sD[TOT + i]) + (sD[2 * TOT + i] + sD[3 * TOT + i]);
    if (tid == 0) a.lpart[blockIdx.x] = (sL[0] + sL[1]) + (sL[2] + sL[3]);
  }
}

// --------------------------------------------------------------------------
// weight gradient of the hidden layer, sums of the gradients' partials
// --------------------------------------------------------------------------

// part[workgroup] = sum_node dhpre[j] x[c] ([64][32]) then sum_node dhpre[j] ([64]): 32 nodes per
// step are the depth of the MFMAs, loaded with the channels of a node on consecutive lanes
__global__ __launch_bounds__(256) void k_hidden_grad(int Nn, const uint16_t* dh, const uint16_t* x, float* part) {
  constexpr int TOT = kH * kW + kH;
  __shared__ float sW[4 * TOT];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, r = lane & 15, q = lane >> 4;
  const s8 ones = {0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
  f4 acc[4][2], db[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    db[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 2; ++u) acc[t][u] = f4{0.f, 0.f, 0.f, 0.f};
  }
  const int groups = (Nn + 31) / 32;
  for (int g = blockIdx.x * 4 + wv; g < groups; g += gridDim.x * 4) {
    uint32_t A[2][2][4], X[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int nd = 32 * g + 16 * h + 4 * q + e;
        uint2 v = make_uint2(0u, 0u);
        X[h][e] = 0u;
        if (nd < Nn) {
          v = *(const uint2*)(dh + (size_t)nd * kH + 4 * r);
          X[h][e] = ((const uint32_t*)x)[(size_t)nd * 16 + r];
        }
        A[0][h][e] = v.x;
        A[1][h][e] = v.y;
      }
    const s8 x0 = node_vec(X, 0), x1 = node_vec(X, 1);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const s8 v = node_vec(A[t >> 1], t & 1);
      acc[t][0] = mfma32(v, x0, acc[t][0]);
      acc[t][1] = mfma32(v, x1, acc[t][1]);
      db[t] = mfma32(v, ones, db[t]);
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int j = 16 * t + 4 * q + e;
      sW[wv * TOT + j * kW + r] = acc[t][0][e];
      sW[wv * TOT + j * kW + 16 + r] = acc[t][1][e];
      if (r == 0) sW[wv * TOT + kH * kW + j] = db[t][e];
    }
  __syncthreads();
  for (int i = tid; i < TOT; i += 256)
    part[(size_t)blockIdx.x * TOT + i] = (sW[i] + sW[TOT + i]) + (sW[2 * TOT + i] + sW[3 * TOT + i]);
}

// Every gradient but the mixing weights': dst[i] = sum over the workgroups' rows, in FP64 and
// in a fixed order.  One launch for all of them: blockIdx.y picks the segment, a block takes 32
// columns with 32 groups of rows (two launches for each of the seven gradients before).
constexpr int kMaxSegs = 11;
struct SumArgs {
  const float* part[kMaxSegs];
  float* dst[kMaxSegs];
  int rows[kMaxSegs], cols[kMaxSegs];
};

__global__ __launch_bounds__(1024) void k_sum_all(SumArgs a) {
  __shared__ double sR[32][33];
  const int s = blockIdx.y, cols = a.cols[s], rows = a.rows[s];
  const int c = threadIdx.x & 31, g = threadIdx.x >> 5, i = blockIdx.x * 32 + c;
  if (blockIdx.x * 32 >= cols) return;
  const float* p = a.part[s] + i;
  double t = 0.0;
  if (i < cols)
    for (int r0 = g; r0 < rows; r0 += 32 * 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = r0 + 32 * u < rows ? p[(size_t)(r0 + 32 * u) * cols] : 0.0f;
#pragma unroll
      for (int u = 0; u < 8; ++u) t += v[u];
    }
  sR[g][c] = t;
  __syncthreads();
  if (g == 0 && i < cols) {
    double v = 0.0;
    for (int j = 0; j < 32; ++j) v += sR[j][c];
    a.dst[s][i] = (float)v;
  }
}

// --------------------------------------------------------------------------
// loss scale
// --------------------------------------------------------------------------

// per-block sums of squares: blocks below gridDim.x / 2 of the [3][Nn] FP32 target, the others
// of the first-iterate channels 9..11 of the input
__global__ __launch_bounds__(256) void k_sq_partial(const float* t, const uint16_t* feat, int Nn, double* part) {
  __shared__ double sred[4];
  const int half = gridDim.x / 2, b = (int)blockIdx.x;
  double s = 0.0;
  if (b < half) {
    for (long long i = (long long)b * 256 + threadIdx.x; i < 3ll * Nn; i += (long long)half * 256) {
      const double v = t[i];
      s += v * v;
    }
  } else {
    for (int i = (b - half) * 256 + threadIdx.x; i < Nn; i += half * 256)
#pragma unroll
      for (int c = 9; c < 12; ++c) {
        const double v = bf2f(feat[(size_t)i * kCh + c]);
        s += v * v;
      }
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if ((threadIdx.x & 63) == 0) sred[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) part[b] = sred[0] + sred[1] + sred[2] + sred[3];
}

// single wave: tsum = sum part, tinv = 1 / tsum
__global__ void k_sq_final(const double* part, int nb, double* tsum, float* tinv) {
  double s = 0.0;
  for (int i = threadIdx.x; i < nb; i += 64) s += part[i];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (threadIdx.x == 0) {
    *tsum = s;
    *tinv = (float)(1.0 / s);
  }
}

__global__ void k_loss_final(const double* lpart, int nb, const double* tsum, double* loss) {
  double s = 0.0;
  for (int i = threadIdx.x; i < nb; i += 64) s += lpart[i];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (threadIdx.x == 0) *loss = s / *tsum;
}

// --------------------------------------------------------------------------
// optimiser and weight images
// --------------------------------------------------------------------------

__global__ void k_adam(float* p, const float* g, float* mo, float* ve, long long P, float lr, float b1, float b2,
                       float eps, float bc1, float bc2) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P) return;
  const float gi = g[i];
  const float mi = b1 * mo[i] + (1.0f - b1) * gi;
  const float vi = b2 * ve[i] + (1.0f - b2) * gi * gi;
  mo[i] = mi;
  ve[i] = vi;
  p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

struct Offsets {
  long long Wl, bl, blk0, blk_stride, Ws, Wb, cb, Wp1, bp1, Wp2, bp2, total;
};

// Part (0 high, 1 what its rounding leaves, 2 what that leaves) of a weight in BF16
__device__ __forceinline__ uint16_t bf_part(float w, int part) {
  for (int i = 0; i < part; ++i) w -= bf2f(f2bf(w));
  return f2bf(w);
}

// Weights as MFMA operands, 64 lanes of 8 BF16 values (1 KB) each, in the layout the kernels
// load: the depth slot 8 q + s of a lane r + 16 q is, for 32 channels stored in pairs, channel
// 4 q + s / 2 + 16 (s mod 2).  Lift: two tiles of outputs (depth = input channel, 12..15 zero); per
// block the forward and the transposed weights, two tiles each; then the output layers'
// operands in the order OP_P .. OP_N.
__global__ __launch_bounds__(256) void k_images(const float* p, Offsets off, int blocks, uint16_t* img) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int f = i >> 9, lane = (i >> 3) & 63, s = i & 7, r = lane & 15, q = lane >> 4;
  const int nf = kOpLift + kOpBlock * blocks + OP_N - OP_P;
  if (f >= nf) return;
  const int ch = 4 * q + (s >> 1) + 16 * (s & 1);
  float w = 0.0f;
  int part = 0;
  if (f < kOpLift) {
    const int c = 8 * q + s;
    if (c < kCin) w = p[off.Wl + (16 * f + r) * kCin + c];
  } else if (f < kOpLift + kOpBlock * blocks) {
    const int b = (f - kOpLift) / kOpBlock, g = (f - kOpLift) % kOpBlock, t = g & 1;
    const float* W = p + off.blk0 + b * off.blk_stride + off.Wb;
    w = g < 2 ? W[(16 * t + r) * kW + ch] : W[ch * kW + 16 * t + r];
  } else {
    const int o = f - kOpLift - kOpBlock * blocks + OP_P;
    const float* W1 = p + off.Wp1;
    const float* W2 = p + off.Wp2;
    if (o < OP_W2) {               // hidden layer, four tiles
      w = W1[(16 * (o - OP_P) + r) * kW + ch];
    } else if (o < OP_T) {         // output layer, half of the hidden channels: row 4 c + part
      const int j = 16 * (s & 3) + 4 * q + 2 * (o - OP_W2) + (s >> 2);
      part = r & 3;
      if ((r >> 2) < kCout && part < 3) w = W2[(r >> 2) * kH + j];
    } else if (o < OP_W2T) {       // transposed hidden layer [tile][half of the hidden channels]
      const int g = o - OP_T;
      w = W1[(16 * (s & 3) + 4 * q + 2 * (g & 1) + (s >> 2)) * kW + 16 * (g >> 1) + r];
    } else {
      // transposed output layer against dy's parts (slots high 0..2, mid 0..2, low 0, low 1, in
      // group 3 low 2): lane group 0 high parts of the weights on all, 1 mid parts on high and
      // mid, 2 low parts on high, 3 the high part on low 2
      const int j = 16 * (o - OP_W2T) + r;
      part = q < 3 ? q : 0;
      if (q == 3) w = s == 6 ? W2[2 * kH + j] : 0.0f;
      else if (s / 3 + q < 3) w = W2[(s % 3) * kH + j];
    }
  }
  img[i] = bf_part(w, part);
}

__global__ void k_zero_f(float* p, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0f;
}

// --------------------------------------------------------------------------
// input channels
// --------------------------------------------------------------------------

__device__ __forceinline__ void young_poisson(double l, double u, double& E, double& nu) {
  const double den = l + u;
  if (den > 0.0) {
    E = u * (3.0 * l + 2.0 * u) / den;
    nu = l / (2.0 * den);
  } else {
    E = 0.0;
    nu = 0.0;
  }
}

__device__ __forceinline__ double load_lame(const void* p, int fp64, long long i) {
  return fp64 ? ((const double*)p)[i] : (double)((const float*)p)[i];
}

__global__ __launch_bounds__(256) void k_emax_partial(FeatArgs a) {
  __shared__ double sred[4];
  double mx = 0.0;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < a.Nv; i += (long long)gridDim.x * 256) {
    double E, nu;
    young_poisson(load_lame(a.lam, a.fp64, i), load_lame(a.mu, a.fp64, i), E, nu);
    mx = fmax(mx, E);
  }
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_down(mx, off, 64));
  if ((threadIdx.x & 63) == 0) sred[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) a.scratch[blockIdx.x] = fmax(fmax(sred[0], sred[1]), fmax(sred[2], sred[3]));
}

__global__ void k_emax_final(FeatArgs a, int nb) {
  double mx = 0.0;
  for (int i = threadIdx.x; i < nb; i += 64) mx = fmax(mx, a.scratch[i]);
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_down(mx, off, 64));
  if (threadIdx.x == 0) a.scratch[256] = mx > 0.0 ? mx : 1.0;
}

__global__ __launch_bounds__(256) void k_features(FeatArgs a) {
  const long long nd = (long long)blockIdx.x * 256 + threadIdx.x;
  if (nd >= a.Nn) return;
  const int x = (int)(nd % a.N[0]), y = (int)((nd / a.N[0]) % a.N[1]), z = (int)(nd / ((long long)a.N[0] * a.N[1]));
  const int X[3] = {x, y, z};
  double Es = 0.0, ns = 0.0;
  int cnt = 0;
  for (int dz = -1; dz <= 0; ++dz)
    for (int dy = -1; dy <= 0; ++dy)
      for (int dx = -1; dx <= 0; ++dx) {
        int v[3] = {x + dx, y + dy, z + dz};
        bool in = true;
        for (int J = 0; J < 3; ++J) {
          if (a.periodic[J]) v[J] = (v[J] + a.n[J]) % a.n[J];
          else if (v[J] < 0 || v[J] >= a.n[J]) in = false;
        }
        if (!in) continue;
        const long long vi = v[0] + (long long)a.n[0] * (v[1] + (long long)a.n[1] * v[2]);
        double E, nu;
        young_poisson(load_lame(a.lam, a.fp64, vi), load_lame(a.mu, a.fp64, vi), E, nu);
        Es += E;
        ns += nu;
        ++cnt;
      }
  float f[kCh];
  for (int c = 0; c < kCh; ++c) f[c] = 0.0f;
  f[0] = (float)(Es / cnt / a.scratch[256]);
  for (int c = 0; c < 3; ++c) f[9 + c] = (float)(a.u1[c * a.Nn + nd] / a.s_u);
  f[1] = (float)(ns / cnt);
  const uint8_t mk = a.mask[nd];
  for (int c = 0; c < 3; ++c) {
    bool fixed = (mk >> c) & 1;
    for (int J = 0; J < 3; ++J) {
      if (a.periodic[J]) continue;
      if (X[J] == 0 && ((a.aface >> (c * 6 + J * 2 + 0)) & 1)) fixed = true;
      if (X[J] == a.n[J] && ((a.aface >> (c * 6 + J * 2 + 1)) & 1)) fixed = true;
    }
    f[2 + c] = fixed ? 1.0f : 0.0f;
  }
  if (a.has_sphere) {
    const int ax = a.face / 2;
    const int idx = (a.face % 2) ? a.n[ax] : 0;
    if (X[ax] == idx) {
      const double ddx = x - a.center[0], ddy = y - a.center[1], ddz = z - a.center[2];
      const double g = sqrt(ddx * ddx + ddy * ddy + ddz * ddz) - a.radius;
      f[8] = (float)tanh(g / (8.0 * a.s_u));
    }
  }
  uint32_t pk[8];
  for (int e = 0; e < 8; ++e) pk[e] = (uint32_t)f2bf(f[2 * e]) | ((uint32_t)f2bf(f[2 * e + 1]) << 16);
  uint4* out = (uint4*)(a.feat + nd * kCh);
  out[0] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
  out[1] = make_uint4(pk[4], pk[5], pk[6], pk[7]);
}

// prescribed values of strong constraints (the mask channel is set by k_features)
__global__ void k_feat_strong(FeatArgs a) {
  const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
  if (e >= a.ms) return;
  a.feat[a.snode[e] * kCh + 5 + a.scomp[e]] = f2bf((float)(a.sval[e] / a.s_u));
}

void launch_features(const FeatArgs& a, hipStream_t s) {
  const int nb = (int)std::min<long long>(256, (a.Nv + 255) / 256);
  hipLaunchKernelGGL(k_emax_partial, dim3(nb), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_emax_final, dim3(1), dim3(64), 0, s, a, nb);
  hipLaunchKernelGGL(k_features, dim3((unsigned)((a.Nn + 255) / 256)), dim3(256), 0, s, a);
  if (a.ms > 0) hipLaunchKernelGGL(k_feat_strong, dim3((unsigned)((a.ms + 255) / 256)), dim3(256), 0, s, a);
}

}  // namespace nnk

// ==========================================================================
// C ABI
// ==========================================================================

using namespace nnk;

// Training target of the learned start: t = (u* - u1) / s_u in FP32 (u* a converged solve,
// u1 the first iterate the input channels carry).
__global__ __launch_bounds__(256) void k_target(const double* __restrict__ u, const double* __restrict__ u1, long long n,
                                                double inv_su, float* __restrict__ t) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n; e += (long long)gridDim.x * blockDim.x)
    t[e] = (float)((u[e] - u1[e]) * inv_su);
}

struct fftc_nn {
  int m = 6, blocks = 4, M3 = 216;
  Offsets off{};
  long long P = 0;
  // state
  float *p = nullptr, *g = nullptr, *mo = nullptr, *ve = nullptr;
  uint16_t* img = nullptr;
  long long img_n = 0;
  int step = 0;
  int state_bound = 0;
  // workspace
  int bound = 0, training = 0;
  Dims d{};
  hipStream_t stream = nullptr;
  float* tab = nullptr;                         // cosine tables
  uint16_t *syn = nullptr, *ana = nullptr;      // their MFMA operands along x
  uint16_t* xs = nullptr;     // activations x_0..x_B (training) or 2 ping-pong buffers
  uint16_t* zs = nullptr;     // pre-activations z_1..z_{B-1} (training)
  uint16_t *dhpre = nullptr, *dz = nullptr;
  float *xh = nullptr, *G = nullptr, *a2 = nullptr;
  float* dw = nullptr;        // per-workgroup weight gradients, one region per layer
  double *dsc = nullptr;      // small FP64 scratch: partials, tsum, loss
  float* tinv = nullptr;
  std::string err;
};

namespace {

constexpr size_t kAlign = 256;

size_t al(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

Offsets make_offsets(int M3, int blocks) {
  Offsets o{};
  o.Wl = 0;
  o.bl = kW * kCin;
  o.blk0 = o.bl + kW;
  o.Ws = 0;
  o.Wb = (long long)M3 * kW * kW;
  o.cb = o.Wb + kW * kW;
  o.blk_stride = o.cb + kW;
  o.Wp1 = o.blk0 + blocks * o.blk_stride;
  o.bp1 = o.Wp1 + kH * kW;
  o.Wp2 = o.bp1 + kH;
  o.bp2 = o.Wp2 + kCout * kH;
  o.total = o.bp2 + kCout;
  return o;
}

int nfail(fftc_nn* nn, int code, const std::string& msg) {
  if (nn) nn->err = msg;
  return code;
}

#define NNCHK(nn, call)                                                                           \
  do {                                                                                            \
    hipError_t e_ = (call);                                                                       \
    if (e_ != hipSuccess) return nfail(nn, FFTC_E_HIP, std::string("HIP: ") + hipGetErrorString(e_)); \
  } while (0)

// Split of the node grid into workgroups of k_line and k_last: a multiple of the four waves'
// lines each, four (one line per wave) up to 2560 workgroups, then more lines for as many
// workgroups.  Measured on whole passes: 65^3 inference 165 us with 4 lines (1105 workgroups), 171
// with 5 or 6, 178 with 8; 129^3 631 us with 8 (2193 workgroups), 654 with 4, 657 with 11.
Dims make_dims(const fftc_nn* nn, const int N[3]) {
  Dims d{};
  for (int J = 0; J < 3; ++J) d.N[J] = N[J];
  d.Nn = N[0] * N[1] * N[2];
  d.m = nn->m;
  d.M3 = nn->M3;
  d.pairs = (N[0] + 31) / 32;
  const long long want = 4 * (((long long)N[1] * N[2] + 10239) / 10240);
  const int most = (int)std::min<long long>(kLines, want);
  d.chunks = (N[1] + most - 1) / most;
  d.lines = (N[1] + d.chunks - 1) / d.chunks;
  return d;
}

int workgroups(const Dims& d) { return d.N[2] * d.chunks; }

constexpr int kDwBlock = kW * kW + kW, kDwLift = kW * kCin + kW, kDwHidden = kH * kW + kH, kDwOut = kCout * kH + kCout;

size_t ws_layout(const fftc_nn* nn, const int N[3], int training, size_t* off /* >= 20 */) {
  const Dims d = make_dims(nn, N);
  const size_t Nn = (size_t)N[0] * N[1] * N[2], wg = (size_t)workgroups(d), B = (size_t)nn->blocks;
  const size_t act = al(2 * Nn * kW);
  size_t o = 0;
  int q = 0;
  off[q++] = o; o += al(4 * (size_t)(N[0] + N[1] + N[2]) * nn->m);               // tab
  off[q++] = o; o += al(2 * (size_t)(32 * d.pairs) * 32);                        // syn
  off[q++] = o; o += al(2 * (size_t)(d.pairs * 3 * nn->m) * 32);                 // ana
  off[q++] = o; o += (training ? (B + 1) : 2) * act;                             // xs
  off[q++] = o; o += training && B > 1 ? (B - 1) * act : 0;                      // zs
  off[q++] = o; o += training ? al(2 * Nn * kH) : 0;                             // dhpre
  off[q++] = o; o += training ? 2 * act : 0;                                     // dz
  off[q++] = o; o += al(4 * std::max<size_t>(B, 1) * (size_t)nn->M3 * kW);       // xh
  off[q++] = o; o += al(4 * (size_t)N[2] * nn->m * nn->m * kW);                  // G
  off[q++] = o; o += al(4 * wg * nn->m * nn->m * kW);                            // a2
  off[q++] = o; o += training ? al(4 * (wg * (B * kDwBlock + kDwLift + kDwOut) + (size_t)kHiddenGrid * kDwHidden)) : 0;  // dw
  off[q++] = o; o += al(8 * (std::max<size_t>(wg, kSqGrid) + 16));               // dsc
  off[q++] = o; o += al(16);                                                     // tinv
  return o;
}

uint16_t* xbuf(fftc_nn* nn, int i) { return nn->xs + (size_t)i * (al(2 * (size_t)nn->d.Nn * kW) / 2); }
uint16_t* zbuf(fftc_nn* nn, int i) { return nn->zs + (size_t)i * (al(2 * (size_t)nn->d.Nn * kW) / 2); }
uint16_t* dzbuf(fftc_nn* nn, int i) { return nn->dz + (size_t)i * (al(2 * (size_t)nn->d.Nn * kW) / 2); }
// weight gradients per workgroup: blocks, lift, output layer, hidden layer
float* dw_block(fftc_nn* nn, int b) { return nn->dw + (size_t)workgroups(nn->d) * b * kDwBlock; }
float* dw_lift(fftc_nn* nn) { return dw_block(nn, nn->blocks); }
float* dw_out(fftc_nn* nn) { return dw_lift(nn) + (size_t)workgroups(nn->d) * kDwLift; }
float* dw_hidden(fftc_nn* nn) { return dw_out(nn) + (size_t)workgroups(nn->d) * kDwOut; }

// weight operands (k_images): lift, block b forward or transposed, output layers
const s8* op_lift(const fftc_nn* nn) { return (const s8*)nn->img; }
const s8* op_block(const fftc_nn* nn, int b, bool t) {
  return (const s8*)nn->img + 64 * (size_t)(kOpLift + kOpBlock * b + (t ? 2 : 0));
}
const s8* op_out(const fftc_nn* nn) { return op_block(nn, nn->blocks, false); }

LineArgs line_args(fftc_nn* nn, const uint16_t* in, const s8* w, const float* bias) {
  LineArgs a{};
  a.d = nn->d;
  a.in = in;
  a.w = w;
  a.bias = bias;
  a.G = nn->G;
  a.tab = nn->tab;
  a.syn = nn->syn;
  a.ana = nn->ana;
  a.a2 = nn->a2;
  return a;
}

template <int IN, bool SYN, int EPI, bool OUT, bool ANA, int AUX>
void line(fftc_nn* nn, const LineArgs& a) {
  hipLaunchKernelGGL((k_line<IN, SYN, EPI, OUT, ANA, AUX>), dim3(workgroups(nn->d)), dim3(256),
                     line_smem(nn->d, SYN, ANA, AUX != AUX_NONE), nn->stream, a);
}

MidArgs mid_args(fftc_nn* nn, float scale, const float* Ws, float* xh) {
  MidArgs a{};
  a.d = nn->d;
  a.rows = workgroups(nn->d);
  a.zmul = (unsigned)((0x100000000ull + nn->d.chunks - 1) / nn->d.chunks);
  a.a2 = nn->a2;
  a.tab = nn->tab;
  a.scale = scale;
  a.Ws = Ws;
  a.xh = xh;
  a.G = nn->G;
  return a;
}

// Lift and the blocks but the last; returns the buffer of the last block's input (of x_0
// without blocks).  Training keeps every activation and pre-activation.
int forward(fftc_nn* nn, const uint16_t* feat) {
  const bool tr = nn->training;
  const float* p = nn->p;
  const Offsets& o = nn->off;
  LineArgs a = line_args(nn, feat, op_lift(nn), p + o.bl);
  a.out = xbuf(nn, 0);
  line<IN_FEAT, false, EPI_NONE, true, true, AUX_NONE>(nn, a);
  int cur = 0;
  for (int b = 0; b < nn->blocks; ++b) {
    const float* blk = p + o.blk0 + b * o.blk_stride;
    const MidArgs ma = mid_args(nn, 1.0f / (float)nn->d.Nn, blk + o.Ws,
                                nn->xh + (size_t)(tr ? b : 0) * nn->M3 * kW);
    hipLaunchKernelGGL(k_mid<false>, dim3(nn->m * nn->m), dim3(1024), 0, nn->stream, ma);
    if (b + 1 == nn->blocks) break;
    const int nxt = tr ? b + 1 : (cur ^ 1);
    a = line_args(nn, xbuf(nn, cur), op_block(nn, b, false), blk + o.cb);
    a.out = xbuf(nn, nxt);
    if (tr) {
      a.zout = zbuf(nn, b);
      line<IN_X, true, EPI_GELU_Z, true, true, AUX_NONE>(nn, a);
    } else {
      line<IN_X, true, EPI_GELU, true, true, AUX_NONE>(nn, a);
    }
    cur = nxt;
  }
  return cur;
}

LastArgs last_args(fftc_nn* nn, int cur) {
  LastArgs a{};
  const Offsets& o = nn->off;
  const int b = nn->blocks - 1;
  a.d = nn->d;
  a.in = xbuf(nn, cur);
  if (b >= 0) {
    a.w = op_block(nn, b, false);
    a.bias = nn->p + o.blk0 + b * o.blk_stride + o.cb;
  }
  a.G = nn->G;
  a.tab = nn->tab;
  a.syn = nn->syn;
  a.wo = op_out(nn);
  a.bp1 = nn->p + o.bp1;
  a.w2 = nn->p + o.Wp2;
  return a;
}

template <bool TRAIN>
void last(fftc_nn* nn, const LastArgs& a) {
  const size_t sm = last_smem(nn->d, nn->blocks > 0, TRAIN);
  if (nn->blocks > 0) hipLaunchKernelGGL((k_last<true, TRAIN>), dim3(workgroups(nn->d)), dim3(256), sm, nn->stream, a);
  else hipLaunchKernelGGL((k_last<false, TRAIN>), dim3(workgroups(nn->d)), dim3(256), sm, nn->stream, a);
}

int check_grid(const int32_t N[3]) {
  for (int J = 0; J < 3; ++J)
    if (N[J] < 2 || N[J] > kMaxN) return 0;
  return 1;
}

}  // namespace

extern "C" {

int fftc_nn_create(fftc_nn_h* out, int32_t modes, int32_t blocks) {
  if (!out) return FFTC_E_ARG;
  *out = nullptr;
  if (modes < 1 || modes > kMaxM || blocks < 0 || blocks > 8) return FFTC_E_UNSUPPORTED;
  fftc_nn* nn = new (std::nothrow) fftc_nn();
  if (!nn) return FFTC_E_ARG;
  nn->m = modes;
  nn->blocks = blocks;
  nn->M3 = modes * modes * modes;
  nn->off = make_offsets(nn->M3, blocks);
  nn->P = nn->off.total;
  nn->img_n = 512ll * (kOpLift + kOpBlock * blocks + OP_N - OP_P);
  *out = nn;
  return FFTC_OK;
}

void fftc_nn_destroy(fftc_nn_h nn) { delete nn; }

int fftc_nn_num_params(fftc_nn_h nn, int64_t* count) {
  if (!nn || !count) return FFTC_E_ARG;
  *count = nn->P;
  return FFTC_OK;
}

int fftc_nn_state_bytes(fftc_nn_h nn, size_t* bytes) {
  if (!nn || !bytes) return FFTC_E_ARG;
  *bytes = 4 * al(4 * (size_t)nn->P) + al(2 * (size_t)nn->img_n);
  return FFTC_OK;
}

int fftc_nn_bind_state(fftc_nn_h nn, void* state_dev, size_t bytes, void* stream) {
  if (!nn || !state_dev) return FFTC_E_ARG;
  size_t need;
  fftc_nn_state_bytes(nn, &need);
  if (bytes < need) return nfail(nn, FFTC_E_WORKSPACE, "state buffer too small");
  if ((uintptr_t)state_dev % kAlign) return nfail(nn, FFTC_E_ARG, "state buffer must be 256-byte aligned");
  char* b = (char*)state_dev;
  const size_t fp = al(4 * (size_t)nn->P);
  nn->p = (float*)b;
  nn->g = (float*)(b + fp);
  nn->mo = (float*)(b + 2 * fp);
  nn->ve = (float*)(b + 3 * fp);
  nn->img = (uint16_t*)(b + 4 * fp);
  nn->stream = (hipStream_t)stream;
  hipLaunchKernelGGL(k_zero_f, dim3((unsigned)((nn->P + 255) / 256)), dim3(256), 0, nn->stream, nn->g, nn->P);
  hipLaunchKernelGGL(k_zero_f, dim3((unsigned)((nn->P + 255) / 256)), dim3(256), 0, nn->stream, nn->mo, nn->P);
  hipLaunchKernelGGL(k_zero_f, dim3((unsigned)((nn->P + 255) / 256)), dim3(256), 0, nn->stream, nn->ve, nn->P);
  nn->step = 0;
  nn->state_bound = 1;
  NNCHK(nn, hipGetLastError());
  return FFTC_OK;
}

int fftc_nn_workspace_bytes(fftc_nn_h nn, const int32_t N[3], int32_t training, size_t* bytes) {
  if (!nn || !N || !bytes) return FFTC_E_ARG;
  if (!check_grid(N)) return FFTC_E_UNSUPPORTED;
  size_t off[20];
  const int Nc[3] = {N[0], N[1], N[2]};
  *bytes = ws_layout(nn, Nc, training, off);
  return FFTC_OK;
}

int fftc_nn_bind(fftc_nn_h nn, const int32_t N[3], int32_t training, void* ws_dev, size_t bytes, void* stream) {
  if (!nn || !N || !ws_dev) return FFTC_E_ARG;
  if (!check_grid(N)) return nfail(nn, FFTC_E_UNSUPPORTED, "node grid must have 2..257 nodes per axis");
  if ((long long)N[0] * N[1] * N[2] >= (1ll << 31) / kH) return nfail(nn, FFTC_E_UNSUPPORTED, "grid too large");
  if ((uintptr_t)ws_dev % kAlign) return nfail(nn, FFTC_E_ARG, "workspace must be 256-byte aligned");
  size_t off[20];
  const int Nc[3] = {N[0], N[1], N[2]};
  const size_t need = ws_layout(nn, Nc, training, off);
  if (bytes < need) return nfail(nn, FFTC_E_WORKSPACE, "workspace too small");
  char* b = (char*)ws_dev;
  int q = 0;
  nn->tab = (float*)(b + off[q++]);
  nn->syn = (uint16_t*)(b + off[q++]);
  nn->ana = (uint16_t*)(b + off[q++]);
  nn->xs = (uint16_t*)(b + off[q++]);
  nn->zs = (uint16_t*)(b + off[q++]);
  nn->dhpre = (uint16_t*)(b + off[q++]);
  nn->dz = (uint16_t*)(b + off[q++]);
  nn->xh = (float*)(b + off[q++]);
  nn->G = (float*)(b + off[q++]);
  nn->a2 = (float*)(b + off[q++]);
  nn->dw = (float*)(b + off[q++]);
  nn->dsc = (double*)(b + off[q++]);
  nn->tinv = (float*)(b + off[q++]);
  nn->training = training ? 1 : 0;
  nn->stream = (hipStream_t)stream;
  nn->d = make_dims(nn, Nc);
  // cosine tables phi_k(i) = cos(pi k (i + 1/2) / N_J), per axis [N_J][m]
  std::vector<float> tab;
  for (int J = 0; J < 3; ++J)
    for (int i = 0; i < N[J]; ++i)
      for (int k = 0; k < nn->m; ++k) tab.push_back((float)cos(M_PI * k * (i + 0.5) / N[J]));
  // the x tables as MFMA operands: the spectral term's slots (high, high, low parts per mode),
  // and the analysis's three parts per mode in the node order of node_vec; nodes past the
  // line are 0
  const Dims& d = nn->d;
  std::vector<uint16_t> syn(32 * (size_t)(32 * d.pairs), 0), ana(32 * (size_t)(d.pairs * 3 * d.m), 0);
  for (int x = 0; x < N[0]; ++x) {
    const int p = x / 32, n = x % 32;
    const int place = 8 * ((n % 16) / 4) + 4 * (n / 16) + n % 4;   // place of node n among the 32 depth slots
    for (int k = 0; k < d.m; ++k) {
      float c = tab[(size_t)x * d.m + k];
      for (int part = 0; part < 3; ++part) {
        const uint16_t h = f2bf(c);
        ana[((size_t)(p * 3 + part) * d.m + k) * 32 + place] = h;
        if (part == 0) syn[(size_t)x * 32 + k] = syn[(size_t)x * 32 + d.m + k] = h;
        if (part == 1) syn[(size_t)x * 32 + 2 * d.m + k] = h;
        const uint32_t hb = (uint32_t)h << 16;
        float hf;
        memcpy(&hf, &hb, 4);
        c -= hf;
      }
    }
  }
  // the three tables are neighbours in the workspace: one copy
  std::vector<char> all((size_t)((char*)nn->ana - (char*)nn->tab) + 2 * ana.size(), 0);
  memcpy(all.data(), tab.data(), 4 * tab.size());
  memcpy(all.data() + ((char*)nn->syn - (char*)nn->tab), syn.data(), 2 * syn.size());
  memcpy(all.data() + ((char*)nn->ana - (char*)nn->tab), ana.data(), 2 * ana.size());
  NNCHK(nn, hipMemcpyAsync(nn->tab, all.data(), all.size(), hipMemcpyHostToDevice, nn->stream));
  NNCHK(nn, hipStreamSynchronize(nn->stream));
  nn->bound = 1;
  return FFTC_OK;
}

int fftc_nn_set_params(fftc_nn_h nn, const float* params_dev) {
  if (!nn || !params_dev) return FFTC_E_ARG;
  if (!nn->state_bound) return nfail(nn, FFTC_E_STATE, "state not bound");
  NNCHK(nn, hipMemcpyAsync(nn->p, params_dev, 4 * nn->P, hipMemcpyDeviceToDevice, nn->stream));
  hipLaunchKernelGGL(k_zero_f, dim3((unsigned)((nn->P + 255) / 256)), dim3(256), 0, nn->stream, nn->mo, nn->P);
  hipLaunchKernelGGL(k_zero_f, dim3((unsigned)((nn->P + 255) / 256)), dim3(256), 0, nn->stream, nn->ve, nn->P);
  hipLaunchKernelGGL(k_images, dim3((unsigned)((nn->img_n + 255) / 256)), dim3(256), 0, nn->stream,
                     (const float*)nn->p, nn->off, nn->blocks, nn->img);
  nn->step = 0;
  NNCHK(nn, hipGetLastError());
  return FFTC_OK;
}

int fftc_nn_get_params(fftc_nn_h nn, float* params_dev) {
  if (!nn || !params_dev) return FFTC_E_ARG;
  if (!nn->state_bound) return nfail(nn, FFTC_E_STATE, "state not bound");
  NNCHK(nn, hipMemcpyAsync(params_dev, nn->p, 4 * nn->P, hipMemcpyDeviceToDevice, nn->stream));
  return FFTC_OK;
}

int fftc_nn_get_grad(fftc_nn_h nn, float* grad_dev) {
  if (!nn || !grad_dev) return FFTC_E_ARG;
  if (!nn->state_bound) return nfail(nn, FFTC_E_STATE, "state not bound");
  NNCHK(nn, hipMemcpyAsync(grad_dev, nn->g, 4 * nn->P, hipMemcpyDeviceToDevice, nn->stream));
  return FFTC_OK;
}

int fftc_nn_forward(fftc_nn_h nn, const uint16_t* feat_dev, float* y_dev, double s_u, const double* base_dev,
                    double* u0_dev) {
  if (!nn || !feat_dev) return FFTC_E_ARG;
  if (!nn->state_bound || !nn->bound) return nfail(nn, FFTC_E_STATE, "state and workspace must be bound");
  const int tr = nn->training;
  nn->training = 0;
  // inference uses the ping-pong buffers even on a training workspace
  const int cur = forward(nn, feat_dev);
  nn->training = tr;
  LastArgs a = last_args(nn, cur);
  a.y = y_dev;
  a.u0 = u0_dev;
  a.base = base_dev;
  a.s_u = s_u;
  last<false>(nn, a);
  NNCHK(nn, hipGetLastError());
  return FFTC_OK;
}

int fftc_nn_train_step(fftc_nn_h nn, const uint16_t* feat_dev, const float* target_dev, double* loss_dev) {
  if (!nn || !feat_dev || !target_dev) return FFTC_E_ARG;
  if (!nn->state_bound || !nn->bound) return nfail(nn, FFTC_E_STATE, "state and workspace must be bound");
  if (!nn->training) return nfail(nn, FFTC_E_STATE, "workspace was bound without training");
  hipStream_t s = nn->stream;
  const Offsets& o = nn->off;
  const int Nn = nn->d.Nn;
  const int B = nn->blocks;
  const int wg = workgroups(nn->d);
  const int cur = forward(nn, feat_dev);
  // 1 / (sum t^2 + sum b^2); dsc: [0] the sum, [1] loss, from [8] per-block partials (squares
  // first, then the loss)
  double* tsum = nn->dsc;
  double* lossd = nn->dsc + 1;
  double* dpart = nn->dsc + 8;
  hipLaunchKernelGGL(k_sq_partial, dim3(kSqGrid), dim3(256), 0, s, target_dev, feat_dev, Nn, dpart);
  hipLaunchKernelGGL(k_sq_final, dim3(1), dim3(64), 0, s, (const double*)dpart, kSqGrid, tsum, nn->tinv);
  // last block, output layers, loss, and back to the pre-activation of the last block
  uint16_t* dcur = dzbuf(nn, 0);
  LastArgs la = last_args(nn, cur);
  la.target = target_dev;
  la.tinv = nn->tinv;
  la.xout = xbuf(nn, B);
  la.dhpre = nn->dhpre;
  la.dz = dcur;
  la.dw2 = dw_out(nn);
  la.lpart = dpart;   // the squares' partials are consumed above
  last<true>(nn, la);
  hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(64), 0, s, (const double*)dpart, wg, (const double*)tsum,
                     loss_dev ? loss_dev : lossd);
  hipLaunchKernelGGL(k_hidden_grad, dim3(kHiddenGrid), dim3(256), 0, s, Nn, (const uint16_t*)nn->dhpre,
                     (const uint16_t*)xbuf(nn, B), dw_hidden(nn));
  float* g = nn->g;
  LineArgs a = line_args(nn, dcur, nullptr, nullptr);
  if (B > 0) {
    a.aux = xbuf(nn, B - 1);
    a.dw = dw_block(nn, B - 1);
    line<IN_D, false, EPI_NONE, false, true, AUX_X>(nn, a);
  } else {
    a.aux = feat_dev;
    a.dw = dw_lift(nn);
    line<IN_D, false, EPI_NONE, false, false, AUX_FEAT>(nn, a);
  }
  int side = 0;
  for (int b = B - 1; b >= 0; --b) {
    // the analysis of dz_b and, but for the first, its weight gradient came with dz_b itself
    MidArgs ma = mid_args(nn, 1.0f, nn->p + o.blk0 + b * o.blk_stride + o.Ws, nn->xh + (size_t)b * nn->M3 * kW);
    ma.dWs = g + o.blk0 + b * o.blk_stride + o.Ws;
    ma.inv_nn = 1.0f / (float)Nn;
    hipLaunchKernelGGL(k_mid<true>, dim3(nn->m * nn->m), dim3(1024), 0, s, ma);
    a = line_args(nn, dcur, op_block(nn, b, true), nullptr);
    if (b > 0) {
      uint16_t* dnext = dzbuf(nn, side ^ 1);
      a.zaux = zbuf(nn, b - 1);
      a.aux = xbuf(nn, b - 1);
      a.out = dnext;
      a.dw = dw_block(nn, b - 1);
      line<IN_X, true, EPI_DGELU, true, true, AUX_X>(nn, a);
      side ^= 1;
      dcur = dnext;
    } else {
      a.aux = feat_dev;
      a.dw = dw_lift(nn);
      line<IN_X, true, EPI_NONE, false, false, AUX_FEAT>(nn, a);
    }
  }
  SumArgs sa{};
  int n = 0, most = 0;
  auto seg = [&](const float* part, int rows, int cols, float* dst) {
    sa.part[n] = part;
    sa.rows[n] = rows;
    sa.cols[n] = cols;
    sa.dst[n] = dst;
    most = std::max(most, cols);
    ++n;
  };
  for (int b = 0; b < B; ++b) seg(dw_block(nn, b), wg, kDwBlock, g + o.blk0 + b * o.blk_stride + o.Wb);
  seg(dw_lift(nn), wg, kDwLift, g + o.Wl);
  seg(dw_hidden(nn), kHiddenGrid, kDwHidden, g + o.Wp1);
  seg(dw_out(nn), wg, kDwOut, g + o.Wp2);
  hipLaunchKernelGGL(k_sum_all, dim3((most + 31) / 32, n), dim3(1024), 0, s, sa);
  NNCHK(nn, hipGetLastError());
  return FFTC_OK;
}

int fftc_nn_adam_step(fftc_nn_h nn, float lr, float beta1, float beta2, float eps) {
  if (!nn) return FFTC_E_ARG;
  if (!nn->state_bound) return nfail(nn, FFTC_E_STATE, "state not bound");
  if (!(beta1 >= 0.f && beta1 < 1.f && beta2 >= 0.f && beta2 < 1.f && eps > 0.f && lr >= 0.f))
    return nfail(nn, FFTC_E_ARG, "invalid Adam hyper-parameters");
  nn->step += 1;
  const float bc1 = (float)(1.0 - pow((double)beta1, nn->step));
  const float bc2 = (float)(1.0 - pow((double)beta2, nn->step));
  hipLaunchKernelGGL(k_adam, dim3((unsigned)((nn->P + 255) / 256)), dim3(256), 0, nn->stream, nn->p,
                     (const float*)nn->g, nn->mo, nn->ve, nn->P, lr, beta1, beta2, eps, bc1, bc2);
  hipLaunchKernelGGL(k_images, dim3((unsigned)((nn->img_n + 255) / 256)), dim3(256), 0, nn->stream,
                     (const float*)nn->p, nn->off, nn->blocks, nn->img);
  NNCHK(nn, hipGetLastError());
  return FFTC_OK;
}

int fftc_nn_make_target(const double* u_dev, const double* u1_dev, int64_t count, double s_u, float* target_dev,
                        void* stream) {
  if (!u_dev || !u1_dev || !target_dev || count < 0 || !(s_u > 0.0)) return FFTC_E_ARG;
  if (count == 0) return FFTC_OK;
  const unsigned nb = (unsigned)std::min<long long>((count + 255) / 256, 8192);
  hipLaunchKernelGGL(k_target, dim3(nb), dim3(256), 0, (hipStream_t)stream, u_dev, u1_dev, (long long)count,
                     1.0 / s_u, target_dev);
  return hipGetLastError() == hipSuccess ? FFTC_OK : FFTC_E_HIP;
}

const char* fftc_nn_last_error(fftc_nn_h nn) { return nn ? nn->err.c_str() : "null network"; }

}  // extern "C"
