// Learned eigensolver preconditioner: a three-layer 3-D convolutional network
//   x (1 channel) -> conv 3^3 (8) -> ReLU -> conv 3^3 (8) -> ReLU -> conv 3^3 (1)
// with zero padding, BF16 weights (FP32 master copies updated by Adam) and FP32 activations
// and accumulation.  Forward, backward (data and weight gradients), the mean-squared loss and
// Adam are hand-written kernels; the C ABI below drives inference and training on the device.
//
// Hidden activations and their gradients are [sample][x][y][z][channel] FP32 (the 32 bytes of a
// point are one row of the matrix-core kernels).  Weights of a layer are [out][in][27] with
// tap t = 9 (dx + 1) + 3 (dy + 1) + (dz + 1) acting on the input at offset (dx, dy, dz).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/ace.h"
#include "ctx.hpp"

namespace {

using ace::host::Buf;
using ace::host::ensure_on;
using ace::host::hip_check;

constexpr int kT = 256;
constexpr int C = 8;  // hidden channels
// output tile of one workgroup of the 8-channel kernels (and its halo of one point)
constexpr int TX = 4, TY = 8, TZ = 16;
constexpr int HX = TX + 2, HY = TY + 2, HZ = TZ + 2;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// parameter layout: [w0 8x1x27][b0 8][w1 8x8x27][b1 8][w2 1x8x27][b2 1]
constexpr int W0 = 0, B0 = W0 + C * 27, W1 = B0 + C, B1 = W1 + C * C * 27, W2 = B1 + C,
              B2 = W2 + C * 27, NPAR = B2 + 1;
static_assert(NPAR == ACE_NET_PARAMS, "parameter count");

struct Tiles {
  int nx, ny, nz;
  explicit Tiles(int n, int tx = TX, int ty = TY, int tz = TZ)
      : nx((n + tx - 1) / tx), ny((n + ty - 1) / ty), nz((n + tz - 1) / tz) {}
  int count() const { return nx * ny * nz; }
};

__device__ __forceinline__ void tile_origin(int bt, int tny, int tnz, int tx, int ty, int tz,
                                            int* x0, int* y0, int* z0) {
  *z0 = bt % tnz * tz;
  *y0 = bt / tnz % tny * ty;
  *x0 = bt / (tnz * tny) * tx;
}
__device__ __forceinline__ bool in_box(int x, int y, int z, int n) {
  return (unsigned)x < (unsigned)n && (unsigned)y < (unsigned)n && (unsigned)z < (unsigned)n;
}

// Weights laid out for the kernels below, rebuilt by k_pack whenever the compute copy changes.
// Every weight is a BF16 value, so the BF16 forms are exact.
struct Packed {
  float to8[27][C];      // layer 0: [tap][out channel]
  float to8t[27][C];     // layer 2 transposed and flipped (its data gradient): [tap][channel]
  __bf16 mid[9][64][8];  // layer 1: MFMA operand of (dx, dy), see k_conv88
  __bf16 midt[9][64][8]; // layer 1 transposed and flipped
  __bf16 to1[2][64][8];  // layer 2: MFMA operand of taps 0-15 and 16-26, see k_conv81
  float zero[C];         // what a point outside the box reads
};

__global__ __launch_bounds__(kT) void k_pack(const float* __restrict__ weff, Packed* __restrict__ pk) {
  const float* w0 = weff + W0;
  const float* w1 = weff + W1;
  const float* w2 = weff + W2;
  const int stride = gridDim.x * kT;
  for (int e = blockIdx.x * kT + threadIdx.x; e < 27 * C; e += stride) {
    const int t = e / C, c = e % C;
    pk->to8[t][c] = w0[c * 27 + t];
    pk->to8t[t][c] = w2[c * 27 + 26 - t];
  }
  for (int e = blockIdx.x * kT + threadIdx.x; e < 9 * 64 * 8; e += stride) {
    const int q = e / 512, l = e / 8 % 64, j = e % 8;
    const int o = l % 8, dz = l / 16 - l % 16 / 8, t = q * 3 + dz;
    const bool on = dz >= 0 && dz < 3;
    pk->mid[q][l][j] = (__bf16)(on ? w1[(o * C + j) * 27 + t] : 0.f);
    pk->midt[q][l][j] = (__bf16)(on ? w1[(j * C + o) * 27 + 26 - t] : 0.f);
  }
  for (int e = blockIdx.x * kT + threadIdx.x; e < 2 * 64 * 8; e += stride) {
    const int mt = e / 512, l = e / 8 % 64, j = e % 8, t = mt * 16 + l % 16;
    pk->to1[mt][l][j] = (__bf16)(l / 16 < 3 && t < 27 ? w2[j * 27 + t] : 0.f);
  }
  if (blockIdx.x == 0 && threadIdx.x < C) pk->zero[threadIdx.x] = 0.f;
}

// An FP32 value as the exact sum of three BF16 ones (8 + 8 + 8 significant bits), each returned
// as the FP32 bits whose upper half is the BF16 value.  FINITE = false: infinities and NaN go to
// the first part alone (else an infinity makes the others NaN).
struct Split3 {
  unsigned hi, mid, lo;
};
template <bool FINITE>
__device__ __forceinline__ Split3 split3(float x) {
  const unsigned h = __float_as_uint(x) & 0xffff0000u;
  const float r = FINITE || __builtin_isfinite(x) ? x - __uint_as_float(h) : 0.f;
  const unsigned m = __float_as_uint(r) & 0xffff0000u;
  return {h, m, __float_as_uint(r - __uint_as_float(m))};
}
// upper halves of a and b as one dword (a in the low half)
__device__ __forceinline__ unsigned hi_halves(unsigned a, unsigned b) {
  return __builtin_amdgcn_perm(b, a, 0x07060302u);
}

// 1 -> 8 channels: out[p][c] = act(b[c] + sum_t w[t][c] in[p + d_t]) (* (mask[p][c] > 0)).
// Four points along x per thread; the 8 weights of a tap are scalar operands (uniform loads), so
// the 216 FMAs of a point need 27 LDS reads and no weight reads.  64^3 x 16: 55 us, vector
// instructions in 60 % of the slots (317 a point, 100 of them for staging and addresses; the tile's
// rows of 18 meet bank conflicts in 48 % of the cycles in which LDS is busy, a fifth of all); 48 us
// with channel-planar stores, which cost the next layer more than the 7 us.
constexpr int QX = 8, QY = 8, QZ = 16;  // its tile
template <bool BIAS, bool RELU, bool MASK>
__global__ __launch_bounds__(kT) void k_conv18(const float* __restrict__ in,
                                               const float (*__restrict__ w)[C],
                                               const float* __restrict__ b,
                                               const float* __restrict__ mask,
                                               float* __restrict__ out, int n, int tny, int tnz) {
  constexpr int RZ = QZ + 2, RY = QY + 2, VOL = (QX + 2) * RY * RZ, XP = 4;
  __shared__ float tile[VOL];
  const size_t ng = (size_t)n * n * n;
  int x0, y0, z0;
  tile_origin(blockIdx.x, tny, tnz, QX, QY, QZ, &x0, &y0, &z0);
  const float* inb = in + blockIdx.y * ng;
  for (int e = threadIdx.x; e < VOL; e += kT) {
    const int gx = x0 + e / (RZ * RY) - 1, gy = y0 + e / RZ % RY - 1, gz = z0 + e % RZ - 1;
    const bool ok = in_box(gx, gy, gz, n);
    const float v = inb[ok ? ((size_t)gx * n + gy) * n + gz : 0];
    tile[e] = ok ? v : 0.f;
  }
  __syncthreads();
  const int lz = threadIdx.x % QZ, ly = threadIdx.x / QZ % QY, lx = threadIdx.x / (QZ * QY) * XP;
  float acc[XP][C];
#pragma unroll
  for (int p = 0; p < XP; ++p)
#pragma unroll
    for (int c = 0; c < C; ++c) acc[p][c] = BIAS ? b[c] : 0.f;
  // (one dx at a time: its 72 weights fit in the scalar registers, all 216 do not)
#pragma unroll 1
  for (int dx = 0; dx < 3; ++dx)
#pragma unroll
    for (int dy = 0; dy < 3; ++dy)
#pragma unroll
      for (int dz = 0; dz < 3; ++dz) {
        float v[XP];
#pragma unroll
        for (int p = 0; p < XP; ++p) v[p] = tile[((lx + p + dx) * RY + ly + dy) * RZ + lz + dz];
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const float wt = w[dx * 9 + dy * 3 + dz][c];
#pragma unroll
          for (int p = 0; p < XP; ++p) acc[p][c] = fmaf(wt, v[p], acc[p][c]);
        }
      }
#pragma unroll
  for (int p = 0; p < XP; ++p) {
    const int gx = x0 + lx + p, gy = y0 + ly, gz = z0 + lz;
    if (!in_box(gx, gy, gz, n)) continue;
    const size_t pt = (blockIdx.y * ng + ((size_t)gx * n + gy) * n + gz) * C;
#pragma unroll
    for (int c = 0; c < C; c += 4) {
      float4 v = make_float4(acc[p][c], acc[p][c + 1], acc[p][c + 2], acc[p][c + 3]);
      if (RELU) v = make_float4(fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f));
      if (MASK) {
        const float4 m = *reinterpret_cast<const float4*>(mask + pt + c);
        v = make_float4(m.x > 0.f ? v.x : 0.f, m.y > 0.f ? v.y : 0.f, m.z > 0.f ? v.z : 0.f,
                        m.w > 0.f ? v.w : 0.f);
      }
      *reinterpret_cast<float4*>(out + pt + c) = v;
    }
  }
}

// 8 -> 8 channels on the matrix cores: out[p][o] = act(b[o] + sum_j sum_t w[o][j][t] in[p + d_t][j])
// (* (mask[p][o] > 0)).  One v_mfma_f32_16x16x32_bf16 takes the taps of one (dx, dy): row = a
// couple of points (z, z + 1), column = (which of the two, output channel), contraction = four
// z taps x 8 channels; of the four taps each point of the couple uses three, the weight of the
// fourth is zero.  The FP32 inputs are split exactly into three BF16 parts (split3) while the
// tile is staged in LDS, one 16-byte row of 8 channels per point and part, so the products are
// exact and only the FP32 sums round, as in the FMA form.  A wavefront computes 2 x 4 lines of
// 16 z points: a row block is read once per input line and used for the up to three output
// lines it touches, 54 KB of LDS reads for 108 MFMAs.
// The products of the two smaller parts have sums of their own: added to the full sum they lose
// bits always in the same direction (outputs 4e-9 too small relative to FP64, against 1e-10 with
// their own sums or as FMAs; the rounding error itself falls from 3.2e-7 to 1.8e-7).
// The zero weights reach one point further than the layer does: an infinity there would turn a
// finite sum into NaN, so a NaN sum is formed again from the definition.
// Workgroups take several tiles and request the next one's points while they work one.
// 64^3 x 16: 272 us as FMAs on the vector units (53 TFLOP/s), 73 us here (199 TFLOP/s of the
// layer's own products); with a tile per workgroup 106 us.
template <bool BIAS, bool RELU, bool MASK>
__global__ __launch_bounds__(kT, 3) void k_conv88(const float* __restrict__ in,
                                               const bf16x8* __restrict__ wq,
                                               const float* __restrict__ b,
                                               const float* __restrict__ mask,
                                               const float* __restrict__ zero,
                                               float* __restrict__ out, int n, int tny, int tnz,
                                               int ntile, int nb) {
  // plane stride HY HZ + 1 points: the two x lines of a row block lie 4 banks apart
  constexpr int PL = HY * HZ + 1, PV = HX * PL, NPT = HX * HY * HZ, LD = (NPT + kT - 1) / kT;
  __shared__ __align__(16) uint4 tile[3][PV];
  const size_t ng = (size_t)n * n * n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  bf16x8 w[9];
#pragma unroll
  for (int q = 0; q < 9; ++q) w[q] = wq[q * 64 + lane];
  const int o = lane & 7;
  const float bias = BIAS ? b[o] : 0.f;
  // this thread's points of the next tile, requested while the current one is worked
  float4 f0[LD], f1[LD];
  auto fetch = [&](int bt) __attribute__((always_inline)) {
    int x0, y0, z0;
    tile_origin(bt % ntile, tny, tnz, TX, TY, TZ, &x0, &y0, &z0);
    const float* inb = in + (size_t)(bt / ntile) * ng * C;
#pragma unroll
    for (int u = 0; u < LD; ++u) {
      const int e = threadIdx.x + u * kT;
      const int gx = x0 + e / (HZ * HY) - 1, gy = y0 + e / HZ % HY - 1, gz = z0 + e % HZ - 1;
      const bool ok = e < NPT && in_box(gx, gy, gz, n);
      const float4* src =
          reinterpret_cast<const float4*>(ok ? inb + (((size_t)gx * n + gy) * n + gz) * C : zero);
      f0[u] = src[0];
      f1[u] = src[1];
    }
  };
  if ((int)blockIdx.x < ntile * nb) fetch(blockIdx.x);
  for (int bt = blockIdx.x; bt < ntile * nb; bt += gridDim.x) {
    __syncthreads();  // the previous tile's readers are done
#pragma unroll
    for (int u = 0; u < LD; ++u) {
      const int e = threadIdx.x + u * kT;
      if (e >= NPT) break;
      const float f[C] = {f0[u].x, f0[u].y, f0[u].z, f0[u].w, f1[u].x, f1[u].y, f1[u].z, f1[u].w};
      Split3 s[C];
#pragma unroll
      for (int c = 0; c < C; ++c) s[c] = split3<true>(f[c]);
      const int at = e / (HZ * HY) * PL + e % (HZ * HY);
      tile[0][at] = make_uint4(hi_halves(s[0].hi, s[1].hi), hi_halves(s[2].hi, s[3].hi),
                               hi_halves(s[4].hi, s[5].hi), hi_halves(s[6].hi, s[7].hi));
      tile[1][at] = make_uint4(hi_halves(s[0].mid, s[1].mid), hi_halves(s[2].mid, s[3].mid),
                               hi_halves(s[4].mid, s[5].mid), hi_halves(s[6].mid, s[7].mid));
      tile[2][at] = make_uint4(hi_halves(s[0].lo, s[1].lo), hi_halves(s[2].lo, s[3].lo),
                               hi_halves(s[4].lo, s[5].lo), hi_halves(s[6].lo, s[7].lo));
    }
    __syncthreads();
    if (bt + (int)gridDim.x < ntile * nb) fetch(bt + gridDim.x);
    const int xw = (wave & 1) * 2, yw = (wave >> 1) * 4;  // the wavefront's lines
    const int row = lane & 15, tap = lane >> 4;
    const bf16x8* base = reinterpret_cast<const bf16x8*>(&tile[0][0]) + (xw + row / 8) * PL +
                         yw * HZ + 2 * (row % 8) + tap;
    f32x4 acc[4] = {}, low[4] = {};
#pragma unroll
    for (int dx = 0; dx < 3; ++dx)
#pragma unroll
      for (int yi = 0; yi < 6; ++yi) {  // input line yw + yi - 1
        const bf16x8* r = base + dx * PL + yi * HZ;
        const bf16x8 hi = r[0], mid = r[PV], lo = r[2 * PV];
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) {
          const int yo = yi - dy;
          if (yo < 0 || yo > 3) continue;
          low[yo] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, w[dx * 3 + dy], low[yo], 0, 0, 0);
          low[yo] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mid, w[dx * 3 + dy], low[yo], 0, 0, 0);
          acc[yo] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, w[dx * 3 + dy], acc[yo], 0, 0, 0);
        }
      }
    // lane: column (point of the couple, channel) = lane % 16, rows 4 (lane / 16) + q: one x, z
    // two apart from row to row
    int x0, y0, z0;
    tile_origin(bt % ntile, tny, tnz, TX, TY, TZ, &x0, &y0, &z0);
    const size_t sb = bt / ntile;
    const int gx = x0 + xw + (lane >> 5), gy = y0 + yw,
              gz = z0 + (lane >> 4 & 1) * 8 + (lane >> 3 & 1);
    const size_t at = (sb * ng + ((size_t)gx * n + gy) * n + gz) * C + o;
    auto put = [&](int yo, int q, float v) {
      const size_t a = at + ((size_t)yo * n + 2 * q) * C;
      if (RELU) v = fmaxf(v, 0.f);
      if (MASK) v = mask[a] > 0.f ? v : 0.f;
      out[a] = v;
    };
    bool nan = false;
    if (gx < n) {
#pragma unroll
      for (int yo = 0; yo < 4; ++yo) {
        if (gy + yo >= n) break;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float v = acc[yo][q] + (low[yo][q] + bias);
          nan |= v != v;
          if (gz + 2 * q < n) put(yo, q, v);
        }
      }
    }
    if (nan) {
      // this lane's outputs from the definition: the weight of (o, j, tap) is in the operand of
      // its (dx, dy), lane 16 dz + o
#pragma unroll 1
      for (int i = 0; i < 16; ++i) {
        const int yo = i / 4, q = i % 4;
        if (gy + yo >= n || gz + 2 * q >= n) continue;
        float v = bias;
#pragma unroll 1
        for (int j = 0; j < C; ++j)
#pragma unroll 1
          for (int t = 0; t < 27; ++t) {
            const int hx = gx + t / 9 - 1, hy = gy + yo + t / 3 % 3 - 1, hz = gz + 2 * q + t % 3 - 1;
            const float f = in_box(hx, hy, hz, n)
                                ? in[(sb * ng + ((size_t)hx * n + hy) * n + hz) * C + j] : 0.f;
            v = fmaf((float)reinterpret_cast<const __bf16*>(wq + t / 3 * 64 + t % 3 * 16 + o)[j], f, v);
          }
        put(yo, q, v);
      }
    }
  }
}

// 8 -> 1 channel: y[p] = b + sum_t (w[t] . in[p + d_t]) over the 8 channels.  The 27 tap products
// w[t] . in[q] of an input point q are two MFMAs per 16 points (rows = taps, columns = points,
// contraction = the three exact BF16 parts of 8 channels: every input value is read and split
// once); they pass through LDS, where each output adds its 27.  A workgroup marches along x
// over 16 x 16 lines, the products of one x plane (with halo) at a time: each plane is used for
// the three outputs x - 1, x, x + 1, carried in registers.  64^3 x 16: 153 us as FMAs with the
// inputs staged in LDS, 67 us here (134 MB read, 2.0 TB/s; the LDS passes and their barriers
// bound it).
// An infinite weight times a part that is zero makes a NaN of an infinite product, so a NaN output
// is formed again from the definition.
// LOSS: instead of y, writes g = (y - t) / count and the workgroup's sum of (y - t)^2.
constexpr int MY = 16, MZ = 16;  // lines of a workgroup; it marches over mx planes
template <bool LOSS>
__global__ __launch_bounds__(kT) void k_conv81(const float* __restrict__ in,
                                               const bf16x8* __restrict__ wq,
                                               const float* __restrict__ b,
                                               const float* __restrict__ t, float inv_count,
                                               float* __restrict__ y, double* __restrict__ part,
                                               int n, int mx, int tny, int tnz) {
  constexpr int RY = MY + 2, RZ = MZ + 2, NPT = RY * RZ, GW = (NPT + 63) / 64, TS = 388;
  // GW 16-point groups per wavefront; all 32 product rows are written, 27 are read
  static_assert(GW * 64 <= TS && TS % 16 == 4, "rows of four lane groups in different banks");
  __shared__ float pr[32 * TS];
  __shared__ double red[LOSS ? kT : 1];
  const size_t ng = (size_t)n * n * n;
  int x0, y0, z0;
  tile_origin(blockIdx.x, tny, tnz, mx, MY, MZ, &x0, &y0, &z0);
  const float* inb = in + blockIdx.y * ng * C;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, quad = lane >> 4;
  const bf16x8 w0 = wq[lane], w1 = wq[64 + lane];
  // lane group quad holds channels 2 quad and 2 quad + 1 of its 16 points
  float2 f[GW];
  auto fetch = [&](int gx) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < GW; ++u) {
      const int p = (wave + 4 * u) * 16 + (lane & 15);
      const int gy = y0 + p / RZ - 1, gz = z0 + p % RZ - 1;
      const bool ok = p < NPT && in_box(gx, gy, gz, n);
      const float2 v = reinterpret_cast<const float2*>(
          inb + (ok ? ((size_t)gx * n + gy) * n + gz : 0) * C)[quad];
      f[u].x = ok ? v.x : 0.f;
      f[u].y = ok ? v.y : 0.f;
    }
  };
  const int ly = threadIdx.x / MZ, lz = threadIdx.x % MZ;
  const bool mine = y0 + ly < n && z0 + lz < n;
  const float bias = b[0];
  float r0 = 0.f, r1 = 0.f;  // sums begun for the outputs x' + 1 and x'
  double loss = 0.0;
  bool nan = false;
  const int xe = min(n, x0 + mx);
  fetch(x0 - 1);
  for (int xp = x0 - 1; xp <= xe; ++xp) {
    if (xp >= x0) __syncthreads();  // the previous plane's readers are done
#pragma unroll
    for (int u = 0; u < GW; ++u) {
      const int grp = wave + 4 * u;
      {
        // the three parts of the lane's channel couple, then transposed over the four lane
        // groups: group k gets part k of all 8 channels (part 3 is zero)
        const Split3 a = split3<false>(f[u].x), c = split3<false>(f[u].y);
        const auto h = __builtin_amdgcn_permlane16_swap(hi_halves(a.hi, c.hi),
                                                        hi_halves(a.mid, c.mid), false, false);
        const auto l = __builtin_amdgcn_permlane16_swap(hi_halves(a.lo, c.lo), 0u, false, false);
        const auto e = __builtin_amdgcn_permlane32_swap(h[0], l[0], false, false);
        const auto g = __builtin_amdgcn_permlane32_swap(h[1], l[1], false, false);
        const u32x4 d = {(unsigned)e[0], (unsigned)g[0], (unsigned)e[1], (unsigned)g[1]};
        const bf16x8 v = __builtin_bit_cast(bf16x8, d);
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        const f32x4 a0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0, v, zero, 0, 0, 0);
        const f32x4 a1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, v, zero, 0, 0, 0);
        float* dst = pr + grp * 16 + (lane & 15) + 4 * quad * TS;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          dst[q * TS] = a0[q];
          dst[(16 + q) * TS] = a1[q];
        }
      }
    }
    if (xp < xe) fetch(xp + 1);
    __syncthreads();
    float s[3];
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
      s[dx] = 0.f;
#pragma unroll
      for (int q = 0; q < 9; ++q)
        s[dx] += pr[(dx * 9 + q) * TS + (ly + q / 3) * RZ + lz + q % 3];
    }
    const float done = r1 + s[2];  // output x' - 1: its planes x' - 2, x' - 1 and x'
    r1 = r0 + s[1];
    r0 = bias + s[0];
    if (xp - 1 >= x0 && mine) {
      const size_t at = blockIdx.y * ng + ((size_t)(xp - 1) * n + y0 + ly) * n + z0 + lz;
      const bool ok = done == done;
      nan |= !ok;
      if (LOSS) {
        const float d = done - t[at];
        y[at] = d * inv_count;
        loss += ok ? (double)d * d : 0.0;
      } else {
        y[at] = done;
      }
    }
  }
  if (nan) {
#pragma unroll 1
    for (int x = x0; x < xe; ++x) {
      const size_t at = blockIdx.y * ng + ((size_t)x * n + y0 + ly) * n + z0 + lz;
      if (y[at] == y[at]) continue;
      // the weight of (tap, channel j) is element j of operand tap / 16, lane tap % 16
      float v = bias;
#pragma unroll 1
      for (int j = 0; j < C; ++j)
#pragma unroll 1
        for (int q = 0; q < 27; ++q) {
          const int hx = x + q / 9 - 1, hy = y0 + ly + q / 3 % 3 - 1, hz = z0 + lz + q % 3 - 1;
          const float a = in_box(hx, hy, hz, n) ? inb[(((size_t)hx * n + hy) * n + hz) * C + j] : 0.f;
          v = fmaf((float)reinterpret_cast<const __bf16*>(wq + q / 16 * 64 + q % 16)[j], a, v);
        }
      if (LOSS) {
        const float d = v - t[at];
        y[at] = d * inv_count;
        loss += (double)d * d;
      } else {
        y[at] = v;
      }
    }
  }
  if (LOSS) {
    red[threadIdx.x] = loss;
    __syncthreads();
    for (int k = kT / 2; k > 0; k >>= 1) {
      if ((int)threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
      __syncthreads();
    }
    if (threadIdx.x == 0) part[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = red[0];
  }
}

// Weight and bias gradient partials of the 8 -> 8 layer: gw[o][i][t] = sum_p g[p][o] in[p + d_t][i],
// gb[o] = sum_p g[p][o], as FP32 matrix products (v_mfma_f32_16x16x4_f32: exact FP32 products and
// sums) with the points as the contraction.  Rows = (s, o): channel o of g at line y + s; columns
// = (c, i): channel i of the input at line y - 1 + 2 c; so one product of a (dx, dz) gives the
// taps dy = -1 (s 0, c 0), +1 (s 0, c 1) and 0 (s 1, c 1).  The lines y run from one before the
// tile to its last, with zeros for g outside it, so each product of a point counts once: 9 lines
// for 8.  A workgroup takes tiles blockIdx.x, blockIdx.x + gridDim.x, ... of all samples, the
// next one's points requested while the current one is worked, and keeps its sums in registers,
// FP32 within a tile and FP64 over tiles; the four wavefronts (one x each) are added in order at
// the end.
// 64^3 x 8: 355 us with one thread per (input channel, tap), whose two LDS reads per FMA bounded
// it; 104 us here, the matrix cores busy in two thirds of the cycles (154 us with the couples
// taken along z, five steps of four points for 16, and no request ahead).
__global__ __launch_bounds__(kT, 2) void k_wgrad88(const float* __restrict__ in,
                                                   const float* __restrict__ g,
                                                   const float* __restrict__ zero,
                                                   float* __restrict__ part, int n, int tny,
                                                   int tnz, int ntile, int nb) {
  constexpr int IY = TY + 3, GY = TY + 2;  // lines of the input (from y0 - 2) and of g (y0 - 1)
  constexpr int NPL = C * C * 27 + C;
  constexpr int NI = HX * HY * HZ * 2, NG = TX * TY * TZ * 2;  // 16-byte halves of points to load
  constexpr int LI = (NI + kT - 1) / kT, LG = NG / kT;
  static_assert(TX == 4 && NG % kT == 0, "one x per wavefront, whole rounds");
  __shared__ __align__(16) float ti[HX * IY * HZ * C];
  __shared__ __align__(16) float tg[TX * GY * TZ * C];
  static_assert(HX * IY * HZ * C >= 4 * 9 * 256 + 4 * 64, "the sums of the wavefronts fit in the tile");
  __shared__ int again;
  const size_t ng = (size_t)n * n * n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane & 15, kk = lane >> 4;
  f32x4 fi[LI], fg[LG];
  auto fetch = [&](int bt) __attribute__((always_inline)) {
    const size_t sb = bt / ntile;
    int x0, y0, z0;
    tile_origin(bt % ntile, tny, tnz, TX, TY, TZ, &x0, &y0, &z0);
    const float* inb = in + sb * ng * C;
    const float* gb = g + sb * ng * C;
#pragma unroll
    for (int u = 0; u < LI; ++u) {
      const int e = threadIdx.x + u * kT, half = e & 1, p = e >> 1;
      const int gx = x0 + p / (HZ * HY) - 1, gy = y0 + p / HZ % HY - 1, gz = z0 + p % HZ - 1;
      const bool ok = e < NI && in_box(gx, gy, gz, n);
      fi[u] = reinterpret_cast<const f32x4*>(ok ? inb + (((size_t)gx * n + gy) * n + gz) * C : zero)[half];
    }
#pragma unroll
    for (int u = 0; u < LG; ++u) {
      const int e = threadIdx.x + u * kT, half = e & 1, p = e >> 1;
      const int gx = x0 + p / (TZ * TY), gy = y0 + p / TZ % TY, gz = z0 + p % TZ;
      const bool ok = in_box(gx, gy, gz, n);
      fg[u] = reinterpret_cast<const f32x4*>(ok ? gb + (((size_t)gx * n + gy) * n + gz) * C : zero)[half];
    }
  };
  // the lines that stay zero: input line y0 - 2, g lines y0 - 1 and y0 + TY
  const f32x4 z4 = {0.f, 0.f, 0.f, 0.f};
  for (int e = threadIdx.x; e < HX * HZ * 2; e += kT)
    reinterpret_cast<f32x4*>(ti)[e / (HZ * 2) * IY * HZ * 2 + e % (HZ * 2)] = z4;
  for (int e = threadIdx.x; e < TX * 2 * TZ * 2; e += kT)
    reinterpret_cast<f32x4*>(tg)[(e / (TZ * 4) * GY + (e / (TZ * 2) & 1) * (GY - 1)) * TZ * 2 + e % (TZ * 2)] = z4;
  if (threadIdx.x == 0) again = 0;
  double sum[9][4], gtot;
  for (bool careful = false;; careful = true) {
    gtot = 0.0;
#pragma unroll
    for (int q = 0; q < 9; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) sum[q][r] = 0.0;
    if ((int)blockIdx.x < ntile * nb) fetch(blockIdx.x);
    for (int bt = blockIdx.x; bt < ntile * nb; bt += gridDim.x) {
      __syncthreads();  // the previous tile's readers are done
#pragma unroll
      for (int u = 0; u < LI; ++u) {
        const int e = threadIdx.x + u * kT, ln = e / (HZ * 2);  // line of HX x HY
        if (e < NI)
          reinterpret_cast<f32x4*>(ti)[(ln / HY * IY + ln % HY + 1) * HZ * 2 + e % (HZ * 2)] = fi[u];
      }
#pragma unroll
      for (int u = 0; u < LG; ++u) {
        const int e = threadIdx.x + u * kT, ln = e / (TZ * 2);
        reinterpret_cast<f32x4*>(tg)[(ln / TY * GY + ln % TY + 1) * TZ * 2 + e % (TZ * 2)] = fg[u];
      }
      __syncthreads();
      if (bt + (int)gridDim.x < ntile * nb) fetch(bt + gridDim.x);
      const float* ga = tg + ((wave * GY + col / 8) * TZ + kk) * C + col % 8;
      const float* ib = ti + ((wave * IY + 2 * (col / 8)) * HZ + kk) * C + col % 8;
      f32x4 acc[9] = {};
      float gsum = 0.f;
#pragma unroll 1
      for (int ly = 0; ly <= TY; ++ly, ga += TZ * C, ib += HZ * C) {
        if (careful && ly == TY && kk >= 2) {  // s = 1 ends before its zero line
#pragma unroll
          for (int q = 0; q < 9; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) sum[q][r] += acc[q][r];
        }
#pragma unroll
        for (int ks = 0; ks < TZ / 4; ++ks) {
          const float a = ga[ks * 4 * C];
          gsum += a;
#pragma unroll
          for (int q = 0; q < 9; ++q) {  // (dx, dz)
            const float v = ib[(q / 3 * IY * HZ + q % 3 + ks * 4) * C];
            acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, v, acc[q], 0, 0, 0);
          }
        }
        if (careful && ly == 0 && kk < 2) {  // s = 0 begins after its zero line
#pragma unroll
          for (int q = 0; q < 9; ++q) acc[q] = z4;
        }
      }
      if (!careful || kk < 2) {
#pragma unroll
        for (int q = 0; q < 9; ++q)
#pragma unroll
          for (int r = 0; r < 4; ++r) sum[q][r] += acc[q][r];
      }
      gtot += gsum;
    }
    // A zero line of g makes a NaN of an infinite input: where a sum is not finite, all is done once
    // more with the sums of rows s (lanes with kk / 2 = s) kept from their zero line.  (Kept from it
    // always: 4 % slower.)
    bool odd = false;
#pragma unroll
    for (int q = 0; q < 9; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) odd |= !__builtin_isfinite(sum[q][r]);
    if (odd) again = 1;
    __syncthreads();
    if (careful || !again) break;
  }
  float* red = ti;  // [wave][(dx, dz)][row][col], then [wave][lane]
#pragma unroll
  for (int q = 0; q < 9; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) red[(wave * 9 + q) * 256 + (4 * kk + r) * 16 + col] = (float)sum[q][r];
  red[4 * 9 * 256 + threadIdx.x] = (float)gtot;
  __syncthreads();
  float* pb = part + (size_t)blockIdx.x * NPL;
  for (int e = threadIdx.x; e < 9 * 256; e += kT) {
    const int q = e / 256, rw = e % 256 / 16, cl = e % 16;
    const int s = rw / 8, c = cl / 8;
    if (s == 1 && c == 0) continue;
    const float v = red[e] + red[e + 9 * 256] + red[e + 18 * 256] + red[e + 27 * 256];
    pb[(rw % 8 * C + cl % 8) * 27 + q / 3 * 9 + (s == 1 ? 1 : 2 * c) * 3 + q % 3] = v;
  }
  if (threadIdx.x < C) {
    float v = 0.f;  // rows s = 0, channel o: lanes 16 k + o of every wavefront
    for (int k = 0; k < 16; ++k) v += red[4 * 9 * 256 + k * 16 + threadIdx.x];
    pb[C * C * 27 + threadIdx.x] = v;
  }
}

// Weight gradient partials between a scalar field s and an 8-channel field f:
// gw[c][t] = sum_p s[p + SIGN d_t] f[p][c], with the points as the contraction of FP32 matrix
// products: rows = the 27 taps (two products of 16) and a row of ones, which gives sum_p f[p][c]
// (the bias gradient of the 1 -> 8 layer, SIGN = 1); columns = channels.  SIGN = -1, s = g,
// f = the input: the 8 -> 1 layer, whose bias gradient sum_p s[p] is added up beside it.
// For SIGN = -1 the sums run over f's points, and s is zero where p - d_t leaves the box; the layer's
// own sum, over s's points, has no such product, but one of s[p] with a zero of f outside the box.
// Both only matter where a value is infinite: such a wavefront forms its sums again point by point.
// Tiles and sums as in k_wgrad88.  64^3 x 8: 138 us (8 -> 1) and 99 us (1 -> 8) with a thread per
// output; 31 and 30 us here (75 MB read).
template <int SIGN>
__global__ __launch_bounds__(kT, 4) void k_wgrad18(const float* __restrict__ s,
                                                const float* __restrict__ f,
                                                const float* __restrict__ zero,
                                                float* __restrict__ part, int n, int tny, int tnz,
                                                int ntile, int nb) {
  constexpr int NPL = C * 27 + (SIGN > 0 ? C : 1), SV = HX * HY * HZ;
  // the scalar tile, then a 1 and zeros that the rows without a tap read
  __shared__ float ts[SV + 32];
  __shared__ __align__(16) float tf[TX * TY * TZ * C];
  __shared__ float red[4][2][256];
  const size_t ng = (size_t)n * n * n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane & 15, kk = lane >> 4;
  if (threadIdx.x < 32) ts[SV + threadIdx.x] = threadIdx.x < 16 ? 1.f : 0.f;
  double sum[2][4] = {};
  double stot = 0.0;
  // where this lane's row starts in the scalar tile for line (0, 0) and z 0, and whether it moves
  // with the point: taps do, the constant rows do not
  int off[2], move[2];
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    const int t = m * 16 + col;
    const int dx = SIGN * (t / 9 - 1), dy = SIGN * (t / 3 % 3 - 1), dz = SIGN * (t % 3 - 1);
    move[m] = t < 27;
    off[m] = t < 27 ? ((1 + dx) * HY + 1 + dy) * HZ + 1 + dz + kk : SV + (t == 27 ? 0 : 16) + kk;
  }
  constexpr int LS = (SV + kT - 1) / kT, LF = TX * TY * TZ * 2 / kT;
  float vs[LS];
  f32x4 vf[LF];
  auto fetch = [&](int bt) __attribute__((always_inline)) {
    const size_t sb = bt / ntile;
    int x0, y0, z0;
    tile_origin(bt % ntile, tny, tnz, TX, TY, TZ, &x0, &y0, &z0);
    const float* sp = s + sb * ng;
    const float* fp = f + sb * ng * C;
#pragma unroll
    for (int u = 0; u < LS; ++u) {
      const int e = threadIdx.x + u * kT;
      const int gx = x0 + e / (HZ * HY) - 1, gy = y0 + e / HZ % HY - 1, gz = z0 + e % HZ - 1;
      const bool ok = e < SV && in_box(gx, gy, gz, n);
      vs[u] = *(ok ? sp + ((size_t)gx * n + gy) * n + gz : zero);
    }
#pragma unroll
    for (int u = 0; u < LF; ++u) {
      const int e = threadIdx.x + u * kT, half = e & 1, p = e >> 1;
      const int gx = x0 + p / (TZ * TY), gy = y0 + p / TZ % TY, gz = z0 + p % TZ;
      const bool ok = in_box(gx, gy, gz, n);
      vf[u] = reinterpret_cast<const f32x4*>(ok ? fp + (((size_t)gx * n + gy) * n + gz) * C : zero)[half];
    }
  };
  if ((int)blockIdx.x < ntile * nb) fetch(blockIdx.x);
  for (int bt = blockIdx.x; bt < ntile * nb; bt += gridDim.x) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < LS; ++u) {
      const int e = threadIdx.x + u * kT;
      if (e < SV) ts[e] = vs[u];
    }
#pragma unroll
    for (int u = 0; u < LF; ++u) reinterpret_cast<f32x4*>(tf)[threadIdx.x + u * kT] = vf[u];
    __syncthreads();
    if (bt + (int)gridDim.x < ntile * nb) fetch(bt + gridDim.x);
    f32x4 acc[2] = {};
    float ssum = 0.f;
    if (SIGN < 0)  // the tile's own points of s (zero outside the box)
      for (int e = threadIdx.x; e < TX * TY * TZ; e += kT)
        ssum += ts[((e / (TZ * TY) + 1) * HY + e / TZ % TY + 1) * HZ + e % TZ + 1];
    for (int line = wave * 8; line < wave * 8 + 8; ++line) {
      const int lx = line / TY, ly = line % TY, at = (lx * HY + ly) * HZ;
      const float* fb = tf + (line * TZ + kk) * C + (col & 7);
      const float* s0 = ts + off[0] + (move[0] ? at : 0);
      const float* s1 = ts + off[1] + (move[1] ? at : 0);
#pragma unroll
      for (int ks = 0; ks < TZ / 4; ++ks) {
        const float v = fb[ks * 4 * C];
        const float bv = col < C ? v : 0.f;
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(s0[move[0] ? ks * 4 : 0], bv, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(s1[move[1] ? ks * 4 : 0], bv, acc[1], 0, 0, 0);
      }
    }
    if (SIGN < 0) {
      bool odd = false;
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) odd |= !__builtin_isfinite(acc[m][r]);
      if (__any(odd)) {
        int x0, y0, z0;
        tile_origin(bt % ntile, tny, tnz, TX, TY, TZ, &x0, &y0, &z0);
#pragma unroll 1
        for (int i = 0; i < 8; ++i) {  // one at a time, for the registers' sake
          const int t = i / 4 * 16 + 4 * kk + i % 4;
          const int dx = t / 9 - 1, dy = t / 3 % 3 - 1, dz = t % 3 - 1;
          float v = 0.f;
#pragma unroll 1
          for (int e = 0; e < TY * TZ && t < 27; ++e) {  // the wavefront's points (x = wave)
            const int py = e / TZ, pz = e % TZ;
            const int gx = x0 + wave, gy = y0 + py, gz = z0 + pz;
            if (!in_box(gx, gy, gz, n)) continue;
            const float* sp = ts + ((wave + 1) * HY + py + 1) * HZ + pz + 1;
            if (in_box(gx - dx, gy - dy, gz - dz, n))
              v = fmaf(sp[-((dx * HY + dy) * HZ + dz)],
                       tf[((wave * TY + py) * TZ + pz) * C + (col & 7)], v);
            if (!in_box(gx + dx, gy + dy, gz + dz, n)) v = fmaf(sp[0], 0.f, v);
          }
#pragma unroll
          for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[m][r] = i == m * 4 + r ? v : acc[m][r];
        }
      }
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) sum[m][r] += acc[m][r];
    stot += ssum;
  }
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][m][(4 * kk + r) * 16 + col] = (float)sum[m][r];
  __syncthreads();
  float* pb = part + (size_t)blockIdx.x * NPL;
  for (int e = threadIdx.x; e < 512; e += kT) {
    const int t = e / 16, c = e % 16;
    if (c >= C || t > 27) continue;
    const float* r = &red[0][0][0] + e;
    const float v = r[0] + r[512] + r[1024] + r[1536];
    if (t < 27)
      pb[c * 27 + t] = v;
    else if (SIGN > 0)
      pb[C * 27 + c] = v;
  }
  if (SIGN < 0) {
    __syncthreads();
    float* q = &red[0][0][0];
    q[threadIdx.x] = (float)stot;
    __syncthreads();
    for (int k = kT / 2; k > 0; k >>= 1) {
      if ((int)threadIdx.x < k) q[threadIdx.x] += q[threadIdx.x + k];
      __syncthreads();
    }
    if (threadIdx.x == 0) pb[C * 27] = q[0];
  }
}

// grad[j] = sum over the partial rows of its layer (FP64, fixed order), and the loss from its
// partials: 16 columns per workgroup, 64 threads each over the rows, so that a row's 16 values
// are one 64-byte read.
struct GradParts {
  const float* part[3];  // layers 0, 1, 2: [rows][npl]
  int npl[3];
  int rows[3];
  const double* lpart;
  int lrows;
  double lscale;
};
constexpr int RC = 16;
__global__ __launch_bounds__(1024) void k_grad_reduce(GradParts gp, float* __restrict__ grad,
                                                      double* __restrict__ loss) {
  __shared__ double red[64][RC];
  const int c = threadIdx.x % RC, k = threadIdx.x / RC;
  if ((int)blockIdx.x == (NPAR + RC - 1) / RC) {
    double s = 0.0;
    for (int i = threadIdx.x; i < gp.lrows; i += 1024) s += gp.lpart[i];
    red[k][c] = s;
    __syncthreads();
    if (threadIdx.x < RC) {
      s = 0.0;
      for (int i = 0; i < 64; ++i) s += red[i][threadIdx.x];
      red[0][threadIdx.x] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      s = 0.0;
      for (int i = 0; i < RC; ++i) s += red[0][i];
      *loss = gp.lscale * s;
    }
    return;
  }
  const int j = blockIdx.x * RC + c;
  const int layer = j >= W2 ? 2 : j >= W1 ? 1 : 0;
  const int col = j - (layer == 2 ? W2 : layer == 1 ? W1 : W0);
  double s = 0.0;
  if (j < NPAR) {
    const float* p = gp.part[layer] + col;
    const int npl = gp.npl[layer], rows = gp.rows[layer];
#pragma unroll 8
    for (int r = k; r < rows; r += 64) s += p[(size_t)r * npl];
  }
  red[k][c] = s;
  __syncthreads();
  if (k == 0 && j < NPAR) {
    s = 0.0;
    for (int i = 0; i < 64; ++i) s += red[i][c];
    grad[j] = (float)s;
  }
}

// round to the nearest BF16 value (ties to even), returned as FP32
__device__ __forceinline__ float bf16_round(float x) {
  unsigned u = __float_as_uint(x);
  u += 0x7fffu + ((u >> 16) & 1u);
  return __uint_as_float(u & 0xffff0000u);
}

__global__ void k_round_params(const float* __restrict__ w, int np, float* __restrict__ weff) {
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < np; e += gridDim.x * blockDim.x)
    weff[e] = bf16_round(w[e]);
}

// Adam (bias-corrected moments) on the FP32 masters; refreshes the BF16 compute copy
__global__ void k_adam(float* __restrict__ w, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, int np, float lr, float b1, float b2,
                       float eps, float c1, float c2, float* __restrict__ weff) {
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < np; e += gridDim.x * blockDim.x) {
    const float ge = g[e];
    const float me = b1 * m[e] + (1.f - b1) * ge;
    const float ve = b2 * v[e] + (1.f - b2) * ge * ge;
    m[e] = me;
    v[e] = ve;
    const float mh = me / c1, vh = ve / c2;
    const float we = w[e] - lr * mh / (sqrtf(vh) + eps);
    w[e] = we;
    weff[e] = bf16_round(we);
  }
}

// minibatch assembly from a counter-based generator (SplitMix64 of seed and slot)
__device__ __forceinline__ unsigned long long splitmix64(unsigned long long z) {
  z += 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

__global__ __launch_bounds__(kT) void k_gather(const float* __restrict__ xs, const float* __restrict__ ts,
                                               int count, size_t ng, unsigned long long seed,
                                               long long step, int batch, int random,
                                               float* __restrict__ xb, float* __restrict__ tb) {
  const int s = blockIdx.y;
  int idx = s % count;
  float sg = 1.f;
  if (random) {
    const unsigned long long hsh = splitmix64(seed ^ splitmix64((unsigned long long)step * batch + s));
    idx = (int)((hsh >> 1) % (unsigned long long)count);
    sg = (hsh & 1ull) ? -1.f : 1.f;
  }
  for (size_t e = (size_t)blockIdx.x * kT + threadIdx.x; e < ng; e += (size_t)gridDim.x * kT) {
    xb[(size_t)s * ng + e] = sg * xs[(size_t)idx * ng + e];
    tb[(size_t)s * ng + e] = sg * ts[(size_t)idx * ng + e];
  }
}

}  // namespace

struct ace_convnet {
  hipStream_t stream = nullptr;
  float* w = nullptr;     // FP32 masters [NPAR]
  float* weff = nullptr;  // BF16-rounded compute copy [NPAR]
  float* m = nullptr;
  float* v = nullptr;
  float* grad = nullptr;
  Packed* pk = nullptr;   // the compute copy as the kernels read it
  double* loss = nullptr; // device scalar
  long long t = 0;        // Adam step counter
  Buf a1, a2, g, g2, g1, part, lpart, xb, tb, lhist;
};

namespace {

int net_alloc(ace_convnet* net) {
  float** bufs[] = {&net->w, &net->weff, &net->m, &net->v, &net->grad};
  for (float** b : bufs)
    if (hipMalloc(b, NPAR * sizeof(float)) != hipSuccess) return ACE_ERR_OOM;
  if (hipMalloc(&net->pk, sizeof(Packed)) != hipSuccess ||
      hipMalloc(&net->loss, sizeof(double)) != hipSuccess)
    return ACE_ERR_OOM;
  return ACE_OK;
}

void pack(ace_convnet* net) { k_pack<<<18, kT, 0, net->stream>>>(net->weff, net->pk); }

// workgroups of the weight-gradient kernels, i.e. partial rows per layer: as many as run at once
// (four on a CU, two for the 8 -> 8 layer with its 58 KB of LDS), each adding up several tiles
constexpr int kGradRows = 1024, kGradRows88 = 512;

// workgroups of k_conv88: three fit on a CU (52 KB of LDS each), each then takes several tiles
int conv_grid(int ntile, int nb) { return (int)std::min<long long>(768, (long long)ntile * nb); }

// planes a workgroup of k_conv81 marches over: three workgroups fit on a CU (50 KB of LDS), so as
// many equal pieces of each line as fill the device once, of at least 8 planes (two planes of
// halo each)
int march(int n, int nb) {
  const int lines = ((n + MY - 1) / MY) * ((n + MZ - 1) / MZ);
  const int pieces = std::max(1, std::min(n / 8, (int)(768 / std::min<long long>(768, (long long)lines * nb))));
  return (n + pieces - 1) / pieces;
}

// activations ([sample][x][y][z][channel]) of a batch of nb samples of edge n
int net_ensure(ace_convnet* net, int n, int nb, bool train) {
  const size_t ng = (size_t)n * n * n;
  hipStream_t s = net->stream;
  int rc = ensure_on(s, net->a1, sizeof(float) * C * ng * nb);
  if (!rc) rc = ensure_on(s, net->a2, sizeof(float) * C * ng * nb);
  if (!rc && train) {
    rc = ensure_on(s, net->g, sizeof(float) * ng * nb);
    if (!rc) rc = ensure_on(s, net->g2, sizeof(float) * C * ng * nb);
    if (!rc) rc = ensure_on(s, net->g1, sizeof(float) * C * ng * nb);
    if (!rc) rc = ensure_on(s, net->part, sizeof(float) * kGradRows * NPAR);
    if (!rc) rc = ensure_on(s, net->lpart, sizeof(double) * Tiles(n, march(n, nb), MY, MZ).count() * nb);
  }
  return rc;
}

// the two hidden layers into a1 and a2
void hidden(ace_convnet* net, int n, const float* x, int nb) {
  const Tiles tq(n, QX, QY, QZ), tl(n);
  float* a1 = (float*)net->a1.p;
  k_conv18<true, true, false><<<dim3(tq.count(), nb), kT, 0, net->stream>>>(
      x, net->pk->to8, net->weff + B0, nullptr, a1, n, tq.ny, tq.nz);
  k_conv88<true, true, false><<<conv_grid(tl.count(), nb), kT, 0, net->stream>>>(
      a1, (const bf16x8*)net->pk->mid, net->weff + B1, nullptr, net->pk->zero,
      (float*)net->a2.p, n, tl.ny, tl.nz,
      tl.count(), nb);
}

void forward(ace_convnet* net, int n, const float* x, int nb, float* y) {
  const int mx = march(n, nb);
  const Tiles tm(n, mx, MY, MZ);
  hidden(net, n, x, nb);
  k_conv81<false><<<dim3(tm.count(), nb), kT, 0, net->stream>>>(
      (const float*)net->a2.p, (const bf16x8*)net->pk->to1, net->weff + B2, nullptr, 0.f, y,
      nullptr, n, mx, tm.ny, tm.nz);
}

// loss into net->loss and its gradient into net->grad, for inputs x and targets t
void gradient(ace_convnet* net, int n, const float* x, const float* t, int nb) {
  const int mx = march(n, nb);
  const Tiles tm(n, mx, MY, MZ), tq(n, QX, QY, QZ), tl(n);
  const size_t ng = (size_t)n * n * n, count = ng * nb;
  hipStream_t s = net->stream;
  float* a1 = (float*)net->a1.p;
  float* a2 = (float*)net->a2.p;
  float* g = (float*)net->g.p;
  float* g2 = (float*)net->g2.p;
  float* g1 = (float*)net->g1.p;
  const int nt = tl.count();
  auto rows = [&](int most) { return (int)std::min<long long>(most, (long long)nt * nb); };
  float* part = (float*)net->part.p;
  GradParts gp{};
  gp.npl[0] = W1 - W0;
  gp.npl[1] = W2 - W1;
  gp.npl[2] = NPAR - W2;
  gp.rows[0] = gp.rows[2] = rows(kGradRows);
  gp.rows[1] = rows(kGradRows88);
  float* p0 = part;
  float* p1 = p0 + (size_t)gp.rows[0] * gp.npl[0];
  float* p2 = p1 + (size_t)gp.rows[1] * gp.npl[1];
  gp.part[0] = p0;
  gp.part[1] = p1;
  gp.part[2] = p2;
  gp.lpart = (const double*)net->lpart.p;
  gp.lrows = tm.count() * nb;
  gp.lscale = 0.5 / (double)count;
  hidden(net, n, x, nb);
  k_conv81<true><<<dim3(tm.count(), nb), kT, 0, s>>>(a2, (const bf16x8*)net->pk->to1, net->weff + B2,
                                                     t, 1.f / (float)count, g,
                                                     (double*)net->lpart.p, n, mx, tm.ny, tm.nz);
  // layer 2 (8 -> 1)
  k_wgrad18<-1><<<gp.rows[2], kT, 0, s>>>(g, a2, net->pk->zero, p2, n, tl.ny, tl.nz, nt, nb);
  k_conv18<false, false, true><<<dim3(tq.count(), nb), kT, 0, s>>>(g, net->pk->to8t, nullptr, a2, g2,
                                                                   n, tq.ny, tq.nz);
  // layer 1 (8 -> 8)
  k_wgrad88<<<gp.rows[1], kT, 0, s>>>(a1, g2, net->pk->zero, p1, n, tl.ny, tl.nz, nt, nb);
  k_conv88<false, false, true><<<conv_grid(nt, nb), kT, 0, s>>>(
      g2, (const bf16x8*)net->pk->midt, nullptr, a1, net->pk->zero, g1, n, tl.ny, tl.nz, nt, nb);
  // layer 0 (1 -> 8)
  k_wgrad18<1><<<gp.rows[0], kT, 0, s>>>(x, g1, net->pk->zero, p0, n, tl.ny, tl.nz, nt, nb);
  k_grad_reduce<<<(NPAR + RC - 1) / RC + 1, 1024, 0, s>>>(gp, net->grad, net->loss);
}

void adam(ace_convnet* net, double lr) {
  const double b1 = 0.9, b2 = 0.999;
  net->t += 1;
  const float c1 = (float)(1.0 - std::pow(b1, (double)net->t));
  const float c2 = (float)(1.0 - std::pow(b2, (double)net->t));
  k_adam<<<(NPAR + kT - 1) / kT, kT, 0, net->stream>>>(net->w, net->m, net->v, net->grad, NPAR,
                                                       (float)lr, (float)b1, (float)b2, 1e-8f,
                                                       c1, c2, net->weff);
  pack(net);
}

}  // namespace

namespace ace {
// preconditioner application for the SCF driver: y_j = net(x_j), FP32 grid vectors
int convnet_apply_internal(ace_convnet* net, int n, const float* x, int nb, float* y,
                           hipStream_t s) {
  hipStream_t keep = net->stream;
  net->stream = s;
  int rc = net_ensure(net, n, nb, false);
  if (!rc) forward(net, n, x, nb, y);
  net->stream = keep;
  return rc ? rc : hip_check(hipGetLastError());
}
}  // namespace ace

extern "C" {

int convnet_create(void* hip_stream, ace_convnet** out) {
  if (!out) return ACE_ERR_INVALID;
  *out = nullptr;
  ace_convnet* net = new (std::nothrow) ace_convnet();
  if (!net) return ACE_ERR_OOM;
  net->stream = (hipStream_t)hip_stream;
  int rc = net_alloc(net);
  if (!rc) {
    std::vector<float> zero(NPAR, 0.f);
    for (float* b : {net->w, net->weff, net->m, net->v, net->grad})
      if (hipMemcpy(b, zero.data(), NPAR * sizeof(float), hipMemcpyHostToDevice) != hipSuccess)
        rc = ACE_ERR_HIP;
    // packed on the network's stream and waited for, as by convnet_set_params: a network may be
    // used on other streams than its own (a memset of the null stream need not have ended by then)
    if (!rc) {
      pack(net);
      if (hipGetLastError() != hipSuccess || hipStreamSynchronize(net->stream) != hipSuccess)
        rc = ACE_ERR_HIP;
    }
  }
  if (rc) {
    (void)hipGetLastError();
    convnet_destroy(net);
    return rc;
  }
  *out = net;
  return ACE_OK;
}

int convnet_destroy(ace_convnet* net) {
  if (!net) return ACE_OK;
  (void)hipStreamSynchronize(net->stream);
  for (float* b : {net->w, net->weff, net->m, net->v, net->grad})
    if (b) (void)hipFree(b);
  if (net->pk) (void)hipFree(net->pk);
  if (net->loss) (void)hipFree(net->loss);
  for (Buf* b : {&net->a1, &net->a2, &net->g, &net->g2, &net->g1, &net->part,
                 &net->lpart, &net->xb, &net->tb, &net->lhist})
    if (b->p) (void)hipFree(b->p);
  delete net;
  return ACE_OK;
}

int convnet_set_params(ace_convnet* net, const float* params) {
  if (!net || !params) return ACE_ERR_INVALID;
  hipStream_t s = net->stream;
  if (hipStreamSynchronize(s) != hipSuccess ||
      hipMemcpy(net->w, params, NPAR * sizeof(float), hipMemcpyHostToDevice) != hipSuccess)
    return ACE_ERR_HIP;
  std::vector<float> zero(NPAR, 0.f);
  if (hipMemcpy(net->m, zero.data(), NPAR * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(net->v, zero.data(), NPAR * sizeof(float), hipMemcpyHostToDevice) != hipSuccess)
    return ACE_ERR_HIP;
  net->t = 0;
  k_round_params<<<(NPAR + kT - 1) / kT, kT, 0, s>>>(net->w, NPAR, net->weff);
  pack(net);
  if (hipStreamSynchronize(s) != hipSuccess) return ACE_ERR_HIP;
  return hip_check(hipGetLastError());
}

int convnet_get_params(ace_convnet* net, float* params, int rounded) {
  if (!net || !params) return ACE_ERR_INVALID;
  if (hipStreamSynchronize(net->stream) != hipSuccess ||
      hipMemcpy(params, rounded ? net->weff : net->w, NPAR * sizeof(float),
                hipMemcpyDeviceToHost) != hipSuccess)
    return ACE_ERR_HIP;
  return ACE_OK;
}

int convnet_forward(ace_convnet* net, int n, const float* x, int nb, float* y) {
  if (!net || !x || !y || n < 1 || nb < 1) return ACE_ERR_INVALID;
  int rc = net_ensure(net, n, nb, false);
  if (rc) return rc;
  forward(net, n, x, nb, y);
  return hip_check(hipGetLastError());
}

int convnet_gradient(ace_convnet* net, int n, const float* x, const float* t, int nb,
                     double* loss, float* grad) {
  if (!net || !x || !t || n < 1 || nb < 1) return ACE_ERR_INVALID;
  int rc = net_ensure(net, n, nb, true);
  if (rc) return rc;
  gradient(net, n, x, t, nb);
  if (hipGetLastError() != hipSuccess || hipStreamSynchronize(net->stream) != hipSuccess)
    return ACE_ERR_HIP;
  if (loss && hipMemcpy(loss, net->loss, sizeof(double), hipMemcpyDeviceToHost) != hipSuccess)
    return ACE_ERR_HIP;
  if (grad && hipMemcpy(grad, net->grad, NPAR * sizeof(float), hipMemcpyDeviceToHost) != hipSuccess)
    return ACE_ERR_HIP;
  return ACE_OK;
}

int convnet_train(ace_convnet* net, int n, const float* inputs, const float* targets, int count,
                  int steps, int batch, double lr, unsigned long long seed, int flags,
                  double* loss_hist) {
  if (!net || !inputs || !targets || n < 1 || count < 1 || steps < 1 || batch < 1 ||
      !(lr > 0.0))
    return ACE_ERR_INVALID;
  const bool random = (flags & ACE_TRAIN_RANDOM) != 0;
  if (!random && batch != count) return ACE_ERR_INVALID;
  const size_t ng = (size_t)n * n * n;
  hipStream_t s = net->stream;
  int rc = net_ensure(net, n, batch, true);
  if (!rc) rc = ensure_on(s, net->xb, sizeof(float) * ng * batch);
  if (!rc) rc = ensure_on(s, net->tb, sizeof(float) * ng * batch);
  if (!rc) rc = ensure_on(s, net->lhist, sizeof(double) * steps);
  if (rc) return rc;
  double* lh = (double*)net->lhist.p;
  for (int st = 0; st < steps; ++st) {
    const float* xb = inputs;
    const float* tb = targets;
    if (random) {
      dim3 g((unsigned)std::min<size_t>(1024, (ng + kT - 1) / kT), batch);
      k_gather<<<g, kT, 0, s>>>(inputs, targets, count, ng, seed, net->t, batch, 1,
                                (float*)net->xb.p, (float*)net->tb.p);
      xb = (const float*)net->xb.p;
      tb = (const float*)net->tb.p;
    }
    gradient(net, n, xb, tb, batch);
    if (hipMemcpyAsync(lh + st, net->loss, sizeof(double), hipMemcpyDeviceToDevice, s) != hipSuccess)
      return ACE_ERR_HIP;
    adam(net, lr);
  }
  if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess) return ACE_ERR_HIP;
  if (loss_hist &&
      hipMemcpy(loss_hist, lh, sizeof(double) * steps, hipMemcpyDeviceToHost) != hipSuccess)
    return ACE_ERR_HIP;
  return ACE_OK;
}

}  // extern "C"
