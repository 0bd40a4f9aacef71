// Shared pieces of the pair-Poisson passes (poisson.hip: one launch sequence per system or
// box edge; poisson_queue.hip: persistent passes over many systems of any edges): launch
// geometry, LDS layout, the pair resolvers and the per-plane bodies of the three passes.
// The bodies compute every item the same way whatever the launch shape, so the two files' 
// kernels give the same bits.
#pragma once

#include "common.hpp"
#include "fftplan.hpp"
#include "internal.hpp"

namespace ace {

namespace {


// threads of the z passes.  Each pass has a phase of N * P2 items (one per column and
// second-factor index) and one of N * P1 items.  From edge 32 on, the z-forward pass takes one
// thread per item of its N * P2 phase and the z-inverse pass one per item of its N * P1 phase
// (rounded up to whole wavefronts, at most 1024), so neither pass runs a partly filled extra
// round; smaller edges use 256.  (Measured at 48^3 against 256 threads for both: z-forward
// 16.8 -> 14.9 us with 576, z-inverse 17.1 -> 15.9 us with 384.)  The z-forward pass at edge
// 56 keeps 512 threads: 832 (13 wavefronts, two workgroups per CU) was 1.5x slower.
constexpr int z_round(int t) { return ((t + 63) / 64) * 64 > 1024 ? 1024 : ((t + 63) / 64) * 64; }
template <int N>
constexpr int zf_threads() {
  return N == 56 ? 512 : (N >= 32 ? z_round(N * Plan<N>::P2) : 256);
}
template <int N>
constexpr int zi_threads() {
  return N >= 32 ? z_round(N * Plan<N>::P1) : 256;
}
// threads of the one-system XY pass (one P x P plane per workgroup): 512 where the phases are
// small (FP32 up to edge 40, FP64 up to 32), else 1024 -- measured per edge with the planes of
// a few dozen transforms (edge 32: 28.6 against 34.5 us, edge 40: 59.0 against 62.8 us, edge 48:
// 77.6 against 71.1 us for 512 against 1024 threads); every shape gives the same bits.
#ifndef ACE_XY_THREADS
#define ACE_XY_THREADS 0
#endif
template <typename T, int N>
constexpr int xy_threads() {
  return ACE_XY_THREADS > 0 ? ACE_XY_THREADS : (N <= (sizeof(T) == 4 ? 40 : 32) ? 512 : 1024);
}

template <typename T>
__device__ __forceinline__ C2<T>* lds() {
  extern __shared__ __align__(16) unsigned char ace_smem[];
  return reinterpret_cast<C2<T>*>(ace_smem);
}

// Table twiddles in LDS, behind the pass's `elems` complex values (those start at LDS address 0,
// so that their accesses need no base: in front of them the table cost the XY pass 4 %).  A lane that works second-factor
// index n2 needs exp(-2 pi i n2 k1 / P) for every k1.  Two layouts:
//   plain  the P entries exp(-2 pi i m / P), read at m = n2 k1;
//   rows   [n2][k1] (P1 P2 = P entries; rows padded by one entry, which spreads them over the
//          banks where the lanes of a wavefront hold different n2): one address per item
//          instead of an index product per k1.
// Rows take 8 % of the XY pass's vector instructions away at edge 64, where a wavefront of the
// column phases holds a single n2 (halves form, 68 FP32 transforms: 321 -> 311 us, 18 FP64 ones:
// 180 -> 177 us).  At the other edges it holds two or three, the row reads wait longer on LDS
// than the instructions they save, and the plain table is as fast or faster (FP32: edge 56 116
// against 119 us for 33 transforms, edge 48 58.8 against 59.6 us for 32).
template <typename T, int N>
struct TwLds {
  static constexpr int P = Plan<N>::P, P1 = Plan<N>::P1, P2 = Plan<N>::P2;
  static constexpr bool rows = P2 == 16;
  static constexpr int S = P1 + 1;  // entries per row
  static constexpr size_t bytes =
      ((rows ? (size_t)P2 * S : (size_t)P) * sizeof(TwE<T>) + 15) / 16 * 16;
};

template <typename T>
constexpr size_t tw_offset(size_t elems) {
  return (elems * sizeof(C2<T>) + 15) / 16 * 16;
}
// LDS bytes of `elems` complex values and the twiddle table.
template <typename T, int N>
constexpr size_t lds_with_twiddles(size_t elems) {
  return tw_offset<T>(elems) + TwLds<T, N>::bytes;
}

// Fill the LDS table from the global one (exp(-2 pi i m / P), m < P).
template <typename T, int N>
__device__ __forceinline__ const TwE<T>* stage_twiddles(C2<T>* base, size_t elems,
                                                        const TwE<T>* __restrict__ tw) {
  typedef TwLds<T, N> L;
  TwE<T>* s = reinterpret_cast<TwE<T>*>(reinterpret_cast<unsigned char*>(base) +
                                        tw_offset<T>(elems));
  for (int m = threadIdx.x; m < L::P; m += blockDim.x) {
    if constexpr (L::rows)
      s[m / L::P1 * L::S + m % L::P1] = tw[(m / L::P1) * (m % L::P1)];
    else
      s[m] = tw[m];
  }
  return s;
}

// exp(-2 pi i n2 k1 / P) from the LDS table
template <typename T, int N>
__device__ __forceinline__ TwE<T> tw_at(const TwE<T>* tw, int n2, int k1) {
  return tw[TwLds<T, N>::rows ? n2 * TwLds<T, N>::S + k1 : n2 * k1];
}

// ---------------------------------------------------------------------------------------
// Where pair q's two orbitals and its output volume live.  PairsByIndex: one pair list of
// (j, i) indices into two orbital arrays and a contiguous output array (one system);
// PairsByPointer: explicit pointers per pair (many systems batched into one launch).
// The indices are clamped to [0, na) and [0, nb) so that no access leaves the orbital arrays
// (a list that the host did not check); an index out of range is recorded in the status word
// (ACE_ERR_INVALID = -1, info = the pair), once.
struct PairsByIndex {
  const void* pa;
  const void* pb;
  const int* pairs;
  void* vout;
  int np;
  int na, nb;
  int* status;
  __device__ __forceinline__ int clamp_index(int j, int lim, int q) const {
    if (j >= 0 && j < lim) return j;
    if (status && atomicCAS(status, 0, -1) == 0) status[1] = q;
    return j < 0 ? 0 : lim - 1;
  }
  template <typename E>
  __device__ __forceinline__ const E* a(int q, size_t ng) const {
    return reinterpret_cast<const E*>(pa) + (size_t)clamp_index(pairs[2 * q], na, q) * ng;
  }
  template <typename E>
  __device__ __forceinline__ const E* b(int q, size_t ng) const {
    return reinterpret_cast<const E*>(pb) + (size_t)clamp_index(pairs[2 * q + 1], nb, q) * ng;
  }
  template <typename E>
  __device__ __forceinline__ E* v(int q, size_t ng) const {
    return reinterpret_cast<E*>(vout) + (size_t)q * ng;
  }
  __device__ __forceinline__ int kind(int) const { return 0; }
  template <typename E>
  __device__ __forceinline__ E* v2(int, size_t) const { return nullptr; }
};

// Complex transforms of one system from 4 ints each (a, b, out0, out1); see launch_pair_slots.
struct SlotsByIndex {
  const void* pa;
  const int* slots;
  void* vout;
  int np;
  template <typename E>
  __device__ __forceinline__ const E* a(int q, size_t ng) const {
    return reinterpret_cast<const E*>(pa) + (size_t)slots[4 * q] * ng;
  }
  template <typename E>
  __device__ __forceinline__ const E* b(int q, size_t ng) const {
    return reinterpret_cast<const E*>(pa) + (size_t)slots[4 * q + 1] * ng;
  }
  template <typename E>
  __device__ __forceinline__ E* v(int q, size_t ng) const {
    return reinterpret_cast<E*>(vout) + (size_t)slots[4 * q + 2] * ng;
  }
  __device__ __forceinline__ int kind(int q) const {
    const int o1 = slots[4 * q + 3];
    return o1 == -1 ? 0 : (o1 == -2 ? 2 : 1);
  }
  template <typename E>
  __device__ __forceinline__ E* v2(int q, size_t ng) const {
    return reinterpret_cast<E*>(vout) + (size_t)slots[4 * q + 3] * ng;
  }
};

struct PairsByPointer {
  const PairPtrs* items;
  int np;
  template <typename E>
  __device__ __forceinline__ const E* a(int q, size_t) const {
    return reinterpret_cast<const E*>(items[q].a);
  }
  template <typename E>
  __device__ __forceinline__ const E* b(int q, size_t) const {
    return reinterpret_cast<const E*>(items[q].b);
  }
  template <typename E>
  __device__ __forceinline__ E* v(int q, size_t) const {
    return reinterpret_cast<E*>(items[q].v);
  }
  __device__ __forceinline__ int kind(int q) const { return items[q].kind; }
  template <typename E>
  __device__ __forceinline__ E* v2(int q, size_t) const {
    return reinterpret_cast<E*>(items[q].v2);
  }
};

// ---------------------------------------------------------------------------------------
// Z-forward pass body: x-plane x of transform p of the resolver res (its pair density formed
// on the fly), pruned FFT along z, written transposed into this transform's work volume wp
// [qz][x][y].  buf: N (P+1) complex values of LDS; tw: the twiddle table in LDS.
template <typename T, int N, bool RP, typename R>
__device__ __forceinline__ void zfwd_plane(const R& res, int p, int x, C2<T>* __restrict__ wp,
                                           const TwE<T>* __restrict__ tw,
                                           C2<T>* __restrict__ buf, int tid, int nt) {
  typedef Plan<N> PL;
  constexpr int P = PL::P, P1 = PL::P1, P2 = PL::P2, H1 = PL::H1, RS = P + 1;
  constexpr size_t NG = (size_t)N * N * N;
  const size_t plane = (size_t)x * N * N;

  const C2<T>* ca = nullptr;
  const C2<T>* cb = nullptr;
  const T *ra0 = nullptr, *rb0 = nullptr, *ra1 = nullptr, *rb1 = nullptr;
  // complex mode: 0 pair density, 1 two real densities |a|^2 + i |b|^2, 2 one real density
  const int kd = RP ? 0 : res.kind(p);
  if constexpr (RP) {
    const int q0 = 2 * p, q1 = 2 * p + 1;
    ra0 = res.template a<T>(q0, NG) + plane;
    rb0 = res.template b<T>(q0, NG) + plane;
    if (q1 < res.np) {
      ra1 = res.template a<T>(q1, NG) + plane;
      rb1 = res.template b<T>(q1, NG) + plane;
    }
  } else {
    ca = res.template a<C2<T>>(p, NG) + plane;
    cb = res.template b<C2<T>>(p, NG) + plane;
  }

  for (int it = tid; it < N * P2; it += nt) {
    const int n2 = it % P2, y = it / P2;
    C2<T> v[P1];
#pragma unroll
    for (int n1 = 0; n1 < H1; ++n1) {
      const int idx = y * N + n1 * P2 + n2;
      if constexpr (RP) {
        v[n1].r = ra0[idx] * rb0[idx];
        v[n1].i = ra1 ? ra1[idx] * rb1[idx] : T(0);
      } else {
        // both orbitals are loaded for every kind (b = a for kind 2) and the kind selects the
        // result, so the loads stay unconditional and issue back to back
        const C2<T> xa = ca[idx], xb = cb[idx];
        const C2<T> pd = cmulc(xa, xb);
        const T da = xa.r * xa.r + xa.i * xa.i, db = xb.r * xb.r + xb.i * xb.i;
        v[n1].r = kd == 0 ? pd.r : da;
        v[n1].i = kd == 0 ? pd.i : (kd == 1 ? db : T(0));
      }
    }
    dft_in_half<T, P1, -1>(v);
    buf[y * RS + n2] = v[0];
#pragma unroll
    for (int k1 = 1; k1 < P1; ++k1)
      buf[y * RS + k1 * P2 + n2] = tw_mul(v[k1], tw_at<T, N>(tw, n2, k1));
  }
  __syncthreads();
  C2<T>* dst0 = wp + (size_t)x * N;
  for (int it = tid; it < N * P1; it += nt) {
    const int y = it % N, k1 = it / N;
    C2<T> v[P2];
#pragma unroll
    for (int k2 = 0; k2 < P2; ++k2) v[k2] = buf[y * RS + k1 * P2 + k2];
    dft<T, P2, -1>(v);
#pragma unroll
    for (int k2 = 0; k2 < P2; ++k2) dst0[(size_t)(k1 * P2 + k2) * N * N + y] = v[k2];
  }
}

// ---------------------------------------------------------------------------------------
// XY pass body: K consecutive qz planes of one transform, each a whole P x P plane in LDS
// (plane j at pl + j P (P+1)), worked by nt threads (tid = this thread).  g: the first
// plane's N x N slice (planes g_stride elements apart), gz: its kernel spectrum in position
// order [qx][qy] (planes P^2 apart), tw: the twiddle table in LDS.  Every item of a phase
// is computed the same way whatever K and nt are, so all launch shapes give the same bits.
template <typename T, int N, int K>
__device__ __forceinline__ void xy_planes(C2<T>* __restrict__ g, size_t g_stride,
                                          const T* __restrict__ gz, C2<T>* __restrict__ pl,
                                          const TwE<T>* __restrict__ tw, int tid, int nt) {
  typedef Plan<N> PL;
  constexpr int P = PL::P, P1 = PL::P1, P2 = PL::P2, H1 = PL::H1, RS = P + 1;
  constexpr int PS = P * RS;  // LDS elements per plane
  // Phases 1 and 7 give each wavefront about 64 / P2 rows of P2 consecutive elements.  With
  // the row stride P + 1, consecutive rows start one bank pair apart and their elements fall
  // on the same LDS banks; so item group q takes row x = (q mod XS) N / XS + q div XS, rows
  // N / XS apart (edge 48: 58.0-58.5 against 58.9-59.4 us).  Only the assignment of items to
  // threads changes, not what an item computes.  (The z passes' LDS phases have the same
  // pattern, but spreading their rows measured no faster.)
  constexpr int XS = N % 4 == 0 ? 4 : 1;
  // 1. y forward, first factor (rows x < N, input y < N): global -> LDS
  for (int it = tid; it < K * N * P2; it += nt) {
    const int j = it / (N * P2), r = it - j * (N * P2);
    const int n2 = r % P2, q = r / P2, x = (q % XS) * (N / XS) + q / XS;
    const C2<T>* gj = g + j * g_stride;
    C2<T>* pj = pl + j * PS;
    C2<T> v[P1];
#pragma unroll
    for (int n1 = 0; n1 < H1; ++n1) v[n1] = gj[x * N + n1 * P2 + n2];
    dft_in_half<T, P1, -1>(v);
    pj[x * RS + n2] = v[0];
#pragma unroll
    for (int k1 = 1; k1 < P1; ++k1)
      pj[x * RS + k1 * P2 + n2] = tw_mul(v[k1], tw_at<T, N>(tw, n2, k1));
  }
  __syncthreads();
  // 2. y forward, second factor
  for (int it = tid; it < K * N * P1; it += nt) {
    const int j = it / (N * P1), r = it - j * (N * P1);
    const int x = r % N, k1 = r / N;
    C2<T> v[P2];
    C2<T>* row = pl + j * PS + x * RS + k1 * P2;
#pragma unroll
    for (int k2 = 0; k2 < P2; ++k2) v[k2] = row[k2];
    dft<T, P2, -1>(v);
#pragma unroll
    for (int k2 = 0; k2 < P2; ++k2) row[k2] = v[k2];
  }
  __syncthreads();
  // 3. x forward, first factor (columns qy, input x < N)
  for (int it = tid; it < K * P * P2; it += nt) {
    const int j = it / (P * P2), r = it - j * (P * P2);
    const int qy = r % P, n2 = r / P;
    C2<T>* pj = pl + j * PS;
    C2<T> v[P1];
#pragma unroll
    for (int n1 = 0; n1 < H1; ++n1) v[n1] = pj[(n1 * P2 + n2) * RS + qy];
    dft_in_half<T, P1, -1>(v);
    pj[n2 * RS + qy] = v[0];
#pragma unroll
    for (int k1 = 1; k1 < P1; ++k1)
      pj[(k1 * P2 + n2) * RS + qy] = tw_mul(v[k1], tw_at<T, N>(tw, n2, k1));
  }
  // the kernel spectrum values of this thread's first phase-4 item are requested before the
  // barrier, so that their latency overlaps the wait and the phase's LDS reads
  T gpre[P2];
  if (tid < K * P * P1) {
    const int j = tid / (P * P1), r = tid - j * (P * P1);
    const int qy = r % P, k1 = r / P;
    const T* gj = gz + (size_t)j * P * P;
#pragma unroll
    for (int k2 = 0; k2 < P2; ++k2) gpre[k2] = gj[(k1 * P2 + k2) * P + qy];
  }
  __syncthreads();
  // 4. x forward second factor, kernel multiply, x inverse first factor (in registers)
  for (int it = tid; it < K * P * P1; it += nt) {
    const int j = it / (P * P1), r = it - j * (P * P1);
    const int qy = r % P, k1 = r / P;
    C2<T>* pj = pl + j * PS;
    const T* gj = gz + (size_t)j * P * P;
    C2<T> v[P2];
#pragma unroll
    for (int k2 = 0; k2 < P2; ++k2) v[k2] = pj[(k1 * P2 + k2) * RS + qy];
    if (it != tid) {
#pragma unroll
      for (int k2 = 0; k2 < P2; ++k2) gpre[k2] = gj[(k1 * P2 + k2) * P + qy];
    }
    dft<T, P2, -1>(v);
#pragma unroll
    for (int k2 = 0; k2 < P2; ++k2) v[k2] = cscale(v[k2], gpre[k2]);
    dft<T, P2, 1>(v);
#pragma unroll
    for (int k2 = 0; k2 < P2; ++k2) pj[(k1 * P2 + k2) * RS + qy] = v[k2];
  }
  __syncthreads();
  // 5. x inverse, second factor, output x < N only
  for (int it = tid; it < K * P * P2; it += nt) {
    const int j = it / (P * P2), r = it - j * (P * P2);
    const int qy = r % P, n2 = r / P;
    C2<T>* pj = pl + j * PS;
    C2<T> v[P1];
    v[0] = pj[n2 * RS + qy];
#pragma unroll
    for (int k1 = 1; k1 < P1; ++k1)
      v[k1] = tw_mul_conj(pj[(k1 * P2 + n2) * RS + qy], tw_at<T, N>(tw, n2, k1));
    dft_out_half<T, P1, 1>(v);
#pragma unroll
    for (int n1 = 0; n1 < H1; ++n1) pj[(n1 * P2 + n2) * RS + qy] = v[n1];
  }
  __syncthreads();
  // 6. y inverse, first factor (rows x < N)
  for (int it = tid; it < K * N * P1; it += nt) {
    const int j = it / (N * P1), r = it - j * (N * P1);
    const int x = r % N, k1 = r / N;
    C2<T> v[P2];
    C2<T>* row = pl + j * PS + x * RS + k1 * P2;
#pragma unroll
    for (int k2 = 0; k2 < P2; ++k2) v[k2] = row[k2];
    dft<T, P2, 1>(v);
#pragma unroll
    for (int k2 = 0; k2 < P2; ++k2) row[k2] = v[k2];
  }
  __syncthreads();
  // 7. y inverse, second factor, output y < N: LDS -> global (in place over the input slice)
  for (int it = tid; it < K * N * P2; it += nt) {
    const int j = it / (N * P2), r = it - j * (N * P2);
    const int n2 = r % P2, q = r / P2, x = (q % XS) * (N / XS) + q / XS;
    C2<T>* gj = g + j * g_stride;
    C2<T>* pj = pl + j * PS;
    C2<T> v[P1];
    v[0] = pj[x * RS + n2];
#pragma unroll
    for (int k1 = 1; k1 < P1; ++k1)
      v[k1] = tw_mul_conj(pj[x * RS + k1 * P2 + n2], tw_at<T, N>(tw, n2, k1));
    dft_out_half<T, P1, 1>(v);
#pragma unroll
    for (int n1 = 0; n1 < H1; ++n1) gj[x * N + n1 * P2 + n2] = v[n1];
  }
}

// ---------------------------------------------------------------------------------------
// Z-inverse pass body: x-plane x of transform p, read from its work volume wp [qz][x][y],
// inverse FFT along z keeping z < N, written to the resolver's output volume(s).
template <typename T, int N, bool RP, typename R>
__device__ __forceinline__ void zinv_plane(const C2<T>* __restrict__ wp, const R& res, int p,
                                           int x, const TwE<T>* __restrict__ tw,
                                           C2<T>* __restrict__ buf, int tid, int nt) {
  typedef Plan<N> PL;
  constexpr int P = PL::P, P1 = PL::P1, P2 = PL::P2, H1 = PL::H1, RS = P + 1;
  constexpr size_t NG = (size_t)N * N * N;
  const C2<T>* src0 = wp + (size_t)x * N;
  for (int it = tid; it < N * P1; it += nt) {
    const int y = it % N, k1 = it / N;
    C2<T> v[P2];
#pragma unroll
    for (int k2 = 0; k2 < P2; ++k2) v[k2] = src0[(size_t)(k1 * P2 + k2) * N * N + y];
    dft<T, P2, 1>(v);
#pragma unroll
    for (int k2 = 0; k2 < P2; ++k2) buf[y * RS + k1 * P2 + k2] = v[k2];
  }
  __syncthreads();
  for (int it = tid; it < N * P2; it += nt) {
    const int n2 = it % P2, y = it / P2;
    C2<T> v[P1];
    v[0] = buf[y * RS + n2];
#pragma unroll
    for (int k1 = 1; k1 < P1; ++k1)
      v[k1] = tw_mul_conj(buf[y * RS + k1 * P2 + n2], tw_at<T, N>(tw, n2, k1));
    dft_out_half<T, P1, 1>(v);
    const size_t base = ((size_t)x * N + y) * N + n2;
    if constexpr (RP) {
      T* o0 = res.template v<T>(2 * p, NG) + base;
      const bool has1 = (2 * p + 1) < res.np;
#pragma unroll
      for (int n1 = 0; n1 < H1; ++n1) o0[n1 * P2] = v[n1].r;
      if (has1) {
        T* o1 = res.template v<T>(2 * p + 1, NG) + base;
#pragma unroll
        for (int n1 = 0; n1 < H1; ++n1) o1[n1 * P2] = v[n1].i;
      }
    } else {
      const int kd = res.kind(p);
      C2<T>* o = res.template v<C2<T>>(p, NG) + base;
      if (kd == 0) {
#pragma unroll
        for (int n1 = 0; n1 < H1; ++n1) o[n1 * P2] = v[n1];
      } else {
        // real densities: the two potentials are the real and imaginary parts
#pragma unroll
        for (int n1 = 0; n1 < H1; ++n1) o[n1 * P2] = C2<T>{v[n1].r, T(0)};
        if (kd == 1) {
          C2<T>* o1 = res.template v2<C2<T>>(p, NG) + base;
#pragma unroll
          for (int n1 = 0; n1 < H1; ++n1) o1[n1 * P2] = C2<T>{v[n1].i, T(0)};
        }
      }
    }
  }
}

template <typename K>
void allow_lds(K kernel, size_t bytes) {
  if (bytes > 65536) (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                         (int)bytes);
}

constexpr size_t kMaxLds = 160 * 1024;

// LDS elements and bytes of the passes: an x-plane of a z pass, K whole P x P planes of the XY
// pass, or one of its planes by halves (P x N).
template <int N>
constexpr size_t z_elems() {
  return (size_t)N * (2 * N + 1);
}
template <int N>
constexpr size_t planes_elems(int k = 1) {
  return (size_t)k * (2 * N) * (2 * N + 1);
}
template <int N>
constexpr size_t halves_elems() {
  return (size_t)(2 * N) * (N + 1);
}
template <typename T, int N>
constexpr size_t z_lds() {
  return lds_with_twiddles<T, N>(z_elems<N>());
}
template <typename T, int N>
constexpr size_t planes_lds(int k = 1) {
  return lds_with_twiddles<T, N>(planes_elems<N>(k));
}
template <typename T, int N>
constexpr size_t halves_lds() {
  return lds_with_twiddles<T, N>(halves_elems<N>());
}

// the whole P x P plane of the XY pass fits in LDS
template <typename T, int N>
constexpr bool fits() {
  return planes_lds<T, N>() <= kMaxLds;
}

// the pair-Poisson passes are compiled for this edge and precision
template <typename T, int N>
constexpr bool supported() {
  return fits<T, N>() || halves_lds<T, N>() <= kMaxLds;
}

// Whether the one-system XY pass (and the per-edge form of the batch) works its planes by
// halves, its threads, and the wavefronts per SIMD its registers must allow.  By halves wherever
// the whole plane leaves one workgroup per CU, whose barriers then stop every wavefront of the
// CU at once (or does not fit at all); where two or more whole planes fit, halving only adds
// barriers.  Measured, whole plane -> halves, us per launch of the stated transforms:
//   FP32  edge 64 (68) 357 -> 311, edge 56 (33) 132 -> 115, edge 48 (32) 58.8 -> 65.6,
//         edge 40 (64) 72 -> 75;
//   FP64  edge 48 (32) 119 -> 114, edge 40 (32) 86 -> 77, edge 32 (32) 35.0 -> 41;
//         edges 64 and 56 (18), against x transforms over strips of 8 and 28 columns beside
//         the N whole rows: 375 -> 177 and 160 -> 141.
// Vector instructions issue in 90 and 87 % of the slots at edges 56 and 64 in FP32 (78 % at 64 in
// whole planes), but in 37 to 43 % in FP64, where two workgroups of 8 wavefronts per CU (one at 56
// and 64) do not cover the LDS reads and barriers.
// 512 threads: 256 and 768 are slower (FP32 edge 64: 346 and 421 us) except FP64 at edge 56,
// where 768 threads take 14 items of each column in whole rounds (153 -> 141 us).
template <typename T, int N>
constexpr bool by_halves() {
  return N >= (sizeof(T) == 4 ? 56 : 40);
}
// But launches of at most one plane per CU have a CU's LDS for each plane either way, and the whole
// plane is worked by twice the threads with half the barriers.  XY pass, halves -> whole plane, us:
// FP32 edge 64, 1 and 2 transforms 13.5 -> 10.8 and 15.4 -> 13.5, edge 56 14.3 -> 10.1 and 16.0 ->
// 12.4; FP64 edge 48 14.0 -> 10.8 and 15.7 -> 13.0, edge 40, 3 transforms (240 planes), 13.6 -> 11.5.
// From the next transform on the halves are as fast or faster (edge 40, 4: 18.2 against 18.9).
template <typename T, int N>
bool by_halves(int transforms) {
  if constexpr (!by_halves<T, N>()) return false;
  return !fits<T, N>() || (long long)transforms * 2 * N > device_cus();
}
template <typename T, int N>
constexpr int halves_threads() {
  return sizeof(T) == 8 && N == 56 ? 768 : 512;
}
template <typename T, int N>
constexpr int halves_waves() {
  return sizeof(T) == 4 ? (N == 56 ? 6 : 4) : (N <= 48 ? 4 : (N == 56 ? 3 : 2));
}

// XY pass of one qz plane in two halves of its y frequencies: the positions k1 P2 + k2 with k1
// even, then those with k1 odd (N columns each).  The even and the odd k1 are the two DFTs that
// dft_in_half / dft_out_half run separately anyway, so each half is complete by itself up to
// the last sum of the y inverse (even part + twiddled odd part), for which the even part waits
// in registers.  Every value is computed as in xy_planes.  LDS holds P x N values instead of
// P x P, in place: row q, column c = (k1 / 2) P2 + k2 at pl[q (N + 1) + c].
template <typename T, int N, int NT>
__device__ __forceinline__ void xy_halves(C2<T>* __restrict__ g, const T* __restrict__ gz,
                                          C2<T>* __restrict__ pl, const TwE<T>* __restrict__ tw,
                                          int tid) {
  typedef Plan<N> PL;
  constexpr int P = PL::P, P1 = PL::P1, P2 = PL::P2, H1 = PL::H1, RS = N + 1;
  constexpr int XS = N % 4 == 0 ? 4 : 1;      // row order of phases 1 and 7, see xy_planes
  constexpr int IT = (N * P2 + NT - 1) / NT;  // phase-1 / phase-7 items per thread
  C2<T> even[IT][H1];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    // 1. y forward, first factor (rows x < N, input y < N), k1 = 2 m + e: global -> LDS
#pragma unroll
    for (int u = 0; u < IT; ++u) {
      const int it = tid + u * NT;
      if (N * P2 % NT == 0 || it < N * P2) {
        const int n2 = it % P2, q = it / P2, x = (q % XS) * (N / XS) + q / XS;
        C2<T> v[H1];
#pragma unroll
        for (int n1 = 0; n1 < H1; ++n1) v[n1] = g[x * N + n1 * P2 + n2];
        if (e == 1) {
#pragma unroll
          for (int m = 0; m < H1; ++m) v[m] = twk<T, P1, -1>(v[m], m);
        }
        dft<T, H1, -1>(v);
#pragma unroll
        for (int m = 0; m < H1; ++m)
          pl[x * RS + m * P2 + n2] = 2 * m + e == 0 ? v[0] : tw_mul(v[m], tw_at<T, N>(tw, n2, 2 * m + e));
      }
    }
    __syncthreads();
    // 2. y forward, second factor
    for (int it = tid; it < N * H1; it += NT) {
      const int x = it % N, m = it / N;
      C2<T> v[P2];
      C2<T>* row = pl + x * RS + m * P2;
#pragma unroll
      for (int k2 = 0; k2 < P2; ++k2) v[k2] = row[k2];
      dft<T, P2, -1>(v);
#pragma unroll
      for (int k2 = 0; k2 < P2; ++k2) row[k2] = v[k2];
    }
    __syncthreads();
    // 3. x forward, first factor (N columns, input x < N)
    for (int it = tid; it < N * P2; it += NT) {
      const int c = it % N, n2 = it / N;
      C2<T> v[P1];
#pragma unroll
      for (int n1 = 0; n1 < H1; ++n1) v[n1] = pl[(n1 * P2 + n2) * RS + c];
      dft_in_half<T, P1, -1>(v);
      pl[n2 * RS + c] = v[0];
#pragma unroll
      for (int k1 = 1; k1 < P1; ++k1)
        pl[(k1 * P2 + n2) * RS + c] = tw_mul(v[k1], tw_at<T, N>(tw, n2, k1));
    }
    // the kernel spectrum of this thread's first phase-4 item, requested before the barrier
    T gpre[P2];
    if (NT == N * P1 || tid < N * P1) {
      const int c = tid % N, k1 = tid / N, qy = (2 * (c / P2) + e) * P2 + c % P2;
#pragma unroll
      for (int k2 = 0; k2 < P2; ++k2) gpre[k2] = gz[(k1 * P2 + k2) * P + qy];
    }
    __syncthreads();
    // 4. x forward second factor, kernel multiply, x inverse first factor (in registers)
    auto column = [&](int it, bool first) {
      const int c = it % N, k1 = it / N;
      C2<T> v[P2];
#pragma unroll
      for (int k2 = 0; k2 < P2; ++k2) v[k2] = pl[(k1 * P2 + k2) * RS + c];
      if (!first) {
        const int qy = (2 * (c / P2) + e) * P2 + c % P2;
#pragma unroll
        for (int k2 = 0; k2 < P2; ++k2) gpre[k2] = gz[(k1 * P2 + k2) * P + qy];
      }
      dft<T, P2, -1>(v);
#pragma unroll
      for (int k2 = 0; k2 < P2; ++k2) v[k2] = cscale(v[k2], gpre[k2]);
      dft<T, P2, 1>(v);
#pragma unroll
      for (int k2 = 0; k2 < P2; ++k2) pl[(k1 * P2 + k2) * RS + c] = v[k2];
    };
    if constexpr (N * P1 == NT) {
      column(tid, true);
    } else {
      for (int it = tid; it < N * P1; it += NT) column(it, it == tid);
    }
    __syncthreads();
    // 5. x inverse, second factor, output x < N only
    for (int it = tid; it < N * P2; it += NT) {
      const int c = it % N, n2 = it / N;
      C2<T> v[P1];
      v[0] = pl[n2 * RS + c];
#pragma unroll
      for (int k1 = 1; k1 < P1; ++k1)
        v[k1] = tw_mul_conj(pl[(k1 * P2 + n2) * RS + c], tw_at<T, N>(tw, n2, k1));
      dft_out_half<T, P1, 1>(v);
#pragma unroll
      for (int n1 = 0; n1 < H1; ++n1) pl[(n1 * P2 + n2) * RS + c] = v[n1];
    }
    __syncthreads();
    // 6. y inverse, first factor (rows x < N)
    for (int it = tid; it < N * H1; it += NT) {
      const int x = it % N, m = it / N;
      C2<T> v[P2];
      C2<T>* row = pl + x * RS + m * P2;
#pragma unroll
      for (int k2 = 0; k2 < P2; ++k2) v[k2] = row[k2];
      dft<T, P2, 1>(v);
#pragma unroll
      for (int k2 = 0; k2 < P2; ++k2) row[k2] = v[k2];
    }
    __syncthreads();
    // 7. y inverse, second factor, output y < N: the even part to registers, then the sum of
    // both parts to global (in place over the input slice)
#pragma unroll
    for (int u = 0; u < IT; ++u) {
      const int it = tid + u * NT;
      if (N * P2 % NT == 0 || it < N * P2) {
        const int n2 = it % P2, q = it / P2, x = (q % XS) * (N / XS) + q / XS;
        C2<T> v[H1];
#pragma unroll
        for (int m = 0; m < H1; ++m) {
          const C2<T> a = pl[x * RS + m * P2 + n2];
          v[m] = 2 * m + e == 0 ? a : tw_mul_conj(a, tw_at<T, N>(tw, n2, 2 * m + e));
        }
        dft<T, H1, 1>(v);
        if (e == 0) {
#pragma unroll
          for (int m = 0; m < H1; ++m) even[u][m] = v[m];
        } else {
#pragma unroll
          for (int m = 0; m < H1; ++m)
            g[x * N + m * P2 + n2] = cadd(even[u][m], twk<T, P1, 1>(v[m], m));
        }
      }
    }
    if (e == 0) __syncthreads();
  }
}

#define ACE_SIZES(X) X(8) X(9) X(10) X(12) X(15) X(16) X(20) X(24) X(32) X(40) X(48) X(56) X(64)


}  // namespace

}  // namespace ace
