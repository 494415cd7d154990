// Device helpers: fixed-order workgroup reductions, the per-replicate
// "last workgroup finishes the reduction" handshake, work-item decoding and
// the Philox4x64-10 block function.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hca_internal.h"

namespace hca {

// Sum over a wavefront, in every lane, in the order of the butterfly over lane
// distances 32, 16, 8, 4, 2, 1, by register moves alone (the same butterfly by
// LDS permutes takes several times as long, and short kernels wait for it: on
// a 100 x 100 slice k_cg_update 5.0 -> 3.5 us, k_guess_dots with its twelve sums
// 7.8 -> 5.3).  The swaps of
// halves and of rows of 16 give each lane both addends; a rotation
// by 8 in a row of 16 is distance 8, one by 4 distance 4 once the lanes at distance 8
// hold the same value.
template <int CTRL>
__device__ inline double dpp_moved(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false),
                          __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false));
}
__device__ inline double wave_sum(double v) {
  {
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    v = __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
  }
  {
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    v = __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
  }
  v += dpp_moved<0x128>(v);   // row_ror:8
  v += dpp_moved<0x124>(v);   // row_ror:4
  v += dpp_moved<0x4e>(v);    // quad_perm:[2,3,0,1]
  v += dpp_moved<0xb1>(v);    // quad_perm:[1,0,3,2]
  return v;
}

// N sums over a 256-thread workgroup, each in a fixed order (wave_sum, then
// the four wavefront sums in index order).  Every thread returns the totals.
template <int N>
__device__ inline void block_sums(double (&v)[N], double (&lds)[4][N]) {
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = wave_sum(v[k]);
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int k = 0; k < N; ++k) lds[wave][k] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = ((lds[0][k] + lds[1][k]) + lds[2][k]) + lds[3][k];
  __syncthreads();
}

__device__ inline double block_sum(double v, double* lds4) {
  v = wave_sum(v);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) lds4[wave] = v;
  __syncthreads();
  double t = ((lds4[0] + lds4[1]) + lds4[2]) + lds4[3];
  __syncthreads();
  return t;
}

__device__ inline unsigned long long block_sum_u64(unsigned long long v,
                                                   unsigned long long* lds4) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) lds4[wave] = v;
  __syncthreads();
  unsigned long long t = lds4[0] + lds4[1] + lds4[2] + lds4[3];
  __syncthreads();
  return t;
}

__device__ inline double block_max(double v, double* lds4) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) lds4[wave] = v;
  __syncthreads();
  double t = fmax(fmax(lds4[0], lds4[1]), fmax(lds4[2], lds4[3]));
  __syncthreads();
  return t;
}

// Persistent launches: G workgroups cover T work items in contiguous chunks.
// Workgroups are dealt to the 8 XCDs round-robin, so logical block
// lb = (b % 8) * (G / 8) + b / 8 gives each XCD one contiguous run of chunks
// (neighbouring tiles, shared halos in that XCD's L2).
__device__ inline void work_range(int T, int& begin, int& end) {
  const int G = gridDim.x, b = blockIdx.x;
  const int lb = (G % 8 == 0) ? (b % 8) * (G / 8) + b / 8 : b;
  begin = (int)((long long)lb * T / G);
  end = (int)((long long)(lb + 1) * T / G);
}

// Stencil tiles: with a grid that is a multiple of 8 * kXcdChunk the tiles
// are dealt to the 8 XCDs in runs of kXcdChunk consecutive tiles, round robin
// (run k to XCD k mod 8), one tile per workgroup: neighbouring tiles share
// their frame rows in one XCD's L2 while every system's tiles still spread
// over all XCDs (systems finish at different iterations).  Otherwise as
// work_range.
__device__ inline void tile_range(int T, int& begin, int& end) {
  const int G = gridDim.x, b = blockIdx.x;
  if (G % (8 * kXcdChunk) == 0) {
    const int x = b % 8, j = b / 8;   // j-th workgroup of XCD x
    const int t = ((j / kXcdChunk) * 8 + x) * kXcdChunk + j % kXcdChunk;
    begin = min(t, T);
    end = min(t + 1, T);
    return;
  }
  work_range(T, begin, end);
}

// A workgroup's three partial sums, stored at its work-item slot (3 doubles);
// a later reduce kernel (one workgroup per replicate) sums the slots of a
// replicate in a fixed order.  The kernel boundary orders the two.
__device__ inline void store_partials(double* slot, double a, double b, double c) {
  if (threadIdx.x == 0) {
    slot[0] = a;
    slot[1] = b;
    slot[2] = c;
  }
}

// The end of system sys's solve on the voxels [off, off + len): x += G_j z_j of
// the kept iterations (CgRing) and the last iteration's x += alpha p if its z is
// not among them.  Thread t takes the voxels t + k kBlock, kPer at a time, loads
// before stores (with kept z, four at a time measured 58 us at 128^3, two 51).
template <typename T>
__device__ inline void cg_finish_span(const CgRing& ring, const T* p0, const T* p1, const SolveScal* ss, int sys,
                                      T* x, long long off, int len) {
  const int n = ss[sys].it;
  if (n == 0) return;
  constexpr bool kKeeps = sizeof(T) == 8;
  const double alpha = ss[sys].alpha;
  const int kept = kKeeps ? min(n, ring.n) : 0;
  const bool last = n > kept;   // alpha p is still to be added
  double w[kZRing];
  if constexpr (kKeeps) {
    const double* h = ring.hist + (size_t)sys * 3 * kZRing;
    double G = 0.0, beta = 0.0;   // of the iteration above
#pragma unroll
    for (int j = kZRing - 1; j >= 0; --j) {
      w[j] = 0.0;
      if (j < kept) {
        G = h[3 * j] + beta * G;
        beta = h[3 * j + 1];
        w[j] = G * h[3 * j + 2];
      }
    }
  }
  constexpr int kPer = kKeeps ? 2 : kFlatChunk / kBlock;
  const T* p = (((n - 1) & 1) ? p0 : p1) + off;   // the direction of iteration n - 1
  x += off;
  for (int l0 = (int)threadIdx.x; l0 < len; l0 += kPer * kBlock) {
    double xv[kPer], pv[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int li = l0 + k * kBlock;
      xv[k] = li < len ? (double)x[li] : 0.0;
      pv[k] = last && li < len ? (double)p[li] : 0.0;
    }
    if constexpr (kKeeps) {
      float zv[kZRing][kPer];
#pragma unroll
      for (int j = 0; j < kZRing; ++j) {
        const float* z = ring.z(j) + off;
#pragma unroll
        for (int k = 0; k < kPer; ++k) zv[j][k] = j < kept && l0 + k * kBlock < len ? z[l0 + k * kBlock] : 0.f;
      }
#pragma unroll
      for (int j = 0; j < kZRing; ++j)
        if (j < kept) {
#pragma unroll
          for (int k = 0; k < kPer; ++k) xv[k] = fma(w[j], (double)zv[j][k], xv[k]);
        }
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int li = l0 + k * kBlock;
      if (li < len) x[li] = (T)(last ? fma(alpha, pv[k], xv[k]) : xv[k]);
    }
  }
}

// A deferred solve end (CgFinish, precision 32) of every field on the voxels
// [off, off + len) of replicate rep; the caller's next barrier publishes the
// values to the rest of the workgroup.
template <typename T>
__device__ inline void cg_finish_run(const CgFinish<T>* __restrict__ finp, int rep, long long off, int len) {
  if (sizeof(T) == 8 || !finp) return;
  const CgFinish<T> fin = *finp;
  for (int f = 0; f < fin.nf; ++f)
    cg_finish_span(CgRing{}, fin.p0, fin.p1, fin.ss, f * fin.nrep + rep, fin.x, (long long)f * fin.ntot + off, len);
}

// ---- Philox4x64-10 (Salmon et al., SC'11) ----------------------------------
struct U64x4 {
  uint64_t v[4];
};

__device__ inline U64x4 philox4x64_10(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3,
                                      uint64_t k0, uint64_t k1) {
  constexpr uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
  constexpr uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += W0;
      k1 += W1;
    }
    const uint64_t lo0 = M0 * c0, hi0 = __umul64hi(M0, c0);
    const uint64_t lo1 = M1 * c2, hi1 = __umul64hi(M1, c2);
    const uint64_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0;
    c1 = lo1;
    c2 = n2;
    c3 = lo0;
  }
  U64x4 o;
  o.v[0] = c0;
  o.v[1] = c1;
  o.v[2] = c2;
  o.v[3] = c3;
  return o;
}

__device__ inline double unit53(uint64_t o) { return (double)(o >> 11) * 0x1.0p-53; }

// Moore neighbour d (0..25, ascending gid order) offsets.
__device__ inline void moore_offset(int d, int& dx, int& dy, int& dz) {
  const int e = d < 13 ? d : d + 1;   // skip the centre (13)
  dz = e / 9 - 1;
  dy = (e / 3) % 3 - 1;
  dx = e % 3 - 1;
}

__device__ inline int moore_opposite(int d) { return 25 - d; }

}  // namespace hca
