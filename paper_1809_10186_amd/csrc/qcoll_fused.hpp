// Building blocks of the on-chip kernels.  The FP32 fused kernels (N <= 32):
// one workgroup of N^2 lanes owns a whole N^3 complex volume, one pencil per
// lane, and changes the pencil axis by transposes through one LDS tile; the
// FP64 kernel shares the XCD-aware block numbering.
#pragma once
#include <hip/hip_runtime.h>

#include "qcoll_fft.hpp"
#include "qcoll_internal.h"

namespace qcoll {

// Raw buffer descriptor over [base, base + bytes): loads through it take the
// per-element stride as a scalar offset (no per-element address VGPRs) and
// return 0 outside the range instead of faulting.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, int(bytes), 0x00020000);
}

__device__ __forceinline__ cplx<float> load_c32(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  const float2 v = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
  return cplx<float>{v.x, v.y};
}

__device__ __forceinline__ cplx<double> load_c64(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  const double2 v = __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
  return cplx<double>{v.x, v.y};
}

// Words per plane of the LDS tile: at least N (N + 1) for the rows of N + 1 words
// of the B <-> C transposes, and N more than a multiple of 64, so that the
// planes that the lanes of one access span (N lanes a plane) continue each
// other's banks (1024 items at 24^3: 5.02 -> 4.65 ms, against N^2 + 32 words).
constexpr int tile_stride(int N) {
  int s = N * (N + 1);
  while (s % 64 != N % 64) ++s;
  return s;
}

template <int N>
struct FusedGeom {
  // pencils per lane (1: N^2 lanes; the loops below also support 2, which
  // halves the lane count at twice the registers per lane)
  static constexpr int PPL = 1;
  static constexpr int NL = N * N / PPL;
  static constexpr int S1 = tile_stride(N);
  // the B <-> C transposes stay inside a wave when a wave owns whole rows
  // (64 lanes = 64/N rows of N lanes, one pencil per lane)
  static constexpr bool WAVE_BC = (PPL == 1) && (64 % N == 0);
  // Below 32 the tile holds both components (N = 24: 112.5 KiB; at 32 it would
  // be 264 KiB, so there the real parts move first, then the imaginary parts).
  // With element (a, b, c) at a S1 + b (N + 1) + c throughout, a lane writes each
  // pencil where it read the one before, and a transpose costs one barrier
  // instead of the four of two components in turn.  It pays although one
  // workgroup of 24^3 then has a CU to itself: 1024 items x 4 nodes, M 6, in
  // 1029 us before (two workgroups of 57 KiB a CU), 1021 without the second,
  // 979 with both components, 878 with pencils written in place, 850 with the
  // components side by side (8-byte accesses).
  static constexpr bool BOTH = N < 32;
  static constexpr size_t lds_bytes = size_t(N) * S1 * (BOTH ? sizeof(float2) : sizeof(float));
  // waves per SIMD the register budget must allow: the 9 waves of 24^3
  static constexpr int WPE = (N == 24) ? 3 : 1;
};

// element addresses of the tile for lane (hi, lo): its pencil along the first,
// second or third index
template <int N>
struct TileAt {
  static constexpr int S1 = FusedGeom<N>::S1, R = N + 1;
  int hi, lo;
  __device__ __forceinline__ int a(int i) const { return i * S1 + hi * R + lo; }
  __device__ __forceinline__ int b(int i) const { return hi * S1 + i * R + lo; }
  __device__ __forceinline__ int c(int i) const { return hi * S1 + lo * R + i; }
};

// orders a wave's LDS writes before its reads of what its other lanes wrote
__device__ __forceinline__ void lds_wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// both components of the lane's pencil into / out of the tile
template <int N, class AT>
__device__ __forceinline__ void tile_put(float *lds, const float *zr, const float *zi, AT at) {
  float2 *l = reinterpret_cast<float2 *>(lds);
  static_for<0, N>([&](auto i) {
    l[at(decltype(i)::value)] = make_float2(zr[decltype(i)::value], zi[decltype(i)::value]);
  });
}
template <int N, class AT>
__device__ __forceinline__ void tile_get(const float *lds, float *zr, float *zi, AT at) {
  const float2 *l = reinterpret_cast<const float2 *>(lds);
  static_for<0, N>([&](auto i) {
    const float2 v = l[at(decltype(i)::value)];
    zr[decltype(i)::value] = v.x;
    zi[decltype(i)::value] = v.y;
  });
}

// move one component (re or im) of every pencil of the lane through LDS; with
// TAIL = false the barrier after the reads is left to the caller (the tile
// must not be written again before one)
template <int N, int PPL, bool TAIL = true, class WA, class RA>
__device__ __forceinline__ void lds_transpose(float *lds, float (*v)[N], WA wa, RA ra) {
  static_for<0, PPL>([&](auto u) {
    static_for<0, N>([&](auto i) {
      lds[wa(decltype(u)::value, decltype(i)::value)] = v[decltype(u)::value][decltype(i)::value];
    });
  });
  __syncthreads();
  static_for<0, PPL>([&](auto u) {
    static_for<0, N>([&](auto i) {
      v[decltype(u)::value][decltype(i)::value] = lds[ra(decltype(u)::value, decltype(i)::value)];
    });
  });
  if constexpr (TAIL) __syncthreads();
}

// Same transpose within one wave: every address a lane writes or reads lies in
// rows owned by its own wave, so ordering the wave's LDS writes before its
// reads is enough (LDS requests of one wave are served in order; the fences
// stop the compiler from moving the accesses across each other).
template <int N, int PPL, class WA, class RA>
__device__ __forceinline__ void lds_transpose_wave(float *lds, float (*v)[N], WA wa, RA ra) {
  static_for<0, PPL>([&](auto u) {
    static_for<0, N>([&](auto i) {
      lds[wa(decltype(u)::value, decltype(i)::value)] = v[decltype(u)::value][decltype(i)::value];
    });
  });
  lds_wave_order();
  static_for<0, PPL>([&](auto u) {
    static_for<0, N>([&](auto i) {
      v[decltype(u)::value][decltype(i)::value] = lds[ra(decltype(u)::value, decltype(i)::value)];
    });
  });
  lds_wave_order();
}

// XCD-aware block numbering: hardware block i runs on XCD i % 8; logical
// indices are handed out so that each XCD gets one contiguous range (the pairs
// of one item then share the item's spectrum in that XCD's L2).
__device__ __forceinline__ long xcd_block() {
  const long nb = gridDim.x;
  const long full = nb / 8, rem = nb % 8;
  const long x = blockIdx.x % 8;
  return x * full + (x < rem ? x : rem) + blockIdx.x / 8;
}

// FP64 gain loops: A_p += Re(u_q)^2 - Im(u_q)^2, q = 1..M-1, from the volumes that
// the kernels' one-term variants stored, one point per lane; with N > 0 they are laid
// out [j3][j1][j2]
template <int N>
__global__ __launch_bounds__(256) void k_gain_acc64(const double2 *__restrict__ U, double *__restrict__ A, long n3,
                                                    long nbp, int nq) {
  const long i = long(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= nbp * n3) return;
  const long bp = i / n3, o = i % n3;
  const double2 *u = U + bp * nq * n3 + o;
  long d = o;
  if constexpr (N > 0) d = (o % (N * N)) * N + o / (N * N);
  double a = A[bp * n3 + d];
#pragma unroll 6
  for (int q = 0; q < nq; ++q) {
    const double2 v = u[q * n3];
    a = __builtin_fma(v.x, v.x, a);
    a = __builtin_fma(-v.y, v.y, a);
  }
  A[bp * n3 + d] = a;
}

// the whole term loop per workgroup, or with U (nbp * (M - 1) volumes) a
// workgroup per term and the sum over the terms after it
template <int N, int CLASSES, int PERM, class Kern>
qcoll_status launch_onchip64(const Plan &p, Kern kern, int lanes, size_t lds, const char *what,
                                    const cplx<double> *H, double *A, cplx<double> *U, long nbp, hipStream_t st) {
  if (hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                          int(lds)) != hipSuccess) {
    set_error("hipFuncSetAttribute failed for the FP64 gain kernel");
    return QCOLL_EDEVICE;
  }
  constexpr long n3 = long(N) * N * N;
  {
    TimedLaunch tl(what, st);
    const double scale = 1.0 / double(n3);
    hipLaunchKernelGGL(kern, dim3(unsigned(nbp * CLASSES * (U ? p.M : 1))), dim3(lanes), lds, st, H,
                       reinterpret_cast<const cplx<double> *>(p.phase), reinterpret_cast<const double *>(p.wq), A, U,
                       nbp, p.M, p.N_rho, scale);
  }
  if (U) {
    TimedLaunch tl("gain acc", st);
    hipLaunchKernelGGL((k_gain_acc64<PERM>), dim3(unsigned((nbp * n3 + 255) / 256)), dim3(256), 0, st,
                       reinterpret_cast<const double2 *>(U), A, n3, nbp, p.M - 1);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error(std::string(what) + ": " + hipGetErrorString(e));
    return QCOLL_EDEVICE;
  }
  return QCOLL_OK;
}

}  // namespace qcoll
