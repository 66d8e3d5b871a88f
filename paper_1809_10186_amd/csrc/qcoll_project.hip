// Conservation projection of Q and the moments of f, FP64.
#include <hip/hip_runtime.h>

#include "qcoll_passes.hpp"

namespace qcoll {

// FP64 conservation projection: one 1024-lane workgroup per item.  Each lane
// walks pairs of consecutive points along the last axis (16-byte loads); the
// velocity of a point is rebuilt from its index.  The five sums are reduced
// in a fixed order, so the result is deterministic.  With PPT > 0 (grids up
// to 32^3: at most 16 pairs per lane) a lane keeps its PPT pairs in registers
// between the sums and the correction, so Q is read once; PPT = 0 reads it
// twice.  Both visit a lane's pairs in the same order: the results are
// bit-identical.  NC > 0 fixes N at compile time, so that rebuilding a point's
// indices takes shifts and multiplications instead of integer divisions by a
// runtime value (which dominated the kernel's instruction count).
constexpr int kConserveBlock = 1024;   // lanes per workgroup of k_conserve

template <int PPT, int NC = 0>
__global__ __launch_bounds__(kConserveBlock) void k_conserve(double *Q, double *mom, const double *ginv, int Nrt, double L,
                                                   int *flag, double dc3, const double *isc, int K) {
  const int N = NC > 0 ? NC : Nrt;
  const long n3 = long(N) * N * N;
  const long b = blockIdx.x;
  double2 *q = reinterpret_cast<double2 *>(Q + b * n3);
  const double dc = 2.0 * L / N;
  const long nh = n3 / 2;   // N is even: a pair never crosses a row
  auto coords = [&](long h, double &c1, double &c2, double &c3a, double &c3b) {
    const long j = 2 * h;
    const int i1 = int(j / (N * N)), i2 = int((j / N) % N), i3 = int(j % N);
    c1 = -L + (i1 + 0.5) * dc;
    c2 = -L + (i2 + 0.5) * dc;
    c3a = -L + (i3 + 0.5) * dc;
    c3b = c3a + dc;
  };
  double s[5] = {0, 0, 0, 0, 0};
  auto add = [&](long h, double2 v) {
    double c1, c2, c3a, c3b;
    coords(h, c1, c2, c3a, c3b);
    const double sv = v.x + v.y;
    const double r12 = c1 * c1 + c2 * c2;
    s[0] += sv;
    s[1] += sv * c1;
    s[2] += sv * c2;
    s[3] += v.x * c3a + v.y * c3b;
    s[4] += v.x * (r12 + c3a * c3a) + v.y * (r12 + c3b * c3b);
  };
  double2 keep[PPT > 0 ? PPT : 1];
  if constexpr (PPT > 0) {
    // every load is issued before the first sum: the index is clamped instead
    // of guarded (a guarded load sits in a branch of its own, and the compiler
    // then waits for each load before the next one is issued)
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
      const long h = threadIdx.x + long(i) * kConserveBlock;
      keep[i] = q[h < nh ? h : nh - 1];
    }
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
      const long h = threadIdx.x + long(i) * kConserveBlock;
      if (h < nh) add(h, keep[i]);
    }
  } else {
    for (long h = threadIdx.x; h < nh; h += blockDim.x) add(h, q[h]);
  }
  // butterflies within the waves, then over the waves' sums in every wave: one
  // barrier (a tree over the workgroup in LDS took eleven)
  __shared__ double red[5][kConserveBlock / 64];
  for (int k = 0; k < 5; ++k)
    for (int o = 32; o > 0; o >>= 1) s[k] += __shfl_xor(s[k], o);
  if (threadIdx.x % 64 == 0)
    for (int k = 0; k < 5; ++k) red[k][threadIdx.x / 64] = s[k];
  __syncthreads();
  double m[5], lam[5];
  for (int k = 0; k < 5; ++k) {
    m[k] = red[k][threadIdx.x % (kConserveBlock / 64)];
    for (int o = kConserveBlock / 128; o > 0; o >>= 1) m[k] += __shfl_xor(m[k], o);
  }
  const double sc = isc ? isc[b % K] : 1.0;   // projection first, then the item's weight
  for (int a = 0; a < 5; ++a) {
    double acc = 0;
    for (int c = 0; c < 5; ++c) acc += ginv[a * 5 + c] * m[c];
    lam[a] = acc;
  }
  bool finite = true;
  for (int k = 0; k < 5; ++k) finite = finite && isfinite(m[k]);
  if (threadIdx.x == 0) {
    if (mom)
      for (int k = 0; k < 5; ++k) mom[b * 5 + k] = m[k] * dc3;
    if (!finite) atomicOr(flag, 1);
  }
  auto fix = [&](long h, double2 v) {
    double c1, c2, c3a, c3b;
    coords(h, c1, c2, c3a, c3b);
    const double base = lam[0] + lam[1] * c1 + lam[2] * c2 + lam[4] * (c1 * c1 + c2 * c2);
    v.x -= base + lam[3] * c3a + lam[4] * c3a * c3a;
    v.y -= base + lam[3] * c3b + lam[4] * c3b * c3b;
    v.x *= sc;
    v.y *= sc;
    q[h] = v;
  };
  if constexpr (PPT > 0) {
    // The lane index goes through an empty asm statement, so that the
    // coordinates are rebuilt here instead of being held in registers from
    // the first pass (64 more live doubles at PPT = 16: they spilled).
    int lane = threadIdx.x;
    asm volatile("" : "+v"(lane));
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
      const long h = lane + long(i) * kConserveBlock;
      if (h < nh) fix(h, keep[i]);
    }
  } else {
    for (long h = threadIdx.x; h < nh; h += blockDim.x) fix(h, q[h]);
  }
}

// Midpoint-rule moments, FP64, one workgroup per item, two passes.
__global__ __launch_bounds__(256) void k_moments(const double *F, double *out, int N, double L) {
  const long n3 = long(N) * N * N;
  const long b = blockIdx.x;
  const double *f = F + b * n3;
  const double dc = 2.0 * L / N, dc3 = dc * dc * dc;
  __shared__ double red[10][256];
  double s[10];
  for (int k = 0; k < 4; ++k) s[k] = 0;
  for (long j = threadIdx.x; j < n3; j += blockDim.x) {
    const int i1 = int(j / (N * N)), i2 = int((j / N) % N), i3 = int(j % N);
    const double v = f[j];
    s[0] += v;
    s[1] += v * (-L + (i1 + 0.5) * dc);
    s[2] += v * (-L + (i2 + 0.5) * dc);
    s[3] += v * (-L + (i3 + 0.5) * dc);
  }
  for (int k = 0; k < 4; ++k) red[k][threadIdx.x] = s[k];
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w)
      for (int k = 0; k < 4; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + w];
    __syncthreads();
  }
  const double n = red[0][0] * dc3;
  const double u1 = red[1][0] * dc3 / n, u2 = red[2][0] * dc3 / n, u3 = red[3][0] * dc3 / n;
  __syncthreads();
  for (int k = 0; k < 10; ++k) s[k] = 0;
  for (long j = threadIdx.x; j < n3; j += blockDim.x) {
    const int i1 = int(j / (N * N)), i2 = int((j / N) % N), i3 = int(j % N);
    const double v = f[j];
    const double d1 = -L + (i1 + 0.5) * dc - u1, d2 = -L + (i2 + 0.5) * dc - u2, d3 = -L + (i3 + 0.5) * dc - u3;
    const double d2s = d1 * d1 + d2 * d2 + d3 * d3;
    s[0] += v * d2s;
    s[1] += v * d1 * d1;
    s[2] += v * d1 * d2;
    s[3] += v * d1 * d3;
    s[4] += v * d2 * d2;
    s[5] += v * d2 * d3;
    s[6] += v * d3 * d3;
    s[7] += v * d1 * d2s;
    s[8] += v * d2 * d2s;
    s[9] += v * d3 * d2s;
  }
  for (int k = 0; k < 10; ++k) red[k][threadIdx.x] = s[k];
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w)
      for (int k = 0; k < 10; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double *o = out + b * 14;
    o[0] = n;
    o[1] = u1;
    o[2] = u2;
    o[3] = u3;
    o[4] = 2.0 / (3.0 * n) * red[0][0] * dc3;
    for (int k = 0; k < 6; ++k) o[5 + k] = 2.0 * red[1 + k][0] * dc3;
    for (int k = 0; k < 3; ++k) o[11 + k] = red[7 + k][0] * dc3;
  }
}

qcoll_status launch_conserve(const Plan &p, int64_t batch, double *Q, double *mom, hipStream_t st, const double *isc,
                             int K) {
  const double dc = 2.0 * p.L / p.N;
  TimedLaunch tl("conserve", st);
  // pairs per lane of the register-resident variant: N^3 / 2 / 1024, rounded up
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(unsigned(batch)), dim3(kConserveBlock), 0, st, Q, mom, p.ginv, p.N, p.L, p.flag,
                       dc * dc * dc, isc, K);
  };
  switch (p.N) {
    case 8: go(k_conserve<1, 8>); break;
    case 12: go(k_conserve<1, 12>); break;
    case 16: go(k_conserve<2, 16>); break;
    case 24: go(k_conserve<7, 24>); break;
    case 32: go(k_conserve<16, 32>); break;
    case 48: go(k_conserve<0, 48>); break;
    case 64: go(k_conserve<0, 64>); break;
    default: go(k_conserve<0>); break;
  }
  QC_LAUNCH_CHECK("conserve");
  return QCOLL_OK;
}

qcoll_status launch_moments(const Plan &p, int64_t batch, const double *f, double *out, hipStream_t st) {
  TimedLaunch tl("moments", st);
  hipLaunchKernelGGL(k_moments, dim3(unsigned(batch)), dim3(256), 0, st, f, out, p.N, p.L);
  QC_LAUNCH_CHECK("moments");
  return QCOLL_OK;
}

}  // namespace qcoll
