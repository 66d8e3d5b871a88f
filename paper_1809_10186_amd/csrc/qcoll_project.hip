// Conservation projection of Q and the moments of f, FP64.
#include <hip/hip_runtime.h>

#include "qcoll_passes.hpp"

namespace qcoll {

// FP64 conservation projection: one workgroup of up to 1024 lanes per item.
// Each lane walks pairs of consecutive points along the last axis (16-byte
// loads); the five sums are reduced in a fixed order, so the result is
// deterministic.  Bound by one CU's FP64 and index arithmetic for few items, by
// memory for many.
// PPT > 0 (grids up to 32^3): the workgroup covers whole planes of the first
// axis per pass, so a lane meets the same (c2, c3) in each of its PPT pairs: it
// sums v, c1 v and c1^2 v, and multiplies the rest in once.  It keeps its pairs in
// registers between the sums and the correction, so Q is read once.  PPT = 0
// rebuilds each point's velocity from its index and reads Q twice.  NC > 0 fixes N
// at compile time.
constexpr int kConserveBlock = 1024;   // most lanes per workgroup of k_conserve

// planes of the first axis per pass, and the passes.  24^3: two planes are nine whole
// waves, three are thirteen and a half, with a test in every pass (1024 items 41.5 ->
// 40.9 us, 39.7 before the planes; 30 items 8.2 -> 7.8, 11.3)
constexpr int conserve_planes(int N) {
  if (N == 24) return 2;
  const int r = kConserveBlock / (N * N / 2);
  return r < N ? r : N;
}
constexpr int conserve_ppt(int N) { return (N + conserve_planes(N) - 1) / conserve_planes(N); }
// lanes: whole waves
constexpr int conserve_lanes(int N) { return (conserve_planes(N) * (N * N / 2) + 63) / 64 * 64; }

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
  // PPT > 0: the lane's pair of a plane, its plane of a pass (lanes past the
  // last whole plane hold nothing) and its velocities
  constexpr int HP = NC > 0 ? NC * NC / 2 : 1, RP = PPT > 0 ? conserve_planes(NC > 0 ? NC : 8) : 1;
  constexpr bool FULL = RP * HP % 64 == 0 && NC % RP == 0;   // every lane has a pair in every pass
  double l1 = 0, l2 = 0, l3a = 0, l3b = 0;
  // its pair of pass i, or nh
  auto pair = [&](int t, int i) {
    const int h = t + i * RP * HP;
    if constexpr (FULL) return h;
    const int lp = t / HP;
    return lp < RP && lp + i * RP < N ? h : int(nh);
  };
  if constexpr (PPT > 0) {
    coords(threadIdx.x, l1, l2, l3a, l3b);
    // every load is issued before the first sum: the index is clamped instead
    // of guarded (a guarded load sits in a branch of its own, and the compiler
    // then waits for each load before the next one is issued)
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
      const int h = pair(threadIdx.x, i);
      keep[i] = q[FULL || h < nh ? h : nh - 1];
    }
    double sx = 0, sy = 0, s11 = 0;
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
      if (!FULL && pair(threadIdx.x, i) >= nh) keep[i] = double2{0.0, 0.0};
      const double c1 = l1 + i * (RP * dc);
      const double sv = keep[i].x + keep[i].y, v1 = sv * c1;
      sx += keep[i].x;
      sy += keep[i].y;
      s[1] += v1;
      s11 += v1 * c1;
    }
    s[0] = sx + sy;
    s[2] = s[0] * l2;
    s[3] = sx * l3a + sy * l3b;
    s[4] = s11 + s[0] * (l2 * l2) + (sx * (l3a * l3a) + sy * (l3b * l3b));
  } else {
    for (long h = threadIdx.x; h < nh; h += blockDim.x) add(h, q[h]);
  }
  // Within a wave the exchanges halve the number of sums that a lane goes on
  // with: 9 of them, where five butterflies take 30 (which cost the many
  // workgroups of a large batch of small grids more than the LDS tree of eleven
  // barriers before them: 1024 items at 16^3 14.5 -> 23.7 us).
  __shared__ double red[5][kConserveBlock / 64];
  {
    const int l = threadIdx.x % 64;
    const bool a = !(l & 32), b = !(l & 16), c = !(l & 8);
    const double t0 = (a ? s[0] : s[3]) + __shfl_xor(a ? s[3] : s[0], 32);
    const double t1 = (a ? s[1] : s[4]) + __shfl_xor(a ? s[4] : s[1], 32);
    const double t2 = (a ? s[2] : 0.0) + __shfl_xor(a ? 0.0 : s[2], 32);
    const double u0 = (b ? t0 : t2) + __shfl_xor(b ? t2 : t0, 16);
    const double u1 = (b ? t1 : 0.0) + __shfl_xor(b ? 0.0 : t1, 16);
    double v = (c ? u0 : u1) + __shfl_xor(c ? u1 : u0, 8);
    for (int o = 4; o > 0; o >>= 1) v += __shfl_xor(v, o);
    const int k = a ? (b ? (c ? 0 : 1) : 2) : (c ? 3 : 4);
    if (l % 8 == 0 && (b || (a && c))) red[k][threadIdx.x / 64] = v;
  }
  __syncthreads();
  // the waves' sums: sixteen lanes a sum
  double m[5], lam[5];
  {
    const int l = threadIdx.x % 64, w = l % 16;
    const bool in = w < int(blockDim.x / 64);
    double x = in ? red[l / 16][w] : 0.0, y = in ? red[4][w] : 0.0;
    for (int o = 8; o > 0; o >>= 1) {
      x += __shfl_xor(x, o);
      y += __shfl_xor(y, o);
    }
    for (int k = 0; k < 4; ++k) m[k] = __shfl(x, 16 * k);
    m[4] = y;
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
    // the lane index and its c1 go through empty asm statements, so that the
    // passes' values are formed again here instead of being held in registers
    // since the sums
    int lane = threadIdx.x;
    asm volatile("" : "+v"(lane));
    asm volatile("" : "+v"(l1));
    const double b0 = lam[0] + lam[2] * l2 + lam[4] * (l2 * l2);
    const double ba = b0 + (lam[3] * l3a + lam[4] * (l3a * l3a)), bb = b0 + (lam[3] * l3b + lam[4] * (l3b * l3b));
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
      const int h = pair(lane, i);
      const double c1 = l1 + i * (RP * dc), b1 = lam[1] * c1 + lam[4] * (c1 * c1);
      if (FULL || h < nh) q[h] = double2{(keep[i].x - (b1 + ba)) * sc, (keep[i].y - (b1 + bb)) * sc};
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
  auto go = [&](auto kern, int lanes) {
    hipLaunchKernelGGL(kern, dim3(unsigned(batch)), dim3(lanes), 0, st, Q, mom, p.ginv, p.N, p.L, p.flag,
                       dc * dc * dc, isc, K);
  };
  switch (p.N) {
    case 8: go(k_conserve<conserve_ppt(8), 8>, conserve_lanes(8)); break;
    case 12: go(k_conserve<conserve_ppt(12), 12>, conserve_lanes(12)); break;
    case 16: go(k_conserve<conserve_ppt(16), 16>, conserve_lanes(16)); break;
    case 24: go(k_conserve<conserve_ppt(24), 24>, conserve_lanes(24)); break;
    case 32: go(k_conserve<conserve_ppt(32), 32>, conserve_lanes(32)); break;
    case 48: go(k_conserve<0, 48>, kConserveBlock); break;
    case 64: go(k_conserve<0, 64>, kConserveBlock); break;
    default: go(k_conserve<0>, kConserveBlock); break;
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
