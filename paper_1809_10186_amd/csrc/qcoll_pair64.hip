// FP64 term loops that need the spectrum of every term's product, at N = 32:
// the gain adjoint of the VJP (VHS kernels) and the gain of VSS kernels.
//
// k_terms_c2 takes a term on chip to velocity space (c2_inverse: one workgroup
// per (item, node) pair and class of j1), forms the product there,
//   adjoint  y = w_q h_p conj(u)             (one volume per term),
//   VSS      t_q + i t_q', t = Re(u)^2 - Im(u)^2 = t1 t2   (two terms a volume),
// transforms it forward along axes 3 and 2 on chip and writes the class's
// planes: 16 bytes a point and volume, written once, where the two-pass
// schedule writes and reads a term's volume twice (and VSS kernels take a
// volume per term).  k_acc_terms reads each volume once, transforms it along
// axis 1 and adds it, weighted, to the item's spectrum
//   adjoint  Z = sum c_s(k) P(k)                  (2 Re ifft3[Z] is used),
//   VSS      Z = sum (alpha_q - i alpha_q')(k) P(k)     (Re ifft3[Z]: alpha is
//            even and real, so C_q t_q + C_q' t_q' is the real part).
// k_terms_c2 is bound like k_gain_c2 (VALU issue, LDS and L2 reads in turn)
// with half of its transforms more, k_acc_terms by its reads.  N_rho 16, M 12,
// through the projection: VJP of 37 items 4.00 ms in passes, 2.25 ms so (a launch
// of 16 items: terms 470 us, sums 320 us); VSS of 45 items 3.08 -> 1.92 ms.
// For few items both are latency, and split further: terms_a_workgroup and
// sum_by_points below.  1 item, N_rho 16, M 12: VSS 102 us in passes, 320 unsplit,
// 100 so; VJP 691, 445 and 213.
#include <hip/hip_runtime.h>

#include "qcoll_c2.hpp"

namespace qcoll {

// C -> B inside a wave's own planes: element (v, j2, k3) at v*S + j2*R + k3
template <int N>
__device__ __forceinline__ void c_to_b(double *tile, int vb, int cb, double *z) {
  constexpr int R = C2Geom<N>::R, S = C2Geom<N>::S;
  static_for<0, N>([&](auto kk) { tile[vb * S + cb * R + decltype(kk)::value] = z[decltype(kk)::value]; });
  lds_wave_order();
  static_for<0, N>([&](auto jj) { z[decltype(jj)::value] = tile[vb * S + decltype(jj)::value * R + cb]; });
  lds_wave_order();
}

// the lanes' parts in a fixed order: wave butterflies, then the waves
template <int NL>
__device__ __forceinline__ void class_dot(double *red, int lane, double dot, double *out) {
  for (int o = 32; o > 0; o >>= 1) dot += __shfl_xor(dot, o);
  if (lane % 64 == 0) red[lane / 64] = dot;
  __syncthreads();
  if (lane == 0) {
    double s = 0.0;
    for (int w = 0; w < NL / 64; ++w) s += red[w];
    *out = s;
  }
}

// MODE 0: adjoint, volumes (pair, q); MODE 1: VSS, volumes (pair, q / 2).
// H: spectra of the items; the launch takes ni of them from it0 on, nn nodes from n0
// on of each; Hp: h_p of every pair (MODE 0); Y: the launch's volumes [j1][k2][k3].
// A workgroup takes nt terms of its pair: all M, or (launches of a few pairs, which
// would leave most CUs idle) a volume's, one for the adjoint and two for VSS, or for
// VSS one: the products then stay in their volumes' places and k_forward_planes does
// the rest.  dots, or null: [2 pairs] parts of <h_p, A_p> by class; with nt < M every
// lane's part of the launch's terms, [pair][class][term][lane], which k_term_dots adds
// in the same order.
// PART = false is nt = M known at compile time (VSS: 45 items 1.41 -> 1.27 ms; the
// adjoint is not slower without).
template <int N, int MODE, bool PART>
__global__ __launch_bounds__(C2Geom<N>::NL) void k_terms_c2(const cplx<double> *__restrict__ H,
                                                           const cplx<double> *__restrict__ phase,
                                                           const double *__restrict__ wq,
                                                           const double *__restrict__ Hp,
                                                           cplx<double> *__restrict__ Y, double *__restrict__ dots,
                                                           long it0, long ni, int n0, int nn, int ntp, int M,
                                                           int Nr, double scale) {
  using Gm = C2Geom<N>;
  constexpr int NV = Gm::NV, S = Gm::S;
  constexpr long n2 = long(N) * N, n3 = n2 * N;
  extern __shared__ double tile[];

  const int MV = MODE == 0 ? M : (M + 1) / 2;   // volumes of a pair
  const int nt = PART ? ntp : M;
  const int nw = PART ? (M + nt - 1) / nt : 1;   // workgroups of a pair and class
  const long lb = xcd_block();
  if (lb >= ni * nn * nw * 2) return;  // uniform per workgroup
  const long bpl = lb / 2 / nw;
  const int g = int(lb % 2), q0 = PART ? int(lb / 2 % nw) * nt : 0;   // the first term
  const long b = it0 + bpl / nn;
  const int p = n0 + int(bpl % nn);
  const long bp = b * Nr + p;
  const int lane = threadIdx.x;
  const int vb = lane / N, cb = lane % N;   // plane v and row j2 (k3 after the transpose back)
  const __amdgpu_buffer_rsrc_t hr = make_rsrc(H + b * n3, unsigned(n3 * sizeof(cplx<double>)));
  cplx<double> *b1s = reinterpret_cast<cplx<double> *>(tile + NV * S);
  if (lane < N) b1s[(q0 & 1) * N + lane] = phase[size_t(p * M + q0) * 3 * N + lane];
  __syncthreads();

  double keep[MODE == 0 ? N : 1];   // the lane's row of h_p
  if constexpr (MODE == 0) {
    const double2 *h = reinterpret_cast<const double2 *>(Hp + bp * n3 + long(2 * vb + g) * n2 + long(cb) * N);
    static_for<0, N / 2>([&](auto j) {
      const double2 v = h[decltype(j)::value];
      keep[2 * decltype(j)::value] = v.x;
      keep[2 * decltype(j)::value + 1] = v.y;
    });
  }
  double dot = 0.0;
  const int yo = (int(2 * vb + g) * int(n2) + cb) * int(sizeof(cplx<double>));
  auto inverse = [&](int q, double sc, double *zr, double *zi) {
    const cplx<double> *ph = phase + size_t(p * M + q) * 3 * N;
    cplx<double> b1n{};
    if (lane < N && q + 1 < M) b1n = ph[3 * N + lane];
    c2_inverse<N>(tile, hr, ph, b1s + (q & 1) * N, g, lane, sc, [&]() {
      if (lane < N && q + 1 < M) b1s[((q + 1) & 1) * N + lane] = b1n;
    }, zr, zi);
  };
  // scratch in a volume: the lane's plane j1 = 2v + g as [q mod 2][j][j2] doubles,
  // which only its own wave writes
  const int ko = int(2 * vb + g) * int(n2 * sizeof(cplx<double>)) + cb * int(sizeof(double));
  const int vol0 = MODE == 0 ? q0 : q0 / 2, vol1 = PART && nt < M ? vol0 + 1 : MV;
  for (int vol = vol0; vol < vol1; ++vol) {
    const __amdgpu_buffer_rsrc_t yr = make_rsrc(Y + (bpl * MV + vol) * n3, unsigned(n3 * sizeof(cplx<double>)));
    double zr[N], zi[N];
    if constexpr (MODE == 0) {
      // u carries sqrt(w_q): y = w_q h conj(u) and w_q h (Re(u)^2 - Im(u)^2)
      const double sw = __builtin_sqrt(wq[vol]);
      inverse(vol, scale * sw, zr, zi);
      double part = 0.0;
      static_for<0, N>([&](auto j) {
        constexpr int jj = decltype(j)::value;
        part += keep[jj] * (zr[jj] * zr[jj] - zi[jj] * zi[jj]);
        const double s = sw * keep[jj];
        zr[jj] = s * zr[jj];
        zi[jj] = -s * zi[jj];
      });
      dot += part;
    } else {
      for (int q = PART && nt == 1 ? q0 : 2 * vol; q < M && q < 2 * vol + 2; ++q) {
        inverse(q, scale, zr, zi);
        static_for<0, N>([&](auto j) {
          constexpr int jj = decltype(j)::value;
          zr[jj] = __builtin_fma(zr[jj], zr[jj], -(zi[jj] * zi[jj]));
        });
        if ((PART && nt == 1) || ((q & 1) == 0 && q + 1 < M)) {
          // the first product waits in the volume's own place (this lane's
          // values, read back below): held in registers it spills as much
          const int qo = ko + (q & 1) * int(n2 * sizeof(double));
          static_for<0, N>([&](auto j) {
            typedef unsigned u2v __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2v, zr[decltype(j)::value]), yr, qo,
                                                  int(decltype(j)::value * N * sizeof(double)), 0);
          });
          if (PART && nt == 1) return;
        }
      }
      const bool two = 2 * vol + 1 < M;
      static_for<0, N>([&](auto j) {
        constexpr int jj = decltype(j)::value;
        double first = 0.0;
        if (two)
          first = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(yr, ko, int(jj * N * sizeof(double)), 0));
        zi[jj] = two ? zr[jj] : 0.0;
        zr[jj] = two ? first : zr[jj];
      });
    }
    fft_reg<N, -1, double>(zr, zi);   // axis 3: lane (v, j2) holds k3
    c_to_b<N>(tile, vb, cb, zr);
    c_to_b<N>(tile, vb, cb, zi);
    fft_reg<N, -1, double>(zr, zi);   // axis 2: lane (v, k3) holds k2
    // streaming stores (nt): read once, by k_acc_terms
    static_for<0, N>([&](auto kk) {
      typedef unsigned u4v __attribute__((ext_vector_type(4)));
      __builtin_amdgcn_raw_buffer_store_b128(
          __builtin_bit_cast(u4v, double2{zr[decltype(kk)::value], zi[decltype(kk)::value]}), yr, yo,
          int(decltype(kk)::value * N * sizeof(cplx<double>)), 2);
    });
  }
  if constexpr (MODE == 0) {
    if (dots) {
      if (nt == M) {
        __syncthreads();
        class_dot<Gm::NL>(tile, lane, dot, dots + bp * 2 + g);
      } else {
        dots[((bpl * 2 + g) * M + q0) * Gm::NL + lane] = dot;
      }
    }
  }
}

// VSS volumes whose planes hold their terms' products: the forward transforms along
// axes 3 and 2 as in k_terms_c2, two planes a wave
template <int N>
__global__ __launch_bounds__(64) void k_forward_planes(cplx<double> *Y, int M) {
  constexpr int n2 = N * N, NV = N / 2;
  static_assert(64 % N == 0 && 64 / N == 2, "two planes a wave");
  __shared__ double tile[2 * C2Geom<N>::S];
  const long vol = blockIdx.x / NV;
  const int vb = int(threadIdx.x) / N, cb = int(threadIdx.x) % N;
  cplx<double> *y = Y + (vol * N + int(blockIdx.x % NV) * 2 + vb) * n2;
  const double *t = reinterpret_cast<const double *>(y);
  const bool two = 2 * int(vol % ((M + 1) / 2)) + 1 < M;
  double zr[N], zi[N];
  static_for<0, N>([&](auto j) {
    constexpr int jj = decltype(j)::value;
    zr[jj] = t[jj * N + cb];
    zi[jj] = two ? t[n2 + jj * N + cb] : 0.0;
  });
  fft_reg<N, -1, double>(zr, zi);
  c_to_b<N>(tile, vb, cb, zr);
  c_to_b<N>(tile, vb, cb, zi);
  fft_reg<N, -1, double>(zr, zi);
  static_for<0, N>([&](auto kk) {
    y[decltype(kk)::value * N + cb] = cplx<double>{zr[decltype(kk)::value], zi[decltype(kk)::value]};
  });
}

// dots of the pairs of a launch of one term a workgroup from the lanes' parts P
template <int N>
__global__ __launch_bounds__(C2Geom<N>::NL) void k_term_dots(const double *__restrict__ P, double *__restrict__ dots,
                                                            long it0, int M, int Nr) {
  constexpr int NL = C2Geom<N>::NL;
  __shared__ double red[NL / 64];
  double dot = 0.0;
  for (int v = 0; v < M; ++v) dot += P[(long(blockIdx.x) * M + v) * NL + threadIdx.x];
  class_dot<NL>(red, threadIdx.x, dot, dots + it0 * Nr * 2 + blockIdx.x);
}

// k1 of sum i of parity G: the outputs of column k = G mod 2 of the decimated
// transform (the others are dropped at compile time, which leaves room for the
// sums beside the pencil)
template <int N, int G>
constexpr int acc_k1(int i) {
  return G + 2 * (i / 4) + (N / 4) * (i % 4);
}

// Weight of a volume's value (x, y) at (k1, pen), and the sum it joins; explicit
// fused operations, so that k_acc_terms and k_acc_points give the same bits.
//   adjoint  c_s = Re(b1 b2 b3) + Im(b1 b2 b3) = b1.re P + b1.im Q
//   VSS      w0 - i w1, the weights of the volume's two terms
template <int N>
struct ShiftFactor {
  const cplx<double> *ph;
  double P, Q;
  __device__ __forceinline__ ShiftFactor(const cplx<double> *phase, int M, int p, int v, int pen)
      : ph(phase + size_t(p * M + v) * 3 * N) {
    const cplx<double> b2 = ph[N + pen / N], b3 = ph[2 * N + pen % N];
    const double cr = __builtin_fma(b2.re, b3.re, -(b2.im * b3.im)), ci = __builtin_fma(b2.re, b3.im, b2.im * b3.re);
    P = cr + ci;
    Q = cr - ci;
  }
  __device__ __forceinline__ void add(int k1, double x, double y, double &ar, double &ai) const {
    const cplx<double> b1 = ph[k1];
    const double c = __builtin_fma(b1.re, P, b1.im * Q);
    ar = __builtin_fma(c, x, ar);
    ai = __builtin_fma(c, y, ai);
  }
};

template <int N>
struct VssWeight {
  // alpha_pq on the planes k1 <= N/2; plane k1 > N/2 at the reflected index
  const double *a0, *a1;
  bool two;
  int pen, refl;
  __device__ __forceinline__ VssWeight(const double *apq, int M, int p, int v, int pen_) : pen(pen_) {
    constexpr long nh = long(N / 2 + 1) * N * N;
    refl = ((N - pen / N) % N) * N + (N - pen % N) % N;
    a0 = apq + (size_t(p) * M + 2 * v) * nh;
    two = 2 * v + 1 < M;
    a1 = two ? a0 + nh : a0;
  }
  __device__ __forceinline__ void add(int k1, double x, double y, double &ar, double &ai) const {
    const int o = k1 <= N / 2 ? k1 * (N * N) + pen : (N - k1) * (N * N) + refl;
    const double w0 = a0[o], r1 = a1[o], w1 = two ? r1 : 0.0;
    ar += __builtin_fma(w0, x, w1 * y);
    ai += __builtin_fma(w0, y, -(w1 * x));
  }
};

template <int N, int MODE>
__device__ __forceinline__ auto term_weight(const cplx<double> *phase, const double *apq, int M, int p, int v,
                                            int pen) {
  if constexpr (MODE == 0) return ShiftFactor<N>(phase, M, p, v, pen);
  else return VssWeight<N>(apq, M, p, v, pen);
}

// the pencil pen of volume y
template <int N>
__device__ __forceinline__ void load_pencil(const cplx<double> *y, int pen, double *xr, double *xi) {
  constexpr int n2 = N * N;
  const __amdgpu_buffer_rsrc_t yr = make_rsrc(y, unsigned(long(n2) * N * sizeof(cplx<double>)));
  static_for<0, N>([&](auto j) {
    const cplx<double> x = load_c64(yr, pen * int(sizeof(cplx<double>)),
                                    int(decltype(j)::value * n2 * sizeof(cplx<double>)));
    xr[decltype(j)::value] = x.re;
    xi[decltype(j)::value] = x.im;
  });
}

// the pencil pen of volume y into the sums of parity G.  Each parity loads for
// itself: with the loads ahead of the branch 18 (MODE 0) and 43 (MODE 1)
// registers spill, none so.
template <int N, int MODE, int G>
__device__ __forceinline__ void acc_term(const cplx<double> *__restrict__ y, const cplx<double> *__restrict__ phase,
                                         const double *__restrict__ apq, int p, int v, int M, int pen, double *ar,
                                         double *ai) {
  double xr[N], xi[N];
  auto sum = [&](const auto &w) {
    fft_reg<N, -1, double>(xr, xi);
    static_for<0, N / 2>([&](auto i) {
      constexpr int ii = decltype(i)::value, k1 = acc_k1<N, G>(ii);
      w.add(k1, xr[k1], xi[k1], ar[ii], ai[ii]);
    });
  };
  if constexpr (MODE == 0) {
    load_pencil<N>(y, pen, xr, xi);   // all of it in flight before the factors are asked for
    __builtin_amdgcn_sched_barrier(0);
    sum(ShiftFactor<N>(phase, M, p, v, pen));
  } else {
    const VssWeight<N> w(apq, M, p, v, pen);
    load_pencil<N>(y, pen, xr, xi);
    sum(w);
  }
}

// Z part: one lane per pencil (k2, k3) of an item and per parity of k1, over the
// volumes of the nodes [part Nr / kAccParts, (part + 1) Nr / kAccParts): a fixed
// split, so that an item's result does not depend on the launch.  A launch of the nodes
// [n0, n0 + nn) goes on from the sums that the nodes before them left.
template <int N, int MODE>
__global__ __launch_bounds__(256, 2) void k_acc_terms(const cplx<double> *__restrict__ Y,
                                                      const cplx<double> *__restrict__ phase,
                                                      const double *__restrict__ apq, cplx<double> *__restrict__ Z,
                                                      long part_stride, int M, int Nr, int n0, int nn) {
  constexpr int n2 = N * N, HN = N / 2;
  constexpr long n3 = long(n2) * N;
  // a workgroup: 128 pencils, waves 0 and 1 their even k1, waves 2 and 3 the odd
  constexpr int GP = n2 / 128;
  const long bl = blockIdx.x / GP;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / 64);
  const int pen = int(blockIdx.x % GP) * 128 + (wave % 2) * 64 + int(threadIdx.x) % 64;
  const int part = int(blockIdx.y);
  const int p0 = part * Nr / kAccParts, p1 = (part + 1) * Nr / kAccParts;
  // the part's nodes in this launch; the first launch clears a part without any
  const int first = p0 > n0 ? p0 : n0, last = p1 < n0 + nn ? p1 : n0 + nn;
  if (first >= last && !(p0 == p1 && n0 == 0)) return;  // uniform per workgroup
  const int MV = MODE == 0 ? M : (M + 1) / 2;
  cplx<double> *z = Z + part * part_stride + bl * n3 + pen + (wave / 2) * n2;
  double ar[HN], ai[HN];
  static_for<0, HN>([&](auto i) { ar[decltype(i)::value] = 0.0; ai[decltype(i)::value] = 0.0; });
  if (first > p0) {
    static_for<0, HN>([&](auto i) {
      const cplx<double> v = z[acc_k1<N, 0>(decltype(i)::value) * n2];
      ar[decltype(i)::value] = v.re;
      ai[decltype(i)::value] = v.im;
    });
  }
  for (int p = first; p < last; ++p) {
    for (int v = 0; v < MV; ++v) {
      // both parities read a volume together (the second from cache): one barrier
      // that all four waves meet, ahead of the branch on the parity
      __syncthreads();
      const cplx<double> *y = Y + ((bl * nn + p - n0) * MV + v) * n3;
      if (wave < 2) acc_term<N, MODE, 0>(y, phase, apq, p, v, M, pen, ar, ai);
      else acc_term<N, MODE, 1>(y, phase, apq, p, v, M, pen, ar, ai);
    }
  }
  static_for<0, HN>([&](auto i) {
    z[acc_k1<N, 0>(decltype(i)::value) * n2] = cplx<double>{ar[decltype(i)::value], ai[decltype(i)::value]};
  });
}

// The same sums for a few items (k_acc_terms has 32 workgroups an item, each with a
// quarter of its volumes in turn): every volume transformed along axis 1 in place by
// k_axis1_terms, then one lane a point and part.
template <int N>
__global__ __launch_bounds__(64) void k_axis1_terms(cplx<double> *Y) {
  constexpr int n2 = N * N, WP = n2 / 64;
  cplx<double> *y = Y + long(blockIdx.x / WP) * (long(n2) * N);
  const int pen = int(blockIdx.x % WP) * 64 + int(threadIdx.x);
  double xr[N], xi[N];
  load_pencil<N>(y, pen, xr, xi);
  fft_reg<N, -1, double>(xr, xi);
  static_for<0, N>([&](auto k) {
    y[decltype(k)::value * n2 + pen] = cplx<double>{xr[decltype(k)::value], xi[decltype(k)::value]};
  });
}

template <int N, int MODE>
__global__ __launch_bounds__(256) void k_acc_points(const cplx<double> *__restrict__ Y,
                                                    const cplx<double> *__restrict__ phase,
                                                    const double *__restrict__ apq, cplx<double> *__restrict__ Z,
                                                    long part_stride, int M, int Nr) {
  constexpr int n2 = N * N, n3 = n2 * N, WG = n3 / 256;
  const long bl = blockIdx.x / WG;
  const int o = int(blockIdx.x % WG) * 256 + int(threadIdx.x);
  const int part = int(blockIdx.y);
  const int p0 = part * Nr / kAccParts, p1 = (part + 1) * Nr / kAccParts;
  const int MV = MODE == 0 ? M : (M + 1) / 2;
  const int k1 = o / n2, pen = o % n2;
  double ar = 0.0, ai = 0.0;
  for (int p = p0; p < p1; ++p) {
    const cplx<double> *y = Y + (bl * Nr + p) * MV * long(n3) + o;
#pragma unroll 4
    for (int v = 0; v < MV; ++v) {
      const cplx<double> x = y[v * long(n3)];
      term_weight<N, MODE>(phase, apq, M, p, v, pen).add(k1, x.re, x.im, ar, ai);
    }
  }
  Z[part * part_stride + bl * n3 + o] = cplx<double>{ar, ai};
}

// dwg[pair] = both classes' parts
__global__ __launch_bounds__(256) void k_class_dots(const double *dots, double *dwg, long n) {
  const long i = long(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) dwg[i] = dots[2 * i] + dots[2 * i + 1];
}

static bool terms64_supported(const Plan &p) { return p.precision == QCOLL_FP64 && p.N == 32 && !p.literal; }

bool use_adjoint_terms64(const Plan &p) { return terms64_supported(p) && p.schedule_user != 1 && !p.is_vss(); }

bool use_vss_terms64(const Plan &p) { return terms64_supported(p) && p.schedule != 1 && p.is_vss(); }

// Terms per workgroup of k_terms_c2 for wgs (pair, class)es, by the rounds of one
// workgroup a CU: fewer where that takes clearly fewer term times (the price of less
// than all is the row of h_p again for every volume, of a single VSS term the products
// through memory).  Terms of all / two / one a workgroup, us, VSS 1.5: N_rho 4, M 6, 1
// item 104 / 41 / 28, 16 items 108 / 83 / 86; 8, 12: 1 item 204 / 41 / 33, 4 items
// 207 / 82 / 86, 16 items 249 / 251 / 330; adjoint, all / one: 4, 6, 1 item 104 / 31;
// 16, 12, 1 item 201 / 60, 4 items 204 / 163, 8 items 245 / 320.
static int terms_a_workgroup(int mode, long wgs, int M) {
  constexpr long cus = 256;
  auto rounds = [](long n) { return (n + cus - 1) / cus; };
  if (mode == 1 && wgs * M <= cus) return 1;
  const int nt = mode == 0 ? 1 : 2;
  return 4 * rounds(wgs * ((M + nt - 1) / nt)) * nt < 3 * rounds(wgs) * M ? nt : M;
}

// The sums by points where the launch has all nodes of a few items: k_acc_terms takes
// about 3 us a volume of the longest part, whatever the items, the other two kernels
// 0.25 us a volume (VSS, N_rho 16, M 12: 1 item 92 / 34 us, 4 items 94 / 102; adjoint
// 1 item 154 / 65, 4 items 149 / 222).
static bool sum_by_points(const Plan &p, long ni, int nn) {
  return nn == p.N_rho && ni * nn <= 12 * ((nn + kAccParts - 1) / kAccParts);
}

template <int MODE>
static qcoll_status launch_terms64(const Plan &p, const cplx<double> *H, const double *Hp, cplx<double> *Y,
                                   cplx<double> *Z, long part_stride, double *dots, double *parts, long it0,
                                   long ni, int n0, int nn, hipStream_t st) {
  constexpr int N = 32;
  using G = C2Geom<N>;
  const int nt = terms_a_workgroup(MODE, ni * nn * 2, p.M);
  const auto terms = MODE == 0 || nt == 1 || nt < p.M ? &k_terms_c2<N, MODE, true> : &k_terms_c2<N, MODE, MODE == 0>;
  if (hipFuncSetAttribute(reinterpret_cast<const void *>(terms),
                          hipFuncAttributeMaxDynamicSharedMemorySize, int(G::lds_bytes)) != hipSuccess) {
    set_error("hipFuncSetAttribute failed for the FP64 term kernel");
    return QCOLL_EDEVICE;
  }
  const auto *ph = reinterpret_cast<const cplx<double> *>(p.phase);
  const int MV = MODE == 0 ? p.M : (p.M + 1) / 2;
  const long n3 = long(N) * N * N;
  {
    TimedLaunch tl(MODE == 0 ? "vjp terms c2" : "vss terms c2", st);
    hipLaunchKernelGGL(terms, dim3(unsigned(ni * nn * 2 * ((p.M + nt - 1) / nt))), dim3(G::NL),
                       G::lds_bytes, st, H, ph, reinterpret_cast<const double *>(p.wq), Hp, Y,
                       dots && nt < p.M ? parts : dots, it0, ni, n0, nn, nt, p.M, p.N_rho, 1.0 / double(n3));
    if (MODE == 1 && nt == 1)
      hipLaunchKernelGGL((k_forward_planes<N>), dim3(unsigned(ni * nn * MV * (N / 2))), dim3(64), 0, st, Y, p.M);
    if (dots && nt < p.M)
      hipLaunchKernelGGL((k_term_dots<N>), dim3(unsigned(ni * nn * 2)), dim3(G::NL), 0, st, parts, dots, it0, p.M,
                         p.N_rho);
  }
  {
    TimedLaunch tl(MODE == 0 ? "vjp terms acc" : "vss terms acc", st);
    if (sum_by_points(p, ni, nn)) {
      hipLaunchKernelGGL((k_axis1_terms<N>), dim3(unsigned(ni * nn * MV * (N * N / 64))), dim3(64), 0, st, Y);
      hipLaunchKernelGGL((k_acc_points<N, MODE>), dim3(unsigned(ni * (n3 / 256)), kAccParts), dim3(256), 0, st, Y, ph,
                         static_cast<const double *>(p.alpha_pq), Z + it0 * n3, part_stride, p.M, p.N_rho);
    } else {
      hipLaunchKernelGGL((k_acc_terms<N, MODE>), dim3(unsigned(ni * (N * N / 128)), kAccParts), dim3(256), 0, st, Y,
                         ph, static_cast<const double *>(p.alpha_pq), Z + it0 * n3, part_stride, p.M, p.N_rho, n0, nn);
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error(std::string("FP64 terms: ") + hipGetErrorString(e));
    return QCOLL_EDEVICE;
  }
  return QCOLL_OK;
}

qcoll_status launch_adjoint_terms64(const Plan &p, const void *H, const double *Hp, void *Y, void *Z,
                                    long part_stride, double *dots, double *parts, double *dwg, long nb, long pc,
                                    hipStream_t st) {
  for (long i0 = 0; i0 < nb; i0 += pc) {
    const qcoll_status s = launch_terms64<0>(p, static_cast<const cplx<double> *>(H), Hp,
                                             static_cast<cplx<double> *>(Y), static_cast<cplx<double> *>(Z),
                                             part_stride, dots, parts, i0, nb - i0 < pc ? nb - i0 : pc, 0, p.N_rho,
                                             st);
    if (s != QCOLL_OK) return s;
  }
  if (dots) {
    const long n = nb * p.N_rho;
    hipLaunchKernelGGL(k_class_dots, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, dots, dwg, n);
    if (hipGetLastError() != hipSuccess) {
      set_error("FP64 terms: class dots launch failed");
      return QCOLL_EDEVICE;
    }
  }
  return QCOLL_OK;
}

qcoll_status launch_vss_terms64(const Plan &p, const void *H, void *Y, void *Z, long part_stride, long nb, long pc,
                                int pn, hipStream_t st) {
  for (long i0 = 0; i0 < nb; i0 += pc) {
    const long ni = nb - i0 < pc ? nb - i0 : pc;
    for (int n0 = 0; n0 < p.N_rho; n0 += pn) {
      const qcoll_status s = launch_terms64<1>(p, static_cast<const cplx<double> *>(H), nullptr,
                                               static_cast<cplx<double> *>(Y), static_cast<cplx<double> *>(Z),
                                               part_stride, nullptr, nullptr, i0, ni, n0,
                                               p.N_rho - n0 < pn ? p.N_rho - n0 : pn, st);
      if (s != QCOLL_OK) return s;
    }
  }
  return QCOLL_OK;
}

}  // namespace qcoll
