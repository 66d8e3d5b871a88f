// FP64 gain loop on chip (N = 16): for one (item, radial node) pair
// and one residue class g of the second output index (j2 = 4u + g), a
// workgroup of N^2/4 lanes runs
//   A_p(j) += w_q (Re(u)^2 - Im(u)^2),  u = ifft3[c_s f^]   for every q
// (Appendix: the product of the two shifted copies of f for one quadrature
// term, packed in one complex transform) and writes its quarter of A_p once.
// Four workgroups cover one pair; nothing of the per-term volumes reaches HBM,
// where the two-pass FP64 schedule writes and re-reads M complex volumes per pair.
//
// Per term, lane (k1, t) (t < N/4):
//   stage 1: the inverse transform along axis 2 of its four pencils
//            (k1, k3 = t + m N/4), evaluated only at the outputs j2 = 4u + g:
//            with k2 = (N/4) a + b, X[4u + g] = sum_b w^(g b) w4^(u b) y_b and
//            y_b = sum_a i^(g a) x[(N/4) a + b]  (w = e^(2 pi i/N), w4 = w^4),
//            i.e. a four-term combination, a twiddle and an N/4-point
//            transform, about a third of a full transform.  The shift
//            multiplier c_s (times sqrt(w_q)) is applied as the pencil loads.
//   stage 2: a transpose among the N/4 lanes of one k1 gives lane (k1, u) all
//            k3 of j2 = 4u + g; inverse transform along axis 3.
//   stage 3: a transpose across the workgroup gives lane (u, j3) all k1 of
//            (j2, j3); inverse transform along axis 1, then the product.
// The transposes move one component at a time through an LDS tile of
// N x (N/4)(N+1) doubles.
//
// The kernel is written for any N divisible by 4, but it is launched only at
// N = 16 (1.4x faster than the two-pass schedule there).  From N = 24 a lane's
// four pencils, their FFT temporaries and the N-double accumulator exceed 256
// VGPRs; at one wave per SIMD the per-term reloads of the item spectrum from L2
// are not hidden.  At N = 32 the kernel below splits j1 in two classes
// instead: one pencil per lane, two waves per SIMD.
#include <hip/hip_runtime.h>

#include "qcoll_c2.hpp"

namespace qcoll {

template <int N>
struct Q64Geom {
  static constexpr int N4 = N / 4;
  static constexpr int NL = N * N4;     // lanes
  static constexpr int R = N + 1;       // tile row stride (doubles)
  static constexpr int S = N4 * R;      // tile stride per k1
  static constexpr size_t lds_bytes = size_t(N) * S * sizeof(double);
  // the stage-2 transpose stays inside a wave when the N/4 lanes of a k1 do
  static constexpr bool WAVE2 = (64 % N4 == 0);
  // rows of stage-1 loads in flight (4 pencils each)
  static constexpr int KG = 4;   // rows of H loaded together (a row at a time 47.9 us a call of one 16^3 item, 45.6 so)
};

// stage 1 for residue class G: v[m N/4 + u] = X_m[4u + G], X_m the inverse
// transform along axis 2 of pencil (k1, t + m N/4) of c_s f^
template <int N, int G>
__device__ __forceinline__ void q64_stage1(__amdgpu_buffer_rsrc_t hr, const cplx<double> *__restrict__ ph, int k1,
                                           int t, double sc, double *vr, double *vi) {
  constexpr int N4 = N / 4, KG = Q64Geom<N>::KG;
  const int vo = int((k1 * N * N + t) * sizeof(cplx<double>));
  const cplx<double> b1 = ph[k1];
  double P[4], Qm[4];
  static_for<0, 4>([&](auto mm) {
    constexpr int m = decltype(mm)::value;
    const cplx<double> b3 = ph[2 * N + t + N4 * m];
    const double xr = __builtin_fma(b1.re, b3.re, -(b1.im * b3.im));
    const double xi = __builtin_fma(b1.re, b3.im, b1.im * b3.re);
    // Re(b1 b2 b3) + Im(b1 b2 b3) = b2.re P + b2.im Qm
    P[m] = (xr + xi) * sc;
    Qm[m] = (xr - xi) * sc;
  });
  static_for<0, 4 * N4>([&](auto j) {
    vr[decltype(j)::value] = 0.0;
    vi[decltype(j)::value] = 0.0;
  });
  // k2 outer (each b2 serves the four pencils); the loads of KG rows are issued
  // together before their arithmetic
  static_for<0, N / KG>([&](auto gg) {
    constexpr int g0 = decltype(gg)::value * KG;
    cplx<double> v[KG][4];
    static_for<0, KG>([&](auto ii) {
      static_for<0, 4>([&](auto mm) {
        v[decltype(ii)::value][decltype(mm)::value] =
            load_c64(hr, vo, int(((g0 + decltype(ii)::value) * N + N4 * decltype(mm)::value) * sizeof(cplx<double>)));
      });
    });
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, KG>([&](auto ii) {
      constexpr int k2 = g0 + decltype(ii)::value;
      constexpr int a = k2 / N4, bb = k2 % N4;
      constexpr int e = (G * a) & 3;   // y_b += i^e c x
      const cplx<double> b2 = ph[N + k2];
      static_for<0, 4>([&](auto mm) {
        constexpr int m = decltype(mm)::value;
        constexpr int o = m * N4 + bb;
        const cplx<double> h = v[decltype(ii)::value][m];
        const double c = __builtin_fma(b2.re, P[m], b2.im * Qm[m]);
        if constexpr (e == 0) {
          vr[o] = __builtin_fma(h.re, c, vr[o]);
          vi[o] = __builtin_fma(h.im, c, vi[o]);
        } else if constexpr (e == 1) {
          vr[o] = __builtin_fma(-h.im, c, vr[o]);
          vi[o] = __builtin_fma(h.re, c, vi[o]);
        } else if constexpr (e == 2) {
          vr[o] = __builtin_fma(-h.re, c, vr[o]);
          vi[o] = __builtin_fma(-h.im, c, vi[o]);
        } else {
          vr[o] = __builtin_fma(h.im, c, vr[o]);
          vi[o] = __builtin_fma(-h.re, c, vi[o]);
        }
      });
    });
    __builtin_amdgcn_sched_barrier(0);
  });
  __builtin_amdgcn_sched_barrier(0);
  static_for<0, 4>([&](auto mm) {
    constexpr int m = decltype(mm)::value;
    static_for<0, N4>([&](auto bb) {
      constexpr int b = decltype(bb)::value;
      twiddle<N, G * b, +1, double>(vr[m * N4 + b], vi[m * N4 + b]);
    });
    fft_reg<N4, +1, double>(vr + m * N4, vi + m * N4);
  });
}

// TERM = true (launches of a few pairs, which leave most CUs idle while each
// workgroup runs its M terms one after the other): a workgroup per (pair,
// class, q) stores its u in U, laid out as A_p (term 0: its product, in A);
// k_gain_acc64 then adds the terms to A_p with the same operations in the same
// order.
template <int N, bool TERM>
__global__ __launch_bounds__(Q64Geom<N>::NL, 2) void k_gain_q64(const cplx<double> *__restrict__ H,
                                                                const cplx<double> *__restrict__ phase,
                                                                const double *__restrict__ wq,
                                                                double *__restrict__ A, cplx<double> *__restrict__ U,
                                                                long nbp, int M, int Nr, double scale) {
  using G = Q64Geom<N>;
  constexpr int N4 = G::N4, R = G::R, S = G::S;
  constexpr long n2 = long(N) * N, n3 = n2 * N;
  extern __shared__ double tile[];

  const long lb = xcd_block();
  if (lb >= nbp * 4 * (TERM ? M : 1)) return;  // uniform per workgroup
  const long bp = TERM ? lb / 4 / M : lb / 4;
  const int g = int(lb % 4);
  const long b = bp / Nr;
  const int p = int(bp % Nr);
  const int lane = threadIdx.x;
  const int k1 = lane / N4, t = lane % N4;   // stages 1 and 2
  const int u3 = lane / N, j3 = lane % N;    // stage 3: pencil (j2 = 4 u3 + g, j3)
  auto sync2 = [&]() {
    if constexpr (G::WAVE2) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
      __syncthreads();
    }
  };

  double acc[N];
  static_for<0, N>([&](auto j) { acc[decltype(j)::value] = 0.0; });
  const __amdgpu_buffer_rsrc_t hr = make_rsrc(H + b * n3, unsigned(n3 * sizeof(cplx<double>)));
  const int q0 = TERM ? int(lb / 4 % M) : 0, q1 = TERM ? q0 + 1 : M;
  for (int q = q0; q < q1; ++q) {
    const cplx<double> *ph = phase + size_t(p * M + q) * 3 * N;
    const double sc = scale * __builtin_sqrt(wq[q]);
    double vr[N], vi[N];
    switch (g) {
      case 0: q64_stage1<N, 0>(hr, ph, k1, t, sc, vr, vi); break;
      case 1: q64_stage1<N, 1>(hr, ph, k1, t, sc, vr, vi); break;
      case 2: q64_stage1<N, 2>(hr, ph, k1, t, sc, vr, vi); break;
      default: q64_stage1<N, 3>(hr, ph, k1, t, sc, vr, vi); break;
    }
    // stage 2: (k1, t) holds k3 = t + m N/4 for every u; gather all k3 of u = t.
    // The previous term's stage-3 reads cross waves: finish them first.
    __syncthreads();
    auto gather2 = [&](double *v) {
      static_for<0, 4>([&](auto mm) {
        constexpr int m = decltype(mm)::value;
        static_for<0, N4>([&](auto uu) {
          constexpr int u = decltype(uu)::value;
          tile[k1 * S + u * R + t + N4 * m] = v[m * N4 + u];
        });
      });
      sync2();
      static_for<0, N>([&](auto kk) { v[decltype(kk)::value] = tile[k1 * S + t * R + decltype(kk)::value]; });
      sync2();
    };
    gather2(vr);
    gather2(vi);
    fft_reg<N, +1, double>(vr, vi);   // axis 3: lane (k1, u = t) now holds j3 = 0..N-1
    // stage 3: gather all k1 of pencil (u3, j3)
    auto gather3 = [&](double *v) {
      static_for<0, N>([&](auto jj) { tile[k1 * S + t * R + decltype(jj)::value] = v[decltype(jj)::value]; });
      __syncthreads();
      static_for<0, N>([&](auto kk) { v[decltype(kk)::value] = tile[decltype(kk)::value * S + u3 * R + j3]; });
      __syncthreads();
    };
    gather3(vr);
    gather3(vi);
    fft_reg<N, +1, double>(vr, vi);   // axis 1: j1 = 0..N-1
    if constexpr (TERM) {
      if (q > 0) {
        cplx<double> *u = U + (bp * (M - 1) + q - 1) * n3 + long(4 * u3 + g) * N + j3;
        static_for<0, N>([&](auto j) {
          constexpr int jj = decltype(j)::value;
          u[jj * n2] = cplx<double>{vr[jj], vi[jj]};
        });
        return;
      }
    }
    static_for<0, N>([&](auto j) {
      constexpr int jj = decltype(j)::value;
      acc[jj] = __builtin_fma(vr[jj], vr[jj], acc[jj]);
      acc[jj] = __builtin_fma(-vi[jj], vi[jj], acc[jj]);
    });
    if constexpr (TERM) break;
  }
  double *a = A + bp * n3 + long(4 * u3 + g) * N + j3;
  static_for<0, N>([&](auto j) { a[decltype(j)::value * n2] = acc[decltype(j)::value]; });
}

// FP64 gain loop on chip at N = 32: one workgroup per (item, node) pair and
// class of j1; lane (v, j2) owns A_p[2v + g][j2][:] across all q.
// TERM: as for k_gain_q64, with u stored as [j3][j1][j2] (coalesced).
template <int N, bool TERM>
__global__ __launch_bounds__(C2Geom<N>::NL) void k_gain_c2(const cplx<double> *__restrict__ H,
                                                          const cplx<double> *__restrict__ phase,
                                                          const double *__restrict__ wq, double *__restrict__ A,
                                                          cplx<double> *__restrict__ U, long nbp, int M, int Nr,
                                                          double scale) {
  using Gm = C2Geom<N>;
  constexpr int NV = Gm::NV, S = Gm::S;
  constexpr long n2 = long(N) * N, n3 = n2 * N;
  extern __shared__ double tile[];

  const long lb = xcd_block();
  if (lb >= nbp * 2 * (TERM ? M : 1)) return;  // uniform per workgroup
  const long bp = TERM ? lb / 2 / M : lb / 2;
  const int g = int(lb % 2);
  const long b = bp / Nr;
  const int p = int(bp % Nr);
  const int lane = threadIdx.x;
  const int vb = lane / N, cb = lane % N;     // plane v and row j2

  double acc[N];
  static_for<0, N>([&](auto j) { acc[decltype(j)::value] = 0.0; });
  const __amdgpu_buffer_rsrc_t hr = make_rsrc(H + b * n3, unsigned(n3 * sizeof(cplx<double>)));
  const int q0 = TERM ? int(lb / 2 % M) : 0, q1 = TERM ? q0 + 1 : M;
  // the axis-1 shift factors of this term and the next behind the tile: as
  // scalar loads they overflow the scalar registers (400 of 1 876 instructions
  // a term moved them in and out of vector lanes; read again for each pencil,
  // the waits for them cost more than that)
  cplx<double> *b1s = reinterpret_cast<cplx<double> *>(tile + NV * S);
  if (lane < N) b1s[(q0 & 1) * N + lane] = phase[size_t(p * M + q0) * 3 * N + lane];
  __syncthreads();
  for (int q = q0; q < q1; ++q) {
    const cplx<double> *ph = phase + size_t(p * M + q) * 3 * N;
    const double sc = scale * __builtin_sqrt(wq[q]);
    double zr[N], zi[N];
    const cplx<double> *b1q = b1s + (q & 1) * N;
    cplx<double> b1n{};
    if (lane < N && q + 1 < q1) b1n = ph[3 * N + lane];
    c2_inverse<N>(tile, hr, ph, b1q, g, lane, sc, [&]() {
      if (lane < N && q + 1 < q1) b1s[((q + 1) & 1) * N + lane] = b1n;
    }, zr, zi);
    if constexpr (TERM) {
      if (q > 0) {
        cplx<double> *u = U + (bp * (M - 1) + q - 1) * n3 + (2 * vb + g) * N + cb;
        static_for<0, N>([&](auto j) {
          constexpr int jj = decltype(j)::value;
          u[jj * n2] = cplx<double>{zr[jj], zi[jj]};
        });
        return;
      }
    }
    static_for<0, N>([&](auto j) {
      constexpr int jj = decltype(j)::value;
      acc[jj] = __builtin_fma(zr[jj], zr[jj], acc[jj]);
      acc[jj] = __builtin_fma(-zi[jj], zi[jj], acc[jj]);
    });
    if constexpr (TERM) break;
  }
  // A_p[2v + g][j2][j3]: N consecutive doubles per lane
  double2 *a = reinterpret_cast<double2 *>(A + bp * n3 + long(2 * vb + g) * n2 + long(cb) * N);
  static_for<0, N / 2>([&](auto j) {
    constexpr int jj = decltype(j)::value;
    a[jj] = make_double2(acc[2 * jj], acc[2 * jj + 1]);
  });
}

bool gain_q64_supported(int N, int precision) { return precision == QCOLL_FP64 && (N == 16 || N == 32); }

bool use_gain_q64(const Plan &p) {
  // at N = 24 the on-chip loop is the automatic choice, not one to request
  if (p.N == 24) return p.schedule == 0 && p.precision == QCOLL_FP64 && !p.is_vss() && !p.literal;
  return p.schedule != 1 && !p.is_vss() && !p.literal && gain_q64_supported(p.N, p.precision);
}

qcoll_status launch_gain_q64(const Plan &p, const void *H, double *A, void *U, long nbp, hipStream_t st) {
  const auto *h = static_cast<const cplx<double> *>(H);
  auto *u = static_cast<cplx<double> *>(U);
  using G16 = Q64Geom<16>;
  using G32 = C2Geom<32>;
  switch (p.N) {
    case 16:
      return launch_onchip64<16, 4, 0>(p, u ? &k_gain_q64<16, true> : &k_gain_q64<16, false>, G16::NL,
                                       G16::lds_bytes, "gain q64", h, A, u, nbp, st);
    case 24: return launch_gain_cls24(p, h, A, U, nbp, st);
    case 32:
      return launch_onchip64<32, 2, 32>(p, u ? &k_gain_c2<32, true> : &k_gain_c2<32, false>, G32::NL,
                                        G32::lds_bytes, "gain c2", h, A, u, nbp, st);
    default: set_error("FP64 on-chip gain kernel: unsupported N"); return QCOLL_ENOTSUP;
  }
}

}  // namespace qcoll
