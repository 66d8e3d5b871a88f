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

#include "qcoll_fused.hpp"

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
  static constexpr int KG = 4;
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

// FP64 gain loop on chip at N = 32, two residue classes of the first output
// index (j1 = 2v + g, v < N/2): a workgroup of N^2/2 lanes (two waves per
// SIMD) runs the same sum for one (item, node) pair and one class, whose
// volume (N/2 x N x N complex doubles) is one N-point pencil per lane.  With
// k1 = (N/2) a + b,
//   u(2v + g) = sum_b e^(2 pi i b v / (N/2)) [e^(2 pi i g b / N) (X(b) + (-1)^g X(N/2 + b))].
//   stage A  lane l holds two pencils (k2, k3) = (l / N + (N/2) m, l % N),
//            m < 2, loaded along k1 with the shift multiplier applied
//            (consecutive lanes read consecutive k3), folded and transformed
//            (N/2 points): v = 0..N/2-1 each;
//   stage B  lane (v, k3) after a transpose across the workgroup: axis 2;
//   stage C  lane (v, j2) after a transpose inside the wave (a wave holds
//            whole planes v): axis 3, then the product; the lane owns
//            A_p[2v + g][j2][:] across all q.
// One component at a time through a tile of N/2 x N x (N+1) doubles (135 KiB);
// the odd row stride keeps the strided reads free of bank conflicts.
template <int N>
struct C2Geom {
  static constexpr int NV = N / 2;
  static constexpr int NL = N * N / 2;
  static constexpr int R = N + 1;
  static constexpr int S = N * R;
  static constexpr size_t lds_bytes = (size_t(NV) * S + 4 * N) * sizeof(double);   // tile, two rows of b1
  static constexpr bool WAVE_BC = (64 % N == 0);
  // stage-A outputs whose two loads each are issued together: eight loads in
  // flight (four outputs) fit beside the accumulator and the outputs; with
  // the loads of one output at a time (waits after every pair) the kernel ran
  // 12% slower, with eight outputs per group it spills 32 registers
  static constexpr int KG = 4;
};

template <int N, int G>
__device__ __forceinline__ void c2_stage_a(__amdgpu_buffer_rsrc_t hr, const cplx<double> *__restrict__ ph,
                                           const cplx<double> *b1q, int lane, double sc, double *zr, double *zi) {
  constexpr int NV = C2Geom<N>::NV, NL = C2Geom<N>::NL;
  constexpr long n2 = long(N) * N;
  static_for<0, 2>([&](auto mm) {
    constexpr int m = decltype(mm)::value;
    const int t = lane + m * NL;   // pencil (k2, k3) = (t / N, t % N)
    const cplx<double> b2 = ph[N + t / N], b3 = ph[2 * N + t % N];
    // c_s(k1) = Re(b1 b2 b3) + Im(b1 b2 b3) = b1.re P + b1.im Qm, times 1/N^3 sqrt(w_q)
    const double xr = __builtin_fma(b2.re, b3.re, -(b2.im * b3.im));
    const double yi = __builtin_fma(b2.re, b3.im, b2.im * b3.re);
    const double P = (xr + yi) * sc, Qm = (xr - yi) * sc;
    // buffer loads with the element offset as a scalar: no per-element
    // address registers to keep across the term loop.  The loads of KG
    // outputs are issued together (2 KG in flight) before their arithmetic.
    const int vo = int(t * sizeof(cplx<double>));
    constexpr int KG = C2Geom<N>::KG;
    static_for<0, NV / KG>([&](auto gg) {
      constexpr int g0 = decltype(gg)::value * KG;
      cplx<double> hl[KG], hh[KG];
      static_for<0, KG>([&](auto ii) {
        constexpr int b = g0 + decltype(ii)::value;
        hl[decltype(ii)::value] = load_c64(hr, vo, int(b * n2 * sizeof(cplx<double>)));
        hh[decltype(ii)::value] = load_c64(hr, vo, int((NV + b) * n2 * sizeof(cplx<double>)));
      });
      __builtin_amdgcn_sched_barrier(0);
      static_for<0, KG>([&](auto ii) {
      constexpr int b = g0 + decltype(ii)::value;
      const cplx<double> h0 = hl[decltype(ii)::value], h1 = hh[decltype(ii)::value];
      const cplx<double> e0 = b1q[b], e1 = b1q[NV + b];
      const double c0 = __builtin_fma(e0.re, P, e0.im * Qm), c1 = __builtin_fma(e1.re, P, e1.im * Qm);
      double yr, yim;
      if constexpr (G == 0) {
        yr = __builtin_fma(h0.re, c0, h1.re * c1);
        yim = __builtin_fma(h0.im, c0, h1.im * c1);
      } else {
        yr = __builtin_fma(h0.re, c0, -(h1.re * c1));
        yim = __builtin_fma(h0.im, c0, -(h1.im * c1));
      }
      twiddle<N, G * b, +1, double>(yr, yim);   // e^(2 pi i G b / N)
      zr[m * NV + b] = yr;
      zi[m * NV + b] = yim;
      });
      __builtin_amdgcn_sched_barrier(0);
    });
    fft_reg<NV, +1, double>(zr + m * NV, zi + m * NV);
  });
}

// TERM: as for k_gain_q64, with u stored as [j3][j1][j2] (coalesced).
template <int N, bool TERM>
__global__ __launch_bounds__(C2Geom<N>::NL) void k_gain_c2(const cplx<double> *__restrict__ H,
                                                          const cplx<double> *__restrict__ phase,
                                                          const double *__restrict__ wq, double *__restrict__ A,
                                                          cplx<double> *__restrict__ U, long nbp, int M, int Nr,
                                                          double scale) {
  using Gm = C2Geom<N>;
  constexpr int NV = Gm::NV, R = Gm::R, S = Gm::S;
  constexpr long n2 = long(N) * N, n3 = n2 * N;
  extern __shared__ double tile[];

  const long lb = xcd_block();
  if (lb >= nbp * 2 * (TERM ? M : 1)) return;  // uniform per workgroup
  const long bp = TERM ? lb / 2 / M : lb / 2;
  const int g = int(lb % 2);
  const long b = bp / Nr;
  const int p = int(bp % Nr);
  const int lane = threadIdx.x;
  const int k2a = lane / N, k3a = lane % N;   // stage A: pencils (k2a + NV m, k3a)
  const int vb = lane / N, cb = lane % N;     // stages B and C: v, and k3 (B) or j2 (C)

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
    if (g == 0) c2_stage_a<N, 0>(hr, ph, b1q, lane, sc, zr, zi);
    else c2_stage_a<N, 1>(hr, ph, b1q, lane, sc, zr, zi);
    // A -> B (across waves): element (v, k2, k3) at v*S + k2*R + k3.  The
    // previous term's stage-C reads stay inside each wave's own planes, so one
    // barrier before the writes orders them against other waves' reads (and
    // the next term's factors against this and the previous term's).
    __syncthreads();
    if (lane < N && q + 1 < q1) b1s[((q + 1) & 1) * N + lane] = b1n;
    auto a_to_b = [&](double *z, bool tail) {
      static_for<0, 2>([&](auto mm) {
        constexpr int m = decltype(mm)::value;
        static_for<0, NV>([&](auto vv) {
          constexpr int v = decltype(vv)::value;
          tile[v * S + (k2a + NV * m) * R + k3a] = z[m * NV + v];
        });
      });
      __syncthreads();
      static_for<0, N>([&](auto kk) { z[decltype(kk)::value] = tile[vb * S + decltype(kk)::value * R + cb]; });
      if (tail) __syncthreads();
    };
    a_to_b(zr, true);
    a_to_b(zi, false);
    fft_reg<N, +1, double>(zr, zi);   // axis 2: lane (v, k3) now holds j2 = 0..N-1
    // B -> C: element (v, j2, k3) at v*S + j2*R + k3; plane v belongs to the
    // N lanes of one wave (64 % N == 0), so the wave orders its own accesses.
    // Before the first write every wave must be done reading the A -> B tile.
    __syncthreads();
    auto b_to_c = [&](double *z) {
      static_for<0, N>([&](auto jj) { tile[vb * S + decltype(jj)::value * R + cb] = z[decltype(jj)::value]; });
      if constexpr (Gm::WAVE_BC) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      } else {
        __syncthreads();
      }
      static_for<0, N>([&](auto kk) { z[decltype(kk)::value] = tile[vb * S + cb * R + decltype(kk)::value]; });
      if constexpr (Gm::WAVE_BC) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      } else {
        __syncthreads();
      }
    };
    b_to_c(zr);
    b_to_c(zi);
    fft_reg<N, +1, double>(zr, zi);   // axis 3: lane (v, j2) holds j3 = 0..N-1
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

// A_p += Re(u_q)^2 - Im(u_q)^2, q = 1..M-1, from the volumes TERM stored, one
// point per lane; with N > 0 they are laid out [j3][j1][j2]
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
static qcoll_status launch_onchip64(const Plan &p, Kern kern, int lanes, size_t lds, const char *what,
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

bool gain_q64_supported(int N, int precision) { return precision == QCOLL_FP64 && (N == 16 || N == 32); }

bool use_gain_q64(const Plan &p) {
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
    case 32:
      return launch_onchip64<32, 2, 32>(p, u ? &k_gain_c2<32, true> : &k_gain_c2<32, false>, G32::NL,
                                        G32::lds_bytes, "gain c2", h, A, u, nbp, st);
    default: set_error("FP64 on-chip gain kernel: unsupported N"); return QCOLL_ENOTSUP;
  }
}

}  // namespace qcoll
