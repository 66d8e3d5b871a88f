// Building blocks of the FP64 on-chip kernels at N = 32, two residue classes of
// the first velocity index: a workgroup of N^2/2 lanes holds one (item, node)
// pair's class, and takes a term's spectrum to its N/2 planes in velocity space.
#pragma once
#include <hip/hip_runtime.h>

#include "qcoll_fused.hpp"

namespace qcoll {

// Inverse transform of one term's c_s f^ for class g of the first output index
// (j1 = 2v + g, v < N/2): the class's volume (N/2 x N x N complex doubles) is
// one N-point pencil per lane of N^2/2 (two waves per SIMD).  With
// k1 = (N/2) a + b,
//   u(2v + g) = sum_b e^(2 pi i b v / (N/2)) [e^(2 pi i g b / N) (X(b) + (-1)^g X(N/2 + b))].
//   stage A  lane l holds two pencils (k2, k3) = (l / N + (N/2) m, l % N),
//            m < 2, loaded along k1 with the shift multiplier applied
//            (consecutive lanes read consecutive k3), folded and transformed
//            (N/2 points): v = 0..N/2-1 each;
//   stage B  lane (v, k3) after a transpose across the workgroup: axis 2;
//   stage C  lane (v, j2) after a transpose inside the wave (a wave holds
//            whole planes v): axis 3.
// One component at a time through a tile of N/2 x N x (N+1) doubles (135 KiB);
// the odd row stride keeps the strided reads free of bank conflicts.  The factors
// b1 of a term come from a two-row ring in LDS: as scalar loads their waits also
// held up the LDS (k_gain_c2, 192 items x 16 nodes, M 12: 3.49 -> 3.18 ms).
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

// stages A to C: lane (v, j2) = divmod(lane, N) ends with u(2v + g, j2, :) in
// (zr, zi).  b1q: this term's axis-1 shift factors in LDS; put_next stores the
// next term's, between two barriers of the workgroup.  Of the tile's previous
// contents only reads inside a wave's own planes may be outstanding.
template <int N, class Next>
__device__ __forceinline__ void c2_inverse(double *tile, __amdgpu_buffer_rsrc_t hr, const cplx<double> *__restrict__ ph,
                                           const cplx<double> *b1q, int g, int lane, double sc, Next put_next,
                                           double *zr, double *zi) {
  using Gm = C2Geom<N>;
  constexpr int NV = Gm::NV, R = Gm::R, S = Gm::S;
  const int k2a = lane / N, k3a = lane % N;   // stage A: pencils (k2a + NV m, k3a)
  const int vb = lane / N, cb = lane % N;     // stages B and C: v, and k3 (B) or j2 (C)
  if (g == 0) c2_stage_a<N, 0>(hr, ph, b1q, lane, sc, zr, zi);
  else c2_stage_a<N, 1>(hr, ph, b1q, lane, sc, zr, zi);
  // A -> B (across waves): element (v, k2, k3) at v*S + k2*R + k3.  The
  // previous term's stage-C reads stay inside each wave's own planes, so one
  // barrier before the writes orders them against other waves' reads (and
  // the next term's factors against this and the previous term's).
  __syncthreads();
  put_next();
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
  // B -> C: element (v, j2, k3) at v*S + j2*R + k3; plane v, also in the reads
  // above, belongs to the N lanes of one wave (64 % N == 0), so the wave orders
  // its own accesses.
  if constexpr (Gm::WAVE_BC) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
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
}

}  // namespace qcoll
