// FP64 gain loop on chip at N = 24: NC = 3 residue classes of the first output
// index, one workgroup of N^2/NC lanes (three waves) per (item, radial node)
// pair and class g (j1 = g mod NC).  It runs, for every half-sphere point q,
// u = ifft3[c_s f^] at its N/NC planes j1 and accumulates
// A_p += w_q (Re(u)^2 - Im(u)^2) there (Appendix: the product of the two shifted
// copies of f for one quadrature term).
//   stage A  lane l holds the NC pencils (k2, k3) = divmod(l + m N^2/NC, N)
//            along k1, loaded with the shift multiplier applied (consecutive
//            lanes read consecutive k3); of the inverse transform only the
//            class's outputs are used, so the compiler drops the arithmetic of
//            the others (the transform decimates in time by four: output
//            k + (N/4) t needs column k of the combine only, and NC divides N/4);
//   stage B  lane (v, k3) after a transpose across the workgroup: axis 2;
//   stage C  lane (v, j2) after a second one: axis 3, then the product; the
//            lane owns A_p[j1(v)][j2][:] across all q.
// Three waves, so that two workgroups (77 KiB of tiles and 256 registers a lane
// each) share a CU and one's barriers overlap the other's arithmetic.  The
// two-class split of N = 32 gives five waves here, of which one workgroup fits a
// CU without spilling.  Bound by VALU issue, L2 reads and LDS in turn.  360 pairs
// of 6 terms: two passes over memory 190 us, two classes 162, these 145 (171
// with the shift factors as scalar loads, whose waits also held up the LDS).
#include <hip/hip_runtime.h>

#include "qcoll_fused.hpp"

namespace qcoll {

// row stride of a plane in the tile (doubles): N^2 words (the B -> C rows of
// N + 1 words need N^2 + N - 1) rounded so that the planes of the lanes of one
// wave fall into different banks (stride = N mod 64)
constexpr int cls_stride(int N) {
  int s = N * N + N - 1;
  while (s % 64 != N % 64) ++s;
  return s;
}

template <int N, int NC>
struct ClsGeom {
  static constexpr int NV = N / NC;             // planes j1 of a class
  static constexpr int NL = N * NV;             // lanes
  static constexpr int S1 = cls_stride(N);
  // both components, two rows of b1
  static constexpr size_t lds_bytes = (size_t(2) * NV * S1 + 4 * N) * sizeof(double);
  // rows of stage-A loads in flight
  static constexpr int KG = 6;
};

// j1 of plane v of class G
template <int N, int NC, int G>
constexpr int cls_j1(int v) {
  return G + NC * (v / 4) + (N / 4) * (v % 4);
}

template <int N, int NC, int G>
__device__ __forceinline__ void cls_stage_a(__amdgpu_buffer_rsrc_t hr, const cplx<double> *__restrict__ ph,
                                            const cplx<double> *b1q, int lane, double sc, double *tr, double *ti) {
  using Gm = ClsGeom<N, NC>;
  constexpr int NV = Gm::NV, NL = Gm::NL, KG = Gm::KG;
  constexpr int n2 = N * N;
  static_for<0, NC>([&](auto mm) {
    constexpr int m = decltype(mm)::value;
    const int t = lane + m * NL;
    const cplx<double> b2 = ph[N + t / N], b3 = ph[2 * N + t % N];
    const double x = b2.re * b3.re - b2.im * b3.im;
    const double y = b2.re * b3.im + b2.im * b3.re;
    const double P = (x + y) * sc, Qm = (x - y) * sc;
    const int vo = t * int(sizeof(cplx<double>));
    double xr[N], xi[N];
    static_for<0, N / KG>([&](auto gg) {
      constexpr int k0 = decltype(gg)::value * KG;
      cplx<double> v[KG];
      static_for<0, KG>([&](auto ii) {
        v[decltype(ii)::value] = load_c64(hr, vo, (k0 + decltype(ii)::value) * n2 * int(sizeof(cplx<double>)));
      });
      __builtin_amdgcn_sched_barrier(0);
      static_for<0, KG>([&](auto ii) {
        constexpr int kk = k0 + decltype(ii)::value;
        const cplx<double> b1 = b1q[kk];
        const double c = b1.re * P + b1.im * Qm;
        xr[kk] = v[decltype(ii)::value].re * c;
        xi[kk] = v[decltype(ii)::value].im * c;
      });
    });
    fft_reg<N, +1, double>(xr, xi);
    // into the tile for A -> B, element (v, k2, k3) at v*S1 + k2*N + k3, once
    // every wave has done the previous term's last reads
    if constexpr (m == 0) __syncthreads();
    static_for<0, NV>([&](auto vv) {
      constexpr int v = decltype(vv)::value;
      tr[v * Gm::S1 + t] = xr[cls_j1<N, NC, G>(v)];
      ti[v * Gm::S1 + t] = xi[cls_j1<N, NC, G>(v)];
    });
    __builtin_amdgcn_sched_barrier(0);
  });
}

// TERM (launches of a few pairs, which leave most CUs idle while each workgroup runs
// its M terms one after the other): a workgroup per (pair, class, q) stores its u as
// [j3][j1][j2] in U (term 0: its product, in A); k_gain_acc64 then adds the terms to A_p
// with the same operations in the same order (one item, N_rho 8, M 12: eval 107 -> 65
// us, 72 in two passes before their other kernels were merged).
template <int N, int NC, bool TERM>
__global__ __launch_bounds__((ClsGeom<N, NC>::NL), 2) void k_gain_cls(const cplx<double> *__restrict__ H,
                                                                      const cplx<double> *__restrict__ phase,
                                                                      const double *__restrict__ wq,
                                                                      double *__restrict__ A,
                                                                      cplx<double> *__restrict__ U, long nbp, int M,
                                                                      int Nr, double scale) {
  using Gm = ClsGeom<N, NC>;
  static_assert(64 % N != 0, "planes straddle waves: workgroup barriers throughout");
  constexpr int NV = Gm::NV, S1 = Gm::S1;
  constexpr long n2 = long(N) * N, n3 = n2 * N;
  extern __shared__ double cls_lds[];
  double *tr = cls_lds, *ti = tr + NV * S1;

  const long lb = xcd_block();
  if (lb >= nbp * NC * (TERM ? M : 1)) return;  // uniform per workgroup
  const long bp = TERM ? lb / NC / M : lb / NC;
  const int g = int(lb % NC);
  const long b = bp / Nr;
  const int p = int(bp % Nr);
  const int lane = threadIdx.x;
  const int vb = lane / N, cb = lane % N;   // stages B and C: plane v, and k3 (B) or j2 (C)

  double acc[N];
  static_for<0, N>([&](auto j) { acc[decltype(j)::value] = 0.0; });
  const __amdgpu_buffer_rsrc_t hr = make_rsrc(H + b * n3, unsigned(n3 * sizeof(cplx<double>)));
  const int j1 = g + NC * (vb / 4) + (N / 4) * (vb % 4);
  const int q0 = TERM ? int(lb / NC % M) : 0, q1 = TERM ? q0 + 1 : M;
  // the axis-1 shift factors of this term and the next
  cplx<double> *b1s = reinterpret_cast<cplx<double> *>(cls_lds + 2 * NV * S1);
  if (lane < N) b1s[(q0 & 1) * N + lane] = phase[size_t(p * M + q0) * 3 * N + lane];
  __syncthreads();
  for (int q = q0; q < q1; ++q) {
    const cplx<double> *ph = phase + size_t(p * M + q) * 3 * N;
    const double sc = scale * __builtin_sqrt(wq[q]);
    const cplx<double> *b1q = b1s + (q & 1) * N;
    double zr[N], zi[N];
    static_for<0, NC>([&](auto gg) {
      if (g == decltype(gg)::value) cls_stage_a<N, NC, decltype(gg)::value>(hr, ph, b1q, lane, sc, tr, ti);
    });
    // the next term's factors: their slot was last read before stage A's barrier
    if (lane < N && q + 1 < q1) b1s[((q + 1) & 1) * N + lane] = ph[3 * N + lane];
    __syncthreads();
    static_for<0, N>([&](auto kk) {
      zr[decltype(kk)::value] = tr[vb * S1 + decltype(kk)::value * N + cb];
      zi[decltype(kk)::value] = ti[vb * S1 + decltype(kk)::value * N + cb];
    });
    fft_reg<N, +1, double>(zr, zi);   // axis 2: lane (v, k3) holds j2 = 0..N-1
    // B -> C inside plane v: element (j2, k3) at k3*(N+1) + j2
    __syncthreads();
    static_for<0, N>([&](auto jj) {
      tr[vb * S1 + cb * (N + 1) + decltype(jj)::value] = zr[decltype(jj)::value];
      ti[vb * S1 + cb * (N + 1) + decltype(jj)::value] = zi[decltype(jj)::value];
    });
    __syncthreads();
    static_for<0, N>([&](auto kk) {
      zr[decltype(kk)::value] = tr[vb * S1 + decltype(kk)::value * (N + 1) + cb];
      zi[decltype(kk)::value] = ti[vb * S1 + decltype(kk)::value * (N + 1) + cb];
    });
    fft_reg<N, +1, double>(zr, zi);   // axis 3: lane (v, j2) holds j3 = 0..N-1
    if constexpr (TERM) {
      if (q > 0) {
        cplx<double> *u = U + (bp * (M - 1) + q - 1) * n3 + j1 * N + cb;
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
  }
  double2 *a = reinterpret_cast<double2 *>(A + bp * n3 + j1 * n2 + long(cb) * N);
  static_for<0, N / 2>([&](auto j) {
    constexpr int jj = decltype(j)::value;
    a[jj] = make_double2(acc[2 * jj], acc[2 * jj + 1]);
  });
}

qcoll_status launch_gain_cls24(const Plan &p, const void *H, double *A, void *U, long nbp, hipStream_t st) {
  constexpr int N = 24, NC = 3;
  using G = ClsGeom<N, NC>;
  return launch_onchip64<N, NC, N>(p, U ? &k_gain_cls<N, NC, true> : &k_gain_cls<N, NC, false>, G::NL, G::lds_bytes,
                                   "gain classes", static_cast<const cplx<double> *>(H), A,
                                   static_cast<cplx<double> *>(U), nbp, st);
}

}  // namespace qcoll
