// Gain loop of the bilinear Q(f, g) on chip (FP32, N <= 32, VHS kernels): one
// workgroup of N^2 lanes per (item, radial node) pair forms
//   A_p = sum_q w_q Re(u_f u_g),  u_h = ifft3[c_s h^]
// (Appendix: (t1_f t2_g + t2_f t1_g) / 2 of one quadrature term) and writes it
// once, where the two-pass schedule writes and reads both per-term volumes.
// Bound by VALU issue, LDS and the L2 reads of the spectra, one after the other
// more than side by side.  96 items at 32^3, N_rho 16, M 12: 4.3 ms in two
// passes, 3.45 ms with k_gain_bil, 2.76 ms with k_gain_bil2, 2.38 ms with its
// shift factors in LDS (as scalar loads their waits also held up the LDS).
//
// Per term and function, as in k_gain_fused but with the axes in the two-pass
// schedule's order, so that the two give the same bits:
//   stage A  lane (k1, k3): pencil along axis 2, loaded with the multiplier;
//   stage B  lane (k1, j2): axis 3, after a transpose inside plane k1 (inside a
//            wave when 64 is a multiple of N);
//   stage C  lane (j2, j3): axis 1, after a transpose across the workgroup; the
//            lane owns A_p[:][j2][j3].
// N < 32: both components go through LDS together, in place; 400 items x 8 nodes
// at 24^3, M 12, take 3.38 ms so, 4.27 ms with one component after the other.
// A lane's registers hold one volume and the accumulator, so u_f waits in a
// scratch volume per pair (written and read by the same lane, 16 bytes a point
// and term) while u_g is formed.
#include <hip/hip_runtime.h>

#include "qcoll_fused.hpp"

namespace qcoll {

// N < 32
template <int N>
__global__ __launch_bounds__(N *N, FusedGeom<N>::WPE) void k_gain_bil(
    const cplx<float> *__restrict__ Hf, const cplx<float> *__restrict__ Hg, const cplx<float> *__restrict__ phase,
    const float *__restrict__ wq, float *__restrict__ A, cplx<float> *S, long bp0, long nbp, int M, int Nr,
    float scale) {
  using G = FusedGeom<N>;
  static_assert(G::PPL == 1 && G::BOTH, "one pencil per lane, both components in the tile");
  constexpr long n2 = long(N) * N, n3 = n2 * N;
  extern __shared__ float lds[];

  const long lb = xcd_block();
  if (lb >= nbp) return;  // uniform per workgroup
  const long bp = bp0 + lb;
  const long b = bp / Nr;
  const int p = int(bp % Nr);
  int lane = threadIdx.x;
  asm volatile("" : "+v"(lane));   // as in k_gain_fused
  const int hi = lane / N, lo = lane % N;
  // plane k1 = hi: element (j2, k3) at k3 (N + 1) + j2, then (j2, j3) at
  // j3 (N + 1) + j2
  const TileAt<N> at{hi, lo};
  auto pa = [=](int i) { return at.c(i); };
  auto pb = [=](int i) { return at.b(i); };
  auto pc = [=](int i) { return i * G::S1 + lo * (N + 1) + hi; };

  float acc[N];
  static_for<0, N>([&](auto j) { acc[decltype(j)::value] = 0.f; });
  // scratch through a buffer descriptor: scalar element offsets, no address
  // registers kept across the term loop
  const __amdgpu_buffer_rsrc_t sr = make_rsrc(S + lb * n3, unsigned(n3 * sizeof(cplx<float>)));
  const int so = lane * int(sizeof(cplx<float>));
  for (int q = 0; q < M; ++q) {
    const cplx<float> *ph = phase + size_t(p * M + q) * 3 * N;
    static_for<0, 2>([&](auto ff) {
      constexpr int fn = decltype(ff)::value;
      // the term's factors b2 are read again for the second function instead of
      // being kept in 2 N scalar registers across the first
      asm volatile("" : "+s"(ph));
      const __amdgpu_buffer_rsrc_t hr = make_rsrc((fn ? Hg : Hf) + b * n3, unsigned(n3 * sizeof(cplx<float>)));
      float zr[1][N], zi[1][N];
      const cplx<float> b1 = ph[hi], b3 = ph[2 * N + lo];
      const float x13 = b1.re * b3.re - b1.im * b3.im, y13 = b1.re * b3.im + b1.im * b3.re;
      const float P = (x13 + y13) * scale, Q = (x13 - y13) * scale;
      static_for<0, N>([&](auto k) {
        constexpr int kk = decltype(k)::value;
        const cplx<float> v = load_c32(hr, int((hi * n2 + lo) * sizeof(cplx<float>)), int(kk * N * sizeof(cplx<float>)));
        const cplx<float> b2 = ph[N + kk];
        const float m = b2.re * P + b2.im * Q;
        zr[0][kk] = v.re * m;
        zi[0][kk] = v.im * m;
      });
      fft_reg<N, +1, float>(zr[0], zi[0]);
      // the previous volume's stage-C reads cross waves: finish them first
      __syncthreads();
      tile_put<N>(lds, zr[0], zi[0], pa);
      if constexpr (G::WAVE_BC) lds_wave_order();
      else __syncthreads();
      tile_get<N>(lds, zr[0], zi[0], pb);
      fft_reg<N, +1, float>(zr[0], zi[0]);
      tile_put<N>(lds, zr[0], zi[0], pb);
      __syncthreads();
      tile_get<N>(lds, zr[0], zi[0], pc);
      fft_reg<N, +1, float>(zr[0], zi[0]);
      if constexpr (fn == 0) {
        static_for<0, N>([&](auto j) {
          constexpr int jj = decltype(j)::value;
          typedef unsigned u2v __attribute__((ext_vector_type(2)));
          __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2v, float2{zr[0][jj], zi[0][jj]}), sr, so,
                                                int(jj * n2 * sizeof(cplx<float>)), 0);
        });
      } else {
        const float w = wq[q];
        constexpr int KG = 8 <= N && N % 8 == 0 ? 8 : 4;
        static_for<0, N / KG>([&](auto gg) {
          constexpr int j0 = decltype(gg)::value * KG;
          cplx<float> u[KG];
          static_for<0, KG>([&](auto i) { 
            u[decltype(i)::value] = load_c32(sr, so, int((j0 + decltype(i)::value) * n2 * sizeof(cplx<float>)));
          });
          __builtin_amdgcn_sched_barrier(0);
          static_for<0, KG>([&](auto i) {
            constexpr int jj = j0 + decltype(i)::value;
            const cplx<float> a = u[decltype(i)::value];
            acc[jj] += w * (a.re * zr[0][jj] - a.im * zi[0][jj]);
          });
        });
      }
    });
  }
  float *a = A + bp * n3 + lane;
  static_for<0, N>([&](auto j) { a[decltype(j)::value * n2] = acc[decltype(j)::value]; });
}

// N = 32: two workgroups of N^2/2 lanes per pair, one per parity class G of the
// second output index (j2 = G mod 2), which leaves a lane 256 registers: u_f
// stays in them while u_g is formed, and nothing of a term reaches memory.
//   stage A  lane l: the two pencils (k1, k3) = divmod(l + m N^2/2, N) along
//            axis 2; only the class's outputs are used, so the compiler drops
//            the arithmetic of the others (the transform decimates in time by
//            four: output k + 8 t needs column k of the combine only);
//   stage B  lane (k1, v), j2 = j2(v): axis 3, after a transpose of the wave's
//            own four planes k1;
//   stage C  lane (v, j3): axis 1, after a transpose across the workgroup.
// Both components go through LDS together (2 x N x N/2 x (N + 1) floats).
template <int N>
struct Bil2Geom {
  static constexpr int NV = N / 2, NL = N * NV;
  static constexpr int R = N + 1, S = NV * R;
  static constexpr size_t lds_bytes = (size_t(2) * N * S + 4 * N) * sizeof(float);   // the tiles, two rows of b2
  static constexpr int KG = 16;   // stage-A loads issued together
  static_assert(N == 32, "a wave holds four planes k1 of N/2 rows");
};

template <int N, int G>
constexpr int bil2_j2(int v) {
  return G + 2 * (v / 4) + (N / 4) * (v % 4);
}

template <int N, int G>
__device__ __forceinline__ void bil2_stage_a(__amdgpu_buffer_rsrc_t hr, const cplx<float> *__restrict__ ph,
                                             const cplx<float> *b2q, int lane, float scale, float *tr, float *ti) {
  using Gm = Bil2Geom<N>;
  constexpr int KG = Gm::KG;
  static_for<0, 2>([&](auto mm) {
    constexpr int m = decltype(mm)::value;
    const int k1 = lane / N + m * Gm::NV, k3 = lane % N;
    const cplx<float> b1 = ph[k1], b3 = ph[2 * N + k3];
    const float x13 = b1.re * b3.re - b1.im * b3.im, y13 = b1.re * b3.im + b1.im * b3.re;
    const float P = (x13 + y13) * scale, Q = (x13 - y13) * scale;
    const int vo = (k1 * N * N + k3) * int(sizeof(cplx<float>));
    float xr[N], xi[N];
    static_for<0, N / KG>([&](auto gg) {
      constexpr int k0 = decltype(gg)::value * KG;
      cplx<float> v[KG];
      static_for<0, KG>([&](auto ii) {
        v[decltype(ii)::value] = load_c32(hr, vo, int((k0 + decltype(ii)::value) * N * sizeof(cplx<float>)));
      });
      __builtin_amdgcn_sched_barrier(0);
      static_for<0, KG>([&](auto ii) {
        constexpr int kk = k0 + decltype(ii)::value;
        const cplx<float> b2 = b2q[kk];
        const float c = b2.re * P + b2.im * Q;
        xr[kk] = v[decltype(ii)::value].re * c;
        xi[kk] = v[decltype(ii)::value].im * c;
      });
    });
    fft_reg<N, +1, float>(xr, xi);
    // the previous volume's stage-C reads cross waves: finish them first
    if constexpr (m == 0) __syncthreads();
    static_for<0, Gm::NV>([&](auto vv) {
      constexpr int v = decltype(vv)::value;
      tr[k1 * Gm::S + v * Gm::R + k3] = xr[bil2_j2<N, G>(v)];
      ti[k1 * Gm::S + v * Gm::R + k3] = xi[bil2_j2<N, G>(v)];
    });
    __builtin_amdgcn_sched_barrier(0);
  });
}

template <int N>
__global__ __launch_bounds__(Bil2Geom<N>::NL, 2) void k_gain_bil2(
    const cplx<float> *__restrict__ Hf, const cplx<float> *__restrict__ Hg, const cplx<float> *__restrict__ phase,
    const float *__restrict__ wq, float *__restrict__ A, long nbp, int M, int Nr, float scale) {
  using Gm = Bil2Geom<N>;
  constexpr int S = Gm::S, R = Gm::R;
  constexpr long n2 = long(N) * N, n3 = n2 * N;
  extern __shared__ float lds[];
  float *tr = lds, *ti = lds + N * S;

  const long lb = xcd_block();
  if (lb >= nbp * 2) return;  // uniform per workgroup
  const long bp = lb / 2;
  const int g = int(lb % 2);
  const long b = bp / Nr;
  const int p = int(bp % Nr);
  const int lane = threadIdx.x;
  // stage B: row (k1, v) among the wave's planes 2w, 2w+1, 2w+N/2, 2w+1+N/2
  const int wl = lane % 64, c4 = wl / Gm::NV;
  const int k1b = 2 * (lane / 64) + (c4 & 1) + Gm::NV * (c4 >> 1);
  const int row = k1b * S + (wl % Gm::NV) * R;
  const int vc = lane / N, j3 = lane % N;   // stage C

  float acc[N];
  static_for<0, N>([&](auto j) { acc[decltype(j)::value] = 0.f; });
  // the axis-2 shift factors of this term and the next, behind the tiles
  cplx<float> *b2s = reinterpret_cast<cplx<float> *>(lds + 2 * N * S);
  if (lane < N) b2s[lane] = phase[size_t(p * M) * 3 * N + N + lane];
  __syncthreads();
  auto volume = [&](const cplx<float> *H, const cplx<float> *ph, const cplx<float> *b2q, float *zr, float *zi) {
    const __amdgpu_buffer_rsrc_t hr = make_rsrc(H + b * n3, unsigned(n3 * sizeof(cplx<float>)));
    if (g == 0) bil2_stage_a<N, 0>(hr, ph, b2q, lane, scale, tr, ti);
    else bil2_stage_a<N, 1>(hr, ph, b2q, lane, scale, tr, ti);
    // A -> B: the wave's own planes
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    static_for<0, N>([&](auto kk) {
      zr[decltype(kk)::value] = tr[row + decltype(kk)::value];
      zi[decltype(kk)::value] = ti[row + decltype(kk)::value];
    });
    fft_reg<N, +1, float>(zr, zi);   // axis 3: j3
    // B -> C: the lane's own row, read across the workgroup
    static_for<0, N>([&](auto jj) {
      tr[row + decltype(jj)::value] = zr[decltype(jj)::value];
      ti[row + decltype(jj)::value] = zi[decltype(jj)::value];
    });
    __syncthreads();
    static_for<0, N>([&](auto kk) {
      zr[decltype(kk)::value] = tr[decltype(kk)::value * S + vc * R + j3];
      zi[decltype(kk)::value] = ti[decltype(kk)::value * S + vc * R + j3];
    });
    fft_reg<N, +1, float>(zr, zi);   // axis 1: j1
  };
  for (int q = 0; q < M; ++q) {
    const cplx<float> *ph = phase + size_t(p * M + q) * 3 * N;
    const cplx<float> *b2q = b2s + (q & 1) * N;
    float fr[N], fi[N], gr[N], gi[N];
    volume(Hf, ph, b2q, fr, fi);
    // the next term's row: its slot was last read in the previous term, and the
    // barriers of the second volume order this write before its reads
    if (lane < N && q + 1 < M) b2s[((q + 1) & 1) * N + lane] = ph[4 * N + lane];
    volume(Hg, ph, b2q, gr, gi);
    const float w = wq[q];
    static_for<0, N>([&](auto j) {
      constexpr int jj = decltype(j)::value;
      acc[jj] += w * (fr[jj] * gr[jj] - fi[jj] * gi[jj]);
    });
  }
  const int j2 = g + 2 * (vc / 4) + (N / 4) * (vc % 4);
  float *a = A + bp * n3 + j2 * N + j3;
  static_for<0, N>([&](auto j) { a[decltype(j)::value * n2] = acc[decltype(j)::value]; });
}

template <int N>
static qcoll_status launch_bil(const Plan &p, const cplx<float> *Hf, const cplx<float> *Hg, float *A, cplx<float> *S,
                               long bp0, long cnt, hipStream_t st) {
  using G = FusedGeom<N>;
  if (hipFuncSetAttribute(reinterpret_cast<const void *>(&k_gain_bil<N>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, int(G::lds_bytes)) != hipSuccess) {
    set_error("hipFuncSetAttribute failed for the bilinear gain kernel");
    return QCOLL_EDEVICE;
  }
  TimedLaunch tl("gain bilinear", st);
  const float scale = float(1.0 / double(long(N) * N * N));
  hipLaunchKernelGGL((k_gain_bil<N>), dim3(unsigned(cnt)), dim3(G::NL), G::lds_bytes, st, Hf, Hg,
                     reinterpret_cast<const cplx<float> *>(p.phase), reinterpret_cast<const float *>(p.wq), A, S, bp0,
                     cnt, p.M, p.N_rho, scale);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error(std::string("gain bilinear: ") + hipGetErrorString(e));
    return QCOLL_EDEVICE;
  }
  return QCOLL_OK;
}

template <int N>
static qcoll_status launch_bil2(const Plan &p, const cplx<float> *Hf, const cplx<float> *Hg, float *A, long nbp,
                                hipStream_t st) {
  using G = Bil2Geom<N>;
  if (hipFuncSetAttribute(reinterpret_cast<const void *>(&k_gain_bil2<N>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, int(G::lds_bytes)) != hipSuccess) {
    set_error("hipFuncSetAttribute failed for the bilinear gain kernel");
    return QCOLL_EDEVICE;
  }
  TimedLaunch tl("gain bilinear", st);
  const float scale = float(1.0 / double(long(N) * N * N));
  hipLaunchKernelGGL((k_gain_bil2<N>), dim3(unsigned(nbp * 2)), dim3(G::NL), G::lds_bytes, st, Hf, Hg,
                     reinterpret_cast<const cplx<float> *>(p.phase), reinterpret_cast<const float *>(p.wq), A, nbp,
                     p.M, p.N_rho, scale);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error(std::string("gain bilinear: ") + hipGetErrorString(e));
    return QCOLL_EDEVICE;
  }
  return QCOLL_OK;
}

// the pairs in launches of at most cap (the scratch S holds cap volumes)
template <int N>
static qcoll_status launch_bil_all(const Plan &p, const cplx<float> *Hf, const cplx<float> *Hg, float *A,
                                   cplx<float> *S, long cap, long nbp, hipStream_t st) {
  for (long bp0 = 0; bp0 < nbp; bp0 += cap) {
    const qcoll_status s = launch_bil<N>(p, Hf, Hg, A, S, bp0, nbp - bp0 < cap ? nbp - bp0 : cap, st);
    if (s != QCOLL_OK) return s;
  }
  return QCOLL_OK;
}

qcoll_status launch_gain_bil(const Plan &p, const void *Hf, const void *Hg, void *A, void *S, long cap, long nbp,
                             hipStream_t st) {
  const auto *f = static_cast<const cplx<float> *>(Hf);
  const auto *g = static_cast<const cplx<float> *>(Hg);
  auto *a = static_cast<float *>(A);
  auto *s = static_cast<cplx<float> *>(S);
  switch (p.N) {
    case 8: return launch_bil_all<8>(p, f, g, a, s, cap, nbp, st);
    case 12: return launch_bil_all<12>(p, f, g, a, s, cap, nbp, st);
    case 16: return launch_bil_all<16>(p, f, g, a, s, cap, nbp, st);
    case 24: return launch_bil_all<24>(p, f, g, a, s, cap, nbp, st);
    case 32: return launch_bil2<32>(p, f, g, a, nbp, st);
    default: set_error("bilinear gain kernel: unsupported N"); return QCOLL_ENOTSUP;
  }
}

}  // namespace qcoll
