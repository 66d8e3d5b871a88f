// Body of the slab kernels over T, N, SIGN, the type Src of src, src, dst, nslab and
// QC_SLAB_TILES, which the including kernel declares: text, not a
// function, because the compiler orders an inlined function's loads differently
// (the shifted gain slab of 48^3 46.4 -> 47.0 us a launch).
  const int s = int(threadIdx.x) / N, c = int(threadIdx.x) % N;
  const long g = long(blockIdx.x) * SPB + s;
  const long gl = g < nslab ? g : nslab - 1;
  T xr[N], xi[N];
  if constexpr (grouped_loads<Src>::value) {
    constexpr int LG = (N % 16 == 0) ? 16 : ((N % 8 == 0) ? 8 : 4);
    static_for<0, N / LG>([&](auto gg) {
      constexpr int r0 = decltype(gg)::value * LG;
      decltype(src.raw(gl, 0, c)) v[LG];
      static_for<0, LG>([&](auto ii) { v[decltype(ii)::value] = src.raw(gl, r0 + decltype(ii)::value, c); });
      __builtin_amdgcn_sched_barrier(0);
      static_for<0, LG>([&](auto ii) {
        xr[r0 + decltype(ii)::value] = T(v[decltype(ii)::value].re);
        xi[r0 + decltype(ii)::value] = T(v[decltype(ii)::value].im);
      });
    });
  } else {
    static_for<0, N>([&](auto r) {
      const C<T> v = src(gl, decltype(r)::value, c);
      xr[decltype(r)::value] = v.re;
      xi[decltype(r)::value] = v.im;
    });
  }
  fft_reg<N, SIGN, T>(xr, xi);
  if constexpr (SPLIT) {
    // one tile, one component at a time: column -> row, row FFT, row -> column
    const int row = c;
    auto to_rows = [&](T *x) {
      static_for<0, N>([&](auto r) { sre[s][decltype(r)::value][c] = x[decltype(r)::value]; });
      __syncthreads();
      static_for<0, N>([&](auto k) { x[decltype(k)::value] = sre[s][row][decltype(k)::value]; });
      __syncthreads();
    };
    auto to_cols = [&](T *x) {
      static_for<0, N>([&](auto k) { sre[s][row][decltype(k)::value] = x[decltype(k)::value]; });
      __syncthreads();
      static_for<0, N>([&](auto r) { x[decltype(r)::value] = sre[s][decltype(r)::value][c]; });
      __syncthreads();
    };
    to_rows(xr);
    to_rows(xi);
    fft_reg<N, SIGN, T>(xr, xi);
    to_cols(xr);
    to_cols(xi);
    if (g < nslab) {
      static_for<0, N>([&](auto r) {
        dst(g, decltype(r)::value, c, C<T>{xr[decltype(r)::value], xi[decltype(r)::value]});
      });
    }
    return;
  } else {
    static_for<0, N>([&](auto r) {
      sre[s][decltype(r)::value][c] = xr[decltype(r)::value];
      sim[s][decltype(r)::value][c] = xi[decltype(r)::value];
    });
    __syncthreads();
    const int row = c;
    static_for<0, N>([&](auto k) {
      xr[decltype(k)::value] = sre[s][row][decltype(k)::value];
      xi[decltype(k)::value] = sim[s][row][decltype(k)::value];
    });
    fft_reg<N, SIGN, T>(xr, xi);
    static_for<0, N>([&](auto k) {
      sre[s][row][decltype(k)::value] = xr[decltype(k)::value];
      sim[s][row][decltype(k)::value] = xi[decltype(k)::value];
    });
    __syncthreads();
    if (g < nslab) {
      static_for<0, N>([&](auto r) {
        dst(g, decltype(r)::value, c, C<T>{sre[s][decltype(r)::value][c], sim[s][decltype(r)::value][c]});
      });
    }
  }
