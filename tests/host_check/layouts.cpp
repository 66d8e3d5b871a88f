// Workspace layouts of the library on the host alone (no device): prints one
// "FAILED ..." line per broken expectation and "layouts: ok" at the end.
#include <cstdio>
#include <cstring>

#include "qcoll_internal.h"

static int g_fail = 0;

#define EXPECT(cond, ...)                      \
  do {                                         \
    if (!(cond)) {                             \
      if (++g_fail < 20) {                     \
        std::printf("FAILED %s: ", #cond);     \
        std::printf(__VA_ARGS__);              \
        std::printf("\n");                     \
      }                                        \
    }                                          \
  } while (0)

static qcoll::Plan plan_of(int N, int Nr, int M, int prec, double vss = 1.0, bool literal = false) {
  qcoll::Plan p;
  p.N = N;
  p.N_rho = Nr;
  p.M = M;
  p.precision = prec;
  p.vss = vss;
  p.literal = literal;
  p.rank = p.nv = Nr;
  return p;
}

// what the two passes take in the fixed scratch, the automatic schedule takes too
static void check_noalloc() {
  for (int prec : {QCOLL_FP64, QCOLL_FP32})
    for (int N : {8, 16, 24, 32, 48})
      for (double vss : {1.0, 1.5})
        for (int Nr = 1; Nr <= 64; Nr += N == 32 ? 1 : 7)
          for (int M = 1; M <= 256; M += N == 32 ? 1 : 5) {
            qcoll::Plan p = plan_of(N, Nr, M, prec, vss);
            qcoll::Layout two, one;
            p.schedule = 1;
            const bool was = qcoll::noalloc_layout(p, 100, two);
            p.schedule = 0;
            const bool is = qcoll::noalloc_layout(p, 100, one);
            EXPECT(is || !was, "N=%d Nr=%d M=%d prec=%d vss=%g needs %zu", N, Nr, M, prec, vss, one.total);
            if (is) EXPECT(one.total <= qcoll::kScratchBytes && one.bc >= 1, "N=%d Nr=%d M=%d", N, Nr, M);
            if (is && prec == QCOLL_FP64 && N == 32 && vss != 1.0) {
              // the launch's volumes end where the parts of the spectra begin
              const size_t y = size_t(one.pc) * one.pn * ((M + 1) / 2) * 32768 * 16;
              EXPECT(one.off_y + y <= one.off_zp && one.pn >= 1 && (one.pn == Nr || one.pc == 1), "Nr=%d M=%d", Nr, M);
            }
          }
}

int main(int argc, char **argv) {
  const char *what = argc > 1 ? argv[1] : "";
  if (!std::strcmp(what, "noalloc")) check_noalloc();
  else return 2;
  if (g_fail) {
    std::printf("layouts: %d failures\n", g_fail);
    return 1;
  }
  std::printf("layouts: ok\n");
  return 0;
}
