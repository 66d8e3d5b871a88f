// Workspace layouts and the autotune cache of the library on the host alone (no device): prints one
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

constexpr size_t kRoom = ~size_t(0);

static void write_cache(const char *file, const char *text) {
  FILE *fp = std::fopen(file, "w");
  if (fp) {
    std::fputs(text, fp);
    std::fclose(fp);
  }
}

// entries of another kernel kind, Nyquist convention or schedule set are not this plan's
static void check_tune_key(const char *file) {
  const qcoll::Plan vhs = plan_of(24, 8, 12, QCOLL_FP64), vss = plan_of(24, 8, 12, QCOLL_FP64, 1.5),
                    lit = plan_of(24, 8, 12, QCOLL_FP64, 1.0, true);
  int sch = -7, ck = -7;
  write_cache(file, "gfx950 s2 N=24 Nr=8 M=12 prec=0 rank=8 batch<=64|1 32\n"
                    "gfx950 s3 N=24 Nr=8 M=12 prec=0 rank=8 batch<=64|1 32\n");
  EXPECT(!qcoll::tune_cache_find(vhs, 50, kRoom, file, sch, ck), "older set");
  write_cache(file, "gfx950 s4 N=24 Nr=8 M=12 prec=0 rank=8 vss batch<=64|1 32\n"
                    "gfx950 s4 N=24 Nr=8 M=12 prec=0 rank=8 literal batch<=64|1 96\n");
  EXPECT(!qcoll::tune_cache_find(vhs, 50, kRoom, file, sch, ck), "VHS plan, VSS and literal entries");
  EXPECT(qcoll::tune_cache_find(vss, 50, kRoom, file, sch, ck) && sch == 1 && ck == 32, "%d %d", sch, ck);
  EXPECT(qcoll::tune_cache_find(lit, 50, kRoom, file, sch, ck) && sch == 1 && ck == 96, "%d %d", sch, ck);
  EXPECT(!qcoll::tune_cache_find(vss, 65, kRoom, file, sch, ck), "another batch");
  // small grids: larger candidates above 256 items, the older entries below
  const qcoll::Plan small = plan_of(8, 4, 6, QCOLL_FP32);
  write_cache(file, "gfx950 s2 N=8 Nr=4 M=6 prec=1 rank=4 batch<=256|2 192\n"
                    "gfx950 s2 N=8 Nr=4 M=6 prec=1 rank=4 batch<=512|2 256\n");
  EXPECT(qcoll::tune_cache_find(small, 256, kRoom, file, sch, ck) && sch == 2 && ck == 192, "%d %d", sch, ck);
  EXPECT(!qcoll::tune_cache_find(small, 300, kRoom, file, sch, ck), "256 items were the largest candidate");
}

// schedules that are no candidate of the plan, negative ones among them
static void check_tune_schedule(const char *file) {
  write_cache(file, "gfx950 s4 N=24 Nr=8 M=12 prec=0 rank=8 vss batch<=64|-1 64\n"
                    "gfx950 s4 N=24 Nr=8 M=12 prec=0 rank=8 vss batch<=64|0 64\n"
                    "gfx950 s4 N=24 Nr=8 M=12 prec=0 rank=8 vss batch<=64|2 64\n"
                    "gfx950 s4 N=24 Nr=8 M=12 prec=0 rank=8 batch<=64|-1 64\n"
                    "gfx950 s4 N=24 Nr=8 M=12 prec=0 rank=8 batch<=64|2 64\n"
                    "gfx950 s4 N=24 Nr=8 M=12 prec=0 rank=8 batch<=64|0 40\n");
  int sch = -7, ck = -7;
  EXPECT(!qcoll::tune_cache_find(plan_of(24, 8, 12, QCOLL_FP64, 1.5), 50, kRoom, file, sch, ck), "%d %d", sch, ck);
  EXPECT(qcoll::tune_cache_find(plan_of(24, 8, 12, QCOLL_FP64), 50, kRoom, file, sch, ck) && sch == 0 && ck == 40, "%d %d", sch,
         ck);
}

// a chunk timed in a larger workspace is no entry for one that does not hold it
static void check_tune_fit(const char *file) {
  qcoll::Plan p = plan_of(8, 4, 6, QCOLL_FP32);
  write_cache(file, "gfx950 s4 N=8 Nr=4 M=6 prec=1 rank=4 batch<=2048|2 2048\n"
                    "gfx950 s4 N=8 Nr=4 M=6 prec=1 rank=4 batch<=2048|2 256\n");
  int sch = -7, ck = -7;
  const size_t all = qcoll::make_layout(p, 2048, 0, 2048).total, part = qcoll::make_layout(p, 2048, 0, 256).total;
  EXPECT(part < all, "%zu %zu", part, all);
  EXPECT(qcoll::tune_cache_find(p, 2048, all, file, sch, ck) && ck == 2048, "%d", ck);
  EXPECT(qcoll::tune_cache_find(p, 2048, all - 1, file, sch, ck) && ck == 256, "%d", ck);
  EXPECT(qcoll::tune_cache_find(p, 2048, part, file, sch, ck) && ck == 256, "%d", ck);
  EXPECT(!qcoll::tune_cache_find(p, 2048, part - 1, file, sch, ck), "%d", ck);
}

int main(int argc, char **argv) {
  const char *what = argc > 1 ? argv[1] : "";
  if (!std::strcmp(what, "noalloc")) check_noalloc();
  else if (!std::strcmp(what, "tune_key") && argc > 2) check_tune_key(argv[2]);
  else if (!std::strcmp(what, "tune_schedule") && argc > 2) check_tune_schedule(argv[2]);
  else if (!std::strcmp(what, "tune_fit") && argc > 2) check_tune_fit(argv[2]);
  else return 2;
  if (g_fail) {
    std::printf("layouts: %d failures\n", g_fail);
    return 1;
  }
  std::printf("layouts: ok\n");
  return 0;
}
