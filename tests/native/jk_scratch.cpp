// Sweeps the host plans of the Coulomb and exchange builds (csrc/kernels.h) and checks that
// what a build writes stays inside what its caller reserves.  Prints the number of
// plans looked at and exits with 1 at the first one that does not fit.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "kernels.h"

using namespace dfx;

// Coulomb: every number of tiles (nt tile rows), of kept ones among them, and naux to 6 nbf
static long coulomb() {
  long seen = 0;
  for (int nt = 1; nt <= 50; ++nt) {
    const int nbf = TILE * nt, all = nt * (nt + 1) / 2;
    const int64_t ncols = tiled_cols(nbf);
    for (int naux = 1; naux <= 6 * nbf; naux += 1 + naux / 256) {
      const size_t jw = j_work_bytes(nbf, naux, ncols), gw = j_gamma_work_bytes(nbf, naux, ncols);
      for (int kept = 0; kept <= all; ++kept, ++seen) {
        const JPlan p = j_plan(naux, ncols, kept);
        // the parts cover all tiles and all auxiliary functions
        const bool whole = p.sg >= 1 && p.sb >= 1 && (int64_t)p.sg * p.tchunk >= kept && (int64_t)p.sb * p.qchunk >= naux;
        const int64_t g = 8 * j_gamma_reach(p, naux, ncols), j = 8 * j_build_reach(p, naux, ncols, kept);
        if (!whole || g > (int64_t)gw || g > (int64_t)jw || j > (int64_t)jw) {
          std::printf("nbf %d naux %d kept %d of %d: gamma %lld of %zu bytes, J %lld of %zu\n", nbf, naux, kept, all,
                      (long long)g, gw, (long long)j, jw);
          std::exit(1);
        }
      }
    }
  }
  return seen;
}

int main(int argc, char** argv) {
  const char* what = argc > 1 ? argv[1] : "";
  long n = 0;
  if (!std::strcmp(what, "coulomb")) n = coulomb();
  std::printf("%ld\n", n);
  return n > 0 ? 0 : 2;
}
