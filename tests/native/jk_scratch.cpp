// Sweeps the host plans of the Coulomb and exchange builds (csrc/kernels.h) and checks that
// what a build writes stays inside what its caller reserves.  Prints the number of
// plans looked at and exits with 1 at the first one that does not fit.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "host.h"
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

// Exchange of a density: every pair of sign counts, as chunks of KD_CH columns, at sizes
// around the tiles' edges and in all precisions
static long exchange() {
  long seen = 0, grows = 0;
  for (int prec = PREC_FP64; prec <= PREC_BF16; ++prec)
    for (int nbf : {1, 17, 31, 32, 33, 35, 45, 64, 65, 100, 127, 129, 200, 520, 700, 1100})
      for (int naux : {1, 16, 40, 157, 202, 292, 600, 3 * nbf, 5 * nbf}) {
        const JKArgs a{nullptr, nullptr, naux, nbf, tiled_cols(nbf), prec};
        const int step = nbf <= 129 ? 1 : nbf / 40;
        for (int np = 0; np <= nbf; np += step)
          for (int nn = 0; np + nn <= nbf; nn += step, ++seen) {
            if (np + nn == 0) continue;
            const size_t have = k_density_work_bytes(a, np, nn);
            for (int n : {np, nn})
              for (int c0 = 0; c0 < n; c0 += KD_CH) {
                const int r = std::min(KD_CH, n - c0);
                const size_t need = k_work_bytes(a, r);
                if (need > have) {
                  std::printf("precision %d nbf %d naux %d: %d and %d columns reserve %zu bytes, %d need %zu\n", prec,
                              nbf, naux, np, nn, have, r, need);
                  std::exit(1);
                }
                grows += need > k_work_bytes(a, std::min(KD_CH, std::max(np, nn)));
              }
          }
      }
  return grows ? seen : 0;  // the case that the larger count does not cover is among them
}

// Workspace of a fit: the raw rows in whole lines, the lists of kept tiles and L's diagonal
// have their place beside the arrays counted one by one, and leave half of the reserve
static long fit() {
  long seen = 0;
  for (int nbf : {1, 2, 3, 33, 66, 67, 300, 2002})
    for (int naux : {1, 7, 250, 5001})
      for (int flags : {0, DFX_KEEP_RAW, DFX_KEEP_METRIC, DFX_KEEP_RAW | DFX_KEEP_METRIC}) {
        HostShells b, a;
        b.nsh = b.nbf = nbf;
        a.nsh = a.nbf = naux;
        b.l.assign(nbf, 0);
        a.l.assign(naux, 0);
        const Eri3Need z = eri3_need(b, a, flags);
        const int64_t nc = (int64_t)nbf * (nbf + 1) / 2, row = (nc + 15) / 16 * 16, nt = ntiles_for(nbf);
        const int64_t raw = 8 * naux * row;  // no pair screened
        const int64_t lists = 8 * nt * ((nt + 63) / 64) + 8 * tiled_cols(nbf) / TILE2;
        const bool kept = flags & DFX_KEEP_RAW;
        const int64_t reserve = z.total - z.bottom - std::max(z.setup, z.jk + 8 * nc);
        if (z.bytes_raw + z.lines < raw || z.stays < lists + (kept ? raw - z.bytes_raw : 0) ||
            z.beside < z.stays + (raw - z.bytes_raw) + 8 * naux || reserve < 2 * z.beside ||
            reserve < (int64_t)16 << 20) {
          std::printf("nbf %d naux %d flags %d: beside %lld reserve %lld\n", nbf, naux, flags, (long long)z.beside,
                      (long long)reserve);
          std::exit(1);
        }
        ++seen;
      }
  return seen;
}

int main(int argc, char** argv) {
  const char* what = argc > 1 ? argv[1] : "";
  long n = 0;
  if (!std::strcmp(what, "coulomb")) n = coulomb();
  if (!std::strcmp(what, "exchange")) n = exchange();
  if (!std::strcmp(what, "fit")) n = fit();
  std::printf("%ld\n", n);
  return n > 0 ? 0 : 2;
}
