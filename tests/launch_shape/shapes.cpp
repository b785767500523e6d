// Prints what the library's launch-shape rule answers for a partial shape that gives the shots per
// block alone, at several batch sizes, beside the same block written out in full. Host code only
// (without a device the library assumes 64 KiB of LDS and 256 compute units). Test infrastructure.
//
// stdin: lines "m n dc dv regular lattice bp seq spb"; stdout: per line
// "accepted-in-full  accepted threads checks lanes  accepted threads checks lanes ..."
#include <cstdio>

#include "laim_internal.h"

using namespace laim;

int main() {
  int m, n, dc, dv, regular, lattice, bp, seq, spb;
  static const int32_t table = 0;
  while (std::scanf("%d %d %d %d %d %d %d %d %d", &m, &n, &dc, &dv, &regular, &lattice, &bp, &seq, &spb) == 9) {
    DevCode c = {};
    c.m = m;
    c.n = n;
    c.dcmax = dc;
    c.dvmax = dv;
    c.regular = regular;
    c.tile_chk = lattice ? &table : nullptr;  // (its presence alone decides)
    ResidentShape sh;
    auto runs = [&](const laim_resident_cfg& cfg, long long nshots) {
      return resident_shape(c, bp, &cfg, &sh, 0, seq != 0, true, nshots);
    };
    // In full: one check per thread up to 256 checks, two up to 512, four up to 1024 (eight on the 2D
    // toric lattice with min-sum), the next compiled number above, else the largest compiled.
    const int start = lattice && bp == 0 && !seq ? 8 : m <= 256 ? 1 : m <= 512 ? 2 : 4;
    int pick = 0;
    for (int a : {1, 2, 4, 8})
      if (runs({0, a, 1}, 0) && (pick < start)) pick = a;
    const bool full = pick > 0 && runs({(m + pick - 1) / pick, pick, spb}, 0);
    std::printf("%d", full ? 1 : 0);
    for (const long long nshots : {0ll, 1ll, 40ll, 256ll, 1024ll, 4096ll, 65536ll, 2147483647ll}) {
      const bool ok = runs({0, 0, spb}, nshots);
      std::printf("  %d %d %d %d", ok ? 1 : 0, ok ? sh.nt : 0, ok ? sh.cpt : 0, ok ? sh.lpc : 0);
    }
    std::printf("\n");
  }
  return 0;
}
