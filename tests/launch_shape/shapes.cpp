// Prints what the library's launch-shape rule answers for a shape that gives the shots per block
// alone (0: nothing at all) and a batch size, beside the same block written out in full. Host code
// only (without a device the library assumes 64 KiB of LDS and 256 compute units). Test
// infrastructure.
//
// stdin: lines "m n dc dv regular lattice bp seq spb nshots brief"; stdout: per line
// "accepted-in-full accepted threads checks lanes shots"
#include <cstdio>

#include "laim_internal.h"

using namespace laim;

int main() {
  int m, n, dc, dv, regular, lattice, bp, seq, spb, brief;
  long long nshots;
  static const int32_t table = 0;
  while (std::scanf("%d %d %d %d %d %d %d %d %d %lld %d", &m, &n, &dc, &dv, &regular, &lattice, &bp, &seq, &spb,
                    &nshots, &brief) == 11) {
    DevCode c = {};
    c.m = m;
    c.n = n;
    c.dcmax = dc;
    c.dvmax = dv;
    c.regular = regular;
    c.tile_chk = lattice ? &table : nullptr;  // (its presence alone decides)
    ResidentShape sh;
    auto runs = [&](const laim_resident_cfg& cfg, long long shots) {
      return resident_shape(c, bp, &cfg, &sh, 0, seq != 0, true, shots, brief != 0);
    };
    // In full: one check per thread up to 256 checks, two up to 512, four up to 1024 (eight on the 2D
    // toric lattice with min-sum), the next compiled number above, else the largest compiled.
    const int start = lattice && bp == 0 && !seq ? 8 : m <= 256 ? 1 : m <= 512 ? 2 : 4;
    int pick = 0;
    for (int a : {1, 2, 4, 8})
      if (runs({0, a, 1}, 0) && pick < start) pick = a;
    const bool full = pick > 0 && spb > 0 && runs({(m + pick - 1) / pick, pick, spb}, 0);
    const bool ok = runs({0, 0, spb}, nshots);
    std::printf("%d %d %d %d %d %d\n", full ? 1 : 0, ok ? 1 : 0, ok ? sh.nt : 0, ok ? sh.cpt : 0, ok ? sh.lpc : 0,
                ok ? sh.spb : 0);
  }
  return 0;
}
