// Whether the wide form is taken for a regular code of m checks and n qubits: host code only. Test
// infrastructure. stdin: lines "m n dc dv bp nshots"; stdout: 0 or 1 per line.
#include <cstdio>

#include "laim_internal.h"

int main() {
  int m, n, dc, dv, bp, nshots;
  while (std::scanf("%d %d %d %d %d %d", &m, &n, &dc, &dv, &bp, &nshots) == 6) {
    laim::DevCode c = {};
    c.m = m;
    c.n = n;
    c.dcmax = dc;
    c.dvmax = dv;
    c.regular = 1;
    laim::KParams kp = {};
    kp.bp = bp;
    kp.alpha = 0.75f;
    std::printf("%d\n", laim::wide_ok(c, kp, nshots) ? 1 : 0);
  }
  return 0;
}
