// Host check of the rule that chooses runs of elements per work-group (test helper,
// built and run by test_rows_rule_cpu.py): reads "dim p nx ny nz n0 n1 n2
// precision" per line and prints row_runs_pay.
#include <hip/hip_runtime.h>

#include <iostream>

#include "../paper_2308_06196_amd/csrc/bgk_rows_rule.hpp"

using namespace bgk;

int main() {
  int dim, p, ne[3], n[3], precision;
  while (std::cin >> dim >> p >> ne[0] >> ne[1] >> ne[2] >> n[0] >> n[1] >> n[2] >> precision) {
    DevGeom g{};
    g.dim = dim;
    g.n1 = p + 1;
    g.ne = 1;
    g.nv = 1;
    for (int k = 0; k < 3; ++k) {
      g.nelem[k] = ne[k];
      g.ne *= ne[k];
      g.nv1[k] = n[k];
      g.nv *= n[k];
      g.vlo[k] = -6.0;
      g.du[k] = 12.0 / (n[k] - 1);
      g.scale[k] = 1.0;
    }
    g.nchunk = (int)((g.nv + kBlock - 1) / kBlock);
    g.ns = ipow(p + 1, dim);
    g.tabw = n[0] + n[1] + n[2] + 1;
    std::cout << row_runs_pay(g, precision, true) << "\n";
  }
  return 0;
}
