// Prints the kernel choice of plan descriptors, without a GPU: one line per
// input line "n0 n1 n2 prec scheme green bc[18]".
//   rc mat | lanes x points per lane of each (component, pass), "-" generic,
//   or the reason of a refusal
// Built for the host only; includes the engine for its make_geometry.
#include "../../paper_2607_05929_amd/csrc/fm_engine.hip"

#include <cstdio>

int main() {
  fm_plan_desc d;
  std::memset(&d, 0, sizeof(d));
  d.h = 1.0; d.lambda0 = 1.0; d.mu0 = 1.0; d.tol = 1e-6;
  d.max_iter = 10; d.aa_depth = 4; d.aa_period = 3; d.max_materials = 2;
  int v[6];
  while (std::scanf("%d %d %d %d %d %d", v, v + 1, v + 2, v + 3, v + 4, v + 5) == 6) {
    for (int i = 0; i < 3; ++i) d.n[i] = v[i];
    d.prec = v[3]; d.scheme = v[4]; d.green = v[5];
    int* bc = &d.bc[0][0][0];
    for (int i = 0; i < 18; ++i)
      if (std::scanf("%d", bc + i) != 1) return 1;
    Geometry g;
    const int rc = make_geometry(&d, g);
    std::printf("%d %d |", rc, rc ? 0 : g.mat);
    for (int q = 0; q < 3 && !rc; ++q)
      for (int p = 0; p < NPASS; ++p) {
        if (g.wE[q][p]) std::printf(" %dx%d", g.wN[q][p], g.wE[q][p]);
        else std::printf(" -");
      }
    std::printf(" %s\n", rc ? fm_last_error() : "");
  }
  return 0;
}
