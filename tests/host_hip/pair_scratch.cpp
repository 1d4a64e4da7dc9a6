// The scratch of split traces against the schedule, over lists of every length (in column tiles) of
// populations of 1 .. 40 column tiles, on devices of 64 to 256 compute units.
#include "pair_sizes.inc"

#include <cstdio>
#include <cstdlib>

int main() {
  const int shapes[][5] = {   // M, N_up, N_dn, N_g, determinants
      {8, 2, 2, 32, 1}, {25, 9, 8, 129, 1}, {33, 17, 16, 257, 1}, {46, 3, 0, 128, 1}, {64, 16, 16, 320, 8},
      {64, 16, 15, 384, 3}, {60, 30, 2, 130, 1}, {128, 32, 32, 800, 1}, {112, 28, 0, 672, 1},
      {150, 37, 37, 900, 1}, {128, 1, 32, 5000, 1}, {40, 20, 1, 40, 12}};
  for (auto& q : shapes) {
    PairTables t;
    pair_plan(t, q[0], q[1], q[2], q[3], q[4]);
    if (!t.on) return printf("no tables for M = %d\n", q[0]), 1;
    const PairDims& p = t.dim;
    for (int C = 1; C <= 40; C += C < 12 ? 1 : 7)
      for (int cus : {64, 256}) {
        const int nw = 64 * C - 3, nwg = pair_grid(p, nw, cus);
        for (int c0 = 0; c0 <= C; ++c0)
          for (int c1 = 0; c1 <= C; ++c1) {
            const PairSched r = pair_sched(p, c0, c1, nwg);
            if (r.ts == 1) continue;
            const size_t need = (size_t)p.n_det * (r.C[0] + r.C[1]) * r.ts * PAIR_W * p.G;
            const size_t have = pair_split_elems(p, nw, true);
            if (need > have)
              return printf("M = %d, %d tiles, lists %d %d: %zu of %zu\n", q[0], C, c0, c1, need, have), 1;
            if (c0 == C && c1 == C && need > pair_split_elems(p, nw, false))
              return printf("M = %d, %d tiles: whole\n", q[0], C), 1;
          }
      }
  }
  return 0;
}
