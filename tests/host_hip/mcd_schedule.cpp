// The modified Cholesky kernels on the host, launch by launch.  In the launch that finds the
// decomposition converged, and in those after it, the wavefronts of a workgroup start at
// different times: the first before and the others after another workgroup of the launch has
// recorded the end.  argv: M, delta, file of v_pqrs (M^4 doubles); prints the number of vectors
// and writes them to the file argv[4].
#include <cstdio>
#include <cstdlib>

#include "kernels_mcd.hpp"

int main(int, char** argv) {
  const int M = atoi(argv[1]), MM = M * M, nb = mcd_blocks(MM), most = 2 * MM;
  const double delta = atof(argv[2]);
  std::vector<double> eri((size_t)MM * MM), L((size_t)(most + 1) * MM, 0.0), D(MM);
  FILE* f = fopen(argv[3], "rb");
  if (!f || fread(eri.data(), 8, eri.size(), f) != eri.size()) return 2;
  fclose(f);
  std::vector<McdBest> best(2 * nb);
  std::vector<unsigned long long> dead(nb);
  McdState st{};
  for (int b = 0; b < nb; ++b)
    host_hip::run_block(b, 64, 1, [] {}, [&] {
      k_mcd_init(M, eri.data(), D.data(), dead.data(), best.data(), &st);
    });
  int after = 0;
  for (int n = 0; n < most && after < 3; ++n) {
    auto kernel = [&] {
      k_mcd_vector(M, n, delta, most, eri.data(), L.data(), D.data(), dead.data(), best.data(), &st);
    };
    // does this launch end the decomposition?  Then the workgroup that records it comes in the
    // middle of every other one.
    double top = -INFINITY;
    for (int b = 0; b < nb; ++b) top = fmax(top, best[(n & 1) * nb + b].d);
    const bool ends = !(top >= delta);
    const McdState was = st;
    const std::vector<double> D0 = D, L0(L.begin() + (size_t)n * MM, L.begin() + (size_t)(n + 1) * MM);
    for (int b = nb - 1; b >= 0; --b)
      host_hip::run_block(b, 1024, ends && b > 0 ? 1 : 16, [&] {
        if (!was.done) st = McdState{1, n, -1, 0, top};
      }, kernel);
    if (!ends && !st.done) continue;
    ++after;
    for (int mu = 0; mu < MM; ++mu)
      if (D[mu] != D0[mu] || L[(size_t)n * MM + mu] != L0[mu]) {
        printf("launch %d, after the end, wrote element %d of its vector\n", n, mu);
        return 1;
      }
    if (st.dmax != top && !was.done) return 3;
  }
  if (!st.done || after < 3) return 4;
  f = fopen(argv[4], "wb");
  fwrite(L.data(), 8, (size_t)st.count * MM, f);
  fclose(f);
  printf("%d\n", st.count);
  return 0;
}
