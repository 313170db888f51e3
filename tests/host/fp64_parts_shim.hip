// C entry points over the FP64 contraction's rules on sizes (fp64_parts.h), built
// host-only for the CPU tests.  Test infrastructure: not part of the library.
#include "fp64_parts.h"

using namespace rbfl;

extern "C" {

// out: first, count and read_end of the variant's part, then of the rest.
void fp_parts(int K, int Kp, long long nb, int variant, long long *out) {
  EvalConsts hc{};
  hc.K = K;
  hc.Kp = Kp;
  const Fp64Parts p = fp64_parts(hc, nb, variant, false);
  const long long v[6] = {p.main.first, p.main.count, p.main.read_end, p.rest.first, p.rest.count, p.rest.read_end};
  for (int i = 0; i < 6; ++i) out[i] = v[i];
}

long long fp_rows_ld(long long n) { return rows_ld(n); }

}  // extern "C"
