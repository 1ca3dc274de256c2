// Whether BP's LDS-state kernel takes a DEM, for every team size, of circuits
// around the limit of a compute unit's LDS:
// "<circuit> <rows> <cols> <lanes> <fits> <bytes> <bytes with tables of the usual length>".
#include <cstdio>
#include <cstring>

#include "host/internal.h"

namespace tmcs {
namespace dec {
bool chunk_fits(const Dem& D, int P, size_t* lds, size_t* usual);
}
}  // namespace tmcs

int main() {
  auto run = [](const char* name, const tmcs_circuit_spec& s) {
    tmcs::Circuit c;
    tmcs::Dem d;
    if (tmcs::build_circuit(s, &c) != TMCS_OK || tmcs::build_dem(c, &d) != TMCS_OK) return false;
    for (int P = 64; P <= 1024; P += 64) {
      size_t lds = 0, usual = 0;
      const bool fits = tmcs::dec::chunk_fits(d, P, &lds, &usual);
      std::printf("%s %d %d %d %d %zu %zu\n", name, d.rows, d.cols, P, fits ? 1 : 0, lds, usual);
    }
    return true;
  };
  tmcs_circuit_spec s;
  std::memset(&s, 0, sizeof s);
  s.p = 1e-3;
  s.p_ebit = 1e-2;
  char name[64];
  // surface code, d = 9 non-local CNOT
  s.code = TMCS_SC;
  s.d = 9;
  s.op = TMCS_NONLOCAL_CNOT;
  for (int r = 28; r <= 31; ++r) {
    s.rounds_before = s.rounds_after = r;
    std::snprintf(name, sizeof name, "sc9_nlcnot_%d", r);
    if (!run(name, s)) return 1;
  }
  // [[36,4,6]] non-local CNOT: checks of up to 60 mechanisms, cut into parts
  s.code = TMCS_BB;
  s.d = 0;
  s.bb_l = 3;
  s.bb_m = 6;
  const int a[3][2] = {{1, 0}, {0, 2}, {0, 3}}, b[3][2] = {{0, 0}, {2, 0}, {0, 1}};
  std::memcpy(s.bb_a, a, sizeof a);
  std::memcpy(s.bb_b, b, sizeof b);
  for (int r = 32; r <= 36; ++r) {
    s.rounds_before = s.rounds_after = r;
    std::snprintf(name, sizeof name, "bb36_nlcnot_%d", r);
    if (!run(name, s)) return 1;
  }
  return 0;
}
