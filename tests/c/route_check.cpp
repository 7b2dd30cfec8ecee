// Host-side check of the library's pass selection (no GPU): which passes an
// operation takes, by grid, DOE, window and wavelengths.  Links libdop.so and
// prints one "key value" pair per line, read by tests/test_routes_cpu.py.
//
//   route_check my mx ny nx n_lambda full ...   (six numbers per problem)
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../include/dop.h"
#include "../../paper_2505_22313_amd/csrc/dop_internal.h"

int main(int argc, char **argv) {
  const std::vector<double> lam(DOP_MAX_LAMBDA, 0.55), nidx(DOP_MAX_LAMBDA, 1.46);
  for (int i = 1; i + 5 < argc; i += 6) {
    dop_problem p{};
    p.my = atoi(argv[i]);
    p.m = atoi(argv[i + 1]);
    p.ny = atoi(argv[i + 2]);
    p.n = atoi(argv[i + 3]);
    p.n_lambda = atoi(argv[i + 4]);
    p.out_mode = atoi(argv[i + 5]) ? DOP_OUT_FULL : DOP_OUT_CROP;
    p.dx = 0.5;
    p.z = 1000.0;
    p.lambda = lam.data();
    p.n_index = nidx.data();
    const char *names[] = {"five", "small", "tri"};
    printf("psf %s\nfield %s\ngradient %s\n", names[dop::route_of(&p, dop::IN_PHASE)],
           names[dop::route_of(&p, dop::IN_FIELD)], names[dop::route_of(&p, dop::IN_GRAD)]);
  }
  return 0;
}
