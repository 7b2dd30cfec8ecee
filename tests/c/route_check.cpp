// Host-side check of the library's pass selection (no GPU): which passes an
// operation takes, by grid, DOE, window and wavelengths.  Links libdop.so and
// prints one "key value" pair per line, read by tests/test_routes_cpu.py.
//
//   route_check my mx ny nx n_lambda full ...   (six numbers per problem)
//   route_check refuse      (what launch_tri must refuse before it launches)
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../include/dop.h"
#include "../../paper_2505_22313_amd/csrc/dop_internal.h"

// launch_tri of a 2048^2 DOE on 4096^2 with one field changed: 1 if refused.
template <class F>
static int refused(F change) {
  dop::KParams p{};
  p.plan = 12;
  p.n = p.nrows_in = p.nrows_out = 2048;
  p.group = 1;
  change(p);
  return dop::launch_tri(p, nullptr, nullptr) == hipErrorInvalidValue;
}

int main(int argc, char **argv) {
  if (argc == 2 && !strcmp(argv[1], "refuse")) {
    printf("group %d\n", refused([](dop::KParams &p) { p.group = 2; }));
    printf("no_group %d\n", refused([](dop::KParams &p) { p.group = 0; }));
    printf("columns %d\n", refused([](dop::KParams &p) { p.n = 2049; }));
    printf("rows %d\n", refused([](dop::KParams &p) { p.nrows_in = p.nrows_out = 2049; }));
    printf("rows_out %d\n", refused([](dop::KParams &p) { p.nrows_out = 4096; }));
    printf("full %d\n", refused([](dop::KParams &p) { p.full = 1; }));
    printf("plan %d\n", refused([](dop::KParams &p) { p.plan = 15; }));
    return 0;
  }
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
