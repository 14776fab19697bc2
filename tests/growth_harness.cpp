// Prints, for `early` additions of a large growth, a test or a new side, and `late`
// additions of a small one: what the account says of the late part and of all, each
// times kGrowth over the exact sum.
#define __host__
#define __device__
#define __forceinline__ inline
#include "growth.hpp"

#include <cstdio>
#include <cstdlib>

int main(int argc, char** argv) {
  if (argc != 6) return 2;
  const int early = atoi(argv[1]), late = atoi(argv[3]);
  const float big = (float)atof(argv[2]), small = (float)atof(argv[4]);
  const bool new_side = atoi(argv[5]) != 0;
  smre::Growth g = {0.0f, 0.0f, 0.0f};
  for (int i = 0; i < early; ++i) g.add(big);
  if (new_side) g.side_done();
  else g.tested();
  for (int i = 0; i < late; ++i) g.add(small);
  const double part = (double)g.since * smre::kGrowth / ((double)small * late);
  g.side_done();
  const double all = (double)g.total * smre::kGrowth / ((double)big * early + (double)small * late);
  printf("%.9f %.9f\n", part, all);
  return 0;
}
