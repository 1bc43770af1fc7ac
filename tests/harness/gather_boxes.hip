// Host-side harness (tests only): the boxes of the adjoint's second pass, compiled for the CPU.
#include "gather_boxes.hpp"

using namespace cosmos;

extern "C" {
void harness_box_point(int shape, int e, int x24, int x16, int p[3]) {
  const BoxPoint b = gather_box_point(shape, e, x24, x16);
  p[0] = b.x, p[1] = b.y, p[2] = b.z;
}
// x, y, z, xy, xz, yz, then k's 12
void harness_place(int tx, int ty, int tz, int shift24, int shift16, int out[18]) {
  const GatherPlace g(tx, ty, tz, shift24, shift16);
  const int v[6] = {g.x, g.y, g.z, g.xy, g.xz, g.yz};
  for (int q = 0; q < 6; ++q) out[q] = v[q];
  for (int q = 0; q < 12; ++q) out[6 + q] = g.k[q / 6][q % 6];
}
int harness_chunks(int shape) { return kGatherChunks[shape]; }
}
