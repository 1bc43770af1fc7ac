// Boxes of the adjoint's second pass (k_vjp_gather_lds): for each field the transposed stencils read boxes
// of its cotangents around a 16x4x4 brick, staged in LDS. Which box element a lane loads, and where a thread
// finds its taps. __host__ __device__, so that the two can be checked against each other on the CPU.
#pragma once
#include <hip/hip_runtime.h>

namespace cosmos {

// Boxes (pairs a lane loads, in chunks of 64 pairs = 1 KB that one wave loads; x rows 24 wide from i0 - 4 or
// 16 wide from i0): lines along x (24x4x4), y (16x8x4), z (16x4x8); mixed differences xy (24x8x4), xz (24x4x8),
// yz (16x8x8); the full lines of kbar along all three axes (24x4x4, then the rows y -3 .. -1, 4 .. 6 and those
// of z). With n0 odd a row that reaches the seam x = n0 - 1, 0 starts one point later (24 wide) or earlier (16
// wide), so that no pair straddles it (HaloDma's rule).
enum GatherShape { SH_X, SH_Y, SH_Z, SH_XY, SH_XZ, SH_YZ, SH_K };
constexpr int kGatherChunks[7] = {3, 4, 4, 6, 6, 8, 9};
constexpr int kGatherOff[7] = {0, 1, 2, 3, 5, 7, 9};  // a lane's first offset of the shape
constexpr int kGatherOffs = 12;
// chunk j of a shape is loaded by wave (j + rot) mod 4: the loads of a field are 13, 13, 13 and 12 a wave
constexpr int kGatherRot[7] = {0, 0, 0, 0, 2, 0, 3};
// place of a box among a field's: first differences, pure second, mixed, kbar
constexpr int GB_D1[3] = {0, 384, 896}, GB_D2[3] = {1408, 1792, 2304}, GB_XY = 2816, GB_XZ = 3584, GB_YZ = 4352;
constexpr int GB_K = 5376, kGatherK = 1152, kGatherLds = GB_K + kGatherK;  // doubles
constexpr int GB_K1 = 1408, kGatherD1 = GB_K1 + kGatherK;  // kbar's place, size, with first differences only
static_assert(3 * kGatherLds * 8 <= 160 * 1024 && 2 * kGatherD1 <= kGatherLds && 5 * kGatherK <= kGatherLds, "LDS budget");

// Box coordinates of the first point of pair e of a shape: y and z relative to the brick, x from the rows'
// starts x24 and x16. Pair e is elements 2 e and 2 e + 1 of the box.
struct BoxPoint {
  int x, y, z;
};
__host__ __device__ constexpr BoxPoint gather_box_point(int s, int e, int x24, int x16) {
  if (s == SH_X || s == SH_XY || s == SH_XZ) {
    const int row = e / 12, ny = s == SH_XY ? 8 : 4;
    return {x24 + 2 * (e % 12), row % ny - (s == SH_XY ? 2 : 0), row / ny - (s == SH_XZ ? 2 : 0)};
  }
  if (s != SH_K) {
    const int row = e / 8, ny = s == SH_Z ? 4 : 8;
    return {x16 + 2 * (e % 8), row % ny - (s == SH_Z ? 0 : 2), row / ny - (s == SH_Y ? 0 : 2)};
  }
  if (e < 192) {
    const int row = e / 12;
    return {x24 + 2 * (e % 12), row % 4, row / 4};
  }
  const int q = (e - 192) % 192, in = q / 8 % 4, o = q / 32, out = o < 3 ? o - 3 : o + 1;
  return {x16 + 2 * (q % 8), e < 384 ? out : in, e < 384 ? in : out};
}

// Element of the box of each shape at the thread's point, and kbar's taps -3 .. -1, 1 .. 3 along y and z (in
// the rows of the brick or in those around it). shift24, shift16: whether the brick's rows reach the seam of
// an odd n0 (start one point later, earlier). In the latter case the last column is outside the grid and has no
// place in the 16-wide rows; its threads read the column before, inside the box, and drop what they form.
struct GatherPlace {
  int x, y, z, xy, xz, yz, k[2][6];
  __host__ __device__ constexpr GatherPlace(int tx, int ty, int tz, int shift24, int shift16)
      : x(0), y(0), z(0), xy(0), xz(0), yz(0), k{} {
    const int x24 = tx + 4 - shift24, x16 = tx + shift16 < 16 ? tx + shift16 : 15;
    x = (tz * 4 + ty) * 24 + x24, y = (tz * 8 + ty + 2) * 16 + x16, z = ((tz + 2) * 4 + ty) * 16 + x16;
    xy = (tz * 8 + ty + 2) * 24 + x24, xz = ((tz + 2) * 4 + ty) * 24 + x24, yz = ((tz + 2) * 8 + ty + 2) * 16 + x16;
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      const int o = q < 3 ? q - 3 : q - 2, yo = ty + o, zo = tz + o;
      k[0][q] = yo >= 0 && yo < 4 ? (tz * 4 + yo) * 24 + x24 : 384 + ((yo < 0 ? yo + 3 : yo - 1) * 4 + tz) * 16 + x16;
      k[1][q] = zo >= 0 && zo < 4 ? (zo * 4 + ty) * 24 + x24 : 768 + ((zo < 0 ? zo + 3 : zo - 1) * 4 + ty) * 16 + x16;
    }
  }
};

}  // namespace cosmos
