// LDS-staged stage kernel: a 512-thread workgroup owns a BX x BY x BZ brick of 256 points with two
// threads per point in two roles, one wave of each role on every SIMD:
//   curvature waves (0-3)  stage the halo boxes, and form from them the second derivatives, the
//       connection, the Ricci tensor, D_iD_j alpha and the Gt^i source: everything that ends in
//       X_ij = -D_iD_j alpha + alpha (R_ij - 8 pi S_ij), its trace-free part, and Gt^i;
//   transport waves (4-7)  form shift advection and dissipation of every field, the fluid and
//       the remaining algebra, and run the RK4 epilogue.
// The whole point evaluation in one thread needs about 470 registers, so one wave per SIMD, whose
// dependent FP64 operations and LDS reads nothing covers: a lone brick of a 16^3 grid, all data in
// cache, took 25 us, nearly the 31 us per brick of a full 256^3 grid. Split by role, each half fits
// 256 registers and the SIMD issues from one wave while the other waits; what the halves owe each
// other is 8 values one way (inverse metric, pressure, 1 / X) and 10 the other, exchanged in LDS.
//
// The 25 fields are visited two per barrier interval in a fixed order (kPairOrder), chosen so that
// the two roles have about equal work in each: the connection algebra runs while the transport
// waves advect At_ij, and X_ij is handed over before the last fields. A field's halo box (brick
// plus width 3, the ghost-zone fill done as an index wrap in the load offsets) goes straight from
// HBM into a ring of three interval slots by LDS-direct loads, two intervals ahead. The curvature
// waves issue no other memory operations in steady state, so a count of their newer loads tells
// when a field has landed; the transport waves' epilogue operands, flux neighbours and stores
// have their own counters and never delay the ring. A workgroup walks several bricks; the next
// brick's first fields, point values and recovery are done during the current one's last intervals.
// The fluid fluxes come from the previous stage (or a pointwise pre-pass) and are differentiated
// from global loads.
//
// The arithmetic is that of bssn_rhs_stream in bssn_device.hpp; only where operands come from, and
// the order of a few sums, differs, so the two variants agree to rounding.
#pragma once
#include "bssn_device.hpp"

namespace cosmos {

// Workgroup barrier for LDS staging. __syncthreads() carries a workgroup-scope release fence,
// which waits for every outstanding global load and store of the wave (s_waitcnt vmcnt(0)) and so
// drains the prefetch of later fields and epilogue operands at every phase. Here only the wave's
// own LDS operations are completed (lgkmcnt 0: its halo writes are visible and its reads of a
// buffer about to be refilled have returned) before s_barrier; global memory is not ordered.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0); vmcnt and expcnt not waited on
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Brick of round `it` for workgroup `blk` in the XCD-blocked order (T.order 2, set up by the
// launcher): XCD blk % 8 owns a slab of T.zr brick layers, and its workgroups take one
// T.gx x T.gy x T.gz block of bricks per round. False when the workgroup's slot lies outside the
// grid's bricks in this round.
__device__ __forceinline__ bool blocked_brick(const Tile& T, int it, int blk, int& bxi, int& byi, int& bzi) {
  const int l = blk >> 3, gxy = T.ngx * T.ngy;
  bxi = (it % T.ngx) * T.gx + l % T.gx;
  byi = ((it / T.ngx) % T.ngy) * T.gy + (l / T.gx) % T.gy;
  const int bzl = (it / gxy) * T.gz + l / (T.gx * T.gy);
  bzi = (blk & 7) * T.zr + bzl;
  return bxi < T.nbx && byi < T.nby && bzl < T.zr && bzi < T.nbz;
}

// Stencil taps read from the LDS halo box: c points at the thread's centre.
template <class B>
__device__ __forceinline__ void lds_line(const double* c, int a, double v[7]) {
  const int st = a == 0 ? 1 : (a == 1 ? B::SY : B::SZ);
#pragma unroll
  for (int o = 0; o < 7; ++o) v[o] = c[(o - 3) * st];
}

// Stencil taps of one field in registers. Taps are loaded one batch ahead of the arithmetic that uses
// them, with a scheduling fence after every batch: left to itself the compiler reads two or three taps
// at a time and waits for each, about a dozen LDS latencies per field with second derivatives.
__device__ __forceinline__ void fence() { __builtin_amdgcn_sched_barrier(0); }
struct Lines {  // offsets -3..+3 along each axis (only the used ones are loaded)
  double v[3][7];
};
template <class B>
__device__ __forceinline__ void lines_load(const double* c, Lines& l) {
#pragma unroll
  for (int a = 0; a < 3; ++a) lds_line<B>(c, a, l.v[a]);
}
struct Cross {  // the 16 taps of a mixed derivative, [offset along a][offset along b] of -2, -1, 1, 2
  double v[4][4];
};
template <class B>
__device__ __forceinline__ void cross_load(const double* c, int a, int b, Cross& x) {
  const int sa = a == 0 ? 1 : (a == 1 ? B::SY : B::SZ);
  const int sb = b == 0 ? 1 : (b == 1 ? B::SY : B::SZ);
  const int o[4] = {-2, -1, 1, 2};
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int q = 0; q < 4; ++q) x.v[p][q] = c[o[p] * sa + o[q] * sb];
}
__device__ __forceinline__ double cross_value(const Cross& x, double i144) {
  double in[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) in[p] = (x.v[p][0] - x.v[p][3]) + 8.0 * (x.v[p][2] - x.v[p][1]);
  return ((in[0] - in[3]) + 8.0 * (in[2] - in[1])) * i144;
}
// Mixed derivatives without the 16 taps each, on bricks whose x-rows are the wave's rows of 16 lanes:
// the inner first difference (along y for xy, along z for xz and yz) at the four neighbours of the
// outer one is what other lanes of the wave hold already. Only the columns x = -2, -1, 16, 17 (xy, xz)
// and, on 16 x 4 bricks, the rows y = -2, -1, 4, 5 (yz) lie outside the wave: 4 taps a lane instead of
// 16. The batches of fields with second derivatives are bound by the LDS reads (111-116 B/clk per CU):
// 61 -> 25 values a point, stage kernel at 256^3 5.84 -> 5.64 ms, 96^3 308 -> 299 us, 32^3
// 21.6 -> 20.2 us, constraints at 128^3 485 -> 440 us a call. Same operations on the same values as cross_value, so the same bits. Every lane of
// the wave must be active; brick points beyond the grid take part with their staged (wrapped) values.
struct Edge {
  double v[4];  // taps -2, -1, 1, 2 of the inner difference at the lane's outside column or row
};
// Lanes 0, 1, 14, 15 of a row stand for the columns -2, -1, 16, 17; the other lanes' taps are not used.
template <class B>
__device__ __forceinline__ void columns_load(const double* c, int b, Edge& e) {
  const int sb = b == 1 ? B::SY : B::SZ;
  const double* o = c + ((threadIdx.x & 15) < 8 ? -2 : 2);
  const int t[4] = {-2, -1, 1, 2};
#pragma unroll
  for (int q = 0; q < 4; ++q) e.v[q] = o[t[q] * sb];
}
// Lane rows 0, 1, 2, 3 stand for y = -2, -1, 4, 5.
template <class B>
__device__ __forceinline__ void rows_load(const double* c, Edge& e) {
  const double* o = c + ((threadIdx.x & 32) ? 2 : -2) * B::SY;
  const int t[4] = {-2, -1, 1, 2};
#pragma unroll
  for (int q = 0; q < 4; ++q) e.v[q] = o[t[q] * B::SZ];
}
// x of the lane that the lane shift CTRL selects in the same row of 16, or `edge` where it has none
template <int CTRL>
__device__ __forceinline__ double lane_shift(double x, double edge) {
  const long long a = __double_as_longlong(x), e = __double_as_longlong(edge);
  const int lo = __builtin_amdgcn_update_dpp((int)e, (int)a, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(e >> 32), (int)(a >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double((long long)(unsigned)lo | (long long)hi << 32);
}
// rows (a0 a1 a2 a3), (b0 b1 b2 b3) -> (a0 a1 b0 b1), (a2 a3 b2 b3)
__device__ __forceinline__ void swap_halves(double& a, double& b) {
  const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  a = __longlong_as_double((long long)((unsigned long long)hi[0] << 32 | lo[0]));
  b = __longlong_as_double((long long)((unsigned long long)hi[1] << 32 | lo[1]));
}
// rows (a0 a1 a2 a3), (b0 b1 b2 b3) -> (a0 b0 a2 b2), (a1 b1 a3 b3)
__device__ __forceinline__ void swap_rows(double& a, double& b) {
  const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  a = __longlong_as_double((long long)((unsigned long long)hi[0] << 32 | lo[0]));
  b = __longlong_as_double((long long)((unsigned long long)hi[1] << 32 | lo[1]));
}
// the inner difference: v is the point's own line along the inner axis
__device__ __forceinline__ double inner_own(const double v[7]) { return (v[1] - v[5]) + 8.0 * (v[4] - v[2]); }
__device__ __forceinline__ double inner_edge(const Edge& e) { return (e.v[0] - e.v[3]) + 8.0 * (e.v[2] - e.v[1]); }
__device__ __forceinline__ double columns_value(const double v[7], const Edge& e, double i144) {
  const double own = inner_own(v), two = inner_edge(e);
  const double one = lane_shift<0xB1>(two, two);  // neighbouring lanes swapped: columns -1, 16 in lanes 0, 15
  const double m2 = lane_shift<0x112>(own, two), m1 = lane_shift<0x111>(own, one);  // from lanes - 2, - 1
  const double p1 = lane_shift<0x101>(own, one), p2 = lane_shift<0x102>(own, two);  // from lanes + 1, + 2
  return ((m2 - p2) + 8.0 * (p1 - m1)) * i144;
}
__device__ __forceinline__ double rows_value(const double v[7], const Edge& e, double i144) {
  const double own = inner_own(v), out = inner_edge(e);  // rows o0 o1 o2 o3; e0 e1 e2 e3
  double m2 = out, s = own, r = own, p2 = out;
  swap_halves(m2, s);                                    // m2 = e0 e1 o0 o1
  swap_halves(r, p2);                                    // p2 = o2 o3 e2 e3
  double m1 = own, p1 = own;
  swap_rows(m1, p1);                                     // o0 o0 o2 o2; o1 o1 o3 o3
  double a = m2, b = p2;
  swap_rows(a, m1);                                      // m1 = e1 o0 o1 o2
  swap_rows(p1, b);                                      // p1 = o1 o2 o3 e2
  return ((m2 - p2) + 8.0 * (p1 - m1)) * i144;
}
// Which mixed derivatives of a brick are formed so; the others take cross_load's 16 taps.
template <class B>
constexpr bool kByColumns = B::X == 16;
template <class B>
constexpr bool kByRows = B::X == 16 && B::Y == 4;

// First and (SECOND) pure second derivatives from the lines.
template <bool SECOND>
__device__ __forceinline__ void lines_derivs(const Lines& l, const DevParams& P, FieldDerivs& r) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double none = 0.0;
    op_line<SECOND, false, false>(l.v[a], 0.0, P.i12h[a], P.i12h2[a], 0.0, 0.0, r.d1[a], SECOND ? r.d2[S(a, a)] : none, none);
  }
}
// All derivatives of one staged field: first (and SECOND: pure and mixed second) derivatives and, with
// ADV / KO, shift advection and dissipation.
template <class B, bool SECOND, bool ADV, bool KO>
__device__ __forceinline__ void lds_derivs(const double* c, const DevParams& P, const double beta[3], FieldDerivs& r) {
  static_assert(!SECOND || kByRows<B>, "16 x 4 bricks");
  Lines l;
  Edge e1, e2, e3;
  lines_load<B>(c, l);
  if constexpr (SECOND) {
    columns_load<B>(c, 1, e1);
    columns_load<B>(c, 2, e2);
    rows_load<B>(c, e3);
  }
  fence();
  double acc = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double d2 = 0.0;
    op_line<SECOND, ADV, KO>(l.v[a], beta[a], P.i12h[a], P.i12h2[a], P.i24h[a], P.iko[a], r.d1[a], d2, acc);
    if (SECOND) r.d2[S(a, a)] = d2;
  }
  r.advko = acc;
  if constexpr (SECOND) {
    r.d2[S(0, 1)] = columns_value(l.v[1], e1, P.i144[0]);
    r.d2[S(0, 2)] = columns_value(l.v[2], e2, P.i144[1]);
    r.d2[S(1, 2)] = rows_value(l.v[2], e3, P.i144[2]);
  }
}

// Halo box for staging by LDS-direct loads: x runs from i0 - 4 to i0 + BX + 3 (BX + 8 points,
// one more on each side than the stencils need), so that with n0 even every aligned pair of
// x-neighbours (2m, 2m + 1) of the box is two consecutive doubles in memory, 16-byte aligned,
// also where the box wraps around the periodic boundary. One lane moves one such pair per load
// (buffer_load_dwordx4 into LDS), NR rounds of 256 pairs per field.
template <int BX, int BY, int BZ>
struct DBrick {
  static constexpr int X = BX, Y = BY, Z = BZ;
  static constexpr int XO = 4;
  static constexpr int HX = BX + 8, HY = BY + 6, HZ = BZ + 6;
  static constexpr int NPR = HX / 2;                 // pairs per row
  static constexpr int NPAIR = NPR * HY * HZ;
  static constexpr int NR = (NPAIR + 255) / 256;     // load rounds per field
  static constexpr int NP = NR * 512;                // doubles per LDS buffer (padded to whole rounds)
  static constexpr int SY = HX, SZ = HX * HY;
  static constexpr int NOFF = 2 * NR;  // two offset sets: fields with and without second derivatives
  static_assert(BX * BY * BZ == 256 && BX % 2 == 0, "one point per thread, even brick width");
};

// The same as an instruction immediate chosen at compile time: at most N outstanding.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt has 6 bits");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}
// Wait until at most n vector-memory operations of this wave are outstanding (expcnt and
// lgkmcnt not waited on). Loads complete in issue order, so a load is complete once n newer
// ones have been issued and the count drops to n.
__device__ __forceinline__ void wait_vm(int n) {
  switch (n) {  // the count is an instruction immediate
    case 0: __builtin_amdgcn_s_waitcnt(0x0F70); break;
    case 5: __builtin_amdgcn_s_waitcnt(0x0F75); break;
    case 10: __builtin_amdgcn_s_waitcnt(0x0F7A); break;
    default: __builtin_amdgcn_s_waitcnt(0x0F70); break;  // any other count: wait for everything
  }
}

// LDS-direct halo staging: each lane loads one pair of x-neighbours per round, straight into an LDS
// buffer (round q of wave w fills pairs [256 q + 64 w, 256 q + 64 w + 64)); no registers hold the data.
// Which box points a lane loads is fixed, in box coordinates: box points that no stencil reads stand
// for a point of a cache line the brick reads anyway, so that only the lines the stencils use are
// requested, with two sets of them. Fields with second derivatives read x-halo points in rows within
// +-2 of the brick in y and z with the other coordinate inside (mixed xy and xz derivatives; +-3 axial
// ones in rows inside in both), the other rows only over the brick's x-range (y and z stencils, mixed
// yz ones within +-2 in both), and the box's corner rows not at all. Fields with first derivatives
// only read the x-halo in rows inside in y and z, the brick's x-range in rows inside in one of them.
// The coordinates are packed five bits each, both sets in one word per round, formed once per launch,
// so a brick costs a few multiply-adds per offset, plus the periodic wrap only where its box crosses
// the grid's faces.
//
// A pair must not straddle the seam between x = n0 - 1 and x = 0. With n0 even the box starts at the
// even i0 - 4 and no pair does. With n0 odd the seam at the upper face falls inside a pair there, so a
// box that reaches it starts one point later (shift 1; its stencils need no more than i0 - 3). One seam
// per box is assumed: n0 >= BX + 5, for the widest brick 21 (halo_fits). Pairs are 8-byte aligned only, then and for any base
// address, which the LDS-direct loads take (checked on the device at every offset).
constexpr bool halo_fits(int n0) { return n0 % 2 == 0 || n0 >= 21; }
template <class B>
struct HaloDma {
  static_assert(B::HX <= 32 && B::HY <= 32 && B::HZ <= 32, "five bits a coordinate");
  uint32_t box[B::NR];    // second-derivative set in the low half, first-derivative set in the high half
  uint32_t off[B::NOFF];  // byte offsets in a field: [0, NR) the first set, [NR, 2 NR) the second
  static __device__ __forceinline__ int shift(int i0, int n0) { return (n0 & 1) && i0 - 4 + B::HX > n0 ? 1 : 0; }
  __device__ __forceinline__ void init(int n0) {
    const int first = n0 & 1 ? 1 : 2;  // pairs [first, NPR - 3] cover the brick's x-range (with either shift)
#pragma unroll
    for (int q = 0; q < B::NR; ++q) {
      const int e = (threadIdx.x & 255) + 256 * q;
      const int ee = e < B::NPAIR ? e : 0;  // padding lanes load an in-box pair into the padding
      const int hx = ee % B::NPR, y = (ee / B::NPR) % B::HY, z = ee / (B::NPR * B::HY);
      const int dy = y - 3, dz = z - 3;
      const bool yin = dy >= 0 && dy < B::Y, zin = dz >= 0 && dz < B::Z;
      const bool y2 = dy >= -2 && dy < B::Y + 2, z2 = dz >= -2 && dz < B::Z + 2;
      const int hi = min(max(hx, first), B::NPR - 3);  // the pair moved into the brick's x-range
      const int yc = min(max(dy, 0), B::Y - 1) + 3;    // the row moved inside the brick in y
      const bool xh2 = (y2 && zin) || (yin && z2), row2 = yin || zin || (y2 && z2);
      const bool xh1 = yin && zin, row1 = yin || zin;
      const uint32_t second = 2 * (xh2 ? hx : hi) | (row2 ? y : yc) << 5 | z << 10;
      const uint32_t first1 = 2 * (xh1 ? hx : hi) | (row1 ? y : yc) << 5 | z << 10;
      box[q] = second | first1 << 16;
    }
  }
  // x in [-n, 3n) to its place in [0, n): the unsigned minimum keeps x - n only where it is not negative
  static __device__ __forceinline__ int wrap(int x, int n) {
    uint32_t u = (uint32_t)(x + n);
    u = min(u, u - (uint32_t)n);
    u = min(u, u - (uint32_t)n);
    u = min(u, u - (uint32_t)n);
    return (int)u;
  }
  __device__ __forceinline__ void locate(int i0, int j0, int k0, const int n[3]) {
    // opaque per brick: the unpacked coordinates are formed here, not kept (and spilled) across bricks
#pragma unroll
    for (int q = 0; q < B::NR; ++q) asm volatile("" : "+v"(box[q]));
    const int x0 = i0 - 4 + shift(i0, n[0]), y0 = j0 - 3, z0 = k0 - 3;
    if (x0 >= 0 && x0 + B::HX <= n[0] && y0 >= 0 && y0 + B::HY <= n[1] && z0 >= 0 && z0 + B::HZ <= n[2]) {  // uniform
      const uint32_t base = (uint32_t)(x0 + n[0] * (y0 + n[1] * z0));
#pragma unroll
      for (int q = 0; q < B::NOFF; ++q) {
        const uint32_t b = box[q % B::NR] >> (q < B::NR ? 0 : 16);
        off[q] = 8u * (base + (b & 31) + (uint32_t)n[0] * (((b >> 5) & 31) + (uint32_t)n[1] * ((b >> 10) & 31)));
      }
    } else {
#pragma unroll
      for (int q = 0; q < B::NOFF; ++q) {
        const uint32_t b = box[q % B::NR] >> (q < B::NR ? 0 : 16);
        const int x = wrap(x0 + (int)(b & 31), n[0]), y = wrap(y0 + (int)((b >> 5) & 31), n[1]);
        const int z = wrap(z0 + (int)((b >> 10) & 31), n[2]);
        off[q] = 8u * (uint32_t)(x + n[0] * (y + n[1] * z));
      }
    }
  }
  // one field's halo box by four waves: SECOND selects the set of the fields with second derivatives
  __device__ __forceinline__ void fetch(const double* F, uint32_t nbytes, double* buf, bool second = true) const {
    const __amdgpu_buffer_rsrc_t r = field_rsrc(F, nbytes);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int q = 0; q < B::NR; ++q)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          r, (__attribute__((address_space(3))) void*)(buf + 2 * (256 * q + 64 * w)), 16, off[second ? q : B::NR + q], 0, 0, 0);
  }
};

// the thread's point in the brick's halo boxes
template <class B>
__device__ __forceinline__ int box_index(int i0, int n0) {
  const int pt = threadIdx.x & 255;
  return (pt % B::X + B::XO - HaloDma<B>::shift(i0, n0)) +
         B::SY * (((pt / B::X) % B::Y + 3) + B::HY * (pt / (B::X * B::Y) + 3));
}

// ---------------------------------------------------------------- the two roles of the stage kernel
constexpr int kPairThreads = 512;  // waves 0-3: curvature waves, waves 4-7: transport waves, one point per thread of each
constexpr int kIntervals = 13;     // barrier intervals per brick, two fields each (the last one)
// Fields of interval i: kPairOrder[2 i] and kPairOrder[2 i + 1].
constexpr int kPairOrder[2 * kIntervals] = {
    F_BET, F_BET + 1, F_BET + 2, F_GT,  F_GT + 1, F_GT + 2, F_GT + 3, F_GT + 4, F_GT + 5, F_GAM, F_GAM + 1, F_GAM + 2, F_AT,
    F_AT + 1, F_AT + 2, F_AT + 3, F_CHI, F_AT + 4, F_ALP, F_AT + 5, F_K, F_ET, F_ST, F_ST + 1, F_ST + 2, -1};
// Fields with second and mixed derivatives: the shift, the conformal metric, chi and the lapse.
constexpr bool pair_second(int f) {
  return (f >= F_GT && f < F_GT + 6) || (f >= F_BET && f < F_BET + 3) || f == F_CHI || f == F_ALP;
}
constexpr int pair_fields(int i) { return kPairOrder[2 * i + 1] < 0 ? 1 : 2; }

// LDS of a workgroup: a ring of three interval slots of two halo boxes each, then the exchange
// (kExSlots values per point).
constexpr int kExSlots = 10;
// exchange, written in the last interval of the previous brick and read in interval 0 ...
constexpr int EX_GI = 0, EX_P = 6, EX_IX = 7;
// ... written in interval 9 (lapse), read in 10 and 11: chi (X_ij - gt_ij X / 3), D^i D_i alpha ...
constexpr int EX_Y = 0, EX_D2A = 6;
// ... written in interval 10, read in 11: the Gt^i right-hand side without advection and dissipation
constexpr int EX_RG = 7;
template <class B>
struct PairRing {
  static constexpr int FULL = B::NPAIR / 256;                   // load rounds of all four waves
  static constexpr int LASTW = (B::NPAIR % 256 + 63) / 64;      // waves of the last, partial round
  static constexpr int PB = 2 * (256 * FULL + 64 * LASTW);      // doubles per halo box
  static constexpr int LDS = 6 * PB + kExSlots * 256;  // the sink's parked values, if any, follow
  static_assert(LDS * 8 <= 160 * 1024, "LDS budget");
  // One field's halo box into LDS by the curvature waves: FULL loads per lane, one more in the
  // first LASTW waves.
  static __device__ __forceinline__ void fetch(const double* F, uint32_t nbytes, double* buf, const uint32_t* off) {
    const __amdgpu_buffer_rsrc_t r = field_rsrc(F, nbytes);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int q = 0; q < FULL; ++q)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          r, (__attribute__((address_space(3))) void*)(buf + 2 * (256 * q + 64 * w)), 16, off[q], 0, 0, 0);
    if (LASTW && w < LASTW)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          r, (__attribute__((address_space(3))) void*)(buf + 2 * (256 * FULL + 64 * w)), 16, off[FULL], 0, 0, 0);
  }
  // Wait until at most K newer fields' loads of this (curvature) wave are outstanding.
  template <int K>
  static __device__ __forceinline__ void wait() {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (LASTW && w < LASTW)
      wait_vmcnt<K*(FULL + 1)>();
    else
      wait_vmcnt<K * FULL>();
  }
};

// What a stage does for one brick, uniform over the workgroup: the arrays and field size of its
// grid, the stage's time and RK4 weights, and the brick's origin.
struct StageItem {
  const double *U, *un;
  double *acc, *out;
  const double* F;  // point fluxes (or KT divergence) of U
  double* Fn;       // where the point fluxes of `out` go (FUSE)
  size_t fs;
  double t, ca, cn;
  int i0, j0, k0;
};
template <class B>
__device__ __forceinline__ int pair_point(const StageItem& m, const int n[3], bool& active) {
  const int pt = threadIdx.x & 255;
  const int i = m.i0 + pt % B::X, j = m.j0 + (pt / B::X) % B::Y, k = m.k0 + pt / (B::X * B::Y);
  active = i < n[0] && j < n[1] && k < n[2];
  return active ? i + n[0] * (j + n[1] * k) : 0;
}
template <class B>
__device__ __forceinline__ void flux_neighbours(const StageItem& m, const int n[3], int c, uint32_t fo[3][4]) {
  constexpr int d[4] = {-2, -1, 1, 2};
  const int st[3] = {1, n[0], n[0] * n[1]};
  if (m.i0 >= 2 && m.i0 + B::X + 2 <= n[0] && m.j0 >= 2 && m.j0 + B::Y + 2 <= n[1] && m.k0 >= 2 &&
      m.k0 + B::Z + 2 <= n[2]) {  // uniform
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int o = 0; o < 4; ++o) fo[a][o] = 8u * (uint32_t)(c + d[o] * st[a]);
  } else {
    const int pt = threadIdx.x & 255;  // a thread outside the grid takes the neighbours of point 0, as c does
    const int q[3] = {m.i0 + pt % B::X, m.j0 + (pt / B::X) % B::Y, m.k0 + pt / (B::X * B::Y)};
    const bool in = q[0] < n[0] && q[1] < n[1] && q[2] < n[2];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int x = in ? q[a] : 0;
#pragma unroll
      for (int o = 0; o < 4; ++o) fo[a][o] = 8u * (uint32_t)(c + (wrap1(x + d[o], n[a]) - x) * st[a]);
    }
  }
}
// Loads for the divergence of conserved variable q: its fluxes at the neighbours, or (KT) the
// divergence the pre-pass left.
template <bool KT>
__device__ __forceinline__ void pair_flux_load(const double* F, size_t fs, int c, const uint32_t fo[3][4], int q,
                                               double v[3][4]) {
  const uint32_t nb = (uint32_t)(fs * 8);
  if constexpr (KT) {
    v[0][0] = bld(field_at(F, q, fs), nb, (uint32_t)c * 8u);
  } else {
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int o = 0; o < 4; ++o) v[a][o] = bld(field_at(F, 4 * a + q, fs), nb, fo[a][o]);
  }
}
__device__ __forceinline__ int ring_next(int s) { return s == 2 ? 0 : s + 1; }
__device__ __forceinline__ int ring_prev(int s) { return s == 0 ? 2 : s - 1; }
// keeps the value in a register here: the arithmetic that forms it stays on this side of the next barrier
__device__ __forceinline__ void pin(double& x) { asm volatile("" : "+v"(x)); }
template <int I>
using iv = std::integral_constant<int, I>;

// The derivatives of an interval's two fields, K0 and K1 = 0 (not differentiated), 1 (first) or 2
// (first and second): use0 / use1 take each as soon as it is there; between() runs while the first
// taps arrive.
template <class B, int K0, int K1, class Between, class Use0, class Use1>
__device__ __forceinline__ void pair_derivs(const double* c0, const double* c1, const DevParams& P, Between between,
                                            Use0 use0, Use1 use1) {
  constexpr bool columns = kByColumns<B>, rows = kByRows<B>;
  Lines l;
  Edge e1, e2, e3;
  Cross x, y;
  FieldDerivs d, e;
  auto load_first = [&](const double* c) {
    lines_load<B>(c, l);
    if constexpr (columns) {
      columns_load<B>(c, 1, e1);
      columns_load<B>(c, 2, e2);
    }
    if constexpr (rows) rows_load<B>(c, e3);
  };
  auto mixed = [&](const double* c, FieldDerivs& r) {  // the taps of the yz derivative follow into x
    if constexpr (columns) {
      if constexpr (!rows) {
        cross_load<B>(c, 1, 2, x);
        fence();
      }
      r.d2[S(0, 1)] = columns_value(l.v[1], e1, P.i144[0]);
      r.d2[S(0, 2)] = columns_value(l.v[2], e2, P.i144[1]);
      if constexpr (rows) r.d2[S(1, 2)] = rows_value(l.v[2], e3, P.i144[2]);
    } else {
      cross_load<B>(c, 0, 1, x);
      cross_load<B>(c, 0, 2, y);
      fence();
      r.d2[S(0, 1)] = cross_value(x, P.i144[0]);
      cross_load<B>(c, 1, 2, x);
      fence();
      r.d2[S(0, 2)] = cross_value(y, P.i144[1]);
    }
  };
  if constexpr (K0 == 2)
    load_first(c0);
  else
    lines_load<B>(c0, l);
  fence();
  between();
  fence();
  lines_derivs<K0 == 2>(l, P, d);
  if constexpr (K0 == 2) mixed(c0, d);
  // the second field's lines are on their way while the first one's last derivative is formed and used
  if constexpr (K1 == 2)
    load_first(c1);
  else if constexpr (K1 == 1)
    lines_load<B>(c1, l);
  fence();
  if constexpr (K0 == 2 && !rows) d.d2[S(1, 2)] = cross_value(x, P.i144[2]);
  use0(d);
  if constexpr (K1 != 0) {
    fence();
    lines_derivs<K1 == 2>(l, P, e);
    if constexpr (K1 == 2) {
      mixed(c1, e);
      if constexpr (!rows) e.d2[S(1, 2)] = cross_value(x, P.i144[2]);
    }
    use1(e);
  }
}

// First derivatives and the advection + dissipation of one field (the arithmetic of op_line with
// the weights formed once per point).
__device__ __forceinline__ void lines_transport(const Lines& l, const DevParams& P, const double wo[3],
                                                const double wd[3], FieldDerivs& r) {
  double acc = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double* v = l.v[a];
    const double t1 = v[4] - v[2], t2 = v[5] - v[1];
    r.d1[a] = (8.0 * t1 - t2) * P.i12h[a];
    const double s1 = v[4] + v[2], s2 = v[5] + v[1];
    const double d6 = ((v[6] + v[0]) - 6.0 * s2) + (15.0 * s1 - 20.0 * v[3]);
    const double odd = ((v[6] - v[0]) - 6.0 * t2) + 21.0 * t1;
    acc += wo[a] * odd;
    acc += wd[a] * d6;
  }
  r.advko = acc;
}

// Dissipation alone (the fluid of the centred scheme).
__device__ __forceinline__ void lines_dissipation(const Lines& l, const DevParams& P, FieldDerivs& r) {
  double acc = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double d1, d2;
    op_line<false, false, true>(l.v[a], 0.0, 0.0, 0.0, 0.0, P.iko[a], d1, d2, acc);
  }
  r.advko = acc;
}

// Curvature waves. Seq walks the workgroup's bricks: first(m) / next(m) give the brick's StageItem
// (false: none), P() the parameters of the run the last one belongs to, fail(bool) counts a point's
// failed fluid recovery.
template <class B, int SC, class Seq>
__device__ __forceinline__ void curvature_waves(Seq& seq, double* smem) {
  using R = PairRing<B>;
  double* ex = smem + 6 * R::PB + threadIdx.x;
  HaloDma<B> halo;
  StageItem m;
  if (!seq.first(m)) return;  // uniform; the transport waves leave too
  double gi[6];
  double cv[11];  // chi, gt_ij, Et, St_i at the next brick's point
  bool act;
  // the point values of a brick, then its inverse metric and fluid recovery, handed to the transport waves
  auto point_load = [&](const StageItem& q, const int n[3]) {
    const uint32_t nb = (uint32_t)(q.fs * 8), c = 8u * (uint32_t)pair_point<B>(q, n, act);
    cv[0] = bld(field_at(q.U, F_CHI, q.fs), nb, c);
#pragma unroll
    for (int s = 0; s < 6; ++s) cv[1 + s] = bld(field_at(q.U, F_GT + s, q.fs), nb, c);
#pragma unroll
    for (int s = 0; s < 4; ++s) cv[7 + s] = bld(field_at(q.U, F_ET + s, q.fs), nb, c);
    COSMOS_PHASE();
  };
  double S3[3], Pr, iX;
  auto point_setup = [&](double w) {
    asm volatile("" : "+v"(w));  // 1 + w and 4 w are formed here, not kept (and spilled) across bricks
    inv_sym(cv + 1, gi);
    Fluid fl;
    seq.fail(recover(w, cv[0], gi, cv[7], cv + 8, fl) && act);
#pragma unroll
    for (int s = 0; s < 6; ++s) ex[(EX_GI + s) * 256] = gi[s];
    ex[EX_P * 256] = Pr = fl.P;
    ex[EX_IX * 256] = iX = fl.invX;
#pragma unroll
    for (int q = 0; q < 3; ++q) S3[q] = fl.S[q];
  };
  auto issue = [&](auto I, const StageItem& q, int slot) {  // the fields of interval I of brick q
    constexpr int i = decltype(I)::value;
    const uint32_t nb = (uint32_t)(q.fs * 8);
    double* buf = smem + slot * (2 * R::PB);
#pragma unroll
    for (int k = 0; k < pair_fields(i); ++k) {
      const int f = kPairOrder[2 * i + k];
      R::fetch(field_at(q.U, f, q.fs), nb, buf + k * R::PB, pair_second(f) ? halo.off : halo.off + B::NR);
    }
  };
  int slot = 0;
  point_load(m, seq.P().n);
  halo.init(seq.P().n[0]);
  halo.locate(m.i0, m.j0, m.k0, seq.P().n);
  issue(iv<0>(), m, 0);
  issue(iv<1>(), m, 1);
  point_setup(seq.P().w);
  R::template wait<2>();
  lds_barrier();
  for (;;) {
    const DevParams P = seq.P();
    const int cidx = box_index<B>(m.i0, P.n[0]);
    StageItem nx;
    const double* cur;  // halo box of the interval's first field, at the thread's point
    auto begin = [&](auto I) {
      constexpr int i = decltype(I)::value;
      if constexpr (i + 2 < kIntervals)
        issue(iv<i + 2>(), m, ring_prev(slot));
      else
        issue(iv<i + 2 - kIntervals>(), nx, ring_prev(slot));
    };
    auto end = [&](auto I) {  // the next interval's fields have landed once only the newer ones remain
      constexpr int i = decltype(I)::value;
      R::template wait<pair_fields((i + 2) % kIntervals)>();
      lds_barrier();
      slot = ring_next(slot);
      cur = smem + slot * (2 * R::PB) + cidx;
      fence();
    };
    double DB[9], RG[3] = {0.0, 0.0, 0.0}, RX[6], G[18], gt[6];
    auto shift = [&](int i, const FieldDerivs& d) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        DB[3 * i + a] = d.d1[a];
        pin(DB[3 * i + a]);
      }
      RG[i] += contract_sym(gi, d.d2);
#pragma unroll
      for (int l = 0; l < 3; ++l) {
        RG[l] += (gi[S(l, 0)] * d.d2[S(0, i)] + gi[S(l, 1)] * d.d2[S(1, i)] + gi[S(l, 2)] * d.d2[S(2, i)]) * (1.0 / 3.0);
        pin(RG[l]);
      }
    };
    auto metric = [&](int s, const FieldDerivs& d) {  // d_a gt_ij kept, -1/2 gt^lm d_l d_m gt_ij into R_ij
      RX[s] = -0.5 * contract_sym(gi, d.d2);
      pin(RX[s]);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        G[3 * s + a] = d.d1[a];
        pin(G[3 * s + a]);
      }
    };
    auto conn = [&](int k, const FieldDerivs& d) {  // gt_k(i d_j) Gt^k into R_ij
#pragma unroll
      for (int s = 0; s < 6; ++s) {
        const int i = SI(s), j = SJ(s);
        RX[s] += 0.5 * (gt[S(k, i)] * d.d1[j] + gt[S(k, j)] * d.d1[i]);
        pin(RX[s]);
      }
    };
    using D = const FieldDerivs&;
    auto put = [&](auto I) { return [&, I] { begin(I); }; };  // this interval's loads two intervals ahead
    cur = smem + slot * (2 * R::PB) + cidx;
    pair_derivs<B, 2, 2>(cur, cur + R::PB, P, put(iv<0>()), [&](D d) { shift(0, d); }, [&](D d) { shift(1, d); });
    end(iv<0>());
    gt[0] = cur[R::PB];
    pair_derivs<B, 2, 2>(cur, cur + R::PB, P, put(iv<1>()), [&](D d) { shift(2, d); }, [&](D d) { metric(0, d); });
    end(iv<1>());
    gt[1] = cur[0], gt[2] = cur[R::PB];
    pair_derivs<B, 2, 2>(cur, cur + R::PB, P, put(iv<2>()), [&](D d) { metric(1, d); }, [&](D d) { metric(2, d); });
    end(iv<2>());
    gt[3] = cur[0], gt[4] = cur[R::PB];
    pair_derivs<B, 2, 2>(cur, cur + R::PB, P, put(iv<3>()), [&](D d) { metric(3, d); }, [&](D d) { metric(4, d); });
    end(iv<3>());
    gt[5] = cur[0];
    pair_derivs<B, 2, 1>(cur, cur + R::PB, P, put(iv<4>()), [&](D d) { metric(5, d); }, [&](D d) { conn(0, d); });
    end(iv<4>());
    pair_derivs<B, 1, 1>(cur, cur + R::PB, P, put(iv<5>()), [&](D d) { conn(1, d); }, [&](D d) { conn(2, d); });
    double Gl[3][6];
    {
      double dgt[6][3];
#pragma unroll
      for (int q = 0; q < 18; ++q) dgt[q / 3][q % 3] = G[q];
      connection_lower(dgt, Gl);
#pragma unroll
      for (int q = 0; q < 18; ++q) pin(Gl[q / 6][q % 6]);
    }
    end(iv<5>());
    double At[6], Gu[3][6], Gd[3];
    begin(iv<6>());
    At[0] = cur[0];
    At[1] = cur[R::PB];
    connection_raise(Gl, gi, Gu, Gd);
#pragma unroll
    for (int q = 0; q < 18; ++q) pin(Gu[q / 6][q % 6]);
#pragma unroll
    for (int k = 0; k < 3; ++k) pin(Gd[k]);
    end(iv<6>());
    double xij[6], xj[3];
    begin(iv<7>());
    At[2] = cur[0];
    At[3] = cur[R::PB];
    ricci_quadratic(Gl, gi, Gu, Gd, RX);
#pragma unroll
    for (int s = 0; s < 6; ++s) pin(RX[s]);
    end(iv<7>());
    double dchi[3], ichi, chi;
    // The scalar field's sources, an interval before their use; issued before the interval's halo loads,
    // so the counted waits cover them.
    bool inside;
    const uint32_t cb = SC != 0 ? 8u * (uint32_t)pair_point<B>(m, P.n, inside) : 0u;
    if constexpr (SC != 0) {
#pragma unroll
      for (int q = 0; q < 6; ++q) xij[q] = bld(field_at(seq.xsrc(), SRC_SIJ + q, m.fs), (uint32_t)(m.fs * 8), cb);
      COSMOS_PHASE();
    }
    At[4] = cur[R::PB];
    chi = cur[0];
    pair_derivs<B, 2, 0>(cur, nullptr, P, put(iv<8>()), [&](D d) {
      ichi = 1.0 / chi;
      ricci_conformal_factor(ichi, d.d1, d.d2, gt, gi, Gu, RX);
#pragma unroll
      for (int s = 0; s < 6; ++s) pin(RX[s]);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        dchi[a] = d.d1[a];
        pin(dchi[a]);
      }
    }, [](D) {});
    end(iv<8>());
    double dal[3], alpha;
    if constexpr (SC != 0) {
#pragma unroll
      for (int q = 0; q < 3; ++q) xj[q] = bld(field_at(seq.xsrc(), SRC_S + q, m.fs), (uint32_t)(m.fs * 8), cb);
      COSMOS_PHASE();
    }
    At[5] = cur[R::PB];
    alpha = cur[0];
    pair_derivs<B, 2, 0>(cur, nullptr, P, put(iv<9>()), [&](D d) {
      double cda = 0.0;
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int l = 0; l < 3; ++l) cda += gi[S(k, l)] * dchi[k] * d.d1[l];
      const double ih = 0.5 * ichi;
      double DDa[6], X[6];
#pragma unroll
      for (int s = 0; s < 6; ++s) {
        const int i = SI(s), j = SJ(s);
        DDa[s] = (d.d2[s] - (Gu[0][s] * d.d1[0] + Gu[1][s] * d.d1[1] + Gu[2][s] * d.d1[2])) +
                 ih * ((dchi[i] * d.d1[j] + dchi[j] * d.d1[i]) - gt[s] * cda);
      }
      ex[EX_D2A * 256] = chi * contract_sym(gi, DDa);
#pragma unroll
      for (int s = 0; s < 6; ++s) {
        double Sij = S3[SI(s)] * S3[SJ(s)] * iX + Pr * gt[s] * ichi;
        if constexpr (SC != 0) Sij += xij[s];
        X[s] = -DDa[s] + alpha * (RX[s] - 8.0 * PI_D * Sij);
      }
      const double trX3 = contract_sym(gi, X) * (1.0 / 3.0);
#pragma unroll
      for (int s = 0; s < 6; ++s) ex[(EX_Y + s) * 256] = chi * (X[s] - gt[s] * trX3);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        dal[a] = d.d1[a];
        pin(dal[a]);
      }
    }, [](D) {});
    end(iv<9>());
    pair_derivs<B, 1, 0>(cur, nullptr, P, put(iv<10>()), [&](D d) {  // Gt^i: every term but advection and dissipation
      double Amix[3][3], Aup[6];
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int j = 0; j < 3; ++j) Amix[k][j] = gi[S(k, 0)] * At[S(0, j)] + gi[S(k, 1)] * At[S(1, j)] + gi[S(k, 2)] * At[S(2, j)];
#pragma unroll
      for (int s = 0; s < 6; ++s) {
        const int i = SI(s), j = SJ(s);
        Aup[s] = Amix[i][0] * gi[S(0, j)] + Amix[i][1] * gi[S(1, j)] + Amix[i][2] * gi[S(2, j)];
      }
      const double divb = DB[0] + DB[4] + DB[8];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        double r = RG[i];
        r -= (4.0 / 3.0) * alpha * (gi[S(i, 0)] * d.d1[0] + gi[S(i, 1)] * d.d1[1] + gi[S(i, 2)] * d.d1[2]);
        r -= Gd[0] * DB[3 * i + 0] + Gd[1] * DB[3 * i + 1] + Gd[2] * DB[3 * i + 2];
        r += (2.0 / 3.0) * Gd[i] * divb;
        r -= 2.0 * (Aup[S(i, 0)] * dal[0] + Aup[S(i, 1)] * dal[1] + Aup[S(i, 2)] * dal[2]);
        double inner = contract_sym(Gu[i], Aup);
        inner -= (1.5 * ichi) * (Aup[S(i, 0)] * dchi[0] + Aup[S(i, 1)] * dchi[1] + Aup[S(i, 2)] * dchi[2]);
        r += 2.0 * alpha * inner;
        double Sj[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          Sj[j] = S3[j];
          if constexpr (SC != 0) Sj[j] += xj[j];
        }
        r -= 16.0 * PI_D * alpha * (gi[S(i, 0)] * Sj[0] + gi[S(i, 1)] * Sj[1] + gi[S(i, 2)] * Sj[2]);
        ex[(EX_RG + i) * 256] = r;
      }
    }, [](D) {});
    end(iv<10>());
    // the next brick: its point values (older than its halo loads) and offsets
    if (!seq.next(nx)) {  // none: the transport waves' last two intervals
      R::template wait<0>();
      lds_barrier();
      lds_barrier();
      return;
    }
    point_load(nx, seq.P().n);
    halo.locate(nx.i0, nx.j0, nx.k0, seq.P().n);
    begin(iv<11>());
    end(iv<11>());
    begin(iv<12>());
    point_setup(seq.P().w);
    end(iv<12>());
    m = nx;
  }
}

// Transport waves: see the file's head. Sink<...> is the stage's epilogue.
template <class B, bool KT, int SC, class Sink, class Seq>
__device__ __forceinline__ void transport_waves(Seq& seq, double* smem) {
  using R = PairRing<B>;
  using Pre = typename Sink::Pre;
  const double* ex = smem + 6 * R::PB + (threadIdx.x & 255);
  double* nvals = smem + R::LDS + (threadIdx.x & 255);  // the sink's parked values
  StageItem m;
  if (!seq.first(m)) return;  // uniform; the curvature waves leave too
  double cen[NF];
  bool active;
  int c = pair_point<B>(m, seq.P().n, active);
  auto centre_load = [&](const StageItem& q, int cp) {
    const uint32_t nb = (uint32_t)(q.fs * 8);
#pragma unroll
    for (int f = 0; f < NF; ++f) cen[f] = bld(field_at(q.U, f, q.fs), nb, 8u * (uint32_t)cp);
  };
  centre_load(m, c);
  int slot = 0;
  lds_barrier();
  for (;;) {
    const DevParams P = seq.P();
    const int cidx = box_index<B>(m.i0, P.n[0]);
    Sink sink(m, c, active, P.alpha_collapse, nvals);
    const double* cur;
    auto end = [&](auto) {
      lds_barrier();
      slot = ring_next(slot);
      __builtin_amdgcn_sched_barrier(0);
    };
    const double chi = cen[F_CHI], K = cen[F_K], alpha = cen[F_ALP];
    const double c32 = chi * sqrt(chi), im32 = 1.0 / c32, ichi = 1.0 / chi;
    double gt[6], beta[3], At[6], Gam[3], Sl[3], Sup[3];
#pragma unroll
    for (int s = 0; s < 6; ++s) gt[s] = cen[F_GT + s], At[s] = cen[F_AT + s];
    const double E = c32 * cen[F_ET];
#pragma unroll
    for (int q = 0; q < 3; ++q) beta[q] = cen[F_BET + q], Gam[q] = cen[F_GAM + q], Sl[q] = c32 * cen[F_ST + q];
    // the inverse metric stays in the exchange (until interval 9) and is read where it is used
    auto inverse = [&](double gi[6]) {
#pragma unroll
      for (int s = 0; s < 6; ++s) gi[s] = ex[(EX_GI + s) * 256];
    };
    const double Pr = ex[EX_P * 256], iX = ex[EX_IX * 256];
    {
      double gi[6];
      inverse(gi);
#pragma unroll
      for (int j = 0; j < 3; ++j) Sup[j] = chi * (gi[S(j, 0)] * Sl[0] + gi[S(j, 1)] * Sl[1] + gi[S(j, 2)] * Sl[2]);
    }
    // shift advection and dissipation along axis a: wo[a] odd differences + wd[a] 6th difference
    double wo[3], wd[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      wo[a] = beta[a] * P.i24h[a];
      wd[a] = fabs(beta[a]) * P.i24h[a];
      wd[a] += P.iko[a];
      pin(wo[a]);
      pin(wd[a]);
    }
    auto Sjk_at = [&](int s) { return Sup[SI(s)] * Sup[SJ(s)] * iX + Pr * chi * ex[(EX_GI + s) * 256]; };

    double DB[9], SG[3] = {0.0, 0.0, 0.0};
    // right-hand sides waiting for their epilogue operand (stored one interval later)
    using Hold = typename Sink::Hold;
    Hold rb[3], rg[6], ag[3], pa[6];
    Pre eb[3], eg[6];
    auto keep = [&](Hold& h, double k, double uc) {
      h = sink.hold(k, uc);
      pin(h.a);
    };
    Lines l0, l1;
    auto load0 = [&] {  // the interval's first field; the second with load1, at once where registers allow
      cur = smem + slot * (2 * R::PB) + cidx;
      lines_load<B>(cur, l0);
      fence();
    };
    auto load1 = [&] {
      lines_load<B>(cur + R::PB, l1);
      fence();
    };
    auto load2 = [&] {
      load0();
      load1();
    };
    auto shift = [&](int i, const Lines& l) {
      FieldDerivs d;
      lines_transport(l, P, wo, wd, d);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        DB[3 * i + a] = d.d1[a];
        pin(DB[3 * i + a]);
      }
      double r = 0.0;
      if (P.evolve_shift) r = d.advko + (0.75 * Gam[i] - P.eta * beta[i]);
      keep(rb[i], r, l.v[0][3]);
    };
    auto metric = [&](int s, const Lines& l) {
      FieldDerivs d;
      lines_transport(l, P, wo, wd, d);
      const double wsym = (s == 0 || s == 3 || s == 5) ? 1.0 : 2.0;
      const double Sjk = Sjk_at(s);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        SG[a] += wsym * Sjk * d.d1[a];
        pin(SG[a]);
      }
      const int i = SI(s), j = SJ(s);
      const double divb = DB[0] + DB[4] + DB[8];
      double r = d.advko;
#pragma unroll
      for (int k = 0; k < 3; ++k) r += gt[S(i, k)] * DB[3 * k + j] + gt[S(j, k)] * DB[3 * k + i];
      r -= (2.0 / 3.0) * gt[s] * divb;
      r -= 2.0 * alpha * At[s];
      keep(rg[s], r, l.v[0][3]);
    };
    auto gamma = [&](int k, const Lines& l) {
      FieldDerivs d;
      lines_transport(l, P, wo, wd, d);
      keep(ag[k], d.advko, l.v[0][3]);
    };
    load0();
    eb[0] = sink.preload(F_BET);
    eb[1] = sink.preload(F_BET + 1);
    fence();
    shift(0, l0);
    load1();
    shift(1, l1);
    end(iv<0>());
    load2();
    eb[2] = sink.preload(F_BET + 2);
    eg[0] = sink.preload(F_GT);
    sink.put(F_BET, rb[0], eb[0]);
    sink.put(F_BET + 1, rb[1], eb[1]);
    fence();
    shift(2, l0);
    metric(0, l1);
    end(iv<1>());
    load2();
    eg[1] = sink.preload(F_GT + 1);
    eg[2] = sink.preload(F_GT + 2);
    sink.put(F_BET + 2, rb[2], eb[2]);
    sink.put(F_GT, rg[0], eg[0]);
    fence();
    metric(1, l0);
    metric(2, l1);
    end(iv<2>());
    load2();
    eg[3] = sink.preload(F_GT + 3);
    eg[4] = sink.preload(F_GT + 4);
    sink.put(F_GT + 1, rg[1], eg[1]);
    sink.put(F_GT + 2, rg[2], eg[2]);
    fence();
    metric(3, l0);
    metric(4, l1);
    end(iv<3>());
    load2();
    eg[5] = sink.preload(F_GT + 5);
    sink.put(F_GT + 3, rg[3], eg[3]);
    sink.put(F_GT + 4, rg[4], eg[4]);
    fence();
    metric(5, l0);
    gamma(0, l1);
    end(iv<4>());
    double Amix[3][3], AK, EpS, KS = 0.0, sgt = 0.0;
    load2();
    sink.put(F_GT + 5, rg[5], eg[5]);
    fence();
    gamma(1, l0);
    gamma(2, l1);
    {  // the point algebra of the trace-K and fluid equations: S^jk K_jk and S^jk gt_jk, and K's source
#pragma unroll
      for (int s = 0; s < 6; ++s) {
        const double Sjk = Sjk_at(s), wS = (s == 0 || s == 3 || s == 5 ? 1.0 : 2.0) * Sjk;
        KS += wS * ((At[s] + gt[s] * K * (1.0 / 3.0)) * ichi);
        sgt += wS * gt[s];
      }
      pin(KS);
      pin(sgt);
      double gi[6];
      inverse(gi);
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          Amix[k][j] = gi[S(k, 0)] * At[S(0, j)] + gi[S(k, 1)] * At[S(1, j)] + gi[S(k, 2)] * At[S(2, j)];
          pin(Amix[k][j]);
        }
      double Aup[6];
#pragma unroll
      for (int s = 0; s < 6; ++s) {
        const int i = SI(s), j = SJ(s);
        Aup[s] = Amix[i][0] * gi[S(0, j)] + Amix[i][1] * gi[S(1, j)] + Amix[i][2] * gi[S(2, j)];
      }
      const double AA = contract_sym(At, Aup);
      const double Str = (Sup[0] * Sl[0] + Sup[1] * Sl[1] + Sup[2] * Sl[2]) * iX + 3.0 * Pr;
      AK = AA + K * K * (1.0 / 3.0);
      EpS = E + Str;
      pin(AK);
      pin(EpS);
    }
    end(iv<5>());
    auto curv = [&](int s, const Lines& l) {  // At_ij: every term but chi (X_ij - gt_ij X / 3)
      FieldDerivs d;
      lines_transport(l, P, wo, wd, d);
      const int i = SI(s), j = SJ(s);
      double r = d.advko;
#pragma unroll
      for (int k = 0; k < 3; ++k) r += At[S(i, k)] * DB[3 * k + j] + At[S(j, k)] * DB[3 * k + i];
      r -= (2.0 / 3.0) * At[s] * (DB[0] + DB[4] + DB[8]);
      double AAij = 0.0;  // At_ik gt^kl At_lj
#pragma unroll
      for (int k = 0; k < 3; ++k) AAij += At[S(i, k)] * Amix[k][j];
      r += alpha * (K * At[s] - 2.0 * AAij);
      keep(pa[s], r, l.v[0][3]);
    };
    load2();
    fence();
    curv(0, l0);
    curv(1, l1);
    end(iv<6>());
    load2();
    fence();
    curv(2, l0);
    curv(3, l1);
    end(iv<7>());
    double DCHI[3], DAL[3];
    Hold rchi, ral;
    uint32_t fo[3][4];  // byte offsets of the flux neighbours at -2, -1, +1, +2 along each axis
    load0();
    const Pre echi = sink.preload(F_CHI);
    fence();
    {
      FieldDerivs d;
      lines_transport(l0, P, wo, wd, d);
      const double divb = DB[0] + DB[4] + DB[8];
      keep(rchi, d.advko + (2.0 / 3.0) * chi * (alpha * K - divb), chi);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        DCHI[a] = d.d1[a];
        pin(DCHI[a]);
      }
    }
    load1();
    curv(4, l1);
    if constexpr (!KT) flux_neighbours<B>(m, P.n, c, fo);
    end(iv<8>());
    double f0[3][4], f1[3][4];
    double eps = 0.0;
    load0();
    const Pre eal = sink.preload(F_ALP);
    Pre ea[6];
#pragma unroll
    for (int s = 0; s < 3; ++s) ea[s] = sink.preload(F_AT + s);
    if constexpr (SC != 0) eps = bld(field_at(seq.xsrc(), SRC_EPS, m.fs), (uint32_t)(m.fs * 8), 8u * (uint32_t)c);
    sink.put(F_CHI, rchi, echi);
    fence();
    {
      FieldDerivs d;
      lines_transport(l0, P, wo, wd, d);
      const double Kbg = P.lapse_bg ? -3.0 * P.H0 / (1.0 + 2.0 * P.H0 * m.t) : 0.0;
      keep(ral, d.advko - 2.0 * alpha * (K - Kbg), alpha);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        DAL[a] = d.d1[a];
        pin(DAL[a]);
      }
    }
    load1();
    curv(5, l1);
    pair_flux_load<KT>(m.F, m.fs, c, fo, 0, f0);
    end(iv<9>());
    Hold rk, ret;
    load0();
    const Pre ek = sink.preload(F_K), eet = sink.preload(F_ET);
#pragma unroll
    for (int s = 3; s < 6; ++s) ea[s] = sink.preload(F_AT + s);
    pair_flux_load<KT>(m.F, m.fs, c, fo, 1, f1);
    sink.put(F_ALP, ral, eal);
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      sink.more(pa[s], ex[(EX_Y + s) * 256]);
      sink.put(F_AT + s, pa[s], ea[s]);
    }
    fence();
    {
      FieldDerivs d;
      lines_transport(l0, P, wo, wd, d);
      if constexpr (SC != 0) EpS += eps;
      keep(rk, d.advko + (-ex[EX_D2A * 256] + alpha * AK + 4.0 * PI_D * alpha * EpS), K);
    }
    {
      load1();
      const double div0 = flux_var_div(f0, P, KT);
      FieldDerivs d;
      if constexpr (!KT) lines_dissipation(l1, P, d);
      const double Sda = Sup[0] * DAL[0] + Sup[1] * DAL[1] + Sup[2] * DAL[2];
      keep(ret, (KT ? 0.0 : d.advko) + (im32 * (alpha * KS - Sda) - div0), l1.v[0][3]);
    }
    pair_flux_load<KT>(m.F, m.fs, c, fo, 2, f0);
    end(iv<10>());
    Hold rs[3];
    auto momentum = [&](int i, const Lines& l, const double f[3][4]) {
      const double divi = flux_var_div(f, P, KT);
      FieldDerivs d;
      if constexpr (!KT) lines_dissipation(l, P, d);
      double src = -E * DAL[i] + (Sl[0] * DB[0 + i] + Sl[1] * DB[3 + i] + Sl[2] * DB[6 + i]);
      src += 0.5 * alpha * (SG[i] * ichi - sgt * DCHI[i] * (ichi * ichi));
      keep(rs[i], (KT ? 0.0 : d.advko) + (im32 * src - divi), l.v[0][3]);
    };
    load0();
    Pre es[3], em[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) em[k] = sink.preload(F_GAM + k);
#pragma unroll
    for (int k = 0; k < 2; ++k) es[k] = sink.preload(F_ST + k);
    sink.put(F_K, rk, ek);
    sink.put(F_ET, ret, eet);
#pragma unroll
    for (int s = 3; s < 6; ++s) {
      sink.more(pa[s], ex[(EX_Y + s) * 256]);
      sink.put(F_AT + s, pa[s], ea[s]);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      sink.more(ag[k], ex[(EX_RG + k) * 256]);
      pin(ag[k].a);
    }
    fence();
    momentum(0, l0, f1);
    load1();
    pair_flux_load<KT>(m.F, m.fs, c, fo, 3, f1);
    momentum(1, l1, f0);
    end(iv<11>());
    load0();
    es[2] = sink.preload(F_ST + 2);
    StageItem nx;
    bool nact = false;
    int nc = 0;
    const bool more = seq.peek(nx, nc, nact);
#pragma unroll
    for (int k = 0; k < 3; ++k) sink.put(F_GAM + k, ag[k], em[k]);
    sink.put(F_ST, rs[0], es[0]);
    sink.put(F_ST + 1, rs[1], es[1]);
    fence();
    momentum(2, l0, f1);
    if (more) {
      centre_load(nx, nc);
    } else {  // so that the old values do not stay live for this case
#pragma unroll
      for (int f = 0; f < NF; ++f) cen[f] = 0.0;
    }
    sink.put(F_ST + 2, rs[2], es[2]);
    sink.finish(m, P, seq);
    end(iv<12>());
    if (!more) return;
    m = nx;
    c = nc;
    active = nact;
    seq.advance();
  }
}

}  // namespace cosmos
