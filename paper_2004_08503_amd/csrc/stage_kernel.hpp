// Fused limited SSP-RK stage for gfx950.  One workgroup owns a tile of
// TX x TY elements (TX elements in 1-D) and runs every step of the stage out
// of registers and LDS.  Global memory is touched once per node for the
// stage input (plus one ring of face-trace nodes around the tile), once for
// u^n on the second and third stages, and once for the output.
//
// The tile's nodes form one grid of GX = TX (p+1) columns and GY = TY (p+1)
// rows (one row in 1-D), surrounded by a ring of halo nodes (the facing
// nodes of the neighbouring elements or, on an open side of the box, the
// exterior states).  Along a grid row, consecutive columns are neighbours
// whether they belong to one element (an interior subcell face) or to two
// (an element face).  One thread owns a grid node and the two faces to its
// left and below; it keeps its node's state and its two faces in registers
// through the whole stage, so a face reads only its left (lower) state from
// LDS, and a node reads only its right and upper faces.  Where the tile
// leaves threads of its last wave idle (15 x 15 nodes of 16 x 16 threads),
// the thread grid has one more column and row, whose threads own the right
// and upper halo nodes and with them the faces on the tile's high edges;
// otherwise one wave evaluates those faces in an extra pass.  A face on the
// tile's edge, which the neighbouring tile evaluates too, gives bitwise the
// same values in both.
//
// Phases (LDS barriers between them):
//   1-2. every thread loads its node (and threads below the number of
//        remaining halo nodes one of those), forms the pointwise physics
//        (fluxes and, for Euler, 1/rho, the sound speed c, c p^{-(gamma-1)/(2
//        gamma)}, (gamma+1)/(2 gamma p), the inputs of the wave-speed bound,
//        and K = p rho^{-gamma}) and puts what a neighbour reads into LDS;
//   3. the thread's two faces: wave-speed bound, low-order flux f^L (eq.
//      lax-friedrichs on the subgrid), bar state of the limited component
//      (eq. bar-states) and on interior subcell faces the high-order subcell
//      flux f^H and the antidiffusive flux f^L - f^H;
//   4. per node: u^L, local bounds (K_min over the node and its four grid
//      neighbours), Zalesak coefficient and, for Euler, the entropy line
//      search of eq. convex-provisional;
//   5. per node: subcell-face coefficients min(alpha_i, alpha_j), the
//      flux-corrected update (eq. convex-fct) and the RK combination.
//
// Face quantities are kept without their common factors: fluxes and bar
// states are stored doubled (the halves of the averages go into the node's
// dt/(2 w h), and the bounds are halved once per node), and the
// antidiffusive flux without its line weight, which cancels against the
// node's mass: dt/m w_b h_y = dt/(w_a h_x) for an x-line.
//
// The high-order subcell flux uses the cumulative derivative matrix: on an
// interior subcell face a+1/2 of a line, f^H = F_0 + sum_e (sum_{c<=a}
// D[c][e]) F_e is the flux whose differences reproduce the strong-form
// residual (eq. dg-strong), so the prefix sums of r^H - r^L of Sec. 4.1.3
// become one short contraction per face.
//
// The file is compiled without multiply-add contraction, and the fused
// operations are written out: results must not depend on how a kernel is
// compiled (plain and batched kernels, tile shapes, and the two routes of a
// tile-edge face agree bitwise).
//
// What bounds it: FP64 vector issue first (the contraction, two wave-speed
// bounds and up to four admissibility tests per node), the LDS port second
// (a ds_read_b64 holds the CU's port for 4 cycles, as long as three to four
// vector instructions of one of its four SIMDs).  Hence the thread that keeps
// its node and its two faces, the fluxes stored once, the arrays indexed by
// the thread, and the cheap certain tests before the exact ones.  Measured,
// 256 x 256 elements of p = 4, gamma = 7/5 (1.64 M nodes), one stage in the
// kernel trace: 104.8 us with one work item per face and every value passed
// through LDS (1268 vector and 176 LDS instructions per wave), 81 to 82.7 us so
// (906 and 100), 1.7 TB/s of the stage's own bytes; issue is 0.53 busy.
#pragma once
#include "common.hpp"

#pragma clang fp contract(off)

namespace idp {

constexpr int up64(int n) { return (n + 63) / 64 * 64; }

template <int EQ, int DIM, int P, int TX, int TY, bool CURV = false>
struct Cfg {
  static constexpr int N1 = P + 1;
  static constexpr int NP = DIM == 2 ? N1 * N1 : N1;    // nodes per element
  static constexpr int TYE = DIM == 2 ? TY : 1;         // elements per tile in y
  static constexpr int NE = TX * TYE;                   // elements per tile
  static constexpr int GX = TX * N1;                    // node columns of the tile
  static constexpr int GY = DIM == 2 ? TYE * N1 : 1;    // node rows
  static constexpr int NOWN = GX * GY;                  // own nodes
  static constexpr int NC = is_euler(EQ) ? DIM + 2 : 1;
  // EDGE: the thread grid also covers the right halo column and the upper
  // halo row where that takes no further wave (p = 4, 15 x 15 nodes: four
  // waves either way).  Those threads would idle, and the extra pass keeps
  // three waves waiting for one; a fifth wave would leave three workgroups on
  // a CU.  1-D grids cover both halos.
  static constexpr bool EDGE = DIM == 1 || up64(GX * GY) == up64((GX + 1) * (GY + 1));
  static constexpr int OL = DIM == 1 ? 1 : 0;           // left halo in the grid (1-D)
  static constexpr int TGX = OL + GX + (EDGE ? 1 : 0);  // thread grid
  static constexpr int TGY = DIM == 2 ? GY + (EDGE ? 1 : 0) : 1;
  static constexpr int BS = up64(TGX * TGY);
  static constexpr int NW = BS / 64;                    // waves per workgroup
  // halo nodes outside the thread grid: left, lower (, right, upper)
  static constexpr int NHX = DIM == 1 ? 0 : (GX + GY) * (EDGE ? 1 : 2);
  static_assert(NHX <= BS, "one halo node per thread");
  // high-edge faces outside the thread grid: right column, upper row
  static constexpr int NEF = EDGE ? 0 : GX + GY;
  static_assert(NEF <= 64, "one wave takes the high-edge faces");
  // Node data that a neighbour reads, one array each over the slot grid:
  // the state, and for Euler the distinct fluxes (F^x_x, F^x_y = F^y_x,
  // F^y_y, F^x_E, F^y_E; the mass fluxes are the momenta), 1/rho, c, c p^-ex,
  // (gamma+1)/(2 gamma p); on a curved mesh the eight metric terms.
  static constexpr int NF = is_euler(EQ) ? (DIM == 2 ? 5 : 2) : 0;
  static constexpr int ZX = NC + NF;                    // first auxiliary
  static constexpr int ZM = ZX + (is_euler(EQ) ? 4 : 0);   // first metric term
  static constexpr int NZ = ZM + (CURV ? 8 : 0);
  // slot grid: own nodes, left and lower halos (, right and upper halos)
  static constexpr int SPX = GX + (EDGE ? 1 : 2);
  static constexpr int SPY = DIM == 2 ? GY + (EDGE ? 1 : 2) : 1;
  static constexpr int NSL = SPX * SPY;
  // K grid: own nodes and the whole ring
  static constexpr int KPX = GX + 2;
  static constexpr int NK = is_euler(EQ) ? (DIM == 2 ? KPX * (GY + 2) : KPX) : 0;
  // region A: phase 1-2 results, read in phase 3
  static constexpr int A_K = NZ * NSL;
  static constexpr int A_END = A_K + NK;
  // region B (aliases A): per direction k the doubled low-order fluxes, bar
  // states and antidiffusive fluxes of the faces a node does not own itself,
  // stored at the node to whose right (above which) they lie: x-face i of
  // row j at node (i-1, j), y-face j of column i at node (i, j-1).  A node's
  // index is its thread's, and the arrays are whole waves long, so one
  // address register serves every array.
  static constexpr int NB = BS;
  static constexpr int b_f(int k) { return k * NC * NB; }
  static constexpr int b_u(int k) { return (DIM * NC + k) * NB; }
  static constexpr int b_g(int k) { return (DIM * NC + DIM + k * NC) * NB; }
  static constexpr int B_END = (2 * DIM * NC + DIM) * NB;
  // region C: Euler search data, written once the low-order fluxes are
  // consumed; it overwrites them where it fits
  static constexpr int C_LEN = is_euler(EQ) ? (NC + 3 + DIM) * NB + DIM * NB / 2 : 0;
  static constexpr int C_UL = C_LEN <= b_g(0) ? 0 : B_END;   // [NC][NB]
  static constexpr int C_KM = C_UL + NC * NB;
  static constexpr int C_AZ = C_KM + NB;                // bound U of the node
  static constexpr int C_G2 = C_AZ + NB;                // [DIM] 2d dt/(2 w h) of the node
  static constexpr int C_PS = C_G2 + DIM * NB;          // largest |P| over the node's faces
  static constexpr int C_LIST = C_PS + NB;              // unsigned short[2*DIM*NB]
  static constexpr int C_END = is_euler(EQ) ? C_UL + C_LEN : 0;
  static_assert(NB * 4 <= 65536, "search items are 16-bit");
  static constexpr int AB0 = A_END > B_END ? A_END : B_END;
  static constexpr int AB = AB0 > C_END ? AB0 : C_END;
  static constexpr int S_AL = AB;                       // nodal alpha; scratch before phase 4
  static constexpr int S_W = S_AL + NB;                 // weights
  static constexpr int S_Q = S_W + N1;                  // high-order flux rows
  static constexpr int S_IW = S_Q + P * N1;             // 1/w
  static constexpr int S_M = S_IW + N1;                 // degree-p Legendre coefficient of a line
  static constexpr int S_LN = S_M + N1;                 // search list length (int)
  static constexpr int S_R = S_LN + 1;                  // per-wave minima of the time-step bound
  static constexpr int LDS = S_R + NW;
  static_assert(LDS * 8 <= 160 * 1024, "tile does not fit in LDS");
  // Waves per SIMD the registers have to leave room for: four, as many as the
  // LDS of 256-thread workgroups does (39 KB each).  Curved Euler tiles hold
  // 47 KB, three per CU, and would spill at 128 registers.
  static constexpr int WPE = is_euler(EQ) && CURV ? 3 : 4;
  // the work-list kernels, whose arguments take a few registers more (generic
  // gamma spills at 128)
  static constexpr int WPEB = EQ == EQ_EULER ? 3 : WPE;

  // slot of grid node (i, j), K slot, and node index
  static __device__ __forceinline__ int sl(int i, int j) { return DIM == 2 ? (j + 1) * SPX + i + 1 : i + 1; }
  static __device__ __forceinline__ int kl(int i, int j) { return DIM == 2 ? (j + 1) * KPX + i + 1 : i + 1; }
  static __device__ __forceinline__ int nd(int i, int j) { return j * TGX + i + OL; }
  // slot array of component c of the flux in direction k
  static constexpr int fz(int k, int c) {
    return c == 0 ? 1 + k : DIM == 1 ? NC + c - 1 : c == 3 ? NC + 3 + k : NC + k + c - 1;
  }
};

// Where a tile lies: its first element column and row, and how many of its
// TX x TY elements exist (tiles on the high edges of the mesh are ragged).
struct TileGeo {
  int ex0, ey0, tw, th;
};
// tile / ntx by the multiplier of idp_magic (tiles < 2^31)
__device__ inline int div_ntx(int tile, unsigned int mul, int shift) {
  return (int)(((unsigned long long)(unsigned int)tile * mul) >> shift);
}
template <int DIM, int TX, int TY>
__device__ inline TileGeo tile_geo(int tile, int ntx, unsigned int mul, int shift, int nx, int ny) {
  TileGeo t;
  const int ty = DIM == 2 ? div_ntx(tile, mul, shift) : 0;
  const int tx = tile - ty * ntx;
  t.ex0 = tx * TX;
  t.ey0 = DIM == 2 ? ty * TY : 0;
  t.tw = min(TX, nx - t.ex0);
  t.th = DIM == 2 ? min(TY, ny - t.ey0) : 1;
  return t;
}

// Workgroups are dealt round-robin to the eight XCDs; give every XCD a
// contiguous range of tiles so that the halo nodes a tile reads from the
// tile rows above and below were fetched into the same XCD's L2.
__device__ inline int xcd_tile(int b, int nb) {
  const int x = b & 7, i = b >> 3;
  const int q = nb >> 3, r = nb & 7;
  return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + i;
}

// Minimum and maximum of two doubles, one instruction each.  (Compiled from
// fmin or fmax, operands that come from memory would first be quieted by an
// instruction of their own.)  A NaN operand gives the other operand.  Their
// operands must not come straight from a transcendental instruction (rcp, rsq,
// exp, log): the compiler sees no hazard in inline assembly.
__device__ __forceinline__ double vmin(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double vmax(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
// max(|a|, |b|), and max(a, 0), min(a, 0)
__device__ __forceinline__ double vmaxabs(double a, double b) {
  double r;
  asm("v_max_f64 %0, |%1|, |%2|" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double vpos(double a) {
  double r;
  asm("v_max_f64 %0, %1, 0" : "=v"(r) : "v"(a));
  return r;
}
__device__ __forceinline__ double vneg(double a) {
  double r;
  asm("v_min_f64 %0, %1, 0" : "=v"(r) : "v"(a));
  return r;
}

// The advection velocity / Burgers direction component k, selected between
// two values already loaded (a select between two fields of the argument
// struct could otherwise become a load from a run-time address, which moves
// a local copy of the struct to scratch memory).
__device__ inline double vel_k(int k, const Phys& ph) {
  const unsigned long long v0 = __double_as_longlong(ph.vel0), v1 = __double_as_longlong(ph.vel1);
  return __longlong_as_double(k == 0 ? v0 : v1);
}

template <int N>
__device__ inline double ipow_c(double x) {
  if constexpr (N == 1) return x;
  else if constexpr (N % 2 == 0) { const double h = ipow_c<N / 2>(x); return h * h; }
  else return x * ipow_c<N - 1>(x);
}

// x^(-1/N) in binary64 for x > 0: a single-precision log2/exp2 seed y
// (within 1e-6, relative) and, with r = 1 - x y^N, the third-order step
// y (1 + r/N + (N+1)/(2 N^2) r^2), which leaves (N+1)(2N+1)/(6 N^3) r^3 <
// 1e-17, below the rounding of the last operation.  An x outside the
// seed's range shows in r, and takes the reduced form:
// x = m 2^e with m in [1/2, 1) and e = N q + k (0 <= k < N), so that
// x^(-1/N) = 2^-q (m 2^k)^(-1/N) with m 2^k in [1/2, 2^(N-1)).
// Non-positive, infinite or NaN x give NaN or infinity.
template <int N>
__device__ inline double root_step(double x, float xs, double* r) {
  const double y = (double)__builtin_amdgcn_exp2f(__builtin_amdgcn_logf(xs) * (-1.0f / N));
  *r = fma(-x, ipow_c<N>(y), 1.0);
  return fma(y * *r, fma(*r, (N + 1.0) / (2.0 * N * N), 1.0 / N), y);
}
template <int N>
__device__ inline double inv_root(double x) {
  double r, y = root_step<N>(x, (float)x, &r);
  if (fabs(r) >= 1e-4) {   // (a NaN stays one in either form)
    int e;
    const double m = frexp(x, &e);
    const int q = (e + 1100 * N) / N - 1100;   // floor(e / N) for e >= -1100 N
    const double xr = ldexp(m, e - N * q);
    y = ldexp(root_step<N>(xr, (float)xr, &r), -q);
  }
  return y;
}

// sqrt(x) for x of normal magnitude: the hardware reciprocal square root y
// (23 bits or better) and, with g = x y and r = 1 - g y, the third-order
// step g (1 + r/2 + 3 r^2/8), within an ulp.  NaN for infinity, zero and
// negative x.
__device__ inline double sqrt_nr(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double g = x * y;
  const double r = fma(-g, y, 1.0);
  return fma(g * r, fma(r, 0.375, 0.5), g);
}

// sqrt_nr for x >= 1 or +infinity: the seed of infinity, 0, is raised to
// 2^-600, far below every other, and g and the result become infinite.  (By
// fmax, not vmax: a value from the transcendental unit may be read by the next
// vector instruction only after a wait, which the compiler does not insert
// before inline assembly.)
__device__ inline double sqrt_ge1(double x) {
  const double y = fmax(__builtin_amdgcn_rsq(x), 0x1p-600);
  const double g = x * y;
  const double r = fma(-g, y, 1.0);
  return fma(g * r, fma(r, 0.375, 0.5), g);
}

// sqrt_nr that keeps zero and +infinity.
__device__ inline double sqrt_any(double x) {
  const double s = sqrt_nr(x);
  return __builtin_amdgcn_class(x, 0x260) ? x : s;
}

// 1/x for x of normal magnitude: the hardware approximation y (23 bits or
// better) and, with e = 1 - x y, the third-order step y (1 + e + e^2), within
// an ulp (NaN for infinity, zero and NaN).
__device__ inline double rcp_nr(double x) {
  const double y = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, y, 1.0);
  return fma(y, fma(e, e, e), y);
}

// rcp_nr for every x: where the approximation is infinite or zero (x zero,
// infinite, or so small that 1/x is past the largest double or next to it) a
// division.  Ordinary states never take that branch, which the empty assembly
// keeps a branch: computed for every x and selected, the division made the
// time-step kernel 295 vector instructions per wave, so 281.
__device__ inline double rcp_any(double x) {
  double r = rcp_nr(x);
  if (__builtin_amdgcn_class(__builtin_amdgcn_rcp(x), 0x264)) {
    asm volatile("" : "+v"(x));
    r = 1.0 / x;
  }
  return r;
}

// x^y for finite x > 0 and a result of normal magnitude; NaN for other x.
// x = m 2^e with m in [1/sqrt 2, sqrt 2), ln m = 2 atanh(s) with s =
// (m-1)/(m+1); s, the product with 1/ln 2 and the sum with e are kept in two
// parts, so that y log2 x carries an absolute error near 1e-17 max(1, |y|)
// and 2^f, |f| <= 1/2, is the Taylor sum to f^13 (next term 4e-18): within two
// ulps.  About 60 operations and no branch; the library's pow, with its
// special cases, made the generic-gamma stage 1.5 times as long.
__device__ inline double pow_pos(double x, double y) {
  int e;
  double m = frexp(x, &e);
  const bool up = m < 0.70710678118654752;
  m = up ? 2.0 * m : m;
  e -= up ? 1 : 0;
  const double r = m - 1.0, d = m + 1.0, t = rcp_nr(d);
  const double s = r * t, sl = (fma(-s, d, r) - s * (m - (d - 1.0))) * t;
  const double z = s * s;
  double a = 2.0 / 21.0;
#pragma unroll
  for (int k = 19; k >= 3; k -= 2) a = fma(a, z, 2.0 / k);
  const double lo = fma(s * z, a, 2.0 * sl), h = 2.0 * s;   // ln m = h + lo
  constexpr double CH = 1.4426950408889634, CL = 2.0355273740931033e-17;   // 1/ln 2 = CH + CL
  const double ph = h * CH, pl = fma(h, CH, -ph) + fma(h, CL, lo * CH);
  const double ed = (double)e, lh = ed + ph, ll = pl + (ph - (lh - ed));   // log2 x (|ph| <= 1/2 <= |e|, or e = 0)
  const double yh = y * lh, yl = fma(y, lh, -yh) + y * ll;
  const double n = rint(yh), f = (yh - n) + yl;
  constexpr double LN2 = 0.69314718055994531;
  double c = LN2 / 13.0;
#pragma unroll
  for (int k = 12; k >= 1; --k) c = fma(c, f, 1.0) * (LN2 / k);
  const double v = ldexp(fma(c, f, 1.0), (int)n);
  return x > 0.0 ? v : NAN;   // (an infinite x has made v NaN)
}

// ----------------------------------------------------------------------
// pointwise physics
// ----------------------------------------------------------------------

// Euler auxiliaries of one state: X = (1/rho, c, c p^-ex, (gamma+1)/(2 gamma
// p)), ex = (gamma-1)/(2 gamma), with WITHK K = p rho^-gamma, and the
// pressure p.  For gamma = 1 + 2/n (GN = n = 5: 7/5, n = 3: 5/3) every
// fractional power is an integer power of z = rho^(-1/n) or of
// x3 = p^(-1/(n+2)): 1/rho = z^n, K = p z^(n+2), 1/p = x3^(n+2); otherwise
// pow and divisions are used.  Without K (the time-step pass) 1/rho is a
// plain reciprocal, cheaper than the root.  Zero and infinite densities and
// pressures give what IEEE division, square root and pow give (the roots of
// integer powers NaN), so that a wave speed, a bound and K_min leave out
// the same faces and nodes whatever way they are computed.
template <int DIM, int GN, bool WITHK>
__device__ inline void euler_aux(const double* U, const Phys& ph, double* X, double& K, double& p, bool& bad) {
  double rinv, z = 0.0;
  if constexpr (GN > 0 && WITHK) {
    z = inv_root<GN>(U[0]);
    rinv = ipow_c<GN>(z);
  } else {
    rinv = rcp_any(U[0]);
  }
  double mm = U[1] * U[1];
  if constexpr (DIM == 2) mm = fma(U[2], U[2], mm);
  p = (ph.gamma - 1.0) * fma(-0.5 * mm, rinv, U[DIM + 1]);
  bad = !(U[0] > 0.0) || !(p > 0.0);
  const double c = sqrt_any(ph.gamma * p * rinv);
  double x3, ip;
  if constexpr (GN > 0) {
    x3 = inv_root<GN + 2>(p);
    ip = ipow_c<GN + 2>(x3);
  } else {
    x3 = pow_pos(p, -ph.ex);
    ip = rcp_nr(p);
  }
  X[0] = rinv;
  X[1] = c;
  X[2] = c * x3;
  X[3] = ph.fac * ip;
  if constexpr (WITHK) {
    if constexpr (GN > 0) K = p * (rinv * (z * z));
    else K = p * (__builtin_amdgcn_class(U[0], 0x260) ? rinv : pow_pos(U[0], -ph.gamma));   // (pow of 0, infinity)
  }
}

// The node data of one state z[0..NC) in place: fluxes and auxiliaries.
template <class C, int EQ, int DIM>
__device__ inline void node_state(double* z, const Phys& ph, double& K, bool& bad) {
  if constexpr (is_euler(EQ)) {
    double p;
    euler_aux<DIM, gn_of(EQ), true>(z, ph, z + C::ZX, K, p, bad);
    constexpr int F = C::NC;
    const double ri = z[C::ZX], H = z[DIM + 1] + p;
    const double v1 = z[1] * ri;
    z[F] = fma(z[1], v1, p);
    if constexpr (DIM == 2) {
      const double v2 = z[2] * ri;
      z[F + 1] = z[2] * v1;
      z[F + 2] = fma(z[2], v2, p);
      z[F + 3] = v1 * H;
      z[F + 4] = v2 * H;
    } else {
      z[F + 1] = v1 * H;
    }
  }
}

// The two-rarefaction bound of the Euler wave speeds (Guermond and Popov,
// J. Comput. Phys. 2016, valid for 1 < gamma <= 5/3) from the normal
// velocities v, sound speeds c, the sum x2 of the two c p^-ex and
// x3 = (gamma+1)/(2 gamma p) of the left and right states: with
// p* = ((c_L + c_R - (gamma-1)/2 (v_R - v_L))_+ / x2)^(1/ex),
// lambda = max((v_L - c_L sqrt(1 + (gamma+1)/(2 gamma) (p* - p_L)_+ / p_L))_-,
//              (v_R + c_R sqrt(1 + (gamma+1)/(2 gamma) (p* - p_R)_+ / p_R))_+).
// Homogeneous of degree one in (v, c, x2): scaled by |n|, it is |n| lambda.
template <int GN>
__device__ inline double euler_lambda(double vl, double vr, double cl, double cr, double x2, double x3l, double x3r,
                                      const Phys& ph) {
  const double num = vpos(fma(-ph.g1, vr - vl, cl + cr));
  const double base = num * rcp_nr(x2);   // c p^-ex > 0 on both sides
  double pstar;
  if constexpr (GN > 0) pstar = ipow_c<GN + 2>(base);
  else pstar = pow_pos(base, ph.inv_ex);
  // 1 + (p*/p - 1)_+ (gamma+1)/(2 gamma), at least 1
  const double sl = sqrt_ge1(vmax(fma(pstar, x3l, ph.f1), 1.0));
  const double sr = sqrt_ge1(vmax(fma(pstar, x3r, ph.f1), 1.0));
  return vpos(vmax(fma(cl, sl, -vl), fma(cr, sr, vr)));
}

// Phi(V) = rho e - K_min rho^gamma / (gamma - 1) along V = uL + t P, with
// its t-derivative.  Phi >= 0 with rho > 0 is the specific-entropy minimum
// principle of Sec. 4.3; Phi is concave.
struct PhiVal {
  double rho, phi, dphi;
};

template <int DIM, int GN>
__device__ inline PhiVal phi_at(double t, const double* uL, const double* P, double kmin,
                                const Phys& ph) {
  // straight-line code (no branches), so that independent evaluations
  // interleave; a non-positive density gives phi = -infinity
  PhiVal r;
  r.rho = fma(t, P[0], uL[0]);
  const bool pos = r.rho > 0.0;
  const double rho = pos ? r.rho : 1.0;
  const double g = ph.gamma;
  double rinv, rg;
  if constexpr (GN > 0) {  // z = rho^(-1/n): 1/rho = z^n, rho^gamma = rho^2 z^(n-2)
    const double z = inv_root<GN>(rho);
    rinv = ipow_c<GN>(z);
    rg = (rho * rho) * ipow_c<GN - 2>(z);
  } else {
    rinv = rcp_nr(rho);
    rg = pow_pos(rho, g);
  }
  const double m1 = fma(t, P[1], uL[1]);
  double mm = m1 * m1, mp = m1 * P[1];
  if constexpr (DIM == 2) {
    const double m2 = fma(t, P[2], uL[2]);
    mm = fma(m2, m2, mm);
    mp = fma(m2, P[2], mp);
  }
  const double E = fma(t, P[DIM + 1], uL[DIM + 1]);
  const double kr = kmin * ph.igm1 * rg;
  const double ke = 0.5 * mm * rinv;          // kinetic energy
  const double phi = fma(-0.5 * mm, rinv, E) - kr;
  // P_E - m.P_m / rho + (ke - gamma kr) P_rho / rho
  const double dphi = fma(rinv, fma(fma(-g, kr, ke), P[0], -mp), P[DIM + 1]);
  r.phi = pos ? phi : -INFINITY;
  r.dphi = pos ? dphi : 0.0;
  return r;
}

__device__ inline bool admissible(const PhiVal& e) { return e.rho > 0.0 && e.phi >= 0.0; }

// Whether V = uL + t P is admissible beyond doubt, from integer powers
// only; false means "not certain" and leaves the decision to phi_at.  For
// gamma = 1 + 2/n and rho > 0, with W = rho (rho e) = E rho - |m|^2 / 2 and
// w = W (gamma - 1) / K_min:  Phi >= 0  <=>  w^n >= rho^(2n+2).  E rho is
// lowered by 64 ulps (where W >= 0, |m|^2 / 2 <= E rho, so that is twice a
// bound on the rounding of W and of a direct evaluation of rho e), and ikg,
// (gamma - 1) / K_min lowered by 3e-13, leaves the powers a relative margin
// of 1e-12 or close to it.  The three comparisons bound both powers away from
// overflow and underflow: rho >= 1e-20 and w^n <= 1e250 with w^n >=
// rho^(2n+2) leave 1e-48 <= w <= 1e84 and rho <= 1e32, and n is odd, so
// w > 0.  A K_min that is not positive, next to a bad node, has ikg = 0 and
// certifies nothing (W / K_min may be positive with both negative).  For other gamma, Phi >= 0 <=> log2 w >= (gamma+1) log2 rho, from
// single-precision logarithms with a margin eight times their error: 2^-24 /
// ln 2 for the rounding of w and gamma + 1 times that for rho, 3.2e-7 together,
// and an ulp, 1.2e-7 of their size, for the logarithms.
template <int DIM, int GN>
__device__ inline bool surely_admissible(double t, const double* uL, const double* P, double ikg, const Phys& ph) {
  const double rho = fma(t, P[0], uL[0]);
  const double m1 = fma(t, P[1], uL[1]);
  double mm = m1 * m1;
  if constexpr (DIM == 2) {
    const double m2 = fma(t, P[2], uL[2]);
    mm = fma(m2, m2, mm);
  }
  const double E = fma(t, P[DIM + 1], uL[DIM + 1]);
  const double w = fma(E * rho, 1.0 - 0x1p-47, -0.5 * mm) * ikg;
  if constexpr (GN > 0) {
    const double r2 = rho * rho, r4 = r2 * r2;
    const double rhs = GN == 5 ? r4 * r4 * r4 : r4 * r4;   // rho^12 or rho^8
    const double lhs = ipow_c<GN>(w);
    return (rho >= 1e-20) & (lhs <= 1e250) & (lhs >= rhs);
  } else {
    const float a = __builtin_amdgcn_logf((float)w), b = __builtin_amdgcn_logf((float)rho) * (float)(ph.gamma + 1.0);
    return (rho >= 1e-20) & (w <= 1e30) & (a - b >= 1e-6f * (3.0f + fabsf(a) + fabsf(b)));
  }
}

// sup { t in [0, U] : uL + t P admissible } for an element's correction of
// one node (elementwise limiting), uL admissible.  U is the tangent bound from
// alpha.
//  - the first point is U itself: an admissible U is the answer; otherwise
//    it is the first infeasible end;
//  - then Newton steps from the infeasible end hi (Phi is concave wherever
//    rho > 0, so the tangent at hi cuts zero at or above the root), each a
//    single evaluation; a tangent step that lands admissible is within
//    rounding of the root and ends the search; without a usable tangent
//    (rho <= 0 at hi), or after three Newton steps in a row that do not
//    halve (convergence slower than quadratic), one bisection; once the
//    Newton step is below half the tolerance, hi sits on the root and the
//    next points are probes under hi at half the tolerance, doubling the
//    distance after each inadmissible probe;
//  - the search stops once the bracket is narrower than 1e-15 or than
//    1e-16 max|uL| / max|P|, and returns the admissible end: one node's t is
//    applied to every node of the element, so that nodes of other scales (the
//    small momentum of a gas near rest next to a node of large energy) still
//    land within rounding.
template <int DIM, int GN>
__device__ double entropy_root(const double* uL, const double* P, double U, double kmin, const Phys& ph) {
  double us = 0.0, ps = 0.0;
#pragma unroll
  for (int c = 0; c < DIM + 2; ++c) {
    us = fmax(us, fabs(uL[c]));
    ps = fmax(ps, fabs(P[c]));
  }
  const double tol = fmax(1e-15, 1e-16 * us / ps);
  double lo = 0.0, hi = U, fhi = -INFINITY, dhi = 0.0, rhi = 0.0;
  double t = U, prev = INFINITY, probe = 0.5 * tol;
  int slow = 0;
  bool tang = true;   // t is a tangent's zero
  for (int it = 0; it < 64; ++it) {
    const PhiVal e = phi_at<DIM, GN>(t, uL, P, kmin, ph);
    if (admissible(e)) {
      if (tang || t >= U) return t;
      lo = t;
    } else {
      hi = t;
      fhi = e.phi;
      dhi = e.dphi;
      rhi = e.rho;
    }
    if (!(hi - lo > tol)) break;
    tang = false;
    if (rhi > 0.0 && dhi < 0.0) {
      const double step = fhi / dhi;  // the Newton step from hi, >= 0
      if (step < 0.5 * tol) {         // hi sits on the root: probe under it
        t = hi - probe;
        probe *= 2.0;
      } else if (slow >= 3) {
        t = 0.5 * (lo + hi);
        slow = 0;
      } else {
        t = hi - step;
        tang = true;
        slow = step > 0.5 * prev ? slow + 1 : 0;
        prev = step;
      }
    } else {
      t = 0.5 * (lo + hi);
    }
    if (!(t > lo && t < hi)) {
      t = 0.5 * (lo + hi);
      tang = false;
    }
  }
  return lo;
}

// sup { t in [0, U] : uL + t P admissible } for one subcell face of a node
// whose u^L is admissible, to within tol = 1e-14 max|uL| / max(|P|, pscale) or
// 1e-15.  The node's t scales more than this P: its coefficient limits every
// face of the node (through min(alpha_i, alpha_j)), so pscale is the largest
// |P| over the node's faces, and the answer moves every face's contribution to
// the state by less than 1e-14 of its largest component from any point of the
// bracket, the supremum included.  The first point is U, the node's alpha (the
// exact value there, which the screen could not certify).  Then Newton steps from the infeasible end hi; Phi is concave
// along the segment, so a Newton point tn lies at or above the root, and the
// point evaluated is tn - tol/2 instead of tn: if it is admissible, the root
// lies in [tn - tol/2, tn] and the search ends there; if not, it is the new
// infeasible end.  Without a usable tangent, or after three Newton steps in
// a row that do not halve, one bisection; a Newton step below tol/4 means
// hi sits on the root, and the next points are probes under hi at tol/2,
// doubling the distance after each inadmissible probe.  Where Phi is zero to
// rounding over a stretch of the segment (a correction that hardly changes the
// entropy) any computed-admissible point of the stretch may end the search.
// (Opening with Newton steps on w^(n/(2n+2)) - rho, the function whose sign
// surely_admissible tests and which is closer to linear, took 244.6 us a step
// instead of 248.2 at 256 x 256, p = 4, but its rounding put answers up to ten
// tolerances under the root, and flows that had run for thousands of steps,
// full of nearly isentropic corrections, took longer: the double Mach
// reflection on 40 x 15, p = 3, after 4300 steps 128 us a step, so 115.)
template <int DIM, int GN>
__device__ double entropy_root_face(const double* uL, const double* P, double U, double kmin, double pscale,
                                    const Phys& ph) {
  double us = 0.0, ps = pscale;
#pragma unroll
  for (int c = 0; c < DIM + 2; ++c) {
    us = vmaxabs(us, uL[c]);
    ps = vmaxabs(ps, P[c]);
  }
  const double tol = vmax(1e-15, 1e-14 * us * rcp_nr(ps));
  double lo = 0.0, hi = U, fhi = -INFINITY, dhi = 0.0;   // dhi = 0 without a usable tangent
  double t = U, prev = INFINITY, probe = 0.5 * tol;
  int slow = 0;
  bool below = false;   // t = tn - tol/2 under a Newton point tn
  for (int it = 0; it < 64; ++it) {
    const PhiVal e = phi_at<DIM, GN>(t, uL, P, kmin, ph);
    if (admissible(e)) {
      if (below || t >= U) return t;
      lo = t;
    } else {
      hi = t;
      fhi = e.phi;
      dhi = e.dphi;
    }
    if (!(hi - lo > tol)) break;
    below = false;
    if (dhi < 0.0) {
      const double step = fhi * rcp_nr(dhi);  // the Newton step from hi, >= 0
      if (step < 0.25 * tol) {        // hi sits on the root: probe under it
        t = hi - probe;
        probe *= 2.0;
      } else if (slow >= 3) {
        t = 0.5 * (lo + hi);
        slow = 0;
      } else {
        t = (hi - step) - 0.5 * tol;
        below = true;
        slow = step > 0.5 * prev ? slow + 1 : 0;
        prev = step;
      }
    } else {
      t = 0.5 * (lo + hi);
    }
    if (!(t > lo && t < hi)) {
      t = 0.5 * (lo + hi);
      below = false;
    }
  }
  return lo;
}

// ----------------------------------------------------------------------
// where a node of the tile's grid or of its halo ring lies
// ----------------------------------------------------------------------

// Node (i, j) of a tile, -1 <= i <= GX, -1 <= j <= GY: the global index of
// its state (periodic wrap), or, beyond an open side of the box (ext), that
// of the boundary node whose exterior state it is, with the side and the
// boundary node's index along it; row and col are its node row and column
// in the box.  LOW: i or j may be -1.
struct Src {
  long long g;
  int side, q, row, col;
  bool ext;
};
template <int DIM, int P, bool LOW>
__device__ inline Src node_src(int i, int j, const TileGeo& t, int nx, int ny, int open) {
  constexpr int N1 = P + 1, NP = DIM == 2 ? N1 * N1 : N1;
  Src r;
  r.ext = false;
  r.side = 0;
  const int lx = LOW ? (int)((unsigned)(i + N1) / N1) - 1 : (int)((unsigned)i / N1);
  int a = i - lx * N1, ex = t.ex0 + lx;
  if (LOW && ex < 0) {
    if (open & 1) r.ext = true, ex = 0, a = 0;
    else ex = nx - 1;
  }
  if (ex >= nx) {
    if (open & 1) r.ext = true, r.side = 1, ex = nx - 1, a = P;
    else ex = 0;
  }
  r.col = ex * N1 + a;
  if constexpr (DIM == 1) {
    r.row = r.q = 0;
    r.g = (long long)ex * NP + a;
  } else {
    const int ly = LOW ? (int)((unsigned)(j + N1) / N1) - 1 : (int)((unsigned)j / N1);
    int b = j - ly * N1, ey = t.ey0 + ly;
    if (LOW && ey < 0) {
      if (open & 2) r.ext = true, r.side = 2, ey = 0, b = 0;
      else ey = ny - 1;
    }
    if (ey >= ny) {
      if (open & 2) r.ext = true, r.side = 3, ey = ny - 1, b = P;
      else ey = 0;
    }
    r.row = ey * N1 + b;
    r.q = r.side < 2 ? r.row : r.col;
    r.g = ((long long)ey * nx + ex) * NP + b * N1 + a;
  }
  return r;
}

// Halo node h of the ring nodes outside the thread grid (left, lower and,
// without EDGE, right and upper): its grid node; false if the tile has none.
template <class C>
__device__ inline bool ring_node(int h, int cw, int ch, int* i, int* j) {
  if (h < C::GY) { *i = -1; *j = h; return h < ch; }
  h -= C::GY;
  if (h < C::GX) { *i = h; *j = -1; return h < cw; }
  if constexpr (!C::EDGE) {
    h -= C::GX;
    if (h < C::GY) { *i = cw; *j = h; return h < ch; }
    h -= C::GY;
    if (h < C::GX) { *i = h; *j = ch; return h < cw; }
  }
  return false;
}

// The exterior state of an open side for a halo node (V holds the own
// boundary node's state on entry): the prescribed state, the own state
// (outflow) or the own state with the normal momentum reversed (slip).  The
// side's arrays are selected between the four pointers already loaded: an
// index into the argument struct at run time would move it to scratch.
template <int EQ, int DIM, int NC>
__device__ inline void exterior_state(const Bnd& bnd, const Src& s, int nx1, int ny1, double* V) {
  const unsigned long long t0 = (unsigned long long)bnd.type[0], t1 = (unsigned long long)bnd.type[1];
  const unsigned long long t2 = (unsigned long long)bnd.type[2], t3 = (unsigned long long)bnd.type[3];
  const unsigned long long s0 = (unsigned long long)bnd.state[0], s1 = (unsigned long long)bnd.state[1];
  const unsigned long long s2 = (unsigned long long)bnd.state[2], s3 = (unsigned long long)bnd.state[3];
  const int sd = s.side;
  const int n = DIM == 1 ? 1 : (sd < 2 ? ny1 : nx1);   // boundary nodes of the side
  const signed char* type = (const signed char*)(sd == 0 ? t0 : sd == 1 ? t1 : sd == 2 ? t2 : t3);
  const double* state = (const double*)(sd == 0 ? s0 : sd == 1 ? s1 : sd == 2 ? s2 : s3);
  const int ty = type[s.q];
  if (ty == BC_STATE && state) {
#pragma unroll
    for (int c = 0; c < NC; ++c) V[c] = state[c * n + s.q];
  } else if (ty == BC_SLIP && is_euler(EQ)) {
    if (sd < 2) V[1] = -V[1];
    else if constexpr (DIM == 2) V[2] = -V[2];
  }
}

// The thread's place in the tile: grid node (i, j), element-local position
// (a, b), and which of its roles apply (cw, ch: the tile's node columns and
// rows): own node, or the halo node whose lower-side face it owns.
template <class C, int DIM>
struct Place {
  int i, j, a, b, cw, ch;
  bool own, right, top, left;
  __device__ inline bool any() const { return own || right || top || left; }
  __device__ inline bool face_x() const { return own || right; }
  __device__ inline bool face_y() const { return own || top; }
};
template <class C, int DIM>
__device__ inline Place<C, DIM> place(const TileGeo& tg) {
  Place<C, DIM> r;
  const unsigned tid = threadIdx.x;
  r.j = tid / C::TGX;
  r.i = (int)(tid - r.j * C::TGX) - C::OL;
  r.cw = tg.tw * C::N1;
  r.ch = DIM == 2 ? tg.th * C::N1 : 1;
  r.a = (unsigned)r.i % C::N1;
  r.b = DIM == 2 ? (unsigned)r.j % C::N1 : 0;
  const bool in_x = (C::OL == 0 || r.i >= 0) && r.i < r.cw, in_y = r.j < r.ch;
  r.own = in_x && in_y;
  r.right = C::EDGE && r.i == r.cw && in_y;
  r.top = C::EDGE && DIM == 2 && r.j == r.ch && in_x;
  r.left = C::OL > 0 && r.i < 0 && in_y;
  return r;
}

// The per-degree tables, fetched into registers by the first threads of
// the workgroup (thread t holds entry t of each table it covers) before the
// state loads are issued, and stored to LDS once the state has arrived, so
// that their latency hides under that of the state.
template <int P>
struct TableRegs {
  static constexpr int N1 = P + 1;
  double w, iw, q, m;
  __device__ inline void fetch(const Tables& T) {
    const int t = threadIdx.x;
    if (t < N1) {
      w = T.w[t];
      iw = T.iw[t];
      m = T.m[t];
    }
    if (t < P * N1) q = T.Q[t];
  }
  __device__ inline void store(double* sw, double* sq, double* siw, double* sm) const {
    const int t = threadIdx.x;
    if (t < N1) {
      sw[t] = w;
      siw[t] = iw;
      sm[t] = m;
    }
    if (t < P * N1) sq[t] = q;
  }
};

// ----------------------------------------------------------------------
// phase 3: subcell faces
// ----------------------------------------------------------------------

// One face: the doubled low-order flux, the doubled bar states of its left
// (lower) and right (upper) node, and the doubled antidiffusive flux without
// its line weight (zero on element faces).
template <int NC>
struct FaceVal {
  double f[NC], g[NC], ul, ur;
};

// The scalar fluxes are F_k(u) = coef_k gu(u).
template <int EQ>
__device__ __forceinline__ double gu(double u) { return EQ == EQ_BURG ? u * u : u; }
template <int EQ>
__device__ __forceinline__ double flux_coef(int k, const Phys& ph, const double* beta) {
  if constexpr (EQ == EQ_BURG) return 0.5 * vel_k(k, ph);
  else if constexpr (EQ == EQ_ADVV) return beta[k];
  else return vel_k(k, ph);
}

// Low-order part of the face in direction K between the node data zl (left
// or lower node) and zr.  beta: the velocity at the face's line (EQ_ADVV; the
// same on both sides, since beta_k is constant along a k-line).
// Curved meshes: ml and mr are the metric rows K of the two nodes: on an
// interior subcell face the corrected rows J, on an element face both the
// high-order row of the lower node (the face's scaled normal n).  Then with
// lt = max(|mr| lambda(L, R, mr/|mr|), |ml| lambda(L, R, ml/|ml|)) (eq. dij's
// two wave speeds, along n_LR and n_RL) the flux is 1/2 (ml.F_L + mr.F_R) -
// lt/2 (U_R - U_L), and the bar states of L and R are 1/2 (U_L + U_R) minus
// mr.(F_R - F_L) / (2 lt) and ml.(F_R - F_L) / (2 lt).
template <class C, int EQ, int DIM, int K, bool CURV>
__device__ __forceinline__ void face_low(const double* zl, const double* zr, const double* beta, const double* ml,
                                         const double* mr, const Phys& ph, FaceVal<C::NC>& o) {
  constexpr int NC = C::NC, X = C::ZX;
  if constexpr (is_euler(EQ)) {
    constexpr int GN = gn_of(EQ);
    double lam;
    if constexpr (CURV) {
      double v[2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const double* n = s == 0 ? mr : ml;
        const double q = sqrt_nr(fma(n[1], n[1], n[0] * n[0]));
        const double vl = fma(zl[2], n[1], zl[1] * n[0]) * zl[X], vr = fma(zr[2], n[1], zr[1] * n[0]) * zr[X];
        v[s] = euler_lambda<GN>(vl, vr, q * zl[X + 1], q * zr[X + 1], q * (zl[X + 2] + zr[X + 2]), zl[X + 3],
                                zr[X + 3], ph);
      }
      lam = vmax(v[0], v[1]);
    } else {
      lam = euler_lambda<GN>(zl[1 + K] * zl[X], zr[1 + K] * zr[X], zl[X + 1], zr[X + 1], zl[X + 2] + zr[X + 2],
                             zl[X + 3], zr[X + 3], ph);
    }
    const double il = lam > 0.0 ? rcp_nr(lam) : 0.0;
    const double s0 = zl[0] + zr[0];
    if constexpr (CURV) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const double fl = fma(zl[C::fz(1, c)], ml[1], zl[C::fz(0, c)] * ml[0]);
        const double fr = fma(zr[C::fz(1, c)], mr[1], zr[C::fz(0, c)] * mr[0]);
        o.f[c] = fma(-lam, zr[c] - zl[c], fl + fr);
      }
      const double d0 = zr[1] - zl[1], d1 = zr[2] - zl[2];
      o.ul = fma(-fma(mr[1], d1, mr[0] * d0), il, s0);
      o.ur = fma(-fma(ml[1], d1, ml[0] * d0), il, s0);
    } else {
#pragma unroll
      for (int c = 0; c < NC; ++c) o.f[c] = fma(-lam, zr[c] - zl[c], zl[C::fz(K, c)] + zr[C::fz(K, c)]);
      o.ul = o.ur = fma(zl[1 + K] - zr[1 + K], il, s0);
    }
  } else {
    const double ul = zl[0], ur = zr[0], s0 = ul + ur, du = ur - ul;
    if constexpr (CURV) {
      const double h = EQ == EQ_BURG ? 0.5 : 1.0;
      const double cl = h * fma(ph.vel1, ml[1], ph.vel0 * ml[0]), cr = h * fma(ph.vel1, mr[1], ph.vel0 * mr[0]);
      double lam = vmaxabs(cl, cr);
      if constexpr (EQ == EQ_BURG) lam = 2.0 * lam * vmaxabs(ul, ur);
      const double gl = gu<EQ>(ul), gr = gu<EQ>(ur);
      const double il = lam > 0.0 ? rcp_nr(lam) : 0.0;
      // an advection's factors of the two states, of which the downwind one's is
      // 0 where both sides have one coefficient, as on element faces: its
      // rounding must not enter a much smaller upwind state's update
      if constexpr (EQ == EQ_BURG) o.f[0] = fma(-lam, du, fma(cl, gl, cr * gr));
      else o.f[0] = fma(cl + lam, ul, (cr - lam) * ur);
      o.ul = fma(-(cr * (gr - gl)), il, s0);
      o.ur = fma(-(cl * (gr - gl)), il, s0);
    } else if constexpr (EQ == EQ_BURG) {
      const double cf = flux_coef<EQ>(K, ph, beta), gl = gu<EQ>(ul), gr = gu<EQ>(ur);
      const double lam = 2.0 * fabs(cf) * vmaxabs(ul, ur);
      const double il = lam > 0.0 ? rcp_nr(lam) : 0.0;
      o.f[0] = fma(-lam, du, cf * (gl + gr));
      o.ul = o.ur = fma(-(cf * (gr - gl)), il, s0);
    } else {
      // F_R - F_L over lambda = |coef| is +-(u_R - u_L): the upwind state.  The
      // flux from both states, of which the downwind one's factor is exactly 0:
      // a finite downwind state leaves no rounding in it, however large, and a
      // NaN or infinite one still makes it NaN.
      const double cf = flux_coef<EQ>(K, ph, beta);
      o.ul = o.ur = cf > 0.0 ? ul + ul : cf < 0.0 ? ur + ur : s0;
      o.f[0] = fma(vneg(cf), ur + ur, vpos(cf) * (ul + ul));
    }
  }
}

// Antidiffusive flux of an interior subcell face from its low-order flux o.f
// and the doubled f^H = F_0 + sum_e Q_e F_e of its element line: q points at
// the row 2 Q_e of the table, s at the slot of the line's first node.  (F_0
// stays out of the sum: folded into Q_0 it would double that entry's
// rounding, which constant states accumulate step by step.)
template <class C, int EQ, int DIM, int K, bool CURV>
__device__ __forceinline__ void face_high(const double* lds, const double* q, int s, const double* beta,
                                          const Phys& ph, FaceVal<C::NC>& o) {
  constexpr int NC = C::NC, N1 = C::N1, NSL = C::NSL, ST = K == 0 ? 1 : C::SPX;
  const double* z = lds + s;
  // p + 1 terms; the loop is unrolled as far as the registers of the loads
  // in flight fit beside the thread's node and faces
  constexpr int UN = CURV ? (N1 > 4 ? 2 : N1) : (N1 > 6 ? 3 : N1);
  // component c of the line's flux at node e, without the scalar laws' factor
  auto flux = [&](int e, int c) -> double {
    if constexpr (CURV) {
      const double m0 = z[(C::ZM + 2 * K) * NSL + e * ST], m1 = z[(C::ZM + 2 * K + 1) * NSL + e * ST];
      if constexpr (is_euler(EQ)) return fma(m1, z[C::fz(1, c) * NSL + e * ST], m0 * z[C::fz(0, c) * NSL + e * ST]);
      else return (EQ == EQ_BURG ? 0.5 : 1.0) * fma(ph.vel1, m1, ph.vel0 * m0) * gu<EQ>(z[e * ST]);
    } else {
      return is_euler(EQ) ? z[C::fz(K, c) * NSL + e * ST] : gu<EQ>(z[e * ST]);
    }
  };
  double acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const double f0 = flux(0, c);
    acc[c] = fma(q[0], f0, f0 + f0);
  }
#pragma unroll UN
  for (int e = 1; e < N1; ++e) {
    const double qe = q[e];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = fma(qe, flux(e, c), acc[c]);
  }
  if constexpr (is_euler(EQ) || CURV) {
#pragma unroll
    for (int c = 0; c < NC; ++c) o.g[c] = o.f[c] - acc[c];
  } else {
    o.g[0] = fma(-flux_coef<EQ>(K, ph, beta), acc[0], o.f[0]);
  }
}

// The face of direction K at grid node (i, j) whose right (upper) node's
// data are zr; the left node's come from the slot grid.  pos: the node's
// position along its element line (0: an element face).
template <class C, int EQ, int DIM, int K, bool CURV>
__device__ __forceinline__ void node_face(const double* lds, const double* zr, const double* beta, int i, int j,
                                          int pos, const Phys& ph, FaceVal<C::NC>& o) {
  constexpr int ST = K == 0 ? 1 : C::SPX;
  const int sl = C::sl(i, j) - ST;
  double zl[C::NZ];
#pragma unroll
  for (int q = 0; q < C::ZM; ++q) {
    // the fluxes of the other direction are read on curved meshes only
    if (is_euler(EQ) && !CURV && DIM == 2 && (q == C::NC + 2 - 2 * K || q == C::NC + 4 - K)) continue;
    zl[q] = lds[q * C::NSL + sl];
  }
  double ml[2], mr[2];
  if constexpr (CURV) {
    const int mo = (C::ZM + (pos ? 4 : 0) + 2 * K) * C::NSL + sl;
    ml[0] = lds[mo];
    ml[1] = lds[mo + C::NSL];
    mr[0] = pos ? zr[C::ZM + 4 + 2 * K] : ml[0];
    mr[1] = pos ? zr[C::ZM + 5 + 2 * K] : ml[1];
  }
  face_low<C, EQ, DIM, K, CURV>(zl, zr, beta, ml, mr, ph, o);
  if (pos) {
    face_high<C, EQ, DIM, K, CURV>(lds, lds + C::S_Q + (pos - 1) * C::N1, sl - (pos - 1) * ST, beta, ph, o);
  } else {
#pragma unroll
    for (int c = 0; c < C::NC; ++c) o.g[c] = 0.0;
  }
}

// log10(x) for normal x > 0: x = m 2^e with m in [1/sqrt 2, sqrt 2) and, with
// s = (m-1)/(m+1), ln m = 2 (s + s^3/3 + s^5/5 + ...), whose terms past s^21
// are below 1e-18.
__device__ inline double log10_series(double x) {
  int e;
  double m = frexp(x, &e);
  const bool up = m < 0.70710678118654752;
  m = up ? 2.0 * m : m;
  e -= up ? 1 : 0;
  const double s = (m - 1.0) * rcp_nr(m + 1.0), z = s * s;
  double a = 1.0 / 21.0;
#pragma unroll
  for (int k = 19; k >= 1; k -= 2) a = fma(a, z, 1.0 / k);
  return fma((double)e, 0.30102999566398120, 2.0 * s * a * 0.43429448190325183);
}

// sin(pi y / 2) for |y| <= 1 by its Taylor series (terms past y^23 are below
// 1e-20).
__device__ inline double sin_half_pi(double y) {
  const double z = (M_PI * 0.5) * (M_PI * 0.5) * y * y;
  double a = 1.0;
#pragma unroll
  for (int k = 11; k >= 1; --k) a = fma(a, -z * (1.0 / (2 * k * (2 * k + 1))), 1.0);
  return M_PI * 0.5 * y * a;
}

// Subcell-resolution smoothness factor of every element of the tile
// (Sec. 4.4) from the limited component in the slot grid: the L2 energy
// fraction of the modes of degree p in any variable, s_K = log10 of it and
// eps_K on the ramp 1/2 + 1/2 sin(pi (s_K - s0)/2) between s0 - 1 (0) and
// s0 + 1 (1).  An element whose polynomial is zero is smooth (0).
// The Gauss-Lobatto sums are the exact Legendre norms n_k = 2/(2k+1) except
// for k = p, whose discrete norm is g = 2/p.  So with D the discrete energy of
// the element, X_b and Y_a the degree-p coefficients of its rows and columns,
// q that of X, and |.|^2 the discrete norm of a line,
//   x = |X|^2 - g q^2, y = |Y|^2 - g q^2   (sum over l < p of n_l c_pl^2, c_lp^2)
//   energy of degree p:  n_p (x + y + n_p q^2)
//   whole energy:        D - (g - n_p) (x + y) - (g^2 - n_p^2) q^2,
// and no other mode is needed: one thread per row and per column, then one
// per element, two barriers.  (The whole modal transform, by one thread per
// row and mode, was a third of a p = 5 stage.)  An infinite energy is no
// fraction of anything: the factor is NaN, and with it the relaxed bounds.  m is the table's row that
// gives the degree-p coefficient, w the weights on [0,1]; uses the exchange
// array scr as scratch; returns the factor of the thread's element.  Sums run
// in a fixed order, so the result does not depend on the launch.
template <int EQ, int DIM, int P, int TX, int TY, bool CURV>
__device__ inline double smoothness_tile(const double* u0, const double* m, const double* w, double s0,
                                         const Place<Cfg<EQ, DIM, P, TX, TY, CURV>, DIM>& pl, double* scr) {
  using C = Cfg<EQ, DIM, P, TX, TY, CURV>;
  constexpr int N1 = P + 1, TP = C::TGX;
  constexpr double NP = 2.0 / (2.0 * P + 1.0), G = 2.0 / P;
  const int tid = threadIdx.x;
  const double* u = u0 + C::sl(pl.i, pl.j);
  double c = 0.0, e = 0.0;
  if (pl.own && pl.a == 0) {   // the row's degree-p coefficient and energy
#pragma unroll
    for (int q = 0; q < N1; ++q) {
      c = fma(m[q], u[q], c);
      e = fma(w[q] * u[q], u[q], e);
    }
    if constexpr (DIM == 2) {
      scr[tid] = c;
      scr[tid + 1] = 2.0 * e;
    }
  }
  if constexpr (DIM == 2) {
    if (pl.own && pl.b == 0) {   // the column's degree-p coefficient
      double d = 0.0;
#pragma unroll
      for (int q = 0; q < N1; ++q) d = fma(m[q], u[q * C::SPX], d);
      scr[tid + pl.a * (TP - 1) + 2] = d;
    }
    __syncthreads();
  }
  if (pl.own && pl.a == 0 && pl.b == 0) {
    double hi, tot, D = 0.0;
    if constexpr (DIM == 2) {
      double X = 0.0, Y = 0.0, q = 0.0;
#pragma unroll
      for (int r = 0; r < N1; ++r) {
        const double x = scr[tid + r * TP], y = scr[tid + r * TP + 2], w2 = 2.0 * w[r];
        D = fma(w2, scr[tid + r * TP + 1], D);
        X = fma(w2 * x, x, X);
        Y = fma(w2 * y, y, Y);
        q = fma(m[r], x, q);
      }
      const double q2 = q * q, xy = fma(-2.0 * G, q2, X + Y);
      hi = NP * fma(NP, q2, xy);
      tot = fma(-(G - NP), xy, fma(-(G * G - NP * NP), q2, D));
    } else {
      hi = NP * c * c;
      D = 2.0 * e;
      tot = fma(-(G - NP) * c, c, D);
    }
    double eps = 0.0;
    if (tot > 0.0 && hi > 0.0) {
      const double y = log10_series(hi / tot) - s0;
      eps = y < -1.0 ? 0.0 : y > 1.0 ? 1.0 : fma(0.5, sin_half_pi(y), 0.5);
    }
    scr[tid] = D < INFINITY || D != D ? eps : NAN;
  }
  __syncthreads();
  return pl.own ? scr[tid - pl.a - pl.b * TP] : 1.0;
}

// Sets a diagnostic flag.  A flag that is up already is only read: where every
// wave of a mesh has a reason to set it (a state that the unlimited scheme has
// driven to NaN), their atomics on one address took most of the step, 2.3 to
// 2.6 ms at 465 x 416, p = 4, which takes 0.49 so.
__device__ inline void raise_flag(unsigned int* flag) {
  if (!__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicOr(flag, 1u);
}

// ----------------------------------------------------------------------
// the fused stage kernel
// ----------------------------------------------------------------------
// One tile of one solve, run by one workgroup of C::BS threads on C::LDS
// doubles of LDS, with the degree tables T.  Shared by the plain kernel
// (the tiles of one solve) and the batched work-list kernel (the tiles of
// every solve of one degree).  FOLD: the time-step bound is folded from the
// minima of F (a step's first stage on a small mesh).
template <int EQ, int DIM, int P, int TX, int TY, bool CURV = false, bool FOLD = false>
__device__ __forceinline__ void stage_tile(double* lds, const StageArgs& A, const Tables& T, const Bnd& bnd,
                                           int tile, const FoldArgs& F = FoldArgs{}) {
  using C = Cfg<EQ, DIM, P, TX, TY, CURV>;
  static_assert(!CURV || (DIM == 2 && EQ != EQ_ADVV), "curved meshes: 2-D, flux F(u)");
  constexpr int NC = C::NC, N1 = C::N1, NB = C::NB, TP = C::TGX, GN = gn_of(EQ);
  const int tid = threadIdx.x;
  const Solve& S = A.S;
  const TileGeo tg = tile_geo<DIM, TX, TY>(tile, S.ntx, S.ntx_mul, S.ntx_shift, S.nx, S.ny);
  if (tg.tw <= 0 || tg.th <= 0) return;  // whole workgroup
  const long long nn = S.nn;

  const Place<C, DIM> at = place<C, DIM>(tg);
  const int i = at.i, j = at.j;

  // ---- phases 1-2: states, pointwise physics ----
  static_assert(P * (P + 1) <= C::BS, "one table entry per thread");
  const bool modal = A.limiter == LIM_SUBCELL_SI;
  TableRegs<P> tr;
  tr.fetch(T);
  const Src src = node_src<DIM, P, (C::OL > 0)>(i, j, tg, S.nx, S.ny, bnd.open);
  double z[C::NZ], detn = 1.0;
  if (at.any()) {
#pragma unroll
    for (int c = 0; c < NC; ++c) z[c] = S.u_s[c * nn + src.g];
    if constexpr (CURV) {
      if (at.own) {
#pragma unroll
        for (int q = 0; q < 8; ++q) z[C::ZM + q] = S.metric[q * nn + src.g];
        detn = S.metric[8 * nn + src.g];
      }
    }
  }
  double beta[2] = {0.0, 0.0};   // the velocity on the node's x-line and y-line
  if constexpr (EQ == EQ_ADVV) {
    if (at.any()) {
      beta[0] = A.ph.vrow[src.row];
      beta[1] = A.ph.vcol[src.col];
    }
  }
  // the halo nodes outside the thread grid, one per thread of the first
  // wave(s); all loads in flight before any use
  double zh[C::NZ];
  Src hs;
  int hi = 0, hj = 0;
  bool halo = false;
  if constexpr (C::NHX > 0) {
    halo = tid < C::NHX && ring_node<C>(tid, at.cw, at.ch, &hi, &hj);
    if (halo) {
      hs = node_src<DIM, P, true>(hi, hj, tg, S.nx, S.ny, bnd.open);
#pragma unroll
      for (int c = 0; c < NC; ++c) zh[c] = S.u_s[c * nn + hs.g];
      if constexpr (CURV) {
#pragma unroll
        for (int q = 0; q < 8; ++q) zh[C::ZM + q] = S.metric[q * nn + hs.g];
      }
    }
  }
  double dt;
  if constexpr (FOLD) {
    const double v = wave_min63(strided_min<C::BS>(F.partial, 0, F.n));
    if ((tid & 63) == 63) lds[C::S_R + (tid >> 6)] = v;
  } else {
    // (scalar loads, in the shadow of the states')
    dt = S.dt_dev ? S.dt_scale * S.dt_dev[0] : S.dt;
    if (!(dt < INFINITY)) dt = 0.0;  // no dissipation anywhere: nothing moves
  }
  bool bad = false;
  double K = INFINITY;   // Euler: p rho^-gamma of the node
  if (at.any()) {
    if (bnd.open && src.ext) exterior_state<EQ, DIM, NC>(bnd, src, S.nx * N1, S.ny * N1, z);
    node_state<C, EQ, DIM>(z, A.ph, K, bad);
    if (at.own || at.left) {
      const int t = C::sl(i, j);
#pragma unroll
      for (int q = 0; q < C::NZ; ++q) lds[q * C::NSL + t] = z[q];
    }
    if constexpr (is_euler(EQ)) lds[C::A_K + C::kl(i, j)] = K;
  }
  if constexpr (C::NHX > 0) {
    if (halo) {
      bool b = false;
      double Kh = INFINITY;
      if (bnd.open && hs.ext) exterior_state<EQ, DIM, NC>(bnd, hs, S.nx * N1, S.ny * N1, zh);
      node_state<C, EQ, DIM>(zh, A.ph, Kh, b);
      bad |= b;
      const int t = C::sl(hi, hj);
#pragma unroll
      for (int q = 0; q < C::NZ; ++q) lds[q * C::NSL + t] = zh[q];
      if constexpr (is_euler(EQ)) lds[C::A_K + C::kl(hi, hj)] = Kh;
    }
  }
  if (bad && A.diag) raise_flag(&A.diag->bad_input);
  tr.store(lds + C::S_W, lds + C::S_Q, lds + C::S_IW, lds + C::S_M);
  if (tid == 0) *reinterpret_cast<int*>(lds + C::S_LN) = 0;
  __syncthreads();

  if constexpr (FOLD) {
    double v = lds[C::S_R];
#pragma unroll
    for (int q = 1; q < C::NW; ++q) v = vmin(v, lds[C::S_R + q]);
    if (blockIdx.x == 0 && tid == 0) F.pub[0] = v;
    dt = S.dt_scale * v;
    if (!(dt < INFINITY)) dt = 0.0;
  }

  // K_min over the node and its 2d grid neighbours (Euler)
  double kmin = K;
  if constexpr (is_euler(EQ)) {
    if (at.own) {
      const double* k = lds + C::A_K + C::kl(i, j);
      kmin = vmin(kmin, vmin(k[-1], k[1]));
      if constexpr (DIM == 2) kmin = vmin(kmin, vmin(k[-C::KPX], k[C::KPX]));
    }
  }

  // smoothness factor of the node's element (SUBCELL_SI; p = 1 keeps the
  // strict bounds); the nodal-alpha array is free scratch until phase 4
  double eps = 1.0;
  if constexpr (P > 1) {
    if (modal)
      eps = smoothness_tile<EQ, DIM, P, TX, TY, CURV>(lds, lds + C::S_M, lds + C::S_W, T.s0, at, lds + C::S_AL);
  }

  // ---- phase 3: the faces to the node's left and below ----
  FaceVal<NC> fx, fy, fe;   // set where the thread owns the face
  if (at.face_x()) node_face<C, EQ, DIM, 0, CURV>(lds, z, beta, i, j, at.a, A.ph, fx);
  if constexpr (DIM == 2) {
    if (at.face_y()) node_face<C, EQ, DIM, 1, CURV>(lds, z, beta, i, j, at.b, A.ph, fy);
  }
  // the faces on the tile's high edges (element faces), where the thread
  // grid has no node for them: taken by the last wave
  int eo = -1, ek = 0;   // exchange node and direction
  if constexpr (C::NEF > 0) {
    const int e = tid - (C::BS - 64);
    if (e >= 0) {
      double ze[C::NZ], be[2] = {0.0, 0.0};
      const bool ex = e < C::GY;
      const int q = ex ? e : e - C::GY;   // row of an x-face, column of a y-face
      if (ex ? q < at.ch : q < at.cw && q < C::GX) {
        const int ei = ex ? at.cw : q, ej = ex ? q : at.ch;
        const int t = C::sl(ei, ej);
#pragma unroll
        for (int m = 0; m < C::ZM; ++m) ze[m] = lds[m * C::NSL + t];
        if constexpr (EQ == EQ_ADVV) {
          if (ex) be[0] = A.ph.vrow[tg.ey0 * N1 + q];
          else be[1] = A.ph.vcol[tg.ex0 * N1 + q];
        }
        if (ex) node_face<C, EQ, DIM, 0, CURV>(lds, ze, be, ei, ej, 0, A.ph, fe);
        else node_face<C, EQ, DIM, 1, CURV>(lds, ze, be, ei, ej, 0, A.ph, fe);
        ek = ex ? 0 : 1;
        eo = C::nd(ei, ej) - (ex ? 1 : TP);
      }
    }
  }
  __syncthreads();  // region A is dead from here on
  const int n = tid;   // the node's index in the exchange arrays
  if (at.face_x() && i > 0) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      lds[C::b_f(0) + c * NB + n - 1] = fx.f[c];
      lds[C::b_g(0) + c * NB + n - 1] = fx.g[c];
    }
    lds[C::b_u(0) + n - 1] = fx.ul;
  }
  if constexpr (DIM == 2) {
    if (at.face_y() && j > 0) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        lds[C::b_f(1) + c * NB + n - TP] = fy.f[c];
        lds[C::b_g(1) + c * NB + n - TP] = fy.g[c];
      }
      lds[C::b_u(1) + n - TP] = fy.ul;
    }
  }
  if constexpr (C::NEF > 0) {
    if (eo >= 0) {
      const int of = ek ? C::b_f(1) : C::b_f(0), og = ek ? C::b_g(1) : C::b_g(0), ou = ek ? C::b_u(1) : C::b_u(0);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        lds[of + c * NB + eo] = fe.f[c];
        lds[og + c * NB + eo] = 0.0;
      }
      lds[ou + eo] = fe.ul;
    }
  }
  __syncthreads();

  // ---- phase 4a: low-order state, bounds, Zalesak, entropy checks ----
  double uL[NC], un[NC], alpha = 1.0, az = 1.0, umin = 0.0, umax = 0.0, hx = 0.0, hy = 0.0;
  bool lov = false;
  const bool elementwise = A.limiter == LIM_ELEMENTWISE;
  int search = 0;   // Euler: the node's faces for the search list
  double g2[2] = {0.0, 0.0}, pm = 0.0;
  if (at.own) {
    // dt / (2 w h) along each direction (a curved mesh: dt / (2 w det(J)))
    const double hdt = 0.5 * dt;
    if constexpr (CURV) {
      const double id = hdt / detn;
      hx = id * lds[C::S_IW + at.a];
      hy = id * lds[C::S_IW + at.b];
    } else {
      hx = hdt * S.ihx * lds[C::S_IW + at.a];
      if constexpr (DIM == 2) hy = hdt * S.ihy * lds[C::S_IW + at.b];
    }
    double gx[NC], gy[NC];   // the antidiffusive fluxes of the right and upper face
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      uL[c] = fma(hx, fx.f[c] - lds[C::b_f(0) + c * NB + n], z[c]);
      gx[c] = lds[C::b_g(0) + c * NB + n];
      if constexpr (DIM == 2) {
        uL[c] = fma(hy, fy.f[c] - lds[C::b_f(1) + c * NB + n], uL[c]);
        gy[c] = lds[C::b_g(1) + c * NB + n];
      }
    }
    const double u2 = z[0] + z[0];
    const double b1 = lds[C::b_u(0) + n];
    umin = vmin(vmin(u2, fx.ur), b1);
    umax = vmax(vmax(u2, fx.ur), b1);
    if constexpr (DIM == 2) {
      const double b2 = lds[C::b_u(1) + n];
      umin = vmin(vmin(umin, fy.ur), b2);
      umax = vmax(vmax(umax, fy.ur), b2);
    }
    umin *= 0.5;
    umax *= 0.5;
    lov = vmin(umax - uL[0], uL[0] - umin) < -1e-12 * vmaxabs(umin, umax);
    if (modal) {  // eq. relaxed-bounds
      umin = eps * umin + (1.0 - eps) * A.gmin;
      umax = eps * umax + (1.0 - eps) * A.gmax;
    }
    if (A.limiter == LIM_TARGET || A.limiter == LIM_LOW) {
      alpha = A.limiter == LIM_TARGET ? 1.0 : 0.0;
    } else if (dt > 0.0) {
      // Zalesak: the room Q over the sum P of the corrections of one sign
      // (of the node's whole correction u^H - u^L in elementwise limiting,
      // Sec. 4.1.2, eq. convex-provisional-elementwise).  Without corrections
      // the ratio is 1; without room it is 0 exactly: anything more puts
      // subnormal values where the state is zero, which then leave their
      // bounds by their own rounding, step after step.  P is raised to at least
      // 2^-1021, the smallest magnitude whose reciprocal is finite, and for the
      // scalar laws lowered to the largest double, so that an infinite P leaves
      // nothing (an Euler correction with one fails the entropy check).
      double Pp, Pm, d[NC];
      if (elementwise) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          d[c] = hx * (gx[c] - fx.g[c]);
          if constexpr (DIM == 2) d[c] = fma(hy, gy[c] - fy.g[c], d[c]);
        }
        Pp = vpos(d[0]);
        Pm = vneg(d[0]);
      } else {
        Pp = hx * (vpos(gx[0]) - vneg(fx.g[0]));
        Pm = hx * (vneg(gx[0]) - vpos(fx.g[0]));
        if constexpr (DIM == 2) {
          Pp = fma(hy, vpos(gy[0]) - vneg(fy.g[0]), Pp);
          Pm = fma(hy, vneg(gy[0]) - vpos(fy.g[0]), Pm);
        }
      }
      constexpr double TINY = 0x1p-1021, BIG = 0x1.fffffffffffffp1023;
      double Sp = vmax(Pp, TINY), Sm = vmax(-Pm, TINY);
      if constexpr (!is_euler(EQ)) {
        Sp = vmin(Sp, BIG);
        Sm = vmin(Sm, BIG);
      }
      const double Rp = vpos(umax - uL[0]) * rcp_nr(Sp), Rm = vpos(uL[0] - umin) * rcp_nr(Sm);
      alpha = vmin(1.0, vmin(Pp > 0.0 ? Rp : 1.0, Pm < 0.0 ? Rm : 1.0));
      az = alpha;
      if constexpr (is_euler(EQ)) {
        // every partial state uL + t 2d dt/m (+-rbar) must stay admissible
        // for t <= alpha (eq. convex-provisional), and in elementwise
        // limiting uL + t (u^H - u^L).  A face whose partial state at
        // t = alpha is not admissible beyond doubt goes to the workgroup's
        // search list, which finds its root on [0, alpha] starting from the
        // exact value at alpha; most faces pass here with integer powers
        // only.  A node whose partial-state corrections are all below the
        // search tolerance (max|P| over its faces <= 1e-14 max|u^L|) needs no
        // search: any t in [0, alpha] moves its state by less than that,
        // which is as close as a search would get (in a uniform region the
        // antidiffusive fluxes are of rounding size and Phi at alpha is zero
        // to rounding, which no test could settle).  The comparisons are such
        // that a NaN correction is searched, and takes nothing.
        g2[0] = 2.0 * DIM * hx;
        g2[1] = 2.0 * DIM * hy;
        const double ikg = vpos(A.ph.gsure * rcp_nr(kmin));
        if (elementwise) {
          search = surely_admissible<DIM, GN>(alpha, uL, d, ikg, A.ph) ? 0 : 1;
        } else {
          // largest component of every face's flux
          double us = vmaxabs(uL[0], uL[1]), r0 = vmaxabs(fx.g[0], fx.g[1]), r1 = vmaxabs(gx[0], gx[1]), r2 = 0.0, r3 = 0.0;
          if constexpr (DIM == 2) {
            r2 = vmaxabs(fy.g[0], fy.g[1]);
            r3 = vmaxabs(gy[0], gy[1]);
          }
#pragma unroll
          for (int c = 2; c < NC; ++c) {
            us = vmaxabs(us, uL[c]);
            r0 = vmaxabs(r0, fx.g[c]);
            r1 = vmaxabs(r1, gx[c]);
            if constexpr (DIM == 2) {
              r2 = vmaxabs(r2, fy.g[c]);
              r3 = vmaxabs(r3, gy[c]);
            }
          }
          pm = g2[0] * vmax(r0, r1);
          if constexpr (DIM == 2) pm = vmax(pm, g2[1] * vmax(r2, r3));
          if (!(pm <= 1e-14 * us)) {
            // the partial state at alpha, uL + (alpha 2d dt/m) (+-rbar): the
            // screen only certifies with margins, so how its scale is
            // rounded does not matter (an uncertified face is searched
            // from the exact value at alpha)
            const double sx = alpha * g2[0], sy = alpha * g2[1];
            if (!surely_admissible<DIM, GN>(-sx, uL, fx.g, ikg, A.ph) && !(r0 <= 0.0)) search |= 1;
            if (!surely_admissible<DIM, GN>(sx, uL, gx, ikg, A.ph) && !(r1 <= 0.0)) search |= 2;
            if constexpr (DIM == 2) {
              if (!surely_admissible<DIM, GN>(-sy, uL, fy.g, ikg, A.ph) && !(r2 <= 0.0)) search |= 4;
              if (!surely_admissible<DIM, GN>(sy, uL, gy, ikg, A.ph) && !(r3 <= 0.0)) search |= 8;
            }
          }
        }
      }
    }
    lds[C::S_AL + n] = alpha;
    if (A.use_un) {   // in flight through the searches
#pragma unroll
      for (int c = 0; c < NC; ++c) un[c] = S.u_n[c * nn + src.g];
    }
  }
  if constexpr (is_euler(EQ)) {
    __syncthreads();  // the low-order fluxes are consumed: region C may overwrite them
    if (search) {
#pragma unroll
      for (int c = 0; c < NC; ++c) lds[C::C_UL + c * NB + n] = uL[c];
      lds[C::C_KM + n] = kmin;
      lds[C::C_AZ + n] = az;
#pragma unroll
      for (int k = 0; k < DIM; ++k) lds[C::C_G2 + k * NB + n] = g2[k];
      lds[C::C_PS + n] = pm;
    }
    // one place in the list per face: a wave counts its faces of each kind,
    // takes the places with one atomic and ranks its lanes
    {
      unsigned short* list = reinterpret_cast<unsigned short*>(lds + C::C_LIST);
      unsigned long long m[2 * DIM];
      int total = 0;
#pragma unroll
      for (int f = 0; f < 2 * DIM; ++f) {
        m[f] = __ballot((search >> f) & 1);
        total += __popcll(m[f]);
      }
      if (total > 0) {   // wave-uniform
        int at0 = 0;
        if ((tid & 63) == 0) at0 = atomicAdd(reinterpret_cast<int*>(lds + C::S_LN), total);
        at0 = __builtin_amdgcn_readfirstlane(at0);
#pragma unroll
        for (int f = 0; f < 2 * DIM; ++f) {
          const int r = __builtin_amdgcn_mbcnt_hi((unsigned)(m[f] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m[f], 0u));
          if ((search >> f) & 1) list[at0 + r] = (unsigned short)(n * 4 + f);
          at0 += __popcll(m[f]);
        }
      }
    }
    __syncthreads();
    // ---- phase 4b: entropy line searches, spread over the workgroup ----
    // u^L itself is checked first where it is not admissible beyond doubt
    // (u^L off the set by rounding leaves the node at alpha = 0)
    const int nact = *reinterpret_cast<const int*>(lds + C::S_LN);
    const unsigned short* list = reinterpret_cast<const unsigned short*>(lds + C::C_LIST);
    for (int w = tid; w < nact; w += C::BS) {
      const int item = list[w];
      const int node = item >> 2, k = (item >> 1) & 1, sd = item & 1;
      double ul[NC], Pv[NC];
      if (elementwise) {   // u^H - u^L, formed as in phase 4a
        const int nj = (unsigned)node / (unsigned)TP, ni = node - nj * TP - C::OL;
        const bool a0 = ni % N1 == 0, b0 = nj % N1 == 0;
        const double qx = lds[C::C_G2 + node] * (0.5 / DIM), qy = DIM == 2 ? lds[C::C_G2 + NB + node] * (0.5 / DIM) : 0.0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const double* g = lds + c * NB + node;
          Pv[c] = qx * (g[C::b_g(0)] - (a0 ? 0.0 : g[C::b_g(0) - 1]));
          if constexpr (DIM == 2) Pv[c] = fma(qy, g[C::b_g(1)] - (b0 ? 0.0 : g[C::b_g(1) - TP]), Pv[c]);
        }
      } else {
        const double gs = lds[C::C_G2 + k * NB + node];
        const double* rb = lds + (k ? C::b_g(1) : C::b_g(0)) + (sd ? node : node - (k ? TP : 1));
#pragma unroll
        for (int c = 0; c < NC; ++c) Pv[c] = (sd ? gs : -gs) * rb[c * NB];
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) ul[c] = lds[C::C_UL + c * NB + node];
      const double km = lds[C::C_KM + node], am = lds[C::C_AZ + node];
      const double zero[NC] = {};
      bool feasible = surely_admissible<DIM, GN>(0.0, ul, zero, vpos(A.ph.gsure * rcp_nr(km)), A.ph);
      if (!feasible) feasible = admissible(phi_at<DIM, GN>(0.0, ul, zero, km, A.ph));
      double t = 0.0;
      if (elementwise) {
        const PhiVal ea = phi_at<DIM, GN>(am, ul, Pv, km, A.ph);
        if (admissible(ea)) {
          t = am;
        } else if (feasible) {
          double tn = ea.rho > 0.0 && ea.dphi < 0.0 ? am - ea.phi / ea.dphi : am;
          tn = vmin(vpos(tn), am);
          t = entropy_root<DIM, GN>(ul, Pv, tn, km, A.ph);
        }
      } else if (feasible) {
        t = entropy_root_face<DIM, GN>(ul, Pv, am, km, lds[C::C_PS + node], A.ph);
      }
      atomicMin(reinterpret_cast<unsigned long long*>(lds + C::S_AL + node),
                (unsigned long long)__double_as_longlong(t));
    }
  }
  __syncthreads();

  // ---- phase 5: subcell-face coefficients, corrected update, RK stage ----
  bool limited = false, ent = false;
  if (at.own) {
    alpha = lds[C::S_AL + n];
    // the node's own coefficient was lowered by the entropy search
    ent = is_euler(EQ) && A.limiter != LIM_TARGET && A.limiter != LIM_LOW && alpha < az;
    if (elementwise) {  // one coefficient per element: the minimum over its nodes
      const double* ae = lds + C::S_AL + n - at.b * TP - at.a;
      for (int bb = 0; bb < (DIM == 2 ? N1 : 1); ++bb)
        for (int aa = 0; aa < N1; ++aa) alpha = vmin(alpha, ae[bb * TP + aa]);
    }
    limited = alpha < 1.0;
    if (A.trace) {
      const bool lim = is_euler(EQ) && dt > 0.0 && A.limiter != LIM_TARGET && A.limiter != LIM_LOW;
      A.trace[src.g] = umin;
      A.trace[nn + src.g] = umax;
      A.trace[2 * nn + src.g] = lim ? kmin : 0.0;
      A.trace[3 * nn + src.g] = az;
      A.trace[4 * nn + src.g] = alpha;
    }
    // the antidiffusive fluxes are read again rather than kept through the
    // searches, whose registers set the kernel's
    double v[NC];
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
      constexpr int ST[2] = {1, TP};
      const int pos = k == 0 ? at.a : at.b;
      const double* g = lds + C::b_g(k) + n;
      double s[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) s[c] = 0.0;
      if (pos < P) {
        const double q = elementwise ? alpha : vmin(alpha, lds[C::S_AL + n + ST[k]]);
#pragma unroll
        for (int c = 0; c < NC; ++c) s[c] = q * g[c * NB];
      }
      if (pos > 0) {
        const double q = elementwise ? alpha : vmin(alpha, lds[C::S_AL + n - ST[k]]);
#pragma unroll
        for (int c = 0; c < NC; ++c) s[c] = fma(-q, g[c * NB - ST[k]], s[c]);
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) v[c] = fma(k == 0 ? hx : hy, s[c], k == 0 ? uL[c] : v[c]);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) S.u_out[c * nn + src.g] = A.use_un ? fma(A.b_s, v[c], A.a_s * un[c]) : v[c];
  }
  if (A.diag) {
    const unsigned long long bl = __ballot(limited), be = __ballot(ent), bv = __ballot(lov);
    if ((tid & 63) == 0) {
      const int slot = (blockIdx.x * C::NW + (tid >> 6)) & (DIAG_SLOTS - 1);
      if (bl) atomicAdd(&A.diag->limited[slot], (unsigned long long)__popcll(bl));
      if (be) atomicAdd(&A.diag->entropy[slot], (unsigned long long)__popcll(be));
      if (bv) raise_flag(&A.diag->lo_violation);
    }
  }
}

template <int EQ, int DIM, int P, int TX, int TY, bool CURV = false>
__global__ __launch_bounds__((Cfg<EQ, DIM, P, TX, TY, CURV>::BS), (Cfg<EQ, DIM, P, TX, TY, CURV>::WPE)) void stage_kernel(StageArgs A) {
  __shared__ double lds[Cfg<EQ, DIM, P, TX, TY, CURV>::LDS];
  stage_tile<EQ, DIM, P, TX, TY, CURV>(lds, A, A.T, A.bnd, xcd_tile(blockIdx.x, gridDim.x));
}

template <int EQ, int DIM, int P, int TX, int TY>
__global__ __launch_bounds__((Cfg<EQ, DIM, P, TX, TY>::BS), (Cfg<EQ, DIM, P, TX, TY>::WPEB)) void stage_fold_kernel(StageArgs A, FoldArgs F) {
  __shared__ double lds[Cfg<EQ, DIM, P, TX, TY>::LDS];
  stage_tile<EQ, DIM, P, TX, TY, false, true>(lds, A, A.T, A.bnd, xcd_tile(blockIdx.x, gridDim.x), F);
}

// ----------------------------------------------------------------------
// low-order CFL bound (eq. cfl-low): min over nodes of m_i/(2 sum dhauij)
// ----------------------------------------------------------------------
// The time-step kernel takes the same tiles and thread grid, and stages per
// slot only what the wave-speed bounds read: for Euler the velocity
// components and the auxiliaries c, c p^-ex, (gamma+1)/(2 gamma p); for
// Burgers the state; on a curved mesh the eight metric terms.  (An advection
// velocity needs no neighbour.)  Bound by vector issue like the stage: about
// 90 instructions of pointwise physics and 65 per face.  256 x 256 elements,
// p = 4, gamma = 7/5: 25.0 us a launch with one work item per face (355 vector
// instructions per wave), 19.6 us with a thread's two faces in registers (279),
// 2.7 TB/s of its 32 bytes per node.
template <int EQ, int DIM, int P, int TX, int TY, bool CURV = false>
struct DtCfg {
  using C = Cfg<EQ, DIM, P, TX, TY, CURV>;
  static constexpr int NV = is_euler(EQ) ? DIM + 3 : EQ == EQ_BURG ? 1 : 0;
  static constexpr int NZ = NV + (CURV ? 8 : 0), NZ1 = NZ > 0 ? NZ : 1;
  static constexpr int L = NZ * C::NSL;                    // wave speeds of the right (upper) faces [DIM][NB]
  static constexpr int IW = L + DIM * C::NB;               // 1/w
  static constexpr int R = IW + C::N1;                     // per-wave maxima
  static constexpr int LDS = R + C::NW;
};

// The wave-speed inputs of one state.
template <int EQ, int DIM>
__device__ inline void wave_inputs(const double* U, const Phys& ph, double* ws) {
  if constexpr (is_euler(EQ)) {
    double X[4], K, pr;
    bool bad;
    euler_aux<DIM, gn_of(EQ), false>(U, ph, X, K, pr, bad);
#pragma unroll
    for (int k = 0; k < DIM; ++k) ws[k] = U[1 + k] * X[0];
    ws[DIM] = X[1];
    ws[DIM + 1] = X[2];
    ws[DIM + 2] = X[3];
  } else if constexpr (EQ == EQ_BURG) {
    ws[0] = U[0];
  }
}

// Wave speed of the face in direction K between the staged inputs wl and wr:
// on a curved mesh scaled by the metric rows as in face_low.
template <class D, int EQ, int DIM, int K, bool CURV>
__device__ __forceinline__ double face_speed(const double* wl, const double* wr, const double* beta, const double* ml,
                                             const double* mr, const Phys& ph) {
  if constexpr (CURV) {
    double v[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const double* n = s == 0 ? mr : ml;
      if constexpr (is_euler(EQ)) {
        const double q = sqrt_nr(fma(n[1], n[1], n[0] * n[0]));
        v[s] = euler_lambda<gn_of(EQ)>(fma(wl[1], n[1], wl[0] * n[0]), fma(wr[1], n[1], wr[0] * n[0]), q * wl[2],
                                       q * wr[2], q * (wl[3] + wr[3]), wl[4], wr[4], ph);
      } else {
        v[s] = fma(ph.vel1, n[1], ph.vel0 * n[0]);
      }
    }
    if constexpr (is_euler(EQ)) return vmax(v[0], v[1]);
    else if constexpr (EQ == EQ_BURG) return vmaxabs(v[0], v[1]) * vmaxabs(wl[0], wr[0]);
    else return vmaxabs(v[0], v[1]);
  } else {
    if constexpr (is_euler(EQ))
      return euler_lambda<gn_of(EQ)>(wl[K], wr[K], wl[DIM], wr[DIM], wl[DIM + 1] + wr[DIM + 1], wl[DIM + 2],
                                     wr[DIM + 2], ph);
    else if constexpr (EQ == EQ_BURG) return vmaxabs(wl[0], wr[0]) * fabs(vel_k(K, ph));
    else return fabs(flux_coef<EQ>(K, ph, beta));
  }
}

template <class D, int EQ, int DIM, int K, bool CURV>
__device__ __forceinline__ double node_speed(const double* lds, const double* wr, const double* beta, int i, int j,
                                             int pos, const Phys& ph) {
  using C = typename D::C;
  const int sl = C::sl(i, j) - (K == 0 ? 1 : C::SPX);
  double wl[D::NZ1], ml[2], mr[2];
#pragma unroll
  for (int x = 0; x < D::NV; ++x) {
    if (is_euler(EQ) && !CURV && DIM == 2 && x == 1 - K) continue;   // the other velocity component
    wl[x] = lds[x * C::NSL + sl];
  }
  if constexpr (CURV) {
    const int mo = (D::NV + (pos ? 4 : 0) + 2 * K) * C::NSL + sl;
    ml[0] = lds[mo];
    ml[1] = lds[mo + C::NSL];
    mr[0] = pos ? wr[D::NV + 4 + 2 * K] : ml[0];
    mr[1] = pos ? wr[D::NV + 5 + 2 * K] : ml[1];
  }
  return face_speed<D, EQ, DIM, K, CURV>(wl, wr, beta, ml, mr, ph);
}

// the minimum of one tile into *out
template <int EQ, int DIM, int P, int TX, int TY, bool CURV = false>
__device__ __forceinline__ void maxdt_tile(double* lds, const MaxDtArgs& A, const Tables& T, const Bnd& bnd,
                                           int tile, double* out) {
  using D = DtCfg<EQ, DIM, P, TX, TY, CURV>;
  using C = typename D::C;
  constexpr int NC = C::NC, N1 = C::N1, NB = C::NB, TP = C::TGX;
  const int tid = threadIdx.x;
  const TileGeo tg = tile_geo<DIM, TX, TY>(tile, A.ntx, A.ntx_mul, A.ntx_shift, A.nx, A.ny);
  if (tg.tw <= 0 || tg.th <= 0) {   // whole workgroup
    if (tid == 0) *out = INFINITY;
    return;
  }
  const Place<C, DIM> at = place<C, DIM>(tg);
  const int i = at.i, j = at.j, n = tid;
  const double iwt = tid < N1 ? T.iw[tid] : 0.0;   // stored once the state has arrived
  const Src src = node_src<DIM, P, (C::OL > 0)>(i, j, tg, A.nx, A.ny, bnd.open);
  double U[NC], V[NC], w[D::NZ1], wh[D::NZ1], detn = 1.0;
  if (D::NV > 0 && at.any()) {
#pragma unroll
    for (int c = 0; c < NC; ++c) U[c] = A.u[c * A.nn + src.g];
  }
  if constexpr (CURV) {
    if (at.own) {
#pragma unroll
      for (int q = 0; q < 8; ++q) w[D::NV + q] = A.metric[q * A.nn + src.g];
      detn = A.metric[8 * A.nn + src.g];
    }
  }
  double beta[2] = {0.0, 0.0};
  if constexpr (EQ == EQ_ADVV) {
    if (at.any()) {
      beta[0] = A.ph.vrow[src.row];
      beta[1] = A.ph.vcol[src.col];
    }
  }
  Src hs;
  int hi = 0, hj = 0;
  bool halo = false;
  if constexpr (C::NHX > 0 && D::NZ > 0) {
    halo = tid < C::NHX && ring_node<C>(tid, at.cw, at.ch, &hi, &hj);
    if (halo) {
      hs = node_src<DIM, P, true>(hi, hj, tg, A.nx, A.ny, bnd.open);
      if constexpr (D::NV > 0) {
#pragma unroll
        for (int c = 0; c < NC; ++c) V[c] = A.u[c * A.nn + hs.g];
      }
      if constexpr (CURV) {
#pragma unroll
        for (int q = 0; q < 8; ++q) wh[D::NV + q] = A.metric[q * A.nn + hs.g];
      }
    }
  }
  if (D::NZ > 0 && at.any()) {
    if (bnd.open && src.ext) exterior_state<EQ, DIM, NC>(bnd, src, A.nx * N1, A.ny * N1, U);
    wave_inputs<EQ, DIM>(U, A.ph, w);
    if (at.own || at.left) {
      const int t = C::sl(i, j);
#pragma unroll
      for (int x = 0; x < D::NZ; ++x) lds[x * C::NSL + t] = w[x];
    }
  }
  if constexpr (C::NHX > 0 && D::NZ > 0) {
    if (halo) {
      if (bnd.open && hs.ext) exterior_state<EQ, DIM, NC>(bnd, hs, A.nx * N1, A.ny * N1, V);
      wave_inputs<EQ, DIM>(V, A.ph, wh);
      const int t = C::sl(hi, hj);
#pragma unroll
      for (int x = 0; x < D::NZ; ++x) lds[x * C::NSL + t] = wh[x];
    }
  }
  if (tid < N1) lds[D::IW + tid] = iwt;
  __syncthreads();
  double lx = 0.0, ly = 0.0;
  if (at.face_x()) {
    lx = node_speed<D, EQ, DIM, 0, CURV>(lds, w, beta, i, j, at.a, A.ph);
    if (i > 0) lds[D::L + n - 1] = lx;
  }
  if constexpr (DIM == 2) {
    if (at.face_y()) {
      ly = node_speed<D, EQ, DIM, 1, CURV>(lds, w, beta, i, j, at.b, A.ph);
      if (j > 0) lds[D::L + NB + n - TP] = ly;
    }
  }
  if constexpr (C::NEF > 0) {   // the faces on the tile's high edges: the last wave
    const int e = tid - (C::BS - 64);
    if (e >= 0) {
      const bool ex = e < C::GY;
      const int q = ex ? e : e - C::GY;
      if (ex ? q < at.ch : q < at.cw && q < C::GX) {
        const int ei = ex ? at.cw : q, ej = ex ? q : at.ch;
        double we[D::NZ1], be[2] = {0.0, 0.0};
        const int t = C::sl(ei, ej);
#pragma unroll
        for (int x = 0; x < D::NV; ++x) we[x] = lds[x * C::NSL + t];
        if constexpr (EQ == EQ_ADVV) {
          if (ex) be[0] = A.ph.vrow[tg.ey0 * N1 + q];
          else be[1] = A.ph.vcol[tg.ex0 * N1 + q];
        }
        if (ex) lds[D::L + C::nd(ei, ej) - 1] = node_speed<D, EQ, DIM, 0, CURV>(lds, we, be, ei, ej, 0, A.ph);
        else lds[D::L + NB + C::nd(ei, ej) - TP] = node_speed<D, EQ, DIM, 1, CURV>(lds, we, be, ei, ej, 0, A.ph);
      }
    }
  }
  __syncthreads();
  // 2 sum dhat / m of the node: the line weights cancel against the mass
  // (m_i = w_a w_b h_x h_y, or w_a w_b det(J)); the bound is the reciprocal of
  // the largest
  double r = 0.0;
  if (at.own) {
    r = (lx + lds[D::L + n]) * lds[D::IW + at.a];
    if constexpr (!CURV) r *= A.ihx;
    if constexpr (DIM == 2) {
      double s = (ly + lds[D::L + NB + n]) * lds[D::IW + at.b];
      if constexpr (!CURV) s *= A.ihy;
      r += s;
    }
    if constexpr (CURV) r /= detn;
  }
  r = wave_max63(r);
  if ((tid & 63) == 63) lds[D::R + (tid >> 6)] = r;
  __syncthreads();
  if (tid == 0) {
    r = lds[D::R];
#pragma unroll
    for (int q = 1; q < C::NW; ++q) r = vmax(r, lds[D::R + q]);
    *out = 1.0 / vpos(r);   // +infinity too where every node's speed is NaN
  }
}

template <int EQ, int DIM, int P, int TX, int TY, bool CURV = false>
__global__ __launch_bounds__((Cfg<EQ, DIM, P, TX, TY, CURV>::BS)) void maxdt_kernel(MaxDtArgs A) {
  __shared__ double lds[DtCfg<EQ, DIM, P, TX, TY, CURV>::LDS];
  maxdt_tile<EQ, DIM, P, TX, TY, CURV>(lds, A, A.T, A.bnd, xcd_tile(blockIdx.x, gridDim.x),
                                       A.partial + blockIdx.x);
}

// ----------------------------------------------------------------------
// one-workgroup steps (1-D): the time-step bound and the three stages in one
// launch, on a tile that holds the whole mesh.  A step of a few hundred nodes
// is all launches and latency: 64 elements of p = 3 advection took 24.5 us
// in five launches of 2 to 4 us each and take 7.3 us in one.
// The stages pass their states through the handle's buffers as the
// launches do; a workgroup sees its own stores after a barrier.
// ----------------------------------------------------------------------
template <int EQ, int P, int TX>
__global__ __launch_bounds__((Cfg<EQ, 1, P, TX, 1>::BS)) void step1_kernel(StepArgs B) {
  using C = Cfg<EQ, 1, P, TX, 1>;
  using D = DtCfg<EQ, 1, P, TX, 1>;
  __shared__ double lds[C::LDS > D::LDS ? C::LDS : D::LDS];
  __shared__ double bound;
  StageArgs A;
  A.S = B.A.S;
  A.ph = B.A.ph;
  A.limiter = B.A.limiter;
  A.diag = B.A.diag;
  A.trace = nullptr;
  A.gmin = B.A.gmin;
  A.gmax = B.A.gmax;
  A.S.dt_dev = nullptr;
  if (B.cfl > 0.0) {
    MaxDtArgs M;
    M.u = B.u;
    M.nn = A.S.nn;
    M.nx = A.S.nx;
    M.ny = A.S.ny;
    M.ntx = A.S.ntx;
    M.ntx_mul = A.S.ntx_mul;
    M.ntx_shift = A.S.ntx_shift;
    M.ihx = A.S.ihx;
    M.ihy = A.S.ihy;
    M.ph = A.ph;
    M.metric = nullptr;
    maxdt_tile<EQ, 1, P, TX, 1>(lds, M, B.A.T, B.A.bnd, 0, &bound);
    __syncthreads();
    A.S.dt = B.cfl * bound;
    if (threadIdx.x == 0) B.dt_pub[0] = bound;
  }
#pragma unroll 1
  for (int s = 0; s < 3; ++s) {
    A.S.u_n = B.u;
    A.S.u_s = s == 0 ? B.u : s == 1 ? B.buf1 : B.buf2;
    A.S.u_out = s == 0 ? B.buf1 : s == 1 ? B.buf2 : B.u;
    A.use_un = s > 0;
    A.a_s = s == 0 ? 0.0 : s == 1 ? 0.75 : 1.0 / 3.0;
    A.b_s = s == 0 ? 1.0 : s == 1 ? 0.25 : 2.0 / 3.0;
    stage_tile<EQ, 1, P, TX, 1>(lds, A, B.A.T, B.A.bnd, 0);
    __syncthreads();   // the stage's stores, and its LDS
  }
}

template <int EQ, int DIM, int P>
hipError_t launch_step1_t(const StepArgs& a, hipStream_t s) {
  if constexpr (DIM == 1) {
    constexpr int T0 = 254 / (P + 1), T1 = step1_nodes(EQ) / (P + 1);
    if (a.A.S.nx <= T0) hipLaunchKernelGGL((step1_kernel<EQ, P, T0>), dim3(1), dim3(Cfg<EQ, 1, P, T0, 1>::BS), 0, s, a);
    else if (a.A.S.nx <= T1) hipLaunchKernelGGL((step1_kernel<EQ, P, T1>), dim3(1), dim3(Cfg<EQ, 1, P, T1, 1>::BS), 0, s, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  } else {
    (void)a;
    (void)s;
    return hipErrorInvalidValue;
  }
}

// ----------------------------------------------------------------------
// tile shapes (TX x TY elements) per degree: variant 0 is a new handle's,
// variant 1 the alternative the tuner may pick, variant 2 that of curved
// meshes.  Variant 0 fills four waves as far as the degree lets it (216 to 256
// own nodes, 19.7 to 23.8 G node-updates/s per Euler stage at 2 M nodes; the
// other shapes are up to 14 % slower: p = 6, 5 x 1 elements 99.9 us a stage,
// 2 x 2 110.5; p = 8, 3 x 1 106.5, 2 x 1 113.8).  On a mesh of one workgroup a
// CU or less the shorter workgroup of shape 1 is up to 9 % faster (p = 6,
// 10 x 21 elements 32.2 and 30.0 us a step; p = 8, 12 x 20 33.6 and 30.6),
// which the tuner finds.  A curved tile stages
// eight metric terms more per slot; where variant 0 then leaves two workgroups
// on a CU, a shape with fewer nodes keeps three (2 M nodes, when chosen: p = 1,
// 8 x 8 159 us a stage, 7 x 7 142; p = 3, 4 x 4 176, 4 x 3 161; p = 7, 2 x 2
// 192, 3 x 1 172; the chosen ones take 149, 168 and 176 now).
// ----------------------------------------------------------------------
constexpr int CURVED_SHAPE = 2;
constexpr int tile_x_for(int dim, int p, int variant) {
  if (dim == 1) return (variant == 0 ? 126 : 254) / (p + 1);   // and two halo nodes per workgroup
  constexpr int v[3][9] = {{0, 8, 5, 4, 3, 3, 5, 2, 3}, {0, 7, 7, 4, 5, 2, 2, 4, 2}, {0, 7, 5, 4, 3, 3, 2, 3, 2}};
  return v[variant][p];
}
constexpr int tile_y_for(int dim, int p, int variant) {
  if (dim == 1) return 1;
  constexpr int v[3][9] = {{0, 8, 5, 4, 3, 2, 1, 2, 1}, {0, 7, 4, 2, 2, 2, 2, 1, 1}, {0, 7, 5, 3, 3, 2, 2, 1, 1}};
  return v[variant][p];
}

// ----------------------------------------------------------------------
// batched work-list kernels: one kernel per degree, its work list holding
// the element tiles of every solve of that degree (same tile shape as the
// plain kernel), one workgroup per item, mapped XCD-aware.  The item's
// arguments are read once at entry, before any store, so that they can live
// in scalar registers; the degree tables go straight from global memory to
// LDS.
// ----------------------------------------------------------------------
template <int EQ, int DIM, int P, int TX, int TY, bool CURV = false>
__global__ __launch_bounds__((Cfg<EQ, DIM, P, TX, TY, CURV>::BS), (Cfg<EQ, DIM, P, TX, TY, CURV>::WPEB)) void batch_stage_kernel(BatchArgs B) {
  __shared__ double lds[Cfg<EQ, DIM, P, TX, TY, CURV>::LDS];
  const int it = xcd_tile(blockIdx.x, gridDim.x);
  if (it >= B.nitems) return;
  const StageArgs* pa = B.args + B.item_solve[it];
  StageArgs A;
  A.S = pa->S;
  A.ph = pa->ph;
  A.a_s = pa->a_s;
  A.b_s = pa->b_s;
  A.use_un = pa->use_un;
  A.limiter = pa->limiter;
  A.diag = pa->diag;
  A.trace = pa->trace;
  A.gmin = pa->gmin;
  A.gmax = pa->gmax;
  // the boundary arrays are indexed at run time: read them where they are
  // (a copy in this local struct would move it to scratch memory)
  stage_tile<EQ, DIM, P, TX, TY, CURV>(lds, A, pa->T, pa->bnd, B.item_tile[it]);
}

template <int EQ, int DIM, int P, int TX, int TY, bool CURV = false>
__global__ __launch_bounds__((Cfg<EQ, DIM, P, TX, TY>::BS)) void batch_maxdt_kernel(BatchDtArgs B) {
  __shared__ double lds[DtCfg<EQ, DIM, P, TX, TY, CURV>::LDS];
  const int it = xcd_tile(blockIdx.x, gridDim.x);
  if (it >= B.nitems) return;
  const MaxDtArgs* pa = B.args + B.item_solve[it];
  MaxDtArgs A;
  A.u = pa->u;
  A.partial = pa->partial;
  A.nn = pa->nn;
  A.nx = pa->nx;
  A.ny = pa->ny;
  A.ntx = pa->ntx;
  A.ntx_mul = pa->ntx_mul;
  A.ntx_shift = pa->ntx_shift;
  A.ihx = pa->ihx;
  A.ihy = pa->ihy;
  A.ph = pa->ph;
  A.metric = pa->metric;
  maxdt_tile<EQ, DIM, P, TX, TY, CURV>(lds, A, pa->T, pa->bnd, B.item_tile[it], B.partial + it);
}

template <int EQ, int DIM, int P, int TX, int TY, bool CURV = false>
void batch_kernels_e(BatchKernels* k) {
  k->stage = reinterpret_cast<const void*>(&batch_stage_kernel<EQ, DIM, P, TX, TY, CURV>);
  k->maxdt = reinterpret_cast<const void*>(&batch_maxdt_kernel<EQ, DIM, P, TX, TY, CURV>);
  k->block = Cfg<EQ, DIM, P, TX, TY, CURV>::BS;
  k->tile_x = TX;
  k->tile_y = DIM == 2 ? TY : 1;
}

template <int EQ, int DIM, int P>
void batch_kernels_t(int variant, BatchKernels* k) {
  if (variant == 1)
    return batch_kernels_e<EQ, DIM, P, tile_x_for(DIM, P, 1), tile_y_for(DIM, P, 1)>(k);
  batch_kernels_e<EQ, DIM, P, tile_x_for(DIM, P, 0), tile_y_for(DIM, P, 0)>(k);
}

// curved meshes: the work-list kernels on their own tile shape
template <int EQ, int DIM, int P>
int batch_kernels_curved_t(BatchKernels* k) {
  if constexpr (DIM == 2 && EQ != EQ_ADVV) {
    batch_kernels_e<EQ, DIM, P, tile_x_for(DIM, P, CURVED_SHAPE), tile_y_for(DIM, P, CURVED_SHAPE), true>(k);
    return 0;
  } else {
    (void)k;
    return -1;
  }
}

// tiles of a mesh of nx x ny elements
inline int num_tiles(int nx, int ny, int tx, int ty) { return ((nx + tx - 1) / tx) * ((ny + ty - 1) / ty); }

template <int EQ, int DIM, int P, int TX, int TY>
hipError_t launch_stage_t(const StageArgs& a, hipStream_t s) {
  using C = Cfg<EQ, DIM, P, TX, TY>;
  const int nb = num_tiles(a.S.nx, a.S.ny, TX, DIM == 2 ? TY : 1);
  hipLaunchKernelGGL((stage_kernel<EQ, DIM, P, TX, TY>), dim3(nb), dim3(C::BS), 0, s, a);
  return hipGetLastError();
}

template <int EQ, int DIM, int P, int TX, int TY>
hipError_t launch_stage_fold_t(const StageArgs& a, const FoldArgs& f, hipStream_t s) {
  using C = Cfg<EQ, DIM, P, TX, TY>;
  const int nb = num_tiles(a.S.nx, a.S.ny, TX, DIM == 2 ? TY : 1);
  hipLaunchKernelGGL((stage_fold_kernel<EQ, DIM, P, TX, TY>), dim3(nb), dim3(C::BS), 0, s, a, f);
  return hipGetLastError();
}

template <int EQ, int DIM, int P>
hipError_t launch_stage_fold_v(int variant, const StageArgs& a, const FoldArgs& f, hipStream_t s) {
  if (variant == 1) return launch_stage_fold_t<EQ, DIM, P, tile_x_for(DIM, P, 1), tile_y_for(DIM, P, 1)>(a, f, s);
  return launch_stage_fold_t<EQ, DIM, P, tile_x_for(DIM, P, 0), tile_y_for(DIM, P, 0)>(a, f, s);
}

template <int EQ, int DIM, int P, int TX, int TY>
hipError_t launch_maxdt_t(const MaxDtArgs& a, hipStream_t s) {
  using C = Cfg<EQ, DIM, P, TX, TY>;
  const int nb = num_tiles(a.nx, a.ny, TX, DIM == 2 ? TY : 1);
  hipLaunchKernelGGL((maxdt_kernel<EQ, DIM, P, TX, TY>), dim3(nb), dim3(C::BS), 0, s, a);
  return hipGetLastError();
}

template <int EQ, int DIM, int P>
hipError_t launch_stage_v(int variant, const StageArgs& a, hipStream_t s) {
  if (variant == 1) return launch_stage_t<EQ, DIM, P, tile_x_for(DIM, P, 1), tile_y_for(DIM, P, 1)>(a, s);
  return launch_stage_t<EQ, DIM, P, tile_x_for(DIM, P, 0), tile_y_for(DIM, P, 0)>(a, s);
}

template <int EQ, int DIM, int P>
hipError_t launch_maxdt_v(int variant, const MaxDtArgs& a, hipStream_t s) {
  if (variant == 1) return launch_maxdt_t<EQ, DIM, P, tile_x_for(DIM, P, 1), tile_y_for(DIM, P, 1)>(a, s);
  return launch_maxdt_t<EQ, DIM, P, tile_x_for(DIM, P, 0), tile_y_for(DIM, P, 0)>(a, s);
}

// Curved meshes: one kernel per degree, on their own tile shape.
template <int EQ, int DIM, int P>
hipError_t launch_stage_curved_t(const StageArgs& a, hipStream_t s) {
  if constexpr (DIM == 2 && EQ != EQ_ADVV) {
    constexpr int TX = tile_x_for(DIM, P, CURVED_SHAPE), TY = tile_y_for(DIM, P, CURVED_SHAPE);
    using C = Cfg<EQ, DIM, P, TX, TY, true>;
    const int nb = num_tiles(a.S.nx, a.S.ny, TX, TY);
    hipLaunchKernelGGL((stage_kernel<EQ, DIM, P, TX, TY, true>), dim3(nb), dim3(C::BS), 0, s, a);
    return hipGetLastError();
  } else {
    (void)a;
    (void)s;
    return hipErrorInvalidValue;
  }
}

template <int EQ, int DIM, int P>
hipError_t launch_maxdt_curved_t(const MaxDtArgs& a, hipStream_t s) {
  if constexpr (DIM == 2 && EQ != EQ_ADVV) {
    constexpr int TX = tile_x_for(DIM, P, CURVED_SHAPE), TY = tile_y_for(DIM, P, CURVED_SHAPE);
    using C = Cfg<EQ, DIM, P, TX, TY>;
    const int nb = num_tiles(a.nx, a.ny, TX, TY);
    hipLaunchKernelGGL((maxdt_kernel<EQ, DIM, P, TX, TY, true>), dim3(nb), dim3(C::BS), 0, s, a);
    return hipGetLastError();
  } else {
    (void)a;
    (void)s;
    return hipErrorInvalidValue;
  }
}

#define IDP_DEFINE_LAUNCHERS(NAME, EQ, DIM)                                              \
  hipError_t launch_stage_##NAME(int p, int variant, const StageArgs& a, hipStream_t s) { \
    switch (p) {                                                                         \
      case 1: return launch_stage_v<EQ, DIM, 1>(variant, a, s);                          \
      case 2: return launch_stage_v<EQ, DIM, 2>(variant, a, s);                          \
      case 3: return launch_stage_v<EQ, DIM, 3>(variant, a, s);                          \
      case 4: return launch_stage_v<EQ, DIM, 4>(variant, a, s);                          \
      case 5: return launch_stage_v<EQ, DIM, 5>(variant, a, s);                          \
      case 6: return launch_stage_v<EQ, DIM, 6>(variant, a, s);                          \
      case 7: return launch_stage_v<EQ, DIM, 7>(variant, a, s);                          \
      case 8: return launch_stage_v<EQ, DIM, 8>(variant, a, s);                          \
    }                                                                                    \
    return hipErrorInvalidValue;                                                         \
  }                                                                                      \
  hipError_t launch_maxdt_##NAME(int p, int variant, const MaxDtArgs& a, hipStream_t s) { \
    switch (p) {                                                                         \
      case 1: return launch_maxdt_v<EQ, DIM, 1>(variant, a, s);                          \
      case 2: return launch_maxdt_v<EQ, DIM, 2>(variant, a, s);                          \
      case 3: return launch_maxdt_v<EQ, DIM, 3>(variant, a, s);                          \
      case 4: return launch_maxdt_v<EQ, DIM, 4>(variant, a, s);                          \
      case 5: return launch_maxdt_v<EQ, DIM, 5>(variant, a, s);                          \
      case 6: return launch_maxdt_v<EQ, DIM, 6>(variant, a, s);                          \
      case 7: return launch_maxdt_v<EQ, DIM, 7>(variant, a, s);                          \
      case 8: return launch_maxdt_v<EQ, DIM, 8>(variant, a, s);                          \
    }                                                                                    \
    return hipErrorInvalidValue;                                                         \
  }                                                                                      \
  hipError_t launch_stage_curved_##NAME(int p, const StageArgs& a, hipStream_t s) {       \
    switch (p) {                                                                         \
      case 1: return launch_stage_curved_t<EQ, DIM, 1>(a, s);                            \
      case 2: return launch_stage_curved_t<EQ, DIM, 2>(a, s);                            \
      case 3: return launch_stage_curved_t<EQ, DIM, 3>(a, s);                            \
      case 4: return launch_stage_curved_t<EQ, DIM, 4>(a, s);                            \
      case 5: return launch_stage_curved_t<EQ, DIM, 5>(a, s);                            \
      case 6: return launch_stage_curved_t<EQ, DIM, 6>(a, s);                            \
      case 7: return launch_stage_curved_t<EQ, DIM, 7>(a, s);                            \
      case 8: return launch_stage_curved_t<EQ, DIM, 8>(a, s);                            \
    }                                                                                    \
    return hipErrorInvalidValue;                                                         \
  }                                                                                      \
  hipError_t launch_maxdt_curved_##NAME(int p, const MaxDtArgs& a, hipStream_t s) {       \
    switch (p) {                                                                         \
      case 1: return launch_maxdt_curved_t<EQ, DIM, 1>(a, s);                            \
      case 2: return launch_maxdt_curved_t<EQ, DIM, 2>(a, s);                            \
      case 3: return launch_maxdt_curved_t<EQ, DIM, 3>(a, s);                            \
      case 4: return launch_maxdt_curved_t<EQ, DIM, 4>(a, s);                            \
      case 5: return launch_maxdt_curved_t<EQ, DIM, 5>(a, s);                            \
      case 6: return launch_maxdt_curved_t<EQ, DIM, 6>(a, s);                            \
      case 7: return launch_maxdt_curved_t<EQ, DIM, 7>(a, s);                            \
      case 8: return launch_maxdt_curved_t<EQ, DIM, 8>(a, s);                            \
    }                                                                                    \
    return hipErrorInvalidValue;                                                         \
  }                                                                                      \
  hipError_t launch_stage_fold_##NAME(int p, int variant, const StageArgs& a,            \
                                      const FoldArgs& f, hipStream_t s) {                \
    switch (p) {                                                                         \
      case 1: return launch_stage_fold_v<EQ, DIM, 1>(variant, a, f, s);                  \
      case 2: return launch_stage_fold_v<EQ, DIM, 2>(variant, a, f, s);                  \
      case 3: return launch_stage_fold_v<EQ, DIM, 3>(variant, a, f, s);                  \
      case 4: return launch_stage_fold_v<EQ, DIM, 4>(variant, a, f, s);                  \
      case 5: return launch_stage_fold_v<EQ, DIM, 5>(variant, a, f, s);                  \
      case 6: return launch_stage_fold_v<EQ, DIM, 6>(variant, a, f, s);                  \
      case 7: return launch_stage_fold_v<EQ, DIM, 7>(variant, a, f, s);                  \
      case 8: return launch_stage_fold_v<EQ, DIM, 8>(variant, a, f, s);                  \
    }                                                                                    \
    return hipErrorInvalidValue;                                                         \
  }                                                                                      \
  hipError_t launch_step1_##NAME(int p, const StepArgs& a, hipStream_t s) {               \
    switch (p) {                                                                         \
      case 1: return launch_step1_t<EQ, DIM, 1>(a, s);                                   \
      case 2: return launch_step1_t<EQ, DIM, 2>(a, s);                                   \
      case 3: return launch_step1_t<EQ, DIM, 3>(a, s);                                   \
      case 4: return launch_step1_t<EQ, DIM, 4>(a, s);                                   \
      case 5: return launch_step1_t<EQ, DIM, 5>(a, s);                                   \
      case 6: return launch_step1_t<EQ, DIM, 6>(a, s);                                   \
      case 7: return launch_step1_t<EQ, DIM, 7>(a, s);                                   \
      case 8: return launch_step1_t<EQ, DIM, 8>(a, s);                                   \
    }                                                                                    \
    return hipErrorInvalidValue;                                                         \
  }                                                                                      \
  void tile_dims_##NAME(int p, int variant, int* tx, int* ty) {                          \
    *tx = tile_x_for(DIM, p, variant);                                                   \
    *ty = tile_y_for(DIM, p, variant);                                                   \
  }                                                                                      \
  int batch_kernels_##NAME(int p, int variant, BatchKernels* k) {                        \
    switch (p) {                                                                         \
      case 1: batch_kernels_t<EQ, DIM, 1>(variant, k); return 0;                         \
      case 2: batch_kernels_t<EQ, DIM, 2>(variant, k); return 0;                         \
      case 3: batch_kernels_t<EQ, DIM, 3>(variant, k); return 0;                         \
      case 4: batch_kernels_t<EQ, DIM, 4>(variant, k); return 0;                         \
      case 5: batch_kernels_t<EQ, DIM, 5>(variant, k); return 0;                         \
      case 6: batch_kernels_t<EQ, DIM, 6>(variant, k); return 0;                         \
      case 7: batch_kernels_t<EQ, DIM, 7>(variant, k); return 0;                         \
      case 8: batch_kernels_t<EQ, DIM, 8>(variant, k); return 0;                         \
    }                                                                                    \
    return -1;                                                                           \
  }                                                                                      \
  int batch_kernels_curved_##NAME(int p, BatchKernels* k) {                             \
    switch (p) {                                                                         \
      case 1: return batch_kernels_curved_t<EQ, DIM, 1>(k);                              \
      case 2: return batch_kernels_curved_t<EQ, DIM, 2>(k);                              \
      case 3: return batch_kernels_curved_t<EQ, DIM, 3>(k);                              \
      case 4: return batch_kernels_curved_t<EQ, DIM, 4>(k);                              \
      case 5: return batch_kernels_curved_t<EQ, DIM, 5>(k);                              \
      case 6: return batch_kernels_curved_t<EQ, DIM, 6>(k);                              \
      case 7: return batch_kernels_curved_t<EQ, DIM, 7>(k);                              \
      case 8: return batch_kernels_curved_t<EQ, DIM, 8>(k);                              \
    }                                                                                    \
    return -1;                                                                           \
  }

}  // namespace idp
