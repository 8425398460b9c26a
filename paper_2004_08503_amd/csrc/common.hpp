// Shared declarations of the gfx950 stage kernels and the host runtime.
#pragma once
#include <hip/hip_runtime.h>

namespace idp {

// Equation codes of the kernels.  Euler comes in three instantiations:
// generic gamma, and gamma = 1 + 2/n with n = 3 (5/3) or n = 5 (7/5), where
// the fractional powers become integer powers of one inverse root.
// EQ_ADVV is advection by a velocity field beta = (beta_x(y), beta_y(x))
// given per node row and column (2-D only).
enum { EQ_ADV = 0, EQ_BURG = 1, EQ_EULER = 2, EQ_EULER53 = 3, EQ_EULER75 = 4, EQ_ADVV = 5 };
constexpr bool is_euler(int eq) { return eq >= EQ_EULER && eq <= EQ_EULER75; }
constexpr int gn_of(int eq) { return eq == EQ_EULER53 ? 3 : eq == EQ_EULER75 ? 5 : 0; }
enum { LIM_SUBCELL = 0, LIM_TARGET = 1, LIM_LOW = 2, LIM_SUBCELL_SI = 3, LIM_ELEMENTWISE = 4 };
constexpr int MAXP = 8;

// Per-degree constants, passed by value in the kernel arguments.
struct Tables {
  double w[MAXP + 1];             // Gauss-Lobatto weights on [0,1]
  double Q[MAXP * (MAXP + 1)];    // 2 sum_{c<=a} D[c][e], a < p; rows of p+1
  double iw[MAXP + 1];            // 1 / w
  double m[MAXP + 1];             // degree-p Legendre coefficient of a line: sum_a m[a] u_a
  double s0;                      // smoothness indicator centre log10(p^-4)
};

// Physics constants of one problem.
struct Phys {
  double vel0, vel1;   // advection velocity / Burgers direction
  const double* vrow;  // EQ_ADVV: beta_x of every node row (ny*(p+1), device)
  const double* vcol;  // EQ_ADVV: beta_y of every node column (nx*(p+1), device)
  double gamma;        // Euler
  double g1;           // (gamma-1)/2
  double igm1;         // 1/(gamma-1)
  double fac;          // (gamma+1)/(2 gamma)
  double f1;           // 1 - fac
  double gsure;        // (gamma-1) (1 - 3e-13), for the admissibility screen
  double ex;           // (gamma-1)/(2 gamma)
  double inv_ex;       // 2 gamma/(gamma-1)
};

// Open boundaries.  Per side (x = 0, x = lx, y = 0, y = ly) the condition
// of every boundary node (node-row order on x-sides, node-column order on
// y-sides, one node per side in 1-D) and the prescribed states [c][node]
// (device arrays, caller-owned).  A face trace on an open side holds the
// exterior state: the prescribed state, the node's own state (outflow), or
// the own state with the normal momentum reversed (slip; outflow for the
// scalar laws).  Other codes, and STATE without a state array, act as
// outflow.
enum { BC_STATE = 1, BC_OUTFLOW = 2, BC_SLIP = 3 };
struct Bnd {
  const signed char* type[4];
  const double* state[4];
  int open;   // bit k set: direction k is open (not periodic)
};

// Diagnostics words in device memory.  Counters are spread over slots
// (indexed by workgroup) so that concurrent workgroups rarely meet on one
// address; the host sums them.
constexpr int DIAG_SLOTS = 1024;
struct Diag {
  unsigned long long limited[DIAG_SLOTS];   // nodes with final alpha < 1
  unsigned long long entropy[DIAG_SLOTS];   // nodes where the entropy search bound alpha
  unsigned int bad_input;                   // rho <= 0 or p <= 0 seen in a stage input
  unsigned int lo_violation;                // u^L outside its bounds (dt above CFL)
};

// Geometry of one solve and where its arrays are.
struct Solve {
  const double* u_n;    // read when use_un
  const double* u_s;    // stage input
  double* u_out;        // stage output
  const double* dt_dev; // when non-null: dt = dt_scale * dt_dev[0]
  double dt, dt_scale;
  long long nn;         // nodes
  int nx, ny;           // elements
  int ntx;              // tiles per row of tiles, and its divider (idp_magic)
  unsigned int ntx_mul;
  int ntx_shift;
  double ihx, ihy;      // 1/h of the elements
  const double* metric; // curved meshes: per node [q][nn] (q < 4 det(J) J^-1, q < 8 the
                        // corrected terms, q = 8 det(J)); NULL on Cartesian meshes
};

struct StageArgs {
  Solve S;
  Phys ph;
  Tables T;
  double a_s, b_s;
  int use_un;
  int limiter;
  Diag* diag;
  double* trace;   // optional per-node [umin, umax, kmin, alpha_z, alpha] x Nn
  double gmin, gmax;   // global bounds (LIM_SUBCELL_SI)
  Bnd bnd;
};

// The minima partial[0..n) that a step's first stage folds into its bound
// (dt = dt_scale times it); the first workgroup writes the bound to pub.
struct FoldArgs {
  const double* partial;
  int n;
  double* pub;
};

// A whole SSP-RK3 step of a 1-D mesh by one workgroup: A is its first stage
// (u -> buf1); cfl > 0: dt = cfl times the bound of u, which goes to dt_pub.
struct StepArgs {
  StageArgs A;
  double* u;
  double* buf1;
  double* buf2;
  double cfl;
  double* dt_pub;
};
// Nodes of the largest such mesh: with the two halo nodes 8 waves for Euler, 12
// for the scalar laws, whose three waves a SIMD leave each the 168 registers
// the loop over the stages takes.  One workgroup has one CU's issue where the
// separate launches have several, which counts with Euler's work per node:
// 508 nodes of p = 3, us a step in separate launches and in one, gamma = 7/5
// 21.0 and 20.1 (with the bound 24.6, 21.7), gamma = 1.3 25.7 and 25.9 (30.0,
// 28.4); with 12 waves, 764 nodes, 23.2 and 24.4, 27.8 and 31.8.  Burgers, 764
// nodes: 11.5 and 7.6 (14.7, 8.5).
constexpr int step1_nodes(int eq) { return is_euler(eq) ? 510 : 766; }

struct MaxDtArgs {
  const double* u;
  double* partial;           // one minimum per workgroup
  long long nn;
  int nx, ny;                // elements
  int ntiles;                // element tiles (read by the host)
  int ntx;                   // tiles per row of tiles, and its divider (idp_magic)
  unsigned int ntx_mul;
  int ntx_shift;
  double ihx, ihy;           // 1/h of the elements
  Phys ph;
  Tables T;
  Bnd bnd;
  const double* metric;      // curved meshes (as Solve::metric), else NULL
};

// Batched execution: per degree, a work list of (solve, tile) items over
// every solve of that degree.
struct BatchArgs {
  const StageArgs* args;     // per solve (this stage's pointers and dt)
  const int* item_solve;
  const int* item_tile;
  int nitems;
};
struct BatchDtArgs {
  const MaxDtArgs* args;     // per solve
  const int* item_solve;
  const int* item_tile;
  double* partial;           // one minimum per item
  int nitems;
};
// The work-list kernels of one degree.
struct BatchKernels {
  const void* stage;         // __global__ void(BatchArgs)
  const void* maxdt;         // __global__ void(BatchDtArgs)
  int block;                 // threads per workgroup
  int tile_x, tile_y;        // elements per tile in x and y
};

// Multiplier and shift that divide by d >= 1: n / d = (n mul) >> shift for
// 0 <= n < 2^31 (mul = floor(2^shift / d) + 1 with shift = 31 + ceil(log2 d),
// so that mul d exceeds 2^shift by at most d <= 2^(shift-31)).
inline void idp_magic(int d, unsigned int* mul, int* shift) {
  int l = 0;
  while ((1LL << l) < d) ++l;
  *shift = 31 + l;
  *mul = (unsigned int)((1ULL << *shift) / (unsigned int)d + 1);
}

// Kernel launchers, one translation unit per (equation, dimension).
// Return hipSuccess or the launch error; variant selects elements-per-block.
#define IDP_DECLARE_LAUNCHERS(NAME)                                               \
  hipError_t launch_stage_##NAME(int p, int variant, const StageArgs& a,          \
                                 hipStream_t s);                                  \
  hipError_t launch_maxdt_##NAME(int p, int variant, const MaxDtArgs& a,          \
                                 hipStream_t s);                                  \
  hipError_t launch_stage_fold_##NAME(int p, int variant, const StageArgs& a,      \
                                      const FoldArgs& f, hipStream_t s);           \
  hipError_t launch_stage_curved_##NAME(int p, const StageArgs& a, hipStream_t s); \
  hipError_t launch_maxdt_curved_##NAME(int p, const MaxDtArgs& a, hipStream_t s); \
  hipError_t launch_step1_##NAME(int p, const StepArgs& a, hipStream_t s);         \
  void tile_dims_##NAME(int p, int variant, int* tx, int* ty);                    \
  int batch_kernels_##NAME(int p, int variant, BatchKernels* k);                  \
  int batch_kernels_curved_##NAME(int p, BatchKernels* k);

IDP_DECLARE_LAUNCHERS(adv1)
IDP_DECLARE_LAUNCHERS(adv2)
IDP_DECLARE_LAUNCHERS(burg1)
IDP_DECLARE_LAUNCHERS(burg2)
IDP_DECLARE_LAUNCHERS(euler1)
IDP_DECLARE_LAUNCHERS(euler2)
IDP_DECLARE_LAUNCHERS(euler53_1)
IDP_DECLARE_LAUNCHERS(euler53_2)
IDP_DECLARE_LAUNCHERS(euler75_1)
IDP_DECLARE_LAUNCHERS(euler75_2)
IDP_DECLARE_LAUNCHERS(advv2)

// min over partial[b..e) by one thread at stride BS: eight independent loads
// in flight per wait (a single chain waits on every load; large meshes have
// hundreds of thousands of partial minima)
template <int BS>
__device__ inline double strided_min(const double* __restrict__ partial, int b, int e) {
  double v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = INFINITY;
  int i = b + (int)threadIdx.x;
  for (; i + 7 * BS < e; i += 8 * BS) {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = fmin(v[j], partial[i + j * BS]);
  }
  for (; i < e; i += BS) v[0] = fmin(v[0], partial[i]);
#pragma unroll
  for (int j = 1; j < 8; ++j) v[0] = fmin(v[0], v[j]);
  return v[0];
}

// The value of the lane that the data-parallel-primitive control CTRL
// selects, moved as two 32-bit halves; lanes of rows outside ROWS (and lanes
// whose source is outside the row) keep x.
template <int CTRL, int ROWS>
__device__ inline double dpp_get(double x) {
  const int lo = __double2loint(x), hi = __double2hiint(x);
  const int lo2 = __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xF, false);
  const int hi2 = __builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xF, false);
  return __hiloint2double(hi2, lo2);
}

// Minimum over the 64 lanes of a wave, valid in lane 63: quad permutations
// [1,0,3,2] and [2,3,0,1], the half-row and row mirrors (every lane then
// holds the minimum of its row of 16), lane 15 of each row broadcast into
// rows 1 and 3, then lane 31 into rows 2 and 3.
__device__ inline double wave_min63(double x) {
  x = fmin(x, dpp_get<0xB1, 0xF>(x));
  x = fmin(x, dpp_get<0x4E, 0xF>(x));
  x = fmin(x, dpp_get<0x141, 0xF>(x));
  x = fmin(x, dpp_get<0x140, 0xF>(x));
  x = fmin(x, dpp_get<0x142, 0xA>(x));
  x = fmin(x, dpp_get<0x143, 0xC>(x));
  return x;
}
// the maximum, the same way
__device__ inline double wave_max63(double x) {
  x = fmax(x, dpp_get<0xB1, 0xF>(x));
  x = fmax(x, dpp_get<0x4E, 0xF>(x));
  x = fmax(x, dpp_get<0x141, 0xF>(x));
  x = fmax(x, dpp_get<0x140, 0xF>(x));
  x = fmax(x, dpp_get<0x142, 0xA>(x));
  x = fmax(x, dpp_get<0x143, 0xC>(x));
  return x;
}

// min over partial[0..n) -> out[0] (one workgroup of 1024 threads)
__global__ void min_reduce_kernel(const double* partial, int n, double* out);
// per solve s: min over partial[range[2s]..range[2s+1]) -> out[s] (one workgroup per solve)
__global__ void segmented_min_kernel(const double* partial, const int* range, double* out);

}  // namespace idp
