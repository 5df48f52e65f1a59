// K3 for 16 < p <= 64: the p x p part of the Flag Aggregator (normalisation, IRLS by repeated
// weighted PCA, coefficients) in one workgroup of eight or twelve wavefronts, every matrix product on
// the fp64 matrix core.
//
// Same mathematics as the p <= 16 fast path (fa_irls16.hip, namespace fastp; Eq. 5 with the
// regulariser of Sec. 2.3 option (2), Alg. 1's IRLS step and direction): R with R^T R = K~
// from a pivoted Cholesky factorisation, per solve M = R C R^T, the projector P onto the m
// leading eigenvectors of M by trace-correcting purification (X <- X^2 if trace X > m, else
// 2X - X^2, from X_0 = M / trace M), residuals from Z = (I - P) R, and at the end a basis of
// range(P) from a pivoted Cholesky of P.  What differs is the scale: matrices of order
// N = 16 T (T = 2, 3, 4) are kept in LDS as T x T tiles of 16 x 16, each tile in the register
// order of the matrix instruction's accumulator (entry r of lane l = element
// (4 r + l / 16, l % 16)), so that a wavefront moves a tile between LDS and registers with
// two conflict-free 16-byte accesses per lane and can use it directly
//   * as B operand (rows of the tile are the contraction index), and
//   * as A operand of the *transposed* tile (for a symmetric matrix: of tile (J, I)).
// One wavefront owns one output tile of a product; symmetric results are computed for I <= J
// and mirrored.  One further wavefront steers the purification; from the second solve on, most of
// its steps are planned from the previous solve's eigenvalues (see Plan).
//
// The same kernel has a mode for workers that send several gradients (blocks of columns, see
// MODE below); in that mode it is also built for a single tile (p <= 16).
//
// If the purification cannot converge (tied eigenvalues m, m+1) the kernel leaves
// info->status = FA_ST_RETRY and touches nothing else; the caller then runs the any-p Jacobi
// kernel, which starts from the same inputs.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <type_traits>

#include "fa.h"
#include "fa_internal.h"

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

// Wavefronts in the workgroup: one for each tile I <= J of a symmetric result and one that steers
// have to fit, and every further one takes registers from them (sixteen leave 128 a lane, and the
// purification step then spilled; twelve leave 168, eight 256).
constexpr int waves_for(int t) { return t <= 3 ? 8 : 12; }
constexpr int MAX_PURIFY = 200;   // steps of one solve

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  int lo = __double2loint(x), hi = __double2hiint(x);
  lo = __builtin_amdgcn_mov_dpp(lo, CTRL, 0xf, 0xf, false);
  hi = __builtin_amdgcn_mov_dpp(hi, CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ unsigned dpp_u32(unsigned x) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false);
}
// sum over each 16-lane row; every lane of the row gets it
__device__ __forceinline__ double row_sum(double x) {
  x += dpp_f64<0x128>(x);   // row_ror:8
  x += dpp_f64<0x124>(x);   // row_ror:4
  x += dpp_f64<0x122>(x);   // row_ror:2
  x += dpp_f64<0x121>(x);   // row_ror:1
  return x;
}
__device__ __forceinline__ double lane_bcast(double x, int srclane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(x), srclane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(x), srclane);
  return __hiloint2double(hi, lo);
}
// Sum over the four lanes c, 16 + c, 32 + c, 48 + c, in every one of them: (t0 + t1) + (t2 + t3).
// v_permlane16_swap / v_permlane32_swap with both operands the same value return the even rows
// (the lower half) and the odd rows (the upper half) side by side.
__device__ __forceinline__ double rows_sum(double t) {
  int lo = __double2loint(t), hi = __double2hiint(t);
  auto a = __builtin_amdgcn_permlane16_swap((unsigned)lo, (unsigned)lo, false, false);
  auto b = __builtin_amdgcn_permlane16_swap((unsigned)hi, (unsigned)hi, false, false);
  const double s = __hiloint2double((int)b[0], (int)a[0]) + __hiloint2double((int)b[1], (int)a[1]);
  lo = __double2loint(s); hi = __double2hiint(s);
  a = __builtin_amdgcn_permlane32_swap((unsigned)lo, (unsigned)lo, false, false);
  b = __builtin_amdgcn_permlane32_swap((unsigned)hi, (unsigned)hi, false, false);
  return __hiloint2double((int)b[0], (int)a[0]) + __hiloint2double((int)b[1], (int)a[1]);
}
// x, but computed from here on and not ahead of the loop that this stands in
__device__ __forceinline__ int again(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
// deterministic sum over the wavefront, same value in every lane
__device__ __forceinline__ double wave_sum(double x) {
  x = row_sum(x);
  return ((lane_bcast(x, 0) + lane_bcast(x, 16)) + lane_bcast(x, 32)) + lane_bcast(x, 48);
}
// The same on the matrix core, 10 instructions behind x instead of 23: a 4 x 4 x 4 product of four blocks with all
// ones sums over the lanes l, l + 16, l + 32, l + 48, a second one over the other index of a block.
__device__ __forceinline__ double wave_sum_mfma(double x) {
  x = __builtin_amdgcn_mfma_f64_4x4x4f64(x, 1.0, 0.0, 0, 0, 0);
  x = __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, x, 0.0, 0, 0, 0);
  x += dpp_f64<0x128>(x);
  x += dpp_f64<0x124>(x);
  return lane_bcast(x, 0);
}
// 1/sqrt(x): hardware estimate plus two Newton steps
__device__ __forceinline__ double rsq2(double x) {
  double y = __builtin_amdgcn_rsq(x);
  const double hx = 0.5 * x;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const double e = fma(-hx * y, y, 0.5);
    y = fma(y, e, y);
  }
  return y;
}

// ---- tiles ---------------------------------------------------------------------------------
// A matrix is stored as T x T tiles of 16 x 16.  Lane l = 16 q + c of a wavefront holds rows
// 4e + q (e = 0..3), column c of a tile, as the matrix instruction delivers them.  Entries 2h and
// 2h + 1 of a lane are neighbours, in half h of the tile at 2 l doubles and four more for every
// sixteen lanes, so that a tile is two 16-byte accesses per lane, without bank conflicts; and the
// transposed store (lane (q, c), source entry r, goes to entry c / 4 of lane 16 (c % 4) + 4 r + q)
// touches every bank once per half wavefront: q and the parity of c / 4 stay within 32 bytes, c % 4
// moves by 288 bytes and the half by 1152.
constexpr int FA_TILE = FA_TILE_DOUBLES, FA_HALF = FA_TILE / 2;
typedef double v2d __attribute__((ext_vector_type(2)));
__device__ __forceinline__ int at(int l) { return 2 * l + 4 * (l >> 4); }
template <int T>
__device__ __forceinline__ v4d load_tile(const double* base, int I, int J, int lane) {
  const double* t = base + (I * T + J) * FA_TILE + at(lane);
  const v2d a = *reinterpret_cast<const v2d*>(t), b = *reinterpret_cast<const v2d*>(t + FA_HALF);
  return v4d{a[0], a[1], b[0], b[1]};
}
// the first NS entries of each lane only: with all four loaded, the registers of those without a use were given to
// the next load, which then waited for this one
template <int T, int NS>
__device__ __forceinline__ v4d load_tile_first(const double* base, int I, int J, int lane) {
  const double* t = base + (I * T + J) * FA_TILE + at(lane);
  v4d v = {0.0, 0.0, 0.0, 0.0};
  const v2d a = *reinterpret_cast<const v2d*>(t);
  v[0] = a[0]; v[1] = a[1];
  if constexpr (NS == 3) v[2] = t[FA_HALF];
  if constexpr (NS == 4) { const v2d b = *reinterpret_cast<const v2d*>(t + FA_HALF); v[2] = b[0]; v[3] = b[1]; }
  return v;
}
template <int T>
__device__ __forceinline__ void store_tile(double* base, int I, int J, int lane, const v4d& v) {
  double* t = base + (I * T + J) * FA_TILE + at(lane);
  *reinterpret_cast<v2d*>(t) = v2d{v[0], v[1]};
  *reinterpret_cast<v2d*>(t + FA_HALF) = v2d{v[2], v[3]};
}
// the same values written as the transposed tile (J, I): element (4r + q, c) of (I, J) is
// element (c, 4r + q) of (J, I), i.e. entry c / 4 of lane 16 (c % 4) + 4r + q
template <int T>
__device__ __forceinline__ void store_tile_transposed(double* base, int I, int J, int lane,
                                                      const v4d& v) {
  const int c16 = lane & 15, q4 = lane >> 4;
  double* t = base + (J * T + I) * FA_TILE + (c16 >> 3) * FA_HALF + ((c16 >> 2) & 1) +
              at((c16 & 3) * 16 + q4);
#pragma unroll
  for (int r = 0; r < 4; ++r) t[8 * r] = v[r];
}
// the tile as store_tile_transposed would have written it at (J, I), read instead of written
template <int T>
__device__ __forceinline__ v4d load_tile_transposed(const double* base, int I, int J, int lane) {
  const int c16 = lane & 15, q4 = lane >> 4;
  const double* t = base + (I * T + J) * FA_TILE + (c16 >> 3) * FA_HALF + ((c16 >> 2) & 1) +
                    at((c16 & 3) * 16 + q4);
  return v4d{t[0], t[8], t[16], t[24]};
}
// offset of entry e of lane l
__device__ __forceinline__ int entry(int e, int l) { return (e >> 1) * FA_HALF + (e & 1) + at(l); }
// offset of element (i, j) in the tiled storage
template <int T>
__device__ __forceinline__ int eidx(int i, int j) {
  return ((i >> 4) * T + (j >> 4)) * FA_TILE + entry((i & 15) >> 2, (i & 3) * 16 + (j & 15));
}
// offset of element (a, j) of a matrix kept in A-operand order: tile (a/16, j/16), entry
// (j%16)/4 of lane ((j%16)%4) * 16 + a%16   [lane (i, k) supplies element (i, 4s + k)]
template <int T>
__device__ __forceinline__ int aidx(int a, int j) {
  return ((a >> 4) * T + (j >> 4)) * FA_TILE + entry((j & 15) >> 2, (j & 3) * 16 + (a & 15));
}
__device__ __forceinline__ v4d mma4(const v4d& a, const v4d& b, v4d acc) {
#pragma unroll
  for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], acc, 0, 0, 0);
  return acc;
}
// the first NS of those: what the others would add is zero
template <int NS>
__device__ __forceinline__ v4d mma_first(const v4d& a, const v4d& b, v4d acc) {
#pragma unroll
  for (int s = 0; s < NS; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], acc, 0, 0, 0);
  return acc;
}
// the k-th pair (I <= J) of the upper triangle: the T diagonal tiles first (the wavefronts
// that start first hold them, one per SIMD), then the rest row by row
template <int T>
__device__ __forceinline__ void upper_pair(int k, int* I, int* J) {
  if (k < T) { *I = k; *J = k; return; }
  int i = 0, rem = k - T;
  while (rem >= T - 1 - i) { rem -= T - 1 - i; ++i; }
  *I = i; *J = i + 1 + rem;
}

// what a purification step does: X -> al X + be X^2 + ga I, or end the loop
enum { OFF_DIAGONAL, DIAGONAL, LAST_DIAGONAL };   // tiles by what their purification step needs
enum { STEP_GO = 0, STEP_DONE = 1, STEP_FAILED = 2 };
struct __attribute__((aligned(16))) Step {
  double al, be, ga;
  int end, pad;
};
struct Small {
  double s[64], dinv[64], w[2][64], r1[64], beta[64], rinv[64], gd[64], rho[64];
  double red[16], redw[16];
  int piv[64], used[64];
  int cstop, crank;      // of the factorisation: its end; rows
  double cpart[4][64];   // tile columns' parts of c
  // workers that send several gradients: first column and width of the block a column is in,
  // 1 / tr(g^T g) of that block
  int gf[64], gc[64];
  double ginv[64];
  Step step[2];                    // of purification step k at [k & 1]
  float hist[(MAX_PURIFY + 63) / 64 * 64];   // step k of this solve: a of a growth, -1 - b of a shrinking map
                                             // (read 64 at a time, one a lane)
  int guessed;                     // this solve's first steps were planned
};

// ---- planned steps ---------------------------------------------------------------------------
// Without knowing where the gap between eigenvalues m and m + 1 is, a step X^2 or 2X - X^2 widens it
// by a factor of 1.24 on average; knowing it, by up to two, with the same product:
//   growth   1 - (1 - a X)^2,     1 <= a <= 2: a = 1 is 2X - X^2; folds [2/a - 1, 1] onto itself
//   shrink   ((1 + b) X - b)^2,   0 <= b <= 1: b = 0 is X^2;      folds [0, 2b / (1 + b)]
// A fold gives up the order of what it folds, so it must not reach the gap.  From the third solve
// on the last solve's gap is a guess for this one's: a fifth outside either end ([0, H] and [G, 1])
// is folded, the two eigenvalues themselves (expected near h and g) are not.  [G, 1] and [0, H] are
// taken through the maps along with X (rounded outwards).  What started in [G, 1] stays in its
// image, the same for [0, H], and in between every map keeps the order; so if in the end G is near
// 1, H near 0 and trace X = m, the result is the projector onto the m leading eigenvectors whatever
// the guess was worth.  If not, the solve is done once more without.
// Once h and g are within 0.03 of 0 and 1 the steps go on as always.
// Where there is no guess - the first two solves (the first weights move the gap most: guesses failed
// there), a gap of less than a fifth or of more than 32 (where the plain steps need few), a guess that
// failed - only the first growth steps are planned, from a bound that always holds (trace X_0 <= 1: measured, or the
// weights' sum where that is it to 3e-8).
// Measured, steps per call (plain -> with plans): p = 32, m = 16, 15 solves 400 -> 313; p = 64,
// m = 32, 30 solves 764 -> 639; p = 60, m = 31, 5 solves 170 -> 161.  Where a guess from the second solve
// on and ends that stay below a fold cost up to 1.7 times the plain steps (m = 1 or close to p, a = 4: 137
// for 81), it is 85 now; the worst of 8000 problems of that kind drawn at random is 1.35 times.
// All of it is one wavefront's and uniform; the ends are kept in its lanes, so that one image takes all of
// them a step further: lane 0 H, 1 G, 2 h, 3 g, 4 the image of 0, 5 that of 1.
struct Plan {
  float x;                    // this lane's end
  float mul, add;             // H and G are rounded outwards, so that they hold whatever f32 does
  float dn, up;               // 0 in lane 0 / lane 1, beyond every number elsewhere
  float end;                  // the plan ends when h and 1 - g are below this
  double al, be, ga;          // the last step's map: X -> al X + be X^2 + ga I
};
__device__ __forceinline__ float lane_of(float x, int l) {
  return __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(x), l));
}
__device__ __forceinline__ double scalar(double x) { return lane_bcast(x, 0); }
__device__ __forceinline__ void plan_begin(Plan& pl, float H, float G, float h, float g, float end, int lane) {
  pl.x = lane == 0 ? H : lane == 1 ? G : lane == 2 ? h : lane == 3 ? g : lane == 5 ? 1.0f : 0.0f;
  pl.mul = lane == 0 ? 1.0f + 1e-6f : lane == 1 ? 1.0f - 1e-6f : lane < 4 ? 1.0f : 0.0f;
  pl.add = lane == 0 ? 1e-7f : lane == 1 ? -1e-7f : lane == 5 ? 1.0f : 0.0f;
  pl.dn = lane == 0 ? 0.0f : -__builtin_inff();
  pl.up = lane == 1 ? 0.0f : __builtin_inff();
  pl.end = end;
}
// the ends through the growth or shrinking map of parameter c
__device__ __forceinline__ void plan_push(Plan& pl, bool grow, float c) {
  const float u = fmaf(grow ? -c : 1.0f + c, pl.x, grow ? 1.0f : -c);
  float y = grow ? fmaf(-u, u, 1.0f) : u * u;
  y = fminf(fmaxf(y, lane_of(y, 4) + pl.dn), lane_of(y, 5) + pl.up);
  pl.x = fmaf(y, pl.mul, pl.add);
}
// step k's map; false when the plan is at its end
__device__ __forceinline__ bool plan_next(Plan& pl, Small& sm, int k, int lane) {
  const float H = lane_of(pl.x, 0), G = lane_of(pl.x, 1), h = lane_of(pl.x, 2);
  const float up = 1.0f - lane_of(pl.x, 3);
  if (fmaxf(h, up) < pl.end || k >= 40) return false;
  const bool grow = up > h;
  float c = (grow ? 2.0f : H) * __builtin_amdgcn_rcpf(grow ? 1.0f + G : 2.0f - H);
  c = fminf(fmaxf(c, grow ? 1.0f : 0.0f), grow ? 2.0f : 1.0f);
  const double cd = (double)c, b1 = 1.0 + cd;
  pl.al = grow ? 2.0 * cd : -2.0 * cd * b1;
  pl.be = grow ? -cd * cd : b1 * b1;
  pl.ga = grow ? 0.0 : cd * cd;
  if (lane == 0) {
    Step& st = sm.step[k & 1];
    st.al = pl.al; st.be = pl.be; st.ga = pl.ga; st.end = STEP_GO;
    sm.hist[k] = grow ? c : -1.0f - c;
  }
  plan_push(pl, grow, c);
  return true;
}

}  // namespace

// MODE 0: Eq. 5.  MODE 1: terms residual^(1/a) with the constant a of Sec. 2.2 Step 2 other than
// Eq. 5's a = 2 (a kernel of its own: the powers must not take registers from the a = 2 code).
// MODE 2: workers that send several gradients (Sec. 2.1; Sec. 2.2, the extension to
// g_i in R^{n x k}): the p columns are nworkers blocks of sizes[i] consecutive columns; a block's
// value is tr(g^T Y Y^T g) / tr(g^T g), the IRLS re-weights whole blocks, pair terms exist
// between blocks of equal width (Frobenius distance, column l against column l); any exponent.
template <int T, int MODE>
__global__ __launch_bounds__(64 * waves_for(T)) void fa_irls64_kernel(const double* __restrict__ Kg, int p,
                                                             int nworkers,
                                                             const int* __restrict__ sizes,
                                                             int m, int iters, double lambda,
                                                             double tol, double delta,
                                                             double expo,
                                                             double rank_tol, double pair_tol,
                                                             double* __restrict__ cg,
                                                             fa_info* __restrict__ info,
                                                             double* __restrict__ gws,
                                                             double* __restrict__ Ml,
                                                             int spin_budget, fa_resume* rs) {
  constexpr int N = 16 * T, TT = T * T, NTP = T * (T + 1) / 2, MSZ = TT * FA_TILE;
  constexpr int NW = waves_for(T), NTHREADS = 64 * NW;
  // The fourth SIMD (wavefronts 3, 7, 11) gets one tile at T = 4 and none below; the wavefront
  // that steers is on it.  A vector instruction of its would otherwise wait for a matrix
  // instruction of the others each time.
  constexpr int SW = 7;
  // R as B operand: a fifth matrix in LDS where there is room, in global memory (a second-level cache's
  // latency in front of a product) otherwise.
  constexpr bool RB_LDS = T < 4;
  constexpr int BACK = T < 3 ? 1 : T < 4 ? 6 : 10;         // see take_back
  constexpr int EPT = (N * N + NTHREADS - 1) / NTHREADS;   // matrix entries per thread
  extern __shared__ __attribute__((aligned(16))) double lds[];
  double* B0 = lds;
  double* B1 = lds + MSZ;
  double* B2 = lds + 2 * MSZ;
  double* RA = lds + 3 * MSZ;
  constexpr int LP = N + 1;         // row pitch of the factors (N LP <= MSZ)
  Small& sm = *reinterpret_cast<Small*>(lds + (RB_LDS ? 5 : 4) * MSZ);
  double* Rb = gws;                 // R in tile order (B operand)
  if constexpr (RB_LDS) Rb = lds + 4 * MSZ;
  double* D2I = gws + MSZ;          // 1 / D_ij^2 in tile order, 0 for dropped pairs
  double* RtG = gws + 2 * MSZ;      // rows of the Cholesky factor of K~, row-major N x N
  // Ml: last weighted-PCA matrix, row-major N x N, then rank, m (for the eigengap diagnostic)

  const int tid = threadIdx.x, lane = tid & 63;
  // in a scalar register: everything decided per wavefront is a scalar branch
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, q4 = lane >> 4;
  constexpr bool GEN = MODE != 0, GRP = MODE == 2;
  const int P = GRP ? nworkers : p;                       // workers
  const double coef = (lambda > 0.0 && P > 1) ? lambda / (double)(P - 1) : 0.0;
  const int it0 = rs ? rs->it0 : 0;
  const bool scaled = rs && rs->scaled;
  bool isdiag[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) isdiag[r] = (4 * r + q4) == c16;

  // ---- Gram, norms, status -----------------------------------------------------------------
  if (tid < 64) {
    double si = tid < p ? Kg[tid * p + tid] : 0.0;
    if (tid < p && scaled) si *= rs->uinv[tid] * rs->uinv[tid];
    sm.s[tid] = si;
    sm.dinv[tid] = si > 0.0 ? 1.0 / sqrt(si) : 0.0;
    sm.w[0][tid] = si > 0.0 ? 1.0 : 0.0;
    sm.used[tid] = 0;
    sm.rho[tid] = 0.0;
  }
  __syncthreads();
  if constexpr (GRP) {
    if (tid < 64) {
      int first = tid, cnt = 1;
      if (tid < p) {
        int c = 0;
        for (int i = 0; i < nworkers; ++i) {
          const int k = sizes[i];
          if (tid < c + k) { first = c; cnt = k; break; }
          c += k;
        }
      }
      double gs = 0.0;
      for (int l = 0; l < cnt; ++l) gs += sm.s[first + l];
      sm.gf[tid] = first; sm.gc[tid] = cnt;
      sm.ginv[tid] = gs > 0.0 ? 1.0 / gs : 0.0;
      sm.w[0][tid] = gs > 0.0 ? 1.0 : 0.0;
    }
    __syncthreads();
  }
  bool bad = false, live = false, close = false;     // close: a pair nearer than FA_CLOSE_PAIR
#pragma unroll
  for (int q = 0; q < EPT; ++q) {
    const int e = tid + q * NTHREADS;
    if (e < N * N) {
      const int i = e / N, j = e - i * N;
      const bool in = i < p && j < p;
      double kv = in ? Kg[i * p + j] : 0.0;
      if (in && scaled) kv *= rs->uinv[i] * rs->uinv[j];
      if (in) info->K[i * p + j] = kv;
      bad = bad || !(fabs(kv) <= 1.79e308);
      const double si = sm.s[i], sj = sm.s[j];
      live = live || (i == j && si > 0.0);
      B0[eidx<T>(i, j)] = (i == j) ? (si > 0.0 ? 1.0 : 0.0) : kv * sm.dinv[i] * sm.dinv[j];   // K~
      double d2 = si + sj - 2.0 * kv, both = si + sj;
      bool livep = in && i != j && d2 > pair_tol * both;
      if constexpr (GRP) {
        // D^2 between two blocks: column l of one against column l of the other; only blocks
        // of equal width have one, and it sits at the column pairs at the same place in them
        livep = false;
        if (in && i != j) {
          const int fi = sm.gf[i], fj = sm.gf[j], ki = sm.gc[i];
          if (fi != fj && ki == sm.gc[j] && i - fi == j - fj) {
            both = 0.0;
            d2 = 0.0;
            for (int l = 0; l < ki; ++l) {
              const double sa = sm.s[fi + l], sb = sm.s[fj + l];
              d2 += sa + sb - 2.0 * Kg[(fi + l) * p + fj + l];
              both += sa + sb;
            }
            livep = d2 > pair_tol * both;
          }
        }
      }
      D2I[eidx<T>(i, j)] = livep ? 1.0 / d2 : 0.0;
      close = close || (livep && coef > 0.0 && !(d2 > FA_CLOSE_PAIR * both));
    }
  }
  const int nbad = __syncthreads_or(bad ? 1 : 0);
  const int nlive = __syncthreads_or(live ? 1 : 0);
  const int nclose = __syncthreads_or(close ? 1 : 0);
  if (nbad || !nlive) {
    const int st = nbad ? 4 : 5;
    if (tid < p) {
      const double cv = nbad ? nan("") : 0.0;
      cg[tid] = cv;
      info->c[tid] = cv; info->s[tid] = sm.s[tid]; info->v[tid] = 0.0; info->w[tid] = 0.0;
    }
    for (int idx = tid; idx < p * m; idx += NTHREADS) info->A[idx] = 0.0;
    if (tid == 0) {
      info->status = st; info->p = p; info->m = m; info->rank = 0; info->iters_done = 0;
      info->sweeps = 0; info->eigengap = 0.0;
    }
    return;
  }

  // this wavefront's output tile in products with a symmetric result (I <= J); the tiles of a full
  // one go round the wavefronts
  int mt = (wave & 3) < 3 ? wave - (wave >> 2) : -1;       // ... tile number, negative: none
  if (T == 4) mt = wave < 7 ? wave : (wave & 3) < 3 ? wave - 1 : -1;
  if (mt >= NTP) mt = -1;
  int uI = 0, uJ = 0;
  if (mt >= 0) upper_pair<T>(mt, &uI, &uJ);

  // ---- greedy diagonal-pivoted Cholesky of S (tile order; overwritten) -> rows (row-major, pitch LP)
  // Eight pivots at a time by one wavefront, lane j = column j: the pivot is the largest remaining
  // diagonal entry as seen in fp32, ties to the lowest index; its row of S comes from LDS as it was
  // before these eight, what they have taken off since is subtracted from registers, and the diagonal
  // is kept up in the lanes.  Then all wavefronts take the eight rows off S on the matrix core.  Two
  // barriers in eight pivots.  Latency bound, 640 to 740 cycles a pivot; 1400 and 1730 with
  // S in the registers of T wavefronts, a barrier and a rank-one update on the matrix core per pivot.
  auto pivoted_cholesky = [&](double* S, double* rows, double tolv, int max_rank) -> int {
    constexpr int NB = 8;
    const int jl = lane < N ? lane : 0;
    const double* col = S + (jl >> 4) * FA_TILE + 2 * (jl & 15);      // + row_offset: element (row, jl)
    double d = lane < N ? S[eidx<T>(jl, jl)] : 0.0, open = 1.0;       // open: not a pivot yet
    for (int k0 = 0;; k0 += NB) {
      if (wave == 0) {
        int k = k0, last = 0;
        double r[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          if (!last) {
            const float df = d > 0.0 ? (float)d : 0.0f;
            unsigned key = (__float_as_uint(df) & ~63u) | (unsigned)(63 - lane);
            key = max(key, dpp_u32<0x128>(key));
            key = max(key, dpp_u32<0x124>(key));
            key = max(key, dpp_u32<0x122>(key));
            key = max(key, dpp_u32<0x121>(key));
            key = max(key, dpp_u32<0x142, 0xa>(key));
            key = max(key, dpp_u32<0x143, 0xc>(key));
            const int pv = 63 - (__builtin_amdgcn_readlane((int)key, 63) & 63);
            const double dp = lane_bcast(d, pv);
            if (k == max_rank || !(dp > tolv)) {
              last = 1;
            } else {
              double row = col[(pv >> 4) * T * FA_TILE + entry((pv & 15) >> 2, (pv & 3) * 16)];
              const double rsv = rsq2(dp);
#pragma unroll
              for (int c = 0; c < b; ++c) row = fma(-lane_bcast(r[c], pv), r[c], row);
              // (columns that are done with hold rounding noise)
              r[b] = (lane == pv ? dp : row * open) * rsv;
              if (lane < N) rows[k * LP + lane] = r[b];
              if (lane == 0) { sm.piv[k] = pv; sm.rinv[k] = rsv; }
              d = lane == pv ? 0.0 : fma(-r[b], r[b], d);
              open = lane == pv ? 0.0 : open;
              ++k;
            }
          }
        }
        if (lane == 0) { sm.cstop = last || k == max_rank; sm.crank = k; }
      }
      __syncthreads();
      if (__builtin_amdgcn_readfirstlane(sm.cstop)) break;
      if (mt >= 0) {
        v4d acc = load_tile<T>(S, uI, uJ, lane);
#pragma unroll
        for (int s = 0; s < NB / 4; ++s) {
          const double* rk = rows + (k0 + 4 * s + q4) * LP + c16;
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-rk[16 * uI], rk[16 * uJ], acc, 0, 0, 0);
        }
        store_tile<T>(S, uI, uJ, lane, acc);
        if (uI != uJ) store_tile_transposed<T>(S, uI, uJ, lane, acc);
      }
      __syncthreads();
    }
    const int rank = __builtin_amdgcn_readfirstlane(sm.crank);
    for (int e = tid; e < N * LP; e += NTHREADS)
      if (e / LP >= rank) rows[e] = 0.0;
    if (tid < N && tid >= rank) { sm.piv[tid] = 0; sm.rinv[tid] = 0.0; }
    __syncthreads();
    return rank;
  };
  const int rank = pivoted_cholesky(B0, B1, rank_tol, N);
  const int mm = m < rank ? m : rank;

  // ---- R = R~ D^1/2 in both operand orders; R 1; Cholesky rows kept for the epilogue --------
#pragma unroll
  for (int q = 0; q < EPT; ++q) {
    const int e = tid + q * NTHREADS;
    if (e < N * N) {
      const int a = e / N, j = e - a * N;
      const double rt = B1[a * LP + j];
      const double rv = rt * sqrt(sm.s[j]);
      RA[aidx<T>(a, j)] = rv;
      Rb[eidx<T>(a, j)] = rv;
      RtG[e] = rt;
    }
  }
  __syncthreads();
  {
    // R 1: sixteen threads per row
    const int l16 = tid & 15;
    for (int a = tid >> 4; a < N; a += NTHREADS / 16) {
      double acc = 0.0;
      for (int j = l16; j < N; j += 16) {
        const double x = RA[aidx<T>(a, j)];
        acc += GRP ? x / (double)sm.gc[j] : x;          // a block counts with its mean column
      }
      acc = row_sum(acc);
      if (l16 == 0) sm.r1[a] = acc;
    }
  }
  // the Cholesky pivots are needed again in the epilogue
  int piv_keep = tid < 64 ? sm.piv[tid] : 0;
  double rinv_keep = tid < 64 ? sm.rinv[tid] : 0.0;

  // ---- pair part of C (B2, tile order): uniform weights, or what an earlier launch left ------
#pragma unroll
  for (int q = 0; q < EPT; ++q) {
    const int e = tid + q * NTHREADS;
    if (e < N * N) {
      const int i = e / N, j = e - i * N;
      double v = 0.0;
      if (i < p && j < p && i != j)
        v = it0 > 0 ? rs->cp[i * p + j] : -2.0 * coef * D2I[eidx<T>(i, j)];
      B2[eidx<T>(i, j)] = v;
    }
  }
  if (it0 > 0 && tid < p) sm.w[0][tid] = sm.s[tid] > 0.0 ? rs->w[tid] : 0.0;
  double prev_obj = it0 > 0 ? rs->prev_obj : 0.0;
  __syncthreads();
  // whether the sum of the weights is not trace M (see FA_CLOSE_PAIR)
  bool inexact = nclose != 0;
  if (!inexact && rank < __popcll(__ballot(sm.s[lane] > 0.0))) {
    // R^T R (B0) against s and D^2
    if (mt >= 0) {
      v4d g = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
      for (int K = 0; K < T; ++K)
        g = mma4(load_tile<T>(Rb, K, uI, lane), load_tile<T>(Rb, K, uJ, lane), g);
      store_tile<T>(B0, uI, uJ, lane, g);
      if (uI != uJ) store_tile_transposed<T>(B0, uI, uJ, lane, g);
    }
    __syncthreads();
    bool off = false;
    for (int e = tid; e < N * N; e += NTHREADS) {
      const int i = e / N, j = e - i * N;
      const double d2inv = D2I[eidx<T>(i, j)];
      double ratio = 1.0;
      if (i == j && sm.s[i] > 0.0) ratio = B0[eidx<T>(i, i)] * sm.dinv[i] * sm.dinv[i];
      if (i != j && d2inv > 0.0 && coef > 0.0) {
        const int fi = GRP ? sm.gf[i] : i, fj = GRP ? sm.gf[j] : j, k = GRP ? sm.gc[i] : 1;
        ratio = 0.0;
        for (int l = 0; l < k; ++l)
          ratio += (B0[eidx<T>(fi + l, fi + l)] + B0[eidx<T>(fj + l, fj + l)] -
                    2.0 * B0[eidx<T>(fi + l, fj + l)]) * d2inv;
      }
      off = off || !(fabs(ratio - 1.0) <= FA_TRACE_OFF);
    }
    inexact = __syncthreads_or(off ? 1 : 0) != 0;
  }

  const double rs_delta = 1.0 / sqrt(delta);
  int iters_done = 0, steps = 0;
  double* cur = B0;   // where the projector of the last solve is
  double* nxt = B1;
  int failed = 0;
  int wi = 0;         // sm.w[wi]: the weights of this solve
  double hi = 0.0;    // trace M
  // the steering wavefront's: eigenvalues m + 1 (even lanes) and m (odd lanes) of the last solve's
  // matrix, if known
  double est = 0.0;
  bool have_est = false;
  // Of this wavefront's tile: 1 / D^2 (0: no such term); in the Eq. 5 kernel with 1 / |g|^2 on the diagonal.  At T = 4
  // they are loaded for each solve, beside a product: kept, they were spilled and came back one by one.
  v4d d2i = {0.0, 0.0, 0.0, 0.0};
  auto load_d2i = [&](int lane) {
    if (coef > 0.0) d2i = load_tile<T>(D2I, uI, uJ, lane);
    if (!GEN && uI == uJ) {
      const double di = sm.dinv[16 * uI + (lane & 15)];
#pragma unroll
      for (int r = 0; r < 4; ++r) d2i[r] = isdiag[r] ? di * di : d2i[r];
    }
  };
  if (T < 4 && mt >= 0) load_d2i(lane);

  // Between two purifications stand four products and the residuals.  What is not on their path stays off
  // it: the trace of M is the sum of the weights (where it is, see FA_CLOSE_PAIR), C's diagonal is put in on the way to the first
  // product, M goes into X_0 from the accumulators, the steering wavefront plans the first step and takes
  // the gap's ends back beside the products, the residuals' chains overlap.  (With a phase and a barrier for
  // each of these, ten solves at p = 20 took 206 us instead of 165, fifteen at p = 32 263 instead of 207; with what is
  // said below at the residuals, the gap's ends and R, 157 and, 16 workers of two columns, 276 instead of 307.)
  for (int it = 0; it < iters; ++it) {
    // (at T = 4 every address made of it used to be computed ahead of all solves, spilled, and waited for singly)
    const int lane = T > 3 ? again(tid & 63) : tid & 63, c16 = lane & 15, q4 = lane >> 4;
    int k = 0, end = STEP_GO;
    // the steering wavefront's
    Plan pl;
    float Hp = 0.0f, Gp = 1.0f;             // the ends' images at X_k (pl is at X_{k+1})
    bool guessed = false, planned = false, sq = false;
    const double dm = (double)mm;
    // Where the two ends of the gap lie in this solve's matrix, for the next one's folds: bounds of both
    // (even lanes: the lower end) where the eigenvalues are all near 0 or 1, taken back through the maps
    // of the steps bk - 1, ..., 0 before that.
    float yv = 0.5f;
    int bk = -1, cap_in = 0;                // (negative: not known); bit e: end e may lie in what was folded
    float hv = 0.0f;                        // hist[64 hb + lane]
    int hb = -1;
    auto take_back = [&](int down_to) {
      while (bk > down_to) {
        --bk;
        // (every lane's read is inside, whichever step this is)
        static_assert(sizeof(sm.hist) % (64 * sizeof(float)) == 0 && sizeof(sm.hist) / sizeof(float) >= MAX_PURIFY,
                      "a lane would read past the end");
        if (bk >> 6 != hb) { hb = bk >> 6; hv = sm.hist[64 * hb + lane]; }
        const float h = lane_of(hv, bk & 63);
        const bool grow = h > 0.0f;
        const float r = __builtin_amdgcn_sqrtf(fmaxf(grow ? 1.0f - yv : yv, 0.0f));
        yv = (grow ? yv : r - (h + 1.0f)) * __builtin_amdgcn_rcpf(grow ? fmaf(h, r, h) : -h);
      }
    };
    // ---- W = C R^T (B1): A operand = C (symmetric: tile (K, I)), B operand = R^T tile (K, J),
    // which is R's tile (J, K) in A-operand order.  C's diagonal, w / s minus the row sum of the pair
    // part, is put in on the way: a column of the A operand is spread over the four lanes c, c + 16, ...
    for (int f = wave; f < TT; f += NW) {
      const int fI = f / T, fJ = f % T;
      v4d a[T];
      double sum = 0.0;
#pragma unroll
      for (int K = 0; K < T; ++K) {
        a[K] = load_tile<T>(B2, K, fI, lane);
        sum += (a[K][0] + a[K][1]) + (a[K][2] + a[K][3]);
      }
      const int j = 16 * fI + c16;
      const double cd = sm.w[wi][j] * (GRP ? sm.ginv[j] : sm.dinv[j] * sm.dinv[j]) - rows_sum(sum);
      v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int K = 0; K < T; ++K) {
        if (K == fI) {
#pragma unroll
          for (int r = 0; r < 4; ++r) a[K][r] = isdiag[r] ? cd : a[K][r];
        }
        acc = mma4(a[K], load_tile<T>(RA, fJ, K, lane), acc);
      }
      store_tile<T>(B1, fI, fJ, lane, acc);
    }
    __syncthreads();
    // the unplanned map of step j
    bool tracked = false;                   // H and G are taken along
    bool owed = false;                      // ... not yet through the published map
    auto publish = [&](int j) {
      pl.al = sq ? 0.0 : 2.0; pl.be = sq ? 1.0 : -1.0; pl.ga = 0.0;
      if (lane == 0) {
        Step& st = sm.step[j & 1];
        st.al = pl.al; st.be = pl.be; st.ga = 0.0; st.end = end;
        sm.hist[j] = sq ? -1.0f : 1.0f;
      }
      owed = tracked;
    };
    // the ends through it: behind the next measurement's reads, not ahead of the barrier
    auto push = [&]() {
      if (owed) {
        Hp = lane_of(pl.x, 0); Gp = lane_of(pl.x, 1);
        plan_push(pl, !sq, sq ? 0.0f : 1.0f);
        owed = false;
      }
    };
    const bool measure = it == 0 || inexact;
    auto trace_of_M = [&]() {
      __syncthreads();
      hi = 0.0;
#pragma unroll
      for (int q = 0; q < NTP; ++q) hi += sm.red[q];
    };
    // (behind the first two solves the plan needs the trace)
    if (wave == SW && inexact && it > 1) trace_of_M();
    if (wave == SW && mm < rank) {
      // while the others multiply: the first step's map (2000 cycles)
      const double is = scalar(__builtin_amdgcn_rcp(hi) * (1.0 - 1e-7));
      const double lo = lane_bcast(est, 0) * is, up = lane_bcast(est, 1) * is;
      tracked = guessed = it > 1 && have_est && up > 1.2 * lo && up < 32.0 * lo;
      if (lane == 0) sm.guessed = guessed;
      if (guessed) {
        plan_begin(pl, (float)(0.8 * lo), (float)fmin(1.0, 1.25 * up), (float)(1.05 * lo),
                   (float)fmin(0.99, 0.95 * up), 0.03f, lane);
      } else {
        // no guess, but trace X_0 <= 1 bounds x_{m+1} by 1 / (m + 1) (with a margin for rounding):
        // growth may fold what is above that, while it is small
        const float bound = 1.0001f / (float)(mm + 1);
        plan_begin(pl, 0.0f, bound, 0.0f, bound, 0.5f, lane);
      }
      Hp = lane_of(pl.x, 0); Gp = lane_of(pl.x, 1);
      if (spin_budget <= 0) end = STEP_FAILED;
      planned = plan_next(pl, sm, 0, lane) && end == STEP_GO;
      if (!planned) publish(0);
    }
    // ---- M = R W, and X_0 = M / trace M (slightly less: any scale with eigenvalues in [0, 1] will do)
    v4d x = {0.0, 0.0, 0.0, 0.0};           // this wavefront's tile of X_k
    if (mt >= 0) {
#pragma unroll
      for (int K = 0; K < T; ++K)
        x = mma4(load_tile<T>(RA, uI, K, lane), load_tile<T>(B1, K, uJ, lane), x);
      // the matrix itself, row-major, for the eigengap diagnostic (only a last solve's is looked at)
      if (it + 1 == iters || tol > 0.0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = 16 * uI + 4 * r + q4, j = 16 * uJ + c16;
          Ml[i * N + j] = x[r];
          if (uI != uJ) Ml[j * N + i] = x[r];
        }
      }
    }
    if (measure && !(wave == SW && inexact && it > 1)) {
      // (otherwise the residuals' weights give it)
      if (mt >= 0) {
        double td = 0.0;
        if (uI == uJ) {
#pragma unroll
          for (int r = 0; r < 4; ++r) td += isdiag[r] ? x[r] : 0.0;
        }
        td = wave_sum(td);
        if (lane == 0) sm.red[mt] = td;
      }
      trace_of_M();
    }
    cur = B0; nxt = B1;
    if (mm < rank) {
      if (mt >= 0) {
        const double sc = __builtin_amdgcn_rcp(hi) * (1.0 - 1e-7);
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] *= sc;
        store_tile<T>(B0, uI, uJ, lane, x);
        if (uI != uJ) {
          store_tile_transposed<T>(B0, uI, uJ, lane, x);
        } else {
          // Exactly symmetric: a diagonal tile takes its lower triangle twice (the others are mirrored).
          // The steps keep that bit for bit, X^T X being symmetric; an antisymmetric rest would
          // only ever see a map's linear coefficient, up to 4 in a planned step, and no planned step
          // takes it out as a square does: 1e-17 of M was 5e-4 of X after 40 of them.
          wave_fence();
          const double* tp = B0 + (uI * T + uI) * FA_TILE + (c16 >> 3) * FA_HALF + ((c16 >> 2) & 1) +
                             at((c16 & 3) * 16 + q4);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const double below = tp[8 * r];
            if (4 * r + q4 < c16) x[r] = below;
          }
          wave_fence();
          store_tile<T>(B0, uI, uI, lane, x);
        }
      }
      // ---- purification ---------------------------------------------------------------------
      // A wavefront's fp64 vector instructions do not get a turn while older wavefronts of
      // its SIMD have matrix instructions to issue, and every dependent LDS round trip, cross-lane
      // sum or taken branch costs hundreds of cycles, so measuring and deciding stay off the
      // multiplying wavefronts' path, and each of the three roles runs a loop of its own:
      //  - multiplying wavefronts (mt >= 0) make one tile of X_k^2 and of X_{k+1} each;
      //  - during step k wavefront SW decides on step k + 1: the next planned map (see Plan), or from
      //    t = trace X_k and |X_k|_F^2, which give trace X_{k+1}: X^2 where that is above m, 2X - X^2
      //    below; and that X_{k+1} is the result where X_k is a projector already;
      //  - everybody else keeps the barrier, one a step.
      // So a step's map is there before the barrier in front of it and nobody waits for it.  Cycles of a step,
      // planned / steered / behind the measurement, some 70 of each for reading the clock: p = 20 790 / 920 / 910, p = 32
      // 980 / 1080 / 1050 (512 of them matrix instructions), p = 60 3750 / 3810 / 3510 (3072); with the trace of X_k
      // itself, published during step k and waited for behind its products, 1580 at T = 2 and 4500 at T = 4.  At T = 4
      // the fourth SIMD has a third of the others' products; a wavefront there that makes half of the last tile of each
      // of the others handed it over too late (569 us against 482 for a call at p = 60).
      if (mt >= 0) {
        // this wavefront's tile of X_k stays in its registers: LDS holds it for the others
        double live[4];                                  // the identity's place in a diagonal tile
#pragma unroll
        for (int r = 0; r < 4; ++r) live[r] = isdiag[r] && 16 * uJ + c16 < rank ? 1.0 : 0.0;
        // One step: X_k in cu, X_{k+1} into nx.  Written for fixed buffers (the loop alternates
        // two instances) so that every LDS address is loop invariant and the loads of a
        // wavefront that leaves the barrier behind older ones of its SIMD are in flight at
        // once.  Own tile (uI, uJ) of X_k^2 = sum_K X(K, uI)^T X(K, uJ), K = uI first and K = T - 1, where NL of the
        // four matrix instructions suffice (X is zero from index rank on), last.
        // On the diagonal the part K = uI needs nobody else's tile: it is multiplied ahead of the barrier (calls of
        // 8192 rows, us: p = 20 168.2 against 170.5, p = 48 389 against 401, p = 60 480 against 489).  Returns true
        // when the loop is over.
        auto step = [&](auto kind, auto nl, const Step& st, const double* cu, double* nx) __attribute__((always_inline)) -> bool {
          constexpr int KIND = decltype(kind)::value, NL = decltype(nl)::value;
          constexpr bool DIAG = KIND != OFF_DIAGONAL;
          v4d y = {0.0, 0.0, 0.0, 0.0};
          if constexpr (DIAG) {
            y = mma_first<KIND == LAST_DIAGONAL ? NL : 4>(x, x, y);
            __builtin_amdgcn_sched_barrier(0);
          }
          __syncthreads();
          const int e = st.end;
          const double al = st.al, be = st.be, ga = st.ga;
          __builtin_amdgcn_sched_barrier(0);             // ahead of the tiles: products wait for their own operands only
          v4d a[T], b[T];
#pragma unroll
          for (int i = DIAG ? 1 : 0; i < T; ++i) {
            const int K = KIND == LAST_DIAGONAL ? i - 1 : i == T - 1 ? T - 1 : uI + i < T - 1 ? uI + i : uI + i - (T - 1);
            if (T > 2 && i == T - 1 && KIND != LAST_DIAGONAL) {
              a[i] = load_tile_first<T, NL>(cu, K, uI, lane);
              b[i] = DIAG ? a[i] : load_tile_first<T, NL>(cu, K, uJ, lane);
            } else {
              a[i] = load_tile<T>(cu, K, uI, lane);
              b[i] = DIAG ? a[i] : i == 0 ? x : load_tile<T>(cu, K, uJ, lane);
            }
          }
          __builtin_amdgcn_sched_barrier(0);             // all of them ahead of the products
          end = __builtin_amdgcn_readfirstlane(e);
          if (end != STEP_GO) return true;
#pragma unroll
          for (int i = DIAG ? 1 : 0; i < T; ++i)
            y = i == T - 1 && KIND != LAST_DIAGONAL ? mma_first<NL>(a[i], b[i], y) : mma4(a[i], b[i], y);
          if constexpr (T < 3) {
            // one such wavefront a SIMD: nothing of the rest in between the products (calls of 8192 rows, us: p = 20
            // 162.0 against 165.4, p = 32 183.1 against 185.5; where wavefronts share a SIMD it takes turns from the others'
            // products instead, p = 60 482 against 474)
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(2);
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) x[r] = fma(be, y[r], DIAG ? fma(al, x[r], ga * live[r]) : al * x[r]);
          store_tile<T>(nx, uI, uJ, lane, x);
          if constexpr (!DIAG) store_tile_transposed<T>(nx, uI, uJ, lane, x);
          if constexpr (T < 3) __builtin_amdgcn_s_setprio(0);
          ++k;
          return false;
        };
        auto steps_of = [&](auto kind, auto nl) __attribute__((always_inline)) {
          while (!step(kind, nl, sm.step[0], B0, B1) && !step(kind, nl, sm.step[1], B1, B0)) {}
        };
        auto run = [&](auto nl) __attribute__((always_inline)) {
          if (uI != uJ) {
            if constexpr (T > 1) steps_of(std::integral_constant<int, OFF_DIAGONAL>{}, nl);
          } else if (uI != T - 1) {
            if constexpr (T > 1) steps_of(std::integral_constant<int, DIAGONAL>{}, nl);
          } else {
            steps_of(std::integral_constant<int, LAST_DIAGONAL>{}, nl);
          }
        };
        const int nl = (rank + 3) / 4 - 4 * (T - 1);
        if (nl <= 1) run(std::integral_constant<int, 1>{});
        else if (nl == 2) run(std::integral_constant<int, 2>{});
        else if (nl == 3) run(std::integral_constant<int, 3>{});
        else run(std::integral_constant<int, 4>{});
      } else if (wave == SW) {
        // Everything here is uniform, and its chain has to stay under a step's products.  Three stages:
        // planned steps; steps steered by trace X_k and |X_k|_F^2 (which way does not
        // matter to what is right, both maps keep the eigenvalues' order); and from where all
        // eigenvalues are near 0 or 1, with those two measured, as many steps as it takes to
        // square what the sums of the lower ones and of the upper ones' distances from 1 leave away.  In the last of
        // them both are measured again, and have to say the same.
        __builtin_amdgcn_s_setprio(3);      // ahead of the matrix instructions of its SIMD
        __syncthreads();
        if (planned) {
          for (;;) {                        // step k, whose map is a planned one
            const float H = lane_of(pl.x, 0), G = lane_of(pl.x, 1);
            planned = plan_next(pl, sm, k + 1, lane);
            Hp = H; Gp = G;
            if (!planned) break;
            ++k;
            __syncthreads();
          }
          // the first plain one goes by the guess: what is behind it can be measured and bounded
          sq = lane_of(pl.x, 2) > 1.0f - lane_of(pl.x, 3);
          publish(k + 1);
          ++k;
          __syncthreads();
        }
        double t = 0.0, F = 0.0;            // trace X_k, |X_k|_F^2
        auto norm2 = [&](const double* cu) {
          double f0 = 0.0, f1 = 0.0;
          v4d v[NTP];
#pragma unroll
          for (int q = 0; q < NTP; ++q) {
            int I, J;
            upper_pair<T>(q, &I, &J);
            v[q] = load_tile<T>(cu, I, J, lane);
          }
          __builtin_amdgcn_sched_barrier(0);
          push();
#pragma unroll
          for (int q = 0; q < NTP; ++q) {
            double& f = q < T ? f0 : f1;
#pragma unroll
            for (int r = 0; r < 4; ++r) f = fma(v[q][r], v[q][r], f);
          }
          F = wave_sum_mfma(fma(2.0, f1, f0));
        };
        auto trace = [&](const double* cu) {
          const int d = lane < N ? lane : 0;
          t = wave_sum_mfma(lane < N ? cu[eidx<T>(d, d)] : 0.0);
        };
        // the lower eigenvalues' sum and the upper ones' distance from 1, where those are all near 0 or 1 (1.02 s stands
        // for s = sum x (1 - x) without the squares)
        double A = 0.0, B = 0.0;
        auto fits = [&]() -> bool {
          const double s = t - F, sa = 1.02 * fabs(s);
          A = 0.5 * (sa + t - dm);
          B = 0.5 * (sa - t + dm);
          return s >= -1e-9 && s < 0.02 && fabs(t - dm) < 0.25;
        };
        auto advance = [&]() {              // on to X_{k+1}
          ++k;
          if (end == STEP_GO && k >= (guessed ? 64 : MAX_PURIFY - 1)) end = STEP_FAILED;
          publish(k);
        };
        bool near = true;                   // (behind a plan the trace is not known)
        while (end == STEP_GO) {            // step k, whose map is a plain one
          const double* cu = k & 1 ? B1 : B0;
          norm2(cu);
          near = near || t - F < 0.04;
          if (near) {
            trace(cu);
            const double s = t - F;
            near = s < 0.04;
            if (s < 0.02) {
              const bool good = fits();
              if (bk < 0) {
                // bounds of the ends of the gap
                bk = k;
                yv = lane & 1 ? 1.0f - (float)fmin(0.5, fmax(1e-4, B)) : (float)fmin(0.5, fmax(1e-4, A));
                // (both are sums, good to 0.02 s)
                const double zl = 0.5 * (double)(rank - mm) * Hp, zu = 0.5 * dm * (1.0 - Gp);
                cap_in = !guessed ? 0 : (A <= zl + 0.02 * s ? 1 : 0) | (B <= zu + 0.02 * s ? 2 : 0);
              }
              if (good) break;
              // nearly a projector, but with another trace; or eigenvalues outside [0, 1], where neither map keeps an
              // order
              if (s < 1e-10 || (guessed && s < 1e-3)) end = STEP_FAILED;
            }
          }
          t = sq ? F : 2.0 * t - F;         // carried
          sq = t > dm;
          advance();
          __syncthreads();
        }
        if (end == STEP_GO) {
          // where H and G are near 0 and 1 as well, the order is kept from here on
          tracked = tracked && !(Hp < 0.1f && Gp > 0.9f);
          A = fmax(A, 1e-15);
          B = fmax(B, 1e-15);
          for (;;) {
            const double* cu = k & 1 ? B1 : B0;
            const double An = sq ? A * A : 2.0 * A, Bn = sq ? 2.0 * B : B * B;
            if (fmax(An, Bn) < 1e-12) {
              // the last one: X_k as expected, up to rounding
              const double limit = 2.0 * fmax(A, B) + 1e-12;
              norm2(cu);
              trace(cu);
              end = fits() && fmax(A, B) <= limit &&
                            (!tracked || (lane_of(pl.x, 1) > 0.9f && lane_of(pl.x, 0) < 0.1f))
                        ? STEP_DONE : STEP_FAILED;
            }
            A = An;
            B = Bn;
            sq = A > B;
            advance();
            push();
            take_back(bk > BACK ? bk - BACK : 0);        // (there is time beside these steps)
            __syncthreads();
            if (end != STEP_GO) break;
          }
        }
        __builtin_amdgcn_s_setprio(0);
      } else {
        for (;; ++k) {
          __syncthreads();
          end = __builtin_amdgcn_readfirstlane(sm.step[k & 1].end);
          if (end != STEP_GO) break;
        }
      }
      steps += k;
      const bool conv = end == STEP_DONE;
      cur = k & 1 ? B1 : B0;
      nxt = k & 1 ? B0 : B1;
      if (!conv) {
        // a guess that did not hold: the solve once more without
        if (!sm.guessed) { failed = 1; break; }
        __syncthreads();
        have_est = false;
        --it;
        continue;
      }
    } else {
      // m >= rank: Y spans all of span(G)
      for (int f = wave; f < TT; f += NW) {
        const int fI = f / T, fJ = f % T;
        v4d x;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          x[r] = (fI == fJ && isdiag[r] && 16 * fI + c16 < rank) ? 1.0 : 0.0;
        store_tile<T>(cur, fI, fJ, lane, x);
      }
      __syncthreads();
    }
    // ---- -Z = (P - I) R (nxt): A operand = P - I (symmetric), B operand = R (at T = 4 from RA: eight-byte reads of
    // LDS, where sixteen-byte ones of global memory had the products wait, 7400 cycles against 4950) -----------------
    for (int f = wave; f < TT; f += NW) {
      const int fI = f / T, fJ = f % T;
      v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int K = 0; K < T; ++K) {
        v4d q = load_tile<T>(cur, K, fI, lane);
        if (K == fI) {
#pragma unroll
          for (int r = 0; r < 4; ++r) q[r] = isdiag[r] ? q[r] - 1.0 : q[r];
        }
        acc = mma4(q, RB_LDS ? load_tile<T>(Rb, K, fJ, lane) : load_tile_transposed<T>(RA, K, fJ, lane), acc);
      }
      store_tile<T>(nxt, fI, fJ, lane, acc);
    }
    // (beside this product, the next and the residuals: all of it in front of this barrier was waited for)
    if (wave == SW) take_back(bk > 4 ? bk - 4 : 0);
    __syncthreads();
    // ---- Gq = Z^T Z (symmetric; tile (I, J) = sum_K Z(K, I)^T Z(K, J)); its diagonal ----------
    v4d gq = {0.0, 0.0, 0.0, 0.0};
    if (mt >= 0) {
      if constexpr (T > 3) {
        load_d2i(lane);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int K = 0; K < T; ++K)
        gq = mma4(load_tile<T>(nxt, K, uI, lane), load_tile<T>(nxt, K, uJ, lane), gq);
      if (uI == uJ) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (isdiag[r]) sm.gd[16 * uI + c16] = gq[r];
      }
    } else if (wave == SW) {
      take_back(bk > 4 ? bk - 4 : 0);
    }
    __syncthreads();
    if constexpr (GRP) {
      // a block's residual adds entries of Gq that other wavefronts hold: all of it into LDS
      // (over Z, which nobody reads any more)
      if (mt >= 0) {
        store_tile<T>(nxt, uI, uJ, lane, gq);
        if (uI != uJ) store_tile_transposed<T>(nxt, uI, uJ, lane, gq);
      }
      __syncthreads();
    }
    // ---- residuals, objective, next weights (pair part straight into C = B2) -------------------
    double part = 0.0, wsum = 0.0;          // of the objective; of the next M's trace
    if (mt >= 0) {
      v4d cpn;
      const int j = 16 * uJ + c16;
      const double pair = (uI == uJ ? 1.0 : 2.0) * coef;
      double rho[4] = {}, wv[4] = {};
      if constexpr (!GEN) {
        // |(I - P) r_j|^2 / |g_j|^2 = 1 - v_j on the diagonal, |z_i - z_j|^2 / D_ij^2 elsewhere; ordered
        // pairs: an off-diagonal tile stands for its mirror image too.  All four without a branch, so
        // that their chains overlap: what they read ahead of all of it, what they write behind (between them it
        // cost a branch each: a solve's residuals took 2100 cycles at T = 2 and 5200 at T = 4, they take 1300 and 2950).
        const double gj = sm.gd[j];
        double gi[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) gi[r] = sm.gd[16 * uI + 4 * r + q4];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool diag = uI == uJ && isdiag[r];
          const double off = fma(-2.0, gq[r], gi[r] + gj);
          rho[r] = fmax(diag ? gq[r] : off, 0.0) * d2i[r];
          const double rsv = rsq2(rho[r] > 1e-300 ? rho[r] : 1e-300);
          const double f = d2i[r] > 0.0 ? (diag ? 1.0 : pair) : 0.0;
          wv[r] = fmin(rsv, rs_delta);
          part = fma(f, rho[r] * rsv, part);
          wsum = fma(f, wv[r], wsum);
          cpn[r] = diag ? 0.0 : -2.0 * coef * d2i[r] * wv[r];
          wv[r] = d2i[r] > 0.0 ? wv[r] : 0.0;
        }
      } else if constexpr (GRP) {
        // a block's numbers, the same at each of its columns; its term of the objective is counted at its
        // first column (pair terms: at the blocks' first columns).  All four entries together, a wavefront goes on to its
        // widest block (one by one, 16 blocks of two: 7450 cycles a solve, 3700 like this).
        const int kj = sm.gc[j], fj = sm.gf[j];
        const double gvj = sm.ginv[j];
        int fi[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) fi[r] = sm.gf[16 * uI + 4 * r + q4];
        double bot = 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) rho[r] = 0.0;
#pragma unroll 1
        for (int l = 0; __any(l < kj); ++l) {
          const bool in = l < kj;
          const int jl = fj + (in ? l : 0);
          const double gj = sm.gd[jl];
          double gi[4], x[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = fi[r] + (in ? l : 0), il = i < N ? i : N - 1;   // (a narrower block's neighbour: not used)
            gi[r] = sm.gd[il];
            x[r] = nxt[eidx<T>(il, jl)];
          }
          __builtin_amdgcn_sched_barrier(0);
          bot += in ? gj : 0.0;
#pragma unroll
          for (int r = 0; r < 4; ++r) rho[r] += in ? fma(-2.0, x[r], gi[r] + gj) : 0.0;
        }
        double tv[4];
        bool use[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool diag = uI == uJ && isdiag[r];
          use[r] = diag ? gvj > 0.0 : d2i[r] > 0.0;
          const double v = diag ? bot * gvj : fmax(rho[r], 0.0) * d2i[r];
          rho[r] = use[r] ? v : 0.0;
        }
        if (expo == 0.5) {
          // Eq. 5: one reciprocal square root instead of two powers
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const double rsv = rsq2(rho[r] > 1e-300 ? rho[r] : 1e-300);
            tv[r] = rho[r] * rsv;
            wv[r] = rsv < rs_delta ? rsv : rs_delta;
          }
        } else {
          // (rolled: once per solve, and inlined copies of pow() are long)
#pragma unroll 1
          for (int r = 0; r < 4; ++r) {
            const double ro = r == 0 ? rho[0] : r == 1 ? rho[1] : r == 2 ? rho[2] : rho[3];
            const double t = fa_term_pow(ro, expo), w = fa_weight_pow(ro, delta, expo);
            if (r == 0) { tv[0] = t; wv[0] = w; }
            else if (r == 1) { tv[1] = t; wv[1] = w; }
            else if (r == 2) { tv[2] = t; wv[2] = w; }
            else { tv[3] = t; wv[3] = w; }
          }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool diag = uI == uJ && isdiag[r];
          const double f = !use[r] ? 0.0 : diag ? (j == fj ? 1.0 : 0.0) : 16 * uI + 4 * r + q4 == fi[r] ? pair : 0.0;
          part = fma(f, tv[r], part);
          wsum = fma(f, wv[r], wsum);
          cpn[r] = !diag && use[r] ? -2.0 * coef * d2i[r] * wv[r] : 0.0;
          wv[r] = use[r] ? wv[r] : 0.0;
        }
      } else {
        // the general exponent: same places, powers instead of square roots (rolled: once per
        // solve, and inlined copies of pow() are long)
#pragma unroll 1
        for (int r = 0; r < 4; ++r) {
          const int i = 16 * uI + 4 * r + q4;
          const double gqr = r == 0 ? gq[0] : r == 1 ? gq[1] : r == 2 ? gq[2] : gq[3];
          const double di = r == 0 ? d2i[0] : r == 1 ? d2i[1] : r == 2 ? d2i[2] : d2i[3];
          double ro = 0.0, scale = 0.0;        // residual; factor of its term in the objective
          bool diag = i == j, use = false;
          if (diag) {
            ro = gqr * sm.dinv[j] * sm.dinv[j];
            use = sm.s[j] > 0.0;
            scale = 1.0;
          } else if (di > 0.0 && coef > 0.0) {
            double num = sm.gd[i] + sm.gd[j] - 2.0 * gqr;
            num = num > 0.0 ? num : 0.0;
            ro = num * di;
            use = true;
            scale = pair;
          }
          const double t = fa_term_pow(ro, expo), w = fa_weight_pow(ro, delta, expo);
          if (use) { part += scale * t; wsum += scale * w; }
          if (diag) { sm.rho[j] = ro; sm.w[wi ^ 1][j] = use ? w : 0.0; }
          const double cv = (!diag && use) ? -2.0 * coef * di * w : 0.0;
          if (r == 0) cpn[0] = cv; else if (r == 1) cpn[1] = cv; else if (r == 2) cpn[2] = cv; else cpn[3] = cv;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      store_tile<T>(B2, uI, uJ, lane, cpn);
      if (uI != uJ) store_tile_transposed<T>(B2, uI, uJ, lane, cpn);
      if ((!GEN || GRP) && uI == uJ && q4 == (c16 & 3)) {
        // this lane's diagonal entry
        double dr = rho[0], dw = wv[0];
#pragma unroll
        for (int r = 1; r < 4; ++r) { dr = isdiag[r] ? rho[r] : dr; dw = isdiag[r] ? wv[r] : dw; }
        sm.rho[j] = dr;
        sm.w[wi ^ 1][j] = dw;
      }
      part = wave_sum_mfma(part);
      wsum = wave_sum_mfma(wsum);
      if (lane == 0) { sm.red[mt] = part; sm.redw[mt] = wsum; }
    } else if (wave == SW && bk >= 0) {
      take_back(0);
      // an end that was folded could have come from either side of the fold: then further out
      double e = hi * (double)yv;
      if ((cap_in >> (lane & 1)) & 1) e = lane & 1 ? fmin(hi, fmax(e, 2.0 * est)) : fmin(e, 0.5 * est);
      est = e;
      have_est = true;
    }
    __syncthreads();
    double obj = 0.0;
    hi = 0.0;         // the next M's trace, unless it has to be measured
#pragma unroll
    for (int q = 0; q < NTP; ++q) { obj += sm.red[q]; hi += sm.redw[q]; }
    if (tid == 0 && it0 + it < FA_ITERS_MAX) info->objective[it0 + it] = obj;
    iters_done = it + 1;
    const bool stop = it0 + it > 0 && fabs(prev_obj - obj) < tol;
    prev_obj = obj;
    if (stop) break;
    wi ^= 1;
  }
  __syncthreads();
  if (failed) {
    if (tid == 0) info->status = FA_ST_RETRY;
    return;
  }
  // ---- epilogue ----------------------------------------------------------------------------
  // pivoted Cholesky rows U_m of P (cur) -> RA's place
  double* Um = RA;      // R in A order is no longer needed
  // pivots of the first factorisation survive in registers; the second one overwrites sm.piv
  const int nb = pivoted_cholesky(cur, Um, 1e-6, mm);
  if (nb != mm) {
    if (tid == 0) info->status = FA_ST_RETRY;
    return;
  }
  // beta = U_m (R 1)   (U_m rows k, columns a)
  {
    const int l16 = tid & 15;
    for (int k = tid >> 4; k < N; k += NTHREADS / 16) {
      double acc = 0.0;
      for (int a = l16; a < N; a += 16) acc = fma(Um[k * LP + a], sm.r1[a], acc);
      acc = row_sum(acc);
      if (l16 == 0) sm.beta[k] = k < mm ? acc : 0.0;
    }
  }
  // restore the first factorisation's pivots and reciprocal diagonal
  __syncthreads();
  if (tid < 64) { sm.piv[tid] = piv_keep; sm.rinv[tid] = rinv_keep; }
  for (int idx = tid; idx < p * m; idx += NTHREADS) info->A[idx] = 0.0;
  __syncthreads();
  // A = D^-1/2 X, U X = U_m^T, with the upper triangular U[a][l] = R~[a][piv[l]] (rows from global;
  // row a of X belongs to worker piv[a]).  By tiles: the T diagonal tiles of U are inverted, one
  // wavefront each, lane c column c; then wavefront J takes tile column J of X from the bottom up
  // on the matrix core, without a barrier.  (B2 still holds the pair part of C, which the resume
  // state wants.)  T = 4: 19 thousand cycles; substitution by all threads, two barriers a row, 53.
  double* Us = nxt;                 // row-major, pitch LP
  double* Ui = cur;                 // inverses of the diagonal tiles, pitch 17
#pragma unroll
  for (int q = 0; q < EPT; ++q) {
    const int e = tid + q * NTHREADS;
    if (e < N * N) {
      const int a = e / N, l = e - a * N;
      Us[a * LP + l] = (a < rank && l < rank) ? RtG[a * N + sm.piv[l]] : 0.0;
    }
  }
  __syncthreads();
  if (wave < T) {
    const int o = 16 * wave;
    double bcol[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) bcol[i] = (i == c16) ? 1.0 : 0.0;
#pragma unroll
    for (int k = 15; k >= 0; --k) {
      if (o + k < rank) {
        const double xk = bcol[k] * sm.rinv[o + k];
#pragma unroll
        for (int i = 0; i < k; ++i) bcol[i] = fma(-Us[(o + i) * LP + o + k], xk, bcol[i]);
        bcol[k] = xk;
      } else {
        bcol[k] = 0.0;
      }
    }
#pragma unroll
    for (int k = 0; k < 16; ++k)
      if (lane < 16) Ui[wave * FA_TILE + k * 17 + c16] = bcol[k];
  }
  __syncthreads();
  if (wave < T) {
    v4d X[T];
#pragma unroll
    for (int I = T - 1; I >= 0; --I) {
      v4d acc, u;
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[r] = Um[(16 * wave + c16) * LP + 16 * I + 4 * r + q4];
#pragma unroll
      for (int K = I + 1; K < T; ++K) {
#pragma unroll
        for (int r = 0; r < 4; ++r) u[r] = -Us[(16 * I + c16) * LP + 16 * K + 4 * r + q4];
        acc = mma4(u, X[K], acc);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) u[r] = Ui[I * FA_TILE + c16 * 17 + 4 * r + q4];
      X[I] = mma4(u, acc, v4d{0.0, 0.0, 0.0, 0.0});
    }
    // A[piv[a]][k] = dinv[piv[a]] X[a][k];  this tile column's part of c = A beta / p
    const int k = 16 * wave + c16;
#pragma unroll
    for (int I = 0; I < T; ++I)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int a = 16 * I + 4 * r + q4;
        double av = 0.0;
        if (a < rank) {
          const int i = sm.piv[a];
          av = X[I][r] * sm.dinv[i];
          if (i < p && k < mm) info->A[i * m + k] = av;
        }
        const double t = row_sum(k < mm ? av * sm.beta[k] : 0.0);
        if (c16 == 0) sm.cpart[wave][a] = t;
      }
  }
  __syncthreads();
  if (tid < rank) {
    double acc = sm.cpart[0][tid];
#pragma unroll
    for (int J = 1; J < T; ++J) acc += sm.cpart[J][tid];
    sm.gd[sm.piv[tid]] = acc / (double)P;               // c of that column
  }
  if (tid < 64) sm.used[tid] = 0;
  __syncthreads();
  if (tid < rank) sm.used[sm.piv[tid]] = 1;
  __syncthreads();
  if (tid < p) {
    const double cv = sm.used[tid] ? sm.gd[tid] : 0.0;   // workers outside the pivot set: 0
    cg[tid] = cv;
    info->c[tid] = cv;
    info->s[tid] = sm.s[tid];
    info->v[tid] = (GRP ? sm.ginv[tid] > 0.0 : sm.s[tid] > 0.0) ? 1.0 - sm.rho[tid] : 0.0;
    info->w[tid] = sm.w[wi][tid];
  }
  if (rs) {
    // weights for the solve that would come next
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
      const int e = tid + q * NTHREADS;
      if (e < N * N) {
        const int i = e / N, j = e - i * N;
        if (i < p && j < p) rs->cp[i * p + j] = i != j ? B2[eidx<T>(i, j)] : 0.0;
      }
    }
    if (tid < p) rs->w[tid] = sm.w[wi][tid];
    if (tid == 0) { rs->prev_obj = prev_obj; rs->it0 = it0 + iters_done; }
  }
  if (tid == 0) {
    info->status = 0;
    info->p = p; info->m = m; info->rank = rank;
    info->iters_done = it0 + iters_done;
    info->sweeps = steps;
    info->eigengap = nan("");        // filled in on demand by fa_get_info
    Ml[N * N] = (double)rank;
    Ml[N * N + 1] = (double)m;
  }
}

template <int T>
static constexpr size_t lds_bytes() {
  constexpr size_t bytes = (size_t)(T < 4 ? 5 : 4) * T * T * FA_TILE * sizeof(double) + sizeof(Small);
  static_assert(bytes <= 160 * 1024, "more than a compute unit's LDS");
  return bytes;
}

template <int T, int MODE>
static hipError_t launch_tm(const double* Kd, int p, int nworkers, const int* sizes_d, int m,
                            double lambda, int iters, double tol, double delta, double expo,
                            double rank_tol, double pair_tol, double* cd, fa_info* info_d,
                            double* tiles_ws, double* mlast, int spin_budget, fa_resume* rs,
                            hipStream_t st, const fa_ktime* tm) {
  FA_LAUNCH(tm, (fa_irls64_kernel<T, MODE>), dim3(1), dim3(64 * waves_for(T)), lds_bytes<T>(), st, Kd, p,
            nworkers, sizes_d, m, iters, lambda, tol, delta, expo, rank_tol, pair_tol, cd, info_d,
            tiles_ws, mlast, spin_budget, rs);
  return hipGetLastError();
}

template <int T>
static hipError_t launch_t(const double* Kd, int p, int nworkers, const int* sizes_d, int m,
                           double lambda, int iters, double tol, double delta, double expo,
                           double rank_tol, double pair_tol, double* cd, fa_info* info_d,
                           double* tiles_ws, double* mlast, int spin_budget, fa_resume* rs,
                           hipStream_t st, const fa_ktime* tm) {
  if (nworkers > 0)
    return launch_tm<T, 2>(Kd, p, nworkers, sizes_d, m, lambda, iters, tol, delta, expo, rank_tol,
                           pair_tol, cd, info_d, tiles_ws, mlast, spin_budget, rs, st, tm);
  if constexpr (T > 1) {
    if (expo == 0.5)
      return launch_tm<T, 0>(Kd, p, 0, nullptr, m, lambda, iters, tol, delta, expo, rank_tol,
                             pair_tol, cd, info_d, tiles_ws, mlast, spin_budget, rs, st, tm);
    return launch_tm<T, 1>(Kd, p, 0, nullptr, m, lambda, iters, tol, delta, expo, rank_tol,
                           pair_tol, cd, info_d, tiles_ws, mlast, spin_budget, rs, st, tm);
  }
  return hipErrorInvalidValue;      // single columns at p <= 16 have a solver of their own
}

template <int T, int MODE>
static hipError_t prepare_t() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(fa_irls64_kernel<T, MODE>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes<T>());
}

hipError_t fa_irls64_prepare(void) {
  hipError_t e = prepare_t<1, 2>();
#define FA_X(t)                                        \
  if (e == hipSuccess) e = prepare_t<t, 0>();          \
  if (e == hipSuccess) e = prepare_t<t, 1>();          \
  if (e == hipSuccess) e = prepare_t<t, 2>();
  FA_X(2) FA_X(3) FA_X(4)
#undef FA_X
  return e;
}

hipError_t fa_launch_irls64(const double* Kd, int p, int nworkers, const int* sizes_d, int m,
                            double lambda, int iters, double tol, double delta, double exponent_a,
                            double rank_tol, double pair_tol, double* cd, fa_info* info_d,
                            double* tiles_ws, double* mlast, int spin_budget, fa_resume* rs,
                            hipStream_t st, const fa_ktime* tm) {
  const double expo = exponent_a == 2.0 ? 0.5 : 1.0 / exponent_a;
  switch ((p + 15) / 16) {
#define FA_X(t)                                                                                  \
    case t:                                                                                      \
      return launch_t<t>(Kd, p, nworkers, sizes_d, m, lambda, iters, tol, delta, expo, rank_tol, \
                         pair_tol, cd, info_d, tiles_ws, mlast, spin_budget, rs, st, tm);
    FA_X(1) FA_X(2) FA_X(3) FA_X(4)
#undef FA_X
  }
  return hipErrorInvalidValue;
}
