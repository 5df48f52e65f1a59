// HIP kernels of the Flag Aggregator hot path for gfx950 (MI355X), and their launchers.
//
//   K1 fa_gram_kernel        norms + Gram matrix K = G^T G, one streaming pass over G
//                            (fp64 matrix core; the bf16 matrix-core pass is fa_gram_lp.hip)
//   K2 fa_gram_reduce_kernel fixed-order reduction of the per-workgroup partial results
//                            (optionally scaled: diag(u) K diag(u), a weighted Gram matrix)
//   K3 fa_irls_kernel        the p x p part for any p <= 64: normalisation, IRLS (weighted
//                            PCA by Jacobi), coefficients c with out = G c
//                            (p <= 16 has its own kernel, fa_irls16.hip)
//   K4 fa_combine_kernel     out = G c, second streaming pass over G
//   K5 fa_proj_kernel        projections G^T (G A) by streaming (re-streaming schedule)
//   K6 fa_restream_weights_kernel  IRLS weights from the streamed projections
//
// Paper: Sec. 2.1 (explained variance needs |g_i|^2 and Y^T g_i), Sec. 2.3 (D_ij^2),
// Eq. 5 (objective), Alg. 1 (IRLS step and d = (1/p) Y Y^T G 1).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <initializer_list>
#include <type_traits>

#include "fa.h"
#include "fa_internal.h"

typedef double v4f64 __attribute__((ext_vector_type(4)));

// tuning of the p <= 16 fp32 Gram kernel: columns per load instruction and waves per CU
// (measured at p = 15, n = 11.2M: CPL 4 x 12 waves 105 us; 2 x 12 111 us; 1 x 8 119 us; wave
// counts that are not a multiple of the four SIMDs lose 10-20 us)
#ifndef FA_GRAM_CPL1
#define FA_GRAM_CPL1 4
#endif
#ifndef FA_GRAM_W1
#define FA_GRAM_W1 12
#endif
// 16 < p <= 32: sixteen waves per CU (measured at p = 32 bf16, n = 124M: 3.00 ms; 8 waves 3.06)
#ifndef FA_GRAM_W2
#define FA_GRAM_W2 16
#endif
#ifndef FA_GRAM_CPL2
#define FA_GRAM_CPL2 4
#endif
#ifndef FA_GRAM_W4
#define FA_GRAM_W4 8
#endif
// 48 < p <= 64 (measured at p = 64, n = 50M: 4 columns per load x 8 waves 4.4 ms; 8 columns per
// load, i.e. tiles of 32 rows, x 12 waves 4.7 ms, x 16 waves 8.5 ms - the accumulators of ten
// tile pairs do not fit 128 registers; the matrix pipe is 77 % busy at the default)
#ifndef FA_GRAM_CPL4
#define FA_GRAM_CPL4 4
#endif

// ------------------------------------------------------------------------------------------
// storage element types: 16 bytes per lane per load
struct ElemF32 {
  static constexpr int SIZE = 4;
  static constexpr int EPL = 4;  // elements per 16-byte lane load
};
struct ElemBF16 {
  static constexpr int SIZE = 2;
  static constexpr int EPL = 8;
};

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

// Streaming access to G and out: every byte is used once per pass, so the loads carry the
// non-temporal hint (measured on MI355X: 15 column streams read at 7.0 TB/s with it, 6.2 TB/s
// without) and the output is written through (one output stream beside the 15 input
// streams: 114 us with write-through stores, 119 us with default ones, n = 11.2M).
__device__ __forceinline__ uint4 load16_stream(const void* src) {
  const uint32_t* s = reinterpret_cast<const uint32_t*>(src);
  uint4 v;   // the four dword loads are merged into one global_load_dwordx4 nt
  v.x = __builtin_nontemporal_load(s);
  v.y = __builtin_nontemporal_load(s + 1);
  v.z = __builtin_nontemporal_load(s + 2);
  v.w = __builtin_nontemporal_load(s + 3);
  return v;
}

typedef uint32_t fa_u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void store16_through(float* dst, fa_u32x4 v) {
  // the trailing s_nop covers the wait states a VALU write of the data registers needs
  // after a store wider than 64 bits (the compiler cannot see inside the asm)
  asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 2" ::"v"(dst), "v"(v) : "memory");
}
__device__ __forceinline__ void store16_through(float* dst, float4 r) {
  store16_through(dst, fa_u32x4{__float_as_uint(r.x), __float_as_uint(r.y), __float_as_uint(r.z),
                                __float_as_uint(r.w)});
}

// 16 bytes of column `base` starting at element row0, zero-filled past row n.
template <typename E>
__device__ __forceinline__ uint4 load16_guarded(const unsigned char* base, int64_t row0,
                                                int64_t n) {
  uint4 v = make_uint4(0u, 0u, 0u, 0u);
  if (row0 + E::EPL <= n) {
    v = load16_stream(base + row0 * E::SIZE);
  } else if (row0 < n) {
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    if constexpr (E::SIZE == 4) {
      const uint32_t* src = reinterpret_cast<const uint32_t*>(base) + row0;
      for (int e = 0; e < 4; ++e)
        if (row0 + e < n) w[e] = src[e];
    } else {
      const uint16_t* src = reinterpret_cast<const uint16_t*>(base) + row0;
      for (int e = 0; e < 8; ++e)
        if (row0 + e < n) w[e >> 1] |= (uint32_t)src[e] << (16 * (e & 1));
    }
    v = make_uint4(w[0], w[1], w[2], w[3]);
  }
  return v;
}

// The 16 bytes at element row0 <= n - 1, zero from element n on, of which some do not exist.  No load depends on a condition,
// so that several of these wait once; element by element under conditions they are a chain of 0.3 to 0.6 us a call.
template <typename E>
__device__ __forceinline__ uint4 load16_end(const unsigned char* base, int64_t row0, int64_t n) {
  const int have = (int)(n - row0 < E::EPL ? n - row0 : E::EPL);
  uint32_t x[E::EPL];
  if constexpr (E::SIZE == 4) {
    const uint32_t* src = reinterpret_cast<const uint32_t*>(base) + row0;
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = src[e < have ? e : have - 1];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = e < have ? x[e] : 0u;
    return make_uint4(x[0], x[1], x[2], x[3]);
  } else {
    const uint16_t* src = reinterpret_cast<const uint16_t*>(base) + row0;
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = src[e < have ? e : have - 1];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = e < have ? x[e] : 0u;
    return make_uint4(x[0] | x[1] << 16, x[2] | x[3] << 16, x[4] | x[5] << 16, x[6] | x[7] << 16);
  }
}

// how G lies in memory and goes to LDS: worker-major; interleaved as it is; interleaved, scattered
enum { FA_MEM_WORKER, FA_MEM_ROWS, FA_MEM_SCATTER };
// and, added to that: at most four, at most eight columns in the last block of sixteen; at most eight in all
enum { FA_NARROW_LAST4 = 4, FA_NARROW_LAST8 = 8, FA_NARROW_ALL8 = 12 };
constexpr int fa_mem(int st) { return st & 3; }
constexpr int fa_narrow(int st) { return st & 12; }

// a pass over some rows of some gradients, whose sums are added to K: which gradients its columns are,
// where they are not simply the first p
struct fa_gram_cols {
  int add, listed;
  uint8_t idx[FA_P_MAX];
};

// ------------------------------------------------------------------------------------------
// K1: Gram matrix by fp64 matrix-core accumulation.
//
// Each wavefront owns a private LDS tile and walks the row tiles w, w + W, w + 2W, ... (w its
// index among the W wavefronts of the launch: a fixed assignment, so results are
// reproducible).  Per tile: 16-byte coalesced global loads (next tile's loads are in flight while this
// tile is multiplied) -> LDS laid out [column][row] (interleaved storage: as the rows are, see ROWS) ->
// each lane reads the four rows of "its" column -> v_mfma_f64_16x16x4_f64, whose A and B operands are the same register for a
// diagonal 16x16 block of G^T G: lane (c, k) supplies G[row_k][c].
// Products of fp32 (or bf16) inputs are exact in fp64 and the accumulation is fp64, which the
// small differences 1 - v_i of the IRLS weights need.
//
// The operands of step t+1 are read from LDS and converted before the matrix instructions
// of step t are issued, so their LDS latency is hidden behind those.
// No masking: over worker-major storage the LDS columns p..16T-1 are zeroed once and never written, over
// interleaved storage they read what lies there, which only reaches entries of K that nobody reads.
//
// Launch shape: one workgroup of WAVES wavefronts (a multiple of the four SIMDs) per compute
// unit, each wavefront with its private LDS tile; the workgroup's LDS request is sized so
// that exactly one fits per CU.  The tile assignment is static (reproducible sums), so an uneven placement
// of workgroups would last for the whole kernel; this shape leaves the dispatcher no choice.
//
// T   = number of 16-column blocks (p <= 16 T)
// CPL = columns covered by one load instruction (1: a wave reads 1 KiB of one column;
//       4: 256 B of each of four columns, which keeps the LDS tile small for large p)
// LAST = only the tiles of the last block of columns with all blocks, itself included (the others'
//       entries of K are there already: see fa_gram_update_rows)
// cols: worker-major storage only, which gradients the p columns are; no other place is read
__device__ __forceinline__ void wave_lds_fence() {
  // orders this wavefront's LDS accesses for the compiler; the hardware executes one
  // wavefront's LDS instructions in order
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// the value of the lane n on within its row of sixteen (CTRL 0x120 + n)
template <int CTRL>
__device__ __forceinline__ double row_ror(double x) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, false),
                          __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, false));
}

template <typename E>
__device__ __forceinline__ void unpack4(const unsigned char* src, double* x) {
  if constexpr (E::SIZE == 4) {
    const float4 f = *reinterpret_cast<const float4*>(src);
    x[0] = (double)f.x; x[1] = (double)f.y; x[2] = (double)f.z; x[3] = (double)f.w;
  } else {
    const uint2 h = *reinterpret_cast<const uint2*>(src);
    x[0] = (double)bf16_bits_to_f32(h.x & 0xffffu); x[1] = (double)bf16_bits_to_f32(h.x >> 16);
    x[2] = (double)bf16_bits_to_f32(h.y & 0xffffu); x[3] = (double)bf16_bits_to_f32(h.y >> 16);
  }
}

// ROWS: G is stored row by row ("interleaved": element i of coordinate k at G + (k*ldg + i)
// * elem_size, ldg <= 16 T).  A tile of R rows is then one contiguous span of memory; it is
// read with the same 16-byte coalesced loads and goes to LDS as it is, and a lane reads the
// elements of "its" column one by one; four rows are a group, and the groups are set apart so
// that the sixteen elements each quarter wavefront reads lie in banks of their own.  The scatter
// of every element to a [column][row] place on the way into LDS, eight 2-byte writes per 16 bytes
// of bf16, bounded the pass: p = 32, bf16, 8M rows 390 -> 244 us, where the matrix core alone needs
// 156; p = 64, bf16, 2M rows 444 -> 177; p = 20, fp32, 3M rows 95 -> 90; fp32, 4M rows at p = 47 262 -> 281
// and at p = 64 443 -> 464, but at 300 thousand 39.6 -> 38.9 and 72 -> 55 (the reads are four where a
// column's rows lie side by side).  What is left is the conversions: a SIMD does not overlap them with
// fp64 products.
// With one tile and many rows the scatter is the quicker one (FA_MEM_SCATTER; the same order of sums, the
// same bits): as they are / scattered, p = 4 bf16 12M rows 138 / 122 us, 4M 56 / 51, 1M 22 / 22, 300 thousand
// 13 / 14; p = 16 fp32 12M 136 / 129, 4M 53 / 52, 1M 22 / 23.
//
// With few columns in the last block most of what is multiplied for it is thrown away.  v_mfma_f64_4x4x4_4b
// multiplies four pairs of blocks of four columns at the rate of the 16 x 16 instruction (18 cycles against 64),
// block b of an operand being columns 4 b .. 4 b + 3: sixteen columns times four, in all four blocks, are one of
// them (FA_NARROW_LAST4), times eight, in two blocks each and in turn, two (FA_NARROW_LAST8; with twelve columns
// nothing is left of the gain); and all pairs of at most eight columns in all are one, of the columns (0, 0, 1, 1) with
// themselves four lanes on (FA_NARROW_ALL8).  The order of an entry's sums, and so its bits, are those of the other
// instruction.  Worker-major columns that the block does not have are not loaded either.
// This pass, us: worker-major fp32 p = 7 n = 10M 85 -> 47, 50M 414 -> 232, p = 18 1M 30 -> 18, p = 23 1M 31 -> 23, p = 36 500
// thousand 34 -> 24, p = 56 900 thousand 83 -> 70; bf16 p = 23 1M 29.6 -> 23.0, p = 50 900 thousand 92 -> 68; interleaved
// p = 7 10M 89 -> 54, bf16 8M 82 -> 52.  With the aggregate's and 12 us between them, interleaved, 3 M rows: fp32 p = 20 173 ->
// 149, 24 167 -> 153, 36 292 -> 251, 40 320 -> 301, 52 512 -> 457, 56 524 -> 472; bf16 152 -> 124, 153 -> 151, 238 -> 190,
// 305 -> 265, 348 -> 292, 364 -> 332.
// LDS bytes of a tile of r interleaved rows, whatever their pitch (at most 16 t elements):
constexpr int fa_rows_tile_bytes(int t, int es, int r) {
  return r / 4 * ((64 * t * es + 255) / 256 * 256 + 16 * es);
}
template <int T, int CPL, typename E, int WAVES, int ST, bool LAST>
__global__ __launch_bounds__(64 * WAVES) void fa_gram_kernel(
                                                     const unsigned char* __restrict__ G,
                                                     int64_t ldg, int p, int64_t n,
                                                     int64_t ntiles,
                                                     double* __restrict__ partials,
                                                     const int* __restrict__ gate,
                                                     fa_gram_cols cols) {
  // as the stand-by of the bf16 matrix-core pass: nothing to do unless that one overflowed
  if (gate != nullptr && *gate == 0) return;
  constexpr bool ROWS = fa_mem(ST) == FA_MEM_ROWS, SCATTER = fa_mem(ST) == FA_MEM_SCATTER;
  constexpr bool ALL8 = fa_narrow(ST) == FA_NARROW_ALL8;
  constexpr int NB = fa_narrow(ST) == FA_NARROW_LAST4 ? 4 : fa_narrow(ST) == FA_NARROW_LAST8 ? 8 : 16;   // columns of the last block
  constexpr int NQ = NB / 4;
  constexpr int EPL = E::EPL;
  constexpr int LPC = 64 / CPL;            // lanes per column in one load instruction
  constexpr int R = LPC * EPL;             // rows per tile
  constexpr int COLS = ROWS || SCATTER ? T * 16 : ALL8 ? 8 : T * 16 - 16 + NB;   // columns that are loaded
  constexpr int NCG = COLS / CPL;          // load instructions per tile
  constexpr int CS = R * E::SIZE + 16;     // LDS bytes per column (+16: bank spread)
  constexpr int NTP = LAST ? T : T * (T + 1) / 2;
  constexpr int NSTEP = R / 16;
  constexpr int TILE = ROWS ? fa_rows_tile_bytes(T, E::SIZE, R) : COLS * CS;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_all[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (a tile's place is a scalar)
  unsigned char* lds = lds_all + wave * TILE;
  const int64_t wid = (int64_t)blockIdx.x * WAVES + wave;   // global wave index
  const int64_t nwaves = (int64_t)gridDim.x * WAVES;

  const int lane = threadIdx.x & 63;
  const int lcol = lane / LPC;
  const int lrow = (lane % LPC) * EPL;
  const int c16 = lane & 15, kq = lane >> 4;

  v4f64 acc[NTP];
#pragma unroll
  for (int i = 0; i < NTP; ++i) acc[i] = v4f64{0.0, 0.0, 0.0, 0.0};

  double accl[T][2];                       // the last block's pairs, where it is narrow
#pragma unroll
  for (int i = 0; i < T; ++i) accl[i][0] = accl[i][1] = 0.0;

  // zero the whole tile once: columns >= p stay zero for the life of the kernel
  // (interleaved storage: the span of a tile overwrites what is read of it)
  for (int off = lane * 16; !ROWS && off < TILE; off += 64 * 16)
    *reinterpret_cast<uint4*>(lds + off) = make_uint4(0u, 0u, 0u, 0u);

  // this lane's source column for each load instruction (clamped: lanes of columns >= p
  // re-read column p-1 and their data is dropped before the LDS write)
  const unsigned char* colbase[NCG];
  bool colon[NCG];
#pragma unroll
  for (int cg = 0; cg < NCG; ++cg) {
    const int col = cg * CPL + lcol;
    colon[cg] = col < p;
    const int src = colon[cg] ? col : p - 1;
    colbase[cg] = G + (int64_t)(cols.listed ? cols.idx[src] : src) * ldg * E::SIZE;
  }

  // interleaved storage: where each of this lane's pieces goes (the span of a tile is R * ldg
  // elements, <= NCG * 64 pieces).  A group of four rows takes gb bytes; where those are whole
  // 16-byte pieces (always, but for bf16 rows of odd length) the next group starts gs >= gb bytes
  // on, gs = 16 elements modulo the 256 bytes of the 64 banks.
  const int ldr = (int)ldg;
  const int gb = 4 * ldr * E::SIZE;
  const int gs = (gb & 15) ? gb : gb + ((16 * E::SIZE - gb) & 255);
  const int tb = R * ldr * E::SIZE;        // bytes of a tile's span
  // An instruction that would reach past the span starts earlier and reads some pieces again, into the same places:
  // a lane that is switched off for a load costs the wavefront a wait for all loads before it.  One that starts past the span,
  // which is so for all lanes, is left out with 49 to 56 columns only (us, all / so: bf16 p = 49, 300 thousand rows 43.6 / 41.5, a
  // million 72.7 / 70.2; fp32 p = 52, a million 71 / 69; but bf16 p = 17, 300 thousand 14.1 / 15.5, p = 24 18 / 25, and with no load
  // to leave out fp32 p = 64, 3 M 239 / 245).
  constexpr bool LEAVE_OUT = T == 4 && NB < 16;
  auto shift = [&](int cg) { return cg * 1024 + 1024 <= tb ? cg * 1024 : tb > 1024 ? tb - 1024 : 0; };
  const int lane16 = lane * 16 < tb ? lane * 16 : tb - 16;
  int pdst[NCG], prow[NCG], pcol[NCG];     // (scattered: row and column of a piece's first element)
#pragma unroll
  for (int cg = 0; cg < NCG; ++cg) {
    const int b = SCATTER ? (cg * 64 + lane) * 16 : shift(cg) + lane16;
    pdst[cg] = ROWS ? b + (b / gb) * (gs - gb) : 0;
    prow[cg] = SCATTER ? (b / E::SIZE) / ldr : 0;
    pcol[cg] = b / E::SIZE - prow[cg] * ldr;
  }

  uint4 regs[NCG];
  auto load_tile = [&](int64_t tl) {
    if constexpr (SCATTER) {
      const unsigned char* base = G + tl * tb;
      const int lim = (int)(n - tl * R < R ? n - tl * R : R) * ldr;   // elements that exist
#pragma unroll
      for (int cg = 0; cg < NCG; ++cg) {
        const int e0 = (cg * 64 + lane) * EPL;
        if (e0 < R * ldr) regs[cg] = load16_guarded<E>(base, e0, lim);
      }
      return;
    }
    if constexpr (ROWS) {
      if ((tl + 1) * R > n) return;        // the ragged last tile: see store_tile_lds
      const unsigned char* base = G + tl * tb;
#pragma unroll
      for (int cg = 0; cg < NCG; ++cg)
        if (!LEAVE_OUT || cg * 1024 < tb) regs[cg] = load16_stream(base + shift(cg) + (uint32_t)lane16);
      return;
    }
    const int64_t row0 = tl * R + lrow;
    if ((tl + 1) * R <= n) {               // uniform: a full tile needs no row guards
#pragma unroll
      for (int cg = 0; cg < NCG; ++cg)
        regs[cg] = load16_stream(colbase[cg] + row0 * E::SIZE);
    } else {
#pragma unroll
      for (int cg = 0; cg < NCG; ++cg) regs[cg] = load16_guarded<E>(colbase[cg], row0, n);
    }
  };
  auto store_tile_lds = [&](int64_t tl) {
    if constexpr (ROWS) {
      if ((tl + 1) * R > n) {
        // the ragged last tile straight from memory, zero past the end (rolled: once per launch)
        const unsigned char* base = G + tl * tb;
        const int lim = (int)(n - tl * R) * ldr;     // elements of this tile that exist
#pragma unroll 1
        for (int b = lane * 16; b < tb; b += 64 * 16)
          *reinterpret_cast<uint4*>(lds + b + (b / gb) * (gs - gb)) =
              load16_guarded<E>(base, b / E::SIZE, lim);
        return;
      }
#pragma unroll
      for (int cg = 0; cg < NCG; ++cg)
        if (!LEAVE_OUT || cg * 1024 < tb) *reinterpret_cast<uint4*>(lds + pdst[cg]) = regs[cg];
      return;
    }
    if constexpr (SCATTER) {
#pragma unroll
      for (int cg = 0; cg < NCG; ++cg) {
        if ((cg * 64 + lane) * EPL >= R * ldr) continue;
        int r = prow[cg], c = pcol[cg];
        const uint32_t w[4] = {regs[cg].x, regs[cg].y, regs[cg].z, regs[cg].w};
#pragma unroll
        for (int j = 0; j < EPL; ++j) {
          if (c < p) {
            if constexpr (E::SIZE == 4)
              *reinterpret_cast<uint32_t*>(lds + c * CS + r * 4) = w[j];
            else
              *reinterpret_cast<uint16_t*>(lds + c * CS + r * 2) =
                  (uint16_t)(w[j >> 1] >> (16 * (j & 1)));
          }
          if (++c == ldr) { c = 0; ++r; }
        }
      }
      return;
    }
#pragma unroll
    for (int cg = 0; cg < NCG; ++cg)
      if (colon[cg])
        *reinterpret_cast<uint4*>(lds + (cg * CPL + lcol) * CS + lrow * E::SIZE) = regs[cg];
  };
  // rows 16 t + 4 kq + j (j = 0..3) of this lane's column of tile column tt.  Interleaved storage:
  // a column >= p reads whatever comes next in the tile's LDS (a row has at most 16 T elements, so
  // that is never past its end); it only reaches entries of its own row and column, which the
  // reduction does not look at.
  // (at most eight columns in all: the first four twice, the others twice)
  const int left16 = ALL8 ? (c16 >> 3) * 4 + (c16 & 3) : c16;
  const unsigned char* src =
      ROWS ? lds + kq * gs + left16 * E::SIZE : lds + left16 * CS + 4 * kq * E::SIZE;
  auto operand = [&](int t, int tt, double* x) {
    if constexpr (ROWS) {
      const unsigned char* at = src + t * (4 * gs) + (tt * 16 + (NB < 16 && tt == T - 1 ? (c16 & (NB - 1)) - c16 : 0)) * E::SIZE;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if constexpr (E::SIZE == 4)
          x[j] = (double)*reinterpret_cast<const float*>(at + j * ldr * 4);
        else
          x[j] = (double)bf16_bits_to_f32(*reinterpret_cast<const uint16_t*>(at + j * ldr * 2));
      }
    } else {
      unpack4<E>(src + (tt * 16 + (NB < 16 && tt == T - 1 ? (c16 & (NB - 1)) - c16 : 0)) * CS + 16 * t * E::SIZE, x);
    }
  };

  wave_lds_fence();
  int64_t tile = wid;
  if (tile < ntiles) load_tile(tile);
  for (; tile < ntiles; tile += nwaves) {
    wave_lds_fence();  // the previous tile's LDS reads precede these writes
    store_tile_lds(tile);
    wave_lds_fence();
    const int64_t next = tile + nwaves;
    if (next < ntiles) load_tile(next);

    double xc[T][4], xn[T][4];
#pragma unroll
    for (int tt = 0; tt < T; ++tt) operand(0, tt, xc[tt]);
#pragma unroll 4
    for (int t = 0; t < NSTEP; ++t) {
      // operands of the next step (the last step re-reads step 0; harmless)
      const int tn = (t + 1 < NSTEP) ? t + 1 : 0;
#pragma unroll
      for (int tt = 0; tt < T; ++tt) operand(tn, tt, xn[tt]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if constexpr (ALL8) {
          accl[0][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(xc[0][j], row_ror<0x124>(xc[0][j]), accl[0][0], 0, 0, 0);
          continue;
        }
        if constexpr (NB < 16) {
          const double y = xc[T - 1][j];
          double z = 0.0;
          if constexpr (NQ == 2) z = row_ror<0x124>(y);
#pragma unroll
          for (int a = 0; a < T; ++a) {
            accl[a][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(xc[a][j], y, accl[a][0], 0, 0, 0);
            if constexpr (NQ == 2)
              accl[a][1] = __builtin_amdgcn_mfma_f64_4x4x4f64(xc[a][j], z, accl[a][1], 0, 0, 0);
          }
        }
        int tp = 0;
#pragma unroll
        for (int a = 0; a < T; ++a)
#pragma unroll
          for (int b = LAST ? T - 1 : a; b < T; ++b) {
            if (NB == 16 || b < T - 1)
              acc[tp] = __builtin_amdgcn_mfma_f64_16x16x4f64(xc[a][j], xc[b][j], acc[tp], 0, 0, 0);
            ++tp;
          }
      }
#pragma unroll
      for (int tt = 0; tt < T; ++tt)
#pragma unroll
        for (int j = 0; j < 4; ++j) xc[tt][j] = xn[tt][j];
    }
  }

  // accumulator register r of lane l is entry (row 4*r + l/16, column l%16) of the block.
  // The workgroup's wavefronts add up in wave order through LDS (the tiles are dead now),
  // one partial Gram per workgroup leaves the kernel.
  __syncthreads();
  double* red = reinterpret_cast<double*>(lds_all);   // WAVES * 256 doubles <= 32 KiB
  double* dst = partials + (int64_t)blockIdx.x * NTP * 256;
#pragma unroll
  for (int tp = 0; tp < NTP; ++tp) {
    // the tile of a block a and the last one; (a, T - 1) is where block a's row of tiles ends
    int narrow = -1;
#pragma unroll
    for (int a = 0, end = -1; a < T; ++a) {
      end += T - a;
      if (NB < 16 && tp == end) narrow = a;
    }
    if constexpr (ALL8) {
      // the same places: block b of the left operand is the columns of left16, the right one's are four lanes on
      const int row = (c16 >> 3) * 4 + kq, from = __builtin_amdgcn_mov_dpp(c16, 0x124, 0xf, 0xf, false);
      red[wave * 256 + (row >> 2) * 64 + (row & 3) * 16 + (from >> 3) * 4 + (from & 3)] = accl[0][0];
    } else if (narrow >= 0) {
      // entry i of lane (i, 4 b + j) belongs to column 4 b + i of the left operand and to the right one's of
      // this lane; the places of columns that the block does not have stay as they are, nobody reads them
#pragma unroll
      for (int q = 0; q < NQ && q < 2; ++q) {
        const int from = q == 0 ? c16 : __builtin_amdgcn_mov_dpp(c16, 0x124, 0xf, 0xf, false);
        const int left = (c16 & ~3) + kq, row = narrow == T - 1 ? left & (NB - 1) : left;
        red[wave * 256 + (row >> 2) * 64 + (row & 3) * 16 + (from & (NB - 1))] = accl[narrow < 0 ? 0 : narrow][q];
      }
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave * 256 + r * 64 + lane] = acc[tp][r];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 256; e += 64 * WAVES) {
      double tot = 0.0;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) tot += red[w * 256 + e];
      dst[tp * 256 + e] = tot;
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------------------------------
// K5: the projections of the gradients on the current basis, measured by streaming G:
//   P = G^T (G A)   (p x m; row i is Y^T g_i for Y = G A, the quantity in the explained
//   variance |Y^T g_i|^2 / |g_i|^2 of Sec. 2.1).
// Same data path as the Gram kernel (coalesced loads -> LDS [column][row] -> matrix core), two
// contractions per 16 rows: first Y_blk = G_blk A (16 rows x m) with the rows of the block as
// the M index of the product, permuted so that the accumulator registers of Y_blk are at once
// the B operand of the second product P += G_blk^T Y_blk (contraction over the 16 rows).
// Y is never written anywhere.  A sits in LDS, zero-padded to 16 T x 16 TM.
template <typename E>
__device__ __forceinline__ double lds_elem(const unsigned char* src) {
  if constexpr (E::SIZE == 4) return (double)*reinterpret_cast<const float*>(src);
  else return (double)bf16_bits_to_f32(*reinterpret_cast<const uint16_t*>(src));
}

template <int T, int TM, int CPL, typename E, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void fa_proj_kernel(
                                                     const unsigned char* __restrict__ G,
                                                     int64_t ldg, int p, int m, int64_t n,
                                                     int64_t ntiles,
                                                     const double* __restrict__ Acoef,
                                                     double* __restrict__ partials) {
  constexpr int EPL = E::EPL;
  constexpr int LPC = 64 / CPL;
  constexpr int R = LPC * EPL;
  constexpr int NCG = T * 16 / CPL;
  constexpr int CS = R * E::SIZE + 16;
  constexpr int NSTEP = R / 16;
  constexpr int NTILE = T * TM;
  constexpr int ALD = TM * 16;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_all[];
  double* Alds = reinterpret_cast<double*>(lds_all);
  unsigned char* tiles = lds_all + (size_t)T * 16 * ALD * sizeof(double);
  const int wave = threadIdx.x >> 6;
  unsigned char* lds = tiles + wave * (T * 16 * CS);
  const int64_t wid = (int64_t)blockIdx.x * WAVES + wave;
  const int64_t nwaves = (int64_t)gridDim.x * WAVES;
  const int lane = threadIdx.x & 63;
  const int lcol = lane / LPC;
  const int lrow = (lane % LPC) * EPL;
  const int c16 = lane & 15, kq = lane >> 4;

  for (int idx = threadIdx.x; idx < T * 16 * ALD; idx += 64 * WAVES) {
    const int i = idx / ALD, a = idx - i * ALD;
    Alds[idx] = (i < p && a < m) ? Acoef[i * m + a] : 0.0;
  }
  for (int off = lane * 16; off < T * 16 * CS; off += 64 * 16)
    *reinterpret_cast<uint4*>(lds + off) = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();

  v4f64 acc[NTILE];
#pragma unroll
  for (int i = 0; i < NTILE; ++i) acc[i] = v4f64{0.0, 0.0, 0.0, 0.0};

  const unsigned char* colbase[NCG];
  bool colon[NCG];
#pragma unroll
  for (int cg = 0; cg < NCG; ++cg) {
    const int col = cg * CPL + lcol;
    colon[cg] = col < p;
    colbase[cg] = G + (int64_t)(colon[cg] ? col : p - 1) * ldg * E::SIZE;
  }
  uint4 regs[NCG];
  auto load_tile = [&](int64_t tl) {
    const int64_t row0 = tl * R + lrow;
    if ((tl + 1) * R <= n) {
#pragma unroll
      for (int cg = 0; cg < NCG; ++cg) regs[cg] = load16_stream(colbase[cg] + row0 * E::SIZE);
    } else {
#pragma unroll
      for (int cg = 0; cg < NCG; ++cg) regs[cg] = load16_guarded<E>(colbase[cg], row0, n);
    }
  };

  // first product: lane (i = c16, k = kq) supplies G[row(i)][4 s + k] with
  // row(i) = 4 (i mod 4) + i / 4, so that register r of lane (kq, a) of the result holds
  // Y[4 kq + r][a]: exactly what the second product wants from that lane for its step j = r
  const int rowA = 4 * (c16 & 3) + (c16 >> 2);
  int64_t tile = wid;
  if (tile < ntiles) load_tile(tile);
  for (; tile < ntiles; tile += nwaves) {
    wave_lds_fence();
#pragma unroll
    for (int cg = 0; cg < NCG; ++cg)
      if (colon[cg])
        *reinterpret_cast<uint4*>(lds + (cg * CPL + lcol) * CS + lrow * E::SIZE) = regs[cg];
    wave_lds_fence();
    const int64_t next = tile + nwaves;
    if (next < ntiles) load_tile(next);

#pragma unroll 2
    for (int t = 0; t < NSTEP; ++t) {
      v4f64 y[TM];
#pragma unroll
      for (int ta = 0; ta < TM; ++ta) y[ta] = v4f64{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int tt = 0; tt < T; ++tt)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int col = 16 * tt + 4 * s + kq;
          const double a1 = lds_elem<E>(lds + col * CS + (16 * t + rowA) * E::SIZE);
#pragma unroll
          for (int ta = 0; ta < TM; ++ta)
            y[ta] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, Alds[col * ALD + 16 * ta + c16],
                                                         y[ta], 0, 0, 0);
        }
      double xc[T][4];
#pragma unroll
      for (int tt = 0; tt < T; ++tt)
        unpack4<E>(lds + (16 * tt + c16) * CS + (16 * t + 4 * kq) * E::SIZE, xc[tt]);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int tt = 0; tt < T; ++tt)
#pragma unroll
          for (int ta = 0; ta < TM; ++ta)
            acc[tt * TM + ta] = __builtin_amdgcn_mfma_f64_16x16x4f64(xc[tt][j], y[ta][j],
                                                                     acc[tt * TM + ta], 0, 0, 0);
    }
  }

  // one partial result per workgroup, summed over its wavefronts in wave order
  __syncthreads();
  double* red = reinterpret_cast<double*>(tiles);
  double* dst = partials + (int64_t)blockIdx.x * NTILE * 256;
#pragma unroll
  for (int tp = 0; tp < NTILE; ++tp) {
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave * 256 + r * 64 + lane] = acc[tp][r];
    __syncthreads();
    for (int e = threadIdx.x; e < 256; e += 64 * WAVES) {
      double tot = 0.0;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) tot += red[w * 256 + e];
      dst[tp * 256 + e] = tot;
    }
    __syncthreads();
  }
}

// The materialised basis Y = G A over interleaved storage (G row by row, row pitch ldr elements): a workgroup copies the
// contiguous span of its 256 rows to LDS as it is, 16 bytes per lane per load and per LDS
// write (no decoding of rows and columns on the way); then thread r adds up row r (fp64) and
// the workgroup writes 256 consecutive outputs of each of up to MB columns of Y (column a, at out + a*ldo, uses the
// coefficients c[i*cstride + a]).  Rows of 16 k elements would put a wavefront's
// reads of element i on a few banks only, so the copy leaves 16 bytes free after every 256:
// byte b of the span sits at b + 16 (b / 256).
#define FA_ROWS_MULTI 8   // columns of a materialised basis per pass over row-major G
__host__ __device__ inline size_t fa_rows_lds_bytes(int ldr, int es) {
  const size_t span = (size_t)256 * ldr * es;
  return span + (span >> 8) * 16 + 16;
}
template <typename E, int MB>
__global__ __launch_bounds__(256) void fa_combine_rows_kernel(const unsigned char* __restrict__ G,
                                                              int ldr, int p, int64_t n,
                                                              const double* __restrict__ c,
                                                              int cstride, int ncols,
                                                              float* __restrict__ out, int64_t ldo) {
  constexpr int EPL = E::EPL;
  constexpr int RB = 256;                  // rows per workgroup pass
  extern __shared__ __attribute__((aligned(16))) unsigned char tile[];
  __shared__ double cs[MB][FA_P_MAX];
  for (int idx = threadIdx.x; idx < MB * FA_P_MAX; idx += 256) {
    const int a = idx / FA_P_MAX, i = idx % FA_P_MAX;
    cs[a][i] = (i < p && a < ncols) ? c[(int64_t)i * cstride + a] : 0.0;
  }
  const int64_t nblk = (n + RB - 1) / RB;
  for (int64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
    const int64_t row_base = blk * RB;
    const int rows_here = (int)(n - row_base < RB ? n - row_base : RB);
    const int lim = rows_here * ldr;                        // elements of this span
    const int npieces = (lim + EPL - 1) / EPL;              // 16-byte pieces, the last one ragged
    const unsigned char* base = G + row_base * ldr * E::SIZE;
    __syncthreads();                                        // the previous pass has been read
    // (fetching the next span into registers before the rows are added up was measured:
    // 126 instead of 134 us at a pitch of 16 fp32 values, 140 instead of 130 at 15)
    constexpr int PCH = 4;                                  // pieces in flight per thread
    for (int pb = (int)threadIdx.x; pb < npieces; pb += 256 * PCH) {
      uint4 v[PCH];
#pragma unroll
      for (int q = 0; q < PCH; ++q) {
        const int pc = pb + q * 256;
        v[q] = make_uint4(0u, 0u, 0u, 0u);
        if ((pc + 1) * EPL <= lim) v[q] = load16_stream(base + (int64_t)pc * 16);
        else if (pc < npieces) v[q] = load16_guarded<E>(base, (int64_t)pc * EPL, lim);
      }
#pragma unroll
      for (int q = 0; q < PCH; ++q) {
        const int pc = pb + q * 256;
        if (pc < npieces) *reinterpret_cast<uint4*>(tile + pc * 16 + (pc >> 4) * 16) = v[q];
      }
    }
    __syncthreads();
    const int r = (int)threadIdx.x;
    if (r < rows_here) {
      const int b0 = r * ldr * E::SIZE;                     // first byte of row r in the span
      auto elem = [&](int i) -> double {
        const int b = b0 + i * E::SIZE;
        const unsigned char* at = tile + b + (b >> 8) * 16;
        if constexpr (E::SIZE == 4) return (double)*reinterpret_cast<const float*>(at);
        else return (double)bf16_bits_to_f32(*reinterpret_cast<const uint16_t*>(at));
      };
      double acc[MB];
#pragma unroll
      for (int a = 0; a < MB; ++a) acc[a] = 0.0;
      for (int i = 0; i < p; ++i) {
        const double t = elem(i);
#pragma unroll
        for (int a = 0; a < MB; ++a) acc[a] = fma(cs[a][i], t, acc[a]);
      }
#pragma unroll
      for (int a = 0; a < MB; ++a)
        if (a < ncols) out[(int64_t)a * ldo + row_base + r] = (float)acc[a];
    }
  }
}

// K4 for interleaved storage, one output: every wavefront has a tile of 64 rows to itself, as it lies in memory, in LDS
// while the next one is on its way to its registers, and a lane adds up one row (even and odd
// elements, in fp64).  NP: 1 KiB loads a tile (ceil(ldr es / 16), rounded up; a load that would reach past the tile starts earlier).
// WHOLE: rows are whole 16-byte pieces, read as such.  The outputs of fa_rows_held tiles, one a lane, stay in registers
// and are written together (see fa_combine_held_kernel), but for the shortest rows, where that costs more than it gives.
// us, one workgroup per span of 256 rows and a barrier either side of its copy to LDS / this: fp32 p = 5, 4M 24.2 / 17.7; p = 16,
// 8M 85.7 / 80.2; p = 20, 3M 52 / 39; p = 28, 4M 77 / 71; p = 40, 3M 98 / 76; p = 64, 3M 161 / 132; bf16 p = 7, 8M 52 / 29; p = 16,
// 8M 64 / 47; p = 32, 8M 98 / 87; p = 64, 3M 75 / 65.
// Tiles held and workgroups a compute unit.  Where the outputs of a set are more than one batch, short batches of many workgroups
// cost more than that kernel did, so it is 64 or 48 tiles and three workgroups for fp32 (32 tiles, four workgroups / so / that
// kernel: p = 12, 50M 461 / 419 / 424; p = 16, 12M 134 / 121 / 128, 50M 628 / 538 / 535, 100M 1308 / 1126 / 1134; p = 18, 50M 700 /
// 599 / 638; p = 20, 3M 42.3 / 39.0 / 52; with p = 12, 80M 763 / 707 / 692 alone above it), six instead of seven for whole rows
// of at most 32 bytes (p = 8, 100M 664 / 614 / 626) and three instead of four for bf16 rows of 49 to 80 bytes once they are more
// than one batch (p = 32, 8M 87 / 89 / 98, 12M 140 / 127 / 144, 60M 782 / 711 / 721; with 64 tiles p = 25, 8M 89.5 instead of 72.2).
// Direct stores: p = 16, 50M 606, bf16 p = 32, 60M 758.
constexpr int fa_rows_held(int es, int np, bool whole) {
  return np < 3 ? 0 : np > 5 ? 64 : es == 2 ? 32 : np == 3 && !whole ? 48 : 64;
}
// workgroups a compute unit
constexpr int fa_rows_wgs(int es, int np, bool whole) {
  if (np < 3) return np < 2 ? 12 : whole ? 6 : 7;
  return np < 6 ? (es == 2 ? 4 : 3) : np < 9 && es == 2 ? 3 : 2;
}
template <int N, int ID = 0>
struct fa_held_rows {
  static constexpr int HALF = N / 2;
  fa_held_rows<HALF, ID> lower;
  fa_held_rows<N - HALF, ID + HALF> upper;
  __device__ __forceinline__ void put(int i, float x) {
    if (i < HALF) lower.put(i, x);
    else upper.put(i - HALF, x);
  }
  __device__ __forceinline__ void write(int count, float* dst, int64_t step) const {
    lower.write(count, dst, step);
    if (count > HALF) upper.write(count - HALF, dst + HALF * step, step);
  }
};
template <int ID>
struct fa_held_rows<1, ID> {
  float a;
  __device__ __forceinline__ void put(int, float x) {
    a = x;
    asm volatile("" ::"n"(ID));        // a branch of its own (as in fa_held_tiles)
  }
  __device__ __forceinline__ void write(int count, float* dst, int64_t) const {
    if (count > 0) __builtin_nontemporal_store(a, dst);
  }
};
template <int ID>
struct fa_held_rows<0, ID> {};
// Wavefronts a SIMD that the registers have to allow: those of the workgroups that are there, and no more with ten loads a tile,
// where the compiler reads a row's elements one by one to get down to the registers of one more (p = 33 fp32, 1M 24.9 us, 23.2
// like this; with twelve loads the same costs 3 to 5 % from four million rows on).
constexpr int fa_rows_waves(int es, int np, bool whole) { return fa_rows_held(es, np, whole) ? fa_rows_wgs(es, np, whole) : 1; }
template <typename E, int NP, bool WHOLE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(fa_rows_waves(E::SIZE, NP, WHOLE),
                                                                     NP == 10 ? fa_rows_waves(E::SIZE, NP, WHOLE) : 8))) void
fa_combine_rows_tiles_kernel(const unsigned char* __restrict__ G, int ldr, int p, int64_t n, const double* __restrict__ c,
                             int cstride, float* __restrict__ out) {
  constexpr int EPL = E::EPL;
  extern __shared__ __attribute__((aligned(16))) unsigned char tile[];
  __shared__ __attribute__((aligned(16))) double cs[FA_P_MAX];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (threadIdx.x < FA_P_MAX) cs[threadIdx.x] = (int)threadIdx.x < p ? c[(int64_t)threadIdx.x * cstride] : 0.0;
  __syncthreads();
  const int tb = 64 * ldr * E::SIZE;
  // byte b of a tile sits at b + 16 (b / 256), so that rows of 16 k elements do not lie on a few banks only; but rows of 40, 60
  // or 120 bytes as they are, of which that would put every sixth, fourth or second one on the same bank (us, with the
  // places: bf16 p = 20, 4M 35.2 -> 28.9, p = 30, 16M 258 -> 173, p = 60, 16M 772 -> 338; fp32 p = 15, 12M 120 -> 115, p = 30, 12M 318 ->
  // 225; other widths lose up to 10 % without them)
  const int row = ldr * E::SIZE;
  const int sh = !WHOLE && row >= 40 && 240 % row == 0 ? 31 : 8;
  unsigned char* const mine = tile + wave * (NP * 1088);
  const int lane16 = lane * 16 < tb ? lane * 16 : tb - 16;
  auto shift = [&](int k) { return k * 1024 + 1024 <= tb ? k * 1024 : tb > 1024 ? tb - 1024 : 0; };
  int dst[NP];
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const int b = shift(k) + lane16;
    dst[k] = b + (b >> sh) * 16;
  }
  const int64_t ntiles = n / 64, nwaves = (int64_t)gridDim.x * 4;   // whole tiles
  int64_t t = (int64_t)blockIdx.x * 4 + wave;
  uint4 regs[NP];
  auto load_tile = [&](int64_t tl) {
    const unsigned char* base = G + tl * tb;
#pragma unroll
    for (int k = 0; k < NP; ++k) regs[k] = load16_stream(base + shift(k) + (uint32_t)lane16);
  };
  const int r0 = lane * row;                               // first byte of this lane's row
  auto row_sum = [&]() -> float {
    double a0 = 0.0, a1 = 0.0;
    if constexpr (WHOLE) {
      // (elements past p are multiplied by 0 only where the row has them: left out)
#pragma unroll 2
      for (int i = 0; i < p; i += EPL) {
        const int b = r0 + i * E::SIZE;
        const uint4 v = *reinterpret_cast<const uint4*>(mine + b + (b >> 8) * 16);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < EPL; e += 2) {
          double x0, x1;
          if constexpr (E::SIZE == 4) {
            x0 = (double)__uint_as_float(w[e]);
            x1 = (double)__uint_as_float(w[e + 1]);
          } else {
            x0 = (double)__uint_as_float(w[e >> 1] << 16);
            x1 = (double)__uint_as_float(w[e >> 1] & 0xffff0000u);
          }
          if (i + e < p) a0 = fma(cs[i + e], x0, a0);
          if (i + e + 1 < p) a1 = fma(cs[i + e + 1], x1, a1);
        }
      }
    } else {
      auto elem = [&](int i) -> double {
        const int b = r0 + i * E::SIZE;
        const unsigned char* at = mine + b + (b >> sh) * 16;
        if constexpr (E::SIZE == 4) return (double)*reinterpret_cast<const float*>(at);
        else return (double)bf16_bits_to_f32(*reinterpret_cast<const uint16_t*>(at));
      };
      int i = 0;
#pragma unroll 4
      for (; i + 1 < p; i += 2) {
        a0 = fma(cs[i], elem(i), a0);
        a1 = fma(cs[i + 1], elem(i + 1), a1);
      }
      if (i < p) a0 = fma(cs[i], elem(i), a0);
    }
    return (float)(a0 + a1);
  };
  constexpr int HELD = fa_rows_held(E::SIZE, NP, WHOLE);
  fa_held_rows<HELD> held;
  int nheld = 0;
  float* dst_out = out + t * 64 + lane;                    // first tile of those held
  if (t < ntiles) load_tile(t);
  for (; t < ntiles; t += nwaves) {
    wave_lds_fence();                                      // the previous tile has been read
#pragma unroll
    for (int k = 0; k < NP; ++k) *reinterpret_cast<uint4*>(mine + dst[k]) = regs[k];
    wave_lds_fence();
    const int64_t next = t + nwaves;
    if (next < ntiles) load_tile(next);
    const float r = row_sum();
    if constexpr (HELD == 0) {
      __builtin_nontemporal_store(r, out + t * 64 + lane);
    } else {
      held.put(nheld, r);
      ++nheld;
      if (nheld == HELD || next >= ntiles) {
        held.write(nheld, dst_out, nwaves * 64);
        dst_out += (int64_t)nheld * nwaves * 64;
        nheld = 0;
      }
    }
  }
  if (t > ntiles || ntiles * 64 == n) return;

  // The ragged last tile, all its pieces at once: a place past the last whole piece is given that piece again (no row
  // that exists is there).  With a wait after each KiB the pass took, us, fp32 p = 32, 30 thousand rows 5.8, p = 64 9.9, 300
  // thousand 19.8, bf16 p = 64, 30 thousand 7.0; 4.3, 6.2, 18.8 and 5.5 like this (64-row tiles of a wavefront are few there).
  const unsigned char* base = G + ntiles * tb;
  const int rows_here = (int)(n - ntiles * 64);
  const int lim = rows_here * ldr, whole = lim / EPL * EPL;     // elements that exist; those in whole pieces
  const int last = whole * E::SIZE - 16;
  wave_lds_fence();
  if (last >= 0) {
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int b = shift(k) + lane16;
      regs[k] = load16_stream(base + (uint32_t)(b < last ? b : last));
    }
#pragma unroll
    for (int k = 0; k < NP; ++k) *reinterpret_cast<uint4*>(mine + dst[k]) = regs[k];
  }
  if (!WHOLE && whole < lim) {
    wave_lds_fence();                                      // (after what its place has been given above)
    *reinterpret_cast<uint4*>(mine + whole * E::SIZE + (whole * E::SIZE >> sh) * 16) = load16_end<E>(base, whole, lim);
  }
  wave_lds_fence();
  const float r = row_sum();
  if (lane < rows_here) out[ntiles * 64 + lane] = r;
}

// The p x p solver text (any p): parallel-for phases over one workgroup.  Included here
// because the kernel below shares its term / weight functions.
#define FA_FN __device__
#define FA_TID ((int)threadIdx.x)
#define FA_NT ((int)blockDim.x)
#define FA_FOR(i, n) for (int i = FA_TID; i < (n); i += FA_NT)
#define FA_SYNC() __syncthreads()
#include "fa_irls_core.inc"

// K6: IRLS weights from the streamed projections (the re-streaming schedule's counterpart of
// the residual step inside the p x p kernel): explained variances v_i = |P_i|^2 / |g_i|^2,
// residuals 1 - v_i and 1 - |P_i - P_j|^2 / D_ij^2 (Eq. 5), the objective, the weights
// max(residual, delta)^(-1/2), and the column scales sqrt(w_i) / |g_i| of the next weighted
// Gram pass.  One workgroup.
__global__ __launch_bounds__(256) void fa_restream_weights_kernel(const fa_info* __restrict__ info,
                                                                  const double* __restrict__ P,
                                                                  int p, int m, double coef,
                                                                  double delta, double pair_tol,
                                                                  double expo,
                                                                  fa_resume* __restrict__ rs) {
  __shared__ double red[256];
  const int tid = threadIdx.x;
  const double* K = info->K;
  double part = 0.0;
  for (int i = tid; i < p; i += 256) {
    const double si = K[i * p + i];
    double pr = 0.0;
    for (int a = 0; a < m; ++a) pr = fma(P[i * m + a], P[i * m + a], pr);
    const double v = si > 0.0 ? pr / si : 0.0;
    const double rho = v < 1.0 ? 1.0 - v : 0.0;
    const double w = si > 0.0 ? fa_weight(rho, delta, expo) : 0.0;
    const double u = si > 0.0 ? sqrt(w / si) : 0.0;
    rs->w[i] = w;
    rs->v_streamed[i] = v;
    rs->u[i] = u;
    rs->uinv[i] = u > 0.0 ? 1.0 / u : 1.0;
    if (si > 0.0) part += fa_term(rho, expo);
  }
  for (int idx = tid; idx < p * p; idx += 256) {
    const int i = idx / p, j = idx - i * p;
    double cpv = 0.0;
    if (i != j && coef > 0.0) {
      const double si = K[i * p + i], sj = K[j * p + j];
      const double d2 = si + sj - 2.0 * K[idx];
      if (d2 > pair_tol * (si + sj)) {
        double pr = 0.0;
        for (int a = 0; a < m; ++a) {
          const double df = P[i * m + a] - P[j * m + a];
          pr = fma(df, df, pr);
        }
        const double q = pr / d2;
        const double rho = q < 1.0 ? 1.0 - q : 0.0;
        part += coef * fa_term(rho, expo);              // ordered pair (i, j)
        cpv = -2.0 * coef * fa_weight(rho, delta, expo) / d2;
      }
    }
    rs->cp[idx] = cpv;
  }
  red[tid] = part;
  __syncthreads();
  if (tid == 0) {
    double tot = 0.0;
    for (int t = 0; t < 256; ++t) tot += red[t];
    const int it = rs->it0 - 1;                         // the solve whose basis was measured
    if (it >= 0 && it < FA_ITERS_MAX) rs->obj_streamed[it] = tot;
    rs->scaled = 1;                                     // the next Gram pass uses rs->u
  }
}

// K2: K = sum over workgroups of their partial Grams, in a fixed order (sixteen interleaved
// strands, each summed in four interleaved sub-strands, then combined in a fixed tree), so the
// result does not depend on timing.  One 1024-thread block per 64 entries.
// TM = 0: the tiles are the upper-triangular tile pairs of a symmetric p x p matrix.
// TM > 0: the tiles are the T x TM blocks of a p x m matrix (row-major, leading dimension m).
// colscale (may be null; symmetric case only): entry (i, j) is multiplied by u_i u_j, which
// makes the result the Gram matrix G^T W G of the columns scaled by u = W^(1/2).
// cols (symmetric case only): the sums may be those of some rows of G, to be added to K, whose order
// is ldk, at the places of the listed columns; last: the tiles are those of the LAST pass.
__global__ __launch_bounds__(1024) void fa_gram_reduce_kernel(const double* __restrict__ partials,
                                                              int nparts, int T, int p,
                                                              double* __restrict__ K, int TM,
                                                              int m,
                                                              const double* __restrict__ colscale,
                                                              const int* __restrict__ gate,
                                                              int last, int ldk,
                                                              fa_gram_cols cols,
                                                              int* __restrict__ nonfinite) {
  if (gate != nullptr && *gate == 0) return;   // stand-by of a pass that did not need it
  const int NTP = TM > 0 ? T * TM : last ? T : T * (T + 1) / 2;
  const int ei = threadIdx.x & 63, g = threadIdx.x >> 6;   // entry, strand 0..15
  const int E = blockIdx.x * 64 + ei;                      // entry in [0, NTP*256)
  const int64_t stride = (int64_t)NTP * 256;
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  for (int b0 = g; b0 < nparts; b0 += 64) {
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int b = b0 + 16 * u;
      v[u] = b < nparts ? partials[(int64_t)b * stride + E] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) a[u] += v[u];
  }
  __shared__ double sh[1024];
  sh[threadIdx.x] = (a[0] + a[1]) + (a[2] + a[3]);
  __syncthreads();
  if (g == 0) {
    double t[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) t[k] = sh[k * 64 + ei];
#pragma unroll
    for (int w = 8; w >= 1; w >>= 1)
#pragma unroll
      for (int k = 0; k < w; ++k) t[k] += t[k + w];
    const double tot = t[0];
    const int tp = E >> 8, e = E & 255;
    const int r = e >> 6, l = e & 63;
    if (TM > 0) {
      const int gi = (tp / TM) * 16 + 4 * r + (l >> 4), ga = (tp % TM) * 16 + (l & 15);
      if (gi < p && ga < m) K[gi * m + ga] = tot;
      return;
    }
    int ta = 0, tb = 0;
    for (int aa = 0, k = 0; aa < T; ++aa)
      for (int bb = last ? T - 1 : aa; bb < T; ++bb, ++k)
        if (k == tp) { ta = aa; tb = bb; }
    const int gi = ta * 16 + 4 * r + (l >> 4), gj = tb * 16 + (l & 15);
    if (gi < p && gj < p && gi <= gj) {
      if (cols.add) {
        const int ki = cols.listed ? cols.idx[gi] : gi, kj = cols.listed ? cols.idx[gj] : gj;
        const double v = K[ki * ldk + kj] + tot;   // (both triangles hold the same bits)
        K[ki * ldk + kj] = v;
        K[kj * ldk + ki] = v;
        return;
      }
      const double v = colscale ? tot * (colscale[gi] * colscale[gj]) : tot;
      if (nonfinite != nullptr && !(fabs(v) <= 1.79e308)) *nonfinite = 1;   // (the pass before has cleared it)
      K[gi * p + gj] = v;
      K[gj * p + gi] = v;
    }
  }
}

// ------------------------------------------------------------------------------------------
// K4: out[k] = sum_i c[i] G[k][i]  (Alg. 1: d = (1/p) Y Y^T G 1 = G c).  Each thread owns 16
// bytes of every column (coalesced 16-byte loads: four rows of fp32, eight of bf16).
// fp32 storage: fp64 accumulation, one rounding to fp32 at the end; a thread's four outputs
// are one 16-byte store and a wavefront's store covers 1 KiB without gaps.
// bf16 storage: fp32 accumulation with c rounded to fp32 (per element at most (p + 1) 2^-24 of
// sum_i |c_i g_i|).  A thread's eight outputs are 32 bytes; stored as they are, each of its two
// stores would leave every other 16 bytes of a line to the other one, so the wavefront turns
// its 2 KiB of outputs round through LDS and stores two gap-free KiB instead.
template <typename E, typename acc_t>
__device__ __forceinline__ void combine_add(acc_t (&acc)[E::EPL], acc_t cc, const uint4& v) {
  if constexpr (E::SIZE == 4) {
    acc[0] += cc * (double)__uint_as_float(v.x);
    acc[1] += cc * (double)__uint_as_float(v.y);
    acc[2] += cc * (double)__uint_as_float(v.z);
    acc[3] += cc * (double)__uint_as_float(v.w);
  } else {
    acc[0] = fmaf(cc, __uint_as_float(v.x << 16), acc[0]);
    acc[1] = fmaf(cc, __uint_as_float(v.x & 0xffff0000u), acc[1]);
    acc[2] = fmaf(cc, __uint_as_float(v.y << 16), acc[2]);
    acc[3] = fmaf(cc, __uint_as_float(v.y & 0xffff0000u), acc[3]);
    acc[4] = fmaf(cc, __uint_as_float(v.z << 16), acc[4]);
    acc[5] = fmaf(cc, __uint_as_float(v.z & 0xffff0000u), acc[5]);
    acc[6] = fmaf(cc, __uint_as_float(v.w << 16), acc[6]);
    acc[7] = fmaf(cc, __uint_as_float(v.w & 0xffff0000u), acc[7]);
  }
}

#ifndef FA_COMBINE_NL
#define FA_COMBINE_NL 8
#endif
// LISTED: columns whose coefficient is 0 are left out if *skip is not 0 (see fa_combine_held_kernel).
template <typename E, bool LISTED>
__global__ __launch_bounds__(256) void fa_combine_kernel(const unsigned char* __restrict__ G,
                                                         int64_t ldg, int p, int64_t n,
                                                         const double* __restrict__ c, int cstride,
                                                         const double* __restrict__ skip,
                                                         float* __restrict__ out) {
  constexpr int EPL = E::EPL;
  constexpr int NL = FA_COMBINE_NL;   // columns in flight per thread
  typedef typename std::conditional<E::SIZE == 4, double, float>::type acc_t;
  __shared__ acc_t cs[FA_P_MAX + NL];
  __shared__ __attribute__((aligned(16))) float turn[E::SIZE == 2 ? 256 * 8 : 4];
  __shared__ int place[LISTED ? FA_P_MAX : 1], ncols;
  if constexpr (LISTED) {
    if (threadIdx.x < 64) {
      const int i = threadIdx.x;
      const double ci = i < p ? c[(int64_t)i * cstride] : 0.0;
      const bool keep = i < p && !(*skip != 0.0 && ci == 0.0);
      const uint64_t mask = __ballot(keep);
      const int at = __popcll(mask & (((uint64_t)1 << i) - 1)), count = __popcll(mask);
      cs[i] = (acc_t)0;
      if (i < NL) cs[FA_P_MAX + i] = (acc_t)0;
      place[i] = 0;
      wave_lds_fence();
      if (keep) { cs[at] = (acc_t)ci; place[at] = i; }
      if (i == 0) ncols = count;
    }
    __syncthreads();
    p = ncols;
  } else {
    if (threadIdx.x < FA_P_MAX + NL)
      cs[threadIdx.x] = (int)threadIdx.x < p ? (acc_t)c[(int64_t)threadIdx.x * cstride] : (acc_t)0;
    __syncthreads();
  }
  const int64_t ngroups = (n + EPL - 1) / EPL;
  for (int64_t gbase = (int64_t)blockIdx.x * 256; gbase < ngroups;
       gbase += (int64_t)gridDim.x * 256) {
    const int64_t gidx = gbase + threadIdx.x;
    const int64_t row0 = gidx * EPL;
    const bool block_full = (gbase + 256) * EPL <= n;   // uniform: no row guards needed
    if (!block_full && gidx >= ngroups) continue;
    acc_t acc[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = (acc_t)0;
    const unsigned char* src = G + row0 * E::SIZE;
    for (int c0 = 0; c0 < p; c0 += NL) {
      uint4 v[NL];
      if (block_full) {
#pragma unroll
        for (int u = 0; u < NL; ++u) {
          // columns past p re-read column p-1; their coefficient is zero
          const int at = c0 + u < p ? c0 + u : p - 1;
          const int col = LISTED ? place[at] : at;
          v[u] = load16_stream(src + (int64_t)col * ldg * E::SIZE);
        }
      } else if (row0 + EPL <= n) {
#pragma unroll
        for (int u = 0; u < NL; ++u) {
          const int at = c0 + u < p ? c0 + u : p - 1;
          const int col = LISTED ? place[at] : at;
          v[u] = load16_stream(src + (int64_t)col * ldg * E::SIZE);
        }
      } else {
        // the piece that the columns end in.  Under a condition for each element these loads were a chain, a wait for every
        // column.  us, whole pieces / a row or three more, before / now: fp32 p = 60, 1.2 M rows 50 / 84 / 61; p = 32, 2 M 44 /
        // 61 / 48; p = 15, 271 thousand 6.0 / 10.0 / 7.8; p = 64, 100 thousand 10 / 44 / 17; bf16 p = 23, 1 M 9.8 / 28 / 13.
#pragma unroll
        for (int u = 0; u < NL; ++u) {
          const int at = c0 + u < p ? c0 + u : p - 1;
          const int col = LISTED ? place[at] : at;
          v[u] = load16_end<E>(G + (int64_t)col * ldg * E::SIZE, row0, n);
        }
      }
#pragma unroll
      for (int u = 0; u < NL; ++u) {
        combine_add<E>(acc, cs[c0 + u], v[u]);
      }
    }
    float* dst = out + row0;
    if constexpr (E::SIZE == 4) {
      if (row0 + 4 <= n) {
        store16_through(dst, make_float4((float)acc[0], (float)acc[1], (float)acc[2],
                                         (float)acc[3]));
      } else {
        for (int e = 0; e < 4; ++e)
          if (row0 + e < n) dst[e] = (float)acc[e];
      }
    } else {
      if (block_full) {
        // the wavefront's 512 outputs, in row order, through its own 2 KiB of LDS
        const int lane = threadIdx.x & 63;
        float* mine = turn + (threadIdx.x & ~63) * 8;
        wave_lds_fence();        // the previous pass of this wavefront has read its part
        *reinterpret_cast<float4*>(mine + lane * 8) = make_float4(acc[0], acc[1], acc[2], acc[3]);
        *reinterpret_cast<float4*>(mine + lane * 8 + 4) =
            make_float4(acc[4], acc[5], acc[6], acc[7]);
        wave_lds_fence();
        const float4 lo = *reinterpret_cast<const float4*>(mine + lane * 4);
        const float4 hi = *reinterpret_cast<const float4*>(mine + 256 + lane * 4);
        float* wdst = out + (gbase + (threadIdx.x & ~63)) * 8;    // the wavefront's first row
        store16_through(wdst + lane * 4, lo);
        store16_through(wdst + 256 + lane * 4, hi);
      } else {
        for (int e = 0; e < 8; ++e)
          if (row0 + e < n) dst[e] = acc[e];
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
// K4 for large sets: the same sums (same order, same bits), but the outputs are held back on the chip and written
// many tiles at a time.  A read stream with writes strewn in between is what bounds the kernel above: p = 32, bf16,
// n = 124M takes 1147 us without its stores and 1510 with them, although 0.5 GB are written in 72.  Here one
// workgroup per compute unit walks its tiles in step with the others, so that the whole chip reads for a while and
// then writes for a while; the more is written at a time the better (with twice the loads in flight: every tile for
// itself 1567 us; 12 KiB a wavefront 1512, 24 1449, 36 1370; with registers beside LDS 66 KiB 1332, 98 KiB 1295).
//
// A wavefront takes the tiles w, w + W, ... (64 lanes x 16 bytes of every column).  Loads run ahead of the sums
// over the ends of columns and tiles: FA_HELD_SLOTS 16-byte slots a lane, one column of one tile each, each refilled as
// soon as it is used.  24 KiB in flight a compute unit are the right amount; with more the reads get in each other's
// way (5 / 6 / 8 / 10 / 14 slots, us: p = 32 bf16, n = 124M 1353 / 1279 / 1297 / 1345 / 1363, 1510 with the kernel
// above; p = 15 fp32, n = 30M 254 / 261 / 269 / 276 / 280, 295 above; p = 64 fp32, n = 8M 288 / 261 / 275 / 283 / 281, 300
// above, but n = 50M 1826 / 1727 / 1650 / 1668 / 1666, 1830 above).  Eight wavefronts are slower than four by 3 to 7 %
// at 3 slots and more beyond.  Workgroups of one XCD (blockIdx mod 8) take neighbouring tiles: p = 15, n = 11.2M 113 -> 110 us
// (14 slots), the others the same.  At p = 15, n = 11.2M the pass now takes 97-103 us, 104-114 above.
//
// RT tiles of a batch stay in registers, LT in LDS.  p <= 16: half the registers and three quarters of the LDS, so that the
// solver of a set on another stream fits beside a workgroup, whose tiles are nobody else's; one batch is
// still all of p = 15, n = 11.2M.  A batch is written at the end of the FA_HELD_SLOTS slots after which another ENDS tiles might not
// fit: 55 tiles (now and then 56 of five columns) or 103 for fp32, 28 or 51 for bf16.  ENDS: most tiles that can end within
// FA_HELD_SLOTS columns, two of five columns, which is the fewest there are (fa_combine_held_applies), one of six and more.
// skip (device, may be null): if *skip is not 0, columns whose coefficient is 0 are not read (Multi-Krum; only where
// no gradient holds a NaN or an infinity, which 0 times it would carry over).
#define FA_HELD_SLOTS 6
#define FA_HELD_WAVES 4

// N tiles of H x 16 bytes a lane, each in registers of its own (an array would be indexed, and so go to scratch memory)
template <int N, int H, int ID = 0>
struct fa_held_tiles {
  static constexpr int HALF = N / 2;
  fa_held_tiles<HALF, H, ID> lower;
  fa_held_tiles<N - HALF, H, ID + HALF> upper;
  __device__ __forceinline__ void put(int i, fa_u32x4 x, fa_u32x4 y) {
    if (i < HALF) lower.put(i, x, y);
    else upper.put(i - HALF, x, y);
  }
  // the first `count` of them, `step` apart
  __device__ __forceinline__ void write(int count, float* dst, int64_t step) const {
    lower.write(count, dst, step);
    if (count > HALF) upper.write(count - HALF, dst + HALF * step, step);
  }
};
template <int H, int ID>
struct fa_held_tiles<1, H, ID> {
  fa_u32x4 a, b;
  __device__ __forceinline__ void put(int, fa_u32x4 x, fa_u32x4 y) {
    a = x;
    if constexpr (H == 2) b = y;
    asm volatile("" ::"n"(ID));        // each place a branch of its own: two merged ones would be one indexed store
  }
  __device__ __forceinline__ void write(int count, float* dst, int64_t) const {
    if (count <= 0) return;
    store16_through(dst, a);
    if constexpr (H == 2) store16_through(dst + 256, b);
  }
};

__device__ __forceinline__ float lane_value(float x, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}
__device__ __forceinline__ double lane_value(double x, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                          __builtin_amdgcn_readlane(__double2loint(x), lane));
}

template <typename E, int RT, int LT, int ENDS>
constexpr size_t fa_held_lds_bytes() { return (size_t)FA_HELD_WAVES * (LT + ENDS) * 64 * E::EPL * sizeof(float); }

// WGS: workgroups a compute unit that the registers have to leave room for
template <typename E, int RT, int LT, int ENDS, int WGS>
__global__ __launch_bounds__(64 * FA_HELD_WAVES, FA_HELD_WAVES / 4 * WGS) void fa_combine_held_kernel(
    const unsigned char* __restrict__ G, int64_t ldg, int p, int64_t n, const double* __restrict__ c,
    int cstride, const double* __restrict__ skip, float* __restrict__ out) {
  constexpr int EPL = E::EPL, ROWS = 64 * EPL, H = ROWS / 256, S = FA_HELD_SLOTS;
  typedef typename std::conditional<E::SIZE == 4, double, float>::type acc_t;
  extern __shared__ __attribute__((aligned(16))) float held[];
  __shared__ acc_t lcoef[FA_P_MAX];
  __shared__ int64_t loff[FA_P_MAX];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // the columns that are read, in ascending order: lane k holds the k-th one's coefficient and place
  int ncols;
  {
    const double ci = lane < p ? c[(int64_t)lane * cstride] : 0.0;
    const bool some = skip != nullptr && *skip != 0.0;
    const bool keep = lane < p && !(some && ci == 0.0);
    const uint64_t mask = __ballot(keep);
    ncols = __popcll(mask);
    if (keep && wave == 0) {
      const int at = __popcll(mask & (((uint64_t)1 << lane) - 1));
      lcoef[at] = (acc_t)ci;
      loff[at] = (int64_t)lane * ldg * E::SIZE;
    }
  }
  __syncthreads();
  const acc_t coef = lane < ncols ? lcoef[lane] : (acc_t)0;
  const int64_t off = loff[lane < ncols ? lane : ncols - 1];
  const int off_lo = (int)off, off_hi = (int)(off >> 32);
  auto column = [&](int k) -> int64_t {
    return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane(off_hi, k) << 32) |
                     (uint32_t)__builtin_amdgcn_readlane(off_lo, k));
  };

  const int64_t W = (int64_t)gridDim.x * FA_HELD_WAVES;
  const int blk = (gridDim.x & 7) == 0 ? (int)((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3))
                                       : (int)blockIdx.x;
  const int64_t w = (int64_t)blk * FA_HELD_WAVES + wave;
  const int64_t ntiles = n / ROWS;
  const int mine = (int)(w < ntiles ? (ntiles - w + W - 1) / W : 0);
  acc_t acc[EPL];
#pragma unroll
  for (int e = 0; e < EPL; ++e) acc[e] = (acc_t)0;

  // The rows that do not fill a tile: the wavefront that would be next, which has a tile less than those before it, ahead of
  // its tiles and eight columns at a time.  Behind them and column by column, each waited for, they made every set of
  // another length than whole tiles slower, 16 tiles a wavefront and no more than the kernel for small sets takes: fp32, us,
  // 4 194 304 rows / 4 234 340 before / now (that kernel): p = 15 42.3 / 45.5 / 42.7 (46.2), p = 64 159 / 187 / 173 (189).
  if (ntiles * ROWS < n && w == ntiles % W) {
    const int64_t row0 = ntiles * ROWS + lane * EPL;
    constexpr int NL = 8;                                     // columns in flight
    if (row0 < n) {
      for (int k0 = 0; k0 < ncols; k0 += NL) {
        uint4 v[NL];
        if (row0 + EPL <= n) {
#pragma unroll
          for (int u = 0; u < NL; ++u)
            v[u] = load16_stream(G + column(k0 + u < ncols ? k0 + u : ncols - 1) + row0 * E::SIZE);
        } else {
#pragma unroll
          for (int u = 0; u < NL; ++u)
            v[u] = load16_end<E>(G + column(k0 + u < ncols ? k0 + u : ncols - 1), row0, n);
        }
#pragma unroll
        for (int u = 0; u < NL; ++u)
          if (k0 + u < ncols) combine_add<E>(acc, lane_value(coef, k0 + u), v[u]);
      }
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        if (row0 + e < n) out[row0 + e] = (float)acc[e];
        acc[e] = (acc_t)0;
      }
    }
  }

  if (mine > 0) {
    float* const kept = held + wave * (LT + ENDS) * ROWS;   // LT tiles, then those that go on to registers
    const unsigned char* base = G + w * (ROWS * E::SIZE) + lane * 16;
    const int64_t step = W * (ROWS * E::SIZE), out_step = W * ROWS;
    int lt = 0, lc = 0;                                     // the next slot to load: tile, column
    uint4 v[S];
    // past the end the last tile is read again (its sums are dropped)
#define FA_HELD_LOAD(s)                                                     \
    do {                                                                    \
      v[s] = load16_stream(base + column(lc));                              \
      if (++lc == ncols) { lc = 0; if (lt + 1 < mine) { ++lt; base += step; } } \
    } while (0)
#pragma unroll
    for (int s = 0; s < S; ++s) {
      FA_HELD_LOAD(s);
      __builtin_amdgcn_sched_barrier(0);                    // in the order they are waited for
    }
    fa_held_tiles<RT, H> regs;
    float* dst = out + w * ROWS + lane * 4;                 // first tile of the batch
    int cc = 0, nb = 0, done = 0;                           // column; tiles of the batch; tiles summed
    while (done < mine) {
      const int nb0 = nb;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        combine_add<E>(acc, lane_value(coef, cc), v[s]);
        FA_HELD_LOAD(s);
        if (++cc == ncols) {
          cc = 0;
          // row order: fp32 lanes hold four rows, bf16 lanes eight, of which a store takes four
          float* o = kept + (nb < LT ? nb : LT + (nb - nb0)) * ROWS + lane * EPL;
          *reinterpret_cast<float4*>(o) = make_float4((float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]);
          if constexpr (EPL == 8)
            *reinterpret_cast<float4*>(o + 4) = make_float4(acc[4], acc[5], acc[6], acc[7]);
#pragma unroll
          for (int e = 0; e < EPL; ++e) acc[e] = (acc_t)0;
          ++nb;
        }
      }
      if (nb == nb0) continue;
      wave_lds_fence();
      for (int j = nb0 < LT ? LT : nb0; j < nb; ++j) {      // (the first of them can only be nb0 or LT)
        const float* from = kept + (LT + (j - nb0)) * ROWS + lane * 4;
        const fa_u32x4 x = *reinterpret_cast<const fa_u32x4*>(from);
        regs.put(j - LT, x, H == 2 ? *reinterpret_cast<const fa_u32x4*>(from + (H - 1) * 256) : x);
      }
      done += nb - nb0;
      if (done >= mine || nb > LT + RT - ENDS) {
        const int here = done > mine ? nb - (done - mine) : nb;    // what came of the last tile read again is dropped
        for (int j = 0; j < here && j < LT; ++j, dst += out_step)
#pragma unroll
          for (int h = 0; h < H; ++h)
            store16_through(dst + h * 256, *reinterpret_cast<const float4*>(kept + j * ROWS + h * 256 + lane * 4));
        if (here > LT) {
          regs.write(here - LT, dst, out_step);
          dst += (here - LT) * out_step;
        }
        nb = 0;
      }
      wave_lds_fence();                                     // the reads above precede the next tiles' writes
    }
#undef FA_HELD_LOAD
  }
}

// ------------------------------------------------------------------------------------------
// One row of the Gram matrix: k_u = g_i . g_{cols[u]} for up to FA_ROW_JB gradients: what is left
// to do for some rows of a wide set (p > 16) when the last gradient to hold them lands and the
// others' share of K is there already (Alg. 1: the server receives the p workers' gradients; see
// fa_gram_update_rows).  Each thread owns 16 bytes of
// gradient i and of every listed gradient per pass; products of the stored values are exact
// in fp64 and are added in fp64.  Static chunk -> workgroup map, fixed-order sums inside the
// workgroup: one partial row per workgroup, bitwise reproducible.
struct fa_row_cols { int idx[FA_ROW_JB]; };

template <typename E>
__global__ __launch_bounds__(256) void fa_gram_row_kernel(const unsigned char* __restrict__ G,
                                                          int64_t ldg, int64_t n, int i,
                                                          fa_row_cols cols, int nj,
                                                          double* __restrict__ partials) {
  constexpr int EPL = E::EPL;
  __shared__ double red[4][FA_ROW_JB];
  double acc[FA_ROW_JB];
#pragma unroll
  for (int u = 0; u < FA_ROW_JB; ++u) acc[u] = 0.0;
  const unsigned char* gi = G + (int64_t)i * ldg * E::SIZE;
  const int64_t ngroups = (n + EPL - 1) / EPL;
  for (int64_t gbase = (int64_t)blockIdx.x * 256; gbase < ngroups;
       gbase += (int64_t)gridDim.x * 256) {
    const int64_t row0 = (gbase + threadIdx.x) * EPL;
    const bool block_full = (gbase + 256) * EPL <= n;   // uniform
    uint4 xi, xj[FA_ROW_JB];
    if (block_full) {
      xi = load16_stream(gi + row0 * E::SIZE);
#pragma unroll
      for (int u = 0; u < FA_ROW_JB; ++u)   // entries past nj repeat the last listed gradient
        xj[u] = load16_stream(G + ((int64_t)cols.idx[u] * ldg + row0) * E::SIZE);
    } else {
      xi = load16_guarded<E>(gi, row0, n);
#pragma unroll
      for (int u = 0; u < FA_ROW_JB; ++u)
        xj[u] = load16_guarded<E>(G + (int64_t)cols.idx[u] * ldg * E::SIZE, row0, n);
    }
    double a[EPL];
    {
      const uint32_t w[4] = {xi.x, xi.y, xi.z, xi.w};
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        if constexpr (E::SIZE == 4) a[e] = (double)__uint_as_float(w[e]);
        else a[e] = (double)bf16_bits_to_f32((w[e >> 1] >> (16 * (e & 1))) & 0xffffu);
      }
    }
#pragma unroll
    for (int u = 0; u < FA_ROW_JB; ++u) {
      const uint32_t w[4] = {xj[u].x, xj[u].y, xj[u].z, xj[u].w};
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        double b;
        if constexpr (E::SIZE == 4) b = (double)__uint_as_float(w[e]);
        else b = (double)bf16_bits_to_f32((w[e >> 1] >> (16 * (e & 1))) & 0xffffu);
        acc[u] = fma(a[e], b, acc[u]);
      }
    }
  }
  // fixed butterfly inside each wavefront, wavefronts in order
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int u = 0; u < FA_ROW_JB; ++u) {
    double x = acc[u];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
    if (lane == 0) red[wave][u] = x;
  }
  __syncthreads();
  if ((int)threadIdx.x < FA_ROW_JB)
    partials[(int64_t)blockIdx.x * FA_ROW_JB + threadIdx.x] =
        (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
}

// Fixed-order sum of the partial rows (four interleaved strands per entry, then a fixed
// tree), added to row and column i of K (row-major p x p; zero when the round opens).
__global__ __launch_bounds__(64 * FA_ROW_JB) void fa_gram_row_reduce_kernel(
    const double* __restrict__ partials, int nparts, fa_row_cols cols, int nj, int i, int p,
    double* __restrict__ K) {
  __shared__ double sh[FA_ROW_JB][64];
  const int u = threadIdx.x >> 6, s = threadIdx.x & 63;
  double a = 0.0;
  for (int b = s; b < nparts; b += 64) a += partials[(int64_t)b * FA_ROW_JB + u];
  sh[u][s] = a;
  __syncthreads();
  if (s == 0 && u < nj) {
    double t[64];
#pragma unroll
    for (int k = 0; k < 64; ++k) t[k] = sh[u][k];
#pragma unroll
    for (int w = 32; w >= 1; w >>= 1)
#pragma unroll
      for (int k = 0; k < w; ++k) t[k] += t[k + w];
    const int j = cols.idx[u];
    const double v = K[i * p + j] + t[0];     // K_ij and K_ji see the same addends in the same order
    K[i * p + j] = v;
    K[j * p + i] = v;
  }
}

__global__ __launch_bounds__(256) void fa_zero_kernel(double* __restrict__ dst, int count) {
  for (int k = blockIdx.x * 256 + threadIdx.x; k < count; k += gridDim.x * 256) dst[k] = 0.0;
}

hipError_t fa_launch_zero(double* dst, int count, hipStream_t st) {
  hipLaunchKernelGGL(fa_zero_kernel, dim3((count + 255) / 256), dim3(256), 0, st, dst, count);
  return hipGetLastError();
}

hipError_t fa_launch_gram_row(const void* G, int64_t ldg, int p, int64_t n, int dtype, int i,
                              double* partials, int max_parts, double* Kd, hipStream_t st) {
  const int epl = dtype == FA_F32 ? 4 : 8;
  const int64_t ngroups = (n + epl - 1) / epl;
  int64_t blocks = (ngroups + 255) / 256;
  if (blocks > max_parts) blocks = max_parts;
  // gradient i against itself and against every other one, FA_ROW_JB of them per pass
  for (int a0 = 0; a0 < p; a0 += FA_ROW_JB) {
    fa_row_cols cols;
    const int nj = p - a0 < FA_ROW_JB ? p - a0 : FA_ROW_JB;
    for (int u = 0; u < FA_ROW_JB; ++u) cols.idx[u] = a0 + (u < nj ? u : nj - 1);
    if (dtype == FA_F32)
      hipLaunchKernelGGL((fa_gram_row_kernel<ElemF32>), dim3((unsigned)blocks), dim3(256), 0, st,
                         (const unsigned char*)G, ldg, n, i, cols, nj, partials);
    else
      hipLaunchKernelGGL((fa_gram_row_kernel<ElemBF16>), dim3((unsigned)blocks), dim3(256), 0, st,
                         (const unsigned char*)G, ldg, n, i, cols, nj, partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fa_gram_row_reduce_kernel, dim3(1), dim3(64 * FA_ROW_JB), 0, st,
                       (const double*)partials, (int)blocks, cols, nj, i, p, Kd);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// ------------------------------------------------------------------------------------------
// Y = G A for MB columns of A at once (the basis of Sec. 2.1 materialised: column a of Y is
// sum_i A[i][a] g_i): the aggregate pass with MB coefficient vectors, so G is read once per MB
// columns of Y instead of once per column.  A is row-major p x lda in device memory; column a
// of Y at Y + a*ldy.  Same thread-to-data map and loads as fa_combine_kernel.
template <typename E, int MB>
__global__ __launch_bounds__(256) void fa_combine_multi_kernel(
    const unsigned char* __restrict__ G, int64_t ldg, int p, int64_t n,
    const double* __restrict__ A, int lda, int ncols, float* __restrict__ Y, int64_t ldy) {
  constexpr int EPL = E::EPL;
  constexpr int NL = 4;                     // columns of G in flight per thread
  // fp32 storage: fp64 sums, one rounding per output; bf16 storage: fp32 sums with the
  // coefficients rounded to fp32, as in the aggregate pass of that storage
  typedef typename std::conditional<E::SIZE == 4, double, float>::type acc_t;
  __shared__ acc_t cs[(FA_P_MAX + NL) * MB];
  for (int t = threadIdx.x; t < (FA_P_MAX + NL) * MB; t += 256) {
    const int i = t / MB, a = t - i * MB;
    cs[t] = (i < p && a < ncols) ? (acc_t)A[(int64_t)i * lda + a] : (acc_t)0;
  }
  __syncthreads();
  const int64_t ngroups = (n + EPL - 1) / EPL;
  for (int64_t gbase = (int64_t)blockIdx.x * 256; gbase < ngroups;
       gbase += (int64_t)gridDim.x * 256) {
    const int64_t gidx = gbase + threadIdx.x;
    const int64_t row0 = gidx * EPL;
    const bool block_full = (gbase + 256) * EPL <= n;   // uniform: no row guards needed
    if (!block_full && gidx >= ngroups) continue;
    acc_t acc[MB][EPL];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[a][e] = (acc_t)0;
    const unsigned char* src = G + row0 * E::SIZE;
    for (int c0 = 0; c0 < p; c0 += NL) {
      uint4 v[NL];
#pragma unroll
      for (int u = 0; u < NL; ++u) {
        const int col = c0 + u < p ? c0 + u : p - 1;    // past p: coefficient zero
        if (block_full) v[u] = load16_stream(src + (int64_t)col * ldg * E::SIZE);
        else v[u] = load16_guarded<E>(G + (int64_t)col * ldg * E::SIZE, row0, n);
      }
#pragma unroll
      for (int u = 0; u < NL; ++u) {
        acc_t x[EPL];
        if constexpr (E::SIZE == 4) {
          x[0] = (double)__uint_as_float(v[u].x); x[1] = (double)__uint_as_float(v[u].y);
          x[2] = (double)__uint_as_float(v[u].z); x[3] = (double)__uint_as_float(v[u].w);
        } else {
          x[0] = __uint_as_float(v[u].x << 16); x[1] = __uint_as_float(v[u].x & 0xffff0000u);
          x[2] = __uint_as_float(v[u].y << 16); x[3] = __uint_as_float(v[u].y & 0xffff0000u);
          x[4] = __uint_as_float(v[u].z << 16); x[5] = __uint_as_float(v[u].z & 0xffff0000u);
          x[6] = __uint_as_float(v[u].w << 16); x[7] = __uint_as_float(v[u].w & 0xffff0000u);
        }
#pragma unroll
        for (int a = 0; a < MB; ++a) {
          const acc_t cc = cs[(c0 + u) * MB + a];
#pragma unroll
          for (int e = 0; e < EPL; ++e) {
            if constexpr (E::SIZE == 4) acc[a][e] = fma(cc, x[e], acc[a][e]);
            else acc[a][e] = fmaf(cc, x[e], acc[a][e]);
          }
        }
      }
    }
#pragma unroll
    for (int a = 0; a < MB; ++a) {
      if (a >= ncols) break;
      float* dst = Y + (int64_t)a * ldy + row0;
      if (row0 + EPL <= n) {
#pragma unroll
        for (int e = 0; e < EPL; e += 4)
          store16_through(dst + e, make_float4((float)acc[a][e], (float)acc[a][e + 1],
                                               (float)acc[a][e + 2], (float)acc[a][e + 3]));
      } else {
        for (int e = 0; e < EPL; ++e)
          if (row0 + e < n) dst[e] = (float)acc[a][e];
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
// Multi-Krum from the Gram matrix (the distance-based aggregator the paper compares with,
// Sec. 3 "Baselines", Sec. 2.3; rule of Blanchard et al., 2017): D_ij^2 = K_ii + K_jj - 2 K_ij,
// worker i is scored by the sum of its k = p - f - 2 smallest distances to the others (added
// in ascending order), the q smallest scores are selected (ties: smaller index), and the
// coefficients of out = G c are 1/q on the selected workers.  A distance's place in its row is
// counted, one thread per distance, and the row's thread adds the first k up in order (an insertion
// sort by one thread per worker took 13.6 us at p = 15 and 185 at p = 64; 4.6 and 28 now).
// p <= 64; scores and selected may be host memory the device can write.  c[FA_P_MAX]: whether the columns that were not
// selected may be left out of the aggregate (a finite K has no NaN and no infinity in any gradient).
__global__ __launch_bounds__(1024) void fa_krum_kernel(const double* __restrict__ K, int p, int k,
                                                       int q, double* __restrict__ c,
                                                       double* __restrict__ scores,
                                                       int* __restrict__ selected) {
  __shared__ double sc[FA_P_MAX];
  __shared__ double dist[FA_P_MAX][FA_P_MAX + 1];
  constexpr int PER = FA_P_MAX * FA_P_MAX / 1024;
  const int tid = threadIdx.x, j = tid & 63, i0 = tid >> 6;      // entries (i0 + 16 u, j)
  double x[PER];
  int pos[PER];
  bool ok = true;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int i = i0 + 16 * u;
    x[u] = 0.0;
    if (i < p && j < p) {
      ok = ok && fabs(K[i * p + j]) <= 1.79e308;
      const double d = K[i * p + i] + K[j * p + j] - 2.0 * K[i * p + j];
      x[u] = d > 0.0 ? d : 0.0;
      dist[i][j] = x[u];
    }
  }
  const int finite = __syncthreads_and(ok ? 1 : 0);
  if (tid == 0) c[FA_P_MAX] = finite ? 1.0 : 0.0;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int i = i0 + 16 * u;
    pos[u] = 0;
    if (i < p && j < p && j != i)
      for (int t = 0; t < p; ++t) {
        const double y = dist[i][t];
        pos[u] += t != i && (y < x[u] || (y == x[u] && t < j)) ? 1 : 0;
      }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int i = i0 + 16 * u;
    if (i < p && j < p && j != i) dist[i][pos[u]] = x[u];       // ascending
  }
  __syncthreads();
  double s = 0.0;
  if (tid < p) {
    for (int t = 0; t < k; ++t) s += dist[tid][t];
    sc[tid] = s;
    scores[tid] = s;
  }
  __syncthreads();
  if (tid < p) {
    int rank = 0;
    for (int t = 0; t < p; ++t) rank += (sc[t] < s || (sc[t] == s && t < tid)) ? 1 : 0;
    const int sel = rank < q ? 1 : 0;
    selected[tid] = sel;
    c[tid] = sel ? 1.0 / (double)q : 0.0;
  }
}

// Y (+ a*ldy, a < m) = G A, A row-major p x m in device memory; eight columns per pass over G
// in either layout.
hipError_t fa_launch_combine_multi(const void* G, int64_t ldg, int p, int64_t n, int dtype,
                                   int layout, const double* A, int m, float* Y, int64_t ldy,
                                   int max_blocks, hipStream_t st) {
  if (layout == FA_ROW_MAJOR) {
    const int ldr = (int)ldg;
    const size_t lds = fa_rows_lds_bytes(ldr, dtype == FA_F32 ? 4 : 2);
    int64_t blocks = (n + 255) / 256;
    // one workgroup per span of 256 rows (measured at p = 15, n = 11.2M: 124 us; eight
    // persistent workgroups per compute unit 133 us, sixty-four 121-127 us)
    if (blocks > 0x7fffffff) blocks = 0x7fffffff;
    for (int a0 = 0; a0 < m; a0 += FA_ROWS_MULTI) {
      const int nc = m - a0 < FA_ROWS_MULTI ? m - a0 : FA_ROWS_MULTI;
      if (dtype == FA_F32)
        hipLaunchKernelGGL((fa_combine_rows_kernel<ElemF32, FA_ROWS_MULTI>), dim3((unsigned)blocks),
                           dim3(256), lds, st, (const unsigned char*)G, ldr, p, n, A + a0, m, nc,
                           Y + (int64_t)a0 * ldy, ldy);
      else
        hipLaunchKernelGGL((fa_combine_rows_kernel<ElemBF16, FA_ROWS_MULTI>), dim3((unsigned)blocks),
                           dim3(256), lds, st, (const unsigned char*)G, ldr, p, n, A + a0, m, nc,
                           Y + (int64_t)a0 * ldy, ldy);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  constexpr int MB = 8;
  const int epl = dtype == FA_F32 ? 4 : 8;
  const int64_t ngroups = (n + epl - 1) / epl;
  int64_t blocks = (ngroups + 255) / 256;
  if (blocks > max_blocks) blocks = max_blocks;
  for (int a0 = 0; a0 < m; a0 += MB) {
    const int nc = m - a0 < MB ? m - a0 : MB;
    if (dtype == FA_F32)
      hipLaunchKernelGGL((fa_combine_multi_kernel<ElemF32, MB>), dim3((unsigned)blocks), dim3(256),
                         0, st, (const unsigned char*)G, ldg, p, n, A + a0, m, nc,
                         Y + (int64_t)a0 * ldy, ldy);
    else
      hipLaunchKernelGGL((fa_combine_multi_kernel<ElemBF16, MB>), dim3((unsigned)blocks), dim3(256),
                         0, st, (const unsigned char*)G, ldg, p, n, A + a0, m, nc,
                         Y + (int64_t)a0 * ldy, ldy);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t fa_launch_krum(const double* Kd, int p, int f, int q, double* cd, double* scores_d,
                          int* selected_d, hipStream_t st) {
  hipLaunchKernelGGL(fa_krum_kernel, dim3(1), dim3(1024), 0, st, Kd, p, p - f - 2, q, cd, scores_d,
                     selected_d);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// Streamed check of a materialised basis Y (n x m, fp32, column a at Y + a*ldy): one pass
// computes W = Y^T [Y | G] in fp64 on the matrix cores: Y^T Y (the identity for the
// orthonormal basis of Sec. 2.1) and Y^T G (row a, column i: the projection of g_i on y_a,
// whose squares add up to the explained variance of Sec. 2.1 times |g_i|^2).
// One workgroup (eight wavefronts) per (row stripe, tile row ta of the result); a wavefront
// takes 16 rows at a time: lane (c, k) holds rows 4k..4k+3 of column c of each 16-column tile
// of [Y | G] (one 16-byte load where the rows are contiguous), and feeds row 4k+s of tile ta
// of Y and of every tile to the s-th matrix instruction - the contraction does not care in
// which order the rows come, as long as both operands agree, and the registers of a tile
// serve as either operand.  [Y | G] is therefore read once per tile row of Y (once at
// m <= 16), all TC result tiles of the row accumulate in registers.
// G is addressed by strides (elements): g_rs between rows, g_cs between columns, which
// covers both storage orders.
template <typename E>
__device__ __forceinline__ double load_elem(const unsigned char* base, int64_t idx) {
  if constexpr (E::SIZE == 4) return (double)reinterpret_cast<const float*>(base)[idx];
  else return (double)bf16_bits_to_f32(reinterpret_cast<const uint16_t*>(base)[idx]);
}
// rows row0..row0+3 of one column (zero past n, zero if the column does not exist)
template <typename E>
__device__ __forceinline__ void load_rows4(const unsigned char* base, int64_t col_off,
                                           int64_t rs, int64_t row0, int64_t n, bool on,
                                           double* x) {
  x[0] = x[1] = x[2] = x[3] = 0.0;
  if (!on || row0 >= n) return;
  if (rs == 1 && row0 + 4 <= n) {
    const unsigned char* src = base + (col_off + row0) * E::SIZE;
    if constexpr (E::SIZE == 4) {
      if (((uintptr_t)src & 15u) == 0) {
        const float4 f = *reinterpret_cast<const float4*>(src);
        x[0] = (double)f.x; x[1] = (double)f.y; x[2] = (double)f.z; x[3] = (double)f.w;
        return;
      }
    } else {
      if (((uintptr_t)src & 7u) == 0) {
        const uint2 h = *reinterpret_cast<const uint2*>(src);
        x[0] = (double)bf16_bits_to_f32(h.x & 0xffffu); x[1] = (double)bf16_bits_to_f32(h.x >> 16);
        x[2] = (double)bf16_bits_to_f32(h.y & 0xffffu); x[3] = (double)bf16_bits_to_f32(h.y >> 16);
        return;
      }
    }
  }
  for (int s = 0; s < 4; ++s)
    if (row0 + s < n) x[s] = load_elem<E>(base, col_off + (row0 + s) * rs);
}

// four rows row0..row0+3 (all inside the matrix) of one column as raw bits: the loads of a
// stage are all issued before any of them is used
template <typename E, bool ROWS>
__device__ __forceinline__ uint4 cross_raw(const unsigned char* base, int64_t col_off, int64_t rs,
                                           int64_t row0) {
  uint4 r = {0u, 0u, 0u, 0u};
  if constexpr (!ROWS) {
    const unsigned char* src = base + (col_off + row0) * E::SIZE;
    if constexpr (E::SIZE == 4) {
      r = *reinterpret_cast<const uint4*>(src);
    } else {
      const uint2 h = *reinterpret_cast<const uint2*>(src);
      r.x = h.x; r.y = h.y;
    }
  } else if constexpr (E::SIZE == 4) {
    const uint32_t* g = reinterpret_cast<const uint32_t*>(base) + col_off + row0 * rs;
    r.x = g[0]; r.y = g[rs]; r.z = g[2 * rs]; r.w = g[3 * rs];
  } else {
    const uint16_t* g = reinterpret_cast<const uint16_t*>(base) + col_off + row0 * rs;
    r.x = g[0]; r.y = g[rs]; r.z = g[2 * rs]; r.w = g[3 * rs];
  }
  return r;
}
template <typename E, bool ROWS>
__device__ __forceinline__ void cross_decode(const uint4& r, double* x) {
  if constexpr (E::SIZE == 4) {
    x[0] = (double)__uint_as_float(r.x); x[1] = (double)__uint_as_float(r.y);
    x[2] = (double)__uint_as_float(r.z); x[3] = (double)__uint_as_float(r.w);
  } else if constexpr (!ROWS) {
    x[0] = (double)bf16_bits_to_f32(r.x & 0xffffu); x[1] = (double)bf16_bits_to_f32(r.x >> 16);
    x[2] = (double)bf16_bits_to_f32(r.y & 0xffffu); x[3] = (double)bf16_bits_to_f32(r.y >> 16);
  } else {
    x[0] = (double)bf16_bits_to_f32(r.x); x[1] = (double)bf16_bits_to_f32(r.y);
    x[2] = (double)bf16_bits_to_f32(r.z); x[3] = (double)bf16_bits_to_f32(r.w);
  }
}

// ROWS: G is stored row-major (g_rs = row pitch, g_cs = 1); otherwise g_rs = 1 and the four
// rows of a lane are one 16-byte (fp32) or 8-byte (bf16) load, aligned because G, Y and their
// column pitches are (the caller checks).
template <typename E, int TC, bool ROWS>
__global__ __launch_bounds__(512) void fa_cross_kernel(const float* __restrict__ Y, int64_t ldy,
                                                       int m,
                                                       const unsigned char* __restrict__ G,
                                                       int64_t g_rs, int64_t g_cs, int p,
                                                       int64_t n, int TMr,
                                                       double* __restrict__ partials) {
  // wavefronts; 16-row chunks per stage (the next stage's loads are in flight while this
  // one is multiplied: two stages of raw bits and TC accumulators share the registers)
  constexpr int NWV = 8, U = TC <= 2 ? 4 : TC <= 4 ? 2 : 1;
  __shared__ double red[NWV * 256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c16 = lane & 15, kq = lane >> 4;
  const int ta = (int)blockIdx.y;            // tile row: columns 16 ta .. of Y on the left
  const unsigned char* Yb = reinterpret_cast<const unsigned char*>(Y);
  const int64_t wid = (int64_t)blockIdx.x * NWV + wave, nw = (int64_t)gridDim.x * NWV;
  v4f64 acc[TC];
#pragma unroll
  for (int tb = 0; tb < TC; ++tb) acc[tb] = v4f64{0.0, 0.0, 0.0, 0.0};

  // operands of tile tb for the rows of one chunk, already as doubles -> TC products
  auto multiply = [&](double (&b)[TC][4]) {
    double a[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      a[s] = b[0][s];
#pragma unroll
      for (int t = 1; t < TC && t < 4; ++t) a[s] = ta == t ? b[t][s] : a[s];
    }
#pragma unroll
    for (int tb = 0; tb < TC; ++tb)
#pragma unroll
      for (int s = 0; s < 4; ++s)
        acc[tb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[tb][s], acc[tb], 0, 0, 0);
  };
  auto issue = [&](int64_t group, uint4 (&raw)[U][TC]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t row0 = (group * U + u) * 16 + 4 * kq;
#pragma unroll
      for (int tb = 0; tb < TC; ++tb) {
        raw[u][tb] = uint4{0u, 0u, 0u, 0u};
        if (tb < TMr) {                      // a tile of Y
          const int col = tb * 16 + c16;
          if (col < m) raw[u][tb] = cross_raw<ElemF32, false>(Yb, (int64_t)col * ldy, 1, row0);
        } else {                             // a tile of G
          const int col = (tb - TMr) * 16 + c16;
          if (col < p) raw[u][tb] = cross_raw<E, ROWS>(G, (int64_t)col * g_cs, g_rs, row0);
        }
      }
    }
  };
  auto consume = [&](uint4 (&raw)[U][TC]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      double b[TC][4];
#pragma unroll
      for (int tb = 0; tb < TC; ++tb) {
        if (tb < TMr) cross_decode<ElemF32, false>(raw[u][tb], b[tb]);
        else cross_decode<E, ROWS>(raw[u][tb], b[tb]);
      }
      multiply(b);
    }
  };

  // groups of U whole chunks, two stages in flight
  const int64_t ngroups = (n / 16) / U;
  uint4 cur[U][TC], nxt[U][TC];
  int64_t g = wid;
  if (g < ngroups) issue(g, cur);
  while (g < ngroups) {
    const int64_t gn = g + nw;
    if (gn < ngroups) issue(gn, nxt);
    consume(cur);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int tb = 0; tb < TC; ++tb) cur[u][tb] = nxt[u][tb];
    g = gn;
  }
  // what is left: fewer than U whole chunks and the ragged one, one wavefront each, with
  // the careful loads
  const int64_t nchunks = (n + 15) / 16;
  const int64_t ch = ngroups * U + wid;
  if (ch < nchunks) {
    const int64_t row0 = ch * 16 + 4 * kq;
    double b[TC][4];
#pragma unroll
    for (int tb = 0; tb < TC; ++tb) {
      if (tb < TMr) {
        const int col = tb * 16 + c16;
        load_rows4<ElemF32>(Yb, (int64_t)col * ldy, 1, row0, n, col < m, b[tb]);
      } else {
        const int col = (tb - TMr) * 16 + c16;
        load_rows4<E>(G, (int64_t)col * g_cs, g_rs, row0, n, col < p, b[tb]);
      }
    }
    multiply(b);
  }
  // the wavefronts add up in wave order; one partial tile per workgroup and result tile
#pragma unroll
  for (int tb = 0; tb < TC; ++tb) {
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave * 256 + r * 64 + lane] = acc[tb][r];
    __syncthreads();
    double* dst = partials + (((int64_t)blockIdx.x * gridDim.y + ta) * TC + tb) * 256;
    for (int e = threadIdx.x; e < 256; e += 64 * NWV) {
      double tot = 0.0;
#pragma unroll
      for (int w = 0; w < NWV; ++w) tot += red[w * 256 + e];
      dst[e] = tot;
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------------------------------
// K3: the p x p solver, one workgroup, matrices in LDS.

__global__ __launch_bounds__(FA_IRLS_THREADS) void fa_irls_kernel(const double* __restrict__ Kg,
                                                                  fa_irls_args ar, double* cg,
                                                                  fa_info* info, double* gws,
                                                                  int big_in_global,
                                                                  fa_resume* rs, int retry_only) {
  // as the stand-by of the matrix-core solver: nothing to do unless that one gave up
  if (retry_only && info->status != FA_ST_RETRY) return;
  extern __shared__ __attribute__((aligned(16))) double dyn[];
  const int p = ar.p;
  const int ld = p | 1;
  fa_irls_mem sm;
  sm.ld = ld;
  double* q = dyn;
  const size_t msz = (size_t)p * ld;
  sm.R = q; q += msz;
  sm.Ut = q; q += msz;
  sm.CM = q; q += msz;
  sm.T = q; q += msz;
  if (big_in_global) {
    sm.D2inv = gws;
    sm.Vt = gws + msz;
  } else {
    sm.D2inv = q; q += msz;
    sm.Vt = q; q += msz;
  }
  sm.s = q; q += FA_P_MAX;
  sm.dinv = q; q += FA_P_MAX;
  sm.w = q; q += FA_P_MAX;
  sm.rho = q; q += FA_P_MAX;
  sm.v = q; q += FA_P_MAX;
  sm.lam0 = q; q += FA_P_MAX;
  sm.mu = q; q += FA_P_MAX;
  sm.beta = q; q += FA_P_MAX;
  sm.ginv = q; q += FA_P_MAX;
  sm.ctop = q; q += FA_P_MAX;
  sm.cbot = q; q += FA_P_MAX;
  sm.rot_c = q; q += FA_P_MAX / 2;
  sm.rot_s = q; q += FA_P_MAX / 2;
  sm.red = q; q += FA_IRLS_THREADS;
  int* qi = reinterpret_cast<int*>(q);
  sm.rot_p = qi; qi += FA_P_MAX / 2;
  sm.rot_q = qi; qi += FA_P_MAX / 2;
  sm.pos = qi; qi += FA_P_MAX;
  sm.order = qi; qi += FA_P_MAX;
  sm.gfirst = qi; qi += FA_P_MAX;
  sm.gcnt = qi; qi += FA_P_MAX;
  sm.flag = qi; qi += 8;
  fa_irls_solve(Kg, ar, sm, cg, info, rs);
}

size_t fa_irls_lds_bytes(int p, int* big_in_global) {
  const size_t msz = (size_t)p * (p | 1) * sizeof(double);
  const size_t small = (11 * FA_P_MAX + FA_P_MAX + FA_IRLS_THREADS) * sizeof(double) +
                       (5 * FA_P_MAX + 8) * sizeof(int);
  size_t need = 6 * msz + small;
  *big_in_global = 0;
  if (need > 60 * 1024) {   // keep the common sizes under the default dynamic-LDS limit
    need = 4 * msz + small;
    *big_in_global = 1;
  }
  return need;
}

// ------------------------------------------------------------------------------------------
// launchers (host).  Shapes are validated by the callers in fa_api.hip.
template <int T, int CPL, typename E, int WAVES, int ST, bool LAST = false>
static hipError_t launch_gram_t(const void* G, int64_t ldg, int p, int64_t n, int max_blocks,
                                double* partials, int* nparts, hipStream_t st,
                                const fa_ktime* tm, const int* gate, const fa_gram_cols& cols) {
  static_assert(WAVES <= FA_GRAM_WAVES_PER_CU, "partials buffer is sized for this many");
  constexpr int R = (64 / CPL) * E::EPL;
  constexpr int CS = R * E::SIZE + 16;
  constexpr size_t tile_bytes =
      fa_mem(ST) == FA_MEM_ROWS ? fa_rows_tile_bytes(T, E::SIZE, R) : (size_t)T * 16 * CS;
  static_assert(WAVES * tile_bytes <= 160 * 1024, "LDS tiles of one workgroup must fit a CU");
  // more than half of the CU's 160 KiB, so that no second workgroup fits beside this one
  const size_t lds_bytes = WAVES * tile_bytes > 84 * 1024 ? WAVES * tile_bytes : 84 * 1024;
  const int64_t ntiles = (n + R - 1) / R;
  int64_t wgs = (ntiles + WAVES - 1) / WAVES;
  if (wgs > max_blocks) wgs = max_blocks;
  *nparts = (int)wgs;
  FA_LAUNCH(tm, (fa_gram_kernel<T, CPL, E, WAVES, ST, LAST>), dim3((unsigned)wgs),
            dim3(64 * WAVES), lds_bytes, st, (const unsigned char*)G, ldg, p, n, ntiles,
            partials, gate, cols);
  return hipGetLastError();
}

// interleaved storage, p <= 16: rows from which on the elements are scattered (see ROWS)
#define FA_SCATTER_MIN_ROWS ((int64_t)1 << 22)

// the tiling of each width class: T -> (columns per load, wavefronts per CU)
#define FA_GRAM_TILINGS(X) \
  X(1, FA_GRAM_CPL1, FA_GRAM_W1) X(2, FA_GRAM_CPL2, FA_GRAM_W2) X(3, 4, 8) X(4, FA_GRAM_CPL4, FA_GRAM_W4)

template <typename E, bool ROWS>
static hipError_t launch_gram_e(const void* G, int64_t ldg, int p, int64_t n, int max_blocks,
                                double* partials, int* nparts, hipStream_t st_,
                                const fa_ktime* tm, const int* gate,
                                const fa_gram_cols& cols = fa_gram_cols{}, bool last = false) {
  constexpr int BASE = ROWS ? FA_MEM_ROWS : FA_MEM_WORKER;
  switch ((p + 15) / 16) {
#define FA_L(t, cpl, w, st, l)                                                                     \
  return launch_gram_t<t, cpl, E, w, st, l>(G, ldg, p, n, max_blocks, partials, nparts, st_, tm, gate, cols)
#define FA_X(t, cpl, w)                                                                            \
    case t:                                                                                        \
      if constexpr (t == 1) {                                                                      \
        if (ROWS && n >= FA_SCATTER_MIN_ROWS) {                                                    \
          if (p <= 8) FA_L(t, cpl, w, FA_MEM_SCATTER + FA_NARROW_ALL8, false);                      \
          FA_L(t, cpl, w, FA_MEM_SCATTER, false);                                                  \
        }                                                                                          \
        if (p <= 8) FA_L(t, cpl, w, BASE + FA_NARROW_ALL8, false);                                  \
      } else {                                                                                     \
        if constexpr (!ROWS)                                                                       \
          if (last) FA_L(t, cpl, w, BASE, true);                                                   \
        if (p <= 16 * t - 12) FA_L(t, cpl, w, BASE + FA_NARROW_LAST4, false);                       \
        if (p <= 16 * t - 8) FA_L(t, cpl, w, BASE + FA_NARROW_LAST8, false);                        \
      }                                                                                            \
      FA_L(t, cpl, w, BASE, false);
    FA_GRAM_TILINGS(FA_X)
#undef FA_X
#undef FA_L
  }
  return hipErrorInvalidValue;
}

template <typename E, bool ROWS>
static hipError_t prepare_gram_e() {
  constexpr int BASE = ROWS ? FA_MEM_ROWS : FA_MEM_WORKER;
  hipError_t e = hipSuccess;
#define FA_SET(...)                                                                               \
  if (e == hipSuccess)                                                                           \
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(fa_gram_kernel<__VA_ARGS__>),          \
                            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
#define FA_X(t, cpl, w)                                                                          \
  FA_SET(t, cpl, E, w, BASE, false)                                                              \
  if constexpr (!ROWS && t > 1) { FA_SET(t, cpl, E, w, BASE, true) }                              \
  if constexpr (t == 1) { FA_SET(t, cpl, E, w, BASE + FA_NARROW_ALL8, false) }                    \
  if constexpr (ROWS && t == 1) { FA_SET(t, cpl, E, w, FA_MEM_SCATTER, false) }                   \
  if constexpr (ROWS && t == 1) { FA_SET(t, cpl, E, w, FA_MEM_SCATTER + FA_NARROW_ALL8, false) }  \
  if constexpr (t > 1) { FA_SET(t, cpl, E, w, BASE + FA_NARROW_LAST4, false) }                    \
  if constexpr (t > 1) { FA_SET(t, cpl, E, w, BASE + FA_NARROW_LAST8, false) }
  FA_GRAM_TILINGS(FA_X)
#undef FA_X
#undef FA_SET
  return e;
}

bool fa_gram_takes_matrix_core(int p, int64_t n, int dtype, int layout, int gram_mode) {
  const bool want_lp = gram_mode == FA_GRAM_BF16_MATRIX ||
                       (gram_mode == FA_GRAM_AUTO && n >= FA_GRAM_AUTO_MIN_ROWS);
  return want_lp && layout == FA_WORKER_MAJOR && fa_gram_lp_applies(p, dtype);
}

hipError_t fa_launch_gram_partials(const void* G, int64_t ldg, int p, int64_t n, int dtype,
                                   int layout, int gram_mode, int max_blocks, double* partials,
                                   int* nparts, hipStream_t st, const fa_ktime* tm,
                                   const int* gate, int* clear) {
  if (fa_gram_takes_matrix_core(p, n, dtype, layout, gram_mode))
    return fa_launch_gram_lp_partials(G, ldg, p, n, dtype, max_blocks, partials, nparts, clear, st, tm);
  const bool rows = layout == FA_ROW_MAJOR;
  if (dtype == FA_F32)
    return rows ? launch_gram_e<ElemF32, true>(G, ldg, p, n, max_blocks, partials, nparts, st, tm, gate)
                : launch_gram_e<ElemF32, false>(G, ldg, p, n, max_blocks, partials, nparts, st, tm, gate);
  return rows ? launch_gram_e<ElemBF16, true>(G, ldg, p, n, max_blocks, partials, nparts, st, tm, gate)
              : launch_gram_e<ElemBF16, false>(G, ldg, p, n, max_blocks, partials, nparts, st, tm, gate);
}

hipError_t fa_launch_gram_reduce(const double* partials, int nparts, int p, double* Kd,
                                 const double* colscale, hipStream_t st, const fa_ktime* tm,
                                 const int* gate, int* nonfinite) {
  const int T = (p + 15) / 16;
  const int NTP = T * (T + 1) / 2;
  FA_LAUNCH(tm, fa_gram_reduce_kernel, dim3(NTP * 4), dim3(1024), 0, st, partials, nparts, T, p,
            Kd, 0, 0, colscale, gate, 0, p, fa_gram_cols{}, nonfinite);
  return hipGetLastError();
}

hipError_t fa_launch_gram_add(const void* G, int64_t ldg, int p, int64_t n, int dtype,
                              uint64_t first, uint64_t then, int max_blocks, double* partials,
                              double* Kd, hipStream_t st) {
  fa_gram_cols cols{};
  cols.add = 1;
  int ncols = 0;
  for (const uint64_t set : {first, then})
    for (int j = 0; j < p; ++j)
      if ((set >> j) & 1u) cols.idx[ncols++] = (uint8_t)j;
  cols.listed = ncols < p;
  const int T = (ncols + 15) / 16;
  const bool last = first != 0;
  int nparts = 0;
  hipError_t e = dtype == FA_F32
      ? launch_gram_e<ElemF32, false>(G, ldg, ncols, n, max_blocks, partials, &nparts, st, nullptr,
                                      nullptr, cols, last)
      : launch_gram_e<ElemBF16, false>(G, ldg, ncols, n, max_blocks, partials, &nparts, st, nullptr,
                                       nullptr, cols, last);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fa_gram_reduce_kernel, dim3((last ? T : T * (T + 1) / 2) * 4), dim3(1024), 0,
                     st, (const double*)partials, nparts, T, ncols, Kd, 0, 0,
                     (const double*)nullptr, (const int*)nullptr, last ? 1 : 0, p, cols, (int*)nullptr);
  return hipGetLastError();
}

// K1 + K2: K = G^T G into Kd.  Where the pass runs on the bf16 matrix core, whose 32-row sums
// are fp32 and overflow for values beyond ~1e18, the fp64 pass stands by behind it: it is
// always enqueued and returns at once unless K came out non-finite (flag_d: one int of device
// scratch, which the first pass clears and its reduction sets; as a kernel of its own that read K 3.4 of 546 us at
// p = 60, 1.2 M rows), so that large finite values - a Byzantine worker may send anything - cost a second
// pass instead of the result.  tm_gram / tm_reduce time the first pass and its reduction.
hipError_t fa_launch_gram(const void* G, int64_t ldg, int p, int64_t n, int dtype, int layout,
                          int gram_mode, int max_blocks, double* partials, double* Kd,
                          int* flag_d, int* nparts, hipStream_t st, const fa_ktime* tm_gram,
                          const fa_ktime* tm_reduce) {
  hipError_t e = fa_launch_gram_partials(G, ldg, p, n, dtype, layout, gram_mode, max_blocks,
                                         partials, nparts, st, tm_gram, nullptr, flag_d);
  if (e != hipSuccess) return e;
  const bool matrix_core = fa_gram_takes_matrix_core(p, n, dtype, layout, gram_mode);
  e = fa_launch_gram_reduce(partials, *nparts, p, Kd, nullptr, st, tm_reduce, nullptr, matrix_core ? flag_d : nullptr);
  if (e != hipSuccess || !matrix_core) return e;
  int np2 = 0;
  e = fa_launch_gram_partials(G, ldg, p, n, dtype, layout, FA_GRAM_FP64, max_blocks, partials, &np2,
                              st, nullptr, flag_d);
  if (e != hipSuccess) return e;
  return fa_launch_gram_reduce(partials, np2, p, Kd, nullptr, st, nullptr, flag_d);
}

hipError_t fa_launch_proj_reduce(const double* partials, int nparts, int p, int m, double* Td,
                                 hipStream_t st, const fa_ktime* tm) {
  const int T = (p + 15) / 16, TM = (m + 15) / 16;
  FA_LAUNCH(tm, fa_gram_reduce_kernel, dim3(T * TM * 4), dim3(1024), 0, st, partials, nparts, T,
            p, Td, TM, m, (const double*)nullptr, (const int*)nullptr, 0, p, fa_gram_cols{}, (int*)nullptr);
  return hipGetLastError();
}

// W = Y^T [Y | G], m x (16 ceil(m/16) + p) row-major into Wd: the partial tiles of at most
// max_parts row stripes go to `partials` (max_parts * tiles * 256 doubles), then K2 adds them.
hipError_t fa_launch_cross(const float* Y, int64_t ldy, int m, const void* G, int64_t ldg, int p,
                           int64_t n, int dtype, int layout, int max_parts, double* partials,
                           double* Wd, hipStream_t st) {
  const int TMr = (m + 15) / 16, TC = TMr + (p + 15) / 16;
  const int64_t g_rs = layout == FA_ROW_MAJOR ? ldg : 1, g_cs = layout == FA_ROW_MAJOR ? 1 : ldg;
  // two workgroups of eight wavefronts per compute unit of a 256-unit chip, at most
  int64_t stripes = (n + 8 * 16 - 1) / (8 * 16);             // a chunk per wavefront at least
  if (stripes > 512 / TMr) stripes = 512 / TMr;
  if (stripes > max_parts) stripes = max_parts;
  if (stripes < 1) stripes = 1;
  const dim3 grid((unsigned)stripes, (unsigned)TMr);
  const bool rows = layout == FA_ROW_MAJOR;
  switch (TC) {
#define FA_Y(E, tc, R)                                                                     \
  hipLaunchKernelGGL((fa_cross_kernel<E, tc, R>), grid, dim3(512), 0, st, Y, ldy, m,       \
                     (const unsigned char*)G, g_rs, g_cs, p, n, TMr, partials)
#define FA_X(tc)                                                       \
    case tc:                                                           \
      if (dtype == FA_F32) {                                           \
        if (rows) FA_Y(ElemF32, tc, true); else FA_Y(ElemF32, tc, false);   \
      } else {                                                         \
        if (rows) FA_Y(ElemBF16, tc, true); else FA_Y(ElemBF16, tc, false); \
      }                                                                \
      break;
    FA_X(2) FA_X(3) FA_X(4) FA_X(5) FA_X(6) FA_X(7) FA_X(8)
#undef FA_X
#undef FA_Y
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int ncols = 16 * TMr + p;
  hipLaunchKernelGGL(fa_gram_reduce_kernel, dim3(TMr * TC * 4), dim3(1024), 0, st,
                     (const double*)partials, (int)stripes, TMr, m, Wd, TC, ncols,
                     (const double*)nullptr, (const int*)nullptr, 0, m, fa_gram_cols{}, (int*)nullptr);
  return hipGetLastError();
}

template <int T, int TM, int CPL, typename E, int WAVES>
static hipError_t launch_proj_t(const void* G, int64_t ldg, int p, int m, int64_t n,
                                int max_blocks, const double* Acoef, double* partials,
                                int* nparts, hipStream_t st, const fa_ktime* tm) {
  constexpr int R = (64 / CPL) * E::EPL;
  constexpr int CS = R * E::SIZE + 16;
  constexpr size_t a_bytes = (size_t)T * 16 * TM * 16 * sizeof(double);
  constexpr size_t tile_bytes = (size_t)T * 16 * CS;
  constexpr size_t need = a_bytes + (WAVES * tile_bytes > WAVES * 2048u ? WAVES * tile_bytes
                                                                        : WAVES * 2048u);
  static_assert(need <= 160 * 1024, "LDS of one workgroup must fit a CU");
  const size_t lds_bytes = need > 84 * 1024 ? need : 84 * 1024;   // one workgroup per CU
  const int64_t ntiles = (n + R - 1) / R;
  int64_t wgs = (ntiles + WAVES - 1) / WAVES;
  if (wgs > max_blocks) wgs = max_blocks;
  *nparts = (int)wgs;
  FA_LAUNCH(tm, (fa_proj_kernel<T, TM, CPL, E, WAVES>), dim3((unsigned)wgs), dim3(64 * WAVES),
            lds_bytes, st, (const unsigned char*)G, ldg, p, m, n, ntiles, Acoef, partials);
  return hipGetLastError();
}

// (T, TM) -> (columns per load, wavefronts per CU); the larger tilings run four wavefronts per
// CU: they need more than 256 registers a lane
#define FA_PROJ_TILINGS(X)                                                        \
  X(1, 1, 4, 12) X(2, 1, 4, 8) X(2, 2, 4, 8) X(3, 1, 4, 8) X(3, 2, 4, 8) X(3, 3, 4, 4) \
  X(4, 1, 8, 8) X(4, 2, 8, 4) X(4, 3, 8, 4) X(4, 4, 8, 4)

template <typename E>
static hipError_t launch_proj_e(const void* G, int64_t ldg, int p, int m, int64_t n,
                                int max_blocks, const double* Acoef, double* partials,
                                int* nparts, hipStream_t st, const fa_ktime* tm) {
  const int T = (p + 15) / 16, TM = (m + 15) / 16;
#define FA_PROJ_CASE(t, tmm, cpl, w)                                                            \
  if (T == t && TM == tmm)                                                                      \
    return launch_proj_t<t, tmm, cpl, E, w>(G, ldg, p, m, n, max_blocks, Acoef, partials, nparts, \
                                            st, tm);
  FA_PROJ_TILINGS(FA_PROJ_CASE)
#undef FA_PROJ_CASE
  return hipErrorInvalidValue;
}

template <typename E>
static hipError_t prepare_proj_e() {
  hipError_t e = hipSuccess;
#define FA_PROJ_CASE(t, tmm, cpl, w)                                                            \
  if (e == hipSuccess)                                                                          \
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(fa_proj_kernel<t, tmm, cpl, E, w>),   \
                            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  FA_PROJ_TILINGS(FA_PROJ_CASE)
#undef FA_PROJ_CASE
  return e;
}

hipError_t fa_launch_proj_partials(const void* G, int64_t ldg, int p, int m, int64_t n, int dtype,
                                   int max_blocks, const double* Acoef, double* partials,
                                   int* nparts, hipStream_t st, const fa_ktime* tm) {
  if (dtype == FA_F32)
    return launch_proj_e<ElemF32>(G, ldg, p, m, n, max_blocks, Acoef, partials, nparts, st, tm);
  return launch_proj_e<ElemBF16>(G, ldg, p, m, n, max_blocks, Acoef, partials, nparts, st, tm);
}

hipError_t fa_launch_restream_weights(const fa_info* info_d, const double* Pd, int p, int m,
                                      double lambda, double delta, double pair_tol,
                                      double exponent_a, fa_resume* rs, hipStream_t st) {
  const double coef = (lambda > 0.0 && p > 1) ? lambda / (double)(p - 1) : 0.0;
  hipLaunchKernelGGL(fa_restream_weights_kernel, dim3(1), dim3(256), 0, st, info_d, Pd, p, m, coef,
                     delta, pair_tol, 1.0 / exponent_a, rs);
  return hipGetLastError();
}

hipError_t fa_launch_irls(const double* Kd, int p, int m, double lambda, int iters, double tol,
                          double delta, double rank_tol, double pair_tol, double exponent_a,
                          double* cd,
                          fa_info* info_d, double* gws, int solver, int spin_budget,
                          fa_resume* rs, hipStream_t st, const fa_ktime* tm) {
  if (p <= 16 && solver != 2)
    return fa_launch_irls16(Kd, p, m, lambda, iters, tol, delta, exponent_a, rank_tol, pair_tol, cd,
                            info_d,
                            gws + FA_GWS_MLAST_OFF, solver == 0 ? 1 : 0, rs, st, tm);
  int retry_only = 0;
  fa_ktime first = {nullptr, nullptr}, second = {nullptr, nullptr};
  if (p > 16 && solver == 0) {
    // timing, if asked for, spans both launches: begin of the first, end of the second
    if (tm) { first.start = tm->start; second.stop = tm->stop; }
    hipError_t e = fa_launch_irls64(Kd, p, 0, nullptr, m, lambda, iters, tol, delta, exponent_a,
                                    rank_tol, pair_tol, cd,
                                    info_d, gws + FA_GWS_GENERIC, gws + FA_GWS_MLAST_OFF,
                                    spin_budget, rs, st, tm ? &first : nullptr);
    if (e != hipSuccess) return e;
    retry_only = 1;   // the Jacobi kernel below runs only if the one above gave up
    tm = tm ? &second : nullptr;
  }
  fa_irls_args ar;
  ar.p = p; ar.m = m; ar.iters = iters; ar.lambda = lambda; ar.tol = tol;
  ar.delta = delta; ar.rank_tol = rank_tol; ar.pair_tol = pair_tol;
  ar.expo = 1.0 / exponent_a;
  ar.nworkers = 0; ar.sizes = nullptr;
  int big = 0;
  const size_t lds = fa_irls_lds_bytes(p, &big);
  FA_LAUNCH(tm, fa_irls_kernel, dim3(1), dim3(FA_IRLS_THREADS), lds, st, Kd, ar, cd, info_d, gws,
            big, rs, retry_only);
  return hipGetLastError();
}

// The same for workers that send several gradients: q columns in nworkers blocks of
// sizes_d[i] consecutive columns (device memory).  solver 0: the matrix-core purification
// kernel, with the any-p kernel behind it as stand-by; otherwise the any-p kernel alone.
hipError_t fa_launch_irls_grouped(const double* Kd, int q, int nworkers, const int* sizes_d, int m,
                                  double lambda, int iters, double tol, double delta,
                                  double rank_tol, double pair_tol, double exponent_a, double* cd,
                                  fa_info* info_d, double* gws, int solver, int spin_budget,
                                  hipStream_t st) {
  int retry_only = 0;
  if (solver == 0) {
    hipError_t e = fa_launch_irls64(Kd, q, nworkers, sizes_d, m, lambda, iters, tol, delta,
                                    exponent_a, rank_tol, pair_tol, cd, info_d,
                                    gws + FA_GWS_GENERIC, gws + FA_GWS_MLAST_OFF, spin_budget,
                                    nullptr, st, nullptr);
    if (e != hipSuccess) return e;
    retry_only = 1;   // the Jacobi kernel below runs only if the one above gave up
  }
  fa_irls_args ar;
  ar.p = q; ar.m = m; ar.iters = iters; ar.lambda = lambda; ar.tol = tol;
  ar.delta = delta; ar.rank_tol = rank_tol; ar.pair_tol = pair_tol;
  ar.expo = 1.0 / exponent_a;
  ar.nworkers = nworkers; ar.sizes = sizes_d;
  int big = 0;
  const size_t lds = fa_irls_lds_bytes(q, &big);
  hipLaunchKernelGGL(fa_irls_kernel, dim3(1), dim3(FA_IRLS_THREADS), lds, st, Kd, ar, cd, info_d,
                     gws, big, (fa_resume*)nullptr, retry_only);
  return hipGetLastError();
}

// Eigenvalues of the last weighted-PCA matrix (N x N row-major, then rank and m, left by the
// purification paths) by the Jacobi routine above; writes the relative gap between
// eigenvalues m and m+1.
__global__ __launch_bounds__(256) void fa_gap_kernel(const double* __restrict__ mlast, int N,
                                                     fa_info* __restrict__ info) {
  extern __shared__ __attribute__((aligned(16))) double gl[];
  const int ld = N + 1;
  double* A = gl;                       // N x ld
  double* vals = A + N * ld;            // 64
  double* rc = vals + 64;               // 32
  double* rsn = rc + 32;                // 32
  double* red = rsn + 32;               // 256
  int* rp = reinterpret_cast<int*>(red + 256);
  int* rq = rp + 32;
  int* pos = rq + 32;
  int* order = pos + 64;
  int* flag = order + 64;
  fa_irls_mem sm;
  sm.ld = ld;
  sm.rot_c = rc; sm.rot_s = rsn; sm.rot_p = rp; sm.rot_q = rq; sm.red = red; sm.flag = flag;
  sm.pos = pos; sm.order = order;
  const int r = (int)mlast[N * N], m = (int)mlast[N * N + 1];
  for (int idx = threadIdx.x; idx < N * N; idx += 256) A[(idx / N) * ld + (idx % N)] = mlast[idx];
  if (threadIdx.x == 0) flag[4] = 0;
  __syncthreads();
  if (r < 1 || r > N) return;
  fa_jacobi(A, r, (double*)0, 0, (double*)0, 0, sm, 60);
  FA_FOR(a, r) vals[a] = A[a * ld + a];
  FA_SYNC();
  fa_rank_desc(vals, r, pos, order);
  if (threadIdx.x == 0) {
    double gap = __builtin_inf();
    if (m < r) gap = (vals[order[m - 1]] - vals[order[m]]) / vals[order[0]];
    info->eigengap = gap;
  }
}

hipError_t fa_launch_gap(const double* mlast, int N, fa_info* info_d, hipStream_t st) {
  const size_t lds = ((size_t)N * (N + 1) + 64 + 32 + 32 + 256) * sizeof(double) +
                     (32 + 32 + 64 + 64 + 8) * sizeof(int);
  hipLaunchKernelGGL(fa_gap_kernel, dim3(1), dim3(256), lds, st, mlast, N, info_d);
  return hipGetLastError();
}

// narrow: at most sixteen columns.  (bf16 never has fewer than ten, so one tile more fits in place of a second end.)
template <typename E, int RT, int LT, int ENDS, int WGS>
static hipError_t launch_held_t(const void* G, int64_t ldg, int p, int64_t n, const double* c,
                                int cstride, const double* skip, float* out, int cus, hipStream_t st,
                                const fa_ktime* tm) {
  FA_LAUNCH(tm, (fa_combine_held_kernel<E, RT, LT, ENDS, WGS>), dim3((unsigned)cus), dim3(64 * FA_HELD_WAVES),
            (fa_held_lds_bytes<E, RT, LT, ENDS>()), st, (const unsigned char*)G, ldg, p, n, c, cstride, skip, out);
  return hipGetLastError();
}
#define FA_HELD_NARROW_F32 ElemF32, 30, 26, 2, 2
#define FA_HELD_NARROW_BF16 ElemBF16, 15, 13, 1, 2
#define FA_HELD_WIDE_F32 ElemF32, 66, 37, 1, 1
#define FA_HELD_WIDE_BF16 ElemBF16, 33, 18, 1, 1
template <typename E, int RT, int LT, int ENDS, int WGS>
static hipError_t prepare_held_t() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(fa_combine_held_kernel<E, RT, LT, ENDS, WGS>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)fa_held_lds_bytes<E, RT, LT, ENDS>());
}

template <typename E>
static hipError_t prepare_e(int layout) {
  if (layout != FA_ROW_MAJOR) {
    hipError_t e = prepare_gram_e<E, false>();
    if constexpr (E::SIZE == 4) {
      if (e == hipSuccess) e = prepare_held_t<FA_HELD_NARROW_F32>();
      if (e == hipSuccess) e = prepare_held_t<FA_HELD_WIDE_F32>();
    } else {
      if (e == hipSuccess) e = prepare_held_t<FA_HELD_NARROW_BF16>();
      if (e == hipSuccess) e = prepare_held_t<FA_HELD_WIDE_BF16>();
    }
    return e == hipSuccess ? prepare_proj_e<E>() : e;      // (the re-streaming schedule is worker-major only)
  }
  hipError_t e = prepare_gram_e<E, true>();
  if constexpr (E::SIZE == 4) {
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(fa_combine_rows_tiles_kernel<E, 16, true>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, 4 * 16 * 1088);
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(fa_combine_rows_tiles_kernel<E, 16, false>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, 4 * 16 * 1088);
  }
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(fa_combine_rows_kernel<E, FA_ROWS_MULTI>),
                            hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)fa_rows_lds_bytes(FA_P_MAX, 4));
  return e;
}

hipError_t fa_kernels_prepare(int dtype, int layout) {
  // the single-workgroup Jacobi solver's large dynamic LDS (p = 64 needs ~140 KiB)
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fa_irls_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e != hipSuccess) return e;
  // the streaming kernels that claim a whole compute unit's LDS, of this storage only: an attribute takes a few
  // microseconds of every fa_create
  return dtype == FA_F32 ? prepare_e<ElemF32>(layout) : prepare_e<ElemBF16>(layout);
}

template <typename E>
static hipError_t launch_combine_rows(const void* G, int ldr, int p, int64_t n, const double* c, int cstride,
                                      float* out, int cus, hipStream_t st, const fa_ktime* tm) {
  const int need = (ldr * E::SIZE + 15) / 16;
  const bool whole = ldr * E::SIZE % 16 == 0;
  const int64_t ntiles = (n + 63) / 64;
#define FA_X(np)                                                                                     \
  if (need <= np) {                                                                                  \
    int64_t blocks = (int64_t)cus * fa_rows_wgs(E::SIZE, np, whole);                                  \
    if (E::SIZE == 2 && np > 3 && np < 6 && ntiles > blocks * 4 * fa_rows_held(2, np, whole))        \
      blocks = (int64_t)cus * 3;                                                                     \
    if (blocks > (ntiles + 3) / 4) blocks = (ntiles + 3) / 4;                                        \
    if (whole)                                                                                       \
      FA_LAUNCH(tm, (fa_combine_rows_tiles_kernel<E, np, true>), dim3((unsigned)blocks), dim3(256),  \
                4 * np * 1088, st, (const unsigned char*)G, ldr, p, n, c, cstride, out);             \
    else                                                                                             \
      FA_LAUNCH(tm, (fa_combine_rows_tiles_kernel<E, np, false>), dim3((unsigned)blocks), dim3(256), \
                4 * np * 1088, st, (const unsigned char*)G, ldr, p, n, c, cstride, out);             \
    return hipGetLastError();                                                                        \
  }
  FA_X(1) FA_X(2) FA_X(3) FA_X(4) FA_X(5) FA_X(6) FA_X(7) FA_X(8)
  if constexpr (E::SIZE == 4) { FA_X(10) FA_X(12) FA_X(14) FA_X(16) }
#undef FA_X
  return hipErrorInvalidValue;
}

// Whether fa_combine_held_kernel takes an aggregate pass that reads `cols` worker-major columns: from ten columns on where a
// wavefront has ten whole tiles, fp32 with five to nine where it has sixteen.  Below, which of the two is ahead changes with the width,
// the type and how full the last round of tiles is.  us, the kernel for small sets / this one, sets of so many tiles a wavefront (262 144
// rows each for fp32, 524 288 for bf16) that do not end on a whole piece: fp32 p = 12 4.03 14.1 / 13.7, 10.03 26.2 / 24.5, 16.2 39.4 /
// 36.2; p = 15 4.03 15.6 / 15.5, 7.03 22.9 / 22.7, 10.03 30.3 / 28.6, 13.03 38.3 / 35.8; p = 64 7.03 88.7 / 83.3, 10.03 123 / 108, 16.03 192 /
// 168; bf16 p = 16 7.03 25.9 / 26.9, 9.03 31.7 / 32.4, 10.03 34.7 / 34.2, 13.03 43.4 / 41.7; p = 32 7.03 48.5 / 48.2, 10.03 66.1 / 61.3; that end on a
// tile: fp32 p = 15 4 13.4 / 13.6, 10 28.4 / 26.8; p = 64 16 177 / 158.  Few columns leave a wavefront little time for a tile: fp32 p = 6
// 12.03 16.6 / 16.7, 16.03 21.4 / 21.1; p = 7 16.03 24.1 / 23.5, 32.03 44.6 / 41.5; bf16 p = 7 32.03 50.2 / 51.4, p = 8 16.03 31.0 / 30.7, 64.03
// 113 / 108.
static bool fa_combine_held_applies(int cols, int64_t n, int dtype, int cus) {
  const int64_t tiles = n / (64 * (dtype == FA_F32 ? 4 : 8)) / ((int64_t)FA_HELD_WAVES * cus);   // per wavefront
  if (cols >= 10) return tiles >= 10;
  return dtype == FA_F32 && cols >= 5 && tiles >= 16;
}

hipError_t fa_launch_combine(const void* G, int64_t ldg, int p, int64_t n, int dtype, int layout,
                             const double* c, int cstride, float* out, int cus,
                             hipStream_t st, const fa_ktime* tm, const double* skip, int nonzero) {
  if (layout == FA_ROW_MAJOR)
    return dtype == FA_F32 ? launch_combine_rows<ElemF32>(G, (int)ldg, p, n, c, cstride, out, cus, st, tm)
                           : launch_combine_rows<ElemBF16>(G, (int)ldg, p, n, c, cstride, out, cus, st, tm);
  const int epl = dtype == FA_F32 ? 4 : 8;
  if (fa_combine_held_applies(skip ? nonzero : p, n, dtype, cus)) {
    const bool wide = (skip ? nonzero : p) > 16;
    if (dtype == FA_F32)
      return wide ? launch_held_t<FA_HELD_WIDE_F32>(G, ldg, p, n, c, cstride, skip, out, cus, st, tm)
                  : launch_held_t<FA_HELD_NARROW_F32>(G, ldg, p, n, c, cstride, skip, out, cus, st, tm);
    return wide ? launch_held_t<FA_HELD_WIDE_BF16>(G, ldg, p, n, c, cstride, skip, out, cus, st, tm)
                : launch_held_t<FA_HELD_NARROW_BF16>(G, ldg, p, n, c, cstride, skip, out, cus, st, tm);
  }
  const int64_t ngroups = (n + epl - 1) / epl;
  int64_t blocks = (ngroups + 255) / 256;
  if (blocks > (1 << 20)) blocks = 1 << 20;
#define FA_X(E, L)                                                                                 \
  FA_LAUNCH(tm, (fa_combine_kernel<E, L>), dim3((unsigned)blocks), dim3(256), 0, st,               \
            (const unsigned char*)G, ldg, p, n, c, cstride, skip, out)
  if (dtype == FA_F32) {
    if (skip) FA_X(ElemF32, true);
    else FA_X(ElemF32, false);
  } else {
    if (skip) FA_X(ElemBF16, true);
    else FA_X(ElemBF16, false);
  }
#undef FA_X
  return hipGetLastError();
}
