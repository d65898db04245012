// Kernel templates; included by the per-configuration instantiation units.
#pragma once
// Fused batched interior-point kernels for gfx950 (MI355X).
//
// One workgroup owns one QP for its whole solve: problem data is read from
// HBM (it stays L2/MALL resident across iterations), the iterate, residuals
// and directions live in LDS, and the bordered KKT factor lives in LDS when
// it fits (else in a per-QP global workspace).  No host synchronisation
// happens inside a solve; each QP exits its Newton loop on its own.
//
// Method (paper section 4): implicit complementarity with the softplus
// retraction b_kappa (eq. softplus, appendix C).  Each Newton step solves the
// reduced symmetric system of eq. implicit_partially_condensed
//
//     [ Q - G'G   G'      A' ] [dx]     [ r_t - G'(r_i + r_z - r_s) ]
//     [ G        -B(-v)   0  ] [dv] = - [ r_i - r_s - c r_kappa     ]
//     [ A         0       0  ] [dy]     [ r_e                       ]
//
// The paper only says the matrix is symmetric and admits LDL'; it is
// indefinite, so it is factored here by a sign-split elimination that is
// exact in exact arithmetic and needs no pivoting:
//   * rows with v_i <= 0 (D_i = b'(-v_i) >= 1/2) are eliminated: pivot
//     -D_i, which folds G_i' (E_i/D_i) G_i into the (1,1) block, with
//     E_i/D_i = z_i/s_i in (0, 1];
//   * rows with v_i > 0 are kept as a border with the change of variable
//     du_i = E_i dv_i, giving the diagonal -D_i/E_i = -s_i/z_i in (-1, 0);
//   * the equality rows A are kept as a border with a zero diagonal.
// The result is the quasi-definite matrix
//
//     M = [ H   C' ]    H = Q + G_I' diag(E/D) G_I  (positive definite),
//         [ C  -Dl ]    C = [G_B; A],  Dl = diag(s_B / z_B, 0_p) >= 0,
//
// factored as M = L diag(sg) L' with known signs sg = (+1 x n, -1 x k):
// a Cholesky whose trailing k pivots are negated.  Every multiplier is
// bounded (E, D in (0,1), E/D <= 1 on eliminated rows, D/E < 1 on border
// rows), which is the spectral bound the paper relies on.  When more than
// kb rows have v_i > 0, the kb rows with the largest v are bordered and the
// rest eliminated (their weight z/s is then > 1 but moderate).
//
// The standard (explicit) arm factors the normal matrix Q + G' diag(z/s) G
// bordered by A (eq. explicit_partially_condensed with dz eliminated) with
// the same signed Cholesky, and runs Mehrotra's predictor-corrector.
#include <hip/hip_runtime.h>
#include <float.h>
#include <stdint.h>

#include <type_traits>

#include "qp_internal.h"
#ifdef QPK_PHASE_TIMING
#include "qp_phase.h"
#endif

namespace qpk {
namespace {

#define QPD __device__ __forceinline__
// Attribute of the solver's phases (residuals, partition, assembly,
// factorisation, solves, refinement, ...).  Small systems inline them into
// the kernel: the calls' saved registers and context copies would otherwise
// go through scratch memory.  Large systems keep them as separate functions,
// which bounds register pressure and compile time; the instantiation unit
// chooses by defining QPK_INLINE_PHASES.
#ifdef QPK_INLINE_PHASES
#define QPK_PHASE __device__ __forceinline__
#else
#define QPK_PHASE __device__ __noinline__
#endif

constexpr int kNB = 16;          // panel width of the blocked factorisation
constexpr float kBig = 3.0e38f;

// Explicit address spaces: LDS (3) and global (1).  Helpers that are not
// inlined keep 32-bit LDS addresses and emit ds_* / global_* instructions.
typedef __attribute__((address_space(3))) float lf;
typedef __attribute__((address_space(3))) int li;
typedef __attribute__((address_space(3))) double ldd;
typedef float f4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) f4v lf4;
typedef __attribute__((address_space(1))) float gf;
typedef __attribute__((address_space(1))) f4v gf4;
// LDS pointer type of a residual accumulator (FP32 or FP64).
template <class AT> struct LdsT;
template <> struct LdsT<float> { typedef __attribute__((address_space(3))) float type; };
template <> struct LdsT<double> { typedef __attribute__((address_space(3))) double type; };
template <class F> struct Vec4;
template <> struct Vec4<lf> { typedef lf4 type; };
template <> struct Vec4<gf> { typedef gf4 type; };
template <> struct Vec4<const lf> { typedef const lf4 type; };
template <> struct Vec4<const gf> { typedef const gf4 type; };
typedef float f2v __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(3))) f2v clf2;

// The thread's index and a uniform size, as values the compiler cannot trace
// back.  The Newton loop inlines every phase; known as loop invariants, each
// phase's lane predicates, row addresses and trip counts would be computed
// before the loop and kept (spilled) for all of it: 212 bytes of scratch per
// lane in the solve kernel of 256 threads and 2 rows per lane, 12 with the index
// opaque (4096 solves of n = 50 5.11 -> 4.62 ms, 1024 of n = 100 5.98 -> 5.18).
// Scalar registers spill either way (536 and 593 there), into lanes of vector
// registers.
QPD int tidx() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}
QPD int opaque(int v) {
  asm volatile("" : "+s"(v));
  return v;
}

QPD bool finitef(float a) { return fabsf(a) <= FLT_MAX; }

QPD float readlane(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}


// Values that are the same in every lane.  Non-inlined helpers receive their
// arguments in VGPRs (or read them from the stack), which hides uniformity
// from the compiler; passing them through readfirstlane at entry puts loop
// bounds and base addresses back into SGPRs and keeps branches scalar.
QPD int rfl(int v) { return __builtin_amdgcn_readfirstlane(v); }
QPD float rflf(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }
template <class T>
QPD T *rflp(T *p) {
  if constexpr (sizeof(T *) == 4) {
    return (T *)(uintptr_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)p);
  } else {
    const uint64_t v = (uint64_t)(uintptr_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return (T *)(uintptr_t)(((uint64_t)hi << 32) | lo);
  }
}

// Optional per-phase cycle counters for profiling builds (-DQPK_PHASE_TIMING):
// thread 0 accumulates clock64() deltas per phase in LDS (a workgroup barrier
// at every mark); the kernel writes them to Params::phase.  Compiled out
// otherwise.
#ifdef QPK_PHASE_TIMING
static __shared__ long long qpk_pt[PH_N];
#define QPK_PT(k)                                       \
  do {                                                  \
    __syncthreads();                                    \
    if (threadIdx.x == 0) {                             \
      const long long _t = clock64();                   \
      qpk_pt[k] += _t - qpk_pt[PH_N - 1];               \
      qpk_pt[PH_N - 1] = _t;                            \
    }                                                   \
  } while (0)
#else
#define QPK_PT(k) ((void)0)
#endif

struct OpSum { template <class V> QPD static V f(V a, V b) { return a + b; } };
struct OpMax { QPD static float f(float a, float b) { return fmaxf(a, b); } };
struct OpMin { QPD static float f(float a, float b) { return fminf(a, b); } };

// One butterfly step: Op(v, value of lane ^ O) in every lane, on the VALU
// (DPP row rotations, gfx950's permlane swaps) instead of the LDS crossbar
// that shuffles use; V is float or double (two 32-bit halves).  Steps run
// in descending O: once the steps above O have run, lanes l and l ^ 2^k
// (2^k > O) hold equal values, so the rotation by O within a 16-lane row,
// which reaches lane (l - O) mod 16, reads the value of lane l ^ O (for
// O = 8 it is that lane); the swaps exchange whole rows (O = 16) or halves
// (O = 32) exactly.  With commutative operations the results are bitwise
// those of the shuffle butterfly.  All lanes of the wave must be active.
template <int O>
QPD int dpp_ror(int v) {
  static_assert(O == 8 || O == 4 || O == 2 || O == 1, "row rotation");
  return __builtin_amdgcn_update_dpp(0, v, 0x120 + O, 0xF, 0xF, false);  // row_ror:O
}
template <int O>
QPD void lane_swap(int v, int &a, int &b) {
  if constexpr (O == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    a = r[0]; b = r[1];
  } else {
    static_assert(O == 16, "row swap");
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    a = r[0]; b = r[1];
  }
}
template <int O, class Op, class V>
QPD V bfly(V v) {
  if constexpr (sizeof(V) == 4) {
    const int iv = __float_as_int(v);
    if constexpr (O >= 16) {
      int a, b;
      lane_swap<O>(iv, a, b);
      return Op::f(__int_as_float(a), __int_as_float(b));
    } else {
      return Op::f(v, __int_as_float(dpp_ror<O>(iv)));
    }
  } else {
    const long long w = __double_as_longlong(v);
    const int lo = (int)(unsigned)w, hi = (int)(unsigned)(w >> 32);
    auto join = [](int l, int h) {
      return __longlong_as_double((long long)(((unsigned long long)(unsigned)h << 32) |
                                              (unsigned)l));
    };
    if constexpr (O >= 16) {
      int al, bl, ah, bh;
      lane_swap<O>(lo, al, bl);
      lane_swap<O>(hi, ah, bh);
      return Op::f(join(al, ah), join(bl, bh));
    } else {
      return Op::f(v, join(dpp_ror<O>(lo), dpp_ror<O>(hi)));
    }
  }
}
// Op over the 16 lanes of each row, in every lane.
template <class Op, class V>
QPD V row_bfly(V v) {
  v = bfly<8, Op>(v);
  v = bfly<4, Op>(v);
  v = bfly<2, Op>(v);
  return bfly<1, Op>(v);
}
// Op over the wave, in every lane.
template <class Op, class V>
QPD V wave_bfly(V v) {
  v = bfly<32, Op>(v);
  v = bfly<16, Op>(v);
  return row_bfly<Op>(v);
}

// Reduce K values across the workgroup; every thread gets the results, as
// scalars: read from LDS they count as different per lane, and a Newton loop
// that leaves on such a value is compiled as a divergent one, with its
// uniform state (sizes, addresses) in vector registers that spill and are
// reloaded one by one in every iteration.
// `red` needs (T/64)*K floats.  Contains two barriers.
template <int T, class Op, int K>
QPD void block_reduce(float (&v)[K], lf *red) {
#pragma unroll
  for (int k = 0; k < K; ++k) {
    v[k] = wave_bfly<Op>(v[k]);
  }
  if constexpr (T > 64) {
    const int w = tidx() >> 6;
    if ((tidx() & 63) == 0) {
#pragma unroll
      for (int k = 0; k < K; ++k) red[w * K + k] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      float r = red[k];
#pragma unroll
      for (int i = 1; i < T / 64; ++i) r = Op::f(r, red[i * K + k]);
      v[k] = rflf(r);
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Softplus retraction, cancellation-free (appendix C): b_kappa(v) =
// (v + r)/2 for v >= 0, 2 kappa / (r - v) for v < 0, r = sqrt(v^2 + 4 kappa).
// Both signs of v at once: one root and one division.
QPD void bk2(float v, float kappa, float &bp, float &bm) {  // b(v), b(-v)
  const float av = fabsf(v), r = sqrtf(fmaf(v, v, 4.f * kappa));
  const float big = 0.5f * (av + r), small = 2.f * kappa / (r + av);
  bp = v >= 0.f ? big : small;
  bm = v <= 0.f ? big : small;
}
// b_kappa'(v): (1 + v/r)/2 for v >= 0, 2 kappa / (r^2 - v r) for v < 0; again
// for both signs, with one division each.
QPD void dbk2(float v, float kappa, float r, float &dp, float &dm) {  // b'(v), b'(-v)
  const float av = fabsf(v);
  const float big = 0.5f * (1.f + av / r), small = 2.f * kappa / (r * (r + av));
  dp = v >= 0.f ? big : small;
  dm = v <= 0.f ? big : small;
}

// ---------------------------------------------------------------------------
// Packed-blocked storage of the lower triangle of the bordered factor: row i
// holds columns 0 .. 16*floor(i/16)+15 (its lower part rounded up to a whole
// 16-column panel) plus 4 floats of padding, so every panel segment
// M[i][k0 .. k0+15] with k0 <= i is a 16-byte-aligned run and consecutive
// rows start on different LDS banks.  Element (i, j), j <= i, is at
// moff(i) + j.
__host__ __device__ inline int moff(int i) {
  const int q = i >> 4, rem = i & 15;
  return 20 * i + 16 * (8 * q * (q - 1) + q * rem);
}

// Addresses inside a factor of N rows.  In LDS the packed-blocked layout
// above.  In global memory 16x16 tiles, row-major and contiguous, tile row by
// tile row (the last one only as many rows as the system has), so that a wave
// reads or writes a tile as one run of 1 KB: with rows kept contiguous instead,
// a tile is 16 runs of 64 bytes in as many pairs of cache lines, and a read
// with a row per lane is 64 of them.  Either takes at most moff(N) floats.
// Row i: element (i, j) is at base + col(j); block q of 16 rows: the segment
// of panel k of its row r is at row(16 q + r).base + k step.
template <class MF>
struct MRow {
  int base, step;
  QPD int col(int j) const {
    if constexpr (std::is_same<MF, lf>::value) return j;
    else return (j >> 4) * step + (j & 15);
  }
  QPD int at(int j) const { return base + col(j); }
};
template <class MF>
QPD MRow<MF> mrow(int N, int i) {
  if constexpr (std::is_same<MF, lf>::value) {
    return {moff(i), kNB};
  } else {
    const int q = i >> 4, last = (N - 1) >> 4;
    return {128 * q * (q + 1) + 16 * (i & 15), q == last ? 16 * (N - 16 * last) : 256};
  }
}

// Lower-triangular tile t -> (ti, tj), tj <= ti, in row order.  The estimate
// is off by at most one for the tile counts in use (up to 32896, the 4x4 tiles
// of n = 1024).
QPD void tile_ij(int t, int &ti, int &tj) {
  int i = (int)((__builtin_amdgcn_sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
  i += (i + 1) * (i + 2) / 2 <= t;
  i -= i * (i + 1) / 2 > t;
  ti = i;
  tj = t - i * (i + 1) / 2;
}

// ---------------------------------------------------------------------------
// Per-QP LDS layout (floats; ints share the float arena).  All blocks are
// 4-float aligned.  Equal sizes stand together, so that an address is a few
// scalar multiply-adds of the sizes away: every phase works its addresses out
// anew (Ctx) instead of keeping them.
struct Layout {
  int n, m, p, kb, Nmax;
  int iflag;                            // 16 flags
  int part, red;                        // partial sums, reduction scratch
  int u0, u1, rr, rd;                   // right-hand sides; residual and last
                                        // correction of the refinement
  int dv0, dv1, dd, ex;                 // dd: FP64 scratch; ex: border exponents
  int z, s, v, h, E, D, c, ri, rz, rs;
  int role, bidx, elist;
  int t0, t1;                           // also rhs copies of the refinement
  int x, q, rt, tGz, tAy;
  int y, b, re;
  int stg, stg_len;  // assembly staging: the span part .. end of ex, which
                     // holds nothing live while the matrix is assembled
  int M;      // offset of M if in LDS, else -1
  int total;  // floats
};

__host__ __device__ inline int al4(int a) { return (a + 3) & ~3; }

__host__ __device__ inline Layout make_layout(int n, int m, int p, int kb, bool m_lds, int T) {
  Layout L;
  L.n = n; L.m = m; L.p = p; L.kb = kb;
  L.Nmax = n + kb + p;
  const int sn = al4(n), sm = al4(max(m, 1)), sp = al4(max(p, 1)), sN = al4(L.Nmax);
  const int st = al4(max(max(m, p), L.Nmax));  // t0, t1: also m- and p-vectors
  L.iflag = 0;
  // partial sums: 2 floats or 1 double per thread (4 floats before them are
  // unused: the plans' LDS bound, and with it the border cap of sizes at the
  // bound, counts them)
  L.part = 20; L.red = L.part + 2 * T;
  const int b0 = L.red + (T / 64) * 16;
  L.u0 = b0; L.u1 = b0 + sN; L.rr = b0 + 2 * sN; L.rd = b0 + 3 * sN;
  L.dv0 = b0 + 4 * sN; L.dv1 = L.dv0 + sm;
  L.dd = L.dv0 + 2 * sm;
  L.ex = L.dd + al4(2 * (2 * m + p + n + 8));
  const int b1 = L.ex + ((L.Nmax + 15) & ~15);
  L.stg = L.part;
  L.stg_len = b1 - L.part;
  L.z = b1; L.s = b1 + sm; L.v = b1 + 2 * sm; L.h = b1 + 3 * sm; L.E = b1 + 4 * sm;
  L.D = b1 + 5 * sm; L.c = b1 + 6 * sm; L.ri = b1 + 7 * sm; L.rz = b1 + 8 * sm;
  L.rs = b1 + 9 * sm; L.role = b1 + 10 * sm; L.bidx = b1 + 11 * sm; L.elist = b1 + 12 * sm;
  const int b2 = b1 + 13 * sm;
  L.t0 = b2; L.t1 = b2 + st;
  const int b3 = b2 + 2 * st;
  L.x = b3; L.q = b3 + sn; L.rt = b3 + 2 * sn; L.tGz = b3 + 3 * sn; L.tAy = b3 + 4 * sn;
  const int b4 = b3 + 5 * sn;
  L.y = b4; L.b = b4 + sp; L.re = b4 + 2 * sp;
  const int b5 = b4 + 3 * sp;
  // in LDS M's storage ends with 16 floats past the last row, a zero row for the
  // triangular solves (the solves on a factor in global memory need none)
  L.M = m_lds ? b5 : -1;
  L.total = m_lds ? b5 + al4(moff(L.Nmax) + kNB) : b5;
  return L;
}

// ---------------------------------------------------------------------------
// Dense helpers on one workgroup of T threads.

// Rows i0 + grp, i0 + grp + T/16, ... (U of them) of R, columns jb + sub +
// 16 q: the loads only, from clamped in-bounds addresses (a use next to a load,
// a select to mask it included, would wait for it).  Row batches past the last
// row are skipped; rows and columns past the last hold entries of the last,
// for the users to mask.
template <int T, int U>
QPD void load_rows(const gf *R, int ld, int rows, int cols, int i0, int jb, float (&e)[U][4]) {
  const int sub = tidx() & 15, grp = tidx() >> 4;
  int j[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) j[q] = min(jb + sub + 16 * q, cols - 1);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (i0 + u * (T / 16) < rows) {
      const int i = min(i0 + u * (T / 16) + grp, rows - 1);
#pragma unroll
      for (int q = 0; q < 4; ++q) e[u][q] = R[(unsigned)(i * ld + j[q])];
    }
  }
}

// out[i] = sum_j R[i*ld + j] x[j] for i < rows.  16 lanes share a row
// (columns jb + sub + 16c, c < 4, in blocks of 64) and T/16 rows go at a
// time, the loads of U batches of rows before their arithmetic.
template <int T, int U, int NV, class RF>
QPD void rowdot(const RF *R, int ld, int rows, int cols, const lf *const (&x)[NV],
                lf *const (&out)[NV]) {
  const int sub = tidx() & 15, grp = tidx() >> 4;
  for (int jb = 0; jb < cols; jb += 64) {
    float xv[NV][4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int j = jb + sub + 16 * c;
#pragma unroll
      for (int k = 0; k < NV; ++k) xv[k][c] = j < cols ? x[k][j] : 0.f;
    }
    for (int i0 = 0; i0 < rows; i0 += U * (T / 16)) {
      float e[U][4];
      load_rows<T, U>(R, ld, rows, cols, i0, jb, e);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (i0 + u * (T / 16) < rows) {
          const int i = i0 + u * (T / 16) + grp;
          float acc[NV];
#pragma unroll
          for (int k = 0; k < NV; ++k) {
            acc[k] = 0.f;
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[k] = fmaf(e[u][c], xv[k][c], acc[k]);
            acc[k] = row_bfly<OpSum>(acc[k]);
          }
          if (sub == 0 && i < rows) {
#pragma unroll
            for (int k = 0; k < NV; ++k) out[k][i] = jb ? out[k][i] + acc[k] : acc[k];
          }
        }
      }
    }
  }
}

// out[j] = sum_i R[i*ld + j] x[i] for j < cols.  The same lane layout as
// rowdot; each lane sums its columns over its rows, then the row groups are
// combined by shuffles inside a wave and through `part` (2T floats) across
// waves.  Barriers inside; `x` must be visible to all threads on entry.
template <int T, int U, int NV, class RF>
QPD void coldot(const RF *R, int ld, int rows, int cols, const lf *const (&x)[NV],
                lf *const (&out)[NV], lf *part) {
  static_assert(NV <= 2, "part holds two floats per thread");
  const int tid = tidx(), sub = tid & 15, grp = tid >> 4, wid = tid >> 6;
  for (int jb = 0; jb < cols; jb += 64) {
    float c[NV][4];
#pragma unroll
    for (int k = 0; k < NV; ++k)
#pragma unroll
      for (int q = 0; q < 4; ++q) c[k][q] = 0.f;
    for (int i0 = 0; i0 < rows; i0 += U * (T / 16)) {
      float e[U][4];
      load_rows<T, U>(R, ld, rows, cols, i0, jb, e);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * (T / 16) + grp;
        if (i < rows) {
#pragma unroll
          for (int k = 0; k < NV; ++k) {
            const float w = x[k][i];
#pragma unroll
            for (int q = 0; q < 4; ++q) c[k][q] = fmaf(e[u][q], w, c[k][q]);
          }
        }
      }
    }
#pragma unroll
    for (int k = 0; k < NV; ++k)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        c[k][q] = bfly<32, OpSum>(bfly<16, OpSum>(c[k][q]));
      }
    if ((tid & 63) < 16) {
#pragma unroll
      for (int k = 0; k < NV; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q) part[k * T + wid * 64 + 16 * q + sub] = c[k][q];
    }
    __syncthreads();
    if (tid < 64 && jb + tid < cols) {
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < T / 64; ++w) sum += part[k * T + w * 64 + tid];
        out[k][jb + tid] = sum;
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Panels of the factorisation, one wave at a time.
//
// A wave works on four 16-row blocks ("slots") of one 16-column panel: first
// as 16x16 tiles in the matrix cores' result layout with rows and columns
// swapped (lane 16 g + c holds row c, columns 4g .. 4g+3 of its block, so a
// tile is one 16-byte load or store per lane), then, for the elimination,
// with a row per lane (lane 16 s + c holds all 16 columns of row c of slot
// s).

// (a, b) <- rows of lanes exchanged: the upper half (odd 16-lane rows) of a
// with the lower half (even rows) of b.
QPD void swap32(float &a, float &b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(a), __float_as_int(b), false, false);
  a = __int_as_float(r[0]); b = __int_as_float(r[1]);
}
QPD void swap16(float &a, float &b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(a), __float_as_int(b), false, false);
  a = __int_as_float(r[0]); b = __int_as_float(r[1]);
}
// Tile layout of four slots -> a row per lane: the 4x4 transposition between
// slot index (register) and column group (16-lane row), register by register.
QPD void tiles_to_rows(const f4v (&t)[4], float (&P)[kNB]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float x0 = t[0][r], x1 = t[1][r], x2 = t[2][r], x3 = t[3][r];
    swap32(x0, x2);
    swap32(x1, x3);
    swap16(x0, x1);
    swap16(x2, x3);
    P[r] = x0; P[4 + r] = x1; P[8 + r] = x2; P[12 + r] = x3;
  }
}

// And back.
QPD void rows_to_tiles(const float (&P)[kNB], f4v (&t)[4]) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float x0 = P[r], x1 = P[4 + r], x2 = P[8 + r], x3 = P[12 + r];
    swap16(x0, x1);
    swap16(x2, x3);
    swap32(x0, x2);
    swap32(x1, x3);
    t[0][r] = x0; t[1][r] = x1; t[2][r] = x2; t[3][r] = x3;
  }
}

// Tiles t[0 .. CNT-1] -= sum over panels k < np of L[block, k] sg L[panel, k]':
// oa[u] and ob are the places in M of this lane's row of block u and of the
// panel's diagonal block (+ 4g), whose 16-byte segments of panel k are k sa[u]
// and k sb floats further on.  Instruction q multiplies component q, so the
// four v_mfma_f32_16x16x4_f32 cover the 16 columns; each panel's sum is formed
// from zero and then subtracted, in ascending order of k.  The segments of the
// next panel are loaded while this one's products run; the loops carry no
// branches (after one, every load waits for all those in flight), so panels
// whose columns all have sign +1 have a loop of their own (a factorisation of
// 440 rows: 494K -> 448K cycles).  Two to six panels in flight, or the
// subtraction one panel behind, took 461K to 503K.
template <int CNT, class MF>
QPD void update_tiles(const MF *M, const int (&oa)[4], const int (&sa)[4], int ob, int sb, int np,
                      int npos, f4v (&t)[4]) {
  typedef typename Vec4<const MF>::type CV4;
  const int g4 = 4 * ((tidx() & 63) >> 4);
  auto at = [&](int o) {
    return *reinterpret_cast<CV4 *>(M + (std::is_same<MF, lf>::value ? o : (unsigned)o));
  };
  f4v a[CNT], b = at(ob);
  int o[CNT];
#pragma unroll
  for (int u = 0; u < CNT; ++u) {
    o[u] = oa[u];
    a[u] = at(o[u]);
  }
  auto step = [&](int k, auto mixed) {
    f4v bs = b, as[CNT];
#pragma unroll
    for (int u = 0; u < CNT; ++u) as[u] = a[u];
    const int d = k + 1 < np ? 1 : 0;  // (the last panel's segments again)
    ob += d * sb;
    b = at(ob);
#pragma unroll
    for (int u = 0; u < CNT; ++u) {
      o[u] += d * sa[u];
      a[u] = at(o[u]);
    }
    if constexpr (decltype(mixed)::value) {
#pragma unroll
      for (int q = 0; q < 4; ++q) bs[q] *= 16 * k + g4 + q < npos ? 1.f : -1.f;
    }
    f4v acc[CNT];
#pragma unroll
    for (int u = 0; u < CNT; ++u) acc[u] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int u = 0; u < CNT; ++u)
        acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(bs[q], as[u][q], acc[u], 0, 0, 0);
#pragma unroll
    for (int u = 0; u < CNT; ++u) t[u] -= acc[u];
  };
  const int kp = min(np, npos >> 4);
#pragma unroll 2
  for (int k = 0; k < kp; ++k) step(k, std::false_type{});
#pragma unroll 1
  for (int k = kp; k < np; ++k) step(k, std::true_type{});
}

// Dynamic regularisation (dyn): a pivot sg*a_jj that is not above
// kPivTol * pmax, with pmax the largest pivot accepted so far in its block
// (the H block, or the border from its first column on), is taken as
// numerically zero (or of the wrong sign through rounding) and replaced by
// kPivReg * pmax; nreg counts the replacements.  The factor is then that of
// M plus a small diagonal, and callers refine against the exact operator.
// This keeps a degenerate system (dependent border rows, e.g. more active
// rows plus equalities than unknowns) factorable in FP32.
constexpr float kPivTol = 1e-6f;
constexpr float kPivReg = 1e-5f;
constexpr float kGrowthMax = 1e2f;  // accepted max|L| / sqrt(largest pivot) with
                                    // replacements (a stable factor stays near 1)

// Eliminate one panel of kb columns from k0 on in a wave's registers (a row
// per lane); lanes 0 .. 15 hold the diagonal block, so that every multiplier
// and pivot is one lane broadcast away.  The border's pivots (its Schur
// complement, of order |C_j|^2 / |H| plus the diagonal Dl, with the rows
// equilibrated: border_exponent) are tested against the border's own largest
// pivot: at the first border column the running maximum restarts (the H
// block's is kept in pmaxh).  The multipliers of column jj are read from
// ps = a[.][jj] / L[jj][jj], which equals L[.][jj] sg_jj exactly.  iv
// receives the signed pivot inverses.  Returns whether a pivot failed.
//
// This form decides pivot by pivot; it runs only when eliminate() has found
// a pivot that needs a decision.
QPD bool eliminate_checked(float (&P)[kNB], float (&iv)[kNB], int k0, int kb, int npos, bool dyn,
                           float &pmax, float &pmaxh, int &nreg) {
  const int lane = tidx() & 63;
  bool fail = false;
#pragma unroll
  for (int jj = 0; jj < kNB; ++jj) {
    if (jj < kb) {
      const float sg = (k0 + jj) < npos ? 1.f : -1.f;
      if (k0 + jj == npos) {
        pmaxh = pmax;
        pmax = 0.f;
      }
      float tt = sg * readlane(P[jj], jj);
      if (dyn && !(tt > kPivTol * pmax) && tt >= -FLT_MAX && pmax > 0.f) {
        tt = kPivReg * pmax;
        ++nreg;
      }
      const bool ok = tt > 0.f && tt <= FLT_MAX;
      if (ok) pmax = fmaxf(pmax, tt);
      fail |= !ok;
      // pivot sqrt(tt) and its signed inverse from one hardware reciprocal
      // square root (about 1 ulp)
      const float rs = ok ? __builtin_amdgcn_rsqf(tt) : 1.f;
      const float d = ok ? tt * rs : 1.f;
      iv[jj] = sg * rs;
      const float ps = P[jj] * rs;  // L sg below the diagonal
      const float nl = ps * -sg;
      P[jj] = lane == jj ? d : -nl;
#pragma unroll
      for (int cc = jj + 1; cc < kNB; ++cc) P[cc] = fmaf(readlane(ps, cc), nl, P[cc]);
    }
  }
  return fail;
}

// Running maximum over the lanes before this one in its 16-lane row
// (0 for the first); x >= 0.
QPD float row_max_before(float x) {
#define QPK_SHR(v, O) __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x110 + O, 0xF, 0xF, true))
  x = QPK_SHR(x, 1);
  x = fmaxf(x, QPK_SHR(x, 1));
  x = fmaxf(x, QPK_SHR(x, 2));
  x = fmaxf(x, QPK_SHR(x, 4));
  return fmaxf(x, QPK_SHR(x, 8));
#undef QPK_SHR
}

// A panel of at most kFewCols columns (the last one) is eliminated column by
// column: eliminate() runs all 16 of its steps whatever the panel holds.  At 5
// to 8 columns the short form takes up to 2% longer; at 1 or 2 (2048 QPs of
// n = 1, m = 1) it takes 291 us and the other 307.
constexpr int kFewCols = 4;

// The same elimination for a panel whose pivots are all good (positive,
// finite and above kPivTol times the largest before them: the common case).
// The chain from one pivot to the next bounds the factorisation of every
// size, so nothing is decided between the columns: the pivots are collected
// (lane jj holds column jj's) and tested together at the end, with a running
// maximum across the lanes.  If one needs a decision, the return value is
// true, pmax and pmaxh are unchanged, and the caller repeats the panel from
// its saved tiles with eliminate_checked().  Alone on a CU a panel takes 5.7K
// cycles decided pivot by pivot, 2.6K here (the lane broadcasts, two vector
// instructions per multiplier with its update, are most of that).  Rows past the last column
// (kb < 16) are replaced by rows of the identity first, whose pivots are 1
// and whose multipliers are 0.
QPD bool eliminate(float (&P)[kNB], float (&iv)[kNB], int k0, int kb, int npos, float &pmax,
                   float &pmaxh) {
  const int lane = tidx() & 63, r = npos - k0;  // columns before r have sign +1
  if (kb < kNB) {
#pragma unroll
    for (int c = 0; c < kNB; ++c)
      P[c] = lane >= kb ? (lane == c ? (c < r ? 1.f : -1.f) : 0.f) : P[c];
  }
  constexpr int kSign = (int)0x80000000;
  float tv = 0.f;
  int sm = 0 < r ? 0 : kSign;
  int tt = __builtin_amdgcn_readlane(__float_as_int(P[0]), 0) ^ sm;
  float rs = __builtin_amdgcn_rsqf(__int_as_float(tt));
  // scheduling fences keep the next pivot's chain (update its column, read
  // the pivot, its reciprocal square root) ahead of this column's other
  // updates, which then run in the chain's shadow
#pragma unroll
  for (int jj = 0; jj < kNB; ++jj) {
    const float ps = P[jj] * rs;
    const float nl = __int_as_float(__float_as_int(ps) ^ (sm ^ kSign));
    float lc[kNB];
    if (jj + 1 < kNB) P[jj + 1] = fmaf(readlane(ps, jj + 1), nl, P[jj + 1]);
    const int s0 = sm, t0 = tt;
    const float rs0 = rs;
    if (jj + 1 < kNB) {
      sm = jj + 1 < r ? 0 : kSign;
      tt = __builtin_amdgcn_readlane(__float_as_int(P[jj + 1]), jj + 1) ^ sm;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int cc = jj + 2; cc < kNB; ++cc) lc[cc] = readlane(ps, cc);
    if (jj + 1 < kNB) rs = __builtin_amdgcn_rsqf(__int_as_float(tt));
    __builtin_amdgcn_sched_barrier(0);
    // (on the diagonal ps sg = tt rs, the pivot's square root)
    P[jj] = __int_as_float(__float_as_int(ps) ^ s0);
    iv[jj] = __int_as_float(__float_as_int(rs0) ^ s0);
    tv = lane == jj ? __int_as_float(t0) : tv;
#pragma unroll
    for (int cc = jj + 2; cc < kNB; ++cc) P[cc] = fmaf(lc[cc], nl, P[cc]);
  }
  const bool own = lane < kb;
  tv = own ? tv : 0.f;
  float before, ph = pmaxh, pm = r == 0 ? 0.f : pmax;
  if (r == 0) ph = pmax;
  if (r > 0 && r < kb) {  // the border begins inside the panel
    const float th = lane < r ? tv : 0.f, tb = lane < r ? 0.f : tv;
    const float bh = fmaxf(row_max_before(th), pm), bb = row_max_before(tb);
    before = lane < r ? bh : bb;
    ph = readlane(fmaxf(bh, th), kNB - 1);
    pm = readlane(fmaxf(bb, tb), kNB - 1);
  } else {
    before = fmaxf(row_max_before(tv), pm);
    pm = readlane(fmaxf(before, tv), kNB - 1);
  }
  if (__any(own && !(tv > kPivTol * before && tv <= FLT_MAX))) return true;
  pmax = pm;
  pmaxh = ph;
  return false;
}

// The same eliminations on 64 further rows, with the diagonal block D (lanes
// 0 .. 15, finished) and the signed pivot inverses of eliminate().
QPD void eliminate_more(float (&P)[kNB], const float (&D)[kNB], const float (&iv)[kNB], int k0,
                        int kb, int npos) {
#pragma unroll
  for (int jj = 0; jj < kNB; ++jj) {
    if (jj < kb) {
      const float sg = (k0 + jj) < npos ? 1.f : -1.f;
      P[jj] *= iv[jj];
#pragma unroll
      for (int cc = jj + 1; cc < kNB; ++cc)
        P[cc] = fmaf(-P[jj], readlane(D[jj], cc) * sg, P[cc]);
    }
  }
}

// Row i's 16-column panel segment from registers.
template <class MF>
QPD void store_row(MF *M, int i, int k0, const float (&P)[kNB]) {
  typedef typename Vec4<MF>::type V4;
  MF *row = M + moff(i) + k0;
#pragma unroll
  for (int c = 0; c < kNB; c += 4)
    *reinterpret_cast<V4 *>(row + c) = f4v{P[c], P[c + 1], P[c + 2], P[c + 3]};
}

// Equilibration of the border for the pivot tests.  The regularisation
// test compares each border pivot with the largest border pivot accepted so
// far, so a border that mixes rows of very different norms (inequality rows
// of G and equality rows of A in different units) would have the small
// rows' pivots taken for numerical zeros.  Before the factorisation, border
// row i (i >= npos) is multiplied by s_i = 2^k_i and its diagonal entry by
// s_i^2, with k_i = floor((e_max - e_i) / 2), e_i the binary exponent of
// |C_i|^2 and e_max the largest one (rows within about a factor of two in
// norm of the largest keep s_i = 1); after it, row i of the factor is
// divided by s_i.  The scalings are powers of two and so exact: the result
// is bit for bit the factor of the unscaled matrix wherever the scaled
// tests decide as the unscaled ones would, and the factor with the scaled
// tests' replacements otherwise.  The assembly computes e_i while it copies
// the border rows and keeps it in ex[i], the per-wave maxima of e in flag[8 ..] (at most 8 waves).
constexpr int kNoExp = -1000;
template <int T>
QPD int border_emax(const li *flag) {
  int e = kNoExp;
#pragma unroll
  for (int w = 0; w < T / 64; ++w) e = max(e, flag[8 + w]);
  return rfl(e);
}
QPD int border_shift(const lf *ex, int i, int emax) {
  const int e = __float_as_int(ex[i]);
  return e == kNoExp ? 0 : min((emax - e) >> 1, 30);
}
// Exponent e_i of the squared norm ss (the same in all 16 lanes of row i's
// group) into ex[i] (if store), and the thread's running maximum.
QPD void border_exponent(lf *ex, int i, bool store, int sub, float ss, float &el) {
  ss = row_bfly<OpSum>(ss);
  int e = kNoExp;
  if (ss > 0.f && ss <= FLT_MAX) (void)frexpf(ss, &e);
  if (store) {
    if (sub == 0) ex[i] = __int_as_float(e);
    el = fmaxf(el, (float)e);
  }
}
// Per-wave maxima of the exponents into flag[8 ..]; read after a barrier.
template <int T>
QPD void border_exponents_done(float el, li *flag) {
  static_assert(T / 64 <= 8, "per-wave exponent slots");
  el = wave_bfly<OpMax>(el);
  if ((tidx() & 63) == 0) flag[8 + (tidx() >> 6)] = (int)el;
}
// Wave 0: f(i, k_i) for every border row i with k_i > 0, in row order (a
// lane per row reads the exponents; the rows to rescale, usually few, are
// then taken one at a time by the whole wave).
template <class F>
QPD void border_shifted_rows(const lf *ex, int N, int npos, int emax, F &&f) {
  const int lane = tidx() & 63, K = N - npos;
  for (int k0 = 0; k0 < K; k0 += 64) {
    const int k = k0 + lane;
    const int sh = k < K ? border_shift(ex, npos + k, emax) : 0;
    unsigned long long b = __ballot(sh > 0);
    while (b) {
      const int l = __builtin_ctzll(b);
      b &= b - 1;
      f(npos + k0 + l, __builtin_amdgcn_readlane(sh, l));
    }
  }
}

// In-place M = L diag(sg) L' (lower triangle, packed-blocked layout),
// sg_j = +1 for j < npos, -1 otherwise.  Left-looking in panels of 16 columns:
// the panel's 16-row blocks are dealt to the waves (block j below the
// diagonal block to wave j mod T/64), each wave subtracts the products of all
// earlier panels from its blocks in registers (update_tiles), wave 0 passes
// the updated diagonal block on through `dsh`, and each wave eliminates the
// panel on the diagonal block and its own rows (eliminate), so that an
// element of M is read once and written once, and two barriers separate the
// panels.  A right-looking form reads and writes the trailing matrix once
// per panel: with the factor in global memory that traffic, one tile in
// flight per wave, took 10 times as long (n = 256).
// The strict upper part of each row's last 16-column segment is left at
// exact zeros.  Returns false (uniformly) if a pivot sg_j * a_jj is not a
// positive finite number.  With dyn, numerically zero pivots are regularised
// (see kPivTol; the tests see the border equilibrated, border_exponent) and
// flag[2] receives their count.  flag[4] is the largest accepted pivot (float
// bits, the border's in equilibrated units); flag[0] is scratch, as are
// flag[8 ..]; flag[1] and flag[3] are left alone.  RPL = rows per lane,
// >= ceil(N / 64).
template <int T, int RPL, class MF>
QPK_PHASE bool signed_cholesky(MF *M, int N, int npos, li *flag, bool dyn, lf *dsh, lf *ex) {
  ex = rflp(ex);
  M = rflp(M); N = opaque(rfl(N)); npos = opaque(rfl(npos)); flag = rflp(flag); dyn = rfl(dyn); dsh = rflp(dsh);
  constexpr int NW = T / 64;
  constexpr int kMaxBlk = 4 * RPL;            // 16-row blocks of the largest system
  constexpr bool kMore = kMaxBlk > 3 * NW + 1;  // blocks beyond the waves' first slots
  constexpr int DS = 2 * T >= 320 ? 20 : 16;  // row stride of dsh (2 T floats)
  typedef typename Vec4<const MF>::type CV4;
  const int tid = tidx(), lane = tid & 63, wid = rfl(tid >> 6);
  const int c16 = lane & 15, sl = lane >> 4, g4 = 4 * sl;
  const int nblk = (N + 15) >> 4;
  float pmax = 0.f, pmaxh = 0.f;  // running pivot scale and count of regularised
  int nreg = 0;                   // pivots: the same in every wave that has rows
  bool fail = false;
  // with the pivot tests on, they see the border equilibrated: wave 0
  // scales the rows first and takes the scaling back out of the factor at
  // the end (see border_exponent)
  bool eq = dyn && N > npos;
  const int emax = eq ? border_emax<T>(flag) : 0;
  if (eq) {
    // (usually no row needs it; every wave looks)
    bool any = false;
    for (int k = lane; k < N - npos; k += 64) any |= border_shift(ex, npos + k, emax) > 0;
    eq = __any(any);
  }
  if (eq) {
    __syncthreads();  // every wave has looked
    if (wid == 0) {
      border_shifted_rows(ex, N, npos, emax, [&](int i, int sh) {
        const MRow<MF> row = mrow<MF>(N, i);
        const float s = ldexpf(1.f, sh);
        for (int j = lane; j < npos; j += 64) M[row.at(j)] *= s;
        if (lane == 0) M[row.at(i)] *= s * s;  // the border block is diagonal here
      });
    }
    __syncthreads();
  }
#pragma unroll 1
  for (int p = 0; p < nblk; ++p) {
    const int k0 = kNB * p, kb = min(kNB, N - k0), below = nblk - 1 - p;
    // this lane's row of block q (clamped: rows past N-1 read row N-1 and are
    // not stored)
    constexpr bool kLds = std::is_same<MF, lf>::value;
    auto row_of = [&](int q, int &step) {
      const int r = min(c16, N - 1 - kNB * q);
      const MRow<MF> row = mrow<MF>(N, kNB * q);
      step = row.step;
      return row.base + r * (kLds ? 20 + kNB * q : kNB) + g4;
    };
    int sb;
    const int ob = row_of(p, sb);
    // slots of this wave: block p + j(s); wave 0's slot 0 is the diagonal
    // block, which the other waves get through dsh
    const int s0 = wid == 0 ? 0 : 1;
    auto block_of = [&](int s) { return wid == 0 ? NW * s : wid + NW * (s - 1); };
    // the updated tiles, slots s0 .. of this wave
    f4v t[4];
    auto update = [&](auto cnt, auto first) {
      constexpr int CNT = decltype(cnt)::value;
      int oa[4], sa[4];
#pragma unroll
      for (int u = 0; u < CNT; ++u) {
        oa[u] = row_of(p + first(u), sa[u]);
        t[u] = *reinterpret_cast<CV4 *>(M + oa[u] + p * sa[u]);
      }
      if (p) update_tiles<CNT>(M, oa, sa, ob, sb, p, npos, t);
    };
    auto update_n = [&](int cnt, auto first) {
      if (cnt == 1) update(std::integral_constant<int, 1>{}, first);
      if constexpr (kMaxBlk > NW)
        if (cnt == 2) update(std::integral_constant<int, 2>{}, first);
      if constexpr (kMaxBlk > 2 * NW)
        if (cnt == 3) update(std::integral_constant<int, 3>{}, first);
      if constexpr (kMaxBlk > 3 * NW)
        if (cnt == 4) update(std::integral_constant<int, 4>{}, first);
    };
    const f4v zero = {0.f, 0.f, 0.f, 0.f};
    t[0] = t[1] = t[2] = t[3] = zero;
    // slots in use: j(s) <= below
    const int used = wid == 0 ? 1 + min(3, below / NW) : (wid <= below ? min(3, (below - wid) / NW + 1) : 0);
    update_n(used, [&](int u) { return block_of(u + s0); });
    if (wid == 0) *reinterpret_cast<lf4 *>(dsh + c16 * DS + g4) = t[0];
    __syncthreads();
    QPK_PT(PH_FACT_UPDATE);
    if (used) {
      if (wid != 0) {
        t[3] = t[2]; t[2] = t[1]; t[1] = t[0];
        t[0] = *reinterpret_cast<const lf4 *>(dsh + c16 * DS + g4);
      }
      float P[kNB], iv[kNB];
      tiles_to_rows(t, P);
      if (kb <= kFewCols || eliminate(P, iv, k0, kb, npos, pmax, pmaxh)) {
        tiles_to_rows(t, P);
        fail |= eliminate_checked(P, iv, k0, kb, npos, dyn, pmax, pmaxh, nreg);
      }
      if (wid == 0) {
#pragma unroll
        for (int c = 1; c < kNB; ++c) P[c] = lane < c ? 0.f : P[c];  // right of the diagonal
      }
      // slots s0 .. : block p + first(s)
      auto store = [&](const float (&R)[kNB], int from, auto first) {
        if constexpr (kLds) {
          const int j = first(sl), i = kNB * (p + j) + c16;
          if (sl >= from && j <= below && i < N) store_row(M, i, k0, R);
        } else {
          typedef typename Vec4<MF>::type V4;
          f4v o[4];
          rows_to_tiles(R, o);
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int j = first(s);
            if (s >= from && j <= below) {
              int step;
              MF *d = M + row_of(p + j, step);
              d += p * step;
              if (kNB * (p + j) + c16 < N) *reinterpret_cast<V4 *>(d) = o[s];
            }
          }
        }
      };
      store(P, s0, block_of);
      if constexpr (kMore) {
        // blocks past the waves' first slots, four per wave at a time
#pragma unroll 1
        for (int j0 = 3 * NW + 1 + wid; j0 <= below; j0 += 4 * NW) {
          t[0] = t[1] = t[2] = t[3] = zero;
          update_n(min(4, (below - j0) / NW + 1), [&](int u) { return j0 + NW * u; });
          float R[kNB];
          tiles_to_rows(t, R);
          eliminate_more(R, P, iv, k0, kb, npos);
          store(R, 0, [&](int s) { return j0 + NW * s; });
        }
      }
    }
    __syncthreads();
    QPK_PT(PH_FACT_ELIM);
  }
  pmax = fmaxf(pmax, pmaxh);
  if (tid == 0) {
    flag[0] = fail;
    flag[2] = nreg;
    flag[4] = __float_as_int(pmax);  // largest accepted pivot (retry scale)
  }
  __syncthreads();
  bool good = rfl(flag[0]) == 0;
  if (rfl(flag[2]) > 0) {
    // with regularised pivots, entries of L far beyond the scale sqrt(pmax)
    // of a stable factor mean the replaced pivots amplified rounding errors:
    // report a failure so the caller factors again with a uniform floor
    float lmax = 0.f;
    for (int i = wid; i < N; i += NW) {
      const MRow<MF> row = mrow<MF>(N, i);
      for (int j = lane; j <= i; j += 64) {
        const float v = fabsf(M[row.at(j)]);
        lmax = v <= FLT_MAX ? fmaxf(lmax, v) : __int_as_float(0x7f800000);
      }
    }
    lmax = wave_bfly<OpMax>(lmax);
    if (lane == 0) flag[8 + wid] = __float_as_int(lmax);
    __syncthreads();
    for (int w = 0; w < NW; ++w) lmax = fmaxf(lmax, __int_as_float(flag[8 + w]));
    lmax = rflf(lmax);
    if (!(lmax <= kGrowthMax * sqrtf(__int_as_float(rfl(flag[4]))))) good = false;
  }
  if (eq) {
    if (wid == 0) {
      border_shifted_rows(ex, N, npos, emax, [&](int i, int sh) {
        const MRow<MF> row = mrow<MF>(N, i);
        const float r = ldexpf(1.f, -sh);
        for (int j = lane; j <= i; j += 64) M[row.at(j)] *= r;
      });
    }
    __syncthreads();
  }
  return good;
}

// o[t] = p[t] for t < RPL (p aligned to RPL floats) if `in`, else zeros, as
// one vector load for RPL <= 4 (16-byte loads above).
template <int RPL>
QPD void load_run(const lf *p, bool in, float (&o)[RPL]) {
  if constexpr (RPL == 1) {
    o[0] = in ? p[0] : 0.f;
  } else if constexpr (RPL == 2) {
    f2v v = {0.f, 0.f};
    if (in) v = *reinterpret_cast<clf2 *>(p);
    o[0] = v.x; o[1] = v.y;
  } else {
#pragma unroll
    for (int t = 0; t < RPL; t += 4) {
      f4v v = {0.f, 0.f, 0.f, 0.f};
      if (in) v = *reinterpret_cast<const lf4 *>(p + t);
      o[t] = v.x; o[t + 1] = v.y; o[t + 2] = v.z; o[t + 3] = v.w;
    }
  }
}

// Solve (L diag(sg) L') u = r in place for the right-hand side r (length N)
// on WG waves (this one is wave g of them), the vector and the pivots' inverses
// in registers.  The forward sweep walks rows of L, the backward sweep reads
// L[j][i] from row j.  16-row blocks are dealt to the waves in turn (block b
// to wave b mod WG), S rows per lane (lane l owns local rows S l .. S l + S-1,
// all in one block), so that a block's rows sit in fixed slots of 16 / S lanes.
// For each 16-column block the owner runs its 16 dependent steps (scale the
// row's value by its pivot's inverse, broadcast it, subtract it from every row) in
// registers; with more than one wave it then passes the 16 values on through
// `ex` (two buffers of 16, taken in turn, so that one workgroup barrier per
// block separates writer and readers), and the other waves subtract them from
// their rows.  Every element sees its subtractions in the same order whatever
// WG is.  The segments of L do not depend on the chain: the next CW columns'
// are loaded before this one's steps.  The factor holds exact zeros right of
// the diagonal inside every row's padded 16-column segment; rows that must
// not be touched in a block read the zero row `zrow` (16 zeros stored after
// M's last row, so both pointers are in M's address space), and rows past N-1
// hold 0 with an inverse of 0, so the steps carry no tests.
template <int S, int WG>
QPD void signed_solve_waves(const lf *M, int N, int npos, lf *r, const lf *zrow, int g,
                            lf *ex, li *bad) {
  static_assert(kNB % S == 0, "row slot must be static within a block");
  // columns in flight: two buffers of S x CW floats per lane
  constexpr int CW = S > 4 ? 4 : (S > 2 ? 8 : kNB);
  const int lane = tidx() & 63;
  const int lr = S * lane;  // this lane's first local row
  const int i0 = kNB * ((lr >> 4) * WG + g) + (lr & 15);
  float a[S], dl[S];
  const lf *row[S];
#pragma unroll
  for (int t = 0; t < S; ++t) {
    const bool in = i0 + t < N;
    a[t] = in ? r[min(i0 + t, N - 1)] : 0.f;
    row[t] = M + moff(min(i0 + t, N - 1));
    dl[t] = in ? 1.f / row[t][min(i0 + t, N - 1)] : 0.f;
  }
  const int nblk = (N + 15) >> 4;
  float nx[S][CW], Lc[S][CW];
  auto load_f = [&](int j) {  // columns j .. j+CW-1 of this lane's rows
    const int jb = j & ~15;
#pragma unroll
    for (int t = 0; t < S; ++t) {
      // rows below the block: L[i][j..]; rows in the block: their lower part
      // with zeros right of the diagonal; finished rows and rows past N-1: zeros
      const lf *p = i0 >= jb && i0 + t < N ? row[t] + j : zrow + (j & 15);
#pragma unroll
      for (int c = 0; c < CW; c += 4) {
        const f4v v4 = *reinterpret_cast<const lf4 *>(p + c);
        nx[t][c] = v4.x; nx[t][c + 1] = v4.y; nx[t][c + 2] = v4.z; nx[t][c + 3] = v4.w;
      }
    }
  };
  auto take = [&] {
#pragma unroll
    for (int t = 0; t < S; ++t)
#pragma unroll
      for (int c = 0; c < CW; ++c) Lc[t][c] = nx[t][c];
  };
  // the owner's step for column (or row) c of the block in lanes l0 ..
  auto step = [&](int h, int c, int l0) {
    const int q = h + c, s = q % S;
    const float w = a[s] * dl[s];
    const float wj = readlane(w, l0 + q / S);
#pragma unroll
    for (int t = 0; t < S; ++t) a[t] = fmaf(-Lc[t][c], wj, a[t]);
    a[s] = lane == l0 + q / S ? w : a[s];
  };
  // pass the block's values on (their owner) or subtract them (the others)
  auto give = [&](int l0, lf *e) {
    if (lane >= l0 && lane < l0 + kNB / S) {
#pragma unroll
      for (int t = 0; t < S; ++t) e[S * (lane - l0) + t] = a[t];
    }
  };
  // With a row per lane, a last block of at most kFewCols rows takes that many
  // steps instead of 16 (QPs of a few rows are nothing but that block: 2048 of
  // n = 1, m = 1 291 -> 283 us).
  const bool few = S == 1 && WG == 1 && N - kNB * (nblk - 1) <= kFewCols;
  const int whole = nblk - (few ? 1 : 0), lf0 = (kNB / S) * whole;
  load_f(0);
#pragma unroll 1
  for (int b = 0; b < whole; ++b) {
    const int l0 = (kNB / S) * (b / WG);
    const bool own = WG == 1 || b % WG == g;
    lf *e = ex + 16 * (b & 1);
    if (own) {
#pragma unroll
      for (int h = 0; h < kNB; h += CW) {
        take();
        load_f(min(kNB * b + h + CW, kNB * nblk - CW));
#pragma unroll
        for (int c = 0; c < CW; ++c) step(h, c, l0);
      }
      if constexpr (WG > 1) give(l0, e);
    }
    if constexpr (WG > 1) {
      __syncthreads();
      if (!own) {
#pragma unroll
        for (int h = 0; h < kNB; h += CW) {
          take();
          load_f(min(kNB * b + h + CW, kNB * nblk - CW));
#pragma unroll
          for (int c = 0; c < CW; c += 4) {
            const f4v w4 = *reinterpret_cast<const lf4 *>(e + h + c);
#pragma unroll
            for (int cc = 0; cc < 4; ++cc)
#pragma unroll
              for (int t = 0; t < S; ++t) a[t] = fmaf(-Lc[t][c + cc], w4[cc], a[t]);
          }
        }
      }
    }
  }
  if (few) {
    take();
#pragma unroll
    for (int c = 0; c < kFewCols; ++c) step(0, c, lf0);
  }
  // sign: w <- sg w
#pragma unroll
  for (int t = 0; t < S; ++t)
    if (i0 + t >= npos) a[t] = -a[t];
  // backward sweep L' u = w: u_j = a_j / L[j][j], then a_i -= L[j][i] u_j, i < j
  auto load_b = [&](int j) {  // rows j .. j+CW-1 at this lane's columns
    // rows b0 .. b0+15 are one block: row b0+c starts c * rstride floats
    // after row b0 (the last rows, past N-1, read row N-1)
    const int b0 = j & ~15, h = j & 15, rstride = 20 + b0;
    const lf *brow = M + moff(b0) + i0;
    // rows above the block read row j; rows in the block read row j's
    // zero padding right of its diagonal; rows below read zeros.  A lane's
    // S rows are all above the block or all at or below it.
    const bool above = i0 < b0 + kNB;
#pragma unroll
    for (int c = 0; c < CW; ++c) {
      float run[S];
      load_run<S>(brow + min(h + c, N - 1 - b0) * rstride, above, run);
#pragma unroll
      for (int t = 0; t < S; ++t) nx[t][c] = run[t];
    }
  };
  load_b(kNB * nblk - CW);
  if (few) {
    take();
    load_b(max(kNB * whole - CW, 0));
#pragma unroll
    for (int c = kFewCols - 1; c >= 0; --c) step(0, c, lf0);
  }
#pragma unroll 1
  for (int b = whole - 1; b >= 0; --b) {
    const int l0 = (kNB / S) * (b / WG);
    const bool own = WG == 1 || b % WG == g;
    // (not the buffer of the forward sweep's last step: it may still be read)
    lf *e = ex + 16 * ((b & 1) ^ 1);
    if (own) {
#pragma unroll
      for (int h = kNB - CW; h >= 0; h -= CW) {
        take();
        load_b(max(kNB * b + h - CW, 0));
#pragma unroll
        for (int c = CW - 1; c >= 0; --c) step(h, c, l0);
      }
      if constexpr (WG > 1) give(l0, e);
    }
    if constexpr (WG > 1) {
      __syncthreads();
      if (!own) {
#pragma unroll
        for (int h = kNB - CW; h >= 0; h -= CW) {
          take();
          load_b(max(kNB * b + h - CW, 0));
#pragma unroll
          for (int c = CW - 4; c >= 0; c -= 4) {
            const f4v w4 = *reinterpret_cast<const lf4 *>(e + h + c);
#pragma unroll
            for (int cc = 3; cc >= 0; --cc)
#pragma unroll
              for (int t = 0; t < S; ++t) a[t] = fmaf(-Lc[t][c + cc], w4[cc], a[t]);
          }
        }
      }
    }
  }
  bool nf = false;
#pragma unroll
  for (int t = 0; t < S; ++t) {
    if (i0 + t < N) r[i0 + t] = a[t];
    nf |= i0 + t < N && !finitef(a[t]);
  }
  if (nf) *bad = 1;
}

// The same solve, of one or two right-hand sides, with a factor in global
// memory (16x16 tiles), by all T/64 = NW waves of the workgroup.  Blocks are
// dealt to the waves in turn; lane 16 s + c holds row c of the wave's local
// blocks 4 t + s (register t), for both right-hand sides, so that a tile of
// the factor is read once, as one run.  The forward sweep transposes the
// tiles it reads into a row per lane (tiles_to_rows), the backward sweep reads
// rows of 16 tiles with a column per lane.  Per block: its owner's 16
// dependent steps, the values passed on through `ex` (64 floats, two buffers
// taken in turn), one barrier, and the other waves' subtractions.  One wave per
// right-hand side, each reading the factor with a row per lane, spent 7K
// cycles per block on the 64 cache lines of every load (n = 256); this takes
// 3.5K there and 2.2K at n = 100.
template <int T, int RPL>
QPD void signed_solve_tiles(const gf *M, int N, int npos, lf *r0, lf *r1, bool both,
                            lf *ex, li *bad) {
  constexpr int NW = T / 64, S = RPL > NW ? RPL / NW : 1;
  const int lane = tidx() & 63, g = rfl(tidx() >> 6), c16 = lane & 15, sl = lane >> 4;
  const int nblk = (N + 15) >> 4, last = nblk - 1;
  float a[2][S], dl[S];
  int qi[S];  // this lane's blocks
#pragma unroll
  for (int t = 0; t < S; ++t) {
    qi[t] = (4 * t + sl) * NW + g;
    const int i = kNB * qi[t] + c16;
    const bool in = i < N;
    a[0][t] = in ? r0[min(i, N - 1)] : 0.f;
    a[1][t] = in && both ? r1[min(i, N - 1)] : 0.f;
    dl[t] = in ? 1.f / M[(unsigned)mrow<gf>(N, min(i, N - 1)).at(min(i, N - 1))] : 0.f;
  }
  f4v nt[S][4];
  // this lane's place in a tile (rows of the last tile row that do not exist
  // read its last one)
  const unsigned po = 16 * c16 + 4 * sl;
  const unsigned pl = 16 * min(c16, N - 1 - kNB * last) + 4 * sl;
  auto load_f = [&](int b) {  // panel b of this wave's blocks
#pragma unroll
    for (int t = 0; t < S; ++t)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int q = (4 * t + u) * NW + g;
        nt[t][u] = f4v{0.f, 0.f, 0.f, 0.f};  // finished blocks
        if (q >= b && q < nblk) {
          const MRow<gf> row = mrow<gf>(N, kNB * q);
          const gf *tile = M + (row.base + b * row.step);
          nt[t][u] = *reinterpret_cast<const gf4 *>(tile + (q == last ? pl : po));
        }
      }
  };
  float Lc[S][kNB];
  // the owner's steps on its block in register to, lanes l0 .. l0+15 (rows
  // past the last one hold 0)
  auto chain = [&](auto tc, int l0, auto upc) {
    constexpr int to = decltype(tc)::value;
    constexpr bool up = decltype(upc)::value;
    a[0][to] = kNB * qi[to] + c16 < N ? a[0][to] : 0.f;
    a[1][to] = kNB * qi[to] + c16 < N ? a[1][to] : 0.f;
#pragma unroll
    for (int k = 0; k < kNB; ++k) {
      const int c = up ? k : kNB - 1 - k;
      const float w0 = a[0][to] * dl[to], w1 = a[1][to] * dl[to];
      const float x0 = readlane(w0, l0 + c), x1 = readlane(w1, l0 + c);
      a[0][to] = fmaf(-Lc[to][c], x0, a[0][to]);
      a[1][to] = fmaf(-Lc[to][c], x1, a[1][to]);
      const bool me = lane == l0 + c;
      a[0][to] = me ? w0 : a[0][to];
      a[1][to] = me ? w1 : a[1][to];
    }
  };
  auto step = [&](int b, auto upc) {
    constexpr bool up = decltype(upc)::value;
    // the buffer after the last step's: down from the last block it is the
    // other one of the pair (its readers passed that block's barrier)
    lf *e = ex + 32 * ((b & 1) ^ (up ? 0 : 1));
    const int lb = b / NW, to = lb >> 2, l0 = 16 * (lb & 3);
    const bool own = b % NW == g;
    if (own) {
#pragma unroll
      for (int t = 0; t < S; ++t)
        if (t == to) {
          if (t == 0) chain(std::integral_constant<int, 0>{}, l0, upc);
          if constexpr (S > 1)
            if (t == 1) chain(std::integral_constant<int, 1>{}, l0, upc);
          if constexpr (S > 2)
            if (t == 2) chain(std::integral_constant<int, 2>{}, l0, upc);
          if constexpr (S > 3)
            if (t == 3) chain(std::integral_constant<int, 3>{}, l0, upc);
          if (lane >= l0 && lane < l0 + kNB) {
            e[lane - l0] = a[0][t];
            e[kNB + lane - l0] = a[1][t];
          }
        }
    }
    __syncthreads();
    if (S > 1 || !own) {
      f4v x0[4], x1[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        x0[k] = *reinterpret_cast<const lf4 *>(e + 4 * k);
        x1[k] = *reinterpret_cast<const lf4 *>(e + kNB + 4 * k);
      }
#pragma unroll
      for (int t = 0; t < S; ++t) {
        if (!own || t != to) {
#pragma unroll
          for (int k = 0; k < kNB; ++k) {
            const int c = up ? k : kNB - 1 - k;
            a[0][t] = fmaf(-Lc[t][c], x0[c >> 2][c & 3], a[0][t]);
            a[1][t] = fmaf(-Lc[t][c], x1[c >> 2][c & 3], a[1][t]);
          }
        }
      }
    }
  };
  static_assert(S <= 4, "owner registers");
  load_f(0);
#pragma unroll 1
  for (int b = 0; b < nblk; ++b) {
#pragma unroll
    for (int t = 0; t < S; ++t) tiles_to_rows(nt[t], Lc[t]);
    load_f(min(b + 1, last));
    step(b, std::true_type{});
  }
#pragma unroll
  for (int t = 0; t < S; ++t)
    if (kNB * qi[t] + c16 >= npos) {
      a[0][t] = -a[0][t];
      a[1][t] = -a[1][t];
    }
  float nx[S][kNB];
  auto load_b = [&](int b) {  // rows 16 b .. at this lane's columns
    const MRow<gf> row = mrow<gf>(N, kNB * b);
    const int rows = b == last ? N - kNB * last : kNB;
#pragma unroll
    for (int t = 0; t < S; ++t) {
      // (zeros right of the diagonal in block b itself; rows past the last
      // read it again: their values are 0)
      const unsigned o = row.base + min(qi[t], b) * row.step + c16;
#pragma unroll
      for (int c = 0; c < kNB; ++c) nx[t][c] = M[o + 16 * min(c, rows - 1)];
    }
  };
  load_b(last);
#pragma unroll 1
  for (int b = last; b >= 0; --b) {
#pragma unroll
    for (int t = 0; t < S; ++t)
#pragma unroll
      for (int c = 0; c < kNB; ++c) Lc[t][c] = qi[t] <= b ? nx[t][c] : 0.f;
    load_b(max(b - 1, 0));
    step(b, std::false_type{});
  }
  bool nf = false;
#pragma unroll
  for (int t = 0; t < S; ++t) {
    const int i = kNB * qi[t] + c16;
    if (i < N) {
      r0[i] = a[0][t];
      if (both) r1[i] = a[1][t];
      nf |= !finitef(a[0][t]) || !finitef(a[1][t]);
    }
  }
  if (nf) *bad = 1;
}

// The solves of one or two right-hand sides side by side.  With the factor in
// LDS, up to 4 rows per lane one wave each (the chain of dependent steps
// bounds them), above that half of the workgroup's waves each (the plans reach
// that with 257 rows at 512 threads only: larger factors do not fit LDS).  A
// barrier must follow.  *bad is set if a solution has a non-finite entry.
template <int T, int RPL, class MF>
QPD void signed_solve(const MF *M, int N, int npos, lf *r0, lf *r1, bool both, const lf *zrow,
                      lf *ex, li *bad) {
  if constexpr (std::is_same<MF, lf>::value) {
    constexpr int WG = RPL > 4 ? T / 128 : 1, S = RPL / WG;
    const int wid = rfl(tidx() >> 6), k = wid / WG;
    if (k == 0 || (k == 1 && both)) {
      signed_solve_waves<S, WG>(M, N, npos, k ? r1 : r0, zrow, wid % WG, ex + 32 * k, bad);
    } else if constexpr (WG > 1) {
      for (int b = 2 * ((N + 15) >> 4); b > 0; --b) __syncthreads();
    }
  } else {
    signed_solve_tiles<T, RPL>(M, N, npos, r0, r1, both, ex, bad);
  }
}

// out[j] (+)= sum_i R[i*ld + j] x[i], accumulated in AT (FP32 or FP64);
// barriers inside.
template <int T, class AT, class RF, class XF>
QPD float coldot_d(const RF *R, int ld, int rows, int cols, const XF *x,
                   typename LdsT<AT>::type *out, bool add, typename LdsT<AT>::type *part) {
  float mx = 0.f;  // largest |column sum| this thread produced
  const int cw = cols <= 64 ? 64 : (cols <= 128 ? (T >= 128 ? 128 : 64) : (T >= 256 ? 256 : T));
  const int groups = T / cw;
  const int g = tidx() / cw, jl = tidx() % cw;
  for (int jb = 0; jb < cols; jb += cw) {
    const int j = jb + jl;
    AT acc = 0;
    if (j < cols) {
      // independent loads first (several in flight), then the accumulation chain
#pragma unroll 8
      for (int i = g; i < rows; i += groups) acc = fma((AT)R[(size_t)i * ld + j], (AT)x[i], acc);
    }
    part[tidx()] = acc;
    __syncthreads();
    if (g == 0 && j < cols) {
      AT s = 0;
      for (int gg = 0; gg < groups; ++gg) s += part[gg * cw + jl];
      out[j] = add ? out[j] + s : s;
      mx = fmaxf(mx, fabsf((float)s));
    }
    __syncthreads();
  }
  return mx;
}

// The products the residuals need, in one pass over Q, G and A (each n
// columns wide), accumulated in AT (FP32, or FP64 for the residuals of the
// FP64 policy and of escalated refinements): gx = G x and ax = A x (row dots) and
// rt = Q'x + G'z + A'y (column sums).  16 lanes share a row (columns
// jb + sub + 16k, k < 4, in blocks of 64), T/16 rows at a time, with the
// loads of several rows in flight before their arithmetic, so each input
// element is read once.  The column sums of each matrix are reduced across
// row groups (shuffles inside a wave, then `part`, T values, across
// waves); their largest magnitudes, which scale the residuals, come back in
// mq, mg, ma (per-thread partial maxima).  Without gcols, G contributes
// its row dots only (z is not read).  No LDS pointer is tested against
// NULL: LDS address 0 is a valid address.  Barriers inside.
template <int T, int U, class AT>
QPD void kkt_matvecs(const gf *Q, const gf *G, const gf *A, int n, int m, int p, const lf *x,
                     const lf *z, bool gcols, const lf *y, typename LdsT<AT>::type *gx,
                     typename LdsT<AT>::type *ax, typename LdsT<AT>::type *rt,
                     typename LdsT<AT>::type *part, float &mq, float &mg, float &ma) {
  typedef typename LdsT<AT>::type la;
  constexpr int RG = T / 16;
  const int tid = tidx(), sub = tid & 15, grp = tid >> 4, wid = tid >> 6;
  mq = mg = ma = 0.f;
  for (int jb = 0; jb < n; jb += 64) {
    AT xv[4], cq[4], cg[4], ca[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int j = jb + sub + 16 * k;
      xv[k] = j < n ? (AT)x[j] : (AT)0;
      cq[k] = cg[k] = ca[k] = 0;
    }
    // rows of R weighted by w (if cols) into c; with dots, also the row dots
    // with x into out
    auto sweep = [&](const gf *R, int rows, const lf *w, bool cols, la *out, bool dots,
                     AT(&c)[4]) {
      for (int i0 = 0; i0 < rows; i0 += U * RG) {
        float e[U][4];
        load_rows<T, U>(R, n, rows, n, i0, jb, e);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (i0 + u * RG < rows) {
            const int i = i0 + u * RG + grp;
            const bool in = i < rows;
            const AT wi = cols && in ? (AT)w[i] : (AT)0;
            AT d = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              if (in) c[k] = fma((AT)e[u][k], wi, c[k]);
              if (dots) d = fma((AT)e[u][k], xv[k], d);
            }
            if (dots) {
              d = row_bfly<OpSum>(d);
              if (sub == 0 && in) out[i] = jb ? out[i] + d : d;
            }
          }
        }
      }
    };
    sweep(Q, n, x, true, gx, false, cq);
    if (m) sweep(G, m, z, gcols, gx, true, cg);
    if (p) sweep(A, p, y, true, ax, true, ca);
    // column sums across the row groups, one matrix at a time
    auto reduce = [&](AT(&c)[4], bool first, float &mx) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        c[k] = bfly<32, OpSum>(bfly<16, OpSum>(c[k]));
      }
      if ((tid & 63) < 16) {
#pragma unroll
        for (int k = 0; k < 4; ++k) part[wid * 64 + 16 * k + sub] = c[k];
      }
      __syncthreads();
      if (tid < 64 && jb + tid < n) {
        AT sum = 0;
#pragma unroll
        for (int w = 0; w < T / 64; ++w) sum += part[w * 64 + tid];
        rt[jb + tid] = first ? sum : rt[jb + tid] + sum;
        mx = fmaxf(mx, fabsf((float)sum));
      }
      __syncthreads();
    };
    reduce(cq, true, mq);
    if (m && gcols) reduce(cg, false, mg);
    if (p) reduce(ca, false, ma);
  }
}

// ---------------------------------------------------------------------------
// The per-QP context: LDS views plus this QP's global problem data.
//
// Each phase makes its own copy (uctx), whose LDS addresses are computed from
// opaque copies of the sizes, so none stays live from one phase to the next
// (kept live, the fifty-odd addresses overflow the scalar register file) and
// those that a phase does not use cost nothing.  Read back from a table in LDS
// instead, every phase began with a chain of LDS loads.
template <int T_, int RPL, class MF>
struct Ctx {
  typedef MF MT;
  static constexpr int T = T_;
  // row batches in flight in the products with Q, G and A: eight from 4 rows
  // per lane on (four: 1024 solves of n = 100 5.18 -> 5.25 ms, 64 of n = 256
  // 13.74 -> 13.86); below, their registers spill (1 QP of n = 8: 235 -> 243 us,
  // 4096 of n = 10 1.02 -> 1.04 ms)
  static constexpr int U = RPL >= 4 ? 8 : 4;
  int n, m, p, kb;
  const gf *Q, *q_g, *A, *b_g, *G, *h_g;
  MF *Mg;  // factor storage when it is global
  MF *M;   // factor storage (LDS or global)
  lf *x, *y, *z, *s, *v, *q, *h, *b, *E, *D, *c;
  lf *rt, *ri, *re, *rz, *rs, *tGz, *tAy;
  lf *t0, *t1, *u0, *u1, *dv0, *dv1, *ex, *part, *red;
  lf *w0, *w1, *rr, *rd;  // w0, w1: rhs copies of the refinement (in t0, t1)
  lf *mz;  // 16 zeros after the last row of a factor in LDS
  ldd *dd;
  li *role, *bidx, *elist, *iflag;
  lf *stg;  // matrix-core assembly staging (aliases part .. ex)
  int amode;  // H-block assembly: 0 FP32 VALU, 1 BF16x3 MFMA, 2 FP32 MFMA
  int dyn;    // bounded form: regularise degenerate factorisations (R13)
  int rmode;  // residual precision: 0 FP32 first (FP64 refinement after a
              // stall), 1 FP64 residuals everywhere, 2 FP32 only
  float bo;   // line-search back-off factor (1 = none)
  int wk;     // count algorithmic flops (FP64 arithmetic; only when asked for)
};

extern __shared__ __attribute__((aligned(16))) float qpk_smem[];

// Addresses of the context's LDS views from its sizes.
template <class CT>
QPD void place(CT &C) {
  constexpr bool mlds = std::is_same<typename CT::MT, lf>::value;
  const Layout L = make_layout(C.n, C.m, C.p, C.kb, mlds, CT::T);
  lf *sm = (lf *)qpk_smem;
  C.x = sm + L.x; C.y = sm + L.y; C.z = sm + L.z; C.s = sm + L.s; C.v = sm + L.v;
  C.q = sm + L.q; C.h = sm + L.h; C.b = sm + L.b; C.E = sm + L.E; C.D = sm + L.D;
  C.c = sm + L.c; C.rt = sm + L.rt; C.ri = sm + L.ri; C.re = sm + L.re; C.rz = sm + L.rz;
  C.rs = sm + L.rs; C.tGz = sm + L.tGz; C.tAy = sm + L.tAy; C.t0 = sm + L.t0; C.t1 = sm + L.t1;
  C.u0 = sm + L.u0; C.u1 = sm + L.u1; C.dv0 = sm + L.dv0; C.dv1 = sm + L.dv1;
  C.ex = sm + L.ex; C.part = sm + L.part; C.red = sm + L.red;
  C.w0 = C.t0; C.w1 = C.t1; C.rr = sm + L.rr; C.rd = sm + L.rd;
  C.dd = reinterpret_cast<ldd *>(sm + L.dd);
  C.role = reinterpret_cast<li *>(sm + L.role);
  C.bidx = reinterpret_cast<li *>(sm + L.bidx);
  C.elist = reinterpret_cast<li *>(sm + L.elist);
  C.iflag = reinterpret_cast<li *>(sm + L.iflag);
  C.stg = sm + L.stg;
  if constexpr (mlds) {
    C.M = sm + L.M;
    C.mz = C.M + moff(L.Nmax);
  } else {
    C.M = C.Mg;
    C.mz = sm;  // (not read)
  }
}

// Uniform copy of a context (see rfl) with its addresses.
template <class CT>
QPD CT uctx(const CT &I) {
  CT C;
  C.n = opaque(rfl(I.n)); C.m = opaque(rfl(I.m)); C.p = opaque(rfl(I.p)); C.kb = opaque(rfl(I.kb));
  C.Q = rflp(I.Q); C.q_g = rflp(I.q_g); C.A = rflp(I.A); C.b_g = rflp(I.b_g);
  C.G = rflp(I.G); C.h_g = rflp(I.h_g); C.Mg = rflp(I.Mg);
  C.amode = rfl(I.amode); C.dyn = rfl(I.dyn); C.rmode = rfl(I.rmode); C.bo = rflf(I.bo);
  C.wk = rfl(I.wk);
  place(C);
  return C;
}

// Residuals at (x, y, z, s) and, for the bounded form, (v, kappa).
// Returns the scaled residual measure (uniform); `bad` = a non-finite value
// was seen.  Complementarity: max(z s) in the solve; in the relaxation
// (kr > 0) |kappa - kr| / kr for the implicit forms, whose retraction keeps
// every z_i s_i equal to kappa (per-row products differ from it only by
// rounding, about 1e-7 relative in FP32), and max|z s - kr| / kr for the
// standard form.  The matrix-vector products are accumulated in AT: FP32 by
// default, FP64 under the FP64 residual policy (the FP32 iterate is exact in
// FP64, so that residual is limited only by the iterate's rounding).
template <int T, class AT, class CT>
QPK_PHASE float residuals(CT &Cin_, bool bounded, float kappa, float kr, bool *bad) {
  CT C = uctx(Cin_);
  bounded = rfl(bounded); kappa = rflf(kappa); kr = rflf(kr);
  typedef typename LdsT<AT>::type la;
  const int n = C.n, m = C.m, p = C.p, tid = tidx();
  // one accumulator for Qx + G'z + A'y; the pieces' norms are taken as they
  // are produced
  la *gxd = reinterpret_cast<la *>(C.dd), *axd = gxd + m, *rtd = gxd + m + p;
  la *pd = reinterpret_cast<la *>(C.part);
  // largest residuals and the scales they are measured against
  enum { RT, RTS, RI, RIS, RE, RES, RZS, RZSS, CC, NF, NK };
  float mx[NK];
#pragma unroll
  for (int k = 0; k < NK; ++k) mx[k] = 0.f;
  float mq, mg, ma;
  kkt_matvecs<T, CT::U, AT>(C.Q, C.G, C.A, n, m, p, C.x, C.z, true, C.y, gxd, axd, rtd, pd, mq, mg,
                            ma);
  mx[RTS] = fmaxf(mq, fmaxf(mg, ma));
  QPK_PT(PH_MATVEC);
  const bool man = bounded && kr > 0.f;  // relaxation of an implicit form
  for (int i = tid; i < n; i += T) {
    const float r = (float)(rtd[i] + (AT)C.q[i]);
    C.rt[i] = r;
    mx[RT] = fmaxf(mx[RT], fabsf(r));
    mx[RTS] = fmaxf(mx[RTS], fabsf(C.q[i]));
    if (!finitef(r)) mx[NF] = 1.f;
  }
  for (int i = tid; i < m; i += T) {
    const AT gx = gxd[i];
    const float si = C.s[i], zi = C.z[i];
    const float r = (float)(gx + (AT)si - (AT)C.h[i]);
    C.ri[i] = r;
    mx[RI] = fmaxf(mx[RI], fabsf(r));
    mx[RIS] = fmaxf(fmaxf(mx[RIS], fabsf((float)gx)), fmaxf(fabsf(si), fabsf(C.h[i])));
    mx[RZSS] = fmaxf(mx[RZSS], fmaxf(fabsf(zi), fabsf(si)));
    float rz = 0.f, rs = 0.f;
    if (bounded) {
      const float vi = C.v[i];
      float bz, bs;
      bk2(vi, kappa, bz, bs);
      rz = zi - bz;
      rs = si - bs;
      C.rz[i] = rz;
      C.rs[i] = rs;
    }
    mx[RZS] = fmaxf(mx[RZS], fmaxf(fabsf(rz), fabsf(rs)));
    const float zs = zi * si;
    if (!man) mx[CC] = fmaxf(mx[CC], kr > 0.f ? fabsf(zs - kr) / kr : zs);
    if (!finitef(r) || !finitef(zs) || !finitef(rz) || !finitef(rs)) mx[NF] = 1.f;
  }
  for (int i = tid; i < p; i += T) {
    const AT ax = axd[i];
    const float r = (float)(ax - (AT)C.b[i]);
    C.re[i] = r;
    mx[RE] = fmaxf(mx[RE], fabsf(r));
    mx[RES] = fmaxf(mx[RES], fmaxf(fabsf((float)ax), fabsf(C.b[i])));
    if (!finitef(r)) mx[NF] = 1.f;
  }
  block_reduce<T, OpMax, NK>(mx, C.red);
  const float rt_s = mx[RT] / (1.f + mx[RTS]);
  const float ri_s = m ? mx[RI] / (1.f + mx[RIS]) : 0.f;
  const float re_s = p ? mx[RE] / (1.f + mx[RES]) : 0.f;
  const float rzs = m ? mx[RZS] / (1.f + mx[RZSS]) : 0.f;
  const float cc = m ? (man ? fabsf(kappa - kr) / kr : mx[CC]) : 0.f;
  *bad = mx[NF] != 0.f;
  return fmaxf(fmaxf(rt_s, ri_s), fmaxf(fmaxf(re_s, rzs), cc));
}

// Workgroup-wide exclusive compaction of rows with flag set, in row order.
// Writes the compacted indices to out[] and returns the count (uniform).
template <int T>
QPD int compact_rows(const li *flag, int m, li *out, lf *red) {
  const int tid = tidx(), lane = tid & 63, w = tid >> 6;
  int base = 0;
  for (int i0 = 0; i0 < m; i0 += T) {
    const int i = i0 + tid;
    const bool f = i < m && flag[i];
    const unsigned long long bal = __ballot(f);
    const int pre = __popcll(bal & ((1ull << lane) - 1ull));
    const int wcnt = __popcll(bal);
    li *wsum = reinterpret_cast<li *>(red);
    if (lane == 0) wsum[w] = wcnt;
    __syncthreads();
    int off = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < T / 64; ++k) {
      const int c = wsum[k];
      off += k < w ? c : 0;
      tot += c;
    }
    if (f) out[base + off + pre] = i;
    base += rfl(tot);
    __syncthreads();
  }
  return base;
}

// Bounded form: retraction derivatives and the sign split.  Returns the
// number of bordered rows nb; fills E, D, c, role (border index or -1),
// bidx (border rows), elist (eliminated rows) and iflag[1] = #eliminated.
template <int T, class CT>
QPK_PHASE int partition_bounded(CT &Cin_, float kappa) {
  CT C = uctx(Cin_);
  kappa = rflf(kappa);
  const int m = C.m, kb = C.kb, tid = tidx(), lane = tid & 63, w = tid >> 6;
  constexpr int NW = T / 64;
  li *ws = reinterpret_cast<li *>(C.red);  // per-wave counts [2][NW]
  const unsigned long long below = (1ull << lane) - 1ull;
  // The border / eliminated lists in row order, from wave ballots: row i goes
  // to the border if bord(i)
  int nb = 0, ne = 0;
  auto lists = [&](auto bord) {
    nb = ne = 0;
    for (int i0 = 0; i0 < m; i0 += T) {
      const int i = i0 + tid;
      const bool valid = i < m;
      const bool f = valid && bord(i);
      const unsigned long long bb = __ballot(f), be = __ballot(valid && !f);
      if (lane == 0) {
        ws[w] = __popcll(bb);
        ws[NW + w] = __popcll(be);
      }
      __syncthreads();
      int ob = 0, oe = 0, tb = 0, te = 0;
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        const int cb = ws[k], ce = ws[NW + k];
        ob += k < w ? cb : 0;
        oe += k < w ? ce : 0;
        tb += cb;
        te += ce;
      }
      if (valid) {
        if (f) {
          const int k = nb + ob + __popcll(bb & below);
          if (k < kb) C.bidx[k] = i;
          C.role[i] = k;
          C.t0[k] = C.v[i];  // the candidates' v, in row order
        } else {
          C.elist[ne + oe + __popcll(be & below)] = i;
          C.role[i] = -1;
        }
      }
      nb += rfl(tb);
      ne += rfl(te);
      __syncthreads();
    }
  };
  // the common case, at most kb rows with v > 0: one sweep with the
  // retraction derivatives
  lists([&](int i) {
    const float vi = C.v[i];
    const float r = sqrtf(fmaf(vi, vi, 4.f * kappa));
    float e, d;
    dbk2(vi, kappa, r, e, d);
    C.E[i] = e;
    C.D[i] = d;
    C.c[i] = 1.f / r;
    return vi > 0.f;
  });
  if (nb > kb) {
    // more candidates than border slots: keep the kb largest v (ties by row
    // index) and eliminate the rest.  The rank of a candidate counts those
    // ahead of it, read four per 16-byte broadcast load (the list's padding
    // is masked).
    const lf4 *v4 = reinterpret_cast<const lf4 *>(C.t0);
    const int nq = (nb + 3) >> 2, cnt = nb;
    for (int i = tid; i < m; i += T) {
      const int k = C.role[i];
      if (k >= 0) {
        const float vi = C.v[i];
        int rank = 0;
        auto ahead = [&](float vj, int j) {
          return (int)(j < cnt && ((vj > vi) || (vj == vi && j < k)));
        };
#pragma unroll 4
        for (int q = 0; q < nq; ++q) {
          const f4v w4 = v4[q];
          rank += ahead(w4.x, 4 * q) + ahead(w4.y, 4 * q + 1) + ahead(w4.z, 4 * q + 2) +
                  ahead(w4.w, 4 * q + 3);
        }
        if (rank >= kb) C.role[i] = -1;
      }
    }
    __syncthreads();
    lists([&](int i) { return C.role[i] >= 0; });
  }
  if (tid == 0) C.iflag[1] = ne;
  __syncthreads();
  return nb;
}

// ---------------------------------------------------------------------------
// H-block assembly on the matrix cores (used for large n).
//
// H = Q + Y'Y with Y = diag(sqrt(w)) G_I (rows of G in elist).  Y is staged
// through LDS 16 rows at a time, column-major: column c of the chunk is a
// record of kStgRec floats, so the MFMA fragment of a lane (4 consecutive
// rows of one column) is a single 8- or 16-byte load, and the A operand of a
// tile (Y_i') and its B operand (Y_j) come from the same records.  Each wave
// owns up to kAsmTiles 16x16 tiles of the lower triangle per pass and
// accumulates them over all chunks in FP32.
//   amode 1 (BF16x3): y = hi + lo with hi = bf16(y), lo = bf16(y - hi);
//     Y_i'Y_j ~ hi_i'hi_j + lo_i'hi_j + hi_i'lo_j on gfx950's 16x16x32 bf16
//     matrix cores with FP32 accumulation: per 16-row chunk one instruction
//     takes K = 32 as [hi; lo]_i against [hi; hi]_j (the first two terms),
//     a second [hi; 0]_i against [lo; 0]_j.  The dropped lo'lo term and the
//     rounding of lo leave a relative error of about 2^-16 per product; the
//     Newton and adjoint solves refine against the exact operator to
//     recover FP32 accuracy.
//   amode 2: FP32 inputs on the 16x16x4 FP32 MFMA.
// Record layout: amode 1: hi of rows 0..15 as 16 bf16 (floats 0..7), lo as
// 16 bf16 (floats 8..15); amode 2: rows 0..15 as floats 0..15.  Floats
// 16..19 pad the record to 80 bytes, which spreads the 16 columns a
// fragment load touches over the LDS banks.
constexpr int kStgRec = 20;
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) unsigned lu;

QPD unsigned bf16_pair(float a, float b) {
  return (unsigned)__builtin_bit_cast(unsigned short, (__bf16)a) |
         ((unsigned)__builtin_bit_cast(unsigned short, (__bf16)b) << 16);
}

// LDS floats the matrix-core assembly stages for n columns.
__host__ __device__ inline int stage_floats(int n) { return ((n + 15) & ~15) * kStgRec; }

// The rows of a chunk are dealt to the waves in pairs (so that a row's address
// and weight are scalars) and loaded one chunk ahead, while the products of the
// present one run; a wave owns every tile it can in one pass (17 at 512 threads
// take n = 256 in one: with 9, G was staged twice).  The square roots of the
// weights are taken once per row, in row order.
template <int T, class CT>
QPD void assemble_h_mfma(CT &C, int N, int ne, const lf *wts) {
  constexpr int W = T / 64;
  constexpr int kAsmTiles = T >= 512 ? 17 : 9;
  constexpr int kPairs = 8 / W > 0 ? 8 / W : 1;  // row pairs per wave
  constexpr int kCols = T >= 512 ? 4 : 2;        // 64-column blocks loaded ahead
  const int n = C.n, tid = tidx(), lane = tid & 63, wid = rfl(tid >> 6);
  const int n16 = (n + 15) & ~15, nt = n16 >> 4;
  const int ntl = nt * (nt + 1) / 2;
  const int passes = (ntl + W * kAsmTiles - 1) / (W * kAsmTiles);
  const int tpw = (ntl + passes * W - 1) / (passes * W);
  const bool bf = C.amode == 1;
  const int g = lane >> 4, c16 = lane & 15;
  lf *stg = C.stg, *sw = C.t0;
  auto *M = C.M;
  for (int k = tid; k < ne; k += T) sw[k] = sqrtf(wts[C.elist[k]]);
  __syncthreads();
  for (int pass = 0; pass < passes; ++pass) {
    int ti[kAsmTiles], tj[kAsmTiles];
    bool val[kAsmTiles];
    f4v acc[kAsmTiles];
#pragma unroll
    for (int j = 0; j < kAsmTiles; ++j) {
      const int t = (pass * W + wid) * tpw + j;
      val[j] = j < tpw && t < ntl;
      ti[j] = tj[j] = 0;
      if (val[j]) {
        tile_ij(t, ti[j], tj[j]);
        ti[j] = rfl(ti[j]);
        tj[j] = rfl(tj[j]);
      }
      acc[j] = f4v{0.f, 0.f, 0.f, 0.f};
    }
    // rows 2 kp, 2 kp + 1 of the chunk at k0, kp = wid + W i, this lane's
    // columns cb + lane + 64 q
    float y[kPairs][kCols][2];
    auto load = [&](int k0, int cb) {
#pragma unroll
      for (int i = 0; i < kPairs; ++i) {
        const int k = k0 + 2 * (wid + W * i);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const bool in = wid + W * i < 8 && k + h < ne;
          const gf *row = C.G + (size_t)rfl(C.elist[in ? k + h : 0]) * n;
          const float w = in ? rflf(sw[k + h]) : 0.f;
#pragma unroll
          for (int q = 0; q < kCols; ++q) {
            const int c = cb + lane + 64 * q;
            y[i][q][h] = in && c < n ? w * row[c] : 0.f;
          }
        }
      }
    };
    auto stage = [&](int cb) {
#pragma unroll
      for (int i = 0; i < kPairs; ++i) {
        const int kp = wid + W * i;
        if (kp < 8) {
#pragma unroll
          for (int q = 0; q < kCols; ++q) {
            const int c = cb + lane + 64 * q;
            if (c < n16) {
              const float y0 = y[i][q][0], y1 = y[i][q][1];
              lf *rec = stg + c * kStgRec;
              if (bf) {
                const float h0 = (float)(__bf16)y0, h1 = (float)(__bf16)y1;
                reinterpret_cast<lu *>(rec)[kp] = bf16_pair(y0, y1);
                reinterpret_cast<lu *>(rec)[8 + kp] = bf16_pair(y0 - h0, y1 - h1);
              } else {
                rec[2 * kp] = y0;
                rec[2 * kp + 1] = y1;
              }
            }
          }
        }
      }
    };
    if (ne > 0) load(0, 0);
    for (int k0 = 0; k0 < ne; k0 += 16) {
      __syncthreads();  // the previous chunk has been consumed
      stage(0);
      for (int cb = 64 * kCols; cb < n16; cb += 64 * kCols) {
        load(k0, cb);
        stage(cb);
      }
      __syncthreads();
      if (k0 + 16 < ne) load(k0 + 16, 0);
#pragma unroll
      for (int j = 0; j < kAsmTiles; ++j) {
        if (!val[j]) continue;
        const lf *ra = stg + (16 * ti[j] + c16) * kStgRec;
        const lf *rb = stg + (16 * tj[j] + c16) * kStgRec;
        if (bf) {
          // lane group g holds K = 8g .. 8g+7 of its row (A) or column (B);
          // a record's 16-byte quarters are hi rows 0-7, hi 8-15, lo 0-7,
          // lo 8-15
          const lf4 *RA = reinterpret_cast<const lf4 *>(ra);
          const lf4 *RB = reinterpret_cast<const lf4 *>(rb);
          const f4v zero = {0.f, 0.f, 0.f, 0.f};
          const f4v a1 = RA[g], b1 = RB[g & 1];
          const f4v a2 = g < 2 ? RA[g] : zero, b2 = g < 2 ? RB[2 + g] : zero;
          acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, a1),
                                                          __builtin_bit_cast(bf8v, b1), acc[j],
                                                          0, 0, 0);
          acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, a2),
                                                          __builtin_bit_cast(bf8v, b2), acc[j],
                                                          0, 0, 0);
        } else {
          const f4v a = *reinterpret_cast<const lf4 *>(ra + 4 * g);
          const f4v b = *reinterpret_cast<const lf4 *>(rb + 4 * g);
          acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, acc[j], 0, 0, 0);
          acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, acc[j], 0, 0, 0);
          acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.z, acc[j], 0, 0, 0);
          acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.w, acc[j], 0, 0, 0);
        }
      }
    }
    // result layout: register r of lane l is row 4(l/16) + r, column l%16;
    // Q's entries of kQ tiles before their stores
    constexpr int kQ = T >= 512 ? 6 : 3;
#pragma unroll
    for (int j0 = 0; j0 < kAsmTiles; j0 += kQ) {
      f4v qv[kQ];
#pragma unroll
      for (int i = 0; i < kQ; ++i) {
        const int j = j0 + i;
        if (j >= kAsmTiles || !val[j]) continue;
        const int col = 16 * tj[j] + c16;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          qv[i][r] = C.Q[(unsigned)(min(16 * ti[j] + 4 * g + r, n - 1) * n + min(col, n - 1))];
      }
#pragma unroll
      for (int i = 0; i < kQ; ++i) {
        const int j = j0 + i;
        if (j >= kAsmTiles || !val[j]) continue;
        const int col = 16 * tj[j] + c16;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * ti[j] + 4 * g + r;
          if (row < n && col <= row)
            M[mrow<typename CT::MT>(N, row).at(col)] = qv[i][r] + acc[j][r];
        }
      }
    }
  }
}

// Assemble M = [[H, C'], [C, -Dl]] (lower triangle) for N = n + nb + p.
// H = Q + sum_{r in elist} w_r g_r g_r' with w = weights (E/D bounded,
// z/s standard); border rows = G[bidx] then A; Dl = dl (per border row) and
// delta on the diagonal of the border block.
template <int T, class CT>
QPK_PHASE void assemble(CT &Cin_, int nb, int ne, const lf *wts, bool bounded, float delta) {
  CT C = uctx(Cin_);
  nb = rfl(nb); ne = rfl(ne); wts = rflp(wts); bounded = rfl(bounded); delta = rflf(delta);
  typedef typename CT::MT MT;
  const int n = C.n, p = C.p, tid = tidx(), N = n + nb + p;
  MT *M = C.M;
  if (C.amode != 0) {
    assemble_h_mfma<T>(C, N, ne, wts);
  } else {
  // H block in 4x4 tiles.  Rows of G_I are staged through LDS in chunks
  // (coalesced cooperative loads), then each tile thread reads its 4 + 4
  // entries per row as 16-byte LDS loads.  The staging area is the (not yet
  // written) border part of M when M is in LDS, else the `part` buffer.
  const int nt = (n + 3) >> 2;
  const int ntiles = nt * (nt + 1) / 2;
  // tile threads are split into `groups` that take every groups-th staged
  // row; group 0 writes Q + its sum, the others add theirs in a fixed order
  const int groups = 1 + (2 * ntiles <= T) + (3 * ntiles <= T) + (4 * ntiles <= T);
  const int ldg = al4(n);
  lf *stage = C.part;
  int cap = 2 * T;
  if constexpr (std::is_same<MT, lf>::value) {
    const int room = moff(N) - moff(n);
    if (room > cap) { stage = C.M + moff(n); cap = room; }
  } else if (groups == 1) {
    // one group takes every row in order, whatever the chunks: the whole span
    // of idle vectors (n = 65: 35 rows at a time instead of 7)
    cap = make_layout(n, C.m, p, C.kb, false, T).stg_len;
  }
  const int R = max(1, cap / ldg);
  for (int tb = 0; tb < ntiles; tb += T) {
    // with more than one group, tb = 0: group g has threads g ntiles ..
    const int g = groups > 1 ? (tid >= ntiles) + (tid >= 2 * ntiles) + (tid >= 3 * ntiles) +
                                   (tid >= 4 * ntiles) : 0;
    const int t = tb + tid - g * ntiles;
    const bool act = t < ntiles && g < groups;
    int i0 = 0, j0 = 0;
    if (act) {
      int ti, tj;
      tile_ij(t, ti, tj);
      i0 = 4 * ti;
      j0 = 4 * tj;
    }
    float acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int bq = 0; bq < 4; ++bq) {
        const int i = min(i0 + a, n - 1), j = min(j0 + bq, n - 1);
        acc[a][bq] = (act && g == 0) ? C.Q[(size_t)i * n + j] : 0.f;
      }
    for (int k0 = 0; k0 < ne; k0 += R) {
      const int kr = min(R, ne - k0);
      __syncthreads();  // the previous chunk has been consumed
      // 16 lanes per staged row (4 columns each, blocks of 64), T/16 rows at
      // a time: the loads of eight row batches first, then the stores; the
      // rows' weights next to them, in row order
      for (int jb = 0; jb < ldg; jb += 64) {
        for (int r0 = 0; r0 < kr; r0 += 8 * (T / 16)) {
          float e[8][4];
          int j[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) j[q] = min(jb + (tid & 15) + 16 * q, n - 1);
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            if (r0 + u * (T / 16) < kr) {
              const int r = C.elist[k0 + min(r0 + u * (T / 16) + (tid >> 4), kr - 1)];
#pragma unroll
              for (int q = 0; q < 4; ++q) e[u][q] = C.G[(unsigned)(r * n + j[q])];
            }
          }
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int r = r0 + u * (T / 16) + (tid >> 4);
            if (r < kr) {
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const int jq = jb + (tid & 15) + 16 * q;
                if (jq < ldg) stage[r * ldg + jq] = jq < n ? e[u][q] : 0.f;
              }
            }
          }
        }
      }
      for (int r = tid; r < kr; r += T) C.t0[r] = wts[C.elist[k0 + r]];
      __syncthreads();
      if (act) {
        const lf *si = stage + i0, *sj = stage + j0, *sw = C.t0;
        // four rows' loads before their arithmetic
        for (int r = g; r < kr; r += 4 * groups) {
          f4v gi[4], gj[4];
          float w[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int ru = min(r + u * groups, kr - 1);
            gi[u] = *reinterpret_cast<const lf4 *>(si + ru * ldg);
            gj[u] = *reinterpret_cast<const lf4 *>(sj + ru * ldg);
            w[u] = sw[ru];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (r + u * groups < kr) {
              const f4v gw = gj[u] * w[u];
#pragma unroll
              for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int bq = 0; bq < 4; ++bq) acc[a][bq] = fmaf(gi[u][a], gw[bq], acc[a][bq]);
            }
          }
        }
      }
    }
    // rows i0 .. i0+3 lie in one 16-row block, and every 4-column run of a
    // row is a 16-byte one (right of the diagonal it is scratch)
    typedef typename Vec4<MT>::type V4;
    const int rs = std::is_same<MT, lf>::value ? 20 + (i0 & ~15) : kNB;
    MT *Mt = M + mrow<MT>(N, i0).at(j0);
    for (int gg = 0; gg < groups; ++gg) {
      __syncthreads();  // staging area (may alias M's border rows) / previous group
      if (act && g == gg) {
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          if (i0 + a < n) {
            V4 *d = reinterpret_cast<V4 *>(Mt + a * rs);
            const f4v v = {acc[a][0], acc[a][1], acc[a][2], acc[a][3]};
            *d = gg == 0 ? v : *d + v;
          }
        }
      }
    }
  }
  }
  __syncthreads();
  QPK_PT(PH_ASM);
  // border rows: [C | -Dl (lower part)].  C = [G_B; A] copied by 16 lanes
  // per row, which also take each row's squared norm for the border
  // equilibration of the factorisation (border_exponent) and write its part
  // of the lower triangle of the diagonal block.  Four row batches' loads go
  // before their stores.
  const int K = nb + p;
  {
    constexpr int NG = T / 16;
    const int sub = tid & 15, grp = tid >> 4;
    float el = (float)kNoExp;
    for (int k0 = 0; k0 < K; k0 += 4 * NG) {
      // groups past the last row repeat it (the row reduction needs all 16
      // lanes) and store nothing
      const gf *src[4];
      float ss[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int kc = min(k0 + u * NG + grp, K - 1);
        src[u] = kc < nb ? C.G + (size_t)C.bidx[kc] * n : C.A + (size_t)(kc - nb) * n;
        ss[u] = 0.f;
      }
      for (int jb = 0; jb < n; jb += 64) {
        float e[4][4];
        int jc[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) jc[q] = min(jb + sub + 16 * q, n - 1);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (k0 + u * NG < K) {
#pragma unroll
            for (int q = 0; q < 4; ++q) e[u][q] = src[u][(unsigned)jc[q]];
          }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = k0 + u * NG + grp;
          const MRow<MT> row = mrow<MT>(N, n + min(k, K - 1));
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int j = jb + sub + 16 * q;
            if (k0 + u * NG < K && j < n) {
              if (k < K) M[row.at(j)] = e[u][q];
              ss[u] = fmaf(e[u][q], e[u][q], ss[u]);
            }
          }
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = k0 + u * NG + grp;
        if (k0 + u * NG < K) {
          border_exponent(C.ex, n + min(k, K - 1), k < K, sub, ss[u], el);
          if (k < K) {
            const MRow<MT> row = mrow<MT>(N, n + k);
            for (int l = sub; l < k; l += 16) M[row.at(n + l)] = 0.f;
            if (sub == 0) {
              float dl = 0.f;
              if (k < nb && bounded) {
                const int r = C.bidx[k];
                dl = C.D[r] / C.E[r];
              }
              M[row.at(n + k)] = -(dl + delta);
            }
          }
        }
      }
    }
    border_exponents_done<T>(el, C.iflag);
  }
  __syncthreads();
  QPK_PT(PH_ASM_BORDER);
}

// Solve for u0 or both right-hand sides u0 and u1.
template <int T, int RPL, class CT>
QPK_PHASE void solve2(CT &Cin_, int N, bool both) {
  CT C = uctx(Cin_);
  N = rfl(N); both = rfl(both);
  signed_solve<T, RPL>(C.M, N, C.n, C.u0, C.u1, both, C.mz, C.part, C.iflag + 6);
  __syncthreads();
}


// Contraction of a refinement step above which the factor is too coarse a
// preconditioner in the arithmetic in use (refine, below).
constexpr float kRefineSlow = 0.5f;

// out = w - K u (sub) or K u, for the augmented operator of refine (below),
// accumulated in AT from the original Q, G, A and rounded to FP32.
// Barriers inside; u must be visible to all threads on entry.
template <int T, class AT, class CT>
QPD void kkt_apply(CT &C, int nb, bool bounded, const lf *w, const lf *u, lf *out, bool sub) {
  typedef typename LdsT<AT>::type la;
  const int n = C.n, m = C.m, p = C.p, tid = tidx();
  la *gx = reinterpret_cast<la *>(C.dd), *ax = gx + m, *phi = gx + m + p, *kx = gx + 2 * m + p;
  la *pd = reinterpret_cast<la *>(C.part);
  // G u, A u and Q'u_x + A'u_y in one pass; then G' phi, which needs G u
  float unused[3];
  kkt_matvecs<T, CT::U, AT>(C.Q, C.G, C.A, n, m, p, u, u, false, u + n + nb, gx, ax, kx, pd, unused[0],
                     unused[1], unused[2]);
  for (int i = tid; i < m; i += T) {
    const int k = C.role[i];
    const AT wi = bounded ? (AT)C.E[i] / (AT)C.D[i] : (AT)C.E[i];
    phi[i] = k >= 0 ? (AT)u[n + k] : wi * gx[i];
  }
  __syncthreads();
  if (m) coldot_d<T, AT>(C.G, n, m, n, phi, kx, true, pd);
  const AT sg = sub ? (AT)-1 : (AT)1;
  for (int j = tid; j < n; j += T) out[j] = (float)((sub ? (AT)w[j] : (AT)0) + sg * kx[j]);
  for (int k = tid; k < nb; k += T) {
    const int i = C.bidx[k];
    const AT dl = bounded ? (AT)C.D[i] / (AT)C.E[i] : (AT)0;
    out[n + k] = (float)((sub ? (AT)w[n + k] : (AT)0) + sg * (gx[i] - dl * (AT)u[n + k]));
  }
  for (int a = tid; a < p; a += T)
    out[n + nb + a] = (float)((sub ? (AT)w[n + nb + a] : (AT)0) + sg * ax[a]);
  __syncthreads();
}

// Largest |r_j| over j < N (kBig if any entry is not finite); uniform.
template <int T>
QPD float maxnorm(const lf *r, int N, lf *red) {
  float mx[2] = {0.f, 0.f};
  for (int j = tidx(); j < N; j += T) {
    const float a = fabsf(r[j]);
    mx[0] = fmaxf(mx[0], a);
    if (!(a <= FLT_MAX)) mx[1] = 1.f;
  }
  block_reduce<T, OpMax, 2>(mx, red);
  return mx[1] != 0.f ? kBig : mx[0];
}

// Iterative refinement of a solution u of the augmented system
//   [[H, C'], [C, -Dl]] u = w,  H = Q + G_I' diag(wts_I) G_I,  C = [G_B; A],
// wts = E/D (bounded form) or E (standard form / initialisation, where E
// holds z/s or 1),
// Dl = D/E on bounded border rows and 0 on equality rows, against the
// operator WITHOUT any regularisation, with the residual w - K u
// accumulated in AT (FP32, or FP64 once a QP's FP32 refinement stalled)
// from the original Q, G, A.  Each step solves for the correction with the
// existing factor (signed_solve, one right-hand side) and adds it; the residual
// after each correction is checked, and a correction that did not make it
// smaller is taken back and ends the refinement.  Returns the contraction of the
// first correction (residual max-norm after it over the one before; 0 if none
// was taken, kBig for a non-finite residual): above kRefineSlow the factor is
// too coarse a preconditioner in this arithmetic.  iflag[7] receives the
// residual max-norm of the returned u (float bits).
template <int T, int RPL, class AT, class CT>
QPK_PHASE float refine(CT &Cin_, int nb, bool bounded, const lf *w, lf *u, int steps) {
  CT C = uctx(Cin_);
  nb = rfl(nb); bounded = rfl(bounded); w = rflp(w); u = rflp(u); steps = rfl(steps);
  const int n = C.n, p = C.p, tid = tidx(), N = n + nb + p;
  lf *r = C.rr;
  float prev = 0.f, first = 0.f, cur = 0.f;
  for (int it = 0; it <= steps; ++it) {
    kkt_apply<T, AT>(C, nb, bounded, w, u, r, true);
    QPK_PT(PH_REFINE_APPLY);
    const float nrm = maxnorm<T>(r, N, C.red);
    cur = nrm;
    if (it > 0) {
      if (it == 1) first = prev > 0.f ? nrm / prev : 0.f;
      if (!(nrm < prev)) {
        // the last correction did not help: take it back and stop
        for (int j = tid; j < N; j += T) u[j] -= C.rd[j];
        cur = prev;
        __syncthreads();
        break;
      }
    } else if (nrm == 0.f) {
      break;  // exact already
    }
    if (it == steps) break;
    prev = nrm;
    signed_solve<T, RPL>(C.M, N, n, r, r, false, C.mz, C.part, C.iflag + 6);
    __syncthreads();
    for (int j = tid; j < N; j += T) {
      C.rd[j] = r[j];
      u[j] += r[j];
    }
    __syncthreads();
  }
  if (tidx() == 0) C.iflag[7] = __float_as_int(cur);
  __syncthreads();
  return first;
}

// Residual precision of the refinement (qp_opts.fp64_residual): refine in
// FP32; under the automatic policy a QP whose FP32 refinement contracts by
// less than kRefineSlow per step continues in FP64 residuals, and keeps
// them for the rest of its solve (iflag[5]).  Returns the contraction of
// the arithmetic that ran last.
template <int T, int RPL, class CT>
QPD float refine_policy(CT &C, int nb, bool bounded, const lf *w, lf *u, int steps) {
  float q;
  if (C.rmode == 1 || rfl(C.iflag[5])) {
    q = refine<T, RPL, double>(C, nb, bounded, w, u, steps);
  } else {
    q = refine<T, RPL, float>(C, nb, bounded, w, u, steps);
    if (C.rmode == 0 && !(q <= kRefineSlow)) {
      __syncthreads();
      if (tidx() == 0) C.iflag[5] = 1;
      __syncthreads();
      q = refine<T, RPL, double>(C, nb, bounded, w, u, steps);
    }
  }
  return q;
}

// Refinement steps of a solve with a factor of the exact operator (neither
// regularised nor assembled from split products): at least `min_steps`
// where the answer needs it (the adjoint solve, the equality-only solve; an
// FP32 factor's backward error grows with the system size, so FP32
// residuals still improve these).
QPD int plain_refine_steps(int rmode, int user_steps, int min_steps) {
  (void)rmode;
  return max(user_steps, min_steps);
}


// Add -delta to the diagonal of the border block, with delta = rel * (largest
// squared border-row norm) / (largest diagonal of H), and at least floor_abs:
// a Tikhonov floor on the Schur complement Dl + C H^-1 C'.
template <int T, class CT>
QPK_PHASE void border_delta(CT &Cin_, int nb, float rel, float floor_abs) {
  CT C = uctx(Cin_);
  nb = rfl(nb); rel = rflf(rel); floor_abs = rflf(floor_abs);
  typedef typename CT::MT MT;
  const int n = C.n, K = nb + C.p, N = n + K, tid = tidx();
  float mx[2] = {0.f, 0.f};
  for (int j = tid; j < n; j += T) mx[0] = fmaxf(mx[0], C.M[mrow<MT>(N, j).at(j)]);
  for (int k = tid; k < K; k += T) {
    float ss = 0.f;
    for (int j = 0; j < n; ++j) {
      const float c = C.M[mrow<MT>(N, n + k).at(j)];
      ss = fmaf(c, c, ss);
    }
    mx[1] = fmaxf(mx[1], ss);
  }
  block_reduce<T, OpMax, 2>(mx, C.red);
  const float delta = fmaxf(fmaxf(rel * mx[1] / fmaxf(mx[0], 1e-30f), floor_abs), 1e-30f);
  for (int k = tid; k < K; k += T) C.M[mrow<MT>(N, n + k).at(n + k)] -= delta;
  __syncthreads();
}

// True (uniformly) if a[0..N) or, with two, b[0..N) holds a
// non-finite value.
template <int T>
QPD bool any_nonfinite(const lf *a, const lf *b, bool two, int N, lf *red) {
  float f[1] = {0.f};
  for (int j = tidx(); j < N; j += T) {
    if (!finitef(a[j]) || (two && !finitef(b[j]))) f[0] = 1.f;
  }
  block_reduce<T, OpMax, 1>(f, red);
  return f[0] != 0.f;
}

// Assemble and factor the bounded-form matrix.  On a pivot breakdown the
// matrix is rebuilt with a border floor and factored again; *regularised
// tells the caller to refine against the unregularised operator.
constexpr float kRetryReg = 1e-4f;
template <int T, int RPL, class CT>
QPD bool factor_bounded(CT &C, int nb, int ne, const lf *wts, float delta_rel, bool *regularised,
                        bool floor = false) {
  const int N = C.n + nb + C.p;
  assemble<T>(C, nb, ne, wts, true, 0.f);
  if (floor) {
    // asked for by a caller whose solve came out non-finite: floor the
    // border at the scale of the previous factorisation's pivots
    border_delta<T>(C, nb, fmaxf(delta_rel, 1e-6f), kRetryReg * __int_as_float(rfl(C.iflag[4])));
  } else if (delta_rel > 0.f) {
    border_delta<T>(C, nb, delta_rel, 0.f);
  }
  QPK_PT(PH_ASM_DIAG);
  bool ok = signed_cholesky<T, RPL>(C.M, N, C.n, C.iflag, C.dyn != 0, C.part, C.ex);
  QPK_PT(PH_FACT);
  *regularised = delta_rel > 0.f || floor || rfl(C.iflag[2]) > 0;
  if (!ok && C.dyn) {
    // the floor is at least kRetryReg times the largest pivot the failed
    // attempt accepted, i.e. scaled like the Schur complement's entries
    const float pmax = __int_as_float(rfl(C.iflag[4]));
    assemble<T>(C, nb, ne, wts, true, 0.f);
    border_delta<T>(C, nb, fmaxf(delta_rel, 1e-6f), kRetryReg * pmax);
    ok = signed_cholesky<T, RPL>(C.M, N, C.n, C.iflag, true, C.part, C.ex);
    *regularised = true;
  }
  return ok;
}

// Bounded-form right-hand sides of the augmented system for two columns:
//   column 0: rho = (r_t - G'(r_i + r_z - r_s), r_i - r_s - c (kappa - kt0), r_e)
//   column 1: rho = (0, c, 0)   (derivative with respect to kappa_target)
// or, for the adjoint (mode adj): column 0 rho = (gx, E gz, gy), no column 1.
// With psi_i = rho2_i / D_i on eliminated rows and rho2_i on border rows:
//   u = [ -rho1 - G' psi ;  -rho2_B ;  -rho3 ].
// rho2 of each column is left in dv0 / dv1 for the recovery.
template <int T, class CT>
QPK_PHASE void rhs_bounded(CT &Cin_, int nb, float kappa, const gf *gx, const gf *gz,
                     const gf *gy, bool adj) {
  CT C = uctx(Cin_);
  nb = rfl(nb); kappa = rflf(kappa); adj = rfl(adj);
  gx = rflp(gx); gz = rflp(gz); gy = rflp(gy);
  const int n = C.n, m = C.m, p = C.p, tid = tidx();
  // phi0 = -(r_i + r_z - r_s) + psi0 would give u_x = -r_t - G' phi0;
  // we compute w0 = (r_i + r_z - r_s) - psi0 so u_x = -r_t + G' w0, and
  // w1 = -psi1 so u_x1 = G' w1.
  for (int i = tid; i < m; i += T) {
    const bool border = C.role[i] >= 0;
    float r2a, w0, w1 = 0.f;
    if (!adj) {
      r2a = C.ri[i] - C.rs[i] - C.c[i] * kappa;
      const float psi0 = border ? r2a : r2a / C.D[i];
      w0 = (C.ri[i] + C.rz[i] - C.rs[i]) - psi0;
      const float r2b = C.c[i];
      const float psi1 = border ? r2b : r2b / C.D[i];
      w1 = -psi1;
      C.dv1[i] = r2b;
    } else {
      r2a = gz ? C.E[i] * gz[i] : 0.f;
      const float psi0 = border ? r2a : r2a / C.D[i];
      w0 = -psi0;
    }
    C.dv0[i] = r2a;
    C.t0[i] = w0;
    C.t1[i] = w1;
  }
  __syncthreads();
  if (m) {
    if (!adj) {
      const lf *xv[2] = {C.t0, C.t1};
      lf *o[2] = {C.tGz, C.tAy};
      coldot<T, CT::U, 2>(C.G, n, m, n, xv, o, C.part);
    } else {
      const lf *xv[1] = {C.t0};
      lf *o[1] = {C.tGz};
      coldot<T, CT::U, 1>(C.G, n, m, n, xv, o, C.part);
    }
  }
  for (int i = tid; i < n; i += T) {
    const float g0 = m ? C.tGz[i] : 0.f;
    if (!adj) {
      C.u0[i] = -C.rt[i] + g0;
      C.u1[i] = m ? C.tAy[i] : 0.f;
    } else {
      C.u0[i] = -gx[i] + g0;
    }
  }
  for (int k = tid; k < nb; k += T) {
    const int r = C.bidx[k];
    C.u0[n + k] = -C.dv0[r];
    if (!adj) C.u1[n + k] = -C.dv1[r];
  }
  for (int k = tid; k < p; k += T) {
    C.u0[n + nb + k] = adj ? (gy ? -gy[k] : 0.f) : -C.re[k];
    if (!adj) C.u1[n + nb + k] = 0.f;
  }
  __syncthreads();
}

// Recover dv for the solved columns: eliminated rows dv = (G dx + rho2)/D,
// border rows dv = du / E.  rho2 is read from dv0 / dv1 and overwritten.
template <int T, class CT>
QPK_PHASE void recover_bounded(CT &Cin_, int nb, bool both) {
  CT C = uctx(Cin_);
  nb = rfl(nb); both = rfl(both);
  const int n = C.n, m = C.m, tid = tidx();
  if (!m) return;
  if (both) {
    const lf *xv[2] = {C.u0, C.u1};
    lf *o[2] = {C.t0, C.t1};
    rowdot<T, CT::U, 2>(C.G, n, m, n, xv, o);
  } else {
    const lf *xv[1] = {C.u0};
    lf *o[1] = {C.t0};
    rowdot<T, CT::U, 1>(C.G, n, m, n, xv, o);
  }
  __syncthreads();
  for (int i = tid; i < m; i += T) {
    const int k = C.role[i];
    if (k >= 0) {
      const float ie = 1.f / C.E[i];
      C.dv0[i] = C.u0[n + k] * ie;
      if (both) C.dv1[i] = C.u1[n + k] * ie;
    } else {
      const float id = 1.f / C.D[i];
      C.dv0[i] = (C.t0[i] + C.dv0[i]) * id;
      if (both) C.dv1[i] = (C.t1[i] + C.dv1[i]) * id;
    }
  }
  __syncthreads();
}

// Ratio test of eq. linesearch over (s, ds), (z, dz); returns the min of the
// ratios (uninclusive of the cap 1).
QPD float ratio(float s, float ds) { return ds < 0.f ? -s / ds : kBig; }

constexpr int ST_CONV = 0, ST_MAXIT = 1, ST_NONFIN = 2, ST_FACT = 3;
constexpr int SG_NONE = 0, SG_SCAL = 1, SG_PRED = 2, SG_CENT = 3, SG_CORR = 4, SG_LS = 5,
              SG_RELAX = 6, SG_BWD = 7;

QPD int mkstatus(int st, int stage) { return st | (stage << 8); }

// Precision events of a QP's run, reported in status bits 16-17: FP64
// refinement residuals were needed; the split-product assembly fell back to
// FP32.
template <class CT>
QPD int precision_bits(const CT &C, int amode0) {
  return (rfl(C.iflag[5]) ? 1 << 16 : 0) | (amode0 == 1 && C.iflag[3] != 1 ? 1 << 17 : 0);
}

// ---------------------------------------------------------------------------
// Initialisation (CVXOPT convention): solve [[Q+G'G, A'], [A, 0]] [x; y] =
// [-q + G'h; b], zt = Gx - h, s = -zt, z = zt, each shifted positive.
template <int T, int RPL, class CT>
QPK_PHASE bool initialize(CT &Cin_, double &work, bool dyn) {
  CT C = uctx(Cin_);
  dyn = rfl(dyn);
  const int n = C.n, m = C.m, p = C.p, tid = tidx();
  for (int i = tid; i < m; i += T) C.E[i] = 1.f;  // unit weights
  for (int i = tid; i < m; i += T) C.role[i] = 1;
  __syncthreads();
  const int ne = compact_rows<T>(C.role, m, C.elist, C.red);
  assemble<T>(C, 0, ne, C.E, false, 0.f);
  const int N = n + p;
  const bool ok = signed_cholesky<T, RPL>(C.M, N, n, C.iflag, dyn, C.part, C.ex);
  if (m) {
    const lf *hv[1] = {C.h};
    lf *o[1] = {C.tGz};
    coldot<T, CT::U, 1>(C.G, n, m, n, hv, o, C.part);
  }
  for (int i = tid; i < n; i += T) C.u0[i] = C.w0[i] = -C.q[i] + (m ? C.tGz[i] : 0.f);
  for (int k = tid; k < p; k += T) C.u0[n + k] = C.w0[n + k] = C.b[k];
  for (int i = tid; i < m; i += T) C.role[i] = -1;
  __syncthreads();
  solve2<T, RPL>(C, N, false);
  // without inequalities this solve is the answer
  const int nref0 = m == 0 ? plain_refine_steps(C.rmode, 0, 2) : 0;
  if (nref0) refine_policy<T, RPL>(C, 0, false, C.w0, C.u0, nref0);
  for (int i = tid; i < n; i += T) C.x[i] = C.u0[i];
  for (int k = tid; k < p; k += T) C.y[k] = C.u0[n + k];
  __syncthreads();
  if (m) {
    const lf *xv[1] = {C.x};
    lf *o[1] = {C.t0};
    rowdot<T, CT::U, 1>(C.G, n, m, n, xv, o);
    __syncthreads();
    float mx[2] = {-kBig, -kBig};
    for (int i = tid; i < m; i += T) {
      const float zt = C.t0[i] - C.h[i];
      C.s[i] = -zt;
      C.z[i] = zt;
      mx[0] = fmaxf(mx[0], zt);    // max(-s)
      mx[1] = fmaxf(mx[1], -zt);   // max(-z)
    }
    block_reduce<T, OpMax, 2>(mx, C.red);
    for (int i = tid; i < m; i += T) {
      if (mx[0] >= 0.f) C.s[i] += 1.f + mx[0];
      if (mx[1] >= 0.f) C.z[i] += 1.f + mx[1];
    }
  }
  __syncthreads();
  if (C.wk) {
    const double dn = n, dm = m, dN = N;
    work += dm * dn * (dn + 1.0) + dN * dN * dN / 3.0 + 2.0 * dN * dN + 4.0 * dm * dn;
    work += nref0 * (2.0 * dN * dN + 2.0 * dn * dn);  // refinement steps
  }
  return ok;
}

// One Newton iteration of the bounded (implicit) form.  Mode of the target:
// kt_mode 0 = predictor-corrector, 1 = fixed sigma, 2 = relax (kt = kr).
// Returns a status code (ST_CONV meaning "keep going"), with the stage in
// *stage on failure.  Updates x, y, v, kappa, z, s; sz receives this thread's
// part of the new s'z (v and sz are what the next iteration starts from).
template <int T, int RPL, class CT>
QPK_PHASE int newton_bounded(CT &Cin_, float &kappa, int kt_mode, float sigma, float kr,
                       float delta_reg, int refine_steps, double &work, int *stage, float &sz) {
  CT C = uctx(Cin_);
  kappa = rflf(kappa); kt_mode = rfl(kt_mode); sigma = rflf(sigma); kr = rflf(kr);
  delta_reg = rflf(delta_reg); refine_steps = rfl(refine_steps);
  const int n = C.n, m = C.m, p = C.p, tid = tidx();
  C.amode = rfl(C.iflag[3]);  // this QP's assembly arithmetic (may have fallen back)
  const int nb = partition_bounded<T>(C, kappa);
  const int ne = rfl(C.iflag[1]);
  QPK_PT(PH_PART);
  const int N = n + nb + p;
  auto count = [&](auto flops) {  // algorithmic flops
    if (C.wk) work += flops((double)n, (double)m, (double)p, (double)N);
  };
  count([](double dn, double dm, double dp, double) {  // residuals
    return 2.0 * dn * dn + 4.0 * dm * dn + 4.0 * dp * dn;
  });
  // Factor, solve and refine.  With split-product (BF16x3) assembly, a
  // refinement that contracts by less than kRefineSlow per step means the
  // assembly error is too large for this system's conditioning: the QP
  // switches to FP32 matrix-core assembly and the step is redone.
  // at most one switch of the assembly arithmetic and one floored redo
  bool ok = false, floor = false;
  for (int attempt = 0; attempt < 3; ++attempt) {
    // weights E/D for eliminated rows (in t1 until the right-hand sides)
    for (int i = tid; i < m; i += T) C.t1[i] = C.E[i] / C.D[i];
    __syncthreads();
    bool reg = false;
    ok = factor_bounded<T, RPL>(C, nb, ne, C.t1, delta_reg, &reg, floor);
    count([&](double dn, double, double, double dN) {  // assembly + factor
      return (double)ne * dn * (dn + 1.0) + dN * dN * dN / 3.0;
    });
    count([](double dn, double dm, double, double dN) {  // two solves
      return 2.0 * (2.0 * dN * dN + 4.0 * dm * dn);
    });
    if (!ok) break;
    if (tid == 0) C.iflag[6] = 0;  // (barriers in the right-hand sides)
    rhs_bounded<T>(C, nb, kappa, nullptr, nullptr, nullptr, false);
    QPK_PT(PH_RHS);
    const int nref = (reg || C.amode == 1) ? max(refine_steps, 2)
                                           : plain_refine_steps(C.rmode, refine_steps, 0);
    if (nref) {
      for (int j = tid; j < N; j += T) { C.w0[j] = C.u0[j]; C.w1[j] = C.u1[j]; }
      __syncthreads();
    }
    solve2<T, RPL>(C, N, true);
    QPK_PT(PH_SOLVE);
    if (nref) {
      const float q0 = refine_policy<T, RPL>(C, nb, true, C.w0, C.u0, nref);
      const float q1 = refine_policy<T, RPL>(C, nb, true, C.w1, C.u1, nref);
      count([&](double dn, double dm, double dp, double dN) {
        return 2.0 * nref * (2.0 * dN * dN + 4.0 * dm * dn + 2.0 * dn * dn + 4.0 * dp * dn);
      });
      if (C.amode == 1 && !(fmaxf(q0, q1) <= kRefineSlow)) {
        C.amode = 2;
        if (tid == 0) C.iflag[3] = 2;
        __syncthreads();
        continue;
      }
    }
    // a factor that passed its checks can still give a non-finite solution
    // when it is nearly singular: redo the step once with a border floor
    // (the solving waves have seen whether theirs is; a refinement may change it)
    if (C.dyn && !floor &&
        (nref ? any_nonfinite<T>(C.u0, C.u1, true, N, C.red) : rfl(C.iflag[6]) != 0)) {
      floor = true;
      continue;
    }
    break;
  }
  if (!ok) { *stage = SG_PRED; return ST_FACT; }
  QPK_PT(PH_REFINE);
  recover_bounded<T>(C, nb, true);
  QPK_PT(PH_RECOVER);
  // predictor step length (kappa_target = 0) and kappa_aff
  float kt;
  if (kt_mode == 0) {
    float mn[2] = {1.f, 0.f};
    for (int i = tid; i < m; i += T) {
      const float dv = C.dv0[i];
      const float dz = -C.rz[i] + C.E[i] * dv - C.c[i] * kappa;
      const float ds = -C.rs[i] - C.D[i] * dv - C.c[i] * kappa;
      mn[0] = fminf(mn[0], fminf(ratio(C.s[i], ds), ratio(C.z[i], dz)));
      if (!finitef(dz) || !finitef(ds)) mn[1] = -1.f;
    }
    block_reduce<T, OpMin, 2>(mn, C.red);
    if (mn[1] < 0.f) { *stage = SG_PRED; return ST_NONFIN; }
    const float aa = mn[0];
    float sm[1] = {0.f};
    for (int i = tid; i < m; i += T) {
      const float dv = C.dv0[i];
      const float dz = -C.rz[i] + C.E[i] * dv - C.c[i] * kappa;
      const float ds = -C.rs[i] - C.D[i] * dv - C.c[i] * kappa;
      sm[0] += (C.s[i] + aa * ds) * (C.z[i] + aa * dz);
    }
    block_reduce<T, OpSum, 1>(sm, C.red);
    const float kaff = sm[0] / (float)m;
    const float ratio_k = kaff / kappa;
    const float sg = ratio_k * ratio_k * ratio_k;
    kt = sg * kappa;
    if (!finitef(kt)) { *stage = SG_CENT; return ST_NONFIN; }
    kt = fmaxf(kt, 1e-12f);  // keep the central-path parameter positive
    QPK_PT(PH_AFFINE);
  } else if (kt_mode == 1) {
    kt = sigma * kappa;
  } else {
    kt = kr;
  }
  // combined direction and its step length
  const float dk = kt - kappa;
  float mn[2] = {1.f, 0.f};
  for (int i = tid; i < m; i += T) {
    const float dv = fmaf(kt, C.dv1[i], C.dv0[i]);
    const float dz = -C.rz[i] + C.E[i] * dv + C.c[i] * dk;
    const float ds = -C.rs[i] - C.D[i] * dv + C.c[i] * dk;
    mn[0] = fminf(mn[0], fminf(ratio(C.s[i], ds), ratio(C.z[i], dz)));
    if (!finitef(dz) || !finitef(ds)) mn[1] = -1.f;
  }
  block_reduce<T, OpMin, 2>(mn, C.red);
  if (mn[1] < 0.f) { *stage = kt_mode == 2 ? SG_RELAX : SG_CORR; return ST_NONFIN; }
  const float alpha = fminf(1.f, C.bo * mn[0]);
  if (!(alpha > 0.f)) { *stage = SG_LS; return ST_NONFIN; }
  // step on (x, y, v, kappa), then retract z, s
  for (int i = tid; i < n; i += T) C.x[i] += alpha * fmaf(kt, C.u1[i], C.u0[i]);
  for (int k = tid; k < p; k += T) C.y[k] += alpha * fmaf(kt, C.u1[n + nb + k], C.u0[n + nb + k]);
  // kappa + alpha (kt - kappa) lies between kt and kappa, but with alpha = 1
  // and kt below kappa's rounding unit the sum rounds to exactly zero: z of
  // every inactive row would then be 0 and the next centering would divide
  // by kappa = 0.  Held at the bound the step cannot cross.
  const float knew = fmaxf(kappa + alpha * dk, fminf(kt, kappa));
  sz = 0.f;
  for (int i = tid; i < m; i += T) {
    const float vn = C.v[i] + alpha * fmaf(kt, C.dv1[i], C.dv0[i]);
    float zn, sn;
    bk2(vn, knew, zn, sn);
    C.z[i] = zn;
    C.s[i] = sn;
    // the next iteration's manifold coordinate and its share of s'z
    C.v[i] = zn - sn;
    sz += sn * zn;
  }
  kappa = knew;
  __syncthreads();
  QPK_PT(PH_STEP);
  return ST_CONV;
}

// One Mehrotra predictor-corrector iteration of the standard form.
template <int T, int RPL, class CT>
QPK_PHASE int newton_standard(CT &Cin_, float mu, int kt_mode, float kr, float delta_reg, double &work,
                        int *stage) {
  CT C = uctx(Cin_);
  mu = rflf(mu); kt_mode = rfl(kt_mode); kr = rflf(kr); delta_reg = rflf(delta_reg);
  const int n = C.n, m = C.m, p = C.p, tid = tidx();
  float bad[1] = {0.f};
  for (int i = tid; i < m; i += T) {
    const float w = C.z[i] / C.s[i];
    C.t1[i] = w;
    C.role[i] = 1;
    if (!finitef(w)) bad[0] = 1.f;
  }
  block_reduce<T, OpMax, 1>(bad, C.red);
  if (bad[0] != 0.f) { *stage = SG_SCAL; return ST_NONFIN; }
  const int ne = compact_rows<T>(C.role, m, C.elist, C.red);
  // the weights t1 must survive: copy to E (unused in the standard form)
  for (int i = tid; i < m; i += T) C.E[i] = C.t1[i];
  __syncthreads();
  const int N = n + p;
  assemble<T>(C, 0, ne, C.E, false, delta_reg);
  const bool ok = signed_cholesky<T, RPL>(C.M, N, n, C.iflag, false, C.part, C.ex);
  if (C.wk) {
    const double dn = n, dm = m, dp = p, dN = N;
    work += 2.0 * dn * dn + 4.0 * dm * dn + 4.0 * dp * dn;
    work += dm * dn * (dn + 1.0) + dN * dN * dN / 3.0;
    work += 2.0 * (2.0 * dN * dN + 4.0 * dm * dn);
  }
  if (!ok) { *stage = SG_PRED; return ST_FACT; }
  // rhs for a given r_c / s =: q_i;  u_x = -r_t - G'(w r_i - q), u_y = -r_e
  // then dz = w (r_i + G dx) - q, ds = -r_i - G dx
  auto rhs_and_solve = [&](const lf *qv) {
    for (int i = tid; i < m; i += T) C.t0[i] = C.E[i] * C.ri[i] - qv[i];
    __syncthreads();
    {
      const lf *xv[1] = {C.t0};
      lf *o[1] = {C.tGz};
      if (m) coldot<T, CT::U, 1>(C.G, n, m, n, xv, o, C.part);
    }
    for (int i = tid; i < n; i += T) C.u0[i] = -C.rt[i] - (m ? C.tGz[i] : 0.f);
    for (int k = tid; k < p; k += T) C.u0[n + k] = -C.re[k];
    __syncthreads();
    solve2<T, RPL>(C, N, false);
    const lf *xv[1] = {C.u0};
    lf *o[1] = {C.t0};
    if (m) rowdot<T, CT::U, 1>(C.G, n, m, n, xv, o);
    __syncthreads();
  };
  float sgm;
  if (kt_mode == 2) {
    // relax: r_c = z s - kr  =>  q = z - kr / s
    for (int i = tid; i < m; i += T) C.dv1[i] = C.z[i] - kr / C.s[i];
    __syncthreads();
    rhs_and_solve(C.dv1);
  } else {
    // affine predictor: q = z
    rhs_and_solve(C.z);
    float mn[2] = {1.f, 0.f};
    for (int i = tid; i < m; i += T) {
      const float gdx = C.t0[i];
      const float dz = C.E[i] * (C.ri[i] + gdx) - C.z[i];
      const float ds = -C.ri[i] - gdx;
      C.dv0[i] = dz;
      C.dv1[i] = ds;
      mn[0] = fminf(mn[0], fminf(ratio(C.s[i], ds), ratio(C.z[i], dz)));
      if (!finitef(dz) || !finitef(ds)) mn[1] = -1.f;
    }
    block_reduce<T, OpMin, 2>(mn, C.red);
    if (mn[1] < 0.f) { *stage = SG_PRED; return ST_NONFIN; }
    const float aa = mn[0];
    float sm[1] = {0.f};
    for (int i = tid; i < m; i += T)
      sm[0] += (C.s[i] + aa * C.dv1[i]) * (C.z[i] + aa * C.dv0[i]);
    block_reduce<T, OpSum, 1>(sm, C.red);
    const float muaff = sm[0] / (float)m;
    const float rr = muaff / mu;
    sgm = rr * rr * rr;
    if (!finitef(sgm) || !finitef(mu)) { *stage = SG_CENT; return ST_NONFIN; }
    // corrector: r_c = z s + ds_a dz_a - sigma mu  =>  q = z + (ds_a dz_a - sigma mu)/s
    for (int i = tid; i < m; i += T)
      C.dv1[i] = C.z[i] + (C.dv1[i] * C.dv0[i] - sgm * mu) / C.s[i];
    __syncthreads();
    rhs_and_solve(C.dv1);
    if (kt_mode == 1) { /* fixed sigma is not used by the standard arm */ }
  }
  float mn[2] = {kBig, 0.f};
  for (int i = tid; i < m; i += T) {
    const float gdx = C.t0[i];
    const float dz = C.E[i] * (C.ri[i] + gdx) - C.dv1[i];
    const float ds = -C.ri[i] - gdx;
    C.dv0[i] = dz;
    C.dv1[i] = ds;
    mn[0] = fminf(mn[0], fminf(ratio(C.s[i], ds), ratio(C.z[i], dz)));
    if (!finitef(dz) || !finitef(ds)) mn[1] = -1.f;
  }
  block_reduce<T, OpMin, 2>(mn, C.red);
  if (mn[1] < 0.f) { *stage = kt_mode == 2 ? SG_RELAX : SG_CORR; return ST_NONFIN; }
  const float alpha = fminf(1.f, C.bo * mn[0]);
  if (!(alpha > 0.f) || !finitef(alpha)) { *stage = SG_LS; return ST_NONFIN; }
  for (int i = tid; i < n; i += T) C.x[i] += alpha * C.u0[i];
  for (int k = tid; k < p; k += T) C.y[k] += alpha * C.u0[n + k];
  for (int i = tid; i < m; i += T) {
    C.z[i] += alpha * C.dv0[i];
    C.s[i] += alpha * C.dv1[i];
  }
  __syncthreads();
  return ST_CONV;
}

// Without inequalities (m = 0) the refined KKT solve of the initialisation
// is the answer, and its accuracy is that of a direct solve: the backward
// error max(|r_t| / (1 + | |Q||x| + |q| + |A'||y| |), |r_e| / (1 + | |A||x|
// + |b| |)) (infinity norms) measures it.  The scaled residual of the
// general test divides by the largest term instead, which for a solution
// with heavy cancellation (|Q||x| >> |Qx|) lies below what any float32
// vector attains.  Uses r_t, r_e from residuals(); uniform result.
template <int T, class CT>
QPD float direct_backward_error(CT &C) {
  const int n = C.n, p = C.p, tid = tidx();
  float mx[4] = {0.f, 0.f, 0.f, 0.f};  // |r_t|, its scale, |r_e|, its scale
  for (int j = tid; j < n; j += T) {
    float a = fabsf(C.q[j]);
    for (int i = 0; i < n; ++i) a = fmaf(fabsf(C.Q[(size_t)i * n + j]), fabsf(C.x[i]), a);
    for (int k = 0; k < p; ++k) a = fmaf(fabsf(C.A[(size_t)k * n + j]), fabsf(C.y[k]), a);
    mx[0] = fmaxf(mx[0], fabsf(C.rt[j]));
    mx[1] = fmaxf(mx[1], a);
  }
  for (int k = tid; k < p; k += T) {
    float a = fabsf(C.b[k]);
    for (int j = 0; j < n; ++j) a = fmaf(fabsf(C.A[(size_t)k * n + j]), fabsf(C.x[j]), a);
    mx[2] = fmaxf(mx[2], fabsf(C.re[k]));
    mx[3] = fmaxf(mx[3], a);
  }
  block_reduce<T, OpMax, 4>(mx, C.red);
  return fmaxf(mx[0] / (1.f + mx[1]), p ? mx[2] / (1.f + mx[3]) : 0.f);
}

// Newton loop shared by the solve, the relaxation and the serving step.
// Returns the final status; iters counts Newton steps taken.
template <int T, int RPL, class CT>
QPD int newton_loop(CT &Cin_, bool bounded, int max_iter, float tol, int kt_mode, float sigma,
                    float kr, float delta_reg, int refine_steps, double &work, int &iters,
                    float &res) {
  int status = ST_MAXIT;
  int stage = SG_NONE;
  float sz = 0.f;
  for (int it = 0;; ++it) {
    CT C = uctx(Cin_);
    const int m = C.m, tid = tidx();
    // manifold coordinates v = z - s, kappa = s'z / m
    float sm[1] = {sz};
    if (it == 0 || !bounded) {
      sm[0] = 0.f;
      for (int i = tid; i < m; i += T) {
        sm[0] += C.s[i] * C.z[i];
        if (bounded) C.v[i] = C.z[i] - C.s[i];
      }
    }
    block_reduce<T, OpSum, 1>(sm, C.red);
    float kappa = m ? sm[0] / (float)m : 0.f;
    QPK_PT(PH_KAPPA);
    bool bad = false;
    // FP64 residuals under the FP64 policy, and for a QP whose refinement
    // has already needed FP64 (FP32 cannot resolve its residuals either)
    const bool r64 = C.rmode == 1 || (C.rmode == 0 && rfl(C.iflag[5]) != 0);
    res = r64 ? residuals<T, double>(C, bounded, kappa, kt_mode == 2 ? kr : 0.f, &bad)
              : residuals<T, float>(C, bounded, kappa, kt_mode == 2 ? kr : 0.f, &bad);
    QPK_PT(PH_RESID);
    if (bad || !finitef(res)) {
      status = ST_NONFIN;
      stage = kt_mode == 2 ? SG_RELAX : (it == 0 ? SG_NONE : SG_LS);
      iters = it;
      break;
    }
    if (res < tol) { status = ST_CONV; iters = it; break; }
    if (m == 0) {
      res = direct_backward_error<T>(C);
      status = res < tol ? ST_CONV : ST_MAXIT;
      iters = it;
      break;
    }
    if (it >= max_iter) {
      // an iteration limit inside Algorithm 2 is reported at the relax stage
      status = ST_MAXIT;
      if (kt_mode == 2) stage = SG_RELAX;
      iters = it;
      break;
    }
    int st;
    if (bounded)
      st = newton_bounded<T, RPL>(C, kappa, kt_mode, sigma, kr, delta_reg, refine_steps, work, &stage,
                                  sz);
    else st = newton_standard<T, RPL>(C, kappa, kt_mode, kr, delta_reg, work, &stage);
    if (st != ST_CONV) {
      status = st;
      // a failure inside the relaxation (Algorithm 2) is attributed to it as
      // a whole, whichever sub-step produced it
      if (kt_mode == 2) stage = SG_RELAX;
      iters = it + 1;
      break;
    }
  }
  return mkstatus(status, stage);
}

// Load this QP's small vectors into LDS.
template <int T, class CT>
QPD void load_vectors(CT &C) {
  const int tid = tidx();
  for (int i = tid; i < C.n; i += T) C.q[i] = C.q_g[i];
  for (int i = tid; i < C.m; i += T) C.h[i] = C.h_g[i];
  for (int i = tid; i < C.p; i += T) C.b[i] = C.b_g[i];
  if constexpr (std::is_same<typename CT::MT, lf>::value) {
    if (tid < kNB) C.mz[tid] = 0.f;
  }
  __syncthreads();
}

// Factor at the current (relaxed) point and solve the adjoint system for
// the upstream gradient; returns dx in u0[0:n], dy in u0[n+nb:], dz in dv0.
// Returns kAdjOk, kAdjFactorFail, or kAdjInaccurate when the refinement of
// the adjoint solve stalled (contraction above 1/2 in the last arithmetic
// it used) with a residual above kAdjResTol of the right-hand side: the
// factor is too coarse a preconditioner for this system and the gradient
// is not reliable.
constexpr int kAdjOk = 0, kAdjFactorFail = 1, kAdjInaccurate = 2;
constexpr float kAdjResTol = 1e-5f;
template <int T, int RPL, class CT>
QPK_PHASE int adjoint(CT &Cin_, bool bounded, const gf *gx, const gf *gy, const gf *gz,
                 float delta_reg, int refine_steps, double &work) {
  CT C = uctx(Cin_);
  bounded = rfl(bounded); gx = rflp(gx); gy = rflp(gy); gz = rflp(gz);
  delta_reg = rflf(delta_reg); refine_steps = rfl(refine_steps);
  const int n = C.n, m = C.m, p = C.p, tid = tidx();
  float sm[1] = {0.f};
  for (int i = tid; i < m; i += T) {
    sm[0] += C.s[i] * C.z[i];
    if (bounded) C.v[i] = C.z[i] - C.s[i];
  }
  block_reduce<T, OpSum, 1>(sm, C.red);
  const float kappa = m ? sm[0] / (float)m : 0.f;
  int nb = 0, ne = 0;
  if (bounded && m) {
    nb = partition_bounded<T>(C, kappa);
    ne = rfl(C.iflag[1]);
    for (int i = tid; i < m; i += T) C.t1[i] = C.E[i] / C.D[i];
  } else {
    for (int i = tid; i < m; i += T) {
      C.t1[i] = C.z[i] / C.s[i];
      C.role[i] = 1;
    }
    __syncthreads();
    ne = compact_rows<T>(C.role, m, C.elist, C.red);
    for (int i = tid; i < m; i += T) C.role[i] = -1;
  }
  __syncthreads();
  // keep the weights: E holds E (bounded) or z/s (standard)
  if (!bounded)
    for (int i = tid; i < m; i += T) C.E[i] = C.t1[i];
  __syncthreads();
  const int N = n + nb + p;
  auto count = [&](int nref) {  // algorithmic flops
    if (C.wk) {
      const double dn = n, dN = N;
      const double wfac = (double)ne * dn * (dn + 1.0) + dN * dN * dN / 3.0 + 2.0 * dN * dN + 8.0 * m * dn;
      const double wstep = 2.0 * dN * dN + 2.0 * dn * dn + 8.0 * m * dn + 4.0 * p * dn;
      work += wfac + nref * wstep;
    }
  };
  bool ok = false, inaccurate = false;
  if (bounded) {
    C.amode = rfl(C.iflag[3]);
    // as in newton_bounded: fall back from split-product assembly when the
    // refinement does not contract, and floor the border when the solve is
    // not finite
    bool floor = false;
    for (int attempt = 0; attempt < 3; ++attempt) {
      if (attempt) {
        for (int i = tid; i < m; i += T) C.t1[i] = C.E[i] / C.D[i];
        __syncthreads();
      }
      bool reg = false;
      ok = factor_bounded<T, RPL>(C, nb, ne, C.t1, delta_reg, &reg, floor);
      // the adjoint solve gives the gradient directly: a regularised or
      // split-product factor is always refined against the exact operator
      const int nref = (reg || C.amode == 1) ? max(refine_steps, 2)
                                             : plain_refine_steps(C.rmode, refine_steps, 2);
      count(nref);
      if (!ok) break;
      rhs_bounded<T>(C, nb, kappa, gx, gz, gy, true);
      for (int j = tid; j < N; j += T) C.w0[j] = C.u0[j];
      __syncthreads();
      const float wn = maxnorm<T>(C.w0, N, C.red);
      solve2<T, RPL>(C, N, false);
      const float q = nref ? refine_policy<T, RPL>(C, nb, true, C.w0, C.u0, nref) : 0.f;
      inaccurate = nref && !(q <= kRefineSlow) &&
                   !(__int_as_float(rfl(C.iflag[7])) <= kAdjResTol * wn);
      if (C.amode == 1 && !(q <= kRefineSlow)) {
        C.amode = 2;
        if (tid == 0) C.iflag[3] = 2;
        __syncthreads();
        continue;
      }
      if (C.dyn && !floor && any_nonfinite<T>(C.u0, C.u0, false, N, C.red)) {
        floor = true;
        continue;
      }
      break;
    }
    if (!ok) return kAdjFactorFail;
    recover_bounded<T>(C, nb, false);
    // dz = E (dv + gz)
    for (int i = tid; i < m; i += T) C.dv0[i] = C.E[i] * (C.dv0[i] + (gz ? gz[i] : 0.f));
  } else {
    assemble<T>(C, nb, ne, C.t1, false, 0.f);
    ok = signed_cholesky<T, RPL>(C.M, N, n, C.iflag, false, C.part, C.ex);
    const int nref = plain_refine_steps(C.rmode, refine_steps, 2);
    count(nref);
    if (!ok) return kAdjFactorFail;
    // standard: [H A'; A 0][a; c] = [-gx - G' W gz; -gy], dz = W (G a + gz)
    for (int i = tid; i < m; i += T) C.t0[i] = gz ? C.E[i] * gz[i] : 0.f;
    __syncthreads();
    if (m) {
      const lf *xv[1] = {C.t0};
      lf *o[1] = {C.tGz};
      coldot<T, CT::U, 1>(C.G, n, m, n, xv, o, C.part);
    }
    for (int i = tid; i < n; i += T) C.u0[i] = C.w0[i] = -gx[i] - (m ? C.tGz[i] : 0.f);
    for (int k = tid; k < p; k += T) C.u0[n + k] = C.w0[n + k] = gy ? -gy[k] : 0.f;
    __syncthreads();
    const float wn = maxnorm<T>(C.w0, N, C.red);
    solve2<T, RPL>(C, N, false);
    if (nref) {
      const float q = refine_policy<T, RPL>(C, 0, false, C.w0, C.u0, nref);
      inaccurate = !(q <= kRefineSlow) && !(__int_as_float(rfl(C.iflag[7])) <= kAdjResTol * wn);
    }
    if (m) {
      const lf *xv[1] = {C.u0};
      lf *o[1] = {C.t0};
      rowdot<T, CT::U, 1>(C.G, n, m, n, xv, o);
    }
    __syncthreads();
    for (int i = tid; i < m; i += T) C.dv0[i] = C.E[i] * (C.t0[i] + (gz ? gz[i] : 0.f));
  }
  // move dy next to dx: u0[n : n+p] = dy
  __syncthreads();
  if (nb) {
    float tmp[4];
    for (int k0 = 0; k0 < p; k0 += 4 * T) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = k0 + tid + u * T;
        tmp[u] = k < p ? C.u0[n + nb + k] : 0.f;
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = k0 + tid + u * T;
        if (k < p) C.u0[n + k] = tmp[u];
      }
      __syncthreads();
    }
  }
  return inaccurate ? kAdjInaccurate : kAdjOk;
}

// Write the parameter gradients of Algorithm 3 with coalesced stores.
template <int T, class CT>
QPK_PHASE void write_grads(CT &Cin_, const Params &P, size_t qi) {
  CT C = uctx(Cin_);
  const int n = C.n, m = C.m, p = C.p, tid = tidx();
  const lf *dx = C.u0, *dy = C.u0 + n, *dz = C.dv0;
  if (P.dQ) {
    gf *o = (gf *)P.dQ + qi * (size_t)n * n;
    for (int e = tid; e < n * n; e += T) {
      const int i = e / n, j = e % n;
      o[e] = 0.5f * (dx[i] * C.x[j] + C.x[i] * dx[j]);
    }
  }
  if (P.dq) {
    gf *o = (gf *)P.dq + qi * (size_t)n;
    for (int i = tid; i < n; i += T) o[i] = dx[i];
  }
  if (P.dA && p) {
    gf *o = (gf *)P.dA + qi * (size_t)p * n;
    for (int e = tid; e < p * n; e += T) {
      const int i = e / n, j = e % n;
      o[e] = dy[i] * C.x[j] + C.y[i] * dx[j];
    }
  }
  if (P.db && p) {
    gf *o = (gf *)P.db + qi * (size_t)p;
    for (int i = tid; i < p; i += T) o[i] = -dy[i];
  }
  if (P.dG && m) {
    gf *o = (gf *)P.dG + qi * (size_t)m * n;
    for (int e = tid; e < m * n; e += T) {
      const int i = e / n, j = e % n;
      o[e] = dz[i] * C.x[j] + C.z[i] * dx[j];
    }
  }
  if (P.dh && m) {
    gf *o = (gf *)P.dh + qi * (size_t)m;
    for (int i = tid; i < m; i += T) o[i] = -dz[i];
  }
}

// ---------------------------------------------------------------------------
template <int T, int RPL, bool MLDS, int MODE>
QPD void qp_body(const Params &P) {
  typedef typename std::conditional<MLDS, lf, gf>::type MF;
  const size_t qi = blockIdx.x;
  // sizes and data pointers: from the batch (solve / backward) or from this
  // block's slot descriptor (serving step)
  int n, m, p, kb;
  const float *Qp, *qp, *Ap, *bp, *Gp, *hp;
  float *wsp;
  if constexpr (MODE == kServe) {
    const SlotDesc &d = P.desc[qi];
    n = d.n; m = d.m; p = d.p; kb = d.kb;
    Qp = d.Q; qp = d.q; Ap = d.A; bp = d.b; Gp = d.G; hp = d.h;
    wsp = d.ws;
  } else {
    n = P.n; m = P.m; p = P.p; kb = P.kb;
    Qp = P.Q + qi * (size_t)n * n;
    qp = P.q + qi * (size_t)n;
    Ap = p ? P.A + qi * (size_t)p * n : nullptr;
    bp = p ? P.b + qi * (size_t)p : nullptr;
    Gp = m ? P.G + qi * (size_t)m * n : nullptr;
    hp = m ? P.h + qi * (size_t)m : nullptr;
    wsp = MLDS ? nullptr : P.ws + (size_t)qi * P.ws_stride;
  }
  Ctx<T, RPL, MF> C;
  C.n = n; C.m = m; C.p = p; C.kb = kb;
  C.Q = (const gf *)Qp; C.q_g = (const gf *)qp; C.A = (const gf *)Ap;
  C.b_g = (const gf *)bp; C.G = (const gf *)Gp; C.h_g = (const gf *)hp;
  if constexpr (MLDS) C.Mg = nullptr;
  else C.Mg = (gf *)wsp;
  place(C);
  if constexpr (MODE == kServe) C.amode = (P.desc[qi].flags >> 1) & 3;
  else C.amode = P.asm_mode;
  const int amode0 = C.amode;
  const int refine = P.refine;
  const int tid = tidx();
  // per-QP assembly mode for the Newton steps (a BF16x3 QP may fall back)
  if (tid == 0) C.iflag[3] = C.amode;
  // implicit complementarity (bounded form 0, or the first partially
  // condensed form 2 as a negative control: no border rows, no
  // regularisation); form 1 is the standard explicit IPM
  const bool bounded = P.form != 1;
  C.dyn = P.form == 0;
  C.rmode = P.rmode;
  C.bo = P.backoff;
  C.wk = MODE != kServe && P.work != nullptr;
  if (tid == 0) {
    C.iflag[5] = 0;  // refinement residuals start in FP32
  }
#ifdef QPK_PHASE_TIMING
  if (tid < PH_N) qpk_pt[tid] = 0;
  __syncthreads();
  if (tid == 0) qpk_pt[PH_N - 1] = clock64();
#endif
  load_vectors<T>(C);
  double work = 0.0;
  const Ctx<T, RPL, MF> C0 = C;
  int iters = 0;
  float res = 0.f;
  int status;
  if constexpr (MODE == kServe) {
    // resume one resident QP for at most d.budget Newton iterations; the
    // iterate (x, y, z, s) and the QP's arithmetic state (its assembly
    // arithmetic after any fallback, FP64 refinement residuals) persist in
    // the slot's state between steps, so the split into steps does not
    // change what is computed
    const SlotDesc &d = P.desc[qi];
    gf *st = (gf *)d.state;
    const int sticky = n + p + 2 * m;
    bool ok = true;
    if (d.flags & 1) {
      ok = initialize<T, RPL>(C, work, C.dyn != 0);
    } else {
      for (int i = tid; i < n; i += T) C.x[i] = st[i];
      for (int k = tid; k < p; k += T) C.y[k] = st[n + k];
      for (int i = tid; i < m; i += T) {
        C.z[i] = st[n + p + i];
        C.s[i] = st[n + p + m + i];
      }
      if (tid == 0) {
        const int f = __float_as_int(st[sticky]);
        C.iflag[3] = f & 3;
        C.iflag[5] = (f >> 2) & 1;
      }
      __syncthreads();
    }
    if (!ok) {
      status = mkstatus(ST_FACT, SG_PRED);
    } else {
      status = newton_loop<T, RPL>(C, bounded, d.budget, P.tol, P.pc ? 0 : 1, P.sigma, 0.f,
                                   P.delta_reg, refine, work, iters, res);
    }
    C = uctx(C0);
    for (int i = tid; i < n; i += T) st[i] = C.x[i];
    for (int k = tid; k < p; k += T) st[n + k] = C.y[k];
    for (int i = tid; i < m; i += T) {
      st[n + p + i] = C.z[i];
      st[n + p + m + i] = C.s[i];
    }
    gf *out = (gf *)d.out;
    for (int i = tid; i < n; i += T) out[i] = C.x[i];
    for (int k = tid; k < p; k += T) out[n + k] = C.y[k];
    for (int i = tid; i < m; i += T) {
      out[n + p + i] = C.z[i];
      out[n + p + m + i] = C.s[i];
    }
    __syncthreads();
    if (tid == 0) st[sticky] = __int_as_float((C.iflag[3] & 3) | ((rfl(C.iflag[5]) & 1) << 2));
    if (tid == 0) {
      *d.status = status | precision_bits(C, amode0);
      *d.iters = iters;
      *d.res = res;
    }
  } else if constexpr (MODE == kSolve) {
    const bool ok = initialize<T, RPL>(C, work, C.dyn != 0);
    QPK_PT(PH_INIT);
    if (!ok) {
      status = mkstatus(ST_FACT, SG_PRED);
      res = __int_as_float(0x7fc00000);
    } else {
      status = newton_loop<T, RPL>(C, bounded, P.max_iter, P.tol, P.pc ? 0 : 1, P.sigma, 0.f,
                                   P.delta_reg, refine, work, iters, res);
    }
    C = uctx(C0);
    gf *xo = (gf *)P.x + qi * (size_t)n;
    for (int i = tid; i < n; i += T) xo[i] = C.x[i];
    if (p && P.y) for (int k = tid; k < p; k += T) ((gf *)P.y)[qi * p + k] = C.y[k];
    if (m && P.z) for (int i = tid; i < m; i += T) ((gf *)P.z)[qi * m + i] = C.z[i];
    if (m && P.s) for (int i = tid; i < m; i += T) ((gf *)P.s)[qi * m + i] = C.s[i];
    __syncthreads();
    if (tid == 0) {
      P.status[qi] = status | precision_bits(C, amode0);
      if (P.iters) P.iters[qi] = iters;
      if (P.res) P.res[qi] = res;
      if (P.work) P.work[qi] = work;
    }
  } else {
    // backward: warm start from the solution
    const gf *xs = (const gf *)P.x, *ys = (const gf *)P.y, *zs = (const gf *)P.z,
             *ss = (const gf *)P.s;
    for (int i = tid; i < n; i += T) C.x[i] = xs[qi * n + i];
    for (int k = tid; k < p; k += T) C.y[k] = ys[qi * p + k];
    for (int i = tid; i < m; i += T) {
      C.z[i] = zs[qi * m + i];
      C.s[i] = ss[qi * m + i];
    }
    __syncthreads();
    // On QPs with at least three inequality rows per variable the
    // relaxation refines its steps: H then sums that many rank-one terms in
    // FP32, and the relaxed multipliers, to which the gradients are
    // sensitive, drift by about 1e-5 relative (n = 56, m = 896, p = 28:
    // gradient entries off by up to 0.8% without; with one refinement step
    // per relaxation step every entry is within 0.4% of its 1e-3 bound;
    // n = 200, m = 800 missed the bound by 2.6x without).  At m = 2n (the
    // benchmark shapes) it would make the backward pass 63% longer (4096 QPs of
    // n = 50: 1.68 -> 2.74 ms) for no measurable gain.
    const int refine_relax = bounded && m >= 3 * n ? max(refine, 1) : refine;
    status = newton_loop<T, RPL>(C, bounded, P.relax_max_iter, P.relax_tol, 2, 0.f, P.kappa_relax,
                                 P.delta_reg, refine_relax, work, iters, res);
    // without inequalities there is nothing to relax: the relaxed point is
    // the solution (whose own status reports its accuracy)
    if (m == 0 && (status & 0xff) == ST_MAXIT) status = mkstatus(ST_CONV, SG_NONE);
    const gf *gx = (const gf *)P.gx + qi * (size_t)n;
    const gf *gy = P.gy ? (const gf *)P.gy + qi * (size_t)p : nullptr;
    const gf *gz = P.gz ? (const gf *)P.gz + qi * (size_t)m : nullptr;
    const int adj = adjoint<T, RPL>(C, bounded, gx, gy, gz, P.delta_reg, refine, work);
    QPK_PT(PH_BWD);
    // Algorithm 2 hands the factorisation at the relaxed point to the
    // gradient computation, so a breakdown there counts as a relax failure;
    // an adjoint solve whose refinement stalled is reported at the backward
    // stage (the gradients are written but not reliable)
    if (adj == kAdjFactorFail) status = mkstatus(ST_FACT, SG_RELAX);
    else if (adj == kAdjInaccurate && (status & 0xff) == ST_CONV) status = mkstatus(ST_MAXIT, SG_BWD);
    __syncthreads();
    C = uctx(C0);
    write_grads<T>(C, P, qi);
    if (P.rx) for (int i = tid; i < n; i += T) ((gf *)P.rx)[qi * n + i] = C.x[i];
    if (P.ry && p) for (int k = tid; k < p; k += T) ((gf *)P.ry)[qi * p + k] = C.y[k];
    if (P.rz && m) for (int i = tid; i < m; i += T) ((gf *)P.rz)[qi * m + i] = C.z[i];
    if (P.rs && m) for (int i = tid; i < m; i += T) ((gf *)P.rs)[qi * m + i] = C.s[i];
    __syncthreads();
    if (tid == 0) {
      if (P.rstatus) P.rstatus[qi] = status | precision_bits(C, amode0);
      if (P.riters) P.riters[qi] = iters;
      if (P.res) P.res[qi] = res;
      if (P.work) P.work[qi] = work;
    }
  }
#ifdef QPK_PHASE_TIMING
  QPK_PT(PH_OUT);
  if (P.phase && tid < PH_N - 1) P.phase[qi * PH_N + tid] = qpk_pt[tid];
#endif
}

// Waves per SIMD the register allocation targets: 3 (168 VGPRs) up to 256
// threads per QP, 2 (256 VGPRs) at 512, and 4 (128 VGPRs) for 256 threads
// with 4 rows per lane and the factor in global memory in the solve and
// serving kernels: their systems (129 to 256 rows) leave a small LDS
// footprint, so four QPs fit a CU (1024 solves of n = 100: 6.88 ms at three,
// 5.18 at four; 24 of them, one per CU, 2.77 and 2.80).  Kernels with the factor
// in LDS and more than 64 rows are held to three QPs per CU or fewer by LDS.
// Two lines date from kernels that spilled more and measure otherwise on these:
// the backward kernel of that size at four waves takes 1.89 instead of 2.51 ms
// (1024 QPs) and 1.04 instead of 1.03 (24), and the kernels of 128 threads at
// four 0.93 instead of 1.02 ms (4096 solves of n = 10), 1.51 instead of 1.67
// (n = 20) and 0.304 instead of 0.294 (64 of n = 10).
#define QPK_MIN_WAVES(T, RPL, MLDS) \
  ((T) >= 512 ? 2 : ((T) == 256 && (RPL) == 4 && !(MLDS) ? 4 : 3))
#define QPK_MIN_WAVES_BWD(T) ((T) >= 512 ? 2 : 3)

// One workgroup per QP: Algorithm 1 (or the standard IPM) end to end.
template <int T, int RPL, bool MLDS>
__global__ void __launch_bounds__(T, QPK_MIN_WAVES(T, RPL, MLDS)) qp_solve_kernel(Params P) {
  qp_body<T, RPL, MLDS, kSolve>(P);
}

// One workgroup per QP: relax (Algorithm 2), adjoint solve and parameter
// gradients (Algorithm 3).
template <int T, int RPL, bool MLDS>
__global__ void __launch_bounds__(T, QPK_MIN_WAVES_BWD(T)) qp_backward_kernel(Params P) {
  qp_body<T, RPL, MLDS, kBackward>(P);
}

// One workgroup per resident serving slot: resume its Newton loop.
template <int T, int RPL, bool MLDS>
__global__ void __launch_bounds__(T, QPK_MIN_WAVES(T, RPL, MLDS)) qp_serve_kernel(Params P) {
  qp_body<T, RPL, MLDS, kServe>(P);
}

template <class K>
hipError_t launch_k(K k, const Params &P, int T, size_t lds, int grid, hipStream_t st) {
  (void)hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(k, dim3(grid), dim3(T), lds, st, P);
  return hipGetLastError();
}

}  // namespace

template <int T, int RPL>
hipError_t launch_t(const Params &P, bool m_in_lds, size_t lds, int grid, hipStream_t st) {
  if (P.mode == kSolve) {
    if (m_in_lds) return launch_k(qp_solve_kernel<T, RPL, true>, P, T, lds, grid, st);
    return launch_k(qp_solve_kernel<T, RPL, false>, P, T, lds, grid, st);
  }
  if (P.mode == kServe) {
    if (m_in_lds) return launch_k(qp_serve_kernel<T, RPL, true>, P, T, lds, grid, st);
    return launch_k(qp_serve_kernel<T, RPL, false>, P, T, lds, grid, st);
  }
  if (m_in_lds) return launch_k(qp_backward_kernel<T, RPL, true>, P, T, lds, grid, st);
  return launch_k(qp_backward_kernel<T, RPL, false>, P, T, lds, grid, st);
}

}  // namespace qpk
