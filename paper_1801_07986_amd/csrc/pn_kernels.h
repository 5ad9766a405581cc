// pn_kernels.h -- gfx950 device code of libpn (included once, by pn_api.hip).
//
// Notation (Sec. 2 of the paper): body 0 is the massive object (the paper's
// #1, mass M); stars are bodies 1..N-1, stored as "star k" = body k+1 in every
// star-indexed array (Ns = N-1 stars).  x_ab = x_a - x_b, R_ab = sqrt(r^2+eps^2)
// (Eq. (10)), lambda = 1/c^2.
//
// Per force evaluation the work is split into
//   k_prologue   O(N)   massive-object/star pair terms u_s = G M / R_s0 and
//                       b_s = G M x_s0 / R_s0^3, star packets for the pair
//                       sweep, block partials of sum m_s b_s, m_s u_s, m_s v_s;
//   k_pair       O(N^2) star-star sweep: per star i the sums
//                         U_i  = sum_j G m_j / R_ij                (potential)
//                         G_i  = sum_j G m_j x_ij / R_ij^3         (= -g_i)
//                         Q_i  = sum_j (G m_j/R^3)[S'_ij x_ij - D'_ij v_j]
//                         C2_i = sum_j (G m_j/R^3) D'_ij        (stored / sqrt(3/2))
//                         Q7_i = sum_j (G m_j/R) (-b_j / 2)
//                       with S'_ij = e_j + 4 v_i.v_j + 3/2 (x_ij.v_j/R)^2
//                       - x_ij.b_j/2, e_j = -2 v_j^2 + u_j, and
//                       D'_ij = x_ij.(4 v_i - 3 v_j); written per j-split;
//   k_epilogue   O(N)   per star: reduces the splits, assembles the Newtonian
//                       and 1PN accelerations (Eqs. (4)-(6)), the star's term
//                       of the massive object's 1PN sum (Eqs. (2)-(3)) as block
//                       partials, and the Runge-Kutta stage update;
//   k_bh_final   O(N)   one block: the massive object's acceleration (Eq. (1))
//                       and stage update.
// The star-star 1PN sum of Eq. (6) needs no pass-1 result of any other star
// (only x, v, m and the O(N) massive-object terms u_j, b_j), so the potential
// sweep and the 1PN sweep share one pass over j.
//
// Runge-Kutta steps chain their evaluations: k_epilogue_chain also performs
// the next stage's prologue (each star's next state is in its registers), and
// k_pair_bh is the sweep with one extra workgroup doing the previous stage's
// k_bh_final work (the sweep reads only star packets), so a step is eight
// kernels.  Massive-object block rows hold 64 stars in every kernel, summed
// in the same tree, so whichever kernel writes a row it holds the same sum.
// For small systems k_stage runs a whole stage in one launch (each workgroup
// sums all j for a few stars and runs their epilogue; every workgroup
// recomputes the massive object's pending update), four kernels per step.
// Sums over a wavefront are folds or xor butterflies.
//
// The same four kernels instantiated on dual numbers (T = S = Dual) give the
// time derivative of the force along the motion (the jerk of the Hermite
// scheme), and their epilogue carries the Hermite corrector and predictor the
// way the FP64 one carries the Runge-Kutta stage update.  In a jerk
// evaluation the FP64 epilogue writes the dual packets (k_epilogue_chain<Dual>)
// and the dual epilogue carries the FP64 massive-object update
// (k_epilogue_dual_bh): six kernels.  Further down:
// Eqs. (7)-(8) diagnostics (k_diag_*), close-encounter search (k_enc_*),
// the unrestricted EIH equations (k_eih_*, reusing k_pair), and batched
// ensembles (k_*_batched: one launch per phase for many systems).
#pragma once

#include <hip/hip_runtime.h>
#include <climits>
#include <type_traits>
#include <stdint.h>

namespace pn {

constexpr int kBlock = 256;  // threads per workgroup (4 wave64)
constexpr int kProRows = kBlock / 64;  // prologue block rows per workgroup (one per 64 stars)
constexpr int kNF = 11;      // pair-sum fields: U, G(3), Q(3), C2, Q7(3)
enum Field { F_U = 0, F_G = 1, F_Q = 4, F_C2 = 7, F_Q7 = 8 };
enum PairMode { MODE_P1 = 1, MODE_P2 = 2, MODE_FUSED = 3 };

// Star packet read by the pair sweep.  Positions stay FP64 so that coordinate
// differences are formed in FP64 in both precisions.  The velocity is stored
// scaled, s = sqrt(3/2) v: then 3/2 (x.v_j / R)^2 = (x.s_j / R)^2, and with
// the per-i vector (4/sqrt(3/2)) v_i the other velocity products come out
// unscaled (4 v_i.v_j = [(4/sqrt(3/2)) v_i].s_j); D'_ij / sqrt(3/2) is
// accumulated and rescaled in the epilogue.  The FP64 packet holds s/2 (see
// PairScale below).
constexpr double kSqrt32 = 1.22474487139158904909864203735;    // sqrt(3/2)
constexpr double kInvSqrt32 = 0.816496580927726032732428024902; // 1/sqrt(3/2)

// Scalings of the pair sweep.  The FP64 sweep refines v_rsq_f64 by a Newton
// step written Y = y (3 - x y^2), which is 2/R (three instructions; the form
// that yields 1/R takes four), and carries the factor 2 through instead of
// removing it: its packets hold s/2, its i-vector is 2 (4/sqrt(3/2)) v_i, the
// D-term coefficient is -8, and a wavefront's sums come out as 2U, 8G, 8Q,
// 16 C2 and 2 Q7, scaled back when it flushes them.  Every factor is a power
// of two, so the FP64 sums are those of the unscaled terms bit for bit except
// for the reciprocal square root itself.  The FP32 and dual-number sweeps use
// 1/R as it is.
template <typename T> struct PairScale {
  static constexpr double sv = kSqrt32;         // packet velocity = sv v
  static constexpr double inv_sv = kInvSqrt32;  // v = inv_sv (packet velocity)
  static constexpr double k = 8.0 / 3.0;        // i-vector = k (packet velocity)
  static constexpr double d = -2.0;             // D term: d (x.s_j) + x.k_i
  static constexpr double u = 1.0, g = 1.0, q = 1.0, c2 = 1.0, q7 = 1.0;  // flush factors
};
template <> struct PairScale<double> {
  static constexpr double sv = 0.5 * kSqrt32;
  static constexpr double inv_sv = 2.0 * kInvSqrt32;
  static constexpr double k = 32.0 / 3.0;
  static constexpr double d = -8.0;
  static constexpr double u = 0.5, g = 0.125, q = 0.125, c2 = 0.0625, q7 = 0.5;
};

struct alignas(16) PkF64 {
  double x, y, z, gm, svx, svy, svz, e, hbx, hby, hbz, pad;
};
struct alignas(16) PkF32 {
  double x, y, z;
  float gm, svx, svy, svz, e, hbx, hby, hbz, pad0, pad1;
};
static_assert(sizeof(PkF64) == 96, "packet layout");
static_assert(sizeof(PkF32) == 64, "packet layout");

template <typename T> struct PkOf;
template <> struct PkOf<double> { using type = PkF64; };
template <> struct PkOf<float> { using type = PkF32; };

// ---------------------------------------------------------------------------
// Reciprocal square root in FP64.  The hardware estimate (v_rsq_f64) is good
// to about 2^-24 relative (measured: 5.2e-8 at worst); one step of the
// third-order series
//   1/sqrt(x) = y (1 - r)^(-1/2) = y (1 + r/2 + 3 r^2/8 + ...),  r = 1 - x y^2
// brings it to full double precision (residual ~ (5/16) r^3 < 2^-70).  The
// O(N) kernels (massive-object terms, epilogues) use this.
//
// The O(N^2) pair sweeps use one Newton step instead: y (1 + e) becomes
// y (1 + r/2) = y (1 - 3/2 e^2 - e^3/2), at most 4.1e-15 below the true value
// (the sweep's accuracy target is 1e-12; measured per-body errors stay at
// 1e-14).  Written y (3 - x y^2) it is twice that in three instructions, two
// fewer than the series.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double rsqrt_f64(double x) {
  double y = __builtin_amdgcn_rsq(x);
  double r = fma(-x * y, y, 1.0);
  double p = fma(0.375, r, 0.5);
  return fma(y * r, p, y);
}
__device__ __forceinline__ double rsqrt_f64_newton(double x) {
  double y = __builtin_amdgcn_rsq(x);
  double r = fma(-x * y, y, 1.0);
  return fma(y * r, 0.5, y);
}
// The same Newton step as 2/sqrt(x) = y (3 - x y^2): one instruction less.
__device__ __forceinline__ double rsqrt2_f64_newton(double x) {
  double y = __builtin_amdgcn_rsq(x);
  return y * fma(-x * y, y, 3.0);
}
__device__ __forceinline__ float rsqrt_t(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsqrt_t(double x) { return rsqrt_f64(x); }

// a*b + c with c wavefront-uniform (held in SGPRs).  For doubles the compiler
// otherwise copies c into a VGPR pair (two v_mov) to use the accumulating
// v_fmac form; one VOP3 v_fma_f64 with a scalar addend is the same operation.
__device__ __forceinline__ double fma_uniform_c(double a, double b, double c) {
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
  return r;
}
__device__ __forceinline__ float fma_uniform_c(float a, float b, float c) { return fmaf(a, b, c); }

// ---------------------------------------------------------------------------
// Forward-mode dual number v + d e (e^2 = 0).  Evaluating the force with every
// input replaced by (value, time derivative along the motion) -- positions
// (x, v), velocities (v, a) -- yields the acceleration in .v and its exact
// time derivative, the jerk, in .d (the Hermite scheme of Sec. 4-5 needs
// both).  Operators are hidden friends, so they never shadow the scalar
// overloads of fma & co. for plain doubles.
// ---------------------------------------------------------------------------
struct Dual {
  double v, d;
  Dual() = default;
  __host__ __device__ constexpr Dual(double x) : v(x), d(0.0) {}
  __host__ __device__ constexpr Dual(double x, double y) : v(x), d(y) {}
  friend __device__ __forceinline__ Dual operator+(Dual a, Dual b) { return {a.v + b.v, a.d + b.d}; }
  friend __device__ __forceinline__ Dual operator-(Dual a, Dual b) { return {a.v - b.v, a.d - b.d}; }
  friend __device__ __forceinline__ Dual operator-(Dual a) { return {-a.v, -a.d}; }
  friend __device__ __forceinline__ Dual operator*(Dual a, Dual b) {
    return {a.v * b.v, fma(a.v, b.d, a.d * b.v)};
  }
  friend __device__ __forceinline__ Dual operator*(double s, Dual b) { return {s * b.v, s * b.d}; }
  friend __device__ __forceinline__ Dual operator*(Dual b, double s) { return {b.v * s, b.d * s}; }
  friend __device__ __forceinline__ Dual operator/(Dual a, double s) { return {a.v / s, a.d / s}; }
  __device__ __forceinline__ Dual& operator+=(Dual b) {
    v += b.v;
    d += b.d;
    return *this;
  }
  __device__ __forceinline__ Dual& operator*=(double s) {
    v *= s;
    d *= s;
    return *this;
  }
  friend __device__ __forceinline__ Dual fma(Dual a, Dual b, Dual c) {
    return {fma(a.v, b.v, c.v), fma(a.v, b.d, fma(a.d, b.v, c.d))};
  }
};
// d(x^-1/2) = -x^-3/2 dx / 2
__device__ __forceinline__ Dual rsqrt_t(Dual x) {
  const double y = rsqrt_f64(x.v);
  return {y, -0.5 * y * y * y * x.d};
}
// the pair sweep's reciprocal square root (FP64: one Newton step, see rsqrt_f64,
// and 2/R rather than 1/R, see PairScale)
__device__ __forceinline__ float rsqrt_pair(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsqrt_pair(double x) { return rsqrt2_f64_newton(x); }

// Helpers that let the O(N) stages run on double or Dual: a Dual quantity
// stored in a row of width 2K keeps its value in column k and its derivative
// in column K + k.
template <typename T> struct IsDual { static constexpr bool value = false; };
template <> struct IsDual<Dual> { static constexpr bool value = true; };
template <typename T> struct Width { static constexpr int n = IsDual<T>::value ? 2 : 1; };
template <typename T> struct ScalarOf { using type = double; };  // O(N) arithmetic of a sweep type
template <> struct ScalarOf<Dual> { using type = Dual; };
template <typename T> struct PosOf { using type = double; };     // position type of a sweep type
template <> struct PosOf<Dual> { using type = Dual; };

__device__ __forceinline__ double val(double x) { return x; }
__device__ __forceinline__ double val(Dual x) { return x.v; }
__device__ __forceinline__ bool finite_s(double x) { return isfinite(x); }
__device__ __forceinline__ bool finite_s(Dual x) { return isfinite(x.v) && isfinite(x.d); }

// element i of a value array (and, for Dual, of its derivative array)
template <typename S> __device__ __forceinline__ S ld(const double* v, const double* d, size_t i);
template <> __device__ __forceinline__ double ld<double>(const double* v, const double*, size_t i) {
  return v[i];
}
template <> __device__ __forceinline__ Dual ld<Dual>(const double* v, const double* d, size_t i) {
  return Dual(v[i], d[i]);
}
// column k of a row holding K quantities
__device__ __forceinline__ void put(double* row, int k, int, double x) { row[k] = x; }
__device__ __forceinline__ void put(double* row, int k, int K, Dual x) {
  row[k] = x.v;
  row[K + k] = x.d;
}
template <typename S> __device__ __forceinline__ S get(const double* row, int k, int K);
template <> __device__ __forceinline__ double get<double>(const double* row, int k, int) {
  return row[k];
}
template <> __device__ __forceinline__ Dual get<Dual>(const double* row, int k, int K) {
  return Dual(row[k], row[K + k]);
}

// Star packet of the jerk sweep: every field with its time derivative.
struct alignas(16) PkDual {
  Dual x, y, z, gm, svx, svy, svz, e, hbx, hby, hbz;
};
static_assert(sizeof(PkDual) == 176, "packet layout");
template <> struct PkOf<Dual> { using type = PkDual; };
__device__ __forceinline__ void clear_pad(PkF64& p) { p.pad = 0.0; }
__device__ __forceinline__ void clear_pad(PkF32& p) { p.pad0 = p.pad1 = 0.f; }
__device__ __forceinline__ void clear_pad(PkDual&) {}

// A double from another lane of the same row of 16 by a DPP move (two 32-bit
// halves); CTRL: 0x141 lane i <- 7 - i within 8, 0x140 i <- 15 - i within 16,
// 0xB1 / 0x4E (quad permutations) i <- i ^ 1 / i ^ 2.
template <int CTRL>
__device__ __forceinline__ double dpp_d(double x) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xF, 0xF, true);
  const unsigned hi =
      (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// x plus the x of lane i ^ 16 (i ^ 32), by one row swap of each 32-bit half:
// v_permlane16_swap exchanges the odd rows of 16 of its first operand with the
// even rows of its second, so on two copies of x the first ends with the even
// row of each pair of rows in both, the second with the odd one
// (v_permlane32_swap: the same with halves of 32).  Both lanes add the same two
// values.
template <int M>
__device__ __forceinline__ double swap_sum(double x) {
  static_assert(M == 16 || M == 32, "row or half");
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = (unsigned)u, hi = (unsigned)(u >> 32);
  if constexpr (M == 16) {
    const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __builtin_bit_cast(double, ((unsigned long long)b[0] << 32) | a[0]) +
           __builtin_bit_cast(double, ((unsigned long long)b[1] << 32) | a[1]);
  } else {
    const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return __builtin_bit_cast(double, ((unsigned long long)b[0] << 32) | a[0]) +
           __builtin_bit_cast(double, ((unsigned long long)b[1] << 32) | a[1]);
  }
}

// Sum over the 64 lanes of a wavefront by six exchanges: lane i with 7 - i
// (within 8), i ^ 1, i ^ 2, 15 - i (within 16), i ^ 16, i ^ 32.  Both lanes
// of every exchange add the same two values, so after each level the lanes it
// joined hold the same bits, and at the end every lane holds the same sum; no
// barrier.  The first four levels are DPP moves within a row, the last two
// row swaps (swap_sum), all in the vector unit (through the LDS crossbar,
// ds_bpermute, those two levels cost a step 2.5 % at N = 100, 35.4 against 34.6
// us, and 1.3 % at N = 1024, 51.5 against 50.8).
template <int K>
__device__ __forceinline__ void wave_allsum(double (&v)[K]) {
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] += dpp_d<0x141>(v[k]);
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] += dpp_d<0xB1>(v[k]);
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] += dpp_d<0x4E>(v[k]);
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] += dpp_d<0x140>(v[k]);
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = swap_sum<16>(v[k]);
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = swap_sum<32>(v[k]);
}

// Sums over lanes 0 .. NS - 1 of a wavefront, in each of them.
template <int NS, int K>
__device__ __forceinline__ void star_sum(double (&v)[K]) {
  static_assert(NS == 2 || NS == 4 || NS == 8 || NS == 16, "stars per workgroup");
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] += dpp_d<0xB1>(v[k]);
  if constexpr (NS >= 4) {
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] += dpp_d<0x4E>(v[k]);
  }
  if constexpr (NS >= 8) {
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] += dpp_d<0x141>(v[k]);
  }
  if constexpr (NS >= 16) {
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] += dpp_d<0x140>(v[k]);
  }
}

// Element col of a register array, chosen per lane without indexing the
// array at run time (a chain of selects).
template <int K>
__device__ __forceinline__ double pick(const double (&v)[K], int col) {
  double r = 0.0;
#pragma unroll
  for (int k = 0; k < K; ++k) r = col == k ? v[k] : r;
  return r;
}

// Wave index as a scalar (so that loop bounds derived from it stay uniform
// and j packets keep coming through scalar loads).
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// Two values folded into one register of sums: the lanes with bit M clear end
// with x[i] + x[i ^ M], those with it set with the same sum of y (M = 32, 16: by
// a swap of halves or rows; 8, 4: by DPP moves within rows, written to the banks
// of four lanes that lack the value).  Reducing K values over a wavefront this
// way takes about as many additions as there are values, where summing each of
// them in all lanes takes one per value and level.
template <int M>
__device__ __forceinline__ double fold(double x, double y) {
  const unsigned long long ux = __builtin_bit_cast(unsigned long long, x);
  const unsigned long long uy = __builtin_bit_cast(unsigned long long, y);
  const unsigned xl = (unsigned)ux, xh = (unsigned)(ux >> 32);
  const unsigned yl = (unsigned)uy, yh = (unsigned)(uy >> 32);
  unsigned al, ah, bl, bh;
  if constexpr (M == 32) {
    const auto l = __builtin_amdgcn_permlane32_swap(xl, yl, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(xh, yh, false, false);
    al = l[0], bl = l[1], ah = h[0], bh = h[1];
  } else if constexpr (M == 16) {
    const auto l = __builtin_amdgcn_permlane16_swap(xl, yl, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(xh, yh, false, false);
    al = l[0], bl = l[1], ah = h[0], bh = h[1];
  } else {
    // a: x, with y shifted up by M in the lanes with bit M set; b: y, with x
    // shifted down in the others
    constexpr int set = M == 8 ? 0xC : 0xA, clear = M == 8 ? 0x3 : 0x5;
    al = __builtin_amdgcn_update_dpp((int)xl, (int)yl, 0x110 + M, 0xF, set, false);
    ah = __builtin_amdgcn_update_dpp((int)xh, (int)yh, 0x110 + M, 0xF, set, false);
    bl = __builtin_amdgcn_update_dpp((int)yl, (int)xl, 0x100 + M, 0xF, clear, false);
    bh = __builtin_amdgcn_update_dpp((int)yh, (int)xh, 0x100 + M, 0xF, clear, false);
  }
  return __builtin_bit_cast(double, ((unsigned long long)ah << 32) | al) +
         __builtin_bit_cast(double, ((unsigned long long)bh << 32) | bl);
}

// Twelve values reduced over the lanes that are NS apart: the lane's results
// r[0 .. fold_regs - 1] are the sums of the values f[0 ..] of residue lane % NS
// (f = -1: a copy of another lane's).
template <int NS>
constexpr int fold_regs() { return NS >= 16 ? 3 : NS == 8 ? 2 : 1; }
template <int NS>
__device__ __forceinline__ void fold12(const double (&x)[12], double (&r)[fold_regs<NS>()],
                                       int (&f)[fold_regs<NS>()]) {
  const int lane = threadIdx.x & 63;
  const int row = (lane >> 4 & 1) * 2 + (lane >> 5);  // which of four values a row of 16 holds
  double z[3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
    z[i] = fold<16>(fold<32>(x[4 * i], x[4 * i + 1]), fold<32>(x[4 * i + 2], x[4 * i + 3]));
  if constexpr (NS >= 16) {
#pragma unroll
    for (int i = 0; i < 3; ++i) r[i] = z[i], f[i] = 4 * i + row;
  } else {
    const int b8 = lane >> 3 & 1;
    const double u = fold<8>(z[0], z[1]), w = z[2] + dpp_d<0x128>(z[2]);
    if constexpr (NS == 8) {
      r[0] = u, f[0] = 4 * b8 + row;
      r[1] = w, f[1] = b8 ? -1 : 8 + row;
    } else {
      const int b4 = lane >> 2 & 1;
      r[0] = fold<4>(u, w);
      f[0] = !b4 ? 4 * b8 + row : b8 ? -1 : 8 + row;
      if constexpr (NS == 2) {
        r[0] += dpp_d<0x4E>(r[0]);  // lane ^ 2
        if (lane & 2) f[0] = -1;
      }
    }
  }
}

// Lane l's x, as a scalar.
__device__ __forceinline__ double lane_value(double x, int l) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)u, l);
  const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(u >> 32), l);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Ten values summed over a wavefront, as scalars.
__device__ __forceinline__ void sum10(double (&v)[10]) {
  const double x[12] = {v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8], v[9], 0.0, 0.0};
  double r[1];
  int f[1];
  fold12<2>(x, r, f);
  r[0] += dpp_d<0xB1>(r[0]);  // lane ^ 1: every lane now holds the whole sum of its value
#pragma unroll
  for (int k = 0; k < 10; ++k) {
    // a lane that holds value k: row of 16 by k % 4, then 8 or 4 by k / 4
    const int lane = (k & 1) * 32 + (k >> 1 & 1) * 16 + (k < 4 ? 0 : k < 8 ? 8 : 4);
    v[k] = lane_value(r[0], lane);
  }
}

// Sums over the wavefront, in every lane, ten at a time by folds: fewer
// instructions than wave_allsum (ten values of a wavefront alone: 0.3 us
// instead of 0.7), and the same additions for every value, so that the block
// sums of a chained epilogue, an epilogue alone and a prologue agree bit for
// bit.
template <int K>
__device__ __forceinline__ void wave_sum(double (&v)[K]) {
#pragma unroll
  for (int k0 = 0; k0 < K; k0 += 10) {
    double x[10];
#pragma unroll
    for (int k = 0; k < 10; ++k) x[k] = k0 + k < K ? v[k0 + k < K ? k0 + k : 0] : 0.0;
    sum10(x);
#pragma unroll
    for (int k = 0; k < 10; ++k)
      if (k0 + k < K) v[k0 + k < K ? k0 + k : 0] = x[k];
  }
}

// Sum of `rows` partial rows of width `stride` (first K columns), fixed order:
// lane l of every wavefront sums rows l, l+64, ..., then wave_sum.  Every
// thread of every workgroup ends with the same bits, without a barrier.
// Split in two so that a kernel can request the rows of several sums before
// waiting for any: rows_load (this lane's partial sums), then rows_sum.
// The lane's first row is loaded, not added, so that up to 64 rows (every
// system of up to 4096 stars) rows_load issues its loads and returns without
// waiting for them.
template <int K>
__device__ __forceinline__ void rows_load(const double* part, int rows, int stride,
                                          double (&v)[K]) {
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = 0.0;
  if (l < rows) {
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = part[(size_t)l * stride + k];
  }
  constexpr int U = K <= 8 ? 3 : 1;  // further rows in flight together
  for (int r = l + 64; r - l < rows; r += U * 64) {
    double w[U][K];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < K; ++k)
        w[u][k] = part[(size_t)min(r + 64 * u, rows - 1) * stride + k];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] += r + 64 * u < rows ? w[u][k] : 0.0;
  }
}
template <int K>
__device__ __forceinline__ void rows_sum(const double (&v)[K], double (&out)[K]) {
#pragma unroll
  for (int k = 0; k < K; ++k) out[k] = v[k];
  wave_sum<K>(out);
}
template <int K>
__device__ __forceinline__ void reduce_rows(const double* part, int rows, int stride,
                                            double (&out)[K]) {
  double v[K];
  rows_load<K>(part, rows, stride, v);
  rows_sum<K>(v, out);
}

// A call's status: two words, set to 1 where a thread finds the fault.  They are
// stored, not combined, so that they may lie in host memory, too: a call that
// waits for its result takes words there, which the host clears before and reads
// after it, and spares the launch that clears words on the device and the copy
// back (pn_accel, N = 300: 48.3 -> 32.1 us; pn_potential_accel and pn_correction,
// N = 6000: 172 -> 139; pn_accel_eih, N = 16384: 597 -> 555).
constexpr int kStatusNonfinite = 0, kStatusMass = 1, kStatusWords = 2;
__device__ __forceinline__ void raise_status(int* status, int word) {
  __hip_atomic_store(status + word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__global__ void k_reset_status(int* status) {
  if (threadIdx.x < kStatusWords) status[threadIdx.x] = 0;
}
// Words on the device to words in host memory, at the end of a call.
__global__ void k_report_status(const int* status, int* host) {
  if (threadIdx.x < kStatusWords)
    __hip_atomic_store(host + threadIdx.x, status[threadIdx.x], __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------------------
// Prologue: massive-object/star pair terms and star packets (O(N), FP64).
// ---------------------------------------------------------------------------
struct ProArgs {
  const double* pos;  // [N][3] (state of this evaluation)
  const double* vel;  // [N][3] or nullptr (Newtonian-only evaluation)
  const double* mass; // [N]
  int Ns;
  double G, eps2;
  void* pk;       // [Ns] packets (PkOf<T>)
  double* ub;     // [Ns][4 W]: u_s, b_s(3)
  double* bpart;  // [gridDim.x * kProRows][8 W]: per 64 stars sum m b (3), sum m u, sum m v (3), 0
  int* status;
  // jerk sweep (T = Dual): time derivatives of pos and vel (the velocity and
  // the acceleration of the evaluation state)
  const double* pos_d = nullptr;
  const double* vel_d = nullptr;
};

// Prologue terms of star k (body k + 1) at position xs, velocity vs, with the
// massive object at x0: writes the packet pk[k] and the row ub[k] = (u, b),
// and returns the star's block-sum terms v = (m b, m u, m v).  Shared by the
// prologue and by the Runge-Kutta epilogue that prepares the next evaluation.
template <typename T, typename S>
__device__ __forceinline__ void star_terms(const S (&x0)[3], const S (&xs)[3], const S (&vs)[3],
                                           double m, double G, double gM, double eps2, void* pk,
                                           double* ub_rows, int k, S (&v)[7]) {
  constexpr int W = Width<T>::n;
  const S dx = xs[0] - x0[0], dy = xs[1] - x0[1], dz = xs[2] - x0[2];
  const S rinv = rsqrt_t(fma(dz, dz, fma(dy, dy, fma(dx, dx, S(eps2)))));
  const S u = gM * rinv;
  const S b3 = u * rinv * rinv;
  const S bx = b3 * dx, by = b3 * dy, bz = b3 * dz;
  const S vx = vs[0], vy = vs[1], vz = vs[2];
  const S v2 = fma(vz, vz, fma(vy, vy, vx * vx));
  using Pk = typename PkOf<T>::type;
  Pk p;
  p.x = xs[0];
  p.y = xs[1];
  p.z = xs[2];
  p.gm = (T)(G * m);
  p.svx = (T)(PairScale<T>::sv * vx);
  p.svy = (T)(PairScale<T>::sv * vy);
  p.svz = (T)(PairScale<T>::sv * vz);
  p.e = (T)fma(S(-2.0), v2, u);
  p.hbx = (T)(-0.5 * bx);
  p.hby = (T)(-0.5 * by);
  p.hbz = (T)(-0.5 * bz);
  clear_pad(p);
  static_cast<Pk*>(pk)[k] = p;
  double* ub = ub_rows + 4 * W * (size_t)k;
  put(ub, 0, 4, u);
  put(ub, 1, 4, bx);
  put(ub, 2, 4, by);
  put(ub, 3, 4, bz);
  v[0] = m * bx;
  v[1] = m * by;
  v[2] = m * bz;
  v[3] = m * u;
  v[4] = m * vx;
  v[5] = m * vy;
  v[6] = m * vz;
}

// W = Width<T>::n doubles per quantity (value, and derivative for Dual).
template <typename T>
__device__ __forceinline__ void prologue_block(const ProArgs& a, int blk) {
  using S = typename ScalarOf<T>::type;
  constexpr int W = Width<T>::n;
  const int k = blk * kBlock + threadIdx.x;
  S v[7] = {0, 0, 0, 0, 0, 0, 0};
  if (k < a.Ns) {
    const int s = k + 1;
    const S x0[3] = {ld<S>(a.pos, a.pos_d, 0), ld<S>(a.pos, a.pos_d, 1),
                     ld<S>(a.pos, a.pos_d, 2)};
    const S xs[3] = {ld<S>(a.pos, a.pos_d, 3 * s), ld<S>(a.pos, a.pos_d, 3 * s + 1),
                     ld<S>(a.pos, a.pos_d, 3 * s + 2)};
    S vs[3] = {0.0, 0.0, 0.0};
    if (a.vel) {
      vs[0] = ld<S>(a.vel, a.vel_d, 3 * s);
      vs[1] = ld<S>(a.vel, a.vel_d, 3 * s + 1);
      vs[2] = ld<S>(a.vel, a.vel_d, 3 * s + 2);
    }
    star_terms<T, S>(x0, xs, vs, a.mass[s], a.G, a.G * a.mass[0], a.eps2, a.pk, a.ub, k, v);
  }
  // a block row per wavefront (64 stars), summed by wave_sum and written
  // from the wavefront's own registers
  double flat[7 * W];
#pragma unroll
  for (int q = 0; q < 7; ++q) put(flat, q, 7, v[q]);
  wave_sum<7 * W>(flat);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  if (l < 8 * W) {
    // row layout: value columns 0..7, derivative columns 8..15 (Dual)
    const int q = l & 7, h = l >> 3;
    a.bpart[((size_t)blk * kProRows + w) * 8 * W + l] = q < 7 ? pick(flat, h * 7 + q) : 0.0;
  }
  if (blk == 0 && threadIdx.x == 0) {
    const double M = a.mass[0];
    if (!(M > 0.0) || !isfinite(M)) raise_status(a.status, kStatusMass);
  }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_prologue(ProArgs a) {
  prologue_block<T>(a, blockIdx.x);
}

// ---------------------------------------------------------------------------
// Star-star sweep.  i-bodies live in registers (IPT per lane); every lane of a
// wavefront visits the same j at the same time, so the j packet is uniform and
// is read through the scalar unit into SGPRs (no LDS traffic, no per-lane
// broadcast).  A workgroup owns the i-range [ilo, ihi) and the j-range of one
// split (gridDim.y splits); with WS = 4 its four wavefronts share the i-range
// and divide the split's j-range into four pieces, reduced in LDS in fixed
// order at the end.  Partial sums go to part[split][field][star].
// T = double: FP64 throughout.  T = float: FP64 coordinate differences, FP32
// pair arithmetic, FP32 partial sums over tiles of kTile j added into FP64
// accumulators after each tile.  T = Dual: the FP64 sweep on dual numbers,
// 2 kNF fields per star (values, then their time derivatives).
// ---------------------------------------------------------------------------
struct PairArgs {
  const void* pk;
  int Ns;
  int jchunk;  // j per split
  double eps2;
  double* part;  // [gridDim.y][kNF W][Ns]
};

constexpr int kTile = 64;  // j per FP32 partial-sum tile (mixed precision)

template <typename T, int IPT>
struct PairAcc {
  T U[IPT], Gx[IPT], Gy[IPT], Gz[IPT], Qx[IPT], Qy[IPT], Qz[IPT], C2[IPT], Q7x[IPT], Q7y[IPT],
      Q7z[IPT];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
      U[i] = Gx[i] = Gy[i] = Gz[i] = Qx[i] = Qy[i] = Qz[i] = C2[i] = Q7x[i] = Q7y[i] = Q7z[i] = T(0);
    }
  }
};

template <typename T, int IPT>
struct PairI {  // the i-side operands of one lane
  typename PosOf<T>::type x[IPT], y[IPT], z[IPT];
  T kx[IPT], ky[IPT], kz[IPT];  // (4/sqrt(3/2)) v_i
  int idx[IPT];
};

// The jerk sweep's pair: pair_one (below) on dual numbers, in fewer operations.  Written on Dual values, every product with a power of
// 1/R carries that power's own derivative (and that of G m, which is zero), 128
// vector operations per pair.  The derivatives of all powers are one number
// apart: with l = (d/dt) ln(1/R) = -(x.x')/R^2,
//   (m/R^n)' = n l (m/R^n),  (m x/R^3)' = (m/R^3) (3 l x + x'),
// and w = 3 l x + x' serves G and the S term of Q alike: 112 operations.  The
// sweep is bound by vector issue: with it a Hermite step at N = 16384 takes
// 1.467 ms instead of 1.585, at N = 4097 133 us instead of 141 (same splits).
template <int MODE, int IPT, bool MASK>
__device__ __forceinline__ void pair_one_dual(const PkDual& p, int j, double eps2,
                                              const PairI<Dual, IPT>& I, PairAcc<Dual, IPT>& A) {
  static_assert(MODE == MODE_FUSED, "the jerk sweep is fused");
  using SC = PairScale<Dual>;
#pragma unroll
  for (int ii = 0; ii < IPT; ++ii) {
    const Dual dx = I.x[ii] - p.x, dy = I.y[ii] - p.y, dz = I.z[ii] - p.z;
    double y = rsqrt_f64_newton(fma(dz.v, dz.v, fma(dy.v, dy.v, fma(dx.v, dx.v, eps2))));
    if (MASK) y = (j == I.idx[ii]) ? 0.0 : y;
    const double y2 = y * y;
    const double l = -(y2 * fma(dz.v, dz.d, fma(dy.v, dy.d, dx.v * dx.d))), l3 = 3.0 * l;
    const double m = p.gm.v * y, md = m * l, m3 = m * y2;
    A.U[ii].v += m;
    A.U[ii].d += md;
    const double wx = fma(l3, dx.v, dx.d), wy = fma(l3, dy.v, dy.d), wz = fma(l3, dz.v, dz.d);
    A.Gx[ii].v = fma(m3, dx.v, A.Gx[ii].v);
    A.Gy[ii].v = fma(m3, dy.v, A.Gy[ii].v);
    A.Gz[ii].v = fma(m3, dz.v, A.Gz[ii].v);
    A.Gx[ii].d = fma(m3, wx, A.Gx[ii].d);
    A.Gy[ii].d = fma(m3, wy, A.Gy[ii].d);
    A.Gz[ii].d = fma(m3, wz, A.Gz[ii].d);
    const Dual sx = p.svx, sy = p.svy, sz = p.svz;  // sqrt(3/2) v_j
    const Dual xs = fma(dz, sz, fma(dy, sy, dx * sx));
    const double t = xs.v * y, td = fma(t, l, xs.d * y);
    // S: e_j + 3/2 (x.v_j/R)^2 + 4 v_i.v_j - x.b_j / 2
    Dual s(fma_uniform_c(t, t, p.e.v), fma_uniform_c(t + t, td, p.e.d));
    s = fma(I.kz[ii], sz, fma(I.ky[ii], sy, fma(I.kx[ii], sx, s)));
    s = fma(dz, p.hbz, fma(dy, p.hby, fma(dx, p.hbx, s)));
    const Dual x4 = fma(dz, I.kz[ii], fma(dy, I.ky[ii], dx * I.kx[ii]));
    const double D = fma(SC::d, xs.v, x4.v), Dd = fma(SC::d, xs.d, x4.d);
    const double c1 = m3 * s.v, c1d = m3 * s.d, c2 = m3 * D, c2d = m3 * fma(l3, D, Dd);
    A.Qx[ii].v = fma(-c2, sx.v, fma(c1, dx.v, A.Qx[ii].v));
    A.Qy[ii].v = fma(-c2, sy.v, fma(c1, dy.v, A.Qy[ii].v));
    A.Qz[ii].v = fma(-c2, sz.v, fma(c1, dz.v, A.Qz[ii].v));
    A.Qx[ii].d = fma(-c2, sx.d, fma(-c2d, sx.v, fma(c1, wx, fma(c1d, dx.v, A.Qx[ii].d))));
    A.Qy[ii].d = fma(-c2, sy.d, fma(-c2d, sy.v, fma(c1, wy, fma(c1d, dy.v, A.Qy[ii].d))));
    A.Qz[ii].d = fma(-c2, sz.d, fma(-c2d, sz.v, fma(c1, wz, fma(c1d, dz.v, A.Qz[ii].d))));
    A.C2[ii].v += c2;
    A.C2[ii].d += c2d;
    A.Q7x[ii].v = fma(m, p.hbx.v, A.Q7x[ii].v);
    A.Q7y[ii].v = fma(m, p.hby.v, A.Q7y[ii].v);
    A.Q7z[ii].v = fma(m, p.hbz.v, A.Q7z[ii].v);
    A.Q7x[ii].d = fma(m, p.hbx.d, fma(md, p.hbx.v, A.Q7x[ii].d));
    A.Q7y[ii].d = fma(m, p.hby.d, fma(md, p.hby.v, A.Q7y[ii].d));
    A.Q7z[ii].d = fma(m, p.hbz.d, fma(md, p.hbz.v, A.Q7z[ii].d));
  }
}

template <typename T, int MODE, int IPT, bool MASK>
__device__ __forceinline__ void pair_one(const typename PkOf<T>::type& p, int j, T eps2,
                                         const PairI<T, IPT>& I, PairAcc<T, IPT>& A) {
  using P = typename PosOf<T>::type;
  const P xj = p.x, yj = p.y, zj = p.z;
  const T gm = p.gm;
#pragma unroll
  for (int ii = 0; ii < IPT; ++ii) {
    const T dx = (T)(I.x[ii] - xj), dy = (T)(I.y[ii] - yj), dz = (T)(I.z[ii] - zj);
    T rinv = rsqrt_pair(fma(dz, dz, fma(dy, dy, fma(dx, dx, eps2))));
    if (MASK) rinv = (j == I.idx[ii]) ? T(0) : rinv;
    const T rinv2 = rinv * rinv;
    const T mr = gm * rinv;
    const T mr3 = mr * rinv2;
    if (MODE & MODE_P1) A.U[ii] += mr;
    A.Gx[ii] = fma(mr3, dx, A.Gx[ii]);
    A.Gy[ii] = fma(mr3, dy, A.Gy[ii]);
    A.Gz[ii] = fma(mr3, dz, A.Gz[ii]);
    if (MODE & MODE_P2) {
      const T sx = p.svx, sy = p.svy, sz = p.svz;  // sqrt(3/2) v_j
      const T xs = fma(dz, sz, fma(dy, sy, dx * sx));
      const T t = xs * rinv;
      T s = fma_uniform_c(t, t, (T)p.e);           // e_j + 3/2 (x.v_j/R)^2
      s = fma(I.kz[ii], sz, fma(I.ky[ii], sy, fma(I.kx[ii], sx, s)));  // + 4 v_i.v_j
      s = fma(dz, (T)p.hbz, fma(dy, (T)p.hby, fma(dx, (T)p.hbx, s)));  // - x.b_j / 2
      const T x4 = fma(dz, I.kz[ii], fma(dy, I.ky[ii], dx * I.kx[ii]));
      const T D = fma(T(PairScale<T>::d), xs, x4);  // x.(4 v_i - 3 v_j) / sqrt(3/2)
      const T c1 = mr3 * s, c2 = mr3 * D;
      A.Qx[ii] = fma(-c2, sx, fma(c1, dx, A.Qx[ii]));
      A.Qy[ii] = fma(-c2, sy, fma(c1, dy, A.Qy[ii]));
      A.Qz[ii] = fma(-c2, sz, fma(c1, dz, A.Qz[ii]));
      A.C2[ii] += c2;
      A.Q7x[ii] = fma(mr, (T)p.hbx, A.Q7x[ii]);
      A.Q7y[ii] = fma(mr, (T)p.hby, A.Q7y[ii]);
      A.Q7z[ii] = fma(mr, (T)p.hbz, A.Q7z[ii]);
    }
  }
}

template <typename T, int MODE, int IPT, bool MASK>
__device__ __forceinline__ void pair_step(const typename PkOf<T>::type& p, int j, T eps2,
                                          const PairI<T, IPT>& I, PairAcc<T, IPT>& A) {
  if constexpr (IsDual<T>::value) pair_one_dual<MODE, IPT, MASK>(p, j, eps2.v, I, A);
  else pair_one<T, MODE, IPT, MASK>(p, j, eps2, I, A);
}

// j loop over [j0, j1).
template <typename T, int MODE, int IPT, bool MASK>
__device__ __forceinline__ void pair_range(const typename PkOf<T>::type* __restrict__ pk, int j0,
                                           int j1, T eps2, const PairI<T, IPT>& I,
                                           PairAcc<T, IPT>& A) {
  using Pk = typename PkOf<T>::type;
  int j = j0;
  // FP64: four j per iteration (the same order of additions, 1-2 % faster
  // than two); FP32 keeps two, where four cost occupancy
  if constexpr (sizeof(T) == 8) {
    for (; j + 3 < j1; j += 4) {
      const Pk p0 = pk[j];
      const Pk p1 = pk[j + 1];
      const Pk p2 = pk[j + 2];
      const Pk p3 = pk[j + 3];
      pair_step<T, MODE, IPT, MASK>(p0, j, eps2, I, A);
      pair_step<T, MODE, IPT, MASK>(p1, j + 1, eps2, I, A);
      pair_step<T, MODE, IPT, MASK>(p2, j + 2, eps2, I, A);
      pair_step<T, MODE, IPT, MASK>(p3, j + 3, eps2, I, A);
    }
  }
  // two j per iteration: two independent dependency chains per wavefront
  for (; j + 1 < j1; j += 2) {
    const Pk p0 = pk[j];
    const Pk p1 = pk[j + 1];
    pair_step<T, MODE, IPT, MASK>(p0, j, eps2, I, A);
    pair_step<T, MODE, IPT, MASK>(p1, j + 1, eps2, I, A);
  }
  if (j < j1) pair_step<T, MODE, IPT, MASK>(pk[j], j, eps2, I, A);
}

template <typename T, int MODE, int IPT>
__device__ __forceinline__ void pair_segment(const typename PkOf<T>::type* __restrict__ pk, int j0,
                                             int j1, int ilo, int ihi, T eps2,
                                             const PairI<T, IPT>& I, PairAcc<T, IPT>& A) {
  // the diagonal j == i can only occur for j in [ilo, ihi)
  const int m0 = max(j0, ilo), m1 = min(j1, ihi);
  if (m0 < m1) {
    pair_range<T, MODE, IPT, false>(pk, j0, m0, eps2, I, A);
    pair_range<T, MODE, IPT, true>(pk, m0, m1, eps2, I, A);
    pair_range<T, MODE, IPT, false>(pk, m1, j1, eps2, I, A);
  } else {
    pair_range<T, MODE, IPT, false>(pk, j0, j1, eps2, I, A);
  }
}

// acc[f] += s x (and acc[kNF + f] += s dx/dt for Dual); s is a PairScale
// factor, a power of two (1 outside the FP64 sweep)
template <int NFO, int IPT>
__device__ __forceinline__ void acc_add(double (&acc)[NFO][IPT], int f, int ii, float x, double s) {
  acc[f][ii] += (double)x * s;
}
template <int NFO, int IPT>
__device__ __forceinline__ void acc_add(double (&acc)[NFO][IPT], int f, int ii, double x,
                                        double s) {
  acc[f][ii] += x * s;
}
template <int NFO, int IPT>
__device__ __forceinline__ void acc_add(double (&acc)[NFO][IPT], int f, int ii, Dual x, double s) {
  acc[f][ii] += x.v * s;
  acc[kNF + f][ii] += x.d * s;
}

template <typename T, int IPT, int NFO>
__device__ __forceinline__ void acc_flush(const PairAcc<T, IPT>& A, double (&acc)[NFO][IPT]) {
#pragma unroll
  for (int ii = 0; ii < IPT; ++ii) {
    using SC = PairScale<T>;
    acc_add(acc, F_U, ii, A.U[ii], SC::u);
    acc_add(acc, F_G, ii, A.Gx[ii], SC::g);
    acc_add(acc, F_G + 1, ii, A.Gy[ii], SC::g);
    acc_add(acc, F_G + 2, ii, A.Gz[ii], SC::g);
    acc_add(acc, F_Q, ii, A.Qx[ii], SC::q);
    acc_add(acc, F_Q + 1, ii, A.Qy[ii], SC::q);
    acc_add(acc, F_Q + 2, ii, A.Qz[ii], SC::q);
    acc_add(acc, F_C2, ii, A.C2[ii], SC::c2);
    acc_add(acc, F_Q7, ii, A.Q7x[ii], SC::q7);
    acc_add(acc, F_Q7 + 1, ii, A.Q7y[ii], SC::q7);
    acc_add(acc, F_Q7 + 2, ii, A.Q7z[ii], SC::q7);
  }
}

__device__ __forceinline__ bool field_written(int f, int mode) {
  f %= kNF;  // derivative fields of the jerk sweep follow the value fields
  if (f == F_U) return (mode & MODE_P1) != 0;
  if (f < F_Q) return true;
  return (mode & MODE_P2) != 0;
}

// Threads of a sweep workgroup: WS wavefronts sharing one i-range of 64 IPT
// lanes (WS = 4 or 8), or 256 lanes (WS = 1).
template <int WS>
constexpr int pair_threads() {
  return WS == 8 ? 2 * kBlock : kBlock;
}

// LDS of pair_block's wavefront reduction: WS = 4, waves 1-3 park their sums;
// WS = 8, waves 4-7 then waves 1-3 (the same four regions).
template <typename T, int IPT, int WS>
constexpr int pair_red_doubles() {
  return WS > 1 ? (WS == 8 ? 4 : WS - 1) * kNF * Width<T>::n * IPT * 64 : 1;
}

// red: pair_red_doubles<T, IPT, WS>() doubles of LDS
template <typename T, int MODE, int IPT, int WS>
__device__ __forceinline__ void pair_block(const PairArgs& a, int ib, int sp, double* red) {
  using Pk = typename PkOf<T>::type;
  constexpr int NFO = kNF * Width<T>::n;  // output fields per star
  static_assert(WS == 1 || WS == 4 || WS == 8, "wavefronts per i-range");
  constexpr int LANES = pair_threads<WS>() / WS;  // distinct i-lanes per workgroup
  constexpr int IB = LANES * IPT;     // i-bodies per workgroup
  const Pk* __restrict__ pk = static_cast<const Pk*>(a.pk);
  const int wave = WS > 1 ? wave_id() : 0;
  const int lane = WS > 1 ? (int)(threadIdx.x & 63) : (int)threadIdx.x;
  const int ilo = ib * IB;
  const int ihi = min(a.Ns, ilo + IB);
  // j-range of this wavefront
  int j0 = sp * a.jchunk;
  int j1 = min(a.Ns, j0 + a.jchunk);
  if (WS > 1) {
    const int q = (j1 - j0 + WS - 1) / WS;
    const int w0 = min(j1, j0 + wave * q);
    j1 = min(j1, w0 + q);
    j0 = w0;
  }
  // One load per 128 bytes of this wavefront's packets, not used: the epilogue
  // that wrote them ran on other XCDs, so each line's first scalar load would go
  // past this XCD's L2, one round trip after the other.  us per RK4 step
  // without and with it: FP64 N = 1200 50.9, 48.1; 3000 117.7, 108.5; 6000 271,
  // 260; 10001 627, 612; 16384 the same; mixed 1200 61.5, 49.5; 5000 160, 139;
  // 10001 471, 431; 30000 3190, 3156; at 2300, 6000 and 8192 mixed about 1 %
  // slower.  Runs of more than twice the 64 lines have enough to do meanwhile
  // (one line then; with all of them N = 65536 mixed takes 0.5 % longer).
  const int run = (j1 - j0) * (int)sizeof(Pk);
  const unsigned touched = *reinterpret_cast<const unsigned*>(
      reinterpret_cast<const char*>(pk + min(j0, a.Ns - 1)) +  // (no j: some packet)
      min((run <= 2 * 64 * 128 ? 128 : 0) * (int)(threadIdx.x & 63), max(0, run - 4)));
  PairI<T, IPT> I;
#pragma unroll
  for (int ii = 0; ii < IPT; ++ii) {
    I.idx[ii] = ilo + lane + ii * LANES;
    const int il = min(I.idx[ii], a.Ns - 1);  // lanes past the end compute on a copy, never stored
    const Pk& p = pk[il];
    I.x[ii] = p.x;
    I.y[ii] = p.y;
    I.z[ii] = p.z;
    // (4/sqrt(3/2)) v_i = (8/3) s_i (times 2 in FP64, see PairScale)
    I.kx[ii] = T(PairScale<T>::k) * (T)p.svx;
    I.ky[ii] = T(PairScale<T>::k) * (T)p.svy;
    I.kz[ii] = T(PairScale<T>::k) * (T)p.svz;
  }
  const T eps2 = (T)a.eps2;

  double acc[NFO][IPT];
#pragma unroll
  for (int f = 0; f < NFO; ++f)
#pragma unroll
    for (int ii = 0; ii < IPT; ++ii) acc[f][ii] = 0.0;

  PairAcc<T, IPT> A;
  if constexpr (sizeof(T) != 4) {
    A.zero();
    pair_segment<T, MODE, IPT>(pk, j0, j1, ilo, ihi, eps2, I, A);
    acc_flush(A, acc);
  } else {
    for (int t0 = j0; t0 < j1; t0 += kTile) {
      const int t1 = min(j1, t0 + kTile);
      A.zero();
      pair_segment<T, MODE, IPT>(pk, t0, t1, ilo, ihi, eps2, I, A);
      acc_flush(A, acc);
    }
  }

  asm volatile("" ::"v"(touched));
  const size_t plane = (size_t)a.Ns;
  double* out = a.part + (size_t)sp * NFO * plane;
  if constexpr (WS == 1) {
#pragma unroll
    for (int ii = 0; ii < IPT; ++ii) {
      if (I.idx[ii] < a.Ns) {
#pragma unroll
        for (int f = 0; f < NFO; ++f)
          if (field_written(f, MODE)) out[f * plane + I.idx[ii]] = acc[f][ii];
      }
    }
  } else {
    // fixed-order reduction over the WS wavefronts: waves 1..WS-1 park their
    // sums in LDS, wave 0 adds them to its own in wave order and stores
    // (LDS of WS-1 waves only, so it does not cap the occupancy).  WS = 8:
    // first wave w < 4 adds wave w + 4's sums to its own.
    if constexpr (WS == 8) {
      if (wave >= 4) {
#pragma unroll
        for (int f = 0; f < NFO; ++f)
#pragma unroll
          for (int ii = 0; ii < IPT; ++ii)
            red[(((wave - 4) * NFO + f) * IPT + ii) * 64 + lane] = acc[f][ii];
      }
      __syncthreads();
      if (wave < 4) {
#pragma unroll
        for (int f = 0; f < NFO; ++f)
#pragma unroll
          for (int ii = 0; ii < IPT; ++ii)
            acc[f][ii] += red[((wave * NFO + f) * IPT + ii) * 64 + lane];
      }
      __syncthreads();
    }
    if (wave > 0 && wave < 4) {
#pragma unroll
      for (int f = 0; f < NFO; ++f)
#pragma unroll
        for (int ii = 0; ii < IPT; ++ii)
          red[(((wave - 1) * NFO + f) * IPT + ii) * 64 + lane] = acc[f][ii];
    }
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int ii = 0; ii < IPT; ++ii) {
        const int idx = ilo + lane + ii * 64;
        if (idx < a.Ns) {
#pragma unroll
          for (int f = 0; f < NFO; ++f) {
            if (field_written(f, MODE)) {
              double sum = acc[f][ii];
#pragma unroll
              for (int w = 1; w < 4; ++w) sum += red[(((w - 1) * NFO + f) * IPT + ii) * 64 + lane];
              out[f * plane + idx] = sum;
            }
          }
        }
      }
    }
  }
}

template <typename T, int MODE, int IPT, int WS>
__global__ __launch_bounds__(pair_threads<WS>()) void k_pair(PairArgs a) {
  __shared__ double red[pair_red_doubles<T, IPT, WS>()];
  pair_block<T, MODE, IPT, WS>(a, blockIdx.x, blockIdx.y, red);
}

// ---------------------------------------------------------------------------
// Epilogue (per star) and final step (massive object).
// ---------------------------------------------------------------------------
struct EpiArgs {
  const double* pos;  // [N][3] state of this evaluation
  const double* vel;  // [N][3] (may be nullptr when newton_only)
  const double* mass;
  int Ns;
  double G, lam, eps2;
  const double* ub;     // [Ns][4 W]
  const double* bpart;  // prologue partials [nbpro][8 W]
  int nbpro;
  const double* part;  // pair partials [nsplit][kNF W][Ns]
  int nsplit;
  int newton_only;      // skip every 1PN term
  const double* phi_in; // correction mode: Newtonian potential of all N bodies (else nullptr)
  const double* accN_in;// correction mode: Newtonian acceleration of all N bodies
  double* acc_newton;   // outputs, [N][3] / [N] (any may be nullptr)
  double* phi;
  double* acc_1pn;
  double* bhpart;  // [gridDim.x][4 W]: the massive object's 1PN sum, block partials
  int nbepi;       // (k_bh_final) number of bhpart rows
  int* status;
  // Runge-Kutta stage update (stage < 0: none)
  int stage;
  double dt;
  double *X, *V, *Xs, *Vs, *KX, *KV;  // [N][3]
  double* acc_tot = nullptr;  // total acceleration [N][3] (optional)
  // jerk evaluation (S = Dual): derivatives of pos and vel, and the jerk [N][3]
  const double* pos_d = nullptr;
  const double* vel_d = nullptr;
  double* jerk = nullptr;
  // Hermite update (herm < 0: none, 0: first evaluation, 1: evaluation at
  // the predicted state): acceleration and jerk kept between steps, and the
  // next predicted state, all [N][3]
  int herm = -1;
  double *HA = nullptr, *HJ = nullptr, *XP = nullptr, *VP = nullptr;
  // chained Runge-Kutta stages (k_epilogue_chain): the next evaluation's
  // packets, u/b rows and block-sum rows (one per epilogue workgroup)
  void* pk_next = nullptr;
  double* ub_next = nullptr;
  double* bpart_next = nullptr;
};

// Classical RK4 bookkeeping for one body component.  The evaluation state of
// stage 0 is (X, V); of stages 1-3 it is (Xs, Vs).  KX/KV accumulate
// k1 + 2 k2 + 2 k3; stage 3 applies y += dt/6 (k1 + 2 k2 + 2 k3 + k4).
// rk4_next gives the component of the next evaluation state (stage 3: the new
// step's state) from the stage derivative k and the step-start value Y; the
// same function serves position and velocity, and the epilogue uses it for
// the massive object's next position too, so that every thread derives that
// position bit for bit as k_bh_final does.
__device__ __forceinline__ double rk4_next(int stage, double dt, double Y, double K, double k) {
  switch (stage) {
    case 0:
    case 1:
      return Y + 0.5 * dt * k;
    case 2:
      return Y + dt * k;
    default:
      return Y + dt / 6.0 * (K + k);
  }
}
// A kernel-argument pointer the compiler may not trace back to its field:
// otherwise it merges stores through X or Xs into one store through a pointer
// selected from a copy of the arguments in scratch memory.
__device__ __forceinline__ double* uniform_ptr(double* p) {
  asm volatile("" : "+s"(p));
  return p;
}

// The step-start state (X, V) and the accumulated stage sums (KX, KV) of one
// body component, read ahead of their use (a kernel requests all its global
// reads up front so that their latencies overlap).
struct Rk4In {
  double X = 0.0, V = 0.0, KX = 0.0, KV = 0.0;
};
__device__ __forceinline__ Rk4In rk4_load(const EpiArgs& a, size_t o) {
  Rk4In r;
  if (a.stage < 0 || a.stage > 3) return r;
  r.X = a.X[o];
  r.V = a.V[o];
  if (a.stage > 0) {
    r.KX = a.KX[o];
    r.KV = a.KV[o];
  }
  return r;
}
// xv: velocity of the evaluation state (the position derivative k_x); returns
// the next evaluation state's position and velocity component in xn, vn.
__device__ __forceinline__ void rk4_update(const EpiArgs& a, size_t o, const Rk4In& in,
                                           double xv, double acc, double& xn, double& vn) {
  if (a.stage < 0 || a.stage > 3) return;
  const double KX = in.KX, KV = in.KV;
  xn = rk4_next(a.stage, a.dt, in.X, KX, xv);
  vn = rk4_next(a.stage, a.dt, in.V, KV, acc);
  if (a.stage < 3) {
    a.KX[o] = a.stage == 0 ? xv : KX + 2.0 * xv;
    a.KV[o] = a.stage == 0 ? acc : KV + 2.0 * acc;
    uniform_ptr(a.Xs)[o] = xn;
    uniform_ptr(a.Vs)[o] = vn;
  } else {
    uniform_ptr(a.X)[o] = xn;
    uniform_ptr(a.V)[o] = vn;
  }
}

// Fourth-order Hermite bookkeeping for one body component, from the
// acceleration ap and jerk jp of the evaluation state.  herm 0 (state
// (X, V)): keeps a = ap, j = jp; snap and crackle are zero.  herm 1 (state
// (XP, VP), the prediction): corrector
//   v' = v + (a + ap) dt/2 + (j - jp) dt^2/12,
//   x' = x + (v + v') dt/2 + (a - ap) dt^2/12,
// snap and crackle at the step's end from the Hermite interpolant of a,
//   k = (12 (a - ap) + 6 dt (j + jp)) / dt^3,
//   s = (-6 (a - ap) - dt (4 j + 2 jp)) / dt^2 + k dt,
// then a = ap, j = jp.  Both cases predict the next evaluation state
//   XP = x + v dt + a dt^2/2 + j dt^3/6 + s dt^4/24 + k dt^5/120,
//   VP = v + a dt + j dt^2/2 + s dt^3/6 + k dt^4/24.
// (The velocity-dependent 1PN force is why the predictor carries s and k: a
// velocity predicted to O(dt^3) only would cap the scheme at third order.)
__device__ __forceinline__ void hermite_update(const EpiArgs& a, size_t o, double ap, double jp) {
  const double dt = a.dt, dt2 = dt * dt, dt3 = dt2 * dt, dt4 = dt3 * dt, dt5 = dt4 * dt;
  double x = a.X[o], v = a.V[o], sn = 0.0, cr = 0.0;
  if (a.herm == 1) {
    const double a0 = a.HA[o], j0 = a.HJ[o];
    const double vn = v + dt / 2.0 * (a0 + ap) + dt2 / 12.0 * (j0 - jp);
    x = x + dt / 2.0 * (v + vn) + dt2 / 12.0 * (a0 - ap);
    v = vn;
    cr = (12.0 * (a0 - ap) + 6.0 * dt * (j0 + jp)) / dt3;
    sn = (-6.0 * (a0 - ap) - dt * (4.0 * j0 + 2.0 * jp)) / dt2 + cr * dt;
    a.X[o] = x;
    a.V[o] = v;
  }
  a.HA[o] = ap;
  a.HJ[o] = jp;
  a.XP[o] = x + dt * v + dt2 / 2.0 * ap + dt3 / 6.0 * jp + dt4 / 24.0 * sn + dt5 / 120.0 * cr;
  a.VP[o] = v + dt * ap + dt2 / 2.0 * jp + dt3 / 6.0 * sn + dt4 / 24.0 * cr;
}

// The massive object's acceleration A0 = a^N_0, potential magnitude V0 = -phi_0
// and the star momentum P, from the prologue partials (or the caller's inputs).
template <typename S>
constexpr int bh_cols() { return IsDual<S>::value ? 16 : 7; }  // columns read per prologue row

// rows: this thread's partial sums of the prologue rows (rows_load)
template <typename S>
__device__ __forceinline__ void bh_quantities(const EpiArgs& a,
                                              const double (&rows)[bh_cols<S>()], S (&A0)[3],
                                              S& V0, S (&P)[3]) {
  constexpr int K = bh_cols<S>();
  double r[K];
  rows_sum<K>(rows, r);
  const double iM = 1.0 / a.mass[0];  // one division for the four quotients
  A0[0] = get<S>(r, 0, 8) * iM;
  A0[1] = get<S>(r, 1, 8) * iM;
  A0[2] = get<S>(r, 2, 8) * iM;
  V0 = get<S>(r, 3, 8) * iM;
  P[0] = get<S>(r, 4, 8);
  P[1] = get<S>(r, 5, 8);
  P[2] = get<S>(r, 6, 8);
  if constexpr (!IsDual<S>::value) {
    if (a.phi_in) {
      V0 = -a.phi_in[0];
      A0[0] = a.accN_in[0];
      A0[1] = a.accN_in[1];
      A0[2] = a.accN_in[2];
    }
  }
}

constexpr int kEpiStars = 64;  // stars per epilogue workgroup
// Split ranges of an epilogue workgroup's sums and its wavefronts: four sum each
// range, side by side, and one more runs the epilogue.  (The dual epilogue's needs
// more than 168 registers per lane, of which nine wavefronts fit a CU: one range.)
// With five the ranges are summed one after the other; with four, too, and the
// last wavefront, which has the fewest fields, then runs the epilogue.  The sums
// are the same.
template <typename S>
constexpr int epi_ranges() { return IsDual<S>::value ? 1 : 2; }
template <typename S>
constexpr int epi_waves() { return 4 * epi_ranges<S>() + 1; }
template <typename S>
constexpr int epi_threads() { return 64 * epi_waves<S>(); }
template <typename S>
constexpr int epi_fsum() { return kNF * Width<S>::n * kEpiStars * epi_ranges<S>(); }

__device__ __forceinline__ bool epi_field_used(int f, const EpiArgs& a) {
  f %= kNF;
  if (f == F_U) return a.phi_in == nullptr;  // correction mode: U is not computed
  if (f < F_Q) return true;
  return !a.newton_only;
}

// S = double: the evaluation; S = Dual: the same arithmetic on dual numbers
// (acceleration and jerk).  PkT (S = double only): also the next sweep's
// prologue into pk_next, ub_next and bpart_next (packets of PkOf<PkT>):
// double / float, a Runge-Kutta stage's, from each star's next state and the
// massive object's next position; Dual, the jerk sweep's at this state, with
// the derivatives (v, a) of (x, v) from the acceleration just computed.
// void: none.

// A star's own inputs, read ahead of their use.
template <typename S>
struct EpiStar {
  S u = 0.0, bx = 0.0, by = 0.0, bz = 0.0, x = 0.0, y = 0.0, z = 0.0;
  S v[3] = {0.0, 0.0, 0.0};
  double m_s = 0.0;  // the star's mass (G m is formed where it is used, after the loads)
  Rk4In rk[3];
};
template <typename S>
__device__ __forceinline__ EpiStar<S> epi_star_load(const EpiArgs& a, int k) {
  constexpr int W = Width<S>::n;
  const int i = k + 1;
  EpiStar<S> in;
  const double* ub = a.ub + 4 * W * (size_t)k;
  in.u = get<S>(ub, 0, 4);
  in.bx = get<S>(ub, 1, 4);
  in.by = get<S>(ub, 2, 4);
  in.bz = get<S>(ub, 3, 4);
  in.x = ld<S>(a.pos, a.pos_d, 3 * i);
  in.y = ld<S>(a.pos, a.pos_d, 3 * i + 1);
  in.z = ld<S>(a.pos, a.pos_d, 3 * i + 2);
  if (!a.newton_only) {
    in.v[0] = ld<S>(a.vel, a.vel_d, 3 * i);
    in.v[1] = ld<S>(a.vel, a.vel_d, 3 * i + 1);
    in.v[2] = ld<S>(a.vel, a.vel_d, 3 * i + 2);
    in.m_s = a.mass[i];
  }
  if constexpr (!IsDual<S>::value) {
    for (int c = 0; c < 3; ++c) in.rk[c] = rk4_load(a, 3 * (size_t)i + c);
  }
  return in;
}

// The massive object at an evaluation: its mass, its position, its acceleration A0 and
// potential magnitude V0, w = -P / M; and, for a chained Runge-Kutta stage, its
// step-start position, the stage sum of its velocities through the previous
// stage and its velocity.
template <typename S>
struct EpiBh {
  double M;
  S x0[3], A0[3], V0, w[3];
  double X[3] = {0.0, 0.0, 0.0}, KX[3] = {0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0};
};

template <typename PkT>
constexpr int epi_next_terms() {  // block-sum terms of the next prologue
  return std::is_same<PkT, Dual>::value ? 14 : 7;
}

// What the epilogue of a star needs of it and the massive object that does not
// wait for its pair sums.
template <typename S>
struct EpiGeo {
  S vi2, d0[3], rinv0, n0[3], kk, vw, dA, n4v, nw, g7;  // the star's own terms
  S ks, nvs, nws, g7s;                                  // the massive object's
};
template <typename S>
__device__ __forceinline__ EpiGeo<S> epi_geo(const EpiArgs& a, const EpiStar<S>& in,
                                             const EpiBh<S>& B) {
  EpiGeo<S> g;
  const double gM = a.G * B.M;
  const S (&vi)[3] = in.v;
  g.vi2 = vi[0] * vi[0] + vi[1] * vi[1] + vi[2] * vi[2];
  g.d0[0] = in.x - B.x0[0];
  g.d0[1] = in.y - B.x0[1];
  g.d0[2] = in.z - B.x0[2];
  g.rinv0 = rsqrt_t(g.d0[0] * g.d0[0] + g.d0[1] * g.d0[1] + g.d0[2] * g.d0[2] + a.eps2);
  for (int c = 0; c < 3; ++c) g.n0[c] = g.d0[c] * g.rinv0;
  g.kk = gM * g.rinv0 * g.rinv0;
  g.vw = vi[0] * B.w[0] + vi[1] * B.w[1] + vi[2] * B.w[2];
  g.dA = g.d0[0] * B.A0[0] + g.d0[1] * B.A0[1] + g.d0[2] * B.A0[2];
  g.n4v = 4.0 * (g.n0[0] * vi[0] + g.n0[1] * vi[1] + g.n0[2] * vi[2]);
  g.nw = g.n0[0] * B.w[0] + g.n0[1] * B.w[1] + g.n0[2] * B.w[2];
  g.g7 = 3.5 * gM * g.rinv0;
  const double gm_s = a.G * in.m_s;
  const S n0s[3] = {-g.n0[0], -g.n0[1], -g.n0[2]};
  g.ks = gm_s * g.rinv0 * g.rinv0;
  g.nvs = n0s[0] * vi[0] + n0s[1] * vi[1] + n0s[2] * vi[2];
  g.nws = n0s[0] * B.w[0] + n0s[1] * B.w[1] + n0s[2] * B.w[2];
  g.g7s = 3.5 * gm_s * g.rinv0;
  return g;
}
// Holds them before a wait: the compiler would move them behind it.
__device__ __forceinline__ void geo_hold(EpiGeo<double>& g) {
  asm volatile("" : "+v"(g.vi2), "+v"(g.kk), "+v"(g.vw), "+v"(g.dA), "+v"(g.n4v), "+v"(g.nw),
               "+v"(g.g7), "+v"(g.n0[0]), "+v"(g.n0[1]), "+v"(g.n0[2]));
  asm volatile("" : "+v"(g.ks), "+v"(g.nvs), "+v"(g.nws), "+v"(g.g7s));
}
__device__ __forceinline__ void geo_hold(EpiGeo<Dual>&) {}

// Star k's epilogue from its pair sums: outputs, stage update and next
// packet.  bh: its term of the massive object's 1PN sum; pro: its block-sum
// terms of the next prologue.
template <typename S, typename PkT>
__device__ __forceinline__ void epi_star(const EpiArgs& a, int k, const EpiStar<S>& in,
                                         const EpiBh<S>& B, const EpiGeo<S>& g, S (&sum)[kNF],
                                         S (&bh)[3], double (&pro)[epi_next_terms<PkT>()]) {
  constexpr bool DUAL = IsDual<S>::value;
  constexpr bool CHAIN = !std::is_void<PkT>::value;
  constexpr bool JNEXT = std::is_same<PkT, Dual>::value;  // the jerk sweep's packets
  static_assert(!CHAIN || !DUAL, "chained epilogues are FP64 evaluations");
  const int i = k + 1;
  const double gM = a.G * B.M;
  const S x0 = B.x0[0], y0 = B.x0[1], z0 = B.x0[2], V0 = B.V0;
  const S (&A0)[3] = B.A0;
  const S (&w)[3] = B.w;
  const S ui = in.u, bx = in.bx, by = in.by, bz = in.bz, xi = in.x, yi = in.y, zi = in.z;
  const S (&vi)[3] = in.v;
  sum[F_C2] *= kSqrt32;  // the sweep accumulates D'/sqrt(3/2)
  // Newtonian part: g_i - b_i with g_i = -G_i
  const S aN[3] = {-sum[F_G] - bx, -sum[F_G + 1] - by, -sum[F_G + 2] - bz};
  S Vi = sum[F_U] + ui;  // -phi_i
  S a1[3] = {0.0, 0.0, 0.0};
  if (!a.newton_only) {
    S Vphi = Vi;
    S aNs[3] = {aN[0], aN[1], aN[2]};
    if constexpr (!DUAL) {
      if (a.phi_in) {  // correction mode: the caller's potential and Newtonian acceleration
        Vphi = -a.phi_in[i];
        aNs[0] = a.accN_in[3 * i];
        aNs[1] = a.accN_in[3 * i + 1];
        aNs[2] = a.accN_in[3 * i + 2];
      }
    }
    // Eq. (6) star-star terms: S_i0 G_i + Q_i + C2_i v_i + 7 Q7_i, S_i0 = -v_i^2 + 4 u_i
    const S Si0 = -g.vi2 + 4.0 * ui;
    S q[3];
    for (int c = 0; c < 3; ++c)
      q[c] = Si0 * sum[F_G + c] + sum[F_Q + c] + sum[F_C2] * vi[c] + 7.0 * sum[F_Q7 + c];
    // massive-object partner (Eq. (5) and the G^2 m M / velocity terms of Eq. (6))
    const S br = -g.vi2 + 4.0 * g.vw + 4.0 * Vphi + V0 + 0.5 * g.dA;
    for (int c = 0; c < 3; ++c) {
      const S pull =
          g.kk * (br * g.n0[c] + g.n4v * (vi[c] - w[c]) - 3.0 * g.nw * vi[c]) + g.g7 * A0[c];
      a1[c] = a.lam * (pull + q[c]);
    }
    // this star's term of the massive object's 1PN sum (Eqs. (2)-(3))
    const S n0s[3] = {-g.n0[0], -g.n0[1], -g.n0[2]};
    const S d0s[3] = {-g.d0[0], -g.d0[1], -g.d0[2]};
    const S dAs = d0s[0] * aNs[0] + d0s[1] * aNs[1] + d0s[2] * aNs[2];
    const S brs = -2.0 * g.vi2 + 4.0 * g.vw + 1.5 * g.nvs * g.nvs + 4.0 * V0 + Vphi + 0.5 * dAs;
    for (int c = 0; c < 3; ++c)
      bh[c] = g.ks * (brs * n0s[c] + 3.0 * g.nvs * vi[c] - 3.0 * g.nvs * w[c] -
                      4.0 * g.nws * vi[c]) +
              g.g7s * aNs[c];
  }
  if (a.acc_newton) {
    a.acc_newton[3 * i] = val(aN[0]);
    a.acc_newton[3 * i + 1] = val(aN[1]);
    a.acc_newton[3 * i + 2] = val(aN[2]);
  }
  if (a.phi) a.phi[i] = -val(Vi);
  if (a.acc_1pn) {
    a.acc_1pn[3 * i] = val(a1[0]);
    a.acc_1pn[3 * i + 1] = val(a1[1]);
    a.acc_1pn[3 * i + 2] = val(a1[2]);
  }
  const S at[3] = {aN[0] + a1[0], aN[1] + a1[1], aN[2] + a1[2]};
  if (a.acc_tot) {
    for (int c = 0; c < 3; ++c) a.acc_tot[3 * i + c] = val(at[c]);
  }
  if (!finite_s(at[0]) || !finite_s(at[1]) || !finite_s(at[2])) raise_status(a.status, kStatusNonfinite);
  if constexpr (DUAL) {
    if (a.jerk) {
      for (int c = 0; c < 3; ++c) a.jerk[3 * i + c] = at[c].d;
    }
    if (a.herm >= 0) {
      for (int c = 0; c < 3; ++c) hermite_update(a, 3 * (size_t)i + c, at[c].v, at[c].d);
    }
  } else {
    if constexpr (JNEXT) {
      // the jerk sweep's prologue terms of this star (as k_prologue<Dual>
      // computes them from pos_d = vel, vel_d = the acceleration)
      const Dual x0d[3] = {Dual(x0, a.vel[0]), Dual(y0, a.vel[1]), Dual(z0, a.vel[2])};
      const Dual xsd[3] = {Dual(xi, vi[0]), Dual(yi, vi[1]), Dual(zi, vi[2])};
      const Dual vsd[3] = {Dual(vi[0], at[0]), Dual(vi[1], at[1]), Dual(vi[2], at[2])};
      Dual pd[7];
      star_terms<Dual, Dual>(x0d, xsd, vsd, in.m_s, a.G, gM, a.eps2, a.pk_next, a.ub_next, k,
                             pd);
#pragma unroll
      for (int q = 0; q < 7; ++q) {
        pro[q] = pd[q].v;
        pro[7 + q] = pd[q].d;
      }
    }
    if (a.stage >= 0) {
      double xn[3] = {0.0, 0.0, 0.0}, vn[3] = {0.0, 0.0, 0.0};
      for (int c = 0; c < 3; ++c)
        rk4_update(a, 3 * (size_t)i + c, in.rk[c], vi[c], at[c], xn[c], vn[c]);
      if constexpr (CHAIN && !JNEXT) {
        // the massive object's next position, as k_bh_final will compute it
        double x0n[3];
        for (int c = 0; c < 3; ++c) x0n[c] = rk4_next(a.stage, a.dt, B.X[c], B.KX[c], B.v[c]);
        star_terms<PkT, double>(x0n, xn, vn, in.m_s, a.G, gM, a.eps2, a.pk_next, a.ub_next,
                                k, pro);
      }
    }
  }
}

// Block sums of the workgroup's stars, which are in the calling wavefront: it
// sums (every lane of them then holds every sum) and writes its row of the
// massive object's 1PN sum and of the next prologue from its registers.
// COLS > 0: the stars are lanes 0 .. COLS - 1 and rows lie across columns
// [column][workgroup] (the one-launch stages); 0: up to 64 stars, rows
// [workgroup][column].
template <typename S, typename PkT, int COLS>
__device__ __forceinline__ void epi_rows(const EpiArgs& a, int blk, const S (&bh)[3],
                                         const double (&pro)[epi_next_terms<PkT>()]) {
  constexpr int W = Width<S>::n;
  constexpr bool CHAIN = !std::is_void<PkT>::value;
  constexpr int NP = epi_next_terms<PkT>();
  constexpr int NB = CHAIN ? 3 + NP : 3 * W;
  static_assert(COLS == 0 || (CHAIN && W == 1 && NP == 7), "columns: the Runge-Kutta stages");
  double bhs[NB];
#pragma unroll
  for (int c = 0; c < 3; ++c) put(bhs, c, 3, bh[c]);
  if constexpr (CHAIN) {
#pragma unroll
    for (int q = 0; q < NP; ++q) bhs[3 + q] = pro[q];
  }
  const int l = threadIdx.x & 63;
  if constexpr (COLS > 0) {
    star_sum<COLS, NB>(bhs);
    if (l == 0) {
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        if (c < 3) a.bhpart[(size_t)c * a.nbpro + blk] = bhs[c];
        else a.bpart_next[(size_t)(c - 3) * a.nbpro + blk] = bhs[c];
      }
    }
  } else {
    wave_sum<NB>(bhs);
    if (l < 4 * W) {
      // row layout: values in columns 0..2, derivatives in 4..6 (Dual)
      const int q = l & 3, h = l >> 2;
      a.bhpart[(size_t)blk * 4 * W + l] = q < 3 ? pick(bhs, h * 3 + q) : 0.0;
    }
    if constexpr (CHAIN) {
      // the prologue's row layout: sum m b (3), sum m u, sum m v (3), 0 (and
      // the same 8 columns of derivatives for the jerk sweep)
      constexpr int RW = NP == 14 ? 16 : 8;
      if (l >= 32 && l < 32 + RW) {
        const int c = l - 32, q = c & 7, h = c >> 3;
        a.bpart_next[(size_t)blk * RW + c] = q < 7 ? pick(bhs, 3 + h * 7 + q) : 0.0;
      }
    }
  }
}

// The epilogue of kEpiStars stars (blk * kEpiStars ...) from the splits'
// partial sums; fsum: epi_fsum doubles of LDS.  It is a chain of latencies, so
// the wavefronts that sum the splits leave everything else to one more, which
// meanwhile loads the stars' own inputs and the prologue rows and prepares
// what does not wait for the sums.  1500 stars, in us from its first
// instruction: loads back 1.0, massive object 1.5, split sums 1.7, terms
// prepared 1.9, barrier 2.4, star 4.0, block sums 4.5, stored 4.6.  With all
// four wavefronts doing everything in turn, 8 splits at a time, an RK4 step
// took 56.1 us instead of 50.9 at N = 1200, 142.0 instead of 137.3 at 4097
// and 633 instead of 627 at 10001 (FP64).
// Nine wavefronts fill a CU (126 registers per lane: sixteen fit), so they pay
// while there is one workgroup per CU at most; ensembles have more, and take
// fewer wavefronts per workgroup then (launch_epilogue_batched).
template <typename S, typename PkT = void, int WAVES = epi_waves<S>()>
__device__ __forceinline__ void epilogue_block(const EpiArgs& a, int blk, double* fsum) {
  constexpr bool DUAL = IsDual<S>::value;
  constexpr int W = DUAL ? 2 : 1;
  constexpr int NFO = kNF * W;
  constexpr int R = epi_ranges<S>();
  static_assert(kEpiStars == 64, "a star per lane");
  static_assert(WAVES == 4 * R + 1 || WAVES == 5 || WAVES == 4, "wavefronts");
  constexpr int SIDE = WAVES / 4;   // ranges summed side by side
  constexpr int EPI = WAVES - 1;    // the wavefront that runs the epilogue
  const int wave = wave_id(), l = threadIdx.x & 63;
  const int k = blk * kEpiStars + l;

  if (wave < 4 * SIDE) {
    // split reduction: wavefront (h, g) sums fields g, g+4, g+8, ... over the
    // splits of range h (and h + SIDE, ...), in split order; the loads of up to 8
    // (dual: 4) splits of all its fields are issued together, then added in order
    constexpr int FPT = (NFO + 3) / 4;   // fields per thread
    constexpr int BATCH = DUAL ? 4 : 8;  // splits per batch of loads
    const int g = wave & 3;
    const int per = (a.nsplit + R - 1) / R;
    if (k < a.Ns) {
      const size_t plane = (size_t)a.Ns;
      const size_t sstride = (size_t)NFO * plane;
      bool use[FPT];
#pragma unroll
      for (int fi = 0; fi < FPT; ++fi) use[fi] = g + 4 * fi < NFO && epi_field_used(g + 4 * fi, a);
      for (int h = wave >> 2; h < R; h += SIDE) {
        const int s0 = h * per, ns = min(a.nsplit - s0, per);
        double sum[FPT];
#pragma unroll
        for (int fi = 0; fi < FPT; ++fi) sum[fi] = 0.0;
        const double* src = a.part + (size_t)g * plane + (size_t)s0 * sstride + k;
        for (int sp = 0; sp < ns; sp += BATCH) {
          double v[FPT][BATCH];
#pragma unroll
          for (int fi = 0; fi < FPT; ++fi)
#pragma unroll
            for (int q = 0; q < BATCH; ++q)
              v[fi][q] = (use[fi] && sp + q < ns)
                             ? src[(size_t)4 * fi * plane + (size_t)(sp + q) * sstride]
                             : 0.0;
#pragma unroll
          for (int fi = 0; fi < FPT; ++fi)
#pragma unroll
            for (int q = 0; q < BATCH; ++q)
              if (sp + q < ns) sum[fi] += v[fi][q];
        }
#pragma unroll
        for (int fi = 0; fi < FPT; ++fi)
          if (g + 4 * fi < NFO) fsum[(h * NFO + g + 4 * fi) * kEpiStars + l] = sum[fi];
      }
    }
    if (wave != EPI) {
      __syncthreads();
      return;
    }
  }

  // the massive object and the stars' epilogue: every global read is requested
  // before the first wait
  __builtin_amdgcn_s_setprio(3);
  const bool star = k < a.Ns;
  EpiStar<S> in;
  if (star) in = epi_star_load<S>(a, k);
  EpiBh<S> B;
  B.M = a.mass[0];
  for (int c = 0; c < 3; ++c) B.x0[c] = ld<S>(a.pos, a.pos_d, c);
  // the massive object's step-start position, stage sum and velocity (uniform:
  // scalar loads)
  if constexpr (!DUAL && !std::is_void<PkT>::value) {
    if (a.stage >= 0) {
      for (int c = 0; c < 3; ++c) {
        B.X[c] = a.X[c];
        B.KX[c] = a.stage == 0 ? 0.0 : a.KX[c];
        B.v[c] = a.vel[c];
      }
    }
  }
  double rows[bh_cols<S>()];
  rows_load<bh_cols<S>()>(a.bpart, a.nbpro, DUAL ? 16 : 8, rows);
  S P[3];
  bh_quantities<S>(a, rows, B.A0, B.V0, P);
  const double iM = 1.0 / B.M;
  for (int c = 0; c < 3; ++c) B.w[c] = -(P[c] * iM);
  EpiGeo<S> geo = epi_geo<S>(a, in, B);
  geo_hold(geo);
  __syncthreads();  // fsum complete

  S bh[3] = {0.0, 0.0, 0.0};
  double pro[epi_next_terms<PkT>()];
#pragma unroll
  for (int q = 0; q < epi_next_terms<PkT>(); ++q) pro[q] = 0.0;
  if (star) {
    S sum[kNF];
#pragma unroll
    for (int f = 0; f < kNF; ++f) {
      if constexpr (DUAL) sum[f] = S(fsum[f * kEpiStars + l], fsum[(kNF + f) * kEpiStars + l]);
      else sum[f] = fsum[f * kEpiStars + l] + fsum[(NFO + f) * kEpiStars + l];
    }
    epi_star<S, PkT>(a, k, in, B, geo, sum, bh, pro);
  }
  epi_rows<S, PkT, 0>(a, blk, bh, pro);
}

template <typename S>
__global__ __launch_bounds__(epi_threads<S>()) void k_epilogue(EpiArgs a) {
  __shared__ double fsum[epi_fsum<S>()];
  epilogue_block<S>(a, blockIdx.x, fsum);
}

// FP64 epilogue that also performs the next sweep's prologue (packets of
// PkOf<T>; T = Dual: the jerk sweep at this state), saving that kernel.
template <typename T>
__global__ __launch_bounds__(epi_threads<double>()) void k_epilogue_chain(EpiArgs a) {
  __shared__ double fsum[epi_fsum<double>()];
  epilogue_block<double, T>(a, blockIdx.x, fsum);
}

template <typename S>
__device__ __forceinline__ void bh_final_block(const EpiArgs& a) {
  constexpr bool DUAL = IsDual<S>::value;
  constexpr int W = DUAL ? 2 : 1;
  // both row sets and the massive object's own state are requested before
  // the first wait (see epilogue_block)
  double rows[bh_cols<S>()], rows1[4 * W - 1];  // 1PN rows: columns 0..2 (4..6: derivatives)
  rows_load<bh_cols<S>()>(a.bpart, a.nbpro, DUAL ? 16 : 8, rows);
  if (!a.newton_only) rows_load<4 * W - 1>(a.bhpart, a.nbepi, 4 * W, rows1);
  // thread c < 3 finishes component c: its velocity and Runge-Kutta state
  const int cc = threadIdx.x;
  S v0c = 0.0;
  Rk4In rkc;
  if (cc < 3) {
    if (!a.newton_only) v0c = ld<S>(a.vel, a.vel_d, cc);
    if constexpr (!DUAL) rkc = rk4_load(a, (size_t)cc);
  }
  S A0[3], V0, P[3];
  bh_quantities<S>(a, rows, A0, V0, P);
  S T[3] = {0.0, 0.0, 0.0};
  if (!a.newton_only) {
    double r[4 * W - 1];
    rows_sum<4 * W - 1>(rows1, r);
    for (int c = 0; c < 3; ++c) T[c] = get<S>(r, c, 4);
  }
  // component c of the massive object's outputs and update (c a constant in
  // each call below, so that nothing is indexed at run time)
  auto finish = [&](int c, const S& A0c, const S& Tc) {
    const S a1c = a.lam * Tc;
    const S atc = A0c + a1c;
    if (a.acc_newton) a.acc_newton[c] = val(A0c);
    if (a.phi && c == 0) a.phi[0] = -val(V0);
    if (a.acc_1pn) a.acc_1pn[c] = val(a1c);
    if (a.acc_tot) a.acc_tot[c] = val(atc);
    if (!finite_s(atc)) raise_status(a.status, kStatusNonfinite);
    if constexpr (DUAL) {
      if (a.jerk) a.jerk[c] = atc.d;
      if (a.herm >= 0) hermite_update(a, (size_t)c, atc.v, atc.d);
    } else {
      if (a.stage >= 0) {
        double xn, vn;
        rk4_update(a, (size_t)c, rkc, v0c, atc, xn, vn);
      }
    }
  };
  if (cc == 0) finish(0, A0[0], T[0]);
  else if (cc == 1) finish(1, A0[1], T[1]);
  else if (cc == 2) finish(2, A0[2], T[2]);
}

template <typename S>
__global__ __launch_bounds__(kBlock) void k_bh_final(EpiArgs a) {
  bh_final_block<S>(a);
}

// The jerk evaluation's dual epilogue with the FP64 pass's massive-object
// update (k_bh_final<double>'s work) in one extra workgroup: the dual
// epilogue reads neither the massive object's FP64 acceleration nor the FP64
// partial rows (its own rows are in separate buffers).
__global__ __launch_bounds__(epi_threads<Dual>()) void k_epilogue_dual_bh(EpiArgs a, EpiArgs e) {
  __shared__ double fsum[epi_fsum<Dual>()];
  if (blockIdx.x == gridDim.x - 1) {
    bh_final_block<double>(e);
    return;
  }
  epilogue_block<Dual>(a, blockIdx.x, fsum);
}

// The sweep of a chained Runge-Kutta stage with the previous stage's
// massive-object update (k_bh_final's work) in one extra workgroup: the sweep
// reads only star packets, which the previous epilogue has written, so the
// two are independent and the stage saves a kernel boundary.  Grid:
// (iblocks or a few columns more) x (1 + nsplit).  Row 0, column 0 runs the
// update; the rest of that row and the columns beyond the stars exit at once.
// The row comes first, so that the sweep's workgroups spread over the
// CUs as if alone (as a last column its workgroups fell between them: a sweep
// of 768 workgroups then did not fill 256 CUs evenly).
// One i per lane: six wavefronts per SIMD (the update's registers would allow
// four; FP64 N = 3600 134.1 us per step with four, 128.9 with six).
template <typename T, int MODE, int IPT, int WS>
__global__ __launch_bounds__(pair_threads<WS>(), IPT == 1 ? 6 : 4) void k_pair_bh(PairArgs a, EpiArgs e) {
  __shared__ double red[pair_red_doubles<T, IPT, WS>()];
  if (blockIdx.y == 0) {
    if (blockIdx.x == 0) bh_final_block<double>(e);
    return;
  }
  constexpr int IB = pair_threads<WS>() / WS * IPT;  // i-bodies per workgroup
  if ((int)blockIdx.x * IB >= a.Ns) return;
  pair_block<T, MODE, IPT, WS>(a, blockIdx.x, blockIdx.y - 1, red);
}

// ---------------------------------------------------------------------------
// Small systems: one launch per Runge-Kutta stage.  Such a stage is a chain of
// latencies (launch, loads, reductions, dependent FP64 arithmetic) rather than
// work: one kernel per stage saves a launch and the split partials' trip
// through memory.  A workgroup owns NS stars.  Its first kStageWaves
// wavefronts sum all their j (lane sl + NS q takes star sl and j = q,
// q + 64 kStageWaves / NS, ...), reduce them in fixed order (exchanges within
// each wavefront, then the wavefronts).  No other workgroup's partials are
// needed, so nothing waits across workgroups.  One more wavefront meanwhile
// loads the stars' own inputs and prepares what their epilogue needs of the
// massive object: its update of the previous stage needs every epilogue's
// rows, and each workgroup computes it itself from the rows the previous
// launch wrote (the same sums in the same order, so the same bits everywhere);
// workgroup 0 stores it.  That wavefront then runs the stars' epilogue.  Rows
// lie across columns, so that its loads are contiguous.  Where every lane has
// one j at most (DIRECT) it loads that packet itself; else each wavefront has a
// run of j and copies its packets to LDS itself, 64 at a time and the next 64
// meanwhile, so that no wavefront waits for another before the sums are due.
// (One tile for all, behind a barrier, waited for the massive object's loads,
// too: 37.0 us per step instead of 32.7 at N = 1024.)
// A stage of 100 stars (2 per workgroup), in us from its first instruction:
// the massive object's loads back at 1.2, its sums 1.5, its update 2.2 (the
// sweep done at 1.7), the epilogue 4.7, its rows 4.9, the next launch 6.2.
// 1024 stars (4 per workgroup): update 3.7, swept 4.5 to 5.5, epilogue 7.6.
// Two stars per lane, four packets at a time, or the next packet ahead of the
// present one: no faster.
// Against two wavefronts' sweep with the epilogue and the update after it, in
// us per RK4 step: 34.6 -> 21.5 (100 stars), 40.0 -> 25.5 (300), and against
// the two-kernel stages 50.3 -> 32.7 (1024), 71.8 -> 56.7 (2048).
// Every buffer a stage reads is one no workgroup of that stage writes:
// packets, u/b rows, block rows, massive-object 1PN rows and the massive
// object's state (X, V, Xs, Vs, KX, KV and its last Newtonian acceleration)
// alternate between two buffers.
// ---------------------------------------------------------------------------
constexpr int kStageFirst = 0;  // the first stage of a call: no pending update
constexpr int kStageFull = 1;   // pending update, sweep and epilogue
constexpr int kStageFinal = 2;  // the last pending update only (one workgroup)
constexpr int kStageWaves = 8;  // wavefronts of the sweep
constexpr int kStageThreads = 64 * (kStageWaves + 1);

struct StageArgs {
  EpiArgs e;             // this stage's epilogue; e.nbpro workgroups (rows in every row buffer)
  const void* pk;        // this stage's packets (PkOf<T>)
  int mode;
  int pstage;            // stage of the pending massive-object update
  const double* phrow;   // that stage's massive-object 1PN rows [3][e.nbpro]
  // the massive object's X, V, Xs, Vs, KX, KV before that update, and its
  // Newtonian acceleration at that stage; the same after it, at this stage
  const double* bhs_in;
  double* bhs_out;
};
constexpr int kBhState = 21;

// Column sums, this lane's part: rows l, l + 64, ... of n, of three columns of
// p3 and seven of p7, in order; the loads of several rows are in flight together.
__device__ __forceinline__ void cols_load(const double* p3, const double* p7, int n,
                                          double (&v)[10]) {
  const int l = threadIdx.x & 63;
  const auto row = [&](double (&w)[10], int r) {
#pragma unroll
    for (int k = 0; k < 10; ++k)
      w[k] = k < 3 ? p3[(size_t)k * n + min(r, n - 1)] : p7[(size_t)(k - 3) * n + min(r, n - 1)];
  };
  const auto add = [&](const double (&w)[10], int r) {
#pragma unroll
    for (int k = 0; k < 10; ++k) v[k] += r < n ? w[k] : 0.0;
  };
#pragma unroll
  for (int k = 0; k < 10; ++k) v[k] = 0.0;
  constexpr int U = 3;
  double w0[10];
  row(w0, l);
  for (int r = l + 64; r - l < n; r += U * 64) {
    double w[U][10];
#pragma unroll
    for (int u = 0; u < U; ++u) row(w[u], r + 64 * u);
    if (r - l == 64) add(w0, l);
#pragma unroll
    for (int u = 0; u < U; ++u) add(w[u], r + 64 * u);
  }
  if (n <= 64) add(w0, l);
}

// The pending update: the massive object's acceleration at stage sa.pstage (as
// k_bh_final), from its Newtonian part bi[18..20] and the sums of its 1PN rows,
// then its Runge-Kutta bookkeeping (as rk4_update) on the state in bi, which
// becomes the state of this stage's evaluation.  Workgroup 0 stores the new
// step-start state after stage 3.
__device__ __forceinline__ void stage_bh_update(const StageArgs& sa, const double* sums1,
                                                double (&bi)[kBhState]) {
  const EpiArgs& a = sa.e;
  const int ps = sa.pstage;
  bool finite = true;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double atc = bi[18 + c] + a.lam * sums1[c];
    finite = finite && isfinite(atc);
    const double X = bi[c], V = bi[3 + c], vs = bi[9 + c], KX = bi[12 + c], KV = bi[15 + c];
    const double xn = rk4_next(ps, a.dt, X, KX, vs);
    const double vn = rk4_next(ps, a.dt, V, KV, atc);
    bi[6 + c] = xn;
    bi[9 + c] = vn;
    if (ps < 3) {
      bi[12 + c] = ps == 0 ? vs : KX + 2.0 * vs;
      bi[15 + c] = ps == 0 ? atc : KV + 2.0 * atc;
    } else {
      bi[c] = xn;
      bi[3 + c] = vn;
      bi[12 + c] = 0.0;
      bi[15 + c] = 0.0;
    }
  }
  if (blockIdx.x == 0) {
    const int l = threadIdx.x & 63;
    if (l == 0 && !finite) raise_status(a.status, kStatusNonfinite);
    if (ps == 3) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if (l == 32 + c) uniform_ptr(a.X)[c] = bi[c];
        if (l == 40 + c) uniform_ptr(a.V)[c] = bi[3 + c];
      }
    }
  }
}

// epi_star_load of a Runge-Kutta stage, without a branch: every load in flight
// together (the stage sums, too, where a stage has none yet).  Lanes beyond the
// workgroup's stars load stars of other workgroups, which may be storing them at
// that moment; those lanes' values are never used.
__device__ __forceinline__ EpiStar<double> stage_star_load(const EpiArgs& a, int k) {
  const size_t i = (size_t)k + 1;
  const double* ub = a.ub + 4 * (size_t)k;
  EpiStar<double> in;
  in.u = ub[0], in.bx = ub[1], in.by = ub[2], in.bz = ub[3];
  in.x = a.pos[3 * i], in.y = a.pos[3 * i + 1], in.z = a.pos[3 * i + 2];
  in.m_s = a.mass[i];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const size_t o = 3 * i + c;
    in.v[c] = a.vel[o];
    in.rk[c].X = a.X[o], in.rk[c].V = a.V[o], in.rk[c].KX = a.KX[o], in.rk[c].KV = a.KV[o];
  }
  return in;
}

// Waits until N copies to LDS at most are on their way.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"i"(N) : "memory");
}

template <typename T, int NS, bool DIRECT>
__global__ __launch_bounds__(kStageThreads) void k_stage(StageArgs sa) {
  using Pk = typename PkOf<T>::type;
  constexpr int W = sizeof(Pk) / 16;  // copies of 16 bytes per lane to stage a tile
  static_assert(sizeof(Pk) % 16 == 0, "copied in 16-byte words");
  __shared__ __align__(16) char tile[DIRECT ? 16 : 2 * kStageWaves * 64 * sizeof(Pk)];
  __shared__ double red[kNF * kStageWaves * NS];
  __shared__ double fsum[kNF * NS];
  const EpiArgs& a = sa.e;
  const int lane = threadIdx.x & 63, wave = wave_id();
  const bool eval = sa.mode != kStageFinal;

  if (wave == kStageWaves) {
    // the massive object and the stars' epilogue; every global read is
    // requested before the first wait
    const bool pend = sa.mode != kStageFirst;
    const int nb = a.nbpro;
    const int k = blockIdx.x * NS + lane;
    const bool star = lane < NS && k < a.Ns;
    // (this chain is what the launch waits for, the sweep is not)
    __builtin_amdgcn_s_setprio(3);
    double v[10], bi[kBhState];  // row sums: 1PN of the pending stage (3), this stage's (7)
    EpiBh<double> B;
    EpiStar<double> in = stage_star_load(a, min(k, a.Ns - 1));
    const double state = sa.bhs_in[min(lane, kBhState - 1)];
    B.M = a.mass[0];
    cols_load(sa.phrow, a.bpart, nb, v);  // (phrow: read, not used, where nothing is pending)
    if (a.stage == 0) {
#pragma unroll
      for (int c = 0; c < 3; ++c) in.rk[c].KX = in.rk[c].KV = 0.0;
    }
    sum10(v);
#pragma unroll
    for (int c = 0; c < kBhState; ++c) bi[c] = lane_value(state, c);
    const double iM = 1.0 / B.M;
    if (pend) stage_bh_update(sa, v, bi);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      B.x0[c] = bi[6 + c];
      bi[18 + c] = B.A0[c] = v[3 + c] * iM;
      B.w[c] = -(v[7 + c] * iM);
      B.X[c] = bi[c];
      B.KX[c] = a.stage == 0 ? 0.0 : bi[12 + c];
      B.v[c] = bi[9 + c];
    }
    B.V0 = v[6] * iM;
    if (blockIdx.x == 0 && lane < kBhState) sa.bhs_out[lane] = pick(bi, lane);
    if (!eval) return;
    EpiGeo<double> g = epi_geo<double>(a, in, B);
    geo_hold(g);
    __syncthreads();  // the sweep's sums are in red
    for (int e = lane; e < kNF * NS; e += 64) {  // field e / NS of star e % NS
      const double* r = red + e / NS * kStageWaves * NS + e % NS;
      double x = r[0];
#pragma unroll
      for (int w = 1; w < kStageWaves; ++w) x += r[w * NS];
      fsum[e] = x;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // fsum, within this wavefront
    double bh[3] = {0.0, 0.0, 0.0}, pro[7] = {0, 0, 0, 0, 0, 0, 0};
    if (star) {
      double sum[kNF];
#pragma unroll
      for (int f = 0; f < kNF; ++f) sum[f] = fsum[f * NS + lane];
      epi_star<double, T>(a, k, in, B, g, sum, bh, pro);
    }
    epi_rows<double, T, NS>(a, blockIdx.x, bh, pro);
    return;
  }

  if (!eval) return;
  const Pk* __restrict__ pk = static_cast<const Pk*>(sa.pk);
  const int sl = threadIdx.x % NS;
  PairI<T, 1> I;
  I.idx[0] = blockIdx.x * NS + sl;
  {
    const Pk& p = pk[min(I.idx[0], a.Ns - 1)];  // lanes past the end compute on a copy, never stored
    I.x[0] = p.x;
    I.y[0] = p.y;
    I.z[0] = p.z;
    I.kx[0] = T(PairScale<T>::k) * (T)p.svx;
    I.ky[0] = T(PairScale<T>::k) * (T)p.svy;
    I.kz[0] = T(PairScale<T>::k) * (T)p.svz;
  }
  const T eps2 = (T)a.eps2;
  PairAcc<T, 1> A;
  A.zero();
  double acc[kNF][1];
#pragma unroll
  for (int f = 0; f < kNF; ++f) acc[f][0] = 0.0;
  if constexpr (DIRECT) {
    if (const int q = threadIdx.x / NS; q < a.Ns) {
      const Pk p = pk[q];
      pair_one<T, MODE_FUSED, 1, true>(p, q, eps2, I, A);
    }
  } else {
    // this wavefront's j, 64 at a time, the next 64 on their way meanwhile
    const int per = (a.Ns + kStageWaves - 1) / kStageWaves;
    const int jb = wave * per, n = min(a.Ns - jb, per);
    char* const mine = tile + wave * (2 * 64 * sizeof(Pk));
    const char* const src = reinterpret_cast<const char*>(pk + jb);
    const auto stage_tile = [&](int j0) {
#pragma unroll
      for (int w = 0; w < W; ++w) {
        // word 64 w + lane of the tile (past the end: the last word again)
        const int word = min(j0 * W + 64 * w + lane, n * W - 1);
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void*)(src + 16 * (size_t)word),
            (__attribute__((address_space(3))) void*)(mine + (j0 & 64) * sizeof(Pk) + 1024 * w),
            16, 0, 0);
      }
    };
    if (n > 0) stage_tile(0);
    if (n > 64) stage_tile(64);
    for (int j0 = 0; j0 < n; j0 += 64) {
      if (j0 + 64 < n) wait_vmcnt<W>();
      else wait_vmcnt<0>();
      const Pk* lp = reinterpret_cast<const Pk*>(mine + (j0 & 64) * sizeof(Pk));
      const int m = min(n - j0, 64);
      constexpr int Q = 64 / NS;  // j at a time
      int j = lane / NS;
      for (; j + Q < m; j += 2 * Q) {
        const Pk p0 = lp[j];
        const Pk p1 = lp[j + Q];
        pair_one<T, MODE_FUSED, 1, true>(p0, jb + j0 + j, eps2, I, A);
        pair_one<T, MODE_FUSED, 1, true>(p1, jb + j0 + j + Q, eps2, I, A);
      }
      if (j < m) pair_one<T, MODE_FUSED, 1, true>(lp[j], jb + j0 + j, eps2, I, A);
      if constexpr (sizeof(T) < 8) {  // FP32 partial sums: of a few terms
        acc_flush(A, acc);
        A.zero();
      }
      if (j0 + 128 < n) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the tile is read
        stage_tile(j0 + 128);
      }
    }
  }
  if constexpr (DIRECT || sizeof(T) == 8) acc_flush(A, acc);
  double x[12], r[fold_regs<NS>()];
  int f[fold_regs<NS>()];
#pragma unroll
  for (int c = 0; c < 12; ++c) x[c] = c < kNF ? acc[c < kNF ? c : 0][0] : 0.0;
  fold12<NS>(x, r, f);
#pragma unroll
  for (int c = 0; c < fold_regs<NS>(); ++c)
    if (f[c] >= 0 && f[c] < kNF) red[(f[c] * kStageWaves + wave) * NS + lane % NS] = r[c];
  __syncthreads();
}

// A call's first packets, u/b rows and block rows in the stage kernel's
// layout (a block row per NS stars, reduced as its epilogue reduces them, so
// that a run resumed from a saved state repeats the continuous run bit for bit).
template <typename T, int NS>
__global__ __launch_bounds__(kBlock) void k_stage_head(EpiArgs a, double* bhs) {
  const int t = threadIdx.x, k = blockIdx.x * NS + t;
  double v[7] = {0, 0, 0, 0, 0, 0, 0};
  if (t < NS && k < a.Ns) {
    const int s = k + 1;
    const double x0[3] = {a.pos[0], a.pos[1], a.pos[2]};
    const double xs[3] = {a.pos[3 * s], a.pos[3 * s + 1], a.pos[3 * s + 2]};
    const double vs[3] = {a.vel[3 * s], a.vel[3 * s + 1], a.vel[3 * s + 2]};
    star_terms<T, double>(x0, xs, vs, a.mass[s], a.G, a.G * a.mass[0], a.eps2, a.pk_next,
                          a.ub_next, k, v);
  }
  if (t < 64) {  // the stars are in wavefront 0 (as in the stage's epilogue)
    star_sum<NS, 7>(v);
    if (t == 0) {
#pragma unroll
      for (int c = 0; c < 7; ++c) a.bpart_next[(size_t)c * gridDim.x + blockIdx.x] = v[c];
    }
  }
  if (blockIdx.x == 0) {  // the massive object's state before the first stage
    if (t < kBhState) bhs[t] = t < 12 ? (t / 3 % 2 ? a.vel : a.pos)[t % 3] : 0.0;
    const double M = a.mass[0];
    if (t == 0 && (!(M > 0.0) || !isfinite(M))) raise_status(a.status, kStatusMass);
  }
}

// ---------------------------------------------------------------------------
// Diagnostics (Eqs. (7)-(8)) and close encounters.  Both need sums (minima)
// over all star pairs only, and every pair term is symmetric, so a pair is
// visited once: lane i takes the j > i.  The grid is (i-blocks of kBlock
// stars) x (j-chunks); a chunk that ends at or before its block's first star
// has no pair and writes an empty row.  Each workgroup reduces its lanes and writes
// one row, a last workgroup sums the rows in fixed order: three kernels, and
// no per-star partial sums in memory.
//
// The sweeps are bound by vector issue: per unordered pair 37 operations and
// one reciprocal square root (diagnostics), 8 operations (encounters, four j at
// a time).  Forms with a sum (minimum) per star took 39 and 11 per ordered
// pair.  At N = 10001 the diagnostics' sweep takes 90 us (250 per ordered
// pair), the encounters' 28 (92), and their stars' and last kernels 21 (44,
// by LDS trees and one serial thread); a record (both calls) 188 us (478).
// ---------------------------------------------------------------------------
struct TriArgs {
  int Ns, jchunk;
  double eps2;
  double* rows;  // [gridDim.y][gridDim.x][kTriRow]
};
constexpr int kTriRow = 8;       // doubles per row
constexpr int kTriFinal = 1024;  // threads of the workgroup that sums the rows

__device__ __forceinline__ bool tri_live(int block, int chunk, int jchunk) {
  return ((int64_t)chunk + 1) * jchunk > (int64_t)block * kBlock;
}

// The pairs of lane i in its workgroup's chunk, from the block's first star
// on: one(j) where j may be <= i, four(j) for the four stars j .. j + 3 beyond
// the block, last(j) for what is left of them.
template <typename One, typename Four, typename Last>
__device__ __forceinline__ void tri_range(const TriArgs& a, One&& one, Four&& four, Last&& last) {
  const int ilo = blockIdx.x * kBlock;
  const int j0 = max((int)blockIdx.y * a.jchunk, ilo);
  const int j1 = (int)min((int64_t)a.Ns, ((int64_t)blockIdx.y + 1) * a.jchunk);
  const int jm = min(j1, ilo + kBlock);
  int j = j0;
  for (; j < jm; ++j) one(j);
  for (; j + 3 < j1; j += 4) four(j);
  for (; j < j1; ++j) last(j);
}

// Sums over the workgroup of K doubles per thread, in every thread of its first
// wavefront: wavefront butterflies, then the wavefronts in order.
template <int K>
__device__ __forceinline__ void group_sum(double (&v)[K], double* lds) {
  wave_allsum<K>(v);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  if (l < K) lds[w * K + l] = pick(v, l);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = lds[k];
  for (int u = 1; u < (int)(blockDim.x >> 6); ++u) {
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] += lds[u * K + k];
  }
}

// Star packet of the diagnostics: q = 3/2 v^2 + u.
struct alignas(64) PkDiag {
  double x, y, z, gm, vx, vy, vz, q;
};

struct DiagArgs {
  const double* pos;
  const double* vel;
  const double* mass;
  int Ns;
  double G, lam, eps2;
  PkDiag* pk;
  double* srow;  // [star blocks][10]: sums of the stars' own terms
  int nsrow;
  double* prow;  // pair rows (TriArgs::rows)
  int nprow;
  double* out;   // [9]: the eight results, then the status
};

// The stars' own terms (columns of srow) and their packets.
//  0: 1/2 m v^2 - m u                     (Newtonian energy, stars)
//  1: 1PN energy bracket without star-star pairs
//  2: m u / M  (sum = U0 = sum_i G m_i / R_1i)
//  3-5: m v                               (Newtonian momentum, stars)
//  6-8: 1PN momentum bracket without star-star pairs
__global__ __launch_bounds__(kBlock) void k_diag_stars(DiagArgs a) {
  __shared__ double lds[9 * kBlock / 64];
  const int k = blockIdx.x * kBlock + threadIdx.x;
  double v[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  if (k < a.Ns) {
    const int i = k + 1;
    const double M = a.mass[0], m = a.mass[i];
    const double* vi = a.vel + 3 * (size_t)i;
    const double* v1 = a.vel;
    const double* xi = a.pos + 3 * (size_t)i;
    const double d[3] = {a.pos[0] - xi[0], a.pos[1] - xi[1], a.pos[2] - xi[2]};  // x_1i
    const double rinv = rsqrt_f64(fma(d[2], d[2], fma(d[1], d[1], fma(d[0], d[0], a.eps2))));
    const double u = a.G * M * rinv;
    const double n[3] = {d[0] * rinv, d[1] * rinv, d[2] * rinv};
    const double vi2 = vi[0] * vi[0] + vi[1] * vi[1] + vi[2] * vi[2];
    const double v12 = v1[0] * v1[0] + v1[1] * v1[1] + v1[2] * v1[2];
    const double v1vi = v1[0] * vi[0] + v1[1] * vi[1] + v1[2] * vi[2];
    const double nv1 = n[0] * v1[0] + n[1] * v1[1] + n[2] * v1[2];
    const double nvi = n[0] * vi[0] + n[1] * vi[1] + n[2] * vi[2];
    a.pk[k] = PkDiag{xi[0], xi[1], xi[2], a.G * m, vi[0], vi[1], vi[2], fma(1.5, vi2, u)};
    v[0] = 0.5 * m * vi2 - m * u;
    v[1] = 0.375 * m * vi2 * vi2 + 1.5 * m * u * vi2 + 0.5 * m * u * u +
           0.5 * m * u * (3.0 * v12 - 7.0 * v1vi - nv1 * nvi);
    v[2] = m * u / M;
    for (int c = 0; c < 3; ++c) {
      v[3 + c] = m * vi[c];
      v[6 + c] = 0.5 * m * vi2 * vi[c] - 0.5 * m * u * (vi[c] + nvi * n[c]) -
                 0.5 * m * u * (v1[c] + nv1 * n[c]);
    }
  }
  group_sum<9>(v, lds);
  if (threadIdx.x < 9) a.srow[(size_t)blockIdx.x * 10 + threadIdx.x] = pick(v, threadIdx.x);
}

// Star pairs, p = G m_i m_j / R, n = x_ij / R: columns of a row
//  0: -sum p                                        (Newtonian energy)
//  1: sum p [q_i + q_j - 7/2 v_i.v_j - 1/2 (n.v_i)(n.v_j)]   (1PN energy)
//  2-4: -1/2 sum p [(v_i + v_j) + (n.(v_i + v_j)) n]         (1PN momentum)
__global__ __launch_bounds__(kBlock) void k_diag_pair(TriArgs a,
                                                     const PkDiag* __restrict__ pk,
                                                     const double* __restrict__ mass) {
  __shared__ double lds[5 * kBlock / 64];
  double* row = a.rows + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * kTriRow;
  if (!tri_live(blockIdx.x, blockIdx.y, a.jchunk)) {
    if (threadIdx.x < 5) row[threadIdx.x] = 0.0;
    return;
  }
  const int i = blockIdx.x * kBlock + threadIdx.x;
  const PkDiag I = pk[min(i, a.Ns - 1)];
  const double hx = -3.5 * I.vx, hy = -3.5 * I.vy, hz = -3.5 * I.vz;
  double s0 = 0.0, s1 = 0.0, vx = 0.0, vy = 0.0, vz = 0.0, yx = 0.0, yy = 0.0, yz = 0.0;
  auto pair = [&](const PkDiag& p, int j, auto masked) {
    const double dx = I.x - p.x, dy = I.y - p.y, dz = I.z - p.z;
    double rinv = rsqrt_f64(fma(dz, dz, fma(dy, dy, fma(dx, dx, a.eps2))));
    if (decltype(masked)::value) rinv = j > i ? rinv : 0.0;  // (lanes past the end: none)
    const double w = p.gm * rinv, rinv2 = rinv * rinv;
    const double xi = fma(dz, I.vz, fma(dy, I.vy, dx * I.vx));
    const double xj = fma(dz, p.vz, fma(dy, p.vy, dx * p.vx));
    const double q = fma(hz, p.vz, fma(hy, p.vy, hx * p.vx)) + p.q;  // q_j - 7/2 v_i.v_j
    s0 += w;
    s1 = fma(w, fma(-0.5 * rinv2, xi * xj, q), s1);
    vx = fma(w, p.vx, vx);
    vy = fma(w, p.vy, vy);
    vz = fma(w, p.vz, vz);
    const double c = w * rinv2 * (xi + xj);
    yx = fma(c, dx, yx);
    yy = fma(c, dy, yy);
    yz = fma(c, dz, yz);
  };
  tri_range(
      a, [&](int j) { pair(pk[j], j, std::true_type{}); },
      [&](int j) {
        const PkDiag p0 = pk[j], p1 = pk[j + 1], p2 = pk[j + 2], p3 = pk[j + 3];
        pair(p0, j, std::false_type{});
        pair(p1, j + 1, std::false_type{});
        pair(p2, j + 2, std::false_type{});
        pair(p3, j + 3, std::false_type{});
      },
      [&](int j) { pair(pk[j], j, std::false_type{}); });
  double v[5] = {0, 0, 0, 0, 0};
  if (i < a.Ns) {
    const double m = mass[i + 1], h = -0.5 * m;
    v[0] = -m * s0;
    v[1] = m * fma(I.q, s0, s1);
    v[2] = h * (fma(I.vx, s0, vx) + yx);
    v[3] = h * (fma(I.vy, s0, vy) + yy);
    v[4] = h * (fma(I.vz, s0, vz) + yz);
  }
  group_sum<5>(v, lds);
  if (threadIdx.x < 5) row[threadIdx.x] = pick(v, threadIdx.x);
}

__global__ __launch_bounds__(kTriFinal) void k_diag_final(DiagArgs a) {
  __shared__ double lds[14 * kTriFinal / 64];
  double r[14];
#pragma unroll
  for (int c = 0; c < 14; ++c) r[c] = 0.0;
  for (int k = threadIdx.x; k < a.nsrow; k += kTriFinal) {
#pragma unroll
    for (int c = 0; c < 9; ++c) r[c] += a.srow[(size_t)k * 10 + c];
  }
#pragma unroll 4
  for (int k = threadIdx.x; k < a.nprow; k += kTriFinal) {
#pragma unroll
    for (int c = 0; c < 5; ++c) r[9 + c] += a.prow[(size_t)k * kTriRow + c];
  }
  group_sum<14>(r, lds);
  if (threadIdx.x == 0) {
    const double M = a.mass[0];
    const double* v1 = a.vel;
    const double v12 = v1[0] * v1[0] + v1[1] * v1[1] + v1[2] * v1[2];
    const double U0 = r[2];
    a.out[0] = 0.5 * M * v12 + (r[0] + r[9]);
    a.out[1] = a.lam * ((r[1] + r[10]) + 0.5 * M * U0 * U0);
    for (int c = 0; c < 3; ++c) {
      a.out[2 + c] = M * v1[c] + r[3 + c];
      a.out[5 + c] = a.lam * (r[6 + c] + r[11 + c]);
    }
    a.out[8] = !(M > 0.0) || !isfinite(M) ? 2.0 : 0.0;
  }
}

// ---------------------------------------------------------------------------
// Close-encounter diagnostics (what the paper's test-model figures follow,
// Sec. 4): the star nearest to the massive object, how many stars lie within
// a given radius of it, and the nearest star-star pair.  Unsoftened
// distances.  Minima carry the smaller index on ties, so results are exact
// and order independent.
// ---------------------------------------------------------------------------
struct EncArgs {
  const double* pos;
  const double* vel;
  const double* mass;
  int Ns;
  double r_close2;  // squared radius for the count
  double G, lam;    // gravitational constant, 1/c^2
  double4* pk;      // star positions
  double* srow;     // [star blocks][10]: nearest BH r^2, its star, close count,
                    //                   largest 1PN/Newton ratio of a BH pair, its star
  int nsrow;
  double* prow;     // pair rows (TriArgs::rows): nearest pair r^2, i, j
  int nprow;
  double* out;      // [8]
};

// Strength of the 1PN term of a star's pair with the massive object: the
// lambda-part of Eq. (5), (G M / r^2) lambda [(4 G M / r - v^2) n + 4 (n.v) v],
// over the Newtonian pull G M / r^2 (unsoftened r, the star's own velocity).
__device__ __forceinline__ double bh_pair_ratio(double dx, double dy, double dz, double r2,
                                                double vx, double vy, double vz, double gM,
                                                double lam) {
  const double r = sqrt(r2);
  const double nx = dx / r, ny = dy / r, nz = dz / r;
  const double v2 = vx * vx + vy * vy + vz * vz;
  const double nv = nx * vx + ny * vy + nz * vz;
  const double k = 4.0 * gM / r - v2;
  const double tx = k * nx + 4.0 * nv * vx, ty = k * ny + 4.0 * nv * vy,
               tz = k * nz + 4.0 * nv * vz;
  return lam * sqrt(tx * tx + ty * ty + tz * tz);
}

// A candidate: value and one or two indices; kNone: no star.
constexpr int kNone = INT_MAX;
struct EncBest {
  double v;
  int i, j;
};
// smaller value, then smaller indices (a NaN never wins)
__device__ __forceinline__ bool enc_less(const EncBest& a, const EncBest& b) {
  return a.v < b.v || (a.v == b.v && (a.i < b.i || (a.i == b.i && a.j < b.j)));
}
__device__ __forceinline__ EncBest enc_min(const EncBest& a, const EncBest& b) {
  return enc_less(b, a) || a.v != a.v ? b : a;
}
// The best over the lanes of a wavefront, in every lane.
__device__ __forceinline__ EncBest enc_wave(EncBest b) {
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) {
    const EncBest o = {__shfl_xor(b.v, m, 64), __shfl_xor(b.i, m, 64), __shfl_xor(b.j, m, 64)};
    b = enc_min(b, o);
  }
  return b;
}
// The best over a workgroup (its first wavefront's lanes hold it).
__device__ __forceinline__ EncBest enc_block(EncBest b, EncBest* lds) {
  b = enc_wave(b);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = b;
  __syncthreads();
  b = lds[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) b = enc_min(b, lds[w]);
  return b;
}

__global__ __launch_bounds__(kBlock) void k_enc_stars(EncArgs a) {
  __shared__ EncBest lr[4], lz[4];
  __shared__ double lc[kBlock / 64];
  const int k = blockIdx.x * kBlock + threadIdx.x;
  EncBest r = {INFINITY, kNone, 0}, z = {INFINITY, kNone, 0};  // z: minus the ratio
  double cnt[1] = {0.0};
  if (k < a.Ns) {
    const double* x = a.pos + 3 * (size_t)(k + 1);
    const double* v = a.vel + 3 * (size_t)(k + 1);
    const double dx = x[0] - a.pos[0], dy = x[1] - a.pos[1], dz = x[2] - a.pos[2];
    const double r2 = dx * dx + dy * dy + dz * dz;
    a.pk[k] = make_double4(x[0], x[1], x[2], 0.0);
    r = {r2, k + 1, 0};
    z = {-bh_pair_ratio(dx, dy, dz, r2, v[0], v[1], v[2], a.G * a.mass[0], a.lam), k + 1, 0};
    cnt[0] = r2 < a.r_close2 ? 1.0 : 0.0;
  }
  r = enc_block(r, lr);
  z = enc_block(z, lz);
  group_sum<1>(cnt, lc);
  if (threadIdx.x == 0) {
    double* o = a.srow + (size_t)blockIdx.x * 10;
    o[0] = r.v;
    o[1] = r.i;
    o[2] = cnt[0];
    o[3] = z.v;
    o[4] = z.i;
  }
}

__global__ __launch_bounds__(kBlock) void k_enc_pair(TriArgs a,
                                                    const double4* __restrict__ pk) {
  __shared__ EncBest lds[4];
  double* row = a.rows + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * kTriRow;
  if (!tri_live(blockIdx.x, blockIdx.y, a.jchunk)) {
    if (threadIdx.x < 3) row[threadIdx.x] = threadIdx.x == 0 ? (double)INFINITY : (double)kNone;
    return;
  }
  const int i = blockIdx.x * kBlock + threadIdx.x;
  const double4 I = pk[min(i, a.Ns - 1)];
  auto dist2 = [&](const double4& p) {
    const double dx = I.x - p.x, dy = I.y - p.y, dz = I.z - p.z;
    return fma(dz, dz, fma(dy, dy, dx * dx));
  };
  double best = INFINITY;
  int bj = -1;         // the first (smallest) j with the smallest r^2 ...
  bool four_j = false; // ... or the first of the four that hold it
  auto take = [&](double r2, int j, bool ok, bool four) {
    const bool less = r2 < best && ok;
    best = less ? r2 : best;
    bj = less ? j : bj;
    four_j = less ? four : four_j;
  };
  tri_range(
      a, [&](int j) { take(dist2(pk[j]), j, j > i, false); },
      [&](int j) {
        const double4 p0 = pk[j], p1 = pk[j + 1], p2 = pk[j + 2], p3 = pk[j + 3];
        // (fmin passes over a NaN, as the comparison does)
        take(fmin(fmin(dist2(p0), dist2(p1)), fmin(dist2(p2), dist2(p3))), j, true, true);
      },
      [&](int j) { take(dist2(pk[j]), j, true, false); });
  if (four_j) {
    const int j = bj;
    bj = dist2(pk[j]) == best ? j : dist2(pk[j + 1]) == best ? j + 1
                                : dist2(pk[j + 2]) == best   ? j + 2
                                                             : j + 3;
  }
  EncBest b = {best, bj < 0 ? kNone : i + 1, bj < 0 ? kNone : bj + 1};  // body indices, i < j
  if (i >= a.Ns) b = {INFINITY, kNone, kNone};
  b = enc_block(b, lds);
  if (threadIdx.x == 0) {
    row[0] = b.v;
    row[1] = b.i;
    row[2] = b.j;
  }
}

__global__ __launch_bounds__(kTriFinal) void k_enc_final(EncArgs a) {
  __shared__ EncBest lr[kTriFinal / 64], lz[kTriFinal / 64], lp[kTriFinal / 64];
  __shared__ double lc[kTriFinal / 64];
  EncBest r = {INFINITY, kNone, 0}, z = {INFINITY, kNone, 0}, p = {INFINITY, kNone, kNone};
  double cnt[1] = {0.0};
  for (int k = threadIdx.x; k < a.nsrow; k += kTriFinal) {
    const double* o = a.srow + (size_t)k * 10;
    r = enc_min(r, EncBest{o[0], (int)o[1], 0});
    z = enc_min(z, EncBest{o[3], (int)o[4], 0});
    cnt[0] += o[2];
  }
#pragma unroll 4
  for (int k = threadIdx.x; k < a.nprow; k += kTriFinal) {
    const double* o = a.prow + (size_t)k * kTriRow;
    p = enc_min(p, EncBest{o[0], (int)o[1], (int)o[2]});
  }
  r = enc_block(r, lr);
  z = enc_block(z, lz);
  p = enc_block(p, lp);
  group_sum<1>(cnt, lc);
  if (threadIdx.x == 0) {
    const double none = (double)LLONG_MAX;
    a.out[0] = sqrt(r.v);
    a.out[1] = r.i == kNone ? none : (double)r.i;
    a.out[2] = cnt[0];
    a.out[3] = sqrt(p.v);
    a.out[4] = p.i == kNone ? none : (double)p.i;
    a.out[5] = p.j == kNone ? none : (double)p.j;
    a.out[6] = z.i == kNone ? -1.0 : -z.v;
    a.out[7] = z.i == kNone ? none : (double)z.i;
  }
}

// ---------------------------------------------------------------------------
// Unrestricted EIH equations for every pair (no massive-object truncation).
// In EIH layout the full 1PN pair term of body a with partner b is
//   (G m_b/R^2) n_ab [-v_a^2 - 2 v_b^2 + 4 v_a.v_b + 3/2 (n_ab.v_b)^2
//                     + 4 V_a + V_b + 1/2 x_ab.a^N_b]
//   + (G m_b/R^2) [n_ab.(4 v_a - 3 v_b)] (v_a - v_b) + 7/2 (G m_b/R) a^N_b,
// the limited star-star term with u_b -> V_b (the full potential) and
// -b_b -> a^N_b (the full Newtonian acceleration).  So it takes two sweeps
// over all N bodies with the same pair kernel: pass 1 (MODE_P1) gives V and
// a^N of every body; k_eih_mid writes them into the packets
// (e = -2 v^2 + V, hb = a^N / 2); pass 2 (MODE_P2) sums the 1PN terms.
// ---------------------------------------------------------------------------
struct EihArgs {
  const double* pos;
  const double* vel;
  const double* mass;
  int N;
  double G, lam;
  void* pk;           // [N] packets of all bodies
  double* va;         // [N][4]: V, a^N (3)
  const double* part; // [nsplit][kNF][N]
  int nsplit;
  double* acc_newton; // outputs (any may be nullptr)
  double* phi;
  double* acc_1pn;
  int* status;
};

template <typename T>
__global__ __launch_bounds__(kBlock) void k_eih_packets(EihArgs a) {
  using Pk = typename PkOf<T>::type;
  const int b = blockIdx.x * kBlock + threadIdx.x;
  if (b < a.N) {
    Pk p;
    p.x = a.pos[3 * b];
    p.y = a.pos[3 * b + 1];
    p.z = a.pos[3 * b + 2];
    p.gm = (T)(a.G * a.mass[b]);
    p.svx = (T)(PairScale<T>::sv * a.vel[3 * b]);
    p.svy = (T)(PairScale<T>::sv * a.vel[3 * b + 1]);
    p.svz = (T)(PairScale<T>::sv * a.vel[3 * b + 2]);
    p.e = T(0);
    p.hbx = T(0);
    p.hby = T(0);
    p.hbz = T(0);
    if constexpr (sizeof(T) == 8) {
      p.pad = 0.0;
    } else {
      p.pad0 = 0.f;
      p.pad1 = 0.f;
    }
    static_cast<Pk*>(a.pk)[b] = p;
  }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_eih_mid(EihArgs a) {
  using Pk = typename PkOf<T>::type;
  const int b = blockIdx.x * kBlock + threadIdx.x;
  if (b < a.N) {
    const size_t plane = (size_t)a.N;
    double U = 0.0, Gx = 0.0, Gy = 0.0, Gz = 0.0;
    for (int sp = 0; sp < a.nsplit; ++sp) {
      const double* pp = a.part + (size_t)sp * kNF * plane + b;
      U += pp[F_U * plane];
      Gx += pp[F_G * plane];
      Gy += pp[(F_G + 1) * plane];
      Gz += pp[(F_G + 2) * plane];
    }
    const double aN[3] = {-Gx, -Gy, -Gz};
    const double vx = a.vel[3 * b], vy = a.vel[3 * b + 1], vz = a.vel[3 * b + 2];
    Pk& p = static_cast<Pk*>(a.pk)[b];
    p.e = (T)(-2.0 * (vx * vx + vy * vy + vz * vz) + U);
    p.hbx = (T)(0.5 * aN[0]);
    p.hby = (T)(0.5 * aN[1]);
    p.hbz = (T)(0.5 * aN[2]);
    double* v4 = a.va + 4 * (size_t)b;
    v4[0] = U;
    v4[1] = aN[0];
    v4[2] = aN[1];
    v4[3] = aN[2];
    if (a.phi) a.phi[b] = -U;
    if (a.acc_newton) {
      a.acc_newton[3 * b] = aN[0];
      a.acc_newton[3 * b + 1] = aN[1];
      a.acc_newton[3 * b + 2] = aN[2];
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_eih_final(EihArgs a) {
  const int b = blockIdx.x * kBlock + threadIdx.x;
  if (b < a.N) {
    const size_t plane = (size_t)a.N;
    double sum[kNF];
#pragma unroll
    for (int f = 0; f < kNF; ++f) sum[f] = 0.0;
    for (int sp = 0; sp < a.nsplit; ++sp) {
      const double* pp = a.part + (size_t)sp * kNF * plane + b;
#pragma unroll
      for (int f = F_G; f < kNF; ++f) sum[f] += pp[f * plane];
    }
    sum[F_C2] *= kSqrt32;
    const double* v4 = a.va + 4 * (size_t)b;
    const double vx = a.vel[3 * b], vy = a.vel[3 * b + 1], vz = a.vel[3 * b + 2];
    const double v[3] = {vx, vy, vz};
    const double S0 = -(vx * vx + vy * vy + vz * vz) + 4.0 * v4[0];
    double a1[3];
    for (int c = 0; c < 3; ++c)
      a1[c] = a.lam * (S0 * sum[F_G + c] + sum[F_Q + c] + sum[F_C2] * v[c] + 7.0 * sum[F_Q7 + c]);
    if (a.acc_1pn) {
      a.acc_1pn[3 * b] = a1[0];
      a.acc_1pn[3 * b + 1] = a1[1];
      a.acc_1pn[3 * b + 2] = a1[2];
    }
    bool bad = false;
    for (int c = 0; c < 3; ++c) bad |= !isfinite(v4[1 + c] + a1[c]);
    if (bad) raise_status(a.status, kStatusNonfinite);
  }
}

// ---------------------------------------------------------------------------
// Batched ensemble: many independent systems in one launch per phase.
// Every phase's workgroups are numbered system after system in the order
// `order` (systems by decreasing cost, so the dispatcher, which starts
// workgroups in index order, hands out the largest systems first);
// `pre_*[r]` is the first workgroup of the r-th system in that order.  A
// workgroup finds its system by binary search over pre_* (scalar loads) and
// runs the same per-block code as the single-system kernels on that system's
// slices of the concatenated arrays.
// ---------------------------------------------------------------------------
struct SysDev {
  int64_t body0;  // first body (the massive object) in the concatenated body arrays
  int64_t star0;  // first star in the concatenated star arrays (packets, u/b)
  int64_t part0;  // first double of the system's pair partials
  int Ns, nsplit, jchunk, iblocks;
  int pro0, epi0;  // first row of the system's prologue / epilogue partials
  int npro, nepi;  // number of those rows
  double G, lam, eps2;
};

struct BatchArgs {
  const SysDev* sys;
  const int* order;
  const int* pre;  // prefix of this phase's workgroups over `order`, n_sys+1 entries
  int n_sys;
  const double* pos;  // evaluation state, concatenated [sum N][3]
  const double* vel;
  const double* mass;
  void* pk;  // packets of all stars
  double* ub;
  double* bpart;
  double* part;
  double* bhpart;
  int* status;
  int stage;
  double dt;
  double *X, *V, *Xs, *Vs, *KX, *KV;
};

// rank r of the system owning workgroup blk: pre[r] <= blk < pre[r+1]
__device__ __forceinline__ int batch_rank(const int* pre, int n, int blk) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (pre[mid] <= blk) lo = mid;
    else hi = mid;
  }
  return lo;
}

template <typename T>
__device__ __forceinline__ ProArgs batch_pro_args(const BatchArgs& b, const SysDev& S) {
  using Pk = typename PkOf<T>::type;
  ProArgs a;
  a.pos = b.pos + 3 * S.body0;
  a.vel = b.vel + 3 * S.body0;
  a.mass = b.mass + S.body0;
  a.Ns = S.Ns;
  a.G = S.G;
  a.eps2 = S.eps2;
  a.pk = static_cast<Pk*>(b.pk) + S.star0;
  a.ub = b.ub + 4 * S.star0;
  a.bpart = b.bpart + 8 * kProRows * (int64_t)S.pro0;
  a.status = b.status;
  return a;
}

__device__ __forceinline__ EpiArgs batch_epi_args(const BatchArgs& b, const SysDev& S) {
  EpiArgs a;
  const int64_t o3 = 3 * S.body0;
  a.pos = b.pos + o3;
  a.vel = b.vel + o3;
  a.mass = b.mass + S.body0;
  a.Ns = S.Ns;
  a.G = S.G;
  a.lam = S.lam;
  a.eps2 = S.eps2;
  a.ub = b.ub + 4 * S.star0;
  a.bpart = b.bpart + 8 * kProRows * (int64_t)S.pro0;
  a.nbpro = S.nepi;  // one prologue row per 64 stars
  a.part = b.part + S.part0;
  a.nsplit = S.nsplit;
  a.newton_only = 0;
  a.phi_in = nullptr;
  a.accN_in = nullptr;
  a.acc_newton = nullptr;
  a.phi = nullptr;
  a.acc_1pn = nullptr;
  a.bhpart = b.bhpart + 4 * (int64_t)S.epi0;
  a.nbepi = S.nepi;
  a.status = b.status;
  a.stage = b.stage;
  a.dt = b.dt;
  a.X = b.X + o3;
  a.V = b.V + o3;
  a.Xs = b.Xs + o3;
  a.Vs = b.Vs + o3;
  a.KX = b.KX + o3;
  a.KV = b.KV + o3;
  return a;
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_prologue_batched(BatchArgs b) {
  const int r = batch_rank(b.pre, b.n_sys, blockIdx.x);
  const SysDev S = b.sys[b.order[r]];
  prologue_block<T>(batch_pro_args<T>(b, S), blockIdx.x - b.pre[r]);
}

// IPT i-bodies per lane for every system of the ensemble (the plan's shape)
template <typename T, int IPT>
__global__ __launch_bounds__(kBlock) void k_pair_batched(BatchArgs b) {
  using Pk = typename PkOf<T>::type;
  const int r = batch_rank(b.pre, b.n_sys, blockIdx.x);
  const SysDev S = b.sys[b.order[r]];
  const int local = blockIdx.x - b.pre[r];
  PairArgs a;
  a.pk = static_cast<const Pk*>(b.pk) + S.star0;
  a.Ns = S.Ns;
  a.jchunk = S.jchunk;
  a.eps2 = S.eps2;
  a.part = b.part + S.part0;
  __shared__ double red[pair_red_doubles<T, IPT, 4>()];
  pair_block<T, MODE_FUSED, IPT, 4>(a, local % S.iblocks, local / S.iblocks, red);
}

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_epilogue_batched(BatchArgs b) {
  __shared__ double fsum[epi_fsum<double>()];
  const int r = batch_rank(b.pre, b.n_sys, blockIdx.x);
  const SysDev S = b.sys[b.order[r]];
  epilogue_block<double, void, WAVES>(batch_epi_args(b, S), blockIdx.x - b.pre[r], fsum);
}

__global__ __launch_bounds__(kBlock) void k_bh_final_batched(BatchArgs b) {
  const SysDev S = b.sys[b.order[blockIdx.x]];
  bh_final_block<double>(batch_epi_args(b, S));
}

}  // namespace pn
