// Fused energy / force / virial kernel for gfx950 (Section 3.1, Eqs. 1-10;
// fusion as in Section 3.4, re-designed for CDNA4).
//
// One persistent work-group (4 wavefronts, one per SIMD) walks a list of
// tiles.  A tile is up to 16 centre atoms of one species, consecutive in the
// cell-sorted order.  Per tile:
//
//   A. Stage the tile's atoms and neighbour rows; keep pairs with r < r_c and
//      bucket them by neighbour species in LDS, in atom order.  Each bucket
//      is cut into 16-pair chunks; all pairs of a chunk share one encoder
//      table (pair conditioning, Section 3.2).
//   B. Pass 1, one chunk per wavefront at a time: the radial encoder (Eq. 2)
//      and its derivative in r run as MFMA products with the 16 pairs as one
//      matrix dimension, the activation and its tangent as two column tiles
//      sharing every weight fragment (8-bit integer digits of both operands,
//      below, or 16x16x4 floating-point products).  The
//      moment P_i = sum_j g_ang (x) g_rad (Eq. 4) is another MFMA product
//      (K = pairs), accumulated into LDS.  The pre-cutoff output m and its
//      tangent dm (2k values per pair) go to a fixed-size per-work-group
//      workspace; nothing is recomputed in pass 2.  When the encoder is
//      recomputed in pass 2 instead (no workspace), pass 1 runs the forward
//      products alone: the moment needs m only.
//   C. Descriptor (Eq. 5), energy head (Eq. 6) and its gradient, and
//      W_i = dE_i/dP_i (Eq. 7) for the tile's atoms, in LDS (W overwrites P).
//   D. Pass 2, per chunk: v = W g and the reassociated radial term
//      s = g_ang^T W g' (Eqs. 8-9; U_i is never formed) as MFMA products,
//      then f_ij (Eq. 10), scatter F_j -= f_ij (global atomics) and
//      F_i += f_ij, w_i -= r_ij (x) f_ij (LDS atomics).
//   E. Write E_i, w_i, add F_i; block-reduce totals.
//
// The kernel is instantiated for two arithmetic types R of the network and
// the contractions: float64 (the paper's evaluation precision, Section 4.1)
// and float32 (the reduced-precision mode evaluated beside it, Sections 3.4
// and 4.4).  The minimum-image difference of positions and every output
// accumulation (F_i, F_j, w_i, E, totals) stay in float64 in both; r, the
// unit vector, the cutoff function, the network, the angular features, the
// moment, W, the two pass-2 contractions and the partial force use R.
//
// MFMA 16x16x4 register layout on gfx950 (lane = 16*g + c), for both types:
//   A operand: lane holds A[c][g]; B operand: lane holds B[g][c].
// The result layout differs: register q of lane holds D[drow(q, g)][c] with
// drow = 4q + g for float64 and 4g + q for float32.  A D-tile X can feed a
// later product as B (contracting over its rows; k-step q covers rows
// drow(q, 0..3)) or as A (X^T, same contraction); the host packs the head's
// weight fragments with the same row map.  The 8-bit integer 16x16x64 product
// of the encoder takes 16 bytes per lane (A[c][16g ..], B[16g ..][c]) and
// returns row 4g + q in both precisions.
//
// The file is compiled in six parts, whose instantiations build in parallel:
// MLIP_FUSED_PART 1 float64 to l_max 3, 2 float64 with l_max 4..5, 3 float32,
// each with the encoder on 8-bit integer digits (MLIP_FUSED_DIGITS 1) and on
// floating-point products (0), which a context takes when its weights are such
// that digits would lose accuracy.
#include <type_traits>

#include "kernel_math.h"
#include "mlip_internal.h"

namespace mlip {
namespace {

constexpr bool kDigits = MLIP_FUSED_DIGITS;

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

template <typename R>
struct Vec4;
template <>
struct Vec4<double> {
  typedef v4d type;
};
template <>
struct Vec4<float> {
  typedef v4f type;
};
template <typename R>
using v4 = typename Vec4<R>::type;

__device__ __forceinline__ v4d mfma(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ v4f mfma(float a, float b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Result row held in register q of a lane of group g.
template <typename R>
__device__ __forceinline__ int drow(int q, int g) {
  return sizeof(R) == 8 ? 4 * q + g : 4 * g + q;
}

// Logistic sigmoid 1 / (1 + exp(-z)) in float64, written out so that the
// vector instructions are few (they, not the matrix products, bound the
// encoder):
//  * exp(t), t = -z clamped to [-700, 700] (beyond that the sigmoid is 0 or 1
//    to far below float64 resolution of the SiLU value), by Cody-Waite
//    reduction t = n ln2 + r with |r| <= ln2/2, a degree-10 polynomial (the
//    interpolant at Chebyshev nodes, below 3.4e-16 relative error) and n
//    added to the exponent; n is rounded by adding 1.5 x 2^52, which leaves
//    it in the low word as an integer;
//  * 1 / (1 + e) from the hardware reciprocal estimate (relative error
//    measured below 2^-24) refined by one third-order step, y (1 + e + e^2).
// The constants are held in scalar registers (as vector constants the
// compiler copies them for every fused multiply-add).
struct SigmoidConst {
  double log2e, ln2hi, ln2lo, shift, top, bottom, c[10];
  __device__ __forceinline__ SigmoidConst()
      : log2e(1.4426950408889634),
        ln2hi(-6.93147180369123816490e-01),  // -ln2 split, high part exact in 32 bits
        ln2lo(-1.90821492927058770002e-10),
        shift(6755399441055744.0), top(700.0), bottom(-700.0),
        // polynomial interpolating exp at the 11 Chebyshev nodes of [-ln2/2,
        // ln2/2] (solved in 80-bit arithmetic, rounded to float64), highest
        // power first, constant term 1
        c{2.762635356445665e-07, 2.764018186396873e-06, 2.4801504368699663e-05, 0.00019841170267682938,
          0.0013888888932453442, 0.008333333385670185, 0.04166666666657336, 0.16666666666554397,
          0.5000000000000006, 1.0000000000000067} {
#pragma unroll
    for (int i = 0; i < 10; ++i) asm("" : "+s"(c[i]));
    asm("" : "+s"(log2e), "+s"(ln2hi), "+s"(ln2lo), "+s"(shift), "+s"(top), "+s"(bottom));
  }
};
__device__ __forceinline__ double sigmoid(double z, const SigmoidConst& k) {
  const double t = fmin(fmax(-z, k.bottom), k.top);
  const double y0 = fma(t, k.log2e, k.shift);
  const double n = y0 - k.shift;
  double r = fma(n, k.ln2hi, t);
  r = fma(n, k.ln2lo, r);
  double p = k.c[0];
#pragma unroll
  for (int i = 1; i < 10; ++i) p = fma(p, r, k.c[i]);
  p = fma(p, r, 1.0);
  const double e2 = __hiloint2double(__double2hiint(p) + (__double2loint(y0) << 20), __double2loint(p));
  const double d = 1.0 + e2;
  const double y = __builtin_amdgcn_rcp(d);
  const double e = fma(-d, y, 1.0);
  return fma(fma(e, e, e), y, y);
}
__device__ __forceinline__ double sigmoid(double z) { return sigmoid(z, SigmoidConst()); }

// Logistic sigmoid in float32 from the hardware base-2 exponential and
// reciprocal (each within about one ulp).  For large -z the exponential
// overflows to +inf and the reciprocal returns 0, the sigmoid's limit; for
// large z it underflows to 0 and the result is 1.
__device__ __forceinline__ float sigmoid(float z) {
  constexpr float kLog2e = 1.44269504f;
  const float e = __builtin_amdgcn_exp2f(-z * kLog2e);
  return __builtin_amdgcn_rcpf(1.0f + e);
}

struct NoConst {};
__device__ __forceinline__ float sigmoid(float z, const NoConst&) { return sigmoid(z); }
template <typename R>
struct SigmoidOf {
  typedef SigmoidConst Const;
};
template <>
struct SigmoidOf<float> {
  typedef NoConst Const;
};

// Slope of the SiLU z s(z), s (1 + z (1 - s)), as two fused multiply-adds:
// t = z - s z = z (1 - s), then s + s t.
template <typename R>
__device__ __forceinline__ R silu_slope(R z, R s) {
  return fma(s, fma(-s, z, z), s);
}

// Pair geometry after the minimum-image difference (which stays in float64):
// IEEE float64 square root and division, or the float32 hardware
// instructions (about one ulp).
__device__ __forceinline__ double vsqrt(double x) { return sqrt(x); }
__device__ __forceinline__ float vsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double vrcp(double x) { return 1.0 / x; }
__device__ __forceinline__ float vrcp(float x) { return __builtin_amdgcn_rcpf(x); }

// cos(x) and sin(x) for 0 <= x < pi (the cutoff function's argument, x =
// pi r / r_c with r < r_c) in float64: Cody-Waite reduction x = k pi/2 + y
// with k = rint(2x / pi) in {0, 1, 2} and |y| <= pi/4, the Taylor
// polynomials of sin (degree 15) and cos (degree 16) in y (truncation below
// 5e-17 and 3e-18; at degrees 13 and 14 the 2e-14 error of fc reached 6e-10
// in the forces of deep networks), then the quadrant rotation.  The general
// library routines carry range reduction for any argument, which this path
// never needs.
__device__ __forceinline__ void cut_sincos(double x, double* sn, double* cs) {
  constexpr double kTwoOverPi = 0.63661977236758134308;
  constexpr double kPio2Hi = 1.57079632679489655800e+00;  // pi/2 = hi + lo
  constexpr double kPio2Lo = 6.12323399573676603587e-17;
  const double k = rint(x * kTwoOverPi);
  double y = fma(-k, kPio2Hi, x);
  y = fma(-k, kPio2Lo, y);
  const double y2 = y * y;
  // 1 / n! for the odd (sin) and even (cos) terms, highest first
  double ps = -7.647163731819816e-13;  // -1/15!
  ps = fma(ps, y2, 1.6059043836821613e-10);  // 1/13!
  ps = fma(ps, y2, -2.505210838544172e-08);  // -1/11!
  ps = fma(ps, y2, 2.7557319223985893e-06);  // 1/9!
  ps = fma(ps, y2, -1.984126984126984e-04);  // -1/7!
  ps = fma(ps, y2, 8.333333333333333e-03);   // 1/5!
  ps = fma(ps, y2, -1.6666666666666666e-01); // -1/3!
  const double sy = fma(ps * y2, y, y);
  double pc = 4.779477332387385e-14;  // 1/16!
  pc = fma(pc, y2, -1.1470745597729725e-11); // -1/14!
  pc = fma(pc, y2, 2.08767569878681e-09);    // 1/12!
  pc = fma(pc, y2, -2.755731922398589e-07);  // -1/10!
  pc = fma(pc, y2, 2.48015873015873e-05);    // 1/8!
  pc = fma(pc, y2, -1.388888888888889e-03);  // -1/6!
  pc = fma(pc, y2, 4.1666666666666664e-02);  // 1/4!
  pc = fma(pc, y2, -0.5);                    // -1/2!
  const double cy = fma(pc, y2, 1.0);
  const int q = int(k);
  *sn = q == 0 ? sy : (q == 1 ? cy : -sy);
  *cs = q == 0 ? cy : (q == 1 ? -sy : -cy);
}

// Cutoff function fc(r) = (1 + cos(pi r / r_c)) / 2 and its derivative
// -(pi / r_c) sin(pi r / r_c) / 2 for r < r_c (Eq. 2): float64 from the
// reduced-range routine above, float32 from the hardware sine and cosine
// (about one ulp; they take revolutions).
__device__ __forceinline__ void cutoff(double r, double pi_rc, double* fc, double* dfc) {
  double sn, cs;
  cut_sincos(r * pi_rc, &sn, &cs);
  *fc = 0.5 * (1.0 + cs);
  *dfc = -0.5 * pi_rc * sn;
}
__device__ __forceinline__ void cutoff(float r, float pi_rc, float* fc, float* dfc) {
  const float x = r * pi_rc * 0.159154943f;
  *fc = 0.5f * (1.0f + __builtin_amdgcn_cosf(x));
  *dfc = -0.5f * pi_rc * __builtin_amdgcn_sinf(x);
}

// Exponents (a, b, c) of the Cartesian monomials of degree <= 5, degree by
// degree and lexicographic with x first within a degree (the column order of
// the angular table; its first 20 entries are the order of `monomials`).
struct MonoExp {
  unsigned char e[56][3];
  constexpr MonoExp() : e{} {
    int i = 0;
    for (int d = 0; d <= 5; ++d)
      for (int a = d; a >= 0; --a)
        for (int b = d - a; b >= 0; --b) {
          e[i][0] = (unsigned char)a;
          e[i][1] = (unsigned char)b;
          e[i][2] = (unsigned char)(d - a - b);
          ++i;
        }
  }
};
constexpr MonoExp kMonoExp{};

// The NM monomials (20: degree <= 3, 56: degree <= 5) of (x, y, z) and, when
// kGrad, their gradients.
template <int NM, bool kGrad, typename R>
__device__ __forceinline__ void monomials_n(R x, R y, R z, R m[NM], R gx[NM], R gy[NM], R gz[NM]) {
  if constexpr (NM == kMonomials) {
    monomials(x, y, z, m);
    if (kGrad) monomial_grads(x, y, z, gx, gy, gz);
  } else {
    R px[6], py[6], pz[6];
    px[0] = py[0] = pz[0] = R(1);
#pragma unroll
    for (int k = 1; k < 6; ++k) {
      px[k] = px[k - 1] * x;
      py[k] = py[k - 1] * y;
      pz[k] = pz[k - 1] * z;
    }
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      const int a = kMonoExp.e[i][0], b = kMonoExp.e[i][1], c = kMonoExp.e[i][2];
      m[i] = px[a] * py[b] * pz[c];
      if (kGrad) {
        gx[i] = a ? R(a) * px[a > 0 ? a - 1 : 0] * py[b] * pz[c] : R(0);
        gy[i] = b ? R(b) * px[a] * py[b > 0 ? b - 1 : 0] * pz[c] : R(0);
        gz[i] = c ? R(c) * px[a] * py[b] * pz[c > 0 ? c - 1 : 0] : R(0);
      }
    }
  }
}

// Slots of the per-tile table of the tile-reduced force scatter: a tile of
// up to 32 atoms has a few hundred distinct neighbours.
constexpr int kFjSlots = 1024;

// Rows of the moment kept in LDS: the angular rows of the configuration (16
// irreducible rows to l_max 3, the Cartesian basis's 20, 36 to l_max 5) of
// the DR rows that its 16-row MFMA tiles span; the rows past them are zero
// in every product and are neither stored nor read.
constexpr int moment_rows(int DR, int NM) { return NM == 56 ? 36 : (DR == 32 ? 20 : DR); }

template <int K, int TM, typename R, int NW, int DR, int NM>
struct Smem {
  R P[TM][moment_rows(DR, NM)][K + 1];  // moment, then its adjoint W (padded columns)
  // Pass 1 reads the first-layer weights; the head runs after pass 1 and
  // before the next tile is staged, so its activations reuse those bytes.
  union {
    struct {
      R l0[kMaxSpecies][2][kEncWidth];  // w0, b0 of the tile's encoder tables, by neighbour species
      R geo[NW][16][4];                 // unit vector and cutoff function of each wavefront's 16 pairs
    } p1;
    struct {
      R xT[(NM == 20 ? 4 : 6) * K][TM > 16 ? 32 : 16];  // head input vec(G), feature-major
      R yT[kHeadWidth][TM > 16 ? 32 : 16];             // head activations
      R gT[kHeadWidth][TM > 16 ? 32 : 16];             // head backward scratch
    } hd;
    // pass 2 of the cached configuration with the tile-reduced force
    // scatter: the tile's F_j contributions summed per neighbour j
    struct {
      int key[kFjSlots];        // neighbour index, -1 = empty
      double val[kFjSlots][3];
    } fj;
  } u;
  R qc[DR][NM];        // angular features over the monomials
  R rw[DR];            // descriptor weight of each angular row (metric C_l)
  double tpos[TM][3];
  double Fi[TM][3];
  double Wi[TM][9];
  double Ei[TM];
  long long row_beg[TM];
  int ent_base[TM + 1];
  int orig[TM];
  int cand[TM][9];     // cells scanned around each atom's cell (decoding coded list entries)
  int cnt[kMaxSpecies][TM];
  int base[kMaxSpecies][TM];
  int pair_j[tile_entry_cap(TM)];
  unsigned char pair_a[tile_entry_cap(TM)];
  int wsum[NW];
  int a0;
  int ch_start[tile_chunk_cap(TM)];
  unsigned char ch_count[tile_chunk_cap(TM)];
  unsigned char ch_s[tile_chunk_cap(TM)];
  int n_chunks;
  int next_chunk[2];  // dynamic chunk hand-out of pass 1 and pass 2
  int n_active;
  int tile_species;
  int na;
};

// Thread index, renewed for a phase of the kernel: what is computed from it
// (lane numbers, LDS and fragment offsets) is formed again in that phase.
// Left to itself the compiler forms all of it once before the tile loop, and
// the registers that hold it are then missing in the encoder.
__device__ __forceinline__ int phase_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Position of the neighbour in column c of chunk ch (or a dummy), fetched
// one chunk ahead so its latency overlaps the previous chunk's work.
struct PairPos {
  double x, y, z;
};

// Value of group g (0..3) among four, by bit masks: a select chain on the
// lane-dependent g would otherwise be compiled into divergent branches.
__device__ __forceinline__ double pick4(int g, double m0, double m1, double m2, double m3) {
  const unsigned long long s1 = 0ull - (unsigned long long)(g & 1), s2 = 0ull - (unsigned long long)((g >> 1) & 1);
  const unsigned long long lo = (__double_as_longlong(m0) & ~s1) | (__double_as_longlong(m1) & s1);
  const unsigned long long hi = (__double_as_longlong(m2) & ~s1) | (__double_as_longlong(m3) & s1);
  return __longlong_as_double((long long)((lo & ~s2) | (hi & s2)));
}
__device__ __forceinline__ float pick4(int g, float m0, float m1, float m2, float m3) {
  const unsigned s1 = 0u - unsigned(g & 1), s2 = 0u - unsigned((g >> 1) & 1);
  const unsigned lo = (__float_as_uint(m0) & ~s1) | (__float_as_uint(m1) & s1);
  const unsigned hi = (__float_as_uint(m2) & ~s1) | (__float_as_uint(m3) & s1);
  return __uint_as_float((lo & ~s2) | (hi & s2));
}

// Next chunk for this wavefront: chunks are handed out in order from an LDS
// counter, so a wavefront that runs ahead of its SIMD partner takes more of
// them and the wavefronts of a tile finish together.
__device__ __forceinline__ int grab_chunk(int* counter) {
  int v = 0;
  if ((threadIdx.x & 63) == 0) v = atomicAdd(counter, 1);
  return __builtin_amdgcn_readfirstlane(__shfl(v, 0, 64));
}

template <int K, int TM, typename R, int NW, int DR, int NM>
__device__ __forceinline__ PairPos load_pair_pos(const FusedArgs& A, const Smem<K, TM, R, NW, DR, NM>& S, int ch) {
  const int c = phase_tid() & 15;
  PairPos p{0.0, 0.0, 0.0};
  if (c < S.ch_count[ch]) {
    const long long j = S.pair_j[S.ch_start[ch] + c];
    p.x = A.pos[3 * j];
    p.y = A.pos[3 * j + 1];
    p.z = A.pos[3 * j + 2];
  }
  return p;
}

// Fragment array at a wave-uniform address, read through a buffer descriptor:
// the descriptor and each group's offset are scalar and the lane offset is
// one fixed vector register, so walking the array costs no vector address
// arithmetic (which on this part would share the pipe with the float64
// MFMAs); a read past `bytes` returns zero instead of touching other memory.
// Group e holds one V per lane, lane l at byte (64 e + l) sizeof(V).
constexpr int kRawBufferConfig = 0x00020000;  // raw untyped access, gfx9-family descriptor word 3
template <typename V>
struct FragStream {
  __amdgpu_buffer_rsrc_t rs;
  int lo;
  __device__ __forceinline__ FragStream(const void* base, int bytes)
      : rs(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, kRawBufferConfig)),
        lo((phase_tid() & 63) * int(sizeof(V))) {}
  __device__ __forceinline__ V operator[](int e) const {
    const int so = e * 64 * int(sizeof(V));
    if constexpr (sizeof(V) == 16) return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rs, lo, so, 0));
    else if constexpr (sizeof(V) == 8) return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(rs, lo, so, 0));
    else return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b32(rs, lo, so, 0));
  }
};

// Per-row values of a weight matrix at a wave-uniform address: the four rows
// 16 To + 4 g + q of a lane.
template <typename R>
struct RowStream {
  const R* p;
  __device__ __forceinline__ RowStream(const R* base, int g) : p(base + 4 * g) {}
  __device__ __forceinline__ void load(int To, R (&v)[4]) const {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = p[16 * To + q];
  }
};

// Row of the encoder's outputs held in register q of a lane of group g, within
// a 16-row tile (with pairs as rows: the pair), and the order in which pass 2
// contracts the columns of m: the integer products return row 4g + q in both
// precisions, floating-point ones drow(q, g).  Row c sits in register hreg(c)
// of the lanes of group hgroup(c).
template <typename R>
constexpr bool kRowsByGroup = kDigits || sizeof(R) == 4;
template <typename R>
__device__ __forceinline__ int hrow(int q, int g) {
  return kRowsByGroup<R> ? 4 * g + q : 4 * q + g;
}
template <typename R>
__device__ __forceinline__ int hgroup(int c) {
  return kRowsByGroup<R> ? c >> 2 : c & 3;
}
template <typename R>
__device__ __forceinline__ int hreg(int c) {
  return kRowsByGroup<R> ? c & 3 : c >> 2;
}

// ---- products on the 8-bit integer matrix pipe ------------------------------
// A float64 MFMA runs at the rate of float64 FMAs and holds the vector pipe
// for its whole duration; 8-bit integer MFMAs run 64 times as fast (32 times a
// float32 MFMA) and leave the vector pipe free.  The encoder's products are
// therefore formed on digits (Ozaki's scheme): with a scale per weight row and
// per activation column, both operands are rounded to integers of balanced
// base-256 digits, X = sum_i d_i 256^(D-1-i), d_i in [-128, 127], and
//   sum_k X_k Y_k = sum_i sum_j 256^(D+D'-2-i-j) sum_k d_i[k] e_j[k],
// whose inner sums are exact in 32 bits (128 products of at most 2^14, at
// most seven of them per i + j: below 2^24).  Digit products of the lowest
// weights are left out.  That and the rounding of both operands err by less
// than 128 x 2^-53 (float32: 128 x 2^-29) of (largest weight of the row) x
// (largest value of the column), where floating-point products err by a part of
// the sum of the absolute terms; for weights whose terms are small beside that
// product of maxima the other encoder below is taken.
//
// float64: seven digits (56 bits), the 28 digit products with i + j <= 6.
// Measured against a float64 reference the outputs are as close as with float64
// MFMAs: 1.08e-15, 4.65e-15 and 4.63e-15 of E, F and w at 1,048,576 atoms,
// 1.09e-15, 4.65e-15 and 4.64e-15 with them.  An encoder call of 16 pairs (two
// hidden layers) takes 59 thousand cycles at 2.1 GHz, 28 us, instead of 91
// thousand at 2.34 GHz, 39 us; the kernel 201.4 ms instead of 252.4 ms at
// 1,048,576 atoms of six species.
//
// float32: four digits (32 bits) of both, the ten digit products with i + j
// <= 3.  Three digits of an activation (24 bits under the column's scale, nine
// products) are 2% faster (85.63 against 87.11 ms, list and evaluation of
// 1,048,576 atoms), but values below the column's largest then have fewer bits
// than float32 gives them: with one hidden unit 100 times the others (and its
// weights in the next layers 1/100) forces were off by 8.4e-6, 1.1e-6 with
// float32 MFMAs and 9.8e-7 with four digits.  With ordinary weights (131,072
// atoms, six species) 1.39e-6, 1.60e-6 with float32 MFMAs.
//
// What takes the time is issue, with one wavefront per SIMD (float64; two in
// float32): counted over the whole kernel, 97 vector instructions and 22 MFMAs
// per activation and tangent in float64, 44 and 8 in float32.  At 4 cycles each
// that is half of a SIMD's cycles in both precisions (two thirds in float64 at
// the 4.5 and 9 measured on one wavefront); the matrix pipe is busy for 40 and
// 35% of them, and a wavefront waits for memory or LDS for 20 and 27% of its own.
template <typename R>
struct Split;
template <>
struct Split<double> {
  [[maybe_unused]] static constexpr int W = 7, D = 7, S = 7;  // digits of weights and activations, sums (i + j < S)
};
template <>
struct Split<float> {
  [[maybe_unused]] static constexpr int W = 4, D = 4, S = 4;
};
static_assert(Split<double>::W == weight_digits(64) && Split<float>::W == weight_digits(32), "packed digits");
typedef int v4i __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4i mfma_i8(v4i a, v4i b, v4i c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}

// Activation columns in digits: s[i][hf] holds digit i of the rows
// 64 hf + 16 t + 4 g + q of column c in byte 4 t + q, which is both the B
// operand (rows as k) and the A operand (columns as rows) of a 16x16x64
// product.  inv: value of a unit of the top three digits.
template <typename R>
struct Digits {
  v4i s[Split<R>::D][2];
  R inv;
};

// Scale that takes a column's largest magnitude (over the lane's 32 values
// and its column's four lanes) to just below 0.99 x 2^23: the closer to the
// full range, the less the digit products that are left out weigh.  A column
// with an infinity or NaN gets a NaN inverse, so everything formed from it is
// NaN; one of zeros (or below 2^-974, in float32 2^-92) gets scale and inverse
// zero.  In float32 the scale returned is that of all four digits, 2^8 times
// as large.
__device__ __forceinline__ int top_bits(double x) { return __double2hiint(x); }
__device__ __forceinline__ int top_bits(float x) { return __float_as_int(x); }
template <typename R>
__device__ __forceinline__ R digit_scale(const R (&h)[8][4], Digits<R>& d) {
  // largest magnitude by the (high) words: as signed integers for positive
  // values, as unsigned for negative ones
  int mp = 0;
  unsigned mn = 0;
#pragma unroll
  for (int T = 0; T < 8; ++T)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int hi = top_bits(h[T][q]);
      mp = max(mp, hi);
      mn = max(mn, unsigned(hi));
    }
  unsigned m = max(unsigned(mp), mn >> 31 ? mn & 0x7fffffffu : 0u);
  m = max(m, unsigned(__shfl_xor(int(m), 16, 64)));
  m = max(m, unsigned(__shfl_xor(int(m), 32, 64)));
  constexpr double kRange = 0.99 * 8388608.0;  // seven balanced digits hold 0.996 x 2^23 x 2^32
  R scale, inv;
  unsigned low, high;  // range of m whose scale and inverse are normal
  if constexpr (sizeof(R) == 8) {
    const double top = __hiloint2double(int(m + 1), 0);  // above every magnitude of the column
    const double y = __builtin_amdgcn_rcp(top);
    scale = kRange * fma(fma(-top, y, 1.0), y, y);
    inv = top * (1.0 / kRange);
    low = 0x03100000u, high = 0x7fd00000u;
  } else {
    const float top = __int_as_float(int(m));
    scale = float(kRange) * __builtin_amdgcn_rcpf(top);
    inv = top * float(1.0 / kRange);
    low = 0x11800000u, high = 0x7e800000u;
  }
  inv = fma(fma(-scale, inv, R(1)), inv, inv);
  if (m - low >= high - low) {
    scale = R(0);
    inv = m >= high ? R(__builtin_nanf("")) : R(0);
  }
  d.inv = inv;
  return sizeof(R) == 8 ? scale : scale * R(256);
}

// Digits of the half hf of a lane's values (tiles 4 hf .. 4 hf + 3): the value
// is rounded to an integer and a remainder, the remainder to 32 bits, by
// adding 1.5 x 2^52, which leaves the integers in the low words (and the
// remainder's carry in its high word).  An offset of 128 in every digit
// (0x808080 in the upper 24 bits, 0x80808080 in the lower 32) makes the digits
// the bytes of a non-negative integer, up to the offset itself, taken off by
// flipping each byte's top bit.
__device__ __forceinline__ void make_digits(const double (&h)[8][4], double scale, int hf, Digits<double>& d) {
  constexpr double kShift = 6755399441055744.0;
  double upper = kShift + 8421504.0, lower = kShift + 2155905152.0, two32 = 4294967296.0;
  // opaque, or their copies for accumulating instructions would outnumber
  // the arithmetic
  asm("" : "+s"(upper), "+s"(two32));
  asm("" : "+v"(lower));
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    unsigned hw[4], lw[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double x = h[4 * hf + t][q];
      const double y = fma(x, scale, upper);
      const double rem = fma(x, scale, upper - y);
      const double v = fma(rem, two32, lower);
      lw[q] = unsigned(__double2loint(v));
      hw[q] = unsigned(__double2loint(y)) + unsigned(__double2hiint(v)) - 0x43380000u;
    }
    // 4 x 4 byte transposes
    const unsigned a = __builtin_amdgcn_perm(hw[1], hw[0], 0x05010400u), b = __builtin_amdgcn_perm(hw[3], hw[2], 0x05010400u);
    const unsigned e = __builtin_amdgcn_perm(hw[1], hw[0], 0x06020602u), f = __builtin_amdgcn_perm(hw[3], hw[2], 0x06020602u);
    const unsigned p = __builtin_amdgcn_perm(lw[1], lw[0], 0x07030602u), q = __builtin_amdgcn_perm(lw[3], lw[2], 0x07030602u);
    const unsigned r = __builtin_amdgcn_perm(lw[1], lw[0], 0x05010400u), z = __builtin_amdgcn_perm(lw[3], lw[2], 0x05010400u);
    const unsigned w[7] = {
        __builtin_amdgcn_perm(f, e, 0x05040100u), __builtin_amdgcn_perm(b, a, 0x07060302u),
        __builtin_amdgcn_perm(b, a, 0x05040100u), __builtin_amdgcn_perm(q, p, 0x07060302u),
        __builtin_amdgcn_perm(q, p, 0x05040100u), __builtin_amdgcn_perm(z, r, 0x07060302u),
        __builtin_amdgcn_perm(z, r, 0x05040100u)};
#pragma unroll
    for (int i = 0; i < 7; ++i) d.s[i][hf][t] = int(w[i] ^ 0x80808080u);
  }
  // kept in accumulation registers: matrix operands only from here on
#pragma unroll
  for (int i = 0; i < 7; ++i) asm("" : "+a"(d.s[i][hf]));
}
// float32: the four digits of the value cut to an integer (24 bits of the
// largest values, so only those below 2^-7 of the column's largest lose any,
// at most 2^-31 of it).
__device__ __forceinline__ void make_digits(const float (&h)[8][4], float scale, int hf, Digits<float>& d) {
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    unsigned x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = unsigned(int(h[4 * hf + t][q] * scale)) + 0x80808080u;
    // 4 x 4 byte transpose
    const unsigned a = __builtin_amdgcn_perm(x[1], x[0], 0x05010400u), b = __builtin_amdgcn_perm(x[3], x[2], 0x05010400u);
    const unsigned e = __builtin_amdgcn_perm(x[1], x[0], 0x07030602u), f = __builtin_amdgcn_perm(x[3], x[2], 0x07030602u);
    const unsigned w[4] = {__builtin_amdgcn_perm(b, a, 0x05040100u), __builtin_amdgcn_perm(b, a, 0x07060302u),
                           __builtin_amdgcn_perm(f, e, 0x05040100u), __builtin_amdgcn_perm(f, e, 0x07060302u)};
#pragma unroll
    for (int i = 0; i < 4; ++i) d.s[i][hf][t] = int(w[3 - i] ^ 0x80808080u);
  }
}
template <typename R>
__device__ __forceinline__ void make_digits(const R (&h)[8][4], Digits<R>& d) {
  const R scale = digit_scale(h, d);
  make_digits(h, scale, 0, d);
  make_digits(h, scale, 1, d);
}

// Sum of the digit products, S[d] = sum over i + j = d:
// 2^8 sum_d S[d] 2^(-8d), exact up to the last rounding (float64: and to 2^-40
// of a unit of S[0]; float32: up to the rounding of the two merged sums).  The
// pairs that are merged as integers stay below 2^31 (at most 1.62e9).
__device__ __forceinline__ double digit_sum(const v4i (&S)[7], int q) {
  const int a = (S[0][q] << 8) + S[1][q], b = (S[2][q] << 8) + S[3][q], e = S[5][q] + (S[6][q] >> 8);
  double t = fma(double(S[4][q]), 0x1p-8, double(b));
  t = fma(double(e), 0x1p-16, t);
  return fma(t, 0x1p-16, double(a));
}
__device__ __forceinline__ float digit_sum(const v4i (&S)[4], int q) {
  const int a = (S[0][q] << 8) + S[1][q], b = (S[2][q] << 8) + S[3][q];
  return fma(float(b), 0x1p-16f, float(a));
}

// Weight tile of an integer product: digit i of half hf is fragment W hf + i
// (64 lanes of 16 bytes).
template <typename R>
constexpr int kTileFrags = 2 * Split<R>::W;
// Values of R that the fragments of n tiles take in a table.
template <typename R>
constexpr int frag_values(int n) {
  return n * kTileFrags<R> * 1024 / int(sizeof(R));
}

// Minimum-image vector r_ij of the pair in column c of chunk ch (Eq. 1), in
// float64; (1, 0, 0) and atom -1 for the padding columns of a partial chunk.
template <int K, int TM, typename R, int NW, int DR, int NM>
__device__ __forceinline__ void pair_delta(const FusedArgs& A, const Smem<K, TM, R, NW, DR, NM>& S, int ch,
                                           const PairPos& pp, double* dx, double* dy, double* dz, int* atom) {
  const int c = phase_tid() & 15;
  *dx = 1.0; *dy = 0.0; *dz = 0.0; *atom = -1;
  if (c >= S.ch_count[ch]) return;
  const int a = S.pair_a[S.ch_start[ch] + c];
  *dx = fold(pp.x - S.tpos[a][0], A.box[0], A.inv_box[0]);
  *dy = fold(pp.y - S.tpos[a][1], A.box[1], A.inv_box[1]);
  *dz = fold(pp.z - S.tpos[a][2], A.box[2], A.inv_box[2]);
  *atom = a;
}

// Encoder table of chunk ch (pair conditioning, Section 3.2).
template <int K, int TM, typename R, int NW, int DR, int NM>
__device__ __forceinline__ const R* chunk_table(const FusedArgs& A, const Smem<K, TM, R, NW, DR, NM>& S, int ch) {
  // the same for every lane: kept in scalar registers, so the weight loads
  // take a scalar base and the k-step offsets cost no vector instructions
  const int sj = __builtin_amdgcn_readfirstlane(S.ch_s[ch]);
  const int si = __builtin_amdgcn_readfirstlane(S.tile_species);
  const int tau = A.enc_cond == 2 ? si * A.C + sj : (A.enc_cond == 1 ? sj : 0);
  return static_cast<const R*>(A.enc) + (long long)tau * A.enc_stride;
}

// What the hidden layers leave for the output layer.
template <typename R>
struct Hidden {
  Digits<R> h, dh;
};

// Products of half a 16-row weight tile (columns 64 hf .., fragments w[W hf ..])
// with the digits x of 16 columns: 28 MFMAs in float64, 10 in float32.  With kNext each fragment's
// registers take the fragment at next + f of the stream after its last use,
// half a tile of products before that one is needed.  kRows: the activation
// columns are the rows of the result.
template <bool kRows, bool kNext, typename R>
__device__ __forceinline__ void half_products(v4i (&w)[kTileFrags<R>], const Digits<R>& x, v4i (&S)[Split<R>::S], int hf,
                                              const FragStream<v4i>& frag, int next) {
  constexpr int W = Split<R>::W, D = Split<R>::D;
  if (hf == 0) {
#pragma unroll
    for (int i = 0; i < Split<R>::S; ++i) S[i] = v4i{0, 0, 0, 0};
  }
#pragma unroll
  for (int i = 0; i < W; ++i) {
    const int f = hf * W + i;
#pragma unroll
    for (int j = 0; j < D && i + j < Split<R>::S; ++j)
      S[i + j] = kRows ? mfma_i8(x.s[j][hf], w[f], S[i + j]) : mfma_i8(w[f], x.s[j][hf], S[i + j]);
    if constexpr (kNext) w[f] = frag[next + f];
  }
}
template <bool kRows, bool kNext, typename R>
__device__ __forceinline__ void tile_products(v4i (&w)[kTileFrags<R>], const Digits<R>& x, v4i (&S)[Split<R>::S],
                                              const FragStream<v4i>& frag, int next) {
  half_products<kRows, kNext>(w, x, S, 0, frag, next);
  half_products<kRows, kNext>(w, x, S, 1, frag, next);
}

// Order of a region that holds the MFMAs of half_products and vector work:
// kValu vector instructions after each MFMA, and with kLoads each fragment's
// load after its last use.  A 16x16x64 integer MFMA occupies the matrix pipe
// for 16 cycles and issue for about 9, a vector instruction issue for 4 to 5
// (measured on one wavefront), so two vector instructions fit beside each.
template <typename R, int kValu, bool kLoads>
__device__ __forceinline__ void interleave() {
#pragma unroll
  for (int i = 0; i < Split<R>::W; ++i) {
#pragma unroll
    for (int j = 0; j < Split<R>::D && i + j < Split<R>::S; ++j) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, kValu, 0);
    }
    if constexpr (kLoads) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
}

// Encoder forward and tangent (Eq. 2 and its derivative in r) up to the last
// hidden layer for the 16 pairs of a chunk: the first layer (scalar input)
// from the LDS copy of (w0, b0), then the residual hidden layers Z = W H.
// Without kTan only the forward runs: the moment needs the encoder output
// alone, so a pass 1 that keeps no workspace skips the tangent's half.  The
// result is the output-layer section of the table.
//
// Each layer's products are formed on digits (above), one 16-row tile at a
// time: first the activations' products, then the tangents'.  The vector work
// that turns a tile's sums into new activations is spread over the products
// that follow, about two instructions per MFMA.
template <int K, int TM, typename R, int NW, int DR, int NM, bool kTan = true>
__device__ __forceinline__ const R* encoder_hidden(const FusedArgs& A, const Smem<K, TM, R, NW, DR, NM>& S, int sj, R r,
                                                   const R* __restrict__ tab, Hidden<R>& out) {
  const int lane = phase_tid() & 63, g = lane >> 4;
  constexpr int kFrags = frag_values<R>(8);
  // float32 runs two wavefronts per SIMD, which fill each other's gaps; there
  // the compiler's own order measured 2% faster
  constexpr bool kOrder = sizeof(R) == 8;
  const int nh = A.enc_hidden;
  const R* __restrict__ layer = tab + 2 * kEncWidth;
  const typename SigmoidOf<R>::Const kc;
  R h[8][4], dh[8][4];
#pragma unroll
  for (int T = 0; T < 8; ++T)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int in = 16 * T + 4 * g + i;
      const R w0 = S.u.p1.l0[sj][0][in], z = w0 * r + S.u.p1.l0[sj][1][in];
      const R s = sigmoid(z, kc);
      h[T][i] = z * s;
      if constexpr (kTan) {
        dh[T][i] = silu_slope(z, s) * w0;
      }
    }
  for (int t = 1; t < nh; ++t) {
    const FragStream<v4i> frag(layer, int(kFrags * sizeof(R)));
    const R* __restrict__ rows = layer + kFrags;  // row scales, then biases
    const RowStream<R> scale(rows, g), bias(rows + kEncWidth, g);
    v4i w[kTileFrags<R>];
#pragma unroll
    for (int f = 0; f < kTileFrags<R>; ++f) w[f] = frag[f];
    const R dsc = digit_scale(h, out.h);
    R dsct = 0;
    if constexpr (kTan) dsct = digit_scale(dh, out.dh);
    make_digits(h, dsc, 0, out.h);
    v4i sf[Split<R>::S], st[Split<R>::S];
    R sc[4], bi[4], z[4], slope[4];
    auto act = [&](int T, int q) {
      const R s = sigmoid(z[q], kc);
      h[T][q] = fma(z[q], s, h[T][q]);
      if constexpr (kTan) slope[q] *= silu_slope(z[q], s);
    };
    auto sum = [&](int q) {
      const R rs = sc[q];
      z[q] = fma(digit_sum(sf, q) * rs, out.h.inv, bi[q]);
      if constexpr (kTan) slope[q] = rs * out.dh.inv;
    };
    auto tan_sum = [&](int T, int q) {
      dh[T][q] = fma(slope[q], digit_sum(st, q), dh[T][q]);
    };
    if constexpr (kOrder) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int To = 0; To <= 8; ++To) {
      const int next = (To + 1) * kTileFrags<R>;
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        if (To < 8 && hf == 1) {
          scale.load(To, sc);
          bias.load(To, bi);
        }
        if (To < 8) half_products<false, !kTan>(w, out.h, sf, hf, frag, next);
        if (To > 0) {
          act(To - 1, 2 + hf);
          if constexpr (kTan) {
            tan_sum(To - 1, 2 * hf);
            tan_sum(To - 1, 2 * hf + 1);
          }
        } else {
          if (hf == 0) make_digits(h, dsc, 1, out.h);
          else if constexpr (kTan) make_digits(dh, dsct, 0, out.dh);
        }
        if constexpr (kOrder) {
          if (To == 0) interleave<R, 5, !kTan>();
          else if (To < 8) interleave<R, 2, !kTan>();
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (To == 8) continue;
      if constexpr (kTan) {
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          half_products<false, true>(w, out.dh, st, hf, frag, next);
          if (hf == 0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) sum(q);
            if (To == 0) make_digits(dh, dsct, 1, out.dh);
          } else {
            act(To, 0);
            act(To, 1);
          }
          if constexpr (kOrder) {
            if (To == 0 && hf == 0) interleave<R, 7, true>();
            else interleave<R, 2, true>();
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) sum(q);
        act(To, 0);
        act(To, 1);
      }
    }
    layer = rows + 2 * kEncWidth;
  }
  make_digits(h, out.h);
  if constexpr (kTan) make_digits(dh, out.dh);
  return layer;
}

// Encoder output layer with pairs as rows: mo[Tc] register q holds
// m[pair 4g + q][16Tc + c] (dmo the same for the tangent).
template <int K, typename R, bool kTan = true>
__device__ __forceinline__ void encoder_out_rows(const R* __restrict__ layer, const Hidden<R>& in, v4<R> (&mo)[K / 16],
                                                 v4<R> (&dmo)[K / 16]) {
  constexpr int KT = K / 16;
  constexpr int kFrags = frag_values<R>(KT);
  const int lane = phase_tid() & 63, g = lane >> 4, c = lane & 15;
  const FragStream<v4i> frag(layer, int(kFrags * sizeof(R)));
  const R* __restrict__ cols = layer + kFrags;
  v4i w[kTileFrags<R>], sf[Split<R>::S], st[Split<R>::S];
#pragma unroll
  for (int f = 0; f < kTileFrags<R>; ++f) w[f] = frag[f];
  R inv[4], dinv[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    inv[q] = __shfl(in.h.inv, 4 * g + q, 64);
    if constexpr (kTan) dinv[q] = __shfl(in.dh.inv, 4 * g + q, 64);
  }
#pragma unroll
  for (int Tc = 0; Tc < KT; ++Tc) {
    const R sc = cols[16 * Tc + c], b = cols[K + 16 * Tc + c];
    tile_products<true, !kTan>(w, in.h, sf, frag, (Tc + 1) * kTileFrags<R>);
    if constexpr (kTan) tile_products<true, true>(w, in.dh, st, frag, (Tc + 1) * kTileFrags<R>);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      mo[Tc][q] = fma(digit_sum(sf, q) * sc, inv[q], b);
      if constexpr (kTan) dmo[Tc][q] = digit_sum(st, q) * sc * dinv[q];
    }
  }
}

// Encoder output layer with pairs as columns: register q of lane (g, c) for
// output tile Tc holds m[pair c][16Tc + 4g + q], the B operand of pass 2's
// W m product.
template <int K, typename R>
__device__ __forceinline__ void encoder_out_cols(const R* __restrict__ layer, const Hidden<R>& in, R (&mB)[K / 16][4],
                                                 R (&dmB)[K / 16][4]) {
  constexpr int KT = K / 16;
  constexpr int kFrags = frag_values<R>(KT);
  const int lane = phase_tid() & 63, g = lane >> 4;
  const FragStream<v4i> frag(layer, int(kFrags * sizeof(R)));
  const R* __restrict__ rows = layer + kFrags;
  const RowStream<R> scale(rows, g), bias(rows + K, g);
  v4i w[kTileFrags<R>], sf[Split<R>::S], st[Split<R>::S];
#pragma unroll
  for (int f = 0; f < kTileFrags<R>; ++f) w[f] = frag[f];
#pragma unroll
  for (int Tc = 0; Tc < KT; ++Tc) {
    R sc[4], b[4];
    scale.load(Tc, sc);
    bias.load(Tc, b);
    tile_products<false, false>(w, in.h, sf, frag, 0);
    tile_products<false, true>(w, in.dh, st, frag, (Tc + 1) * kTileFrags<R>);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      mB[Tc][q] = fma(digit_sum(sf, q) * sc[q], in.h.inv, b[q]);
      dmB[Tc][q] = digit_sum(st, q) * sc[q] * in.dh.inv;
    }
  }
}

// ---- the encoder on floating-point products ---------------------------------
// For weights whose terms the digits would not hold (digits_hold in api.cpp):
// 16x16x4 MFMAs of the network's type, the activation and its tangent sharing
// every weight fragment.  A float64 one holds the vector pipe for its duration,
// so products and activation functions add up: 1,048,576 atoms of six species
// take 252.4 ms instead of 201.4, in float32 119.5 instead of 84.
//
// Fragments of VW consecutive output tiles per 16-byte load stream through
// register rings issued kRing - 1 (hidden layers) or kRingO - 1 (output layer)
// k-steps ahead of the MFMAs that consume them.  An output-layer k-step is
// only 2 KT products, so its ring runs further ahead.  The float32 kernel runs
// two wavefronts per SIMD, which cover each other's load latency; there
// shallower rings leave more registers and measured faster (ring depths 2 and
// 4 against 3 and 8).
template <int K, typename R>
struct Stream {
  static constexpr int KT = K / 16;
  static constexpr int VW = 16 / int(sizeof(R));  // fragments per load
  static constexpr int NH = 8 / VW;               // loads per hidden-layer k-step
  static constexpr int VO = KT < VW ? KT : VW;    // fragments per output-layer load
  static constexpr int NO = KT / VO;              // loads per output-layer k-step
  static constexpr int kRing = sizeof(R) == 8 ? 3 : 2;
  static constexpr int kRingO = sizeof(R) == 8 ? 8 : 4;
  typedef R vh_t __attribute__((ext_vector_type(VW)));
  typedef R vo_t __attribute__((ext_vector_type(VO)));
};

// Bias vector of a hidden layer at a wave-uniform address, read through a
// buffer descriptor in the accumulator row order: element (To, q) of lane
// (g, c) is row 16 To + drow(q, g); the lane part of that offset is one
// fixed vector register, the rest a scalar offset.  With bytes = 0 every
// read returns zero without touching memory.
template <typename R>
struct BiasStream {
  __amdgpu_buffer_rsrc_t rs;
  int lo;
  __device__ __forceinline__ BiasStream(const void* base, int bytes, int g)
      : rs(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, kRawBufferConfig)),
        lo((sizeof(R) == 8 ? g : 4 * g) * int(sizeof(R))) {}
  __device__ __forceinline__ R operator()(int To, int q) const {
    const int so = (16 * To + (sizeof(R) == 8 ? 4 * q : q)) * int(sizeof(R));
    if constexpr (sizeof(R) == 8) return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b64(rs, lo, so, 0));
    else return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b32(rs, lo, so, 0));
  }
};

// What the hidden layers leave for the output layer: rows 16T + drow(i, g) of
// column c.
template <typename R>
struct FloatHidden {
  R h[8][4], dh[8][4];
};

// Encoder forward and tangent up to the last hidden layer, as above, with the
// hidden layers as 8 x 32 MFMA steps.
template <int K, int TM, typename R, int NW, int DR, int NM, bool kTan = true>
__device__ __forceinline__ const R* encoder_hidden(const FusedArgs& A, const Smem<K, TM, R, NW, DR, NM>& S, int sj, R r,
                                                   const R* __restrict__ tab, FloatHidden<R>& out) {
  typedef Stream<K, R> St;
  typedef typename St::vh_t vh_t;
  constexpr int NH = St::NH, VW = St::VW, kRing = St::kRing;
  const int lane = phase_tid() & 63, g = lane >> 4;
  const typename SigmoidOf<R>::Const kc;
  R (&h)[8][4] = out.h;
  R (&dh)[8][4] = out.dh;
  constexpr int kLayerBytes = int(kEncWidth * kEncWidth * sizeof(R));
  constexpr int kBiasBytes = int(kEncWidth * sizeof(R));
  const int nh = A.enc_hidden;
  // The first hidden layer's leading weight fragments are requested before
  // the elementwise first layer, whose activation work covers their
  // latency; each hidden layer requests the next one's in its last k-steps,
  // so they arrive during its own activation phase.  Past the last hidden
  // layer that descriptor has size 0 and reads zeros.  At k = 64 the wider
  // output tiles leave no registers for fragments held across an activation
  // phase (it measured slower): there each layer fills its ring at its start.
  constexpr bool kCross = K <= 32;
  const R* __restrict__ layer = tab + 2 * kEncWidth;
  vh_t wb[kRing][NH];
  v4<R> acc[8], dacc[8];
  if constexpr (kCross) {
    const FragStream<vh_t> frag(layer, nh > 1 ? kLayerBytes : 0);
#pragma unroll
    for (int p = 0; p < kRing - 1; ++p)
#pragma unroll
      for (int u = 0; u < NH; ++u) wb[p][u] = frag[p * NH + u];
  }
#pragma unroll
  for (int T = 0; T < 8; ++T)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int in = 16 * T + drow<R>(i, g);
      const R w0 = S.u.p1.l0[sj][0][in], z = w0 * r + S.u.p1.l0[sj][1][in];
      const R s = sigmoid(z, kc);
      h[T][i] = z * s;
      if constexpr (kTan) dh[T][i] = silu_slope(z, s) * w0;
    }
  for (int t = 1; t < nh; ++t) {
    const FragStream<vh_t> frag(layer, kLayerBytes);
    const R* __restrict__ next = layer + kEncWidth * kEncWidth + kEncWidth;
    const bool more = t + 1 < nh;
    const FragStream<vh_t> nfrag(next, more ? kLayerBytes : 0);
    if constexpr (!kCross) {
#pragma unroll
      for (int p = 0; p < kRing - 1; ++p)
#pragma unroll
        for (int u = 0; u < NH; ++u) wb[p][u] = frag[p * NH + u];
    }
    // the tangent has no bias
    {
      const BiasStream<R> bias(layer + kEncWidth * kEncWidth, kBiasBytes, g);
#pragma unroll
      for (int To = 0; To < 8; ++To) acc[To] = v4<R>{bias(To, 0), bias(To, 1), bias(To, 2), bias(To, 3)};
    }
#pragma unroll
    for (int To = 0; To < 8; ++To) dacc[To] = v4<R>{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 32; ++ks) {
      const int kn = ks + kRing - 1;
      if (kCross || kn < 32) {
#pragma unroll
        for (int u = 0; u < NH; ++u) wb[kn % kRing][u] = kn < 32 ? frag[kn * NH + u] : nfrag[(kn - 32) * NH + u];
      }
      __builtin_amdgcn_sched_barrier(0);
      const int T = ks >> 2, i = ks & 3;
#pragma unroll
      for (int To = 0; To < 8; ++To) {
        const R wv = wb[ks % kRing][To / VW][To % VW];
        acc[To] = mfma(wv, h[T][i], acc[To]);
        if constexpr (kTan) dacc[To] = mfma(wv, dh[T][i], dacc[To]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // the next layer's k-step p sits in slot (32 + p) mod kRing; it starts
    // from slot p (a no-op when kRing divides 32)
    if constexpr (kCross && 32 % kRing != 0) {
      vh_t nx[kRing - 1][NH];
#pragma unroll
      for (int p = 0; p < kRing - 1; ++p)
#pragma unroll
        for (int u = 0; u < NH; ++u) nx[p][u] = wb[(32 + p) % kRing][u];
#pragma unroll
      for (int p = 0; p < kRing - 1; ++p)
#pragma unroll
        for (int u = 0; u < NH; ++u) wb[p][u] = nx[p][u];
    }
#pragma unroll
    for (int To = 0; To < 8; ++To) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const R z = acc[To][q];
        const R s = sigmoid(z, kc);
        h[To][q] += z * s;
        if constexpr (kTan) dh[To][q] = fma(silu_slope(z, s), dacc[To][q], dh[To][q]);
      }
    }
    layer = next;
  }
  return layer;
}

// Encoder output layer with pairs as rows: mo[Tc] register q holds
// m[pair drow(q, g)][16Tc + c] (dmo the same for the tangent).  Even and odd
// k-steps accumulate separately so 4 KT independent MFMA chains are in flight;
// the bias is added at the end so the first products do not wait for its load.
template <int K, typename R, bool kTan = true>
__device__ __forceinline__ void encoder_out_rows(const R* __restrict__ layer, const FloatHidden<R>& in,
                                                 v4<R> (&mo)[K / 16], v4<R> (&dmo)[K / 16]) {
  typedef Stream<K, R> St;
  typedef typename St::vo_t vo_t;
  constexpr int KT = St::KT, NO = St::NO, VO = St::VO, kRing = St::kRingO;
  const int lane = phase_tid() & 63, c = lane & 15;
  const R* __restrict__ bout = layer + K * kEncWidth;
  v4<R> mo2[2][KT], dmo2[2][KT];
  R b[KT];
#pragma unroll
  for (int Tc = 0; Tc < KT; ++Tc) {
    b[Tc] = bout[16 * Tc + c];
    mo2[0][Tc] = mo2[1][Tc] = dmo2[0][Tc] = dmo2[1][Tc] = v4<R>{0, 0, 0, 0};
  }
  const FragStream<vo_t> frag(layer, int(K * kEncWidth * sizeof(R)));
  vo_t wo[kRing][NO];
#pragma unroll
  for (int p = 0; p < kRing - 1; ++p)
#pragma unroll
    for (int u = 0; u < NO; ++u) wo[p][u] = frag[p * NO + u];
#pragma unroll
  for (int ks = 0; ks < 32; ++ks) {
    if (ks + kRing - 1 < 32) {
#pragma unroll
      for (int u = 0; u < NO; ++u) wo[(ks + kRing - 1) % kRing][u] = frag[(ks + kRing - 1) * NO + u];
    }
    __builtin_amdgcn_sched_barrier(0);
    const int T = ks >> 2, i = ks & 3;
#pragma unroll
    for (int Tc = 0; Tc < KT; ++Tc) {
      const R wv = wo[ks % kRing][Tc / VO][Tc % VO];
      mo2[ks & 1][Tc] = mfma(in.h[T][i], wv, mo2[ks & 1][Tc]);
      if constexpr (kTan) dmo2[ks & 1][Tc] = mfma(in.dh[T][i], wv, dmo2[ks & 1][Tc]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int Tc = 0; Tc < KT; ++Tc) {
    mo[Tc] = mo2[0][Tc] + mo2[1][Tc] + v4<R>{b[Tc], b[Tc], b[Tc], b[Tc]};
    if constexpr (kTan) dmo[Tc] = dmo2[0][Tc] + dmo2[1][Tc];
  }
}

// Encoder output layer with pairs as columns (the same fragments serve as the A
// operand): register q of lane (g, c) for output tile Tc holds
// m[pair c][16Tc + drow(q, g)].
template <int K, typename R>
__device__ __forceinline__ void encoder_out_cols(const R* __restrict__ layer, const FloatHidden<R>& in,
                                                 R (&mB)[K / 16][4], R (&dmB)[K / 16][4]) {
  typedef Stream<K, R> St;
  typedef typename St::vo_t vo_t;
  constexpr int KT = St::KT, NO = St::NO, VO = St::VO, kRing = St::kRingO;
  const int lane = phase_tid() & 63, g = lane >> 4;
  const R* __restrict__ bout = layer + K * kEncWidth;
  v4<R> acc[KT], dacc[KT];
#pragma unroll
  for (int Tc = 0; Tc < KT; ++Tc) {
    acc[Tc] = v4<R>{bout[16 * Tc + drow<R>(0, g)], bout[16 * Tc + drow<R>(1, g)], bout[16 * Tc + drow<R>(2, g)],
                    bout[16 * Tc + drow<R>(3, g)]};
    dacc[Tc] = v4<R>{0, 0, 0, 0};
  }
  const FragStream<vo_t> frag(layer, int(K * kEncWidth * sizeof(R)));
  vo_t wo[kRing][NO];
#pragma unroll
  for (int p = 0; p < kRing - 1; ++p)
#pragma unroll
    for (int u = 0; u < NO; ++u) wo[p][u] = frag[p * NO + u];
#pragma unroll
  for (int ks = 0; ks < 32; ++ks) {
    if (ks + kRing - 1 < 32) {
#pragma unroll
      for (int u = 0; u < NO; ++u) wo[(ks + kRing - 1) % kRing][u] = frag[(ks + kRing - 1) * NO + u];
    }
    __builtin_amdgcn_sched_barrier(0);
    const int T = ks >> 2, i = ks & 3;
#pragma unroll
    for (int Tc = 0; Tc < KT; ++Tc) {
      const R wv = wo[ks % kRing][Tc / VO][Tc % VO];
      acc[Tc] = mfma(wv, in.h[T][i], acc[Tc]);
      dacc[Tc] = mfma(wv, in.dh[T][i], dacc[Tc]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int Tc = 0; Tc < KT; ++Tc)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      mB[Tc][q] = acc[Tc][q];
      dmB[Tc][q] = dacc[Tc][q];
    }
}

template <typename R>
using HiddenOf = std::conditional_t<kDigits, Hidden<R>, FloatHidden<R>>;

// Pair that takes row c of the feature product, so that its result registers
// hold the pairs hrow(q, g) of the encoder's output.
template <typename R>
__device__ __forceinline__ int moment_pair(int c) {
  return kDigits && sizeof(R) == 8 ? 4 * (c & 3) + (c >> 2) : c;
}

// Pass 1 on one chunk: encoder forward, moment accumulation and, when kWs,
// the encoder tangent and the workspace write of (m, dm).  Nothing but the
// encoder's own state is held across its hidden layers: the pairs' unit
// vectors wait in LDS, and the next chunk is taken and its positions are
// requested (into pp) beside the output layer.
template <int K, int TM, typename R, int NW, int DR, int NM, bool kWs>
__device__ void pass1_chunk(const FusedArgs& A, Smem<K, TM, R, NW, DR, NM>& S, int ch, int nch, int* next_ch,
                            PairPos& pp, R* __restrict__ wsc) {
  constexpr int KT = K / 16;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  v4<R> mo[KT], dmo[KT];
  {
    const int lane = phase_tid() & 63, g = lane >> 4, c = lane & 15;
    double dxd, dyd, dzd;
    int atom;
    pair_delta(A, S, ch, pp, &dxd, &dyd, &dzd, &atom);
    const R dx = R(dxd), dy = R(dyd), dz = R(dzd);
    const R r = vsqrt(dx * dx + dy * dy + dz * dz);
    if (g == 0) {
      const R ir = vrcp(r);
      R fc, dfc_unused;
      cutoff(r, R(A.pi_rc), &fc, &dfc_unused);
      S.u.p1.geo[wave][c][0] = dx * ir;
      S.u.p1.geo[wave][c][1] = dy * ir;
      S.u.p1.geo[wave][c][2] = dz * ir;
      S.u.p1.geo[wave][c][3] = atom < 0 ? R(0) : fc;
    }
    HiddenOf<R> hid;
    const R* __restrict__ layer =
        encoder_hidden<K, TM, R, NW, DR, NM, kWs>(A, S, S.ch_s[ch], r, chunk_table(A, S, ch), hid);
    *next_ch = grab_chunk(&S.next_chunk[0]);
    if (*next_ch < nch) pp = load_pair_pos(A, S, *next_ch);
    encoder_out_rows<K, R, kWs>(layer, hid, mo, dmo);
  }
  const int lane = phase_tid() & 63, g = lane >> 4, c = lane & 15;
  // chunk-wide values, in scalar registers
  const int start = __builtin_amdgcn_readfirstlane(S.ch_start[ch]);
  const int count = __builtin_amdgcn_readfirstlane(S.ch_count[ch]);

  // moment: P[mm][col] += sum_pairs fc * a_mm(u) * m[pair][col], one MFMA
  // product per centre atom present in the chunk and 16-row tile of the
  // angular features (pairs of other atoms are masked to zero in the A
  // operand).  The features themselves are an MFMA product over the
  // monomials, F[pair][mm] = sum_m fc m_m(u_pair) Q[mm][m], whose result
  // registers (register q: pair drow(q, g), row c) are exactly the A operand
  // of the moment product; each lane forms only its own pair's monomials.
  constexpr int NA = DR / 16;
  static_assert(NM % 4 == 0, "monomial count must be a multiple of the MFMA k-step");
  v4<R> av[NA];
  int aa[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int p = hrow<R>(q, g);
    aa[q] = p < count ? S.pair_a[start + p] : -1;
  }
  {
    const R* geo = S.u.p1.geo[wave][moment_pair<R>(c)];
    const R ax = geo[0], ay = geo[1], az = geo[2], fa = geo[3];
    R mono[NM];
    monomials_n<NM, false>(ax, ay, az, mono, mono, mono, mono);
#pragma unroll
    for (int ta = 0; ta < NA; ++ta) av[ta] = v4<R>{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < NM / 4; ++i) {
      // A[pair c][m = 4i + g] = fc m_m(u_c); B[m = 4i + g][row c] = Q[row][m]
      const R x = fa * pick4(g, mono[4 * i], mono[4 * i + 1], mono[4 * i + 2], mono[4 * i + 3]);
#pragma unroll
      for (int ta = 0; ta < NA; ++ta) av[ta] = mfma(x, S.qc[16 * ta + c][4 * i + g], av[ta]);
    }
  }
  const int a_first = __builtin_amdgcn_readfirstlane(S.pair_a[start]);
  const int a_last = __builtin_amdgcn_readfirstlane(S.pair_a[start + count - 1]);
  for (int a = a_first; a <= a_last; ++a) {
#pragma unroll
    for (int ta = 0; ta < NA; ++ta) {
      v4<R> pacc[KT];
#pragma unroll
      for (int Tc = 0; Tc < KT; ++Tc) pacc[Tc] = v4<R>{0, 0, 0, 0};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const R av_a = aa[q] == a ? av[ta][q] : R(0);
#pragma unroll
        for (int Tc = 0; Tc < KT; ++Tc) pacc[Tc] = mfma(av_a, mo[Tc][q], pacc[Tc]);
      }
      constexpr int DRS = moment_rows(DR, NM);
#pragma unroll
      for (int Tc = 0; Tc < KT; ++Tc)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = 16 * ta + drow<R>(q, g);
          if (16 * ta + 16 <= DRS || row < DRS) atomicAdd(&S.P[a][row][16 * Tc + c], pacc[Tc][q]);
        }
    }
  }

  if (kWs) {
    // workspace in the B-operand order pass 2 loads, contiguous per lane:
    // lane 16 g' + c' holds m[pair c'][16Tc + hrow(i, g')] at 4 KT lane' +
    // 4 Tc + i (then the same for dm)
#pragma unroll
    for (int Tc = 0; Tc < KT; ++Tc)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int off = (16 * hgroup<R>(c) + hrow<R>(q, g)) * (4 * KT) + Tc * 4 + hreg<R>(c);
        wsc[off] = mo[Tc][q];
        wsc[K * 16 + off] = dmo[Tc][q];
      }
  }
}

// Inputs of pass 2 for one chunk: the workspace tiles (m, dm) in B-operand
// order and the neighbour position; loaded one chunk ahead.
template <int K, typename R>
struct Pass2In {
  R mB[K / 16][4], dmB[K / 16][4];
  PairPos pp;
};

template <int K, int TM, typename R, int NW, int DR, int NM>
__device__ __forceinline__ void pass2_load(const FusedArgs& A, const Smem<K, TM, R, NW, DR, NM>& S, int ch,
                                           const R* __restrict__ wsc, Pass2In<K, R>& in) {
  constexpr int VW = 16 / int(sizeof(R));
  constexpr int NV = K / 4 / VW;  // 16-byte loads per lane for m (and for dm)
  typedef R vw_t __attribute__((ext_vector_type(VW)));
  const int lane = phase_tid() & 63;
  const vw_t* __restrict__ pm = reinterpret_cast<const vw_t*>(wsc + lane * (K / 4));
  const vw_t* __restrict__ pd = reinterpret_cast<const vw_t*>(wsc + K * 16 + lane * (K / 4));
  vw_t vm[NV], vd[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    vm[v] = pm[v];
    vd[v] = pd[v];
  }
#pragma unroll
  for (int Tc = 0; Tc < K / 16; ++Tc)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      in.mB[Tc][i] = vm[(Tc * 4 + i) / VW][(Tc * 4 + i) % VW];
      in.dmB[Tc][i] = vd[(Tc * 4 + i) / VW][(Tc * 4 + i) % VW];
    }
  in.pp = load_pair_pos(A, S, ch);
}

// Inputs of pass 2 for one chunk by recomputing the encoder instead of
// reading the workspace (the paper's mega-fusion, Section 3.4).
template <int K, int TM, typename R, int NW, int DR, int NM>
__device__ __forceinline__ void pass2_recompute(const FusedArgs& A, const Smem<K, TM, R, NW, DR, NM>& S, int ch,
                                                const PairPos& pp, Pass2In<K, R>& in) {
  double dxd, dyd, dzd;
  int atom;
  pair_delta(A, S, ch, pp, &dxd, &dyd, &dzd, &atom);
  const R dx = R(dxd), dy = R(dyd), dz = R(dzd);
  const R r = vsqrt(dx * dx + dy * dy + dz * dz);
  HiddenOf<R> hid;
  const R* __restrict__ layer = encoder_hidden<K, TM, R, NW, DR, NM>(A, S, S.ch_s[ch], r, chunk_table(A, S, ch), hid);
  encoder_out_cols<K, R>(layer, hid, in.mB, in.dmB);
  in.pp = pp;
}

// F_j -= f_ij through the tile's table in LDS (open addressing by a
// multiplicative hash of j, linear probing); when every probe position of j
// is taken by other neighbours the contribution goes straight to HBM.
template <int K, int TM, typename R, int NW, int DR, int NM>
__device__ __forceinline__ void scatter_fj_tile(const FusedArgs& A, Smem<K, TM, R, NW, DR, NM>& S, int j, double fx,
                                                double fy, double fz) {
  constexpr int kProbes = 32;
  int slot = int((unsigned(j) * 0x9E3779B1u) >> 22);  // 10 bits: kFjSlots = 1024
  for (int p = 0; p < kProbes; ++p) {
    const int prev = atomicCAS(&S.u.fj.key[slot], -1, j);
    if (prev == -1 || prev == j) {
      atomicAdd(&S.u.fj.val[slot][0], -fx);
      atomicAdd(&S.u.fj.val[slot][1], -fy);
      atomicAdd(&S.u.fj.val[slot][2], -fz);
      return;
    }
    slot = (slot + 1) & (kFjSlots - 1);
  }
  atomicAdd(&A.forces[3 * (long long)j], -fx);
  atomicAdd(&A.forces[3 * (long long)j + 1], -fy);
  atomicAdd(&A.forces[3 * (long long)j + 2], -fz);
}

// Pass 2 on one chunk: W contractions, partial forces and scatter (F_j by
// global atomics, or with kTileFj through the tile's table).
template <int K, int TM, typename R, int NW, int DR, int NM, bool kTileFj = false>
__device__ void pass2_chunk(const FusedArgs& A, Smem<K, TM, R, NW, DR, NM>& S, int ch, const Pass2In<K, R>& in) {
  constexpr int KT = K / 16;
  const int lane = phase_tid() & 63, g = lane >> 4, c = lane & 15;
  // chunk-wide values, in scalar registers
  const int start = __builtin_amdgcn_readfirstlane(S.ch_start[ch]);
  const int count = __builtin_amdgcn_readfirstlane(S.ch_count[ch]);

  const bool valid = c < count;
  int atom = -1, j = 0;
  double dx = 1.0, dy = 0.0, dz = 0.0;  // minimum image in float64, kept for the virial
  if (valid) {
    const int e = start + c;
    j = S.pair_j[e];
    atom = S.pair_a[e];
    dx = fold(in.pp.x - S.tpos[atom][0], A.box[0], A.inv_box[0]);
    dy = fold(in.pp.y - S.tpos[atom][1], A.box[1], A.inv_box[1]);
    dz = fold(in.pp.z - S.tpos[atom][2], A.box[2], A.inv_box[2]);
  }
  const R rx = R(dx), ry = R(dy), rz = R(dz);
  const R r = vsqrt(rx * rx + ry * ry + rz * rz);
  const R ir = vrcp(r);
  const R ux = rx * ir, uy = ry * ir, uz = rz * ir;
  R fc, dfc;
  cutoff(r, R(A.pi_rc), &fc, &dfc);
  if (!valid) fc = dfc = R(0);

  // (W m) and (W dm) for this column's own centre atom, one 16-row tile of
  // the angular features at a time
  constexpr int NA = DR / 16;
  v4<R> wm[NA], wdm[NA];
#pragma unroll
  for (int ta = 0; ta < NA; ++ta) wm[ta] = wdm[ta] = v4<R>{0, 0, 0, 0};
  const int a_first = __builtin_amdgcn_readfirstlane(S.pair_a[start]);
  const int a_last = __builtin_amdgcn_readfirstlane(S.pair_a[start + count - 1]);
  for (int a = a_first; a <= a_last; ++a) {
#pragma unroll
    for (int ta = 0; ta < NA; ++ta) {
      v4<R> t1 = v4<R>{0, 0, 0, 0}, t2 = v4<R>{0, 0, 0, 0};
#pragma unroll
      for (int Tc = 0; Tc < KT; ++Tc)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          constexpr int DRS = moment_rows(DR, NM);
          const R w = 16 * ta + 16 <= DRS || 16 * ta + c < DRS ? S.P[a][16 * ta + c][16 * Tc + hrow<R>(i, g)] : R(0);
          t1 = mfma(w, in.mB[Tc][i], t1);
          t2 = mfma(w, in.dmB[Tc][i], t2);
        }
      if (atom == a) {
        wm[ta] = t1;
        wdm[ta] = t2;
      }
    }
  }

  // angular features a_mm and gradients for rows mm = 16 ta + drow(q, g) of
  // this pair, accumulated monomial by monomial so that each monomial and
  // its gradient are live only for their own step
  R mono[NM], gx[NM], gy[NM], gz[NM];
  monomials_n<NM, true>(ux, uy, uz, mono, gx, gy, gz);
  R fv[NA][4], fgx[NA][4], fgy[NA][4], fgz[NA][4];
#pragma unroll
  for (int ta = 0; ta < NA; ++ta)
#pragma unroll
    for (int q = 0; q < 4; ++q) fv[ta][q] = fgx[ta][q] = fgy[ta][q] = fgz[ta][q] = R(0);
#pragma unroll
  for (int m = 0; m < NM; ++m)
#pragma unroll
    for (int ta = 0; ta < NA; ++ta)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const R co = S.qc[16 * ta + drow<R>(q, g)][m];
        fv[ta][q] += co * mono[m];
        fgx[ta][q] += co * gx[m];
        fgy[ta][q] += co * gy[m];
        fgz[ta][q] += co * gz[m];
      }
  R s = 0, tx = 0, ty = 0, tz = 0;
#pragma unroll
  for (int ta = 0; ta < NA; ++ta)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const R v = fc * wm[ta][q];                       // v = W g
      const R wg = dfc * wm[ta][q] + fc * wdm[ta][q];   // W g'
      s += fv[ta][q] * wg;
      tx += fgx[ta][q] * v;
      ty += fgy[ta][q] * v;
      tz += fgz[ta][q] * v;
    }
#pragma unroll
  for (int o = 16; o <= 32; o <<= 1) {
    s += __shfl_xor(s, o, 64);
    tx += __shfl_xor(tx, o, 64);
    ty += __shfl_xor(ty, o, 64);
    tz += __shfl_xor(tz, o, 64);
  }
  // f = s u + (I - u u^T) t / r  (Eq. 10, reassociated), accumulated in float64
  const R ut = ux * tx + uy * ty + uz * tz;
  const double fx = double(s * ux + (tx - ut * ux) * ir);
  const double fy = double(s * uy + (ty - ut * uy) * ir);
  const double fz = double(s * uz + (tz - ut * uz) * ir);
  if (valid) {
    if (g == 0) {
      if constexpr (kTileFj) {
        scatter_fj_tile(A, S, j, fx, fy, fz);
      } else {
        atomicAdd(&A.forces[3 * (long long)j], -fx);
        atomicAdd(&A.forces[3 * (long long)j + 1], -fy);
        atomicAdd(&A.forces[3 * (long long)j + 2], -fz);
      }
    } else if (g == 1) {
      atomicAdd(&S.Fi[atom][0], fx);
      atomicAdd(&S.Fi[atom][1], fy);
      atomicAdd(&S.Fi[atom][2], fz);
    } else if (g == 2) {
      atomicAdd(&S.Wi[atom][0], -dx * fx);
      atomicAdd(&S.Wi[atom][1], -dx * fy);
      atomicAdd(&S.Wi[atom][2], -dx * fz);
      atomicAdd(&S.Wi[atom][3], -dy * fx);
      atomicAdd(&S.Wi[atom][4], -dy * fy);
    } else {
      atomicAdd(&S.Wi[atom][5], -dy * fz);
      atomicAdd(&S.Wi[atom][6], -dz * fx);
      atomicAdd(&S.Wi[atom][7], -dz * fy);
      atomicAdd(&S.Wi[atom][8], -dz * fz);
    }
  }
}

// Radial kernel of the unfused configuration (Eq. 2 as a kernel of its own)
// on one chunk: g = fc(r) MLP(r) and dg/dr of each pair from the distance
// the setup kernel stored for its neighbour-list entry, written back by
// entry.  The chunk's pair slots hold entry indices relative to the tile's
// first entry.
template <int K, int TM, typename R, int NW, int DR, int NM>
__device__ void radial_chunk(const FusedArgs& A, const Smem<K, TM, R, NW, DR, NM>& S, int ch) {
  constexpr int KT = K / 16;
  const int lane = phase_tid() & 63, g = lane >> 4, c = lane & 15;
  const bool valid = c < S.ch_count[ch];
  const long long e = S.row_beg[0] + (valid ? S.pair_j[S.ch_start[ch] + c] : 0);
  const R r = valid ? R(A.geo[4 * e + 3]) : R(1);
  R fc, dfc;
  cutoff(r, R(A.pi_rc), &fc, &dfc);
  if (!valid) fc = dfc = R(0);
  HiddenOf<R> hid;
  const R* __restrict__ layer = encoder_hidden<K, TM, R, NW, DR, NM>(A, S, S.ch_s[ch], r, chunk_table(A, S, ch), hid);
  R mB[KT][4], dmB[KT][4];
  encoder_out_cols<K, R>(layer, hid, mB, dmB);
  if (valid) {
    R* __restrict__ gr = static_cast<R*>(A.grad) + e * K;
    R* __restrict__ gp = static_cast<R*>(A.gprime) + e * K;
#pragma unroll
    for (int Tc = 0; Tc < KT; ++Tc)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int col = 16 * Tc + hrow<R>(q, g);
        gr[col] = fc * mB[Tc][q];
        gp[col] = dfc * mB[Tc][q] + fc * dmB[Tc][q];
      }
  }
}

// Descriptor value x[in] = vec(G)[in] of tile atom a (Eq. 5): the l = 0
// block is linear, a block l >= 1 (angular rows lrow[l] .. lrow[l+1]-1) is
// the quadratic form sum_m rw[m] P[m][col]^2 with the block's diagonal
// metric (1 for the irreducible basis, the multinomial coefficients for the
// Cartesian one).
template <int K, int TM, typename R, int NW, int DR, int NM>
__device__ __forceinline__ R descriptor_value(const FusedArgs& A, const Smem<K, TM, R, NW, DR, NM>& S, int a, int in) {
  const int l = in / K, col = in % K;
  if (l == 0) return S.P[a][0][col];
  R v = 0;
  for (int mm = A.lrow[l]; mm < A.lrow[l + 1]; ++mm) v += S.rw[mm] * S.P[a][mm][col] * S.P[a][mm][col];
  return v;
}

// W = dE/dP (Eq. 7) for tile atom a from dE/dx[in]: W[0][col] = dE/dG[0][col],
// W[m][col] = 2 dE/dG[l][col] rw[m] P[m][col]; overwrites P.
template <int K, int TM, typename R, int NW, int DR, int NM>
__device__ __forceinline__ void adjoint_from_grad(const FusedArgs& A, Smem<K, TM, R, NW, DR, NM>& S, int a, int in,
                                                  R d) {
  const int l = in / K, col = in % K;
  if (l == 0) {
    S.P[a][0][col] = d;
  } else {
    for (int mm = A.lrow[l]; mm < A.lrow[l + 1]; ++mm) S.P[a][mm][col] *= R(2) * S.rw[mm] * d;
  }
}

// Weight fragments of the head products, consumed in groups of 16 k-steps.
// Group G of a wavefront that owns output rows (w < 4): the first layer's
// k-steps 16G .. 16G+15, then the hidden layers forward, the hidden layers
// backward (A_t^T), then the A0^T output tiles tt = w, w + NW, ...; the
// other wavefronts only take A0^T tiles.  Element ks of a group is at
// p[ks * stride * 64]; n is the group's k-step count (0 past the end).
template <typename R>
struct HeadGroup {
  const R* p;
  int stride, n;
};

template <typename R>
__device__ __forceinline__ HeadGroup<R> head_group(int G, bool rw, int w, int nw, int nin, int nhid,
                                                   const R* __restrict__ A0f, const R* __restrict__ A0Tf,
                                                   const R* __restrict__ hid) {
  constexpr int RW = kHeadWidth;
  constexpr int HS = 2 * RW * RW + RW;
  const int lane = phase_tid() & 63;
  const int tin = nin / 16, k0 = nin / 4, nl0 = (k0 + 15) / 16;
  if (rw) {
    if (G < nl0) return {A0f + (64 * G + w) * 64 + lane, 4, k0 - 16 * G < 16 ? k0 - 16 * G : 16};
    G -= nl0;
    if (G < nhid) return {hid + G * HS + w * 64 + lane, 4, 16};
    G -= nhid;
    if (G < nhid) return {hid + (nhid - 1 - G) * HS + RW * RW + w * 64 + lane, 4, 16};
    G -= nhid;
  }
  const int tt = w + nw * G;
  if (tt < tin) return {A0Tf + tt * 64 + lane, tin, 16};
  return {A0Tf, 0, 0};
}

template <typename R>
__device__ __forceinline__ void head_load(const HeadGroup<R>& d, R (&f)[16]) {
#pragma unroll
  for (int ks = 0; ks < 16; ++ks) f[ks] = ks < d.n ? d.p[ks * d.stride * 64] : R(0);
}

// Descriptor (Eq. 5), head forward and backward (Eq. 6) and W = dE/dP
// (Eq. 7) for the tile on MFMA: the tile's atoms are the 16 columns of every
// product and wavefront w < 4 owns rows 16w..16w+15 of each 64-wide layer.
// Activations live in LDS feature-major ([feature][atom]) so that B-operand
// reads are contiguous; pre-activations stay in registers for the backward
// pass.  Each wavefront streams its weight fragments one 16-k-step group
// ahead of the products (the first group before the descriptor is formed),
// so a layer's fragments arrive while the previous layer and its barriers
// run.  With kRegress (the regression kernel of the three-kernel and unfused
// configurations) the descriptor comes from HBM and dE/dx goes back to HBM
// in its place instead of forming W.
template <int K, int TM, typename R, int NW, int DR, int NM, bool kRegress>
__device__ void head_stage(const FusedArgs& A, Smem<K, TM, R, NW, DR, NM>& S) {
  constexpr int RW = kHeadWidth;
  constexpr int HS = 2 * RW * RW + RW;  // one hidden layer: A_t and A_t^T fragments, c_t
  constexpr int NC = TM > 16 ? 32 : 16;  // atom columns: one or two groups of 16
  constexpr int CG = NC / 16;
  const int tid = phase_tid(), lane = tid & 63, g = lane >> 4, c = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int na = S.na;
  const int nin = (A.lmax + 1) * K;
  const int tin = nin / 16;
  const int nhid = A.reg_hidden - 1;
  const int rho = A.reg_cond ? S.tile_species : 0;
  const R* __restrict__ A0f = static_cast<const R*>(A.head) + (long long)rho * A.head_stride;  // A0 fragments
  const R* __restrict__ A0Tf = A0f + RW * nin;                                               // A0^T fragments
  const R* __restrict__ c0 = A0Tf + RW * nin;
  const R* __restrict__ hid = c0 + RW;
  const R* __restrict__ aout = hid + nhid * HS;
  // this lane's result rows are 16 w + drow(q, g); with more than 4
  // wavefronts the others only join the barriers of the row-parallel steps
  // and take A0^T tiles.  Each weight fragment multiplies the CG column
  // groups of atoms.
  const bool rw = w < RW / 16;
  int G = 0;
  R fcur[16], fnext[16];
  head_load(head_group(G, rw, w, NW, nin, nhid, A0f, A0Tf, hid), fnext);
  // next group: the fetched one becomes current and the one after it is fetched
#define ADVANCE()                                                          \
  do {                                                                     \
    _Pragma("unroll") for (int ks_ = 0; ks_ < 16; ++ks_) fcur[ks_] = fnext[ks_]; \
    ++G;                                                                   \
    head_load(head_group(G, rw, w, NW, nin, nhid, A0f, A0Tf, hid), fnext); \
  } while (0)

  // B-operand reads from the feature-major activations: element
  // [16 (k >> 2) + drow(k & 3, g)][16 cg + c] sits at a per-lane base plus an
  // offset that depends on k and cg only, so every read is that base with an
  // immediate offset instead of an address register of its own (no
  // __restrict__: yT and gT are also written through S between the barriers)
  const R* xl = &S.u.hd.xT[0][0] + drow<R>(0, g) * NC + c;
  const R* yl = &S.u.hd.yT[0][0] + drow<R>(0, g) * NC + c;
  const R* gl = &S.u.hd.gT[0][0] + drow<R>(0, g) * NC + c;
#define BOFF(k) ((16 * ((k) >> 2) + drow<R>((k) & 3, 0)) * NC)

  R* __restrict__ gbuf = kRegress ? static_cast<R*>(A.gbuf) + (long long)S.a0 * nin : nullptr;
  for (int u = tid; u < NC * nin; u += (64 * NW)) {
    const int a = u % NC, in = u / NC;
    R v = 0;
    if (a < na) v = kRegress ? gbuf[(long long)a * nin + in] : descriptor_value(A, S, a, in);
    S.u.hd.xT[in][a] = v;
  }
  __syncthreads();

#define ROW(q) (16 * w + drow<R>(q, g))

  // layer 0: z0 = A0 x + c0, over nin / 4 k-steps in groups of 16 with two
  // accumulators alternating
  v4<R> z0[CG];
#pragma unroll
  for (int cg = 0; cg < CG; ++cg) z0[cg] = v4<R>{0, 0, 0, 0};
  if (rw) {
    v4<R> z0b[CG];
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) {
      z0[cg] = v4<R>{c0[ROW(0)], c0[ROW(1)], c0[ROW(2)], c0[ROW(3)]};
      z0b[cg] = v4<R>{0, 0, 0, 0};
    }
    const int k0 = nin / 4;
    for (int kb = 0; kb < k0; kb += 16) {
      ADVANCE();
      const R* xk = xl + 4 * kb * NC;  // kb is a multiple of 16
#pragma unroll
      for (int ks = 0; ks < 16; ks += 2) {
        if (kb + ks < k0) {
#pragma unroll
          for (int cg = 0; cg < CG; ++cg) {
            z0[cg] = mfma(fcur[ks], xk[BOFF(ks) + 16 * cg], z0[cg]);
            z0b[cg] = mfma(fcur[ks + 1], xk[BOFF(ks + 1) + 16 * cg], z0b[cg]);
          }
        }
      }
    }
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) {
      z0[cg] += z0b[cg];
#pragma unroll
      for (int q = 0; q < 4; ++q) S.u.hd.yT[ROW(q)][16 * cg + c] = z0[cg][q] * sigmoid(z0[cg][q]);
    }
  }
  __syncthreads();

  // residual layers: y <- y + silu(A_t y + c_t)
  v4<R> zeta[kMaxHidden][CG];
#pragma unroll
  for (int t = 1; t < kMaxHidden; ++t) {
    if (t >= A.reg_hidden) break;
    const R* __restrict__ ct = hid + (t - 1) * HS + 2 * RW * RW;
    v4<R> z[CG];
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) z[cg] = v4<R>{0, 0, 0, 0};
    if (rw) {
      ADVANCE();
#pragma unroll
      for (int cg = 0; cg < CG; ++cg) z[cg] = v4<R>{ct[ROW(0)], ct[ROW(1)], ct[ROW(2)], ct[ROW(3)]};
#pragma unroll
      for (int ks = 0; ks < 16; ++ks)
#pragma unroll
        for (int cg = 0; cg < CG; ++cg)
          z[cg] = mfma(fcur[ks], yl[BOFF(ks) + 16 * cg], z[cg]);
    }
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) zeta[t][cg] = z[cg];
    __syncthreads();
    if (rw) {
#pragma unroll
      for (int cg = 0; cg < CG; ++cg)
#pragma unroll
        for (int q = 0; q < 4; ++q) S.u.hd.yT[ROW(q)][16 * cg + c] += z[cg][q] * sigmoid(z[cg][q]);
    }
    __syncthreads();
  }
  if (tid < na) {
    R e = aout[RW];
    for (int o = 0; o < RW; ++o) e += aout[o] * S.u.hd.yT[o][tid];
    S.Ei[tid] = double(e);
  }

  // backward: d <- d + A_t^T (silu'(zeta_t) d), starting from d = a_out
  v4<R> d[CG];
#pragma unroll
  for (int cg = 0; cg < CG; ++cg)
    d[cg] = rw ? v4<R>{aout[ROW(0)], aout[ROW(1)], aout[ROW(2)], aout[ROW(3)]} : v4<R>{0, 0, 0, 0};
#pragma unroll
  for (int t = kMaxHidden - 1; t >= 1; --t) {
    if (t >= A.reg_hidden) continue;
    if (rw) {
#pragma unroll
      for (int cg = 0; cg < CG; ++cg)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const R z = zeta[t][cg][q], sg = sigmoid(z);
          S.u.hd.gT[ROW(q)][16 * cg + c] = silu_slope(z, sg) * d[cg][q];
        }
    }
    __syncthreads();
    if (rw) {
      ADVANCE();
      v4<R> acc[CG];
#pragma unroll
      for (int cg = 0; cg < CG; ++cg) acc[cg] = v4<R>{0, 0, 0, 0};
#pragma unroll
      for (int ks = 0; ks < 16; ++ks)
#pragma unroll
        for (int cg = 0; cg < CG; ++cg)
          acc[cg] = mfma(fcur[ks], gl[BOFF(ks) + 16 * cg], acc[cg]);
#pragma unroll
      for (int cg = 0; cg < CG; ++cg) d[cg] += acc[cg];
    }
    __syncthreads();
  }
  if (rw) {
#pragma unroll
    for (int cg = 0; cg < CG; ++cg)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const R z = z0[cg][q], sg = sigmoid(z);
        S.u.hd.gT[ROW(q)][16 * cg + c] = silu_slope(z, sg) * d[cg][q];
      }
  }
  __syncthreads();
  // dE/dx = A0^T g0, then W[0][col] = dE/dG[0][col], W[m][col] = 2 dE/dG[l][col] P[m][col]
  for (int tt = w; tt < tin; tt += NW) {
    ADVANCE();
    v4<R> acc[CG];
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) acc[cg] = v4<R>{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
#pragma unroll
      for (int cg = 0; cg < CG; ++cg)
        acc[cg] = mfma(fcur[ks], gl[BOFF(ks) + 16 * cg], acc[cg]);
    }
#pragma unroll
    for (int cg = 0; cg < CG; ++cg) {
      const int a = 16 * cg + c;
      if (a < na) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int in = 16 * tt + drow<R>(q, g);
          if (kRegress)
            gbuf[(long long)a * nin + in] = acc[cg][q];
          else
            adjoint_from_grad(A, S, a, in, acc[cg][q]);
        }
      }
    }
  }
  __syncthreads();
#undef BOFF
#undef ROW
#undef ADVANCE
}

// First-layer weights (w0, b0) of the tile's encoder tables, one per
// neighbour species, into LDS.
template <int K, int TM, typename R, int NW, int DR, int NM>
__device__ __forceinline__ void stage_first_layer(const FusedArgs& A, Smem<K, TM, R, NW, DR, NM>& S,
                                                  const R* __restrict__ enc) {
  for (int u = threadIdx.x; u < A.C * 2 * kEncWidth; u += 64 * NW) {
    const int sj = u / (2 * kEncWidth), rem = u % (2 * kEncWidth);
    const int si = S.tile_species;
    const int tau = A.enc_cond == 2 ? si * A.C + sj : (A.enc_cond == 1 ? sj : 0);
    S.u.p1.l0[sj][rem / kEncWidth][rem % kEncWidth] = enc[(long long)tau * A.enc_stride + rem];
  }
}

// What one launch does (Section 3.4 fusion configurations): the single
// kernel that caches (m, dm) between its two passes or recomputes them in
// pass 2; one of the three kernels of the partial configuration: encoding
// (Eqs. 1-5, G to HBM), regression (Eq. 6, E and dE/dG to HBM) and
// derivation (Eqs. 7-10, recomputing P); or the radial kernel of the unfused
// configuration (Eq. 2 alone, which uses the regression kernel as well).
enum Mode { kCached = 0, kRecompute = 1, kEncode = 2, kRegress = 3, kDerive = 4, kRadial = 5, kCachedTileFj = 6 };
static_assert(kCachedTileFj == kModeCachedTileFj, "mode number of the tile-reduced scatter");
static_assert(kRegress == kModeRegress && kRadial == kModeRadial, "mode numbers of the unfused configuration");

template <int K, int TM, typename R, int NW, int DR, int NM, int MODE, bool kDig>
__global__ __launch_bounds__(64 * NW, 1) void k_fused(FusedArgs A) {
  static_assert(TM <= 64, "the bucket table gives one lane to each atom of a tile");
  extern __shared__ __align__(16) unsigned char smem_raw[];
  Smem<K, TM, R, NW, DR, NM>& S = *reinterpret_cast<Smem<K, TM, R, NW, DR, NM>*>(smem_raw);
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const long long chunk_elems = 2LL * K * 16;
  R* __restrict__ ws_slot = static_cast<R*>(A.ws) + (long long)blockIdx.x * A.ws_slot;
  const R* __restrict__ enc = static_cast<const R*>(A.enc);
  const R* __restrict__ qc = static_cast<const R*>(A.qc);

  for (int u = threadIdx.x; u < DR * NM; u += (64 * NW)) S.qc[u / NM][u % NM] = qc[u];
  for (int u = threadIdx.x; u < DR; u += 64 * NW) S.rw[u] = qc[DR * NM + u];

  // XCD-aware assignment: blocks are dispatched round-robin over the 8 XCDs,
  // so block b works on the b%8-th contiguous eighth of the tile list and
  // spatially adjacent tiles share an L2.
  const int G = gridDim.x;
  const int nx = (G % 8 == 0) ? 8 : 1;
  const int xcd = blockIdx.x % nx, slot = blockIdx.x / nx, per = G / nx;
  const int lo = int((long long)A.n_tiles * xcd / nx), hi = int((long long)A.n_tiles * (xcd + 1) / nx);

  for (int tile = lo + slot; tile < hi; tile += per) {
    // ---- A: stage atoms and rows -----------------------------------------
    // The rows of consecutive sorted atoms are one contiguous run of the
    // neighbour list, and each row is grouped by neighbour species, so the
    // bucket position of an entry follows from a block-wide prefix count of
    // active entries; every thread handles 8 consecutive entries.
    const int tid = phase_tid();
    if (tid == 0) {
      int s = 0;
      while (s + 1 < A.C && tile >= A.tile_start[s + 1]) ++s;
      const int first = A.species_start[s] + (tile - A.tile_start[s]) * A.tile_atoms;
      const int rem = A.species_start[s + 1] - first;
      S.tile_species = s;
      S.na = rem < A.tile_atoms ? rem : A.tile_atoms;
      S.a0 = first;
    }
    __syncthreads();
    const int na = S.na;
    const int a0 = S.a0;
    if (tid < TM) {
      if (tid < na) {
        const int o = A.perm[a0 + tid];
        S.orig[tid] = o;
        if (A.list.idx16) centre_cells(A.list, A.list.key[o], S.cand[tid]);
        S.tpos[tid][0] = A.pos[3 * (long long)o];
        S.tpos[tid][1] = A.pos[3 * (long long)o + 1];
        S.tpos[tid][2] = A.pos[3 * (long long)o + 2];
      }
#pragma unroll
      for (int k = 0; k < 3; ++k) S.Fi[tid][k] = 0.0;
#pragma unroll
      for (int k = 0; k < 9; ++k) S.Wi[tid][k] = 0.0;
      S.Ei[tid] = 0.0;
    }
    int nch = 0;
    if constexpr (MODE != kRegress) {
    stage_first_layer(A, S, enc);
    if (tid <= TM) {
      const int k = tid < na ? tid : na;
      S.ent_base[tid] = int(A.offsets[a0 + k] - A.offsets[a0]);
      if (tid == 0) S.row_beg[0] = A.offsets[a0];
    }
    for (int u = tid; u < kMaxSpecies * TM; u += (64 * NW)) S.cnt[u / TM][u % TM] = 0;
    if constexpr (MODE != kRadial)
      for (int u = tid; u < TM * moment_rows(DR, NM) * (K + 1); u += (64 * NW)) (&S.P[0][0][0])[u] = R(0);
    __syncthreads();
    const int nent = S.ent_base[na];
    const long long ebase = S.row_beg[0];
    constexpr int kPer = tile_entry_cap(TM) / (64 * NW);
    static_assert(kPer * 64 * NW == tile_entry_cap(TM), "every listed entry of a tile needs a thread");
    int ej[kPer], ea[kPer], es[kPer];
    int my_active = 0;
    {
      const int e0 = tid * kPer;
      int a = 0;
      while (a + 1 < na && e0 >= S.ent_base[a + 1]) ++a;
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        while (a + 1 < na && e0 + k >= S.ent_base[a + 1]) ++a;
        ea[k] = a;
      }
      if (A.list.idx32) {
#pragma unroll
        for (int k = 0; k < kPer; ++k) ej[k] = e0 + k < nent ? A.list.idx32[ebase + e0 + k] : -1;
      } else {
        // coded entries: bucket start through the centre's candidate cells,
        // then the permutation (each level's loads issued together)
        unsigned code[kPer];
        int slot[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) code[k] = e0 + k < nent ? A.list.idx16[ebase + e0 + k] : 0u;
#pragma unroll
        for (int k = 0; k < kPer; ++k) slot[k] = e0 + k < nent ? code_slot(A.list, S.cand[ea[k]], code[k]) : -1;
#pragma unroll
        for (int k = 0; k < kPer; ++k) ej[k] = slot[k] >= 0 ? A.list.perm[slot[k]] : -1;
      }
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        const int e = e0 + k;
        a = ea[k];
        es[k] = -1;
        const int j = ej[k];
        if (j >= 0) {
          bool active;
          if constexpr (MODE == kRadial) {
            // the setup kernel marked entries beyond the cutoff
            active = A.geo[4 * (ebase + e) + 3] >= 0.0;
          } else {
            const double dx = fold(A.pos[3 * (long long)j] - S.tpos[a][0], A.box[0], A.inv_box[0]);
            const double dy = fold(A.pos[3 * (long long)j + 1] - S.tpos[a][1], A.box[1], A.inv_box[1]);
            const double dz = fold(A.pos[3 * (long long)j + 2] - S.tpos[a][2], A.box[2], A.inv_box[2]);
            active = dx * dx + dy * dy + dz * dz < A.rc2;
          }
          if (active) {
            es[k] = A.types[j];
            atomicAdd(&S.cnt[es[k]][a], 1);
            ++my_active;
          }
        }
      }
    }
    // exclusive prefix of active entries over the block (entry order)
    int prefix;
    {
      int inc = my_active;
      const int ln = tid & 63;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o, 64);
        if (ln >= o) inc += t;
      }
      if (ln == 63) S.wsum[wave] = inc;
      __syncthreads();
      prefix = inc - my_active;
      for (int w = 0; w < wave; ++w) prefix += S.wsum[w];
    }
    if (wave == 0) {
      // Bucket layout (species-major, atoms in order), chunk table, and the
      // offset turning an entry's block-wide active prefix (atom-major) into
      // its bucket slot: base[s][a] = (active entries of buckets before
      // (s, a) in species-major order) - (active entries before (a, s) in
      // atom-major order).  Lane a holds atom a; one lane scan per species.
      const int ln = tid;
      int run = 0, nchunk = 0, cum = 0;  // cum: this atom's entries of the species so far
      for (int s = 0; s < A.C; ++s) {
        const int x = ln < na ? S.cnt[s][ln] : 0;
        int inc = x;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int t = __shfl_up(inc, o, 64);
          if (ln >= o) inc += t;
        }
        const int tot = __shfl(inc, 63, 64);
        if (ln < na) S.base[s][ln] = run + inc - x - cum;
        cum += x;
        const int nb = (tot + 15) >> 4;
        for (int k = ln; k < nb; k += 64) {
          S.ch_start[nchunk + k] = run + 16 * k;
          S.ch_count[nchunk + k] = (unsigned char)(tot - 16 * k < 16 ? tot - 16 * k : 16);
          S.ch_s[nchunk + k] = (unsigned char)s;
        }
        nchunk += nb;
        run += tot;
      }
      // cum is now this atom's row total; subtract the atom-major row start
      int inc = cum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o, 64);
        if (ln >= o) inc += t;
      }
      const int row_start = inc - cum;
      if (ln < na)
        for (int s = 0; s < A.C; ++s) S.base[s][ln] -= row_start;
      if (ln == 0) {
        S.n_chunks = nchunk;
        S.next_chunk[0] = NW;  // chunk w < NW starts on wavefront w
        S.next_chunk[1] = NW;
        S.n_active = run;
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if (es[k] >= 0) {
        const int s = es[k], a = ea[k];
        const int p = S.base[s][a] + prefix;
        // the list builder groups every row by species, so p always lies in
        // the (species, atom) run; the bound only keeps LDS accesses in range
        if (p >= 0 && p < S.n_active) {
          S.pair_j[p] = MODE == kRadial ? tid * kPer + k : ej[k];
          S.pair_a[p] = (unsigned char)a;
        }
        ++prefix;
      }
    }
    __syncthreads();

    // ---- B: pass 1 ---------------------------------------------------------
    nch = S.n_chunks;
    if constexpr (MODE == kRadial) {
      int ch = wave;
      while (ch < nch) {
        const int ch2 = grab_chunk(&S.next_chunk[0]);
        radial_chunk<K, TM, R, NW, DR, NM>(A, S, ch);
        ch = ch2;
      }
      if (tid == 0) atomicAdd(&A.counters[0], (unsigned long long)S.n_active);
      __syncthreads();
      continue;
    } else {
      constexpr bool kWs = MODE == kCached || MODE == kCachedTileFj || MODE == kDerive;
      int ch = wave;
      PairPos pp = ch < nch ? load_pair_pos(A, S, ch) : PairPos{0.0, 0.0, 0.0};
      while (ch < nch) {
        int ch2;
        pass1_chunk<K, TM, R, NW, DR, NM, kWs>(A, S, ch, nch, &ch2, pp, ws_slot + ch * chunk_elems);
        ch = ch2;
      }
    }
    __syncthreads();
    }  // MODE != kRegress

    // ---- C: descriptor, head, W ------------------------------------------
    if constexpr (MODE == kCached || MODE == kCachedTileFj || MODE == kRecompute) {
      head_stage<K, TM, R, NW, DR, NM, false>(A, S);
    } else if constexpr (MODE == kRegress) {
      head_stage<K, TM, R, NW, DR, NM, true>(A, S);
    } else if constexpr (MODE == kEncode || MODE == kDerive) {
      // encoding kernel: G to HBM; derivation kernel: W from dE/dG in HBM
      const int nin = (A.lmax + 1) * K;
      R* __restrict__ gbuf = static_cast<R*>(A.gbuf) + (long long)a0 * nin;
      for (int u = tid; u < na * nin; u += 64 * NW) {
        const int a = u / nin, in = u % nin;
        if constexpr (MODE == kEncode)
          gbuf[u] = descriptor_value(A, S, a, in);
        else
          adjoint_from_grad(A, S, a, in, gbuf[u]);
      }
      __syncthreads();
    }

    // ---- D: pass 2 ---------------------------------------------------------
    if constexpr (MODE == kCached || MODE == kCachedTileFj || MODE == kDerive) {
      constexpr bool kTileFj = MODE == kCachedTileFj;
      if constexpr (kTileFj) {
        // the head is done with the union: an empty table for this tile
        for (int u = tid; u < kFjSlots; u += 64 * NW) {
          S.u.fj.key[u] = -1;
          S.u.fj.val[u][0] = S.u.fj.val[u][1] = S.u.fj.val[u][2] = 0.0;
        }
        __syncthreads();
      }
      // inputs of the next chunk are loaded while this one is processed
      // (float64 at k = 64: two chunks' inputs alone are 256 registers)
      constexpr bool kAhead = K * sizeof(R) <= 256;
      int ch = wave;
      Pass2In<K, R> next;
      if (kAhead && ch < nch) pass2_load(A, S, ch, ws_slot + ch * chunk_elems, next);
      while (ch < nch) {
        if (!kAhead) pass2_load(A, S, ch, ws_slot + ch * chunk_elems, next);
        const Pass2In<K, R> cur = next;
        const int ch2 = grab_chunk(&S.next_chunk[1]);
        if (kAhead && ch2 < nch) pass2_load(A, S, ch2, ws_slot + ch2 * chunk_elems, next);
        pass2_chunk<K, TM, R, NW, DR, NM, kTileFj>(A, S, ch, cur);
        ch = ch2;
      }
      if constexpr (kTileFj) {
        // one atomic per distinct neighbour of the tile instead of one per pair
        __syncthreads();
        for (int u = tid; u < kFjSlots; u += 64 * NW) {
          const int j = S.u.fj.key[u];
          if (j >= 0) {
            atomicAdd(&A.forces[3 * (long long)j], S.u.fj.val[u][0]);
            atomicAdd(&A.forces[3 * (long long)j + 1], S.u.fj.val[u][1]);
            atomicAdd(&A.forces[3 * (long long)j + 2], S.u.fj.val[u][2]);
          }
        }
      }
    } else if constexpr (MODE == kRecompute) {
      // the head's activations overwrote the first-layer weights in LDS
      stage_first_layer(A, S, enc);
      __syncthreads();
      int ch = wave;
      PairPos next = ch < nch ? load_pair_pos(A, S, ch) : PairPos{0.0, 0.0, 0.0};
      while (ch < nch) {
        const PairPos cur = next;
        const int ch2 = grab_chunk(&S.next_chunk[1]);
        if (ch2 < nch) next = load_pair_pos(A, S, ch2);
        Pass2In<K, R> in;
        pass2_recompute(A, S, ch, cur, in);
        pass2_chunk<K, TM, R, NW, DR, NM>(A, S, ch, in);
        ch = ch2;
      }
    }
    __syncthreads();

    // ---- E: outputs --------------------------------------------------------
    constexpr bool kEnergy = MODE == kCached || MODE == kCachedTileFj || MODE == kRecompute || MODE == kRegress;
    constexpr bool kForces = MODE == kCached || MODE == kCachedTileFj || MODE == kRecompute || MODE == kDerive;
    if (tid < na) {
      const long long o = S.orig[tid];
      if (kEnergy && A.energy) A.energy[o] = S.Ei[tid];
      if (kForces) {
        if (A.virial) {
#pragma unroll
          for (int k = 0; k < 9; ++k) A.virial[9 * o + k] = S.Wi[tid][k];
        }
        atomicAdd(&A.forces[3 * o], S.Fi[tid][0]);
        atomicAdd(&A.forces[3 * o + 1], S.Fi[tid][1]);
        atomicAdd(&A.forces[3 * o + 2], S.Fi[tid][2]);
      }
    }
    if (wave == 0 && MODE != kEncode) {
      double v[10];
      const bool own = tid < na;
      v[0] = kEnergy && own ? S.Ei[tid] : 0.0;
#pragma unroll
      for (int k = 0; k < 9; ++k) v[1 + k] = kForces && own ? S.Wi[tid][k] : 0.0;
#pragma unroll
      for (int k = 0; k < 10; ++k)
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) v[k] += __shfl_xor(v[k], o, 64);
      if (tid < 10) {
        double mine = v[0];
#pragma unroll
        for (int k = 1; k < 10; ++k)
          if (tid == k) mine = v[k];
        // a small system's one-atom tiles are many additions to one value: what
        // each of them rounds away is summed too (mlip_internal.h: kTotals)
        const double old = atomicAdd(&A.totals[tid], mine);
        const double sum = old + mine, part = sum - old;
        atomicAdd(&A.totals[kTotalsRest + tid], (old - (sum - part)) + (mine - part));
      }
      if (tid == 0 && kForces) atomicAdd(&A.counters[0], (unsigned long long)S.n_active);
    }
    __syncthreads();
  }
}

template <int K, int TM, typename R, int NW, int DR, int NM, int MODE>
hipError_t launch_k(const FusedArgs& a, int n_blocks, hipStream_t s) {
  static_assert(sizeof(Smem<K, TM, R, NW, DR, NM>) <= 160 * 1024, "tile state exceeds the 160 KB LDS of a CU");
  const size_t smem = sizeof(Smem<K, TM, R, NW, DR, NM>);
  static bool attr_set = false;
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_fused<K, TM, R, NW, DR, NM, MODE, kDigits>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, int(smem));
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  k_fused<K, TM, R, NW, DR, NM, MODE, kDigits><<<dim3(unsigned(n_blocks)), dim3(64 * NW), smem, s>>>(a);
  return hipGetLastError();
}

#if MLIP_FUSED_PART != 2
template <int K, int TM, typename R, int NW, int DR, int NM>
hipError_t launch_mode(int mode, const FusedArgs& a, int n_blocks, hipStream_t s) {
  switch (mode) {
    case kCached: return launch_k<K, TM, R, NW, DR, NM, kCached>(a, n_blocks, s);
    case kRecompute: return launch_k<K, TM, R, NW, DR, NM, kRecompute>(a, n_blocks, s);
    case kEncode: return launch_k<K, TM, R, NW, DR, NM, kEncode>(a, n_blocks, s);
    case kDerive: return launch_k<K, TM, R, NW, DR, NM, kDerive>(a, n_blocks, s);
    case kRadial: return launch_k<K, TM, R, NW, DR, NM, kRadial>(a, n_blocks, s);
    case kCachedTileFj: return launch_k<K, TM, R, NW, DR, NM, kCachedTileFj>(a, n_blocks, s);
    default: break;
  }
  // the regression kernel has no encoder: one instantiation serves both
  if constexpr (kDigits)
    if (mode == kRegress) return launch_k<K, TM, R, NW, DR, NM, kRegress>(a, n_blocks, s);
  return hipErrorInvalidValue;
}
#endif

}  // namespace

#if MLIP_FUSED_DIGITS
#define MLIP_ENTRY(name) name##_digits
#else
#define MLIP_ENTRY(name) name##_float
#endif

#if MLIP_FUSED_PART == 1 && MLIP_FUSED_DIGITS
// Angular configurations: 0 = irreducible basis with l_max <= 3 (16 rows,
// 20 monomials), 1 = Cartesian basis with l_max <= 3 (20 rows in two 16-row
// tiles), 2 = irreducible basis with l_max 4 or 5 (up to 36 rows in three
// tiles, 56 monomials of degree <= 5).
int angular_config(int angular, int lmax) { return angular == 1 ? 1 : (lmax > 3 ? 2 : 0); }

void angular_table_shape(int acfg, int* rows, int* cols) {
  *rows = acfg == 0 ? 16 : (acfg == 1 ? 32 : 48);
  *cols = acfg == 2 ? 56 : kMonomials;
}

// Instantiations: k in {16, 32, 64}; float64 with one wavefront per SIMD,
// float32 with two.  Atoms per tile: float64 16, float32 32 (two column
// groups in the head), fewer where the moment would not fit LDS: at k = 64
// 8 (float64) and 16 (float32); l_max 4..5, whose 36-row moment and 6k-wide
// head input grow with k, 16 / 9 / 3 atoms at k = 16 / 32 / 64 in float64
// and 32 / 16 / 11 in float32 (a tile's listed entries are spread evenly
// over the work-group's threads, which rules out 17-19 at k = 32).  The
// other fusion configurations are built for k = 32 with the irreducible
// basis and l_max <= 3.
int fused_tile_max(int k, int precision, int acfg) {
  if (acfg == 1) return precision == 64 ? 16 : 32;
  if (acfg == 2) {
    if (precision == 64) return k == 16 ? 16 : (k == 32 ? 9 : 3);
    return k == 16 ? 32 : (k == 32 ? 16 : 11);
  }
  if (precision == 64) return k == 64 ? 8 : 16;
  return k == 64 ? 16 : 32;
}

hipError_t launch_fused(int k, int precision, int acfg, int mode, bool digits, const FusedArgs& a, int n_blocks,
                        hipStream_t s) {
  if (mode != kCached && (k != 32 || acfg != 0)) return hipErrorInvalidValue;
  if (acfg == 1 && k != 32) return hipErrorInvalidValue;
  if (precision != 64 && precision != 32) return hipErrorInvalidValue;
  digits = digits || mode == kRegress;
  if (precision == 32) return (digits ? launch_fused_f32_digits : launch_fused_f32_float)(k, acfg, mode, a, n_blocks, s);
  if (acfg == 2) return (digits ? launch_fused_f64_high_digits : launch_fused_f64_high_float)(k, a, n_blocks, s);
  return (digits ? launch_fused_f64_digits : launch_fused_f64_float)(k, acfg, mode, a, n_blocks, s);
}
#endif

#if MLIP_FUSED_PART == 1
hipError_t MLIP_ENTRY(launch_fused_f64)(int k, int acfg, int mode, const FusedArgs& a, int n_blocks, hipStream_t s) {
  if (acfg == 1) return launch_k<32, 16, double, 4, 32, 20, kCached>(a, n_blocks, s);
  switch (k) {
    case 16: return launch_k<16, 16, double, 4, 16, 20, kCached>(a, n_blocks, s);
    case 32: return launch_mode<32, 16, double, 4, 16, 20>(mode, a, n_blocks, s);
    case 64: return launch_k<64, 8, double, 4, 16, 20, kCached>(a, n_blocks, s);
    default: return hipErrorInvalidValue;
  }
}
#elif MLIP_FUSED_PART == 2
hipError_t MLIP_ENTRY(launch_fused_f64_high)(int k, const FusedArgs& a, int n_blocks, hipStream_t s) {
  switch (k) {
    case 16: return launch_k<16, 16, double, 4, 48, 56, kCached>(a, n_blocks, s);
    case 32: return launch_k<32, 9, double, 4, 48, 56, kCached>(a, n_blocks, s);
    case 64: return launch_k<64, 3, double, 4, 48, 56, kCached>(a, n_blocks, s);
    default: return hipErrorInvalidValue;
  }
}
#elif MLIP_FUSED_PART == 3
hipError_t MLIP_ENTRY(launch_fused_f32)(int k, int acfg, int mode, const FusedArgs& a, int n_blocks, hipStream_t s) {
  if (acfg == 1) return launch_k<32, 32, float, 8, 32, 20, kCached>(a, n_blocks, s);
  if (acfg == 2) {
    switch (k) {
      case 16: return launch_k<16, 32, float, 8, 48, 56, kCached>(a, n_blocks, s);
      case 32: return launch_k<32, 16, float, 8, 48, 56, kCached>(a, n_blocks, s);
      case 64: return launch_k<64, 11, float, 8, 48, 56, kCached>(a, n_blocks, s);
      default: return hipErrorInvalidValue;
    }
  }
  switch (k) {
    case 16: return launch_k<16, 32, float, 8, 16, 20, kCached>(a, n_blocks, s);
    case 32: return launch_mode<32, 32, float, 8, 16, 20>(mode, a, n_blocks, s);
    case 64: return launch_k<64, 16, float, 8, 16, 20, kCached>(a, n_blocks, s);
    default: return hipErrorInvalidValue;
  }
}
#endif

}  // namespace mlip
