// Encoder tables in the device layout (mlip_create): the first layer's values
// as they are, each weight matrix as digits for the 16x16x64 8-bit integer MFMA
// (fused.hip) with one scale per row, or as values for the 16x16x4 one, and the
// biases; and the measure by which mlip_create chooses between the two.
//
// The integers of a row are round(w 2^(8 D) / scale) = sum_i d_i 256^(D - 1 - i)
// with digits in [-128, 127], where the row's scale takes its largest weight to
// 0.99 x 2^(8 D - 1) (balanced digits hold 0.996 times that) and is rounded to
// the type it is stored in first: rounded after the integers are formed, all
// 128 weights of a row would share its rounding error, which does not average
// over pairs and atoms.  It is NaN for a row with an infinity or NaN, whose
// digits are zero.  Digit i of the half
// hf (columns 64 hf ..) of output tile t is fragment 2 D t + D hf + i, 16 bytes at
// lane 16 g + c: byte 4 T + q is row 16 t + c, column 64 hf + 16 T + 4 g + q.
#include "mlip_internal.h"

namespace mlip {
namespace {

constexpr int W = kEncWidth;

// One work-group per row of the table's matrices (and one for the first
// layer), one thread per column.
template <typename R, bool kDig>
__global__ __launch_bounds__(W) void k_pack_encoder(const double* __restrict__ blob, int hidden, int k, R* __restrict__ out,
                                                    size_t stride) {
  constexpr int D = weight_digits(8 * int(sizeof(R)));
  const int c = threadIdx.x, row = blockIdx.x;
  const size_t square = size_t(W) * W + W;  // a hidden layer of the blob
  const double* __restrict__ src = blob + size_t(blockIdx.y) * (2 * W + (hidden - 1) * square + size_t(k) * W + k);
  R* __restrict__ dst = out + size_t(blockIdx.y) * stride;
  const int rows = (hidden - 1) * W + k;
  if (row == rows) {
    dst[c] = R(src[c]);
    dst[W + c] = R(src[W + c]);
    return;
  }
  const int layer = row / W < hidden - 1 ? row / W : hidden - 1;
  const int o = row - layer * W, nout = layer < hidden - 1 ? W : k;
  const double* __restrict__ m = src + 2 * W + layer * square;
  R* __restrict__ to = dst + 2 * W + size_t(layer) * W * (kDig ? W * D / sizeof(R) + 2 : W + 1);
  const double w = m[size_t(o) * W + c];
  if constexpr (!kDig) {
    // fragment of block (T, i) and output tile t: element [16 t + r][16 T +
    // kin(i, g)] at lane 16 g + r, kin = 4 i + g for float64 and 4 g + i for
    // float32 (the row map of the result registers); vw output tiles
    // interleaved per lane, so that a 16-byte load fetches them
    constexpr bool k64 = sizeof(R) == 8;
    const int T = c / 16, i = k64 ? c % 16 / 4 : c % 4, g = k64 ? c % 4 : c % 16 / 4;
    const int nt = nout / 16, vw = nt < int(16 / sizeof(R)) ? nt : int(16 / sizeof(R)), t = o / 16;
    to[((size_t(4 * T + i) * (nt / vw) + t / vw) * 64 + 16 * g + o % 16) * vw + t % vw] = R(w);
    if (c == 0) to[size_t(nout) * W + o] = R(m[size_t(nout) * W + o]);
    return;
  }

  // largest magnitude by bit pattern (an infinity or NaN is above all others)
  __shared__ unsigned long long part[W / 64];
  unsigned long long top = static_cast<unsigned long long>(__double_as_longlong(fabs(w)));
  for (int x = 32; x > 0; x >>= 1) {
    const unsigned long long other = __shfl_xor(top, x, 64);
    top = other > top ? other : top;
  }
  if ((c & 63) == 0) part[c >> 6] = top;
  __syncthreads();
  top = part[0] > part[1] ? part[0] : part[1];
  const bool finite = top < 0x7ff0000000000000ull;
  // the row's largest weight by an exact power of two into [0.5, 1), then its
  // scale; the integer in two steps, since beyond 2^53 a product is rounded
  int E = 0;
  double lead = 1.0;
  if (finite && top > 0) lead = frexp(__longlong_as_double(static_cast<long long>(top)), &E);
  const R scale = R(ldexp(lead * (2.0 / 0.99), E));
  const double unit = ldexp(double(R(lead * (2.0 / 0.99))), -8 * D), v = finite ? ldexp(w, -E) : 0.0;
  const double first = rint(v / unit);
  const long long X = static_cast<long long>(first) + llrint(fma(-first, unit, v) / unit);
  // an offset of 128 in every digit turns them into plain bytes
  constexpr unsigned long long kOffset = 0x80808080808080ull >> (8 * (7 - D));
  const unsigned long long x = (static_cast<unsigned long long>(X) + kOffset) ^ kOffset;
  const int hf = c / 64, T = c % 64 / 16, g = c % 16 / 4, q = c % 4;
  unsigned char* p = reinterpret_cast<unsigned char*>(to) + (size_t(o / 16) * 2 * D + size_t(hf) * D) * 1024 +
                     (16 * g + o % 16) * 16 + 4 * T + q;
#pragma unroll
  for (int i = 0; i < D; ++i) p[i * 1024] = static_cast<unsigned char>(x >> (8 * (D - 1 - i)));
  if (c == 0) {
    R* const tail = to + size_t(nout) * W * D / sizeof(R);
    tail[o] = finite ? scale : R(__builtin_nan(""));
    tail[nout + o] = R(m[size_t(nout) * W + o]);
  }
}

// Points in the distance at which the digits' terms are looked at.
constexpr int kRatioPoints = 64;
constexpr int kRatioAt = 2;  // by one work-group

// The encoder of a table at distances up to the cutoff, in float64 and plain
// order, and for each of its matrix products the largest
//   (largest weight of the row) x (largest value of the column) / sum of the
//   absolute terms:
// an error of integer digits is a fixed part of the numerator, of a
// floating-point product of the denominator (api.cpp: digits_hold).  Both the
// values and their slopes in the distance are columns.  Infinite where a value
// is not finite or a maximum is outside [low, high].
__global__ __launch_bounds__(W) void k_digit_ratio(const double* __restrict__ blob, int hidden, int k, double cutoff,
                                                   double low, double high, double* __restrict__ worst) {
  constexpr int P = kRatioAt;
  __shared__ double col[W][2 * P];  // values, then slopes
  __shared__ double part[W / 64][2 * P];
  const int o = threadIdx.x;
  const double* __restrict__ src = blob + size_t(blockIdx.x) * (2 * W + (hidden - 1) * (size_t(W) * W + W) + size_t(k) * W + k);
  double h[2 * P], z[2 * P];
  auto activate = [&](int p) {
    const double s = 1.0 / (1.0 + exp(-z[p]));
    h[P + p] += s * (1.0 + z[p] * (1.0 - s)) * z[P + p];
    h[p] += z[p] * s;
  };
  for (int p = 0; p < P; ++p) {
    z[p] = src[o] * (cutoff * (blockIdx.y * P + p + 1) / kRatioPoints) + src[W + o];
    z[P + p] = src[o];
    h[p] = h[P + p] = 0.0;
    activate(p);
  }
  double ratio = 0.0;
  for (int t = 1; t <= hidden; ++t) {
    __syncthreads();
    for (int p = 0; p < 2 * P; ++p) {
      col[o][p] = h[p];
      double v = fabs(h[p]);
      for (int x = 32; x > 0; x >>= 1) v = fmax(v, __shfl_xor(v, x, 64));
      if ((o & 63) == 0) part[o >> 6][p] = v;
    }
    __syncthreads();
    const double* __restrict__ m = src + 2 * W + (t - 1) * (size_t(W) * W + W);
    const int nout = t < hidden ? W : k;
    if (o < nout) {
      double top = 0.0, sums[2 * P];
      for (int p = 0; p < 2 * P; ++p) {
        z[p] = p < P ? m[size_t(nout) * W + o] : 0.0;
        sums[p] = 0.0;
      }
#pragma unroll 8
      for (int c = 0; c < W; ++c) {
        const double w = m[size_t(o) * W + c];
        top = fmax(top, fabs(w));
        for (int p = 0; p < 2 * P; ++p) {
          const double x = w * col[c][p];
          z[p] += x;
          sums[p] += fabs(x);
        }
      }
      auto fits = [&](double v) { return v == 0.0 || (v >= low && v <= high); };
      for (int p = 0; p < 2 * P; ++p) {
        // a NaN or infinity anywhere in the row or column is in its sum
        const double most = fmax(part[0][p], part[1][p]);
        const bool ok = isfinite(sums[p]) && fits(top) && fits(most);
        const double r = top * most > 0.0 ? top * most / sums[p] : 0.0;
        ratio = ok && r >= 0.0 ? fmax(ratio, r) : __builtin_inf();
      }
    }
    if (t < hidden)
      for (int p = 0; p < P; ++p) activate(p);
  }
  for (int x = 32; x > 0; x >>= 1) ratio = fmax(ratio, __shfl_xor(ratio, x, 64));
  // non-negative doubles order like their bit patterns
  if ((o & 63) == 0)
    atomicMax(reinterpret_cast<unsigned long long*>(worst), static_cast<unsigned long long>(__double_as_longlong(ratio)));
}

}  // namespace

hipError_t launch_pack_encoder(const double* blob, int tables, int hidden, int k, int precision, bool digits, void* out,
                               size_t stride, hipStream_t s) {
  const dim3 grid(unsigned((hidden - 1) * W + k + 1), unsigned(tables));
  double* const d = static_cast<double*>(out);
  float* const f = static_cast<float*>(out);
  if (precision == 64 && digits) k_pack_encoder<double, true><<<grid, W, 0, s>>>(blob, hidden, k, d, stride);
  else if (precision == 64) k_pack_encoder<double, false><<<grid, W, 0, s>>>(blob, hidden, k, d, stride);
  else if (digits) k_pack_encoder<float, true><<<grid, W, 0, s>>>(blob, hidden, k, f, stride);
  else k_pack_encoder<float, false><<<grid, W, 0, s>>>(blob, hidden, k, f, stride);
  return hipGetLastError();
}

hipError_t launch_digit_ratio(const double* blob, int tables, int hidden, int k, double cutoff, int precision,
                              double* worst, hipStream_t s) {
  // maxima whose scales, and their products with a value, are normal numbers
  const double range = precision == 64 ? 0x1p+900 : 0x1p+80;
  k_digit_ratio<<<dim3(unsigned(tables), kRatioPoints / kRatioAt), W, 0, s>>>(blob, hidden, k, cutoff, 1.0 / range, range, worst);
  return hipGetLastError();
}

}  // namespace mlip
