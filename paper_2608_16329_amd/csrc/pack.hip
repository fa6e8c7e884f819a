// Encoder tables in the device layout (mlip_create): the first layer's values
// as they are, each weight matrix as digits for the 16x16x64 8-bit integer MFMA
// (fused.hip) with one scale per row, and the biases.
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
template <typename R>
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
  R* __restrict__ to = dst + 2 * W + size_t(layer) * W * (W * D / sizeof(R) + 2);
  const double w = m[size_t(o) * W + c];

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

}  // namespace

hipError_t launch_pack_encoder(const double* blob, int tables, int hidden, int k, int precision, void* out, size_t stride,
                               hipStream_t s) {
  const dim3 grid(unsigned((hidden - 1) * W + k + 1), unsigned(tables));
  if (precision == 64)
    k_pack_encoder<double><<<grid, W, 0, s>>>(blob, hidden, k, static_cast<double*>(out), stride);
  else
    k_pack_encoder<float><<<grid, W, 0, s>>>(blob, hidden, k, static_cast<float*>(out), stride);
  return hipGetLastError();
}

}  // namespace mlip
