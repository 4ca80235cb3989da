// Omnidirectional feature front end (Section 3): the magnitude of the
// discrete Fourier transform of 1-D panoramic signals, bins 0 .. d-1, is the
// rotation-invariant feature the database and the queries hold.
//
// Everything is computed in FP64 and rounded once to fp32. The real signal
// of length L = 2n is read as n complex points z_t = x_{2t} + i x_{2t+1},
// transformed at length n, and unpacked into the spectrum of x:
// X_j = E_j + exp(-i pi j / n) O_j, with E_j = (Z_j + conj Z_{n-j}) / 2 and
// O_j = (Z_j - conj Z_{n-j}) / 2i the transforms of the even and odd samples.
// The twiddles exp(-i pi j / n), j = 0 .. n, are tabulated in LDS once per
// block with sincospi.
//
// n = R1 R2 = 16 .. 1024 (L = 32 .. 2048; R1 = R2 or 2 R2): four-step transform,
// R2 lanes per signal and 64 / R2 signals per wave. Lane c loads points
// R2 t1 + c (R2 lanes read 8 R2 contiguous bytes per instruction), transforms
// them over t1 in registers, multiplies by exp(-2 pi i k1 c / n), and the wave
// transposes its signals through padded LDS rows of its own (real parts, then
// imaginary parts: half the LDS of a complex transpose, more waves per compute
// unit); lane c then transforms rows k1 = c + R2 b over t2 in registers and
// holds Z_{k1 + R1 k2}. The partner Z_{n-j} of its bin j sits in lane R2 - c
// (lane 0: its own registers) and comes by a lane shuffle; one lane of the two
// computes both X_j = E + w O and X_{n-j} = conj(E - w O). Up to 16 points a
// lane the next signals' points are loaded while the current ones are
// transformed. Any other n (1 .. 8): one wave per signal, iterative radix-2
// transform in LDS.
//
// Both read 4L and write 4d bytes per signal and do about 5 n log2 n + 20 d
// FP64 operations; FP64 instructions and their latency bound it, not memory.
// 200,000 signals to L / 2 bins, against one bin at a time with the library's
// square root (L = 128, 512) and the LDS transform (other lengths): L = 32 75 ->
// 11.5 us, 64 93 -> 22, 128 41 -> 35, 256 211 -> 79, 512 186 -> 156 (4 TB/s);
// 97,000 of 1,024 593 -> 371, 48,000 of 2,048 965 -> 384. Two waves per SIMD at 16
// points a lane; a third spills and loses half the speed.
#include <cmath>

#include "hloc_host.h"

namespace hloc {

constexpr int kFftMaxLen = 2048;   // LDS per block (2n + 1) * 16 bytes <= 32 KB
constexpr int kFftBlocksPerCu = 32;  // one wave each; 8 waves per SIMD at 45 VGPRs

constexpr int bit_reverse(int t, int bits) {
  int r = 0;
  for (int i = 0; i < bits; ++i) r |= ((t >> i) & 1) << (bits - 1 - i);
  return r;
}

__device__ __forceinline__ double2 cmul(double2 w, double2 v) {
  return make_double2(w.x * v.x - w.y * v.y, w.x * v.y + w.y * v.x);
}

// exp(-2 pi i k / 32), k = 0 .. 15, from cos(pi/8) = sqrt(2 + sqrt 2) / 2,
// sin(pi/8) = sqrt(2 - sqrt 2) / 2, cos(pi/4) = sqrt(2) / 2 and the halvings
// cos(x/2) = sqrt((1 + cos x) / 2), sin(x/2) = sqrt((1 - cos x) / 2) of pi/8 and
// 3 pi/8 (rounded to double by the compiler).
constexpr double kC8 = 0.9238795325112867561281831893967882868225;
constexpr double kS8 = 0.3826834323650897717284599840303988667612;
constexpr double kH2 = 0.7071067811865475244008443621048490392848;
constexpr double kC16 = 0.98078528040323044912618223613424;
constexpr double kS16 = 0.19509032201612826784828486847702;
constexpr double kC316 = 0.83146961230254523707878837761791;
constexpr double kS316 = 0.55557023301960222474283081394853;
__device__ constexpr double cos32(int k) {  // cos(2 pi k / 32), k = 0 .. 8
  return k == 0 ? 1.0 : k == 1 ? kC16 : k == 2 ? kC8 : k == 3 ? kC316 : k == 4 ? kH2
       : k == 5 ? kS316 : k == 6 ? kS8 : k == 7 ? kS16 : 0.0;
}
__device__ constexpr double w32_re(int k) { return k <= 8 ? cos32(k) : -cos32(16 - k); }
__device__ constexpr double w32_im(int k) { return k <= 8 ? -cos32(8 - k) : -cos32(k - 8); }

// In-register transform of R = 4 .. 32 points (bit-reversed input, natural
// output), radix-2 decimation in time with compile-time twiddles; the
// twiddles 1 and -i cost no multiply.
template <int R>
__device__ __forceinline__ void dft_regs(double2 *a) {
#pragma unroll
  for (int h = 1; h < R; h <<= 1) {
#pragma unroll
    for (int b = 0; b < R / 2; ++b) {
      const int pos = b & (h - 1);
      const int i = ((b - pos) << 1) + pos;
      const int k = pos * (32 / (2 * h));  // exp(-2 pi i pos / 2h) = w32(k)
      double2 v = a[i + h];
      if (k == 8)
        v = make_double2(v.y, -v.x);
      else if (k != 0)
        v = cmul(make_double2(w32_re(k), w32_im(k)), v);
      const double2 u = a[i];
      a[i] = make_double2(u.x + v.x, u.y + v.y);
      a[i + h] = make_double2(u.x - v.x, u.y - v.y);
    }
  }
}

// sqrt(s) / 2 rounded to float, s >= 0 (or NaN), by Goldschmidt's iteration from
// the hardware's reciprocal square root: one coupled step for sqrt(s) and
// 1 / (2 sqrt(s)) and one residual correction leave about a double's last bits,
// far below the float's; the library's square root is correctly rounded and
// also rescales for arguments this one cannot meet (s is 0 or above 1e-250:
// sums of squares of float values and their differences).
__device__ __forceinline__ float half_sqrt(double s) {
  const double y = __builtin_amdgcn_rsq(s);
  double g = s * y, h = 0.5 * y;
  const double r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  g = fma(fma(-g, g, s), h, g);
  return (float)(0.5 * (__builtin_amdgcn_class(s, 0x240) ? s : g));  // +0 and +inf as they are
}

// |X_j| from Z_j (A), Z_{n-j} (B) and tw[j], computed as |2 X_j| / 2 from
// 2 E_j and 2 O_j (scaling by powers of two is exact, so the result is the
// same as with the halvings applied first).
__device__ __forceinline__ float unpack_mag(double2 A, double2 B, double2 w) {
  const double er = A.x + B.x, ei = A.y - B.y;    // 2 E_j
  const double orr = A.y + B.y, oi = B.x - A.x;   // 2 O_j
  const double xr = er + (w.x * orr - w.y * oi);
  const double xi = ei + (w.x * oi + w.y * orr);
  return (float)(0.5 * sqrt(xr * xr + xi * xi));
}

__global__ __launch_bounds__(64) void k_fft_magnitude(const float *__restrict__ x, int64_t nsig,
                                                      int len, int log2n, int d,
                                                      float *__restrict__ out) {
  extern __shared__ double2 lds[];
  const int n = len >> 1;
  double2 *tw = lds;           // tw[j] = exp(-i pi j / n), j = 0 .. n
  double2 *a = lds + (n + 1);  // the length-n transform, in place
  const int lane = threadIdx.x;
  for (int j = lane; j <= n; j += 64) {
    double s, c;
    sincospi((double)j / (double)n, &s, &c);
    tw[j] = make_double2(c, -s);
  }
  for (int64_t sig = blockIdx.x; sig < nsig; sig += gridDim.x) {
    const float2 *row = reinterpret_cast<const float2 *>(x + sig * len);
    __syncthreads();  // the twiddles are written; the previous signal is read out
    for (int t = lane; t < n; t += 64) {
      const float2 v = row[t];
      const int r = log2n ? (int)(__builtin_bitreverse32((uint32_t)t) >> (32 - log2n)) : 0;
      a[r] = make_double2((double)v.x, (double)v.y);
    }
    for (int h = 1; h < n; h <<= 1) {
      __syncthreads();
      const int stride = n / h;  // exp(-2 pi i pos / 2h) = tw[pos * n / h]
      for (int b = lane; b < (n >> 1); b += 64) {
        const int pos = b & (h - 1);
        const int i = ((b - pos) << 1) + pos;
        const double2 w = tw[pos * stride];
        const double2 u = a[i], v = a[i + h];
        const double tr = w.x * v.x - w.y * v.y;
        const double ti = w.x * v.y + w.y * v.x;
        a[i] = make_double2(u.x + tr, u.y + ti);
        a[i + h] = make_double2(u.x - tr, u.y - ti);
      }
    }
    __syncthreads();
    float *o = out + sig * d;
    for (int j = lane; j < d; j += 64) {
      o[j] = unpack_mag(a[j & (n - 1)], a[(n - j) & (n - 1)], tw[j]);  // Z_j, Z_{n-j}
    }
  }
}

// Waves per block of the four-step kernel (they share the twiddles), whether
// the table reaches every index 2 k1 c (else those past n use the period), and
// its entries.
template <int R1, int R2>
struct FftShape {
  static constexpr int r1 = R1, r2 = R2;
  static constexpr int n = R1 * R2, G = 64 / R2, B = R1 / R2;
  static constexpr int waves = n >= 512 ? 2 : 4;
  static constexpr bool full = n <= 256;
  static constexpr int table = full ? 2 * (R1 - 1) * (R2 - 1) + 1 : n + 1;
  static constexpr int rows = G * R1 * (R2 + 1);  // doubles per wave
  static constexpr uint32_t lds = table * sizeof(double2) + waves * rows * sizeof(double);
  static constexpr bool ahead = R1 <= 16;
};

constexpr int log2_of(int v) { return v <= 1 ? 0 : 1 + log2_of(v / 2); }

template <class S>
__device__ __forceinline__ void fft_four_step(const float *__restrict__ x, int64_t nsig, int d,
                                              float *__restrict__ out) {
  constexpr int R1 = S::r1, R2 = S::r2;
  constexpr int n = S::n, G = S::G, B = S::B, LD = R2 + 1;
  constexpr int L1 = log2_of(R1), L2 = log2_of(R2);
  static_assert(R1 == R2 || R1 == 2 * R2, "one or two rows per lane");
  extern __shared__ double2 lds[];
  double2 *tw = lds;  // tw[j] = exp(-i pi j / n)
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane / R2, c = lane % R2;
  // this signal's R1 x (R2 + 1) rows (real parts, then imaginary parts)
  double *rows = reinterpret_cast<double *>(lds + S::table) + w * S::rows + g * R1 * LD;
  for (int j = threadIdx.x; j < S::table; j += 64 * S::waves) {
    double sn, cs;
    sincospi((double)j / (double)n, &sn, &cs);
    tw[j] = make_double2(cs, -sn);
  }
  __syncthreads();
  // orders the wave's LDS accesses (its rows are its own)
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  const int64_t first = ((int64_t)blockIdx.x * S::waves + w) * G;
  const int64_t stride = (int64_t)gridDim.x * S::waves * G;
  float2 cur[R1];
  auto load = [&](int64_t s) {
    const float2 *p = reinterpret_cast<const float2 *>(x) + s * n + c;
#pragma unroll
    for (int t = 0; t < R1; ++t) cur[t] = s < nsig ? p[t * R2] : make_float2(0.f, 0.f);
  };
  if (S::ahead && first < nsig) load(first + g);
  for (int64_t base = first; base < nsig; base += stride) {
    const int64_t s = base + g;
    if (!S::ahead) load(s);
    double2 a[R1];
#pragma unroll
    for (int t = 0; t < R1; ++t)
      a[bit_reverse(t, L1)] = make_double2((double)cur[t].x, (double)cur[t].y);
    if (S::ahead && base + stride < nsig) load(s + stride);
    dft_regs<R1>(a);  // a[k1] = sum_t1 z[R2 t1 + c] exp(-2 pi i t1 k1 / R1)
#pragma unroll
    for (int k1 = 1; k1 < R1; ++k1) {
      const int m = 2 * k1 * c;  // exp(-2 pi i k1 c / n) = tw[m], or -tw[m - n]
      if (S::full) {
        a[k1] = cmul(tw[m], a[k1]);
      } else {
        const double2 v = cmul(tw[m <= n ? m : m - n], a[k1]);
        a[k1] = m <= n ? v : make_double2(-v.x, -v.y);
      }
    }
#pragma unroll
    for (int k1 = 0; k1 < R1; ++k1) rows[k1 * LD + c] = a[k1].x;
    wave_sync();
    double re[R1];
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
      for (int t = 0; t < R2; ++t) re[b * R2 + t] = rows[(c + R2 * b) * LD + t];
    wave_sync();
#pragma unroll
    for (int k1 = 0; k1 < R1; ++k1) rows[k1 * LD + c] = a[k1].y;
    wave_sync();
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
      for (int t = 0; t < R2; ++t)
        a[b * R2 + bit_reverse(t, L2)] =
            make_double2(re[b * R2 + t], rows[(c + R2 * b) * LD + t]);
    wave_sync();  // the rows are read out before the next signals write them
    // a[b R2 + k2] = Z_{k1 + R1 k2}, k1 = c + R2 b
#pragma unroll
    for (int b = 0; b < B; ++b) dft_regs<R2>(a + b * R2);
    const bool valid = s < nsig;
    float *o = out + s * d;
    const int partner = g * R2 + ((R2 - c) & (R2 - 1));
#pragma unroll
    for (int b = 0; b < B; ++b) {
#pragma unroll
      for (int k2 = 0; k2 < R2 / 2; ++k2) {
        // Z_{n-j}: row R1 - k1, column R2 - 1 - k2 (row 0: column -k2)
        const double2 q = a[(B - 1 - b) * R2 + R2 - 1 - k2];
        const double2 p = make_double2(__shfl(q.x, partner), __shfl(q.y, partner));
        const double2 own = b == 0 ? a[(R2 - k2) & (R2 - 1)] : a[(B - b) * R2 + R2 - 1 - k2];
        const double2 A = a[b * R2 + k2];
        const double2 Q = make_double2(c == 0 ? own.x : p.x, c == 0 ? own.y : p.y);
        const int j = c + R2 * b + R1 * k2;
        const double2 t = tw[j];
        // 2 E_j, 2 O_j and w 2 O_j; both halvings wait for the end (exact)
        const double er = A.x + Q.x, ei = A.y - Q.y;
        const double orr = A.y + Q.y, oi = Q.x - A.x;
        const double vr = t.x * orr - t.y * oi, vi = t.x * oi + t.y * orr;
        const double xr = er + vr, xi = ei + vi, yr = er - vr, yi = ei - vi;
        const float mj = half_sqrt(xr * xr + xi * xi), mn = half_sqrt(yr * yr + yi * yi);
        if (valid && j < d) o[j] = mj;
        if (valid && n - j < d) o[n - j] = mn;
      }
    }
    // j = n / 2 is its own partner: X_j = conj Z_j
    const double2 h = a[R2 / 2];
    if (valid && c == 0 && n / 2 < d) o[n / 2] = half_sqrt(4.0 * (h.x * h.x + h.y * h.y));
  }
}

// n = R R (L = 32, 128, 512, 2048) and n = 2 R R (L = 64, 256, 1024).
template <int R>
using FftSq = FftShape<R, R>;
template <int R>
using FftSq2 = FftShape<2 * R, R>;
template <int R>
__global__ __launch_bounds__(64 * FftSq<R>::waves) void k_fft_magnitude_sq(
    const float *__restrict__ x, int64_t nsig, int d, float *__restrict__ out) {
  fft_four_step<FftSq<R>>(x, nsig, d, out);
}
template <int R>
__global__ __launch_bounds__(64 * FftSq2<R>::waves) void k_fft_magnitude_sq2(
    const float *__restrict__ x, int64_t nsig, int d, float *__restrict__ out) {
  fft_four_step<FftSq2<R>>(x, nsig, d, out);
}

template <int R1, int R2>
hipError_t launch_fft_4s(const float *x, int64_t nsig, int d, float *out, int cus,
                         hipStream_t s) {
  using S = FftShape<R1, R2>;
  void (*kernel)(const float *, int64_t, int, float *);
  if constexpr (R1 == R2) kernel = k_fft_magnitude_sq<R2>;
  else kernel = k_fft_magnitude_sq2<R2>;
  static int per_cu = 0;
  if (per_cu == 0) {
    const void *k = reinterpret_cast<const void *>(kernel);
    int occ = 0;
    if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::lds) !=
            hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k, 64 * S::waves, S::lds) !=
            hipSuccess ||
        occ < 1) {
      (void)hipGetLastError();
      occ = std::max(1, kLdsPerCu / (int)S::lds);
    }
    per_cu = occ;
  }
  // the blocks that the compute units hold at once, each wave 64 / R2 signals
  // at a time
  const int64_t per_block = (int64_t)S::G * S::waves;
  const int64_t grid = std::min<int64_t>((nsig + per_block - 1) / per_block, (int64_t)cus * per_cu);
  return launch_kernel(kernel, dim3((unsigned)grid), dim3(64 * S::waves), S::lds, s, x, nsig, d,
                       out);
}

}  // namespace hloc

using namespace hloc;

extern "C" int hloc_fft_features_async(const float *signals, int64_t nsig, int32_t len, int32_t d,
                                       float *out, void *stream) {
  if (nsig < 0) return fail(HLOC_EINVAL, "nsig must be >= 0 (got %lld)", (long long)nsig);
  if (len < 2 || len > kFftMaxLen || (len & (len - 1)) != 0)
    return fail(HLOC_EINVAL, "len must be a power of two in 2..%d (got %d)", kFftMaxLen, len);
  if (d < 1 || d > len / 2 + 1)
    return fail(HLOC_EINVAL, "d must be in 1..%d for len %d (got %d)", len / 2 + 1, len, d);
  if (nsig == 0) return HLOC_OK;
  if (!signals || !out) return fail(HLOC_EINVAL, "signals and out must not be NULL");
  int dev = 0, num_cu = 0;
  HIPCHK(hipGetDevice(&dev));
  HIPCHK(hipDeviceGetAttribute(&num_cu, hipDeviceAttributeMultiprocessorCount, dev));
  const int n = len / 2;
  const uint32_t lds = (uint32_t)(2 * n + 1) * sizeof(double2);
  const int per_cu = std::max(1, std::min<int>(kFftBlocksPerCu, kLdsPerCu / (int)lds));
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const int cus = std::max(num_cu, 1);
  const int64_t grid = std::min<int64_t>(nsig, (int64_t)cus * per_cu);
  switch (n) {
#define HLOC_FFT_CASE(R1, R2)                                                 \
  case (R1) * (R2):                                                           \
    HIPCHK((launch_fft_4s<R1, R2>(signals, nsig, (int)d, out, cus, st)));     \
    return HLOC_OK;
    HLOC_FFT_CASE(4, 4)
    HLOC_FFT_CASE(8, 4)
    HLOC_FFT_CASE(8, 8)
    HLOC_FFT_CASE(16, 8)
    HLOC_FFT_CASE(16, 16)
    HLOC_FFT_CASE(32, 16)
    HLOC_FFT_CASE(32, 32)
#undef HLOC_FFT_CASE
    default:
      break;
  }
  int log2n = 0;
  while ((1 << log2n) < n) ++log2n;
  HIPCHK(launch_kernel(k_fft_magnitude, dim3((unsigned)grid), dim3(64), lds,
                       st, signals, nsig, (int)len, log2n,
                       (int)d, out));
  return HLOC_OK;
}
