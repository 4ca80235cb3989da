// Low-precision distance screens on MFMA and the copies they read: bf16
// (v_mfma_f32_16x16x32_bf16) and OCP fp8 e4m3 with one fp32 scale per vector
// (v_mfma_f32_16x16x32_fp8_fp8).
//
// Same work items and lane layout as the fp32 register screen, with fewer
// bytes per row: lane l holds row (l % 16) and frame (l % 16) and takes the
// 16-byte pieces 4 s + l / 16 of their rows, so the 16 rows of a block are
// read as 64-byte runs. A bf16 piece (8 values) feeds one MFMA, an fp8 piece
// (16 values) two; rows and frames use the same assignment of values to MFMA
// k slots, so every piece of a row meets the same piece of the frame.
// Products are accumulated in fp32 (fp8 products are exact in fp32); the fp8
// sum is multiplied by the frame's and the row's scale. The screen value is
// |q|^2 + |d|^2 - 2 q~.d~ with the norms of the fp32 vectors and the dot
// product of their roundings q~, d~ (for fp8: scale times the e4m3 value);
// its error against the exact distance is bounded by the select kernel from
// |q~ - q| and |q~| (per frame, from the prep kernel) and the largest
// |d~ - d| and |d~| over the rows (from the copy kernels below).
#include "hloc_device.h"
#include "hloc_internal.h"

#include <algorithm>

namespace hloc {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));  // 16-byte piece (native vector)

constexpr float kFp8Max = 448.f;  // largest finite OCP e4m3 value

// Round-to-nearest-even fp32 -> bf16 bits (finite inputs).
__device__ __forceinline__ uint16_t bf16_rne(float x) {
  const uint32_t u = __float_as_uint(x);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Value of an OCP e4m3 byte (sign, 4 exponent bits of bias 7, 3 mantissa
// bits; exponent 0 is subnormal). The two NaN codes are never produced here.
__device__ __forceinline__ float fp8_to_f32(uint32_t b) {
  const int e = (b >> 3) & 15, m = b & 7;
  const float v = e == 0 ? ldexpf((float)m, -9) : ldexpf((float)(8 + m), e - 10);
  return (b & 0x80) ? -v : v;
}

// Nearest e4m3 bytes of x0 and x1 (|x| <= 448), in the low two bytes.
__device__ __forceinline__ uint32_t fp8_pair(float x0, float x1) {
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(x0, x1, 0, false) & 0xFFFFu;
}

__device__ __forceinline__ float clamp_fp8(float x) { return fminf(fmaxf(x, -kFp8Max), kFp8Max); }

constexpr int kLpRowsPerWave = 16;

// Low-precision copy of n rows of dp floats, kLpRowsPerWave rows per wave.
// bf16: dst holds dp 16-bit values per row. fp8: dst holds dp bytes per row
// and scale[i] = max |row| / 448 (1 for a zero row), the row being
// scale[i] * e4m3(row / scale[i]). Per-row FP64 norms of the rounding error
// and of the rounded row; maxima into max_err / max_norm (float bits, one
// atomic per block).
template <int FMT>
__global__ void k_rows_to_lp(const float *__restrict__ src, int64_t n, int dp, void *dst_,
                             float *__restrict__ scale, float *max_err, float *max_norm) {
  __shared__ float s_e[4], s_n[4];
  const int lane = lane_id();
  const int64_t i0 = ((int64_t)blockIdx.x * 4 + wave_id()) * kLpRowsPerWave;
  float me = 0.f, mn = 0.f;
  for (int64_t i = i0; i < min(n, i0 + kLpRowsPerWave); ++i) {
    const float *r = src + i * dp;
    double e2 = 0.0, n2 = 0.0;
    if (FMT == HLOC_BF16) {
      uint16_t *o = static_cast<uint16_t *>(dst_) + i * dp;
      for (int c = lane; c < dp; c += 64) {
        const uint16_t h = bf16_rne(r[c]);
        o[c] = h;
        const double t = (double)bf16_to_f32(h);
        e2 = fma(t - (double)r[c], t - (double)r[c], e2);
        n2 = fma(t, t, n2);
      }
    } else {
      uint8_t *o = static_cast<uint8_t *>(dst_) + i * dp;
      float amax = 0.f;
      for (int c = lane; c < dp; c += 64) amax = fmaxf(amax, fabsf(r[c]));
      for (int o2 = 32; o2 > 0; o2 >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o2));
      const float sc = amax > 0.f ? amax / kFp8Max : 1.f;
      const float inv = amax > 0.f ? kFp8Max / amax : 1.f;
      if (lane == 0) scale[i] = sc;
      // two values per lane per step: dp is a multiple of 32
      for (int c = 2 * lane; c < dp; c += 128) {
        const uint32_t p = fp8_pair(clamp_fp8(r[c] * inv), clamp_fp8(r[c + 1] * inv));
        o[c] = (uint8_t)p;
        o[c + 1] = (uint8_t)(p >> 8);
        const double t0 = (double)fp8_to_f32(p & 0xFF) * sc, t1 = (double)fp8_to_f32(p >> 8) * sc;
        e2 = fma(t0 - (double)r[c], t0 - (double)r[c], e2);
        e2 = fma(t1 - (double)r[c + 1], t1 - (double)r[c + 1], e2);
        n2 = fma(t0, t0, n2);
        n2 = fma(t1, t1, n2);
      }
    }
    e2 = wave_sum_f64(e2);
    n2 = wave_sum_f64(n2);
    me = fmaxf(me, (float)sqrt(e2));
    mn = fmaxf(mn, (float)sqrt(n2));
  }
  if (lane == 0) {
    s_e[wave_id()] = me;
    s_n[wave_id()] = mn;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) {
      s_e[0] = fmaxf(s_e[0], s_e[w]);
      s_n[0] = fmaxf(s_n[0], s_n[w]);
    }
    atomicMax(reinterpret_cast<unsigned int *>(max_err), __float_as_uint(s_e[0]));
    atomicMax(reinterpret_cast<unsigned int *>(max_norm), __float_as_uint(s_n[0]));
  }
}

hipError_t launch_rows_to_lp(int32_t fmt, const float *src, int64_t n, int32_t dp, void *dst,
                             float *scale, float *max_err, float *max_norm, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const dim3 grid((unsigned)((n + 4 * kLpRowsPerWave - 1) / (4 * kLpRowsPerWave)));
  if (fmt == HLOC_BF16)
    return launch_kernel(k_rows_to_lp<HLOC_BF16>, grid, dim3(256), 0, s, src, n, dp, dst, scale,
                         max_err, max_norm);
  if (fmt == HLOC_FP8)
    return launch_kernel(k_rows_to_lp<HLOC_FP8>, grid, dim3(256), 0, s, src, n, dp, dst, scale,
                         max_err, max_norm);
  return hipErrorInvalidValue;
}

// One frame per wave, its values in registers (4 consecutive ones per lane
// and 256-value chunk): padded fp32 copy and squared norm and, for the low-
// precision screens, the copy rounded the same way as the rows (fp8: with a
// scale per frame) with the norms of the rounding error (q_err) and of the
// rounded frame (q_lon), rounded up. FMT: the fine screen's copy (0: none);
// COARSE: a bf16 copy beside it for the coarse screen. One launch and one read
// of the frames instead of two or three (32,768 frames x 512 to bf16 54 -> 32
// us, 2,048 frames to fp8 and bf16 18 -> 8.3).
constexpr int kPrepDim = HLOC_MAX_DIM;  // padded length at most (a multiple of 32)
static_assert(kPrepDim <= 1024, "four chunks of 256 values");

// fp8 with terms = 2: the frame as the sum of two e4m3 vectors of one scale,
// the rounded frame and, behind it, the rounding of what that leaves out (at
// most 2^-4 of each value, so it rounds at the same scale to 2^-8 of it).
template <int FMT, int CH>
__device__ __forceinline__ void frame_copy(const float4 (&v)[CH], int f, int dp, int terms,
                                           void *dst, float *__restrict__ scale,
                                           float *__restrict__ q_err,
                                           float *__restrict__ q_lon) {
  const int lane = lane_id();
  double e2 = 0.0, n2 = 0.0;
  auto add = [&](double t, float x) {
    e2 = fma(t - (double)x, t - (double)x, e2);
    n2 = fma(t, t, n2);
  };
  if (FMT == HLOC_BF16) {
    uint16_t *o = static_cast<uint16_t *>(dst) + (int64_t)f * dp;
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int c = 256 * u + 4 * lane;
      if (c >= dp) continue;
      const ushort4 h = make_ushort4(bf16_rne(v[u].x), bf16_rne(v[u].y), bf16_rne(v[u].z),
                                     bf16_rne(v[u].w));
      *reinterpret_cast<ushort4 *>(o + c) = h;
      add((double)bf16_to_f32(h.x), v[u].x);
      add((double)bf16_to_f32(h.y), v[u].y);
      add((double)bf16_to_f32(h.z), v[u].z);
      add((double)bf16_to_f32(h.w), v[u].w);
    }
  } else {
    uint8_t *o = static_cast<uint8_t *>(dst) + (int64_t)f * terms * dp;
    float amax = 0.f;
#pragma unroll
    for (int u = 0; u < CH; ++u)
      amax = fmaxf(amax, fmaxf(fmaxf(fabsf(v[u].x), fabsf(v[u].y)),
                               fmaxf(fabsf(v[u].z), fabsf(v[u].w))));
    for (int o2 = 32; o2 > 0; o2 >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o2));
    const float sc = amax > 0.f ? amax / kFp8Max : 1.f;
    const float inv = amax > 0.f ? kFp8Max / amax : 1.f;
    if (lane == 0) scale[f] = sc;
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int c = 256 * u + 4 * lane;
      if (c >= dp) continue;
      const float x[4] = {clamp_fp8(v[u].x * inv), clamp_fp8(v[u].y * inv),
                          clamp_fp8(v[u].z * inv), clamp_fp8(v[u].w * inv)};
      const uint32_t h = fp8_pair(x[0], x[1]) | fp8_pair(x[2], x[3]) << 16;
      *reinterpret_cast<uint32_t *>(o + c) = h;
      float t[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) t[e] = fp8_to_f32(h >> (8 * e) & 0xFF);
      if (terms == 2) {
        const uint32_t l = fp8_pair(x[0] - t[0], x[1] - t[1]) |
                           fp8_pair(x[2] - t[2], x[3] - t[3]) << 16;
        *reinterpret_cast<uint32_t *>(o + dp + c) = l;
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] += fp8_to_f32(l >> (8 * e) & 0xFF);  // (exact)
      }
      add((double)t[0] * sc, v[u].x);
      add((double)t[1] * sc, v[u].y);
      add((double)t[2] * sc, v[u].z);
      add((double)t[3] * sc, v[u].w);
    }
  }
  e2 = wave_sum_f64(e2);
  n2 = wave_sum_f64(n2);
  if (lane == 0) {
    q_err[f] = (float)sqrt(e2) * (1.0f + 1e-6f);
    q_lon[f] = (float)sqrt(n2) * (1.0f + 1e-6f);
  }
}

template <int FMT, bool COARSE, int CH>
__global__ __launch_bounds__(256) void k_prep_frames(PrepArgs a) {
  if (blockIdx.x == 0)
    for (int t = threadIdx.x; t < kMiscInts; t += 256) a.zero[t] = 0;
  for (int t = blockIdx.x * 256 + threadIdx.x; t < a.n_counts; t += gridDim.x * 256) a.counts[t] = 0;
  const int f = blockIdx.x * 4 + wave_id(), lane = lane_id();
  if (f >= a.nq) return;
  const float *src = a.q + (int64_t)(a.period > 0 ? f % a.period : f) * a.d;
  // whole 16-byte loads where every row starts on 16 bytes
  const bool vec = a.d % 4 == 0 && (reinterpret_cast<uintptr_t>(a.q) & 15) == 0;
  float4 v[CH];
#pragma unroll
  for (int u = 0; u < CH; ++u) {
    const int c = 256 * u + 4 * lane;
    v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (vec) {
      if (c < a.d) v[u] = *reinterpret_cast<const float4 *>(src + c);
    } else {
      if (c < a.d) v[u].x = src[c];
      if (c + 1 < a.d) v[u].y = src[c + 1];
      if (c + 2 < a.d) v[u].z = src[c + 2];
      if (c + 3 < a.d) v[u].w = src[c + 3];
    }
  }
  float acc = 0.f;
#pragma unroll
  for (int u = 0; u < CH; ++u) {
    const int c = 256 * u + 4 * lane;
    if (c < a.dp) *reinterpret_cast<float4 *>(a.qp + (int64_t)f * a.dp + c) = v[u];
    acc = fmaf(v[u].x, v[u].x, acc);
    acc = fmaf(v[u].y, v[u].y, acc);
    acc = fmaf(v[u].z, v[u].z, acc);
    acc = fmaf(v[u].w, v[u].w, acc);
  }
  acc = wave_sum_f32(acc);
  if (lane == 0) a.qn2[f] = acc;
  if constexpr (FMT != 0) frame_copy<FMT, CH>(v, f, a.dp, a.terms, a.lp, a.scale, a.err, a.lon);
  if constexpr (COARSE) frame_copy<HLOC_BF16, CH>(v, f, a.dp, 1, a.c_lp, nullptr, a.c_err, a.c_lon);
}

template <int CH>
hipError_t launch_prep_ch(int32_t fmt, const PrepArgs &a, hipStream_t s) {
  const dim3 grid((unsigned)((a.nq + 3) / 4)), block(256);
  if (fmt == 0) return launch_kernel(k_prep_frames<0, false, CH>, grid, block, 0, s, a);
  if (fmt == HLOC_BF16)
    return launch_kernel(k_prep_frames<HLOC_BF16, false, CH>, grid, block, 0, s, a);
  if (fmt != HLOC_FP8) return hipErrorInvalidValue;
  return a.c_lp ? launch_kernel(k_prep_frames<HLOC_FP8, true, CH>, grid, block, 0, s, a)
                : launch_kernel(k_prep_frames<HLOC_FP8, false, CH>, grid, block, 0, s, a);
}

hipError_t launch_prep_frames(int32_t fmt, const PrepArgs &a, hipStream_t s) {
  if (a.nq <= 0) return hipSuccess;
  if (a.dp > kPrepDim) return hipErrorInvalidValue;
  if (a.dp <= 256) return launch_prep_ch<1>(fmt, a, s);
  if (a.dp <= 512) return launch_prep_ch<2>(fmt, a, s);
  return launch_prep_ch<4>(fmt, a, s);
}

// One 16-byte piece of a row against the same piece of a frame.
template <int FMT>
__device__ __forceinline__ v4f lp_mfma(uint4 a, uint4 b, v4f acc) {
  if (FMT == HLOC_BF16) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a),
                                                   __builtin_bit_cast(v8bf, b), acc, 0, 0, 0);
  } else {
    const long a0 = (long)(((uint64_t)a.y << 32) | a.x), a1 = (long)(((uint64_t)a.w << 32) | a.z);
    const long b0 = (long)(((uint64_t)b.y << 32) | b.x), b1 = (long)(((uint64_t)b.w << 32) | b.z);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a0, b0, acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a1, b1, acc, 0, 0, 0);
  }
}

// The same on native vectors (kept in registers across loops).
template <int FMT>
__device__ __forceinline__ v4f lp_mfma_v(v4u a, v4u b, v4f acc) {
  if (FMT == HLOC_BF16) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a),
                                                   __builtin_bit_cast(v8bf, b), acc, 0, 0, 0);
  } else {
    const long a0 = (long)(((uint64_t)a.y << 32) | a.x), a1 = (long)(((uint64_t)a.w << 32) | a.z);
    const long b0 = (long)(((uint64_t)b.y << 32) | b.x), b1 = (long)(((uint64_t)b.w << 32) | b.z);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a0, b0, acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a1, b1, acc, 0, 0, 0);
  }
}

// Screen word of a row with squared norm rn against a frame with squared norm
// qn, from the low-precision dot product (times the two scales for fp8).
template <int FMT>
__device__ __forceinline__ uint32_t lp_word(float qn, float rn, float acc, float qs, float rs) {
  if (__builtin_isinf(rn)) return 0xFFFFFFFFu;
  const float dot = FMT == HLOC_FP8 ? acc * (qs * rs) : acc;
  float dd = (qn + rn) - 2.f * dot;
  dd = dd > 0.f ? dd : 0.f;
  return __float_as_uint(dd);
}

// Dense items and narrow list items, one item per block, one 16-row block per
// wave, as the fp32 register screen. NS = 16-byte pieces per lane and row
// (row bytes / 64).
template <int FMT, int NS, bool DENSE>
__global__ __launch_bounds__(256) void k_screen_lp(ScreenArgs a) {
  constexpr int ROWU4 = 4 * NS;  // 16-byte pieces per row
  const int lane = lane_id(), w = wave_id(), nw = blockDim.x >> 6;
  const int i = lane & 15, g = lane >> 4;
  const uint4 *rows = static_cast<const uint4 *>(a.rows_lp);
  const uint4 *frames = static_cast<const uint4 *>(a.q_lp);
  int lo = 0, hi, nchunks = 1;
  const int terms = FMT == HLOC_FP8 ? a.terms : 1;
  // dense mode: frames 0 .. nq - 1, or the listed ones
  const int nqd = DENSE && a.frame_list ? *a.frame_count : a.nq;
  if (DENSE) {
    nchunks = (a.nrows + a.rows_per_item - 1) / a.rows_per_item;
    hi = nchunks * ((nqd + kGroup - 1) / kGroup);
  } else {
    hi = a.n_items[4];  // the narrow items: at most kGroup frames each
  }
  // list items: the next item's descriptor and frame entry are fetched while
  // the current one is screened
  Item nx{};
  int2 ne = make_int2(0, 0);
  if (!DENSE && lo + (int)blockIdx.x < hi) {
    nx = a.items[lo + blockIdx.x];
    if (i < (nx.nrows_gq & 0xFFFF)) ne = a.rq[nx.q0 + i];
  }
  for (int it = lo + blockIdx.x; it < hi; it += gridDim.x) {
    int row_begin, chunk_row, nrows, gq, fr = 0;
    int64_t off = 0;
    const int itn = it + gridDim.x;
    if (DENSE) {
      const int c = it % nchunks, grp = it / nchunks;
      row_begin = c * a.rows_per_item;
      chunk_row = row_begin;
      nrows = min(a.rows_per_item, a.nrows - row_begin);
      gq = min(kGroup, nqd - grp * kGroup);
      fr = grp * kGroup + i;
      if (a.frame_list) fr = i < gq ? a.frame_list[fr] : 0;
      off = (int64_t)fr * a.cap + chunk_row;
    } else {
      row_begin = nx.row_begin;
      chunk_row = nx.block;
      nrows = nx.nrows_gq >> 16;
      gq = nx.nrows_gq & 0xFFFF;
      if (i < gq) {
        fr = ne.x;
        off = (int64_t)ne.x * a.cap + ne.y + chunk_row;
      }
      if (itn < hi) nx = a.items[itn];
    }
    if (i >= gq) fr = 0;
    const int nrb = (nrows + 15) >> 4;
    for (int rb = w; rb < nrb; rb += nw) {
      const int rl = min(rb * 16 + i, nrows - 1);
      const uint4 *rp = rows + (int64_t)(row_begin + rl) * ROWU4 + g;
      const uint4 *qp = frames + (int64_t)fr * (terms * ROWU4) + g;
      uint4 av[NS], bv[NS];
#pragma unroll
      for (int s = 0; s < NS; ++s) av[s] = rp[4 * s];
#pragma unroll
      for (int s = 0; s < NS; ++s) bv[s] = qp[4 * s];
      const float qn = a.qn2[fr];
      const float qs = FMT == HLOC_FP8 ? a.q_scale[fr] : 1.f;
      v4f acc = {0.f, 0.f, 0.f, 0.f};
      if (FMT == HLOC_FP8 && terms == 2) {
        uint4 cv[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) cv[s] = qp[ROWU4 + 4 * s];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          acc = lp_mfma<FMT>(av[s], bv[s], acc);
          acc = lp_mfma<FMT>(av[s], cv[s], acc);
        }
      } else {
#pragma unroll
        for (int s = 0; s < NS; ++s) acc = lp_mfma<FMT>(av[s], bv[s], acc);
      }
      // the lane's four rows are consecutive rows of its frame's list
      const int row0 = rb * 16 + 4 * g;
      uint32_t wd[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int grow = row_begin + min(row0 + r, nrows - 1);
        const float rs = FMT == HLOC_FP8 ? a.row_scale[grow] : 1.f;
        wd[r] = row0 + r < nrows ? lp_word<FMT>(qn, a.row_n2[grow], acc[r], qs, rs) : 0xFFFFFFFFu;
      }
      if (DENSE) {
        if (i < gq) {
          if (row0 + 3 < nrows) {
            store_words4(a.cand + off + row0, wd[0], wd[1], wd[2], wd[3]);
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (row0 + r < nrows) a.cand[off + row0 + r] = wd[r];
          }
        }
      } else {
        const uint32_t m = block_min16(wd);
        if (i < gq && g == 0) a.cand[off + rb] = m;
      }
      if (!DENSE && rb == w && itn < hi) {
        ne = make_int2(0, 0);
        if (i < (nx.nrows_gq & 0xFFFF)) ne = a.rq[nx.q0 + i];
      }
    }
    if (!DENSE && w >= nrb && itn < hi) {
      ne = make_int2(0, 0);
      if (i < (nx.nrows_gq & 0xFFFF)) ne = a.rq[nx.q0 + i];
    }
  }
}

// Fine screen without an item list (direct mode), as the fp32 one.
template <int FMT, int NS>
__global__ __launch_bounds__(256) void k_screen_direct_lp(ScreenArgs a) {
  constexpr int ROWU4 = 4 * NS;
  const int lane = lane_id(), i = lane & 15, g = lane >> 4;
  const uint4 *rows = static_cast<const uint4 *>(a.rows_lp);
  const uint4 *frames = static_cast<const uint4 *>(a.q_lp);
  const int terms = FMT == HLOC_FP8 ? a.terms : 1;
  direct_groups(a, i, [&](int4 t, int2 e, int left) {
    const int row0 = 4 * g;
    const uint4 *rp = rows + (int64_t)(t.x + min(i, t.y - 1)) * ROWU4 + g;
    const uint4 *qp = frames + (int64_t)e.x * (terms * ROWU4) + g;
    uint4 av[NS], bv[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) av[s] = rp[4 * s];
#pragma unroll
    for (int s = 0; s < NS; ++s) bv[s] = qp[4 * s];
    const float qn = a.qn2[e.x];
    const float qs = FMT == HLOC_FP8 ? a.q_scale[e.x] : 1.f;
    v4f acc = {0.f, 0.f, 0.f, 0.f};
    if (FMT == HLOC_FP8 && terms == 2) {
      uint4 cv[NS];
#pragma unroll
      for (int s = 0; s < NS; ++s) cv[s] = qp[ROWU4 + 4 * s];
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        acc = lp_mfma<FMT>(av[s], bv[s], acc);
        acc = lp_mfma<FMT>(av[s], cv[s], acc);
      }
    } else {
#pragma unroll
      for (int s = 0; s < NS; ++s) acc = lp_mfma<FMT>(av[s], bv[s], acc);
    }
    uint32_t wd[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = t.x + min(row0 + r, t.y - 1);
      const float rs = FMT == HLOC_FP8 ? a.row_scale[row] : 1.f;
      wd[r] = row0 + r < t.y ? lp_word<FMT>(qn, a.row_n2[row], acc[r], qs, rs) : 0xFFFFFFFFu;
    }
    const uint32_t m = block_min16(wd);
    if (i < left && g == 0) a.cand[(int64_t)e.x * a.cap + e.y + t.w] = m;
  });
}

// Wide list items, as the fp32 wide screen: the chunk's rows (and fp8 scales)
// staged in LDS once, a 16-frame group per wave at a time.
template <int FMT, int NS>
__global__ __launch_bounds__(256) void k_screen_wide_lp(ScreenArgs a) {
  constexpr int ROWU4 = 4 * NS;
  constexpr int LDR = ROWU4 + 1;  // pieces per LDS row, one of padding
  extern __shared__ uint4 s_rows[];  // 64 x LDR
  __shared__ float s_rn[64], s_rs[64];
  const int tid = threadIdx.x, lane = lane_id(), w = wave_id(), nw = blockDim.x >> 6;
  const int i = lane & 15, g = lane >> 4;
  const uint4 *rows = static_cast<const uint4 *>(a.rows_lp);
  const uint4 *frames = static_cast<const uint4 *>(a.q_lp);
  const int terms = FMT == HLOC_FP8 ? a.terms : 1;
  // the chunk of the block's next item is read into registers (all of a
  // thread's pieces at once) while the current one is screened, with the rq
  // entry of each lane's frame in the wave's first group
  constexpr int PER = 64 * ROWU4 / 256;  // pieces per thread (256 threads)
  static_assert(64 * ROWU4 % 256 == 0, "whole pieces per thread");
  uint4 pv[PER];
  float prn = 0.f, prs = 1.f;
  WideItem wn{};
  int2 pe = make_int2(0, 0);
  auto fetch = [&](int item) {
    wn = wide_item(a, item);
    pe = wide_entry(a, wn, w * kGroup + i);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = tid + u * 256, row = e / ROWU4, c = e - row * ROWU4;
      pv[u] = row < wn.nrows ? rows[(int64_t)(wn.row_begin + row) * ROWU4 + c]
                             : make_uint4(0u, 0u, 0u, 0u);
    }
    if (tid < 64) {
      prn = tid < wn.nrows ? a.row_n2[wn.row_begin + tid] : 0.f;
      prs = (FMT == HLOC_FP8 && tid < wn.nrows) ? a.row_scale[wn.row_begin + tid] : 1.f;
    }
  };
  int lo;
  const int hi = wide_range(a, &lo);
  if (lo + (int)blockIdx.x < hi) fetch(lo + blockIdx.x);
  for (int it = lo + blockIdx.x; it < hi; it += gridDim.x) {
    const WideItem wi = wn;
    const int nrows = wi.nrows, gq = wi.gq;
    int2 ce = pe;
    __syncthreads();  // the previous item's rows are no longer read
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = tid + u * 256, row = e / ROWU4, c = e - row * ROWU4;
      s_rows[row * LDR + c] = pv[u];
    }
    if (tid < 64) {
      s_rn[tid] = prn;
      s_rs[tid] = prs;
    }
    __syncthreads();
    if (it + (int)gridDim.x < hi) fetch(it + gridDim.x);
    for (int grp = w; grp * kGroup < gq; grp += nw) {
      const int gs = min(kGroup, gq - grp * kGroup);
      int fr = 0;
      int64_t off = 0;
      if (i < gs) wide_frame(a, wi, grp * kGroup + i, ce, &fr, &off);
      const uint4 *qp = frames + (int64_t)fr * (terms * ROWU4) + g;
      uint4 bv[NS], cv[FMT == HLOC_FP8 ? NS : 1];
#pragma unroll
      for (int s = 0; s < NS; ++s) bv[s] = qp[4 * s];
      if (FMT == HLOC_FP8 && terms == 2) {
#pragma unroll
        for (int s = 0; s < (FMT == HLOC_FP8 ? NS : 1); ++s) cv[s] = qp[ROWU4 + 4 * s];
      }
      const float qn = a.qn2[fr];
      const float qs = FMT == HLOC_FP8 ? a.q_scale[fr] : 1.f;
      ce = wide_entry(a, wi, (grp + nw) * kGroup + i);  // the wave's next group
      uint32_t bm[4];  // list items: the frame's block words of the chunk
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) {
        bm[rb] = 0xFFFFFFFFu;
        if (rb * 16 >= nrows) continue;
        const uint4 *rp = s_rows + (rb * 16 + i) * LDR + g;
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        if (FMT == HLOC_FP8 && terms == 2) {
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            const uint4 av = rp[4 * s];
            acc = lp_mfma<FMT>(av, bv[s], acc);
            acc = lp_mfma<FMT>(av, cv[FMT == HLOC_FP8 ? s : 0], acc);
          }
        } else {
#pragma unroll
          for (int s = 0; s < NS; ++s) acc = lp_mfma<FMT>(rp[4 * s], bv[s], acc);
        }
        // the lane's four rows are consecutive rows of its frame's list
        const int row0 = rb * 16 + 4 * g;
        uint32_t wd[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = min(row0 + r, 63);
          wd[r] = row0 + r < nrows ? lp_word<FMT>(qn, s_rn[row], acc[r], qs, s_rs[row])
                                   : 0xFFFFFFFFu;
        }
        if (a.dense) {
          if (i < gs) {
            if (row0 + 3 < nrows) {
              store_words4(a.cand + off + row0, wd[0], wd[1], wd[2], wd[3]);
            } else {
#pragma unroll
              for (int r = 0; r < 4; ++r)
                if (row0 + r < nrows) a.cand[off + row0 + r] = wd[r];
            }
          }
        } else {
          bm[rb] = block_min16(wd);
        }
      }
      if (!a.dense && i < gs && g == 0) {
        const int nrb = (nrows + 15) >> 4;
        if (nrb == 4) {
          store_words4(a.cand + off, bm[0], bm[1], bm[2], bm[3]);
        } else {
#pragma unroll
          for (int rb = 0; rb < 4; ++rb)
            if (rb < nrb) a.cand[off + rb] = bm[rb];
        }
      }
    }
  }
}

// Wide list items with the rows held in registers and the frames staged
// through LDS, 16 at a time, double-buffered (wide items of the bf16 and fp8
// screens when the padded length gives NS % 4 == 0).
// A block of four waves takes one wide item: up to kWideRunsRs runs of 128
// rows of one region against the item's gq frames. For each run, wave w
// holds rows 32 w .. 32 w + 31 as the MFMA A operand (two 16-row tiles over
// the whole padded length), so each row is read from memory once per item
// and every LDS read of a frame piece feeds both row tiles (two MFMAs for
// bf16, four for fp8). The item's frame entries are staged in LDS once; its
// frame groups then stream through the two buffers run after run (across a
// run boundary comes group 0 again): while one (run, group) step is
// multiplied, the group after the next is requested into one of two register
// sets and the next one, in the other set since the step before, is written to
// the other buffer. A run's rows are requested after the last step of the run
// before; its first step is written apart so that no other step finds row
// loads in flight. An item's set-up requests its entries, then its first
// frame group, its first run and the entries' norms together; the next
// item's descriptor is requested one item ahead.
// The epilogue takes, per frame and row tile, the smallest of the tile's 16
// screen words (the block word) and stores it at the frame's block position;
// |q|^2 is added to the smallest of the lane's four rows only, and the two
// tiles share one lane swap (64 -> 40 vector instructions a step beside 16
// multiplies at 256 values).
// Measured with those, the second register set and the bank swizzle below:
// 2,048 frames on 200k x 256 bf16, every row, 361 -> 291 us (720 TFLOP/s, 37 ->
// 46 % of the matrix rate: barriers and the epilogue); 32,768 frames on 2M x 512
// 796 -> 708 (it reads 3.4 GB at 4.8 TB/s, rows once per 512 frames of a region);
// 2,048 frames on 500k x 512 137 -> 125; fp8 90 -> 77. Without the second set
// 304, 765, 131 and 77; with the request pinned to the step's start (more
// registers, a wave fewer) 315, 717, 135 and 78.
// Items are dealt to the XCDs in contiguous runs (blocks go to the eight
// XCDs round-robin): the chunks of one region, which stage the same frames,
// run on one XCD and find them in its L2.
constexpr int kRsAhead = 4;  // frame pieces in flight ahead of the multiplies

template <int FMT, int NS, int TERMS>
__global__ __launch_bounds__(256, 2) void k_screen_wide_rs(ScreenArgs a) {
  constexpr int ROWU4 = 4 * NS;                 // 16-byte pieces per row
  constexpr int FRU4 = TERMS * ROWU4;           // and per frame
  constexpr int NSF = TERMS * NS;
  // piece x of frame j lies at j * FRU4 + (x ^ j): the 16 lanes that an LDS
  // read serves at once (of lanes l: 0-3, 12-15, 20-27 and the like) then hit
  // distinct banks, where rows padded by one piece had one pair collide, four
  // cycles on each read of eight
  constexpr int TPF = 256 / kGroup;             // threads staging one frame
  static_assert(ROWU4 % TPF == 0, "whole pieces per thread");
  constexpr int PERF = FRU4 / TPF;              // pieces per thread per group
  constexpr int U = kListFrames / 256;          // item entries per thread
  extern __shared__ v4u s_fr[];                 // 2 x kGroup x FRU4
  // the item's frames: rq entries, squared norms, scales (read once per item)
  __shared__ int2 s_e[kListFrames];
  __shared__ float s_qn[kListFrames], s_qs[kListFrames];
  const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
  const int i = lane & 15, g = lane >> 4;
  const v4u *rows = static_cast<const v4u *>(a.rows_lp);
  const v4u *frames = static_cast<const v4u *>(a.q_lp);
  int lo;
  const int hi = wide_range(a, &lo);
  // this block's run of items: XCD x = b % 8 owns [x span, (x + 1) span)
  constexpr int kXcd = 8;
  const int nb = gridDim.x / kXcd, x = blockIdx.x % kXcd, jb = blockIdx.x / kXcd;
  const int span = (hi - lo + kXcd - 1) / kXcd;
  const int it0 = lo + x * span, it1 = min(hi, it0 + span);
  // staging: thread t loads pieces (t % TPF) + TPF u of frame t / TPF
  const int sj = tid / TPF, sc = tid % TPF;
  // With item counters block jb of XCD x begins with item jb of x's span; the
  // blocks then take the span's other items in order, one counter increment
  // each, then those left in the other spans (x + 1, x + 2, ... mod 8), so no
  // block idles while items remain; thread 0 takes the next item at an item's start and the block reads it after
  // the item's first barrier (two slots by item parity: the slot thread 0
  // writes was last read before the previous item's set-up barrier). Without
  // them block jb of XCD x takes items it0 + jb, + nb, ...
  const bool dyn = a.item_ctr != nullptr;
  __shared__ int s_nx[2];
  int xs = 0;  // spans thread 0 has emptied
  auto grab = [&]() -> int {
    while (xs < kXcd) {
      const int xx = x + xs < kXcd ? x + xs : x + xs - kXcd;
      const int b0 = lo + xx * span, b1 = min(hi, b0 + span);
      int32_t *ctr = a.item_ctr + xx * kItemCtrStride;
      // another XCD's span is looked at first: reads of a finished span run
      // side by side, additions would queue up
      if (xs > 0 &&
          b0 + nb + __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= b1) {
        ++xs;
        continue;
      }
      const int j = nb + atomicAdd(ctr, 1);
      if (b0 + j < b1) return b0 + j;
      ++xs;
    }
    return hi;
  };
  int it = it0 + jb, lim = it1;
  if (dyn) {
    if (it >= it1) {  // more blocks than items in this span
      if (tid == 0) s_nx[0] = grab();
      __syncthreads();
      it = s_nx[0];
    }
    lim = hi;
  }
  Item nxt = it < lim ? a.items[it] : Item{};
  for (int par = 1; it < lim; par ^= 1) {
    const Item cur = nxt;
    int itn = it + nb;
    if (dyn) {
      if (tid == 0) s_nx[par] = grab();
    } else if (itn < lim) {
      nxt = a.items[itn];
    }
    const int row_begin = cur.row_begin, block0 = cur.block, q0 = cur.q0;
    const int nrows = cur.nrows_gq >> 16, gq = cur.nrows_gq & 0xFFFF;
    const int nrun = (nrows + kWideRowsRs - 1) / kWideRowsRs;
    const int ng = (gq + kGroup - 1) / kGroup;
    v4u av[2][NS];
    float rn[2][4], rs[2][4];
    v4u pva[PERF], pvb[PERF];
    // the wave's rows of run C (clamped to the item's last row; words of rows
    // past it are no candidates), then their norms and scales
#define HLOC_RS_ROWS(C)                                                          \
  _Pragma("unroll") for (int h = 0; h < 2; ++h) {                                \
    const int rl = min((C) * kWideRowsRs + 32 * w + 16 * h + i, nrows - 1);      \
    const v4u *rp = rows + (int64_t)(row_begin + rl) * ROWU4 + g;                \
    _Pragma("unroll") for (int s = 0; s < NS; ++s) av[h][s] = rp[4 * s];         \
  }
#define HLOC_RS_NORMS(C)                                                         \
  _Pragma("unroll") for (int h = 0; h < 2; ++h) {                                \
    _Pragma("unroll") for (int r = 0; r < 4; ++r) {                              \
      const int row = (C) * kWideRowsRs + 32 * w + 16 * h + 4 * g + r;           \
      const int grow = row_begin + min(row, nrows - 1);                          \
      const float n2 = a.row_n2[grow];                                           \
      rn[h][r] = row < nrows ? n2 : __builtin_inff();                            \
      rs[h][r] = FMT == HLOC_FP8 ? a.row_scale[grow] : 1.f;                      \
    }                                                                            \
  }
#define HLOC_RS_FETCH_FRAME(PV, FR)                                              \
  {                                                                              \
    const v4u *fp = frames + (int64_t)(FR) * FRU4 + sc;                          \
    _Pragma("unroll") for (int u = 0; u < PERF; ++u) PV[u] = fp[TPF * u];        \
  }
#define HLOC_RS_STAGE(PV, BUF)                                                   \
  {                                                                              \
    _Pragma("unroll") for (int u = 0; u < PERF; ++u)                             \
        s_fr[((BUF) * kGroup + sj) * FRU4 + ((sc ^ sj) + TPF * u)] = PV[u];      \
  }
    __syncthreads();  // the previous item's entries and frames are no longer read
    if (dyn) {
      itn = s_nx[par];
      if (itn < lim) nxt = a.items[itn];
    }
    {
      // the item's frame entries (frames past gq: frame 0, never stored) and
      // the frame of this thread's piece of the first group
      const int2 ef = sj < gq ? a.rq[q0 + sj] : make_int2(0, 0);
      int2 e[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = u * 256 + tid;
        e[u] = j < gq ? a.rq[q0 + j] : make_int2(0, 0);
      }
      // the first group, the first run and the entries' norms together
      HLOC_RS_FETCH_FRAME(pva, ef.x)
      float qv[U], sv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        qv[u] = a.qn2[e[u].x];
        sv[u] = FMT == HLOC_FP8 ? a.q_scale[e[u].x] : 1.f;
      }
      HLOC_RS_ROWS(0)
      HLOC_RS_NORMS(0)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = u * 256 + tid;
        if (j < ng * kGroup) {
          s_e[j] = e[u];
          s_qn[j] = qv[u];
          s_qs[j] = sv[u];
        }
      }
      HLOC_RS_STAGE(pva, 0)
    }
    __syncthreads();
    int gn = ng > 1 ? 1 : 0;  // group of the next step
    HLOC_RS_FETCH_FRAME(pva, s_e[gn * kGroup + sj].x)
    // piece 4 s + g of the lane's frame
    int sw[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) sw[u] = (4 * u + g) ^ i;
#define HLOC_RS_PIECE(S) (sw[(S) & 3] + 16 * ((S) >> 2))
    // One (run c, group K) step. P holds the next step's group (requested a
    // step ago), Q receives the one after it; both wrap around to group 0 at
    // the run's end (past the item's last step they are not used). P is
    // staged as soon as the multiply is done, when only Q's loads are younger,
    // so nothing waits for Q.
#define HLOC_RS_STEP(K, P, Q)                                                    \
  {                                                                              \
    const int buf = st & 1;                                                      \
    gn = gn + 1 < ng ? gn + 1 : 0;                                               \
    HLOC_RS_FETCH_FRAME(Q, s_e[gn * kGroup + sj].x)                              \
    v4f acc[2] = {v4f{0.f, 0.f, 0.f, 0.f}, v4f{0.f, 0.f, 0.f, 0.f}};             \
    const v4u *bp = s_fr + (buf * kGroup + i) * FRU4;                            \
    /* frame pieces read kRsAhead steps ahead of their multiplies, the */       \
    /* order pinned: the first reads, then per k step two multiplies and */     \
    /* the next read */                                                          \
    v4u bq[NSF];                                                                 \
    _Pragma("unroll") for (int s = 0; s < kRsAhead && s < NSF; ++s) bq[s] = bp[HLOC_RS_PIECE(s)]; \
    __builtin_amdgcn_sched_group_barrier(0x100, kRsAhead < NSF ? kRsAhead : NSF, 0); \
    _Pragma("unroll") for (int s = 0; s < NSF; ++s) {                            \
      if (s + kRsAhead < NSF) bq[s + kRsAhead] = bp[HLOC_RS_PIECE(s + kRsAhead)]; \
      acc[0] = lp_mfma_v<FMT>(av[0][s % NS], bq[s], acc[0]);                     \
      acc[1] = lp_mfma_v<FMT>(av[1][s % NS], bq[s], acc[1]);                     \
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);                         \
      if (s + kRsAhead < NSF) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0); \
    }                                                                            \
    HLOC_RS_STAGE(P, buf ^ 1)                                                    \
    /* the smallest |d|^2 - 2 q.d of the lane's four rows of each tile, */       \
    /* + |q|^2, then the tiles' minima over lanes l, l ^ 16, l ^ 32, l ^ 48: */  \
    /* one swap of both tiles leaves the first in even rows of 16 lanes and */   \
    /* the second in odd ones; a tile whose rows are all marked (norm +inf) */   \
    /* has no word */                                                            \
    if ((K) == 0) {                                                              \
      _Pragma("unroll") for (int h = 0; h < 2; ++h) {                            \
        bool fin = false;                                                        \
        _Pragma("unroll") for (int r = 0; r < 4; ++r) fin |= !__builtin_isinf(rn[h][r]); \
        none[h] = __ballot(fin) == 0;                                            \
      }                                                                          \
    }                                                                            \
    const int2 e = s_e[(K) * kGroup + i];                                        \
    const float qn = s_qn[(K) * kGroup + i], qs = s_qs[(K) * kGroup + i];        \
    uint32_t wd[2];                                                              \
    _Pragma("unroll") for (int h = 0; h < 2; ++h) {                              \
      float t[4];                                                                \
      _Pragma("unroll") for (int r = 0; r < 4; ++r)                              \
          t[r] = FMT == HLOC_FP8 ? fmaf(acc[h][r] * rs[h][r], -2.f * qs, rn[h][r]) \
                                 : fmaf(acc[h][r], -2.f, rn[h][r]);              \
      const float m = fminf(fminf(t[0], t[1]), fminf(t[2], t[3])) + qn;          \
      wd[h] = none[h] ? 0xFFFFFFFFu : __float_as_uint(fmaxf(m, 0.f));            \
    }                                                                            \
    const auto p16 = __builtin_amdgcn_permlane16_swap(wd[0], wd[1], false, false); \
    const uint32_t b16 = min((uint32_t)p16[0], (uint32_t)p16[1]);                \
    const auto p32 = __builtin_amdgcn_permlane32_swap(b16, b16, false, false);   \
    const uint32_t word = min((uint32_t)p32[0], (uint32_t)p32[1]);               \
    const int row = c * kWideRowsRs + 32 * w + 16 * g; /* g < 2: the lane's tile */ \
    if ((K) * kGroup + i < gq && g < 2 && row < nrows)                           \
      a.cand[(int64_t)e.x * a.cap + e.y + block0 + (row >> 4)] = word;           \
    __syncthreads();                                                             \
    ++st;                                                                        \
  }
    int st = 0;  // steps done
    bool none[2] = {false, false};
    for (int c = 0; c < nrun; ++c) {
      // the run's first step (its multiply waits for the run's rows), written
      // apart so that no other step may find row loads in flight
      HLOC_RS_STEP(0, pva, pvb)
      int k = 1;
      for (; k + 1 < ng; k += 2) {
        HLOC_RS_STEP(k, pvb, pva)
        HLOC_RS_STEP(k + 1, pva, pvb)
      }
      if (k < ng) {
        HLOC_RS_STEP(k, pvb, pva)
      } else {
        // an odd run leaves the next group in pvb
#pragma unroll
        for (int u = 0; u < PERF; ++u) pva[u] = pvb[u];
      }
      if (c + 1 < nrun) {
        HLOC_RS_ROWS(c + 1)
        HLOC_RS_NORMS(c + 1)
      }
    }
#undef HLOC_RS_STEP
#undef HLOC_RS_PIECE
#undef HLOC_RS_ROWS
#undef HLOC_RS_NORMS
#undef HLOC_RS_FETCH_FRAME
#undef HLOC_RS_STAGE
    it = itn;
  }
}

template <int NS>
size_t wide_lp_lds_bytes() {
  return (size_t)64 * (4 * NS + 1) * sizeof(uint4);
}

constexpr size_t wide_rs_lds_bytes(int pieces) {
  return (size_t)2 * kGroup * 4 * pieces * sizeof(v4u);
}
// static LDS of the register-row kernels: the item's frames (entry, norm,
// scale of each) and two item numbers, padded to 16 bytes
constexpr size_t kRsStaticLds = kListFrames * (sizeof(int2) + 2 * sizeof(float)) + 16;
constexpr size_t kDefaultLds = 64 * 1024;
constexpr int kRsBlocksPerCu = 2;  // blocks per compute unit if the occupancy query fails

// Pieces per lane for a padded length: bf16 rows take dp / 32, fp8 rows
// dp / 64 (0: no kernel for this length).
int lp_pieces(int32_t fmt, int32_t dp) {
  const int bytes = fmt == HLOC_BF16 ? 2 * dp : fmt == HLOC_FP8 ? dp : 0;
  if (bytes <= 0 || bytes % 64 != 0) return 0;
  switch (bytes / 64) {
    case 1: case 2: case 3: case 4: case 5: case 6: case 8: case 10: case 12: case 16:
      return bytes / 64;
    default:
      return 0;
  }
}

bool lp_screen_supports(int32_t fmt, int32_t dp) { return lp_pieces(fmt, dp) > 0; }

int32_t lp_terms(int32_t fmt, int32_t dp) { return fmt == HLOC_FP8 && dp <= kFp8TermsDim ? 2 : 1; }

bool lp_wide_rs(int32_t fmt, int32_t dp) {
  const int ns = lp_pieces(fmt, dp);
  return ns > 0 && ns % 4 == 0;
}

template <int FMT, int NS, int TERMS>
hipError_t launch_rs(const ScreenArgs &a, int32_t wide_cu, hipStream_t s) {
  // as many blocks as the compute units hold at once (registers and LDS)
  constexpr size_t lds = wide_rs_lds_bytes(TERMS * NS);
  static int per_cu = 0;
  if (per_cu == 0) {
    int occ = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &occ, reinterpret_cast<const void *>(&k_screen_wide_rs<FMT, NS, TERMS>), 256, lds) !=
            hipSuccess || occ < 1) {
      (void)hipGetLastError();
      occ = kRsBlocksPerCu;
    }
    per_cu = occ;
  }
  // every block resident at once, a multiple of the eight XCDs
  const int64_t resident = std::max<int64_t>(8, (int64_t)wide_cu * per_cu / 8 * 8);
  return launch_kernel(k_screen_wide_rs<FMT, NS, TERMS>, dim3((int32_t)resident), dim3(256),
                       (uint32_t)lds, s, a);
}

template <int FMT, int NS>
hipError_t launch_lp_ns(const ScreenArgs &a, int32_t grid, int32_t wide_cu, hipStream_t s) {
  if constexpr (NS % 4 == 0) {
    if (wide_cu > 0 && !a.dense) {
      if constexpr (FMT == HLOC_FP8 && 64 * NS <= kFp8TermsDim) {
        if (a.terms == 2) return launch_rs<FMT, NS, 2>(a, wide_cu, s);
      }
      return launch_rs<FMT, NS, 1>(a, wide_cu, s);
    }
  }
  if (wide_cu > 0) {
    const int64_t resident =
        (int64_t)wide_cu * std::max<int64_t>(1, kLdsPerCu / wide_lp_lds_bytes<NS>());
    return launch_kernel(k_screen_wide_lp<FMT, NS>, dim3((int32_t)std::min<int64_t>(grid, resident)),
                         dim3(256), (uint32_t)wide_lp_lds_bytes<NS>(), s, a);
  }
  return a.dense ? launch_kernel(k_screen_lp<FMT, NS, true>, dim3(grid), dim3(256), 0, s, a)
                 : launch_kernel(k_screen_lp<FMT, NS, false>, dim3(grid), dim3(256), 0, s, a);
}

// wide_cu: compute units for the wide kernel, 0 for the narrow one
template <int FMT>
hipError_t launch_lp_fmt(const ScreenArgs &a, int32_t grid, int32_t wide_cu, hipStream_t s) {
  switch (lp_pieces(FMT, a.dp)) {
#define HLOC_LP_CASE(N) \
  case N:               \
    return launch_lp_ns<FMT, N>(a, grid, wide_cu, s);
    HLOC_LP_CASE(1)
    HLOC_LP_CASE(2)
    HLOC_LP_CASE(3)
    HLOC_LP_CASE(4)
    HLOC_LP_CASE(5)
    HLOC_LP_CASE(6)
    HLOC_LP_CASE(8)
    HLOC_LP_CASE(10)
    HLOC_LP_CASE(12)
    HLOC_LP_CASE(16)
#undef HLOC_LP_CASE
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_screen_lp(int32_t fmt, const ScreenArgs &a, int32_t grid, hipStream_t s) {
  if (grid <= 0) return hipSuccess;
  if (a.rows_per_item % 16 != 0) return hipErrorInvalidValue;
  if (fmt == HLOC_BF16) return launch_lp_fmt<HLOC_BF16>(a, grid, 0, s);
  if (fmt == HLOC_FP8) return launch_lp_fmt<HLOC_FP8>(a, grid, 0, s);
  return hipErrorInvalidValue;
}

template <int FMT>
hipError_t launch_direct_lp(const ScreenArgs &a, int32_t max_blocks, hipStream_t s) {
  const dim3 grid(direct_grid(a, max_blocks));
  switch (lp_pieces(FMT, a.dp)) {
#define HLOC_LP_CASE(N) \
  case N:               \
    return launch_kernel(k_screen_direct_lp<FMT, N>, grid, dim3(256), 0, s, a);
    HLOC_LP_CASE(1)
    HLOC_LP_CASE(2)
    HLOC_LP_CASE(3)
    HLOC_LP_CASE(4)
    HLOC_LP_CASE(5)
    HLOC_LP_CASE(6)
    HLOC_LP_CASE(8)
    HLOC_LP_CASE(10)
    HLOC_LP_CASE(12)
    HLOC_LP_CASE(16)
#undef HLOC_LP_CASE
    default:
      return hipErrorInvalidValue;
  }
}

hipError_t launch_screen_direct_lp(int32_t fmt, const ScreenArgs &a, int32_t max_blocks,
                                   hipStream_t s) {
  if (a.n_blk <= 0 || a.nq <= 0) return hipSuccess;
  if (a.splits < 1) return hipErrorInvalidValue;
  if (fmt == HLOC_BF16) return launch_direct_lp<HLOC_BF16>(a, max_blocks, s);
  if (fmt == HLOC_FP8) return launch_direct_lp<HLOC_FP8>(a, max_blocks, s);
  return hipErrorInvalidValue;
}

hipError_t launch_screen_wide_lp(int32_t fmt, const ScreenArgs &a, int32_t grid, int32_t num_cu,
                                 hipStream_t s) {
  if (grid <= 0) return hipSuccess;
  num_cu = std::max(num_cu, 1);
  if (a.rows_per_item % 16 != 0 || (a.dense && a.rows_per_item > kWideRows))
    return hipErrorInvalidValue;
  if (fmt == HLOC_BF16) return launch_lp_fmt<HLOC_BF16>(a, grid, num_cu, s);
  if (fmt == HLOC_FP8) return launch_lp_fmt<HLOC_FP8>(a, grid, num_cu, s);
  return hipErrorInvalidValue;
}

// The register-row kernel's limit, where its static LDS and its frame buffers
// pass the default (fp8 frames of 768 padded values as two vectors: 65,552 B).
template <int FMT, int NS, int TERMS>
hipError_t set_rs_lds() {
  constexpr size_t lds = wide_rs_lds_bytes(TERMS * NS);
  static_assert(lds + kRsStaticLds <= kLdsPerCu / kRsBlocksPerCu, "two blocks per compute unit");
  if (lds + kRsStaticLds <= kDefaultLds) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void *>(&k_screen_wide_rs<FMT, NS, TERMS>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}
template <int FMT, int NS>
hipError_t set_wide_lds() {
  if constexpr (NS % 4 == 0) {
    hipError_t e = set_rs_lds<FMT, NS, 1>();
    if constexpr (FMT == HLOC_FP8 && 64 * NS <= kFp8TermsDim)
      if (e == hipSuccess) e = set_rs_lds<FMT, NS, 2>();
    if (e != hipSuccess) return e;
  }
  return hipFuncSetAttribute(reinterpret_cast<const void *>(&k_screen_wide_lp<FMT, NS>),
                             hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)wide_lp_lds_bytes<NS>());
}

// LDS limits of the wide kernels (above the 64 KB default).
hipError_t prepare_screen_lp_kernels() {
#define HLOC_LP_ATTR(F, N)                   \
  {                                          \
    const hipError_t e = set_wide_lds<F, N>(); \
    if (e != hipSuccess) return e;           \
  }
#define HLOC_LP_ATTRS(F) \
  HLOC_LP_ATTR(F, 1)     \
  HLOC_LP_ATTR(F, 2)     \
  HLOC_LP_ATTR(F, 3)     \
  HLOC_LP_ATTR(F, 4)     \
  HLOC_LP_ATTR(F, 5)     \
  HLOC_LP_ATTR(F, 6)     \
  HLOC_LP_ATTR(F, 8)     \
  HLOC_LP_ATTR(F, 10)    \
  HLOC_LP_ATTR(F, 12)    \
  HLOC_LP_ATTR(F, 16)
  HLOC_LP_ATTRS(HLOC_BF16)
  HLOC_LP_ATTRS(HLOC_FP8)
#undef HLOC_LP_ATTRS
#undef HLOC_LP_ATTR
  return hipSuccess;
}

}  // namespace hloc
