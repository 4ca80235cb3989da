// Multi-frame candidate aggregation (Section 3.2, Algorithm 2), W waves per
// request, integer arithmetic throughout:
//   1. the request's frames pool their k candidates each (or the first
//      req_k[r] of them; duplicates count, padding -1 is dropped) and every
//      candidate becomes its tile key (iy, ix) from the precomputed
//      floor(coord / cell) table. The frames are req_offsets[r] ..
//      req_offsets[r+1]-1 of the batch, or, with a frame list, the batch
//      frames that list names there (sliding windows over a video share
//      frames, each retrieved once: Section 3.1);
//   2. the keys go into a hash table in LDS of at least twice as many slots,
//      which counts each distinct tile (the 2-D binning of the location
//      distribution array);
//   3. tiles rank by (count desc, iy asc, ix asc). They are taken in that
//      order, one block-wide search of the table each, for as long as the
//      tests below fail, TopC of them at most;
//   4. the tile's tolerance circle sums the counts of the tiles within rho
//      tiles (dx^2 + dy^2 <= rho^2);
//   5. the first tile with 100 * circle > pct * total wins; if none does, the
//      rank-1 tile is returned with HLOC_FLAG_LOW_CONFIDENCE.
// The estimate is the tile centre ((ix + 0.5) * cell, (iy + 0.5) * cell) with
// one rounded FP64 add and one rounded multiply, so it is reproducible bit
// for bit from the tile.
// What bounds it is the chain of dependent reads (offsets, frame list, index,
// tile) and the steps between barriers: sorting the keys, then the tiles'
// ranks, in two bitonic networks cost some 100 barriers where one or two
// searches do (246 requests of 176 candidates 16.8 -> 5.0 us, 23 of 825 that
// try every tile 39.8 -> 19.1, 4,096 of 256 52 -> 21).
#include "hloc_device.h"
#include "hloc_host.h"
#include "hloc_internal.h"

#include <algorithm>

namespace hloc {

constexpr int kAggMax = 4096;  // pooled candidates of one request
constexpr int kFlagLow = 1, kFlagEmpty = 2, kFlagBad = 4;

__device__ __forceinline__ uint32_t flip(int32_t v) { return (uint32_t)v ^ 0x80000000u; }
__device__ __forceinline__ int32_t unflip(uint32_t v) { return (int32_t)(v ^ 0x80000000u); }

constexpr int kAggSmall = 512;  // pooled candidates up to which a request takes the small kernel
constexpr int kAggWaves = 4;    // waves per request of the large kernel

// Optional frame list: request r pools batch frames frames[req_offsets[r] ..
// req_offsets[r+1]-1] (n entries). With labels > 0 the batch holds `per` frames
// once per label (frame p * per + f is frame f under label p) and a request of
// frames req_offsets[r] .. pools each under every label: entries labels *
// req_offsets[r] .. of a list (n = labels * per) whose entry labels * f + p is
// that frame. Neither: the frames themselves.
struct FrameList {
  const int32_t *frames;
  int32_t n;
  int32_t labels, per;
  __device__ __forceinline__ int limit(int nq) const { return frames || labels > 0 ? n : nq; }
  __device__ __forceinline__ int at(int i) const {
    return labels > 0 ? i % labels * per + i / labels : frames ? frames[i] : i;
  }
};

// First and last + 1 list entry of request req.
__device__ __forceinline__ int2 entries_of(const AggArgs &a, const FrameList &fl, int req) {
  const int scale = fl.labels > 0 ? fl.labels : 1;
  const int f0 = a.req_offsets ? a.req_offsets[req] : req;
  const int f1 = a.req_offsets ? a.req_offsets[req + 1] : req + 1;
  return make_int2(scale * f0, scale * f1);
}

// Pooled candidates of request req (0 for an empty or malformed request).
__device__ __forceinline__ int pooled_of(const AggArgs &a, const FrameList &fl, int req) {
  const int2 e = entries_of(a, fl, req);
  const int kr = a.req_k ? a.req_k[req] : a.k;
  if (e.x < 0 || e.y < e.x || e.y > fl.limit(a.nq) || kr < 1 || kr > a.k) return 0;
  return (int)min<int64_t>((int64_t)(e.y - e.x) * kr, (int64_t)kAggMax + 1);
}

// Slots of the table for P candidates (at least twice as many).
__host__ __device__ constexpr int agg_slots(int P) {
  int s = 64;
  while (s < 2 * P) s <<= 1;
  return s;
}
constexpr size_t agg_lds(int cap) { return (size_t)agg_slots(cap) * 12; }

// A wave's best-ranked tile, combined over the waves through LDS.
struct AggShared {
  uint64_t key[kAggWaves];
  int count[kAggWaves], circle[kAggWaves], valid[kAggWaves], used[2][kAggWaves];
};

__device__ __forceinline__ uint32_t agg_min(uint32_t v) {
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x111, 0xf, 0xf, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x112, 0xf, 0xf, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x114, 0xf, 0xf, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x118, 0xf, 0xf, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x142, 0xa, 0xf, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x143, 0xc, 0xf, false));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ int agg_sum(int v) {
  return __builtin_amdgcn_readlane(wave_incl_scan(v), 63);
}

// Ranks of tiles: more candidates first, then the smaller key.
__device__ __forceinline__ bool tile_before(int c0, uint64_t k0, int c1, uint64_t k1) {
  return c0 > c1 || (c0 == c1 && k0 < k1);
}

// Algorithm 2 for one request of at most CAP candidates (or a malformed one),
// by W waves; key / count hold agg_slots(CAP) entries.
template <int CAP, int W>
__device__ void aggregate_one(const AggArgs &a, const FrameList &fl, int req, uint64_t *key, int *count,
                              AggShared &sh) {
  constexpr int kThreads = 64 * W;
  const int tid = threadIdx.x, lane = lane_id(), w = W == 1 ? 0 : wave_id();
  auto sync = [&]() {
    if (W == 1) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
      __syncthreads();
    }
  };
  const int2 ent = entries_of(a, fl, req);
  const int f0 = ent.x, f1 = ent.y;
  const int kr = a.req_k ? a.req_k[req] : a.k;  // candidates pooled per frame
  auto none = [&](int flag) {
    if (tid == 0) {
      a.tile[2 * req] = 0;
      a.tile[2 * req + 1] = 0;
      a.xy[2 * req] = __builtin_nan("");
      a.xy[2 * req + 1] = __builtin_nan("");
      a.flags[req] = flag;
    }
  };
  if (f0 < 0 || f1 < f0 || f1 > fl.limit(a.nq) || kr < 1 || kr > a.k ||
      (int64_t)(f1 - f0) * kr > (int64_t)CAP) {
    none(kFlagBad);
    return;
  }
  const int P = (f1 - f0) * kr, S = agg_slots(P);
  for (int s = tid; s < S; s += kThreads) {
    key[s] = kKeyNone;
    count[s] = 0;
  }
  sync();
  // candidates into the table (linear probing; it never fills up); valid
  // counts them, or is negative if a listed frame is not one of the batch
  int valid = 0;
  bool bad = false;
  constexpr int U = 4;  // candidates per thread whose dependent reads run side by side
  for (int p0 = tid; p0 < P; p0 += U * kThreads) {
    int frame[U], at[U];
    int64_t j[U];
    int2 t[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = min(p0 + u * kThreads, P - 1), fr = p / kr;
      at[u] = p - fr * kr;
      frame[u] = fl.at(f0 + fr);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool ok = frame[u] >= 0 && frame[u] < a.nq;
      bad |= !ok;
      j[u] = ok && p0 + u * kThreads < P ? a.idx[(int64_t)frame[u] * a.k + at[u]] : -1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) t[u] = a.tile_of[j[u] < 0 ? 0 : j[u]];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (j[u] < 0) continue;
      const uint64_t k = ((uint64_t)flip(t[u].y) << 32) | flip(t[u].x);
      uint32_t s = ((uint32_t)t[u].x * 0x9E3779B1u ^ (uint32_t)t[u].y * 0x85EBCA77u);
      s = (s ^ (s >> 15)) & (uint32_t)(S - 1);
      for (;;) {
        const uint64_t old =
            atomicCAS(reinterpret_cast<unsigned long long *>(&key[s]), kKeyNone, k);
        if (old == kKeyNone || old == k) break;
        s = (s + 1) & (uint32_t)(S - 1);
      }
      atomicAdd(&count[s], 1);
      ++valid;
    }
  }
  valid = __ballot(bad) ? -(1 << 20) : agg_sum(valid);
  if (W > 1 && lane == 0) sh.valid[w] = valid;
  sync();
  int total = valid;
  if (W > 1) {
    total = 0;
    for (int i = 0; i < W; ++i) total += sh.valid[i];
  }
  if (total <= 0) {
    none(total < 0 ? kFlagBad : kFlagEmpty);
    return;
  }
  // the used slots to the front (a slot never moves up: the slots read in a
  // step are written after its barrier), so that the searches read only them
  int T = 0;
  for (int s0 = 0, par = 0; s0 < S; s0 += kThreads, par ^= 1) {
    const int s = s0 + tid;
    const int n = s < S ? count[s] : 0;
    const uint64_t k = s < S ? key[s] : kKeyNone;
    const uint64_t bal = __ballot(n > 0);
    if (W > 1 && lane == 0) sh.used[par][w] = __popcll(bal);
    sync();
    int at = T + __popcll(bal & ((1ull << lane) - 1ull));
    if (W > 1) {
      for (int i = 0; i < W; ++i) {
        if (i < w) at += sh.used[par][i];
        T += sh.used[par][i];
      }
    } else {
      T += __popcll(bal);
    }
    if (n > 0) {
      key[at] = k;
      count[at] = n;
    }
  }
  sync();
  const int64_t rho = a.rho, rho2 = rho * rho;
  int pc = INT32_MAX, flag = kFlagLow;  // the previous tile: count, key
  uint64_t pk = 0, chosen = 0;
  for (int c = 0; c < a.top_c; ++c) {
    // the best-ranked tile after the previous one
    int bc = 0;
    uint64_t bk = kKeyNone;
    for (int s = tid; s < T; s += kThreads) {
      const int n = count[s];
      const uint64_t k = key[s];
      if (tile_before(pc, pk, n, k) && tile_before(n, k, bc, bk)) {
        bc = n;
        bk = k;
      }
    }
    const int mc = kAggMax - (int)agg_min((uint32_t)(kAggMax - bc));
    bool in = bc == mc && mc > 0;
    const uint32_t hi = agg_min(in ? (uint32_t)(bk >> 32) : 0xFFFFFFFFu);
    in = in && (uint32_t)(bk >> 32) == hi;
    const uint32_t lo = agg_min(in ? (uint32_t)bk : 0xFFFFFFFFu);
    int tc = mc;
    uint64_t tk = ((uint64_t)hi << 32) | lo;
    if (W > 1) {
      if (lane == 0) {
        sh.count[w] = tc;
        sh.key[w] = tk;
      }
      sync();
      for (int i = 0; i < W; ++i) {
        if (tile_before(sh.count[i], sh.key[i], tc, tk)) {
          tc = sh.count[i];
          tk = sh.key[i];
        }
      }
    }
    if (tc <= 0) break;  // fewer tiles than TopC
    if (c == 0) chosen = tk;
    // its tolerance circle
    int circle = 0;
    const int64_t cx = unflip((uint32_t)tk), cy = unflip((uint32_t)(tk >> 32));
    for (int s = tid; s < T; s += kThreads) {
      const int n = count[s];
      const uint64_t k = key[s];
      const int64_t dx = unflip((uint32_t)k) - cx, dy = unflip((uint32_t)(k >> 32)) - cy;
      if (dx <= rho && dx >= -rho && dy <= rho && dy >= -rho && dx * dx + dy * dy <= rho2)
        circle += n;
    }
    circle = agg_sum(circle);
    if (W > 1) {
      if (lane == 0) sh.circle[w] = circle;
      sync();
      circle = 0;
      for (int i = 0; i < W; ++i) circle += sh.circle[i];
    }
    if ((int64_t)100 * circle > (int64_t)a.toler_pct * total) {
      chosen = tk;
      flag = 0;
      break;
    }
    pc = tc;
    pk = tk;
  }
  if (tid == 0) {
    const int32_t ix = unflip((uint32_t)chosen), iy = unflip((uint32_t)(chosen >> 32));
    a.tile[2 * req] = ix;
    a.tile[2 * req + 1] = iy;
    a.xy[2 * req] = __dmul_rn(__dadd_rn((double)ix, 0.5), a.cell);
    a.xy[2 * req + 1] = __dmul_rn(__dadd_rn((double)iy, 0.5), a.cell);
    a.flags[req] = flag;
  }
}

// One wave per request. Requests pooling more than kAggSmall candidates (up to
// kAggMax) are listed for k_aggregate_big instead: the small table lets many
// waves share a compute unit.
__global__ __launch_bounds__(64) void k_aggregate(AggArgs a, FrameList fl) {
  __shared__ uint64_t key[agg_slots(kAggSmall)];
  __shared__ int count[agg_slots(kAggSmall)];
  __shared__ AggShared sh;
  const int req = blockIdx.x;
  if (req >= a.nreq) return;
  const int P = pooled_of(a, fl, req);
  if (P > kAggSmall && P <= kAggMax) {
    if (threadIdx.x == 0) a.big_list[atomicAdd(a.big_count, 1)] = req;
    return;
  }
  aggregate_one<kAggSmall, 1>(a, fl, req, key, count, sh);
}

// The listed requests, a persistent grid over them; without a list, request
// blockIdx.x (every request of a batch that fits one round of blocks).
__global__ __launch_bounds__(64 * kAggWaves) void k_aggregate_big(AggArgs a, FrameList fl) {
  extern __shared__ uint64_t lds_big[];
  __shared__ AggShared sh;
  int *count = reinterpret_cast<int *>(lds_big + agg_slots(kAggMax));
  if (!a.big_list) {
    if ((int)blockIdx.x < a.nreq)
      aggregate_one<kAggMax, kAggWaves>(a, fl, blockIdx.x, lds_big, count, sh);
    return;
  }
  const int n = *a.big_count;
  for (int i = blockIdx.x; i < n; i += gridDim.x) {
    __syncthreads();  // the previous request's table is no longer read
    aggregate_one<kAggMax, kAggWaves>(a, fl, a.big_list[i], lds_big, count, sh);
  }
}

constexpr size_t kAggLds = agg_lds(kAggMax);
static_assert(kAggLds + sizeof(AggShared) <= (size_t)kLdsPerCu, "aggregation table above 160 KB");

// LDS limit of the aggregation kernel, set once per device.
hipError_t prepare_aggregate_kernels() {
  static int done_dev = -1;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || done_dev == dev) return e;
  e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_aggregate_big),
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)kAggLds);
  if (e == hipSuccess) done_dev = dev;
  return e;
}

static hipError_t launch_listed(const AggArgs &a, const FrameList &fl, hipStream_t s) {
  if (a.nreq <= 0) return hipSuccess;
  if (a.top_c < 1 || a.top_c > 64) return hipErrorInvalidValue;
  const int32_t cus = std::max(a.num_cu, 1);
  if (a.nreq <= cus) {
    // one round of blocks: a single launch with the large lists
    AggArgs b = a;
    b.big_list = nullptr;
    return launch_kernel(k_aggregate_big, dim3(a.nreq), dim3(64 * kAggWaves), kAggLds, s, b, fl);
  }
  hipError_t e = launch_kernel(k_aggregate, dim3(a.nreq), dim3(64), 0, s, a, fl);
  if (e != hipSuccess) return e;
  // one resident block per compute unit at most (the table takes 98 KB of LDS)
  return launch_kernel(k_aggregate_big, dim3(cus), dim3(64 * kAggWaves), kAggLds, s, a, fl);
}

hipError_t launch_aggregate_frames(const AggArgs &a, const int32_t *frames, int32_t n_frames,
                                   hipStream_t s) {
  return launch_listed(a, FrameList{frames, frames ? n_frames : 0, 0, 0}, s);
}

hipError_t launch_aggregate_labels(const AggArgs &a, int32_t labels, int32_t per, hipStream_t s) {
  return launch_listed(a, FrameList{nullptr, labels * per, labels, per}, s);
}

}  // namespace hloc
