// Scheduling of the fine screen of large batches: the frame -> regions lists
// chosen by the coarse stage are inverted into region -> frames lists (the
// coarse selection has counted each region's frames and given each frame its
// place among them), and every touched
// region is cut into chunks of T rows (for wide regions W rows, or a few runs
// of W rows) crossed with groups of up to kListFrames frames. This takes the place of the paper's
// one-stream-per-subspace launch (Section 3.1): uneven regions become many
// equal-sized work items for persistent screen kernels, and every count lives
// in device memory (no host round trip).
//
// Items come in two classes. A region kept by at most kGroup frames gives
// narrow items (one MFMA column block of frames); a region kept by more
// frames gives wide items of up to kListFrames frames, screened by a kernel
// that reads each row once for all of them. Narrow items are numbered first:
// items [0, n_items[4]) are narrow, [n_items[4], n_items[0]) wide. Regions
// are laid out in that order (narrow regions by id, then wide regions by id)
// in vord, with their first item in iof (non-decreasing), so the owner of an
// item is found by binary search.
#include "hloc_device.h"
#include "hloc_internal.h"

#include <algorithm>

namespace hloc {

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int grid = (int)std::min<int64_t>((n + 255) / 256, 4096);
  return launch_kernel(k_fill_i32, dim3(grid), dim3(256), 0, s, p, n, v);
}

// Slot owning work item t: the last k with iof[k] <= t, for non-decreasing
// iof with iof[0] = 0 <= t < iof[R]; that slot has at least one item.
__device__ __forceinline__ int owner_slot(const int32_t *iof, int R, int t) {
  int lo = 0, hi = R;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (iof[mid] <= t) lo = mid;
    else hi = mid;
  }
  return lo;
}

// How a region of `rows` rows kept by g frames is cut into items: chunks of
// rows, each against runs of frames.
struct Cut {
  int rows, frames, nrun;
};

// Narrow regions: chunks of T rows, one run of frames. Wide regions: the unit
// of work is a step, W rows against c.gu groups of kGroup frames; an item aims
// at `target` of them, first by its frames (their rows are read again for
// every further run), then, with WM > 1 (the register-row kernels take such
// an item W rows at a time with its frames staged once), by up to WM runs of
// W rows, so that items of few frames still hide their set-up.
// (Not inlined, here and below: one block runs this code once, and its
// instruction fetches cost more than the calls.)
__device__ __noinline__ Cut cut_region(int g, SchedCut c, int target) {
  Cut k;
  k.rows = c.T;
  k.frames = kListFrames;
  k.nrun = 1;
  if (g <= kGroup) return k;
  const int most = kListFrames / kGroup;
  const int groups = (g + kGroup - 1) / kGroup;
  int gi = target >= c.max_steps ? most : min(most, target << c.log_gu);
  if (groups > gi) {
    // even runs of whole units
    k.nrun = (groups + gi - 1) / gi;
    gi = min(most, ((groups + k.nrun - 1) / k.nrun + (1 << c.log_gu) - 1) >> c.log_gu << c.log_gu);
    k.nrun = (groups + gi - 1) / gi;
  }
  k.frames = gi * kGroup;
  const int steps = (min(groups, gi) + (1 << c.log_gu) - 1) >> c.log_gu;
  k.rows = c.W * max(1, min(c.WM, (min(target, c.max_steps) + steps - 1) / steps));
  return k;
}

__device__ __forceinline__ int items_of(int g, int rows, const SchedCut &c, int target) {
  if (g <= 0) return 0;
  const Cut k = cut_region(g, c, target);
  return (rows + k.rows - 1) / k.rows * k.nrun;
}

// Work item t of a region whose rows are [r0, r0 + rows) and whose frames are
// rq[q_begin, q_end): chunk-major, frame runs inner, so consecutive items
// re-read the same rows.
// Its first row is block blk0 of the lists that the rq entries point into.
__device__ __forceinline__ Item make_item(int t, int item_begin, int q_begin, int q_end, int blk0,
                                          int r0, int rows, const SchedCut &sc, int target) {
  const int g = q_end - q_begin;
  const Cut k = cut_region(g, sc, target);
  const int local = t - item_begin, c = local / k.nrun, b = local - c * k.nrun;
  Item it;
  it.row_begin = r0 + c * k.rows;
  it.block = blk0 + c * (k.rows / kBlockRows);
  it.q0 = q_begin + b * k.frames;
  it.nrows_gq = (min(k.rows, rows - c * k.rows) << 16) | min(k.frames, g - b * k.frames);
  return it;
}

// Block-wide (blockDim.x <= 1024) scans over the regions, each thread taking a
// contiguous range of them: rq_off (R + 1, first frame of each region in id
// order; with `all` > 0, where every region is kept by `all` frames, its first
// 16-row block instead), vord / iof (the regions in narrow-then-wide order and
// their first item), n_items[0] (all items), n_items[4] (narrow items) and
// n_items[5] (the step target of the wide items).
// reg_start: first row of each region (R + 1 entries).
//
// Step target: S steps over all wide regions make items of c.steps_scale S
// (about two for each block that runs at once, to balance with), up to
// max_steps, where a longer item gains nothing more. Items used to be cut for
// max_steps whatever S: a batch of 2,048 frames on 500k x 512 bf16 rows then
// had 408 wide items for 512 blocks, and the longest set the launch's time;
// with this cut (and item counters on lines of their own) the launch takes
// 105 us instead of 169, 67 instead of 134 on fp8 rows (2,048 frames of 256
// requests), and 256 frames of one video on 200k x 256 fp32 rows (18 regions
// kept by all) 10.5 instead of 30. The host sizes the item buffer for the cut
// at max_steps (c.max_items): a finer cut that does not fit falls back to it.
__global__ __launch_bounds__(1024) void k_sched_scan(const int32_t *__restrict__ count, int all_fr,
                                                     int R, const int64_t *__restrict__ reg_start,
                                                     SchedCut c, int32_t *rq_off, int32_t *vord,
                                                     int32_t *iof, int32_t *n_items) {
  __shared__ int s_red[80];
  const int tid = threadIdx.x, nt = blockDim.x;
  const int per = (R + nt - 1) / nt;
  const int r0 = min(R, tid * per), r1 = min(R, r0 + per);
  const int lane = tid & 63, wv = tid >> 6, nw = nt >> 6;
  // first the cut at max_steps, with the sum of the steps beside it; if that
  // asks for shorter items, the cut again
  int target = c.max_steps;
  int v[4], inc[4], all[4];
#pragma unroll 1
  for (int pass = 0;; ++pass) {
    // frames, narrow items, wide items, narrow regions
    v[0] = v[1] = v[2] = v[3] = 0;
    float steps = 0.f;  // (an estimate is enough: the cut never changes a result)
#pragma unroll 1
    for (int r = r0; r < r1; ++r) {
      const int rows = (int)(reg_start[r + 1] - reg_start[r]);
      const int g = all_fr ? all_fr : count[r];
      const int m = items_of(g, rows, c, target);
      v[0] += all_fr ? (rows + kBlockRows - 1) / kBlockRows : g;
      if (g <= kGroup) {
        v[1] += m;
        v[3] += 1;
      } else {
        v[2] += m;
        steps += (float)(rows + c.W - 1) * (float)((g + kGroup - 1) / kGroup + (1 << c.log_gu) - 1);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) inc[q] = wave_incl_scan(v[q]);
    steps = wave_incl_scan_f32(steps);
    if (lane == 63) {
#pragma unroll
      for (int q = 0; q < 4; ++q) s_red[q * 16 + wv] = inc[q];
      s_red[64 + wv] = __float_as_int(steps);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) inc[q] += waves_before(s_red + q * 16, wv, nw, &all[q]);
    steps = lane < nw ? __int_as_float(s_red[64 + lane]) : 0.f;
    steps = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_incl_scan_f32(steps)), 63));
    // (uniform from here on)
    const bool fits = all[1] + all[2] <= c.max_items;
    if (pass == 0 && all[2] > 0) {
      target = (int)fminf(fmaxf(steps * c.steps_scale, 1.f), (float)c.max_steps);
      if (target >= c.max_steps) break;
    } else if (pass != 1 || fits) {
      break;
    } else {
      target = c.max_steps;
    }
    __syncthreads();
  }
  const int BN = all[1], CN = all[3];
  int pa = inc[0] - v[0], pbn = inc[1] - v[1], pbw = inc[2] - v[2], pcn = inc[3] - v[3];
#pragma unroll 1
  for (int r = r0; r < r1; ++r) {
    const int rows = (int)(reg_start[r + 1] - reg_start[r]);
    const int g = all_fr ? all_fr : count[r];
    const int m = items_of(g, rows, c, target);
    rq_off[r] = pa;
    pa += all_fr ? (rows + kBlockRows - 1) / kBlockRows : g;
    int pos;
    if (g <= kGroup) {
      pos = pcn;
      iof[pos] = pbn;
      pbn += m;
      pcn += 1;
    } else {
      pos = CN + (r - pcn);  // wide regions before r: r minus the narrow ones
      iof[pos] = BN + pbw;
      pbw += m;
    }
    vord[pos] = r;
  }
  if (tid == nt - 1) {
    rq_off[R] = inc[0];
    iof[R] = inc[1] + inc[2];
    n_items[0] = inc[1] + inc[2];
    n_items[4] = inc[1];
    n_items[5] = target;
  }
}

// The first pair_blocks blocks: one thread per (frame, region) pair puts it at
// its place in the region's frame list (all: every frame is in every list, so
// one list of them serves all regions). The others: one thread per work item
// (grid-stride), each finding its region by binary search, so that a region
// kept by many frames is expanded by many threads.
__global__ void k_sched_place(const int32_t *__restrict__ regions, int nq, int nr, int all, int R,
                              const int32_t *__restrict__ place, const int32_t *__restrict__ off,
                              const int32_t *__restrict__ vord, const int32_t *__restrict__ iof,
                              const int32_t *__restrict__ rq_off,
                              const int64_t *__restrict__ reg_start, SchedCut sc,
                              const int32_t *__restrict__ n_items, int pair_blocks, int2 *rq,
                              Item *items) {
  if ((int)blockIdx.x < pair_blocks) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (all) {
      if (t < nq) rq[t] = make_int2((int)t, 0);
    } else if (t < (int64_t)nq * nr) {
      const int r = regions[t];
      if (r >= 0 && r < R) rq[rq_off[r] + place[t]] = make_int2((int)(t / nr), off[t]);
    }
    return;
  }
  const int n = iof[R], target = n_items[5];
  for (int t = (blockIdx.x - pair_blocks) * blockDim.x + threadIdx.x; t < n;
       t += (gridDim.x - pair_blocks) * blockDim.x) {
    const int k = owner_slot(iof, R, t);
    const int r = vord[k];
    const int64_t r0 = reg_start[r];
    const int q0 = all ? 0 : rq_off[r], q1 = all ? nq : rq_off[r + 1];
    items[t] = make_item(t, iof[k], q0, q1, all ? rq_off[r] : 0, (int)r0,
                         (int)(reg_start[r + 1] - r0), sc, target);
  }
}

// Two launches: the scan needs every region's count, the placing the scan.
// (Counting and ranking the frames per region in kernels of their own, and for
// the exhaustive search writing out every region's list of all frames, took
// four launches more and 75 us of a 705 us pass over 2,048 frames x 200k rows.)
hipError_t launch_sched(const int32_t *regions, int32_t nq, int32_t nr, int32_t R,
                        const int64_t *reg_start, const SchedCut &sc, const int32_t *rcount,
                        const int32_t *place, const int32_t *off, int32_t *vord, int32_t *rq_off,
                        int32_t *item_off, int32_t *n_items, int2 *rq, Item *items,
                        hipStream_t s) {
  if (nq <= 0) return hipSuccess;
  const int all = rcount ? 0 : nq;
  const hipError_t e = launch_kernel(k_sched_scan, dim3(1), dim3(1024), 0, s, rcount, all, R,
                                     reg_start, sc, rq_off, vord, item_off, n_items);
  if (e != hipSuccess) return e;
  const int64_t pairs = all ? nq : (int64_t)nq * nr;
  const int pair_blocks = (int)((pairs + 255) / 256);
  const int item_blocks = (int)std::min<int64_t>(1024, ((int64_t)sc.max_items + 255) / 256);
  return launch_kernel(k_sched_place, dim3(pair_blocks + std::max(item_blocks, 1)), dim3(256), 0,
                       s, regions, nq, nr, all, R, place, off, vord, item_off, rq_off, reg_start,
                       sc, n_items, pair_blocks, rq, items);
}

}  // namespace hloc
