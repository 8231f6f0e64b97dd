// Host-side helpers shared by the C-ABI entry points (not part of the ABI).
#pragma once

#include <cstring>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <string>
#include <vector>

#include "bip_internal.h"

namespace bip {

inline int64_t roundup(int64_t a, int64_t b) { return (a + b - 1) / b * b; }

inline int err(int code, const std::string& msg) {
  set_error(msg);
  return code;
}

#define HIPCHK(expr, what)                         \
  do {                                             \
    hipError_t e_ = (expr);                        \
    if (e_ != hipSuccess) return hip_fail(e_, what); \
  } while (0)

inline hipEvent_t take_event(bip_plan* p) {
  if (!p->event_pool.empty()) {
    hipEvent_t e = p->event_pool.back();
    p->event_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

// Run `launch` on stream `st`; when profiling, bracket it with events.
template <typename F>
hipError_t timed(bip_plan* p, int stage, hipStream_t st, F&& launch) {
  if (!p->profiling) return launch();
  hipEvent_t a = take_event(p), b = take_event(p);
  if (!a || !b) return hipErrorOutOfMemory;
  hipError_t e = hipEventRecord(a, st);
  if (e == hipSuccess) e = launch();
  if (e == hipSuccess) e = hipEventRecord(b, st);
  p->timed.push_back({stage, a, b});
  return e;
}

// One device block from the caller's allocator, or stream-ordered from the
// HIP pool when there is none.
inline void* raw_alloc(const bip_alloc* al, size_t bytes, hipStream_t s) {
  if (al && al->alloc) return al->alloc(bytes, (void*)s, al->ctx);
  void* ptr = nullptr;
  if (hipMallocAsync(&ptr, bytes, s) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  return ptr;
}
inline void raw_release(const bip_alloc* al, void* ptr, size_t bytes, hipStream_t s) {
  if (!ptr) return;
  if (al && al->release) al->release(ptr, bytes, (void*)s, al->ctx);
  else (void)hipFreeAsync(ptr, s);
}

// Tables of a call that lie in one device block (from `base`): gathered on the
// host and copied at once.  Every copy from pageable memory costs the host a
// staging round of its own, 2.4 us (a map of one atom took 210 us with six copies,
// 197 with one).  The host block outlives the call.
class TableCopy {
 public:
  TableCopy(std::vector<char>& host, void* base) : host_(host), base_((char*)base) { host_.clear(); }
  template <typename T>
  void add(const T* dst, const std::vector<T>& v) {
    const size_t at = (const char*)dst - base_, n = v.size() * sizeof(T);
    if (n == 0) return;
    if (host_.size() < at + n) host_.resize(at + n);
    std::memcpy(host_.data() + at, v.data(), n);
  }
  hipError_t copy(hipStream_t s) const {
    return host_.empty() ? hipSuccess : hipMemcpyAsync(base_, host_.data(), host_.size(), hipMemcpyHostToDevice, s);
  }

 private:
  std::vector<char>& host_;
  char* base_;
};

inline const bip_alloc* plan_alloc(const bip_plan* p) { return p->has_alloc ? &p->alloc : nullptr; }

// A block owned by the plan until bip_plan_destroy; null when the device has no room for it.
inline void* take_block(bip_plan* p, size_t bytes, hipStream_t s) {
  void* ptr = raw_alloc(plan_alloc(p), bytes, s);
  if (!ptr) return nullptr;
  p->allocations.push_back({ptr, bytes});
  p->bytes_now += (int64_t)bytes;
  p->bytes_peak = std::max(p->bytes_peak, p->bytes_now);
  return ptr;
}
inline int no_room(size_t bytes) {
  return err(BIP_ENOMEM, "device allocation of " + std::to_string(bytes) + " bytes failed");
}
inline int plan_block(bip_plan* p, void** out, size_t bytes, hipStream_t s) {
  *out = take_block(p, bytes, s);
  return *out ? BIP_OK : no_room(bytes);
}
inline void plan_release(bip_plan* p, void* ptr, hipStream_t s) {
  for (size_t i = 0; i < p->allocations.size(); ++i)
    if (p->allocations[i].ptr == ptr) {
      raw_release(plan_alloc(p), ptr, p->allocations[i].bytes, s);
      p->bytes_now -= (int64_t)p->allocations[i].bytes;
      p->allocations.erase(p->allocations.begin() + i);
      return;
    }
}

template <typename T>
int dalloc(bip_plan* p, T** out, size_t count, hipStream_t s) {
  *out = nullptr;
  if (count == 0) return BIP_OK;
  void* ptr = nullptr;
  int rc = plan_block(p, &ptr, count * sizeof(T), s);
  *out = (T*)ptr;
  return rc;
}

// Copy a host table into a new plan block.  The source must stay alive until
// the stream has passed the copy.
template <typename T>
int upload(bip_plan* p, T** out, const std::vector<T>& v, hipStream_t s) {
  int rc = dalloc(p, out, v.size(), s);
  if (rc) return rc;
  if (!v.empty()) HIPCHK(hipMemcpyAsync(*out, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, s), "upload");
  return BIP_OK;
}

struct Workspace {
  char* base = nullptr;
  size_t used = 0;
  void* take(size_t bytes) {
    void* p = base + used;
    used += roundup((int64_t)bytes, 256);
    return p;
  }
};

// Grow the plan's workspace to `bytes`; false when the device has no room.  The
// old block is released in stream order, so no synchronization is needed.
inline bool grow_work(bip_plan* p, size_t bytes, hipStream_t s) {
  if (p->work_bytes >= bytes) return true;
  if (p->d_work) {
    plan_release(p, p->d_work, s);
    p->d_work = nullptr;
    p->work_bytes = 0;
  }
  p->d_work = take_block(p, bytes, s);
  if (!p->d_work) return false;
  p->work_bytes = bytes;
  return true;
}
inline int ensure_work(bip_plan* p, size_t bytes, hipStream_t s) {
  return grow_work(p, bytes, s) ? BIP_OK : no_room(bytes);
}

// Largest parent-column batch of a sweep: BIP_COLUMN_BATCH if set (0 = all
// columns), else as many as fit in kColumnBatchBytes of state (224 MiB: a
// batch and what the passes read besides stay inside the 256 MB Infinity
// Cache.  On 50 slices of 256 x 256 with 447 + 2233 columns, batches of at most
// 96, 144, 192, 224, 256 and 320 MiB: 56.5, 52.2, 50.8, 49.7, 49.3 and 53.8 ms).
constexpr int64_t kColumnBatchBytes = (int64_t)224 << 20;
inline int column_batch(int64_t G) {
  const char* env = std::getenv("BIP_COLUMN_BATCH");
  int64_t b = env ? std::atoll(env) : kColumnBatchBytes / (G * 8);
  if (b <= 0) b = INT32_MAX;
  return (int)std::min<int64_t>(b, INT32_MAX);
}
// Split precision runs the Gram matrix on single FP16 products when its sum
// runs over at least this many detector beams: the FP16 rounding of the
// operand (2^-11) then averages to well under the 1e-4 target (measured
// 5e-6 at 32,417 beams); smaller detectors keep the hi+lo BF16 products.
constexpr int kGramFp16MinBeams = 4096;
inline int gram_precision(int precision, int ndet) {
  return precision == BIP_PREC_SPLIT_BF16 && ndet >= kGramFp16MinBeams ? BIP_PREC_FP16 : precision;
}

// The batch actually used for a sweep over n columns: the fewest batches of
// at most cap columns, of equal size (the last one at most a column short).
inline int balanced_batch(int n, int cap) {
  if (n <= 0) return 1;
  const int64_t nb = ((int64_t)n + cap - 1) / cap;
  return (int)((n + nb - 1) / nb);
}

// Most a launch may add to the workspace for partial products of split
// contractions, within what a budget that the caller set leaves of it and while
// the device has room; without it they run whole.
constexpr int64_t kSplitBytes = (int64_t)512 << 20;

// Plans that keep checkpoints differentiate the map: their contractions run
// whole (no K segments, every tile of a diagonal block), in the job groups of
// quad_groups, so that a gradient does not move with the splits chosen below.
// (A tile below the diagonal taken as the conjugate transpose of the one above
// would add its two imaginary products in the other order.)  Maps of plans with
// and without checkpoints therefore agree to rounding only.
inline bool fixed_order(const bip_plan* p) { return p->o.ckpt_stride > 0; }

// Job groups of the quadratic form without K segments: qt tiles of 128 x 128 x
// z groups run in ceil(qt z / n_cu) rounds of ceil(nat / z) jobs per
// workgroup: take the z with the fewest job-rounds, the smallest on ties
// (fewer partial rows to reduce).
inline int quad_groups(int64_t qt, int nat, int n_cu) {
  int best = 1;
  int64_t cost = INT64_MAX;
  for (int z = 1; z <= std::min(GEMM_MAX_ZSPLIT, nat); ++z) {
    const int64_t c = (qt * z + n_cu - 1) / n_cu * ((nat + z - 1) / z);
    if (c < cost) {
      cost = c;
      best = z;
    }
  }
  return best;
}

// Job groups (z) and K segments (k) of the quadratic form, at most GEMM_MAX_ZSPLIT
// partial rows.  The workgroups (mt row tiles x nt column tiles x z k) go to the
// CUs as these come free, the column tiles in order: tile y runs the K chunks from
// its own column on (per_tile of them a tile), so the first tiles are the longest.
// A job costs a workgroup its chunks and about kQuadFill chunk times of filling and
// epilogue (psi staging).  Modelled time: the longest workgroup where every CU gets
// one at most; else the work of a CU and, for the uneven end, half the longest.
// The smallest split within a hundredth of the best (fewer rows to reduce).
//   Counted as if every tile ran all chunks, 24 windows of 32 x 32 against 4096 scans
// took one group, each CU one workgroup of its own length: 2.08 ms, 1.44 so; 112 windows
// of 24 x 24 8 groups: 2.37 and 2.27.
constexpr double kQuadFill = 6.0;
inline void quad_split(int64_t mt, int64_t nt, int per_tile, int nat, int chunks, int64_t n_cu, int& z_out, int& k_out) {
  z_out = k_out = 1;
  double cost = 1e300;
  for (int z = 1; z <= std::min(GEMM_MAX_ZSPLIT, nat); ++z)
    for (int k = 1; z * k <= GEMM_MAX_ZSPLIT && k <= std::max(1, chunks / 2); ++k) {
      const int seg = (chunks + k - 1) / k;
      const double longest = (double)((nat + z - 1) / z) * (seg + kQuadFill);
      double work = 0;
      for (int64_t y = 0; y < nt; ++y) {
        const int64_t mine = std::max<int64_t>(0, chunks - y * per_tile);
        work += (double)mine + kQuadFill * (double)((mine + seg - 1) / seg);
      }
      work *= (double)mt * nat / n_cu;
      const double c = mt * nt * z * k <= n_cu ? longest : std::max(longest, work + 0.5 * longest);
      if (c < 0.99 * cost) {
        z_out = z;
        k_out = k;
        cost = c;
      }
    }
}

// Job groups of the per-beam products: tiles x z workgroups, ceil(tiles z /
// n_cu) of them per CU, of ceil(njobs / z) jobs each.  More than one group costs a slice of
// the output each, written and summed: only for a gain above a tenth, and only
// while the slices fit in max_z.
inline int abs2_groups(int64_t tiles, int njobs, int64_t n_cu, int64_t max_z) {
  int best = 1;
  double cost = 1e300;
  for (int z = 1; z <= std::min<int64_t>({GEMM_MAX_ZSPLIT, njobs, std::max<int64_t>(1, max_z)}); ++z) {
    const double c = (double)((tiles * z + n_cu - 1) / n_cu) * (double)((njobs + z - 1) / z);
    if (c < 0.9 * cost) {
      best = z;
      cost = c;
    }
  }
  return best;
}

inline GatherArgs gather_args(const bip_plan* p, int side) {
  GatherArgs g;
  g.rec = side == 1 ? p->d_grec1 : p->d_grec2;
  g.win = side == 1 ? p->d_win1 : p->d_win2;
  return g;
}

inline ReconArgs recon_args(const bip_plan* p, int a, int side) {
  ReconArgs r;
  r.win = (side == 1 ? p->d_win1 + p->off1[a] : p->d_win2 + p->off2[a]);
  r.rowptr = side == 1 ? p->d_rp1 : p->d_rp2;
  r.col = side == 1 ? p->d_col1 : p->d_col2;
  r.w = side == 1 ? p->d_w1 : p->d_w2;
  r.ellc = side == 1 ? p->d_ellc1 : p->d_ellc2;
  r.ellw = side == 1 ? p->d_ellw1 : p->d_ellw2;
  r.tstart = side == 1 ? p->d_tstart1 : p->d_tstart2;
  r.tpar = side == 1 ? p->d_tpar1 : p->d_tpar2;
  r.ell_loc = side == 1 ? p->d_eloc1 : p->d_eloc2;
  r.tile_np = side == 1 ? p->tile_np1 : p->tile_np2;
  r.scale = 1.f;
  r.beams = side == 1 ? p->d_beams : p->d_det;
  r.nb = side == 1 ? p->B : p->ndet;
  r.W = side == 1 ? p->W1[a] : p->W[a];  // S1: the enlarged window in focal mode
  r.oy = side == 1 ? p->oy1[a] : p->oy[a];
  r.ox = side == 1 ? p->ox1[a] : p->ox[a];
  r.ny = p->g.ny;
  r.nx = p->g.nx;
  r.tw = p->d_tw;
  r.L = p->L;
  r.retilt_sign = side == 1 ? +1 : -1;
  r.mode = p->o.recon_mode;
  r.n_cu = p->n_cu;
  return r;
}

}  // namespace bip
