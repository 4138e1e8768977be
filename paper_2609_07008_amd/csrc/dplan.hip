// Device half of the plan (Alg. 2: ProtectedRows feeding SelectiveMLA in the same
// layer without a trip through the host): the work items, the partial index with
// its segment bookkeeping, and the protected flags.
//
// The host fixes, once per request, everything that depends only on the segment
// table: segment visibility in request order, the chunking of each visible list,
// the Global partial index and the launch order of the item groups (one group
// per kind, segment and chunk, largest upper-bound cost first).  Per call, the
// protected rows A and |A| are read from device memory and the plan is finished:
//   count  validates A (ascending, in range, at most the capacity the plan was
//     built for), finds each segment's run of protected rows by binary search (A is
//     sorted and segments are contiguous in storage), the Local partial base of
//     each segment (a scan in storage order), each group's item count and their
//     prefix (a scan in launch order), and the call's counts;
//   items  one thread per item: its group by binary search in the prefix, then its
//     head-row range.  Inside a group items run from the segment's last head-rows
//     down, so that the costliest items of the group start first;
//   slots  one thread per slot: part_ptr and part_seg;
//   rows   one thread per row: row_src.
// A rejected A leaves zero items, zero slots and status MLA_ERR_ROWS: the
// attention kernels then do nothing.
//
// What bounds it is launches: every phase is a chain of a few dependent reads.
// Requests of up to kPlanOneRows rows take one launch, in which every workgroup
// counts for itself, in LDS, and takes its share of items, slots and rows (the
// 2.1K-row step's four plan launches 21 us, this one 9.6).  Every workgroup then reads
// the whole protected list, which the separate launches do once; larger requests keep
// those.  Measured at the line (65,536 rows, 16 segments, one Local head; one launch
// against four): 1310 protected rows 11.4 us against 21.3, 16,384 20.0 against 30.6, every
// row 46.6 against 60.0; 512 segments 13.2 against 25.2 and 50.8 against 65.2.
#include "common.h"

#include <algorithm>

namespace mla {

constexpr int kPlanThreads = 1024;
// protected lists up to this length are searched in LDS (32 KB, so that two workgroups
// share a compute unit): the binary searches are chains of a dozen dependent reads.
// One launch for 65,536 rows: 14.6 us with 8192 protected rows, 20.0 with 16,384
constexpr int kPlanLdsRows = 8192;

// exclusive prefix of v over the workgroup's threads (in thread order); *total
// receives the sum.  Every thread of the workgroup calls it.
__device__ int64_t block_exclusive_scan(int64_t v, int64_t* total) {
  __shared__ int64_t wsum[kPlanThreads / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int64_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  int64_t before = 0, all = 0;
  for (int i = 0; i < kPlanThreads / 64; ++i) {
    before += i < w ? wsum[i] : 0;
    all += wsum[i];
  }
  __syncthreads();   // wsum may be rewritten by the next call
  *total = all;
  return before + x - v;
}

// first index in prot[0, n) whose value is >= r
template <class P>
__device__ __forceinline__ int lower_bound_i32(P prot, int n, int64_t r) {
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if ((int64_t)prot[mid] < r) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// the count phase, by one workgroup; a's tables are its outputs, in device memory
// or in LDS (generic pointers)
__device__ void plan_count(const DPlanArgs& a, int32_t MLA_LDS* s_prot) {   // [kPlanLdsRows]
  __shared__ int s_ok;
  __shared__ int s_np;
  const int tid = threadIdx.x;
  if (tid == 0) {
    const int np = *a.n_prot_dev;
    s_np = np;
    s_ok = (np >= 0 && np <= a.prot_cap) ? 1 : 0;
  }
  __syncthreads();
  const int np = s_ok ? s_np : 0;
  // validation: rows in range and strictly increasing
  int bad = 0;
  const bool in_lds = np <= kPlanLdsRows;
  for (int i = tid; i < np; i += kPlanThreads) {
    const int32_t r = a.prot[i];
    if (in_lds) s_prot[i] = r;
    if (r < 0 || (int64_t)r >= a.n_rows || (i > 0 && a.prot[i - 1] >= r)) bad = 1;
  }
  if (__syncthreads_or(bad) || !s_ok) {
    if (tid == 0) {
      a.dyn->n_slots = 0;
      a.dyn->n_parts = 0;
      a.dyn->n_items = 0;
      a.dyn->n_prot = 0;
      a.dyn->status = MLA_ERR_ROWS;
      if (a.status_out != nullptr) *a.status_out = MLA_ERR_ROWS;
    }
    return;
  }
  // each segment's run of protected rows, and its Local partial base in storage order
  int64_t carry = 0;
  for (int base = 0; base < a.n_segs; base += kPlanThreads) {
    const int i = base + tid;
    int64_t parts = 0;
    if (i < a.n_segs) {
      const int s = a.storage[i];
      const SegInfo si = a.segs[s];
      const int lo = in_lds ? lower_bound_i32(s_prot, np, si.kv_start)
                            : lower_bound_i32(a.prot, np, si.kv_start);
      const int hi = in_lds ? lower_bound_i32(s_prot, np, si.kv_start + si.length)
                            : lower_bound_i32(a.prot, np, si.kv_start + si.length);
      a.seg_prot_lo[s] = lo;
      a.seg_prot_cnt[s] = hi - lo;
      parts = (int64_t)(hi - lo) * a.n_local * si.n_chunks;
    }
    int64_t total;
    const int64_t ex = block_exclusive_scan(parts, &total);
    if (i < a.n_segs) a.seg_local_base[a.storage[i]] = carry + ex;
    carry += total;
  }
  const int64_t local_parts = carry;
  __syncthreads();   // seg_prot_cnt of every segment is written
  // item counts of the groups in launch order, and their prefix
  int64_t items = 0;
  for (int base = 0; base < a.n_item_groups; base += kPlanThreads) {
    const int i = base + tid;
    int64_t cnt = 0;
    if (i < a.n_item_groups) {
      const ItemGroup g = a.groups[i];
      cnt = g.kind == 0 ? g.n_items
                        : ((int64_t)a.seg_prot_cnt[g.seg] * a.n_local + kTileRows - 1) / kTileRows;
    }
    int64_t total;
    const int64_t ex = block_exclusive_scan(cnt, &total);
    if (i < a.n_item_groups) a.group_base[i] = (int32_t)(items + ex);
    items += total;
  }
  if (tid == 0) {
    // the host's bounds hold for every list of at most prot_cap rows; should one
    // not hold, nothing runs rather than anything being written out of range
    const bool fits = items <= a.max_items && a.global_parts + local_parts <= a.max_parts;
    a.group_base[a.n_item_groups] = (int32_t)items;
    a.dyn->n_slots = fits ? a.n_rows * a.n_groups + (int64_t)np * a.n_local : 0;
    a.dyn->n_parts = fits ? a.global_parts + local_parts : 0;
    a.dyn->n_items = fits ? (int32_t)items : 0;
    a.dyn->n_prot = fits ? np : 0;
    a.dyn->status = fits ? MLA_OK : MLA_ERR_WORKSPACE;
    if (a.status_out != nullptr) *a.status_out = a.dyn->status;
  }
}

__global__ __launch_bounds__(kPlanThreads) void dplan_count_kernel(DPlanArgs a) {
  __shared__ int32_t s_prot[kPlanLdsRows];
  plan_count(a, (int32_t MLA_LDS*)s_prot);
}

__device__ void plan_item(const DPlanArgs& a, int i, WorkItem* items) {
  // the group holding item i: the last g with group_base[g] <= i
  int lo = 0, hi = a.n_item_groups - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.group_base[mid] <= i) lo = mid; else hi = mid - 1;
  }
  const ItemGroup g = a.groups[lo];
  const int k = i - a.group_base[lo];
  const SegInfo si = a.segs[g.seg];
  int64_t h0, h1;   // head-row range of the group
  if (g.kind == 0) {
    h0 = si.kv_start * a.n_groups;
    h1 = (si.kv_start + si.length) * a.n_groups;
  } else {
    h0 = (int64_t)a.seg_prot_lo[g.seg] * a.n_local;
    h1 = h0 + (int64_t)a.seg_prot_cnt[g.seg] * a.n_local;
  }
  const int64_t end = h1 - (int64_t)k * kTileRows;
  const int64_t begin = end - kTileRows > h0 ? end - kTileRows : h0;
  const int64_t last_row = g.kind == 0 ? (end - 1) / a.n_groups : (int64_t)a.prot[(end - 1) / a.n_local];
  WorkItem w;
  w.hr_begin = begin;
  w.count = (int32_t)(end - begin);
  w.kind = g.kind;
  w.seg = g.seg;
  w.chunk = g.chunk;
  w.max_u = (int32_t)(last_row - si.kv_start);
  w.pad = 0;
  items[i] = w;
}

__global__ __launch_bounds__(256) void dplan_items_kernel(DPlanArgs a) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < a.dyn->n_items) plan_item(a, i, a.items);
}


// segment (storage order) holding storage row r: the last one whose kv_start <= r
__device__ __forceinline__ int segment_of_row(const AttendArgs& a, int64_t r) {
  int lo = 0, hi = a.n_segs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.segs[a.storage[mid]].kv_start <= r) lo = mid; else hi = mid - 1;
  }
  return a.storage[lo];
}

// part_ptr (and part_seg) of slot i; i = n_slots closes the index; seg_of(r): the
// segment of storage row r
template <class SegOf>
__device__ __forceinline__ void plan_slot(const AttendArgs& a, int64_t i, int64_t n_slots, int64_t n_parts, SegOf seg_of) {
  const int64_t nglob = a.n_rows * a.n_groups;
  if (i == n_slots) {
    a.part_ptr[i] = n_parts;
    return;
  }
  int s;
  int64_t base;
  if (i < nglob) {
    const int64_t r = i / a.n_groups, g = i - r * a.n_groups;
    s = seg_of(r);
    const SegInfo si = a.segs[s];
    base = si.cum_global + ((r - si.kv_start) * a.n_groups + g) * si.n_chunks;
  } else {
    const int64_t k = i - nglob;
    const int64_t ai = k / a.n_local, jj = k - ai * a.n_local;
    if (a.dyn == nullptr) {
      s = a.prot_seg[ai];
      base = a.global_parts + a.cum_local[ai] + jj * a.segs[s].n_chunks;
    } else {
      s = seg_of((int64_t)a.prot[ai]);
      const int64_t nch = a.segs[s].n_chunks;
      base = a.global_parts + a.seg_local_base[s] + ((ai - a.seg_prot_lo[s]) * a.n_local + jj) * nch;
    }
  }
  a.part_ptr[i] = base;
  if (a.part_seg != nullptr) {
    const SegInfo si = a.segs[s];
    for (int c = 0; c < si.n_chunks; ++c) {
      const ChunkInfo ch = a.chunks[si.chunk_off + c];
      a.part_seg[2 * (base + c)] = a.rank_seg[ch.first_rank];
      a.part_seg[2 * (base + c) + 1] = a.rank_seg[ch.last_rank];
    }
  }
}

// is row r in the protected list?
template <class P>
__device__ __forceinline__ void plan_row(const AttendArgs& a, int64_t r, P prot, int n_prot) {
  const int lo = lower_bound_i32(prot, n_prot, r);
  a.row_src[r] = (lo < n_prot && prot[lo] == r) ? 1 : 0;
}

__global__ __launch_bounds__(256) void plan_slots_kernel(AttendArgs a) {
  const int64_t n_slots = a.dyn != nullptr ? a.dyn->n_slots : a.n_slots;
  const int64_t n_parts = a.dyn != nullptr ? a.dyn->n_parts : a.n_parts;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= n_slots;
       i += (int64_t)gridDim.x * blockDim.x)
    plan_slot(a, i, n_slots, n_parts, [&](int64_t r) { return segment_of_row(a, r); });
}

__global__ __launch_bounds__(256) void row_src_kernel(AttendArgs a) {
  const int n_prot = a.dyn != nullptr ? a.dyn->n_prot : a.n_prot;
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < a.n_rows;
       r += (int64_t)gridDim.x * blockDim.x)
    plan_row(a, r, a.prot, n_prot);
}

// part_ptr / part_seg (when part_ptr is set) and row_src (when set); grids cover
// the host count of slots and rows (for a device plan, the capacity bound)
hipError_t launch_plan(const AttendArgs& a, hipStream_t s) {
  if (a.part_ptr != nullptr) {
    const int64_t n = a.n_slots + 1;
    const unsigned blocks = (unsigned)std::min<int64_t>((n + 255) / 256, 8192);
    plan_slots_kernel<<<dim3(blocks), dim3(256), 0, s>>>(a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (a.row_src == nullptr) return hipSuccess;
  const unsigned rb = (unsigned)std::min<int64_t>((a.n_rows + 255) / 256, 4096);
  row_src_kernel<<<dim3(rb), dim3(256), 0, s>>>(a);
  return hipGetLastError();
}

// requests of the one-launch form; the segment and group tables are held in LDS (20 KB)
constexpr int64_t kPlanOneRows = 65536;
constexpr int kPlanOneSegs = 512, kPlanOneGroups = 2048;

// every phase of a device plan in one launch: workgroup 0 also leaves the counts
// in device memory for the attention kernels
__global__ __launch_bounds__(kPlanThreads) void dplan_one_kernel(DPlanArgs d, AttendArgs a) {
  __shared__ int32_t s_lo[kPlanOneSegs], s_cnt[kPlanOneSegs], s_group[kPlanOneGroups + 1];
  __shared__ int64_t s_base[kPlanOneSegs];
  __shared__ int32_t s_kv[kPlanOneSegs], s_seg[kPlanOneSegs];   // in storage order
  __shared__ int32_t s_prot[kPlanLdsRows];
  __shared__ DynPlan s_dyn;
  DPlanArgs p = d;
  p.seg_prot_lo = s_lo;
  p.seg_prot_cnt = s_cnt;
  p.seg_local_base = s_base;
  p.group_base = s_group;
  p.dyn = &s_dyn;
  if (blockIdx.x != 0) p.status_out = nullptr;
  int32_t MLA_LDS* prot = (int32_t MLA_LDS*)s_prot;
  if (threadIdx.x < d.n_segs) {   // at most kPlanOneSegs; read after the barriers of the count
    const int sg = d.storage[threadIdx.x];
    s_seg[threadIdx.x] = sg;
    s_kv[threadIdx.x] = (int32_t)d.segs[sg].kv_start;
  }
  plan_count(p, prot);
  __syncthreads();
  if (blockIdx.x == 0 && threadIdx.x == 0) *d.dyn = s_dyn;
  const int64_t first = (int64_t)blockIdx.x * kPlanThreads + threadIdx.x, stride = (int64_t)gridDim.x * kPlanThreads;
  for (int64_t i = first; i < s_dyn.n_items; i += stride) plan_item(p, (int)i, d.items);
  a.seg_prot_lo = s_lo;
  a.seg_local_base = s_base;
  const int32_t MLA_LDS* kv = (const int32_t MLA_LDS*)s_kv;
  auto seg_of = [&](int64_t r) -> int {
    int lo = 0, hi = d.n_segs - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (kv[mid] <= r) lo = mid; else hi = mid - 1;
    }
    return s_seg[lo];
  };
  if (a.part_ptr != nullptr)
    for (int64_t i = first; i <= s_dyn.n_slots; i += stride) plan_slot(a, i, s_dyn.n_slots, s_dyn.n_parts, seg_of);
  if (a.row_src != nullptr) {
    const int np = s_dyn.n_prot;
    for (int64_t r = first; r < a.n_rows; r += stride)
      if (np <= kPlanLdsRows) plan_row(a, r, (const int32_t MLA_LDS*)prot, np); else plan_row(a, r, a.prot, np);
  }
}

// d: the counts and items; a: the index and flags of the same call (a.dyn = d.dyn)
hipError_t launch_dplan(const DPlanArgs& d, const AttendArgs& a, hipStream_t s) {
  if (d.n_rows <= kPlanOneRows && d.n_segs <= kPlanOneSegs && d.n_item_groups <= kPlanOneGroups) {
    int64_t n = std::max<int64_t>(d.max_items, 1);
    if (a.part_ptr != nullptr) n = std::max(n, a.n_slots + 1);
    if (a.row_src != nullptr) n = std::max(n, a.n_rows);
    const unsigned blocks = (unsigned)std::min<int64_t>((n + kPlanThreads - 1) / kPlanThreads, 256);
    dplan_one_kernel<<<dim3(blocks), dim3(kPlanThreads), 0, s>>>(d, a);
    return hipGetLastError();
  }
  dplan_count_kernel<<<dim3(1), dim3(kPlanThreads), 0, s>>>(d);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (d.max_items > 0) {
    dplan_items_kernel<<<dim3((unsigned)((d.max_items + 255) / 256)), dim3(256), 0, s>>>(d);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return launch_plan(a, s);
}

}  // namespace mla
