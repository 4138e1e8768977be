// Device helpers shared by the attention kernels: tile layout and direct-to-LDS
// tile loads, the work item as a wave sees it, and the query-side RoPE relocation.
#pragma once

#include "common.h"
#include "restart.h"

namespace mla {

// The softmax reference of a head-row is its max over this many first keys of an item
// (those of the item's first segment, where it is shorter).  The weight at the max is
// exactly 1; weights above it carry bf16's rounding, so fewer keys cost accuracy.
constexpr int kRefKeys = 64;

template <int DC, int DR>
struct Cfg {
  static constexpr int D = DC + DR;
  static constexpr int KS = D / 16;          // 16-wide K steps of Q.K
  static constexpr int CS = DC / 16;         // latent K steps
  static constexpr int RS = DR / 16;         // RoPE K steps
  static constexpr int CH = D / 8;           // 16-byte chunks per key row
  static constexpr int CG = (CH + 7) / 8;    // groups of 8 chunks
  static constexpr int CGF = CH / 8;         // full groups (swizzled)
  static constexpr int BK = 64;              // keys per tile
  // LDS tile: 8 key-blocks of 8 keys; block kb8 starts at kb8*KB8 and holds CG
  // 1 KB sub-blocks (one per chunk group).  Inside a sub-block key k%8 sits at
  // (k%8)*128 and chunk c%8 at slot (c%8) ^ rotl3(k%8) (full groups only), so
  // both the row reads of K and the transposing column reads of V hit distinct
  // banks.  KB8 = 128 mod 256 keeps 16-lane 16-byte reads conflict-free on 64 banks.
  static constexpr int KB8 = CG * 1024 + 128;
  static constexpr int TILE_BYTES = 8 * KB8;
  static constexpr int OB = DC / 32;         // 32-dim output blocks of O^T
  static constexpr int PS = BK / 16;         // 16-key contraction steps of P.V per tile
  static_assert(DR == 16 || DR % 32 == 0, "d_rope must be 16 or a multiple of 32");
  static_assert(DC % 64 == 0, "d_latent must be a multiple of 64");
  static_assert(BK == kRefKeys, "the reference is the first tile's max");
  static_assert(kTileRows == 128, "one work item is 4 waves x 32 head-rows");
};

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ int rotl3(int k) { return ((k << 1) | (k >> 2)) & 7; }

__device__ __forceinline__ int wave_min_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const int w = __shfl_xor(v, o, 64);
    v = w < v ? w : v;
  }
  return v;
}

// Tile barrier: this wave's direct-to-LDS loads and LDS accesses are complete,
// then all waves meet.  One asm statement with a memory clobber, so the
// compiler moves no LDS access across it.
__device__ __forceinline__ void tile_barrier() {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// value of lane l%32 and of lane l%32 + 32, in every lane (one permlane swap)
__device__ __forceinline__ void lane_halves(float v, float& x, float& y) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  x = __uint_as_float(r[0]);
  y = __uint_as_float(r[1]);
}

// What a work item's waves take from the plan: the tables, the item, and this
// lane's head-row (its storage row, query, output slot and request position).
// Blocks are dispatched round-robin over the 8 XCDs; each XCD gets 32
// consecutive items (similar key ranges) per group of 256.
struct ItemView {
  const SegInfo* segs;
  const int32_t* rank_seg;
  const double* theta_rev;
  WorkItem it;
  SegInfo own;
  ChunkInfo chk;
  bool valid;    // this lane has a head-row
  bool active;   // wave-uniform: the wave has head-rows
  int64_t row, slot, t_pos;
  const uint16_t* qsrc;
};

__device__ __forceinline__ int xcd_item_id(int b) {
  const int xcd = b & 7, kx = b >> 3;
  return (kx >> 5) * 256 + xcd * 32 + (kx & 31);
}

// work items of this launch: the host plan's count, or the device plan's
__device__ __forceinline__ int item_count(const AttendArgs& a) {
  return a.dyn != nullptr ? a.dyn->n_items : a.n_items;
}

template <class C>
__device__ __forceinline__ ItemView item_view(const AttendArgs& a, int item_id, int wave, int l32) {
  ItemView v;
  v.segs = a.segs;
  v.rank_seg = a.rank_seg;
  v.theta_rev = a.theta_rev;
  const int32_t* prot = a.prot;
  v.it = a.items[item_id];
  v.own = v.segs[v.it.seg];
  v.chk = a.chunks[v.own.chunk_off + v.it.chunk];
  const int hr_local = wave * 32 + l32;
  v.valid = hr_local < v.it.count;
  v.active = wave * 32 < v.it.count;
  const int64_t hr = v.it.hr_begin + (v.valid ? hr_local : 0);
  if (v.it.kind == 0) {
    v.row = hr / a.n_groups;
    v.qsrc = (const uint16_t*)a.q_glob + hr * C::D;
    v.slot = hr;
  } else {
    v.row = prot[hr / a.n_local];
    v.qsrc = (const uint16_t*)a.q_loc + hr * C::D;
    v.slot = a.local_slot_base + hr;
  }
  v.t_pos = v.own.req_offset + (v.row - v.own.kv_start);
  return v;
}

// visible keys of segment s for the item: its own segment up to the item's last row
__device__ __forceinline__ int64_t seg_keys(const ItemView& v, const SegInfo& s, bool is_own) {
  return is_own ? (int64_t)v.it.max_u + 1 : s.length;
}

// Direct-to-LDS loads of tile `tile` of segment `s` (n_keys visible keys) into
// dbuf: wave w fills key-blocks 2w, 2w+1; lane l loads key l>>3 of a block, the
// 16-byte chunk at physical slot l&7 of each 8-chunk group.  Rows past the
// segment's end repeat its last row.
template <class C>
__device__ __forceinline__ void issue_tile(const void* kv, const SegInfo& s, int64_t n_keys, int64_t tile,
                                           unsigned char MLA_LDS* dbuf, int wave, int lkey, int lchunk_full,
                                           int lchunk_part) {
  const int64_t k0 = tile * C::BK;
  const int last = (int)(n_keys - 1 - k0);
  const bool full = last >= C::BK - 1;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int kb8 = 2 * wave + h;
    // uniform base: first row of the 8-key block; lane offset: its key row and chunk
    int64_t brow = k0 + kb8 * 8;
    int kr = lkey;
    if (!full) {
      const int lb = last - kb8 * 8;   // last valid key of this block, relative to its first
      if (lb < 0) {                    // whole block past the end: repeat the segment's last row
        brow = k0 + last;
        kr = 0;
      } else if (kr > lb) {
        kr = lb;
      }
    }
    const unsigned char* base = (const unsigned char*)kv + (s.kv_start + brow) * (C::D * 2);
    const uint32_t roff = (uint32_t)(kr * (C::D * 2));   // never negative
#pragma unroll
    for (int cg = 0; cg < C::CG; ++cg) {
      const int ch = cg * 8 + (cg < C::CGF ? lchunk_full : lchunk_part);
      dma16(base, roff + ch * 16, dbuf + kb8 * C::KB8 + cg * 1024);
    }
  }
}

// Relocation for a new segment s (Sec. 2.3 eq:rope): rotate the RoPE part of
// this lane's query by R(t - p_s) into qf's RoPE steps; the angle is reduced in
// double precision (in revolutions) and fed to the hardware sin/cos.  Returns
// the lane's largest visible canonical offset in s (INT_MAX without a head-row).
template <class C, int DC, int DR, bool RELOAD = true>
__device__ __forceinline__ int relocate_query(bf16x8 (&qf)[C::KS], const ItemView& v, const SegInfo& s, int half) {
  const int64_t delta = v.t_pos - s.req_offset;
  const int64_t lm = delta < s.length - 1 ? delta : s.length - 1;
  bf16x8 raw[C::RS];
#pragma unroll
  for (int rs = 0; rs < C::RS; ++rs) {
    if (!RELOAD) {
      raw[rs] = qf[C::CS + rs];   // still the unrotated query
    } else if (DR == 16) {
      const u32x2 lo = *(const u32x2*)(v.qsrc + DC + half * 4);
      const u32x2 hi = *(const u32x2*)(v.qsrc + DC + 8 + half * 4);
      raw[rs] = __builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], hi[0], hi[1]});
    } else {
      raw[rs] = *(const bf16x8*)(v.qsrc + DC + rs * 16 + half * 8);
    }
  }
  const double dd = (double)delta;
#pragma unroll
  for (int rs = 0; rs < (DR == 16 ? 1 : C::RS / 2); ++rs) {
#pragma unroll
    for (int i = 0; i < (DR == 16 ? 4 : 8); ++i) {
      // pair (j, j + d_r/2): first element at (rs, slot i), partner at (prs, ps)
      const int j0 = DR == 16 ? i : rs * 16 + i;
      const int jstep = DR == 16 ? 4 : 8;       // frequency offset of the upper lane half
      const int prs = DR == 16 ? rs : rs + DR / 32;
      const int ps = DR == 16 ? i + 4 : i;
      const double rev = dd * v.theta_rev[j0 + half * jstep];
      const float r = (float)(rev - rint(rev));
      const float sn = __builtin_amdgcn_sinf(r), cn = __builtin_amdgcn_cosf(r);
      const float x1 = (float)raw[rs][i], x2 = (float)raw[prs][ps];
      qf[C::CS + rs][i] = v.valid ? (__bf16)(x1 * cn - x2 * sn) : (__bf16)0.f;
      qf[C::CS + prs][ps] = v.valid ? (__bf16)(x1 * sn + x2 * cn) : (__bf16)0.f;
    }
  }
  return v.valid ? (int)lm : 0x7fffffff;
}

// the latent-value 512 + 64 kernel (attend_pair.hip)
hipError_t launch_attend_pair(const AttendArgs& a, unsigned grid, hipStream_t s);

}  // namespace mla
