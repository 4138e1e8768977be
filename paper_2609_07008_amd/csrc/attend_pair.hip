// Query-side RoPE relocation and segment-wise absorbed-MLA attention (Sec. 2.3
// eq:rope, Alg. 2 SelectiveMLA) for the 512 + 64 latent with the latent as the
// value: two specialised waves per SIMD.
//
// What bounds it.  With one 512-register wave per SIMD (the form that the rotary
// value still takes) a wave's tile loads, softmax and barriers leave its SIMD's
// matrix core idle for 40 % of the time.  With them filled the card's power limit
// comes next: on random bf16 values 32x32x16 MFMAs that read one 1 KB LDS fragment
// each settle at 1.56 GHz and 1584 TFLOP/s, pairs of 16x16x32 ones (the same
// fragment bytes and flop) at 1.74 GHz and 1731, so this kernel takes 16x16x32.
//
// A work item is up to 128 head-rows that share every key of the latent stream
// (common.h); one 512-thread workgroup takes it.  Waves w and w + 4 share a SIMD
// and the item's head-rows 32 w .. +31:
//   score wave w      holds the 576-dim queries (144 registers); per 32-key tile
//                     S^T = K Q^T, the softmax weights against a fixed reference
//                     max, and output dims 0 .. 63
//   value wave w + 4  holds output dims 64 .. 511 (224 registers): O^T += V^T P^T
//                     with the weights handed over through LDS; issues the direct
//                     global->LDS loads (global_load_lds_dwordx4) of the tiles
// Neither half fits beside the other's state in one 256-register wave; split so,
// the value waves' MFMAs run while the score waves are in the softmax, at the
// barrier or waiting for LDS.
//
// Step t (one barrier each): tile t + 1 is loaded into one of three tile buffers,
// the score waves take tile t, the value waves tile t - 1.  V fragments serve two
// MFMAs (the two 16-row halves of a pair's head-rows), K fragments too.  The score
// waves' instruction issue (about 5 clk each) is what a step waits for, so their
// vector work sits between MFMAs where it is free: the weights of a tile's first
// 16 keys between the MFMAs of the second 16, the row sums between those of their
// own output dims; rare branches are laid out of line.
//
// The item's queries are contiguous in memory and come in through the idle tile
// buffers with direct loads (fetched by each lane from its own rows they held up
// the first tile: 27K clk from a workgroup's start to its first tile against 16K).
// Head outputs leave through LDS as whole rows.
//
// Measured against the one-wave kernel (same box, whole calls, the other kernels'
// changes included): the 264,192-row step 594 -> 531 ms, the 33,792-row one 12.2 ->
// 10.9, with partials 11.4 -> 10.5, the 67,584-row one with 128 heads 102.5 -> 91.3, the
// 33K-row producer 5.03 -> 4.63; this kernel alone took the 2.1K-row step from 245 to
// 227 us.  3060 clk per 32 keys and workgroup at 1.95 GHz against 3630 at 2.1.  Without
// the value waves' MFMAs a step takes 2350 clk, without the score waves' 2640.
// Reading V or K two, three or four fragments ahead, wave priorities and the tile
// loads' place in the step change the clock and the cycles together and leave the
// time as it is.
//
// The reference of the softmax weights is taken before the tile loop, from the item's
// first 64 keys as in the one-wave kernel: tiles 0 and 1 are loaded together and the
// score waves run K Q^T over them once for the max alone.  From the first 16 keys,
// inside the first step, it cost nothing, but rounded the weight of every larger key
// after them: errors against 64 bits grew (2.1K-row step, lse 1.83e-5 -> 1.89e-5; now
// 1.83e-5), and outputs were 1e-3 to 2.7e-3 off the one-wave kernel's (now 2e-4 and
// less, the order of the sums).  The pass takes an item about 3K clk, its MFMAs: the
// 33K-row producer 4.51 -> 4.61 ms, steps up to 1 %, 1.6 % where documents are short.
//
// Restart policy: restart.h.  A wave that sees a tile's weights sum to 2^64 or more
// records the next step's index in restart_at (LDS atomic min); at the end of step
// t every wave tests restart_at <= t on a value read after the step's barrier, which
// votes cast in step t cannot satisfy, so all leave at the same step.
#include "attend.h"

namespace mla {

template <int DC, int DR>
struct PairCfg {
  static constexpr int D = DC + DR;
  static constexpr int KS = D / 32;                // 32-dim K steps of Q.K
  static constexpr int CS = DC / 32;               // latent K steps
  static constexpr int CG = D / 64;                // chunk groups of 8 x 16 bytes per key row
  static constexpr int BK = 32;                    // keys per tile
  // LDS tile: 4 key-blocks of 8 keys, block kb8 at kb8*KB8, holding CG 1 KB
  // sub-blocks (one per chunk group); inside one, key k%8 sits at (k%8)*128 and
  // chunk c%8 at slot (c%8) ^ key_swz(k%8).  KB8 = 128 mod 256.
  static constexpr int KB8 = CG * 1024 + 128;
  static constexpr int TILE_BYTES = BK / 8 * KB8;
  static constexpr int NBUF = 3;
  static constexpr int OB = DC / 16;               // 16-dim output blocks of O^T
  static constexpr int OBS = 4;                    // output blocks of a score wave
  static constexpr int OBV = OB - OBS;             // output blocks of a value wave
  static constexpr int P_OFF = NBUF * TILE_BYTES;  // 4 pairs x 2 buffers x 2 KB
  static constexpr int Q_OFF = P_OFF + 4 * 2 * 2048;   // 4 pairs x 4 KB: unrotated RoPE query parts
  static constexpr int INV_OFF = Q_OFF + 4 * 4096;     // 4 pairs x 32 reciprocal row sums
  static constexpr int TH_OFF = INV_OFF + 512;         // RoPE frequencies, a copy a score wave
  static constexpr int QSTAGE = kTileRows / 8 * KB8;   // the item's queries at its start, in the tile layout
  static constexpr int LDS_BYTES = QSTAGE > TH_OFF + 4 * (DR / 2 * 8) ? QSTAGE : TH_OFF + 4 * (DR / 2 * 8);
  static_assert(DR == 64 && DC % 64 == 0, "rotation pairs (j, j + 32) sit in one lane of two K steps");
  static_assert(kRefKeys == 2 * BK && NBUF >= 2, "the reference's keys are tiles 0 and 1");
  static_assert(OBS % 4 == 0 && OBV % 4 == 0, "output blocks come in whole chunk groups");
};

// The lane id through an opaque asm: per-lane addresses are recomputed from it at
// each tile rather than held in registers across the tile loop.
__device__ __forceinline__ int lane_now() {
  int v;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(v));
  return v;
}

// Slot of 16-byte chunk c of key k (of its 8-key block) in an LDS sub-block: c ^
// key_swz(k).  A 16-byte read is served in groups of 16 lanes {0-3, 12-15, 20-23,
// 24-27} (and their complements): a K fragment read then takes keys 0-3 of an even
// and 4-7 of an odd key-block for one chunk and the other halves for the next, and
// this swizzle spreads each group over all 64 banks (with c ^ k every K read took
// twice its cycles).  The transposing V reads (8 keys x 2 chunks a half-wave) need
// the even keys, and the odd ones, in four distinct chunk pairs: also true.
__device__ __forceinline__ int key_swz(int k) { return k ^ ((~k & 1) << 2); }

// Tile cursor over a chunk's segments in request order, in scalar registers (the
// tables are constant while the kernel runs; all counts fit 31 bits).
#define MLA_CONST __attribute__((address_space(4)))
struct PairView {   // the item and its tables
  const SegInfo* segs;
  const int32_t* rank_seg;
  WorkItem it;
  ChunkInfo chk;
};
struct TileCursor {
  int rank, kv_start, length, req_offset, n_keys, tile;
};

template <class C>
__device__ __forceinline__ void cursor_open(TileCursor& c, const PairView& v, int rank) {
  c.rank = rank;
  const int sidx = ((const int32_t MLA_CONST*)(uintptr_t)v.rank_seg)[rank];
  const SegInfo MLA_CONST* s = (const SegInfo MLA_CONST*)(uintptr_t)v.segs + sidx;
  c.kv_start = (int)s->kv_start;
  c.length = (int)s->length;
  c.req_offset = (int)s->req_offset;
  c.n_keys = sidx == v.it.seg ? v.it.max_u + 1 : c.length;
  c.tile = 0;
}
// next tile; 0: none, 1: same segment, 2: a new segment
template <class C>
__device__ __forceinline__ int cursor_next(TileCursor& c, const PairView& v) {
  if (__builtin_expect((c.tile + 1) * C::BK < c.n_keys, 1)) {
    ++c.tile;
    return 1;
  }
  if (c.rank >= v.chk.last_rank) return 0;
  cursor_open<C>(c, v, c.rank + 1);
  return 2;
}

// Direct-to-LDS loads of one 8-key block of the cursor's tile into dbuf: lane l
// loads key l>>3, the 16-byte chunk at physical slot l&7 of each 8-chunk group.
// Rows past the segment's visible keys repeat its last one.
template <class C>
__device__ __forceinline__ void issue_block(const void* kv, const TileCursor& c, unsigned char MLA_LDS* dbuf, int kb8) {
  const int lane = lane_now();
  int brow = c.tile * C::BK + kb8 * 8;
  const int last = c.n_keys - 1 - brow;   // last valid key relative to the block's first
  int kr = lane >> 3;
  kr = kr < (last < 0 ? 0 : last) ? kr : (last < 0 ? 0 : last);
  brow = last < 0 ? brow + last : brow;   // whole block past the end
  const unsigned char* base = (const unsigned char*)kv + (int64_t)(c.kv_start + brow) * (C::D * 2);
  const uint32_t voff = (uint32_t)(kr * (C::D * 2) + (((lane & 7) ^ key_swz(lane >> 3)) * 16));
#pragma unroll
  for (int cg = 0; cg < C::CG; ++cg) dma16(base + cg * 128, voff, dbuf + kb8 * C::KB8 + cg * 1024);
}

// maximum / sum over the four lanes that hold a head-row's keys
__device__ __forceinline__ float quad_max(float v) {
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ float quad_sum(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

template <int DC, int DR>
__global__ __launch_bounds__(512, 2) void attend_pair_kernel(AttendArgs a) {
  using C = PairCfg<DC, DR>;
  __shared__ __attribute__((aligned(16))) unsigned char lds[C::LDS_BYTES];
  __shared__ unsigned restart_at;

  unsigned char MLA_LDS* L = (unsigned char MLA_LDS*)lds;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pair = wave & 3;
  const int lg = lane >> 4, lc = lane & 15;   // lane group, and head-row / key / dim inside a 16-block

  const int item_id = xcd_item_id(blockIdx.x);
  if (item_id >= item_count(a)) return;
  PairView v;
  v.segs = a.segs;
  v.rank_seg = a.rank_seg;
  v.it = a.items[item_id];
  const WorkItem& it = v.it;
  // The item's queries are contiguous: direct loads bring them into LDS in the tile
  // layout (two 8-row blocks a wave, rows past the item repeat its last one), and
  // the score waves read their fragments from there.
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int qb = 2 * wave + h;
    int r = qb * 8 + (lane >> 3);
    r = r < it.count ? r : it.count - 1;
    const unsigned char* base = (const unsigned char*)(it.kind == 0 ? a.q_glob : a.q_loc) + it.hr_begin * (C::D * 2);
    const uint32_t voff = (uint32_t)(r * (C::D * 2) + (((lane & 7) ^ key_swz(lane >> 3)) * 16));
#pragma unroll
    for (int cg = 0; cg < C::CG; ++cg) dma16(base + cg * 128, voff, L + qb * C::KB8 + cg * 1024);
  }
  const SegInfo own = v.segs[v.it.seg];
  v.chk = a.chunks[own.chunk_off + v.it.chunk];

  // V^T fragments (A operand, 16 dims x 32 keys) by transposing reads: lane group
  // lg takes keys lg*4 + 0..3 and 16 + lg*4 + 0..3, the order in which a score
  // wave holds its weights; in each group lane rr*4 + cb addresses key lg*4 + rr,
  // dims cb*4 .. +3 and receives dim lane%16 of the four keys.
  auto vbase = [&](int off) {
    const int ln = lane_now();
    const int key = ((ln >> 4) & 1) * 4 + ((ln >> 2) & 3), cb = ln & 3;
    return off + (ln >> 5) * C::KB8 + key * 128 + (((cb >> 1) ^ key_swz(key)) * 16) + (cb & 1) * 8;
  };
  auto vfrag = [&](int vb, int d) -> bf16x8 {
    const unsigned char MLA_LDS* p = L + (vb ^ ((d & 3) * 32)) + (d >> 2) * 1024;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((MLA_LDS bf16x4*)p);
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((MLA_LDS bf16x4*)(p + 2 * C::KB8));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  const int pair_p = C::P_OFF + pair * 4096;   // this pair's weight buffers
  if (tid == 0) restart_at = ~0u;
  float MLA_LDS* linv = (float MLA_LDS*)(L + C::INV_OFF) + pair * 32;

  // staged output rows (the tile, weight and query buffers are idle then): 32 rows
  // a pair, 1040 bytes apart (4 banks mod 64, so 16 rows x 4 banks cover them all):
  // a whole bf16 row, or half an f32 row
  constexpr int SROW = DC * 2 + 16;
  static_assert(4 * 32 * SROW <= C::INV_OFF, "staging");
  unsigned char MLA_LDS* stage = L + pair * 32 * SROW;
  const bool bf16_out = a.out_direct != nullptr && a.out_direct_bf16;
  auto stage_bf16 = [&](int d, const f32x4 (&o)[2], const float (&inv)[2]) {
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
      *(u32x2 MLA_LDS*)(stage + (rb * 16 + lc) * SROW + d * 32 + lg * 8) =
          u32x2{pack_bf16x2(o[rb][0] * inv[rb], o[rb][1] * inv[rb]), pack_bf16x2(o[rb][2] * inv[rb], o[rb][3] * inv[rb])};
  };
  auto stage_f32 = [&](int d, const f32x4 (&o)[2], const float (&inv)[2]) {   // d: block within the half row
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
      *(f32x4 MLA_LDS*)(stage + (rb * 16 + lc) * SROW + d * 64 + lg * 16) =
          f32x4{o[rb][0] * inv[rb], o[rb][1] * inv[rb], o[rb][2] * inv[rb], o[rb][3] * inv[rb]};
  };
  const int64_t slot0 = (it.kind == 0 ? 0 : a.local_slot_base) + it.hr_begin + pair * 32;
  const int nrow = it.count - pair * 32;   // valid rows of the pair (may exceed 32 or be negative)
  // this wave writes 16 of the pair's staged rows, eight reads ahead of their
  // stores, one contiguous kilobyte a store; h: half of an f32 row
  auto write_rows = [&](int h) {
#pragma unroll 1
    for (int p0 = (wave >> 2) * 16; p0 < (wave >> 2) * 16 + 16; p0 += 8) {
      u32x4 t[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) t[j] = *(const u32x4 MLA_LDS*)(stage + (p0 + j) * SROW + lane * 16);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int r = p0 + j;
        if (r >= nrow) continue;
        unsigned char* dst;
        if (bf16_out)
          dst = (unsigned char*)a.out_direct + (slot0 + r) * a.dv * 2;
        else
          dst = (unsigned char*)(a.out_direct != nullptr ? (float*)a.out_direct + (slot0 + r) * a.dv
                                                         : a.part_o + (a.part_ptr[slot0 + r] + it.chunk) * a.dv) + h * (DC * 2);
        *(u32x4*)(dst + lane * 16) = t[j];
      }
    }
  };

  if (wave < 4) {
    // ------------------------------------------------------------------ score wave
    // Q fragments (B operand of S^T = K Q^T): qf[ks][rb] holds dims ks*32 + lg*8 ..
    // +7 of head-row rb*16 + lc
    bf16x8 qf[C::KS][2];
    int t_pos[2];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      const int r = rb * 16 + lc;
      const int64_t hr = it.hr_begin + (r < nrow ? pair * 32 + r : 0);
      const int row = it.kind == 0 ? (int)(hr / a.n_groups) : a.prot[hr / a.n_local];
      t_pos[rb] = (int)own.req_offset + (row - (int)own.kv_start);
    }
    const double th0 = a.theta_rev[lane & (DR / 2 - 1)];
    tile_barrier();   // the queries have landed
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int ks = 0; ks < C::KS; ++ks) {
        const int at = (pair * 4 + rb * 2 + (lc >> 3)) * C::KB8 + (lc & 7) * 128 + ((lg ^ key_swz(lc & 7)) * 16);
        qf[ks][rb] = *(const bf16x8 MLA_LDS*)(L + (at ^ ((ks & 1) * 64)) + (ks >> 1) * 1024);
        if (rb * 16 + lc >= nrow) qf[ks][rb] = bf16x8{};
      }
    tile_barrier();   // every fragment is read: the tiles may come in
    unsigned char MLA_LDS* qraw0 = L + C::Q_OFF + pair * 4096;
    double MLA_LDS* theta = (double MLA_LDS*)(L + C::TH_OFF) + pair * (DR / 2);
    if (lane < DR / 2) theta[lane] = th0;
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int rs = 0; rs < 2; ++rs) *(bf16x8 MLA_LDS*)(qraw0 + (rb * 2 + rs) * 1024 + lane * 16) = qf[C::CS + rs][rb];
    // K fragments (A operand, 16 keys x 32 dims): key kb*16 + lc, chunk 4 ks + lg
    const int abase = (lc >> 3) * C::KB8 + (lc & 7) * 128 + ((lg ^ key_swz(lc & 7)) * 16);

    f32x4 o[C::OBS][2];
    float m_run[2], l_run[2], m_seen[2];
    int lim[2], wave_lim;
    auto relocate = [&](const TileCursor& s) {
      const int ln = lane_now();
      const double MLA_LDS* th = theta + (ln >> 4) * 8;
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        const int delta = t_pos[rb] - s.req_offset;
        const int lm = delta < s.length - 1 ? delta : s.length - 1;
        lim[rb] = rb * 16 + (ln & 15) < nrow ? lm : 0x7fffffff;
        const double dd = (double)delta;
        const bf16x8 lo = *(const bf16x8 MLA_LDS*)(qraw0 + rb * 2048 + ln * 16);
        const bf16x8 hi = *(const bf16x8 MLA_LDS*)(qraw0 + rb * 2048 + 1024 + ln * 16);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const double rev = dd * th[i];
          const float r = (float)(rev - rint(rev));
          const float sn = __builtin_amdgcn_sinf(r), cn = __builtin_amdgcn_cosf(r);
          const float x1 = (float)lo[i], x2 = (float)hi[i];
          qf[C::CS][rb][i] = (__bf16)(x1 * cn - x2 * sn);
          qf[C::CS + 1][rb][i] = (__bf16)(x1 * sn + x2 * cn);
        }
      }
      // an item's rows ascend, so the pair's first row sees least
      wave_lim = __builtin_amdgcn_readfirstlane(lim[0]);
    };
    const float sl2 = a.scale_log2;
    const int vbl = vbase(0), pwl = pair_p + lane * 16;
    int attempt = 0;
    TileCursor c;
    cursor_open<C>(c, v, v.chk.first_rank);
    relocate(c);
    tile_barrier();   // tiles 0 and 1 have landed
    // The reference: each head-row's max over the item's first kRefKeys keys (of its
    // first segment).  Once per item, before the tile loop, 16 keys at a time.
    {
      float m[2] = {-INFINITY, -INFINITY};
      const int n16 = c.n_keys > C::BK ? kRefKeys / 16 : C::BK / 16;
#pragma unroll 1
      for (int b = 0; b < n16; ++b) {
        const int at = abase + (b >> 1) * C::TILE_BYTES + (b & 1) * 2 * C::KB8;
        f32x4 s[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
        bf16x8 ka[4];
        auto kfrag = [&](int ks) -> bf16x8 { return *(const bf16x8 MLA_LDS*)(L + (at ^ ((ks & 1) * 64)) + (ks >> 1) * 1024); };
#pragma unroll
        for (int j = 0; j < 3; ++j) ka[j] = kfrag(j);
#pragma unroll
        for (int ks = 0; ks < C::KS; ++ks) {
          if (ks + 3 < C::KS) ka[(ks + 3) % 4] = kfrag(ks + 3);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int rb = 0; rb < 2; ++rb) s[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[ks % 4], qf[ks][rb], s[rb], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
        const int k0 = b * 16 + (lane_now() >> 4) * 4;
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
          for (int i = 0; i < 4; ++i) m[rb] = fmaxf(m[rb], i > lim[rb] - k0 ? -INFINITY : s[rb][i]);
      }
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        m_run[rb] = quad_max(m[rb]) * sl2;
        m_seen[rb] = fmaxf(-1e30f, m_run[rb]);
      }
    }
    for (;;) {
#pragma unroll
      for (int d = 0; d < C::OBS; ++d)
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) o[d][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
      l_run[0] = l_run[1] = 0.f;
      const bool may_vote = restart_allowed(attempt);
      bf16x8 pf[2] = {bf16x8{}, bf16x8{}};
      bf16x8 vt[C::OBS];
#pragma unroll
      for (int j = 0; j < C::OBS; ++j) vt[j] = bf16x8{};
      bool done = false, restart = false;
      unsigned t = 0;
      int cur = 0, pcur = 0;   // buffers of tile t and of its weights
      for (;;) {
        tile_barrier();
        int ab[2];
        ab[0] = abase + cur;
        ab[1] = ab[0] ^ 64;
        // K fragment f = kb*KS + ks
        auto kfrag = [&](int f) -> bf16x8 {
          const int kb = f / C::KS, ks = f % C::KS;
          return *(const bf16x8 MLA_LDS*)(L + ab[ks & 1] + (ks >> 1) * 1024 + kb * 2 * C::KB8);
        };
        constexpr int KD = 4;   // fragments in flight
        bf16x8 ka[KD];
#pragma unroll
        for (int j = 0; j < KD - 1; ++j) ka[j] = kfrag(j);
        const unsigned vote = *(volatile unsigned MLA_LDS*)&restart_at;
        __builtin_amdgcn_sched_barrier(0);
        // the previous tile's weights into this wave's output blocks while the first K
        // fragments arrive, and its row sums
        const bf16x2 one2 = {(__bf16)1.0f, (__bf16)1.0f};
        float rsum[2];
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
          const bf16x8 w = pf[rb];
          o[0][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[0], w, o[0][rb], 0, 0, 0);
          float r = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(w, w, 0, 1), one2, 0.f, false);
          __builtin_amdgcn_sched_barrier(0);
          o[1][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[1], w, o[1][rb], 0, 0, 0);
          r = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(w, w, 2, 3), one2, r, false);
          __builtin_amdgcn_sched_barrier(0);
          o[2][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[2], w, o[2][rb], 0, 0, 0);
          r = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(w, w, 4, 5), one2, r, false);
          __builtin_amdgcn_sched_barrier(0);
          o[3][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[3], w, o[3][rb], 0, 0, 0);
          rsum[rb] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(w, w, 6, 7), one2, r, false);
          __builtin_amdgcn_sched_barrier(0);
        }
        f32x4 s[2][2];
        auto qk = [&](int f) {
          const int kb = f / C::KS, ks = f % C::KS;
          if (f + KD - 1 < 2 * C::KS) ka[(f + KD - 1) % KD] = kfrag(f + KD - 1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int rb = 0; rb < 2; ++rb)
            s[kb][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[f % KD], qf[ks][rb],
                                                                ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : s[kb][rb], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        };
        // S^T = K Q^T of the first 16 keys
        qk(0);
        l_run[0] += rsum[0];
        l_run[1] += rsum[1];
        const float rmax = fmaxf(rsum[0], rsum[1]);   // a NaN sum never votes
        __builtin_amdgcn_sched_barrier(0);
        qk(1);
        const bool votes = may_vote && __builtin_amdgcn_ballot_w64(restart_vote(rmax)) != 0;
        restart = (unsigned)__builtin_amdgcn_readfirstlane((int)vote) <= t;
        qk(2);
        if (__builtin_expect(votes, 0)) {
#pragma unroll
          for (int rb = 0; rb < 2; ++rb)
            m_seen[rb] = raised_reference(m_seen[rb], m_run[rb], quad_max(restart_raise(rsum[rb])), -INFINITY);
          if (lane_now() == 0) atomicMin(&restart_at, t + 1);
        }
        if (__builtin_expect(done || restart, 0)) break;
        const int tk0 = c.tile * C::BK;
        const int nx = cursor_next<C>(c, v);
#pragma unroll
        for (int f = 3; f < C::KS + 2; ++f) qk(f);
        // register i of s[kb][rb]: key kb*16 + lg*4 + i, head-row rb*16 + lc
        auto mask = [&](int kb) {
          const int k0 = tk0 + kb * 16 + (lane_now() >> 4) * 4;
#pragma unroll
          for (int rb = 0; rb < 2; ++rb) {
            const int rel = lim[rb] - k0;
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (i > rel) s[kb][rb][i] = -INFINITY;
          }
        };
        if (__builtin_expect(tk0 + C::BK - 1 > wave_lim, 0)) mask(0);
        // The second 16 keys' scores; between their MFMAs the first 16 keys' weights
        // and the reads of this wave's V^T fragments.
        const int vb = vbl + cur;
        u32x2 pw0[2];
#pragma unroll
        for (int f = 2; f < C::KS; ++f) {
          qk(C::KS + f);
          if (f < 10) {
            const int rb = (f - 2) >> 2, i = (f - 2) & 3;
            float w = __builtin_amdgcn_exp2f(__builtin_fmaf(s[0][rb][i], sl2, -m_run[rb]));
            asm volatile("" : "+v"(w));   // computed here, not sunk below the loop
            s[0][rb][i] = w;
          } else if (f < 14) {
            const int rb = (f - 10) >> 1, i = ((f - 10) & 1) * 2;
            uint32_t w = pack_bf16x2(s[0][rb][i], s[0][rb][i + 1]);
            asm volatile("" : "+v"(w));
            pw0[rb][i >> 1] = w;
            vt[f - 10] = vfrag(vb, f - 10);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if (__builtin_expect(tk0 + C::BK - 1 > wave_lim, 0)) mask(1);
        unsigned char MLA_LDS* pw = L + pwl + pcur;
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
          float w[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) w[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[1][rb][i], sl2, -m_run[rb]));
          pf[rb] = __builtin_bit_cast(bf16x8, u32x4{pw0[rb][0], pw0[rb][1], pack_bf16x2(w[0], w[1]), pack_bf16x2(w[2], w[3])});
          *(bf16x8 MLA_LDS*)(pw + rb * 1024) = pf[rb];
        }
        ++t;
        done = nx == 0;
        if (__builtin_expect(nx == 2, 0)) relocate(c);
        cur = cur == (C::NBUF - 1) * C::TILE_BYTES ? 0 : cur + C::TILE_BYTES;
        pcur ^= 2048;
      }
      tile_barrier();   // the last tile's votes are cast
      restart = restart || *(volatile unsigned MLA_LDS*)&restart_at != ~0u;
      if (!restart) break;
      tile_barrier();
      if (tid == 0) restart_at = ~0u;
      ++attempt;
      m_run[0] = m_seen[0];
      m_run[1] = m_seen[1];
      int first = v.chk.first_rank;
      asm volatile("" : "+s"(first));   // opened anew, not held across the loop
      cursor_open<C>(c, v, first);
      relocate(c);
      tile_barrier();   // tiles 0 and 1 have landed
    }
    float inv[2];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
      const float l_tot = quad_sum(l_run[rb]);
      inv[rb] = 1.f / l_tot;
      if (lg == rb) {
        const int r = rb * 16 + lc;
        linv[r] = inv[rb];
        if (r < nrow && a.part_lse != nullptr) {
          const int64_t at = a.out_direct != nullptr ? slot0 + r : a.part_ptr[slot0 + r] + it.chunk;
          a.part_lse[at] = (m_run[rb] + __log2f(l_tot)) * 0.6931471805599453f;
        }
      }
    }
    tile_barrier();   // the value waves read linv; every tile and weight buffer is idle
#pragma unroll
    for (int d = 0; d < C::OBS; ++d)
      if (bf16_out) stage_bf16(d, o[d], inv); else stage_f32(d, o[d], inv);
    tile_barrier();
    write_rows(0);
    if (!bf16_out) {
      tile_barrier();
      tile_barrier();
      write_rows(1);
    }
  } else {
    // ------------------------------------------------------------------ value wave
    f32x4 o[C::OBV][2];
    TileCursor c;
    tile_barrier();   // the queries have landed
    tile_barrier();   // and are in the score waves' registers
    for (;;) {
      int first = v.chk.first_rank;
      asm volatile("" : "+s"(first));   // opened anew by each attempt, not held across the loop
      cursor_open<C>(c, v, first);
      issue_block<C>(a.kv, c, L, pair);
      bool have = cursor_next<C>(c, v) != 0;   // tile t (from 1) exists
      if (have) issue_block<C>(a.kv, c, L + C::TILE_BYTES, pair);
#pragma unroll
      for (int d = 0; d < C::OBV; ++d)
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) o[d][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
      bool restart = false;
      tile_barrier();                      // tiles 0 and 1 have landed
      tile_barrier();                      // step 0
      unsigned t = 1;
      int cur = 0;                         // buffer of tile t - 1
      int pcur = 0;                        // weight buffer of tile t - 1
      for (;;) {
        tile_barrier();                    // step t: tile t has landed, the weights of tile t - 1 are written
        const unsigned vote = *(volatile unsigned MLA_LDS*)&restart_at;
        const int buf = cur;
        cur = cur == (C::NBUF - 1) * C::TILE_BYTES ? 0 : cur + C::TILE_BYTES;
        const bool last = !have;
        if (__builtin_expect(have, 1)) {
          const int nxt = cur == (C::NBUF - 1) * C::TILE_BYTES ? 0 : cur + C::TILE_BYTES;
          have = cursor_next<C>(c, v) != 0;
          if (__builtin_expect(have, 1)) issue_block<C>(a.kv, c, L + nxt, pair);
        }
        {
          bf16x8 pf[2];
          const unsigned char MLA_LDS* pr = L + pair_p + pcur + lane_now() * 16;
          pf[0] = *(const bf16x8 MLA_LDS*)pr;
          pf[1] = *(const bf16x8 MLA_LDS*)(pr + 1024);
          const int vb = vbase(buf);
          // blocks in the order of their chunk slot, so that few addresses are live
          auto blk = [](int st) { return C::OBS + (st % (C::OBV / 4)) * 4 + st / (C::OBV / 4); };
          constexpr int VD = 3;
          bf16x8 vt[VD + 1];
#pragma unroll
          for (int j = 0; j < VD; ++j) vt[j] = vfrag(vb, blk(j));
#pragma unroll
          for (int st = 0; st < C::OBV; ++st) {
            if (st + VD < C::OBV) vt[(st + VD) % (VD + 1)] = vfrag(vb, blk(st + VD));
            __builtin_amdgcn_sched_barrier(0);
            const int d = blk(st) - C::OBS;
            o[d][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[st % (VD + 1)], pf[0], o[d][0], 0, 0, 0);
            o[d][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt[st % (VD + 1)], pf[1], o[d][1], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        restart = (unsigned)__builtin_amdgcn_readfirstlane((int)vote) <= t;
        if (__builtin_expect(restart || last, 0)) break;
        ++t;
        pcur ^= 2048;
      }
      tile_barrier();
      restart = restart || *(volatile unsigned MLA_LDS*)&restart_at != ~0u;
      if (!restart) break;
      tile_barrier();
    }
    tile_barrier();
    const float inv[2] = {linv[lc], linv[16 + lc]};
    if (bf16_out) {
#pragma unroll
      for (int d = 0; d < C::OBV; ++d) stage_bf16(C::OBS + d, o[d], inv);
      tile_barrier();
      write_rows(0);
    } else {
#pragma unroll
      for (int d = C::OBS; d < C::OB / 2; ++d) stage_f32(d, o[d - C::OBS], inv);
      tile_barrier();
      write_rows(0);
      tile_barrier();
#pragma unroll
      for (int d = C::OB / 2; d < C::OB; ++d) stage_f32(d - C::OB / 2, o[d - C::OBS], inv);
      tile_barrier();
      write_rows(1);
    }
  }
}

hipError_t launch_attend_pair(const AttendArgs& a, unsigned grid, hipStream_t s) {
  attend_pair_kernel<512, 64><<<dim3(grid), dim3(512), 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace mla
