// Adaptive MoE fanout (Sec. 2.4, eq:moe).  For each token row the router's
// top_k experts (the paper's Top-6) are ranked by weight, their weights are
// normalized only to choose the fanout
//   K = min{k in [min_k, top_k] : sum_{j<=k} p_(j) / sum_{r<=top_k} p_(r) >= tau}
// (top_k when no k qualifies), and the executed experts keep their original
// weights.  The integer K is decided in float32, in rank order: the sum of the
// top_k weights left to right, each share a correctly rounded division, the
// shares accumulated left to right.
//
// Ranking keys are the weight's IEEE-754 totalOrder bits above the inverted expert
// index: unique, larger weights first, equal weights to the lower expert.
//
// Up to 256 experts a row is held by 16 lanes (four rows per wave), loaded four
// experts a lane at a time while the row before is ranked.  Keys are 32-bit here:
// the low 8 bits of the weight's code give way to the index.  Each lane keeps its
// four largest keys sorted (a max and three medians per key); a round takes the
// row's maximum of the lanes' largest (four DPP steps) and the owner drops it.  The
// weights are then fetched, and the list is right if they stand in order and top_k - 1
// experts come before the last.  The order is compared in every row (equal weights are
// in order: the lower expert first).  The count, a second read of the row, only in waves
// with a row where something could belong inside: a runner-up that shares the upper
// bits of the last rank's code, or a lane whose four keys are all taken; one wave in
// seventy on softmax weights, one in four where the logits were bf16 and weights repeat.
// A wave that finds a wrong list ranks its rows over with 64-bit keys (rank_exact): one
// in a thousand, weights that differ in the low 8 bits of their codes only.
// Above 256 experts a whole wave holds a row and every round is exact.
//
// What bounds it is vector issue: 64-bit rounds over all of a lane's experts took 278
// wave instructions a row, these 115, 134 with repeated weights.  264,192 rows x 256
// experts 127 -> 73 us (3.9 TB/s; bf16 logits 127 -> 84, all weights equal 127 -> 102),
// x 128 83 -> 51, x 64 68 -> 45, x 16 52 -> 33.  Any two neighbours with like upper bits,
// equal weights too, sent to the exact ranking took bf16 logits 160 us.  Four waves a
// SIMD, nothing spilled; three and five are within 2 %, with six (80 registers) the rare
// paths spill: 86 us, 122 on bf16 logits.
// A second kernel over a few blocks counts the rows that execute each expert
// (per-block LDS histograms added into expert_count, which the first one clears).
#include "moe.h"

#include <algorithm>

namespace mla {
namespace {

__device__ __forceinline__ uint32_t total_order_bits(float x) {
  const uint32_t u = __float_as_uint(x);
  return (u >> 31) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float from_total_order_bits(uint32_t t) {
  return __uint_as_float((t >> 31) ? (t & 0x7FFFFFFFu) : ~t);
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}

__device__ __forceinline__ uint64_t join(uint32_t lo, uint32_t hi) { return ((uint64_t)hi << 32) | lo; }

// maximum over each group of LPR consecutive lanes (16 or 64), in every lane of
// the group: quad butterflies and row mirrors (DPP) inside each 16-lane row,
// then, for 64-lane groups, the gfx950 row swaps across 16 and 32 lanes
template <int LPR>
__device__ __forceinline__ uint64_t group_max_u64(uint64_t v) {
  static_assert(LPR == 16 || LPR == 64, "lanes per row");
  uint64_t o;
  o = join(dpp<0xB1>((uint32_t)v), dpp<0xB1>((uint32_t)(v >> 32)));     // lane ^ 1
  v = o > v ? o : v;
  o = join(dpp<0x4E>((uint32_t)v), dpp<0x4E>((uint32_t)(v >> 32)));     // lane ^ 2
  v = o > v ? o : v;
  o = join(dpp<0x141>((uint32_t)v), dpp<0x141>((uint32_t)(v >> 32)));   // mirror in 8 lanes: quad pairs
  v = o > v ? o : v;
  o = join(dpp<0x140>((uint32_t)v), dpp<0x140>((uint32_t)(v >> 32)));   // mirror in 16 lanes: halves
  v = o > v ? o : v;
  if (LPR == 64) {
    {
      const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
      const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(v >> 32), (uint32_t)(v >> 32), false, false);
      const uint64_t a = join(lo[0], hi[0]), b = join(lo[1], hi[1]);       // rows r and r ^ 1
      v = a > b ? a : b;
    }
    {
      const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
      const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(v >> 32), (uint32_t)(v >> 32), false, false);
      const uint64_t a = join(lo[0], hi[0]), b = join(lo[1], hi[1]);       // halves of the wave
      v = a > b ? a : b;
    }
  }
  return v;
}

template <int LPR, int NV>
__device__ __forceinline__ void load_row(const MoeArgs& a, int64_t r, int sl, float (&v)[NV]) {
  const float* p = a.router + r * a.n_experts;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int e = LPR * i + sl;
    v[i] = p[e < a.n_experts ? e : a.n_experts - 1];   // clamped: no branch; masked below
  }
}

// top_k experts of the row held by LPR lanes (lane sl: experts sl, sl + LPR, ...), by
// 64-bit keys: the rank-j expert and its key's weight, in every lane of the row
template <int LPR, int NV>
__device__ __forceinline__ void rank_exact(const MoeArgs& a, const float (&cur)[NV], int sl, int32_t (&id)[kMoeMaxTopK],
                                           float (&w)[kMoeMaxTopK]) {
  const int E = a.n_experts, TK = a.top_k;
  // totalOrder codes of the lane's weights; a taken mask marks experts already
  // ranked (and the lane's slots past E)
  uint32_t tob[NV];
  uint32_t taken = 0;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    tob[i] = total_order_bits(cur[i]);
    if (LPR * i + sl >= E) taken |= 1u << i;
  }
  // top_k rounds: the lane's best remaining expert (ascending i keeps the lower
  // expert on equal codes), the row maximum of the 64-bit keys, the owner marks it
#pragma unroll
  for (int j = 0; j < kMoeMaxTopK; ++j) {
    id[j] = 0;
    w[j] = 0.0f;
    if (j < TK) {
      uint32_t bt = 0;
      int bi = -1;
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const bool better = !((taken >> i) & 1u) && (bi < 0 || tob[i] > bt);
        bt = better ? tob[i] : bt;
        bi = better ? i : bi;
      }
      const uint64_t mine =
          bi < 0 ? 0ull : ((uint64_t)bt << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)(LPR * bi + sl));
      const uint64_t m = group_max_u64<LPR>(mine);
      if (bi >= 0 && mine == m) taken |= 1u << bi;                     // keys are unique
      id[j] = (int32_t)(0xFFFFFFFFu - (uint32_t)m);
      w[j] = from_total_order_bits((uint32_t)(m >> 32));
    }
  }
}

__device__ __forceinline__ void zero_counts(const MoeArgs& a) {
  if (a.expert_count != nullptr && blockIdx.x == 0)
    for (int i = threadIdx.x; i < a.n_experts; i += blockDim.x) a.expert_count[i] = 0;
}

// a whole wave per row
template <int NV>
__global__ __launch_bounds__(256) void moe_fanout_wave_kernel(MoeArgs a) {
  zero_counts(a);
  const int sl = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int TK = a.top_k;
  const int64_t stride = (int64_t)gridDim.x * 4;
  int64_t r = (int64_t)blockIdx.x * 4 + wave;
  if (r >= a.n_rows) return;
  float cur[NV];
  load_row<64, NV>(a, r, sl, cur);
  for (; r < a.n_rows; r += stride) {
    float nxt[NV];
    const bool more = r + stride < a.n_rows;
    if (more) load_row<64, NV>(a, r + stride, sl, nxt);
    int32_t id[kMoeMaxTopK];
    float w[kMoeMaxTopK];
    rank_exact<64, NV>(a, cur, sl, id, w);
    // fanout, decided in float32 in rank order
    float S = w[0];
#pragma unroll
    for (int j = 1; j < kMoeMaxTopK; ++j)
      if (j < TK) S = S + w[j];
    float cum = 0.0f;
    int K = TK;
    bool done = false;
    int32_t my_id = 0;
    float my_w = 0.0f;
#pragma unroll
    for (int j = 0; j < kMoeMaxTopK; ++j) {
      if (j < TK) {
        cum = cum + w[j] / S;
        if (!done && j + 1 >= a.min_k && cum >= a.tau) {
          K = j + 1;
          done = true;
        }
      }
      if (sl == j) {
        my_id = id[j];
        my_w = w[j];
      }
    }
    if (sl < TK) {
      a.expert_idx[r * TK + sl] = my_id;
      a.expert_w[r * TK + sl] = my_w;
    }
    if (sl == 0) a.fanout[r] = K;
    if (more) {
#pragma unroll
      for (int i = 0; i < NV; ++i) cur[i] = nxt[i];
    }
  }
}

__device__ __forceinline__ uint32_t max_u32(uint32_t x, uint32_t y) { return x > y ? x : y; }
__device__ __forceinline__ uint32_t med_u32(uint32_t x, uint32_t y, uint32_t z) {
  uint32_t m;
  asm("v_med3_u32 %0, %1, %2, %3" : "=v"(m) : "v"(x), "v"(y), "v"(z));
  return m;
}
// maximum over each row of 16 lanes, in every lane
__device__ __forceinline__ uint32_t row_max_u32(uint32_t v) {
  v = max_u32(v, dpp<0xB1>(v));
  v = max_u32(v, dpp<0x4E>(v));
  v = max_u32(v, dpp<0x141>(v));
  return max_u32(v, dpp<0x140>(v));
}
__device__ __forceinline__ uint32_t row_sum_u32(uint32_t v) {
  v += dpp<0xB1>(v);
  v += dpp<0x4E>(v);
  v += dpp<0x141>(v);
  return v + dpp<0x140>(v);
}
// lane J of each row of 16, in every lane of the row (row_newbcast)
template <int J>
__device__ __forceinline__ float row_bcast(float v) {
  return __uint_as_float(dpp<0x150 + J>(__float_as_uint(v)));
}

// expert of register i: VEC: 64 (i / 4) + 4 sl + i % 4 (16-byte loads), else 16 i + sl
template <int NV, bool VEC>
__device__ __forceinline__ int expert_of(int i, int sl) {
  return VEC ? 64 * (i >> 2) + 4 * sl + (i & 3) : 16 * i + sl;
}
template <int NV, bool VEC>
__device__ __forceinline__ void load_row16(const MoeArgs& a, int64_t r, int sl, float (&v)[NV]) {
  const float* p = a.router + r * a.n_experts;
  if constexpr (VEC) {
#pragma unroll
    for (int i = 0; i < NV; i += 4) {
      const int e = 64 * (i >> 2) + 4 * sl;   // a.n_experts is a multiple of 4
      const f32x4 x = *(const f32x4*)(p + (e < a.n_experts ? e : a.n_experts - 4));
#pragma unroll
      for (int c = 0; c < 4; ++c) v[i + c] = x[c];
    }
  } else {
    load_row<16, NV>(a, r, sl, v);
  }
}

// 16 lanes per row, four rows per wave
template <int NV, bool VEC>
__global__ __launch_bounds__(256, 4) void moe_fanout_kernel(MoeArgs a) {
  zero_counts(a);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sl = lane & 15, slot = lane >> 4;
  const int E = a.n_experts, TK = a.top_k;
  const int64_t stride = (int64_t)gridDim.x * 16;
  int64_t r = ((int64_t)blockIdx.x * 4 + wave) * 4 + slot;
  // every lane runs the same number of iterations (rows past the end compute on
  // a clamped copy and write nothing), so the DPP exchanges see whole groups
  const int64_t last = a.n_rows - 1;
  if (r - slot > last) return;
  float cur[NV];
  load_row16<NV, VEC>(a, r < last ? r : last, sl, cur);
  for (; r - slot <= last; r += stride) {
    const int64_t rc = r < last ? r : last;
    constexpr int DEPTH = NV < 4 ? NV : 4;
    uint32_t m[DEPTH];
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) m[d] = 0;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int e = expert_of<NV, VEC>(i, sl);
      uint32_t x = (total_order_bits(cur[i]) & ~0xFFu) | (uint32_t)(255 - e);
      x = e < E ? x : 0u;
#pragma unroll
      for (int d = DEPTH - 1; d > 0; --d) m[d] = med_u32(m[d - 1], m[d], x);
      m[0] = max_u32(m[0], x);
    }
    // the next row, over the registers just consumed
    if (r - slot + stride <= last) {
      const int64_t rn = r + stride;
      load_row16<NV, VEC>(a, rn < last ? rn : last, sl, cur);
    }
    int32_t my_id = 0;
    uint32_t last_key = 0;   // of rank top_k
#pragma unroll
    for (int j = 0; j < kMoeMaxTopK; ++j) {
      if (j < TK) {
        const uint32_t M = row_max_u32(m[0]);
        last_key = M;
        if (sl == j) my_id = 255 - (int32_t)(M & 0xFFu);
        const bool own = m[0] == M;
#pragma unroll
        for (int d = 0; d + 1 < DEPTH; ++d) m[d] = own ? m[d + 1] : m[d];
        m[DEPTH - 1] = own ? 0u : m[DEPTH - 1];
      }
    }
    float my_w = a.router[rc * E + my_id];   // lanes past top_k: expert 0, not used
    // The key order is the weights' unless two weights whose codes share their upper 24
    // bits stand the wrong way round.  Inside the ranked list neighbours show that.
    const uint32_t code = total_order_bits(my_w);
    const uint32_t prev = dpp<0x111>(code);   // row_shr:1: the rank before
    bool wrong = sl > 0 && sl < TK && prev < code;
    // Past it only a runner-up with the last rank's upper bits, or the unknown fifth key
    // of a lane that gave its four, could belong inside.
    const bool open = (row_max_u32(m[0]) >> 8) == (last_key >> 8) || (NV > DEPTH && m[0] == 0);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(wrong || open) != 0, 0)) {
      int ln = sl;
      asm volatile("" : "+v"(ln));   // the addresses below are formed here, not held across the rows
      {
        // a ranked list in order is right if top_k - 1 experts come before its last
        const int end = (lane & 48) + TK - 1;
        const uint32_t end_code = (uint32_t)__shfl((int)code, end, 64);
        const int end_id = __shfl(my_id, end, 64);
        float row[NV];
        load_row<16, NV>(a, rc, ln, row);
        uint32_t before = 0;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
          const uint32_t c = total_order_bits(row[i]);
          const int e = 16 * i + ln;
          before += e < E && (c > end_code || (c == end_code && e < end_id));
        }
        wrong |= row_sum_u32(before) != (uint32_t)(TK - 1);
      }
      if (__builtin_amdgcn_ballot_w64(wrong) != 0) {
        asm volatile("" : "+v"(ln));   // and the row is read again, not kept until here
        float row[NV];
        load_row<16, NV>(a, rc, ln, row);
        int32_t id[kMoeMaxTopK];
        float w[kMoeMaxTopK];
        rank_exact<16, NV>(a, row, ln, id, w);
        my_w = 0.0f;
#pragma unroll
        for (int j = 0; j < kMoeMaxTopK; ++j)
          if (sl == j) {
            my_id = id[j];
            my_w = w[j];
          }
      }
    }
    // fanout, decided in float32 in rank order: lane j of the row holds rank j
    float S = row_bcast<0>(my_w);
    auto add = [&](float acc, float v, int j) { return j < TK ? acc + v : acc; };
    S = add(S, row_bcast<1>(my_w), 1);
    S = add(S, row_bcast<2>(my_w), 2);
    S = add(S, row_bcast<3>(my_w), 3);
    S = add(S, row_bcast<4>(my_w), 4);
    S = add(S, row_bcast<5>(my_w), 5);
    S = add(S, row_bcast<6>(my_w), 6);
    S = add(S, row_bcast<7>(my_w), 7);
    const float share = my_w / S;
    float cum = 0.0f;
    int K = TK;
    bool done = false;
    auto step = [&](float v, int j) {
      if (j < TK) {
        cum = cum + v;
        if (!done && j + 1 >= a.min_k && cum >= a.tau) {
          K = j + 1;
          done = true;
        }
      }
    };
    step(row_bcast<0>(share), 0);
    step(row_bcast<1>(share), 1);
    step(row_bcast<2>(share), 2);
    step(row_bcast<3>(share), 3);
    step(row_bcast<4>(share), 4);
    step(row_bcast<5>(share), 5);
    step(row_bcast<6>(share), 6);
    step(row_bcast<7>(share), 7);
    if (r <= last) {
      if (sl < TK) {
        a.expert_idx[r * TK + sl] = my_id;
        a.expert_w[r * TK + sl] = my_w;
      }
      if (sl == 0) a.fanout[r] = K;
    }
  }
}
static_assert(kMoeMaxTopK <= 8, "ranks 0 .. 7 are broadcast");

// rows that execute each expert: per-block LDS histograms over a few blocks,
// added into expert_count (zeroed by the previous kernel)
__global__ __launch_bounds__(256) void moe_count_kernel(MoeArgs a) {
  __shared__ uint32_t hist[kMoeMaxExperts];
  const int E = a.n_experts, TK = a.top_k;
  for (int i = threadIdx.x; i < E; i += 256) hist[i] = 0;
  __syncthreads();
  for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < a.n_rows; r += (int64_t)gridDim.x * 256) {
    const int K = a.fanout[r];
    for (int j = 0; j < TK; ++j) {
      const int32_t e = a.expert_idx[r * TK + j];
      if (j < K && (uint32_t)e < (uint32_t)E) atomicAdd(&hist[e], 1u);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < E; i += 256) {
    const uint32_t h = hist[i];
    if (h) atomicAdd((uint32_t*)&a.expert_count[i], h);
  }
}

__global__ __launch_bounds__(256) void moe_zero_counts_kernel(int32_t* c, int n) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) c[i] = 0;
}

}  // namespace

hipError_t launch_moe_fanout(const MoeArgs& a, hipStream_t s) {
  hipError_t e;
  if (a.n_rows == 0) {
    if (a.expert_count == nullptr) return hipSuccess;
    moe_zero_counts_kernel<<<dim3((unsigned)((a.n_experts + 255) / 256)), dim3(256), 0, s>>>(a.expert_count,
                                                                                        a.n_experts);
    return hipGetLastError();
  }
  const dim3 blk(256);
  const int E = a.n_experts;
  auto grid = [&](int rows_per_wave) {
    // a few row groups per wave, so that each wave's next row loads while it ranks one
    return dim3((unsigned)std::min<int64_t>((a.n_rows + 4 * rows_per_wave - 1) / (4 * rows_per_wave), 2048));
  };
  // four experts a lane and load where every row starts on 16 bytes
  const bool vec = E % 4 == 0 && (reinterpret_cast<uintptr_t>(a.router) & 15u) == 0;
  if (E <= 16) moe_fanout_kernel<1, false><<<grid(4), blk, 0, s>>>(a);
  else if (E <= 32) moe_fanout_kernel<2, false><<<grid(4), blk, 0, s>>>(a);
  else if (E <= 64 && vec) moe_fanout_kernel<4, true><<<grid(4), blk, 0, s>>>(a);
  else if (E <= 64) moe_fanout_kernel<4, false><<<grid(4), blk, 0, s>>>(a);
  else if (E <= 128 && vec) moe_fanout_kernel<8, true><<<grid(4), blk, 0, s>>>(a);
  else if (E <= 128) moe_fanout_kernel<8, false><<<grid(4), blk, 0, s>>>(a);
  else if (E <= 256 && vec) moe_fanout_kernel<16, true><<<grid(4), blk, 0, s>>>(a);
  else if (E <= 256) moe_fanout_kernel<16, false><<<grid(4), blk, 0, s>>>(a);
  else if (E <= 512) moe_fanout_wave_kernel<8><<<grid(1), blk, 0, s>>>(a);
  else moe_fanout_wave_kernel<16><<<grid(1), blk, 0, s>>>(a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (a.expert_count != nullptr) {
    const unsigned cblocks = (unsigned)std::min<int64_t>((a.n_rows + 1023) / 1024, 256);
    moe_count_kernel<<<dim3(cblocks), dim3(256), 0, s>>>(a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace mla
